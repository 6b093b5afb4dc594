"""State copies at the sizes where the kernels change: the 16 KiB and 32 KiB chunk edges, fewer and
more chunks than the workgroups of a suspend walk, and device-to-device copies on both sides of the
128 MiB from which they are non-temporal; against the range copy by definition, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ts = pytest.importorskip("paper_2606_19271_amd")

K = 1 << 10


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ts.load()


@pytest.mark.parametrize("where", ["dev->host", "host->dev", "dev->dev"])
@pytest.mark.parametrize("sizes", [[16], [16 * K - 16, 16 * K, 16 * K + 16], [32 * K - 16, 32 * K + 16, 0, 48 * K],
                                   [512 * K, 512 * K + 16], [3 << 20, 16, 5 * K], [(32 << 20) - 4 * 16 * K, 16],
                                   [(32 << 20) + 16, 16 * K + 48, 0, 1 << 20], [(128 << 20) - 2 * 16 * K, 16],
                                   [128 << 20, 32]], ids=str)
def test_copy_paths(where, sizes):
    print("[gpu-test] copy", where, sizes, flush=True)
    src_at, dst_at = where.split("->")
    total = sum(sizes) + 64 * len(sizes)
    g = torch.Generator().manual_seed(len(sizes) + total)
    data = torch.randint(0, 256, (total + 32,), dtype=torch.uint8, generator=g)
    data = data[: total // 16 * 16].contiguous()
    ranges, s, d = [], 16, 0
    for n in sizes:
        ranges.append((s, d, n))
        s, d = s + n + 16, d + n + 48
    src = data.cuda() if src_at == "dev" else data.pin_memory()
    dst = torch.full((d + 16,), 7, dtype=torch.uint8)
    want = dst.numpy().copy()
    for a, b, n in ranges:
        want[b:b + n] = data.numpy()[a:a + n]
    dst = dst.cuda() if dst_at == "dev" else dst.pin_memory()
    ts.ts_state_copy(src, dst, ranges)
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy(), want)


def test_copy_of_more_chunks_than_a_grid_holds():
    """64 ranges of 2 GiB out of one source: 2^23 chunks of 16 KiB and some more."""
    n = (2 << 30) + 16
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GiB of device memory")
    print("[gpu-test] copy of 128 GiB in one list", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    src = torch.randint(-(1 << 62), 1 << 62, ((n + 64 * 16) // 8,), generator=g, device="cuda").view(torch.uint8)
    dst = torch.empty(64 * n, dtype=torch.uint8, device="cuda")
    ranges = [(16 * r, n * r, n) for r in range(64)]
    ts.ts_state_copy(src, dst, ranges)
    for s, d, n in ranges:
        assert torch.equal(dst[d:d + n].view(torch.int64), src[s:s + n].view(torch.int64))
