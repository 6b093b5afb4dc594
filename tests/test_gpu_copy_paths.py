"""State copies at the sizes where the kernels change: the 16 KiB and 32 KiB chunk edges, fewer and
more chunks than the workgroups of a suspend walk, and device-to-device copies on both sides of the
32 MiB from which they are non-temporal; against the range copy by definition, bit for bit."""
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
                                   [(32 << 20) + 16, 16 * K + 48, 0, 1 << 20]], ids=str)
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
