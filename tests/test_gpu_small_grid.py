"""Calls that cannot fill the GPU run in 64-query items, others in 256-query ones, and batches of up to
64 segments in few items are planned by the attention kernel itself, others by a planning kernel.  Neither
choice may change a bit of a row's result: the same sequences are computed alone and in a batch large
enough to change the path.  The small path is checked against the fp64 oracle as well.
"""
import math

import numpy as np
import pytest
import torch

import workloads as W
from metrics import assert_rows
from oracle import ts_ref

pytestmark = pytest.mark.gpu

ts = pytest.importorskip("paper_2606_19271_amd")

CUS = 256  # more 64-query items than CUs: 256-query items


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ts.load()


def say(*a):
    print("[gpu-test]", *a, flush=True)


def draw(lq, lk, H, d, seed, kind):
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((lq, H, d), generator=g)
    k = torch.randn((lk, H, d), generator=g)
    v = torch.randn((lk, H, d), generator=g)
    if kind == "peaked":  # weights reach 2 again and again: maxima are taken mid-sequence
        q *= 8
    if kind == "jump" and lk > 140:  # one block's scores far above all earlier ones, for some queries
        k[lk // 2 + 3] = 30 * q[: min(lq, 20)].mean(dim=0)
    return [t.to(torch.bfloat16) for t in (q, k, v)]


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


def kv(q, k, v, lq, lk, copies, splits, scale):
    """The chunk call on `copies` copies of one segment; (o, lse) of every copy."""
    cq = torch.arange(copies + 1, dtype=torch.int32, device="cuda") * lq
    ck = torch.arange(copies + 1, dtype=torch.int32, device="cuda") * lk
    o, lse = ts.ts_attn_fwd_kvcache(q.repeat(copies, 1, 1), k.repeat(copies, 1, 1), v.repeat(copies, 1, 1),
                                    cq, ck, lq, lk, scale=scale, return_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    return o.view(copies, lq, *o.shape[1:]), lse.view(copies, lq, -1)


def fill(lq, H, splits=1):
    return math.ceil((CUS + 1) / (H * splits * math.ceil(lq / 64)))


# query tails around 32 (one block), 64 (an item) and 256 (thin tiles); key tails around both key tiles
EDGES = [(33, 65), (64, 128), (65, 129), (96, 192), (128, 127), (129, 64), (191, 257), (256, 256), (257, 640), (288, 300),
         (289, 383), (320, 1), (500, 700), (513, 66)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["normal", "peaked", "jump"])
def test_item_size_does_not_change_a_bit(d, kind):
    H = 2
    for n, (lq, lk) in enumerate(EDGES):
        q, k, v = draw(lq, lk, H, d, 900 + n, kind)
        qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
        scale = [None, -0.3, 0.0][n % 3]
        for splits in (1, 3):
            say("item size", d, kind, lq, lk, "splits", splits, "scale", scale)
            o, lse = kv(qd, kd, vd, lq, lk, 1, splits, scale)
            many, many_lse = kv(qd, kd, vd, lq, lk, fill(lq, H, splits), splits, scale)
            for c in (0, many.shape[0] - 1):
                assert torch.equal(bits(many[c]), bits(o[0])), (lq, lk, splits, c)
                assert torch.equal(bits(many_lse[c]), bits(lse[0])), (lq, lk, splits, c)
            sc = 1.0 / math.sqrt(d) if scale is None else scale
            ref, ref_lse = ts_ref.attn_kv_full(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v),
                                               np.array([0, lq], np.int32), np.array([0, lk], np.int32),
                                               float(np.float32(sc)))
            assert_rows(o[0].float().cpu().numpy().astype(np.float64), ref, "%d x %d" % (lq, lk),
                        elementwise=False)
            # as in the chunk tests: the bf16 weights' rounding changes the lse by at most 2e-3
            assert float(np.abs(lse[0].cpu().numpy() - ref_lse).max()) <= 1e-2


@pytest.mark.parametrize("d", [64, 128])
def test_dense_item_size_does_not_change_a_bit(d):
    H = 2
    for L in (64, 65, 200, 257, 288, 289, 1000):
        q, k, v = (t.cuda() for t in draw(L, L, H, d, L, "normal"))
        B = fill(L, H)
        say("dense item size", d, L, B)
        one = ts.ts_attn_fwd(q[None], k[None], v[None])
        many = ts.ts_attn_fwd(*(t[None].repeat(B, 1, 1, 1) for t in (q, k, v)))
        torch.cuda.synchronize()
        assert torch.equal(bits(many[0]), bits(one[0])) and torch.equal(bits(many[-1]), bits(one[0])), L


@pytest.mark.parametrize("lens", [[70, 0, 130, 300], [0, 0, 64], [257] * 3], ids=str)
def test_planned_by_wave_or_kernel_is_the_same(lens):
    """63, 64 and 65 segments around the lens: the last count is planned by the planning kernel."""
    H, d = 2, 64
    results = []
    for nseq in (63, 64, 65):
        ls = lens + [33 + s % 50 for s in range(nseq - len(lens))]
        q, k, v = (t.cuda() for t in draw(sum(ls), sum(ls), H, d, 17, "normal"))
        cu = torch.tensor(np.concatenate([[0], np.cumsum(ls)]), dtype=torch.int32, device="cuda")
        # every segment's own rows are drawn again, so that they do not depend on the total
        at = 0
        for s, n in enumerate(ls):
            g = torch.Generator().manual_seed(s)
            for t in (q, k, v):
                t[at:at + n] = torch.randn((n, H, d), generator=g).to(torch.bfloat16)
            at += n
        for splits in (None, 1, 2):
            if splits is None:
                o = ts.ts_attn_fwd_varlen(q, k, v, cu, max(ls))
            else:
                o = ts.ts_attn_fwd_kvcache(q, k, v, cu, cu, max(ls), max(ls), num_splits=splits)
            torch.cuda.synchronize()
            results.append((nseq, splits, o[: sum(ls[:63])]))
    for splits in (None, 1, 2):
        a, b, c = [o for n, s, o in results if s == splits]
        assert torch.equal(bits(a), bits(b)) and torch.equal(bits(a), bits(c)), (lens, splits)


def test_bad_offsets_are_a_no_op_without_a_plan():
    H, d, T = 2, 64, 400
    q, k, v = (t.cuda() for t in draw(T, T, H, d, 3, "normal"))
    for cu in ([1, 100, 400], [0, 100, 399], [0, 401, 400], [0, 300, 200, 400], [0, -5, 400],
               [0, 2 ** 31 - 1, 400], [0, 350, 400]):
        c = torch.tensor(cu, dtype=torch.int32, device="cuda")
        for splits in (1, 2):
            out = torch.full_like(q, 7.0)
            lse = torch.full((T, H), 7.0, device="cuda")
            ts.ts_attn_fwd_kvcache(q, k, v, c, c, 300, 300, out=out, lse=lse, num_splits=splits)
            torch.cuda.synchronize()
            assert bool((out == 7.0).all()) and bool((lse == 7.0).all()), (cu, splits)


# chunks against caches of even and uneven length, and the key ranges that the library takes for them
CHOICES = [((256, 256, 256, 256), (1536, 512, 1280, 1536), 4, 64, 3), ((768,), (2816,), 12, 128, 7),
           ((768, 256, 256, 768, 256, 768), (1024, 4608, 1536, 1280, 1536, 1024), 12, 128, 12),
           ((256,) * 4, (5120,) * 4, 16, 128, 4), ((1560, 1560), (7800, 4680), 4, 64, 9), ((256,), (5376,), 16, 64, 9),
           ((500, 500), (400, 400), 2, 128, 1)]


@pytest.mark.parametrize("lq,lk,H,d,n", CHOICES, ids=str)
def test_automatic_key_ranges(lq, lk, H, d, n):
    """num_splits = 0 gives the bits of the n it stands for; without allocation, of the most ranges up to
    n whose float32 partial results fit the scratch array."""
    q, _, _ = draw(sum(lq), 1, H, d, 11, "normal")
    _, k, v = draw(1, sum(lk), H, d, 12, "normal")
    cq, ck = (torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32, device="cuda") for x in (lq, lk))
    args = (q.cuda(), k.cuda(), v.cuda(), cq, ck, max(lq), max(lk))
    fits = n
    while fits > 1 and 4 * fits * sum(lq) * H * (d + 1) + 1024 > 32 << 20:
        fits -= 1
    say("automatic key ranges", lq, lk, H, d, n, fits)
    for entry, ranges in ((ts.ts_attn_fwd_kvcache, n), (ts.ts_attn_fwd_kvcache_noalloc, fits)):
        want, want_lse = ts.ts_attn_fwd_kvcache(*args, return_lse=True, num_splits=ranges)
        o, lse = entry(*args, return_lse=True, num_splits=0)
        torch.cuda.synchronize()
        assert torch.equal(bits(o), bits(want)) and torch.equal(bits(lse), bits(want_lse)), entry


@pytest.mark.parametrize("H", [2, 40])  # items of 64 and of 256 queries
@pytest.mark.parametrize("splits", [1, 2])
def test_segments_without_keys_are_zeros(H, splits):
    lq, lk = [1, 31, 32, 33, 64, 65, 255, 256, 257, 300], [0] * 9 + [200]
    q, _, _ = draw(sum(lq), 1, H, 128, 21, "normal")
    _, k, v = draw(1, sum(lk), H, 128, 22, "normal")
    cq, ck = (torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32, device="cuda") for x in (lq, lk))
    say("segments without keys", H, splits)
    out = torch.full(q.shape, 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full(q.shape[:2], 7.0, dtype=torch.float32, device="cuda")
    ts.ts_attn_fwd_kvcache(q.cuda(), k.cuda(), v.cuda(), cq, ck, max(lq), max(lk), out=out, lse=lse, num_splits=splits)
    torch.cuda.synchronize()
    empty = sum(lq[:-1])
    assert bool((out[:empty] == 0).all()) and bool((lse[:empty] == -math.inf).all())
    assert bool((out[empty:] != 7.0).any()) and bool(torch.isfinite(lse[empty:]).all())
