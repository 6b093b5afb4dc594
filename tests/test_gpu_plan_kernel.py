"""Batches whose segments a planning kernel checks and orders before the attention kernel: more than 64
segments, or few in many work items.  The plan lies in the cached workspace (taken in turn by calls of
all streams), or, without allocation and in captured graphs, in the static scratch array.
"""
import numpy as np
import pytest
import torch

import workloads as W
from metrics import assert_rows
from oracle import ts_ref

pytestmark = pytest.mark.gpu

ts = pytest.importorskip("paper_2606_19271_amd")


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ts.load()


def say(*a):
    print("[gpu-test]", *a, flush=True)


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


class Batch:
    """A chunk batch of nseq segments of uneven length, some without queries and some without keys."""

    def __init__(self, nseq, H, d, seed):
        rng = np.random.default_rng(nseq)
        self.lq = rng.integers(0, 40, nseq)
        self.lk = rng.integers(0, 40, nseq)
        self.lq[::9], self.lk[::7] = 0, 0
        self.lq[5], self.lk[5], self.lq[nseq - 2], self.lk[nseq - 2] = 300, 700, 65, 1
        self.cq, self.ck = (np.concatenate([[0], np.cumsum(x)]).astype(np.int32) for x in (self.lq, self.lk))
        g = torch.Generator().manual_seed(seed)
        self.host = [torch.randn((n, H, d), generator=g).to(torch.bfloat16)
                     for n in (self.cq[-1], self.ck[-1], self.ck[-1])]
        self.qkv = [t.cuda() for t in self.host]
        self.offsets = [torch.tensor(c, device="cuda") for c in (self.cq, self.ck)]
        self.longest = int(self.lq.max()), int(self.lk.max())

    def call(self, splits, entry=ts.ts_attn_fwd_kvcache, **out):
        return entry(*self.qkv, *self.offsets, *self.longest, return_lse=True, num_splits=splits, **out)


def same(a, b):
    return torch.equal(bits(a[0]), bits(b[0])) and torch.equal(bits(a[1]), bits(b[1]))


@pytest.mark.parametrize("nseq,H,d", [(65, 2, 128), (1500, 1, 64)])
def test_against_the_oracle(nseq, H, d):
    b = Batch(nseq, H, d, 1)
    ref, ref_lse = ts_ref.attn_kv_full(*(W.bf16_bits(t) for t in b.host), b.cq, b.ck, float(np.float32(d ** -0.5)))
    fin = np.isfinite(ref_lse)
    for splits in (1, 2, 3):
        for entry in (ts.ts_attn_fwd_kvcache, ts.ts_attn_fwd_kvcache_noalloc):
            say("plan kernel", nseq, H, d, "splits", splits, entry.__name__)
            o, lse = b.call(splits, entry)
            torch.cuda.synchronize()
            assert_rows(o.float().cpu().numpy().astype(np.float64), ref, "%d segments" % nseq, elementwise=False)
            lse = lse.cpu().numpy()
            assert np.array_equal(np.isfinite(lse), fin) and np.all(lse[~fin] == -np.inf)
            # as in the chunk tests: the bf16 weights' rounding changes the lse by at most 2e-3
            assert float(np.abs(lse[fin] - ref_lse[fin]).max()) <= 1e-2


@pytest.mark.parametrize("nseq,length,H", [(64, 130, 16), (24, 500, 40), (65, 70, 4)])
def test_segments_alone_and_in_a_batch_are_the_same(nseq, length, H):
    g = torch.Generator(device="cuda").manual_seed(2)
    q, k, v = (torch.randn((nseq * length, H, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    cu = torch.arange(nseq + 1, dtype=torch.int32, device="cuda") * length
    say("plan kernel, many items", nseq, length, H)
    many = ts.ts_attn_fwd_varlen(q, k, v, cu, length)
    for s in (0, nseq // 2, nseq - 1):
        rows = slice(s * length, (s + 1) * length)
        one = ts.ts_attn_fwd_varlen(q[rows], k[rows], v[rows], cu[:2].contiguous(), length)
        torch.cuda.synchronize()
        assert torch.equal(bits(many[rows]), bits(one)), s


@pytest.mark.parametrize("splits", [1, 2])
def test_graph_replays(splits):
    sets = [Batch(70, 2, 128, seed) for seed in (3, 4)]
    refs = [b.call(splits) for b in sets]  # outside the capture, in the workspace
    torch.cuda.synchronize()
    b = Batch(70, 2, 128, 5)
    out, lse = torch.empty_like(b.qkv[0]), torch.empty(b.qkv[0].shape[:2], dtype=torch.float32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    say("plan kernel, capture, splits", splits)
    with torch.cuda.graph(graph):
        b.call(splits, out=out, lse=lse)
    for rep in range(5):
        for dst, src in zip(b.qkv, sets[rep % 2].qkv):  # eager work between replays: new inputs in place
            dst.copy_(src)
        out.fill_(0)
        lse.fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        assert same((out, lse), refs[rep % 2]), rep


def test_streams_take_the_plan_in_turn():
    batches = [Batch(70, 2, 128, 6), Batch(200, 2, 128, 7)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for splits in (1, 2):
        say("plan kernel on two streams, splits", splits)
        refs = [b.call(splits) for b in batches]
        torch.cuda.synchronize()
        results = [[], []]
        for _ in range(6):
            for j in range(2):
                with torch.cuda.stream(streams[j]):
                    results[j].append(batches[j].call(splits))
        torch.cuda.synchronize()
        for j in range(2):
            assert all(same(r, refs[j]) for r in results[j]), j


def test_bad_offsets_are_a_no_op():
    b = Batch(70, 2, 64, 8)
    for at, value in ((0, 1), (30, -5), (30, 2 ** 31 - 1), (40, 0), (70, int(b.ck[-1]) - 1)):
        ck = b.ck.copy()
        ck[at] = value
        b.offsets[1] = torch.tensor(ck, device="cuda")
        for splits in (1, 2):
            for entry in (ts.ts_attn_fwd_kvcache, ts.ts_attn_fwd_kvcache_noalloc):
                say("plan kernel, bad offset", at, value, "splits", splits)
                out = torch.full_like(b.qkv[0], 7.0)
                lse = torch.full(out.shape[:2], 7.0, dtype=torch.float32, device="cuda")
                b.call(splits, entry, out=out, lse=lse)
                torch.cuda.synchronize()
                assert bool((out == 7.0).all()) and bool((lse == 7.0).all()), (at, value, splits)
