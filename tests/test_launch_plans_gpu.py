"""Every launch plan of the decode step and of the attention calls, at the edges of its range: the route
that a shape is meant to take is asked from the library's own rules, so that a case which a
changed rule sends elsewhere fails.  Inputs are made on the GPU; outputs are compared with the
oracle on sampled streams, and across the calls that have to agree bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests import routes

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Case:
    def __init__(self, B, Hq, Hkv, D, N, G, k, n_tail=0, seed=0):
        g = torch.Generator(device=DEV)
        g.manual_seed(1000 * N + k + seed)
        self.B, self.Hq, self.Hkv, self.D, self.N, self.G, self.R = B, Hq, Hkv, D, N, G, Hq // Hkv
        new = lambda *s: torch.randn(*s, device=DEV, generator=g, dtype=torch.bfloat16)
        self.K, self.V, self.q = new(B, Hkv, N, D), new(B, Hkv, N, D), new(B, Hq, D)
        self.c = stc.RoutedCache(B, Hq, Hkv, D, N, G, k, device=DEV, tail_cap=n_tail + 2 if n_tail else 0)
        self.c.build(self.K, self.V, logits=torch.randn(B, Hkv, N, G, device=DEV, generator=g), fixed_k=(G + 1) // 2)
        if n_tail:
            self.c.K_tail.copy_(new(*self.c.K_tail.shape))
            self.c.V_tail.copy_(new(*self.c.V_tail.shape))
            self.c.n_tail = n_tail

    def streams(self):
        return sorted({(0, 0), (self.B // 2, self.Hkv // 2), (self.B - 1, self.Hkv - 1)})

    def heads(self, b, h):
        return PT.host_bf16(self.q[b, h * self.R:(h + 1) * self.R])

    def attention(self, b, h, pages, qh=None):
        """The oracle's output of stream (b, h) over the given pages and the tail."""
        n = self.c.n_tail
        tail = dict(K_tail=PT.host_bf16(self.c.K_tail[b, h, :n]), V_tail=PT.host_bf16(self.c.V_tail[b, h, :n])) if n else {}
        return O.decode_attention(self.heads(b, h) if qh is None else qh, PT.host_bf16(self.K[b, h]),
                                  PT.host_bf16(self.V[b, h]), PT.host_u16(self.c.mask[b, h]), pages, self.G, **tail)

    def check(self, out, b, h, pages):
        got = out[b, h * self.R:(h + 1) * self.R].cpu().numpy()
        assert np.abs(got - self.attention(b, h, pages)).max() < PT.TIGHT

    def ws(self, which, k):
        return torch.full((max(16, stc.stc_workspace_bytes(self.c.shape, which, k)),), 0xA5, dtype=torch.uint8, device=DEV)


# B, Hq, Hkv, D, N, G, k, tail tokens, launches, pairs of pages per wavefront
STEPS = [
    # one launch, 5 .. 8 pairs; the last slots of the eighth pair empty, half full and full
    (48, 4, 4, 64, 1300, 4, 65, 0, "one", 5), (64, 4, 4, 128, 1700, 8, 96, 0, "one", 6),
    (48, 8, 4, 128, 1900, 8, 112, 0, "one", 7), (64, 8, 4, 128, 2000, 8, 113, 0, "one", 8),
    (50, 4, 4, 64, 2090, 4, 127, 0, "one", 8), (48, 4, 4, 64, 2200, 4, 128, 0, "one", 8),
    # the tail takes the last slots, and one more than there are
    (48, 4, 4, 64, 2200, 4, 120, 128, "one", 8), (48, 4, 4, 64, 2200, 4, 120, 129, "with scores", 1),
    # pages per stream that one launch scores: 192 for many heads, 256, up to 1024 for many streams
    (1, 14, 2, 128, 192 * 16, 8, 14, 0, "one", 1), (1, 14, 2, 128, 192 * 16 + 1, 8, 14, 0, "in attention", 1),
    (3, 8, 2, 64, 256 * 16, 4, 16, 0, "one", 1), (3, 8, 2, 64, 256 * 16 + 1, 4, 16, 0, "in attention", 1),
    (48, 4, 4, 64, 257 * 16 - 5, 4, 20, 0, "one", 2), (48, 4, 4, 64, 1023 * 16, 4, 33, 0, "one", 3),
    (48, 28, 4, 64, 1000 * 16 - 1, 4, 40, 0, "one", 3), (24, 64, 8, 64, 600 * 16, 4, 9, 0, "one", 1),
    (64, 16, 4, 128, 1024 * 16 - 3, 8, 100, 0, "one", 7), (128, 4, 4, 64, 300 * 16, 4, 50, 30, "one", 4),
    # one page more: selection inside the attention kernel with several pairs
    (48, 4, 4, 64, 1025 * 16 - 9, 4, 20, 0, "in attention", 2), (48, 4, 4, 64, 1100 * 16, 4, 70, 0, "in attention", 5),
    (64, 16, 4, 128, 1100 * 16, 8, 128, 0, "in attention", 8), (48, 4, 4, 64, 1200 * 16, 4, 60, 50, "in attention", 4),
    (48, 4, 4, 64, 2048 * 16, 4, 33, 0, "in attention", 3), (64, 36, 3, 128, 300 * 16, 8, 20, 0, "in attention", 2),
    (16, 192, 12, 64, 500 * 16, 4, 90, 17, "in attention", 6),
    # more pages than it orders, more streams than are resident, fewer than fill the chip
    (48, 4, 4, 64, 2049 * 16, 4, 33, 0, "three", 3), (86, 3, 3, 128, 400 * 16, 8, 40, 0, "with scores", 1),
    (47, 8, 4, 128, 300 * 16, 8, 30, 0, "in attention", 1),
    (129, 4, 4, 64, 300 * 16, 4, 40, 0, "with scores", 1),
    # 4 wavefronts that select, 8 keys per thread
    (1, 4, 2, 128, 257 * 16, 8, 8, 0, "in attention", 1), (1, 2, 2, 64, 2048 * 16, 4, 8, 0, "in attention", 1),
    (2, 18, 2, 128, 900 * 16 + 3, 8, 5, 0, "in attention", 1), (1, 3, 1, 128, 1500 * 16, 8, 4, 60, "in attention", 1),
]


@pytest.mark.parametrize("case", STEPS, ids=lambda c: "B%d_Hq%d_Hkv%d_D%d_N%d_G%d_k%d_t%d_%s_%d" % c)
def test_step(case):
    """Page list, scores and output of the one-call step equal the two calls' bit for bit, the list and
    the scores the oracle's, the output within the tight bound."""
    *shape, n_tail, launches, pairs = case
    B, Hq, Hkv, D, N, G, k = shape
    assert routes.step(B, Hq, Hkv, D, N, k, n_tail) == launches
    assert routes.pairs(B, Hq, Hkv, D, N, k, n_tail=n_tail) == pairs
    t = Case(*shape, n_tail=n_tail)
    got = {}
    for one in (False, True):
        t.c.page_score.fill_(float("nan"))
        t.c.page_idx.fill_(-7)
        t.c.out.fill_(float("nan"))
        t.c.step(t.q, one_call=one)
        torch.cuda.synchronize()
        got[one] = (t.c.page_idx.clone(), t.c.out.clone(), t.c.page_score.view(torch.int32).clone())
    assert torch.equal(got[False][0], got[True][0]) and torch.equal(got[False][1], got[True][1])
    assert torch.equal(got[False][2], got[True][2])
    for b, h in t.streams():
        want = O.page_scores(t.heads(b, h), O.page_bounds(PT.host_bf16(t.K[b, h])))
        assert np.array_equal(t.c.page_score[b, h].cpu().numpy().view(np.uint32), want.view(np.uint32))
        pages = O.select_pages(want, k)
        assert np.array_equal(t.c.page_idx[b, h].cpu().numpy(), pages)
        t.check(t.c.out, b, h, pages)


@pytest.mark.parametrize("B,Hq,Hkv,D,N,G,k,n_tail", [
    (48, 4, 4, 64, 2049 * 16, 4, 17, 0), (48, 8, 4, 128, 4096 * 16 - 5, 8, 32, 0), (51, 5, 5, 64, 4096 * 16, 4, 32, 0),
    (51, 5, 5, 128, 2049 * 16, 8, 17, 0), (32, 6, 6, 64, 2500 * 16, 4, 20, 60), (48, 4, 4, 128, 2049 * 16, 8, 30, 17),
    (51, 5, 5, 64, 4096 * 16, 4, 16, 1)])
def test_many_long_streams_with_several_pairs(B, Hq, Hkv, D, N, G, k, n_tail):
    """192 to 255 streams of more pages than a launch of several pairs per wavefront orders: the largest
    scores are those of the pages from 2048 on, and the step finds them as the two calls do."""
    assert routes.pairs(B, Hq, Hkv, D, N, k, n_tail=n_tail) == 2
    assert routes.step(B, Hq, Hkv, D, N, k, n_tail) == "three"
    t = Case(B, Hq, Hkv, D, N, G, k, n_tail=n_tail)
    t.K[:, :, 2048 * 16:] *= 2
    stc.stc_build_page_bounds(t.c.shape, t.K, t.c.bounds)
    got = {}
    for one in (False, True):
        t.c.page_idx.fill_(-7)
        t.c.out.fill_(float("nan"))
        t.c.step(t.q, one_call=one)
        torch.cuda.synchronize()
        got[one] = (t.c.page_idx.clone(), t.c.out.clone())
    assert torch.equal(got[False][0], got[True][0]) and torch.equal(got[False][1], got[True][1])
    for b, h in t.streams():
        pages = O.select_pages(O.page_scores(t.heads(b, h), O.page_bounds(PT.host_bf16(t.K[b, h]))), k)
        assert pages[-1] >= 2048 and np.array_equal(t.c.page_idx[b, h].cpu().numpy(), pages)
        t.check(t.c.out, b, h, pages)


@pytest.mark.parametrize("B,Hq,Hkv,D,N,G,pairs", [(48, 4, 4, 64, 100 * 16 - 3, 4, 7), (48, 4, 4, 128, 128 * 16, 8, 8),
                                                  (64, 28, 4, 128, 33 * 16 - 15, 8, 3), (4, 4, 2, 128, 17 * 16, 8, 1)])
def test_every_page_attended_and_the_list_written(B, Hq, Hkv, D, N, G, pairs):
    NP = (N + 15) // 16
    assert routes.pairs(B, Hq, Hkv, D, N, NP) == pairs
    t = Case(B, Hq, Hkv, D, N, G, NP)
    lst = torch.full((B, Hkv, NP), -7, dtype=torch.int32, device=DEV)
    out, out2 = torch.full_like(t.c.out, float("nan")), torch.full_like(t.c.out, float("nan"))
    args = (t.c.shape, t.q)
    stc.stc_decode_step(*args, t.c.bounds, t.K, t.c.vpacked, t.c.mask, t.c.tok_off, NP, lst, out, t.ws(stc.STC_WS_STEP, NP))
    stc.stc_decode_attention(*args, t.K, t.c.vpacked, t.c.mask, t.c.tok_off, None, NP, out2, t.ws(stc.STC_WS_ATTENTION, NP))
    torch.cuda.synchronize()
    assert torch.equal(lst, torch.arange(NP, dtype=torch.int32, device=DEV).expand(B, Hkv, NP))
    assert torch.equal(out, out2)
    for b, h in t.streams():
        t.check(out, b, h, np.arange(NP))


@pytest.mark.parametrize("B,Hq,Hkv,D,k,pairs", [(64, 4, 4, 128, 40, 3), (48, 8, 4, 64, 128, 8), (48, 28, 4, 128, 81, 6)])
def test_lists_in_any_order_with_skipped_entries_and_several_pairs(B, Hq, Hkv, D, k, pairs):
    """Entries outside [0, NP) count for nothing, wherever they lie: alone, as both pages of a pair, and
    as all pages of a wavefront."""
    NP = 140
    N = 16 * NP - 6
    assert routes.pairs(B, Hq, Hkv, D, N, k) == pairs
    t = Case(B, Hq, Hkv, D, N, 8, k)
    rng = np.random.default_rng(k)
    lists = np.stack([rng.permutation(NP)[:k] for _ in range(B * Hkv)]).reshape(B, Hkv, k).astype(np.int32)
    skip = rng.random(lists.shape) < 0.3
    lists[skip] = rng.choice([-1, NP, NP + 1, -(1 << 31), (1 << 31) - 1], size=int(skip.sum()))
    lists[0, 0, :2 * pairs] = -1
    lists[B - 1, Hkv - 1] = -1                              # nothing at all: zeros
    t.c.page_idx.copy_(torch.from_numpy(lists))
    t.c.out.fill_(float("nan"))
    t.c.attend(t.q)
    torch.cuda.synchronize()
    assert not t.c.out[B - 1, Hq - t.R:].any() and bool(torch.isfinite(t.c.out).all())
    for b, h in t.streams()[:-1]:
        t.check(t.c.out, b, h, lists[b, h][(lists[b, h] >= 0) & (lists[b, h] < NP)])


@pytest.mark.parametrize("B,Hq,Hkv,D,N,G,k,pairs,upairs", [
    (8, 28, 4, 128, 200 * 16 - 7, 8, 40, 3, 1), (64, 4, 1, 64, 150 * 16, 4, 17, 2, 1),
    (8, 28, 4, 128, 200 * 16, 8, 49, 1, 1), (48, 16, 4, 128, 150 * 16 - 1, 8, 20, 1, 5),
    (64, 12, 3, 64, 128 * 16, 4, 32, 1, 8), (64, 8, 4, 128, 300 * 16, 8, 64, 1, 8), (64, 8, 4, 128, 300 * 16, 8, 65, 1, 1)])
def test_lists_per_query_head_and_their_union(B, Hq, Hkv, D, N, G, k, pairs, upairs):
    """Attention over a list per query head (heads of a KV head share its cache), and over the union of
    the lists with the set of heads of each page, which is padded with skipped entries."""
    NP, R = (N + 15) // 16, Hq // Hkv
    U = min(NP, R * k)
    assert routes.pairs(B, Hq, Hq, D, N, k, kv_div=R) == pairs
    assert routes.pairs(B, Hq, Hkv, D, N, U) == upairs
    t = Case(B, Hq, Hkv, D, N, G, k)
    c = t.c
    idx = torch.full((B, Hq, k), -9, dtype=torch.int32, device=DEV)
    out, out_u = (torch.full((B, Hq, D), float("nan"), dtype=torch.float32, device=DEV) for _ in range(2))
    uidx = torch.full((B, Hkv, U), -5, dtype=torch.int32, device=DEV)
    uheads = torch.full((B, Hkv, U), -1, dtype=torch.int16, device=DEV)
    stc.stc_select_pages_per_head(c.shape, t.q, c.bounds, k, idx, None, t.ws(stc.STC_WS_SELECT_PER_HEAD, k))
    stc.stc_decode_attention_per_head(c.shape, t.q, c.K, c.vpacked, c.mask, c.tok_off, idx, k, out,
                                      t.ws(stc.STC_WS_ATTENTION_PER_HEAD, k))
    stc.stc_union_pages(c.shape, idx, k, uidx, uheads)
    stc.stc_decode_attention_union(c.shape, t.q, c.K, c.vpacked, c.mask, c.tok_off, uidx, uheads, out_u,
                                   t.ws(stc.STC_WS_ATTENTION, U))
    torch.cuda.synchronize()
    assert bool((uidx == -1).any()) or U == NP
    for b, h in t.streams():
        bounds, qh = O.page_bounds(PT.host_bf16(t.K[b, h])), t.heads(b, h)
        for r in range(R):
            pages = O.select_pages(O.page_scores(qh[r:r + 1], bounds), k)
            assert np.array_equal(idx[b, h * R + r].cpu().numpy(), pages)
            want = t.attention(b, h, pages, qh[r:r + 1])[0]
            for o in (out, out_u):
                assert np.abs(o[b, h * R + r].cpu().numpy() - want).max() < PT.TIGHT


def test_steps_in_one_launch_replayed_from_a_hip_graph():
    """Steps in one launch, with and without a tail, and attention that selects with several pairs,
    captured into one graph and replayed four times with fresh queries and eager work in between."""
    specs = [((2, 8, 2, 128, 700, 8, 14), 0, "one"), ((1, 4, 4, 64, 1000, 4, 9), 40, "one"),
             ((48, 4, 4, 64, 3000, 4, 40), 0, "one"), ((48, 4, 4, 64, 1100 * 16, 4, 24), 0, "in attention")]
    cases = []
    for shape, n_tail, launches in specs:
        assert routes.step(*shape[:5], shape[6], n_tail) == launches
        cases.append(Case(*shape, n_tail=n_tail))
    for t in cases:
        t.c.step(t.q)                                       # eager first: set-up of the launches
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            for t in cases:
                t.c.step(t.q)
    torch.cuda.synchronize()
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    for rep in range(4):
        want = []
        for t in cases:
            t.q.copy_(torch.randn(t.q.shape, device=DEV, generator=g))
            t.c.step(t.q)                                   # eager
            want.append((t.c.page_idx.clone(), t.c.out.clone()))
            t.c.page_idx.fill_(-1)
            t.c.out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, (wi, wo) in zip(cases, want):
            assert torch.equal(t.c.page_idx, wi) and torch.equal(t.c.out, wo), rep
