"""Attention with one page per wavefront, at the edges of where it is taken and of its workgroups, and
the merge of few and of many partial results: the one-call step equals the two calls bit for bit,
and the oracle within the tight bound."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests import routes
from tests.test_launch_plans_gpu import Case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# B, Hq, Hkv, D, N, G, k, tail tokens, pages per wavefront
STEPS = [
    # workgroups of 8 pages: one page, seven pages and none missing in the last
    (1, 4, 2, 128, 500 * 16, 8, 17, 0, 1), (1, 8, 8, 64, 400 * 16 - 3, 4, 23, 0, 1), (1, 14, 2, 128, 300 * 16, 16, 24, 0, 1),
    (2, 16, 1, 128, 600 * 16, 8, 33, 0, 1), (3, 3, 3, 64, 290 * 16, 8, 63, 0, 1),
    # at most 256 of them, and more
    (2, 32, 32, 64, 260 * 16, 8, 32, 0, 1), (4, 4, 4, 128, 1000 * 16, 8, 128, 0, 1), (2, 32, 32, 64, 260 * 16, 8, 33, 0, 2),
    (17, 4, 1, 128, 1000 * 16, 8, 128, 0, 2),
    # pairs on more than 256 workgroups, and single pages on at most 512 that select, or more
    (87, 4, 1, 128, 300 * 16 - 5, 8, 33, 0, 1), (43, 2, 1, 64, 700 * 16, 8, 90, 0, 2), (44, 2, 1, 64, 700 * 16, 8, 88, 0, 1),
    (40, 4, 1, 128, 300 * 16, 8, 90, 100, 1), (128, 1, 1, 64, 300 * 16, 4, 32, 1, 1), (129, 1, 1, 64, 300 * 16, 4, 32, 1, 2),
    # tail pages in the last workgroup, alone in several, and in the middle of one
    (1, 4, 1, 128, 290 * 16, 8, 16, 1, 1), (2, 4, 2, 64, 300 * 16, 4, 20, 200, 1), (1, 7, 1, 128, 400 * 16, 8, 24, 127, 1),
    # 16 keys per thread; the selection as a launch of its own; every page
    (1, 14, 2, 128, 2049 * 16, 8, 130, 0, 1), (1, 4, 2, 64, 8192 * 16, 8, 257, 40, 1), (1, 2, 1, 64, 8193 * 16, 4, 300, 0, 1),
    # merges of 2, 3, 15, 16 and 17 partial results of 1 to 9 heads
    (1, 1, 1, 128, 300 * 16, 8, 17, 0, 1), (1, 1, 1, 64, 300 * 16, 8, 20, 0, 1), (3, 3, 3, 64, 260 * 16, 4, 17, 0, 1),
    (1, 5, 1, 128, 260 * 16, 8, 120, 0, 1), (1, 9, 1, 64, 260 * 16, 8, 128, 0, 1), (1, 3, 1, 128, 260 * 16, 8, 128, 0, 1),
    (1, 5, 1, 64, 260 * 16, 8, 129, 0, 1), (3, 2, 2, 128, 260 * 16, 8, 136, 0, 1),
    # merges of 33, 64, 65, 129 and 300 partial results
    (1, 5, 1, 64, 2500 * 16, 8, 264, 0, 1), (1, 4, 1, 128, 1500 * 16, 8, 512, 0, 1), (1, 16, 1, 64, 2000 * 16, 8, 513, 0, 1),
    (1, 4, 1, 64, 2200 * 16, 8, 1025, 0, 1), (1, 4, 1, 128, 2401 * 16, 8, 2400, 0, 2),
]


def wave_pages(B, Hq, Hkv, D, N, k, n_tail=0, kv_div=1):
    f = routes._rule("_ZN3stc20attention_wave_pagesERK9stc_shapeiii", routes._P, routes._I, routes._I, routes._I,
                     restype=routes._I)
    return f(routes._shape(B, Hq, Hkv, D, N), k, (n_tail + 15) // 16, kv_div)


@pytest.mark.parametrize("case", STEPS, ids=lambda c: "B%d_Hq%d_Hkv%d_D%d_N%d_G%d_k%d_t%d_%d" % c)
def test_step_with_single_pages(case):
    *shape, n_tail, pages_per_wave = case
    B, Hq, Hkv, D, N, G, k = shape
    assert wave_pages(B, Hq, Hkv, D, N, k, n_tail) == pages_per_wave
    t = Case(*shape, n_tail=n_tail)
    got = {}
    for one in (False, True):
        t.c.page_idx.fill_(-7)
        t.c.out.fill_(float("nan"))
        t.c.step(t.q, one_call=one)
        torch.cuda.synchronize()
        got[one] = (t.c.page_idx.clone(), t.c.out.clone())
    assert torch.equal(got[False][0], got[True][0]) and torch.equal(got[False][1], got[True][1])
    for b, h in t.streams():
        want = O.page_scores(t.heads(b, h), O.page_bounds(PT.host_bf16(t.K[b, h])))
        pages = O.select_pages(want, k)
        assert np.array_equal(t.c.page_idx[b, h].cpu().numpy(), pages)
        t.check(t.c.out, b, h, pages)


@pytest.mark.parametrize("B,Hq,Hkv,D,k", [(1, 8, 4, 128, 40), (2, 4, 2, 64, 100), (1, 16, 1, 128, 17)])
def test_lists_with_skipped_entries_and_single_pages(B, Hq, Hkv, D, k):
    """Entries outside [0, NP) count for nothing: single ones, a whole workgroup's, and all."""
    NP = 140
    N = 16 * NP - 6
    assert wave_pages(B, Hq, Hkv, D, N, k) == 1
    t = Case(B, Hq, Hkv, D, N, 8, k)
    rng = np.random.default_rng(k)
    lists = np.stack([rng.permutation(NP)[:k] for _ in range(B * Hkv)]).reshape(B, Hkv, k).astype(np.int32)
    skip = rng.random(lists.shape) < 0.3
    lists[skip] = rng.choice([-1, NP, NP + 1, -(1 << 31), (1 << 31) - 1], size=int(skip.sum()))
    lists[0, 0, :8] = -1
    if B * Hkv > 1:
        lists[B - 1, Hkv - 1] = -1                          # nothing at all: zeros
    t.c.page_idx.copy_(torch.from_numpy(lists))
    t.c.out.fill_(float("nan"))
    t.c.attend(t.q)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(t.c.out).all())
    for b in range(B):
        for h in range(Hkv):
            kept = lists[b, h][(lists[b, h] >= 0) & (lists[b, h] < NP)]
            if len(kept):
                t.check(t.c.out, b, h, kept)
            else:
                assert not t.c.out[b, h * t.R:(h + 1) * t.R].any()
