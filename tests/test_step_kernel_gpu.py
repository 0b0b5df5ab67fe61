"""Decode steps that one launch does (one workgroup per stream scores, selects and attends), and
attention with several pairs of pages per wavefront: against the two calls, bit for bit, and
against the oracle."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests.helpers import randn_bf16
from tests.test_parity_gpu import _rand_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# B, Hq, Hkv, D, N, G, k, tail tokens: every bound on the heads per KV head, one page and one pair
# over, last pairs that are half full or missing, tails that end inside a page, two workgroups
# per CU
CASES = [
    (2, 4, 4, 64, 700, 4, 16, 0), (1, 8, 8, 64, 1024, 4, 16, 0), (2, 4, 2, 128, 300, 8, 9, 0),
    (2, 6, 2, 128, 270, 8, 1, 0), (1, 8, 2, 64, 260, 8, 8, 0), (1, 14, 2, 128, 2500, 16, 15, 0),
    (2, 8, 1, 128, 4096, 8, 16, 0), (1, 5, 1, 64, 1000, 2, 12, 40), (3, 3, 3, 128, 290, 1, 13, 33),
    (2, 7, 1, 128, 500, 8, 14, 17), (64, 8, 4, 128, 530, 8, 17, 0), (64, 4, 4, 128, 600, 8, 33, 0),
    (64, 12, 4, 64, 900, 4, 48, 0), (65, 28, 4, 128, 1040, 8, 64, 0), (64, 4, 4, 128, 700, 8, 37, 70),
    (130, 16, 4, 64, 560, 8, 31, 16), (128, 8, 8, 128, 500, 8, 30, 0), (80, 16, 4, 128, 2100, 8, 127, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d_Hq%d_Hkv%d_D%d_N%d_G%d_k%d_t%d" % c)
def test_step_in_one_launch(case):
    B, Hq, Hkv, D, N, G, k, n_tail = case
    R = Hq // Hkv
    K, V, q, logits, kcount = _rand_case(17 * N + k, B, Hq, Hkv, D, N, G, outliers=True)
    rng = np.random.default_rng(5)
    c = stc.RoutedCache(B, Hq, Hkv, D, N, G, k, device=DEV, tail_cap=n_tail + 3 if n_tail else 0)
    c.build(PT.to_dev_bf16(K), PT.to_dev_bf16(V), logits=torch.from_numpy(logits).to(DEV),
            kcount=torch.from_numpy(kcount).to(DEV))
    if n_tail:
        Kt, Vt = randn_bf16(rng, (B, Hkv, n_tail, D)), randn_bf16(rng, (B, Hkv, n_tail, D))
        c.K_tail[:, :, :n_tail] = PT.to_dev_bf16(Kt)
        c.V_tail[:, :, :n_tail] = PT.to_dev_bf16(Vt)
        c.n_tail = n_tail
    dq = PT.to_dev_bf16(q)
    got = {}
    for one in (False, True):
        c.page_score.fill_(float("nan"))
        c.page_idx.fill_(-7)
        c.out.fill_(float("nan"))
        c.step(dq, one_call=one)
        torch.cuda.synchronize()
        got[one] = (c.page_idx.clone(), c.out.clone(), c.page_score.clone())
    assert torch.equal(got[False][0], got[True][0]) and torch.equal(got[False][1], got[True][1])
    assert torch.equal(got[False][2].view(torch.int32), got[True][2].view(torch.int32))
    idx, out, score = (t.cpu().numpy() for t in got[True])
    for s in sorted({0, 1, B * Hkv // 2, B * Hkv - 1} & set(range(B * Hkv))):
        b, h = s // Hkv, s % Hkv
        m = O.route_mask(logits[b, h], kcount[b, h])
        qh = q[b, h * R:(h + 1) * R]
        want = O.page_scores(qh, O.page_bounds(K[b, h]))
        assert np.array_equal(score[b, h].view(np.uint32), want.view(np.uint32))
        pages = O.select_pages(want, k)
        assert np.array_equal(idx[b, h], pages)
        tail = dict(K_tail=Kt[b, h], V_tail=Vt[b, h]) if n_tail else {}
        ref = O.decode_attention(qh, K[b, h], V[b, h], m, pages, G, **tail)
        assert np.abs(out[b, h * R:(h + 1) * R] - ref).max() < PT.TIGHT
