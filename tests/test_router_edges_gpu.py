"""The router's projection on both sides of every change of its launch shape, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests.helpers import randn_bf16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# wavefronts that share tokens (up to 3000, then up to 12000 or 131072 tokens), wavefronts of their own
# with 16 and with 32 tokens; token counts that fill no wavefront; more than 64 chunks, whose
# sums meet in two rounds; fewer chunks than wavefronts
@pytest.mark.parametrize("B,N,dm,G", [
    (1, 1, 128, 8), (3, 7, 1152, 8), (2, 1499, 256, 8), (2, 1501, 256, 8), (1, 5, 8448, 8), (1, 9, 8320, 4),
    (1, 11999, 128, 8), (1, 12001, 128, 8), (1, 23999, 256, 8), (3, 8011, 256, 8), (1, 3001, 256, 1), (1, 3001, 384, 2),
    (1, 2999, 256, 16), (1, 11999, 256, 16), (1, 24007, 256, 16), (1, 24001, 128, 4), (1, 131073, 128, 4),
    (1, 131079, 128, 2), (1, 131080, 128, 1)])
def test_router_logits_on_both_sides_of_every_rule(B, N, dm, G):
    rng = np.random.default_rng(N + dm)
    h, Wr = randn_bf16(rng, (B, N, dm)), randn_bf16(rng, (G, dm))
    for a in (h, Wr):                                      # zeros and subnormals of either sign
        hit = rng.random(a.shape)
        a[hit < 0.05] = 0x8000
        a[(hit >= 0.05) & (hit < 0.1)] &= 0x807F
    bias = rng.standard_normal(G).astype(np.float32)
    logits = torch.full((B, 1, N, G), float("nan"), dtype=torch.float32, device=DEV)
    stc.stc_router_logits(PT.to_dev_bf16(h), PT.to_dev_bf16(Wr), torch.from_numpy(bias).to(DEV), logits, 1)
    torch.cuda.synchronize()
    got = logits.cpu().numpy()
    for b in range(B):
        want = O.router_logits(h[b], Wr, bias)
        assert np.array_equal(got[b, 0].view(np.uint32), want.view(np.uint32))
