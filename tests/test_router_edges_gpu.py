"""The router's projection on both sides of every change of its launch shape, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests import routes
from tests.helpers import randn_bf16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# wavefronts that share 8 tokens (up to 3000, or elements of up to 8) or 16, wavefronts of their own
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


@pytest.mark.parametrize("B,N,dm,G,form", [
    (3001, 1, 128, 8, routes.OWN16), (3001, 1, 1024, 8, routes.OWN16), (400, 8, 256, 4, routes.SPLIT8),
    (1, 2048, 128, 4, routes.SPLIT8), (1, 2049, 128, 4, routes.SPLIT16), (2049, 1, 1024, 16, routes.SPLIT8),
    (600, 9, 256, 16, routes.OWN16), (300, 17, 128, 8, routes.OWN16), (300, 33, 128, 8, routes.OWN16),
    (300, 63, 256, 2, routes.OWN16), (455, 65, 128, 16, routes.OWN32), (400, 97, 128, 4, routes.OWN32),
    (3001, 1, 3584, 8, routes.SPLIT8),
    (1, 24001, 128, 4, routes.OWN16), (1, 32769, 128, 2, routes.OWN16), (1, 32769, 2048, 4, routes.SPLIT16),
    (1, 57313, 2048, 1, routes.OWN32), (1, 43681, 256, 16, routes.OWN16), (7, 6241, 128, 16, routes.OWN16),
    (1, 65535, 128, 8, routes.OWN32)])
def test_router_logits_of_many_elements_and_of_every_form(B, N, dm, G, form):
    """Elements that end inside a wavefront or leave wavefronts of a workgroup without tokens, and both
    sides of the lines between the forms: the first, last and some other tokens bit for bit, every
    logit written."""
    assert routes.router_form(B, N, dm, G) == form
    g = torch.Generator(device=DEV)
    g.manual_seed(N + dm)
    h = torch.randn(B, N, dm, device=DEV, generator=g).bfloat16()
    Wr = torch.randn(G, dm, device=DEV, generator=g).bfloat16()
    bias = torch.randn(B, G, device=DEV, generator=g)
    logits = torch.full((B, 2, N, G), float("nan"), dtype=torch.float32, device=DEV)
    stc.stc_router_logits(h, Wr, bias, logits, 2)
    torch.cuda.synchronize()
    assert torch.equal(logits[:, 0], logits[:, 1]) and bool(torch.isfinite(logits).all())
    rng = np.random.default_rng(N)
    for b in sorted({0, B // 2, B - 1}):
        at = sorted({*range(min(N, 40)), *range(max(0, N - 40), N), *rng.integers(0, N, 100).tolist()})
        want = O.router_logits(PT.host_bf16(h[b, at]), PT.host_bf16(Wr), bias[b].cpu().numpy())
        assert np.array_equal(logits[b, 0, at].cpu().numpy().view(np.uint32), want.view(np.uint32))
