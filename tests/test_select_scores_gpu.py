"""The selection of pages on scores of every kind, in every kernel that selects: the list is the k
largest of the scores that the call itself left, by the order of their bits as numbers (-0 does
not occur, NaN above or below everything by its sign), the lowest pages first among equal ones."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 64


def kinds(streams, NP, k, g):
    """name -> [streams, NP, 2] values; a page's score is about the sum of its two."""
    u = lambda *s: torch.rand(*s, generator=g, device=DEV)
    z = torch.randn(streams, NP, 2, generator=g, device=DEV)
    pages = torch.arange(NP, device=DEV).float()
    out = {"positive": 40 + 5 * z, "mixed signs": z, "negative": -40 + 5 * z,
           "equal": torch.full_like(z, 3.0), "zeros": torch.zeros_like(z),
           "few values": (u(streams, NP, 2) * 4).floor() + 1,
           "8 octaves and more": torch.exp(8 * z), "all magnitudes": torch.exp(25 * z.clamp(-3, 3)),
           "rising": (pages[None, :, None] / 64 + 1).expand(streams, NP, 2),
           "large at the end": 8 + z.abs() + 100 * (pages >= NP - k - 3)[None, :, None],
           "mostly zero": torch.where(u(streams, NP, 1) < 0.03, 5 + z.abs(), torch.zeros_like(z)),
           # as many pages above the equal ones that only some of them are taken
           "ties at the end": torch.where(u(streams, NP, 1) < 0.5 * k / NP, 50 + z, torch.full_like(z, 20.0)),
           "tiny": 1e-37 * (1 + u(streams, NP, 2)), "close together": 64 + z.clamp(-3, 3) * 0.5,
           # fewer positive scores than are kept; enough of them, but not among the maxima of adjacent pages
           "half positive": torch.where(pages[None, :, None] < k / 2, 5 + z.abs(), -5 - z.abs()),
           "positive at the end": torch.where(pages[None, :, None] >= NP - k - 3, 5 + z.abs(), -5 - z.abs()),
           "one far below": torch.where(pages[None, :, None] == 1, torch.full_like(z, 1e-30), 40 + 5 * z)}
    nan = 40 + 5 * z
    nan[:, NP // 2] = float("inf")        # times the zeros of the other channels
    out["not finite"] = nan
    return out


def expected(score, k):
    b = score.contiguous().view(torch.int32).cpu().numpy().astype(np.int64) & 0xffffffff
    key = np.where(b & 0x80000000, 0xffffffff - b, b | 0x80000000)
    order = np.argsort(-key, axis=-1, kind="stable")[..., :k]
    return np.sort(order, axis=-1)


@pytest.mark.parametrize("B,Hkv,R,NP,ks", [
    # query heads per KV head, pages: the selecting kernel
    (1, 2, 9, 3, (1, 2)), (1, 2, 9, 31, (1, 30)), (2, 2, 9, 64, (1, 17, 63)), (2, 2, 9, 65, (16, 64)), (2, 2, 9, 256, (1, 17, 255)),      # 256 threads: 1 key each
    (2, 2, 9, 257, (9, 100)), (1, 2, 9, 511, (64, 510)),                             # 2 keys
    (2, 1, 9, 513, (1, 40, 112, 113)), (1, 2, 9, 1023, (20, 200, 223, 224, 1000)),   # 4 keys
    (2, 1, 9, 1025, (8, 60, 223, 224)), (2, 2, 9, 2048, (7, 128, 447, 448, 2047)),   # 512 threads: 4 keys
    (1, 2, 9, 2049, (128, 300)), (1, 2, 9, 4096, (200, 511, 600, 896, 897)),         # 8 keys
    (1, 3, 2, 4097, (9, 100, 500)), (1, 2, 7, 8191, (16, 256, 512, 1000)), (1, 2, 1, 8192, (255, 700, 1792, 1793)),
    (1, 2, 2, 8193, (100,)),                                                         # the loop over all keys
    (3, 2, 1, 2, (1,)), (3, 2, 2, 64, (1, 16, 63)), (2, 2, 4, 65, (8, 16)), (2, 2, 1, 127, (16, 40, 126)), (2, 2, 2, 128, (1, 16, 127)),
    (2, 2, 1, 129, (16, 128)), (2, 2, 1, 255, (16, 17, 254)),   # a whole step, scoring and selection
    (50, 4, 1, 1001, (12, 128)), (50, 4, 4, 700, (100,)), (35, 4, 3, 640, (90, 639)),
])
def test_select_scores(B, Hkv, R, NP, ks):
    Hq, N = Hkv * R, NP * 16 - 3
    q = torch.zeros(B, Hq, D, dtype=torch.bfloat16, device=DEV)
    q[:, ::R, :2] = 1.0                   # the other heads of a group score 0 ..
    q[:, :, :2] += (torch.arange(Hq, device=DEV) % R != 0).to(torch.bfloat16)[None, :, None]  # .. or the same
    for k in ks:
        g = torch.Generator(device=DEV)
        g.manual_seed(100 * NP + k)
        c = stc.RoutedCache(B, Hq, Hkv, D, N, 4, k, device=DEV)
        V = torch.zeros(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
        for name, v in kinds(B * Hkv, NP, k, g).items():
            K = torch.zeros(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
            K[..., :2] = v.view(B, Hkv, NP, 1, 2).expand(B, Hkv, NP, 16, 2).reshape(B, Hkv, NP * 16, 2)[:, :, :N].bfloat16()
            c.build(K, V, mask_in=torch.full((B, Hkv, N), 15, dtype=torch.int16, device=DEV))
            for call in ("select", "step"):
                c.page_idx.fill_(-7)
                c.page_score.fill_(float("nan"))
                c.select(q) if call == "select" else c.step(q)
                want = expected(c.page_score.view(B * Hkv, NP), k)
                got = c.page_idx.view(B * Hkv, k).cpu().numpy()
                assert (got == want).all(), (name, call, k)
