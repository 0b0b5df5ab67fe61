"""Cache construction at the edges of its kernels' tiles: page bounds (2 pages per wavefront,
8 per tile), the packed copy (64 tokens per workgroup, chunks of 256), against the oracle, bit
for bit."""
import numpy as np
import pytest
import torch

import paper_2604_21335_amd as stc
from oracle import stc_oracle as O
from tests import parity as PT
from tests.helpers import randn_bf16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D,G,room", [(128, 8, 0), (128, 16, 37), (128, 1, 0), (64, 4, 5), (64, 8, 0)])
@pytest.mark.parametrize("N", [1, 15, 17, 63, 64, 65, 129, 255, 256, 257, 321, 528])
def test_bounds_and_packed_copy_at_tile_edges(N, D, G, room):
    """Every array of the cache, with and without spare token capacity; slots behind the kept
    groups stay untouched, and so do those behind a capacity that ends inside a workgroup's run."""
    B, Hkv = 2, 3
    rng = np.random.default_rng(1000 * D + 10 * G + N)
    K, V = randn_bf16(rng, (B, Hkv, N, D)), randn_bf16(rng, (B, Hkv, N, D))
    K[0, 0, ::3] = 0x8000                                  # -0 next to ordinary values
    mask = rng.integers(0, 1 << G, size=(B, Hkv, N)).astype(np.uint16)
    mask[1, 1] = 0                                         # a stream that keeps nothing
    mask[1, 2] = (1 << G) - 1                              # and one that keeps everything
    want = [[(m := mask[b, h], off := O.token_offsets(m, G), O.pack_values(V[b, h], m, off, G))
             for h in range(Hkv)] for b in range(B)]
    # one less than the kept groups of the second stream, so that its last slot is dropped
    tight = max(1, int(want[0][1][1][-1]) - 1)
    for cap in ((N + room) * G, tight):
        c = stc.RoutedCache(B, Hkv, Hkv, D, N, G, 1, v_cap_groups=cap, device=DEV,
                            n_cap=N + room if room else 0)
        c.vpacked.view(torch.int16).fill_(0x7FC0)
        c.build(PT.to_dev_bf16(K), PT.to_dev_bf16(V), mask_in=PT.to_dev_u16(mask))
        torch.cuda.synchronize()
        rows, vp = PT.host_bf16(c.bounds_rows()), PT.host_bf16(c.vpacked)
        over = False
        for b in range(B):
            for h in range(Hkv):
                m, off, packed = want[b][h]
                n = min(int(off[-1]), cap)
                over |= int(off[-1]) > cap
                assert np.array_equal(rows[b, h], O.page_bounds(K[b, h]))
                assert np.array_equal(PT.host_u16(c.mask)[b, h, :N], m)
                assert np.array_equal(c.tok_off.cpu().numpy().view(np.uint32)[b, h, :N + 1], off)
                assert np.array_equal(vp[b, h, :n], packed[:n])
                assert np.all(vp[b, h, n:] == 0x7FC0)
        assert int(c.dev_status.item()) == int(over)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N", [1, 16, 17, 32, 33, 97, 128, 130, 145, 208, 225, 241, 256, 257, 273, 289])
@pytest.mark.parametrize("room", [0, 200])
def test_bounds_of_short_streams_and_their_padding_pages(D, N, room):
    """Streams of up to 8 wavefronts of 2 pages are one workgroup, longer ones several of 4: bounds
    equal the oracle's, the padding pages of the last tile hold zeros, further tiles are untouched."""
    B, Hkv = 2, 5
    rng = np.random.default_rng(31 * N + D)
    K = randn_bf16(rng, (B, Hkv, N, D))
    c = stc.RoutedCache(B, Hkv, Hkv, D, N, 1, 1, device=DEV, n_cap=N + room if room else 0)
    if room:
        c.K.fill_(float("inf"))                            # rows behind the last token count for nothing
        c.K[:, :, :N].copy_(PT.to_dev_bf16(K))
    else:
        c.K = PT.to_dev_bf16(K)
    c.bounds.view(torch.int16).fill_(0x7FC0)
    stc.stc_build_page_bounds(c.shape, c.K, c.bounds)
    torch.cuda.synchronize()
    rows = PT.host_bf16(c.bounds_rows())
    NP = (N + 15) // 16
    nt = (NP + 7) // 8
    raw = PT.host_bf16(c.bounds).reshape(B * Hkv, -1, D // 32, 2, 8, 4, 4, 2)
    for b in range(B):
        for h in range(Hkv):
            assert np.array_equal(rows[b, h], O.page_bounds(K[b, h]))
    for page in range(NP, 8 * nt):
        assert not raw[:, page // 8, :, page % 8 // 4, :, page % 4].any()
    assert np.all(raw[:, nt:] == 0x7FC0)


@pytest.mark.parametrize("N,G,room", [(1, 8, 0), (33, 1, 2), (2047, 8, 1), (2048, 8, 0), (2049, 8, 0), (4096, 8, 0),
                                      (4097, 8, 3), (8192, 8, 0), (8193, 8, 0), (16384, 2, 0), (16385, 2, 0),
                                      (16385, 1, 0), (4095, 16, 0), (4097, 16, 0), (513, 4, 0)])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("tied", [False, True])
def test_global_budget_at_the_limits_of_its_one_workgroup_form(N, G, room, shared, tied):
    """Sets of up to 65536 logits and 16384 tokens are selected by one workgroup (16, 32 or 64 keys
    per thread), larger ones in passes over the chip: masks and offsets equal the oracle's for
    both, with logits that are mostly equal and with a set per stream or per batch element."""
    B, Hkv, D = 2, 2, 128
    rng = np.random.default_rng(7 * N + G)
    H = 1 if shared else Hkv
    logits = rng.standard_normal((B, H, N, G)).astype(np.float32)
    if tied:
        logits = np.round(logits).astype(np.float32)
        logits[rng.random(logits.shape) < 0.3] = -0.0
    V = torch.zeros(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
    K = torch.zeros_like(V)
    for gk in sorted({0, 1, (G + 1) // 2, G}):
        c = stc.RoutedCache(B, Hkv, Hkv, D, N, G, 1, device=DEV, n_cap=N + room if room else 0)
        c.build(K, V, logits=torch.from_numpy(logits).to(DEV), global_k=gk, shared=shared)
        torch.cuda.synchronize()
        for b in range(B):
            for h in range(Hkv):
                m = O.route_mask_global(logits[b, 0 if shared else h], N * gk)
                assert np.array_equal(PT.host_u16(c.mask)[b, h, :N], m), (b, h, gk)
                assert np.array_equal(c.tok_off.cpu().numpy().view(np.uint32)[b, h, :N + 1],
                                      O.token_offsets(m, G))


def _uneven(rng, shape, kind):
    """Logits that a selection by bins or digits has to work for."""
    x = rng.standard_normal(shape).astype(np.float32)
    tok = rng.random(shape[:-1] + (1,))
    if kind == "equal":
        x[:] = -0.25
    elif kind == "two values":
        x = np.where(x > 0.5, np.float32(1.5), np.float32(-0.0)).astype(np.float32)
    elif kind == "halves":
        x = np.round(2 * x) / 2
    elif kind == "masked":                                 # tokens at a large negative number
        x = np.where(tok < 0.3, np.float32(-1e9), x)
    elif kind == "mostly masked":
        x = np.where(tok < 0.9, np.float32(-1e9), x)
    elif kind == "outliers":
        x = np.where(rng.random(shape) < 0.002, x * np.float32(1e4), x)
    elif kind == "nested":                                 # every round of bins leaves most in one
        e = rng.integers(0, 9, size=shape)
        x = x * np.float32(10.0) ** (4 * e - 30)
    elif kind == "lowest":
        x = np.where(tok < 0.3, np.finfo(np.float32).min, x)
    elif kind == "wide":                                   # a range beyond the largest float
        x = np.where(tok < 0.1, np.float32(3.2e38), np.where(tok > 0.9, np.float32(-3.2e38), x))
    elif kind == "infinite":
        x = np.where(tok < 0.1, np.float32(np.inf), np.where(tok > 0.8, np.float32(-np.inf), x))
    elif kind == "subnormal":
        x = (x * np.float32(1e-41)).astype(np.float32)
    return np.ascontiguousarray(x, dtype=np.float32)


@pytest.mark.parametrize("N,G", [(8192, 8), (4096, 8), (1500, 4), (4096, 16), (16384, 2), (16384, 4), (3000, 1),
                                 (20000, 8)])
@pytest.mark.parametrize("kind", ["equal", "two values", "halves", "masked", "mostly masked", "outliers", "nested",
                                  "lowest", "wide", "infinite", "subnormal"])
def test_global_budget_of_uneven_logits(N, G, kind):
    """Ties, logits far from the others, ranges that cannot be divided: masks and offsets equal the
    oracle's in the one-workgroup form (and in the passes over the chip, last size)."""
    B, Hkv, D = 2, 2, 128
    rng = np.random.default_rng(3 * N + G)
    logits = _uneven(rng, (B, Hkv, N, G), kind)
    V = torch.zeros(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
    c = stc.RoutedCache(B, Hkv, Hkv, D, N, G, 1, device=DEV)
    dl = torch.from_numpy(logits).to(DEV)
    for gk in sorted({1, (G + 1) // 2, max(1, G - 1)}):
        stc.stc_route_and_pack_values(c.shape, stc.STC_ROUTE_GLOBAL, V, dl, None, gk, None, c.mask, c.tok_off,
                                      c.vpacked, c.dev_status, c._ws_route)
        torch.cuda.synchronize()
        for b in range(B):
            for h in range(Hkv):
                m = O.route_mask_global(logits[b, h], N * gk)
                assert np.array_equal(PT.host_u16(c.mask)[b, h], m), (b, h, gk)
                assert np.array_equal(c.tok_off.cpu().numpy().view(np.uint32)[b, h], O.token_offsets(m, G))


@pytest.mark.parametrize("N", [524288, 524289, 524289 + 700])
def test_packed_copy_on_both_sides_of_the_scan_launch(N):
    """Up to 2048 chunks of 256 tokens the packed copy adds up the chunk sums itself, beyond a launch
    scans them: offsets and packed values equal the oracle's."""
    D, G = 64, 8
    rng = np.random.default_rng(N)
    V = rng.integers(0, 1 << 16, size=(1, 1, N, D)).astype(np.uint16) & 0xBFFF
    mask = rng.integers(0, 1 << G, size=(1, 1, N)).astype(np.uint16)
    c = stc.RoutedCache(1, 1, 1, D, N, G, 1, device=DEV)
    c.vpacked.view(torch.int16).fill_(0x7FC0)
    c.build(torch.zeros(1, 1, N, D, dtype=torch.bfloat16, device=DEV), PT.to_dev_bf16(V),
            mask_in=PT.to_dev_u16(mask))
    torch.cuda.synchronize()
    off = O.token_offsets(mask[0, 0], G)
    kept = ((mask[0, 0][:, None] >> np.arange(G, dtype=np.uint16)) & 1).astype(bool)
    packed = V.reshape(N, G, D // G)[kept]
    assert np.array_equal(c.tok_off.cpu().numpy().view(np.uint32)[0, 0], off)
    vp = PT.host_bf16(c.vpacked)[0, 0]
    assert np.array_equal(vp[:len(packed)], packed) and np.all(vp[len(packed):] == 0x7FC0)


@pytest.mark.parametrize("N", [1, 64, 65, 208, 256, 257])
def test_masks_given_in_the_array_they_are_written_to(N):
    """mask_in may be the mask array itself: streams of one chunk, whose packing workgroups also
    read the masks of tokens in front of theirs, and longer ones; bits past the groups are cleared."""
    B, Hkv, D, G = 3, 5, 128, 8
    rng = np.random.default_rng(N)
    V = randn_bf16(rng, (B, Hkv, N, D))
    given = rng.integers(0, 1 << 16, size=(B, Hkv, N)).astype(np.uint16)
    c = stc.RoutedCache(B, Hkv, Hkv, D, N, G, 1, device=DEV)
    c.vpacked.view(torch.int16).fill_(0x7FC0)
    c.mask.copy_(PT.to_dev_u16(given))
    c.build(torch.zeros(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV), PT.to_dev_bf16(V), mask_in=c.mask)
    torch.cuda.synchronize()
    vp = PT.host_bf16(c.vpacked)
    for b in range(B):
        for h in range(Hkv):
            m = given[b, h] & np.uint16((1 << G) - 1)
            off = O.token_offsets(m, G)
            assert np.array_equal(PT.host_u16(c.mask)[b, h], m)
            assert np.array_equal(c.tok_off.cpu().numpy().view(np.uint32)[b, h], off)
            assert np.array_equal(vp[b, h, :int(off[-1])], O.pack_values(V[b, h], m, off, G))
