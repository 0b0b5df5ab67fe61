"""Moving tail tokens into the cache, at the edges of the tiles of tokens and of pages: the result is,
bit for bit, the cache that construction over all tokens gives, and the rows that stay move to
the front of the tail."""
import pytest
import torch

import paper_2604_21335_amd as stc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(t):
    return t.contiguous().view(torch.int16)


@pytest.mark.parametrize("D,G", [(64, 8), (64, 1), (128, 16), (128, 2), (128, 8)])
@pytest.mark.parametrize("N,n,stay", [
    (1, 1, 0), (16, 16, 3), (15, 1, 40), (33, 14, 0), (97, 63, 1), (128, 64, 0), (31, 65, 7),
    (130, 127, 16), (112, 128, 5), (113, 128, 0), (95, 129, 33), (7, 256, 1), (201, 257, 150), (121, 263, 0)])
@pytest.mark.parametrize("given_masks", [False, True])
def test_flush_at_tile_edges(D, G, N, n, stay, given_masks):
    flush_case(2, 3, D, G, N, n, stay, given_masks)


@pytest.mark.parametrize("B,Hkv,D,G,N,n,stay", [
    (43, 6, 64, 8, 33, 1, 0), (43, 6, 128, 8, 97, 31, 1), (65, 4, 128, 16, 1, 32, 3), (37, 7, 64, 1, 15, 33, 0),
    (43, 6, 128, 2, 95, 49, 20), (65, 4, 64, 4, 130, 64, 33), (65, 4, 128, 8, 31, 63, 0), (96, 8, 64, 8, 121, 97, 5),
    (96, 8, 64, 8, 113, 128, 40)])
@pytest.mark.parametrize("given_masks", [False, True])
def test_flush_of_few_tokens_of_many_streams(B, Hkv, D, G, N, n, stay, given_masks):
    """More than 256 streams: workgroups that take 32 tokens at a time."""
    flush_case(B, Hkv, D, G, N, n, stay, given_masks)


def flush_case(B, Hkv, D, G, N, n, stay, given_masks):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000 * N + n)
    rand = lambda *s: torch.randn(*s, generator=g, device=DEV)
    T = N + n + stay
    K, V = rand(B, Hkv, T, D).bfloat16(), rand(B, Hkv, T, D).bfloat16()
    logits, counts = rand(B, Hkv, T, G), torch.randint(0, G + 1, (B, Hkv, T), generator=g, device=DEV).to(torch.uint8)
    masks = torch.randint(0, 1 << G, (B, Hkv, T), generator=g, device=DEV).to(torch.int16)
    # the last tokens find the store full when counts are drawn high: one case of a short store
    cap = (N + n) * G if N != 97 else (N + n) * G // 3

    def route(a, b):
        if given_masks:
            return dict(mask_in=masks[:, :, a:b].contiguous())
        return dict(logits=logits[:, :, a:b].contiguous(), kcount=counts[:, :, a:b].contiguous())

    c = stc.RoutedCache(B, Hkv, Hkv, D, N, G, 1, v_cap_groups=cap, device=DEV, tail_cap=n + stay + 2, n_cap=N + n + 5)
    ref = stc.RoutedCache(B, Hkv, Hkv, D, N + n, G, 1, v_cap_groups=cap, device=DEV, n_cap=N + n + 5)
    for x in (c, ref):
        for t in (x.K, x.vpacked, x.bounds):
            t.zero_()
    c.build(K[:, :, :N], V[:, :, :N].contiguous(), **route(0, N))
    c.K_tail[:, :, :n + stay].copy_(K[:, :, N:])
    c.V_tail[:, :, :n + stay].copy_(V[:, :, N:])
    c.n_tail = n + stay
    c.flush(n, **route(N, N + n))
    ref.build(K[:, :, :N + n], V[:, :, :N + n].contiguous(), **route(0, N + n))
    assert torch.equal(c.mask[:, :, :N + n], ref.mask[:, :, :N + n])
    assert torch.equal(c.tok_off[:, :, :N + n + 1], ref.tok_off[:, :, :N + n + 1])
    assert torch.equal(bits(c.K[:, :, :N + n]), bits(K[:, :, :N + n]))
    assert torch.equal(bits(c.vpacked), bits(ref.vpacked))
    tiles = (N + n + 127) // 128          # tiles in use; the store has room for as many or one more
    per = c.bounds.numel() // (B * Hkv)
    used = lambda x: bits(x.bounds.view(B * Hkv, per)[:, :tiles * 8 * D * 2])
    assert torch.equal(used(c), used(ref))
    assert torch.equal(bits(c.K_tail[:, :, :stay]), bits(K[:, :, N + n:]))
    assert torch.equal(bits(c.V_tail[:, :, :stay]), bits(V[:, :, N + n:]))
    assert int(c.dev_status) == int(ref.dev_status) and c.n_tail == stay
