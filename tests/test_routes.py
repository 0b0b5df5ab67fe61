"""Dispatch rules that depend on more than one size, on the CPU."""
import pytest

from tests import routes


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("dm", [128, 512, 1024, 3584, 8192])
def test_router_form_fits_the_tokens_of_a_batch_element(G, dm):
    """A wavefront's tokens lie in one batch element.  The token slots that a launch computes are never
    more than those of workgroups of 64 tokens, whatever the number of elements."""
    tokens_of = {routes.SPLIT8: 8, routes.SPLIT16: 16, routes.OWN16: 16, routes.OWN32: 32}
    for N in [*range(1, 70), 95, 97, 129, 208, 576, 4097]:
        for B in (1, 3, 64, 500, 2048, 32768, 65535):
            if B * N > 1 << 27:
                continue
            t = tokens_of[routes.router_form(B, N, dm, G)]
            assert (N + t - 1) // t * t <= (N + 63) // 64 * 64, (B, N)


def test_router_forms_are_all_reached():
    for G in (1, 2, 4, 8, 16):
        assert {routes.router_form(B, N, 1024, G) for B, N in [(1, 100), (1, 4000), (1, 16384), (4, 32768)]} == {
            routes.SPLIT8, routes.SPLIT16, routes.OWN16, routes.OWN32}


@pytest.mark.parametrize("D,streams", [(128, 192), (128, 224), (128, 256), (64, 192), (64, 512)])
def test_several_pairs_of_pages_per_wavefront(D, streams):
    """Up to 8 where a stream's pages are its own, up to 3 where heads of a KV head share pages; one
    where the streams do not fill the chip or do not all fit on it."""
    for k in (16, 17, 48, 49, 64, 128, 129):
        full = (k + 15) // 16
        assert routes.pairs(streams, 1, 1, D, 4096, k) == (full if k <= 128 else 1)
        assert routes.pairs(streams // 4, 4, 4, D, 4096, k, kv_div=4) == (full if k <= 48 else 1)
        assert routes.pairs(191, 1, 1, D, 4096, k) == 1
        assert routes.pairs(513, 1, 1, D, 4096, k) == 1


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("NP", [2047, 2048, 2049, 4096, 8192, 8193])
def test_a_launch_that_selects_can_order_the_pages_of_its_streams(NP, D):
    """Whatever the number of streams, kept pages and tail tokens: at most 8192 pages by pages or pairs
    of pages, at most 2048 by several pairs per wavefront, and what the form itself says."""
    for streams in range(1, 601):
        for k in (7, 8, 9, 16, 17, 20, 32, 33, 48, 128, 256):
            for n_tail in (0, 1, 60, 130):
                if routes.step(streams, 1, 1, D, NP * 16, k, n_tail) != "in attention":
                    continue
                several = routes.pairs(streams, 1, 1, D, NP * 16, k, n_tail=n_tail) > 1
                assert NP <= (2048 if several else 8192), (streams, k, n_tail)
                assert NP <= routes.select_pages(streams, 1, 1, D, NP * 16, k, n_tail), (streams, k, n_tail)
