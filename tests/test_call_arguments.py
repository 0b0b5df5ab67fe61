"""What the calls refuse before anything is launched: these need no device."""
import ctypes

import pytest

import paper_2604_21335_amd as stc


def a_shape():
    return stc.stc_shape_t()


class NotAShape(ctypes.Structure):
    _fields_ = [("bytes", ctypes.c_char * ctypes.sizeof(stc.stc_shape_t))]


@pytest.mark.parametrize("shape", [None, bytes(ctypes.sizeof(stc.stc_shape_t)), NotAShape(),
                                   [1, 2, 3]])
def test_the_shape_must_be_one(shape):
    with pytest.raises(TypeError):
        stc.stc_build_page_bounds(shape, None, None)


@pytest.mark.parametrize("mode", [0.0, "0", None])
def test_the_mode_must_be_a_whole_number(mode):
    with pytest.raises(TypeError):
        stc.stc_route_and_pack_values(a_shape(), mode, None, None, None, 0, None, None, None, None,
                                      None, None)


@pytest.mark.parametrize("at", range(5))
@pytest.mark.parametrize("bad", [1.0, "1", None])
def test_sizes_of_a_compaction_must_be_whole_numbers(at, bad):
    sizes = [1, 1, 16, 8, 64]
    sizes[at] = bad
    with pytest.raises(TypeError):
        stc.stc_compact_tokens(None, None, None, *sizes)


@pytest.mark.parametrize("k,error", [(None, TypeError), ("four", ValueError),
                                     (float("nan"), ValueError)])
def test_the_page_count_is_what_int_takes(k, error):
    with pytest.raises(error):
        stc.stc_select_pages(a_shape(), None, None, k, None, None, None)
