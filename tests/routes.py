"""Which launches a call takes, asked from the library's own dispatch rules (host code, no GPU): tests
that mean to run a particular kernel form assert that their shape still reaches it."""
import ctypes

import paper_2604_21335_amd as stc

SPLIT8, SPLIT16, OWN16, OWN32 = range(4)                   # forms of the router's launch


def _rule(name, *argtypes, restype=ctypes.c_bool):
    f = getattr(stc.load_library(), name)
    f.argtypes, f.restype = argtypes, restype
    return f


def _shape(B, Hq, Hkv, D, N, G=8):
    return stc.make_shape(B, Hq, Hkv, D, N, G, N * G)


_P, _I = ctypes.POINTER(stc.stc_shape_t), ctypes.c_int


def router_form(B, N, d_model, G):
    return _rule("_ZN3stc11router_formEiiii", _I, _I, _I, _I, restype=_I)(B, N, d_model, G)


def pairs(B, Hq, Hkv, D, N, k, kv_div=1, n_tail=0):
    """Pairs of pages per wavefront of the attention over k listed pages and a tail.  A launch with page
    lists per query head has Hkv = Hq and kv_div query heads per KV head."""
    s, tp = _shape(B, Hq, Hkv, D, N), (n_tail + 15) // 16
    f = _rule("_ZN3stc16attention_splitsERK9stc_shapeiii", _P, _I, _I, _I, restype=_I)
    splits = f(s, k, tp, kv_div)
    full = (k + tp + 15) // 16
    return full if splits == 1 else 1


def step(B, Hq, Hkv, D, N, k, n_tail=0):
    """Launches of a decode step before the merge: "one", "in attention" (scores, then attention that
    selects), "with scores" (scores and selection in one, attention) or "three"."""
    s, tp = _shape(B, Hq, Hkv, D, N), (n_tail + 15) // 16
    if _rule("_ZN3stc18step_is_one_kernelERK9stc_shapeii", _P, _I, _I)(s, k, tp):
        return "one"
    if _rule("_ZN3stc20attention_can_selectERK9stc_shapeii", _P, _I, _I)(s, k, tp):
        return "in attention"
    return "with scores" if selects_with_scores(B, Hq, Hkv, D, N, k) else "three"


def selects_with_scores(B, Hq, Hkv, D, N, k):
    """stc_select_pages as one launch that scores and selects."""
    return _rule("_ZN3stc16score_can_selectERK9stc_shapei", _P, _I)(_shape(B, Hq, Hkv, D, N), k)


def select_pages(B, Hq, Hkv, D, N, k, n_tail=0):
    """Most pages per stream that the attention launch of this step could order itself."""
    f = _rule("_ZN3stc22attention_select_pagesERK9stc_shapeii", _P, _I, _I, restype=_I)
    return f(_shape(B, Hq, Hkv, D, N), k, (n_tail + 15) // 16)
