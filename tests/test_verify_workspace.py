"""The workspace a warped verification asks for (host arithmetic of the built library, no device needed): what the
static scratch array has to hold fits it."""
import ctypes as C

import pytest

import paper_2409_16560_amd.binding as b

MIB32 = 32 << 20


def _bytes(prompts, trees, nodes, V, top_k, depth=2, W_cap=16):
    f = b._Forest(prompts, prompts * trees, prompts * trees * nodes, None, None, None, None, None, nodes, min(depth, nodes - 1), trees)
    p = b._Params(0, 1, max(W_cap, trees), -1.0, top_k, 0.8)
    return b.load_library().dsbd_verify_forest_workspace_bytes(C.byref(f), V, C.byref(p))


@pytest.mark.parametrize("prompts,trees,nodes,V,top_k,depth", [
    (1134, 8, 64, 24, 10, 2), (837, 8, 64, 74, 20, 2), (2317, 16, 26, 6, 5, 0), (1301, 12, 39, 101, 31, 0), (751, 6, 57, 308, 25, 0),
    (1092, 13, 39, 31, 18, 1), (2056, 8, 64, 12, 2, 0), (1366, 5, 64, 66, 17, 2), (606, 8, 12, 1000, 32, 2), (607, 8, 12, 1000, 32, 2),
])
def test_batches_over_short_vocabularies_fit_the_static_array(prompts, trees, nodes, V, top_k, depth):
    assert 0 < _bytes(prompts, trees, nodes, V, top_k, depth) <= MIB32
