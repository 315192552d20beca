"""The workspace a warped verification asks for (host arithmetic of the built library, no device needed): it rises with the
batch, and what the static scratch array has to hold fits it."""
import ctypes as C

import pytest

import paper_2409_16560_amd.binding as b

MIB32 = 32 << 20


def _bytes(prompts, trees, nodes, V, top_k, depth=2, W_cap=16):
    f = b._Forest(prompts, prompts * trees, prompts * trees * nodes, None, None, None, None, None, nodes, min(depth, nodes - 1), trees)
    p = b._Params(0, 1, max(W_cap, trees), -1.0, top_k, 0.8)
    return b.load_library().dsbd_verify_forest_workspace_bytes(C.byref(f), V, C.byref(p))


@pytest.mark.parametrize("trees,nodes,V,top_k", [
    (8, 12, 1000, 32), (8, 64, 24, 10), (8, 64, 74, 20), (5, 10, 300, 16), (1, 64, 1, 1), (8, 40, 32000, 10), (8, 31, 128256, 10),
    (4, 8, 257, 32), (8, 64, 1025, 32), (16, 32, 4097, 5),
])
def test_a_buffer_for_the_largest_batch_serves_the_smaller_ones(trees, nodes, V, top_k):
    last = 0
    for prompts in list(range(1, 64)) + list(range(64, 8000, 13)):
        n = _bytes(prompts, trees, nodes, V, top_k)
        assert n >= last, (prompts, n, last)
        last = n
    assert last >= MIB32                                     # (the sweep goes through the change of records)


@pytest.mark.parametrize("prompts,trees,nodes,V,top_k,depth", [
    (1134, 8, 64, 24, 10, 2), (837, 8, 64, 74, 20, 2), (2317, 16, 26, 6, 5, 0), (1301, 12, 39, 101, 31, 0), (751, 6, 57, 308, 25, 0),
    (1092, 13, 39, 31, 18, 1), (2056, 8, 64, 12, 2, 0), (1366, 5, 64, 66, 17, 2), (606, 8, 12, 1000, 32, 2), (607, 8, 12, 1000, 32, 2),
])
def test_batches_over_short_vocabularies_fit_the_static_array(prompts, trees, nodes, V, top_k, depth):
    assert 0 < _bytes(prompts, trees, nodes, V, top_k, depth) <= MIB32


def test_smaller_records_are_taken_only_where_they_bring_the_size_down_to_the_static_array():
    # 50000 nodes x 32000: tokens alone would still take over 100 MB, so the records keep their logits (16 + 4 bytes a part and 16
    # a chunk of 1024, 96 a record)
    n = _bytes(125, 8, 50, 32000, 10)
    assert n >= 100000 * (32 * (16 + 4 * 4) + 96)
