"""The order in which the attention's (query chunk, key split) items are dealt to the workgroups of a single sequence's causal pass:
worked out on the host once per forward, read from the library through the C++ symbol (no GPU)."""
import ctypes as C

import pytest


class RowDesc(C.Structure):
    """Mirrors RowDesc of csrc/tidar_internal.h; AttnPlan, Segs and WorkOrder likewise."""
    _fields_ = [(n, C.c_int) for n in ("nc", "nb", "bl", "cond0", "cstride", "nm", "R", "seq_base")]


class AttnPlan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("splits", "splits_bound", "n_chunks", "tiles_per_chunk")] + [
        ("tiled", C.c_bool), ("max_keys", C.c_int), ("per", C.c_int)]


class Segs(C.Structure):
    _fields_ = [("n", C.c_int), ("row0", C.c_int * 33)]


class WorkOrder(C.Structure):
    _fields_ = [("n", C.c_int), ("item2", C.c_uint32 * 256)]


def plan_and_order(n_kv, group, nc, nm, max_keys, B=1, segs=None):
    import paper_2511_08923_amd as T
    lib = C.CDLL(T.LIB_PATH)
    plan, order = lib._Z14plan_attentioniiiRK7RowDescRK4Segsi, lib._Z15attention_orderRK8AttnPlaniiiRK7RowDescRK4Segs
    plan.argtypes = [C.c_int, C.c_int, C.c_int, C.POINTER(RowDesc), C.POINTER(Segs), C.c_int]
    order.argtypes = [C.POINTER(AttnPlan), C.c_int, C.c_int, C.c_int, C.POINTER(RowDesc), C.POINTER(Segs)]
    plan.restype, order.restype = AttnPlan, WorkOrder
    d, sg = RowDesc(nc, 1 if nm else 0, max(nm, 1), nc, 1, nm, nc + nm, 0), Segs()
    if segs:
        sg.n = len(segs)
        for i, r in enumerate(segs):
            sg.row0[i + 1] = sg.row0[i] + r
    p = plan(B, n_kv, group, C.byref(d), C.byref(sg), max_keys)
    o = order(C.byref(p), B, n_kv, group, C.byref(d), C.byref(sg))
    ids = [o.item2[i >> 1] >> (16 * (i & 1)) & 0xffff for i in range(o.n)]
    return p, [(x >> 10, x & 1023) for x in ids]


# one XCD and four XCDs per kv head; fewer than 33 items per XCD, up to 64, more; several key splits; chunks that straddle heads
@pytest.mark.parametrize("n_kv,group,nc,nm,cached", [(8, 4, 1030, 0, 0), (8, 4, 2048, 16, 0), (8, 4, 1333, 7, 1001), (2, 6, 700, 0, 0),
                                                     (2, 6, 1501, 16, 300), (2, 6, 2047, 0, 4000), (4, 3, 3000, 8, 0)])
def test_every_item_is_dealt_once(n_kv, group, nc, nm, cached):
    p, items = plan_and_order(n_kv, group, nc, nm, cached + nc + nm)
    assert p.n_chunks * p.splits * n_kv > 256 and len(items) == p.n_chunks * p.splits
    assert sorted(items) == [(s, c) for s in range(p.splits) for c in range(p.n_chunks)]


def test_the_two_items_of_a_compute_unit_add_up_alike():
    """2048 causal rows, 64 items of one XCD, 32 compute units: by index both items of a unit see the same rows."""
    p, items = plan_and_order(8, 4, 2048, 0, 2048)
    assert p.splits == 1 and len(items) == 64
    keys = lambda chunk: (chunk % 16 + 1) * 128               # the furthest key of a chunk of 128 rows of one head
    pairs = [keys(items[i][1]) + keys(items[i + 32][1]) for i in range(32)]
    assert max(pairs) <= 2048 + 2 * 128 and max(keys(i) + keys(i + 32) for i in range(32)) == 2 * 2048


@pytest.mark.parametrize("n_kv,group,nc,nm,max_keys,B,segs", [
    (8, 4, 16, 256, 4368, 1, None),                  # a decode step
    (8, 4, 200, 0, 200, 1, None),                    # no more workgroups than compute units
    (8, 4, 2000, 0, 2000, 2, None),                  # more groups than XCDs
    (3, 4, 2000, 0, 2000, 1, None),                  # groups that do not divide them
    (8, 4, 1000, 16, 1016, 2, [1016, 700])])         # sequences of different length
def test_the_others_keep_the_plain_order(n_kv, group, nc, nm, max_keys, B, segs):
    assert plan_and_order(n_kv, group, nc, nm, max_keys, B, segs)[1] == []
