"""Which kernel and which grouping of a row's sum the bf16 GEMM plan picks: pure host arithmetic, read from the library
through the C++ symbol of the planner (no GPU)."""
import ctypes as C

import pytest

import tidar_inputs as TI


class GemmPlan(C.Structure):
    """Mirrors GemmPlan of csrc/tidar_internal.h."""
    _fields_ = [(n, C.c_int) for n in ("mt", "nt", "splits", "bk", "m_chunks", "wide", "nw", "rows", "mid", "swz")]


def planner():
    import paper_2511_08923_amd as T
    f = C.CDLL(T.LIB_PATH)._Z14plan_gemm_bf16iiib           # plan_gemm_bf16(int M, int N, int K, bool force_single_split)
    f.argtypes, f.restype = [C.c_int, C.c_int, C.c_int, C.c_bool], GemmPlan
    return f


def products():
    """(N, K) of every projection of this repository's model shapes, and generic ones between and beyond them."""
    out = set()
    for sh in TI.SHAPES.values():
        if sh.d_model % 32 == 0 and sh.d_ff % 32 == 0:
            out |= {(sh.q_dim + 2 * sh.kv_dim, sh.d_model), (sh.d_model, sh.q_dim), (2 * sh.d_ff, sh.d_model),
                    (sh.d_model, sh.d_ff)}
    out |= {(N, K) for N in (48, 784, 1536, 2560, 5120, 9216, 16400, 32768) for K in (96, 608, 1536, 4096, 11008)}
    return sorted(out)


@pytest.mark.parametrize("N,K", products())
def test_grouping_of_a_sum_does_not_follow_the_row_count(N, K):
    """33-480 rows: one kernel family (one chain of 32x32x16 MFMAs per split, or the K-splitting waves) and one split count
    per (N, K).  From 481 rows on: one per (N, K) and number of 256-row multiples."""
    plan = planner()
    classes = [range(33, 481)] + [range(max(481, 256 * n + 1), 256 * n + 257) for n in range(1, 36)]
    for rows in classes:
        seen = {}
        for M in rows:
            p = plan(M, N, K, False)
            seen.setdefault((p.rows, p.mid, p.splits), M)
        assert len(seen) == 1, (N, K, seen)
