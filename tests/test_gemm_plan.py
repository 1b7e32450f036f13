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


# Sizes of the GPU tests, (M, N, K), by the kernel they are there for.
# kernels_gemm_rows: two passes of 8+8, 9+8 and 9+9 row tiles with one, two, three and five chunks of K (fewer than the four
# LDS buffers, odd counts; an odd 32-column tile, ragged column blocks and rows), passes that differ by one tile, all
# passes of five, split K, more workgroups than compute units
MANY_ROWS = [(481, 24560, 32), (513, 24560, 64), (545, 24592, 96), (576, 24560, 160), (600, 5392, 160), (640, 5136, 96),
             (650, 5136, 608), (864, 5168, 1056), (864, 1536, 1536), (1665, 8208, 288), (2305, 256, 4096)]
# kernels_gemm_mid: one to eight row tiles per pass with unequal passes, one k step per wave and fewer (K = 32: two of the
# four waves have none), a share of K that is no multiple of the ring, ragged N, the row counts beyond 480
K_SPLIT = [(33, 48, 32), (100, 784, 608), (272, 1536, 1536), (300, 1040, 96), (470, 2048, 1536), (480, 528, 288), (481, 272, 32),
           (513, 784, 96), (545, 528, 64), (576, 1040, 1056), (608, 4112, 160), (650, 304, 608), (768, 1552, 288),
           (160, 1536, 1536), (420, 5136, 288), (369, 2064, 1056)]
# kernels_gemm, two row passes of four waves side by side: 1+1, 2+1, 2+2, 3+2, 4+3, 6+5, 7+6 and 8+7 row tiles, ragged N and K;
# in the second half passes on both sides of five row tiles with long shares of K, and one split: weights together and one by one
TWO_PASS = [(33, 2064, 2080), (65, 4096, 2048), (100, 2064, 2080), (160, 4096, 1056), (200, 4096, 2048), (350, 2064, 2080),
            (416, 2064, 2080), (470, 2064, 2080),
            (100, 6160, 4128), (300, 6160, 4128), (350, 6160, 4128), (400, 6160, 4128), (480, 6160, 4128), (100, 16368, 288)]
# kernels_gemm, one split of many column blocks: 2 x 2 waves, one pass of six tiles, 256-column workgroups of eight waves
WIDE = [(97, 16400, 160), (160, 24576, 608), (170, 16400, 96), (300, 16400, 160), (420, 24576, 96), (470, 24560, 512)]


@pytest.mark.parametrize("sizes,kernel", [(MANY_ROWS, "rows"), (K_SPLIT, "mid"), (TWO_PASS, "two pass"), (WIDE, "wide")])
def test_sizes_of_the_gpu_tests_reach_the_kernel_they_are_for(sizes, kernel):
    plan, heights = planner(), set()
    for M, N, K in sizes:
        p = plan(M, N, K, False)
        reached = "rows" if p.rows else "mid" if p.mid else "two pass" if p.wide and p.nw == 4 and p.m_chunks == 2 else "wide"
        assert reached == kernel, (M, N, K, reached)
        assert kernel != "wide" or (p.splits == 1 and N >= 128 * 128), (M, N, K)
        heights.add(p.mt)
    assert heights >= {"rows": {5, 6, 7, 8, 9}, "mid": set(range(1, 9)), "two pass": {1, 2, 3, 4, 6, 7, 8}, "wide": {2, 3, 5, 6}}[kernel]


@pytest.mark.parametrize("N,K", products())
def test_grouping_of_a_sum_does_not_follow_the_row_count(N, K):
    """33-480 rows: one kernel family (one chain of products per split, with either MFMA shape, or the K-splitting waves) and one split
    count per (N, K).  From 481 rows on: one per (N, K) and number of 256-row multiples."""
    plan = planner()
    classes = [range(33, 481)] + [range(max(481, 256 * n + 1), 256 * n + 257) for n in range(1, 36)]
    for rows in classes:
        seen = {}
        for M in rows:
            p = plan(M, N, K, False)
            seen.setdefault((p.rows, p.mid, p.splits), M)
        assert len(seen) == 1, (N, K, seen)
