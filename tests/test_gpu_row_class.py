"""A row's sums across the kernels that a row class alternates between by the row count: the kernels add the products of a row in one
order, some with two 32x32x16 MFMAs per 32 k and some with one 16x16x32, and documented results (a step's tokens do not follow what
else is in the batch) rest on these giving the same bits.  Also with operands of very different size and sums that cancel, where the
order would show most.  The LM head's products are launched through the library's C++ symbols: no entry point hands out the logits of
a chosen row count alone."""
import ctypes as C

import pytest
import torch

import tidar_inputs as TI
from test_gemm_plan import GemmPlan, planner
from test_gpu_ops import _gemm

ROWMAJOR, ARGMAX = 1, 3                      # GEMM_EPI_* of csrc/tidar_internal.h

# (N, K, rows): many short shares of K (two row passes / all row tiles in one workgroup), gate/up (all row tiles / 256-column
# workgroups of eight waves / two passes of all row tiles), one split in an odd number of 32-k steps
PRODUCTS = [(1536, 8192, (33, 160, 192, 193, 272, 320, 321, 480)), (1536, 8960, (40, 320, 321, 480)),
            (17920, 1536, (72, 288, 289, 400, 480)), (24576, 1056, (33, 288, 289, 340, 384, 385, 480)),
            (6144, 4096, (96, 97, 272, 350, 480))]
# LM head: 160-column workgroups in one pass against the two-pass and 2 x 2 kernels on both sides of each of its lines
HEADS = [(76816, 160, (33, 288, 289, 480)), (76816, 1536, (64, 96, 128, 160, 192, 224, 256, 288, 289)),
         (76816, 4096, (40, 256, 257)), (82000, 1536, (33, 160, 161, 224, 272))]


def operands(kind, M, N, K, seed):
    a = TI.make_normal((M, K), seed=seed, dtype=torch.float32).cuda()
    w = TI.make_normal((N, K), seed=seed + 1, dtype=torch.float32, std=0.02).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if kind == "spread":                     # exponents over 2^-12 .. 2^12, element by element
        a *= torch.exp2(torch.randint(-12, 13, a.shape, generator=g, device="cuda").float())
        w *= torch.exp2(torch.randint(-12, 13, w.shape, generator=g, device="cuda").float())
    if kind == "cancel":                     # every product has a negative almost like it somewhere else in the row's sum
        order = torch.randperm(K, generator=g, device="cuda")
        one, other = order[:K // 2], order[K // 2:]
        a[:, other], w[:, other] = -a[:, one], w[:, one] * (1 + 2.0 ** -7)
    return a.to(torch.bfloat16), w.to(torch.bfloat16)


def kernel_of(p):
    return p.wide, p.nw, p.m_chunks, p.swz


@pytest.mark.parametrize("N,K,rows", PRODUCTS)
def test_products_cross_kernels(N, K, rows):
    assert len({kernel_of(planner()(M, N, K, False)) for M in rows}) >= 2
    assert len({planner()(M, N, K, False).splits for M in rows}) == 1


@pytest.mark.parametrize("N,K,rows", HEADS)
def test_heads_cross_kernels(N, K, rows):
    assert {planner()(M, N, K, True).wide == 3 for M in rows} == {True, False}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["normal", "spread", "cancel"])
@pytest.mark.parametrize("N,K,rows", PRODUCTS)
def test_a_rows_sum_is_the_same_in_every_kernel(N, K, rows, kind):
    import paper_2511_08923_amd as T
    print(f"row class N={N} K={K} {kind}", flush=True)
    ctx = T.tidar_create(T.make_config(TI.SHAPE_8B.with_layers(1), T.TIDAR_BF16, max_k=16, max_batch=4))
    a, w = operands(kind, rows[-1], N, K, seed=N + K)
    most = _gemm(T, ctx, a, w)
    assert not torch.isnan(most).any()
    for M in rows[:-1]:
        assert torch.equal(_gemm(T, ctx, a[:M].contiguous(), w), most[:M]), (M, N, K)
    T.tidar_destroy(ctx)


@pytest.fixture(scope="module")
def head():
    """head(a, packed, N, K, epi) -> logits [M][N], or (largest value, its lowest column) of every row."""
    import paper_2511_08923_amd as T
    lib = C.CDLL(T.LIB_PATH)
    gemm = lib._Z16launch_gemm_bf16PKDF16bS0_PfiiiRK8GemmPlaniP12ihipStream_tPK10ChooseArgs
    gemm.argtypes = [C.c_void_p] * 3 + [C.c_int] * 3 + [C.POINTER(GemmPlan), C.c_int, C.c_void_p, C.c_void_p]
    gemm.restype = None
    pack = lib._Z15launch_pack_actiPKviiPvP12ihipStream_t
    pack.argtypes, pack.restype = [C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_void_p], None
    plan = planner()

    def run(a, packed, N, K, epi):
        M, st = a.shape[0], torch.cuda.current_stream().cuda_stream
        p = plan(M, N, K, True)
        frag = torch.zeros((M + 31) // 32 * 32, K, dtype=torch.bfloat16, device="cuda")
        pack(T.TIDAR_BF16, a.data_ptr(), M, K, frag.data_ptr(), st)
        groups = (N + 159) // 160 * 2 if p.wide == 3 else (N + 63) // 64
        out = torch.full((M, N) if epi == ROWMAJOR else (2, groups, M), float("nan"), device="cuda")
        gemm(frag.data_ptr(), packed.data_ptr(), out.data_ptr(), M, N, K, C.byref(p), epi, st, None)
        torch.cuda.synchronize()
        if epi == ROWMAJOR:
            return out
        best, col = out[0], out[1].view(torch.int32)
        top = best.max(0).values
        return top, torch.where(best == top, col, N).min(0).values
    return run


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["normal", "spread", "cancel"])
@pytest.mark.parametrize("N,K,rows", HEADS)
def test_head_logits_are_the_same_in_every_kernel(head, N, K, rows, kind):
    """Bit for bit; the largest row count against fp64; and every row's fused maximum against its logits."""
    import paper_2511_08923_amd as T
    print(f"LM head N={N} K={K} {kind}", flush=True)
    a, w = operands(kind, rows[-1], N, K, seed=N + K)
    packed = torch.zeros(T.tidar_packed_weight_bytes(T.TIDAR_BF16, N, K) // 2, dtype=torch.bfloat16, device="cuda")
    T.tidar_pack_weight(T.TIDAR_BF16, w, packed, N)
    most = head(a, packed, N, K, ROWMAJOR)
    # K products added in fp32: fewer than K + 1 roundings of at most 2^-24 of what a partial sum can reach
    size = a.abs().double() @ w.abs().double().T
    assert bool(((most.double() - a.double() @ w.double().T).abs() <= (K + 1) * 2.0 ** -24 * size).all())
    for M in rows:
        some = a[:M].contiguous()
        logits = head(some, packed, N, K, ROWMAJOR)
        assert torch.equal(logits, most[:M]), (M, N, K)
        top, col = head(some, packed, N, K, ARGMAX)
        assert torch.equal(top, logits.max(1).values), (M, N, K)
        first = torch.where(logits == top[:, None], torch.arange(N, device="cuda"), N).min(1).values
        assert torch.equal(col.long(), first), (M, N, K)
