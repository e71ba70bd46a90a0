"""adaptcore_matmul_noalloc: the plain product with the library's fixed
device scratch as workspace, checked through the C ABI against
adaptcore_matmul (same plan, same kernels: equal bit for bit) and against
the oracle, on two calls in a row, the second with a smaller input; a
split-K plan, a column-major operand (prologue copy in the scratch), a plan
without workspace, decode products whose column-major weights (read in place)
are larger than the scratch, and a plan whose workspace exceeds the scratch
(refused, nothing written)."""
import numpy as np
import pytest

import paper_2608_10803_amd as ac
from oracle import gemm_ref, layout_ref
from workloads import gen

from gpu_util import all_candidates, forced_plan, tol, torch

pytestmark = pytest.mark.gpu

F32, BF16 = ac.AC_BF16_F32OUT, ac.AC_BF16_BF16OUT


def _dev(bits):
    t = torch()
    return t.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda()


def _vals(C, dtype):
    if dtype == F32:
        return C.cpu().numpy().astype(np.float64)
    return gemm_ref.decode(C.view(torch().int16).cpu().numpy().view(np.uint16))


def _both(plan, Ad, lda, Bd, ldb, M, N, dtype, stream):
    """C from adaptcore_matmul_noalloc and from adaptcore_matmul (outputs
    pre-filled with NaN)."""
    t = torch()
    tdt = t.float32 if dtype == F32 else t.bfloat16
    C1 = t.full((M, N), float("nan"), dtype=tdt, device="cuda")
    C2 = t.full((M, N), float("nan"), dtype=tdt, device="cuda")
    ac.adaptcore_matmul_noalloc(plan, Ad.data_ptr(), lda, Bd.data_ptr(), ldb, C1.data_ptr(), N, stream)
    ac.adaptcore_matmul(plan, Ad.data_ptr(), lda, Bd.data_ptr(), ldb, C2.data_ptr(), N, stream)
    t.cuda.synchronize()
    return C1, C2


def _split_key(M, N, K, dtype, pk_min):
    """The tile configuration with the smallest split count >= pk_min."""
    keys = [c for c in all_candidates(M, N, K, dtype) if c["family_name"] == "tile" and c["pk"] >= pk_min]
    assert keys
    return min(keys, key=lambda c: (c["pk"], c["variant_key"]))["variant_key"]


def test_noalloc_matches_matmul_on_two_calls_second_smaller():
    t = torch()
    s = t.cuda.Stream()
    cap = ac.adaptcore_noalloc_scratch_bytes()
    assert cap == 64 << 20
    cases = [(512, 512, 16384, F32, 16), (96, 80, 5000, BF16, 4)]  # the second input is smaller
    for (M, N, K, dtype, pk_min) in cases:
        plan = forced_plan(M, N, K, dtype, _split_key(M, N, K, dtype, pk_min))
        d = ac.adaptcore_plan_info(plan)
        assert d["pk"] >= pk_min and 0 < d["workspace_bytes"] <= cap
        A, B = gen.operands(M, N, K, seed=M + N + K)
        Ad, Bd = _dev(A), _dev(B)
        C1, C2 = _both(plan, Ad, K, Bd, N, M, N, dtype, s.cuda_stream)
        v1, v2 = _vals(C1, dtype), _vals(C2, dtype)
        assert np.array_equal(v1.view(np.uint64), v2.view(np.uint64)), (M, N, K)
        R, D = gemm_ref.gemm(A, B)
        assert gemm_ref.err_metric(v1, R, D) <= tol(dtype), (M, N, K)


def test_noalloc_default_plans_and_column_major():
    t = torch()
    # the planner's own plans: a split-K shape, one without workspace, and a
    # column-major B (its row-major copy lives in the scratch); then a
    # smaller one of each again
    for (M, N, K, lay) in [(64, 64, 30000, 0), (700, 500, 300, 0), (300, 260, 900, ac.AC_LAYOUT_B_COL),
                           (33, 17, 4000, 0), (40, 30, 50, ac.AC_LAYOUT_B_COL)]:
        plan = ac.adaptcore_plan(M, N, K, F32, lay)
        A, B = gen.operands(M, N, K, seed=3 * M + K)
        if lay:
            Bs = np.ascontiguousarray(B.T)  # B stored column-major: N x K
            Ad, Bd = _dev(A), _dev(Bs)
            ldb = K
            R, D = layout_ref.gemm_layout(A.reshape(-1), Bs.reshape(-1), M, N, K, K, K, lay)
        else:
            Ad, Bd = _dev(A), _dev(B)
            ldb = N
            R, D = gemm_ref.gemm(A, B)
        C1, C2 = _both(plan, Ad, K, Bd, ldb, M, N, F32, 0)
        v1, v2 = _vals(C1, F32), _vals(C2, F32)
        assert np.array_equal(v1.view(np.uint64), v2.view(np.uint64)), (M, N, K, lay)
        assert gemm_ref.err_metric(v1, R, D) <= tol(F32), (M, N, K, lay)


def _decode_weights(M, N, K, b_off):
    """A, B stored N x K `b_off` elements past an aligned address, and the
    product and its absolute-value product in 64 bits on the device."""
    t = torch()
    g = t.Generator(device="cuda").manual_seed(M + N + K)
    A = t.empty(M, K, dtype=t.float32, device="cuda").uniform_(-1, 1, generator=g).bfloat16()
    B = t.empty(N * K + b_off, dtype=t.float32, device="cuda").uniform_(-1, 1, generator=g).bfloat16()[b_off:]
    Ad, Bd = A.double(), B.view(N, K).double().t().contiguous()
    return A, B, (Ad @ Bd, Ad.abs() @ Bd.abs())


def _close(C, ref):
    R, D = (x.cpu().numpy() for x in ref)
    assert gemm_ref.err_metric(_vals(C, F32), R, D) <= tol(F32)


# weights of 117 MB: read in place
@pytest.mark.parametrize("shape", [(4, 4096, 14336), (16, 14336, 4096), (64, 8192, 8192)],
                         ids=lambda s: "x".join(map(str, s)))
def test_noalloc_decode_weights_larger_than_the_scratch(shape):
    M, N, K = shape
    A, B, ref = _decode_weights(M, N, K, 0)
    plan = ac.adaptcore_plan(M, N, K, F32, ac.AC_LAYOUT_B_COL)
    C1, C2 = _both(plan, A, K, B, K, M, N, F32, 0)
    assert bool((C1 == C2).all())
    _close(C1, ref)


# weights that cannot be read in place, one element past an aligned address or
# of an odd pitch: the small-M kernel, no copy of them
@pytest.mark.parametrize("shape,b_off", [((4, 4096, 14336), 1), ((16, 14336, 4096), 1), ((4, 4096, 14331), 0)],
                         ids=["4x4096x14336+1", "16x14336x4096+1", "4x4096x14331"])
def test_noalloc_misaligned_decode_weights(shape, b_off):
    M, N, K = shape
    A, B, ref = _decode_weights(M, N, K, b_off)
    plan = ac.adaptcore_plan(M, N, K, F32, ac.AC_LAYOUT_B_COL)
    call = ac.adaptcore_call_info(plan, A.data_ptr(), K, B.data_ptr(), K)
    n0 = ac.adaptcore_stats()["launches"]
    C1, C2 = _both(plan, A, K, B, K, M, N, F32, 0)
    assert call["n_kernels"] <= 2 and ac.adaptcore_stats()["launches"] - n0 == 2 * call["n_kernels"], call
    assert bool((C1 == C2).all())
    _close(C1, ref)


def test_capture_of_decode_weights_needs_the_partials_only():
    t = torch()
    M, N, K = 4, 4096, 14336
    A, B, ref = _decode_weights(M, N, K, 0)
    plan = ac.adaptcore_plan(M, N, K, F32, ac.AC_LAYOUT_B_COL)
    s = t.cuda.Stream()
    ac.adaptcore_reserve_workspace(s.cuda_stream, 4 << 20)
    C = t.empty(M, N, dtype=t.float32, device="cuda")
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g, stream=s):
        ac.adaptcore_matmul(plan, A.data_ptr(), K, B.data_ptr(), K, C.data_ptr(), N, s.cuda_stream)
    for _ in range(3):
        C.fill_(float("nan"))
        t.cuda.synchronize()
        g.replay()
        t.cuda.synchronize()
        _close(C, ref)


def test_noalloc_runs_a_configuration_that_fits():
    """Plans whose workspace (padded copies, partials) exceeds the scratch:
    the best configuration of the search that fits it runs instead."""
    t = torch()
    cap = ac.adaptcore_noalloc_scratch_bytes()
    over = 0
    for (M, N, K, dtype) in [(26095, 476, 2819, BF16), (5461, 392, 17806, F32), (20011, 600, 2001, BF16),
                             (9001, 1500, 6003, F32)]:
        g = t.Generator(device="cuda").manual_seed(M)
        A = t.empty(M, K, device="cuda").uniform_(-1, 1, generator=g).bfloat16()
        B = t.empty(K, N, device="cuda").uniform_(-1, 1, generator=g).bfloat16()
        plan = ac.adaptcore_plan(M, N, K, dtype)
        over += ac.adaptcore_call_info(plan, A.data_ptr(), K, B.data_ptr(), N)["workspace_bytes"] > cap
        C = t.full((M, N), float("nan"), dtype=t.float32 if dtype == F32 else t.bfloat16, device="cuda")
        ac.adaptcore_matmul_noalloc(plan, A.data_ptr(), K, B.data_ptr(), N, C.data_ptr(), N, 0)
        t.cuda.synchronize()
        rows = t.arange(0, M, 97, device="cuda")
        Ad, Bd = A[rows].double(), B.double()
        err = gemm_ref.err_metric(_vals(C[rows].contiguous(), dtype), (Ad @ Bd).cpu().numpy(),
                                  (Ad.abs() @ Bd.abs()).cpu().numpy())
        assert err <= tol(dtype), (M, N, K, err)
    assert over >= 2, over


def test_noalloc_refuses_a_workspace_beyond_the_scratch():
    t = torch()
    M, N, K = 2048, 2048, 65536
    key = _split_key(M, N, K, F32, 8)
    plan = forced_plan(M, N, K, F32, key)
    assert ac.adaptcore_plan_info(plan)["workspace_bytes"] > ac.adaptcore_noalloc_scratch_bytes()
    A = t.zeros(M * K, dtype=t.bfloat16, device="cuda")
    B = t.zeros(K * N, dtype=t.bfloat16, device="cuda")
    C = t.full((M, N), 3.0, dtype=t.float32, device="cuda")
    with pytest.raises(ac.AdaptCoreError) as e:
        ac.adaptcore_matmul_noalloc(plan, A.data_ptr(), K, B.data_ptr(), N, C.data_ptr(), N, 0)
    assert e.value.status == ac.AC_ERR_UNSUPPORTED
    t.cuda.synchronize()
    assert bool((C == 3.0).all())
