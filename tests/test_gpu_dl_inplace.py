"""GPU parity of the direct-to-LDS kernels' in-place column-major operands and
grouped form.

A column-major operand with aligned rows is loaded in place: every dl
configuration of shapes at the edges of tiles, k-blocks and stages runs on
it, is checked against the fp64 oracle and, bit for bit, against the same
configuration on operands stored one element further on, which takes the
transposing copy (the same fragments in the same k order). Grouped and
batched products with aligned operands run the direct-to-LDS tile; one
element further on they run the register-staged tile of the same plan: the
same bits again. What each call launched is checked by the library's count of
launches and its description of the call.
"""
import numpy as np
import pytest

import paper_2608_10803_amd as ac
from oracle import addmm_ref, grouped_ref, layout_ref
from workloads import gen

from gpu_util import Out, all_candidates, check, fmt_of, forced_plan, run, run_addmm, to_device, tol, torch
from oracle import gemm_ref

pytestmark = pytest.mark.gpu

F32, BF16, F16F16 = ac.AC_BF16_F32OUT, ac.AC_BF16_BF16OUT, ac.AC_F16_F16OUT


@pytest.fixture(scope="module", autouse=True)
def device():
    torch()
    ac.adaptcore_init()
    yield


def stored(M, N, K, layouts, dtype, seed, pad):
    """A and B as stored, every stored row `pad` elements longer than its
    matrix (other values there)."""
    dist = "uniform_f16" if fmt_of(dtype) == "fp16" else "uniform"
    A, B = gen.operands(M, N, K, seed=seed, dist=dist)
    mk = gen.uniform_f16 if dist == "uniform_f16" else gen.uniform_bf16
    out = []
    for m, i in ((A.T if layouts & 1 else A, 3), (B.T if layouts & 2 else B, 4)):
        s = mk(m.shape[0], m.shape[1] + pad, (seed, i), -9.0, 9.0)
        s[:, :m.shape[1]] = m
        out.append(s)
    return out[0], out[0].shape[1], out[1], out[1].shape[1]


def launches(f):
    n0 = ac.adaptcore_stats()["launches"]
    r = f()
    return r, ac.adaptcore_stats()["launches"] - n0


# (M, N, K, layouts): the operand in place has whole 16-byte chunks (M, or K, a
# multiple of 8); the other dimensions are odd, K one block and less, just
# over a block, a whole and a partial group of stages
SHAPES = [(264, 77, 45, 1), (136, 261, 130, 1), (8, 130, 8, 1), (72, 130, 8, 1), (520, 513, 321, 1),
          (37, 261, 72, 2), (300, 515, 264, 2), (130, 129, 8, 2), (65, 257, 1032, 2), (5, 300, 520, 2),
          (136, 270, 200, 3)]


@pytest.mark.parametrize("dtype", [F32, BF16, F16F16], ids=["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_column_major_in_place(shape, dtype):
    M, N, K, layouts = shape
    sa, lda, sb, ldb = stored(M, N, K, layouts, dtype, seed=M + N + K, pad=0 if K == 72 else 8)
    ref = layout_ref.gemm_layout(sa, sb, M, N, K, lda, ldb, layouts, fmt=fmt_of(dtype))
    cands = [c for c in all_candidates(M, N, K, dtype, layouts) if c["family_name"] == "dl"]
    assert cands
    # tiles of 64 x 512 read neither in place, those of fewer than 128 rows only B
    can = [c for c in cands if c["tile_n"] != 512 and (layouts & 2 or c["tile_m"] >= 128)]
    assert bool(can) == (layouts >= 2 or M >= 64)  # (no tile of more than twice the rows is offered)
    for c in cands:
        plan = forced_plan(M, N, K, dtype, c["variant_key"], layouts)
        whole = len(ac.adaptcore_plan_kernels(plan))
        (vals, ok), n = launches(lambda: run(plan, sa, sb, M, N, K, dtype, lda=lda, ldb=ldb))
        assert n == whole - (c in can), (shape, c, n, whole)
        check(vals, ok, None, None, dtype, ref=ref, label="%s %s" % (shape, c))
        (v2, ok2), n = launches(lambda: run(plan, sa, sb, M, N, K, dtype, lda=lda, ldb=ldb, a_off=layouts & 1,
                                            b_off=layouts >> 1))
        assert n == whole and ok2 and np.array_equal(vals.view(np.uint64), v2.view(np.uint64)), (shape, c)
        if layouts == 3:  # A in place, B copied to where A's copy would be
            (v3, ok3), n = launches(lambda: run(plan, sa, sb, M, N, K, dtype, lda=lda, ldb=ldb, b_off=1))
            assert n == whole - (c["tile_m"] >= 128), (shape, c)
            assert ok3 and np.array_equal(vals.view(np.uint64), v3.view(np.uint64)), (shape, c)


NAN = 0x7FC0  # bf16


@pytest.mark.parametrize("shape", [(264, 77, 45, 1), (37, 261, 72, 2), (300, 515, 264, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_nothing_outside_the_operands_counts(shape):
    """NaN in the pads of the stored rows and around the matrices, and an
    infinity in one row of A: the other rows are those of the oracle."""
    M, N, K, layouts = shape
    dist = gen.operands(M, N, K, seed=1)
    A, B = dist[0].copy(), dist[1]
    inf_row = M - 1
    A[inf_row, K // 2] = 0x7F80
    mem, ops = [], []
    for m in (A.T if layouts & 1 else A, B.T if layouts & 2 else B):
        host = np.full((m.shape[0] + 600, m.shape[1] + 24), NAN, np.uint16)
        ld = host.shape[1] // 8 * 8  # aligned rows
        host = host.reshape(-1)[:host.shape[0] * ld].reshape(-1, ld)
        host[300:300 + m.shape[0], 8:8 + m.shape[1]] = m
        d = torch().from_numpy(host.view(np.int16)).to("cuda")
        mem.append(d)
        ops += [d.data_ptr() + 2 * (300 * ld + 8), ld]
    C_ref, D = gemm_ref.gemm(dist[0], B)
    rows = np.arange(M) != inf_row
    ran = 0
    for c in all_candidates(M, N, K, F32, layouts):
        if c["family_name"] != "dl":
            continue
        plan = forced_plan(M, N, K, F32, c["variant_key"], layouts)
        if not ac.adaptcore_call_info(plan, *ops)["in_place"]:
            continue
        ran += 1
        out = Out(M, N, N, F32)
        ac.adaptcore_matmul(plan, *ops, out.addr, N, 0)
        torch().cuda.synchronize()
        vals, ok = out.read()
        assert ok and gemm_ref.err_metric(vals[rows], C_ref[rows], D[rows]) <= tol(F32), (shape, c)
        assert not np.isfinite(vals[inf_row]).any(), (shape, c)
    assert ran >= 5


@pytest.mark.parametrize("layouts", [1, 2])
def test_pitch_next_to_the_limit(layouts):
    """Rows almost 2^22 elements apart: 255 of them end 8 MB below the 2^31
    bytes that a tile's offsets reach. At 2^22 the operand is copied."""
    M, N, K = (264, 70, 136) if layouts == 1 else (33, 300, 136)
    t = torch()
    A, B = gen.operands(M, N, K, seed=4)
    m = np.ascontiguousarray(A.T if layouts == 1 else B.T)
    C_ref, D = gemm_ref.gemm(A, B)
    other, _ = to_device(B if layouts == 1 else A)
    for pitch in ((1 << 22) - 8, 1 << 22):
        big = t.full((m.shape[0] * pitch,), 1, dtype=t.int16, device="cuda")
        big.view(m.shape[0], pitch)[:, :m.shape[1]].copy_(t.from_numpy(m.view(np.int16)).to("cuda"))
        ops = (big.data_ptr(), pitch, other.data_ptr(), N) if layouts == 1 else (other.data_ptr(), K, big.data_ptr(), pitch)
        ran = 0
        for c in all_candidates(M, N, K, F32, layouts):
            if c["family_name"] != "dl" or c["pk"] > 1:
                continue
            plan = forced_plan(M, N, K, F32, c["variant_key"], layouts)
            in_place = ac.adaptcore_call_info(plan, *ops)["in_place"]
            assert not (in_place and pitch == 1 << 22)
            ran += in_place != 0
            out = Out(M, N, N, F32)
            ac.adaptcore_matmul(plan, *ops, out.addr, N, 0)
            t.cuda.synchronize()
            vals, ok = out.read()
            assert ok and gemm_ref.err_metric(vals, C_ref, D) <= tol(F32), (pitch, c)
        assert (ran >= 3) == (pitch < 1 << 22)
        del big


def test_addmm_column_major_in_place():
    M, N, K = 40, 264, 328
    bias = gen.uniform_f32(1, N, 9).reshape(-1)
    old = gen.uniform_f32(M, N, 10)
    sa, lda, sb, ldb = stored(M, N, K, 2, F32, seed=3, pad=0)
    A, B = sa, np.ascontiguousarray(sb.T)
    ref = addmm_ref.addmm(A, B, old, -1.5, 0.75, bias)
    for c in all_candidates(M, N, K, F32, 2):
        if c["family_name"] != "dl":
            continue
        plan = forced_plan(M, N, K, F32, c["variant_key"], 2)
        vals, ok = run_addmm(plan, sa, sb, M, N, K, F32, old, -1.5, 0.75, bias, lda=lda, ldb=ldb)
        check(vals, ok, None, None, F32, ref=ref, label=str(c))


def grouped(plan, counts, A, B, rows, G, N, K, dtype, a_off, alpha=None, bias=None):
    t = torch()
    Ad, a = to_device(A, K, a_off)
    Bd = t.from_numpy(B.view(np.int16)).to("cuda")
    cnt = t.from_numpy(np.asarray(counts, np.int32)).to("cuda")
    out = Out(rows, N, N, dtype)
    if alpha is None:
        ac.adaptcore_grouped_matmul(plan, cnt.data_ptr(), a, K, Bd.data_ptr(), N, K * N, out.addr, N, 0)
    else:
        bd = t.from_numpy(bias).to("cuda")
        ac.adaptcore_grouped_addmm(plan, cnt.data_ptr(), a, K, Bd.data_ptr(), N, K * N, out.addr, N, alpha, 0.0,
                                   bd.data_ptr(), N, 0)
    t.cuda.synchronize()
    return out.read()


# more and fewer tiles than a round of the tile order (8 XCDs x 8 tiles), row
# tiles with remainders, empty groups, rows no group covers, more than 64 groups
GROUPS = [([100, 0, 37, 250, 1, 0, 129, 64, 50], 700, 296, 200), ([1] * 9, 9, 8, 72),
          ([300, 0, 5], 305, 1304, 136), (list(range(70)), 2500, 136, 264)]


GROUPED_DL = (1, 2, 3, 5, 8)  # tile configurations with a direct-to-LDS kernel


@pytest.mark.parametrize("dtype", [F32, BF16, F16F16], ids=["f32", "bf16", "f16"])
@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "x".join(map(str, (len(c[0]),) + c[1:])))
def test_grouped_direct_to_lds(case, dtype):
    counts, rows, N, K = case
    G = len(counts)
    mk = gen.uniform_f16 if dtype == F16F16 else gen.uniform_bf16
    A = mk(rows, K, 5)
    B = np.concatenate([mk(K, N, 6 + g).reshape(-1) for g in range(G)])
    C_ref, D, cov = grouped_ref.grouped_gemm(A, B, np.asarray(counts, np.int32), rows, N, K, K, N, K * N,
                                             fmt=fmt_of(dtype))
    ran = set()
    for cfg in range(11):
        for sw in (0, 1):
            key = ac.AC_FAMILY_GROUPED | (cfg << 4) | (sw << 12) | (1 << 16) | (dtype << 48)
            try:
                plan = ac.adaptcore_grouped_plan_variant(rows, G, N, K, dtype, 0, key)
            except ac.AdaptCoreError:
                continue
            for off, form in ((0, "k_grouped_dl<" if cfg in GROUPED_DL else "k_grouped<"), (1, "k_grouped<")):
                assert form in ac.adaptcore_call_info(plan, 4096 + 2 * off, K, 4096, N, 0, K * N)["kernels"][0], (cfg, off)
            ran.add(cfg)
            vals, ok = grouped(plan, counts, A, B, rows, G, N, K, dtype, 0)
            assert ok and gemm_ref.err_metric(vals[cov], C_ref[cov], D[cov]) <= tol(dtype), (cfg, sw)
            v2, ok2 = grouped(plan, counts, A, B, rows, G, N, K, dtype, 1)
            assert ok2 and np.array_equal(vals.view(np.uint64), v2.view(np.uint64)), (cfg, sw)
            bias = gen.uniform_f32(G, N, 8).reshape(-1)
            v3, ok3 = grouped(plan, counts, A, B, rows, G, N, K, dtype, 0, -2.0, bias)
            v4, ok4 = grouped(plan, counts, A, B, rows, G, N, K, dtype, 1, -2.0, bias)
            assert ok3 and ok4 and np.array_equal(v3.view(np.uint64), v4.view(np.uint64)), (cfg, sw)
    assert ran >= set(GROUPED_DL)


# products whose misaligned operands take another tiling than aligned ones
@pytest.mark.parametrize("off", [0, 1])
def test_default_grouped_and_batched_plans(off):
    t = torch()
    took = set()
    for counts, rows, N, K in GROUPS + [([60, 200, 40], 300, 440, 344)]:
        G = len(counts)
        A = gen.uniform_bf16(rows, K, 5)
        B = np.concatenate([gen.uniform_bf16(K, N, 6 + g).reshape(-1) for g in range(G)])
        C_ref, D, cov = grouped_ref.grouped_gemm(A, B, np.asarray(counts, np.int32), rows, N, K, K, N, K * N)
        plan = ac.adaptcore_grouped_plan(rows, G, N, K, F32)
        vals, ok = grouped(plan, counts, A, B, rows, G, N, K, F32, off)
        assert ok and gemm_ref.err_metric(vals[cov], C_ref[cov], D[cov]) <= tol(F32), (counts, N, K)
        took.add(ac.adaptcore_call_info(plan, 4096 + 2 * off, K, 4096, N, 0, K * N)["variant_key"] !=
                 ac.adaptcore_plan_info(plan)["variant_key"])
    for batch, M, N, K in [(37, 183, 16, 336), (3, 1000, 136, 72), (61, 70, 304, 80)]:
        A = gen.uniform_bf16(batch * M, K, 1)
        B = gen.uniform_bf16(batch * K, N, 2)
        Ad, a = to_device(A, K, off)
        Bd = t.from_numpy(B.view(np.int16)).to("cuda")
        out = Out(batch * M, N, N, F32)
        plan = ac.adaptcore_batched_plan(batch, M, N, K, F32)
        ac.adaptcore_batched_matmul(plan, a, K, M * K, Bd.data_ptr(), N, K * N, out.addr, N, M * N, 0)
        t.cuda.synchronize()
        vals, ok = out.read()
        C_ref, D = grouped_ref.batched_gemm(A.reshape(-1), B.reshape(-1), batch, M, N, K, K, N, M * K, K * N)
        assert ok and gemm_ref.err_metric(vals, C_ref.reshape(-1, N), D.reshape(-1, N)) <= tol(F32), (batch, M, N, K)
        took.add(ac.adaptcore_call_info(plan, a, K, Bd.data_ptr(), N, M * K, K * N)["variant_key"] !=
                 ac.adaptcore_plan_info(plan)["variant_key"])
    assert (True in took) == (off == 1), took


@pytest.mark.parametrize("shape", [(5, 70, 304, 200), (3, 300, 136, 72), (9, 1, 8, 264), (2, 129, 520, 128)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [F32, BF16, F16F16], ids=["f32", "bf16", "f16"])
def test_batched_direct_to_lds(shape, dtype):
    batch, M, N, K = shape
    t = torch()
    mk = gen.uniform_f16 if dtype == F16F16 else gen.uniform_bf16
    A = mk(batch * M, K, 1)
    B = mk(batch * K, N, 2)
    bias = gen.uniform_f32(1, N, 3).reshape(-1)
    bd = t.from_numpy(bias).to("cuda")
    refs = [gemm_ref.gemm(A[b * M:(b + 1) * M], B[b * K:(b + 1) * K], fmt=fmt_of(dtype)) for b in range(batch)]
    ran = set()
    Bd = t.from_numpy(B.view(np.int16)).to("cuda")
    for cfg in range(11):
        for sw in (0, 1):
            key = ac.AC_FAMILY_BATCHED | (cfg << 4) | (sw << 12) | (1 << 16) | (dtype << 48)
            try:
                plan = ac.adaptcore_batched_plan_variant(batch, M, N, K, dtype, 0, key)
            except ac.AdaptCoreError:
                continue
            ran.add(cfg)
            got, epi = [], []
            for off in (0, 1):
                Ad, a = to_device(A, K, off)
                form = ac.adaptcore_call_info(plan, a, K, Bd.data_ptr(), N, M * K, K * N)["kernels"][0]
                assert ("k_grouped_dl<" in form) == (off == 0 and cfg in GROUPED_DL), (cfg, off, form)
                out = Out(batch * M, N, N, dtype)
                ac.adaptcore_batched_matmul(plan, a, K, M * K, Bd.data_ptr(), N, K * N, out.addr, N, M * N, 0)
                t.cuda.synchronize()
                got.append(out.read())
                out = Out(batch * M, N, N, dtype)
                ac.adaptcore_batched_addmm(plan, a, K, M * K, Bd.data_ptr(), N, K * N, out.addr, N, M * N, -0.5, 0.0,
                                           bd.data_ptr(), 0)
                t.cuda.synchronize()
                epi.append(out.read())
            for two in (got, epi):
                assert two[0][1] and two[1][1] and np.array_equal(two[0][0].view(np.uint64), two[1][0].view(np.uint64))
            for b, (C_ref, D) in enumerate(refs):
                rows = slice(b * M, (b + 1) * M)
                assert gemm_ref.err_metric(got[0][0][rows], C_ref, D) <= tol(dtype), (cfg, sw, b)
                err = gemm_ref.err_metric(epi[0][0][rows], -0.5 * C_ref + bias, 0.5 * D + np.abs(bias))
                assert err <= tol(dtype), (cfg, sw, b, err)
    assert ran >= set(GROUPED_DL)
