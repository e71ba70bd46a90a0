"""What a call launches on given operands (adaptcore_call_info), on the CPU:
column-major operands read in place or copied, the fallbacks of misaligned
rows, and the two forms of the grouped kernel."""
import random

import pytest

import paper_2608_10803_amd as ac

F32, BF16, F16 = ac.AC_BF16_F32OUT, ac.AC_BF16_BF16OUT, ac.AC_F16_F16OUT
A0, B0 = 0x10000, 0x20000  # aligned addresses; never read


def info(plan, M, N, K, layouts=0, a_off=0, b_off=0, a_pad=0, b_pad=0):
    """Operands `off` elements past an aligned address, their stored rows `pad`
    elements longer than the matrix."""
    lda, ldb = (M if layouts & 1 else K) + a_pad, (K if layouts & 2 else N) + b_pad
    return ac.adaptcore_call_info(plan, A0 + 2 * a_off, lda, B0 + 2 * b_off, ldb)


def candidates(M, N, K, dtype, layouts, family):
    for c in ac.adaptcore_candidates(M, N, K, dtype, layouts):
        if c["family"] == family:
            yield ac.adaptcore_plan_variant(M, N, K, dtype, layouts, c["variant_key"]), c


@pytest.mark.parametrize("layouts,bad", [(1, {"a_off": 1}), (1, {"a_pad": 3}), (2, {"b_off": 1}), (2, {"b_pad": 4})])
def test_in_place_or_copied(layouts, bad):
    seen = 0
    for M, N, K in [(136, 520, 264), (2048, 14336, 4096), (16, 14336, 4096)]:
        for plan, c in candidates(M, N, K, BF16, layouts, ac.AC_FAMILY_DL):
            whole, d = ac.adaptcore_plan_kernels(plan), ac.adaptcore_plan_info(plan)
            got = info(plan, M, N, K, layouts, **bad)
            assert got["kernels"] == whole and got["in_place"] == 0 and got["n_kernels"] == len(whole), (c, got)
            assert got["predicted_s"] == d["predicted_s"] and got["variant_key"] == c["variant_key"]
            got = info(plan, M, N, K, layouts)
            assert got["n_kernels"] == len(got["kernels"]) and got["variant_key"] == c["variant_key"]
            if got["in_place"]:
                seen += 1
                name = whole[1].replace("k_dl<", "k_dlc<").replace(">", ", %d>" % layouts)
                assert got["in_place"] == layouts and got["kernels"] == [name] + whole[2:], (got, whole)
                assert got["predicted_s"] < d["predicted_s"]
            else:  # the 64 x 512 tile, and tiles of fewer than 128 rows for A
                assert got["kernels"] == whole and (c["tile_m"] < 128 if layouts == 1 else c["tile_n"] == 512), (c, got)
    assert seen >= 20


def test_workspace_is_that_of_the_copies_made():
    up = lambda n: -(-n // 256) * 256
    for M, N, K in [(4, 4096, 14336), (136, 520, 264)]:
        for layouts in (1, 2, 3):
            for plan, c in candidates(M, N, K, F32, layouts, ac.AC_FAMILY_DL):
                part = up(c["pk"] * M * -(-N // 8) * 8 * 4) if c["pk"] > 1 else 0
                size_a, size_b = up(2 * M * K) if layouts & 1 else 0, 2 * K * -(-N // 8) * 8 if layouts & 2 else 0
                got = info(plan, M, N, K, layouts)
                want = part + (size_a if not got["in_place"] & 1 else 0) + (size_b if not got["in_place"] & 2 else 0)
                assert up(got["workspace_bytes"]) == up(want), (c, got, want)
                copied = info(plan, M, N, K, layouts, a_off=1, b_off=1)
                if copied["variant_key"] == c["variant_key"]:  # (a misaligned row-major operand takes another form)
                    assert copied["workspace_bytes"] == ac.adaptcore_plan_info(plan)["workspace_bytes"]


def test_one_operand_of_two_in_place():
    for plan, c in candidates(264, 520, 328, BF16, 3, ac.AC_FAMILY_DL):
        both = info(plan, 264, 520, 328, 3)
        only_a = info(plan, 264, 520, 328, 3, b_off=1)
        copied = info(plan, 264, 520, 328, 3, a_off=1, b_off=1)
        assert both["in_place"] == (0 if c["tile_n"] == 512 else 2)
        assert only_a["in_place"] == (1 if c["tile_m"] >= 128 else 0)
        assert copied["in_place"] == 0 and copied["kernels"].count("k_transpose16") == 2
        assert both["kernels"].count("k_transpose16") == 2 - (both["in_place"] != 0)


def test_in_place_weights_at_every_size():
    """No size of B at which a plan goes back to a kernel priced higher: the pick
    has the lowest prediction among the configurations, each with the copies
    that a call on aligned operands makes."""
    rng = random.Random(5)
    shapes = [(M, 4096, K) for M in (1, 4, 16, 64) for K in (1024, 4088, 4096, 4104)]
    while len(shapes) < 60:
        shapes.append((int(2 ** rng.uniform(0, 8)), int(2 ** rng.uniform(4, 13)), int(2 ** rng.uniform(4, 13)) // 8 * 8))
    for M, N, K in shapes:
        t = {}
        for c in ac.adaptcore_candidates(M, N, K, BF16, 2):
            plan = ac.adaptcore_plan_variant(M, N, K, BF16, 2, c["variant_key"])
            t[c["variant_key"]] = info(plan, M, N, K, 2)["predicted_s"]
        got = info(ac.adaptcore_plan(M, N, K, BF16, 2), M, N, K, 2)
        assert got["predicted_s"] == pytest.approx(min(t.values()), rel=1e-12), (M, N, K, got)


# (the last two: A misaligned, which takes the register-load form and would copy B)
@pytest.mark.parametrize("bad", [{"b_off": 1}, {"b_pad": 4}, {"a_off": 1}, {"a_pad": 3}])
def test_decode_weights_that_cannot_be_read_in_place(bad):
    """The planned configuration reads aligned weights in place; other operands
    take the best configuration of the search with every copy counted, which
    for large weights is the small-M kernel (any alignment, no copy)."""
    rng = random.Random(3)
    shapes = [(4, 4096, 14336), (16, 14336, 4096), (32, 8192, 8192), (1, 14336, 4096)]
    while len(shapes) < 60:
        M, N, K = rng.choice([1, 2, 5, 16, 33, 64]), int(2 ** rng.uniform(10, 14)), int(2 ** rng.uniform(10, 14)) // 8 * 8
        shapes.append((M, N, K))
    small_m = 0
    for M, N, K in shapes:
        plan = ac.adaptcore_plan(M, N, K, BF16, 2)
        cands = ac.adaptcore_candidates(M, N, K, BF16, 2)
        best = min(cands, key=lambda c: (c["predicted_s"], c["variant_key"]))
        got = info(plan, M, N, K, 2, **bad)
        d = ac.adaptcore_plan_info(plan)
        assert got["workspace_bytes"] <= d["workspace_bytes"]
        if d["family"] != ac.AC_FAMILY_DL or not info(plan, M, N, K, 2)["in_place"]:
            assert got["variant_key"] == d["variant_key"]
        elif best["family"] == ac.AC_FAMILY_SKINNY_M:
            small_m += 1
            assert got["variant_key"] == best["variant_key"] and got["predicted_s"] == best["predicted_s"]
            assert "k_transpose16" not in got["kernels"], (M, N, K, got)
            assert got["workspace_bytes"] <= 16 << 20  # partials
        elif "b_off" in bad or "b_pad" in bad:
            assert got["variant_key"] == best["variant_key"], (M, N, K, got, best)
    assert small_m >= 10
    # a forced configuration runs whatever the alignment
    for plan, c in candidates(4, 4096, 14336, BF16, 2, ac.AC_FAMILY_DL):
        got = info(plan, 4, 4096, 14336, 2, b_off=1)
        assert got["kernels"][0] == "k_transpose16" and got["variant_key"] == c["variant_key"]


def test_row_major_plans_and_fallbacks():
    rng = random.Random(7)
    shapes = [tuple(int(2 ** rng.uniform(0, 12)) for _ in range(3)) for _ in range(40)] + [(520, 333, 265)]
    for M, N, K in shapes:
        for dtype in (BF16, F32, F16):
            plan = ac.adaptcore_plan(M, N, K, dtype)
            got = info(plan, M, N, K)
            assert got["kernels"] == ac.adaptcore_plan_kernels(plan) and got["n_kernels"] == len(got["kernels"])
            assert got["variant_key"] == ac.adaptcore_plan_info(plan)["variant_key"] and got["in_place"] == 0
    # misaligned rows of operands that are not copied: the register-load form, or the tile kernel
    for plan, c in candidates(512, 512, 512, BF16, 0, ac.AC_FAMILY_DL):
        got = info(plan, 512, 512, 512, a_off=1)
        assert got["kernels"][0].startswith(("k_dlu<", "k_tile<")), got
        assert got["variant_key"] != c["variant_key"] and got["n_kernels"] == len(got["kernels"])
    # a misaligned B beside an A that the plan would pad: no copy at all
    for plan, c in candidates(512, 512, 515, BF16, 0, ac.AC_FAMILY_DL):
        if (c["variant_key"] >> 13) & 1:
            continue
        assert info(plan, 512, 512, 515)["kernels"][0] == "k_pad16"
        got = info(plan, 512, 512, 515, b_off=1)
        assert "k_pad16" not in got["kernels"] and got["n_kernels"] == len(got["kernels"]), got
    # nothing to launch
    got = info(ac.adaptcore_plan(0, 8, 8, BF16), 0, 8, 8)
    assert got["kernels"] == [] and got["n_kernels"] == 0
    with pytest.raises(ac.AdaptCoreError) as e:
        ac.adaptcore_call_info(None, A0, 8, B0, 8)
    assert e.value.status == ac.AC_ERR_INVALID_VALUE


@pytest.mark.parametrize("dtype", [BF16, F32, F16])
def test_grouped_forms(dtype):
    dl = (1, 2, 3, 5, 8)  # tile configurations with a direct-to-LDS kernel
    ns = "f16::" if dtype == F16 else ""
    seen = set()
    for make, fam, args in [
            (lambda k, K, N: ac.adaptcore_grouped_plan_variant(500, 7, N, K, dtype, 0, k), ac.AC_FAMILY_GROUPED, (0,)),
            (lambda k, K, N: ac.adaptcore_batched_plan_variant(6, 130, N, K, dtype, 0, k), ac.AC_FAMILY_BATCHED, (1,))]:
        for cfg in range(11):
            for N, K in [(264, 200), (264, 64), (260, 200), (264, 196)]:
                key = fam | (cfg << 4) | (1 << 12) | (1 << 16) | (dtype << 48)
                try:
                    plan = make(key, K, N)
                except ac.AdaptCoreError:
                    continue
                sa = 130 * K if args[0] else 0
                for off, lda, ldb, stride, ok in [(0, K, N, K * N, True), (1, K, N, K * N, False),
                                                  (0, K + 4, N, K * N, False), (0, K, N + 8, K * (N + 8), True),
                                                  (0, K, N, K * N + 4, False)]:
                    got = ac.adaptcore_call_info(plan, A0 + 2 * off, lda, B0, ldb, stride_a=sa, stride_b=stride)
                    direct = ok and cfg in dl and N % 8 == 0 and K % 8 == 0 and K > 64
                    assert got["kernels"][0].startswith(ns + ("k_grouped_dl<" if direct else "k_grouped<")), (cfg, got)
                    assert got["n_kernels"] == 1 and got["workspace_bytes"] == 0
                    if direct:
                        seen.add(cfg)
    assert seen == set(dl)


# (kind, groups, rows, N, K): tile configuration for aligned and for misaligned operands, with the planner's
# table of workgroups per CU
GROUP_PICKS = [("g", 64, 8192, 1536, 4096, 2, 3), ("g", 6, 1744, 440, 1344, 5, 6), ("g", 36, 4609, 1352, 832, 1, 3),
               ("g", 48, 6691, 784, 3968, 1, 5), ("b", 128, 300, 320, 192, 3, 4), ("b", 37, 183, 16, 336, 5, 6),
               ("b", 61, 221, 872, 80, 3, 1)]


def test_misaligned_grouped_products_take_the_register_staged_pick():
    """Misaligned operands run the register-staged kernel: with the tiling that
    is best for it, not the one picked at the direct-to-LDS costs."""
    try:
        ac.adaptcore_init()
        pytest.skip("a device reports its own workgroups per CU")
    except ac.AdaptCoreError:
        pass
    for kind, G, M, N, K, direct, staged in GROUP_PICKS:
        if kind == "g":
            plan, sa = ac.adaptcore_grouped_plan(M, G, N, K, BF16), 0
        else:
            plan, sa = ac.adaptcore_batched_plan(G, M, N, K, BF16), M * K
        for off, lda, stride, want, kernel in [(0, K, K * N, direct, "k_grouped_dl<"), (1, K, K * N, staged, "k_grouped<"),
                                               (0, K + 1, K * N, staged, "k_grouped<"),
                                               (0, K, K * N + 4, staged, "k_grouped<")]:
            got = ac.adaptcore_call_info(plan, A0 + 2 * off, lda, B0, N, stride_a=sa, stride_b=stride)
            assert (got["variant_key"] >> 4) & 0xFF == want and got["kernels"][0].startswith(kernel), (kind, G, M, N, K, got)
