"""Host-side chooser and traffic model (no GPU): capacity constraints, bytes never below the
compulsory minimum, the paper's counting identities, plans that can actually run, and the
rules of the boundary that are decided before any device work."""
import ctypes
import itertools
import math

import pytest

from paper_2512_12949_amd import binding as ff

SHAPES = [  # (M, K, N1, N2, dtype, gated)
    (128, 256, 1024, 256, ff.DT_BF16, False), (4096, 4096, 16384, 4096, ff.DT_BF16, False),
    (2048, 4096, 11008, 4096, ff.DT_BF16, True), (16, 8192, 28672, 8192, ff.DT_BF16, True),
    (64, 8192, 28672, 8192, ff.DT_BF16, True), (32768, 1024, 8192, 1024, ff.DT_F16, False),
    (128, 4096, 16384, 4096, ff.DT_BF16, False), (1, 64, 64, 64, ff.DT_BF16, False), (300, 200, 328, 136, ff.DT_F16, True),
    (8192, 512, 4096, 512, ff.DT_BF16, False), (20000, 1000, 520, 1016, ff.DT_F16, False), (50000, 264, 136, 136, ff.DT_BF16, False),
]


def test_every_ranked_plan_respects_the_capacities_and_the_compulsory_bytes():
    """Sec. 4.3, Eq. 3 (capacity of every level) for every plan the chooser ranks: LDS per workgroup
    within 160 KB, accumulators within 256 registers per lane; and no level's modelled volume
    below what the method itself must move (X, the weights and Y once)."""
    seen_families = set()
    for M, K, N1, N2, dt, gated in SHAPES:
        ranked = ff.ffuse_rank_plans(dt, 2, gated, M, K, N1, N2, 512)
        assert ranked, (M, K, N1, N2)
        times = [t for _, t in ranked]
        assert times == sorted(times)
        e, g = 2, (2 if gated else 1)
        q_min = e * (M * K + g * K * N1 + N1 * N2 + M * N2)
        for plan, t_pred in ranked:
            tr = ff.ffuse_traffic_model(plan, dt, gated, M, K, N1, N2)
            assert tr.feasible == 1
            assert tr.lds_used <= 160 * 1024, plan.as_dict()
            assert tr.acc_regs <= 256, plan.as_dict()
            assert tr.q_min == q_min and tr.q_unfused == q_min + 2 * e * M * N1
            assert tr.hbm_bytes >= q_min, plan.as_dict()
            assert tr.fabric_bytes >= 0.999 * q_min or plan.family == ff.FAMILY_REDUCE, plan.as_dict()
            assert tr.t_pred > 0 and abs(tr.t_pred - t_pred) < 1e-12
            seen_families.add(plan.family)
    assert {ff.FAMILY_REDUCE, ff.FAMILY_TWOPHASE, ff.FAMILY_EXCHANGE, ff.FAMILY_ROWS} <= seen_families


def test_the_intermediate_is_charged_to_hbm_when_it_cannot_stay_in_the_memory_side_cache():
    """The two-phase family writes the intermediate through and reads it back: 512 MiB of it cannot
    come back from a 256 MB cache (the unfused path is charged by the same rule); 128 MiB can."""
    large = ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=256, bn2=256, bk=32, splits=1, raster=4)
    t = ff.ffuse_traffic_model(large, ff.DT_F16, False, 32768, 1024, 8192, 1024)
    assert t.hbm_bytes == t.q_unfused
    t = ff.ffuse_traffic_model(large, ff.DT_BF16, False, 4096, 4096, 16384, 4096)
    assert t.hbm_bytes == t.q_min
    rows = ff.make_plan(ff.FAMILY_ROWS, bm=64, bh=64)
    t = ff.ffuse_traffic_model(rows, ff.DT_F16, False, 32768, 1024, 8192, 1024)
    assert t.hbm_bytes == t.q_min and t.exchange_bytes == 0 and t.reduce_bytes == 0
    assert t.fabric_bytes < t.q_unfused                      # the family exists to move fewer bytes than the unfused path
    assert t.acc_regs == 256 and t.lds_used <= 160 * 1024


def test_model_is_monotone_in_the_rows():
    for fam_plan in (ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=256, bn2=256, bk=32, splits=1, raster=4),
                     ff.make_plan(ff.FAMILY_ROWS, bm=64, bh=64)):
        last = 0.0
        for M in (4096, 8192, 16384, 32768, 65536):
            t = ff.ffuse_traffic_model(fam_plan, ff.DT_BF16, False, M, 1024, 8192, 1024)
            assert t.t_pred >= last and t.flops == 2 * M * 8192 * (1024 + 1024)
            last = t.t_pred


def test_counting_identities_of_the_search_space():
    """Table of spatial / temporal partitions (Sec. 4.3): C(4, s) (4 - s)! schedules with s spatial
    dimensions, 24 + 12 + 4 + 1 = 41 in all; checked against a brute-force enumeration."""
    dims = "mnkl"
    brute = {s: 0 for s in range(1, 5)}
    for s in range(1, 5):
        for spatial in itertools.combinations(dims, s):
            rest = [d for d in dims if d not in spatial]
            brute[s] += len(set(itertools.permutations(rest)))
    assert [brute[s] for s in range(1, 5)] == [24, 12, 4, 1]
    assert [ff.ffuse_loop_schedule_count(s) for s in range(1, 5)] == [24, 12, 4, 1]
    assert ff.ffuse_loop_schedule_count(0) == 41 == sum(brute.values())
    assert ff.ffuse_loop_schedule_count(5) == 0
    # the size of the unpruned space the paper quotes for M = 256, N = 16384, K = L = 4096
    space = 41 * 5 ** 4 * (256 // 16) * (16384 // 16) * (4096 // 16) * (4096 // 16)
    assert abs(space / 2.75e13 - 1) < 0.01


def test_shuffle_and_reduce_group_sizes():
    """Sec. 4.1, the two worked examples: cluster (2, 4, 2, 4) has shuffle groups of 2 blocks and 2
    groups to reduce; cluster (2, 4, 2, 8) has shuffle groups of 4 and nothing to reduce."""
    assert ff.ffuse_cluster_exchange(4, 2, 4) == (2, 2)
    assert ff.ffuse_cluster_exchange(4, 2, 8) == (4, 1)
    assert ff.ffuse_cluster_exchange(1, 1, 1) == (1, 1)
    with pytest.raises(ff.FfuseError):
        ff.ffuse_cluster_exchange(4, 2, 3)
    with pytest.raises(ff.FfuseError):
        ff.ffuse_cluster_exchange(3, 2, 4)


def test_rows_family_geometry():
    ok = ff.make_plan(ff.FAMILY_ROWS, bm=64, bh=64)
    L = ff.lib()
    t = ff.Traffic()
    call = lambda M, K, N1, N2, gated, plan=ok: L.ffuse_traffic_model(ctypes.byref(plan), ff.DT_BF16, int(gated), M, K, N1, N2, ctypes.byref(t))
    assert call(32768, 1024, 8192, 1024, False) == 0
    assert call(100, 8, 8, 8, False) == 0
    assert call(32768, 1032, 8192, 1024, False) == -8        # X no longer fits the registers
    assert call(32768, 1024, 8192, 1032, False) == -8        # the output block no longer fits the accumulators
    assert call(32768, 1024, 8192, 1024, True) == -8         # two accumulator sets of the first product do not fit
    assert call(32768, 1024, 8192, 1024, False, ff.make_plan(ff.FAMILY_ROWS, bm=128, bh=64)) == -8
    assert ff.ffuse_workspace_bytes(ff.DT_BF16, False, 32768, 1024, 8192, 1024, False) > 0   # (sized for every family)


def test_bytes_objective_prefers_the_rows_family_where_it_is_close_enough():
    ff.ffuse_plan_table_clear()
    try:
        shape = (32768, 1024, 8192, 1024)
        ff.ffuse_set_objective(ff.OBJECTIVE_BYTES)
        p, _ = ff.ffuse_plan_lookup(ff.DT_F16, 1, False, *shape)
        assert p.family == ff.FAMILY_ROWS
        tb = ff.ffuse_traffic_model(p, ff.DT_F16, False, *shape)
        ff.ffuse_set_objective(ff.OBJECTIVE_TIME)
        # the fastest plan by the model is a 256-row two-phase plan; the rows family is predicted within a few per
        # cent of it with less than half its fabric bytes, and such a near-tie goes to it under the time objective too
        fastest, t_fastest = ff.ffuse_rank_plans(ff.DT_F16, 1, False, *shape)[0]
        tq = ff.ffuse_traffic_model(fastest, ff.DT_F16, False, *shape)
        assert fastest.family == ff.FAMILY_TWOPHASE and fastest.bm == 256
        assert tq.t_pred <= tb.t_pred <= 1.06 * tq.t_pred and tb.fabric_bytes < 0.5 * tq.fabric_bytes
        q, _ = ff.ffuse_plan_lookup(ff.DT_F16, 1, False, *shape)
        assert q.family == ff.FAMILY_ROWS
        # where the family is clearly slower (short K and few output columns: smaller chunks, the same fixed part per
        # row block) the time objective keeps the fastest plan
        for other in ((32768, 512, 4096, 512), (65536, 256, 2048, 256), (128, 1024, 4096, 1024)):
            r, _ = ff.ffuse_plan_lookup(ff.DT_F16, 1, False, *other)
            assert r.family != ff.FAMILY_ROWS
        # a shape the family cannot run keeps the time plan under either objective
        ff.ffuse_set_objective(ff.OBJECTIVE_BYTES)
        g, _ = ff.ffuse_plan_lookup(ff.DT_BF16, 2, False, 4096, 4096, 16384, 4096)
        assert g.family == ff.FAMILY_TWOPHASE
        with pytest.raises(ff.FfuseError):
            ff.ffuse_set_objective(7)
    finally:
        ff.ffuse_set_objective(ff.OBJECTIVE_TIME)
        ff.ffuse_plan_table_clear()


HUGE = [(262144, 64, 8192, 64), (65536, 1024, 16384, 1024), (131072, 512, 16384, 512), (131072, 1024, 16384, 1024)]


def test_an_intermediate_of_2_gib_or_more_is_a_shape_error():
    """The kernels that keep the intermediate in the workspace address it with 32-bit offsets: a
    problem whose M x N1 intermediate reaches 2 GiB is refused by every entry point before any
    device work (dummy pointers are never dereferenced)."""
    L = ff.lib()
    a = ctypes.c_void_p(0x1000)
    for M, K, N1, N2 in HUGE:
        assert (M + 256) * N1 * 2 >= 1 << 31
        for name in ("ffuse_ffn", "ffuse_ffn_f16", "ffuse_ffn_unfused", "ffuse_ffn_unfused_f16"):
            assert getattr(L, name)(a, a, None, a, 1, M, K, N1, N2, a, None) == -2, (name, M, K, N1, N2)
        assert L.ffuse_ffn_ws(ff.DT_BF16, a, a, None, a, 1, M, K, N1, N2, a, a, 1 << 20, None) == -2
        assert L.ffuse_tune(ff.DT_BF16, a, a, None, a, 1, M, K, N1, N2, a, 4, 2, None, None, None) == -2
    # just below the limit the call gets past validation (and then fails for want of a device or a workspace)
    assert L.ffuse_ffn(a, a, None, a, 1, 32768, 1024, 8192, 1024, a, None) != -2


def test_the_chooser_never_returns_a_plan_that_cannot_run():
    """Whatever the shape -- including intermediates of 2 GiB and more, which the boundary refuses
    anyway -- the chosen plan is valid for the problem, and a two-phase plan is never chosen when its
    intermediate does not fit the 32-bit offsets of the kernel."""
    shapes = [(s[0], s[1], s[2], s[3]) for s in SHAPES] + HUGE + [(1 << 20, 8, 1024, 8), (500000, 64, 2048, 64)]
    for M, K, N1, N2 in shapes:
        for gated in (False, True):
            for objective in (ff.OBJECTIVE_TIME, ff.OBJECTIVE_BYTES):
                ff.ffuse_set_objective(objective)
                try:
                    p, _ = ff.ffuse_plan_lookup(ff.DT_BF16, 3, gated, M, K, N1, N2)
                finally:
                    ff.ffuse_set_objective(ff.OBJECTIVE_TIME)
                t = ff.Traffic()
                rc = ff.lib().ffuse_traffic_model(ctypes.byref(p), ff.DT_BF16, int(gated), M, K, N1, N2, ctypes.byref(t))
                assert rc == 0 and t.feasible == 1, (M, K, N1, N2, gated, p.as_dict())
                if p.family == ff.FAMILY_TWOPHASE:
                    assert (M + 256) * N1 * 2 < 1 << 31, (M, K, N1, N2, p.as_dict())
    ff.ffuse_plan_table_clear()
    # a forced two-phase plan for such a shape is not a valid plan
    big = ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=256, bn2=256, bk=32, splits=1, raster=4)
    t = ff.Traffic()
    assert ff.lib().ffuse_traffic_model(ctypes.byref(big), ff.DT_BF16, 0, 131072, 1024, 16384, 1024, ctypes.byref(t)) == -8


def test_per_call_workspace_arguments_are_validated_first():
    L = ff.lib()
    a, odd = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1008)
    for name in ("ffuse_ffn_ws", "ffuse_ffn_unfused_ws"):
        f = getattr(L, name)
        assert f(7, a, a, None, a, 1, 8, 8, 8, 8, a, a, 256, None) == -4          # unknown operand type
        assert f(ff.DT_BF16, None, a, None, a, 1, 8, 8, 8, 8, a, a, 256, None) == -1
        assert f(ff.DT_BF16, a, a, None, a, 1, 8, 12, 8, 8, a, a, 256, None) == -2
        assert f(ff.DT_BF16, a, a, None, a, 1, 8, 8, 8, 8, a, odd, 256, None) == -3   # workspace alignment
        assert f(ff.DT_BF16, a, a, None, a, 1, 8, 8, 8, 8, a, a, 250, None) == -2     # workspace size not a multiple of 16
        assert f(ff.DT_BF16, a, a, None, a, 1, 8, 8, 8, 8, a, None, 256, None) == -1  # a size without a buffer
    assert L.ffuse_debug_barrier(-1, 10) == -2 and L.ffuse_debug_barrier(0, 0) == -2
    assert L.ffuse_debug_barrier(0, 1 << 24) == 0


def test_split_gate_plans_are_valid_only_where_the_kernel_can_run_them():
    """Gated chain with its branches on different workgroups (Sec. 4.1): two-phase family only, gated only,
    hidden size a multiple of 64 (tiles of the two intermediates must not share cache lines); the
    workspace holds both intermediates; the model never prefers it to its one-workgroup twin."""
    import ctypes
    split = ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=256, bn2=256, bk=32, gate_split=1)
    twin = ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=128, bn2=256, bk=32)
    shape = (2048, 4096, 11008, 4096)
    t1 = ff.ffuse_traffic_model(split, ff.DT_BF16, True, *shape)
    t0 = ff.ffuse_traffic_model(twin, ff.DT_BF16, True, *shape)
    assert t1.feasible and t1.t_pred > t0.t_pred and t1.fabric_bytes == t0.fabric_bytes + 3 * 2 * 2048 * 11008
    t = ff.Traffic()
    L = ff.lib()
    assert L.ffuse_traffic_model(ctypes.byref(split), ff.DT_BF16, 0, *shape, ctypes.byref(t)) == -8          # not gated
    assert L.ffuse_traffic_model(ctypes.byref(split), ff.DT_BF16, 1, 2048, 4096, 11016, 4096, ctypes.byref(t)) == -8   # N1 % 64
    for fam in (ff.FAMILY_REDUCE, ff.FAMILY_EXCHANGE, ff.FAMILY_ROWS):
        other = ff.make_plan(fam, bm=128, bh=128, gate_split=1)
        assert L.ffuse_traffic_model(ctypes.byref(other), ff.DT_BF16, 1, *shape, ctypes.byref(t)) == -8
    bad = ff.make_plan(ff.FAMILY_TWOPHASE, bm=256, bh=256, bn2=256, bk=32, gate_split=2)
    assert L.ffuse_traffic_model(ctypes.byref(bad), ff.DT_BF16, 1, *shape, ctypes.byref(t)) == -8
    # room for both intermediates
    assert ff.ffuse_workspace_bytes(ff.DT_BF16, True, *shape) >= 2 * 2 * 2048 * 11008
    for shp in (shape, (128, 4096, 11008, 4096), (16, 8192, 28672, 8192)):
        ranked = ff.ffuse_rank_plans(ff.DT_BF16, 3, True, *shp)
        splits = [i for i, (p, _) in enumerate(ranked) if p.gate_split]
        assert len(splits) == 1 and splits[0] > 0 and ranked[0][0].gate_split == 0
        assert all(p.gate_split == 0 for p, _ in ff.ffuse_rank_plans(ff.DT_BF16, 2, False, *shp))


def test_the_shipped_plan_table_loads_and_every_entry_is_runnable():
    """The plan table measured offline on an MI355X (paper_2512_12949_amd/plans_mi355x.txt, written by
    paper_2512_12949_amd.tune_plans): it parses, it covers the benchmark configurations and the paper's
    m = 128 tables, every plan is valid for its shape, and a lookup returns it for any M of its bin."""
    from paper_2512_12949_amd import inputs
    ff.ffuse_plan_table_clear()
    try:
        n = ff.ffuse_load_shipped_plans()
        names = ["gpt", "llama", "large", "decode16", "decode64"] + [f"G{i}" for i in range(1, 11)] + [f"S{i}" for i in range(1, 9)]
        assert n == len(names)
        for name in names:
            w = inputs.WORKLOADS[name]
            dt = ff.DTYPE_CODE[w.dtype]
            plan, ms = ff.ffuse_plan_lookup(dt, w.act, w.gated, w.M, w.K, w.N1, w.N2)
            assert ms > 0.0, name                                    # a measured entry, not the model's choice
            t = ff.ffuse_traffic_model(plan, dt, w.gated, w.M, w.K, w.N1, w.N2)     # raises on a plan that is not valid here
            assert t.feasible and 0.3 * t.t_pred < ms * 1e-3 < 3.0 * t.t_pred, (name, ms, t.t_pred)
        # the bin of M, not the exact M: 100 rows share the 65..128 bin with the table's 128
        w = inputs.WORKLOADS["G8"]
        a, ms_a = ff.ffuse_plan_lookup(ff.DT_BF16, w.act, False, 100, w.K, w.N1, w.N2)
        b, ms_b = ff.ffuse_plan_lookup(ff.DT_BF16, w.act, False, 128, w.K, w.N1, w.N2)
        assert ms_a == ms_b > 0 and a.as_dict() == b.as_dict()
        _, ms_c = ff.ffuse_plan_lookup(ff.DT_BF16, w.act, False, 300, w.K, w.N1, w.N2)
        assert ms_c == 0.0
    finally:
        ff.ffuse_plan_table_clear()


def test_no_shipped_entry_is_slower_than_the_models_best_plan():
    """A measured entry overrides the model: recorded times lie within 25 % of what the model expects of its best plan
    (predictions scatter by 8 %), or the table predates a faster kernel and has to be measured again."""
    from paper_2512_12949_amd import inputs
    ff.ffuse_plan_table_clear()
    try:
        ff.ffuse_load_shipped_plans()
        for name in ["gpt", "llama", "large", "decode16", "decode64"] + [f"G{i}" for i in range(1, 11)] + [f"S{i}" for i in range(1, 9)]:
            w = inputs.WORKLOADS[name]
            dt = ff.DTYPE_CODE[w.dtype]
            _, ms = ff.ffuse_plan_lookup(dt, w.act, w.gated, w.M, w.K, w.N1, w.N2)
            _, best = ff.ffuse_rank_plans(dt, w.act, w.gated, w.M, w.K, w.N1, w.N2)[0]
            assert 0.0 < ms * 1e-3 < 1.25 * best, (name, ms, best)
    finally:
        ff.ffuse_plan_table_clear()


# Measured on an MI355X, us per call, back to back on rotating operands: (shape, type, gated, {(family, bm, bh, bk, splits, raster): us}).
# The plans that three models of this chooser ranked first, the best measured one and two others of 30 each.
MEASURED = [
    ((128, 2560, 9728, 2560), ff.DT_BF16, True, {(5, 64, 128, 32, 8, 2): 68.5, (5, 64, 64, 32, 8, 2): 85.1,
      (5, 128, 64, 32, 16, 1): 68.3, (5, 64, 128, 32, 4, 2): 82.4, (5, 64, 64, 64, 8, 2): 100.2}),
    ((128, 1536, 8960, 1536), ff.DT_BF16, True, {(5, 64, 128, 32, 16, 2): 36.3, (5, 64, 64, 32, 16, 2): 42.3,
      (5, 64, 128, 32, 8, 2): 35.0, (5, 128, 128, 32, 32, 1): 45.5, (5, 128, 128, 64, 16, 1): 51.9}),
    ((2551, 2792, 896, 2792), ff.DT_F16, True, {(5, 128, 128, 32, 1, 4): 57.3, (5, 128, 64, 32, 1, 4): 73.7,
      (5, 128, 128, 32, 2, 4): 78.5}),
    ((308, 3000, 6688, 3000), ff.DT_F16, True, {(5, 128, 128, 32, 4, 2): 87.4, (5, 128, 64, 32, 4, 2): 105.7,
      (5, 128, 128, 64, 16, 2): 117.7, (5, 128, 64, 64, 8, 2): 130.1}),
    ((137, 3200, 10048, 3200), ff.DT_F16, True, {(5, 128, 128, 32, 8, 2): 76.4, (5, 128, 64, 32, 8, 2): 89.5,
      (5, 128, 128, 64, 16, 2): 99.6, (5, 256, 128, 32, 8, 1): 111.0}),
    ((384, 1896, 5576, 1896), ff.DT_BF16, False, {(5, 128, 128, 32, 4, 2): 50.3, (5, 128, 64, 32, 8, 2): 58.9,
      (5, 128, 128, 32, 8, 2): 47.1, (5, 128, 256, 32, 16, 2): 61.9, (5, 128, 64, 64, 8, 2): 69.6}),
    ((5573, 1008, 1344, 1008), ff.DT_BF16, False, {(5, 128, 128, 32, 1, 4): 49.2, (5, 128, 256, 32, 1, 4): 57.5,
      (5, 128, 128, 32, 2, 4): 67.9, (5, 128, 256, 32, 2, 4): 73.7}),
    ((71, 1408, 9416, 1408), ff.DT_BF16, True, {(5, 64, 128, 32, 16, 2): 32.5, (5, 64, 64, 32, 16, 2): 38.0,
      (5, 64, 128, 32, 4, 2): 41.5, (5, 128, 64, 64, 8, 1): 48.1}),
    ((812, 2800, 2432, 2800), ff.DT_BF16, True, {(5, 128, 128, 32, 1, 4): 66.2, (5, 128, 64, 32, 2, 4): 77.2,
      (5, 128, 128, 32, 2, 4): 61.1, (5, 128, 128, 64, 1, 4): 83.5, (5, 128, 128, 64, 4, 4): 84.6}),
    ((1382, 2968, 9416, 2968), ff.DT_F16, False, {(5, 256, 256, 32, 2, 4): 209.3, (5, 128, 256, 32, 2, 4): 256.9,
      (5, 128, 128, 32, 1, 4): 284.6, (5, 128, 64, 32, 4, 4): 312.1}),
    ((2662, 3120, 10608, 3120), ff.DT_BF16, False, {(5, 256, 256, 32, 1, 4): 393.4, (5, 128, 256, 32, 1, 4): 479.7,
      (5, 128, 128, 32, 1, 4): 526.9, (5, 128, 64, 32, 2, 4): 576.5}),
    ((711, 3328, 13136, 3328), ff.DT_BF16, False, {(5, 256, 256, 32, 4, 2): 173.0, (5, 128, 256, 32, 4, 4): 210.7,
      (5, 256, 256, 32, 2, 2): 229.7, (5, 128, 128, 64, 4, 4): 244.8}),
    ((1908, 2680, 14760, 2680), ff.DT_BF16, True, {(5, 256, 128, 32, 2, 8): 480.6, (5, 128, 128, 32, 2, 4): 580.6,
      (5, 256, 128, 32, 2, 4): 490.2, (5, 128, 128, 64, 2, 4): 602.8, (5, 128, 64, 32, 1, 4): 713.5}),
    ((1666, 1160, 13576, 1160), ff.DT_BF16, True, {(5, 256, 128, 32, 4, 4): 208.2, (5, 128, 128, 32, 4, 4): 245.3,
      (5, 256, 128, 32, 2, 4): 264.1, (5, 128, 64, 32, 4, 4): 299.9}),
    ((8369, 776, 2888, 776), ff.DT_BF16, False, {(5, 256, 256, 32, 1, 4): 132.7, (5, 128, 256, 32, 1, 4): 146.8,
      (5, 128, 64, 32, 1, 4): 175.0, (5, 128, 128, 64, 2, 4): 183.6}),
    ((578, 1024, 4608, 1024), ff.DT_BF16, True, {(5, 128, 128, 32, 2, 4): 52.2, (5, 128, 128, 32, 8, 4): 39.3,
      (5, 128, 64, 64, 8, 4): 54.5, (5, 128, 64, 64, 4, 4): 58.6}),
    ((641, 1080, 3944, 1080), ff.DT_BF16, True, {(5, 128, 128, 32, 2, 4): 51.9, (5, 128, 128, 32, 8, 4): 42.6,
      (5, 128, 128, 64, 16, 4): 57.4, (5, 128, 128, 64, 2, 4): 61.5}),
    ((10918, 256, 1152, 256), ff.DT_BF16, False, {(5, 256, 256, 32, 1, 4): 53.3, (5, 128, 256, 32, 1, 4): 41.8,
      (5, 128, 128, 64, 1, 4): 52.8, (5, 128, 64, 64, 2, 4): 62.4}),
    ((128, 384, 1536, 384), ff.DT_BF16, False, {(5, 64, 64, 32, 16, 2): 16.4, (1, 16, 64, 32, 24, 1): 10.8,
      (1, 32, 64, 32, 16, 1): 14.6, (5, 64, 64, 32, 32, 2): 16.1}),
    ((231, 512, 1024, 512), ff.DT_BF16, False, {(5, 128, 64, 32, 8, 2): 20.2, (1, 16, 64, 32, 8, 1): 12.5,
      (1, 32, 64, 32, 8, 1): 15.2, (1, 16, 64, 32, 4, 1): 17.0, (1, 16, 64, 32, 16, 1): 12.1}),
    ((4, 7040, 15616, 7040), ff.DT_BF16, True, {(5, 32, 128, 32, 8, 1): 127.4, (5, 32, 128, 64, 16, 1): 149.5,
      (5, 32, 128, 32, 2, 1): 173.8}),
    ((126, 1920, 5136, 1920), ff.DT_F16, False, {(5, 64, 64, 32, 8, 2): 27.3, (5, 64, 64, 32, 16, 2): 28.2,
      (5, 64, 64, 64, 16, 2): 36.8, (5, 128, 64, 32, 4, 1): 40.5}),
    ((4096, 4096, 16384, 4096), ff.DT_BF16, False, {(5, 256, 256, 32, 1, 4): 867.2, (5, 128, 128, 32, 1, 4): 1076.3}),
    ((2048, 4096, 11008, 4096), ff.DT_BF16, True, {(5, 256, 128, 32, 2, 4): 469.2, (5, 128, 64, 32, 1, 4): 607.4,
      (5, 128, 64, 32, 2, 4): 633.6}),
    ((128, 4096, 11008, 4096), ff.DT_BF16, True, {(5, 64, 128, 32, 8, 2): 90.3, (5, 128, 64, 32, 16, 1): 87.4,
      (5, 64, 128, 32, 32, 2): 108.6, (5, 64, 128, 32, 2, 2): 128.1, (5, 128, 64, 32, 8, 1): 87.8}),
    ((142, 1152, 1664, 1152), ff.DT_BF16, True, {(5, 128, 64, 32, 8, 2): 28.4, (1, 16, 64, 32, 26, 1): 23.3,
      (5, 128, 128, 32, 16, 2): 32.5, (5, 128, 64, 64, 8, 2): 34.0, (5, 64, 64, 32, 8, 2): 23.2,
      (5, 64, 64, 32, 8, 3): 22.6}),
]


def test_the_models_choice_against_measured_plans():
    """Regression set of the chooser: its choice is among the measured plans and within 5 % of the best of them.
    Predictions scatter by 8 % round the measured time where a plan is worth running; the worst of this set is 1.46 off
    (a plan that measures 25 % behind).  (A model that priced a lone partial round of items as a whole
    one, but the last of two rounds low, lost 10-29 % on the first fifteen.)"""
    for (shape, dt, gated, plans) in MEASURED:
        act = 3 if gated else 2
        c = ff.ffuse_choose_plan(dt, act, gated, *shape)
        key = (c.family, c.bm, c.bh, c.bk, c.splits, c.raster)
        assert key in plans, (shape, gated, key)
        assert plans[key] <= 1.05 * min(plans.values()), (shape, gated, key, plans)
        for (family, bm, bh, bk, splits, raster), us in plans.items():
            p = ff.make_plan(family, bm=bm, bh=bh, bn2=256, bk=bk, splits=splits, raster=raster)
            t = ff.ffuse_traffic_model(p, dt, gated, *shape).t_pred * 1e6
            assert us / 1.5 < t < 1.5 * us, (shape, gated, (family, bm, bh, bk, splits, raster), us, t)


def test_accumulators_of_the_small_row_blocks():
    """bm rows x 256 ng output columns of fp32 over the 512 lanes of eight waves (over 256 of them where ng = 1: the others
    hold the other half of the hidden columns), over 256 lanes with four waves: gated with K above 256."""
    for N2, ng in ((8, 1), (256, 1), (264, 2), (512, 2), (1000, 4), (2048, 8)):
        for bm in (16, 32):
            if bm == 32 and N2 > 512:
                continue
            plan = ff.make_plan(ff.FAMILY_REDUCE, bm=bm, bh=64, bk=32, splits=2)
            t = ff.ffuse_traffic_model(plan, ff.DT_BF16, False, 100, 512, 512, N2)
            assert t.feasible and t.acc_regs == bm * max(1, ng // 2), (N2, bm, t.acc_regs)
            t = ff.ffuse_traffic_model(plan, ff.DT_BF16, True, 100, 512, 512, N2)
            assert t.feasible and t.acc_regs == bm * ng <= 256, (N2, bm, t.acc_regs)


def test_lds_of_the_small_row_blocks():
    """The model's LDS bytes are the kernels': the figures of the compiler's resource report (-Rpass-analysis=kernel-resource-usage)."""
    # (rows, K, N1, N2, bm, ranges, gated): K up to 256 and past it, one slice a range and several, fewer and more workgroups than
    # the 256 compute units
    for M, K, N1, N2, bm, splits, gated, lds in (
            (100, 512, 512, 256, 16, 2, False, 35072), (100, 256, 512, 256, 16, 2, False, 35072), (100, 512, 512, 256, 32, 2, False, 70144),
            (100, 256, 512, 512, 32, 2, False, 70144), (100, 512, 512, 256, 16, 2, True, 35072), (100, 512, 512, 256, 32, 2, True, 70144),
            (100, 256, 512, 256, 16, 2, True, 67840), (100, 256, 512, 512, 32, 2, True, 135680), (100, 264, 512, 256, 16, 8, False, 35072),
            (4096, 64, 64, 64, 16, 1, False, 35072), (4097, 64, 64, 64, 16, 1, False, 18688), (4097, 64, 128, 64, 16, 1, False, 35072),
            (4097, 64, 64, 264, 16, 1, False, 35072), (8200, 64, 64, 64, 32, 1, False, 70144), (4097, 64, 64, 64, 16, 1, True, 67840)):
        t = ff.ffuse_traffic_model(ff.make_plan(ff.FAMILY_REDUCE, bm=bm, bh=64, bk=32, splits=splits), ff.DT_BF16, gated, M, K, N1, N2)
        assert t.feasible and t.lds_used == lds, (M, K, N1, N2, bm, splits, gated, t.lds_used)


def test_fp32_predictions_against_measured_calls():
    """fp32 mode on an MI355X, us per call: one row to 8192, gated and not (a prediction within a factor 1.5)."""
    plain = {(16, 256, 1024, 256): 8.1, (128, 256, 1024, 256): 10.1, (256, 512, 2048, 512): 29.3, (512, 512, 2048, 512): 46.8,
             (2048, 512, 2048, 512): 151.6, (8192, 256, 1024, 256): 152.8, (512, 1024, 4096, 1024): 146.8, (2048, 1024, 4096, 1024): 484.6,
             (16, 4096, 11008, 4096): 168.2, (128, 64, 256, 64): 7.7, (64, 1000, 264, 1000): 18.3, (333, 1016, 2744, 1016): 99.7,
             (1, 512, 2048, 512): 10.6}
    gated = {(128, 256, 1024, 256): 13.3, (512, 512, 2048, 512): 55.8, (2048, 512, 2048, 512): 174.7, (2048, 1024, 4096, 1024): 605.6,
             (16, 4096, 11008, 4096): 229.7, (128, 64, 256, 64): 7.7}
    for table, g in ((plain, False), (gated, True)):
        for shape, us in table.items():
            p = ff.ffuse_choose_plan(ff.DT_F32, 2, g, *shape)
            t = ff.ffuse_traffic_model(p, ff.DT_F32, g, *shape).t_pred * 1e6
            print(shape, g, us, round(t, 1))
            assert us / 1.5 < t < 1.5 * us, (shape, g, us, t)


# Small row blocks, bf16, us per call: (shape, gated, rows, ranges, us).  Two or fewer of each variant, drawn from the timings within
# 12 % of their shape's best plan.
SMALL_BLOCKS = [
    ((87, 2296, 96, 144), False, 16, 2, 10.9), ((53, 456, 1984, 456), False, 16, 31, 10.1), ((34, 496, 72, 320), False, 16, 2, 6.6),
    ((182, 768, 2048, 768), False, 16, 16, 20.2), ((58, 568, 4192, 920), False, 16, 32, 22.1), ((108, 1944, 544, 1944), False, 16, 9, 19.3),
    ((14, 320, 352, 1632), False, 16, 6, 10.6), ((13, 1200, 1592, 72), False, 32, 25, 11.1), ((180, 328, 1872, 328), False, 32, 16, 13.7),
    ((176, 520, 336, 144), True, 16, 6, 8.7), ((158, 384, 512, 384), True, 16, 8, 9.6), ((105, 512, 1536, 512), True, 16, 24, 12.3),
    ((23, 448, 1480, 592), True, 16, 24, 11.8), ((68, 2152, 656, 760), True, 16, 11, 21.1), ((64, 1976, 192, 1800), True, 16, 3, 20.5),
    ((128, 768, 2688, 128), True, 32, 32, 18.5), ((193, 512, 1408, 512), True, 32, 22, 16.5), ((36, 208, 1352, 208), False, 16, 22, 6.9),
    ((10, 208, 2248, 208), False, 16, 32, 8.1), ((49, 72, 512, 288), False, 16, 8, 5.7), ((166, 128, 9968, 128), False, 32, 32, 14.9),
    ((569, 200, 1408, 312), False, 32, 16, 14.3), ((118, 136, 752, 144), True, 16, 12, 6.7), ((893, 64, 80, 240), True, 16, 1, 5.2),
    ((964, 64, 560, 400), True, 16, 4, 12.5), ((214, 128, 5632, 128), True, 32, 32, 14.6), ((2734, 96, 632, 352), True, 32, 2, 21.2),
]


def test_small_row_blocks_are_priced_as_they_run():
    """Predictions scatter by 7 % round 3600 timings: 27 of them average within 3 % (two standard errors), each within three times
    the scatter.  (The constants of the four-wave kernel are 5 % high here, 8 % over all.)"""
    logs = []
    for shape, gated, rows, ranges, us in SMALL_BLOCKS:
        p = ff.make_plan(1, bm=rows, bh=64, bn2=256, bk=32, splits=ranges, h_level=1, raster=1)
        logs.append(math.log(ff.ffuse_traffic_model(p, ff.DT_BF16, gated, *shape).t_pred * 1e6 / us))
        assert abs(logs[-1]) <= 0.21, (shape, us, logs[-1])
    assert abs(sum(logs) / len(logs)) <= 0.03, sum(logs) / len(logs)


# 64-row blocks against their neighbours, as above: the six fastest plans of about thirteen.
MEASURED_64 = [
    ((225, 512, 13312, 512), False, {(5, 128, 128, 32, 32, 2): 30.5, (5, 128, 128, 32, 16, 2): 31.2, (5, 64, 128, 32, 16, 4): 31.7,
      (5, 128, 128, 32, 32, 1): 32.4, (5, 128, 256, 32, 32, 2): 32.5, (5, 64, 128, 32, 32, 4): 33.2}),
    ((96, 1152, 1920, 1152), False, {(1, 16, 64, 32, 30, 1): 17.3, (5, 64, 64, 32, 8, 1): 21.3, (5, 64, 64, 32, 8, 2): 21.6,
      (5, 64, 64, 32, 16, 2): 21.7, (1, 16, 64, 32, 16, 1): 22.7, (5, 64, 64, 32, 4, 2): 22.8}),
    ((208, 1920, 1024, 1920), True, {(5, 64, 64, 32, 4, 4): 25.5, (5, 64, 64, 32, 2, 4): 26.7, (1, 16, 64, 32, 16, 1): 29.2,
      (5, 128, 64, 32, 4, 2): 30.6}),
    ((215, 424, 1120, 1680), True, {(5, 64, 64, 32, 4, 4): 19.9, (5, 64, 64, 32, 8, 4): 20.1, (5, 128, 64, 32, 8, 2): 22.7,
      (1, 16, 64, 32, 16, 1): 24.6}),
    ((128, 984, 2768, 984), False, {(1, 16, 64, 32, 32, 1): 20.0, (5, 64, 64, 32, 8, 2): 22.4, (5, 64, 64, 32, 8, 1): 22.9,
      (5, 64, 64, 32, 16, 2): 22.9, (5, 64, 128, 32, 8, 2): 23.2}),
    # three row blocks: one patch of weight slices for all of them
    ((192, 1216, 10096, 1216), True, {(5, 64, 128, 32, 16, 3): 34.5, (5, 128, 128, 32, 16, 2): 39.7, (5, 64, 64, 32, 16, 3): 39.8,
      (5, 64, 128, 32, 16, 2): 42.4, (5, 128, 128, 32, 16, 1): 42.5}),
    ((141, 1664, 5248, 1664), True, {(5, 64, 64, 32, 8, 3): 29.4, (5, 64, 128, 32, 8, 3): 32.6, (5, 64, 128, 32, 8, 2): 33.6,
      (5, 64, 64, 32, 8, 2): 34.7, (5, 128, 64, 32, 16, 2): 35.7}),
    ((131, 2568, 4448, 2568), True, {(5, 64, 64, 32, 4, 3): 38.7, (5, 128, 64, 32, 8, 2): 43.3, (5, 64, 64, 32, 4, 2): 43.5,
      (5, 64, 64, 32, 16, 2): 45.8, (5, 64, 64, 32, 4, 1): 45.9}),
    ((152, 984, 8720, 2472), False, {(5, 64, 128, 32, 8, 3): 33.8, (5, 64, 128, 32, 8, 2): 36.5, (5, 64, 64, 32, 8, 3): 37.0,
      (5, 128, 128, 32, 8, 2): 37.1}),
]


@pytest.mark.parametrize("shape,gated,plans", MEASURED_64)
def test_64_row_blocks_where_they_are_the_faster_ones(shape, gated, plans):
    """No layer is kept from them by its sizes, and they are priced as they run."""
    c = ff.ffuse_choose_plan(ff.DT_BF16, 3 if gated else 2, gated, *shape)
    key = (c.family, c.bm, c.bh, c.bk, c.splits, c.raster)
    assert key in plans and plans[key] <= 1.03 * min(plans.values()), (key, plans)


@pytest.mark.parametrize("shape,gated,plans", [
    # three sets of operands in turn; on one set 77.7 / 86.3 / 80.2, and 31.5 / 34.5
    ((128, 4096, 11008, 4096), True, {(5, 128, 64, 32, 8, 1): 87.8, (5, 128, 64, 32, 16, 1): 89.3, (5, 64, 128, 32, 8, 2): 89.6}),
    ((128, 2048, 8192, 2048), False, {(5, 64, 64, 32, 8, 2): 32.0, (5, 64, 64, 32, 16, 2): 35.2}),
])
def test_planes_are_bytes_of_the_second_phase(shape, gated, plans):
    """More hidden ranges fill the second phase's CUs, and each writes a plane beside the weights it reads."""
    c = ff.ffuse_choose_plan(ff.DT_BF16, 3 if gated else 2, gated, *shape)
    key = (c.family, c.bm, c.bh, c.bk, c.splits, c.raster)
    assert key in plans and plans[key] == min(plans.values()), (key, plans)


def test_small_row_blocks_fill_each_l2_with_what_its_ranges_read():
    """Workgroups go round the XCDs range by range: eight ranges read an eighth of the weights each, 25 all of them."""
    shape = (148, 1144, 3192, 128)
    weights = 2 * (2 * 1144 * 3192 + 3192 * 128)
    fabric = {}
    for ranges in (8, 10, 13, 25):   # of 50 slices: all of them are kept
        p = ff.make_plan(1, bm=16, bh=64, bn2=256, bk=32, splits=ranges, h_level=1, raster=1)
        t = ff.ffuse_traffic_model(p, ff.DT_BF16, True, *shape)
        fabric[ranges] = (t.fabric_bytes - t.reduce_bytes) / weights
    # (ranges of 7, 5, 4 and 2 slices: 8, 10, 13 and 25 of them)
    assert fabric[8] < 1.2 and 4.0 <= fabric[10] < 4.3 and 8.0 <= fabric[13] < 8.3 and 8.0 <= fabric[25] < 8.3, fabric
    # where every XCD reads all of it, the layer is better off in the two-phase kernel: 25.0 us
    c = ff.ffuse_choose_plan(ff.DT_BF16, 3, True, *shape)
    assert c.family == ff.FAMILY_TWOPHASE, c.as_dict()
