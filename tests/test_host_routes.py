"""How calls go out (binding.tile_route, grid.route: the library's own plans, on the CPU): the rules that were measured, and that
the GPU tests' cases take the kernels they are there for.  256 compute units, as on MI355X."""
import itertools
import random

import pytest
import torch

CUS = 256


@pytest.fixture(scope="module")
def a2d():
    from paper_2503_15758_amd import binding
    binding._ext()
    return binding


def tile(a2d, heads, nq, nkv, H, **more):
    return a2d.tile_route(heads, nq, nkv, H, compute_units=CUS, **more)


def test_keeping_ds_does_not_change_dk_dv(a2d):
    """The choice for dK and dV is the same with A2D_DESC_KEEP_DS as without: their bits are part of the contract."""
    rng, kept = random.Random(5), 0
    for _ in range(400):
        kv = int(2 ** rng.uniform(0, 7))
        heads = kv * rng.choice([1, 1, 2, 4])
        nq, nkv = (int(2 ** rng.uniform(5, 13)) for _ in range(2))
        more = dict(kv_heads=kv, causal=rng.random() < 0.5, q_off=rng.randint(0, nkv), backward=True, scratch=rng.random() < 0.7)
        plain, keep = (tile(a2d, heads, nq, nkv, 128, ds_handover=k, **more) for k in (False, True))
        case = (heads, nq, nkv, more)
        assert ("bwd_small_kernel" in plain["kernels"]) == ("bwd_small_kernel" in keep["kernels"]), case
        assert (plain["keys"], plain["parts_kv"]) == (keep["keys"], keep["parts_kv"]), case
        kept += "bwd_dq_ds_kernel" in keep["kernels"]
    assert kept > 50


# heads, kv_heads, nq, nkv, H, causal, q_off; us on MI355X in one launch and in two (dQ, then dK/dV)
MEASURED = [
    (51, 51, 2015, 438, 64, False, 0, 95.9, 87.8),
    (51, 51, 3000, 1185, 64, False, 0, 226.0, 215.1),
    (16, 16, 4096, 4096, 64, False, 0, 265.3, 261.7),
    (72, 18, 651, 861, 64, False, 0, 87.7, 76.6),
    (6, 6, 9048, 1290, 128, False, 0, 196.6, 173.6),
    (8, 1, 11144, 5593, 64, False, 0, 603.1, 557.3),
    (18, 9, 1125, 1107, 80, False, 0, 80.7, 60.6),
    (72, 72, 575, 304, 64, True, 246, 44.6, 35.6),
    (46, 23, 541, 1027, 128, False, 0, 94.3, 77.2),
    (9, 9, 563, 2404, 80, False, 0, 50.2, 42.9),
    (7, 7, 7700, 1656, 64, False, 0, 149.2, 121.7),
    (14, 14, 4494, 358, 64, True, 0, 54.8, 48.7),
    (16, 16, 1024, 1024, 128, False, 0, 50.3, 71.1),
    (16, 16, 2048, 2048, 128, False, 0, 129.3, 136.7),
    (32, 32, 1999, 2777, 80, True, 778, 171.8, 174.6),
    (7, 7, 780, 426, 80, False, 0, 15.2, 27.3),
    (31, 31, 1897, 1815, 80, True, 0, 103.4, 120.5),
    (6, 3, 4206, 2488, 64, False, 0, 85.4, 98.9),
    (48, 6, 1282, 2778, 128, False, 0, 389.0, 516.0),
    (84, 84, 4318, 80, 80, False, 0, 118.5, 128.3),
    (2, 2, 146, 5176, 128, False, 0, 24.0, 35.0),
    # many keys that few rows see: one launch with the dQ workgroups first, by the time of that order
    (124, 31, 782, 5816, 64, True, 0, 133.2, 112.7),
    (88, 22, 1364, 7717, 64, True, 0, 208.4, 179.1),
    (24, 12, 4219, 10402, 128, True, 0, 487.7, 433.1),
]


@pytest.mark.parametrize("case", MEASURED, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_one_launch_only_where_it_is_not_slower(a2d, case):
    heads, kvh, nq, nkv, H, causal, q_off, one, two = case
    for scratch in (True, False):                  # (without scratch memory the walks are whole: the rule holds, the times do not)
        kernels = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, backward=True, scratch=scratch)["kernels"]
        assert ("bwd_dq_kernel" in kernels) == (not {"bwd_one_kernel", "bwd_small_kernel"} & set(kernels))
        if scratch:
            assert ("bwd_dq_kernel" in kernels) == (two < one), kernels


# heads, kv_heads, nq, nkv, H, causal; us on MI355X in whole walks and in the parts of dK/dV and dQ that are taken
F32_MEASURED = [(8, 8, 256, 900, 80, False, 31.8, 27.5), (2, 2, 361, 157, 80, True, 13.9, 9.1),
                (16, 8, 334, 116, 64, False, 21.8, 15.8), (6, 6, 879, 282, 64, True, 28.7, 20.7)]


@pytest.mark.parametrize("case", F32_MEASURED, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_fp32_walks_are_shared_where_three_workgroups_fit(a2d, case):
    heads, kvh, nq, nkv, H, causal, whole, shared = case
    r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, dtype=torch.float32, backward=True, split_groups=kvh != heads)
    assert (r["parts_q"] * r["parts_kv"] > 1) == (shared < whole)


def test_route_refuses_what_the_calls_refuse(a2d):
    with pytest.raises(a2d.A2DError):
        tile(a2d, 4, 100, 100, 72)
    with pytest.raises(a2d.A2DError):
        tile(a2d, 4, 100, 100, 64, kv_heads=3)
    with pytest.raises(a2d.A2DError):
        tile(a2d, 4, 100, 100, 64, segments=[(0, 99)])
    from paper_2503_15758_amd import grid as g2d
    assert g2d.route(4, 128, 72, 2, compute_units=CUS) is None


# heads, kv_heads, nq, nkv, H, causal, q_off; us on MI355X in the form before and in the one that is taken, its rows and key lanes
FORWARD_MEASURED = [(84, 21, 12746, 306, 64, False, 0, 204, 139, (128, 1)), (88, 44, 16347, 158, 96, False, 0, 250, 180, (128, 1)),
                    (60, 15, 14581, 193, 96, False, 0, 187, 134, (128, 1)), (1, 1, 65, 1125, 96, False, 0, 12.3, 8.7, (32, 8)),
                    (96, 96, 4096, 4096, 128, False, 0, 743, 720, (256, 1)), (96, 96, 4096, 4096, 128, True, 0, 406, 400, (256, 1))]


@pytest.mark.parametrize("case", FORWARD_MEASURED, ids=lambda c: "%dq%dkv_%dx%dH%d_%s" % (*c[:5], "causal" if c[5] else "full"))
def test_forward_takes_the_form_that_is_faster_now(a2d, case):
    heads, kvh, nq, nkv, H, causal, q_off, _, _, form = case
    r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off)
    assert (r["rows"], r["lanes"]) == form and r["parts_q"] == 1, r


def test_parts_need_scratch_memory(a2d):
    for dtype in (torch.bfloat16, torch.float32):
        for backward in (False, True):
            shared, alone = (tile(a2d, 1, 60, 20000, 128, dtype=dtype, backward=backward, scratch=s) for s in (True, False))
            assert shared["parts_q"] > 1 and alone["parts_q"] == alone["parts_kv"] == 1
            assert shared["kernels"][-1] == ("sum_parts_kernel" if backward else "fix_kernel")
            assert "sum_parts_kernel" not in alone["kernels"] and "fix_kernel" not in alone["kernels"]


@pytest.mark.parametrize("workload", ["c2", "c3", "c4", "c5"])
def test_bench_names_the_kernels_of_the_library(a2d, workload, monkeypatch):
    """What bench.py logs for a call, and reports times of, is what the library launches: the form of the dK/dV kernel too."""
    import bench
    from paper_2503_15758_amd import synth
    route = a2d.tile_route
    monkeypatch.setattr(a2d, "tile_route", lambda *x, **more: route(*x, **dict(more, compute_units=CUS)))
    kernels = bench.call_kernels.__wrapped__
    monkeypatch.setattr(bench, "call_kernels", kernels)
    w = synth.WORKLOADS[workload]
    for recompute in (False, True):
        got = [kernels("partial_bwd_" + tag, w, recompute) for tag in ("full", "diag")]
        want = ["delta_kernel", "bwd_one_kernel"] if workload == "c2" else \
            ["bwd_dq_kernel", "bwd_dkdv_wide_kernel"] if recompute else \
            ["delta_kernel", "bwd_dkdv_wide_kernel", "bwd_dq_ds_kernel"]
        if w.backward:
            assert got == [want, want]
            assert bench.bwd_path(["partial_bwd_full"], w, recompute) == \
                ("recompute" if recompute or workload == "c2" else "dS hand-over")
        assert kernels("partial_fwd_full", w, recompute) == ["fwd_mfma_kernel"]


# ---- the GPU tests' cases take the kernels that they are there for
FORMS = [(256, 1), (128, 2), (128, 1)]             # rows, key lanes of the forward and dQ kernels of large tiles
SIZES = (64, 80, 96, 128)


def every(*axes):
    return set(itertools.product(*axes))


def test_launch_variant_cases(a2d):
    import test_gpu_launch_variants as t
    fwd, masked, dq, shared, dkdv, kept, grouped = (set() for _ in range(7))
    for heads, kvh, nq, nkv, H, causal, q_off, kv_off in t.ROUTES:
        route = lambda **more: tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, kv_off=kv_off, **more)
        f, b, d = route(), route(backward=True), route(backward=True, ds_handover=True)
        if f["kernels"] == ("fwd_mfma_kernel",):
            form = (f["rows"], f["lanes"])
            fwd.add((form, H))
            masked.add(("forward", form, causal))
            grouped.add(("forward", form, heads > kvh))
        if "bwd_dq_kernel" in b["kernels"]:
            form = (b["rows"], b["lanes"])
            dq.add((form, H))
            dkdv.add((b["kernels"][1], H))
            masked.add(("dQ", form, causal))
            grouped.add(("dQ", form, heads > kvh))
            if b["parts_q"] > 1:
                shared.add(form)
        if "bwd_dq_ds_kernel" in d["kernels"]:
            form = (d["rows"], d["lanes"])
            kept.add((form, d["keys"]))
            masked.add(("dQ from dS", form, causal))
            grouped.add(("dQ from dS", form, heads > kvh))
    kinds = ("forward", "dQ", "dQ from dS")
    assert fwd == dq == every(FORMS, SIZES) and shared == set(FORMS)
    assert dkdv == every(("bwd_dkdv_kernel", "bwd_dkdv_wide_kernel"), SIZES) and kept == every(FORMS, (128, 256))
    assert masked == grouped == every(kinds, FORMS, (False, True))
    strided = [tile(a2d, 72, n, n, 96, causal=True) for n in (700, 900)]
    assert [(r["rows"], r["lanes"]) for r in strided] == [(256, 1), (128, 1)]


def test_hidden_score_cases(a2d):
    import test_gpu_hidden_scores as t
    took = set()
    for dtype, heads, H in t.CASES:
        for keep in (False, True) if dtype == "bf16" else ():
            r = tile(a2d, heads, t.NQ, t.NKV, H, causal=True, q_off=t.OFF, backward=True, ds_handover=keep)
            took |= {(k, r["keys"], H) for k in r["kernels"]}
    assert {("bwd_small_kernel", 32, 128), ("bwd_one_kernel", 128, 80), ("bwd_one_kernel", 128, 128),
            ("bwd_dkdv_kernel", 128, 64), ("bwd_dq_ds_kernel", 256, 128)} <= took
    assert {("bwd_one_kernel", 256, H) for H in SIZES} | {("bwd_dkdv_wide_kernel", 256, H) for H in SIZES} <= took


def test_wide_key_cases(a2d):
    import test_gpu_wide_keys as t
    took = set()
    for cases, keys in ((t.CASES, 256), (t.NARROW, 128)):
        for heads, kvh, nq, nkv, H, causal, q_off, segs in cases:
            for keep in (False, True):
                r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, segments=segs, backward=True,
                         ds_handover=keep)
                assert r["keys"] == keys, (heads, nq, nkv, H)
                took |= {(k, H) for k in r["kernels"]}
    assert {("bwd_one_kernel", H) for H in SIZES} | {("bwd_dkdv_wide_kernel", H) for H in SIZES} <= took
    assert ("bwd_dq_ds_kernel", 128) in took


def test_few_row_cases(a2d):
    import test_gpu_small_bwd as b
    import test_gpu_small_rows as f
    rows64 = set()
    for cases, form in ((f.ROWS32, (32, 8)), (f.ROWS64, (64, 4)), (f.PAIRS, (128, 1))):
        for heads, kvh, nq, nkv, H, causal, q_off, segs, *_ in cases:
            r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, segments=segs)
            assert (r["rows"], r["lanes"]) == form, (heads, nq, nkv, H)
            if form == (64, 4):
                rows64.add((H, causal and q_off < 0 or segs is not None))
    assert {H for H, _ in rows64} == set(SIZES) and {(64, True), (80, True), (96, True), (128, True)} <= rows64
    apart = set()
    for cases, small in ((b.CASES, True), (b.PAIRS, False), (b.BOTH, True)):
        for heads, kvh, nq, nkv, H, causal, q_off, segs, _ in cases:
            r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, segments=segs, backward=True)
            assert ("bwd_small_kernel" in r["kernels"]) == small, (heads, nq, nkv, H)
            assert not (r["apart"] and cases is b.BOTH), (heads, nq, nkv, H)
            if small:
                apart.add((r["apart"], H))
    assert {c[4] for c in b.CASES} == set(SIZES) and apart == every((False, True), SIZES)


def test_backward_route_cases(a2d):
    import test_gpu_bwd_routes as t
    for cases, one in ((t.ONE, True), (t.MANY, False)):
        for heads, kvh, nq, nkv, H, causal, q_off, segs, _ in cases:
            r = tile(a2d, heads, nq, nkv, H, kv_heads=kvh, causal=causal, q_off=q_off, segments=segs, backward=True,
                     ds_handover=H == 128)
            assert bool({"bwd_one_kernel", "bwd_small_kernel"} & set(r["kernels"])) == one, (heads, nq, nkv, H)
            assert ("bwd_dq_ds_kernel" in r["kernels"]) == (not one and H == 128)
    took = {tile(a2d, *c, H, causal=True, backward=True, ds_handover=k)["kernels"] for c in t.DELTA for H in SIZES for k in (False, True)}
    assert {("bwd_small_kernel",), ("bwd_one_kernel",), ("delta_kernel", "bwd_one_kernel"),
            ("bwd_dq_kernel", "bwd_dkdv_wide_kernel"), ("delta_kernel", "bwd_dkdv_wide_kernel", "bwd_dq_ds_kernel")} <= took


def test_grid_row_cases(a2d):
    import test_gpu_grid_rows as t
    from paper_2503_15758_amd import grid as g2d
    layouts = ("cyclic", "contiguous")
    fwd, shared, sizes, bwd, heads_of, apart = (set() for _ in range(6))
    for heads, kvh, rows, side, H in t.CASES:
        for causal, layout in every((False, True), layouts):
            route = lambda backward: g2d.route(heads, rows * side, H, side, kvh, causal, layout, backward, CUS)
            f, b = route(False), route(True)
            form = (f["rows"], f["lanes"])
            (shared if f["parts_q"] > 1 else fwd).add((form, layout, causal))
            if f["parts_q"] == 1:
                sizes.add((form, H))
                heads_of.add((form, heads > kvh))
            kind = (b["keys"], b["rows"], b["lanes"])
            bwd.add((kind, layout, causal))
            if b["keys"] == 32:
                apart.add((b["apart"], layout, causal))
            sizes.add((b["keys"], H))
            heads_of.add((b["keys"], heads > kvh))
    forms = FORMS + [(64, 4), (32, 8)]
    kinds = [(32, 32, 8)] + [(keys, *form) for keys in (128, 256) for form in FORMS[:2]]
    assert fwd == every(forms, layouts, (False, True)) and sizes == every(forms + [32, 128, 256], SIZES)
    # (the 64-row form shares unmasked walks only)
    assert shared == every(forms, layouts, (False, True)) - every([(64, 4)], layouts, [True])
    assert bwd == every(kinds, layouts, (False, True)) and apart == every((False, True), layouts, (False, True))
    assert heads_of == every(forms + [32, 128, 256], (False, True))


def test_phased_grid_cases(a2d):
    import test_gpu_grid_rows as t
    from paper_2503_15758_amd import grid as g2d
    layouts, took, shared = ("cyclic", "contiguous"), set(), set()
    for heads, kvh, rows, side, H in t.PHASED:
        for causal, layout in every((False, True), layouts):
            r = g2d.route(heads, rows * side, H, side, kvh, causal, layout, False, CUS)
            if r["phased"]:
                (shared if r["parts_q"] > 1 else took).add(((r["rows"], r["lanes"]), layout, causal))
    assert took == every(FORMS[:2], layouts, (False, True)) and shared >= every(FORMS[:2], layouts, [False])


def test_phases_need_long_walks_of_heads_of_128(a2d):
    """us on MI355X in order / in phases: 16 x 2048 x 2048 38.2 / 37.6, 96 x 4096 x 4096 852 / 824; 9 x 2616 x 288 19.9 / 20.9, 39 x 9559 x 1886, H = 80 916 / 957."""
    for heads, nq, nkv, H, phased in [(16, 2048, 2048, 128, True), (96, 4096, 4096, 128, True), (9, 2616, 288, 128, False), (39, 9559, 1886, 80, False)]:
        assert tile(a2d, heads, nq, nkv, H)["phased"] == phased, (heads, nq, nkv, H)
