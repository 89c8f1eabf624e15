"""The tables of bench.py's line where both gradients of a layer share one launch and so one interval of the timeline."""
import types

import pytest

import bench


def _tables(layers):
    rows, gemms = {}, []
    for li, (name, M, K, N) in enumerate(layers):
        for gemm, m, n, k in (("fwd", M, N, K), ("dX", M, K, N), ("dW", K, N, M)):
            ops, nbytes = 2.0 * m * n * k, float(m * k + n * k + 4 * m * n)
            gemms.append(dict(layer=name, layer_index=li, gemm=gemm, M=m, N=n, K=k, ops=ops, bytes=nbytes, us=5.0, us_loop_min=4.0,
                              bound="hbm", core_clock_mhz=None))
            r = rows.setdefault("gemm_" + gemm, dict(kernel="k", t=0.0, tmin=0.0, launches=0, bytes=0.0, ops=0.0))
            for key, v in (("t", 5e-6), ("tmin", 4e-6), ("launches", 1), ("bytes", nbytes), ("ops", ops)):
                r[key] += v
    return rows, gemms


# both layers with a launch for both gradients, none, one of each
@pytest.mark.parametrize("paired", [(0, 1), (), (1,)])
def test_rows_follow_the_intervals(paired):
    layers = [("a", 256, 256, 256), ("b", 64, 512, 128)]
    rows, gemms = _tables(layers)
    total = {k: sum(r[k] for r in rows.values()) for k in ("ops", "bytes", "t")}
    in_step = {}
    for li in range(2):
        in_step[(li, "gemm_fwd")] = 40.0
        for g in (("gemm_dW+dX",) if li in paired else ("gemm_dW", "gemm_dX")):
            in_step[(li, g)] = 60.0
    bench.join_paired_gradients(rows, gemms, [types.SimpleNamespace(name=l[0]) for l in layers], in_step)
    bench.set_in_step_times(rows, gemms, in_step, 10)
    assert set(rows) == {g for _, g in in_step}
    assert [(g["layer_index"], "gemm_" + g["gemm"]) for g in gemms] == sorted(
        in_step, key=lambda k: (k[0], ["gemm_fwd", "gemm_dX", "gemm_dW+dX", "gemm_dW"].index(k[1])))
    assert all(r["t"] > 0.0 for r in rows.values()) and all(g["us"] > 0.0 for g in gemms)
    for key, loop in (("ops", "ops"), ("bytes", "bytes"), ("t", "t_loop")):
        assert sum(r[loop] for r in rows.values()) == pytest.approx(total[key])
    assert sum(r["launches"] for r in rows.values()) == 6 - len(paired)
    assert sum(g["ops"] for g in gemms) == total["ops"] and sum(g["bytes"] for g in gemms) == total["bytes"]


@pytest.mark.parametrize("sizes,joint", [([(256, 256, 256)], True), ([(256, 256, 256), (25088, 1152, 128)], False)])
def test_small_layers_have_no_scale_row(sizes, joint):
    layers = [types.SimpleNamespace(M=M, K=K, N=N) for M, K, N in sizes]
    rows = {r: dict(kernel=r, t=t, tmin=t, launches=2, bytes=b, ops=0.0) for r, t, b in (("map", 6e-6, 600.0), ("scale", 2e-6, 400.0))}
    in_step = {(li, r): us for li in range(len(layers)) for r, us in (("map", 50.0), ("scale", 10.0))}
    bench.join_small_scales(rows, layers, in_step)
    bench.set_in_step_times(rows, [], in_step, 10)
    assert set(rows) == ({"map"} if joint else {"map", "scale"})
    assert rows["map"]["t"] == pytest.approx(5e-6 * len(layers)) and (joint or rows["scale"]["t"] == pytest.approx(1e-6 * len(layers)))
    assert sum(r["t_loop"] for r in rows.values()) == pytest.approx(8e-6) and rows["map"]["bytes"] == 600.0


def test_tags_of_the_header():
    import os
    import re
    text = open(os.path.join(bench.ROOT, "include", "fxp.h")).read()
    tags = {int(v): name for name, v in re.findall(r"FXP_TL_(\w+) = (\d+)", text)}
    assert set(bench.TIMELINE_ROWS) | {0} == set(tags)
