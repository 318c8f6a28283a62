"""Distances on the vector ALU: both tile sizes (64 x 64 while there are fewer than 512 of 128 x 128), edges of either, contracted
labels of less than a stage, of whole stages and with whole 16-byte vectors or single elements behind them, both layouts and types.
Squared differences against the oracle; the largest absolute difference exactly, with NaN among the operands."""
import numpy as np
import pytest

from tests._parity import RTOL_F32, single_vertex, violations
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu

SHAPES = [("ij,jk->ik", 64, 64, 8), ("ij,kj->ik", 136, 72, 24), ("ij,jk->ik", 200, 136, 64), ("ij,kj->ik", 72, 264, 136), ("ji,jk->ik", 136, 200, 77), ("ji,jk->ik", 64, 72, 131),
          ("ij,jk->ik", 2824, 3080, 40), ("ij,kj->ik", 2824, 3080, 72)]      # the last two: 575 tiles of 128 x 128


def _operands(spec, m, n, k, dtype, poison):
    ext = {"i": m, "j": k, "k": n}
    t = []
    for pos, labels in enumerate(spec.split("->")[0].split(",")):
        b = tuple(ext[l] for l in labels)
        a = uniform_pm1(61, pos, int(np.prod(b))).reshape(b).copy()
        if poison and pos == 0:
            a.ravel()[:: 97] = np.nan
        t.append(HostTensor.from_f32(a, dtype))
    return t


def _run(w, x, y):
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    r = GraphRunner(w, "d")
    try:
        r.bind({"X": to_device(x), "Y": to_device(y)})
        assert r.plan("Z")["kernel"] == "contract_alu"
        r.run()
        torch.cuda.synchronize()
        return to_host(r.output("Z")).as_f64()
    finally:
        r.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spec,m,n,k", SHAPES)
def test_squared_differences_match_oracle(spec, m, n, k, dtype):
    print(f"squared differences {spec} {m} x {k} x {n} {dtype}", flush=True)
    x, y = _operands(spec, m, n, k, dtype, False)
    w = single_vertex(spec, x, y, "f32", otimes="sqdiff", parts={"d": {}})
    bad, worst = violations(_run(w, x, y), run_graph(w, {"X": x, "Y": y})["Z"].as_f64(), RTOL_F32)
    assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spec,m,n,k", SHAPES)
def test_largest_absolute_difference_is_exact_and_passes_over_nan(spec, m, n, k, dtype):
    print(f"largest absolute difference {spec} {m} x {k} x {n} {dtype}", flush=True)
    x, y = _operands(spec, m, n, k, dtype, m * n <= 65536)
    w = single_vertex(spec, x, y, "f32", otimes="absdiff", oplus="max", parts={"d": {}})
    got = _run(w, x, y)
    lx, ly = spec.split("->")[0].split(",")
    a = x.as_f64().astype(np.float32) if lx == "ij" else x.as_f64().astype(np.float32).T
    b = y.as_f64().astype(np.float32) if ly == "jk" else y.as_f64().astype(np.float32).T
    rows = range(m) if m * n <= 65536 else (0, 1, 127, 128, 1500, m - 1)
    for i in rows:
        want = np.fmax.reduce(np.abs(a[i][:, None] - b), axis=0, initial=-np.inf)
        assert np.array_equal(got[i].astype(np.float32), want), (i, got[i], want)
