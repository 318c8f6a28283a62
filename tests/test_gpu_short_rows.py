"""Reductions over short rows and in front of the outputs' innermost label (Section 3 of the paper), around the sizes at which
their kernels change: groups of four outputs and their remainders, both operand types, either operand read as one value."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, single_vertex, violations
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu

CASES = [
    ("bhd,bthd->bht", (2, 3, 128), (2, 512, 3, 128)),         # groups of four outputs behind one another
    ("bhd,bthd->bht", (2, 3, 64), (2, 403, 3, 64)),           # a remainder of three: output by output
    ("bthd->bht", (2, 260, 4, 72), None),                     # rows that do not fill their lanes
    ("ij,ij->i", (1028, 256), (1028, 256)),
    ("abcd->ab", (40, 28, 4, 24), None),                      # two reduced labels
    ("bht,bthd->bhd", (2, 3, 500), (2, 500, 3, 64)),          # one value of X for a vector of Y
    ("bthd,bht->bhd", (2, 131, 3, 64), (2, 3, 131)),          # and the other way round
    ("ij,ij->j", (333, 72), (333, 72)),
    ("ij->j", (1001, 264), None),
    ("abij->ij", (5, 7, 16, 40), None),
]


@pytest.mark.parametrize("spec,bx,by", CASES)
@pytest.mark.parametrize("dx,dy", [("bf16", "bf16"), ("f32", "f32"), ("f32", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("oplus", ["sum", "max"])
def test_short_and_column_reductions_match_the_oracle(spec, bx, by, dx, dy, oplus):
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    x = HostTensor.from_f32(uniform_pm1(83, 0, int(np.prod(bx))).reshape(bx), dx)
    y = HostTensor.from_f32(uniform_pm1(83, 1, int(np.prod(by))).reshape(by), dy) if by else None
    w = single_vertex(spec, x, y, "f32", "mul" if by else "ident", oplus)
    inp = {"X": x, "Y": y} if by else {"X": x}
    ref = run_graph(w, inp)["Z"].as_f64()
    r = GraphRunner(w, "whole")
    try:
        r.bind({k: to_device(t) for k, t in inp.items()})
        assert r.plan("Z")["kernel"] == "reduce_row"
        r.run()
        torch.cuda.synchronize()
        got = to_host(r.output("Z")).as_f64()
    finally:
        r.close()
    # sums of up to 1001 fp32 products of order one: at most 10 + 3 levels of rounding of 2^-24 of the terms' sum of magnitudes
    assert violations(got, ref, RTOL_F32)[0] == 0


@pytest.mark.parametrize("b,j", [(2, 32), (2, 33), (20971, 17), (20972, 17)])
def test_one_output_per_lane_where_parameters_are_fetched_ahead_and_where_not(b, j):
    """Up to 32 elements a lane and 524288 lanes, and the first beyond."""
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    print(f"one output per lane {b} x 5 x {j} x 5", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(97, i, int(np.prod(s))).reshape(s), "bf16") for i, s in enumerate(((b, 5, j), (b, j, 5))))
    w = single_vertex("bij,bjk->bik", x, y, "f32", parts={"d": {}})
    r = GraphRunner(w, "d")
    try:
        assert r.plan("Z")["kernel"] == "generic"
        r.bind({"X": to_device(x), "Y": to_device(y)})
        r.run()
        torch.cuda.synchronize()
        bad, worst = violations(to_host(r.output("Z")).as_f64(), run_graph(w, {"X": x, "Y": y})["Z"].as_f64(), RTOL_F32)
        assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"
    finally:
        r.close()
