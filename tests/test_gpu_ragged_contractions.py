"""Contractions whose blocks are no whole 16-byte vectors (Section 4.3 of the paper puts no condition on a block's extents):
odd extents and row pitches, blocks that start anywhere, against the oracle."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, single_vertex, violations
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu


def _inputs(bx, by, dtype):
    x = HostTensor.from_f32(uniform_pm1(71, 0, int(np.prod(bx))).reshape(bx), dtype)
    y = HostTensor.from_f32(uniform_pm1(71, 1, int(np.prod(by))).reshape(by), dtype)
    return x, y


def test_merged_aggregation_takes_a_pitch_that_leaves_no_contraction_kernel():
    """1000 rows cut eight ways are blocks of 125: the aggregation of such blocks is not merged, so a row pitch that keeps the
    vertex off the 16-byte kernels is accepted with tr_set_fused_aggregation on, as it is with it off."""
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    x, y = _inputs((256, 1000), (256, 128), "bf16")
    w = single_vertex("ji,jk->ik", x, y, "f32", parts={"d": {"i": 8, "j": 2}})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    wide = torch.zeros((256, 1001), dtype=torch.bfloat16, device="cuda")
    wide[:, :1000].copy_(to_device(x))
    r = GraphRunner(w, "d")
    try:
        E.tr_set_fused_aggregation(r.g, True)
        r.bind({"X": wide[:, :1000], "Y": to_device(y)})
        r.run()
        torch.cuda.synchronize()
        got = to_host(r.output("Z")).as_f64()
    finally:
        r.close()
    assert violations(got, ref, RTOL_F32)[0] == 0


# spec, bounds of X and Y, dtypes of operands and result, cuts, kernel.  Extents around the tiles (64, 128) and the depth of a stage
# (64 bf16, 32 fp32), odd pitches, every layout of the two operands, runs that end inside a vector, blocks that start anywhere.
RAGGED = [
    ("ij,jk->ik", (65, 63), (63, 127), "bf16", "bf16", {}),
    ("ij,jk->ik", (129, 131), (131, 65), "bf16", "f32", {"i": 3}),
    ("ij,kj->ik", (257, 67), (129, 67), "bf16", "bf16", {}),
    ("ij,kj->ik", (127, 201), (63, 201), "bf16", "f32", {"j": 3}),
    ("ji,jk->ik", (33, 77), (33, 91), "bf16", "f32", {"i": 7, "k": 7}),
    ("ji,kj->ik", (85, 71), (83, 85), "bf16", "bf16", {"j": 5}),
    ("ij,jk->ki", (71, 19), (19, 101), "bf16", "f32", {}),
    ("ij,jk->ik", (2049, 130), (130, 2047), "bf16", "bf16", {}),             # 128 x 128 tiles
    ("ij,jk->ik", (67, 33), (33, 65), "f32", "f32", {}),
    ("ji,jk->ik", (131, 63), (131, 129), "f32", "f32", {"i": 9, "k": 3}),
    ("ij,kj->ik", (65, 129), (97, 129), "f32", "bf16", {"j": 3}),
    ("bhst,bthd->bshd", (2, 3, 131, 37), (2, 37, 3, 8), "bf16", "bf16", {"h": 3}),
    ("bshd,bthd->bhst", (2, 67, 3, 16), (2, 45, 3, 16), "bf16", "bf16", {"s": 1}),
    ("iab,abk->ik", (65, 5, 17), (5, 17, 67), "bf16", "f32", {"a": 5}),       # two contracted labels, an odd run
    ("aib,kab->ik", (5, 65, 13), (67, 5, 13), "bf16", "bf16", {}),            # runs of 13 that do not join: vectors cross them
    ("iaj,jbk->iabk", (19, 7, 33), (33, 5, 11), "f32", "f32", {}),
]


# Other scalar functions take the tiles from 64 of 128 x 128 on: fewer stay on one output per lane.
RAGGED_ALU = [
    ("ij,jk->ik", (1025, 33), (33, 901), "f32", "f32", "contract_alu"),
    ("ij,kj->ik", (900, 65), (1027, 65), "bf16", "f32", "contract_alu"),
    ("ji,jk->ik", (67, 1025), (67, 903), "bf16", "bf16", "contract_alu"),
    ("aib,kab->ik", (3, 1021, 11), (901, 3, 11), "f32", "f32", "contract_alu"),
    ("ij,jk->ik", (250, 33), (33, 129), "f32", "f32", "generic"),
]


def _check(spec, bx, by, dt, out, cut, otimes, oplus, kernel):
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    x, y = _inputs(bx, by, dt)
    w = single_vertex(spec, x, y, out, otimes, oplus, 1.0, parts={"d": cut})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    r = GraphRunner(w, "d")
    try:
        r.bind({"X": to_device(x), "Y": to_device(y)})
        assert r.plan("Z")["kernel"] == kernel
        r.run()
        torch.cuda.synchronize()
        got = to_host(r.output("Z")).as_f64()
    finally:
        r.close()
    # the common bounds of fp32 and bf16 results; K <= 201 terms of order one, summed to 2^-23 of their absolute values' sum,
    # stay below 201 * 2^-23 = 2.4e-5 of a term, 2e-6 of a result's root mean square
    assert violations(got, ref, RTOL_F32 if out == "f32" else RTOL_BF16)[0] == 0


@pytest.mark.parametrize("spec,bx,by,dt,out,cut", RAGGED)
def test_ragged_products_match_the_oracle(spec, bx, by, dt, out, cut):
    _check(spec, bx, by, dt, out, cut, "mul", "sum", "contract_mfma")


@pytest.mark.parametrize("otimes,oplus", [("sqdiff", "sum"), ("absdiff", "max"), ("absdiff", "sum")])
@pytest.mark.parametrize("spec,bx,by,dt,out,kernel", RAGGED_ALU)
def test_ragged_distances_match_the_oracle(spec, bx, by, dt, out, kernel, otimes, oplus):
    _check(spec, bx, by, dt, out, {}, otimes, oplus, kernel)


def test_operands_that_start_on_an_odd_element():
    """The last element read is the last one of the buffer, the first one lies two bytes into it."""
    import torch
    import paper_2410_02682_amd as E  # noqa: F401
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    x, y = _inputs((130, 96), (96, 136), "bf16")
    w = single_vertex("ij,jk->ik", x, y, "bf16", parts={"d": {"i": 2}})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    base = torch.zeros(130 * 96 + 1, dtype=torch.bfloat16, device="cuda")
    view = base[1:].view(130, 96)
    view.copy_(to_device(x))
    r = GraphRunner(w, "d")
    try:
        r.bind({"X": view, "Y": to_device(y)})
        r.run()
        torch.cuda.synchronize()
        got = to_host(r.output("Z")).as_f64()
    finally:
        r.close()
    assert violations(got, ref, RTOL_BF16)[0] == 0
