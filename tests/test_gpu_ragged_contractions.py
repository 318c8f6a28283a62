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
