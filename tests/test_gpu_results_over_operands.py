"""Cut contractions whose result is bound over one of their own operands.  Every block's sums go to the workspace first and the result is
written when all blocks have been multiplied, so such calls are well defined; the forms that write the result while other
workgroups still read the operands (totals in the kernel, sums that wait for a second block, few rows in one piece) must
stand back.  Bit for bit what the slabs give into memory of their own."""
import numpy as np
import pytest

from tests._parity import single_vertex
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu


def _run(w, x, y, tiled, over=None):
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device

    r = GraphRunner(w, "d", tiled_partials=tiled)
    try:
        dev = {"X": to_device(x), "Y": to_device(y)}
        r.bind(dev, outputs={"Z": dev[over]} if over else None)
        E.tr_profile_enable(r.g, 8)
        r.run()
        torch.cuda.synchronize()
        return r.output("Z").clone(), [q["stage"] for q in E.tr_profile_read(r.g)]
    finally:
        r.close()


@pytest.mark.parametrize("spec,bx,by,cut,dt,over", [
    ("ij,jk->ik", (1024, 1024), (1024, 1024), 4, "bf16", "X"),                # totals kept by the kernel otherwise
    ("ij,jk->ik", (1024, 1024), (1024, 1024), 4, "f32", "Y"),
    ("ij,jk->ik", (4096, 4096), (4096, 4096), 2, "bf16", "X"),                # the first block's sums wait for the second's
    ("ij,jk->ik", (1035, 1035), (1035, 1035), 3, "bf16", "X"),                # ragged
    ("ij,jk->ik", (8, 10240), (10240, 10240), 4, "bf16", "X"),                # few rows, one piece
    ("ij,jk->ik", (8, 4096), (4096, 4096), 8, "bf16", "X"),                   # four
])
def test_result_over_an_operand(spec, bx, by, cut, dt, over):
    import torch
    print(f"{spec} X{bx} Y{by} j cut {cut} {dt}, Z over {over}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(89, p, int(np.prod(b))).reshape(b), dt) for p, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, dt, parts={"d": {"j": cut}})
    ref, _ = _run(w, x, y, False)
    got, launches = _run(w, x, y, True, over)
    assert launches == ["join", "aggregate"], launches
    assert torch.equal(got, ref)
