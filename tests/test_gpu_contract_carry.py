"""Contractions whose 256 x 256 tiles walk over two blocks of an aggregated label, the first one's sums waiting in memory: one launch,
bit for bit what partial slabs and their aggregation give (the same sums in the same order), in every layout, with partial last
stages, odd and even stage counts and tiles that do not divide among the workgroups."""
import numpy as np
import pytest

from tests._parity import kernel_names, single_vertex
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu


def _run(w, x, y, tiled, pad=0, out=None):
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device

    r = GraphRunner(w, "d", tiled_partials=tiled)
    try:
        dev = {"X": to_device(x), "Y": to_device(y)}
        for n, t in dev.items() if pad else ():          # rows that start so many elements inside a 128-byte line
            big = torch.full((t.shape[0], t.shape[1] + 64), float("nan"), dtype=t.dtype, device="cuda")
            dev[n] = big[:, pad:pad + t.shape[1]]
            dev[n].copy_(t)
        r.bind(dev, outputs=None if out is None else {"Z": out})
        E.tr_profile_enable(r.g, 8)
        for _ in range(2):                            # the second pass meets the totals the first one left behind
            r.run()
        torch.cuda.synchronize()
        n = [q["stage"] for q in E.tr_profile_read(r.g)]
        return r.output("Z").clone(), n[:len(n) // 2]
    finally:
        r.close()


@pytest.mark.parametrize("spec,bx,by,part,odt", [
    ("ij,jk->ik", (4096, 2 * 2048), (2 * 2048, 4096), {"j": 2}, "bf16"),
    ("ij,kj->ik", (4096, 2 * 2056), (4096, 2 * 2056), {"j": 2}, "f32"),           # 33 stages, the last one of 8
    ("ji,jk->ik", (2 * 2048, 4096), (2 * 2048, 7168), {"j": 2}, "f32"),           # 448 tiles on 256 compute units
    ("ji,kj->ik", (2 * 2120, 4096), (8192, 2 * 2120), {"j": 2}, "f32"),
    ("bij,bjk->bik", (2, 2048, 2 * 2048), (2, 2 * 2048, 4096), {"j": 2, "b": 2}, "bf16"),
    ("ijl,jlk->ik", (4096, 4, 1024), (4, 1024, 8192), {"j": 2, "i": 2}, "bf16"),  # blocks of two joined labels
])
def test_same_bits_as_partial_slabs(spec, bx, by, part, odt):
    import torch
    print(f"carried totals {spec} X{bx} Y{by} d {part} -> {odt}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(83, p, int(np.prod(b))).reshape(b), "bf16") for p, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, odt, alpha=-0.7, parts={"d": part})
    got, launches = _run(w, x, y, True)
    ref, slabs = _run(w, x, y, False)
    assert launches == ["join"] and slabs == ["join", "aggregate"], (launches, slabs)
    assert torch.equal(got, ref)


@pytest.mark.parametrize("spec,by,pad,zpad", [
    ("ij,jk->ik", (2 * 2072, 4096), 0, 40),              # rows of Z further apart; every other block of X starts 16 bytes inside a line
    ("ij,kj->ik", (4096, 2 * 2072), 8, 0),               # and its rows as well
    ("ij,kj->ik", (4096, 2 * 2072), 24, 13),             # rows of Z that are no whole vectors apart: stored one by one
])
def test_strided_results_and_slices_inside_a_line(spec, by, pad, zpad):
    import torch
    print(f"carried totals {spec} pad {pad}, result {zpad}", flush=True)
    bx = (4096, 2 * 2072)
    x, y = (HostTensor.from_f32(uniform_pm1(101, p, int(np.prod(b))).reshape(b), "bf16") for p, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, "f32", alpha=0.5, parts={"d": {"j": 2}})
    outs = []
    for tiled in (True, False):
        big = torch.full((4096, 4096 + zpad), 7.0, dtype=torch.float32, device="cuda")
        z, launches = _run(w, x, y, tiled, pad, big[:, :4096])
        assert launches == (["join"] if tiled else ["join", "aggregate"]), launches
        big[:, :4096] = 7.0
        assert bool((big == 7.0).all())
        outs.append(z)
    assert torch.equal(outs[0], outs[1])
    names = kernel_names(lambda: _run(w, x, y, True, pad))
    assert sum("k_contract_dma<256, 256, 128, 2, 2, 8," in n and ", 2>" in n for n in names) == 2, names
