"""Contractions of a few rows with a large matrix (k_contract_rows): row counts up to 16 and the first beyond, columns that are
no whole strip, contracted labels that are no whole iteration and leave waves or pieces without work, both layouts of the
matrix, cuts of every label, results in either dtype.  Against the oracle, with operands inside tensors of NaN."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, single_vertex, violations
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu

CASES = [
    ("ij,jk->ik", (2, 256), (256, 64), {}, "f32", 1.0),
    ("ij,jk->ik", (3, 264), (264, 72), {}, "bf16", 1.0),                    # a strip and eight columns; a wave with eight k, six without any
    ("ij,jk->ik", (16, 1000), (1000, 520), {"j": 5}, "f32", -0.5),          # five slabs
    ("ij,jk->ik", (8, 4104), (4104, 1032), {}, "bf16", 1.0),                # cut by the execution
    ("ij,jk->ik", (8, 4096), (4096, 4096), {"k": 8}, "bf16", 1.0),
    ("ij,jk->ik", (5, 2752), (2752, 33000), {"j": 2}, "f32", 1.0),          # many strips: eight columns a lane
    ("ij,jk->ik", (17, 512), (512, 256), {}, "f32", 1.0),                   # one row too many
    ("ij,kj->ik", (2, 256), (64, 256), {}, "f32", 1.0),
    ("ij,kj->ik", (16, 2312), (1000, 2312), {}, "bf16", 2.0),               # 62 strips and a half
    ("ij,kj->ik", (9, 4096), (520, 4096), {"j": 16}, "f32", 1.0),           # 16 slabs: two pieces at least
    ("ba,ahd->bhd", (4, 1024), (1024, 8, 64), {"h": 8}, "bf16", 1.0),
    ("bhd,ahd->ba", (8, 8, 128), (1024, 8, 128), {"h": 8}, "bf16", 1.0),
    ("bhd,ahd->ba", (3, 16, 64), (264, 16, 64), {"h": 2, "a": 3}, "f32", 1.0),
]


@pytest.mark.parametrize("spec,bx,by,part,out_dtype,alpha", CASES)
def test_few_rows_match_oracle(spec, bx, by, part, out_dtype, alpha):
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    print(f"few rows {spec} X{bx} Y{by} d {part} -> {out_dtype}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(59, i, int(np.prod(b))).reshape(b), "bf16") for i, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, out_dtype, alpha=alpha, parts={"d": part})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    rtol = RTOL_BF16 if out_dtype == "bf16" else RTOL_F32

    def padded(t):                                                           # the same values inside a tensor of NaN, rows 16 bytes apart
        t = to_device(t)
        big = torch.full((t.shape[0] + 2,) + tuple(t.shape[1:-1]) + (t.shape[-1] + 16,), float("nan"), dtype=t.dtype, device="cuda")
        view = big[1:-1, ..., 8:-8]
        view.copy_(t)
        return view

    for dense in (True, False):
        r = GraphRunner(w, "d")
        try:
            big = torch.full((ref.shape[0] + 2,) + ref.shape[1:-1] + (ref.shape[-1] + 16,), 7.0, dtype=torch.float32 if out_dtype == "f32" else torch.bfloat16, device="cuda")
            r.bind({"X": to_device(x), "Y": to_device(y)} if dense else {"X": padded(x), "Y": padded(y)}, outputs=None if dense else {"Z": big[1:-1, ..., 8:-8]})
            r.run()
            torch.cuda.synchronize()
            bad, worst = violations(to_host(r.output("Z")).as_f64(), ref, rtol)
            assert bad == 0, f"dense {dense}: {bad} elements out of tolerance (worst {worst:.2f}x)"
            if not dense:
                big[1:-1, ..., 8:-8] = 7.0
                assert bool((big == 7.0).all())
        finally:
            r.close()


@pytest.mark.parametrize("spec,bx,by,cut,most", [
    ("ij,jk->ik", (16, 1000), (1000, 520), 5, 3),                            # a piece is 256 of the contracted label at least
    ("ij,kj->ik", (9, 4096), (520, 4096), 16, 15),
    ("ij,jk->ik", (8, 1024), (1024, 16384), 4, 1),                           # 256 strips of 64: no aggregation
])
def test_pieces_replace_the_blocks_unless_the_slabs_are_asked_for(spec, bx, by, cut, most):
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    print(f"few rows, switch {spec} X{bx} Y{by} j cut {cut}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(61, i, int(np.prod(b))).reshape(b), "bf16") for i, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, "f32", parts={"d": {"j": cut}})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    for tiled in (True, False):
        r = GraphRunner(w, "d", tiled_partials=tiled)
        try:
            r.bind({"X": to_device(x), "Y": to_device(y)})
            E.tr_profile_enable(r.g, 8)
            r.run()
            torch.cuda.synchronize()
            launches = [(q["stage"], q["slabs"]) for q in E.tr_profile_read(r.g)]
            slabs = max(launches[0][1], 1)
            assert launches == ([("join", slabs), ("aggregate", slabs)] if slabs > 1 else [("join", 0)])
            assert -(-cut // 8) <= slabs <= most if tiled else slabs == cut, launches
            bad, worst = violations(to_host(r.output("Z")).as_f64(), ref, RTOL_F32)
            assert bad == 0, f"tiled {tiled}: {bad} elements out of tolerance (worst {worst:.2f}x)"
        finally:
            r.close()
