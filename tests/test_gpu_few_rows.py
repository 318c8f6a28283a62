"""Contractions of a few rows with a large matrix (k_contract_rows): row counts up to 16 and the first beyond, columns that are
no whole strip, contracted labels that are no whole iteration and leave waves or pieces without work, both layouts of the
matrix, cuts of every label, results in either dtype.  Against the oracle, with operands inside tensors of NaN."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, kernel_names, same_values, single_vertex, violations
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


def _zeros(spec, bx, by, part, out_dtype):
    import torch
    from paper_2410_02682_amd.runner import GraphRunner
    x, y = (HostTensor(np.zeros(b, np.uint16), "bf16") for b in (bx, by))
    r = GraphRunner(single_vertex(spec, x, y, out_dtype, parts={"d": part}), "d")
    r.bind({n: torch.zeros(b, dtype=torch.bfloat16, device="cuda") for n, b in (("X", bx), ("Y", by))})
    return r


@pytest.mark.parametrize("spec,bx,by,part,out_dtype,rows", [c[:5] + (c[1][0] <= 16,) for c in CASES] + [
    ("ij,kj->ik", (8, 4096), (10240, 4096), {}, "bf16", True),
    ("ij,kj->ik", (9, 4096), (10240, 4096), {}, "bf16", False),              # a large matrix along k under more than eight rows
    ("ij,kj->ik", (9, 4104), (10240, 4104), {}, "bf16", True),               # whose rows are no whole 128-byte lines
    ("ij,kj->ik", (5, 8192), (10240, 8192), {}, "bf16", False),
    ("ij,kj->ik", (4, 8192), (10240, 8192), {}, "bf16", True),
])
def test_which_products_run_on_the_few_row_kernel(spec, bx, by, part, out_dtype, rows):
    r = _zeros(spec, bx, by, part, out_dtype)
    try:
        names = kernel_names(r.run)
        assert any("k_contract_rows" in n for n in names) == rows, names
    finally:
        r.close()


@pytest.mark.parametrize("spec,bx,by", [("ij,jk->ik", (3, 520), (520, 200)), ("ij,jk->ik", (5, 264), (264, 33000)), ("ij,kj->ik", (7, 520), (200, 520))])
def test_infinities_and_nan_stay_where_they_belong(spec, bx, by):
    """The rows up to 16 and the elements behind the last k that the kernel adds are zeros, and no other column is touched."""
    import torch
    from paper_2410_02682_amd.runner import GraphRunner
    gen = torch.Generator().manual_seed(5)
    x, y = (torch.empty(b).uniform_(0.5, 1.0, generator=gen).bfloat16() for b in (bx, by))
    yt = y if spec == "ij,jk->ik" else y.t()
    yt[0, 7], yt[-1, 8], yt[300 % yt.shape[0], 190] = float("inf"), float("nan"), float("-inf")
    x[1, 100] = float("inf")
    x[2, 3] = 0.0
    yt[3, 100] = float("inf")                                                # 0 times an infinity
    ref = x.double() @ yt.double()
    w = single_vertex(spec, HostTensor(np.zeros(bx, np.uint16), "bf16"), HostTensor(np.zeros(by, np.uint16), "bf16"), "f32", parts={"d": {}})
    r = GraphRunner(w, "d")
    try:
        r.bind({"X": x.cuda(), "Y": y.cuda()})
        names = kernel_names(r.run)
        assert any("k_contract_rows" in n for n in names), names
        assert same_values(r.output("Z").cpu().numpy(), ref.numpy(), RTOL_F32)
    finally:
        r.close()
