"""Contractions whose kernel adds the sums of the blocks along the aggregated labels itself (Section 4.3's two stages in one
launch): with two stages in LDS the sums are those of the partial slabs in the same order, so the result must equal theirs bit for
bit; with four stages two groups of waves share a tile's reduction and the oracle decides.  Ragged tile edges, odd numbers of
stages per block, several aggregated labels, batch labels, every operand layout, slices that start inside a 128-byte line."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, kernel_names, same_values, single_vertex, violations
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu

JOIN, SLABS = [("join", "contract_mfma")], [("join", "contract_mfma"), ("aggregate", "none")]
# spec, bound X, bound Y, partitioning, operand dtype, result dtype, alpha, waves (4: the two-stage kernel)
CASES = [
    ("ij,jk->ik", (1000, 264), (264, 1032), {"j": 3}, "bf16", "f32", 1.0, 0),              # blocks of a stage and a half, ragged edges
    ("ij,kj->ik", (1032, 320), (1000, 320), {"j": 5, "i": 2}, "bf16", "bf16", -0.3, 4),      # rows cut as well
    ("ji,jk->ik", (320, 1032), (320, 1000), {"j": 4}, "bf16", "f32", 1.0, 4),
    ("ji,kj->ik", (640, 1032), (1000, 640), {"j": 2}, "bf16", "bf16", 1.0, 4),
    ("ij,jk->ki", (1000, 384), (384, 1032), {"j": 2}, "bf16", "f32", 1.0, 4),              # the operands change places
    ("bshd,ahd->bsa", (2, 520, 4, 64), (520, 4, 64), {"h": 4, "d": 2}, "bf16", "f32", 1.0, 4),   # two aggregated labels
    ("bij,bjk->bik", (3, 520, 192), (3, 192, 520), {"j": 3, "b": 3}, "bf16", "f32", 1.0, 4),     # a batch label, cut
    ("ij,jk->ik", (768, 1216), (1216, 768), {"j": 2}, "bf16", "f32", 1.0, 4),              # slices of 9.5 stages, every other one inside a line
    ("ij,jk->ik", (2312, 192), (192, 2056), {"j": 2}, "bf16", "bf16", 1.0, 0),             # more tiles than compute units
    ("ij,jk->ik", (1288, 96), (96, 776), {"j": 3}, "f32", "f32", 1.0, 0),
    ("ij,jk->ik", (1032, 1024), (1024, 1000), {"j": 2}, "bf16", "bf16", 0.5, 0),           # four stages from here on
    ("ij,kj->ik", (768, 1216), (768, 1216), {"j": 2}, "bf16", "f32", 1.0, 0),
    ("ji,jk->ik", (576, 1032), (576, 1000), {"j": 8}, "bf16", "f32", -2.0, 0),             # 16 stages, two a block, the second an eighth full
    ("ji,kj->ik", (1720, 1032), (1000, 1720), {"j": 5}, "bf16", "f32", 1.0, 0),            # blocks of 344: 30 stages
]
# four stages without blocks: M, N, K per layout, stage counts from 8 to 11 and runs of two contracted labels
PLAIN = [("ij,jk->ik", (264, 512), (512, 392)), ("ij,kj->ik", (392, 576), (264, 576)), ("ji,jk->ik", (608, 136), (608, 128)), ("ji,kj->ik", (704, 392), (392, 704)),
         ("bshd,ahd->bsa", (2, 72, 3, 192), (136, 3, 192)), ("bij,bjk->bik", (5, 200, 552), (5, 552, 136))]


def _run(w, x, y, tiled, waves, out=None):
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device
    r = GraphRunner(w, "d", contract=dict(kernel="dma", waves=waves), tiled_partials=tiled)
    try:
        r.bind({"X": to_device(x), "Y": to_device(y)}, outputs=out)
        E.tr_profile_enable(r.g, 8)
        r.run()
        torch.cuda.synchronize()
        return r.output("Z").clone(), [(q["stage"], q["kernel"]) for q in E.tr_profile_read(r.g)]
    finally:
        r.close()


def _operands(bx, by, dtype):
    return [HostTensor.from_f32(uniform_pm1(53, i, int(np.prod(b))).reshape(b), dtype) for i, b in enumerate((bx, by))]


@pytest.mark.parametrize("spec,bx,by,part,in_dtype,out_dtype,alpha,waves", CASES)
def test_totals_kept_in_the_kernel(spec, bx, by, part, in_dtype, out_dtype, alpha, waves):
    import torch
    from paper_2410_02682_amd.runner import to_host
    print(f"totals {spec} X{bx} Y{by} d {part} {in_dtype}->{out_dtype} waves {waves}", flush=True)
    x, y = _operands(bx, by, in_dtype)
    w = single_vertex(spec, x, y, out_dtype, alpha=alpha, parts={"d": part})
    totals, launches = _run(w, x, y, True, waves)
    assert launches == JOIN, launches
    slabs, launches = _run(w, x, y, False, waves)
    assert launches == SLABS, launches
    contracted = int(np.prod([n for l, n in zip(spec.split(",")[0], bx) if l not in spec.split("->")[1]]))
    tiles = int(np.prod([-(-n // 128) for n in totals.shape[-2:]])) * int(np.prod(totals.shape[:-2]))
    if waves == 4 or in_dtype == "f32" or contracted < 512 or tiles > 256:
        kind = torch.int16 if out_dtype == "bf16" else torch.int32
        assert torch.equal(totals.view(kind), slabs.view(kind))
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    bad, worst = violations(to_host(totals).as_f64(), ref, RTOL_BF16 if out_dtype == "bf16" else RTOL_F32)
    assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"


@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spec,bx,by", PLAIN)
def test_four_stages_match_oracle(spec, bx, by, out_dtype):
    from paper_2410_02682_amd.runner import to_host
    print(f"four stages {spec} X{bx} Y{by} -> {out_dtype}", flush=True)
    x, y = _operands(bx, by, "bf16")
    w = single_vertex(spec, x, y, out_dtype, alpha=0.7, parts={"d": {}})
    got, launches = _run(w, x, y, True, 0)
    assert launches == JOIN, launches
    bad, worst = violations(to_host(got).as_f64(), run_graph(w, {"X": x, "Y": y})["Z"].as_f64(), RTOL_BF16 if out_dtype == "bf16" else RTOL_F32)
    assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"


def test_totals_into_a_strided_destination():
    import torch
    x, y = _operands((1000, 256), (256, 1032), "bf16")
    w = single_vertex("ij,jk->ik", x, y, "f32", parts={"d": {"j": 4}})
    outs = []
    for tiled in (True, False):
        big = torch.full((1010, 1100), 7.0, dtype=torch.float32, device="cuda")
        z, launches = _run(w, x, y, tiled, 0, out={"Z": big[5:1005, 36:1068]})
        assert launches == (JOIN if tiled else SLABS), launches
        big[5:1005, 36:1068] = 7.0
        assert bool((big == 7.0).all())
        outs.append(z)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("spec,bx,by,cut,out_dtype,totals", [
    ("ij,jk->ik", (2632, 2048), (2048, 144), 16, "f32", False),              # 42 tiles: slabs 22.8 us, totals 32.0
    ("ji,kj->ik", (4608, 1504), (952, 4608), 3, "bf16", False),              # 96 tiles: 29.9 and 39.5
    ("ij,jk->ik", (696, 1280), (1280, 648), 4, "bf16", False),               # 36 tiles: 13.8 and 17.7
    ("ij,jk->ik", (1072, 2048), (2048, 2968), 16, "bf16", True),             # 216 tiles: 85 and 37
    ("ij,jk->ik", (2168, 512), (512, 728), 2, "bf16", True),                 # 102 tiles: 17.5 and 12.0
])
def test_totals_only_where_they_are_faster_than_slabs(spec, bx, by, cut, out_dtype, totals):
    print(f"totals or slabs {spec} X{bx} Y{by} j cut {cut}", flush=True)
    assert _stages(spec, bx, by, cut, "bf16", out_dtype) == (["join"] if totals else ["join", "aggregate"])


def _stages(spec, bx, by, cut, in_dtype, out_dtype):
    """The launches of one vertex as the library routes it; operands of zeros."""
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import TORCH_DTYPE, GraphRunner
    w = single_vertex(spec, HostTensor(np.zeros(bx, np.uint16 if in_dtype == "bf16" else np.float32), in_dtype),
                      HostTensor(np.zeros(by, np.uint16 if in_dtype == "bf16" else np.float32), in_dtype), out_dtype, parts={"d": {"j": cut}})
    r = GraphRunner(w, "d")
    try:
        r.bind({n: torch.zeros(b, dtype=TORCH_DTYPE[in_dtype], device="cuda") for n, b in (("X", bx), ("Y", by))})
        E.tr_profile_enable(r.g, 8)
        r.run()
        torch.cuda.synchronize()
        return [q["stage"] for q in E.tr_profile_read(r.g)]
    finally:
        r.close()


@pytest.mark.parametrize("spec,bx,by,part,stages", [c + ({}, 4) for c in PLAIN] + [(c[0], c[1], c[2], c[3], 2 if c[7] == 4 or i < 10 else 4) for i, c in enumerate(CASES)] + [
    ("ij,jk->ik", (264, 504), (504, 392), {}, 2),                            # reductions under 512 keep two
])
def test_number_of_stages(spec, bx, by, part, stages):
    """k_contract_dma<tile rows, tile columns, bytes of k, stages, ...>: that the cases above reach the kernel they are about."""
    import torch
    from paper_2410_02682_amd.runner import GraphRunner
    case = next((c for c in CASES if (c[0], c[1], c[2], c[3]) == (spec, bx, by, part)), None)
    dt = case[4] if case else "bf16"
    t = torch.float32 if dt == "f32" else torch.bfloat16
    w = single_vertex(spec, *(HostTensor(np.zeros(b, np.float32 if dt == "f32" else np.uint16), dt) for b in (bx, by)), "f32", parts={"d": part})
    r = GraphRunner(w, "d", contract=dict(kernel="dma", waves=case[7] if case else 0))
    try:
        r.bind({n: torch.zeros(b, dtype=t, device="cuda") for n, b in (("X", bx), ("Y", by))})
        names = kernel_names(r.run)
        assert len(names) == 1 and f"k_contract_dma<128, 128, 128, {stages}," in names[0], names
    finally:
        r.close()


@pytest.mark.parametrize("part", [{}, {"j": 2}])
@pytest.mark.parametrize("spec", ["ij,jk->ik", "ij,kj->ik"])
def test_infinities_and_nan_with_four_stages(spec, part):
    """Zeros behind the last stage and the exchange between the two groups of waves leave other rows and columns alone."""
    import torch
    from paper_2410_02682_amd.runner import GraphRunner
    gen = torch.Generator().manual_seed(7)
    bx, by = (392, 1096), (1096, 264) if spec == "ij,jk->ik" else (264, 1096)
    x, y = (torch.empty(b).uniform_(0.5, 1.0, generator=gen).bfloat16() for b in (bx, by))
    yt = y if spec == "ij,jk->ik" else y.t()
    yt[0, 7], yt[1095, 130], yt[600, 263] = float("inf"), float("nan"), float("-inf")
    x[5, 1000], x[391, 17], x[64, 3] = float("-inf"), float("nan"), 0.0
    yt[3, 100] = float("inf")
    ref = x.double() @ yt.double()
    w = single_vertex(spec, HostTensor(np.zeros(bx, np.uint16), "bf16"), HostTensor(np.zeros(by, np.uint16), "bf16"), "f32", parts={"d": part})
    r = GraphRunner(w, "d", contract=dict(kernel="dma"), tiled_partials=True)
    try:
        r.bind({"X": x.cuda(), "Y": y.cuda()})
        names = kernel_names(r.run)
        if not part:
            assert "k_contract_dma<128, 128, 128, 4," in names[0], names
        assert same_values(r.output("Z").cpu().numpy(), ref.numpy(), RTOL_F32)
    finally:
        r.close()
