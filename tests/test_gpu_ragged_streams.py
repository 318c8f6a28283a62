"""Ragged products whose operands are one run each (k_contract_ragged): contracted labels around half a stage, a stage and the depth
of the prefetch, rows and columns around a chunk and a tile in every layout, operands inside tensors of NaN, and blocks along the
contracted label that one workgroup walks over (no aggregation launch; totals in 64 bits over all of them)."""
import numpy as np
import pytest

from tests._parity import RTOL_BF16, RTOL_F32, kernel_names, single_vertex, violations
from tests.test_gpu_contract_totals import _stages
from oracle.graph_ref import run_graph
from synth_inputs.prng import HostTensor, uniform_pm1

pytestmark = pytest.mark.gpu

LAYOUTS = ["ij,jk->ik", "ij,kj->ik", "ji,jk->ik", "ji,kj->ik"]
TYPES = [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32")]
# rows, columns, contracted
SIZES = [(65, 63, 17), (77, 129, 33), (9, 513, 63), (130, 67, 65), (64, 67, 97), (201, 73, 127), (67, 64, 129), (71, 61, 257), (65, 129, 515)]


def _run(w, x, y, pad=False, tiled=None, out=None):
    import torch
    import paper_2410_02682_amd as E
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host

    def bound(t):
        t = to_device(t)
        if not pad:
            return t
        big = torch.full(tuple(t.shape[:-1]) + (t.shape[-1] + 5,), float("nan"), dtype=t.dtype, device="cuda")
        view = big[..., 3:-2]
        view.copy_(t)
        return view

    r = GraphRunner(w, "d", tiled_partials=tiled)
    try:
        r.bind({"X": bound(x), "Y": bound(y)}, outputs=None if out is None else {"Z": out})
        kernel = r.plan("Z")["kernel"]
        E.tr_profile_enable(r.g, 8)
        r.run()
        torch.cuda.synchronize()
        return to_host(r.output("Z")).as_f64(), kernel, [q["stage"] for q in E.tr_profile_read(r.g)]
    finally:
        r.close()


@pytest.mark.parametrize("dt,odt", TYPES)
@pytest.mark.parametrize("spec", LAYOUTS)
@pytest.mark.parametrize("m,n,k", SIZES)
def test_edges_of_stages_and_tiles(m, n, k, spec, dt, odt):
    print(f"ragged {spec} {m} x {k} x {n} {dt}->{odt}", flush=True)
    ext = {"i": m, "j": k, "k": n}
    x, y = (HostTensor.from_f32(uniform_pm1(67, p, int(np.prod(b))).reshape(b), dt) for p, b in enumerate(tuple(ext[l] for l in o) for o in spec.split("->")[0].split(",")))
    w = single_vertex(spec, x, y, odt, alpha=-1.5, parts={"d": {}})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    for pad in (False, True):
        got, _, _ = _run(w, x, y, pad)
        bad, worst = violations(got, ref, RTOL_BF16 if odt == "bf16" else RTOL_F32)
        assert bad == 0, f"padded {pad}: {bad} elements out of tolerance (worst {worst:.2f}x)"


@pytest.mark.parametrize("spec,bx,by,part,dt,odt", [
    ("ij,jk->ik", (1027, 8 * 41), (8 * 41, 1101), {"j": 8}, "bf16", "f32"),
    ("ij,kj->ik", (1027, 3 * 131), (1101, 3 * 131), {"j": 3}, "bf16", "bf16"),
    ("ji,jk->ik", (2 * 65, 1027), (2 * 65, 1101), {"j": 2}, "f32", "f32"),
    ("bij,bjk->bik", (3, 517, 5 * 27), (3, 5 * 27, 643), {"j": 5, "b": 3}, "bf16", "f32"),
    ("ijl,jlk->ik", (1027, 6, 35), (6, 35, 1101), {"j": 3}, "bf16", "f32"),                 # blocks of two joined labels
])
def test_blocks_along_the_contracted_label(spec, bx, by, part, dt, odt):
    print(f"ragged blocks {spec} X{bx} Y{by} d {part} {dt}->{odt}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(71, p, int(np.prod(b))).reshape(b), dt) for p, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, odt, parts={"d": part})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    for tiled, stages in ((True, ["join"]), (False, ["join", "aggregate"])):
        got, kernel, launches = _run(w, x, y, tiled=tiled)
        assert kernel == "contract_mfma" and launches == stages, (kernel, launches)
        bad, worst = violations(got, ref, RTOL_BF16 if odt == "bf16" else RTOL_F32)
        assert bad == 0, f"tiled {tiled}: {bad} elements out of tolerance (worst {worst:.2f}x)"


@pytest.mark.parametrize("dt,odt", TYPES)
@pytest.mark.parametrize("spec,bx,by,pad,joins", [
    ("ij,jk->ik", (1027, 3 * 41), (3 * 41, 1101), (0, 21), True),
    ("jab,jk->abk", (3 * 41, 25, 41), (3 * 41, 1101), (0, 3, 0), False),       # row labels that join in a dense result only
    ("ij,jab->iab", (1027, 3 * 41), (3 * 41, 23, 49), (0, 0, 3), False),       # column labels
])
def test_blocks_into_a_strided_result(spec, bx, by, pad, joins, dt, odt):
    import torch
    print(f"ragged blocks into a strided result {spec} X{bx} Y{by} {dt}->{odt}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(73, p, int(np.prod(b))).reshape(b), dt) for p, b in enumerate((bx, by)))
    w = single_vertex(spec, x, y, odt, parts={"d": {"j": 3}})
    ref = run_graph(w, {"X": x, "Y": y})["Z"].as_f64()
    big = torch.full([n + p for n, p in zip(ref.shape, pad)], 7.0, dtype=torch.float32 if odt == "f32" else torch.bfloat16, device="cuda")
    view = big[tuple(slice(0, n) for n in ref.shape)]
    got, kernel, launches = _run(w, x, y, out=view)
    assert kernel == "contract_mfma" and launches == (["join"] if joins else ["join", "aggregate"]), (kernel, launches)
    bad, worst = violations(got, ref, RTOL_BF16 if odt == "bf16" else RTOL_F32)
    assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"
    view.fill_(7.0)
    assert bool((big == 7.0).all())


@pytest.mark.parametrize("spec,bx,by,cut,dt,odt,totals", [
    ("ji,jk->ik", (16 * 324, 315), (16 * 324, 200), 16, "bf16", "bf16", False),       # 20 tiles: slabs 16.9 us, totals 88.9
    ("ij,kj->ik", (1871, 3 * 1335), (706, 3 * 1335), 3, "bf16", "f32", False),        # 360 tiles, two rounds: 259 and 300
    ("ij,jk->ik", (53, 8 * 20), (8 * 20, 999), 8, "bf16", "bf16", False),             # 16 tiles: 9.8 and 13.5
    ("ij,jk->ik", (2477, 8 * 81), (8 * 81, 1273), 8, "bf16", "bf16", True),           # 780 tiles: 85 and 41
    ("ij,jk->ik", (3001, 8 * 125), (8 * 125, 1530), 8, "f32", "f32", True),           # 1128 tiles: 287 and 215
])
def test_totals_only_where_they_are_faster_than_slabs(spec, bx, by, cut, dt, odt, totals):
    print(f"ragged totals or slabs {spec} X{bx} Y{by} j cut {cut} {dt}->{odt}", flush=True)
    assert _stages(spec, bx, by, cut, dt, odt) == (["join"] if totals else ["join", "aggregate"])


@pytest.mark.parametrize("dt,odt,m,n,k,streams", [
    ("bf16", "bf16", 2051, 2051, 64, False), ("bf16", "bf16", 2051, 2051, 65, True), ("bf16", "bf16", 2045, 2047, 64, True),     # 1089 tiles, 1024
    ("bf16", "f32", 1473, 1409, 112, False), ("bf16", "f32", 1473, 1409, 113, True), ("bf16", "f32", 1471, 1407, 112, True),     # 576, 506
    ("f32", "f32", 1473, 1409, 72, False), ("f32", "f32", 1473, 1409, 73, True), ("f32", "f32", 1471, 1407, 72, True),
])
def test_short_reductions_under_many_tiles(dt, odt, m, n, k, streams):
    """They take the tiles with run-by-run loads; either way the values are right."""
    import torch
    from paper_2410_02682_amd.runner import GraphRunner, to_device, to_host
    print(f"short ragged {m} x {k} x {n} {dt}->{odt}", flush=True)
    x, y = (HostTensor.from_f32(uniform_pm1(103, p, int(np.prod(b))).reshape(b), dt) for p, b in enumerate(((m, k), (k, n))))
    w = single_vertex("ij,jk->ik", x, y, odt, parts={"d": {}})
    r = GraphRunner(w, "d")
    try:
        r.bind({"X": to_device(x), "Y": to_device(y)})
        names = kernel_names(r.run)
        assert len(names) == 1 and ("k_contract_ragged" in names[0]) == streams, names
        ref = (torch.from_numpy(x.as_f64()) @ torch.from_numpy(y.as_f64())).numpy()
        bad, worst = violations(to_host(r.output("Z")).as_f64(), ref, RTOL_BF16 if odt == "bf16" else RTOL_F32)
        assert bad == 0, f"{bad} elements out of tolerance (worst {worst:.2f}x)"
    finally:
        r.close()
