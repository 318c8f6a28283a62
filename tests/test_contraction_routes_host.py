"""Which kernel a cut contraction runs on, how much workspace it takes and which calls are accepted (host code, no GPU needed)."""
import ctypes
import math

import pytest

import paper_2410_02682_amd as E


def vertex(spec, bx, by, cut, out="f32", dt="bf16", otimes="mul", oplus="sum", relu=False, merged=False):
    """(kernel, workspace bytes) of one vertex, with an element-wise vertex behind it if asked for."""
    g = E.einsum_graph_create()
    try:
        if merged:
            E.tr_set_fused_aggregation(g, True)
        x, y = E.einsum_graph_add_input(g, list(bx), dt), E.einsum_graph_add_input(g, list(by), dt)
        z = E.einsum_graph_add_einsum(g, spec, otimes, oplus, 1.0, [x, y], out)
        lhs, lz = spec.split("->")
        labels = list(dict.fromkeys(lhs.replace(",", "")))
        E.einsum_graph_set_partition(g, z, [cut.get(l, 1) for l in labels])
        last = z
        if relu:
            last = E.einsum_graph_add_einsum(g, lz + "->" + lz, "relu", "none", 1.0, [z], out)
            E.einsum_graph_set_partition(g, last, [1] * len(lz))
        E.einsum_graph_mark_output(g, last)
        return E.einsum_graph_plan(g, z)["kernel"], E.tr_workspace_bytes(g)
    finally:
        E.einsum_graph_destroy(g)


def test_blocks_of_one_row_keep_the_kernel_that_compensates():
    """The uncut product runs on 16-byte tiles with fp32 accumulation; cut into single rows it is a compensated column reduction,
    and walking the rows as one index space may not change that."""
    assert vertex("ij,jk->ik", (8, 4096), (4096, 1024), {})[0] == "contract_mfma"
    assert vertex("ij,jk->ik", (8, 4096), (4096, 1024), {"i": 8})[0] == "reduce_row"


@pytest.mark.parametrize("spec,bx,by,cut", [
    ("ji,jk->ik", (4096, 1000), (4096, 1000), {"i": 8, "k": 8}),
    ("ij,jk->ik", (1024, 4096), (4096, 1000), {"k": 8}),
])
def test_ragged_blocks_of_whole_tensors_take_no_workspace(spec, bx, by, cut):
    """Blocks of 125: no contracted label is cut, and ragged vertices are never cut further."""
    assert vertex(spec, bx, by, cut)[1] == 0


def test_ragged_blocks_of_whole_tensors_fit_the_static_workspace():
    need = vertex("ij,jk->ik", (1024, 4096), (4096, 2040), {"k": 8}, relu=True)[1]
    assert need == 1024 * 2040 * 4 <= 32 << 20                    # the product alone


@pytest.mark.parametrize("spec,bx,by,cut,kw", [
    ("iab,abk->ik", (240, 512, 384), (512, 384, 2712), {"i": 8}, {"otimes": "sqdiff"}),     # 176 tiles of 30 rows, 44 over the whole
    ("ij,kj->ik", (240, 8192), (3072, 8192), {"i": 8}, {}),                                 # 192 and 48
])
def test_walking_blocks_as_one_index_space_takes_no_more_slabs(spec, bx, by, cut, kw):
    """The executor cuts a long reduction further where tiles are few: the blocks' tiles count, not the fewer ones of the whole."""
    assert vertex(spec, bx, by, cut, **kw)[1] == 0


@pytest.mark.parametrize("spec,bx,by,dt,out,kernel,slabs", [
    # a long reduction under few tiles: cut into slabs, or a wave per output
    ("ij,jk->ik", (64, 100001), (100001, 64), "bf16", "f32", "reduce_row", 64),
    ("ij,jk->ik", (2, 100001), (100001, 2048), "bf16", "bf16", "reduce_row", 64),
    ("bv,vh->bh", (8, 50257), (50257, 4096), "bf16", "f32", "reduce_row", 16),
    ("bi,ij->bj", (4, 100001), (100001, 1024), "f32", "f32", "reduce_row", 64),
    ("ij,kj->ik", (8, 10001), (512, 10001), "f32", "f32", "reduce_row", 1),
    # columns in whole vectors: a column reduction (129 x 321 x 72 6.7 us, on tiles 12.4; 119 x 62 x 336 4.6 and 8.3)
    ("ji,jk->ik", (129, 321), (129, 72), "bf16", "f32", "reduce_row", 1),
    ("ij,jk->ik", (119, 62), (62, 336), "bf16", "f32", "reduce_row", 1),
    ("bij,bjk->bik", (32, 11, 82), (32, 82, 16), "f32", "f32", "reduce_row", 1),           # 7.3 and 8.9
    # tiles that would be almost empty
    ("bij,bjk->bik", (100000, 5, 17), (100000, 17, 5), "bf16", "f32", "generic", 1),
    # full ones, however short or long the reduction
    ("ij,jk->ik", (1001, 17), (17, 1003), "bf16", "bf16", "contract_mfma", 1),
    ("ij,jk->ik", (1001, 50257), (50257, 1003), "bf16", "f32", "contract_mfma", 1),
    ("bhsd,bhtd->bhst", (8, 16, 149, 80), (8, 16, 149, 80), "bf16", "bf16", "contract_mfma", 1),
])
def test_ragged_products_take_tiles_where_these_fill_the_chip(spec, bx, by, dt, out, kernel, slabs):
    ext = dict(zip(spec.split("->")[0].replace(",", ""), bx + by))
    elems = math.prod(ext[l] for l in spec.split("->")[1])
    assert vertex(spec, bx, by, {}, out=out, dt=dt) == (kernel, slabs * elems * 4 if slabs > 1 else 0)


@pytest.mark.parametrize("otimes,oplus,kernel", [("sqdiff", "sum", "contract_alu"), ("absdiff", "max", "contract_alu"), ("absdiff", "sum", "contract_alu"),
                                                  ("add", "sum", "generic"), ("sqdiff", "max", "generic"), ("mul", "max", "generic")])
def test_ragged_scalar_functions_with_tiles(otimes, oplus, kernel):
    """Operators read at run time take ten times as long on a tile, so only the compiled pairs have ragged tiles."""
    assert vertex("ij,jk->ik", (1025, 63), (63, 2051), {}, dt="f32", otimes=otimes, oplus=oplus)[0] == kernel


def refusal(spec, bx, by, cut, dt, out, zstrides=None):
    """What tr_execute answers to one vertex before it launches anything.  Every launcher makes its checks first, so without a GPU
    the error is that of the missing device (EG_ERR_HIP), or an earlier refusal; the operands' addresses are never touched."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("stops at the missing device")
    room = ctypes.create_string_buffer(512)
    at = (ctypes.addressof(room) + 255) // 256 * 256
    g, rels = E.einsum_graph_create(), []
    try:
        x, y = E.einsum_graph_add_input(g, list(bx), dt), E.einsum_graph_add_input(g, list(by), dt)
        z = E.einsum_graph_add_einsum(g, spec, "mul", "sum", 1.0, [x, y], out)
        names = spec.split("->")[0].replace(",", "")
        E.einsum_graph_set_partition(g, z, [cut.get(l, 1) for l in dict.fromkeys(names)])
        E.einsum_graph_mark_output(g, z)
        ext = dict(zip(names, tuple(bx) + tuple(by)))
        bz = [ext[l] for l in spec.split("->")[1]]
        for k, (b, t, st) in enumerate(((bx, dt, None), (by, dt, None), (bz, out, zstrides))):     # (apart from each other)
            rels.append(E.tensor_partition(at + ((k + 1) << 40), t, list(b), [1] * len(b), st))
        with pytest.raises(E.EgError) as e:
            E.tr_execute(g, rels[:2], rels[2:], at, 1 << 50)
        return str(e.value)
    finally:
        for r in rels:
            E.tensor_relation_destroy(r)
        E.einsum_graph_destroy(g)


@pytest.mark.parametrize("dt,out", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32")])
@pytest.mark.parametrize("spec,bx,by,cut,zstrides", [
    ("jab,jk->abk", (130, 13, 79), (130, 1101), {"j": 2}, [82 * 1101, 1101, 1]),          # row labels that do not join in the result
    ("jab,jk->abk", (123, 30, 35), (123, 1101), {"j": 3}, [40 * 1101, 1101, 1]),
    ("ij,jab->iab", (1101, 130), (130, 13, 79), {"j": 2}, [13 * 82, 82, 1]),              # column labels
    ("bf,bhd->fhd", (123, 3001), (123, 5, 77), {"b": 3}, [400, 80, 1]),
])
def test_ragged_cut_products_into_strided_results_are_accepted(spec, bx, by, cut, zstrides, dt, out):
    for z in (None, zstrides):
        assert "error -12:" in refusal(spec, bx, by, cut, dt, out, z)


@pytest.mark.parametrize("rows", [2, 16])
@pytest.mark.parametrize("cut", [262144, 524280, 524288, 600000])
def test_few_rows_cut_into_more_blocks_than_a_grid_has_pieces(rows, cut):
    """Eight blocks a piece at most, 65535 pieces a launch: beyond 524280 blocks the vertex stays on the tiles."""
    assert "error -12:" in refusal("ij,jk->ik", (rows, 8 * cut), (8 * cut, 64), {"j": cut}, "bf16", "f32")
