"""The work that users of the library run, as cases that can be timed and compared.

A case is a graph family with its sizes.  Every family goes through the public calls of the Python binding the way a program
does: the graph, its relations, its outputs and its workspace are built once (prepare), a pass is one tr_execute (run).
Sizes are those of the repository's workloads (matrix chains, a classifier's training step, a decoder block, a split
reduction, distances), the same graphs in smaller, ragged and single-token form, and the element-wise and reduction vertices
that stand between contractions.
"""
import math
import random

import torch

import paper_2410_02682_amd as E

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "bf16": 2}


def labels_of(spec):
    lhs, z = spec.split("->")
    ops = lhs.split(",")
    seen = []
    for c in "".join(ops):
        if c not in seen:
            seen.append(c)
    return ops, z, seen


class Net:
    """A graph as plain data: inputs (name, bound, dtype, how they are drawn), vertices, outputs."""

    def __init__(self):
        self.inputs, self.vertices, self.outputs = [], [], []
        self.bound, self.dtype = {}, {}

    def input(self, name, bound, dtype, dist="normal", std=1.0):
        self.inputs.append((name, tuple(bound), dtype, dist, std))
        self.bound[name], self.dtype[name] = tuple(bound), dtype

    def vertex(self, name, spec, inputs, dtype, otimes="mul", oplus="sum", alpha=1.0, cut=None, out=False):
        ops, z, seen = labels_of(spec)
        ext = {}
        for o, i in zip(ops, inputs):
            ext.update(zip(o, self.bound[i]))
        # a cut that does not divide its label's bound is left out, as a program has to (blocks are whole)
        d = {l: c for l, c in (cut or {}).items() if l in seen and ext[l] % c == 0}
        self.vertices.append((name, spec, tuple(inputs), dtype, otimes, oplus, alpha, [d.get(l, 1) for l in seen]))
        self.bound[name], self.dtype[name] = tuple(ext[l] for l in z), dtype
        if out:
            self.outputs.append(name)

    def contraction_ops(self):
        n = 0.0
        for _, spec, inputs, _, otimes, oplus, _, _ in self.vertices:
            ops, z, seen = labels_of(spec)
            if len(ops) == 2 and set(seen) - set(z):
                ext = {}
                for o, i in zip(ops, inputs):
                    ext.update(zip(o, self.bound[i]))
                n += (2.0 if otimes == "mul" else 3.0) * math.prod(ext[l] for l in seen)
        return n


# ------------------------------------------------------------------------------------------------
# the families
# ------------------------------------------------------------------------------------------------
def matmul(c):
    """One fp32 product, all three labels cut: the smallest call, and ordinary fp32 work."""
    n = Net()
    n.input("X", (c["i"], c["j"]), "f32", "uniform")
    n.input("Y", (c["j"], c["k"]), "f32", "uniform")
    n.vertex("Z", "ij,jk->ik", ("X", "Y"), "f32", cut={"i": c["cut"], "j": c["cut"], "k": c["cut"]}, out=True)
    return n


def chain(c):
    """(A B) C in bf16, the second product cut otherwise than the first (a repartition lies between them)."""
    n = Net()
    n.input("A", (c["i"], c["j"]), "bf16", std=c["j"] ** -0.5)
    n.input("B", (c["j"], c["k"]), "bf16")
    n.input("C", (c["k"], c["l"]), "bf16", std=c["k"] ** -0.5)
    n.vertex("AB", "ij,jk->ik", ("A", "B"), "bf16", cut={"i": 2, "j": 2, "k": 2})
    n.vertex("ABC", "ik,kl->il", ("AB", "C"), "f32", cut={"k": 2, "l": 4}, out=True)
    return n


def skewed(c):
    """A B + C (D E) with long thin factors; the long contraction is cut, the two summands are cut differently."""
    n = Net()
    n.input("A", (c["i"], c["j"]), "bf16", std=c["j"] ** -0.25)
    n.input("B", (c["j"], c["k"]), "bf16", std=c["j"] ** -0.25)
    n.input("C", (c["i"], c["m"]), "bf16", std=c["m"] ** -0.5)
    n.input("D", (c["m"], c["n"]), "bf16", std=c["n"] ** -0.25)
    n.input("E", (c["n"], c["k"]), "bf16", std=c["n"] ** -0.25)
    n.vertex("AB", "ij,jk->ik", ("A", "B"), "bf16", cut={"i": 4, "k": 2})
    n.vertex("DE", "mn,nk->mk", ("D", "E"), "bf16", cut={"n": 8})
    n.vertex("CDE", "im,mk->ik", ("C", "DE"), "bf16", cut={"i": 2, "k": 4})
    n.vertex("Z", "ik,ik->ik", ("AB", "CDE"), "f32", "add", "none", cut={"i": 8}, out=True)
    return n


def ffnn(c):
    """A training step of a two-layer classifier: forward, softmax cross-entropy, backward to both weight matrices; data parallel."""
    n, d = Net(), {"b": c["cut"]}
    b, f, h, k = c["b"], c["f"], c["h"], c["c"]
    n.input("X", (b, f), "bf16")
    n.input("W1", (f, h), "bf16", std=0.02)
    n.input("W2", (h, k), "bf16", std=0.02)
    n.input("Y", (b, k), "bf16", "onehot")
    n.vertex("H1", "bf,fh->bh", ("X", "W1"), "bf16", cut=d)
    n.vertex("A1", "bh->bh", ("H1",), "bf16", "relu", "none", cut=d)
    n.vertex("L", "bh,hc->bc", ("A1", "W2"), "f32", cut=d)
    n.vertex("Cmax", "bc->b", ("L",), "f32", "ident", "max", cut=d)
    n.vertex("Ex", "bc,b->bc", ("L", "Cmax"), "f32", "exp_sub", "none", cut=d)
    n.vertex("S", "bc->b", ("Ex",), "f32", "ident", "sum", cut=d)
    n.vertex("P", "bc,b->bc", ("Ex", "S"), "f32", "div", "none", cut=d)
    n.vertex("D", "bc,b->bc", ("L", "Cmax"), "f32", "sub", "none", cut=d)
    n.vertex("logS", "b->b", ("S",), "f32", "log", "none", cut=d)
    n.vertex("logP", "bc,b->bc", ("D", "logS"), "f32", "sub", "none", cut=d)
    n.vertex("loss", "bc,bc->", ("Y", "logP"), "f32", alpha=-1.0 / b, cut=d, out=True)
    n.vertex("dL", "bc,bc->bc", ("P", "Y"), "bf16", "sub", "none", alpha=1.0 / b, cut=d)
    n.vertex("dW2", "bh,bc->hc", ("A1", "dL"), "f32", cut=d, out=True)
    n.vertex("dA1", "bc,hc->bh", ("dL", "W2"), "bf16", cut=d)
    n.vertex("dH1", "bh,bh->bh", ("dA1", "H1"), "bf16", "relu_grad", "none", cut=d)
    n.vertex("dW1", "bf,bh->fh", ("X", "dH1"), "f32", cut=d, out=True)
    return n


def prefill(c):
    """A decoder block over whole prompts: causal attention and a gated feed-forward layer.  heads: attention cut by heads and the
    hidden label of the feed-forward layer; otherwise everything is cut by query position."""
    n = Net()
    b, s, a, h, d, f, q = c["b"], c["s"], c["a"], c["h"], c["d"], c["f"], c["cut"]

    def cut(labs):
        if not c["heads"]:
            return {"s": q} if "s" in labs else {"t": q}
        return {"h": q} if "h" in labs else {"f": q} if "f" in labs else {"s": q}

    def v(name, spec, inputs, dtype, *args, **kw):
        n.vertex(name, spec, inputs, dtype, *args, cut=cut(spec), **kw)

    n.input("X", (b, s, a), "bf16")
    for w in ("Wq", "Wk", "Wv", "Wo"):
        n.input(w, (a, h, d), "bf16", std=0.02)
    n.input("M", (s, s), "f32", "causal")
    n.input("Wg", (a, f), "bf16", std=0.02)
    n.input("Wu", (a, f), "bf16", std=0.02)
    n.input("Wd", (f, a), "bf16", std=0.02)
    v("Q", "bsa,ahd->bshd", ("X", "Wq"), "bf16")
    v("K", "bta,ahd->bthd", ("X", "Wk"), "bf16")
    v("V", "bta,ahd->bthd", ("X", "Wv"), "bf16")
    v("T1", "bshd,bthd->bhst", ("Q", "K"), "bf16")
    v("T2", "bhst,st->bhst", ("T1", "M"), "bf16", "add", "none", d ** -0.5)
    v("Cmax", "bhst->bhs", ("T2",), "f32", "ident", "max")
    v("Ex", "bhst,bhs->bhst", ("T2", "Cmax"), "bf16", "exp_sub", "none")
    v("S", "bhst->bhs", ("Ex",), "f32", "ident", "sum")
    v("P", "bhst,bhs->bhst", ("Ex", "S"), "bf16", "div", "none")
    v("O", "bhst,bthd->bshd", ("P", "V"), "bf16")
    v("Yatt", "bshd,ahd->bsa", ("O", "Wo"), "bf16")
    v("G", "bsa,af->bsf", ("Yatt", "Wg"), "bf16")
    v("U", "bsa,af->bsf", ("Yatt", "Wu"), "bf16")
    v("Hh", "bsf,bsf->bsf", ("G", "U"), "bf16", "silu_mul", "none")
    v("Out", "bsf,fa->bsa", ("Hh", "Wd"), "f32", out=True)
    return n


def decode(c):
    """The same block for one new token per sequence against cached keys and values; the token's own key and value come back."""
    n = Net()
    b, t, a, h, d, f, q = c["b"], c["t"], c["a"], c["h"], c["d"], c["f"], c["cut"]

    def v(name, spec, inputs, dtype, *args, **kw):
        n.vertex(name, spec, inputs, dtype, *args, cut={"h": q} if "h" in spec else {"f": q} if "f" in spec else {}, **kw)

    n.input("X", (b, a), "bf16")
    for w in ("Wq", "Wk", "Wv", "Wo"):
        n.input(w, (a, h, d), "bf16", std=0.02)
    n.input("Kc", (b, t, h, d), "bf16")
    n.input("Vc", (b, t, h, d), "bf16")
    n.input("Wg", (a, f), "bf16", std=0.02)
    n.input("Wu", (a, f), "bf16", std=0.02)
    n.input("Wd", (f, a), "bf16", std=0.02)
    v("Q", "ba,ahd->bhd", ("X", "Wq"), "bf16")
    v("Knew", "ba,ahd->bhd", ("X", "Wk"), "bf16", out=True)
    v("Vnew", "ba,ahd->bhd", ("X", "Wv"), "bf16", out=True)
    v("T", "bhd,bthd->bht", ("Q", "Kc"), "bf16", alpha=d ** -0.5)
    v("Cmax", "bht->bh", ("T",), "f32", "ident", "max")
    v("Ex", "bht,bh->bht", ("T", "Cmax"), "bf16", "exp_sub", "none")
    v("S", "bht->bh", ("Ex",), "f32", "ident", "sum")
    v("P", "bht,bh->bht", ("Ex", "S"), "bf16", "div", "none")
    v("O", "bht,bthd->bhd", ("P", "Vc"), "bf16")
    v("Yatt", "bhd,ahd->ba", ("O", "Wo"), "bf16")
    v("G", "ba,af->bf", ("Yatt", "Wg"), "bf16")
    v("U", "ba,af->bf", ("Yatt", "Wu"), "bf16")
    v("Hh", "bf,bf->bf", ("G", "U"), "bf16", "silu_mul", "none")
    v("Out", "bf,fa->ba", ("Hh", "Wd"), "f32", out=True)
    return n


def split(c):
    """One contraction whose contracted label is cut many ways: the aggregation of partial blocks weighs as much as it ever does."""
    n = Net()
    n.input("X", (c["i"], c["j"], c["k"]), "bf16", "uniform")
    n.input("Y", (c["k"], c["l"]), "bf16", "uniform")
    n.vertex("Z", "ijk,kl->ijl", ("X", "Y"), "f32", cut={"k": c["cut"]}, out=True)
    return n


def distances(c):
    """Squared L2 and L-infinity distances of all pairs of rows, in fp32 and in bf16."""
    n, d = Net(), {"i": 2, "j": 2, "k": 2}
    n.input("X", (c["i"], c["j"]), "f32", "uniform")
    n.input("Y", (c["j"], c["k"]), "f32", "uniform")
    n.input("Xh", (c["i"], c["j"]), "bf16", "uniform")
    n.input("Yh", (c["k"], c["j"]), "bf16", "uniform")
    n.vertex("L2", "ij,jk->ik", ("X", "Y"), "f32", "sqdiff", cut=d, out=True)
    n.vertex("Linf", "ij,jk->ik", ("X", "Y"), "f32", "absdiff", "max", cut=d, out=True)
    n.vertex("L2h", "ij,kj->ik", ("Xh", "Yh"), "f32", "sqdiff", cut=d, out=True)
    n.vertex("Linfh", "ij,kj->ik", ("Xh", "Yh"), "bf16", "absdiff", "max", cut=d, out=True)
    return n


def tensor_ops(c):
    """What stands between contractions: a sum of two tensors, a permutation, row and column reductions, a row softmax, and an
    aggregation of partial slabs that the program holds itself."""
    n, q = Net(), c["cut"]
    b, s, h, d = c["b"], c["s"], c["h"], c["d"]
    n.input("X", (b, s, h, d), "bf16")
    n.input("R", (b, s, h, d), "bf16")
    n.input("W", (b * s, h * d), "f32", std=2.0)
    n.vertex("Sum", "bshd,bshd->bshd", ("X", "R"), "bf16", "add", "none", cut={"h": q}, out=True)
    n.vertex("Perm", "bshd->bhsd", ("X",), "bf16", "ident", "none", cut={"h": q}, out=True)
    n.vertex("Bias", "bshd->hd", ("X",), "f32", "ident", "sum", cut={"s": q}, out=True)
    n.vertex("Dot", "bshd,bshd->bsh", ("X", "R"), "f32", cut={"s": q}, out=True)
    n.vertex("Cmax", "rc->r", ("W",), "f32", "ident", "max", cut={"r": q})
    n.vertex("Ex", "rc,r->rc", ("W", "Cmax"), "f32", "exp_sub", "none", cut={"r": q})
    n.vertex("S", "rc->r", ("Ex",), "f32", "ident", "sum", cut={"r": q})
    n.vertex("P", "rc,r->rc", ("Ex", "S"), "bf16", "div", "none", cut={"r": q}, out=True)
    return n


FAMILIES = {f.__name__: f for f in (matmul, chain, skewed, ffnn, prefill, decode, split, distances, tensor_ops)}


def listed():
    return [
        # a single small fp32 product in 2 x 2 x 2 blocks: latency and launches
        {"name": "matmul_f32_256", "family": "matmul", "i": 256, "j": 256, "k": 256, "cut": 2},
        # matrix-chain arithmetic at an ordinary and at the benchmark's size
        {"name": "chain_2048", "family": "chain", "i": 2048, "j": 2048, "k": 2048, "l": 2048},
        {"name": "chain_8192", "family": "chain", "i": 8192, "j": 8192, "k": 8192, "l": 8192},
        # the five-matrix chain with skewed factors
        {"name": "skewed_10240", "family": "skewed", "i": 10240, "j": 1024, "k": 10240, "m": 1024, "n": 102400},
        # a training step, forward and backward, at the wide classifier's size and with sizes as they come
        {"name": "ffnn_4096", "family": "ffnn", "b": 4096, "f": 8192, "h": 4096, "c": 1024, "cut": 8},
        {"name": "ffnn_ragged", "family": "ffnn", "b": 1000, "f": 3001, "h": 1530, "c": 1003, "cut": 8},
        # prompts through a decoder block, every vertex on its own and with attention as one pass
        {"name": "prefill_4x2048", "family": "prefill", "b": 4, "s": 2048, "a": 4096, "h": 32, "d": 128, "f": 11008, "cut": 8, "heads": True, "one_pass": False},
        {"name": "prefill_1x4096_one_pass", "family": "prefill", "b": 1, "s": 4096, "a": 4096, "h": 32, "d": 128, "f": 11008, "cut": 8, "heads": False, "one_pass": True},
        # one token for each of eight sequences
        {"name": "decode_8x2048", "family": "decode", "b": 8, "t": 2048, "a": 4096, "h": 32, "d": 128, "f": 11008, "cut": 8},
        # a large reduction cut sixteen ways
        {"name": "split_k16", "family": "split", "i": 64, "j": 1024, "k": 16384, "l": 4096, "cut": 16},
        # distances off the matrix pipes
        {"name": "distances_8192", "family": "distances", "i": 8192, "j": 1024, "k": 8192},
        # maps, a permutation, reductions, a softmax and an aggregation on 64 MB tensors
        {"name": "tensor_ops_4x2048", "family": "tensor_ops", "b": 4, "s": 2048, "h": 32, "d": 128, "cut": 8, "slabs": 8},
    ]


def draw(rng: random.Random):
    """One more case of a family.  Half of the sizes are whole tiles, a quarter whole 16-byte vectors, a quarter as they come."""
    rag = rng.choice((64, 64, 8, 1))

    def size(lo, hi, step=None):
        step = step or rag
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return max(step, int(v / step) * step + (0 if step > 1 else 1 - int(v) % 2 if rng.random() < 0.5 else 0))

    # sizes that are no whole vectors stay ordinary ones; multiples of eight and sixteen vectors reach the largest
    top = {64: 1.0, 8: 0.5, 1: 0.25}[rag]
    fam = rng.choice(sorted(FAMILIES))
    if fam == "matmul":
        return {"family": fam, "i": size(64, 2048), "j": size(64, 2048), "k": size(64, 2048), "cut": rng.choice((1, 2, 4))}
    if fam == "chain":
        hi = 8192 * top
        return {"family": fam, "i": size(256, hi), "j": size(256, hi), "k": size(256, hi), "l": size(256, hi)}
    if fam == "skewed":
        s = size(512, 10240 * top)
        t = size(64, 1024 * top)
        return {"family": fam, "i": s, "j": t, "k": size(512, 10240 * top), "m": size(64, 1024 * top), "n": size(4096, 102400 * top)}
    if fam == "ffnn":
        return {"family": fam, "b": size(128, 4096 * top), "f": size(256, 8192 * top), "h": size(256, 4096 * top), "c": size(16, 1024), "cut": rng.choice((1, 2, 4, 8))}
    if fam == "prefill":
        h, d = rng.choice(((8, 64), (16, 64), (8, 128), (16, 128), (32, 128), (32, 64)))
        b = rng.choice((1, 2, 4))
        one = rng.random() < 0.5
        return {"family": fam, "b": b, "s": size(128, (4096 if one else 2048) * top * 2 / (1 + b)), "a": h * d, "h": h, "d": d, "f": size(512, 11008, max(8, rag)), "cut": rng.choice((1, 2, 4, 8)),
                "heads": rng.random() < 0.5, "one_pass": one}
    if fam == "decode":
        h, d = rng.choice(((8, 64), (16, 64), (8, 128), (16, 128), (32, 128), (32, 64)))
        return {"family": fam, "b": rng.choice((1, 2, 3, 4, 8, 16)), "t": size(128, 4096 * min(1.0, 2 * top)), "a": h * d, "h": h, "d": d, "f": size(512, 11008, max(8, rag)), "cut": rng.choice((1, 2, 4, 8))}
    if fam == "split":
        cut = rng.choice((2, 4, 8, 16))
        step = {64: 64, 8: 8, 1: 2}[rag]
        return {"family": fam, "i": rng.choice((1, 2, 4, 8, 16, 32)), "j": size(64, 1024 * top), "k": cut * size(64, 1024, step), "l": size(128, 4096 * top), "cut": cut}
    if fam == "distances":
        hi = 8192 * top
        return {"family": fam, "i": size(128, hi), "j": size(32, 1024), "k": size(128, hi)}
    return {"family": fam, "b": rng.choice((1, 2, 4)), "s": size(128, 2048), "h": rng.choice((8, 16, 32)), "d": rng.choice((64, 80, 128)), "cut": rng.choice((1, 2, 4, 8)), "slabs": rng.choice((2, 4, 8, 16))}


# ------------------------------------------------------------------------------------------------
# state and passes
# ------------------------------------------------------------------------------------------------
def values(bound, dtype, dist, std, gen):
    t = torch.empty(bound, dtype=DTYPES[dtype], device="cuda")
    if dist == "normal":
        return t.normal_(0.0, std, generator=gen)
    if dist == "uniform":
        return t.uniform_(-1.0, 1.0, generator=gen)
    if dist == "onehot":
        cls = torch.randint(0, bound[1], (bound[0], 1), generator=gen, device="cuda")
        return t.zero_().scatter_(1, cls, 1.0)
    return t.fill_(float("-inf")).triu_(1)                                    # causal: zero up to the query's own position


class State:
    """What a program keeps: graph, relations over its tensors, workspace."""

    def __init__(self, case, seed):
        net = FAMILIES[case["family"]](case)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        self.tensors, self.rels = {}, []
        self.g = E.einsum_graph_create()
        if case.get("one_pass"):
            E.tr_set_fused_attention(self.g, True)
        ids = {}
        for name, bound, dtype, dist, std in net.inputs:
            self.tensors[name] = values(bound, dtype, dist, std, gen)
            ids[name] = E.einsum_graph_add_input(self.g, bound, dtype)
        for name, spec, inputs, dtype, otimes, oplus, alpha, d in net.vertices:
            ids[name] = E.einsum_graph_add_einsum(self.g, spec, otimes, oplus, alpha, [ids[i] for i in inputs], dtype)
            E.einsum_graph_set_partition(self.g, ids[name], d)
        for name in net.outputs:
            E.einsum_graph_mark_output(self.g, ids[name])
            self.tensors[name] = torch.empty(net.bound[name], dtype=DTYPES[net.dtype[name]], device="cuda")
        self.ins = [self.relation(name, net) for name, *_ in net.inputs]
        self.outs = [self.relation(name, net) for name in net.outputs]
        self.results = [self.tensors[name] for name in net.outputs]
        self.ws = torch.empty(max(256, E.tr_workspace_bytes(self.g)), dtype=torch.uint8, device="cuda")
        self.slabs = None
        if case.get("slabs"):
            shape = (case["b"] * case["s"], case["h"] * case["d"])
            self.slabs = values((case["slabs"],) + shape, "f32", "normal", 1.0, gen)
            self.total = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
            self.total_rel = E.tensor_partition(self.total.data_ptr(), "bf16", shape, [1, 1])
            self.rels.append(self.total_rel)
            self.results.append(self.total)

    def relation(self, name, net):
        r = E.tensor_partition(self.tensors[name].data_ptr(), net.dtype[name], net.bound[name], [1] * len(net.bound[name]))
        self.rels.append(r)
        return r

    def __del__(self):
        for r in self.rels:
            E.tensor_relation_destroy(r)
        E.einsum_graph_destroy(self.g)


def prepare(case, seed):
    return State(case, seed)


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    E.tr_execute(s.g, s.ins, s.outs, s.ws.data_ptr(), s.ws.numel(), stream)
    if s.slabs is not None:
        E.tr_aggregate("sum", s.slabs.data_ptr(), s.slabs.shape[0], s.slabs[0].numel(), s.total_rel, stream)
    return s.results


def work(case):
    net = FAMILIES[case["family"]](case)
    n = sum(math.prod(b) * SIZE[net.dtype[name]] for name, b in [(x[0], x[1]) for x in net.inputs] + [(o, net.bound[o]) for o in net.outputs])
    if case.get("slabs"):
        n += case["b"] * case["s"] * case["h"] * case["d"] * (4 * case["slabs"] + 2)
    return {"bytes": float(n), "flops": net.contraction_ops()}


# About four times what the path differs by from the same graph evaluated in 64 bits with the tensors' own roundings, and from
# itself with its sums taken in another order: a bf16 tensor's value on a rounding boundary falls to the other side then, and
# what is computed from it moves by a unit in its last place.
TOLERANCE = {
    "matmul": (4e-6, 4e-5),         # exact inputs, fp32 sums, fp32 results
    "split": (4e-6, 4e-5),
    "distances": (4e-6, 4e-5),
    "tensor_ops": (1e-4, 3e-2),
    "chain": (2e-4, 8e-3),
    "skewed": (1.2e-3, 5e-2),
    "ffnn": (1.3e-3, 0.2),
    "prefill": (5e-3, 0.15),
    "decode": (1e-2, 7e-2),
}


def tolerance(case):
    rel, most = TOLERANCE[case["family"]]
    if case.get("one_pass"):        # attention as one pass divides by the row sum after the second product instead of before
        rel, most = 2.3e-2, 0.6
    return {"rel": rel, "max": most}
