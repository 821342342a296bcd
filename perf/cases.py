"""What a user of this library has it do, as cases that can be timed and compared.

Every case goes through the public entry points of `paper_2311_13225_amd.binding`. The kinds:

  step        one training step (sample, gather, forward, loss, backward, SGD, cache refresh), with the batch sampled in
              the call or prepared ahead by the call before it
  superbatch  n steps with the bulk refresh of all hot rows committed before the first and started again behind it
  sample      sampling a batch alone (no cache): every array of every block
  gather      feature rows of an id list
  layer       one GraphSAGE-mean layer over a caller's block, forward and backward
  csr         edge list -> in-neighbour CSR
  hot         pre-sampling and ranking of the hot vertices

Graphs are R-MAT (0.57, 0.19, 0.19, 0.05) with permuted ids, made on the device; features are N(0, 1); labels are
uniform; weights are Glorot-uniform. Sizes follow the named workloads of `synth_inputs.py`.
"""
import math

import torch

from paper_2311_13225_amd import binding as b

# Named graphs: vertices, directed edges, whether made of pairs in both directions, row-pointer width.
TINY = dict(vertices=10_000, edges=100_000, symmetrise=False, rowptr_bits=32)
DENSE = dict(vertices=233_000, edges=114_000_000, symmetrise=False, rowptr_bits=64)
SPARSE = dict(vertices=2_400_000, edges=124_000_000, symmetrise=True, rowptr_bits=32)
# the largest workload at a quarter of its vertices and edges: tables and column array far beyond every cache, and still
# quick to make again and again
LARGE = dict(vertices=27_750_000, edges=400_000_000, symmetrise=False, rowptr_bits=64)

ARCH = {"sage": b.NO_ARCH_SAGE_MEAN, "gcn": b.NO_ARCH_GCN, "gcn_sum": b.NO_ARCH_GCN_SUM, "gcn_sym": b.NO_ARCH_GCN_SYM}
TRAIN_SHARE = 0.65
N_BATCHES = 64           # seed batches a state holds; a pass takes the next one
WARM_STEPS = 2           # steps a training state has behind it: the cache holds rows, a next batch is prepared
LR = 0.01
KEY = 7                  # the sampling seed of every case


def _step(name, graph, feat_dim, dtype, classes, hidden, fanouts, batch, hot_fraction, staleness, arch="sage", ahead=True,
          presample_batches=0, kind="step", n_steps=1):
    c = dict(kind=kind, feat_dim=feat_dim, dtype=dtype, classes=classes, hidden=hidden, fanouts=fanouts, batch=batch,
             hot_fraction=hot_fraction, staleness=staleness, arch=arch, ahead=ahead, presample_batches=presample_batches,
             n_steps=n_steps, **graph)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest training step: exact training (no cache), sampled in the call; launches and their gaps
        _step("step_tiny_exact", TINY, 64, "f32", 16, 64, "10,5", 256, 0.0, 0, ahead=False),
        # ordinary training, dense neighbourhoods and wide rows, next batch prepared ahead
        _step("step_dense_ahead", DENSE, 602, "f32", 41, 256, "25,10", 1024, 0.10, 1),
        # ordinary training of a three-layer model for a caller that does not know its next batch yet
        _step("step_sparse", SPARSE, 100, "f32", 47, 256, "15,10,5", 1024, 0.10, 2, ahead=False),
        # the flagship: bf16 features, three layers, tables far larger than any cache
        _step("step_large_bf16_ahead", LARGE, 128, "bf16", 172, 256, "15,10,5", 1024, 0.10, 2, presample_batches=64),
        # the largest batches: matrix products and row traffic
        _step("step_sweep_ahead", SPARSE, 256, "f32", 47, 256, "15,10,5", 4096, 0.10, 2),
        # the other layer family: GCN-style average with one matrix
        _step("step_dense_gcn_ahead", DENSE, 602, "f32", 41, 256, "25,10", 1024, 0.10, 1, arch="gcn"),
        # the paper's schedule: four steps beside the bulk refresh of every hot row, bound 2n - 1
        _step("superbatch_sparse", SPARSE, 100, "f32", 47, 256, "15,10,5", 1024, 0.10, 7, kind="superbatch", n_steps=4),
        # sampling for evaluation: no cache, no training behind it, a ragged batch
        dict(name="sample_sparse", kind="sample", fanouts="15,10,5", batch=1000, **SPARSE),
        # feature collection of a bottom hop's sources out of a table in HBM
        dict(name="gather_large_bf16", kind="gather", rows=27_750_000, n=118_000, feat_dim=128, dtype="bf16", counted=False),
        # a hidden layer by itself, both directions, input gradient included
        dict(name="layer_hidden", kind="layer", n_dst=3_400, n_src=25_000, fanout=10, feat_dim=256, out_dim=256, dtype="f32",
             relu=True, input_grad=True),
        # what every program pays before its first step: the graph ...
        dict(name="csr_sparse", kind="csr", ids64=False, **SPARSE),
        # ... and the hot set (one epoch of pre-sampling)
        dict(name="hot_sparse", kind="hot", fanouts="15,10,5", batch=1024, hot_fraction=0.10, hidden=256, epochs=1, **SPARSE),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_graph(rng, most_edges):
    v = _log(rng, 10_000, 2_400_000)
    e = min(most_edges, v * _log(rng, 8, 490))
    sym = rng.random() < 0.4
    return dict(vertices=v, edges=e - e % 2 if sym else e, symmetrise=sym, rowptr_bits=rng.choice((32, 64)))


def _fit_batch(batch, fanouts, feat_dim):
    """The batch, cut down so that the widest hop stays within that of the largest listed step."""
    grow = 1
    for f in fanouts.split(","):
        grow *= int(f) + 1
    return max(64, min(batch, 4096 * 16 * 11 * 6 * 256 // (grow * max(64, feat_dim))))


def _size(case):
    """One number for a case's work: bytes, or operations at 50 a byte."""
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_size(c) for c in listed())
    while True:
        case = _draw(rng)
        if _size(case) <= most:
            return case


def _draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "step", "superbatch", "sample", "gather", "layer", "csr", "hot"))
    fanouts = rng.choice(("10,5", "25,10", "10,10", "15,10,5", "25,10,5", "5,5,5", "4,3,3,2"))
    if kind in ("step", "superbatch"):
        arch = rng.choice(("sage", "sage", "sage", "gcn", "gcn_sum", "gcn_sym")) if kind == "step" else "sage"
        feat = _log(rng, 32, 602)
        c = _step(None, _draw_graph(rng, 114_000_000), feat, rng.choice(("f32", "bf16")), rng.randint(10, 172),
                  rng.choice((64, 100, 128, 200, 256)), fanouts, _fit_batch(_log(rng, 64, 4096), fanouts, feat),
                  rng.choice((0.0, 0.05, 0.1, 0.3)), rng.randint(0, 4), arch=arch, ahead=rng.random() < 0.6,
                  presample_batches=64, kind=kind)
        if kind == "superbatch":
            n = rng.choice((2, 4, 8))
            c.update(n_steps=n, staleness=2 * n - 1, hot_fraction=rng.choice((0.05, 0.1)), ahead=True)
        return c
    if kind == "sample":
        return dict(kind=kind, fanouts=fanouts, batch=_fit_batch(_log(rng, 64, 10_000), fanouts, 256), **_draw_graph(rng, 114_000_000))
    if kind == "gather":
        feat = _log(rng, 16, 602)
        return dict(kind=kind, rows=_log(rng, 10_000, 6_000_000), n=_log(rng, 256, 400_000), feat_dim=feat,
                    dtype=rng.choice(("f32", "bf16")), counted=rng.random() < 0.5)
    if kind == "layer":
        n_dst = _log(rng, 100, 60_000)
        fanout = rng.randint(3, 25)
        return dict(kind=kind, n_dst=n_dst, n_src=int(n_dst * rng.uniform(1.0, 1.0 + fanout)), fanout=fanout,
                    feat_dim=_log(rng, 32, 602), out_dim=_log(rng, 16, 256), dtype=rng.choice(("f32", "bf16")),
                    relu=rng.random() < 0.7, input_grad=rng.random() < 0.7)
    if kind == "csr":
        return dict(kind=kind, ids64=rng.random() < 0.3, **_draw_graph(rng, 60_000_000))
    graph = _draw_graph(rng, 114_000_000)
    return dict(kind="hot", fanouts=fanouts, batch=max(_log(rng, 256, 4096), graph["vertices"] // 1500),
                hot_fraction=rng.choice((0.05, 0.1, 0.3)), hidden=128, epochs=1, **graph)


# ------------------------------------------------------------------------------------------------------- inputs

def _generator(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * (seed + 1) + tag)
    return g


def _edges(case, seed):
    """(src, dst) int32 on the device: `edges` of them, or half as many pairs where the graph is symmetric."""
    v, m = case["vertices"], case["edges"] // (2 if case["symmetrise"] else 1)
    gen = _generator(seed, 1)
    levels = max(1, math.ceil(math.log2(v)))
    ta, tb, tc = (int(round(p * 65536)) for p in (0.57, 0.76, 0.95))
    src = torch.empty(m, dtype=torch.int32, device="cuda")
    dst = torch.empty(m, dtype=torch.int32, device="cuda")
    filled = 0
    while filled < m:
        k = min(1 << 24, int((m - filled) * 1.2) + 1024)
        s = torch.zeros(k, dtype=torch.int32, device="cuda")
        d = torch.zeros(k, dtype=torch.int32, device="cuda")
        for _ in range(levels):
            u = torch.randint(0, 65536, (k,), generator=gen, dtype=torch.int32, device="cuda")
            lower = u >= tb
            s.mul_(2).add_(lower)
            d.mul_(2).add_(((u >= ta) & ~lower) | (u >= tc))
        ok = (s < v) & (d < v)
        s, d = s[ok], d[ok]
        n = min(m - filled, s.numel())
        src[filled:filled + n] = s[:n]
        dst[filled:filled + n] = d[:n]
        filled += n
    perm = torch.randperm(v, generator=gen, device="cuda", dtype=torch.int32)
    for t in (src, dst):
        for lo in range(0, m, 1 << 26):
            t[lo:lo + (1 << 26)] = perm[t[lo:lo + (1 << 26)].long()]
    return src, dst


def _graph(case, seed):
    src, dst = _edges(case, seed)
    return b.no_build_csr(src, dst, case["vertices"], case["rowptr_bits"], symmetrise=case["symmetrise"])


def _table(rows, dim, dtype, seed):
    gen = _generator(seed, 2)
    t = torch.empty((rows, dim), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    step = max(1, (1 << 28) // dim)
    for lo in range(0, rows, step):
        n = min(step, rows - lo)
        t[lo:lo + n] = torch.randn((n, dim), generator=gen, device="cuda")
    return t


def _train_ids(case, seed):
    perm = torch.randperm(case["vertices"], generator=_generator(seed, 3), device="cuda", dtype=torch.int32)
    return perm[: max(case["batch"], int(case["vertices"] * TRAIN_SHARE))].contiguous()


def _batches(train, batch, count):
    n = max(1, min(count, train.numel() // batch))
    return [train[i * batch:(i + 1) * batch].clone() for i in range(n)]


def _fanouts(case):
    return [int(f) for f in case["fanouts"].split(",")]


def _dims(case):
    return [case["feat_dim"]] + [case["hidden"]] * (len(_fanouts(case)) - 1) + [case["classes"]]


def _uniform(shape, limit, gen):
    return (torch.rand(shape, generator=gen, device="cuda") * 2 - 1) * limit


def _glorot(d_in, d_out, gen):
    limit = math.sqrt(6.0 / (2 * d_in + d_out))
    return _uniform((d_in, d_out), limit, gen), _uniform((d_in, d_out), limit, gen), _uniform((d_out,), 0.1, gen)


class _Training:
    """A training program between two passes: graph, table, labels, model, cache and the batches to come."""

    def __init__(self, case, seed):
        fan, dims = _fanouts(case), _dims(case)
        self.graph = _graph(case, seed)
        self.table = _table(case["vertices"], case["feat_dim"], case["dtype"], seed)
        gen = _generator(seed, 4)
        self.labels = torch.randint(0, case["classes"], (case["vertices"],), generator=gen, dtype=torch.int32, device="cuda")
        train = _train_ids(case, seed)
        self.batches = _batches(train, case["batch"], N_BATCHES)
        self.cache = None
        arch = ARCH[case["arch"]]
        if case["hot_fraction"] > 0.0:
            n = case["presample_batches"] * case["batch"]
            self.cache = b.no_select_hot(self.graph, train[:n].contiguous() if 0 < n < train.numel() else train, case["batch"], fan, 1,
                                         case["hot_fraction"], case["staleness"], case["hidden"], KEY)
            if case["arch"] != "sage":
                b.no_cache_set_layer_form(self.cache, arch)
        self.model = b.no_model_create(self.graph, dims, case["batch"], fan, b.NO_F32 if case["dtype"] == "f32" else b.NO_BF16)
        b.no_model_set_arch(self.model, arch)
        for layer in range(1, len(dims)):
            for t, w in zip(b.no_model_params(self.model, layer), _glorot(dims[layer - 1], dims[layer], gen)):
                t.copy_(w)
        self.w1 = b.no_model_params(self.model, 1)
        self.n_steps, self.super = case["n_steps"], case["kind"] == "superbatch"
        self.ahead, self.bottom_fanout, self.step, self.pending = case["ahead"], fan[-1], 0, False
        self.out = {}
        one_matrix = case["arch"] != "sage"
        for layer in range(1, len(dims)):
            for what, three in (("param", b.no_model_params(self.model, layer)), ("grad", b.no_model_grads(self.model, layer))):
                for part, t in zip(("self", "neigh", "bias"), three):
                    if not (one_matrix and part == "neigh"):
                        self.out["%s%d_%s" % (what, layer, part)] = t
        # the last layer's output over the seeds
        self.out["logits"] = b.no_model_activations(self.model, len(dims) - 1, case["batch"], case["batch"])[0]
        self._see_cache(case["vertices"])
        if self.super:
            for _ in range(2):           # from the second super-batch on every hot vertex is served
                self.super_batch()
                self._see_cache(case["vertices"])
        else:
            for _ in range(WARM_STEPS):
                self.one_step()
        torch.cuda.synchronize()

    def _see_cache(self, n_vertices):
        if self.cache is not None:
            view = b.no_cache_view(self.cache, n_vertices)
            which = "" if not self.super else "_%d" % (self.step > self.n_steps)
            self.out["version" + which], self.out["rows" + which] = view["version"], view["emb"]

    def one_step(self, commit=False):
        t, n = self.step, len(self.batches)
        if self.ahead:
            b.no_train_step_ahead(self.model, self.graph, self.table, self.labels, self.batches[t % n], self.batches[(t + 1) % n],
                                  commit, self.cache, t, KEY, LR, want_stats=False)
        else:
            b.no_train_step(self.model, self.graph, self.table, self.labels, self.batches[t % n], self.cache, t, KEY, LR,
                            want_stats=False)
        self.step = t + 1

    def super_batch(self):
        for i in range(self.n_steps):
            if i == 0:
                b.no_refresh_hot_begin(self.cache, self.graph, self.table, self.w1[0], self.w1[1], self.w1[2], self.bottom_fanout,
                                       self.step, KEY)
            # the rows refreshed during this super-batch become current behind its last step
            self.one_step(commit=i == self.n_steps - 1)


class _Sampling:
    """Batches to sample and the block arrays at their capacities, zero where no batch has written yet (sizes depend on the batch)."""

    def __init__(self, case, seed):
        self.graph = _graph(case, seed)
        self.blocks = b.no_blocks_create(self.graph, case["batch"], _fanouts(case))
        self.batches = _batches(_train_ids(case, seed), case["batch"], 8)
        self.at, self.out = 0, {}
        for hop in range(len(_fanouts(case))):
            v = b.no_blocks_view(self.blocks, hop)
            for key, ptr, n in (("src", v.d_src_global, v.n_src_cap), ("indptr", v.d_indptr, v.n_dst_cap + 1),
                                ("nbr", v.d_nbr_global, v.nnz_cap), ("indices", v.d_indices, v.nnz_cap),
                                ("csc_indptr", v.d_csc_indptr, v.n_src_cap + 1), ("csc_dst", v.d_csc_dst, v.nnz_cap),
                                ("csc_eid", v.d_csc_eid, v.nnz_cap), ("n_dst", v.d_n_dst, 1), ("n_src", v.d_n_src, 1), ("nnz", v.d_nnz, 1)):
                if ptr:
                    self.out["%s%d" % (key, hop)] = b._view(ptr, (n,), "<i4", self.blocks).zero_()

    def sample(self):
        i = self.at
        self.at = (i + 1) % len(self.batches)
        b.no_sample_blocks(self.graph, self.batches[i], KEY, i, None, self.blocks)
        return self.out


class _Gather:
    """A table, and eight id lists with their outputs: between two uses of a list the others pass through the caches."""

    def __init__(self, case, seed):
        self.table = _table(case["rows"], case["feat_dim"], case["dtype"], seed)
        gen = _generator(seed, 5)
        n = case["n"]
        self.lists = [torch.randint(0, case["rows"], (n,), generator=gen, dtype=torch.int32, device="cuda") for _ in range(8)]
        self.outs = [torch.zeros((n, case["feat_dim"]), dtype=self.table.dtype, device="cuda") for _ in range(8)]
        # a device count that leaves the last rows of the capacity alone, as a sampled block's does
        self.count = torch.tensor([n - n // 8], dtype=torch.int32, device="cuda") if case["counted"] else None
        self.at = 0

    def gather(self):
        i = self.at
        self.at = (i + 1) % 8
        return b.no_gather_features(self.table, self.lists[i], self.outs[i], n_ids=self.count)


class _Layer:
    """A block of a caller's own, its transpose, one layer's weights and every output buffer."""

    def __init__(self, case, seed):
        gen = _generator(seed, 6)
        n_dst, n_src, fan, d_in, d_out = (case[k] for k in ("n_dst", "n_src", "fanout", "feat_dim", "out_dim"))
        i32 = dict(dtype=torch.int32, device="cuda")
        lens = torch.randint(0, fan + 1, (n_dst,), generator=gen, device="cuda")
        indptr = torch.zeros(n_dst + 1, **i32)
        indptr[1:] = lens.cumsum(0)
        nnz = int(indptr[-1])
        # sources by popularity: a share of the edges goes to a few of them
        r = torch.rand(nnz, generator=gen, device="cuda", dtype=torch.float64)
        indices = (r * r * n_src).to(torch.int32).clamp_(0, n_src - 1)
        rows = torch.repeat_interleave(torch.arange(n_dst, device="cuda"), lens)
        order = torch.argsort(indices.long(), stable=True)
        csc_indptr = torch.zeros(n_src + 1, **i32)
        csc_indptr[1:] = torch.bincount(indices.long(), minlength=n_src).cumsum(0)
        self.block = b.block_view_from_tensors(torch.tensor([n_dst], **i32), torch.tensor([n_src], **i32), indptr, indices, n_dst, n_src,
                                               csc_indptr, rows[order].to(torch.int32))
        self.x = torch.randn((n_src, d_in), generator=gen, device="cuda").to(torch.float32 if case["dtype"] == "f32" else torch.bfloat16)
        self.w_self, self.w_neigh, self.bias = _glorot(d_in, d_out, gen)
        self.grad_h = torch.randn((n_dst, d_out), generator=gen, device="cuda")
        f32 = dict(dtype=torch.float32, device="cuda")
        self.mean, self.h = torch.empty((n_dst, d_in), **f32), torch.empty((n_dst, d_out), **f32)
        self.grads = [torch.empty((d_in, d_out), **f32), torch.empty((d_in, d_out), **f32), torch.empty((d_out,), **f32)]
        self.grad_x = torch.empty((n_src, d_in), **f32) if case["input_grad"] else None
        self.ws = torch.empty(b.no_sage_layer_ws_bytes(n_dst, n_src, d_in, d_out), dtype=torch.uint8, device="cuda")
        self.relu = case["relu"]

    def forward_backward(self):
        b.no_sage_layer_fwd(self.block, self.x, self.w_self, self.w_neigh, self.bias, self.relu, self.mean, self.h, self.ws)
        b.no_sage_layer_bwd(self.block, self.x, self.mean, self.h, self.grad_h, self.w_self, self.w_neigh, self.relu, *self.grads,
                            self.grad_x, self.ws)
        return [self.mean, self.h] + self.grads + ([self.grad_x] if self.grad_x is not None else [])


class _EdgeList:
    def __init__(self, case, seed):
        self.src, self.dst = _edges(case, seed)
        if case["ids64"]:
            self.src, self.dst = self.src.long(), self.dst.long()
        self.args = (case["vertices"], case["rowptr_bits"])
        self.symmetrise = case["symmetrise"]

    def build(self):
        g = b.no_build_csr(self.src, self.dst, *self.args, symmetrise=self.symmetrise)
        return list(b.no_graph_view(g)[3:])


class _HotSet:
    def __init__(self, case, seed):
        self.graph = _graph(case, seed)
        self.train = _train_ids(case, seed)
        self.n_vertices = case["vertices"]
        self.args = (case["batch"], _fanouts(case), case["epochs"], case["hot_fraction"], 2, case["hidden"], KEY)

    def select(self):
        view = b.no_cache_view(b.no_select_hot(self.graph, self.train, *self.args), self.n_vertices)
        return [view[k] for k in ("hot_ids", "slot_of_vertex", "version", "freq")]


_STATES = {"step": _Training, "superbatch": _Training, "sample": _Sampling, "gather": _Gather, "layer": _Layer, "csr": _EdgeList,
           "hot": _HotSet}


def prepare(case, seed):
    return _STATES[case["kind"]](case, seed)


def run(state):
    if isinstance(state, _Training):
        if state.super:
            state.super_batch()
        else:
            state.one_step()
        return state.out
    if isinstance(state, _Sampling):
        return state.sample()
    if isinstance(state, _Gather):
        return state.gather()
    if isinstance(state, _Layer):
        return state.forward_backward()
    if isinstance(state, _EdgeList):
        return state.build()
    return state.select()


# ------------------------------------------------------------------------------------------------------- work

def _capped_poisson(lam, k):
    """Expectation of min(X, k), X ~ Poisson(lam): neighbours drawn from a row of about lam entries."""
    if lam > 40 + 4 * k:
        return float(k)
    p = total = math.exp(-lam)
    s = 1.0 - total
    for j in range(1, k):
        p *= lam / j
        total += p
        s += max(0.0, 1.0 - total)
    return s


def _frontiers(case):
    """Expected (destinations, edges, sources) of every hop, and what the cache saves at the bottom one, (hits, refreshed rows).

    An R-MAT vertex with k set bits (before the permutation) is an endpoint with probability 0.24^k 0.76^(s - k), at either
    end: its vertices fall into s + 1 classes of equal expected degree and popularity, and m draws reach
    N_k (1 - exp(-m p_k)) of the N_k vertices of class k."""
    v, e = case["vertices"], case["edges"]
    s = max(1, math.ceil(math.log2(v)))
    count = [math.comb(s, k) * v / 2.0 ** s for k in range(s + 1)]
    p = [0.24 ** k * 0.76 ** (s - k) for k in range(s + 1)]
    norm = sum(n * q for n, q in zip(count, p))
    p = [q / norm for q in p]
    here = [case["batch"] * n / v for n in count]
    hops, hits, refreshed = [], 0.0, 0.0
    fan = _fanouts(case)
    for h, f in enumerate(fan):
        if h == len(fan) - 1 and h > 0 and case.get("hot_fraction", 0.0) > 0.0 and "staleness" in case:
            room = case["hot_fraction"] * v
            bound = case["staleness"]
            for k in range(s + 1):
                hot = max(0.0, min(1.0, room / count[k]))
                room -= hot * count[k]
                q = here[k] / count[k]
                served = hot * here[k] * bound * q / (1.0 + bound * q)
                refreshed += hot * here[k] - served
                hits += served
                here[k] -= served
        draws = sum(n * _capped_poisson(e * q, f) for n, q in zip(here, p))
        reached = [n + (c - n) * -math.expm1(-draws * q) for n, c, q in zip(here, count, p)]
        hops.append((sum(here), draws, sum(reached)))
        here = reached
    return hops, hits, refreshed


def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "gather":
        n = case["n"] - (case["n"] // 8 if case["counted"] else 0)
        return {"bytes": n * (4 + 2 * case["feat_dim"] * es), "flops": 0}
    if kind == "layer":
        n_dst, n_src, d_in, d_out = case["n_dst"], case["n_src"], case["feat_dim"], case["out_dim"]
        nnz = n_dst * case["fanout"] / 2
        products = 3 if case["input_grad"] else 2
        # sources, indices, weights, output gradient in; mean, output, gradients out
        moved = n_src * d_in * es + nnz * 4 + 4 * d_in * d_out * 4 + n_dst * (d_in + 2 * d_out) * 4
        if case["input_grad"]:
            moved += n_src * d_in * 4 + nnz * 4
        return {"bytes": moved, "flops": products * 2 * n_dst * 2 * d_in * d_out + 2 * nnz * d_in}
    rp = case["rowptr_bits"] // 8
    if kind == "csr":
        pairs = case["edges"] // (2 if case["symmetrise"] else 1)
        return {"bytes": pairs * 2 * (8 if case["ids64"] else 4) + case["edges"] * 4 + (case["vertices"] + 1) * rp, "flops": 0}
    hops, hits, refreshed = _frontiers(case)
    drawing = lambda h: h[0] * (2 * rp + 4) + h[1] * 4      # row pointers, ids and column entries read
    if kind == "hot":
        n_batches = math.ceil(max(case["batch"], int(case["vertices"] * TRAIN_SHARE)) / case["batch"])
        hot = int(case["vertices"] * case["hot_fraction"])
        per_batch = sum(drawing(h) for h in hops[:-1])
        return {"bytes": case["epochs"] * n_batches * per_batch + case["vertices"] * 8 + hot * 8 + hot * case["hidden"] * 4, "flops": 0}
    if kind == "sample":
        out = sum(h[2] * 4 + h[0] * 4 + h[1] * 8 for h in hops) + sum(h[2] * 4 + h[1] * 8 for h in hops[:-1])
        return {"bytes": sum(drawing(h) for h in hops) + out, "flops": 0}
    dims, n_mat = _dims(case), 2 if case["arch"] == "sage" else 1
    params = sum(n_mat * i * o + o for i, o in zip(dims, dims[1:]))
    # sampling, the bottom hop's feature rows, labels and seeds in, cached rows in, refreshed rows out, weights in and out, gradients
    # and logits out
    moved = (sum(drawing(h) for h in hops) + hops[-1][2] * dims[0] * es + case["batch"] * (8 + dims[-1] * 4) +
             (hits + refreshed) * case["hidden"] * 4 + params * 12)
    flops = sum((2 if layer == 1 else 3) * 2 * hops[-layer][0] * n_mat * dims[layer - 1] * dims[layer] for layer in range(1, len(dims)))
    if kind == "superbatch":
        hot = int(case["vertices"] * case["hot_fraction"])
        fan = _fanouts(case)[-1]
        moved, flops = moved * case["n_steps"], flops * case["n_steps"]
        # popular vertices have full rows; their neighbours are distinct up to the vertex count
        moved += hot * (2 * rp + 4) + hot * fan * 4 + min(case["vertices"], hot * fan) * dims[0] * es + hot * case["hidden"] * 4
        flops += 2 * hot * n_mat * dims[0] * case["hidden"]
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] in ("sample", "gather", "csr", "hot"):
        return "exact"
    if case["dtype"] == "bf16" and case["kind"] != "layer" and case["arch"] == "sage":
        return {"rel": 1e-2, "max": 0.2}       # bf16 operands in layer 1's products
    # Sums of 32-bit floats in another order (1e-5), and what follows from them: about one in a million pre-activations is
    # zero to within that rounding, and its ReLU decision then takes or leaves one row's share of a gradient.
    return {"rel": 1e-3, "max": 0.04}
