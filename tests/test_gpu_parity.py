"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same seeded
inputs. Integer outputs (CSR, sampled blocks, transposes, hot sets, cache versions, gathered
bytes) must match bit for bit; fp32 activations and gradients must satisfy
|gpu - ora| <= 1e-4 * |ora| + 1e-4 * max|ora| per tensor."""
import dataclasses

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import oracle as ora

pytestmark = pytest.mark.gpu

RTOL = 1e-4
# Steps on a bf16 feature table (GraphSAGE-mean): layer 1's products take bf16 operands on both sides, but the values
# that get rounded (the fp32 mean, the weights after an update, the output gradient) differ between the kernel (fp32)
# and the oracle (fp64) in their last bits, and now and then one of them sits on a bf16 rounding boundary: one operand
# of one of a product's 2K terms is then off by a bf16 ulp (2^-8 of its size), i.e. an output by up to ~2^-8 / sqrt(2K)
# of its typical size (3e-4 at K = 64). Tolerance for such runs (well inside the 2e-2 allowed for bf16 features):
RTOL_BF16 = 1e-3
# Whole-step tests let the oracle's backward pass take the kernel's ReLU decision where the oracle's own
# pre-activation is zero to within rounding (|z| <= 1e-5 max|z|); how many decisions that may be is bounded:
RELU_FLIP_SHARE = 1e-5      # of a layer's pre-activations (observed at full size: about 1e-6)
RELU_FLIP_FLOOR = 2


def nb():
    from paper_2311_13225_amd import binding
    return binding


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def assert_close(gpu, ref, what="", rtol=RTOL):
    gpu = np.asarray(gpu, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert gpu.shape == ref.shape, (what, gpu.shape, ref.shape)
    if ref.size == 0:
        return
    tol = rtol * np.abs(ref) + rtol * np.abs(ref).max()
    err = np.abs(gpu - ref)
    bad = err > tol
    assert not bad.any(), "%s: %d of %d outside tolerance, worst err %.3e (tol %.3e)" % (
        what, bad.sum(), ref.size, err.max(), tol[np.unravel_index(err.argmax(), err.shape)])


def make_graph(V, E, seed, bits, symmetrise=False):
    src, dst = si.rmat_edges(V, E, seed, symmetrise=symmetrise)
    og = ora.build_csr(src, dst, V)
    gg = nb().no_build_csr(src, dst, V, bits)
    return src, dst, og, gg


# --------------------------------------------------------------------------------------- CSR

@pytest.mark.parametrize("V,E,bits", [(50, 0, 32), (1, 5, 64), (300, 4000, 32), (10_000, 100_000, 64),
                                      (70_000, 1_500_000, 32)])
def test_build_csr_matches_oracle(V, E, bits):
    print("case", V, E, bits, flush=True)
    src, dst, og, gg = make_graph(V, E, 1, bits)
    v, e, b, rowptr, col = nb().no_graph_view(gg)
    assert (v, e, b) == (V, E, bits)
    assert np.array_equal(rowptr.cpu().numpy().astype(np.int64), og.rowptr)
    if E:
        assert np.array_equal(col.cpu().numpy(), og.col)


@pytest.mark.parametrize("V,E,symmetrise,ids64", [
    (2, 8191, False, False), (513, 8192, False, True), (512, 8193, True, False),      # tiles of 8192 edges, digits of up to 9 bits
    (600_000, 4_300_001, False, False),     # more tiles than chunks, three passes a key
    (70_001, 2_150_003, True, True)])       # the two directions meet inside a thread's run, off 16-byte alignment
def test_build_csr_tile_and_digit_edges(V, E, symmetrise, ids64):
    rng = np.random.default_rng(5)
    src = rng.integers(0, V, E).astype(np.int32)
    dst = (rng.integers(0, V, E) * rng.integers(0, 2, E)).astype(np.int32)       # half of all edges meet in vertex 0
    og = ora.build_csr(src, dst, V, symmetrise=symmetrise)
    ids = np.int64 if ids64 else np.int32
    rowptr, col = nb().no_graph_view(nb().no_build_csr(dev(src.astype(ids)), dev(dst.astype(ids)), V, 64, symmetrise=symmetrise))[3:]
    assert np.array_equal(rowptr.cpu().numpy(), og.rowptr)
    assert np.array_equal(col.cpu().numpy(), og.col)


def test_graphs_built_and_destroyed_by_several_threads():
    """The library's memory is reused across calls: threads with streams of their own must never share a block in use."""
    import threading
    wrong = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(6):
                V, E = 3000 + 997 * i, 40_000 + 9001 * k
                src, dst = si.random_graph_small(V, E, 10 * i + k)
                og = ora.build_csr(src, dst, V)
                gg = nb().no_build_csr(dev(src), dev(dst), V, 64)
                rowptr, col = nb().no_graph_view(gg)[3:]
                if not (np.array_equal(rowptr.cpu().numpy(), og.rowptr) and np.array_equal(col.cpu().numpy(), og.col)):
                    wrong.append((i, k))
                del rowptr, col, gg

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_memory_is_kept_only_while_a_handle_exists():
    """Neither the temporaries of a build that fails nor the memory of the last graph stay with the library."""
    import gc
    b = nb()
    gc.collect()
    src, dst = (np.random.default_rng(i).integers(0, 1000, 20_000_000, dtype=np.int32) for i in range(2))
    bad = src.copy()
    bad[5] = -1

    def fail(n):
        with pytest.raises(b.NoError):
            b.no_build_csr(bad[:n], dst[:n], 1000, 32)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    free = fail(100)
    assert free - fail(len(bad)) < 64 << 20              # (its temporaries: 16 bytes an edge)
    gg = b.no_build_csr(src, dst, 1000, 32)
    assert free - torch.cuda.mem_get_info()[0] >= 4 * len(src)
    gg.close()
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20


def test_build_csr_from_device_and_rejects_bad_ids():
    src, dst = si.rmat_edges(500, 5000, 2)
    og = ora.build_csr(src, dst, 500)
    gg = nb().no_build_csr(dev(src), dev(dst), 500, 64)
    assert np.array_equal(nb().no_graph_view(gg)[4].cpu().numpy(), og.col)
    bad = src.copy()
    bad[7] = 500
    with pytest.raises(nb().NoError) as ei:
        nb().no_build_csr(bad, dst, 500, 64)
    assert ei.value.code == -2
    with pytest.raises(nb().NoError):
        nb().no_build_csr(src, dst, 500, 48)


@pytest.mark.parametrize("V,dedup", [(1, False), (3, True), (512, False), (513, True), (8192, False), (8193, True), (1 << 18, False),
                                     ((1 << 18) + 1, True), (1 << 22, False), ((1 << 22) + 1, False)])
def test_build_csr_digits_within_and_across_the_ids(V, dedup):
    # 2 * 9, 2 * 13 and 2 * 22 bits are the most for 2, 3 and 5 passes: a digit across both ids, or none, on each side of these
    print("case", V, dedup, flush=True)
    rng = np.random.default_rng(V)
    E = 40_001
    src, dst = (rng.choice(np.concatenate([rng.integers(0, V, 300), V - 1 - rng.integers(0, min(V, 300), 300)]), E).astype(np.int32)
                for _ in range(2))
    og = ora.build_csr(src, dst, V, dedup=dedup)
    rowptr, col = nb().no_graph_view(nb().no_build_csr(dev(src), dev(dst), V, 32, dedup=dedup))[3:]
    assert np.array_equal(rowptr.cpu().numpy().astype(np.int64), og.rowptr)
    assert np.array_equal(col.cpu().numpy()[:len(og.col)], og.col)


@pytest.mark.parametrize("symmetrise,dedup,ids64,on_device", [(True, False, False, False), (False, True, False, True),
                                                              (True, True, True, False), (False, False, True, True)])
def test_build_csr_flags(symmetrise, dedup, ids64, on_device):
    """Optional preparations of the edge list: both directions, duplicates dropped, 64-bit ids on input."""
    b = nb()
    V, E = 5000, 120_000
    src, dst = si.rmat_edges(V, E, 3)
    og = ora.build_csr(src, dst, V, symmetrise=symmetrise, dedup=dedup)
    s_in, d_in = (src.astype(np.int64), dst.astype(np.int64)) if ids64 else (src, dst)
    if on_device:
        s_in, d_in = dev(s_in), dev(d_in)
    gg = b.no_build_csr(s_in, d_in, V, 64, symmetrise=symmetrise, dedup=dedup)
    v, e, bits, rowptr, col = b.no_graph_view(gg)
    assert e == og.n_edges and (not dedup or e < (2 * E if symmetrise else E))
    assert np.array_equal(rowptr.cpu().numpy(), og.rowptr)
    assert np.array_equal(col.cpu().numpy()[:e], og.col)
    if ids64:
        bad = src.astype(np.int64)
        bad[11] = 1 << 40
        with pytest.raises(b.NoError) as ei:
            b.no_build_csr(bad, dst.astype(np.int64), V, 64)
        assert ei.value.code == -2


# --------------------------------------------------------------------------------------- sampling

def compare_blocks(b, blocks, sb, with_cache=False):
    sizes = b.no_blocks_sizes(blocks)
    L = len(sb.blocks)
    for h, ob in enumerate(sb.blocks):
        assert sizes[h, 0] == ob.n_dst and sizes[h, 1] == ob.n_src and sizes[h, 2] == ob.nnz, (h, sizes[h], ob.n_dst, ob.n_src, ob.nnz)
        ga = b.block_arrays(blocks, h, sizes)
        for name in ["dst_global", "src_global", "indptr", "nbr_global", "indices"]:
            assert np.array_equal(ga[name], getattr(ob, name)), (h, name)
        if h < L - 1:
            for name in ["csc_indptr", "csc_dst", "csc_eid"]:
                assert np.array_equal(ga[name], getattr(ob, name)), (h, name)
        else:
            assert ga["csc_indptr"] is None
        if with_cache and h == L - 1:
            assert sizes[h, 3] == len(sb.hit_pos)
            assert np.array_equal(ga["compute_pos"], sb.compute_pos)
            assert np.array_equal(ga["hit_pos"], sb.hit_pos)
            assert np.array_equal(ga["hit_slot"], sb.hit_slot)
    return sizes


@pytest.mark.parametrize("bits", [32, 64])
def test_sample_blocks_tiny_config(bits):
    b = nb()
    w = si.WORKLOADS["tiny"]
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, bits)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    blocks = b.no_blocks_create(gg, w.batch, w.fanouts)
    for step in [0, 1, 7]:
        seeds = si.batch_seeds(train, w.batch, step)
        b.no_sample_blocks(gg, dev(seeds), 0, step, None, blocks)
        compare_blocks(b, blocks, ora.sample_blocks(og, seeds, w.fanouts, 0, step))
    # ragged batch smaller than the capacity, other seed
    seeds = train[:37].copy()
    b.no_sample_blocks(gg, dev(seeds), 12345678901234567, 3, None, blocks)
    compare_blocks(b, blocks, ora.sample_blocks(og, seeds, w.fanouts, 12345678901234567, 3))


@pytest.mark.parametrize("fanouts", [(1,), (3, 2), (8, 8), (9, 16, 2), (17, 5), (32, 3), (33, 2), (64,), (25, 10)])
def test_sample_blocks_group_widths_and_dense_rows(fanouts):
    """Every lane-group width (8/16/32/64), rows shorter and much longer than the fanout."""
    b = nb()
    V = 3000
    src, dst, og, gg = make_graph(V, 150_000, 5, 64)
    train = si.train_split(V, 0.65, 5)
    cap = 64 if len(fanouts) < 3 else 16
    blocks = b.no_blocks_create(gg, cap, fanouts)
    for step in range(2):
        seeds = si.batch_seeds(train, cap, step)
        b.no_sample_blocks(gg, dev(seeds), 99, step, None, blocks)
        compare_blocks(b, blocks, ora.sample_blocks(og, seeds, fanouts, 99, step))


def test_sample_blocks_sparse_graph_with_isolated_vertices():
    b = nb()
    V = 5000
    src, dst, og, gg = make_graph(V, 6000, 9, 32)
    seeds = si.train_split(V, 0.9, 9)[:512]
    blocks = b.no_blocks_create(gg, 512, (5, 5, 5))
    b.no_sample_blocks(gg, dev(seeds), 1, 0, None, blocks)
    sizes = compare_blocks(b, blocks, ora.sample_blocks(og, seeds, (5, 5, 5), 1, 0))
    assert sizes[0, 2] < 512 * 5       # some rows are short or empty


def test_sample_blocks_rejects_bad_arguments():
    b = nb()
    src, dst, og, gg = make_graph(300, 2000, 1, 32)
    blocks = b.no_blocks_create(gg, 8, (2, 2))
    seeds = dev(np.arange(9, dtype=np.int32))
    with pytest.raises(b.NoError) as ei:
        b.no_sample_blocks(gg, seeds, 0, 0, None, blocks)
    assert ei.value.code == -3
    with pytest.raises(b.NoError):
        b.no_blocks_create(gg, 8, (0, 2))
    with pytest.raises(b.NoError):
        b.no_blocks_create(gg, 8, (65,))


# --------------------------------------------------------------------------------------- hot set

@pytest.mark.parametrize("fanouts,frac", [((10, 5), 0.05), ((4, 3, 2), 0.1), ((6,), 0.2)])
def test_select_hot_matches_oracle(fanouts, frac):
    b = nb()
    V = 10_000
    src, dst, og, gg = make_graph(V, 100_000, 0, 32)
    train = si.train_split(V, 0.3, 0)
    oc = ora.select_hot(og, train, 256, fanouts, 2, frac, 1, 16, 42)
    gc = b.no_select_hot(gg, dev(train), 256, fanouts, 2, frac, 1, 16, 42)
    view = b.no_cache_view(gc, V)
    assert view["n_hot"] == oc.n_hot and view["emb_dim"] == 16 and view["staleness"] == 1
    assert np.array_equal(view["freq"].cpu().numpy().astype(np.int64), oc.freq)
    assert np.array_equal(view["hot_ids"].cpu().numpy(), oc.hot_ids)
    assert np.array_equal(view["slot_of_vertex"].cpu().numpy(), oc.slot_of_vertex)
    assert (view["version"].cpu().numpy() == -1).all()
    assert not view["emb"].cpu().numpy().any()


@pytest.mark.parametrize("V,E,n_train,batch,fanouts,bits", [
    (1003, 20_000, 651, 1, (4, 3), 32),            # more batches than a counter of the bitmap count holds, a last word of 11 vertices
    (1003, 20_000, 650, 3, (33, 5, 2), 64),        # a lane group per row as wide as a wavefront, a ragged last batch
    (4096, 60_000, 4096, 1500, (17, 9, 4), 64),    # a batch of more seeds than a workgroup has threads
    (10_000, 100_000, 9_000, 9_000, (10, 5), 32)]) # one large batch: spread over the chip by the training sampler
def test_select_hot_batch_counts_and_sizes(V, E, n_train, batch, fanouts, bits):
    b = nb()
    src, dst, og, gg = make_graph(V, E, 3, bits)
    train = si.train_split(V, 1.0, 3)[:n_train]
    oc = ora.select_hot(og, train, batch, fanouts, 1, 0.25, 1, 4, 9)
    view = b.no_cache_view(b.no_select_hot(gg, dev(train), batch, fanouts, 1, 0.25, 1, 4, 9), V)
    assert np.array_equal(view["freq"].cpu().numpy().astype(np.int64), oc.freq)
    assert np.array_equal(view["hot_ids"].cpu().numpy(), oc.hot_ids)


@pytest.mark.parametrize("V,fanouts,batch", [
    (1_245_184, (16, 4, 2), 256),      # the most vertices that one bitmap in LDS holds; a thread draws 16 slots at most
    (1_245_185, (17, 3, 2), 256),      # two parts, and 17 slots
    (2_500_000, (32, 2), 4),           # room for three parts, but few seeds a batch: bitmaps in memory, more batches than compute units
    (4_980_736, (5, 16, 2), 256),      # four full parts
    (4_980_737, (5, 5, 2), 256),       # one vertex too many: bitmaps in memory
    (1_300_000, (33, 2), 256)])        # one slot too many: bitmaps in memory
def test_select_hot_bitmaps_in_parts(V, fanouts, batch):
    check_hot_against_oracle(V, fanouts, batch, 2)


@pytest.mark.parametrize("V,fanouts,batch,epochs", [
    (2_500_000, (32, 3, 2), 256, 1),   # three parts, 32 slots: just too few of them for LDS
    (2_500_000, (32, 4, 2), 256, 1),   # enough
    (2_500_000, (32, 4, 2), 256, 70),  # more batches than workgroups
    (1_245_184, (16, 4, 2), 31, 1), (1_245_184, (16, 4, 2), 32, 1),            # one part: the least seeds a batch
    (1_245_184, (5, 5, 2), 35, 1), (1_245_184, (5, 5, 2), 36, 1),              # and slots
    (1_245_185, (7, 2, 2), 108, 1), (1_245_185, (7, 2, 2), 109, 1),            # two parts
    (1_245_185, (17, 16, 2), 78, 1), (1_245_185, (17, 16, 2), 79, 1)])         # and wide rows
def test_select_hot_bitmaps_in_lds_and_in_memory(V, fanouts, batch, epochs):
    check_hot_against_oracle(V, fanouts, batch, epochs)


def check_hot_against_oracle(V, fanouts, batch, epochs):
    b = nb()
    rng = np.random.default_rng(V)
    E = 3_000_000                      # most vertices have a few neighbours, some thousands have far more than a draw takes
    dst = np.where(rng.random(E) < 0.5, rng.integers(0, 5000, E) * (V // 5000), rng.integers(0, V, E)).astype(np.int32)
    src = np.where(rng.random(E) < 0.5, rng.integers(0, 5000, E) * (V // 5000) + V // 5000 - 1, rng.integers(0, V, E)).astype(np.int32)
    og, gg = ora.build_csr(src, dst, V), b.no_build_csr(dev(src), dev(dst), V, 32)
    train = np.concatenate([rng.choice(5000, 900, replace=False) * (V // 5000), [0, 1, V - 1, V - 2]])
    train = np.unique(train).astype(np.int32)
    rng.shuffle(train)
    print("V %d, %d train ids" % (V, len(train)), flush=True)
    oc = ora.select_hot(og, train, batch, fanouts, epochs, 0.01, 1, 4, 5)
    view = b.no_cache_view(b.no_select_hot(gg, dev(train), batch, fanouts, epochs, 0.01, 1, 4, 5), V)
    assert oc.freq.max() > 1 and (oc.freq > 0).sum() > 5000
    assert np.array_equal(view["freq"].cpu().numpy().astype(np.int64), oc.freq)
    assert np.array_equal(view["hot_ids"].cpu().numpy(), oc.hot_ids)


@pytest.mark.parametrize("V,batch,n_batches", [
    (130, 2, 17),                      # two bitmaps and a bit for each wavefront that shares them
    (10_000, 3, 2),                    # fewer bitmaps than wavefronts
    (10_000, 1, 2100),                 # 263 for each: three rounds of what seven planes hold
    (3_145_600, 4, 121), (3_145_600, 4, 122),      # small batches: too few to share, just enough
    (3_145_729, 4, 130),               # too long to share
    (3_200_000, 1, 8320),              # 520 in a launch: more than nine planes hold
    (4_980_736, 8192, 51), (4_980_736, 8192, 52)])      # large batches: too few, just enough
def test_select_hot_counts_of_few_and_many_bitmaps(V, batch, n_batches):
    """Every vertex has one in-neighbour, so a batch's V^1 is its seeds and theirs; one seed is in nine batches of ten or more."""
    b = nb()
    rng = np.random.default_rng(V + n_batches)
    parent = rng.integers(0, V, V).astype(np.int32)
    train = np.where(rng.random(batch * n_batches) < 0.9, V // 3, rng.integers(0, V, batch * n_batches)).astype(np.int32)
    print("V %d, %d batches of %d" % (V, n_batches, batch), flush=True)
    job = np.repeat(np.arange(n_batches, dtype=np.int64), batch)
    met = np.unique(np.concatenate([job * V + train, job * V + parent[train]]))
    freq = np.bincount(met % V, minlength=V)
    gg = b.no_build_csr(dev(parent), dev(np.arange(V, dtype=np.int32)), V, 32)
    view = b.no_cache_view(b.no_select_hot(gg, dev(train), batch, (2, 1), 1, 0.01, 1, 4, 5), V)
    assert freq.max() > 0.8 * n_batches
    assert np.array_equal(view["freq"].cpu().numpy().astype(np.int64), freq)
    assert np.array_equal(view["hot_ids"].cpu().numpy(), np.lexsort((np.arange(V), -freq))[:V // 100])


@pytest.mark.parametrize("fanouts", [(10, 5), (6,)])
@pytest.mark.parametrize("batch", [100, 9_000])       # batches by bitmap; one large batch, by the training sampler
def test_select_hot_counts_a_repeated_train_id_once_a_batch(fanouts, batch):
    """Against the oracle's counts batch by batch, of the ids without repetition (a draw depends on the vertex, not on its place)."""
    b = nb()
    V, epochs = 10_000, 2
    src, dst, og, gg = make_graph(V, 100_000, 3, 32)
    train = si.train_split(V, 1.0, 3)[:9_000].copy()
    train[1::50] = train[::50]                            # next to each other
    train[8_999], train[7] = train[8_901], train[8_999]   # far apart, and in two batches
    n_batches = -(-len(train) // batch)
    freq = np.zeros(V, np.int64)
    for job in range(epochs * n_batches):
        ids = train[job % n_batches * batch:][:batch]
        ids = ids[np.sort(np.unique(ids, return_index=True)[1])]
        freq += ora.presample_counts(og, ids, len(ids), fanouts, 1, 9 + job)
    view = b.no_cache_view(b.no_select_hot(gg, dev(train), batch, fanouts, epochs, 0.25, 1, 4, 9), V)
    assert np.array_equal(view["freq"].cpu().numpy().astype(np.int64), freq)
    assert np.array_equal(view["hot_ids"].cpu().numpy(), np.lexsort((np.arange(V), -freq))[:V // 4])


def test_sample_blocks_with_cache_lookup():
    b = nb()
    w = si.WORKLOADS["tiny"]
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    oc = ora.select_hot(og, train, w.batch, w.fanouts, 1, 0.2, 2, 8, 0)
    gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, 0.2, 2, 8, 0)
    rng = np.random.default_rng(0)
    ver = rng.integers(-1, 6, oc.n_hot).astype(np.int32)       # empty, fresh and stale slots
    oc.version[:] = ver
    b.no_cache_view(gc, w.n_vertices)["version"].copy_(dev(ver))
    blocks = b.no_blocks_create(gg, w.batch, w.fanouts)
    total_hits = 0
    for step in [5, 6, 9]:
        seeds = si.batch_seeds(train, w.batch, step)
        b.no_sample_blocks(gg, dev(seeds), 0, step, gc, blocks)
        sb = ora.sample_blocks(og, seeds, w.fanouts, 0, step, oc)
        compare_blocks(b, blocks, sb, with_cache=True)
        total_hits += len(sb.hit_pos)
    assert total_hits > 0


@pytest.mark.parametrize("V,batch", [
    (262_144, 8192),      # 248 tiles of slots, 256 of V^1 (as many as there are vertices): both scans in one launch
    (300_000, 8200),      # 249 and 257: the split of V^1 in two launches
    (250_000, 8457),      # 257 and 253: the compaction in two
    (300_000, 8457)])     # 257 and 265: both in two
def test_sample_blocks_scans_in_one_launch_and_in_two(V, batch):
    b = nb()
    fanouts = (31, 3)
    slots, v1 = batch * 31, min(batch * 32, V + batch)      # (room for: a batch of different seeds may have as many)
    expected = {(262_144, 8192): (1, 1), (300_000, 8200): (1, 2), (250_000, 8457): (2, 1), (300_000, 8457): (2, 2)}[V, batch]
    assert tuple(1 if -(-n // 1024) <= 256 else 2 for n in (slots, v1)) == expected
    src, dst, og, gg = make_graph(V, 8 * V, 3, 32)
    train = si.train_split(V, 0.65, 3)
    oc = ora.select_hot(og, train[:4096], 1024, fanouts, 1, 0.2, 2, 8, 0)
    gc = b.no_select_hot(gg, dev(train[:4096]), 1024, fanouts, 1, 0.2, 2, 8, 0)
    ver = np.random.default_rng(1).integers(-1, 6, oc.n_hot).astype(np.int32)
    oc.version[:] = ver
    b.no_cache_view(gc, V)["version"].copy_(dev(ver))
    blocks = b.no_blocks_create(gg, batch, fanouts)
    for step, n in [(5, batch), (6, batch - 37), (7, 1)]:
        seeds = train[:n].copy()
        print("V %d, %d of %d seeds" % (V, n, batch), flush=True)
        for with_cache in (True, False):
            b.no_sample_blocks(gg, dev(seeds), 0, step, gc if with_cache else None, blocks)
            compare_blocks(b, blocks, ora.sample_blocks(og, seeds, fanouts, 0, step, oc if with_cache else None), with_cache=with_cache)


@pytest.mark.parametrize("V,E,batch,fanouts", [
    (600_000, 3_000_000, 400_000, (64,)),             # 25,000 tiles of slots: their sums by a launch of their own
    (26_000_000, 4_000_000, 450_000, (64, 2))])       # and room for as many of V^1
def test_sample_blocks_scans_of_very_many_tiles(V, E, batch, fanouts):
    b = nb()
    rng = np.random.default_rng(E)
    src, dst = (rng.integers(0, V, E).astype(np.int32) for _ in range(2))
    dst[:E // 4] = rng.integers(0, 2000, E // 4)      # (some rows of more entries than a draw takes)
    og, gg = ora.build_csr(src, dst, V), b.no_build_csr(dev(src), dev(dst), V, 32)
    seeds = np.concatenate([np.arange(2000, dtype=np.int32), 2000 + rng.permutation(V - 2000)[:batch - 2000].astype(np.int32)])
    assert batch * 64 > 24_576 * 1024 and (len(fanouts) == 1 or min(batch * 65, V + batch) > 24_576 * 1024)
    oc = gc = None
    if len(fanouts) > 1:
        args = (1024, fanouts, 1, 0.02, 2, 8, 0)
        oc, gc = ora.select_hot(og, seeds[:4096], *args), b.no_select_hot(gg, dev(seeds[:4096]), *args)
        oc.version[:] = np.random.default_rng(1).integers(-1, 6, oc.n_hot)
        b.no_cache_view(gc, V)["version"].copy_(dev(oc.version.astype(np.int32)))
    blocks = b.no_blocks_create(gg, batch, fanouts)
    for step, n in [(5, batch), (6, 3)]:
        print("V %d, %d of %d seeds" % (V, n, batch), flush=True)
        b.no_sample_blocks(gg, dev(seeds[:n]), 0, step, gc, blocks)
        compare_blocks(b, blocks, ora.sample_blocks(og, seeds[:n], fanouts, 0, step, oc), with_cache=oc is not None)


# --------------------------------------------------------------------------------------- gather

@pytest.mark.parametrize("dim,dtype", [(64, "f32"), (602, "f32"), (100, "f32"), (7, "f32"), (256, "f32"),
                                       (128, "bf16"), (6, "bf16"), (5, "bf16")])
def test_gather_is_bit_copy(dim, dtype):
    b = nb()
    V, n = 5000, 3001
    table = si.features(V, dim, 3, dtype)
    ids = np.random.default_rng(1).integers(0, V, n).astype(np.int32)
    t = dev(table.view(np.int16) if dtype == "bf16" else table)
    out = b.no_gather_features(t, dev(ids))
    assert np.array_equal(out.cpu().numpy().view(table.dtype), ora.gather_features(table, ids))
    # device-side count: only the first rows are written
    out2 = torch.zeros_like(out)
    b.no_gather_features(t, dev(ids), out2, dev(np.array([1234], np.int32)))
    got = out2.cpu().numpy().view(table.dtype)
    assert np.array_equal(got[:1234], table[ids[:1234]]) and not got[1234:].any()
    b.no_gather_features(t, dev(ids), out2, dev(np.array([0], np.int32)))


# --------------------------------------------------------------------------------------- layers

def layer_case(V, E, F, d_out, fanouts, B, seed, bf16=False, edges=None, seeds=None):
    src, dst = edges if edges is not None else si.rmat_edges(V, E, seed)
    og = ora.build_csr(src, dst, V)
    if seeds is None:
        seeds = si.train_split(V, 0.65, seed)[:B]
    sb = ora.sample_blocks(og, seeds, fanouts, seed, 0)
    blk = sb.blocks[-1]
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((blk.n_src, F)).astype(np.float32)
    if bf16:
        xb = si.f32_to_bf16_bits(x)
        x = si.bf16_bits_to_f32(xb)
    else:
        xb = None
    (w_self, w_neigh, bias), = si.init_weights([F, d_out], seed)
    return blk, x, xb, w_self, w_neigh, bias, rng


@pytest.mark.parametrize("F,d_out,relu,bf16", [(64, 64, True, False), (602, 256, True, False), (100, 47, False, False),
                                               (33, 5, True, False), (256, 130, True, False), (128, 256, True, True),
                                               (6, 3, False, True), (40, 200, True, False), (70, 41, False, False),
                                               (256, 41, False, False), (200, 50, True, False), (256, 256, True, True)])
def test_sage_layer_forward_backward(F, d_out, relu, bf16):
    check_layer_forward_backward(layer_case(4000, 60_000, F, d_out, (7, 6), 300, 11, bf16), F, d_out, relu, bf16)


@pytest.mark.parametrize("n,cap,F,d_out", [
    (0, 5000, 64, 64), (1, 5000, 8, 256), (31, 5000, 9, 100), (33, 9000, 33, 48), (63, 5000, 128, 128),      # fewer rows than a step or a tile
    (257, 5000, 129, 65), (1000, 30_000, 100, 256), (5001, 30_000, 66, 7),                                   # remainders of every tile size
    (4097, 4097, 127, 129), (9000, 9000, 3, 130), (20_100, 30_000, 130, 172),                               # large tiles; a layer of 3 columns
    (2500, 2500, 1800, 1792), (700, 700, 1800, 1790), (20, 70, 9000, 9), (5001, 9000, 66, 5),                                 # few slices: planes in the rows' place too; no planes
    (20_100, 30_000, 130, 32), (20_100, 30_000, 32, 130), (20_100, 30_000, 130, 33), (9000, 30_000, 2, 1),                   # narrow: small tiles at every number of rows
    (65, 65, 64, 64), (130, 5000, 64, 64), (2049, 5000, 64, 64), (4200, 5000, 64, 30), (300, 300, 602, 40)])                       # slices of 64 rows and their remainders
def test_sage_layer_gradient_products_at_tile_edges(n, cap, F, d_out):
    """Weight and input gradients against exact sums. Bound: every term of a sum of K products may be off by the rounding of
    one fp32 product and every addition by that of its partial sum, together below (K + 8) 2^-24 sum |a b|."""
    b = nb()
    rng = np.random.default_rng(n + F)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    x, mean, gh, w_self, w_neigh = f32(cap, F), f32(cap, F), f32(cap, d_out), f32(F, d_out), f32(F, d_out)
    i32 = lambda a: dev(np.asarray(a, np.int32))
    # row v samples itself once; source u is sampled by row u
    blk = b.block_view_from_tensors(i32([n]), i32([n]), i32(np.minimum(np.arange(cap + 1), n)), i32(np.arange(cap)), cap, cap,
                                    i32(np.minimum(np.arange(cap + 1), n)), i32(np.arange(cap)))
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    gs, gn, gb, gx = (torch.full(s, float("nan"), device="cuda") for s in ((F, d_out), (F, d_out), (d_out,), (cap, F)))
    b.no_sage_layer_bwd(blk, dev(x), dev(mean), dev(gh), dev(gh), dev(w_self), dev(w_neigh), False, gs, gn, gb, gx, ws)
    x, mean, gh = (a[:n].astype(np.float64) for a in (x, mean, gh))
    w = w_self.astype(np.float64) + w_neigh.astype(np.float64)
    w_abs = np.abs(w_self).astype(np.float64) + np.abs(w_neigh)
    for got, ref, mag, terms in ((gs, x.T @ gh, np.abs(x).T @ np.abs(gh), n), (gn, mean.T @ gh, np.abs(mean).T @ np.abs(gh), n),
                                 (gb, gh.sum(0), np.abs(gh).sum(0), n), (gx[:n], gh @ w.T, np.abs(gh) @ w_abs.T, 2 * d_out)):
        assert (np.abs(got.cpu().numpy() - ref) <= (terms + 8) * 2.0 ** -24 * mag).all()
    assert torch.isnan(gx[n:]).all()


@pytest.mark.parametrize("n,cap,F,d_out", [
    (13_990, 14_000, 256, 250), (19_990, 20_000, 256, 256), (20_004, 20_004, 250, 256), (1, 20_000, 256, 256),     # input and weight gradients in one launch, or not
    (40_000, 40_000, 100, 256), (40_010, 40_010, 100, 250),                                                     # the same with blocks of 64 rows
    (28_000, 28_000, 64, 256), (28_010, 28_010, 63, 250)])                                                     # narrow input gradient: small tiles alone, or large ones
def test_sage_layer_gradient_products_about_the_longest_short_launches(n, cap, F, d_out):
    """Sizes about which a layer call stops to take small tiles for its weight gradients, beside the input gradient and alone. Bound as above."""
    test_sage_layer_gradient_products_at_tile_edges(n, cap, F, d_out)


def forward_layer(b, n, cap, x, w_self, w_neigh, bias, relu):
    """One layer whose row v samples itself: the mean is x, h = act(x (W_self + W_neigh) + bias)."""
    F, d_out = w_self.shape
    i32 = lambda a: dev(np.asarray(a, np.int32))
    blk = b.block_view_from_tensors(i32([n]), i32([n]), i32(np.minimum(np.arange(cap + 1), n)), i32(np.arange(cap)), cap, cap)
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    mean, h = torch.empty((cap, F), device="cuda"), torch.full((cap, d_out), -7.0, device="cuda")
    b.no_sage_layer_fwd(blk, dev(x), dev(w_self), dev(w_neigh), dev(bias), relu, mean, h, ws)
    return h


def forward_error(h, ref):
    return np.linalg.norm(h - ref) / np.linalg.norm(ref)


def forward_error_bound(K):
    """Relative 2-norm error of sums of K products on pieces. A chain of 6 K / 16 additions rounds each to 2^-24 of a partial sum at most: taken as
    independent, below 2^-24 sqrt(6 K / 16) / 2, and two roundings for the bias and the output. (A product without one of the six partial products
    is off by 1.2e-6 and more: the middle pieces are about 2^-9 / sqrt(3) of their operands, 1.3e-6 together; the small ones 2^-17.)"""
    return 2.0 ** -24 * (1.0 + np.sqrt(6 * K / 16) / 2)


@pytest.mark.parametrize("n,cap,F,d_out", [
    (1, 9000, 256, 256), (63, 42_000, 8, 256), (65, 41_000, 9, 250),             # fewer rows than a tile; the shortest reductions
    (4096, 30_000, 31, 256), (4097, 30_000, 33, 256), (8200, 36_000, 40, 129),  # the last row of small tiles in one round, the first beyond
    (8193, 22_000, 64, 193), (32_800, 81_000, 70, 47), (16_500, 16_500, 602, 130),   # remainders of both tile sizes and of the steps
    (9600, 9600, 200, 256), (9536, 9536, 200, 256), (42_000, 42_000, 7, 256),   # the least work for planes, a row of tiles less; too few columns
    (8192, 8192, 3000, 256)])                                                    # planes of a layer as wide as it has rows
def test_sage_layer_forward_products_at_tile_edges(n, cap, F, d_out):
    """Against exact sums. Bound as for the gradients: (K + 8) 2^-24 sum |a b| (the bias among the terms)."""
    b = nb()
    rng = np.random.default_rng(n + F)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    x, w_self, w_neigh, bias = f32(cap, F), f32(F, d_out), f32(F, d_out), f32(d_out)
    for relu in (False, True):
        h = forward_layer(b, n, cap, x, w_self, w_neigh, bias, relu).cpu().numpy()
        x64 = x[:n].astype(np.float64)
        ref = x64 @ w_self.astype(np.float64) + x64 @ w_neigh.astype(np.float64) + bias
        mag = np.abs(x64) @ (np.abs(w_self).astype(np.float64) + np.abs(w_neigh)) + np.abs(bias)
        assert (np.abs(h[:n] - (np.maximum(ref, 0.0) if relu else ref)) <= (2 * F + 9) * 2.0 ** -24 * mag).all()
        assert (h[n:] == -7.0).all()
        if not relu:
            assert forward_error(h[:n], ref) <= forward_error_bound(2 * F)


@pytest.mark.parametrize("n,cap,F,d_out", [
    (1, 12_000, 400, 256), (65, 12_000, 410, 250),                       # fewer rows than a tile, a tile and a row
    (17_300, 17_301, 150, 256), (17_200, 17_200, 149, 256),              # about the least work for planes with one product
    (29_000, 29_000, 128, 129), (90_000, 90_000, 127, 129),              # a column tile that is half empty: the least reduction, one less
    (16_500, 22_000, 602, 130), (8_193, 33_000, 333, 100), (20_000, 20_000, 300, 64)])
def test_gcn_layer_forward_products_at_tile_edges(n, cap, F, d_out):
    """One matrix. Rows that sample nothing: the aggregate is the row itself. Bounds as above."""
    b = nb()
    rng = np.random.default_rng(n + F)
    x, w, bias = (rng.standard_normal(sh).astype(np.float32) for sh in ((cap, F), (F, d_out), d_out))
    i32 = lambda a: dev(np.asarray(a, np.int32))
    blk = b.block_view_from_tensors(i32([n]), i32([n]), i32(np.zeros(cap + 1)), i32(np.zeros(1)), cap, cap)
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    agg, h = torch.empty((cap, F), device="cuda"), torch.full((cap, d_out), -7.0, device="cuda")
    ref = x[:n].astype(np.float64) @ w + bias
    mag = np.abs(x[:n]).astype(np.float64) @ np.abs(w) + np.abs(bias)
    for _ in range(2):                                                   # (a second call finds the first one's planes in the workspace)
        print("one product", n, cap, F, d_out, flush=True)
        b.no_gcn_layer_fwd(blk, dev(x), dev(w), dev(bias), False, agg, h, ws)
        got = h.cpu().numpy()
        assert (np.abs(got[:n] - ref) <= (F + 9) * 2.0 ** -24 * mag).all() and (got[n:] == -7.0).all()
        assert forward_error(got[:n], ref) <= forward_error_bound(F)
        w, ref = -w, 2.0 * bias.astype(np.float64) - ref


@pytest.mark.parametrize("n,cap,F,d_out", [(4750, 4801, 200, 256), (4700, 4736, 200, 256), (2900, 2945, 201, 190), (11_140, 11_140, 64, 250), (1, 4801, 300, 256),
                                           (31_990, 32_000, 16, 256), (41_500, 41_600, 8, 250), (42_000, 42_000, 100, 128)])
def test_sage_layer_forward_products_from_the_fewest_tiles_on(n, cap, F, d_out):
    """Sizes about which a layer call takes its product to planes, whose weights the aggregation's launch cuts. Bounds as above."""
    test_sage_layer_forward_products_at_tile_edges(n, cap, F, d_out)


def test_sage_layer_forward_products_of_infinities_and_the_largest_numbers():
    """Infinite and NaN operands, and one near the end of the range, give what sums of fp32 products give, and nothing else changes."""
    b = nb()
    rng = np.random.default_rng(6)
    n, F, d_out = 17_000, 100, 256
    f32 = lambda *s: (rng.standard_normal(s) * 1e-3).astype(np.float32)
    x, w_self, w_neigh, bias = f32(n, F), f32(F, d_out), f32(F, d_out), f32(d_out)
    x[5, 3], x[70, 0], x[200, 99], x[8999, 50] = np.inf, -np.inf, np.nan, 3.4e38
    w_self[7, 9], w_neigh[40, 200] = np.inf, 3.4e38
    h = forward_layer(b, n, n, x, w_self, w_neigh, bias, False).cpu().numpy()
    x64 = x.astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = x64 @ w_self.astype(np.float64) + x64 @ w_neigh.astype(np.float64) + bias
        mag = np.abs(x64) @ (np.abs(w_self).astype(np.float64) + np.abs(w_neigh)) + np.abs(bias)
    big = np.isfinite(ref) & (mag > 3e38)                      # (fp32 sums may overflow on the way there)
    assert np.array_equal(np.isnan(h), np.isnan(ref))
    assert np.array_equal(np.isinf(h) & ~big, np.isinf(ref)) and (np.sign(h)[np.isinf(ref)] == np.sign(ref)[np.isinf(ref)]).all()
    ok = np.isfinite(ref) & ~big
    assert ok.sum() > 0.9 * ref.size and (np.abs(h[ok] - ref[ok]) <= (2 * F + 9) * 2.0 ** -24 * mag[ok]).all()


def test_sage_layer_gradient_products_of_infinities_and_the_largest_numbers():
    """An infinite gradient gives infinite products (NaN where infinities of both signs meet, and there only), one near the end of
    the fp32 range finite ones, as sums of fp32 products do."""
    b = nb()
    rng = np.random.default_rng(5)
    n, cap, F, d_out = 300, 5000, 100, 64
    f32 = lambda *s: (rng.standard_normal(s) * 1e-3).astype(np.float32)
    x, mean, gh, w_self, w_neigh = f32(cap, F), f32(cap, F), f32(cap, d_out), f32(F, d_out), f32(F, d_out)
    gh[5, 3], gh[40, 9], gh[299, 9], gh[120, 33] = np.inf, -np.inf, np.inf, 3.4e38
    x[17, 99], mean[200, 0] = 3.4e38, -np.inf
    i32 = lambda a: dev(np.asarray(a, np.int32))
    ptr = i32(np.minimum(np.arange(cap + 1), n))
    blk = b.block_view_from_tensors(i32([n]), i32([n]), ptr, i32(np.arange(cap)), cap, cap, ptr, i32(np.arange(cap)))
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    gs, gn, gb, gx = (torch.empty(s, device="cuda") for s in ((F, d_out), (F, d_out), (d_out,), (cap, F)))
    b.no_sage_layer_bwd(blk, dev(x), dev(mean), dev(gh), dev(gh), dev(w_self), dev(w_neigh), False, gs, gn, gb, gx, ws)
    x, mean, gh = (a[:n].astype(np.float64) for a in (x, mean, gh))
    ws64, wn64 = w_self.astype(np.float64), w_neigh.astype(np.float64)
    with np.errstate(invalid="ignore"):
        refs = (x.T @ gh, mean.T @ gh, gh.sum(0), gh @ ws64.T + gh @ wn64.T)
    for got, ref in zip((gs, gn, gb, gx[:n]), refs):
        got = got.cpu().numpy()
        assert np.isfinite(ref).any() and not np.isfinite(ref).all()
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.where(np.isinf(got), np.sign(got), 0), np.where(np.isinf(ref), np.sign(ref), 0))


@pytest.mark.parametrize("e_rows,e_grad", [(-116, 0), (-124, 0), (0, -132), (-145, 60), (10, -147), (60, 58), (110, -20)])
def test_sage_layer_gradient_products_at_the_ends_of_the_range(e_rows, e_grad):
    """Operands around 2^e (down to subnormal ones) whose results are ordinary numbers, against exact sums of them: the bound of
    test_sage_layer_gradient_products_at_tile_edges, which does not depend on where the operands lie. n = 70 rows keep it tight."""
    b = nb()
    rng = np.random.default_rng(7)
    n, cap, F, d_out = 70, 5000, 100, 64
    f32 = lambda e, *s: (rng.standard_normal(s) * 2.0 ** e).astype(np.float32)
    x, mean, gh, w_self, w_neigh = f32(e_rows, cap, F), f32(e_rows, cap, F), f32(e_grad, cap, d_out), f32(e_rows, F, d_out), f32(e_rows, F, d_out)
    i32 = lambda a: dev(np.asarray(a, np.int32))
    ptr = i32(np.minimum(np.arange(cap + 1), n))
    blk = b.block_view_from_tensors(i32([n]), i32([n]), ptr, i32(np.arange(cap)), cap, cap, ptr, i32(np.arange(cap)))
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    gs, gn, gb, gx = (torch.full(s, float("nan"), device="cuda") for s in ((F, d_out), (F, d_out), (d_out,), (cap, F)))
    b.no_sage_layer_bwd(blk, dev(x), dev(mean), dev(gh), dev(gh), dev(w_self), dev(w_neigh), False, gs, gn, gb, gx, ws)
    x, mean, gh = (a[:n].astype(np.float64) for a in (x, mean, gh))
    w = w_self.astype(np.float64) + w_neigh.astype(np.float64)
    w_abs = np.abs(w_self).astype(np.float64) + np.abs(w_neigh)
    for got, ref, mag, terms in ((gs, x.T @ gh, np.abs(x).T @ np.abs(gh), n), (gn, mean.T @ gh, np.abs(mean).T @ np.abs(gh), n),
                                 (gb, gh.sum(0), np.abs(gh).sum(0), n), (gx[:n], gh @ w.T, np.abs(gh) @ w_abs.T, 2 * d_out)):
        # (below the normal range every sum that is stored, one to a slice of 64 rows, is off by up to 2^-150)
        assert (np.abs(got.cpu().numpy() - ref) <= (terms + 8) * 2.0 ** -24 * mag + 2 * 2.0 ** -150).all()


def test_sage_layer_gradient_products_that_end_just_inside_the_range():
    """Products of two finite numbers that stay below the largest one are finite, though their operands round up to a product above it."""
    b = nb()
    n, cap, F, d_out = 40, 5000, 100, 64
    top = np.float32(2.0 ** 64 * (1 - 2.0 ** -24))          # top * top = 2^128 (1 - 2^-23 + 2^-48): the largest fp32 number, to half its last bit
    x, gh, w = np.zeros((cap, F), np.float32), np.zeros((cap, d_out), np.float32), np.zeros((F, d_out), np.float32)
    x[5, 7], x[21, 99], gh[5, 3], gh[21, 63], w[50, 63], w[99, 3] = top, top, top, -top, top, -top
    i32 = lambda a: dev(np.asarray(a, np.int32))
    ptr = i32(np.minimum(np.arange(cap + 1), n))
    blk = b.block_view_from_tensors(i32([n]), i32([n]), ptr, i32(np.arange(cap)), cap, cap, ptr, i32(np.arange(cap)))
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap, cap, F, d_out), dtype=torch.uint8, device="cuda")
    gs, gn, gb, gx = (torch.empty(s, device="cuda") for s in ((F, d_out), (F, d_out), (d_out,), (cap, F)))
    b.no_sage_layer_bwd(blk, dev(x), dev(x), dev(gh), dev(gh), dev(w), dev(np.zeros_like(w)), False, gs, gn, gb, gx, ws)
    x, gh = x[:n].astype(np.float64), gh[:n].astype(np.float64)
    for got, ref in ((gs, x.T @ gh), (gn, x.T @ gh), (gb, gh.sum(0)), (gx[:n], gh @ w.astype(np.float64).T)):
        assert np.count_nonzero(ref) == 2 and np.array_equal(got.cpu().numpy(), ref.astype(np.float32))


def layer_backward_us(n, F, d_out, fill=None):
    """(time of one backward call of a layer over n rows, its outputs); operands from N(0, 1), or all of them `fill`."""
    b = nb()
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda") if fill is None else torch.full(s, fill, device="cuda")
    x, gh, w_self, w_neigh = rnd(n, F), rnd(n, d_out), rnd(F, d_out), rnd(F, d_out)
    d_n, ptr = dev(np.array([n], np.int32)), torch.arange(n + 1, dtype=torch.int32, device="cuda")
    blk = b.block_view_from_tensors(d_n, d_n, ptr, ptr[:n].clone(), n, n, ptr, ptr[:n].clone())
    ws = torch.empty(b.no_sage_layer_ws_bytes(n, n, F, d_out), dtype=torch.uint8, device="cuda")
    outs = [torch.empty(s, device="cuda") for s in ((F, d_out), (F, d_out), (d_out,), (n, F))]

    def call_us():
        call = lambda: b.no_sage_layer_bwd(blk, x, x, gh, gh, w_self, w_neigh, False, *outs, ws)
        call()
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(20):
            call()
        t1.record()
        torch.cuda.synchronize()
        return t0.elapsed_time(t1) / 20 * 1e3

    return min(call_us() for _ in range(3)), outs


def test_sage_layer_gradients_of_a_diverged_run_keep_their_pace():
    """NaN in every operand: the gradients are NaN, and the call stays within a few times of one with ordinary numbers (outputs
    summed one by one took 54 times as long; measured: 3 times)."""
    ordinary = layer_backward_us(3400, 256, 256)[0]
    diverged, outs = layer_backward_us(3400, 256, 256, float("nan"))
    assert all(torch.isnan(t).all() for t in outs)
    print("ordinary %.1f us, all NaN %.1f us" % (ordinary, diverged))
    assert diverged < 10 * ordinary


@pytest.mark.parametrize("n,F,d_out,other,at_most", [(60_000, 1792, 1792, 1024, 4.4), (60_000, 256, 4, 8, 1.33)])
def test_sage_layer_gradients_of_wide_and_narrow_layers_keep_their_pace(n, F, d_out, other, at_most):
    """Against the same layer with F = d_out = other, or d_out = other columns. Layers so wide that the weight gradients use few row
    slices (products: 3.06 times the other's; measured: 3.1 times the time, 5.7 with the input gradient on the kernel for small
    products), and ones with fewer columns than are cut together (half the products; measured: 1.07 to 1.19 times the time, 1.46)."""
    ours, others = layer_backward_us(n, F, d_out)[0], layer_backward_us(n, other if F == d_out else F, other)[0]
    print("%d columns %.1f us, %d columns %.1f us" % (d_out, ours, other, others))
    assert ours < at_most * others


def test_sage_layer_gradients_of_few_rows_keep_their_pace():
    """A layer of few columns has few tiles: a thousand rows are cut into slices that occupy the chip, and take hardly longer than 64
    (measured: 1.10 times as long; in slices of 256 rows 1.37)."""
    many, few = layer_backward_us(1000, 100, 47)[0], layer_backward_us(64, 100, 47)[0]
    print("1000 rows %.1f us, 64 rows %.1f us" % (many, few))
    assert many < 1.25 * few


def test_sage_layer_gradients_of_whole_tiles_keep_their_pace():
    """128 columns, a whole tile, leave the row of column sums a tile of its own, which is not work enough to choose the tiles by:
    they took 1.21 times as long as 127."""
    whole, less = layer_backward_us(5000, 128, 256)[0], layer_backward_us(5000, 127, 256)[0]
    print("128 columns %.1f us, 127 columns %.1f us" % (whole, less))
    assert whole < 1.1 * less


def test_weight_gradients_of_one_product_in_a_step_keep_their_pace():
    """GCN-style layers have one product of the two that their workspace has room for: without reuse it is cut into as many slices as fill the chip too, and takes about half of
    the time of two (measured over 20 K rows, 602 x 256: 0.53; in half as many slices, a block a compute unit, 0.66)."""
    b = nb()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    V = 100_000
    ids = lambda: torch.randint(0, V, (4_000_000,), device="cuda", generator=gen, dtype=torch.int32)
    g = b.no_build_csr(ids(), ids(), V, 32)
    feat, lab = torch.randn((V, 602), device="cuda", generator=gen), torch.zeros(V, dtype=torch.int32, device="cuda")
    seeds = torch.arange(1024, dtype=torch.int32, device="cuda")
    models = []
    for arch in ("gcn", "sage"):
        models.append(b.no_model_create(g, [602, 256, 41], 1024, (25, 10)))
        b.no_model_set_arch(models[-1], b.ARCH_OF_NAME[arch])
    times = [[], []]
    for _ in range(5):
        for model, of in zip(models, times):
            b.no_model_profile(model, False)
            b.no_train_step(model, g, feat, lab, seeds, None, 0, 1, 0.0)
            b.no_model_profile(model, True)
            for step in range(8):
                b.no_train_step(model, g, feat, lab, seeds, None, step, 1, 0.0)
            of.append(b.no_model_stage_ms(model)[0]["gemm_dw_l1"] / 8 * 1e3)
    one, two = (sorted(of)[2] for of in times)
    print("one product %.1f us, two %.1f us" % (one, two))
    assert one < 0.6 * two


@pytest.mark.parametrize("bf16", [False, True])
def test_parameters_written_through_kept_views_between_steps(bf16):
    """A caller with an optimiser of its own keeps the views of the parameters and writes them between two steps (and says so by
    asking for them again, which layer 1's copies on a bf16 table need)."""
    b = nb()
    V, dims, batch, fanouts = 4000, [24, 256, 250, 16], 1100, [5, 4, 3]
    src, dst, og, gg = make_graph(V, 40_000, 3, 32)
    feat = si.features(V, dims[0], 3, "bf16" if bf16 else "f32")
    feat, lab = dev(feat.view(np.int16) if bf16 else feat), dev(si.labels(V, dims[-1], 3))
    seeds = dev(si.batch_seeds(si.train_split(V, 0.65, 3), batch, 0))

    def grads_after(*weight_seeds):
        model = b.no_model_create(gg, dims, batch, fanouts, b.NO_BF16 if bf16 else b.NO_F32)
        views = [b.no_model_params(model, l + 1) for l in range(3)]
        for s in weight_seeds:
            for three, new in zip(views, si.init_weights(dims, s)):
                for t, a in zip(three, new):
                    t.copy_(dev(a))
            if bf16:
                b.no_model_params(model, 1)
            b.no_train_step(model, gg, feat, lab, seeds, None, 0, 3, 0.0)
        return [t.clone() for l in range(3) for t in b.no_model_grads(model, l + 1)]

    for got, ref in zip(grads_after(1, 2), grads_after(2)):
        assert torch.equal(got, ref)


def test_layer_form_changed_between_steps_on_a_bf16_table():
    """Layer 1's bf16 copies of its matrices belong to GraphSAGE-mean steps: the first of them after steps of another form makes them
    from the parameters as those left them."""
    b = nb()
    V, dims, batch, fanouts, lr = 3000, [40, 64, 16], 200, [5, 4], 0.1
    src, dst, og, gg = make_graph(V, 30_000, 3, 32)
    feat, lab = dev(si.features(V, dims[0], 3, "bf16").view(np.int16)), dev(si.labels(V, dims[-1], 3))
    seeds = dev(si.batch_seeds(si.train_split(V, 0.65, 3), batch, 0))
    weights = si.init_weights(dims, 3)

    def new_model(values):
        model = b.no_model_create(gg, dims, batch, fanouts, b.NO_BF16)
        for l in range(2):
            for t, a in zip(b.no_model_params(model, l + 1), values[l]):
                t.copy_(a if torch.is_tensor(a) else dev(a))
        return model

    def step(model, form):
        b.no_model_set_arch(model, form)
        b.no_train_step(model, gg, feat, lab, seeds, None, 0, 3, lr)
        return [t.clone() for l in range(2) for t in b.no_model_grads(model, l + 1)]

    views = lambda model: [b.no_model_params(model, l + 1) for l in range(2)]
    for forms in ((b.NO_ARCH_GCN,), (b.NO_ARCH_SAGE_MEAN, b.NO_ARCH_GCN)):
        ran, still = new_model(weights), new_model(weights)
        for form in forms:
            step(ran, form)
            step(still, form)
        still = new_model(views(still))               # the same parameters, and no copies yet
        for got, ref in zip(step(ran, b.NO_ARCH_SAGE_MEAN), step(still, b.NO_ARCH_SAGE_MEAN)):
            assert torch.equal(got, ref)


def test_sage_layer_backward_with_a_popular_source():
    """One source that every destination samples: its transposed segment has several hundred entries (more than the 64
    indices a wavefront reads at a time, and a tail that is no multiple of 16), next to ordinary short segments."""
    V = 700
    hub = np.zeros(V - 1, np.int32)
    v = np.arange(1, V, dtype=np.int32)
    src = np.concatenate([hub, v - 1, (v % (V - 1)) + 1, ((v * 7) % (V - 1)) + 1]).astype(np.int32)
    dst = np.concatenate([v, v, v, v]).astype(np.int32)
    seeds = np.arange(1, 1 + 333, dtype=np.int32)
    case = layer_case(V, 0, 256, 64, (6,), 333, 5, False, edges=(src, dst), seeds=seeds)
    blk = case[0]
    seg = np.diff(blk.csc_indptr)
    assert seg.max() >= 300 and seg.max() % 16 != 0 and np.median(seg) <= 3
    check_layer_forward_backward(case, 256, 64, True, False)


def check_layer_forward_backward(case, F, d_out, relu, bf16):
    b = nb()
    blk, x, xb, w_self, w_neigh, bias, rng = case
    n_dst, n_src, nnz = blk.n_dst, blk.n_src, blk.nnz
    cap_dst, cap_src = n_dst + 77, n_src + 130          # capacities larger than the actual sizes
    d_n_dst, d_n_src = dev(np.array([n_dst], np.int32)), dev(np.array([n_src], np.int32))
    indptr = dev(np.concatenate([blk.indptr, np.zeros(77, np.int32)]))
    view = b.block_view_from_tensors(d_n_dst, d_n_src, indptr, dev(blk.indices), cap_dst, cap_src,
                                     dev(np.concatenate([blk.csc_indptr, np.zeros(130, np.int32)])), dev(blk.csc_dst))
    xs = dev(xb.view(np.int16)) if bf16 else dev(x)
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap_dst, cap_src, F, d_out), dtype=torch.uint8, device="cuda")
    mean = torch.full((cap_dst, F), 7.0, device="cuda")
    h = torch.full((cap_dst, d_out), 7.0, device="cuda")
    tw_self, tw_neigh, tbias = dev(w_self), dev(w_neigh), dev(bias)
    b.no_sage_layer_fwd(view, xs, tw_self, tw_neigh, tbias, relu, mean, h, ws)
    o_mean, o_h = ora.sage_layer_fwd(blk, x, w_self, w_neigh, bias, relu)
    assert_close(mean[:n_dst].cpu().numpy(), o_mean, "mean")
    assert_close(h[:n_dst].cpu().numpy(), o_h, "h")
    assert (h[n_dst:] == 7.0).all() and (mean[n_dst:] == 7.0).all()      # rows past n_dst untouched

    # backward: feed the oracle's own forward values so the ReLU masks agree
    grad_h = rng.standard_normal((n_dst, d_out)).astype(np.float32)
    o_h32 = o_h.astype(np.float32)
    gws = torch.zeros((F, d_out), device="cuda")
    gwn = torch.zeros((F, d_out), device="cuda")
    gb = torch.zeros((d_out,), device="cuda")
    gx = torch.full((cap_src, F), 3.0, device="cuda")
    hh = torch.zeros((cap_dst, d_out), device="cuda")
    hh[:n_dst] = dev(o_h32)
    gh = torch.zeros((cap_dst, d_out), device="cuda")
    gh[:n_dst] = dev(grad_h)
    mm = torch.zeros((cap_dst, F), device="cuda")
    mm[:n_dst] = dev(o_mean.astype(np.float32))
    for need_gx in (True, False):
        b.no_sage_layer_bwd(view, xs, mm, hh, gh, tw_self, tw_neigh, relu, gws, gwn, gb, gx if need_gx else None, ws)
        r = ora.sage_layer_bwd(blk, x, o_mean.astype(np.float32), o_h32, grad_h, w_self, w_neigh, relu, need_gx)
        assert_close(gws.cpu().numpy(), r[0], "gw_self")
        assert_close(gwn.cpu().numpy(), r[1], "gw_neigh")
        assert_close(gb.cpu().numpy(), r[2], "gbias")
        if need_gx:
            assert_close(gx[:n_src].cpu().numpy(), r[3], "grad_x")
            assert (gx[n_src:] == 3.0).all()
    # bit-stable: the same call twice gives identical bits (fixed reduction order, no float atomics)
    g1 = gws.clone()
    b.no_sage_layer_bwd(view, xs, mm, hh, gh, tw_self, tw_neigh, relu, gws, gwn, gb, None, ws)
    assert torch.equal(g1, gws)


def test_sage_layer_empty_block_and_small_workspace():
    b = nb()
    n0 = dev(np.array([0], np.int32))
    view = b.block_view_from_tensors(n0, n0, dev(np.zeros(9, np.int32)), dev(np.zeros(4, np.int32)), 8, 8)
    x = torch.zeros((8, 4), device="cuda")
    w = torch.ones((4, 3), device="cuda")
    bias = torch.ones(3, device="cuda")
    mean = torch.zeros((8, 4), device="cuda")
    h = torch.full((8, 3), 5.0, device="cuda")
    ws = torch.empty(b.no_sage_layer_ws_bytes(8, 8, 4, 3), dtype=torch.uint8, device="cuda")
    b.no_sage_layer_fwd(view, x, w, w, bias, True, mean, h, ws)
    assert (h == 5.0).all()
    with pytest.raises(b.NoError) as ei:
        b.no_sage_layer_fwd(view, x, w, w, bias, True, mean, h, ws[:16])
    assert ei.value.code == -3


# --------------------------------------------------------------------------------------- whole step

def make_relu_hook(b, model, st, n_layers, ambiguous, band=1e-5):
    """The ReLU decision is a float deciding a bit. Where the oracle's pre-activation is zero to
    within rounding (|z| <= 1e-5 max|z|) the decision the kernel took in fp32 is as valid as the
    oracle's, so the oracle's backward uses the kernel's; everywhere else the two must agree exactly
    (asserted here), so a wrong mask cannot hide behind this. How many decisions may be taken over is bounded.
    (`band`: the relative width of "zero to within rounding"; wider for runs whose products take bf16 operands.)"""
    def relu_decisions(layer, z_ora):
        blocks_ = b.no_model_blocks(model)
        sizes_ = b.no_blocks_sizes(blocks_)
        n_rows = st.n_v1 if (layer == 1 and n_layers >= 2) else z_ora.shape[0]
        gh = b.no_model_activations(model, layer, n_rows, 1)[0].cpu().numpy()
        if gh.shape[0] != z_ora.shape[0]:
            gh = gh[b.block_arrays(blocks_, n_layers - 1, sizes_)["compute_pos"]]
        if z_ora.size == 0:
            return np.zeros(z_ora.shape, dtype=bool)
        tau = band * max(np.abs(z_ora).max(), 1e-30)
        assert (gh[z_ora > tau] > 0).all(), "layer %d: kernel masks a clearly positive pre-activation" % layer
        assert (gh[z_ora < -tau] == 0).all(), "layer %d: kernel keeps a clearly negative pre-activation" % layer
        flips = int(((gh > 0) != (z_ora > 0)).sum())
        in_band = int((np.abs(z_ora) <= tau).sum())
        ambiguous.append((layer, flips, in_band, z_ora.size))
        # the witness may only decide a vanishing share of the entries: at most RELU_FLIP_SHARE of a layer's
        # pre-activations (plus RELU_FLIP_FLOOR for tiny layers) may differ from the oracle's own decision
        assert flips <= RELU_FLIP_FLOOR + RELU_FLIP_SHARE * z_ora.size, (
            "layer %d: %d of %d ReLU decisions taken from the kernel (in band: %d)" % (layer, flips, z_ora.size, in_band))
        return gh > 0
    return relu_decisions


def check_step_outputs(b, model, st, r, n_layers, step, with_cache_blocks, gcn, feat_dtype, rtol=RTOL):
    """One step of the library (its statistics `st`, the model's blocks, activations, gradients and parameters)
    against the oracle's StepResult `r`: integers bit for bit, floats within the tolerance."""
    pick = (lambda three: (three[0], three[2])) if gcn else (lambda three: three)
    blocks = b.no_model_blocks(model)
    sizes = compare_blocks(b, blocks, r.batch, with_cache=with_cache_blocks)
    for h in range(n_layers):
        assert (st.n_dst[h], st.n_src[h], st.nnz[h]) == tuple(int(x) for x in sizes[h, :3])
    assert st.n_hit == r.n_hit
    # gathered rows (the step materialises the bottom destinations' rows; the rest is read in place): bit copy
    n_dst_bottom = r.batch.blocks[-1].n_dst
    if not gcn:
        x0 = b.no_model_gathered(model, n_dst_bottom).cpu().numpy()
        assert np.array_equal(x0.view(feat_dtype), r.x0[:n_dst_bottom])
    # floats
    assert abs(st.loss - r.loss) <= rtol * abs(r.loss) + 1e-6, (st.loss, r.loss)
    for l in range(1, n_layers + 1):
        n_rows = r.h[l - 1].shape[0]
        n_dst = r.batch.blocks[n_layers - l].n_dst
        gh, gm = b.no_model_activations(model, l, n_rows, n_dst)
        assert_close(gm.cpu().numpy(), r.mean[l - 1], "mean%d step %d" % (l, step), RTOL if l == 1 else rtol)
        assert_close(gh.cpu().numpy(), r.h[l - 1], "h%d step %d" % (l, step), rtol)
        names = ["gw", "gbias"] if gcn else ["gw_self", "gw_neigh", "gbias"]
        for t, ref, name in zip(pick(b.no_model_grads(model, l)), r.grads[l - 1], names):
            assert_close(t.cpu().numpy(), ref, "%s%d step %d" % (name, l, step), rtol)
        for t, ref, name in zip(pick(b.no_model_params(model, l)), r.new_weights[l - 1], names):
            assert_close(t.cpu().numpy(), ref, "%s%d step %d" % (name[1:], l, step), rtol)


def run_steps(w, n_steps, use_cache, lr=0.05, V=None, E=None, hot_fraction=None, bits=32, presample=1,
              n_train_presample=None, superbatch=0, arch="sage", ahead=False, joined=None):
    b = nb()
    V = V or w.n_vertices
    E = E or w.n_edges
    src, dst, og, gg = make_graph(V, E, w.seed, bits, w.symmetrise)
    feat = si.features(V, w.feat_dim, w.seed, w.feat_dtype)
    lab = si.labels(V, w.n_classes, w.seed)
    train = si.train_split(V, 0.65, w.seed)
    weights = si.init_weights(w.dims, w.seed)
    bf16 = w.feat_dtype == "bf16"
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts, b.NO_BF16 if bf16 else b.NO_F32)
    gcn = arch != "sage"
    bf16_products = bf16 and not gcn          # layer 1's products take bf16 operands (kernel and oracle)
    rtol = RTOL_BF16 if bf16_products else RTOL
    if gcn:
        b.no_model_set_arch(model, b.ARCH_OF_NAME[arch])
    assert joined is None or b.no_model_last_layer_joined(model, w.batch) == joined
    for l in range(w.n_layers):
        for t, a in zip(b.no_model_params(model, l + 1), weights[l]):
            t.copy_(dev(a))
    pick = (lambda three: (three[0], three[2])) if gcn else (lambda three: three)     # GCN-style: (w, bias)
    frac = w.hot_fraction if hot_fraction is None else hot_fraction
    oc = gc = None
    if use_cache:
        # hotness may be pre-sampled on a prefix of the train ids to bound the oracle's cost at full size
        pre = train if n_train_presample is None else train[:n_train_presample]
        oc = ora.select_hot(og, pre, w.batch, w.fanouts, presample, frac, w.staleness, w.hidden, w.seed)
        gc = b.no_select_hot(gg, dev(pre), w.batch, w.fanouts, presample, frac, w.staleness, w.hidden, w.seed)
        assert np.array_equal(b.no_cache_view(gc, V)["hot_ids"].cpu().numpy(), oc.hot_ids)
        if gcn:
            b.no_cache_set_layer_form(gc, b.ARCH_OF_NAME[arch])
    tfeat = dev(feat.view(np.int16) if bf16 else feat)
    tlab = dev(lab)
    ow = [tuple(np.asarray(t, np.float64) for t in pick(x)) for x in weights]
    hits = 0
    pending = None
    pending_snap = current_snap = None          # layer-1 parameters behind the pending / the committed rows
    seed_tensors = [dev(si.batch_seeds(train, w.batch, t)) for t in range(n_steps)]
    commit = False
    stamped_ahead = None
    for step in range(n_steps):
        seeds = si.batch_seeds(train, w.batch, step)
        print("step", step, flush=True)
        if superbatch and step % superbatch == 0:
            # super-batch boundary (Section 4.2): install the rows refreshed during the last super-batch, then
            # start the refresh for the next one from the parameters as they stand now
            if pending is not None:
                ora.commit_refresh(oc, *pending)
                current_snap = pending_snap
                if not ahead:           # sampling ahead: committed inside the previous step's call
                    b.no_refresh_hot_commit(gc)
            pending_snap = ow[0]
            pending = ora.refresh_hot(og, feat, oc, ow[0], w.fanouts[-1], step, w.seed, feat_is_bf16=bf16,
                                      norm=ora.gcn_norm_of(arch) if gcn else "mean")
            p1 = b.no_model_params(model, 1)
            b.no_refresh_hot_begin(gc, gg, tfeat, p1[0], None if gcn else p1[1], p1[2], w.fanouts[-1], step, w.seed)
        if ahead:
            nxt = seed_tensors[step + 1] if step + 1 < n_steps else None
            commit = bool(superbatch) and nxt is not None and (step + 1) % superbatch == 0
            st = b.no_train_step_ahead(model, gg, tfeat, tlab, seed_tensors[step], nxt, commit, gc, step, w.seed, lr)
        else:
            st = b.no_train_step(model, gg, tfeat, tlab, seed_tensors[step], gc, step, w.seed, lr)
        ambiguous = []
        relu_decisions = make_relu_hook(b, model, st, w.n_layers, ambiguous, band=1e-3 if bf16_products else 1e-5)
        r = ora.train_step(og, feat, lab, seeds, w.fanouts, ow, lr, w.seed, step, oc, feat_is_bf16=bf16,
                           relu_decisions=relu_decisions, arch=arch)
        print("  relu decisions taken from the kernel (layer, flips, in band, entries):", ambiguous, flush=True)
        check_step_outputs(b, model, st, r, w.n_layers, step, use_cache and w.n_layers >= 2 and oc.n_hot > 0, gcn, feat.dtype,
                           rtol)
        hits += r.n_hit
        if superbatch and not ahead:
            # weight-drift monitor (Section 4.3): largest change of a layer-1 parameter in this update, and the drift
            # from the parameters behind the rows now in the cache
            upd, drift = b.no_model_weight_drift(model, gc, lr)
            o_upd = ora.max_weight_update(ow[0], r.new_weights[0])
            assert abs(upd - o_upd) <= rtol * o_upd + 1e-12, (upd, o_upd)
            if current_snap is None:
                assert drift == -1.0
            else:
                o_drift = ora.weight_drift(r.new_weights[0], current_snap)
                assert abs(drift - o_drift) <= rtol * o_drift + 1e-7, (drift, o_drift)
        ow = r.new_weights
        if use_cache and oc.n_hot > 0:
            view = b.no_cache_view(gc, V)
            gv = view["version"].cpu().numpy()
            # A batch prepared ahead has been split already, and its split stamps the slots that batch will recompute
            # with its step (the rows follow with its layer-1 product): those entries run one step ahead of the
            # oracle's; which slots they are is checked against the oracle's next step.
            stamped = (gv == step + 1) if (ahead and step + 1 < n_steps) else np.zeros(gv.shape, dtype=bool)
            if ahead and commit:
                # the boundary commit ran inside this call (after the step's last use of the cache): the cache
                # already holds what the oracle installs at the start of the next step
                assert np.array_equal(gv[~stamped], pending[1][~stamped])
                assert_close(view["emb"].cpu().numpy(), pending[0], "committed emb step %d" % step, rtol)
            else:
                assert np.array_equal(gv[~stamped], oc.version[~stamped])
                assert_close(view["emb"].cpu().numpy(), oc.emb, "emb step %d" % step, rtol)
            if stamped_ahead is not None:
                # the slots stamped ahead by the previous call are exactly those this step refreshed in the oracle
                assert np.array_equal(np.flatnonzero(stamped_ahead), np.flatnonzero(oc.version == step)), step
            stamped_ahead = stamped if ahead and step + 1 < n_steps else None
    return hits


def test_train_steps_tiny_config_exact():
    run_steps(si.WORKLOADS["tiny"], 3, use_cache=False)


def test_train_steps_tiny_config_with_cache_S0_never_hits():
    assert run_steps(si.WORKLOADS["tiny"], 3, use_cache=True) == 0      # the tiny config has S = 0


def test_train_steps_with_reuse():
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    assert run_steps(w, 5, use_cache=True, lr=0.02) > 0


def test_train_steps_three_layers_with_reuse():
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(4, 3, 3), staleness=1, hot_fraction=0.3, n_classes=47,
                            feat_dim=100, hidden=40, batch=128)
    assert run_steps(w, 4, use_cache=True, lr=0.02, bits=64) > 0


@pytest.mark.parametrize("feat_dim,hidden", [(1, 16), (3, 64), (5, 33), (70, 129), (128, 256), (130, 300), (258, 300)])
def test_bf16_weight_gradient_products_at_tile_edges(feat_dim, hidden):
    """Rows that start on odd halves of a word, fewer columns than a unit, remainders of the 64- and the 128-wide tiles."""
    w = dataclasses.replace(si.WORKLOADS["tiny"], feat_dtype="bf16", feat_dim=feat_dim, hidden=hidden, staleness=2, hot_fraction=0.1)
    run_steps(w, 2, True)


def test_train_step_single_layer_and_bf16_features():
    import dataclasses
    w1 = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(6,), batch=200)
    run_steps(w1, 2, use_cache=False)
    wb = dataclasses.replace(si.WORKLOADS["tiny"], feat_dtype="bf16", feat_dim=128, staleness=2, hot_fraction=0.1)
    run_steps(wb, 3, use_cache=True)
    # a single layer on a bf16 table: the bf16-operand products feed the logits directly (16 columns: one partly
    # filled column group), and a feature width that is no multiple of 8 or 16 (element-wise staging, padded weights)
    wb1 = dataclasses.replace(si.WORKLOADS["tiny"], feat_dtype="bf16", feat_dim=128, fanouts=(6,), batch=200)
    run_steps(wb1, 2, use_cache=False)
    wb2 = dataclasses.replace(si.WORKLOADS["tiny"], feat_dtype="bf16", feat_dim=70, hidden=300, staleness=2, hot_fraction=0.1)
    run_steps(wb2, 3, use_cache=True, ahead=True)


@pytest.mark.parametrize("fanouts,arch,ahead", [((5, 4, 3, 3), "sage", False), ((4, 3, 3, 2, 2), "sage", True),
                                                ((4, 3, 3, 2, 2), "gcn", False), ((5, 4, 3, 3), "gcn", True),
                                                ((5, 4, 3, 3), "gcn_sym", True), ((4, 3, 3, 2, 2), "gcn_sum", False)])
def test_deeper_models_four_and_five_layers(fanouts, arch, ahead):
    """The depths of the paper's model-depth experiments (the fanout list repeats its last value): every hop, the
    cache split at the bottom one, reuse and the look-ahead on a 4- and a 5-layer model, both layer forms."""
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=fanouts, staleness=2, hot_fraction=0.2, batch=64, hidden=48)
    assert run_steps(w, 4, use_cache=True, lr=0.002 if arch == "gcn_sum" else 0.02, ahead=ahead, arch=arch) > 0
    if arch == "sage":
        # the same depth on a bf16 table: bf16-operand products at the bottom, fp32 weight-gradient products of the
        # layers above launched beside them
        wb = dataclasses.replace(w, feat_dtype="bf16", feat_dim=96)
        assert run_steps(wb, 3, use_cache=True, lr=0.02, ahead=ahead, arch=arch) > 0


@pytest.mark.parametrize("ahead", [False, True])
def test_deepest_model_eight_layers(ahead):
    """The largest number of layers the library takes (NO_MAX_LAYERS): seven upper layers hand their weight-gradient
    work to the bottom layer's launches, which then carry all eight."""
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(3, 2, 2, 2, 2, 2, 2, 2), staleness=2, hot_fraction=0.2, batch=16,
                            hidden=24)
    assert run_steps(w, 3, use_cache=True, lr=0.02, ahead=ahead) > 0


@pytest.mark.parametrize("hot_fraction,staleness", [(0.0, 2), (0.1, 0), (0.1, 2), (0.1, 4), (0.3, 2), (0.3, 4)])
def test_hot_reuse_sweep_points(hot_fraction, staleness):
    """The hot-reuse sweep (hot fraction x staleness bound, the shape of the paper's Fig. 14 experiment) on a
    shrunken copy of the sweep workload's graph."""
    import dataclasses
    w = dataclasses.replace(si.scaled(si.WORKLOADS["sweep"], 0.01), batch=256, hot_fraction=hot_fraction,
                            staleness=staleness, feat_dim=64, hidden=32)
    hits = run_steps(w, 6, use_cache=True, lr=0.02, bits=32)
    if hot_fraction == 0.0 or staleness == 0:
        assert hits == 0
    else:
        assert hits > 0


def test_large_config_shape_scaled_bf16():
    """The large workload's shape (bf16 features, int64 row pointers, 3 layers, 172 classes) on a shrunken graph."""
    w = si.scaled(si.WORKLOADS["large"], 0.0005)
    assert run_steps(w, 4, use_cache=True, lr=0.01, bits=64) > 0


@pytest.mark.parametrize("bf16", [False, True])
def test_refresh_hot_rows_match_oracle(bf16):
    """Bulk refresh (Section 4.2, Stage 2) alone: rows and versions of every hot vertex against the oracle; the
    pending copy stays invisible until the commit; misuse is refused."""
    b = nb()
    V, E, F, D = 3000, 40_000, 70 if not bf16 else 64, 48
    src, dst, og, gg = make_graph(V, E, 4, 32)
    feat = si.features(V, F, 4, "bf16" if bf16 else "f32")
    train = si.train_split(V, 0.65, 4)
    (w_self, w_neigh, bias), = si.init_weights([F, D], 4)
    fan = (5, 4)
    oc = ora.select_hot(og, train, 64, fan, 1, 0.15, 3, D, 4)
    gc = b.no_select_hot(gg, dev(train), 64, fan, 1, 0.15, 3, D, 4)
    tfeat = dev(feat.view(np.int16) if bf16 else feat)
    tw = [dev(w_self), dev(w_neigh), dev(bias)]
    with pytest.raises(b.NoError):
        b.no_refresh_hot_commit(gc)                       # nothing pending
    b.no_refresh_hot_begin(gc, gg, tfeat, *tw, fan[-1], 6, 99)
    tw[0].mul_(2.0)                                       # later updates on the stream do not reach the snapshot
    with pytest.raises(b.NoError):
        b.no_refresh_hot_begin(gc, gg, tfeat, *tw, fan[-1], 7, 99)    # one refresh at a time
    torch.cuda.synchronize()
    view = b.no_cache_view(gc, V)
    assert (view["version"] == -1).all() and (view["emb"] == 0).all()     # not installed yet
    b.no_refresh_hot_commit(gc)
    emb, ver = ora.refresh_hot(og, feat, oc, (w_self, w_neigh, bias), fan[-1], 6, 99, feat_is_bf16=bf16)
    view = b.no_cache_view(gc, V)
    assert np.array_equal(view["version"].cpu().numpy(), ver)
    assert_close(view["emb"].cpu().numpy(), emb, "refreshed rows")
    with pytest.raises(b.NoError):
        b.no_refresh_hot_begin(gc, gg, tfeat, *tw, fan[-1] + 1, 8, 99)      # buffers were sized for another fanout
    # a second round lands in the other copy and replaces the first at its commit
    tw[0].copy_(dev(w_self))
    b.no_refresh_hot_begin(gc, gg, tfeat, *tw, fan[-1], 9, 99)
    b.no_refresh_hot_commit(gc)
    emb2, ver2 = ora.refresh_hot(og, feat, oc, (w_self, w_neigh, bias), fan[-1], 9, 99, feat_is_bf16=bf16)
    view = b.no_cache_view(gc, V)
    assert np.array_equal(view["version"].cpu().numpy(), ver2)
    assert_close(view["emb"].cpu().numpy(), emb2, "refreshed rows, second round")
    assert not np.array_equal(emb, emb2)


@pytest.mark.parametrize("k", [1, 8, 9, 17, 32, 33, 64])
@pytest.mark.parametrize("bits", [32, 64])
def test_refresh_draws_at_the_widths_of_its_lane_groups(k, bits):
    """Rows shorter and longer than the fanout (and, but for 64, as long), on both kinds of row pointers, against the oracle's draws."""
    b = nb()
    V, F, D, fan = 2500, 24, 40, (5, k)
    src, dst, og, gg = make_graph(V, 80_000, 7, bits)
    lens = np.diff(og.rowptr)
    assert (lens < k).any() and (lens > k).any()
    feat, train = si.features(V, F, 7), si.train_split(V, 0.65, 7)
    (w_self, w_neigh, bias), = si.init_weights([F, D], 7)
    oc = ora.select_hot(og, train, 64, fan, 1, 1.0, 3, D, 7)
    gc = b.no_select_hot(gg, dev(train), 64, fan, 1, 1.0, 3, D, 7)
    b.no_refresh_hot_begin(gc, gg, dev(feat), dev(w_self), dev(w_neigh), dev(bias), k, 6, 99)
    b.no_refresh_hot_commit(gc)
    emb, ver = ora.refresh_hot(og, feat, oc, (w_self, w_neigh, bias), k, 6, 99, feat_is_bf16=False)
    view = b.no_cache_view(gc, V)
    assert np.array_equal(view["version"].cpu().numpy(), ver)
    assert_close(view["emb"].cpu().numpy(), emb, "refreshed rows")


@pytest.mark.parametrize("form", ["sage", "gcn", "gcn_sum", "gcn_sym"])
@pytest.mark.parametrize("bf16", [False, True])
def test_refresh_of_many_hot_rows(form, bf16):
    """Enough rows for the product on planes (36,002 and, twice in a row, with other weights; 70 features are no whole step), and the forms with
    one matrix."""
    b = nb()
    V, F, D, fan = 40_003, 70, 250, (5, 4)
    src, dst, og, gg = make_graph(V, 300_000, 4, 32)
    feat = si.features(V, F, 4, "bf16" if bf16 else "f32")
    oc = ora.select_hot(og, si.train_split(V, 0.65, 4), 512, fan, 1, 0.9, 3, D, 4)
    gc = b.no_select_hot(gg, dev(si.train_split(V, 0.65, 4)), 512, fan, 1, 0.9, 3, D, 4)
    gcn = form != "sage"
    if gcn:
        b.no_cache_set_layer_form(gc, b.ARCH_OF_NAME[form])
    tfeat = dev(feat.view(np.int16) if bf16 else feat)
    for version in (6, 9):
        print(form, bf16, version, flush=True)
        (w_self, w_neigh, bias), = si.init_weights([F, D], version)
        b.no_refresh_hot_begin(gc, gg, tfeat, dev(w_self), None if gcn else dev(w_neigh), dev(bias), fan[-1], version, 99)
        b.no_refresh_hot_commit(gc)
        emb, ver = ora.refresh_hot(og, feat, oc, (w_self, bias) if gcn else (w_self, w_neigh, bias), fan[-1], version, 99, feat_is_bf16=bf16,
                                   norm=ora.gcn_norm_of(form) if gcn else "mean")
        view = b.no_cache_view(gc, V)
        assert np.array_equal(view["version"].cpu().numpy(), ver)
        got = view["emb"].cpu().numpy()
        assert_close(got, emb, "refreshed rows")
        # (the aggregate, of up to five rows, is rounded to fp32 before the product)
        assert forward_error(got, emb) <= forward_error_bound(F if gcn else 2 * F) + 2.0 ** -23


@pytest.mark.parametrize("ahead", [False, True])
@pytest.mark.parametrize("arch", ["sage", "gcn", "gcn_sym"])
def test_train_steps_with_forward_products_on_planes(arch, ahead):
    import dataclasses
    b = nb()
    w = dataclasses.replace(si.WORKLOADS["tiny"], n_vertices=100_000, n_edges=600_000, batch=8000, fanouts=(10, 5), feat_dim=300, hidden=250,
                            staleness=2, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    b.no_model_set_arch(model, b.ARCH_OF_NAME[arch] if arch != "sage" else b.NO_ARCH_SAGE_MEAN)
    assert b.no_model_forward_planes(model, 1) and not b.no_model_forward_planes(model, 2)
    with pytest.raises(b.NoError):
        b.no_model_forward_planes(model, 3)
    assert run_steps(w, 3, use_cache=True, lr=0.02, arch=arch, ahead=ahead) > 0


def test_train_step_with_the_weights_of_two_layers_cut_beside_their_aggregations():
    import dataclasses
    b = nb()
    w = dataclasses.replace(si.WORKLOADS["tiny"], n_vertices=100_000, n_edges=600_000, batch=2500, fanouts=(10, 5, 5), feat_dim=300, hidden=252,
                            staleness=2, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    assert [b.no_model_forward_planes(model, layer) for layer in (1, 2, 3)] == [True, True, False]
    assert run_steps(w, 2, use_cache=True, lr=0.02) > 0


JOINED_LAST_LAYERS = [
    ("sage", 1, (10, 5), 64, 16), ("sage", 15, (64, 2), 4, 4), ("gcn", 16, (17, 3), 8, 5), ("sage", 17, (3, 16, 2), 12, 15),    # a block's rows, short rows of few units
    ("sage", 300, (33, 3), 256, 64), ("gcn_sum", 33, (9, 3), 60, 65), ("gcn", 129, (15, 3), 128, 17), ("sage", 100, (1, 2), 252, 47),    # column groups and 16s of classes
    ("sage", 257, (7, 3), 100, 128), ("gcn", 260, (7, 3), 256, 129), ("sage", 65, (8, 4), 200, 192), ("sage", 65, (8, 4), 132, 193), ("gcn_sum", 40, (25, 3), 256, 256),
    ("sage", 4100, (4, 2), 64, 20), ("sage", 4096, (4, 2), 64, 65), ("sage", 40, (8, 4), 192, 256), ("gcn", 4097, (4, 2), 64, 65)]      # about as many row blocks as fit at once; whole tiles
SEPARATE_LAST_LAYERS = [("sage", 40, (8, 4), 260, 20), ("sage", 40, (8, 4), 66, 20), ("gcn", 40, (8, 4), 64, 3), ("sage", 40, (8, 4), 64, 257), ("gcn_sym", 40, (8, 4), 64, 20),
                        ("sage", 4097, (4, 2), 64, 65), ("sage", 40, (8, 4), 196, 256)]      # more row blocks than fit at once; whole tiles of a wide layer


def test_the_line_of_the_joined_last_layer_goes_by_the_seeds_of_a_step():
    b = nb()
    src = np.zeros(0, np.int32)
    g = b.no_build_csr(src, src, 20_000, 32)
    for arch, classes, most in (("sage", 64, 9000), ("sage", 65, 4096), ("sage", 192, 4096), ("gcn", 128, 8192), ("gcn_sum", 129, 4096), ("gcn", 256, 4096)):
        model = b.no_model_create(g, [8, 256, classes], 9000, (4, 2))
        if arch != "sage":
            b.no_model_set_arch(model, b.ARCH_OF_NAME[arch])
        assert b.no_model_last_layer_joined(model, most) and b.no_model_last_layer_joined(model, 1)
        assert most == 9000 or not b.no_model_last_layer_joined(model, most + 1)


@pytest.mark.parametrize("arch,batch,fanouts,hidden,classes,joined", [c + (True,) for c in JOINED_LAST_LAYERS] + [c + (False,) for c in SEPARATE_LAST_LAYERS])
def test_train_steps_at_the_edges_of_the_last_layers_launch(arch, batch, fanouts, hidden, classes, joined):
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], batch=batch, fanouts=fanouts, hidden=hidden, n_classes=classes, feat_dim=20, staleness=2, hot_fraction=0.2)
    run_steps(w, 2, use_cache=True, lr=0.02, arch=arch, joined=joined)


@pytest.mark.parametrize("arch,batch,fanouts,hidden,classes", [
    ("sage", 1, (10, 5), 64, 16), ("sage", 17, (3, 16, 2), 12, 15), ("gcn", 129, (15, 3, 2), 128, 17), ("sage", 65, (8, 4, 3), 132, 193), ("gcn_sum", 40, (25, 3), 256, 256)])
def test_the_last_layers_launch_takes_the_side_tasks_of_batches_prepared_ahead(arch, batch, fanouts, hidden, classes):
    """Tasks that the sampling and the aggregation of a batch prepared ahead leave go with the launch of its last layer, whose blocks have twice their threads."""
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], batch=batch, fanouts=fanouts, hidden=hidden, n_classes=classes, feat_dim=20, staleness=2, hot_fraction=0.2)
    run_steps(w, 3, use_cache=True, lr=0.02, arch=arch, ahead=True, joined=True)


def test_a_last_layer_on_planes_is_what_the_model_says_it_is():
    """Room for so many seeds that the last product is long enough for planes: it takes a launch of its own, and the model says so; with a little less
    room it goes with the loss. Bound of the logits' error: as of products on pieces."""
    b = nb()
    V = 60_000
    src, dst = si.random_graph_small(V, 200_000, 3)
    g = b.no_build_csr(src, dst, V, 32)
    for cap, planes in ((20_480, True), (20_000, False)):
        model = b.no_model_create(g, [602, 256, 200], cap, (4, 3))
        assert b.no_model_forward_planes(model, 1)
        assert (b.no_model_forward_planes(model, 2), b.no_model_last_layer_joined(model, 1500)) == (planes, not planes)
        for layer, three in enumerate(si.init_weights([602, 256, 200], 3)):
            for t, a in zip(b.no_model_params(model, layer + 1), three):
                t.copy_(dev(a))
        feat, lab = dev(si.features(V, 602, 3, "f32")), dev(si.labels(V, 200, 3))
        seeds = torch.arange(1500, dtype=torch.int32, device="cuda")
        st = b.no_train_step(model, g, feat, lab, seeds, None, 0, 1, 0.0)
        n1 = st.n_src[0]
        h1, mean2 = b.no_model_activations(model, 1, n1, n1)[0], b.no_model_activations(model, 2, 1500, 1500)[1]
        w_self, w_neigh, bias = (t.double() for t in b.no_model_params(model, 2))
        ref = h1[:1500].double() @ w_self + mean2.double() @ w_neigh + bias
        z = b.no_model_activations(model, 2, 1500, 1500)[0].double()
        assert float(torch.linalg.norm(z - ref) / torch.linalg.norm(ref)) <= forward_error_bound(2 * 256)


@pytest.mark.parametrize("arch,cap,hidden,classes", [("sage", 40, 64, 16), ("sage", 1024, 256, 172), ("gcn", 1024, 256, 64), ("gcn_sum", 200, 100, 255), ("sage", 4096, 256, 47),
                                                     ("gcn", 4096, 252, 41), ("sage", 500, 256, 128), ("gcn", 300, 256, 65), ("sage", 1024, 256, 129)])
def test_input_gradients_of_a_joined_last_layer_against_64_bits(arch, cap, hidden, classes):
    """A seed that samples nothing: the bias gradients are its row of the output gradients of both layers, and layer 1's are all kept. Up to 64 classes sums are made in
    64 bits of exact products: off by 2^-53 of the sum of their terms' sizes a term, nothing beside the rounding to fp32 that ends them. Of more classes runs of R = 8, or
    16 from 129 on, terms are made in fp32: each addition of a run is off by 2^-24 of its partial sum at most, and where these errors are independent (uniform: a third of the
    square) the worst place of the one large term, the label's, in its run leaves (R + 1) / 3 of 2^-48 of the result's square."""
    b = nb()
    src = np.zeros(0, np.int32)
    g = b.no_build_csr(src, src, 5000, 32)
    model = b.no_model_create(g, [8, hidden, classes], cap, (3, 2))
    if arch != "sage":
        b.no_model_set_arch(model, b.ARCH_OF_NAME[arch])
    assert b.no_model_last_layer_joined(model, 1)
    rng = np.random.default_rng(classes)
    feat, seed = torch.ones((5000, 8), device="cuda"), dev(np.array([17], np.int32))
    for t, v in zip(b.no_model_params(model, 1), (0.0, 0.0, 1.0)):
        t.fill_(v)
    run = 0 if classes <= 64 else 8 if classes <= 128 else 16
    err2 = ref2 = 0.0
    for step in range(16):
        print("step", step, flush=True)
        w = (rng.standard_normal((hidden, classes)) * 0.1).astype(np.float32)
        b.no_model_params(model, 2)[0].copy_(dev(w))
        lab = np.full(5000, step * (classes - 1) // 15, np.int32)
        b.no_train_step(model, g, feat, dev(lab), seed, None, step, 1, 0.0)
        gz2, gz1 = (b.no_model_grads(model, layer)[2].cpu().numpy().astype(np.float64) for layer in (2, 1))
        ref, mag = w.astype(np.float64) @ gz2, np.abs(w).astype(np.float64) @ np.abs(gz2)
        assert (np.abs(gz1 - ref) <= 2.0 ** -24 * (np.abs(ref) + run * mag) + (classes + 1) * 2.0 ** -52 * mag).all()
        err2, ref2 = err2 + ((gz1 - ref) ** 2).sum(), ref2 + (ref ** 2).sum()
    assert np.sqrt(err2 / ref2) <= 2.0 ** -24 * np.sqrt((run + 1) / 3)


@pytest.mark.parametrize("arch,cap,F,hidden,classes,bf16,planes", [
    ("sage", 40, 20, 64, 47, False, False), ("gcn", 40, 20, 252, 172, False, False),             # layer 1's product in small blocks
    ("sage", 2500, 20, 256, 47, False, False), ("sage", 2500, 602, 256, 41, False, True),        # in tiles, on planes
    ("sage", 2500, 20, 256, 47, True, False), ("gcn_sum", 2500, 602, 256, 256, False, False),    # with bf16 operands; one product in tiles
    ("sage", 40, 20, 260, 47, False, False), ("sage", 40, 20, 66, 47, False, False)])            # the last layer not in one launch; decisions read from the outputs
def test_infinities_and_nan_stay_where_they_arise_in_a_step(arch, cap, F, hidden, classes, bf16, planes):
    """Seeds that sample nothing, so that every row is its own, and one seed (amid a block of 16 rows) whose features hold NaN or an infinity; a class that is
    switched off. A NaN is not above 0, so that row's outputs are zeros with no gradient; an infinity is, where it is positive, and makes that row's logits NaN;
    with a label outside the classes the row adds nothing to any gradient. What is finite in 64 bits is within the tolerance, and nothing else changes."""
    b = nb()
    n, V, at = 37, 30_000, 21
    rng = np.random.default_rng(hidden + classes)
    gcn = arch != "sage"
    src = np.zeros(0, np.int32)
    g = b.no_build_csr(src, src, V, 32)
    for value, label_on, off in ((np.nan, True, None), (np.inf, True, None), (-np.inf, False, None), (1.0, True, 2)):
        print("step", value, label_on, off, flush=True)
        model = b.no_model_create(g, [F, hidden, classes], cap, (10, 3), b.NO_BF16 if bf16 else b.NO_F32)
        if gcn:
            b.no_model_set_arch(model, b.ARCH_OF_NAME[arch])
        assert b.no_model_forward_planes(model, 1) == planes and b.no_model_last_layer_joined(model, n) == (hidden in (64, 252, 256))
        weights = si.init_weights([F, hidden, classes], 5)
        for layer in (1, 2):
            weights[layer - 1][2][:] = rng.standard_normal(weights[layer - 1][2].shape) * 0.1
        if off is not None:
            weights[1][2][off] = -np.inf
        for layer in (1, 2):
            for t, a in zip(b.no_model_params(model, layer), weights[layer - 1]):
                t.copy_(dev(a))
        feat = torch.from_numpy(rng.standard_normal((V, F)).astype(np.float32))
        seeds = rng.permutation(V)[:n].astype(np.int32)
        lab = rng.integers(3, classes, V).astype(np.int32)
        feat[int(seeds[at]), 7] = value
        if not label_on:
            lab[seeds[at]] = classes
        feat = feat.to(torch.bfloat16) if bf16 else feat
        st = b.no_train_step(model, g, feat.cuda(), dev(lab), dev(seeds), None, 0, 1, 0.0)
        assert st.bad_label == (0 if label_on else 1)
        w1 = torch.from_numpy(weights[0][0])
        w1 = (w1.to(torch.bfloat16) if bf16 else w1).double().numpy()
        x, w2 = feat.double().numpy()[seeds], weights[1][0].astype(np.float64)
        with np.errstate(invalid="ignore"):
            z1 = x @ w1 + weights[0][2]
            h1 = np.where(z1 > 0, z1, 0.0)
            z2 = h1 @ w2 + weights[1][2]
            e = np.exp(z2 - z2.max(1, keepdims=True))
            p = e / e.sum(1, keepdims=True)
            gz2 = (p - (np.arange(classes) == lab[seeds][:, None])) / n
            if not label_on:
                gz2[at] = 0.0
            gz1 = np.where(z1 > 0, gz2 @ w2.T, 0.0)
            refs = [h1, z2, gz2.sum(0), h1.T @ gz2, gz1.sum(0)] + ([] if bf16 else [x.T @ gz1])
        got = [b.no_model_activations(model, layer, n, n)[0] for layer in (1, 2)] + [b.no_model_grads(model, 2)[i] for i in (2, 0)]
        got += [b.no_model_grads(model, 1)[i] for i in ((2,) if bf16 else (2, 0))]
        assert not np.isfinite(refs[1]).all() or np.isnan(value)
        for a, ref, what in zip(got, refs, ("h1", "logits", "gbias2", "gw2", "gbias1", "gw1")):
            a = a.cpu().numpy()
            assert np.array_equal(np.isnan(a), np.isnan(ref)), (what, value)
            assert np.array_equal(np.where(np.isinf(a), np.sign(a), 0), np.where(np.isinf(ref), np.sign(ref), 0)), (what, value)
            ok = np.isfinite(ref)
            assert_close(a[ok], ref[ok], "%s with %s" % (what, value), RTOL_BF16 if bf16 else RTOL)


@pytest.mark.parametrize("forms", [("gcn", "sage"), ("sage", "gcn"), ("gcn_sym", "gcn_sum")])
def test_a_batch_prepared_for_one_layer_form_is_not_used_for_another(forms):
    b = nb()
    w = si.WORKLOADS["tiny"]
    _, _, _, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat, lab = dev(si.features(w.n_vertices, w.feat_dim, w.seed, "f32")), dev(si.labels(w.n_vertices, w.n_classes, w.seed))
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(2)]
    code = lambda form: b.NO_ARCH_SAGE_MEAN if form == "sage" else b.ARCH_OF_NAME[form]
    grads = []
    for ahead in (True, False):
        model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
        for layer, three in enumerate(si.init_weights(w.dims, w.seed)):
            for t, a in zip(b.no_model_params(model, layer + 1), three):
                t.copy_(dev(a))
        for step, form in enumerate(forms):
            b.no_model_set_arch(model, code(form))
            if ahead:
                b.no_train_step_ahead(model, gg, feat, lab, seeds[step], seeds[1] if step == 0 else None, False, None, step, w.seed, 0.01)
            else:
                b.no_train_step(model, gg, feat, lab, seeds[step], None, step, w.seed, 0.01)
        grads.append([t.cpu().numpy() for layer in (1, 2) for i, t in enumerate(b.no_model_grads(model, layer)) if i != 1 or forms[1] == "sage"])
    for x, y in zip(*grads):
        assert np.array_equal(x, y)


def test_superbatch_schedule_with_bulk_refresh():
    """n = 3 batches per super-batch, bound 2n - 1 = 5: every step against the oracle walking the same schedule;
    from the second super-batch on every hot vertex of V^1 is served from the cache."""
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=5, hot_fraction=0.2)
    assert run_steps(w, 9, use_cache=True, lr=0.02, superbatch=3) > 0
    w3 = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(4, 3, 3), staleness=3, hot_fraction=0.3, n_classes=47,
                             feat_dim=100, hidden=40, batch=128, feat_dtype="bf16")
    assert run_steps(w3, 6, use_cache=True, lr=0.02, bits=64, superbatch=2) > 0


@pytest.mark.parametrize("form", ["gcn", "gcn_sum", "gcn_sym"])
@pytest.mark.parametrize("F,d_out,relu,bf16", [(64, 64, True, False), (602, 256, True, False), (100, 47, False, False),
                                               (33, 5, True, False), (128, 256, True, True), (70, 41, False, False)])
def test_gcn_layer_forward_backward(F, d_out, relu, bf16, form):
    """GCN-style layer (Eq. 1 over N_in(v) U {v}: average, sum, or the symmetric normalisation of Table 1; one matrix)
    through its own entry points."""
    b = nb()
    norm = ora.gcn_norm_of(form)
    fcode = b.ARCH_OF_NAME[form]
    blk, x, xb, w_self, _, bias, rng = layer_case(4000, 60_000, F, d_out, (7, 6), 300, 11, bf16)
    n_dst, n_src = blk.n_dst, blk.n_src
    cap_dst, cap_src = n_dst + 77, n_src + 130
    d_n_dst, d_n_src = dev(np.array([n_dst], np.int32)), dev(np.array([n_src], np.int32))
    indptr = dev(np.concatenate([blk.indptr, np.zeros(77, np.int32)]))
    view = b.block_view_from_tensors(d_n_dst, d_n_src, indptr, dev(blk.indices), cap_dst, cap_src,
                                     dev(np.concatenate([blk.csc_indptr, np.zeros(130, np.int32)])), dev(blk.csc_dst))
    xs = dev(xb.view(np.int16)) if bf16 else dev(x)
    ws = torch.empty(b.no_sage_layer_ws_bytes(cap_dst, cap_src, F, d_out), dtype=torch.uint8, device="cuda")
    agg = torch.full((cap_dst, F), 7.0, device="cuda")
    h = torch.full((cap_dst, d_out), 7.0, device="cuda")
    tw, tbias = dev(w_self), dev(bias)
    b.no_gcn_layer_fwd(view, xs, tw, tbias, relu, agg, h, ws, form=fcode)
    o_agg, o_h = ora.gcn_layer_fwd(blk, x, w_self, bias, relu, norm)
    assert_close(agg[:n_dst].cpu().numpy(), o_agg, "agg")
    assert_close(h[:n_dst].cpu().numpy(), o_h, "h")
    assert (h[n_dst:] == 7.0).all() and (agg[n_dst:] == 7.0).all()
    grad_h = rng.standard_normal((n_dst, d_out)).astype(np.float32)
    o_h32 = o_h.astype(np.float32)
    gw = torch.zeros((F, d_out), device="cuda")
    gb = torch.zeros((d_out,), device="cuda")
    gx = torch.full((cap_src, F), 3.0, device="cuda")
    hh = torch.zeros((cap_dst, d_out), device="cuda")
    hh[:n_dst] = dev(o_h32)
    gh = torch.zeros((cap_dst, d_out), device="cuda")
    gh[:n_dst] = dev(grad_h)
    aa = torch.zeros((cap_dst, F), device="cuda")
    aa[:n_dst] = dev(o_agg.astype(np.float32))
    for need_gx in (True, False):
        b.no_gcn_layer_bwd(view, aa, hh, gh, tw, relu, gw, gb, gx if need_gx else None, ws, form=fcode)
        r = ora.gcn_layer_bwd(blk, o_agg.astype(np.float32), o_h32, grad_h, w_self, relu, need_gx, norm=norm)
        assert_close(gw.cpu().numpy(), r[0], "gw")
        assert_close(gb.cpu().numpy(), r[1], "gbias")
        if need_gx:
            assert_close(gx[:n_src].cpu().numpy(), r[2], "grad_x")
            assert (gx[n_src:] == 3.0).all()
    g1 = gw.clone()
    b.no_gcn_layer_bwd(view, aa, hh, gh, tw, relu, gw, gb, None, ws, form=fcode)
    assert torch.equal(g1, gw)
    if form == "gcn_sym":
        # the column sums come from the transpose: a view without one is refused
        bare = b.block_view_from_tensors(d_n_dst, d_n_src, indptr, dev(blk.indices), cap_dst, cap_src)
        with pytest.raises(b.NoError) as ei:
            b.no_gcn_layer_fwd(bare, xs, tw, tbias, relu, agg, h, ws, form=fcode)
        assert ei.value.code == -1


@pytest.mark.parametrize("arch", ["gcn", "gcn_sum", "gcn_sym"])
def test_gcn_train_steps(arch):
    """Whole steps with GCN-style layers (average, sum, symmetric normalisation): plain, with reuse (2 and 3 layers,
    bf16 table), under the super-batch schedule with bulk refresh, and with batches prepared ahead."""
    import dataclasses
    lr = 0.02 if arch != "gcn_sum" else 0.002        # (sums over up to 16 rows make larger activations)
    run_steps(si.WORKLOADS["tiny"], 3, use_cache=False, arch=arch, lr=lr)
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    assert run_steps(w, 5, use_cache=True, lr=lr, arch=arch) > 0
    w3 = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(4, 3, 3), staleness=3, hot_fraction=0.3, n_classes=47,
                             feat_dim=100, hidden=40, batch=128, feat_dtype="bf16")
    assert run_steps(w3, 6, use_cache=True, lr=lr, bits=64, superbatch=2, arch=arch) > 0
    assert run_steps(w3, 4, use_cache=True, lr=lr, bits=64, superbatch=2, arch=arch, ahead=True) > 0
    w1 = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(6,), batch=200)
    run_steps(w1, 2, use_cache=False, arch=arch, lr=lr)


def test_sampling_ahead_gives_the_same_steps():
    """no_train_step_ahead samples batch t+1 on a second stream while batch t trains: every step must equal the
    oracle's sequential step, with and without reuse, under the super-batch schedule (commit inside the call),
    for both layer forms; a lookahead that is not consumed is dropped."""
    import dataclasses
    run_steps(si.WORKLOADS["tiny"], 4, use_cache=False, ahead=True)
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    assert run_steps(w, 6, use_cache=True, lr=0.02, ahead=True) > 0
    w5 = dataclasses.replace(si.WORKLOADS["tiny"], staleness=5, hot_fraction=0.2)
    assert run_steps(w5, 9, use_cache=True, lr=0.02, superbatch=3, ahead=True) > 0
    w3 = dataclasses.replace(si.WORKLOADS["tiny"], fanouts=(4, 3, 3), staleness=3, hot_fraction=0.3, n_classes=47,
                             feat_dim=100, hidden=40, batch=128, feat_dtype="bf16")
    assert run_steps(w3, 6, use_cache=True, lr=0.02, bits=64, superbatch=2, ahead=True) > 0
    assert run_steps(w3, 4, use_cache=True, lr=0.02, bits=64, ahead=True, arch="gcn") > 0


@pytest.mark.parametrize("ahead", [False, True])
def test_every_vertex_hot_leaves_an_empty_bottom_hop(ahead):
    """Degenerate case of the reuse rule: with every vertex hot, a bulk refresh committed and the bound not yet
    exceeded, all of V^1 is served from the cache: the bottom hop has no destinations, layer 1 computes nothing and
    its gradients are exactly zero."""
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=3, hot_fraction=1.0)
    hits = run_steps(w, 5, use_cache=True, lr=0.02, superbatch=2, ahead=ahead)
    assert hits > 0


def test_sampling_ahead_dropped_when_not_consumed():
    """A batch prepared ahead that the next call does not ask for is dropped: the steps, and the cache they leave,
    equal those of plain stepping. The prepared batch's split had stamped the versions of the slots it would have
    recomputed; the call that drops it (or the model's destruction) must take those stamps back."""
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat = si.features(w.n_vertices, w.feat_dim, w.seed)
    lab = si.labels(w.n_vertices, w.n_classes, w.seed)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    weights = si.init_weights(w.dims, w.seed)
    losses, caches = [], []
    for mode in ("plain", "mismatch", "destroyed"):
        model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
        for l in range(w.n_layers):
            for t, a in zip(b.no_model_params(model, l + 1), weights[l]):
                t.copy_(dev(a))
        gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
        tfeat, tlab = dev(feat), dev(lab)
        seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(4)]
        out = []
        stamped_seen = 0
        for t in range(4):
            if mode == "plain":
                st = b.no_train_step(model, gg, tfeat, tlab, seeds[t], gc, t, w.seed, 0.02)
            else:
                # announce a batch that never comes (wrong tensor), then ask for the right one
                st = b.no_train_step_ahead(model, gg, tfeat, tlab, seeds[t], seeds[0], False, gc, t, w.seed, 0.02)
                torch.cuda.synchronize()
                stamped_seen += int((b.no_cache_view(gc, w.n_vertices)["version"] == t + 1).sum().item())
            out.append((st.loss, st.n_hit, tuple(st.n_src[:2])))
        if mode == "mismatch":
            assert stamped_seen > 0          # the case is exercised: prepared batches did stamp slots
            # one more plain call drops the last prepared batch
            st = b.no_train_step(model, gg, tfeat, tlab, seeds[0], gc, 4, w.seed, 0.0)
        elif mode == "plain":
            st = b.no_train_step(model, gg, tfeat, tlab, seeds[0], gc, 4, w.seed, 0.0)
        else:
            # the model goes away with a prepared batch pending; the cache must read as after four plain steps
            model.close()
            model = None
        torch.cuda.synchronize()
        view = b.no_cache_view(gc, w.n_vertices)
        caches.append((view["version"].cpu().numpy().copy(), view["emb"].cpu().numpy().copy()))
        losses.append(out)
        if model is not None:
            model.close()
        gc.close()
    assert losses[0] == losses[1] == losses[2]
    assert np.array_equal(caches[0][0], caches[1][0]) and np.array_equal(caches[0][1], caches[1][1])
    # "destroyed" stopped one (lr = 0) step earlier: its versions are those of plain stepping before that step, i.e.
    # no entry carries step 4
    assert (caches[2][0] <= 3).all()
    untouched = caches[0][0] <= 3
    assert np.array_equal(caches[2][0][untouched], caches[0][0][untouched])


def test_batch_prepared_ahead_and_dropped_after_an_error_copies_no_rows():
    """A call that ends in an error may leave a batch sampled ahead whose destination rows are not copied yet. The call that drops it
    must not copy them late: the table they come from may be gone."""
    b = nb()
    w = si.WORKLOADS["tiny"]
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    lab = dev(si.labels(w.n_vertices, w.n_classes, w.seed))
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    for l in range(w.n_layers):
        for t in b.no_model_params(model, l + 1):
            t.zero_()
    seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(4)]
    one = seeds[3][:1].clone()
    table, other = (torch.full((w.n_vertices, w.feat_dim), v, device="cuda") for v in (1.0, 3.0))
    n_rows = b.no_train_step_ahead(model, gg, table, lab, seeds[0], seeds[1], False, None, 0, 7, 0.0).n_dst[-1 + w.n_layers]
    torch.cuda.synchronize()
    table.fill_(2.0)                              # (the rows of batches 0 and 1 are copied)
    # an error of the caller's, not asked for yet, is what the step's first check of a launch finds: batch 2 is left sampled
    assert b.lib().hipSetDevice(1 << 20) != 0
    with pytest.raises(b.NoError) as ei:
        b.no_train_step_ahead(model, gg, table, lab, seeds[1], seeds[2], False, None, 1, 7, 0.0)
    assert ei.value.code == -5
    b.no_train_step(model, gg, other, lab, seeds[0], None, 2, 7, 0.0)                               # drops it
    b.no_train_step_ahead(model, gg, other, lab, seeds[0], one, False, None, 3, 7, 0.0)             # one seed: few rows, written over
    few = b.no_train_step(model, gg, other, lab, one, None, 4, 7, 0.0).n_dst[-1 + w.n_layers]      # the first rows of batch 0's copy
    rows = b.no_model_gathered(model, n_rows // 2)
    assert few < n_rows // 2 and (rows[:few] == 3.0).all() and (rows[few:] == 1.0).all()


def test_cache_invalidate_and_set_staleness():
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=3, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat = si.features(w.n_vertices, w.feat_dim, w.seed)
    lab = si.labels(w.n_vertices, w.n_classes, w.seed)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    for l in range(w.n_layers):
        for t, a in zip(b.no_model_params(model, l + 1), si.init_weights(w.dims, w.seed)[l]):
            t.copy_(dev(a))
    gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
    tfeat, tlab = dev(feat), dev(lab)
    step = lambda t: b.no_train_step(model, gg, tfeat, tlab, dev(si.batch_seeds(train, w.batch, t)), gc, t, 0, 0.01)
    assert step(0).n_hit == 0 and step(0).n_refresh >= 0
    assert step(1).n_hit > 0
    b.no_cache_invalidate(gc)
    assert step(2).n_hit == 0                      # every slot is empty again
    assert step(3).n_hit > 0
    b.no_cache_set_staleness(gc, 0)
    assert step(4).n_hit == 0                      # bound 0: nothing may be reused
    with pytest.raises(b.NoError):
        b.no_cache_set_staleness(gc, -1)
    st = step(5)
    assert st.n_v1 == st.n_dst[1] + st.n_hit and st.n_refresh <= st.n_dst[1]


def test_out_of_range_seed_is_flagged_not_followed():
    b = nb()
    w = si.WORKLOADS["tiny"]
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    feat, lab = dev(si.features(w.n_vertices, w.feat_dim, 0)), dev(si.labels(w.n_vertices, w.n_classes, 0))
    seeds = si.train_split(w.n_vertices, 0.65, 0)[:64].copy()
    st = b.no_train_step(model, gg, feat, lab, dev(seeds), None, 0, 0, 0.01)
    assert st.bad_seed == 0
    seeds[5] = w.n_vertices + 12345
    seeds[9] = -7
    st = b.no_train_step(model, gg, feat, lab, dev(seeds), None, 1, 0, 0.01)
    assert st.bad_seed == 1
    with pytest.raises(b.NoError) as ei:
        b.no_blocks_sizes(b.no_model_blocks(model))
    assert ei.value.code == -2
    # the flag belongs to the step that raised it: a clean batch afterwards reads 0 again
    seeds = si.train_split(w.n_vertices, 0.65, 0)[:64].copy()
    st = b.no_train_step(model, gg, feat, lab, dev(seeds), None, 2, 0, 0.01)
    assert st.bad_seed == 0 and st.bad_label == 0 and st.scan_timeout == 0
    b.no_blocks_sizes(b.no_model_blocks(model))
    # a label outside [0, C): flagged, and that seed adds nothing to the loss
    lab_bad = lab.clone()
    lab_bad[int(seeds[3])] = w.n_classes + 3
    lab_bad[int(seeds[4])] = -1
    m2 = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    m3 = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    for l in range(w.n_layers):
        for t2, t3, a in zip(b.no_model_params(m2, l + 1), b.no_model_params(m3, l + 1), si.init_weights(w.dims, 0)[l]):
            t2.copy_(dev(a))
            t3.copy_(dev(a))
    s_bad = b.no_train_step(m2, gg, feat, lab_bad, dev(seeds), None, 0, 0, 0.0)
    s_ok = b.no_train_step(m3, gg, feat, lab, dev(seeds), None, 0, 0, 0.0)
    assert s_bad.bad_label == 1 and s_ok.bad_label == 0
    gh = b.no_model_activations(m3, w.n_layers, 64, 64)[0].cpu().numpy().astype(np.float64)
    rows = ora.softmax_xent(gh, lab.cpu().numpy()[seeds])[0]        # mean over 64 rows
    per_row = [ora.softmax_xent(gh[i:i + 1], lab.cpu().numpy()[seeds[i:i + 1]])[0] for i in (3, 4)]
    assert abs(s_bad.loss - (rows * 64 - sum(per_row)) / 64) <= 1e-4 * abs(rows)
    # a train id outside [0, V) is refused by the hot selection, with and without sampled hops
    bad_train = dev(np.array([1, 2, w.n_vertices, 3], np.int32))
    for fan in ((3, 2), (3,)):
        with pytest.raises(b.NoError) as ei:
            b.no_select_hot(gg, bad_train, 2, fan, 1, 0.1, 1, 8, 0)
        assert ei.value.code == -2


@pytest.mark.parametrize("arch", ["sage", "gcn_sym"])
def test_seeds_that_are_not_different_vertices_stay_inside_the_arrays(arch):
    """Seeds outside [0, V) are all read as vertex 0, so that a batch may list more sources than the graph has vertices. Every array has
    room for them: the blocks agree with themselves, the step is flagged, and the next good batch is what it always is."""
    b = nb()
    V, batch, fanouts, dims = 1000, 1000, (10, 10, 5), [24, 32, 32, 8]
    src, dst, og, gg = make_graph(V, 30_000, 3, 32)
    order = np.random.default_rng(3).permutation(V).astype(np.int32)
    bad = order.copy()
    bad[::2] = V + 5
    blocks = b.no_blocks_create(gg, batch, fanouts)
    b.no_sample_blocks(gg, dev(bad), 1, 0, None, blocks)
    sizes = np.zeros((len(fanouts), 4), np.int32)
    assert b.lib().no_blocks_sizes(blocks.h, None, sizes.ctypes.data_as(b.C.POINTER(b.C.c_int32))) == -2
    assert sizes[:, 1].max() > V
    for h in range(len(fanouts)):
        a = b.block_arrays(blocks, h, sizes)
        new = a["src_global"][sizes[h, 0]:]
        assert len(np.unique(new)) == len(new) and new.min() >= 0 and new.max() < V
        assert np.array_equal(a["nbr_global"], a["src_global"][a["indices"]])
        if h < len(fanouts) - 1:
            e = a["csc_eid"]
            assert np.array_equal(np.sort(e), np.arange(len(e))) and (np.diff(a["indices"][e]) >= 0).all()
    good = order[:300]
    b.no_sample_blocks(gg, dev(good), 1, 1, None, blocks)
    compare_blocks(b, blocks, ora.sample_blocks(og, good, fanouts, 1, 1))

    feat, lab, train = dev(si.features(V, dims[0], 3)), dev(si.labels(V, dims[-1], 3)), dev(order)
    grads = []
    for batches in ((bad, good), (good,)):
        gc = b.no_select_hot(gg, train, 100, fanouts, 1, 0.3, 0, dims[1], 3)
        model = b.no_model_create(gg, dims, batch, fanouts)
        b.no_model_set_arch(model, b.ARCH_OF_NAME[arch])
        for l in range(3):
            for t, a in zip(b.no_model_params(model, l + 1), si.init_weights(dims, 3)[l]):
                t.copy_(dev(a))
        for ids in batches:
            st = b.no_train_step(model, gg, feat, lab, dev(ids), gc, 5, 3, 0.0)
            assert st.bad_seed == int(ids is bad)
            b.no_cache_invalidate(gc)
        grads.append([t.clone() for l in range(3) for t in b.no_model_grads(model, l + 1)])
    assert all(torch.equal(x, y) for x, y in zip(*grads))


def test_step_statistics_account_for_every_vertex_of_v1():
    """The statistics block of a step: hits, hot misses and cold vertices add up to |V^1|; bytes gathered are the
    bottom hop's distinct source rows and the reused layer-1 rows (Section 4.2, Stage 3 moves exactly these)."""
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat = si.features(w.n_vertices, w.feat_dim, w.seed)
    lab = si.labels(w.n_vertices, w.n_classes, w.seed)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    weights = si.init_weights(w.dims, w.seed)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    for l in range(w.n_layers):
        for t, a in zip(b.no_model_params(model, l + 1), weights[l]):
            t.copy_(dev(a))
    oc = ora.select_hot(og, train, w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
    gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
    tfeat, tlab = dev(feat), dev(lab)
    ow = [tuple(np.asarray(t, np.float64) for t in x) for x in weights]
    seen_hit = seen_miss = 0
    for step in range(4):
        seeds = si.batch_seeds(train, w.batch, step)
        before = oc.copy()
        st = b.no_train_step(model, gg, tfeat, tlab, dev(seeds), gc, step, w.seed, 0.02)
        r = ora.train_step(og, feat, lab, seeds, w.fanouts, ow, 0.02, w.seed, step, oc)
        ow = r.new_weights
        v1 = r.batch.blocks[-2].src_global
        hot = before.slot_of_vertex[v1] >= 0
        n_hit = len(r.batch.hit_pos)
        assert (st.n_v1, st.n_hit) == (len(v1), n_hit)
        assert st.n_miss_hot == int(hot.sum()) - n_hit == st.n_refresh
        assert st.n_cold == int((~hot).sum())
        assert st.n_hit + st.n_miss_hot + st.n_cold == st.n_v1
        assert st.bytes_gathered_features == r.batch.blocks[-1].n_src * w.feat_dim * 4
        assert st.bytes_gathered_embeddings == n_hit * w.hidden * 4
        seen_hit += n_hit
        seen_miss += st.n_miss_hot
    assert seen_hit > 0 and seen_miss > 0


SCAN_TILE = 1024      # slots per tile of the library's scans


@pytest.mark.parametrize("fanouts,batch,which", [((10, 10), 512, "edge scan"), ((1, 10), 1000, "V^1 split")])
def test_scan_wait_expiry_is_reported_and_every_kernel_still_ends(fanouts, batch, which):
    """Error path of the one-launch scans: the host makes tile 0 withhold its status word and shortens the bounded
    wait, so the tile after it must give up. The scan then leaves a consistent empty hop behind (so that no later
    kernel follows a wrong prefix out of its arrays), every kernel runs to its end, the step and the block sizes report
    NO_ERR_TIMEOUT, and the next call (limits restored) is clean again. Case 1: hop 0 spans several tiles of slots;
    case 2: hop 0 is a single tile and V^1 spans two."""
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2, batch=batch, fanouts=fanouts)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat, lab = dev(si.features(w.n_vertices, w.feat_dim, 0)), dev(si.labels(w.n_vertices, w.n_classes, 0))
    train = si.train_split(w.n_vertices, 0.65, 0)
    model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
    for l in range(w.n_layers):
        for t, a in zip(b.no_model_params(model, l + 1), si.init_weights(w.dims, 0)[l]):
            t.copy_(dev(a))
    gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, 0)
    seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(3)]
    st0 = b.no_train_step(model, gg, feat, lab, seeds[0], gc, 0, 0, 0.01)
    assert st0.scan_timeout == 0
    if which == "edge scan":
        assert st0.n_dst[0] * fanouts[0] > SCAN_TILE
    else:
        assert st0.n_dst[0] * fanouts[0] <= SCAN_TILE < st0.n_v1
    blocks = b.no_blocks_create(gg, w.batch, w.fanouts)
    try:
        b.no_debug_scan_wait(4, True)
        print("forcing the wait of the %s to expire" % which, flush=True)
        with pytest.raises(b.NoError) as ei:
            b.no_train_step(model, gg, feat, lab, seeds[1], gc, 1, 0, 0.0)
        st = ei.value.stats
        assert ei.value.code == -7 and st.scan_timeout == 1
        print("  sizes after the expiry:", list(st.n_dst[:2]), list(st.n_src[:2]), list(st.nnz[:2]), flush=True)
        assert st.nnz[0] == 0                                      # the hop the failed scan belongs to (or feeds) is empty
        if which == "edge scan":
            assert st.n_src[0] == st.n_dst[0]
        else:
            assert st.n_dst[1] == 0 and st.n_hit == 0
        with pytest.raises(b.NoError) as ei:
            b.no_blocks_sizes(b.no_model_blocks(model))
        assert ei.value.code == -7
        if which == "edge scan":
            b.no_sample_blocks(gg, seeds[1], 0, 1, None, blocks)
            with pytest.raises(b.NoError) as ei:
                b.no_blocks_sizes(blocks)
            assert ei.value.code == -7
    finally:
        b.no_debug_scan_wait(0, False)
    torch.cuda.synchronize()
    b.no_cache_invalidate(gc)          # the failed step may have stamped slots it never filled
    # the id map was left empty: the next calls are clean and exact again
    st2 = b.no_train_step(model, gg, feat, lab, seeds[2], gc, 2, 0, 0.01)
    assert st2.scan_timeout == 0
    compare_blocks(b, b.no_model_blocks(model), ora.sample_blocks(og, si.batch_seeds(train, w.batch, 2), w.fanouts, 0, 2))
    b.no_sample_blocks(gg, seeds[1], 0, 1, None, blocks)
    compare_blocks(b, blocks, ora.sample_blocks(og, si.batch_seeds(train, w.batch, 1), w.fanouts, 0, 1))


def test_refresh_commit_between_two_ahead_calls_drops_the_prepared_batch():
    """A batch prepared ahead was split against the cache as it stood. A bulk-refresh commit (or an invalidate, or a
    new bound) between the two calls replaces what it was split against: the prepared batch must be dropped and
    sampled again, and nothing may be 'restored' into the copy that holds the new rows. Steps and cache must equal
    plain stepping with the same commits."""
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=3, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat = si.features(w.n_vertices, w.feat_dim, w.seed)
    lab = si.labels(w.n_vertices, w.n_classes, w.seed)
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    weights = si.init_weights(w.dims, w.seed)
    results = []
    for mode in ("plain", "ahead"):
        model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
        for l in range(w.n_layers):
            for t, a in zip(b.no_model_params(model, l + 1), weights[l]):
                t.copy_(dev(a))
        gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
        tfeat, tlab = dev(feat), dev(lab)
        seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(7)]
        p1 = b.no_model_params(model, 1)
        out = []
        for t in range(6):
            if t == 2:
                b.no_refresh_hot_begin(gc, gg, tfeat, p1[0], p1[1], p1[2], w.fanouts[-1], t, w.seed)
            if t == 4:
                b.no_refresh_hot_commit(gc)           # between the call that prepared batch 4 and the one that trains it
            if t == 5:
                b.no_cache_set_staleness(gc, 1)       # a new bound also changes what a split would give
            if mode == "plain":
                st = b.no_train_step(model, gg, tfeat, tlab, seeds[t], gc, t, w.seed, 0.02)
            else:
                st = b.no_train_step_ahead(model, gg, tfeat, tlab, seeds[t], seeds[t + 1], False, gc, t, w.seed, 0.02)
            out.append((st.loss, st.n_hit, st.n_miss_hot, tuple(st.n_src[:2])))
        if mode == "ahead":
            b.no_train_step(model, gg, tfeat, tlab, seeds[0], gc, 6, w.seed, 0.0)     # drops the last prepared batch
        else:
            b.no_train_step(model, gg, tfeat, tlab, seeds[0], gc, 6, w.seed, 0.0)
        torch.cuda.synchronize()
        view = b.no_cache_view(gc, w.n_vertices)
        results.append((out, view["version"].cpu().numpy().copy(), view["emb"].cpu().numpy().copy()))
        model.close()
        gc.close()
    assert results[0][0] == results[1][0]
    assert np.array_equal(results[0][1], results[1][1]) and np.array_equal(results[0][2], results[1][2])
    assert any(o[1] > 0 for o in results[0][0])


def test_models_with_batches_prepared_ahead_come_and_go():
    """Every model that prepares batches ahead owns a helper thread, streams and events: several models created, stepped
    (alternately with and without a next batch, and with a next batch larger than the capacity, which is refused before
    anything is enqueued) and destroyed in turn leave nothing behind that disturbs the next one, and all give the same
    losses."""
    b = nb()
    import dataclasses
    w = dataclasses.replace(si.WORKLOADS["tiny"], staleness=2, hot_fraction=0.2)
    src, dst, og, gg = make_graph(w.n_vertices, w.n_edges, w.seed, 32)
    feat, lab = dev(si.features(w.n_vertices, w.feat_dim, w.seed)), dev(si.labels(w.n_vertices, w.n_classes, w.seed))
    train = si.train_split(w.n_vertices, 0.65, w.seed)
    weights = si.init_weights(w.dims, w.seed)
    seeds = [dev(si.batch_seeds(train, w.batch, t)) for t in range(5)]
    too_many = dev(train[: w.batch + 1].copy())
    runs = []
    for trial in range(4):
        model = b.no_model_create(gg, w.dims, w.batch, w.fanouts)
        for l in range(w.n_layers):
            for t, a in zip(b.no_model_params(model, l + 1), weights[l]):
                t.copy_(dev(a))
        gc = b.no_select_hot(gg, dev(train), w.batch, w.fanouts, 1, w.hot_fraction, w.staleness, w.hidden, w.seed)
        out = []
        for t in range(4):
            nxt = seeds[t + 1] if (t + trial) % 2 == 0 else None
            if t == 2:
                with pytest.raises(b.NoError) as ei:
                    b.no_train_step_ahead(model, gg, feat, lab, seeds[t], too_many, False, gc, t, w.seed, 0.02)
                assert ei.value.code == -3
            st = b.no_train_step_ahead(model, gg, feat, lab, seeds[t], nxt, False, gc, t, w.seed, 0.02)
            out.append((st.loss, st.n_hit, st.n_miss_hot))
        runs.append(out)
        model.close()
        gc.close()
    assert all(r == runs[0] for r in runs[1:])
    assert any(o[1] > 0 for o in runs[0])
