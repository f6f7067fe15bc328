"""GPU parity of kv_evict_topk: the keep list is bit-exact with the oracle's
selection, and the compacted K/V rows, positions and chunk ids are bit-exact
with the oracle's gather (position-keyed rows regenerate the expected cache)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ds():
    import paper_2609_27470_amd as ds
    ds.lib()
    return ds


def make_cache(L, row_elems, capacity, chunk, pos):
    """K/V planes whose row at slot i is the hash row of position pos[i]."""
    n = len(pos)
    pos_t = torch.zeros(capacity, dtype=torch.int64, device=DEV)
    pos_t[:n] = torch.as_tensor(np.asarray(pos, np.int64), device=DEV)
    ks, vs = [], []
    for l in range(L):
        kk = torch.zeros((capacity, row_elems), dtype=torch.int16, device=DEV)
        vv = torch.zeros((capacity, row_elems), dtype=torch.int16, device=DEV)
        kk[:n] = synth.kv_row_bits_torch(l, 0, pos_t[:n], row_elems)
        vv[:n] = synth.kv_row_bits_torch(l, 1, pos_t[:n], row_elems)
        ks.append(kk)
        vs.append(vv)
    p = torch.zeros(capacity, dtype=torch.int32, device=DEV)
    c = torch.zeros(capacity, dtype=torch.int32, device=DEV)
    p[:n] = torch.as_tensor(np.asarray(pos, np.int32), device=DEV)
    c[:n] = torch.as_tensor(np.asarray(chunk, np.int32), device=DEV)
    return ks, vs, p, c


def check_cache(ks, vs, p, c, M, exp_pos, exp_chunk):
    assert np.array_equal(p[:M].cpu().numpy(), exp_pos)
    assert np.array_equal(c[:M].cpu().numpy(), exp_chunk)
    ep = torch.as_tensor(np.asarray(exp_pos, np.int64), device=DEV)
    for l, (kk, vv) in enumerate(zip(ks, vs)):
        assert torch.equal(kk[:M], synth.kv_row_bits_torch(l, 0, ep, kk.shape[1])), f"K layer {l}"
        assert torch.equal(vv[:M], synth.kv_row_bits_torch(l, 1, ep, vv.shape[1])), f"V layer {l}"


def one_event(ds, L, row_elems, chunk, pos, scores, M, ns, nw, nb, capacity=None):
    n = len(pos)
    capacity = capacity or n
    ks, vs, p, c = make_cache(L, row_elems, capacity, chunk, pos)
    sc = torch.as_tensor(np.asarray(scores, np.float32), device=DEV)
    keep = torch.full((max(M, 1),), -1, dtype=torch.int32, device=DEV)
    new_len, ws = ds.kv_evict_topk(ks, vs, p, c, sc, n, M, ns, nw, nb, keep_out=keep)
    torch.cuda.synchronize()
    ref = oracle.select_keep(chunk, pos, scores, n, M, ns, nw, nb)
    if n <= M:
        assert new_len == n
        check_cache(ks, vs, p, c, n, np.asarray(pos), np.asarray(chunk))
        return
    assert new_len == M
    assert keep[:M].cpu().tolist() == ref
    st = ds.kv_device_status(ws)
    assert st[0] == 0 and st[2] == 0, st
    check_cache(ks, vs, p, c, M, np.asarray(pos)[ref], np.asarray(chunk)[ref])


def random_cache(rng, n_chunks, lo, hi, thin=0.8):
    lens = rng.integers(lo, hi + 1, n_chunks)
    chunk = np.repeat(np.arange(n_chunks), lens)
    keep = rng.random(len(chunk)) < thin
    chunk = chunk[keep]
    pos = (np.nonzero(keep)[0] + 3).astype(np.int64)
    return chunk.astype(np.int32), pos.astype(np.int32)


@pytest.mark.parametrize("seed", range(12))
def test_random_small_caches(ds, seed):
    rng = np.random.default_rng(1000 + seed)
    chunk, pos = random_cache(rng, int(rng.integers(3, 40)), 1, 60)
    n = len(chunk)
    scores = rng.choice([0.1, 0.25, 0.5, 1.0, 2.0], size=int(chunk.max()) + 1).astype(np.float32)
    if seed % 3 == 0:
        scores[0] = np.inf
    ns = int(rng.integers(0, 5))
    nw = int(rng.integers(0, 40))
    M = int(rng.integers(ns + nw, n + 3))
    nb = int(rng.integers(0, 9))
    one_event(ds, 2, 64 * (1 + seed % 3), chunk, pos, scores, M, ns, nw, nb)


@pytest.mark.parametrize("n_chunks,lo,hi,nb,window", [(1024, 1, 20, 1, False), (1500, 1, 16, 5, True),
                                                      (2048, 2, 6, 3, False), (3000, 1, 8, 4, True)])
def test_many_runs(ds, n_chunks, lo, hi, nb, window):
    """About 1000 to 3000 runs: the ranking sorts up to 2048 runs in LDS (the
    2048-chunk case without sinks and window has exactly 2048 candidate runs)
    and compares every pair in global memory beyond that (the 3000-chunk
    case).  Scores from a small set, so many runs tie on the score and are
    ordered by chunk id."""
    rng = np.random.default_rng(n_chunks + nb)
    chunk, pos = random_cache(rng, n_chunks, lo, hi, thin=0.9)
    if n_chunks == 2048:  # every chunk present: exactly 2048 runs
        chunk = np.repeat(np.arange(n_chunks), 3).astype(np.int32)
        pos = np.arange(len(chunk), dtype=np.int32) * 2 + 1
    n = len(chunk)
    scores = rng.choice([0.1, 0.2, 0.3, 0.5, 1.0], size=int(chunk.max()) + 1).astype(np.float32)
    scores[rng.integers(0, len(scores), 3)] = np.inf
    ns, nw = (4, n // 10) if window else (0, 0)
    one_event(ds, 1, 8, chunk, pos, scores, n * 2 // 3, ns, nw, nb)


def test_golden_examples_on_gpu(ds):
    import json, math, os
    gd = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "select_examples.json")))
    chunk = np.array(gd["cache"]["chunk_id"], np.int32)
    pos = np.array(gd["cache"]["pos"], np.int32)
    for c in gd["cases"]:
        sc = [math.inf if s == "inf" else float(s) for s in c["chunk_scores"]]
        one_event(ds, 1, 8, chunk, pos, sc, c["M"], c["n_sink"], c["n_window"], c["n_buckets"])


def test_equal_scores_keep_newest(ds):
    chunk = np.repeat(np.arange(10), 50).astype(np.int32)
    pos = np.arange(500, dtype=np.int32)
    one_event(ds, 1, 64, chunk, pos, np.full(10, 0.5, np.float32), 123, 0, 0, 1)


@pytest.mark.parametrize("policy", [(0, 0, 1), (4, 1024, 4)])
def test_eviction_loop_shape(ds, policy):
    """The eviction-loop cache at full size: 8 layers x (K, V) x 8 heads x 256
    bf16 (4 KiB rows), 17 chunks of 1024 tokens, budget 16384, capacity 17408."""
    ns, nw, nb = policy
    rng = np.random.default_rng(5)
    chunk = np.repeat(np.arange(17), 1024).astype(np.int32)
    pos = np.arange(17 * 1024, dtype=np.int32) + 40000
    scores = rng.random(17).astype(np.float32)
    scores[3] = np.inf
    one_event(ds, 8, 2048, chunk, pos, scores, 16384, ns, nw, nb)


def test_two_shifts_in_one_event(ds):
    """64 KiB of rows per token (8 layers x 4 KiB K and V): the first moved
    rows shift by 512 slots and the later ones by 1536, in one event: 512 oldest
    tokens of chunk 2 and all of chunk 12 are evicted."""
    chunk = np.concatenate([np.repeat(np.arange(17), 1024), np.full(512, 17)]).astype(np.int32)
    pos = np.arange(len(chunk), dtype=np.int32) + 7
    scores = np.linspace(0.5, 1.0, 18).astype(np.float32)
    scores[12] = 0.01
    scores[2] = 0.02
    one_event(ds, 8, 2048, chunk, pos, scores, 16384, 0, 0, 1)


def test_small_shifts_full_shape(ds):
    """The paper's policy on the eviction-loop shape with chunks of 125
    tokens: every event removes a few scattered tokens, so every moved row
    shifts by at most 125 slots (strips in two segments, whose tails are staged)."""
    rng = np.random.default_rng(9)
    chunk = np.repeat(np.arange(140), 125)[:16384 + 125].astype(np.int32)
    pos = np.arange(len(chunk), dtype=np.int32)
    scores = rng.random(140).astype(np.float32)
    one_event(ds, 8, 2048, chunk, pos, scores, 16384, 4, 1024, 4)


def test_repeated_events_stream(ds):
    """Append a chunk per step and evict down to M every time the cache
    overflows; after every step the cache equals the oracle's replay."""
    L, row, M, F, capacity = 3, 128, 700, 96, 700 + 96
    rng = np.random.default_rng(11)
    steps = 40
    scores_all = rng.random(steps).astype(np.float32)
    scores_all[0] = np.inf
    ks, vs, p, c = make_cache(L, row, capacity, [], [])
    sc = torch.as_tensor(scores_all, device=DEV)
    ref_pos, ref_chunk = np.zeros(0, np.int64), np.zeros(0, np.int64)
    n = 0
    ws = None
    for f in range(steps):
        new_pos = np.arange(f * F, (f + 1) * F, dtype=np.int64)
        pt = torch.as_tensor(new_pos, device=DEV)
        for l in range(L):
            ks[l][n:n + F] = synth.kv_row_bits_torch(l, 0, pt, row)
            vs[l][n:n + F] = synth.kv_row_bits_torch(l, 1, pt, row)
        p[n:n + F] = pt.to(torch.int32)
        c[n:n + F] = f
        n += F
        ref_pos = np.concatenate([ref_pos, new_pos])
        ref_chunk = np.concatenate([ref_chunk, np.full(F, f)])
        new_len, ws = ds.kv_evict_topk(ks, vs, p, c, sc, n, M, 4, 64, 4, workspace=ws)
        if n > M:
            keep = oracle.select_keep(ref_chunk, ref_pos, scores_all, n, M, 4, 64, 4)
            ref_pos, ref_chunk = ref_pos[keep], ref_chunk[keep]
        n = new_len
        torch.cuda.synchronize()
        check_cache(ks, vs, p, c, n, ref_pos, ref_chunk)


def test_broken_invariants_leave_cache_untouched(ds):
    chunk = np.repeat(np.arange(6), 20).astype(np.int32)
    chunk[50] = 0                                   # chunk ids go backwards
    pos = np.arange(120, dtype=np.int32)
    ks, vs, p, c = make_cache(1, 64, 120, chunk, pos)
    before = ks[0].clone()
    sc = torch.ones(6, dtype=torch.float32, device=DEV)
    new_len, ws = ds.kv_evict_topk(ks, vs, p, c, sc, 120, 60, 0, 0, 1)
    torch.cuda.synchronize()
    assert ds.kv_device_status(ws)[0] == 1
    assert torch.equal(ks[0], before)
    assert np.array_equal(p.cpu().numpy(), pos)


# ---------------------------------------------------------------- slot-indexed variant
def indexed_event(ds, chunk, pos, scores, M, ns, nw, nb, seed=0, capacity=None):
    """kv_evict_topk_indexed on a table whose rows are scattered over the
    physical cache; keep list, compacted table and free list bit-exact with
    the oracle."""
    n = len(pos)
    capacity = capacity or n + 5
    rng = np.random.default_rng(seed)
    slot = rng.permutation(capacity)[:n].astype(np.int32)
    mk = lambda a: torch.as_tensor(np.concatenate([np.asarray(a, np.int32),
                                                   np.full(capacity - n, -7, np.int32)]), device=DEV)
    p, c, s = mk(pos), mk(chunk), mk(slot)
    sc = torch.as_tensor(np.asarray(scores, np.float32), device=DEV)
    keep = torch.full((max(M, 1),), -1, dtype=torch.int32, device=DEV)
    new_len, ws, free = ds.kv_evict_topk_indexed(p, c, s, sc, n, M, ns, nw, nb, keep_out=keep)
    torch.cuda.synchronize()
    if n <= M:
        assert new_len == n
        assert np.array_equal(s[:n].cpu().numpy(), slot) and np.array_equal(p[:n].cpu().numpy(), pos)
        return
    ref = oracle.select_keep(chunk, pos, scores, n, M, ns, nw, nb)
    assert new_len == M
    assert ds.kv_device_status(ws)[0] == 0
    assert keep[:M].cpu().tolist() == ref
    ep, ec, es, efree = oracle.compact_indexed(pos, chunk, slot, ref, n)
    assert np.array_equal(p[:M].cpu().numpy(), ep)
    assert np.array_equal(c[:M].cpu().numpy(), ec)
    assert np.array_equal(s[:M].cpu().numpy(), es)
    assert np.array_equal(free[:n - M].cpu().numpy(), efree)
    assert np.array_equal(s[n:].cpu().numpy(), np.full(capacity - n, -7))   # beyond len: untouched


@pytest.mark.parametrize("seed", range(8))
def test_indexed_random_small_caches(ds, seed):
    rng = np.random.default_rng(2000 + seed)
    chunk, pos = random_cache(rng, int(rng.integers(3, 40)), 1, 60)
    n = len(chunk)
    scores = rng.choice([0.1, 0.25, 0.5, 1.0, 2.0], size=int(chunk.max()) + 1).astype(np.float32)
    ns = int(rng.integers(0, 5))
    nw = int(rng.integers(0, 40))
    M = int(rng.integers(ns + nw, n + 3))
    indexed_event(ds, chunk, pos, scores, M, ns, nw, int(rng.integers(0, 9)), seed=seed)


@pytest.mark.parametrize("policy", [(0, 0, 1), (4, 1024, 4)])
def test_indexed_eviction_loop_shape(ds, policy):
    """17 chunks of 1024 tokens down to 16384, capacity 17408."""
    rng = np.random.default_rng(6)
    chunk = np.repeat(np.arange(17), 1024).astype(np.int32)
    pos = np.arange(17 * 1024, dtype=np.int32) + 40000
    scores = rng.random(17).astype(np.float32)
    indexed_event(ds, chunk, pos, scores, 16384, *policy, seed=3, capacity=17408)


def test_indexed_long_cache_several_blocks(ds):
    """A cache of ~100k tokens, so that selection and the table compaction
    both run over several 32768-slot blocks."""
    rng = np.random.default_rng(8)
    chunk, pos = random_cache(rng, 90, 900, 1400, thin=0.9)
    scores = rng.random(90).astype(np.float32)
    n = len(chunk)
    indexed_event(ds, chunk, pos, scores, n // 2, 4, 1000, 5, seed=4)


@pytest.mark.parametrize("n_chunks", [1500, 2600])
def test_indexed_many_runs(ds, n_chunks):
    """The slot-indexed eviction over caches of 1500 and 2600 short chunks:
    its ranking takes the sorted path (up to 2048 runs) and the pairwise one
    over the global run table (beyond)."""
    rng = np.random.default_rng(70 + n_chunks)
    chunk, pos = random_cache(rng, n_chunks, 1, 12, thin=0.9)
    scores = rng.choice([0.1, 0.2, 0.5, 1.0], size=n_chunks).astype(np.float32)
    n = len(chunk)
    indexed_event(ds, chunk, pos, scores, n * 3 // 4, 4, 64, 3, seed=9)


def test_indexed_matches_gather_in_a_stream(ds):
    """Appends write each new chunk's K/V rows into the rows the previous
    eviction freed (an index_copy by the caller); after every step the rows
    read through the table equal the position-keyed rows of the gather-based
    cache, which the gather variant itself rebuilds in the same loop."""
    L, row, M, F, capacity = 2, 128, 700, 96, 700 + 96
    rng = np.random.default_rng(12)
    steps = 30
    scores_all = rng.random(steps).astype(np.float32)
    scores_all[0] = np.inf
    sc = torch.as_tensor(scores_all, device=DEV)
    # gather-based cache
    ks, vs, p, c = make_cache(L, row, capacity, [], [])
    # indexed cache: physical rows + table
    kx = [torch.zeros((capacity, row), dtype=torch.int16, device=DEV) for _ in range(L)]
    tp = torch.zeros(capacity, dtype=torch.int32, device=DEV)
    tc = torch.zeros(capacity, dtype=torch.int32, device=DEV)
    ts = torch.zeros(capacity, dtype=torch.int32, device=DEV)
    free = torch.arange(capacity, dtype=torch.int32, device=DEV)
    n, ws_g, ws_x = 0, None, None
    for f in range(steps):
        pt = torch.arange(f * F, (f + 1) * F, dtype=torch.int64, device=DEV) + 77
        dst = free[:F].to(torch.int64)
        for l in range(L):
            rows_k = synth.kv_row_bits_torch(l, 0, pt, row)
            ks[l][n:n + F] = rows_k
            vs[l][n:n + F] = synth.kv_row_bits_torch(l, 1, pt, row)
            kx[l].index_copy_(0, dst, rows_k)
        p[n:n + F] = pt.to(torch.int32)
        c[n:n + F] = f
        tp[n:n + F] = pt.to(torch.int32)
        tc[n:n + F] = f
        ts[n:n + F] = dst.to(torch.int32)
        n += F
        kg = torch.empty(M, dtype=torch.int32, device=DEV)
        kxk = torch.empty(M, dtype=torch.int32, device=DEV)
        new_len, ws_g = ds.kv_evict_topk(ks, vs, p, c, sc, n, M, 4, 64, 4, keep_out=kg, workspace=ws_g)
        new_x, ws_x, freed = ds.kv_evict_topk_indexed(tp, tc, ts, sc, n, M, 4, 64, 4, keep_out=kxk,
                                                      workspace=ws_x)
        assert new_x == new_len
        free = free[F:]                              # rows never used so far
        if n > M:
            assert torch.equal(kg, kxk)
            free = torch.cat([free, freed[:n - M]])
        n = new_len
        torch.cuda.synchronize()
        assert torch.equal(tp[:n], p[:n]) and torch.equal(tc[:n], c[:n])
        idx = ts[:n].to(torch.int64)
        for l in range(L):
            assert torch.equal(kx[l][idx], ks[l][:n]), f"step {f} layer {l}"
        assert sorted(torch.cat([ts[:n], free]).cpu().tolist()) == list(range(capacity))


def test_indexed_broken_invariants_leave_table_untouched(ds):
    chunk = np.repeat(np.arange(6), 20).astype(np.int32)
    pos = np.arange(120, dtype=np.int32)
    pos[70] = pos[69]                                # positions not increasing
    p = torch.as_tensor(pos, device=DEV)
    c = torch.as_tensor(chunk, device=DEV)
    s = torch.arange(120, dtype=torch.int32, device=DEV)
    free = torch.full((60,), -3, dtype=torch.int32, device=DEV)
    sc = torch.ones(6, dtype=torch.float32, device=DEV)
    new_len, ws, _ = ds.kv_evict_topk_indexed(p, c, s, sc, 120, 60, 0, 0, 1, free_out=free)
    torch.cuda.synchronize()
    assert ds.kv_device_status(ws)[0] == 1
    assert np.array_equal(p.cpu().numpy(), pos) and np.array_equal(c.cpu().numpy(), chunk)
    assert torch.equal(s, torch.arange(120, dtype=torch.int32, device=DEV))
    assert torch.equal(free, torch.full((60,), -3, dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("na,nb,T,n,row", [(50, 30, 40, 10, 64), (50, 30, 70, 20, 4096), (0, 80, 80, 0, 16),
                                           (80, 0, 0, 7, 64), (300, 700, 257, 600, 4096), (1024, 0, 1, 0, 48)])
def test_append_indexed_matches_indexing(ds, na, nb, T, n, row):
    """kv_append_indexed against plain tensor indexing: each plane's rows at
    the first T entries of free_a ++ free_b hold the new rows, every other row
    keeps its bytes; pos, chunk_id and slot [n, n + T) hold the positions,
    the chunk id and those rows, the rest of each table is untouched; the
    rest of the list lands in free_rest.  Bit for bit, spanning several
    256-entry blocks of the list copy and both list segments."""
    capacity = 1024 + 64
    g = torch.Generator(device=DEV).manual_seed(na * 7 + nb + T)
    L = 3
    kp = torch.randint(-30000, 30000, (L, capacity, row // 2), dtype=torch.int16, device=DEV, generator=g)
    vp = torch.randint(-30000, 30000, (L, capacity, row // 2), dtype=torch.int16, device=DEV, generator=g)
    kn = torch.randint(-30000, 30000, (L, T + 5, row // 2), dtype=torch.int16, device=DEV, generator=g)
    vn = torch.randint(-30000, 30000, (L, T + 5, row // 2), dtype=torch.int16, device=DEV, generator=g)
    perm = torch.randperm(capacity, generator=torch.Generator().manual_seed(T)).to(torch.int32).to(DEV)
    fa, fb = perm[:na].clone(), perm[na:na + nb].clone()
    rest = torch.full((capacity,), -9, dtype=torch.int32, device=DEV)
    tabs = [torch.randint(-100, 100, (capacity,), dtype=torch.int32, device=DEV, generator=g) for _ in range(3)]
    exp_k, exp_v, exp_tabs = kp.clone(), vp.clone(), [t.clone() for t in tabs]
    lst = torch.cat([fa, fb]).to(torch.int64)
    dst = lst[:T]
    exp_k[:, dst] = kn[:, :T]
    exp_v[:, dst] = vn[:, :T]
    exp_tabs[0][n:n + T] = torch.arange(5000, 5000 + T, dtype=torch.int32, device=DEV)
    exp_tabs[1][n:n + T] = 37
    exp_tabs[2][n:n + T] = dst.to(torch.int32)
    ds.kv_append_indexed(kp, vp, kn, vn, fa if na else None, na, fb if nb else None, nb, rest, T, n, 5000, 37,
                         *tabs)
    torch.cuda.synchronize()
    assert torch.equal(kp, exp_k) and torch.equal(vp, exp_v)
    for t, e in zip(tabs, exp_tabs):
        assert torch.equal(t, e)
    r = na + nb - T
    assert torch.equal(rest[:r], lst[T:].to(torch.int32)) and bool((rest[r:] == -9).all())


@pytest.mark.parametrize("L,row_elems", [(1, 8), (1, 24), (3, 72), (2, 1032), (1, 2048), (16, 64)])
@pytest.mark.parametrize("n,M,step", [(700, 699, 1), (1500, 900, 40), (2000, 64, 50), (4100, 4000, 100), (3001, 1500, 7)])
def test_strips_and_segments(ds, L, row_elems, n, M, step):
    """The in-place move at its edges: rows of one 16-byte unit, rows that end in
    the middle of a 128-byte strip, few planes (many segments, whose tails are
    staged) and many; one evicted token, tails longer than a segment, more
    evicted than kept, a budget smaller than a batch of rows.  Scores with many
    ties; the tokens evicted are spread over spans."""
    rng = np.random.default_rng(n + M + L + row_elems)
    chunk = (np.arange(n) // step).astype(np.int32)
    pos = (np.arange(n) * 2 + 5).astype(np.int32)
    scores = rng.choice([0.1, 0.2, 0.4, 0.8], size=int(chunk[-1]) + 1).astype(np.float32)
    one_event(ds, L, row_elems, chunk, pos, scores, M, min(4, M // 8), M // 10, 3, capacity=n + 13)


def test_many_strips_of_wide_rows(ds):
    """64 KiB rows (512 strips a plane) and a first chunk evicted: every row moves, in one segment."""
    chunk = np.repeat(np.arange(5), 60).astype(np.int32)
    scores = np.array([0.1, 1, 1, 1, 1], np.float32)
    one_event(ds, 1, 32768, chunk, np.arange(300, dtype=np.int32), scores, 240, 0, 0, 1)


@pytest.mark.parametrize("n,runs,M,ns,nw,nb", [
    (20480, 1, 20479, 0, 0, 1), (20481, 2, 20480, 4, 255, 2), (20479, 15, 16384, 0, 0, 4), (24577, 16, 20481, 256, 256, 1),
    (41000, 17, 30000, 5, 1023, 3), (4096, 31, 1, 0, 0, 1), (4097, 64, 4096, 3, 1, 5), (6000, 127, 5000, 0, 100, 2),
    (9000, 511, 8000, 1, 0, 4), (9000, 512, 4000, 0, 7, 1), (9000, 513, 4000, 7, 0, 7), (300, 300, 150, 0, 0, 1),
    (1024, 1, 600, 300, 300, 1), (8317, 1040, 8192, 4, 0, 4), (8200, 2047, 8100, 0, 9, 3), (8200, 2049, 8000, 3, 0, 1),
    (4000, 3999, 2000, 0, 0, 4), (12000, 380, 9000, 4, 64, 2), (40000, 1300, 16000, 16, 1000, 8)])
def test_selection_edges(ds, n, runs, M, ns, nw, nb):
    """Lengths around a step of the selection (20480 slots), run counts around a run per wave, the lanes that share a
    run's comparisons and the sorted ranking (from 513 on), short runs that share a wave (with a long one among them in
    test_long_runs_among_short_ones), budgets within and beyond the copy of the keep list."""
    rng = np.random.default_rng(n + runs)
    cuts = np.sort(rng.choice(np.arange(1, n), runs - 1, replace=False))
    chunk = np.searchsorted(cuts, np.arange(n), side="right").astype(np.int32)
    pos = np.cumsum(rng.integers(1, 4, n)).astype(np.int32)
    scores = rng.choice([0.1, 0.2, 0.5, 1.0, np.inf], size=runs).astype(np.float32)
    one_event(ds, 1, 8, chunk, pos, scores, M, ns, nw, nb)
    indexed_event(ds, chunk, pos, scores, M, ns, nw, nb, seed=2)


@pytest.mark.parametrize("n,at", [(700, 1), (700, 699), (5000, 4096), (20480, 257), (20480, 20479), (41000, 1024),
                                  (41000, 15 * 256 + 3), (41000, 20480), (41000, 25000), (41000, 40999)])
def test_one_violation_anywhere_leaves_the_cache_untouched(ds, n, at):
    """A position that repeats its predecessor, seen by one lane of one wave (the first wave, which clears the flag it
    raises, the last, a later block or step): nothing is moved or rewritten, in either form of the cache."""
    chunk = torch.arange(n, dtype=torch.int32, device=DEV) // 50
    pos = torch.arange(n, dtype=torch.int32, device=DEV)
    pos[at] = pos[at - 1]
    scores = torch.rand(int(chunk[-1]) + 1, device=DEV)
    M = n - 40
    k = torch.randint(-99, 99, (n, 8), dtype=torch.int16, device=DEV)
    k0, p0, c0, keep = k.clone(), pos.clone(), chunk.clone(), torch.full((M,), -1, dtype=torch.int32, device=DEV)
    _, ws = ds.kv_evict_topk([k], [k0.clone()], pos, chunk, scores, n, M, 4, 100, 2, keep_out=keep)
    assert ds.kv_device_status(ws)[0] == 1
    assert torch.equal(k, k0) and torch.equal(pos, p0) and torch.equal(chunk, c0) and bool((keep == -1).all())
    slot = torch.randperm(n, device=DEV).to(torch.int32)
    s0, free = slot.clone(), torch.full((40,), -1, dtype=torch.int32, device=DEV)
    _, ws, _ = ds.kv_evict_topk_indexed(pos, chunk, slot, scores, n, M, 4, 100, 2, keep_out=keep, free_out=free)
    assert ds.kv_device_status(ws)[0] == 1
    assert torch.equal(pos, p0) and torch.equal(chunk, c0) and torch.equal(slot, s0)
    assert bool((keep == -1).all()) and bool((free == -1).all())


@pytest.mark.parametrize("n_long,long,n_short,short", [(1, 9000, 2000, 1), (3, 700, 900, 4), (40, 130, 1500, 3), (2, 33, 300, 4),
                                                       (2, 32, 300, 4), (1, 20000, 1900, 2), (5, 300, 2500, 2)])
def test_long_runs_among_short_ones(ds, n_long, long, n_short, short):
    """Runs far from the average length, which whole waves write while groups of lanes write the others: first, last and in
    the middle, evicted and kept."""
    rng = np.random.default_rng(n_long + long)
    lens = np.full(n_short + n_long, short)
    lens[np.sort(rng.choice(len(lens), n_long, replace=False))] = long
    if n_long > 1:
        lens[0] = lens[-1] = long
    chunk = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    n = len(chunk)
    pos = np.cumsum(rng.integers(1, 4, n)).astype(np.int32)
    scores = rng.random(len(lens)).astype(np.float32)
    for M in (n - 3, n // 2):
        one_event(ds, 1, 8, chunk, pos, scores, M, 4, 0, 2)
        indexed_event(ds, chunk, pos, scores, M, 0, min(50, M), 1, seed=3)


def test_many_short_runs_take_their_share_of_the_time(ds):
    """16509 slots in 2064 runs take 3.3 times as long to select from as in 258 runs (the ranking sorts 8 times as many);
    with a whole wave a run it was 4.8 times."""
    M, n = 16384, 16509
    i = torch.arange(n, dtype=torch.int32, device=DEV)
    ws = torch.empty(ds.kv_indexed_workspace_bytes(n), dtype=torch.uint8, device=DEV)
    free = torch.empty(n - M, dtype=torch.int32, device=DEV)

    def of(run):
        chunk0 = i // run
        scores = torch.rand(int(chunk0[-1]) + 1, generator=torch.Generator().manual_seed(1)).to(DEV)
        pos, chunk, slot = i.clone(), chunk0.clone(), i.clone()

        def restore():
            pos.copy_(i), chunk.copy_(chunk0), slot.copy_(i)

        def event():
            restore()
            ds.kv_evict_topk_indexed(pos, chunk, slot, scores, n, M, 4, 1024, 4, free_out=free, workspace=ws)

        def per_call(f):
            f()
            best = float("inf")
            for _ in range(5):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                for _ in range(20):
                    f()
                e1.record()
                e1.synchronize()
                best = min(best, e0.elapsed_time(e1) / 20)
            return best
        return per_call(event) - per_call(restore)
    for _ in range(3):   # (times of a shared machine)
        few, many = of(64), of(8)
        if many <= 4.1 * few:
            return
    assert False, (many, few)
