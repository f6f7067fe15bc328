"""gdn_layers_fwd (every layer of a chunk in one call, rows at a pitch) against
one gdn_chunk_fwd call per layer, and gdn_pack_layers against plain copies.

Where both take the per-slice kernel the results are the same bits.  From 64
heads on the layers take the whole-head kernel: the same operations on the same
operands, but where the compiler fuses a product with its rounding to fp16 in one
kernel only, an element in about 2^13 may be rounded the other way (2^-11 of it):
5e-6 of the norm, ten times that is allowed; a bf16 o may flip (2^-8) in one element
in 2^10 besides."""
import pytest
import torch

from gpu_helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ds():
    import paper_2609_27470_amd as ds
    ds.lib()
    return ds


def layers(L, T, H_k, H_v, d, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(torch.bfloat16)  # noqa: E731
    return [(unit(rnd(T, H_k, d)), unit(rnd(T, H_k, d)), rnd(T, H_v, d).to(torch.bfloat16),
             -torch.nn.functional.softplus(rnd(T, H_v)), torch.sigmoid(rnd(T, H_v))) for _ in range(L)]


def packed_like(ds, xs, T, pitch):
    out = tuple(torch.full((len(xs), pitch) + t.shape[1:], 7, dtype=t.dtype, device=DEV) for t in xs[0])
    ds.gdn_pack_layers(xs, T, out)
    return out


def rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("per_slice", [True, False])
@pytest.mark.parametrize("L,T,pitch,H_k,H_v,d,odt", [
    (3, 1, 1, 2, 2, 64, torch.float32), (3, 65, 70, 2, 4, 64, torch.bfloat16), (1, 125, 132, 2, 4, 128, torch.float32),
    (15, 129, 132, 2, 4, 128, torch.bfloat16), (16, 63, 64, 2, 4, 128, torch.float32),
    (16, 128, 131, 1, 4, 128, torch.bfloat16), (5, 132, 132, 8, 16, 128, torch.float32),
    (24, 64, 132, 8, 16, 128, torch.bfloat16)])
def test_layers_match_one_call_per_layer(ds, L, T, pitch, H_k, H_v, d, odt, per_slice):
    xs = layers(L, T, H_k, H_v, d)
    S0 = 0.3 * torch.randn(L, 1, H_v, d, d, device=DEV)
    pairs = H_v * (d // 16) if per_slice else H_v
    ref_o, ref_S = torch.empty(L, T, H_v, d, dtype=odt, device=DEV), S0.clone()
    ref_p = torch.empty(L, 1, pairs, 2, device=DEV)
    for l, x in enumerate(xs):
        ds.gdn_chunk_fwd(*x, [T], 0, state_in=ref_S[l], state_out=ref_S[l], o=ref_o[l], drift_partials=ref_p[l],
                         drift_per_slice=per_slice)
    S, p = S0.clone(), torch.empty_like(ref_p)
    o = torch.full((L, pitch, H_v, d), 5, dtype=odt, device=DEV)
    ws = torch.empty(ds.gdn_workspace_bytes(ds.gdn_shape([T] * L, H_k, H_v, d, 0, per_slice)), dtype=torch.uint8, device=DEV)
    ds.gdn_layers_fwd(*packed_like(ds, xs, T, pitch), T, S, o, p, ws, drift_per_slice=per_slice)
    torch.cuda.synchronize()
    if L * H_v < 64 or d == 64:
        assert torch.equal(o[:, :T], ref_o) and torch.equal(S, ref_S) and torch.equal(p, ref_p)
    else:
        assert rel(o[:, :T], ref_o) <= (5e-5 if odt == torch.float32 else 2e-4) and rel(S, ref_S) <= 5e-5
        assert rel(p, ref_p) <= 1e-4
    assert bool((o[:, T:] == 5).all())


def test_small_q_in_the_first_tile(ds):
    """Layers on the whole-head kernel take P from the bf16 inputs: a q whose fp16 copies would be subnormal costs the
    first tile's o nothing."""
    L, T, H_k, H_v, d, scale = 24, 64, 8, 16, 128, 2.0 ** 17
    xs = [((x[0].float() / scale).to(torch.bfloat16),) + x[1:] for x in layers(L, T, H_k, H_v, d)]
    S, p = torch.zeros(L, 1, H_v, d, d, device=DEV), torch.empty(L, 1, H_v, 2, device=DEV)
    o = torch.empty(L, T, H_v, d, device=DEV)
    ws = torch.empty(ds.gdn_workspace_bytes(ds.gdn_shape([T] * L, H_k, H_v, d, 0)), dtype=torch.uint8, device=DEV)
    ds.gdn_layers_fwd(*packed_like(ds, xs, T, T), T, S, o, p, ws, scale=scale)
    for l, x in enumerate(xs):
        assert rel(o[l], ds.gdn_chunk_fwd(*x, [T], 0, scale=scale)["o"]) <= 5e-5, l


@pytest.mark.parametrize("L,T,pitch,H_k,H_v,d", [(1, 1, 1, 1, 1, 64), (64, 3, 5, 1, 2, 64), (65, 2, 2, 1, 3, 64),
                                                 (2, 131, 132, 16, 32, 128)])
def test_pack_copies_every_row_and_no_other(ds, L, T, pitch, H_k, H_v, d):
    xs = layers(L, T + 1, H_k, H_v, d, seed=1)
    out = packed_like(ds, xs, T, pitch)
    torch.cuda.synchronize()
    for i, t in enumerate(out):
        assert torch.equal(t[:, :T], torch.stack([x[i][:T] for x in xs]))
        assert bool((t[:, T:] == 7).all())


def test_stream_in_layer_groups(ds, monkeypatch):
    """A session whose workspace bound splits its layers over several calls gives the same chunks."""
    from paper_2609_27470_amd import streaming
    L, H_k, H_v, d = 5, 2, 4, 64
    new = lambda: streaming.DeltaSStream(L, H_k, H_v, d, 1, 64, 256, 80, 16, 4, 64, 2, device=DEV)  # noqa: E731
    a = new()
    monkeypatch.setattr(streaming, "LAYERS_WORKSPACE", ds.gdn_workspace_bytes(ds.gdn_shape([80] * 2, H_k, H_v, d, 0)))
    b = new()
    assert a.group == L and b.group == 2
    rows = torch.zeros(1, 80, 64, dtype=torch.int16, device=DEV)
    for c, T in enumerate([80, 33, 64]):
        xs = layers(L, T, H_k, H_v, d, seed=c)
        for s in (a, b):
            s.step(xs, rows, rows)
    assert torch.equal(a.state, b.state) and torch.equal(a.o, b.o) and torch.equal(a.scores[:3], b.scores[:3])


def test_refused_arguments(ds):
    xs = layers(2, 4, 1, 2, 64)
    packed = packed_like(ds, xs, 4, 4)
    S, p = torch.zeros(2, 1, 2, 64, 64, device=DEV), torch.zeros(2, 1, 2, 2, device=DEV)
    o = torch.zeros(2, 4, 2, 64, device=DEV)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    with pytest.raises(ds.DeltasError):
        ds.gdn_layers_fwd(*packed, 5, S, o, p, ws)  # more tokens than the pitch
    with pytest.raises(ds.DeltasError):
        ds.gdn_layers_fwd(*packed, 4, S, o, p, ws[:64])
    with pytest.raises(ValueError):
        ds.gdn_layers_fwd(*packed, 4, S[:1], o, p, ws)
    with pytest.raises(ValueError):
        ds.gdn_pack_layers(xs, 5, packed)
    with pytest.raises(ValueError):
        ds.gdn_pack_layers([x[:2] + (x[2][:, :1],) + x[3:] for x in xs], 4, packed)
    with pytest.raises(ValueError, match="another device"):
        ds.gdn_pack_layers([xs[0], xs[1][:3] + (xs[1][3].cpu(),) + xs[1][4:]], 4, packed)
    with pytest.raises(ValueError, match="same GPU"):
        ds.gdn_layers_fwd(*packed, 4, S, o.cpu(), p, ws)


@pytest.mark.parametrize("form", ["contiguous", "slice", "strided", "host", "misaligned"])
def test_rows_of_every_layout_join_the_contiguous_cache(ds, form):
    """The compacted cache takes a chunk's rows in one launch where it can read them as they are, else by copies."""
    from paper_2609_27470_amd.streaming import DeltaSStream
    KL, row, T = 2, 64, 40
    s = DeltaSStream(2, 1, 2, 64, KL, row, 200, 64, 16, 4, 32, 2, device=DEV, indexed=False)
    want = torch.empty(KL, 0, row, dtype=torch.int16, device=DEV)
    for c in range(4):
        rows = torch.randint(-999, 999, (KL, T, row), dtype=torch.int16, device=DEV)
        want = torch.cat([want, rows], 1)
        if form == "slice":
            rows = torch.cat([rows, rows], 1)[:, :T]
        elif form == "strided":
            rows = rows.transpose(0, 1).contiguous().transpose(0, 1)
        elif form == "host":
            rows = rows.cpu()
        elif form == "misaligned":
            rows = torch.cat([torch.zeros(1, dtype=torch.int16, device=DEV), rows.flatten()])[1:].view(KL, T, row)
        s.step(layers(2, T, 1, 2, 64, seed=c), rows, rows)
    n = 4 * T
    assert s.length == n and torch.equal(s.k[:, :n], want) and torch.equal(s.v[:, :n], want)
    assert s.pos[:n].tolist() == list(range(n)) and s.chunk_id[:n].tolist() == [i // T for i in range(n)]


def test_first_step_allocates_nothing_and_can_be_captured(ds):
    """The buffers of step are there from the start: the first step allocates no device memory, and captured into a graph
    it gives the chunk that the eager session gives."""
    from paper_2609_27470_amd.streaming import DeltaSStream
    L, H_k, H_v, d, T = 5, 2, 4, 64, 50
    new = lambda: DeltaSStream(L, H_k, H_v, d, 1, 64, 256, 80, 16, 4, 64, 2, device=DEV)  # noqa: E731
    a, b, c = new(), new(), new()
    rows, xs = torch.randint(-99, 99, (1, T, 64), dtype=torch.int16, device=DEV), layers(L, T, H_k, H_v, d)
    torch.cuda.synchronize()
    count = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]  # noqa: E731
    before = count()
    a.step(xs, rows, rows)
    assert count() == before
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.step(xs, rows, rows)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(a.state, b.state) and torch.equal(a.o[:, :T], b.o[:, :T]) and torch.equal(a.scores[:1], b.scores[:1])
    assert torch.equal(a.k, b.k) and torch.equal(a.pos, b.pos) and a.length == b.length
    bad = xs[:4] + [xs[4][:1] + (xs[4][1].half(),) + xs[4][2:]]
    with pytest.raises(ValueError):
        c.step(bad, rows, rows)
    assert bool((c.state == 0).all()) and c.n_chunks == 0


def test_workspace_bound_of_a_session(ds):
    """layers_workspace bounds what the layers of one call take together, and the copy of their inputs with it; a later
    group's input is refused before the first group runs."""
    from paper_2609_27470_amd.streaming import DeltaSStream
    L, H_k, H_v, d, T = 5, 2, 4, 64, 50
    new = lambda **kw: DeltaSStream(L, H_k, H_v, d, 1, 64, 256, 80, 16, 4, 64, 2, device=DEV, **kw)  # noqa: E731
    need = lambda n: ds.gdn_workspace_bytes(ds.gdn_shape([80] * n, H_k, H_v, d, 0))  # noqa: E731
    rows, xs = torch.zeros(1, T, 64, dtype=torch.int16, device=DEV), layers(L, T, H_k, H_v, d)
    whole = new()
    whole.step(xs, rows, rows)
    for bound, group in ((need(5), 5), (need(5) - 1, 3), (need(2), 2), (need(1), 1), (0, 1)):
        s = new(layers_workspace=bound)
        assert s.group == group and s.gdn_ws.numel() <= max(bound, need(1))
        assert s._packed is None if group == 1 else s._packed[0].shape[0] == group
        t = new(layers_workspace=bound)
        t.capture_graph()
        for i, buf in enumerate(t.inputs):
            for l in range(L):
                buf[l, :T].copy_(xs[l][i])
        s.step(xs, rows, rows)
        t.step_inputs(T, rows, rows)
        for u in (s, t):
            assert torch.equal(u.state, whole.state) and torch.equal(u.o[:, :T], whole.o[:, :T])
            assert torch.equal(u.scores[:1], whole.scores[:1])
        s2 = new(layers_workspace=bound)
        with pytest.raises(ValueError):
            s2.step(xs[:4] + [xs[4][:3] + (xs[4][3][:, :1].expand(T, H_v),) + xs[4][4:]], rows, rows)
        assert bool((s2.state == 0).all())


@pytest.mark.parametrize("per_slice", [True, False])
@pytest.mark.parametrize("L,T,pitch,H_k,H_v,d,frame_len", [
    (3, 200, 210, 2, 4, 64, 64), (4, 130, 130, 2, 4, 128, 128),        # per-slice kernel
    (16, 300, 333, 2, 4, 128, 64), (20, 64, 100, 2, 4, 128, 64),       # half heads
    (40, 257, 300, 2, 4, 128, 64), (9, 129, 132, 8, 16, 128, 128)])    # whole heads, as a call that may be split
def test_frames_at_a_pitch(ds, L, T, pitch, H_k, H_v, d, frame_len, per_slice):
    """The C entry takes frames of any length: each layer's frames, numbered layer by layer, are those of its own call."""
    import ctypes
    xs = layers(L, T, H_k, H_v, d, seed=7)
    S0 = 0.3 * torch.randn(L, H_v, d, d, device=DEV)
    packed = packed_like(ds, xs, T, pitch)
    F, pairs = -(-T // frame_len), H_v * (d // 16) if per_slice else H_v
    o, S = torch.full((L, pitch, H_v, d), 5.0, device=DEV), torch.empty_like(S0)
    room = L * T // frame_len + L     # frames that so many tokens may hold: those not reached read zero
    p = torch.full((room, pairs, 2), float("nan"), device=DEV)
    shape = ds.GdnShape(L, L * T, H_k, H_v, d, d, frame_len, room, int(per_slice))
    ws = torch.empty(ds.gdn_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    P = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = ds.lib().gdn_layers_fwd(ctypes.byref(shape), pitch, *[P(t) for t in packed], P(S0), P(S), P(o), ds.DS_F32, 1.0, P(p),
                                 P(ws), ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0
    for l, x in enumerate(xs):
        r = ds.gdn_chunk_fwd(*x, [T], frame_len, state_in=S0[l:l + 1].contiguous(), drift_per_slice=per_slice)
        assert rel(o[l, :T], r["o"]) <= 5e-5 and rel(S[l], r["state"][0]) <= 5e-5, l
        assert rel(p[l * F:(l + 1) * F], r["drift_partials"]) <= 1e-4, l
    assert bool((p[L * F:] == 0).all()) and bool((o[:, T:] == 5).all())


@pytest.mark.parametrize("H_k,H_v,d,T", [(1, 2, 64, 40), (2, 4, 128, 130), (2, 4, 128, 90), (32, 64, 128, 70)])
def test_session_of_one_layer(ds, H_k, H_v, d, T):
    """A single layer's inputs are taken as they are: step holds no copy of them and gives step_inputs' bits, also for
    tensors of more rows; what it refuses of several layers it refuses here."""
    from paper_2609_27470_amd.streaming import DeltaSStream
    new = lambda: DeltaSStream(1, H_k, H_v, d, 1, 64, 400, 140, 16, 4, 64, 2, device=DEV)  # noqa: E731
    a, b = new(), new()
    b.capture_graph()
    assert a._packed is None
    rows = torch.randint(-99, 99, (1, T, 64), dtype=torch.int16, device=DEV)
    for c in range(3):
        x = layers(1, T, H_k, H_v, d, seed=c)[0]
        for buf, t in zip(b.inputs, x):
            buf[0, :T].copy_(t)
        longer = tuple(torch.cat([t, t]) for t in x)
        a.step([x[:1] + longer[1:] if c == 1 else x], rows, rows)
        b.step_inputs(T, rows, rows)
        assert torch.equal(a.state, b.state) and torch.equal(a.o[:, :T], b.o[:, :T])
        assert torch.equal(a.scores[:c + 1], b.scores[:c + 1])
    for bad in (x[:2] + (x[2].half(),) + x[3:], x[:3] + (x[3][:, :1].expand(T, H_v),) + x[4:], x[:4] + (x[4].cpu(),), x[:4]):
        with pytest.raises(ValueError):
            a.step([bad], rows, rows)
    assert a.n_chunks == 3 and torch.equal(a.state, b.state)
