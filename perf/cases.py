"""The work a user has this framework do, as cases that can be timed and compared.

Four kinds, each through the package's public entry points:

* ``forward``  gdn_chunk_fwd over packed streams with its drift sums, and
  deltas_drift over the frames: prefill of whole videos, one frame of a layer
  stack with the state carried, batches of streams; head dims 64 and 128, bf16
  and fp32 outputs, per-head and per-slice drift pairs, the write signal and
  the snapshots;
* ``decode``   gdn_decode_step: one token for every stream of a batch;
* ``evict``    kv_evict_topk: one eviction of a contiguous K/V cache, its
  tables put back first (the rows hold whatever the last pass left);
* ``stream``   DeltaSStream.step_inputs: one chunk of a streamed video through
  every layer, the score, the append and the eviction.

Shapes are those of the repository's workloads (H_k = 16, H_v = 32, d = 128, 24
layers; 8 K/V layers; budgets of 8192 and 16384 tokens; chunks of 118 - 132
tokens; frames of 1024) and their surroundings.
"""
from __future__ import annotations

import torch

import paper_2609_27470_amd as ds
from paper_2609_27470_amd.streaming import DeltaSStream, Snapshot

DEV = "cuda"
MAX_CHUNKS = 1 << 18  # chunk scores a session can hold: more than any run of passes consumes


def _forward(name, lens, **kw):
    case = dict(name=name, kind="forward", lens=" ".join(str(n) for n in lens), H_k=16, H_v=32, d=128, frame_len=1024,
                bf16=True, state=False, per_slice=False, write=False, snapshots=False, memory=False)
    case.update(kw)
    return case


def listed():
    return [
        # answering a question on one GPU's few live streams, and a full serving batch
        dict(name="decode_8", kind="decode", B=8, H_k=16, H_v=32, d=128, bf16=True),
        dict(name="decode_256", kind="decode", B=256, H_k=16, H_v=32, d=128, bf16=True),
        # the smallest forward: the tiny workload (latency)
        _forward("tiny_d64", [1024], H_k=2, H_v=2, d=64, frame_len=256, bf16=False),
        # one frame through one layer of the stack, the state carried in place
        _forward("frame_1024", [1024], state=True, per_slice=True),
        # one layer over a whole video: the headline's layer
        _forward("layer_32768", [32768]),
        # both retention signals and the states at the frame ends, an odd length, fp32 outputs, slow decay
        _forward("signals_4999", [4999], H_k=8, H_v=16, bf16=False, write=True, snapshots=True, memory=True),
        # a few streams prefilled together, odd lengths
        _forward("batch_4", [6151, 4097, 8190, 5333], state=True),
        # the packed varlen batch
        _forward("varlen_8", [77817, 66883, 110520, 51901, 110997, 91056, 16761, 58358]),
        # whole-frame eviction of the 16384-token cache (eviction loop), and the paper's policy on the 8192-token one
        dict(name="evict_frames", kind="evict", M=16384, length=17408, chunk=1024, layers=8, row=2048, n_sink=0, n_window=0,
             n_buckets=1),
        dict(name="evict_policy", kind="evict", M=8192, length=8317, chunk=125, layers=8, row=1024, n_sink=4, n_window=1024,
             n_buckets=4),
        # a streamed chunk: the default slot-indexed cache, and the cache whose rows are compacted
        dict(name="stream_indexed", kind="stream", T=125, M=16384, layers=24, H_k=16, H_v=32, d=128, kv_layers=8, row=2048,
             indexed=True),
        dict(name="stream_rows", kind="stream", T=131, M=8192, layers=24, H_k=16, H_v=32, d=128, kv_layers=8, row=2048,
             indexed=False),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "decode", "evict", "stream"])
    if kind == "decode":
        H_k = rng.choice([4, 8, 16])
        return dict(kind=kind, B=_log(rng, 1, 256), H_k=H_k, H_v=H_k * rng.choice([1, 2, 4]), d=rng.choice([64, 128]),
                    bf16=rng.random() < 0.7)
    if kind == "evict":
        M = _log(rng, 1024, 16384)
        chunk = rng.choice([rng.randint(60, 140), rng.randint(250, 1024)])
        n_sink, n_window, n_buckets = rng.choice([(0, 0, 1), (4, M // 8, 4), (16, M // 4, rng.randint(1, 16))])
        return dict(kind=kind, M=M, length=M + rng.choice([chunk, 2 * chunk, M]), chunk=chunk, layers=rng.choice([2, 4, 8]),
                    row=rng.choice([512, 1024, 2048]), n_sink=n_sink, n_window=n_window, n_buckets=n_buckets)
    if kind == "stream":
        H_k = rng.choice([8, 16])
        return dict(kind=kind, T=rng.randint(20, 132), M=_log(rng, 2048, 16384), layers=rng.choice([12, 18, 24]), H_k=H_k,
                    H_v=2 * H_k, d=128, kv_layers=rng.choice([4, 8]), row=rng.choice([1024, 2048]),
                    indexed=rng.random() < 0.7)
    B = rng.choice([1, 1, 1, 2, 3, 4, 6, 8, 12, 16])
    top = max(64, 131072 // B)
    lens = [_log(rng, 64, top) for _ in range(B)] if rng.random() < 0.5 else [_log(rng, 64, top)] * B
    d = rng.choice([64, 128, 128, 128])
    H_k = rng.choice([2, 4, 8, 16, 16])
    H_v = H_k * rng.choice([1, 2, 2, 4]) if H_k < 16 else rng.choice([16, 32, 32])
    case = _forward("", lens, H_k=H_k, H_v=H_v, d=d, frame_len=64 * _log(rng, 1, 32), bf16=rng.random() < 0.7,
                    state=rng.random() < 0.5, per_slice=rng.random() < 0.5, write=rng.random() < 0.2,
                    memory=rng.random() < 0.3)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(0x5EED + seed)
    return g


def _unit(x):
    return (x / x.norm(dim=-1, keepdim=True)).to(torch.bfloat16)


def _tokens(gen, T, H_k, H_v, d, memory=False):
    """q, k (unit rows, keys of a head from a 32-dim subspace as a scene's tokens are), v, log decay g and write
    strength beta of T tokens; memory: heads that decay slowly."""
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=gen)  # noqa: E731
    q, k, v = (torch.empty(T, h, d, dtype=torch.bfloat16, device=DEV) for h in (H_k, H_k, H_v))
    basis = rnd(H_k, 32, d)
    for a in range(0, T, 16384):  # in pieces: the fp32 draws of a long stream would outgrow the tensors themselves
        n = min(16384, T - a)
        q[a:a + n] = _unit(rnd(n, H_k, d))
        k[a:a + n] = _unit(torch.matmul(rnd(H_k, n, 32), basis).transpose(0, 1))
        v[a:a + n] = rnd(n, H_v, d).to(torch.bfloat16)
    x = rnd(T, H_v)
    if memory:
        x = 0.1 * x + torch.linspace(-10.0, -2.0, H_v, device=DEV)
    return q, k, v, -torch.nn.functional.softplus(x), torch.sigmoid(rnd(T, H_v))


def _lens(case):
    return [int(n) for n in case["lens"].split()]


def _forward_inputs(case, seed):
    gen = _gen(seed)
    lens, H_v, d = _lens(case), case["H_v"], case["d"]
    x = _tokens(gen, sum(lens), case["H_k"], H_v, d, case["memory"])
    S = 0.3 * torch.randn(len(lens), H_v, d, d, device=DEV, generator=gen) if case["state"] else None
    return x, S


def _decode_inputs(case, seed):
    gen = _gen(seed)
    B, H_v, d = case["B"], case["H_v"], case["d"]
    return _tokens(gen, B, case["H_k"], H_v, d), 0.3 * torch.randn(B, H_v, d, d, device=DEV, generator=gen)


def _stream_inputs(case, seed):
    """The layers' inputs of one chunk, the layers' states and the scores of the chunks seen so far."""
    gen = _gen(seed)
    L, T, H_v, d = case["layers"], case["T"], case["H_v"], case["d"]
    x = _tokens(gen, L * T, case["H_k"], H_v, d)
    S = 0.3 * torch.randn(L, 1, H_v, d, d, device=DEV, generator=gen)
    seen = case["M"] // 100 + 2
    return [t.view(L, T, *t.shape[1:]) for t in x], S, torch.rand(seen, device=DEV, generator=gen) + 0.5, gen


def _table(n, chunk):
    """Positions and chunk ids of n cached tokens, some older ones already evicted."""
    i = torch.arange(n, dtype=torch.int32, device=DEV)
    return i + (i // chunk) * 3, i // chunk


def _planes(gen, layers, rows, row):
    return torch.randint(-2 ** 15, 2 ** 15, (layers, rows, row), dtype=torch.int16, device=DEV, generator=gen)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "decode":
        x, S = _decode_inputs(case, seed)
        o = torch.empty(case["B"], case["H_v"], case["d"], dtype=torch.bfloat16 if case["bf16"] else torch.float32, device=DEV)
        return dict(case=case, x=x, S=S, o=o, out=torch.empty_like(S))
    if kind == "forward":
        x, S = _forward_inputs(case, seed)
        lens, H_v, d, T = _lens(case), case["H_v"], case["d"], x[0].shape[0]
        shape = ds.gdn_shape(lens, case["H_k"], H_v, d, case["frame_len"], case["per_slice"])
        F, pairs = shape.n_frames, H_v * (d // 16) if case["per_slice"] else H_v
        cu = torch.tensor([0] + lens, dtype=torch.int32, device=DEV).cumsum(0).to(torch.int32) if len(lens) > 1 else None
        new = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV)  # noqa: E731
        return dict(case=case, x=x, S=S, lens=lens, cu=cu, out=new(len(lens), H_v, d, d),
                    o=torch.empty(T, H_v, d, dtype=torch.bfloat16 if case["bf16"] else torch.float32, device=DEV),
                    drift=new(F, pairs, 2), write=new(F, H_v, 2) if case["write"] else False,
                    snaps=new(F, H_v, d, d) if case["snapshots"] else False, scores=new(F),
                    ws=torch.empty(max(1, ds.gdn_workspace_bytes(shape, case["write"])), dtype=torch.uint8, device=DEV))
    if kind == "evict":
        gen = _gen(seed)
        n, layers, row = case["length"], case["layers"], case["row"]
        pos0, chunk0 = _table(n, case["chunk"])
        return dict(case=case, k=_planes(gen, layers, n, row), v=_planes(gen, layers, n, row), pos0=pos0, chunk0=chunk0,
                    pos=pos0.clone(), chunk=chunk0.clone(), keep=torch.empty(case["M"], dtype=torch.int32, device=DEV),
                    scores=torch.rand(int(chunk0[-1]) + 1, device=DEV, generator=gen) + 0.5,
                    ws=torch.empty(ds.kv_workspace_bytes(layers, 2 * row, n), dtype=torch.uint8, device=DEV))
    # stream: a session in the middle of a video, put back from a saved memory with a full cache
    x, S, scores, gen = _stream_inputs(case, seed)
    T, M, KL, row = case["T"], case["M"], case["kv_layers"], case["row"]
    s = DeltaSStream(case["layers"], case["H_k"], case["H_v"], case["d"], KL, row, M, 132, MAX_CHUNKS,
                     n_window=min(1024, M // 4), device=DEV, indexed=case["indexed"])
    pos, chunk = _table(M, 100)
    rows = s.capacity if case["indexed"] else M
    k, v = _planes(gen, KL, rows, row), _planes(gen, KL, rows, row)
    perm = torch.randperm(s.capacity, device=DEV, generator=gen).to(torch.int32)
    s.restore(Snapshot(S, k, v, pos, chunk, scores, perm[:M] if case["indexed"] else None,
                       perm[M:] if case["indexed"] else None, M, scores.numel(), int(pos[-1]) + 1))
    s.capture_graph()
    for buf, t in zip(s.inputs, x):
        buf[:, :T].copy_(t)
    return dict(case=case, s=s, k=_planes(gen, KL, T, row), v=_planes(gen, KL, T, row))


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "decode":
        q, k, v, g, b = st["x"]
        r = ds.gdn_decode_step(q, k, v, g, b, state_in=st["S"], state_out=st["out"], o=st["o"])
        return {"o": r["o"], "state": r["state"]}
    if kind == "forward":
        q, k, v, g, b = st["x"]
        r = ds.gdn_chunk_fwd(q, k, v, g, b, st["lens"], case["frame_len"], cu_seqlens=st["cu"], state_in=st["S"],
                             state_out=st["out"], o=st["o"], drift_partials=st["drift"], write_partials=st["write"],
                             snapshots=st["snaps"], workspace=st["ws"], drift_per_slice=case["per_slice"])
        ds.deltas_drift(st["drift"][None], ds.LAYER_FROB, scores=st["scores"])
        out = {"o": r["o"], "state": r["state"], "drift": st["drift"], "scores": st["scores"]}
        if case["write"]:
            out["write"] = st["write"]
        if case["snapshots"]:
            out["snapshots"] = st["snaps"]
        return out
    if kind == "evict":
        st["pos"].copy_(st["pos0"])
        st["chunk"].copy_(st["chunk0"])
        M = case["M"]
        ds.kv_evict_topk(list(st["k"]), list(st["v"]), st["pos"], st["chunk"], st["scores"], case["length"], M, case["n_sink"],
                         case["n_window"], case["n_buckets"], keep_out=st["keep"], workspace=st["ws"])
        return {"k": st["k"][:, :M], "v": st["v"][:, :M], "pos": st["pos"][:M], "chunk": st["chunk"][:M], "keep": st["keep"]}
    s = st["s"]
    n = s.step_inputs(case["T"], st["k"], st["v"])
    out = {"state": s.state, "o": s.o[:, :case["T"]], "score": s.scores[s.n_chunks - 1:s.n_chunks], "pos": s.pos[:n],
           "chunk": s.chunk_id[:n]}
    if case["indexed"]:  # which row of the cache a token lies in is the session's own choice
        out.update(slot=s.slot[:n], k=s.k, v=s.v)
    else:
        out.update(k=s.k[:, :n], v=s.v[:, :n])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _forward_work(T, H_k, H_v, d, states, o_bytes):
    """Tokens in and out, states in and out; dense 64-token tiles with the Gram products shared per qk-head."""
    return (T * (4 * H_k * d + 2 * H_v * d + o_bytes * H_v * d + 8 * H_v) + states * H_v * d * d * 4,
            T * (H_k * 4 * 64 * d + H_v * (4 * 64 * d + 6 * d * d + 2 * 64 * 64 // 3)))


def work(case):
    kind = case["kind"]
    if kind == "decode":
        B, H_k, H_v, d, ob = case["B"], case["H_k"], case["H_v"], case["d"], 2 if case["bf16"] else 4
        return {"bytes": B * (8 * H_v * d * d + 4 * H_k * d + (2 + ob) * H_v * d + 8 * H_v), "flops": B * H_v * 7 * d * d}
    if kind == "forward":
        lens, H_v, d = _lens(case), case["H_v"], case["d"]
        F = sum(ds.frames_of_length(n, case["frame_len"]) for n in lens)
        b, f = _forward_work(sum(lens), case["H_k"], H_v, d, len(lens) * (2 if case["state"] else 1), 2 if case["bf16"] else 4)
        b += F * H_v * 8 * (d // 16 if case["per_slice"] else 1) + (F * H_v * 8 if case["write"] else 0)
        return {"bytes": b + (F * H_v * d * d * 4 if case["snapshots"] else 0), "flops": f}
    if kind == "evict":
        # every row kept from behind the first evicted token moves (a chunk somewhere in the middle half, on average)
        return {"bytes": 2 * case["M"] // 2 * 2 * case["layers"] * 2 * case["row"] + 16 * case["length"], "flops": 0}
    T, KL, row, M = case["T"], case["kv_layers"], case["row"], case["M"]
    b, f = _forward_work(T, case["H_k"], case["H_v"], case["d"], 2, 2)
    b, f = case["layers"] * b, case["layers"] * f
    b += 2 * T * 2 * KL * 2 * row + 24 * M + (0 if case["indexed"] else M * 2 * KL * 2 * row)
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "evict":
        return "exact"
    if case["kind"] == "decode":
        return {"rel": 2e-3 if case["bf16"] else 1e-5}  # fp32 sums; one rounding to bf16
    # k, the state and the writes meet the matrix cores in fp16: 3.6e-4 off 64 bits, and a bf16 output's own rounding
    return {"rel": 4e-3 if case.get("bf16", True) else 1.5e-3}


# ---------------------------------------------------------------------------
# the recurrence in 64 bits, token by token
# ---------------------------------------------------------------------------
def _recurrence(q, k, v, g, beta, S, frame_len):
    """[N] independent layers or streams of T tokens: q, k [N][T][H_k][d], S [N][H_v][d][d]; returns o, S, and per frame the
    drift sums of every 16-row slice, the write sums and the state."""
    N, T, H_v, d = v.shape
    rep = H_v // q.shape[2]
    a = g.double().exp()
    b = beta.double()
    S = S.double().clone()
    o = torch.empty(N, T, H_v, d, dtype=torch.float64, device=DEV)
    S0, wsum, pairs, writes, snaps = S.clone(), torch.zeros(N, H_v, dtype=torch.float64, device=DEV), [], [], []
    begin = 0
    for t in range(T):
        kt = k[:, t].double().repeat_interleave(rep, 1)
        qt = q[:, t].double().repeat_interleave(rep, 1)
        S.mul_(a[:, t, :, None, None])
        e = b[:, t, :, None] * (v[:, t].double() - torch.matmul(S, kt[..., None])[..., 0])
        S.addcmul_(e[..., None], kt[:, :, None])
        o[:, t] = torch.matmul(S, qt[..., None])[..., 0]
        wsum += e.norm(dim=-1)
        if t + 1 == T or (frame_len > 0 and (t + 1) % frame_len == 0):
            sl = lambda x: x.square().view(N, H_v, d // 16, 16, d).sum((-1, -2))  # noqa: E731
            pairs.append(torch.stack([sl(S - S0), sl(S0)], -1))
            writes.append(torch.stack([wsum, torch.full_like(wsum, t + 1 - begin)], -1))
            snaps.append(S.clone())
            S0, wsum, begin = S.clone(), torch.zeros_like(wsum), t + 1
    return o, S, torch.stack(pairs, 1), torch.stack(writes, 1), torch.stack(snaps, 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "evict":
        return None
    if kind == "decode":
        (q, k, v, g, b), S = _decode_inputs(case, seed)
        o, S, _, _, _ = _recurrence(q[:, None], k[:, None], v[:, None], g[:, None], b[:, None], S, 0)
        return {"o": o[:, 0], "state": S}
    if kind == "stream":
        (q, k, v, g, b), S, scores, _ = _stream_inputs(case, seed)
        o, S, pairs, _, _ = _recurrence(q, k, v, g, b, S[:, 0], 0)
        p = pairs.sum((1, 2, 3))  # Eq. 3 pools a layer's heads; one frame
        score = (p[:, 0] / p[:, 1]).sqrt().mean()[None]
        out = {"state": S[:, None], "o": o, "score": score, "pos": None, "chunk": None, "k": None, "v": None}
        return {**out, "slot": None} if case["indexed"] else out
    lens = _lens(case)
    if sum(lens) > 70000:
        return None
    (q, k, v, g, b), S = _forward_inputs(case, seed)
    parts, t0 = [], 0
    for i, n in enumerate(lens):
        sl = slice(t0, t0 + n)
        s0 = S[i:i + 1] if S is not None else torch.zeros(1, case["H_v"], case["d"], case["d"], device=DEV)
        parts.append(_recurrence(*(x[None, sl] for x in (q, k, v, g, b)), s0, case["frame_len"]))
        t0 += n
    o, S1, pairs, writes, snaps = (torch.cat([p[j] for p in parts], 0 if j == 1 else 1) for j in range(5))
    pairs = pairs[0]
    tot = pairs.sum((1, 2))
    score = torch.where(tot[:, 1] > 0, (tot[:, 0] / tot[:, 1]).sqrt(), torch.full_like(tot[:, 0], float("inf")))
    out = {"o": o[0], "state": S1, "drift": pairs.flatten(1, 2) if case["per_slice"] else pairs.sum(2), "scores": score}
    if case["write"]:
        out["write"] = writes[0]
    if case["snapshots"]:
        out["snapshots"] = snaps[0]
    return out
