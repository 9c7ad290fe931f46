"""The work this framework is timed on: decode attention as a program calls it.

A case is one pass through the Python binding over caches, queries and
selection states that already sit in GPU memory, in one of four forms:

* ``step``   the fused decode step of every layer (``decode_step``);
* ``calls``  the same step as ``plan``, ``decode_attention`` and ``select``;
* ``dense``  ``decode_attention`` over every decoded row (no selection);
* ``image``  one layer's whole image: ``state_reset``, then a ``decode_step``
  for each position from the first to the last.

``launch`` says how the program issues it: ``graph`` replays a HIP graph
captured once (a serving loop), ``eager`` calls the binding each time.
Positions are ragged: evenly spread over the image and dealt to the requests
at random (``idle`` requests are unused slots).  Selection histories are
random ones that the method could have produced, with the kept lists the
previous step would have left.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_19702_amd import binding as B

FP8_MAX = 448.0
MODES = {"dense": B.MODE_DENSE, "diagonal": B.MODE_DIAGONAL, "window": B.MODE_WINDOW}


def _case(name, form, launch, layers, batch, heads, dim, prompt, grid, window, n_att, **more):
    c = {"form": form, "launch": launch, "layers": layers, "batch": batch,
         "q_heads": heads[0], "kv_heads": heads[1], "dim": dim, "prompt": prompt,
         "grid_h": grid[0], "grid_w": grid[1], "window": window, "n_att": n_att,
         "mode": "dense" if form == "dense" else "diagonal", "sinks": 0, "ring": False,
         "kv": "bf16", "outliers": 0.0, "idle": 0}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # One call of the smallest workload (1 request, 8 heads): what a
        # single launch costs a program that calls the binding directly.
        _case("tiny_call", "step", "eager", 1, 1, (8, 8), 64, 32, (16, 16), 64, 13),
        # Two images of LlamaGen-XL-like heads from the first token to the
        # last: every phase of the method, one short launch after another.
        _case("image_b2", "image", "graph", 1, 2, (20, 20), 64, 120, (24, 24), 128, 29),
        # A single Janus-Pro-7B-like image: all 30 layers of one token.
        _case("janus_b1", "step", "graph", 30, 1, (32, 32), 128, 256, (24, 24), 256, 29),
        # The LlamaGen-XL-like serving batch (eight of its layers).
        _case("llamagen_b64", "step", "graph", 8, 64, (20, 20), 64, 120, (24, 24), 128, 29),
        # The Janus-Pro-7B-like serving batch, one layer per call.
        _case("janus_b128", "step", "eager", 1, 128, (32, 32), 128, 256, (24, 24), 256, 29),
        # The same over an fp8 cache.
        _case("janus_b128_fp8", "step", "eager", 1, 128, (32, 32), 128, 256, (24, 24), 256, 29,
              kv="fp8"),
        # The Emu3-8B-like grouped-query batch with outlier keys.
        _case("emu3_b32", "step", "graph", 8, 32, (32, 8), 128, 256, (64, 64), 512, 205,
              outliers=0.01),
        # A large image under the method's default window (half the image).
        _case("default_window_b16", "step", "eager", 1, 16, (32, 32), 128, 256, (96, 96), 4608,
              461),
        # The step as three calls (a program that keeps the plan or changes
        # the logits in between): 8 query heads per KV head, 90% sparsity, a
        # ragged prompt, two unused slots.
        _case("calls_gqa8_b23", "calls", "graph", 4, 23, (32, 4), 128, 77, (64, 64), 2048, 410,
              idle=2),
        # StreamingLLM over a ring cache in fp8, grouped heads, odd grid.
        _case("stream_ring_fp8_b48", "step", "graph", 4, 48, (32, 8), 128, 77, (45, 61), 256, 137,
              mode="window", sinks=4, ring=True, kv="fp8"),
        # The dense baseline on grouped heads (the Emu3-8B-like batch).
        _case("dense_emu3_b32", "dense", "eager", 1, 32, (32, 8), 128, 256, (64, 64), 512, 205,
              outliers=0.01),
        # The dense baseline on the Janus head shape, a larger image: the
        # most bytes of the list.
        _case("dense_48x48_b64", "dense", "eager", 1, 64, (32, 32), 128, 256, (48, 48), 256, 115),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    form = rng.choice(["step", "step", "step", "step", "calls", "dense", "dense", "image"])
    q_heads = rng.choice([8, 16, 20, 32, 32, 64])
    kv_heads = q_heads // rng.choice([g for g in (1, 1, 2, 4, 8) if q_heads % g == 0])
    dim = rng.choice([64, 128])
    prompt = _log_int(rng, 16, 512)
    grid = (_log_int(rng, 12, 96), _log_int(rng, 12, 96))
    if form == "image":
        grid = (rng.randint(12, 24), rng.randint(12, 24))
    length = grid[0] * grid[1]
    window = length // 2 if rng.random() < 0.5 else min(length, _log_int(rng, 64, 1024))
    mode = "dense" if form == "dense" else rng.choice(["diagonal"] * 4 + ["window"])
    sinks = 0 if mode == "dense" else rng.choice([0, 0, 4])
    n_att = max(sinks + 1, int((1 - rng.choice([0.9, 0.95, 0.95, 0.98])) * length + 0.5))
    if mode != "window":
        n_att = min(n_att, window)
    batch = _log_int(rng, 1, 4) if form == "image" else _log_int(rng, 1, 128)
    launch = "graph" if form == "image" else rng.choice(["graph", "eager"])
    c = _case(None, form, launch, 4 if launch == "graph" and form != "image" else 1, batch,
              (q_heads, kv_heads), dim, prompt, grid, window, n_att, mode=mode,
              sinks=sinks, ring=form in ("step", "calls") and rng.random() < 0.2,
              kv=rng.choice(["bf16", "bf16", "fp8"]))
    while c["batch"] > 1 and (work(c)["bytes"] > most or _cache_bytes(c) > 4e9):
        c["batch"] = max(1, c["batch"] * 3 // 4)
    return c


# ---- sizes and positions -------------------------------------------------------

def _length(c):
    return c["grid_h"] * c["grid_w"]


def _elem(c):
    return 1 if c["kv"] == "fp8" else 2


def _ring_rows(c):
    """Decode slots of a ring cache: the least its mode allows."""
    if not c["ring"]:
        return 0
    return c["sinks"] + (c["window"] if c["mode"] == "diagonal" else c["n_att"] - c["sinks"])


def _rows(c):
    return c["prompt"] + (_ring_rows(c) or _length(c))


def _cache_bytes(c):
    return c["layers"] * c["batch"] * c["kv_heads"] * _rows(c) * c["dim"] * 2 * _elem(c)


def _spread(c):
    """Decode positions, evenly over the image (unused slots: -1)."""
    n = c["batch"] - c["idle"]
    return [int((i + 0.5) * _length(c) / n) for i in range(n)] + [-1] * c["idle"]


def _positions(c, seed):
    at = np.random.default_rng([seed, 1]).permutation(c["batch"])
    return [_spread(c)[i] for i in at]


def work(c):
    kv_row = 2 * c["dim"] * _elem(c)
    layers = c["layers"]
    at = _spread(c)
    if c["form"] == "image":  # every position of every request, one layer
        at, layers = [t for t in range(_length(c)) for _ in range(c["batch"])], 1
    cap = min(c["n_att"], _length(c))
    total = flops = 0
    for t in at:
        n = 0 if t < 0 else t + 1 if c["mode"] == "dense" else min(t + 1, cap)
        keys = 0 if t < 0 else c["prompt"] + n
        total += c["kv_heads"] * keys * kv_row + c["q_heads"] * c["dim"] * (2 + 4)
        if c["mode"] != "dense":  # window logits and plan rows out, the kept offsets in
            total += n * (4 * c["q_heads"] + 4 * c["kv_heads"])
            total += 2 * n * c["kv_heads"] if c["mode"] == "diagonal" else 0
        flops += 4 * c["dim"] * keys * c["q_heads"]
    return {"bytes": layers * total, "flops": layers * flops}


def tolerance(c):
    # Outputs and logits are fp32 sums over at most a few thousand keys: 1.7e-7
    # off the 64-bit result with one query head per KV head, 1.8e-6 with
    # several (weights as two bf16 terms); 1e-5 is about four times what two
    # such results differ by.  Whole values (plans, skip lists) may differ
    # where two scores nearly tie.
    return {"rel": 1e-5, "max": 2e-4, "differ": 1e-3}


# ---- selection histories ---------------------------------------------------------

def _capacity(c):
    return c["window"] - (c["n_att"] - c["sinks"]) if c["mode"] == "diagonal" else 0


def _history(c, seed):
    """Skip entries of every (request, head) before its position, in order,
    and the window offsets then kept, largest first: the k-th selection takes
    one of the n kept offsets, and offset n + k enters the window."""
    n, cap, pairs = c["n_att"] - c["sinks"], _capacity(c), c["batch"] * c["kv_heads"]
    rng = np.random.default_rng([seed, 2])
    have = np.repeat([min(max(t - (c["n_att"] - 1), 0), cap) for t in _positions(c, seed)],
                     c["kv_heads"])
    skipped = np.zeros((pairs, cap), np.uint16)
    kept = np.tile(np.arange(n, dtype=np.int32), (pairs, 1))
    for k in range(int(have.max()) if cap else 0):
        on = np.nonzero(have > k)[0]
        j = rng.integers(0, n, len(on))
        skipped[on, k] = kept[on, j]
        kept[on, j] = n + k
    return have, skipped, -np.sort(-kept, axis=1)


def _offsets_kept(c, t, kept):
    """Kept offsets ``t - j`` after the sinks at position ``t``, oldest first
    (``kept``: the list after the skip entries stored so far)."""
    last = t - c["sinks"]  # the oldest offset decoded so far
    if c["mode"] == "window":
        return np.tile(np.arange(min(last, c["n_att"] - c["sinks"] - 1), -1, -1), (len(kept), 1))
    if t < c["n_att"] or _capacity(c) == 0:
        return np.tile(np.arange(min(last, c["window"] - 1), -1, -1), (len(kept), 1))
    return kept


# ---- inputs ----------------------------------------------------------------------

def _gen(seed, *what):
    s = seed
    for w in what:
        s = s * 1000003 + w
    return torch.Generator(device="cuda").manual_seed(s % (1 << 62))


def _tensors(c, seed, layer, steps=None):
    """K, V (with fp8 scales or None) and queries of one layer."""
    shape = (c["batch"], c["kv_heads"], _rows(c), c["dim"])
    kv, scales = [], []
    for i in (0, 1):
        g = _gen(seed, layer, i)
        x = torch.randn(shape, generator=g, device="cuda",
                        dtype=torch.float32 if c["kv"] == "fp8" else torch.bfloat16)
        if i == 0 and c["outliers"]:
            big = torch.rand(shape[:3], generator=g, device="cuda") < c["outliers"]
            x *= torch.where(big, 8.0, 1.0).unsqueeze(-1).to(x.dtype)
        if c["kv"] == "fp8":
            s = x.abs().amax(dim=(2, 3)) / FP8_MAX
            x = (x / s[:, :, None, None]).clamp(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn)
            scales.append(s.reshape(-1).contiguous())
        kv.append(x)
    many = () if steps is None else (steps,)
    q = torch.randn(many + (c["batch"], c["q_heads"], c["dim"]), generator=_gen(seed, layer, 2),
                    device="cuda", dtype=torch.bfloat16)
    return kv[0], kv[1], (scales or [None, None]), q


class _State:
    pass


def prepare(case, seed):
    c, st = case, _State()
    dense = c["mode"] == "dense"
    p = B.make_params(c["prompt"], c["grid_h"], c["grid_w"], c["window"], c["n_att"],
                      MODES[c["mode"]], c["sinks"])
    s = B.make_shape(c["batch"], c["q_heads"], c["kv_heads"], c["dim"])
    pairs, layers = c["batch"] * c["kv_heads"], c["layers"]
    image = c["form"] == "image"
    steps = _length(c) if image else None
    zeros = lambda *n, dtype=torch.float32: torch.zeros(n, dtype=dtype, device="cuda")  # noqa: E731
    st.case, st.p, st.s, st.scale = c, p, s, 1 / math.sqrt(c["dim"])
    lead = steps if image else layers
    st.out = zeros(lead, c["batch"], c["q_heads"], c["dim"])
    st.result = {"out": st.out}
    st.ws = zeros(max(B.workspace_bytes(p, s), 1), dtype=torch.uint8)
    st.plan = st.logits = st.states = None
    if not dense:
        st.plan = zeros(layers, B.plan_bytes(p, s), dtype=torch.uint8)
        st.logits = zeros(lead, B.window_logits_count(p, s))
        st.states = zeros(layers, B.state_bytes(p, s), dtype=torch.uint8)
        pl, sl = B.plan_layout(p, s), B.state_layout(p, s)

        def words(buf, off, n, dtype):
            return buf[:, off:off + n * torch.empty((), dtype=dtype).element_size()].view(dtype)

        st.result.update(
            logits=st.logits, plan_count=words(st.plan, pl.count_offset, pairs, torch.int32),
            plan_rows=words(st.plan, pl.indices_offset, pairs * pl.cap, torch.int32))
        if sl.cap:
            count = words(st.states, sl.count_offset, pairs, torch.int32)
            skipped = words(st.states, sl.offsets_offset, pairs * sl.cap, torch.int16)
            st.result.update(state_count=count, state_skipped=skipped)
            if not image:
                have, skip, kept = _history(c, seed)
                count[:] = torch.from_numpy(have.astype(np.int32)).cuda()
                skipped[:] = torch.from_numpy(skip.view(np.int16).reshape(-1)).cuda()
                # the kept lists, where the previous step's selection left them
                tags = np.zeros((pairs, 2), np.int32)
                lists = np.zeros((pairs, 2, sl.kept_stride), np.uint16)
                tags[np.arange(pairs), have % 2] = np.where(have > 0, have + 1, 0)
                lists[np.arange(pairs), have % 2, :sl.kept_cap] = kept
                words(st.states, sl.kept_count_offset, 2 * pairs, torch.int32)[:] = \
                    torch.from_numpy(tags.reshape(-1)).cuda()
                words(st.states, sl.kept_offset, lists.size, torch.int16)[:] = \
                    torch.from_numpy(lists.view(np.int16).reshape(-1)).cuda()
    if image:
        st.pos = [torch.full((c["batch"],), t, dtype=torch.int32, device="cuda")
                  for t in range(steps)]
    else:
        st.pos = torch.tensor(_positions(c, seed), dtype=torch.int32, device="cuda")
    st.layers = []
    for i in range(layers):
        k, v, (ks, vs), q = _tensors(c, seed, i, steps)
        st.layers.append((k, v, q, B.kv_layout(k, ring_rows=_ring_rows(c), k_scale=ks, v_scale=vs),
                          ks, vs))
    st.graph = None
    if c["launch"] == "graph":
        before = None if st.states is None else st.states.clone()
        _issue(st)  # loads the kernels
        if before is not None:
            st.states.copy_(before)
        torch.cuda.synchronize()
        st.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st.graph):
            _issue(st)
    return st


def _issue(st):
    form, p, s = st.case["form"], st.p, st.s
    if form == "image":
        k, v, q, lay = st.layers[0][:4]
        B.state_reset(p, s, st.states[0])
        for t, pos in enumerate(st.pos):
            B.decode_step(p, s, q[t], k, v, lay, pos, st.states[0], st.plan[0], st.scale,
                          st.out[t], st.logits[t], st.ws)
        return
    for i, layer in enumerate(st.layers):
        k, v, q, lay = layer[:4]
        if form == "dense":
            B.decode_attention(p, s, q, k, v, lay, st.pos, None, st.scale, st.out[i], None, st.ws)
        elif form == "step":
            B.decode_step(p, s, q, k, v, lay, st.pos, st.states[i], st.plan[i], st.scale,
                          st.out[i], st.logits[i], st.ws)
        else:
            B.plan(p, s, st.pos, st.states[i], st.plan[i])
            B.decode_attention(p, s, q, k, v, lay, st.pos, st.plan[i], st.scale, st.out[i],
                               st.logits[i], st.ws)
            B.select(p, s, st.pos, st.plan[i], st.logits[i], st.states[i])


def run(state):
    if state.graph is not None:
        state.graph.replay()
    else:
        _issue(state)
    return state.result


# ---- the same in 64 bits -----------------------------------------------------------

def _cache_rows(c, pos):
    """Cache rows of decode positions (a linear cache, or a ring after the sinks)."""
    r = _ring_rows(c)
    if r and r < _length(c):
        pos = np.where(pos < c["sinks"], pos,
                       c["sinks"] + (pos - c["sinks"]) % (r - c["sinks"]))
    return c["prompt"] + pos


def _attend(c, q, k, v, ks, vs, rows):
    """Outputs ``[Hkv, G, d]`` and logits ``[Hkv, G, rows]`` of one request;
    ``rows``: the cache rows each KV head attends."""
    head = torch.arange(c["kv_heads"], device="cuda")[:, None]
    kk = k[head, rows].float().double()
    vv = v[head, rows].float().double()
    if ks is not None:
        kk *= ks.double()[:, None, None]
        vv *= vs.double()[:, None, None]
    outs, logits = [], []
    for x in q.view(c["kv_heads"], -1, c["dim"]).double().unbind(1):
        z = (kk * x[:, None, :]).sum(-1) / math.sqrt(c["dim"])
        outs.append((torch.softmax(z, -1)[:, :, None] * vv).sum(1))
        logits.append(z)
    return torch.stack(outs, 1), torch.stack(logits, 1)


def exact(case, seed):
    c = case
    lp, heads = c["prompt"], c["kv_heads"]
    prompt = np.tile(np.arange(lp), (heads, 1))
    cap = min(c["n_att"], _length(c))
    image = c["form"] == "image"
    at = None if image else _positions(c, seed)
    lead = _length(c) if image else c["layers"]
    out = torch.zeros((lead, c["batch"], c["q_heads"], c["dim"]), dtype=torch.float64,
                      device="cuda")
    logits = torch.zeros((lead, c["batch"], c["q_heads"], cap), dtype=torch.float64, device="cuda")

    def one(i, b, t, kept, layer):
        """Request ``b`` at position ``t`` of output ``i``; returns its kept
        offsets and the window logits after the sinks."""
        k, v, ks, vs, q = layer
        sinks = np.tile(np.arange(min(c["sinks"], t + 1)), (heads, 1))
        if c["mode"] == "dense":
            offs, pos = None, np.tile(np.arange(t + 1), (heads, 1))
        else:
            offs = _offsets_kept(c, t, kept)
            pos = np.concatenate([sinks, t - offs], 1)
        rows = torch.from_numpy(np.concatenate([prompt, _cache_rows(c, pos)], 1)).cuda()
        o, z = _attend(c, q, k[b], v[b], ks, vs, rows)
        out[i, b] = o.reshape(-1, c["dim"])
        z = z[:, :, lp:]
        if c["mode"] != "dense":
            logits[i, b, :, :z.shape[-1]] = z.reshape(-1, z.shape[-1])
        return offs, z[:, :, sinks.shape[1]:]

    def layer_of(i, b, x):
        k, v, (ks, vs), q = x
        span = slice(b * heads, (b + 1) * heads)
        return (k, v, None if ks is None else ks[span], None if vs is None else vs[span],
                q[i][b] if image else q[b])

    if image:
        x = _tensors(c, seed, 0, lead)
        n = c["n_att"] - c["sinks"]
        for b in range(c["batch"]):
            kept = np.tile(np.arange(n - 1, -1, -1), (heads, 1))
            for t in range(lead):
                offs, z = one(t, b, t, kept, layer_of(t, b, x))
                k = t - (c["n_att"] - 1)
                if 0 <= k < _capacity(c):  # the least attended kept key leaves
                    score = torch.softmax(z, -1).sum(1) if z.shape[1] > 1 else z[:, 0]
                    drop = score.argmin(-1).cpu().numpy()
                    stay = np.arange(n)[None, :] != drop[:, None]
                    kept = np.concatenate([np.full((heads, 1), n + k),
                                           offs[stay].reshape(heads, n - 1)], 1)
    else:
        _, _, kept = _history(c, seed) if c["mode"] == "diagonal" else (
            None, None, np.zeros((c["batch"] * heads, 0), np.int32))
        for i in range(c["layers"]):
            x = _tensors(c, seed, i)
            for b, t in enumerate(at):
                if t >= 0:
                    one(i, b, t, kept[b * heads:(b + 1) * heads], layer_of(i, b, x))
    got = {"out": out}
    if c["mode"] != "dense":
        got.update(logits=logits.reshape(lead, -1), plan_count=None, plan_rows=None)
        if _capacity(c):
            got.update(state_count=None, state_skipped=None)
    return got
