"""The work that is measured: calls of the library as a decoder makes them, each through a public
entry point, over the range of sizes that the library is used at.

A case is one attention layer of a model at one point of its decoding (a step, a block of steps, a
prompt) or one discounted sum; only the ragged case runs several layers, because its work list is
built once for all of them.  Inputs are N(0, 1) from the seed, as in the library's own workloads.
"""
import math
import random

import torch

from paper_2501_05408_amd import tempo as T
from paper_2501_05408_amd.store import BlockStore

DEVICE = "cuda:0"
THETA = 500000.0
DTYPES = {"bf16": (T.TEMPO_BF16, torch.bfloat16), "f32": (T.TEMPO_F32, torch.float32)}

# Attention-layer shapes: (query heads, kv heads, head_dim).  The first is the Llama-3.2-3B layer.
LLAMA = (24, 8, 128)
NARROW = (32, 8, 64)
TINY = (8, 2, 64)


def _case(name, kind, shape, dtype="bf16", **more):
    c = {"kind": kind, "dtype": dtype, "q_heads": shape[0], "kv_heads": shape[1], "head_dim": shape[2],
         "block": 256, "batch": 1, "t": 0, "count": 1, "window": 0, "ring": False, "rope": False, "layers": 1}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # One user, early in the answer: the smallest call, rotary producer fused in.
        _case("step_one", "step", LLAMA, t=299, rope=True),
        # The layer of a batch of 16 at the end of a 4096-token context.
        _case("step_causal", "step", LLAMA, batch=16, t=4095),
        # One sequence with a very long context.
        _case("step_long", "step", LLAMA, t=65535),
        # Sliding-window decoding in constant memory, far into the sequence.
        _case("step_window", "step", LLAMA, batch=16, t=16383, window=512, ring=True),
        # A serving batch: every sequence at its own length, shared pool, random block table, one
        # work list for all layers of the step.
        _case("step_ragged", "ragged", LLAMA, batch=64, t=8191, layers=4),
        # The tight-tolerance data type at a size people verify a model with.
        _case("step_f32", "step", LLAMA, "f32", batch=16, t=2047),
        # Chunked prompts and speculative decoding: a block of steps in front of a long history.
        _case("block", "block", LLAMA, batch=16, t=4075, count=21),
        # One user's prompt of an odd, ordinary length; narrow heads.
        _case("prompt_one", "prompt", NARROW, count=499),
        # A batch of long prompts.
        _case("prompt_batch", "prompt", LLAMA, batch=16, count=4096),
        # Prompts of a sliding-window model, written into its ring store.
        _case("prompt_window", "prompt", LLAMA, batch=4, count=2048, window=512, ring=True),
        # The small fp32 layer, its 512 steps answered as one prompt.
        _case("prompt_f32", "prompt", TINY, "f32", block=64, count=512),
        # The returns of a batch of episodes: the whole future, discounted.
        {"name": "returns", "kind": "returns", "batch": 64, "T": 1000, "n": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 4 + ["window", "ragged", "step_f32", "block", "block"] + ["prompt"] * 3 +
                      ["prompt_window", "prompt_f32", "returns"])
    shape = rng.choice([LLAMA, LLAMA, NARROW, (32, 4, 128), (16, 16, 64)])
    block = rng.choice([32, 64, 256])
    if kind == "step":
        batch = _log(rng, 1, 64)
        t = _log(rng, 16, min(65536, 65536 * 4 // batch)) - 1
        return _case("", "step", shape, block=block, batch=batch, t=t, rope=rng.random() < 0.4)
    if kind == "window":
        window = _log(rng, 64, 4096)
        return _case("", "step", shape, block=block, batch=_log(rng, 1, 32), t=window + rng.randrange(20000),
                     window=window, ring=rng.random() < 0.6)
    if kind == "ragged":
        return _case("", "ragged", LLAMA, batch=rng.randrange(9, 65), t=rng.randrange(600, 8192), layers=rng.randrange(1, 5),
                     block=block)
    if kind == "step_f32":
        shape = rng.choice([LLAMA, TINY, NARROW])
        return _case("", "step", shape, "f32", block=64, batch=_log(rng, 1, 16), t=_log(rng, 64, 2048) - 1)
    if kind == "block":
        count = rng.randrange(2, 128 // (shape[0] // shape[1]) + 1) if shape[0] > shape[1] else rng.randrange(2, 65)
        return _case("", "block", shape, block=block, batch=_log(rng, 1, 16), t=_log(rng, 128, 8000), count=count,
                     rope=rng.random() < 0.4)
    if kind == "prompt":
        batch = _log(rng, 1, 16)
        count = _log(rng, 33, 4096 if shape[0] * shape[2] <= 3072 else 2900)
        history = rng.choice([0, 0, rng.randrange(1, 2000)]) if batch * count <= 16384 else 0
        window = rng.choice([0, 0, 0, _log(rng, 64, 1024)])
        return _case("", "prompt", shape, block=block, batch=batch, t=history, count=count, window=window,
                     rope=rng.random() < 0.4)
    if kind == "prompt_window":
        batch = _log(rng, 1, 8)
        return _case("", "prompt", LLAMA, batch=batch, count=_log(rng, 64, 8192 // batch), window=_log(rng, 64, 512),
                     ring=True, block=block)
    if kind == "prompt_f32":
        return _case("", "prompt", TINY, "f32", block=64, count=_log(rng, 16, 512))
    T_ = _log(rng, 50, 20000)
    n = rng.choice([0, 5, min(T_, _log(rng, 2, 512))])
    return {"kind": "returns", "batch": _log(rng, 1, 512), "T": T_, "n": n}


# ---- inputs ------------------------------------------------------------------------------------

def _normal(shape, generator, dtype):
    return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, 1.0, generator=generator)


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _rope_tables(positions, head_dim):
    half = head_dim // 2
    inv = THETA ** (-torch.arange(half, dtype=torch.float64, device=DEVICE) * 2.0 / head_dim)
    angle = torch.arange(positions, dtype=torch.float64, device=DEVICE)[:, None] * inv[None, :]
    return torch.cos(angle).to(torch.float32).contiguous(), torch.sin(angle).to(torch.float32).contiguous()


def _rotate64(x, cos, sin):
    """x [..., steps, heads, D] in 64 bits turned by rows of cos, sin [steps][D/2]."""
    half = x.shape[-1] // 2
    c, s = cos.double()[:, None, :], sin.double()[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _first_key(c):
    """First step whose key any query of the call sees."""
    return max(0, c["t"] - c["window"] + 1) if c["window"] else 0


def _inputs(c, seed):
    """q and the call's new rows, and the history before the call (rows _first_key .. t-1)."""
    g = _generator(seed)
    dt = DTYPES[c["dtype"]][1]
    B, C, Hq, Hkv, D = c["batch"], c["count"], c["q_heads"], c["kv_heads"], c["head_dim"]
    past = c["t"] - _first_key(c)
    return {"q": _normal((B, C, Hq, D), g, dt), "k": _normal((B, C, Hkv, D), g, dt), "v": _normal((B, C, Hkv, D), g, dt),
            "k_past": _normal((B, past, Hkv, D), g, dt), "v_past": _normal((B, past, Hkv, D), g, dt)}


def _ragged_inputs(c, seed):
    """Per-sequence steps, and per layer q, the new rows and all earlier rows, sequence after sequence."""
    g = _generator(seed)
    B, Hq, Hkv, D = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"]
    # steps uniform in 0 .. t: the same set for every seed, so that every seed is the same work
    lengths = random.Random(B * 65536 + c["t"])
    steps = torch.tensor([lengths.randrange(c["t"] + 1) for _ in range(B)], dtype=torch.int32, device=DEVICE)
    steps = steps[torch.randperm(B, generator=g, device=DEVICE)].contiguous()
    total = int(steps.sum())
    bf = torch.bfloat16
    layers = [{"q": _normal((B, Hq, D), g, bf), "k": _normal((B, Hkv, D), g, bf), "v": _normal((B, Hkv, D), g, bf),
               "k_past": _normal((total, Hkv, D), g, bf), "v_past": _normal((total, Hkv, D), g, bf)}
              for _ in range(c["layers"])]
    return g, steps, layers


def _fill(store, k, v, t0):
    """Earlier rows into the block store, in calls that a ring store accepts."""
    most = store.ring_blocks * store.Z if store.ring_blocks else 65536
    for i in range(0, k.shape[1], most):
        n = min(most, k.shape[1] - i)
        store.append_block(k[:, i:i + n].contiguous(), v[:, i:i + n].contiguous(), t0 + i, n)


def _random_table(blocks, generator):
    return torch.randperm(blocks, generator=generator, device=DEVICE).to(torch.int32)


def prepare(case, seed):
    c = case
    if c["kind"] == "returns":
        r = _normal((c["batch"], c["T"]), _generator(seed), torch.float32)
        return {"case": c, "r": r, "g": torch.empty_like(r)}
    if c["kind"] == "ragged":
        return _prepare_ragged(c, seed)
    Hq, Hkv, D, Z = c["q_heads"], c["kv_heads"], c["head_dim"], c["block"]
    x = _inputs(c, seed)
    last = c["t"] + c["count"] - 1
    ring = 0
    if c["ring"]:
        ring = T.tempo_ring_blocks(c["window"], Z, min(c["count"], 128 // (Hq // Hkv)))
    columns = ring if ring else last // Z + 1
    table = _random_table(c["batch"] * columns, _generator(seed + 1)).reshape(c["batch"], columns)
    store = BlockStore(c["batch"], Hq, Hkv, D, Z, last, DTYPES[c["dtype"]][0], device=DEVICE, ring_blocks=ring,
                       block_table=table)
    past = x["k_past"]
    if c["rope"]:
        cos, sin = _rope_tables(last + 1, D)
        store.set_rope(cos, sin)
        first = _first_key(c)
        past = _rotate64(past.double(), cos[first:c["t"]], sin[first:c["t"]]).to(past.dtype)
    if past.shape[1]:
        _fill(store, past, x["v_past"], _first_key(c))
    s = {"case": c, "store": store, "q": x["q"], "k": x["k"], "v": x["v"]}
    if c["kind"] == "step":
        s["q"], s["k"], s["v"] = x["q"][:, 0].contiguous(), x["k"][:, 0].contiguous(), x["v"][:, 0].contiguous()
    s["out"] = torch.empty_like(s["q"])
    return s


def _prepare_ragged(c, seed):
    B, Hq, Hkv, D, Z = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"], c["block"]
    g, steps, layers = _ragged_inputs(c, seed)
    host_steps = steps.tolist()
    columns = c["t"] // Z + 1
    need = [t // Z + 1 for t in host_steps]
    blocks = sum(need)
    stores = []
    for x in layers:
        free = _random_table(blocks, g).cpu()
        table = torch.zeros((B, columns), dtype=torch.int32)
        at = 0
        for b in range(B):
            table[b, :need[b]] = free[at:at + need[b]]
            at += need[b]
        store = BlockStore(B, Hq, Hkv, D, Z, c["t"], T.TEMPO_BF16, device=DEVICE, num_blocks=blocks, block_table=table)
        at = 0
        for b in range(B):
            n = host_steps[b]
            if n:
                one = T.make_kv(store.k_pool, store.v_pool, store.block_table[b], blocks, columns, Z, Hkv, D, T.TEMPO_BF16)
                T.tempo_kv_append_block(one, x["k_past"][at:at + n], x["v_past"][at:at + n], 1, 0, None, n)
            at += n
        stores.append(store)
    nbytes = T.tempo_attn_worklist_bytes(stores[0].kv, B, Hq, c["t"], 0)
    return {"case": c, "stores": stores, "steps": steps, "layers": [(x["q"], x["k"], x["v"]) for x in layers],
            "outs": [torch.empty_like(x["q"]) for x in layers], "list_bytes": nbytes,
            "list": torch.empty(nbytes // 4, dtype=torch.int32, device=DEVICE)}


# ---- one pass ----------------------------------------------------------------------------------

def _call(s):
    c = s["case"]
    store = s["store"]
    if c["kind"] == "step":
        if c["rope"]:
            store.rope_step(s["q"], s["k"], s["v"], s["out"], c["t"], c["window"])
        elif c["window"]:
            store.step_window(s["q"], s["k"], s["v"], s["out"], c["t"], c["window"])
        else:
            store.step_causal(s["q"], s["k"], s["v"], s["out"], c["t"])
    elif c["kind"] == "block":
        if c["rope"]:
            store.rope_append_block(s["k"], s["v"], c["t"], c["count"])
        else:
            store.append_block(s["k"], s["v"], c["t"], c["count"])
        store.attend_block(s["q"], s["out"], c["t"], c["count"], rope=c["rope"])
    else:
        store.prefill_attend(s["q"], s["k"], s["v"], s["out"], c["t"], c["count"], window=c["window"], rope=c["rope"])
    return [s["out"], store.k_pool, store.v_pool]


def run(state):
    c = state["case"]
    if c["kind"] == "returns":
        T.tempo_discounted_sum(state["r"], state["g"], c["batch"], c["T"], c["n"], 0.95)
        return [state["g"]]
    if c["kind"] != "ragged":
        return _call(state)
    first = state["stores"][0]
    T.tempo_attn_worklist_build(first.kv, c["batch"], c["q_heads"], c["t"], state["steps"], 0, state["list"],
                                state["list_bytes"])
    got = []
    for store, (q, k, v), out in zip(state["stores"], state["layers"], state["outs"]):
        store.step_ragged(q, k, v, out, c["t"], state["steps"], state["list"])
        got += [out, store.k_pool, store.v_pool]
    return got


# ---- what a pass cannot do without, and what it has to give ------------------------------------

def _pairs(c):
    """(query step, visible key) pairs of one sequence, and its distinct visible keys."""
    last = c["t"] + c["count"] - 1
    if not c["window"]:
        return sum(range(c["t"] + 1, last + 2)), last + 1
    return sum(min(t + 1, c["window"]) for t in range(c["t"], last + 1)), last + 1 - _first_key(c)


def work(case):
    c = case
    if c["kind"] == "returns":
        return {"bytes": 8 * c["batch"] * c["T"], "flops": 2 * c["batch"] * c["T"]}
    e = 2 if c["dtype"] == "bf16" else 4
    Hq, Hkv, D, B = c["q_heads"], c["kv_heads"], c["head_dim"], c["batch"]
    if c["kind"] == "ragged":
        lengths = random.Random(B * 65536 + c["t"])
        keys = sum(lengths.randrange(c["t"] + 1) + 1 for _ in range(B))
        return {"bytes": c["layers"] * e * D * (2 * Hkv * keys + 2 * B * Hq + 2 * B * Hkv),
                "flops": c["layers"] * 4 * D * Hq * keys}
    pairs, keys = _pairs(c)
    # keys and values read once (the new ones from the call's rows) and the new ones written, q in, out out
    return {"bytes": B * e * D * (2 * Hkv * keys + 2 * Hkv * c["count"] + 2 * Hq * c["count"]),
            "flops": B * 4 * D * Hq * pairs}


def tolerance(case):
    if case["kind"] == "returns" or case["dtype"] == "f32":
        return {"rel": 1.5e-6, "max": 1e-4}  # 32-bit sums: 1e-7 to 2.3e-7 from exact() at these sizes
    # 2e-3 to 2.8e-3 from exact(): bf16 weights of the products and a bf16 result
    return {"rel": 1e-2, "max": 1e-1}


# ---- the same in 64 bits -----------------------------------------------------------------------

def _attend64(q, k, v, t, first, window):
    """q [C][Hq][D] of steps t .. t+C-1 over k, v [n][Hkv][D] of steps first .. first+n-1, all in 64 bits."""
    C, Hq, D = q.shape
    n, Hkv = k.shape[0], k.shape[1]
    G = Hq // Hkv
    j = torch.arange(first, first + n, device=q.device)[None, :]
    out = torch.empty_like(q)
    for c0 in range(0, C, 1024):
        steps = torch.arange(t + c0, t + min(C, c0 + 1024), device=q.device)[:, None]
        seen = (j <= steps) & (j > steps - window) if window else j <= steps
        seen = seen.repeat_interleave(G, dim=0)
        for h in range(Hkv):
            qh = q[c0:c0 + 1024, h * G:(h + 1) * G].reshape(-1, D)
            x = (qh @ k[:, h].t()) * (1.0 / math.sqrt(D))
            p = torch.softmax(x.masked_fill(~seen, float("-inf")), dim=-1)
            out[c0:c0 + 1024, h * G:(h + 1) * G] = (p @ v[:, h]).reshape(-1, G, D)
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "returns":
        r = prepare(c, seed)["r"].double()
        T_, n = c["T"], c["n"] if c["n"] else c["T"]
        gamma = float(torch.tensor(0.95, dtype=torch.float32))
        g = torch.zeros_like(r)
        # g[t] = r[t] + gamma g[t+1], less the reward that leaves a window of n steps
        nxt = torch.zeros_like(r[:, 0])
        if n >= T_:
            rows = r.cpu()
            nxt = nxt.cpu()
            g = g.cpu()
            for t in range(T_ - 1, -1, -1):
                nxt = rows[:, t] + gamma * nxt
                g[:, t] = nxt
            return [g]
        for m in range(n):
            g[:, :T_ - m] += gamma ** m * r[:, m:]
        return [g]
    if c["kind"] == "ragged":
        _, steps, layers = _ragged_inputs(c, seed)
        got = []
        for x in layers:
            out = torch.empty(x["q"].shape, dtype=torch.float64, device=DEVICE)
            at = 0
            for b, n in enumerate(steps.tolist()):
                k = torch.cat([x["k_past"][at:at + n], x["k"][b:b + 1]]).double()
                v = torch.cat([x["v_past"][at:at + n], x["v"][b:b + 1]]).double()
                out[b] = _attend64(x["q"][b:b + 1].double(), k, v, n, 0, 0)[0]
                at += n
            got += [out, None, None]
        return got
    x = _inputs(c, seed)
    first, last = _first_key(c), c["t"] + c["count"] - 1
    out = torch.empty(x["q"].shape, dtype=torch.float64, device=DEVICE)
    for b in range(c["batch"]):
        q, k, v = x["q"][b].double(), x["k"][b].double(), torch.cat([x["v_past"][b], x["v"][b]]).double()
        past = x["k_past"][b].double()
        if c["rope"]:
            cos, sin = _rope_tables(last + 1, c["head_dim"])
            q, k = _rotate64(q, cos[c["t"]:], sin[c["t"]:]), _rotate64(k, cos[c["t"]:], sin[c["t"]:])
            past = _rotate64(past, cos[first:c["t"]], sin[first:c["t"]])
            past = past.to(x["k"].dtype).double()  # the history holds rounded keys before the call begins
        out[b] = _attend64(q, torch.cat([past, k]), v, c["t"], first, c["window"])
    return [out[:, 0] if c["kind"] == "step" else out, None, None]
