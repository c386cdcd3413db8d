"""The work that a user of this framework has it do, as cases that can be timed and compared.

Three kinds of call, each through the package's public functions:

  step    one generation step of a cache (kf_decode_select_step): append, attention, score, eviction.  With
          "apart" a model's layers hold caches of their own and one pass is a whole token: one
          kf_decode_select_step_at call per layer, captured once in a HIP graph and replayed.
  prompt  prompt scoring (kf_prefill_score): the causal column sums that seed the scores.
  evict   the eviction after the prompt (kf_select_evict_into): n staged tokens -> the k-token cache.

Sizes are those of kf_workloads.CONFIGS (whole workloads, or one layer of them, which is what a model that
runs its layers one after the other calls) or generic.  exact() is the method in float64, written here in
plain torch.
"""
import math

import numpy as np
import torch

import paper_2403_09054_amd as kf

RING = 8  # distinct generated tokens (q, k_new, v_new) that the steps take in turn
DTYPES = {"f32": (kf.F32, torch.float32), "bf16": (kf.BF16, torch.bfloat16), "f16": (kf.F16, torch.float16)}
TAU = (1.0, 2.0)


def _step(name, L, B, H, d, k, w, n, T, dtype="bf16", layout="ordered", G=1, alibi=False, outliers=0.0, apart=False):
    return {"name": name, "call": "step", "L": L, "B": B, "H": H, "d": d, "k": k, "w": w, "n": n, "T": T, "dtype": dtype,
            "layout": layout, "G": G, "alibi": alibi, "outliers": outliers, "apart": apart}


def _prompt(name, L, B, H, d, n, dtype="bf16", G=1, alibi=False, outliers=0.0, padded=False, noise="gumbel"):
    return {"name": name, "call": "prompt", "L": L, "B": B, "H": H, "d": d, "n": n, "dtype": dtype, "G": G,
            "alibi": alibi, "outliers": outliers, "padded": padded, "noise": noise}


def _evict(name, L, B, H, d, n, k, w, dtype="bf16"):
    return {"name": name, "call": "evict", "L": L, "B": B, "H": H, "d": d, "n": n, "k": k, "w": w, "dtype": dtype}


def listed():
    return [
        # the smallest call: one small layer in fp32, where launches and host time are everything
        _step("tiny_step", 1, 1, 2, 64, 64, 16, 128, 32, dtype="f32"),
        # serving one sequence: a token through 28 layers, one call per layer, replayed from a graph
        _step("gptj_token_graph", 28, 1, 16, 256, 1024, 205, 2048, 512, outliers=0.01, apart=True),
        # the same model with all layers' caches in one call
        _step("gptj_step", 28, 1, 16, 256, 1024, 205, 2048, 512, outliers=0.01),
        # one layer of a batch of 8 with position bias, in the layout that moves one row per step
        _step("mpt_layer_step_slot", 1, 8, 32, 128, 2048, 410, 4096, 1024, layout="slot", alibi=True),
        # all layers of that batch, order-preserving: the largest step (8.6 GB of cache)
        _step("mpt_step", 32, 8, 32, 128, 2048, 410, 4096, 1024, alibi=True),
        # one layer of a large batch
        _step("batched_layer_step", 1, 64, 32, 128, 1024, 205, 2048, 1024),
        # one layer of one long sequence: few, long units
        _step("long_layer_step", 1, 1, 32, 128, 9830, 1966, 32768, 2048, outliers=0.005),
        # grouped-query attention in half precision, a budget that is no multiple of anything
        _step("grouped_step_f16", 4, 8, 8, 128, 1501, 300, 3002, 512, dtype="f16", G=4),
        # prompt scoring of one layer: one sequence of a model with wide heads
        _prompt("gptj_prompt_layer", 1, 1, 16, 256, 2048, outliers=0.01),
        # ... a batch with position bias
        _prompt("mpt_prompt_layer", 1, 8, 32, 128, 4096, alibi=True),
        # ... one long document: the most work of one call
        _prompt("long_prompt_layer", 1, 1, 32, 128, 32768, outliers=0.005),
        # the eviction after the prompt of one layer of a large batch
        _evict("batched_evict_layer", 1, 64, 32, 128, 2048, 1024, 205),
    ]


def draw(rng):
    """One more case: sizes over the whole range, their logarithms even."""
    case = _drawn(rng)
    del case["name"]
    return case


def _drawn(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("step", "step", "prompt", "evict"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f16", "f32"))
    d = rng.choice((64, 128, 128) if dtype == "f32" else (64, 128, 128, 256))
    eb = 4 if dtype == "f32" else 2
    B, H = rng.choice((1, 1, 2, 4, 8, 16, 32, 64)), rng.choice((2, 8, 12, 16, 32, 32))
    outliers = rng.choice((0.0, 0.005, 0.01))
    if kind == "step":
        k = log(64, 9830)
        L = max(1, min(log(1, 32), int(4e9 / (B * H * k * 2.0 * d * eb))))
        B = max(1, min(B, int(8e9 / (L * H * k * 2.0 * d * eb))))
        G = rng.choice((1, 1, 1, 2, 4, 8))
        return _step("", L, B, H, d, k, int(k * rng.uniform(0.05, 0.4)), 2 * k, 1024, dtype,
                     rng.choice(("ordered", "ordered", "slot")), G, rng.random() < 0.3, outliers, L <= 4 and rng.random() < 0.25)
    if kind == "prompt":
        n = log(120, 16000)
        G = rng.choice((1, 1, 1, 2, 4))
        most = 6e12 if dtype != "f32" else 5e11
        L = max(1, min(log(1, 28), int(0.5 * most / (B * H * G * float(n) * n * d))))
        B = max(1, min(B, int(0.5 * most / (L * H * G * float(n) * n * d)), int(4e9 / (L * H * G * n * d * eb))))
        return _prompt("", L, B, H, d, n, dtype, G, rng.random() < 0.3, outliers, B > 1 and rng.random() < 0.3,
                       rng.choice(("gumbel", "gumbel", "gumbel", "none")))
    n = log(200, 32768)
    k = max(2, int(n * rng.uniform(0.2, 0.6)))
    L = max(1, min(log(1, 8), int(4e9 / (B * H * n * 2.0 * d * eb))))
    B = max(1, min(B, int(8e9 / (L * H * n * 2.0 * d * eb))))
    return _evict("", L, B, H, d, n, k, int(k * rng.uniform(0.05, 0.4)), dtype)


# ---------------------------------------------------------------- inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream * 7919 + 20240309) & 0x7FFFFFFFFFFFFFFF)
    return g


def _normal(shape, dt, g):
    """N(0,1) in the element type (large tensors in pieces: no float32 copy of the whole)."""
    t = torch.empty(shape, dtype=dt, device="cuda")
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        piece = flat[i:i + (1 << 28)]
        piece.copy_(torch.randn(piece.numel(), generator=g, device="cuda"))
    return t


def _scale_rows(K, frac, g):
    """A share of the key rows four times as long: the tokens that attract attention."""
    if frac > 0:
        hit = torch.rand(K.shape[:-1], generator=g, device="cuda") < frac
        K.mul_(torch.where(hit, 4.0, 1.0).to(K.dtype).unsqueeze(-1))


def _slopes(case):
    if not case["alibi"]:
        return None
    HQ = case["H"] * case["G"]
    return torch.tensor([2.0 ** (-8.0 * (h + 1) / HQ) for h in range(HQ)], dtype=torch.float32, device="cuda")


def _seeds(case, seed):
    return (torch.arange(case["B"], dtype=torch.int64, device="cuda") ^ (20240309 + int(seed)))


def _scale(case):
    return float(np.float32(1.0) / np.sqrt(np.float32(case["d"])))


def _workspace(c, n=0):
    return kf.new_workspace(c, n)


def _t0(case):
    return case["T"] // 2  # the step that a run begins at: the middle of the generation


def _prepare_step(case, seed):
    L, B, H, d, k, w, G, n = (case[x] for x in ("L", "B", "H", "d", "k", "w", "G", "n"))
    code, dt = DTYPES[case["dtype"]]
    g = _gen(seed, 1)
    U, cap = L * B * H, k + 1
    K, V = _normal((L, B, H, cap, d), dt, g), _normal((L, B, H, cap, d), dt, g)
    _scale_rows(K, case["outliers"], g)
    # the w newest positions, and k-w of the others; scores: what the key tokens gathered since the prompt,
    # and, in the window, what a token of that age has gathered so far
    q0 = case["n"] + _t0(case) - 2  # position of the newest cached token
    keys = torch.rand((U, q0 + 1 - w), generator=g, device="cuda").topk(k - w, dim=1).indices.sort(dim=1).values
    pos = torch.zeros((U, cap), dtype=torch.int32, device="cuda")
    pos[:, :k - w] = keys.int()
    pos[:, k - w:k] = torch.arange(q0 + 1 - w, q0 + 1, device="cuda", dtype=torch.int32)
    noise = torch.randn((U, k), generator=g, device="cuda")
    score = torch.zeros((U, cap), dtype=torch.float32, device="cuda")
    score[:, :k - w] = 0.3 + torch.exp(0.7 * noise[:, :k - w])
    age = torch.arange(w, 0, -1, device="cuda", dtype=torch.float32) / (k + 1)
    score[:, k - w:k] = age * torch.exp(0.4 * noise[:, k - w:])
    if case["layout"] == "slot":  # the entries in any order, as a generation in this layout leaves them
        perm = torch.rand((U, k), generator=g, device="cuda").argsort(dim=1)
        pos[:, :k], score[:, :k] = pos[:, :k].gather(1, perm), score[:, :k].gather(1, perm)
    pos, score = pos.view(L, B, H, cap), score.view(L, B, H, cap)
    lens = torch.full((L, B, H), k, dtype=torch.int32, device="cuda")
    qkv = [(_normal((L, B, H * G, d), dt, g), _normal((L, B, H, d), dt, g), _normal((L, B, H, d), dt, g)) for _ in range(RING)]
    for _, kn, _ in qkv:
        _scale_rows(kn, case["outliers"], g)
    cache = kf.Cache(K=K, V=V, score=score, pos=pos, len=lens, L=L, B=B, H=H, d=d, cap=cap, dtype=code, q_per_kv=G)
    s = {"case": case, "cache": cache, "out": torch.zeros((L, B, H * G, d), dtype=torch.float32, device="cuda"),
         "seeds": _seeds(case, seed), "slopes": _slopes(case), "qkv": qkv, "t": _t0(case),
         "layout": kf.LAYOUT_SLOT if case["layout"] == "slot" else kf.LAYOUT_ORDERED}
    if not case["apart"]:
        s["ws"] = _workspace(cache)
        return s
    # one cache per layer (slices of the same buffers), one captured call each; the step number of each layer
    # lives in device memory, the token's inputs are copied into the buffers that the graph reads
    layers = [kf.Cache(K=K[l:l + 1], V=V[l:l + 1], score=score[l:l + 1], pos=pos[l:l + 1], len=lens[l:l + 1], L=1, B=B, H=H,
                       d=d, cap=cap, dtype=code, layer0=l, q_per_kv=G) for l in range(L)]
    ws = _workspace(layers[0])
    now = tuple(t.clone() for t in qkv[0])
    step = torch.full((L,), _t0(case), dtype=torch.int32, device="cuda")

    def calls(which):
        for l in which:
            kf.kf_decode_select_step_at(layers[l], now[0][l], now[1][l], now[2][l], n, case["T"], TAU[0], TAU[1],
                                        step[l:l + 1], cap, _scale(case), kf.NOISE_GUMBEL, s["seeds"], s["slopes"],
                                        s["out"][l], k=k, w=w, layout=s["layout"], workspace=ws)

    keep = [t[:1].clone() for t in (K, V, score, pos, lens)] + [step.clone()]
    calls([0])  # loads the kernels; its results are taken back
    for t, old in zip((K, V, score, pos, lens), keep):
        t[:1].copy_(old)
    step.copy_(keep[-1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(range(L))
    s.update(layers=layers, ws=ws, now=now, step=step, graph=graph)
    return s


def _lens(case, seed):
    """Prompt lengths of a batch padded to n: between a quarter of it and all of it, one of them whole."""
    r = np.random.RandomState((int(seed) * 31 + 7) & 0x7FFFFFFF)
    v = r.randint(max(1, case["n"] // 4), case["n"] + 1, case["B"])
    v[r.randint(case["B"])] = case["n"]
    return v.astype(np.int32)


def _prepare_prompt(case, seed):
    L, B, H, d, n, G = (case[x] for x in ("L", "B", "H", "d", "n", "G"))
    code, dt = DTYPES[case["dtype"]]
    g = _gen(seed, 2)
    K = _normal((L, B, H, n, d), dt, g)
    _scale_rows(K, case["outliers"], g)
    Q = _normal((L, B, H * G, n, d), dt, g)
    cache = kf.Cache(K=K, V=K, score=torch.zeros((L, B, H, n), dtype=torch.float32, device="cuda"),  # V is not touched
                     pos=torch.zeros((L, B, H, n), dtype=torch.int32, device="cuda"),
                     len=torch.zeros((L, B, H), dtype=torch.int32, device="cuda"), L=L, B=B, H=H, d=d, cap=n, dtype=code,
                     q_per_kv=G)
    return {"case": case, "cache": cache, "Q": Q, "seeds": _seeds(case, seed), "slopes": _slopes(case),
            "seq_n": torch.from_numpy(_lens(case, seed)).cuda() if case["padded"] else None, "ws": _workspace(cache, n)}


def _prepare_evict(case, seed):
    L, B, H, d, n, k = (case[x] for x in ("L", "B", "H", "d", "n", "k"))
    code, dt = DTYPES[case["dtype"]]
    g = _gen(seed, 3)
    U = L * B * H
    K, V = _normal((L, B, H, n, d), dt, g), _normal((L, B, H, n, d), dt, g)
    # column sums of a causal softmax: a token that i rows see gathers about log(n/i), widely spread
    mean = torch.log(n / (torch.arange(n, device="cuda", dtype=torch.float32) + 1.0)) + 1.0 / n
    score = mean * torch.exp(0.8 * torch.randn((U, n), generator=g, device="cuda"))
    src = kf.Cache(K=K, V=V, score=score.view(L, B, H, n),
                   pos=torch.arange(n, device="cuda", dtype=torch.int32).expand(L, B, H, n).contiguous(),
                   len=torch.full((L, B, H), n, dtype=torch.int32, device="cuda"), L=L, B=B, H=H, d=d, cap=n, dtype=code)
    return {"case": case, "src": src, "dst": kf.Cache.allocate(L, B, H, d, k + 1, code), "ws": _workspace(src)}


def prepare(case, seed):
    return {"step": _prepare_step, "prompt": _prepare_prompt, "evict": _prepare_evict}[case["call"]](case, seed)


# ---------------------------------------------------------------- one pass
def _live(c, n):
    return {"K": c.K[..., :n, :], "V": c.V[..., :n, :], "score": c.score[..., :n], "pos": c.pos[..., :n], "len": c.len}


def run(s):
    case = s["case"]
    if case["call"] == "step":
        q, kn, vn = s["qkv"][s["t"] % RING]
        t = s["t"]
        s["t"] += 1
        if case["apart"]:
            for dst, src in zip(s["now"], (q, kn, vn)):
                dst.copy_(src)
            s["graph"].replay()
        else:
            kf.kf_decode_select_step(s["cache"], q, kn, vn, case["n"] + t - 1, case["k"] + 1, kf.kf_tau(min(t, case["T"]), case["T"], *TAU),
                                     _scale(case), kf.NOISE_GUMBEL, s["seeds"], s["slopes"], s["out"], k=case["k"], w=case["w"],
                                     layout=s["layout"], workspace=s["ws"])
        return {"out": s["out"], **_live(s["cache"], case["k"])}
    if case["call"] == "prompt":
        c = s["cache"]
        kf.kf_prefill_score(c, s["Q"], case["n"], TAU[0], _scale(case), kf.NOISE_GUMBEL if case["noise"] == "gumbel" else kf.NOISE_NONE,
                            s["seeds"], s["slopes"], s["ws"], seq_n=s["seq_n"])
        return {"score": c.score, "pos": c.pos, "len": c.len}
    kf.kf_select_evict_into(s["src"], s["dst"], 0, case["k"], case["w"], None, s["ws"])
    return _live(s["dst"], case["k"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    eb = 4 if case["dtype"] == "f32" else 2
    U, d = case["L"] * case["B"] * case["H"], case["d"]
    if case["call"] == "step":
        k, w, G = case["k"], case["w"], case["G"]
        # K and V rows, scores and positions in; scores out; q, k_new, v_new in and the attention output out
        b = k * (2.0 * d * eb + 12) + (G + 2) * d * eb + 4.0 * G * d
        # the window's rows move down by one slot (the slot layout stores one row)
        b += (w if case["layout"] == "ordered" else 1) * (2.0 * d * eb + 8)
        return {"bytes": U * b, "flops": U * G * (k + 1) * 4.0 * d}
    if case["call"] == "prompt":
        n, G = case["n"], case["G"]
        rows = _lens(case, 1).astype(float) if case["padded"] else np.full(case["B"], float(n))
        per = case["L"] * case["H"]
        return {"bytes": per * rows.sum() * ((1 + G) * d * eb + 8.0), "flops": per * G * float((rows * (rows + 1)).sum()) * d}
    n, k = case["n"], case["k"]
    return {"bytes": U * (n * 4.0 + k * (4.0 * d * eb + 12)), "flops": 0.0}


def tolerance(case):
    if case["call"] == "evict":
        return "exact"  # a choice among the given scores, and moves
    if case["call"] == "prompt":  # a column's sum over up to n rows in 32 bits: 4e-7 measured at 4096 rows, 1e-5 at 32768
        return {"rel": 4e-5 if case["n"] > 8192 else 1e-5}
    return {"rel": 1e-5}  # sums in 32 bits: 3e-7 measured, 2e-6 with 8 query heads (the same rows move on either side)


# ---------------------------------------------------------------- the method in float64
M32 = 0xFFFFFFFF


def _mix32(x):
    x = x ^ (x >> 16)
    x = (x * 0x6A09E667) & M32
    x = x ^ (x >> 15)
    x = (x * 0xBB67AE85) & M32
    return x ^ (x >> 16)


def _mix64(z):
    z = z ^ (z >> np.uint64(32))
    z = z * np.uint64(0x6A09E667F3BCC909)
    z = z ^ (z >> np.uint64(29))
    z = z * np.uint64(0xBB67AE8584CAA73B)
    return z ^ (z >> np.uint64(32))


def _unit_keys(seeds, L, HQ):
    """The two halves of each (layer, sequence, query head)'s noise key: [L*B*HQ] int64 tensors."""
    with np.errstate(over="ignore"):
        sb = _mix64(seeds.cpu().numpy().astype(np.uint64) + np.uint64(0x9E3779B97F4A7C15))
        lh = (np.arange(L, dtype=np.uint64)[:, None] << np.uint64(32)) | np.arange(HQ, dtype=np.uint64)[None, :]
        u = _mix64(sb[None, :, None] + lh[:, None, :]).reshape(-1)
    lo, hi = (u & np.uint64(M32)).astype(np.int64), (u >> np.uint64(32)).astype(np.int64)
    return torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()


def _row_keys(ka, kb, q_pos):
    return _mix32((_mix32(ka ^ ((q_pos * 0x9E3779B9) & M32)) + kb) & M32)


def _gumbel(rkey, k_pos):
    bits = _mix32(rkey ^ ((k_pos * 0x243F6A89) & M32))
    u = (2 * (bits >> 9) + 1).double() * 2.0 ** -24
    return -torch.log(-torch.log(u))


def _tau32(t, T):
    return float(np.float32(TAU[0]) + np.float32(t) * (np.float32(TAU[1] - TAU[0]) / np.float32(T)))


def _exact_step(case, seed):
    s = _prepare_step(dict(case, apart=False), seed)
    c, t = s["cache"], s["t"]
    q, kn, vn = s["qkv"][t % RING]
    L, B, H, d, k, w, G = (case[x] for x in ("L", "B", "H", "d", "k", "w", "G"))
    U, q_pos, tau = L * B * H, case["n"] + t - 1, _tau32(min(t, case["T"]), case["T"])
    ka, kb = (x.view(U, G) for x in _unit_keys(s["seeds"], L, H * G))
    K, V = c.K.view(U, k + 1, d), c.V.view(U, k + 1, d)
    q, kn, vn = q.view(U, G, d), kn.view(U, 1, d), vn.view(U, 1, d)
    pos, f = c.pos.view(U, k + 1).long(), c.score.view(U, k + 1)
    out, score = torch.empty((U, G, d), dtype=torch.float64, device="cuda"), torch.empty((U, k), dtype=torch.float64, device="cuda")
    step = max(1, int(1.5e8 // ((k + 1) * max(d, 8 * G))))
    for a in range(0, U, step):
        z = slice(a, min(U, a + step))
        Kz = torch.cat([K[z, :k], kn[z]], 1).double()
        Vz = torch.cat([V[z, :k], vn[z]], 1).double()
        pz = torch.cat([pos[z, :k], torch.full_like(pos[z, :1], q_pos)], 1)
        x = (q[z].double() @ Kz.transpose(1, 2).contiguous()) * _scale(case)
        if s["slopes"] is not None:
            heads = torch.arange(a, z.stop, device="cuda") % H
            sl = s["slopes"].double().view(H, G)[heads]
            x = x - sl[:, :, None] * (q_pos - pz)[:, None, :]
        out[z] = torch.softmax(x, -1) @ Vz
        rk = _row_keys(ka[z], kb[z], q_pos)
        df = torch.softmax((x + _gumbel(rk[:, :, None], pz[:, None, :])) / tau, -1).sum(1)
        fn = torch.cat([f[z, :k].double(), torch.zeros_like(df[:, :1])], 1) + df
        # one token leaves: the smallest score outside the window of the w newest
        cand = torch.where(pz <= q_pos - w, fn, math.inf) if w > 0 else fn
        e = cand.argmin(1, keepdim=True)
        if case["layout"] == "slot":
            score[z] = fn[:, :k].scatter(1, e.clamp(max=k - 1), fn[:, k:])
        else:
            j = torch.arange(k, device="cuda")[None, :]
            score[z] = fn.gather(1, j + (j >= e))
    return {"out": out.view(L, B, H * G, d), "K": None, "V": None, "score": score.view(L, B, H, k), "pos": None, "len": None}


def _exact_prompt(case, seed):
    s = _prepare_prompt(case, seed)
    L, B, H, d, n, G = (case[x] for x in ("L", "B", "H", "d", "n", "G"))
    UQ = L * B * H * G
    if UQ * float(n) * n > 4e10:
        return None
    ka, kb = _unit_keys(s["seeds"], L, H * G)
    Q, K = s["Q"].view(UQ, n, d), s["cache"].K.view(L * B * H, n, d)
    lens = _lens(case, seed) if case["padded"] else [n] * B
    score = torch.zeros((L * B * H, n), dtype=torch.float64, device="cuda")
    rows = max(64, int(1e8 // n))
    for u in range(UQ):
        h, m = u % (H * G), int(lens[(u // (H * G)) % B])
        Ku = K[u // G].double()
        for i0 in range(0, m, rows):
            i1 = min(m, i0 + rows)
            i, j = torch.arange(i0, i1, device="cuda")[:, None], torch.arange(i1, device="cuda")[None, :]
            x = (Q[u, i0:i1].double() @ Ku[:i1].t().contiguous()) * _scale(case)
            if s["slopes"] is not None:
                x = x - float(s["slopes"][h]) * (i - j)
            if case["noise"] == "gumbel":
                x = x + _gumbel(_row_keys(ka[u], kb[u], i), j)
            x.masked_fill_(j > i, -math.inf)
            score[u // G, :i1] += torch.softmax(x / TAU[0], -1).sum(0)
    return {"score": score.view(L, B, H, n), "pos": None, "len": None}


def exact(case, seed):
    if case["call"] == "evict":
        return None  # nothing is computed
    return _exact_step(case, seed) if case["call"] == "step" else _exact_prompt(case, seed)
