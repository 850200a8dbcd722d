"""The work that a serving program has this library do, as cases that can be
timed and compared.

Three kinds of pass, each through the public entry points:

* "decode": one block of `s` decode steps over `layers` layers (a refresh, then
  reuse of the shared sets), through DecodeRunner / GatedDecodeRunner.  With
  graph the block was captured once and a pass replays it, which is how a
  serving loop runs it; without, the pass makes the library calls one by one.
* "dense": dense decode attention of one step over `layers` layers.
* "prefill": causal attention of whole prompts, with or without the
  progressive sliding window.

A decode or dense case holds enough layers that its caches do not stay in the
chip's last-level cache from one layer to the next, as in a whole model, unless
the calls themselves are so small that they stay there in real use as well.
"""

import math

import torch

from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import schedule, synth

DEV = "cuda"


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "dtype": "bf16", "batch": 1, "hq": 32, "hkv": 8, "d": 128,
         "n": 4096, "ragged": False, "layers": 1, "paged": False, "page": 16}
    if kind == "decode":
        c.update(k=0, k_num=0, k_den=0, window=64, sink=4, s=4, G=1, r=1, layer_corr=0.0,
                 heavy=8, heavy_tail=False, graph=True, per_step=False, tau=-1.0, psaw=False)
    if kind == "prefill":
        c.update(psaw=False, psaw_layer=0, num_layers=32, sink=16)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest calls: one fp32 layer of a short context, call by call;
        # what counts is the calls themselves and their launches
        _case("tiny-f32-1k", "decode", dtype="f32", hq=4, hkv=4, d=64, n=1024, k=64, window=32,
              graph=False),
        # an fp32 model with grouped queries, mixed lengths, the shared set
        # rebuilt at each step, call by call
        _case("f32-gqa-4k", "decode", dtype="f32", batch=4, n=4001, ragged=True, layers=2, k=256,
              per_step=True, graph=False),
        # a small model with 64-dim heads, odd mixed lengths, call by call
        _case("d64-mha-2k", "decode", batch=6, hq=12, hkv=12, d=64, n=2035, ragged=True, layers=2,
              k=128, graph=False),
        # LLaMA-2-7B-shaped decoding at 4k with sets shared over 4 layers
        _case("llama2-mha-4k", "decode", batch=8, hkv=32, layers=8, k=256, G=4, layer_corr=0.8),
        # the same model under the similarity gate and the sliding window:
        # some units retrieve and some share at every step
        _case("llama2-mha-4k-gated", "decode", batch=8, hkv=32, layers=4, k=256, G=4,
              layer_corr=0.8, tau=0.8, psaw=True),
        # Mistral-7B-shaped decoding at 32k
        _case("mistral-gqa-32k", "decode", batch=4, n=32768, layers=8, k=1024, window=128, s=8,
              G=4, layer_corr=0.8),
        # LLaMA-3-8B-shaped decoding of one sequence at 128k, paged
        _case("llama3-gqa-128k-paged", "decode", n=131072, layers=4, k=2048, window=256, s=8,
              paged=True, heavy=655, heavy_tail=True),
        # the throughput sweep's largest batch, mixed lengths up to 16k
        _case("sweep-b64-16k", "decode", batch=64, n=16384, ragged=True, layers=4, k_num=1,
              k_den=20, window=128),
        # a serving batch on a paged cache, mixed lengths up to 8k
        _case("serve-b48-8k-paged", "decode", batch=48, n=8191, ragged=True, layers=4, k_num=1,
              k_den=20, window=128, paged=True),
        # the dense baseline over a long paged context
        _case("dense-b2-64k-paged", "dense", batch=2, n=65536, paged=True),
        # a LLaMA-2-7B-shaped prompt of 4k, causal
        _case("prefill-mha-4k", "prefill", hkv=32),
        # two grouped-query prompts of different lengths on a paged cache, a
        # deep layer under the sliding window
        _case("prefill-gqa-12k-paged", "prefill", batch=2, n=12289, ragged=True, paged=True,
              psaw=True, psaw_layer=30),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "dense", "prefill"])
    d = rng.choice([64, 128, 128, 128])
    hkv = rng.choice([4, 8, 8, 32])
    hq = hkv * (1 if hkv == 32 else rng.choice([1, 2, 4, 8]))
    paged = rng.random() < 0.4
    page = rng.choice([16, 16, 32, 64])
    ragged = rng.random() < 0.6
    name = "drawn"
    if kind == "prefill":
        n = _log(rng, 130, 9000)
        batch = rng.choice([1, 1, 2, 4]) if n * n * hq <= 2_000_000_000 else 1
        c = _case(name, kind, batch=batch, hq=hq, hkv=hkv, d=d, n=n, ragged=ragged, paged=paged,
                  page=page, psaw=rng.random() < 0.5, psaw_layer=rng.randrange(24, 32))
    else:
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        n = _log(rng, 300, 16000 if dtype == "f32" else 120000)
        # at most 3 GiB of K and V per layer, spread over up to 4 layers
        row = 2 * hkv * d * (4 if dtype == "f32" else 2)
        batch = max(1, min(_log(rng, 1, 64), (1 << 31) // (row * n)))
        layers = max(1, min(4, (4 << 30) // (row * n * batch)))
        if kind == "dense":
            c = _case(name, kind, dtype=dtype, batch=batch, hq=hq, hkv=hkv, d=d, n=n,
                      ragged=ragged, layers=layers, paged=paged, page=page)
        else:
            window = rng.choice([32, 64, 128, 255])
            k = max(16, min(2048, n // rng.choice([8, 16, 24, 64])))
            gated = dtype == "bf16" and rng.random() < 0.2
            c = _case(name, kind, dtype=dtype, batch=batch, hq=hq, hkv=hkv, d=d, n=n,
                      ragged=ragged, layers=layers, paged=paged, page=page, k=k, window=window,
                      sink=rng.choice([0, 4, 16]), s=rng.choice([2, 4, 8]),
                      G=rng.choice([1, 1, 2, 4]), r=rng.choice([1, 1, 1, 2]),
                      graph=layers > 1 or rng.random() < 0.5, per_step=rng.random() < 0.2,
                      tau=0.8 if gated else -1.0, psaw=rng.random() < 0.2)
            if gated:
                c["per_step"] = False
    del c["name"]
    return c


# -- inputs ------------------------------------------------------------------

def _lengths(case, seed, steps):
    """Cached tokens before the first step: all n, or between n/2 and n."""
    n, b = case["n"], case["batch"]
    if not case["ragged"]:
        return (n,) * b
    gen = torch.Generator().manual_seed(seed * 2 + 1)
    x = torch.randint((n + 1) // 2, n - steps + 1, (b,), generator=gen).tolist()
    x[seed % b] = n - steps
    return tuple(int(v) for v in x)


def _workload(case, seed, steps):
    get = case.get
    return synth.Workload(
        "perf", case["dtype"], case["layers"], case["batch"], case["hq"], case["hkv"], case["d"],
        _lengths(case, seed, steps), steps, k=get("k", 0), window=get("window", 0),
        sink=get("sink", 0), s=get("s", 1), G=get("G", 1), r=get("r", 1), k_num=get("k_num", 0),
        k_den=get("k_den", 0), paged=case["paged"], page_size=case["page"], heavy=get("heavy", 8),
        heavy_tail=get("heavy_tail", False), layer_corr=get("layer_corr", 0.0), seed=seed)


def _steps(case):
    return case["s"] if case["kind"] == "decode" else 1


def _inputs(case, seed):
    return synth.generate(_workload(case, seed, _steps(case)), device=DEV)


def _prompt_queries(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 17)
    q = torch.randn(case["batch"], case["hq"], case["n"], case["d"], generator=gen, device=DEV)
    return (torch.clamp(torch.round(q * 16), -255, 255) / 16).to(torch.bfloat16)


def prepare(case, seed):
    inp = _inputs(case, seed)
    L, bt = case["layers"], case["batch"]
    if case["kind"] == "prefill":
        q = _prompt_queries(case, seed)
        lens = torch.tensor(inp.w.n_ctx, dtype=torch.int32, device=DEV)
        table = inp.block_table
        kv = B.KV(inp.K[0], inp.V[0], lens, case["n"], case["hq"], table)
        ps = None
        if case["psaw"]:
            l_s, phi, alpha = schedule.psaw_defaults(case["num_layers"])
            ps = B.psaw(case["psaw_layer"], case["num_layers"], l_s, phi, alpha, case["sink"])
        out = torch.zeros(q.shape, dtype=torch.float32, device=DEV)
        lse = torch.zeros(q.shape[:3], dtype=torch.float32, device=DEV)
        return {"case": case, "inp": inp, "kv": kv, "q": q, "ps": ps, "out": out, "lse": lse,
                "scale": 1.0 / math.sqrt(case["d"])}
    steps = _steps(case)
    out = torch.zeros(steps, L, bt, case["hq"], case["d"], dtype=torch.float32, device=DEV)
    lse = torch.zeros(steps, L, bt, case["hq"], dtype=torch.float32, device=DEV)
    outs = [[(out[j, l], lse[j, l]) for l in range(L)] for j in range(steps)]
    st = {"case": case, "inp": inp, "out": out, "lse": lse, "outs": outs, "graph": None}
    if case["kind"] == "dense":
        st["runner"] = schedule.DecodeRunner(inp, device=DEV)
        return st
    ps = schedule.psaw_defaults(L) if case["psaw"] else None
    if case["tau"] >= 0:
        r = schedule.GatedDecodeRunner(inp, device=DEV, tau=case["tau"], psaw=ps)
        st["sets"] = [r.choice, r.pool, r.pool_len]
    else:
        r = schedule.DecodeRunner(inp, device=DEV, per_step_sets=case["per_step"], psaw=ps)
        st["sets"] = [r.anchor_set, r.anchor_len, r.shared_set, r.shared_len]
    st["sets"] += [r.topk_idx, r.topk_len]
    st["runner"] = r
    if case["graph"]:
        st["graph"] = schedule.capture_steps(lambda j: r.step(j, outs[j]), range(steps))
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "prefill":
        B.prhs_prefill_attn(st["kv"], st["q"], st["scale"], st["out"], st["lse"], psaw=st["ps"])
        return [st["out"], st["lse"]]
    if case["kind"] == "dense":
        st["runner"].dense_step(0, st["outs"][0])
        return [st["out"], st["lse"]]
    if st["graph"] is not None:
        st["graph"].replay()
    else:
        for j in range(case["s"]):
            st["runner"].step(j, st["outs"][j])
    return [st["out"], st["lse"]] + st["sets"]


# -- what a pass cannot do without ---------------------------------------------

def _mean_len(case, power=1):
    """Mean over the batch of the cached lengths, or of their squares."""
    part = (1.0 if not case["ragged"] else 0.75 if power == 1 else 7 / 12) * (case["batch"] - 1)
    return (1.0 + part) / case["batch"] * float(case["n"]) ** power


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    bt, hq, hkv, d, L = case["batch"], case["hq"], case["hkv"], case["d"], case["layers"]
    n = _mean_len(case)
    if case["kind"] == "prefill":
        pairs = bt * hq * (_mean_len(case, 2) + n) / 2
        if case["psaw"]:
            l_s, phi, alpha = schedule.psaw_defaults(case["num_layers"])
            l = case["psaw_layer"] + 1
            f = 1 - phi ** (alpha * (l - l_s) / (case["num_layers"] - l_s)) if l > l_s else 0.0
            pairs *= 1 - f
        rows = bt * hq * case["n"]
        return {"bytes": 2 * bt * hkv * n * d * e + rows * d * (e + 4) + rows * 4,
                "flops": 4.0 * d * pairs}
    io = bt * hq * (d * e + (d + 1) * 4)   # query in, output and lse out
    if case["kind"] == "dense":
        return {"bytes": L * (2 * bt * hkv * n * d * e + io), "flops": L * 4.0 * bt * hq * n * d}
    k = int(case["k_num"] * n) // case["k_den"] if case["k_den"] else case["k"]
    mid = max(0.0, n - case["sink"] - case["window"])
    k = min(k, mid)
    crit = min(n, case["sink"] + k + case["window"])
    shared = min(n, crit + 2 * case["r"] * (k // 3) * 0.9)
    groups = -(-L // case["G"])
    s = case["s"]
    refreshes = groups * (s / 2 if case["tau"] >= 0 else 1)
    by = refreshes * bt * (hkv * (mid * d * e + (2 * k + crit + shared) * 4) + hq * d * e)
    fl = refreshes * 2.0 * bt * hq * mid * d
    rows = groups * crit + (s * L - groups) * shared
    by += bt * hkv * rows * (2 * d * e + 4) + s * L * io
    fl += 4.0 * bt * hq * rows * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # fp32 inputs: 32-bit sums in another order.  bf16 inputs: products are
    # exact, the probabilities keep about 16 bits as two bf16 parts and sums
    # are 32-bit.  About four times what the library is from 64 bits: 1.9e-7
    # and 2.4e-6.  Index sets are the same: scores of these inputs are exact
    # in 32 bits.
    return {"rel": 1e-6 if case["dtype"] == "f32" else 1e-5, "differ": 0.0}


# -- the same in 64 bits, in plain torch -----------------------------------------

def _unit_kv(inp, l, b, n):
    """K, V [Hkv][n][d] of sequence b in 64 bits."""
    if inp.block_table is None:
        return inp.K[l][b, :, :n].double(), inp.V[l][b, :, :n].double()
    ps = inp.w.page_size
    tab = inp.block_table[b, : (n + ps - 1) // ps].long()

    def rows(x):
        x = x[tab].permute(1, 0, 2, 3)
        return x.reshape(x.shape[0], -1, x.shape[3])[:, :n].double()
    return rows(inp.K[l]), rows(inp.V[l])


def _attend(q, K, V, mask, scale):
    """q [H][T][d], K, V [Hkv][n][d], mask broadcastable to [Hkv][G][T][n];
    out [H][T][d], lse [H][T]."""
    H, T, d = q.shape
    hkv, n, _ = K.shape
    x = torch.matmul(q.reshape(hkv, -1, d), K.transpose(1, 2).contiguous())
    x = x.reshape(hkv, H // hkv, T, n) * scale
    if mask is not None:
        x = x.masked_fill(~mask, -math.inf)
    lse = torch.logsumexp(x, dim=-1)
    p = torch.exp(x - lse.clamp_min(-1e300).unsqueeze(-1))
    o = torch.matmul(p.reshape(hkv, -1, n), V)
    return o.reshape(H, T, d), lse.reshape(H, T)


def _first_visible(case, layer, num_layers, n):
    """Start of the visible band, for n tokens in view (an int or a tensor)."""
    l_s, phi, alpha = (3 * num_layers) // 4, 0.7, 1.0
    l = layer + 1
    f = 1.0 - phi ** (alpha * (l - l_s) / (num_layers - l_s)) if l >= l_s else 0.0
    n = torch.as_tensor(n, dtype=torch.float64, device=DEV)
    return torch.maximum(n.clamp(max=case["sink"]), torch.floor(f * n) - 1).long()


def _exact_prefill(case, seed):
    inp = _inputs(case, seed)
    q = _prompt_queries(case, seed)
    T, scale = case["n"], 1.0 / math.sqrt(case["d"])
    out = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.full(q.shape[:3], -math.inf, dtype=torch.float64, device=DEV)
    for b, n in enumerate(inp.w.n_ctx):
        K, V = _unit_kv(inp, 0, b, n)
        step = max(16, (1 << 28) // (n * case["hq"]))
        for i0 in range(0, n, step):
            i1 = min(n, i0 + step)
            i = torch.arange(i0, i1, device=DEV)[:, None]
            p = torch.arange(i1, device=DEV)[None, :]
            mask = p <= i
            if case["psaw"]:
                vis = _first_visible(case, case["psaw_layer"], case["num_layers"], i + 1)
                mask &= (p < case["sink"]) | (p >= vis)
            o, s = _attend(q[b, :, i0:i1].double(), K[:, :i1], V[:, :i1], mask[None, None], scale)
            out[b, :, i0:i1], lse[b, :, i0:i1] = o, s
    return [out, lse]


def _sets(case, K, q, n0):
    """Critical and dilated shared set [Hkv][n0] (boolean) of one sequence."""
    hkv, hq = case["hkv"], case["hq"]
    dev = K.device
    se = min(case["sink"], n0)
    ws = max(se, n0 - case["window"])
    k = (case["k_num"] * n0) // case["k_den"] if case["k_den"] else case["k"]
    m, k = k // 3, min(k, ws - se)
    m = min(m, k)
    crit = torch.zeros(hkv, n0, dtype=torch.bool, device=dev)
    crit[:, :se] = True
    crit[:, ws:] = True
    shared = crit.clone()
    if k > 0:
        x = torch.matmul(q.reshape(hkv, hq // hkv, -1), K[:, se:ws].transpose(1, 2).contiguous())
        top = torch.sort(x.amax(1), dim=1, descending=True, stable=True)[1][:, :k] + se
        crit.scatter_(1, top, True)
        shared.scatter_(1, top, True)
        for delta in range(-case["r"], case["r"] + 1):
            shared.scatter_(1, (top[:, :m] + delta).clamp(0, n0 - 1), True)
    return crit, shared


def _exact_decode(case, seed):
    inp = _inputs(case, seed)
    w = inp.w
    steps, L, bt, hq, hkv = w.steps, case["layers"], case["batch"], case["hq"], case["hkv"]
    g, scale = hq // hkv, 1.0 / math.sqrt(case["d"])
    out = torch.zeros(steps, L, bt, hq, case["d"], dtype=torch.float64, device=DEV)
    lse = torch.zeros(steps, L, bt, hq, dtype=torch.float64, device=DEV)
    dense = case["kind"] == "dense"
    for b, n in enumerate(w.n_ctx):
        kept = []   # per retrieving step of the group: (q, units, crit, shared, n0)
        for l in range(L):
            first = not dense and l % case["G"] == 0
            K, V = _unit_kv(inp, l, b, n + steps)
            if first:
                kept, choice = [], []
                for j in range(steps):
                    q = inp.q[l, j, b].double()
                    pick = torch.full((hkv,), -1, dtype=torch.long, device=DEV)
                    if case["tau"] < 0:
                        if j > 0:
                            pick[:] = 0
                    else:
                        for i, (qi, units, *_) in enumerate(kept):
                            dot = (q * qi).sum(-1)
                            t2 = case["tau"] * case["tau"]
                            ok = (dot > 0) & (dot * dot > (t2 * (q * q).sum(-1)) * (qi * qi).sum(-1))
                            pick = torch.where(ok.reshape(hkv, g).all(1) & units, i, pick)
                    crit, shared = _sets(case, K[:, : n + j + 1], q, n + j + 1) \
                        if bool((pick < 0).any()) else (None, None)
                    kept.append((q, pick < 0, crit, shared, n + j + 1))
                    choice.append(pick)
            for j in range(steps):
                t = n + j + 1
                mask = None
                if not dense:
                    mask = torch.zeros(hkv, t, dtype=torch.bool, device=DEV)
                    for i in range(j + 1):
                        u = choice[j] < 0 if i == j else choice[j] == i
                        if not bool(u.any()):
                            continue
                        _, _, crit, shared, n0 = kept[i]
                        mask[u, :n0] = (crit if i == j and first else shared)[u]
                        mask[u, n0:] = True
                    if case["psaw"]:
                        p = torch.arange(t, device=DEV)
                        mask &= (p < case["sink"]) | (p >= _first_visible(case, l, L, t))
                    mask = mask[:, None, None]
                o, s = _attend(inp.q[l, j, b].double()[:, None], K[:, :t], V[:, :t], mask, scale)
                out[j, l, b], lse[j, l, b] = o[:, 0], s[:, 0]
    return [out, lse]


def exact(case, seed):
    """Outputs and log-sum-exp; the index sets of a decode block, which `run`
    returns after them, have no 64-bit value of their own."""
    if case["kind"] == "prefill":
        return _exact_prefill(case, seed)
    o = _exact_decode(case, seed)
    return o if case["kind"] == "dense" else o + [None] * (5 if case["tau"] >= 0 else 6)
