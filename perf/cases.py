"""The work a serving program has this library do, as cases to measure: prefill batches, decode steps and both at once on
a CU split, through `paper_2504_19516_amd.sts.Engine`, on the model shapes of `paper_2504_19516_amd.synth`.

A case is a stack of `layers` decoder layers of one model shape with an LM head of `vocab` rows, weights drawn on the device
from the seed, KV pages handed out in random order, cached contexts filled with the library's synthetic deviates. `run` is
one call of the step and returns the logits it computed (and the greedy tokens of a decode step). The sequences are rolled
back to their drawn lengths after each pass, as the benchmark does, so that a pass can be repeated.

`exact` recomputes the logits in 64 bits with plain torch: the weights and cached contexts come from the documented
counter-based recipe, written out again here.
"""
import math

import numpy as np
import torch

from paper_2504_19516_amd import sts, synth

PAGE = 16
MIN_TOKENS = 16          # greedy tokens are compared from this many requests up: of a few, one near tie would be a large share
PROFILES = {"8b": "paper_2504_19516_amd/data/mi355x_llama8b.profile", "70b": "paper_2504_19516_amd/data/mi355x_llama70b.profile"}


# ------------------------------------------------------------------------------------------ the cases
def _case(name, model, layers, vocab, prompts="", priors="", batch=0, ctx=0, spread=0.0, prefill_cus=256, decode_cus=256):
    """prompts: new tokens of each sequence of the prefill batch, comma separated; priors: tokens each of them has cached.
    batch: decode requests, their contexts lognormal with median `ctx` and sigma `spread` (cap 16384)."""
    c = dict(model=model, layers=layers, vocab=vocab, prompts=prompts, priors=priors, batch=batch, ctx=ctx, spread=spread,
             prefill_cus=prefill_cus, decode_cus=decode_cus)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the small parity configuration: launches and host time decide
        _case("tiny_step", "tiny", 2, 1024, prompts="128", batch=8, ctx=128, spread=0.5, prefill_cus=128, decode_cus=128),
        # one user's token: the weights of every layer, nothing to share them with
        _case("decode_1", "8b", 4, 1024, batch=1, ctx=1031),
        # the benchmark's decode batch on the whole GPU (no prompt waiting)
        _case("decode_64", "8b", 8, 1024, batch=64, ctx=1024, spread=0.8),
        # a large conversational batch, an odd one (past capacity the serving runs hold 200 and more requests)
        _case("decode_223", "8b", 4, 1024, batch=223, ctx=500, spread=0.9),
        # most live prefill batches are one prompt of a few hundred tokens
        _case("prefill_301", "8b", 2, 1024, prompts="301"),
        # a ragged batch of waiting prompts
        _case("prefill_ragged", "8b", 2, 1024, prompts="613,97,1201,35,744,1290"),
        # one chunk of a long document: 1024 tokens over 15 000 cached ones
        _case("prefill_chunk", "8b", 2, 1024, prompts="1024", priors="15000"),
        # the longest conversational prompt, in one pass
        _case("prefill_8192", "8b", 2, 1024, prompts="8192"),
        # the benchmark's step: a 2048-token chunk beside 64 decodes, 224 / 32 CUs
        _case("concurrent", "8b", 2, 1024, prompts="2048", batch=64, ctx=1024, spread=0.8, prefill_cus=224, decode_cus=32),
        # the larger shape: groups of eight query heads, hidden 8192, MLP 28672
        _case("decode_70b", "70b", 2, 1024, batch=24, ctx=900, spread=0.8),
        _case("prefill_70b", "70b", 2, 1024, prompts="700"),
        # the whole 32-layer model at its real vocabulary, a handful of users: logits and greedy tokens of one decode step
        _case("model_8b", "8b", 32, 128256, batch=4, ctx=600, spread=0.9),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    model = rng.choice(["8b"] * 7 + ["70b"] * 2 + ["tiny"])
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "concurrent"])
    top = {"tiny": 8192, "8b": 8192, "70b": 2000}[model]
    layers = 2 if model != "8b" or kind != "decode" else rng.choice([2, 4, 6])
    prompts, priors, batch, ctx, spread, pm, dm = "", "", 0, 0, 0.0, 256, 256
    if kind != "decode":
        total = _log_int(rng, 16, top if kind == "prefill" else top // 2)
        n = rng.randint(1, max(1, min(6, total // 16)))
        cuts = sorted(rng.sample(range(1, total), n - 1)) if n > 1 else []
        lens = [b - a for a, b in zip([0] + cuts, cuts + [total])]
        prompts = ",".join(map(str, lens))
        if n == 1 and total <= 2048 and rng.random() < 0.4:
            priors = str(_log_int(rng, 16, 15000))
    if kind != "prefill":
        batch = _log_int(rng, 1, 256)
        ctx = _log_int(rng, 64, min(8192, max(65, 120000 // batch)))
        spread = rng.choice([0.3, 0.8])
    if kind == "concurrent":
        pm = rng.choice([128, 192, 224])
        dm = 256 - pm
    return _case(None, model, layers, 1024, prompts, priors, batch, ctx, spread, pm, dm)


# ------------------------------------------------------------------------------------------ inputs
def _desc(case):
    n, v = case["layers"], case["vocab"]
    if case["model"] == "tiny":
        d = synth.tiny_model("bf16")
        assert (d.n_layers, d.vocab) == (n, v)
        return d
    return synth.llama8b_model(n, v) if case["model"] == "8b" else synth.llama70b_model(n, v)


def _ints(text):
    return [int(x) for x in text.split(",")] if text else []


def _inputs(case, seed):
    """Sizes and tokens of the step, from the seed alone."""
    rng = np.random.default_rng([int(seed), 71])
    lens = _ints(case["prompts"])
    priors = _ints(case["priors"]) or [0] * len(lens)
    # contexts are drawn once for a case, whatever the seed: every seed then is the same amount of work
    fixed = np.random.default_rng(97).normal(0.0, 1.0, size=case["batch"])
    ctx = np.clip(np.floor(max(1, case["ctx"]) * np.exp(fixed * case["spread"])), 1, 16384).astype(int).tolist()
    tok = [rng.integers(0, case["vocab"], n, dtype=np.int32) for n in lens]
    dtok = rng.integers(0, case["vocab"], case["batch"], dtype=np.int32)
    return dict(lens=lens, priors=priors, ctx=ctx, tokens=tok, dtokens=dtok, wseed=1000 + int(seed),
                kv_seeds=[(int(seed) * 4096 + 17 + i) for i in range(len(lens) + case["batch"])])


def prepare(case, seed):
    desc, x = _desc(case), _inputs(case, seed)
    need = [(p + n + PAGE) // PAGE for p, n in zip(x["priors"], x["lens"])] + [(c + 1 + PAGE) // PAGE for c in x["ctx"]]
    pool = sum(need) + 64
    eng = sts.Engine(desc, weight_seed=x["wseed"], init_weights=True, kv_pool_pages=pool, max_prefill_tokens=max(64, sum(x["lens"])),
                     max_prefill_seqs=max(1, len(x["lens"])), max_decode_batch=max(1, case["batch"]), max_seqs=len(need) + 2,
                     max_pages_per_seq=max(need) + 8)
    if case["model"] in PROFILES:                  # the rates measured on this part, as the serving loop hands them over
        prof = sts.Profile(path=PROFILES[case["model"]])
        eng.set_tile_model(*prof.tile_model())
        eng.set_stream_model(*prof.stream_model())
    eng.set_partition(case["prefill_cus"], case["decode_cus"])
    perm = np.random.default_rng([int(seed), 72]).permutation(pool).astype(np.int32)
    seqs, off = [], 0
    for n_pages, cached, kv_seed in zip(need, x["priors"] + x["ctx"], x["kv_seeds"]):
        s = eng.seq_create()
        eng.seq_set_block_table(s, perm[off:off + n_pages])
        off += n_pages
        if cached:
            eng.kv_fill_random(s, cached, kv_seed)
        seqs.append(s)
    k = len(x["lens"])
    return dict(eng=eng, layers=desc.n_layers, pseqs=seqs[:k], priors=x["priors"], tokens=x["tokens"], dseqs=seqs[k:], ctx=x["ctx"],
                dtokens=x["dtokens"])


def run(state):
    e, out = state["eng"], {}
    if state["pseqs"] and state["dseqs"]:
        out["prefill"], out["decode"], out["next"] = e.step_concurrent(state["pseqs"], state["tokens"], 0, state["layers"], state["dseqs"],
                                                                       state["dtokens"])
    elif state["pseqs"]:
        out["prefill"] = e.prefill_batch(state["pseqs"], state["tokens"])
    else:
        out["decode"], out["next"] = e.decode_step(state["dseqs"], state["dtokens"])
    if len(state["dseqs"]) < MIN_TOKENS:
        out.pop("next", None)
    for s, n in zip(state["pseqs"], state["priors"]):
        e.seq_truncate(s, n)
    for s, n in zip(state["dseqs"], state["ctx"]):
        e.seq_truncate(s, n)
    return out


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    d, x = _desc(case), _inputs(case, 0)
    qd, kvd = d.n_q_heads * d.head_dim, d.n_kv_heads * d.head_dim
    layer = (qd + 2 * kvd) * d.hidden + d.hidden * qd + 3 * d.mlp * d.hidden          # weights of one layer
    new = sum(x["lens"]) + case["batch"]
    heads = len(x["lens"]) + case["batch"]                                            # rows of logits
    cached = sum(x["priors"]) + sum(x["ctx"])
    pairs = sum(n * p + n * (n + 1) // 2 for n, p in zip(x["lens"], x["priors"])) + sum(c + 1 for c in x["ctx"])
    phases = (1 if x["lens"] else 0) + (1 if case["batch"] else 0)                    # each phase reads the weights for itself
    flops = d.n_layers * (2.0 * new * layer + 4.0 * qd * pairs) + 2.0 * heads * d.vocab * d.hidden
    nbytes = (phases * 2.0 * (d.n_layers * layer + d.vocab * d.hidden) + d.n_layers * 4.0 * kvd * (cached + new)
              + 4.0 * new + 2.0 * new * d.hidden + 4.0 * heads * d.vocab)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 weights, activations and probabilities, fp32 sums and residual stream; rounding adds up over the layers. Measured
    distance of the logits from the 64-bit ones, 2-norm: 0.004 on the tiny shape, 0.008 to 0.014 on one to four large layers,
    0.015 on eight. The bounds are about four times that, the largest single difference five times the norm's. `differ` is for
    greedy tokens whose two best logits lie closer than the rounding (3 to 5 % of the rows)."""
    rel = 1.6e-2 if case["model"] == "tiny" else 5e-2 if case["layers"] <= 4 else 6e-2 if case["layers"] <= 8 else 1.2e-1
    return {"rel": rel, "max": 5 * rel, "differ": 0.2}


# ------------------------------------------------------------------------------------------ the same step in 64 bits
def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _mix_int(z):
    m = (1 << 64) - 1
    z = (z + 0x9E3779B97F4A7C15) & m
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def _mix(z):
    """The same on int64 tensors (products wrap, shifts are made logical)."""
    z = z + _i64(0x9E3779B97F4A7C15)
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _i64(0x94D049BB133111EB)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _deviates(seed, tid, start, count, dev):
    """Elements [start, start + count) of a stream: sums of twelve 16-bit fields, centred (int64)."""
    base = _i64(_mix_int((seed ^ _mix_int(tid)) & ((1 << 64) - 1)))
    out = torch.empty(count, dtype=torch.int32, device=dev)
    step = 1 << 25
    for a in range(0, count, step):
        n = min(step, count - a)
        i4 = torch.arange(start + a, start + a + n, dtype=torch.int64, device=dev) * 4
        acc = torch.full((n,), -393210, dtype=torch.int64, device=dev)
        for j in range(3):
            r = _mix((i4 + j) ^ base)
            for sh in (0, 16, 32, 48):
                acc += (r >> sh) & 0xFFFF
        out[a:a + n] = acc.to(torch.int32)
    return out


def _weight(desc, seed, name, layer, dev):
    r, c = desc.shape(name)
    slots = {"wq": 0, "wk": 1, "wv": 2, "wo": 3, "wg": 4, "wu": 5, "wd": 6}
    tid = {"emb": 0, "lm": 1}[name] if name in ("emb", "lm") else (layer + 1) * 16 + slots[name]
    w = _deviates(seed, tid, 0, r * c, dev).to(torch.float32) * torch.tensor(0.02, dtype=torch.float32, device=dev)
    return (w * 2.0 ** -16).to(torch.bfloat16).to(torch.float64).reshape(r, c)


def _cached(desc, seed, layer, n, dev):
    """K and V of positions [0, n) of a synthetic context: [n, n_kv, d] each."""
    per = desc.n_kv_heads * desc.head_dim
    return [(_deviates(seed, 0x4B000000 + 2 * layer + i, 0, n * per, dev).to(torch.float32) * 2.0 ** -16).to(torch.bfloat16)
            .to(torch.float64).reshape(n, desc.n_kv_heads, desc.head_dim) for i in (0, 1)]


def _norm(x, eps):
    return x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + eps)


def _rope(x, pos, theta):
    """x: [rows, heads, d], element i turns with element i + d / 2."""
    half = x.shape[2] // 2
    f = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[2])
    a = pos.to(torch.float64)[:, None] * f[None, :]
    cs, sn = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    p, q = x[:, :, :half], x[:, :, half:]
    return torch.cat([p * cs - q * sn, p * sn + q * cs], dim=2)


def _attend(q, k, v, prior):
    """q: [t, n_q, d] at positions prior ..; k, v: [prior + t, n_kv, d]. Causal."""
    t, n_q, d = q.shape
    g = n_q // k.shape[1]
    out = torch.empty_like(q)
    hidden = torch.arange(k.shape[0], device=q.device)[None, :] > prior + torch.arange(t, device=q.device)[:, None]
    for h in range(n_q):
        s = (q[:, h].contiguous() @ k[:, h // g].t().contiguous()) / math.sqrt(d)
        s.masked_fill_(hidden, -math.inf)
        out[:, h] = torch.softmax(s, dim=1) @ v[:, h // g].contiguous()
    return out


def exact(case, seed):
    d, x = _desc(case), _inputs(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if d.n_layers > 8:
        return None                                # the whole model takes too long in 64 bits
    pieces = [(n, p) for n, p in zip(x["lens"], x["priors"])] + [(1, c) for c in x["ctx"]]
    tokens = torch.from_numpy(np.concatenate(x["tokens"] + [x["dtokens"]]).astype(np.int64)).to(dev)
    pos = torch.cat([torch.arange(p, p + n, device=dev) for n, p in pieces])
    X = _weight(d, x["wseed"], "emb", None, dev)[tokens]
    rows = X.shape[0]
    for layer in range(d.n_layers):
        W = lambda name: _weight(d, x["wseed"], name, layer, dev).t().contiguous()  # noqa: E731
        xn = _norm(X, d.rms_eps)
        q = _rope((xn @ W("wq")).reshape(rows, d.n_q_heads, d.head_dim), pos, d.rope_theta)
        k = _rope((xn @ W("wk")).reshape(rows, d.n_kv_heads, d.head_dim), pos, d.rope_theta)
        v = (xn @ W("wv")).reshape(rows, d.n_kv_heads, d.head_dim)
        a, r0 = torch.empty_like(q), 0
        for (n, p), kv_seed in zip(pieces, x["kv_seeds"]):
            kk, vv = k[r0:r0 + n], v[r0:r0 + n]
            if p:
                ck, cv = _cached(d, kv_seed, layer, p, dev)
                kk, vv = torch.cat([ck, kk]), torch.cat([cv, vv])
            a[r0:r0 + n] = _attend(q[r0:r0 + n], kk, vv, p)
            r0 += n
        X = X + a.reshape(rows, -1) @ W("wo")
        xn = _norm(X, d.rms_eps)
        X = X + (torch.nn.functional.silu(xn @ W("wg")) * (xn @ W("wu"))) @ W("wd")
    last = torch.tensor(np.cumsum([n for n, _ in pieces]) - 1, device=dev)
    logits = (_norm(X[last], d.rms_eps) @ _weight(d, x["wseed"], "lm", None, dev).t().contiguous()).cpu().numpy()
    k, out = len(x["lens"]), {}
    if k:
        out["prefill"] = logits[:k]
    if case["batch"]:
        out["decode"] = logits[k:]
        if case["batch"] >= MIN_TOKENS:
            out["next"] = None
    return out
