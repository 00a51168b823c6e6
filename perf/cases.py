"""The work that a program has this library do, as cases whose time is measured.

A case is one call pattern of the library's public entry points: a rollout from
its prompts to its last token, decode steps of a running batch, the prefill of a
new batch, a teacher-forced evaluation step, the loss of a finished batch.  The
model pairs are the repository's own workloads: "tiny" (float32), "small" (bf16,
head size 64) and "qwen" (the Qwen3-4B-shaped senior beside the
Qwen3-0.6B-shaped junior, bf16, head size 128, q/k norms), the last one at its
full depth once and otherwise at two layers of each model, as the parity tests
run it.  Weights are random at the scale of the workloads, prompts are uniform
token ids.
"""
import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_28166_amd import _lib as L
from paper_2606_28166_amd.engine import LAYER_KEYS, TandemEngine, grpo_loss, model_cfg

DEV = "cuda:0"
REDRAW, SWITCH, ALTERNATE = 0, 1, 2


def _shape(layers, d, nq, nkv, hd, ffn, vocab, qk_norm, dtype):
    return SimpleNamespace(n_layers=layers, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, ffn_dim=ffn,
                           vocab=vocab, rope_theta=1.0e6, rms_eps=1.0e-6, qk_norm=qk_norm, dtype=dtype)


def _shapes(case):
    """(senior, junior) of a case; junior None: the senior alone."""
    ls, lj, v = case["senior_layers"], case["junior_layers"], case["vocab"]
    if case["pair"] == "tiny":
        s = _shape(ls, 128, 4, 2, 32, 512, v, False, "f32")
        j = _shape(lj, 64, 2, 1, 32, 256, v, False, "f32")
    elif case["pair"] == "small":
        s = _shape(ls, 1024, 16, 4, 64, 4096, v, False, "bf16")
        j = _shape(lj, 512, 8, 2, 64, 2048, v, False, "bf16")
    else:
        s = _shape(ls, 2560, 32, 8, 128, 9728, v, True, "bf16")
        j = _shape(lj, 1024, 16, 8, 128, 3072, v, True, "bf16")
    return s, (j if lj else None)


_DEPTH = {"tiny": (2, 1, 512), "small": (8, 4, 32000), "qwen": (2, 2, 151936)}


def _case(kind, pair, prompts, group, prompt, **kw):
    ls, lj, v = _DEPTH[pair]
    c = dict(kind=kind, pair=pair, senior_layers=ls, junior_layers=lj, vocab=v, prompts=prompts, group=group,
             prompt=prompt, prompt_min=prompt, max_new=2048, steps=1, logits=False, prefill_rows=4096,
             mode=SWITCH, p=0.1, cap=-1, density=1.0, first=1, temperature=1.0, eos=False)
    c.update(kw)
    return c


def listed():
    return [
        # the float32 pair's whole rollout, four sequences: every launch is tiny, so latency and launches count
        dict(_case("rollout", "tiny", 1, 4, 16, max_new=32, p=0.2), name="tiny_rollout"),
        # decode of the small pair's ordinary batch, 64 rows
        dict(_case("decode", "small", 8, 8, 128, steps=16), name="small_decode"),
        # long chains of thought: ragged prompts, an EOS token (so the batch is compacted every 32 steps) and
        # ownership in 32-token chunks, 256 rows
        dict(_case("decode", "small", 32, 8, 512, prompt_min=64, steps=32, p=0.3, cap=31, density=0.0, eos=True),
             name="longcot_decode"),
        # the widest batch, 1024 rows, owners switching at every other token
        dict(_case("decode", "small", 64, 16, 256, steps=4, p=0.5), name="wide_decode"),
        # the benchmark's batch at full depth, 128 rows early in a rollout
        dict(_case("decode", "qwen", 16, 8, 256, max_new=1024, steps=2, senior_layers=36, junior_layers=28),
             name="qwen_decode"),
        # the same shapes late in a long response: 128 rows, each with a context of its own of over 2000 positions
        dict(_case("decode", "qwen", 128, 1, 2040, steps=2, max_new=1024, mode=REDRAW, p=0.5, cap=32, density=0.351,
                   first=2, temperature=0.6), name="qwen_long_decode"),
        # one sequence of one user, where only the weights' stream and latency count
        dict(_case("decode", "qwen", 1, 1, 512, steps=4, mode=ALTERNATE, density=0.0208, temperature=0.6),
             name="qwen_one_row_decode"),
        # the senior alone (the single-model baseline), a small batch
        dict(_case("decode", "qwen", 2, 8, 1000, steps=4, junior_layers=0), name="solo_decode"),
        # prefill of long prompts, read back through one teacher-forced step
        dict(_case("prefill", "qwen", 16, 1, 512, max_new=64, logits=True, prefill_rows=8192), name="qwen_prefill"),
        # prefill of ragged prompts in several passes, eight responses each
        dict(_case("prefill", "small", 32, 8, 512, prompt_min=40, max_new=64, logits=True), name="small_prefill"),
        # teacher-forced evaluation: both models' logits and the dual-distribution scores of a step, 128 rows
        dict(_case("teacher", "qwen", 16, 8, 256, logits=True, mode=REDRAW, p=0.5, cap=32, density=0.351, first=2,
                   temperature=0.6), name="qwen_teacher_score"),
        # the loss of a finished batch of the training schedule: 16 prompts x 8 responses of at most 3000 tokens
        dict(kind="grpo", groups=16, group=8, max_new=3000, clip=0.2, ratio=True, name="grpo_loss"),
    ]


def _log_int(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "teacher", "rollout", "grpo"])
    if kind == "grpo":
        groups, group = _log_int(rng, 1, 32), rng.choice([1, 4, 5, 8, 16])
        return dict(kind="grpo", groups=groups, group=group, max_new=_log_int(rng, 32, 4096), clip=0.2,
                    ratio=rng.random() < 0.8)
    if kind == "rollout":
        return _case("rollout", "tiny", rng.randint(1, 3), rng.randint(1, 8), _log_int(rng, 2, 80), max_new=32,
                     p=round(rng.uniform(0.0, 1.0), 3))
    pair = rng.choice(["small", "qwen"])
    longest = _log_int(rng, 17, 2040)
    opts = dict(prompt_min=longest if rng.random() < 0.5 else max(1, longest // rng.randint(2, 8)))
    opts.update(rng.choice([
        dict(mode=SWITCH, p=round(rng.uniform(0.05, 0.5), 3)),
        dict(mode=REDRAW, p=0.5, cap=32, density=0.351, first=2, temperature=0.6),
        dict(mode=ALTERNATE, density=0.0208, temperature=0.6)]))
    if rng.random() < 0.25:
        opts["junior_layers"] = 0
    if kind == "prefill":
        group = rng.choice([1, 4, 8])
        prompts = max(1, min(_log_int(rng, 1, 64), 16384 // longest, 128 // group))
        return _case("prefill", pair, prompts, group, longest, max_new=64, logits=True,
                     prefill_rows=rng.choice([2048, 4096, 8192]), **opts)
    group = rng.choice([1, 2, 4, 8, 16])
    if kind == "teacher":
        rows = _log_int(rng, 1, 160)
        return _case("teacher", pair, max(1, min(rows // group, 16384 // longest)), group, longest,
                     logits=rng.random() < 0.5, max_new=1024, **opts)
    rows = _log_int(rng, 1, 256 if pair == "qwen" else 1024)
    prompts = max(1, min(rows // group, 131072 // longest))
    if pair == "small" and rng.random() < 0.3:
        opts["eos"] = True
    return _case("decode", pair, prompts, group, longest, steps=rng.choice([1, 2, 4]), **opts)


# ------------------------------------------------------------------ inputs

def _weights(shape, gen):
    """Random weights at the workloads' scale (matrices N(0, 0.02), gains around 1)."""
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32
    d, hd, q = shape.d_model, shape.head_dim, (shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim

    def mat(n, k):
        return torch.empty((n, k), dtype=dt, device=DEV).normal_(0.0, 0.02, generator=gen)

    def gain(n):
        return torch.empty(n, dtype=torch.float32, device=DEV).normal_(1.0, 0.1, generator=gen)

    t = {"embed": mat(shape.vocab, d), "final_norm": gain(d), "lm_head": mat(shape.vocab, d)}
    for i in range(shape.n_layers):
        w = dict(attn_norm=gain(d), w_qkv=mat(q, d), w_o=mat(d, shape.n_q_heads * hd), ffn_norm=gain(d),
                 w_gate_up=mat(2 * shape.ffn_dim, d), w_down=mat(d, shape.ffn_dim))
        if shape.qk_norm:
            w.update(q_norm=gain(hd), k_norm=gain(hd))
        t.update({f"layers.{i}.{k}": v for k, v in w.items()})
    return t


class _Model:
    """Weights on the device and their descriptor, as TandemEngine(models=...) takes them."""

    def __init__(self, shape, tensors):
        self.shape, self.t = shape, tensors
        ptrs = [tensors[f"layers.{i}.{k}"].data_ptr() if f"layers.{i}.{k}" in tensors else 0
                for i in range(shape.n_layers) for k in LAYER_KEYS]
        self.layer_ptrs = (ctypes.c_void_p * len(ptrs))(*ptrs)
        self.desc = L.Model(model_cfg(shape), tensors["embed"].data_ptr(),
                            ctypes.cast(self.layer_ptrs, ctypes.POINTER(ctypes.c_void_p)),
                            tensors["final_norm"].data_ptr(), tensors["lm_head"].data_ptr())


def _generated(case, seed):
    """(senior weights, junior weights or None, prompts, boundary bits or None, forced tokens), from the seed alone."""
    sen, jun = _shapes(case)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    ws, wj = _weights(sen, gen), (_weights(jun, gen) if jun else None)
    rng = np.random.default_rng(seed)
    hi = case["vocab"] - 1                               # the last id is the EOS token where there is one
    lens = rng.integers(case["prompt_min"], case["prompt"] + 1, case["prompts"])
    prompts = [rng.integers(0, hi, n).astype(np.int32) for n in lens]
    bits = None
    if case["density"] < 1.0:
        words = np.zeros((case["vocab"] + 31) // 32, np.uint32)
        v = np.flatnonzero(rng.random(case["vocab"]) < case["density"])
        np.bitwise_or.at(words, v >> 5, np.left_shift(np.uint32(1), (v & 31).astype(np.uint32)))
        bits = words
    forced = rng.integers(0, hi, (case["prompts"] * case["group"], 64)).astype(np.int32)
    return ws, wj, prompts, bits, forced


def _grpo_inputs(case, seed):
    """Binary rewards whose success rate differs by group, ragged lengths, alternating authorship, recorded
    log-probs and the current policy's near them."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    s, t = case["groups"] * case["group"], case["max_new"]

    def uniform(*n):
        return torch.rand(*n, generator=g, device=DEV)

    rate = uniform(case["groups"], 1).expand(-1, case["group"]).reshape(-1)
    old = -torch.empty(s, t, device=DEV).exponential_(1.0, generator=g)
    new = old + torch.empty(s, t, device=DEV).normal_(0.0, 0.15, generator=g) if case["ratio"] else None
    return SimpleNamespace(rewards=(uniform(s) < rate).float(), owner=(uniform(s, t) < 0.5).to(torch.uint8),
                           length=torch.randint(0, t + 1, (s,), generator=g, device=DEV, dtype=torch.int32),
                           old=old, new=new)


def prepare(case, seed):
    if case["kind"] == "grpo":
        st = _grpo_inputs(case, seed)
        st.case = case
        st.workspace = torch.empty(L.tandem_grpo_workspace_size(
            L.GrpoCfg(case["groups"], case["group"], case["max_new"], case["clip"])), dtype=torch.uint8, device=DEV)
        return st
    ws, wj, prompts, bits, forced = _generated(case, seed)
    sen, jun = _shapes(case)
    switch = SimpleNamespace(mode=case["mode"], p=case["p"], cap_k=case["cap"], first_owner=case["first"])
    # the EOS biases are the long chain-of-thought workload's (a stop about every 4000 tokens)
    sample = SimpleNamespace(temperature=case["temperature"], eos_id=case["vocab"] - 1 if case["eos"] else -1,
                             eos_bias_senior=2.2608, eos_bias_junior=2.0414, max_new=case["max_new"])
    n = case["prompts"] * case["group"]
    eng = TandemEngine(None, None, None, None, switch, sample, seed, max_seqs=n,
                       max_ctx=case["prompt"] - 1 + case["max_new"], max_prefill_tokens=case["prefill_rows"],
                       boundary_words=bits, device=DEV, models=(_Model(sen, ws), _Model(jun, wj) if jun else None))
    st = SimpleNamespace(case=case, eng=eng, prompts=prompts, forced=forced, left=0, at=0, scores=None)
    if case["kind"] in ("decode", "teacher"):            # a batch that is under way
        eng.prefill(prompts, case["group"])
        st.left = case["max_new"]
    if case["kind"] == "teacher" and case["logits"] and jun:
        st.scores = torch.zeros((n, 3), dtype=torch.float32, device=DEV)
    return st


def _arenas(eng):
    return {"tokens": eng.tokens, "owner": eng.owner, "logprob": eng.logprob, "length": eng.length}


def run(st):
    c = st.case
    if c["kind"] == "grpo":
        return grpo_loss(st.rewards, st.owner, st.length, st.old, st.new, c["group"], c["clip"],
                         workspace=st.workspace)
    eng = st.eng
    if c["kind"] == "rollout":
        eng.prefill(st.prompts, c["group"])
        for _ in range(c["max_new"]):
            eng.step()
        return _arenas(eng)
    if c["kind"] == "prefill" or st.left < c["steps"]:   # a new batch, or the running one has reached its last token
        eng.prefill(st.prompts, c["group"])
        st.left, st.at = c["max_new"], 0
    st.left -= c["steps"]
    if c["kind"] == "decode":
        for _ in range(c["steps"]):
            eng.step()
        return _arenas(eng)
    # one teacher-forced step.  The library's own sample and its margin are left out: a near tie flips the sample,
    # and one of few rows is a large share
    dbg = eng.step_forced(st.forced[:, st.at % 64], debug=c["logits"], logits=c["logits"])
    st.at += 1
    out = _arenas(eng)
    out.update({k: dbg[k] for k in ("logits_senior", "logits_junior") if k in dbg})
    if c["junior_layers"] == 0:
        out.pop("logits_junior", None)
    if st.scores is not None:
        out["scores"] = eng.score(st.scores)
    return out


# ------------------------------------------------------- what a pass needs

def _layer_weights(s):
    q = (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim
    return s.d_model * (q + s.n_q_heads * s.head_dim + 3 * s.ffn_dim)


def work(case):
    """Weights once per forward, every attended K/V position once (a prompt shared by its responses once), the new
    K/V and the outputs written once."""
    if case["kind"] == "grpo":
        n = case["groups"] * case["group"] * case["max_new"]
        used = n / 2                                     # positions below the length, half of them the senior's
        return {"bytes": used * (1 + (8 if case["ratio"] else 4) / 2) + 4 * n, "flops": 10 * used}
    rows = case["prompts"] * case["group"]
    mean = (case["prompt"] + case["prompt_min"]) / 2
    steps = {"rollout": case["max_new"], "decode": case["steps"]}.get(case["kind"], 1)
    byt = flop = 0.0
    for s in _shapes(case):
        if s is None:
            continue
        e = 2 if s.dtype == "bf16" else 4
        lw, kv, att = _layer_weights(s), 2 * s.n_kv_heads * s.head_dim * e, 4 * s.n_q_heads * s.head_dim
        own = (steps + 1) / 2                            # positions a row has generated, on average over the steps
        byt += steps * (e * (s.n_layers * lw + s.vocab * s.d_model + rows * s.d_model)
                        + s.n_layers * kv * (case["prompts"] * mean + rows * own + rows))
        flop += steps * rows * (2 * (s.n_layers * lw + s.vocab * s.d_model) + s.n_layers * att * (mean + own))
        if case["kind"] in ("prefill", "rollout"):
            tok = case["prompts"] * (mean - 1)
            byt += e * s.n_layers * lw + tok * (s.n_layers * kv + e * s.d_model)
            flop += tok * s.n_layers * (2 * lw + att * mean / 2)
        if case["logits"]:
            byt += 4 * rows * s.vocab
    return {"bytes": byt + 13 * rows * steps, "flops": flop}


def tolerance(case):
    if case["kind"] == "grpo":
        return {"rel": 1e-5, "max": 1e-3}                # float32 sums; 7e-8 off 64 bits was seen
    if case["pair"] == "tiny":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}  # float32 throughout; 8e-8 was seen
    if case["kind"] == "decode":
        # a near tie that rounding decides gives the sequence another token and other tokens after it: their
        # log-probs (around -12) then differ by about 1.  One token in a few thousand is such a tie, and the 128
        # rows of the full-depth pair may hold several
        return {"rel": 2e-2, "max": 0.9, "differ": 5e-3}
    # logits of bf16 models (K/V rounded to bf16): 6e-4 to 8e-4 off 64 bits were seen
    return {"rel": 3e-3, "max": 0.03}


# ------------------------------------------------------------ in 64 bits

def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, theta):
    """x [positions][heads][hd], positions 0, 1, ..; dimension i is paired with i + hd / 2."""
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / (2 * half))
    a = torch.arange(x.shape[0], dtype=torch.float64, device=x.device)[:, None] * inv
    c, s = a.cos()[:, None], a.sin()[:, None]
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


def _last_logits(s, w, seqs):
    """Logits [len(seqs)][vocab] after the last token of each sequence, in float64; keys and values are kept in the
    model's own type."""
    lens, cuts = [len(x) for x in seqs], np.cumsum([0] + [len(x) for x in seqs])
    nq, nkv, hd = s.n_q_heads, s.n_kv_heads, s.head_dim
    keep = (lambda a: a.to(torch.bfloat16).double()) if s.dtype == "bf16" else (lambda a: a)
    h = w["embed"][torch.from_numpy(np.concatenate(seqs)).long().to(DEV)].double()
    for i in range(s.n_layers):
        p = {k: w.get(f"layers.{i}.{k}") for k in LAYER_KEYS}
        qkv = _norm(h, p["attn_norm"], s.rms_eps) @ p["w_qkv"].double().t().contiguous()
        att = torch.empty((h.shape[0], nq * hd), dtype=torch.float64, device=DEV)
        for a, n in zip(cuts, lens):
            q, k, v = qkv[a:a + n].view(n, -1, hd).split([nq, nkv, nkv], 1)
            if s.qk_norm:
                q, k = _norm(q, p["q_norm"], s.rms_eps), _norm(k, p["k_norm"], s.rms_eps)
            q, k, v = _rope(q, s.rope_theta), keep(_rope(k, s.rope_theta)), keep(v)
            mask = torch.ones((n, n), dtype=torch.bool, device=DEV).tril()
            for g in range(nkv):
                qg = q[:, g * nq // nkv:(g + 1) * nq // nkv].transpose(0, 1).contiguous()
                sc = (qg @ k[:, g].t().contiguous()) / math.sqrt(hd)
                o = sc.masked_fill(~mask, -math.inf).softmax(-1) @ v[:, g].contiguous()
                att[a:a + n, g * nq // nkv * hd:(g + 1) * nq // nkv * hd] = o.transpose(0, 1).reshape(n, -1)
        h = h + att @ p["w_o"].double().t().contiguous()
        gu = _norm(h, p["ffn_norm"], s.rms_eps) @ p["w_gate_up"].double().t().contiguous()
        h = h + (torch.nn.functional.silu(gu[:, :s.ffn_dim]) * gu[:, s.ffn_dim:]) @ p["w_down"].double().t().contiguous()
    last = _norm(h[torch.from_numpy(cuts[1:] - 1).to(DEV)], w["final_norm"], s.rms_eps)
    return last @ w["lm_head"].double().t().contiguous()


def _philox(block, t, s, stream, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of the counters (block, t, s, stream): all four words, [..., 4]."""
    m = (1 << 32) - 1
    c = [np.asarray(block, np.uint64), np.uint64(t), np.uint64(s), np.uint64(stream)]
    k0, k1 = seed & m, seed >> 32
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & np.uint64(m),
             (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & np.uint64(m)]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return np.stack(np.broadcast_arrays(*c), -1)


def _rollout_logprobs(case, seed, sen, jun, ws, wj, prompts):
    """The free-running rollout in 64 bits: the log-prob arena (float32 pairs, where near ties do not arise)."""
    v, steps = case["vocab"], case["max_new"]
    seqs = [p for p in prompts for _ in range(case["group"])]
    owner = [1] * len(seqs)
    out = torch.zeros((len(seqs), steps), dtype=torch.float64, device=DEV)
    for t in range(1, steps + 1):
        zs, zj = _last_logits(sen, ws, seqs), _last_logits(jun, wj, seqs)
        lp = torch.log_softmax(zs / case["temperature"], -1)
        for s in range(len(seqs)):
            x = _philox(np.arange((v + 3) // 4), t, s, 0, seed).reshape(-1)[:v]
            u = ((x >> np.uint64(9)) * np.uint64(2) + np.uint64(1)).astype(np.float64) * 2.0 ** -24
            z = (zs if owner[s] else zj)[s].cpu().numpy() / case["temperature"]
            y = int(np.argmax(z - np.log(-np.log(u))))
            out[s, t - 1] = lp[s, y]
            seqs[s] = np.append(seqs[s], np.int32(y))
            coin = int(_philox(0, t, s, 1, seed).reshape(-1)[0]) < int(case["p"] * 4294967296.0)
            owner[s] = 1 - owner[s] if coin else owner[s]        # SWITCH, every token a boundary
    return out


def exact(case, seed):
    if case["kind"] == "grpo":
        st = _grpo_inputs(case, seed)
        s, t = st.owner.shape
        r = st.rewards.double().view(case["groups"], case["group"])
        sd = r.std(1, keepdim=True) if case["group"] > 1 else torch.zeros_like(r[:, :1])
        adv = ((r - r.mean(1, keepdim=True)) / (sd + 1e-6)).reshape(-1)
        mask = (torch.arange(t, device=DEV)[None] < st.length[:, None]) & (st.owner != 0)
        old = st.old.double()
        rho = torch.exp((st.new.double() if st.new is not None else old) - old)
        un, cl = rho * adv[:, None], rho.clamp(1 - case["clip"], 1 + case["clip"]) * adv[:, None]
        n = int(mask.sum())
        loss = -(torch.minimum(un, cl) * mask).sum().reshape(1) / max(n, 1)
        grad = torch.where(mask & (un <= cl), -un / max(n, 1), torch.zeros_like(un))
        return {"advantages": adv, "loss": loss, "grad": grad}
    if case["kind"] == "decode":
        return None                # the tokens that the path drew decide what follows
    sen, jun = _shapes(case)
    ws, wj, prompts, _, forced = _generated(case, seed)
    if case["kind"] == "rollout":
        return {"logprob": _rollout_logprobs(case, seed, sen, jun, ws, wj, prompts)}
    # one step from the prompts: the responses of a prompt have its logits in common
    g = case["group"]
    z = {"logits_senior": _last_logits(sen, ws, prompts).repeat_interleave(g, 0)}
    if jun:
        z["logits_junior"] = _last_logits(jun, wj, prompts).repeat_interleave(g, 0)
    n = case["prompts"] * g
    y = torch.from_numpy(forced[:, 0]).long().to(DEV)
    out = {"logprob": torch.zeros((n, case["max_new"]), dtype=torch.float64, device=DEV)}
    lp = torch.log_softmax(z["logits_senior"] / case["temperature"], -1)
    out["logprob"][:, 0] = lp.gather(1, y[:, None])[:, 0]
    if case["logits"]:
        out.update(z)
    if case["kind"] == "teacher" and case["logits"] and jun:
        ps, pj = torch.log_softmax(z["logits_senior"], -1), torch.log_softmax(z["logits_junior"], -1)
        out["scores"] = torch.stack([-pj.gather(1, y[:, None])[:, 0], torch.minimum(ps, pj).exp().sum(1),
                                     (ps.exp() * (ps - pj)).sum(1)], 1)
    return out
