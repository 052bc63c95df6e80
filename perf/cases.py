"""What a user of this library has it do, as measured cases: drafting, pre-verification, verification, acceptance and
prompt ingestion through the C ABI's binding, over the sizes and types of the synthetic workloads.

Models are Llama-shaped with random weights (N(0, 0.02^2), gains 1 + 0.1 N(0, 1)), as wide as the workloads' own; most
target models are cut to a few layers, which leaves every launch what it is in the full model.  Token ids are uniform.
"""
import math

import numpy as np
import torch

from paper_2602_01274_amd import binding as B
from paper_2602_01274_amd.engine import Session

# d_model, n_heads, head_dim, d_ffn, vocab, n_layers of the workloads' models
TARGETS = {"mid": (768, 12, 64, 2048, 32000, 12), "7b": (4096, 32, 128, 11008, 32000, 32),
           "13b": (5120, 40, 128, 13824, 32000, 40), "33b": (7168, 56, 128, 19200, 32256, 54),
           "tiny": (256, 4, 64, 688, 1024, 4)}
DRAFTS = {"mid": (768, 12, 64, 2048, 32000, 2), "7b": (768, 12, 64, 3072, 32000, 2), "13b": (768, 12, 64, 3072, 32000, 2),
          "33b": (2048, 16, 128, 5504, 32256, 24), "tiny": (256, 4, 64, 688, 1024, 1)}
THETA, EPS = 1e4, 1e-5
RNG_SEED, STEP = 20240817, 3


def _case(kind, pair, **kw):
    c = dict(kind=kind, pair=pair, layers=1, seqs=1, ctx=512, ctx_hi=512, gamma=4, block=4, sample=True)
    c.update(kw)
    c["ctx_hi"] = max(c["ctx"], c["ctx_hi"]) if c["seqs"] > 1 else c["ctx"]
    return c


def listed():
    return [
        # one round of the drafting loop at batch 1 (68M draft): four draft tokens, one pre-verification block, its flag
        dict(_case("round", "7b", ctx=530), name="draft_round_68m"),
        # one draft token for each of 16 sequences of different lengths
        dict(_case("draft", "13b", seqs=16, ctx=256, ctx_hi=2048), name="draft_step_68m_batch16"),
        # one draft token of the 1.35B draft model, batch 1
        dict(_case("draft", "33b", ctx=640), name="draft_step_1b"),
        # a short window's verification at batch 1, 7B width
        dict(_case("verify", "7b", layers=8, ctx=600, gamma=8), name="verify_7b_9rows"),
        # the whole 7B-shaped target with a full window, which is the headline workload's most frequent pass
        dict(_case("verify", "7b", layers=32, ctx=515, gamma=16), name="verify_7b_full_17rows"),
        # verification at long context
        dict(_case("verify", "7b", layers=8, ctx=4100, gamma=12), name="verify_7b_long"),
        # ragged verification of 16 sequences, 13B width
        dict(_case("verify", "13b", layers=4, seqs=16, ctx=256, ctx_hi=2048, gamma=16), name="verify_13b_batch16"),
        # the mid pair's whole target: small matrices, many launches
        dict(_case("verify", "mid", layers=12, ctx=200, gamma=12), name="verify_mid"),
        # a request's start: prompt ingestion and the first round of drafts with its verification, 7B width
        dict(_case("prompt", "7b", layers=4, ctx=512), name="prompt_7b_512"),
        # the same for a long prompt
        dict(_case("prompt", "7b", layers=4, ctx=4001), name="prompt_7b_4001"),
        # acceptance of a full window by sampling, on logits that the caller holds
        dict(_case("accept", "7b", gamma=16, sample=True), name="accept_16"),
        # the f32 pair: a drafting round of two, then verification
        dict(_case("step", "tiny", layers=4, ctx=33, gamma=2, block=2, sample=False), name="tiny_f32_step"),
    ]


def _loguniform(rng, lo, hi):
    return min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    cap = [max(work(c)[k] for c in listed()) for k in ("flops", "bytes")]
    while True:
        kind = rng.choice(["round", "draft", "draft", "verify", "verify", "verify", "prompt", "prompt", "accept", "step"])
        if kind == "round":
            b = rng.choice([1, 2, 3, 4, 5, 8])
            c = _case(kind, rng.choice(["mid", "7b"]), ctx=_loguniform(rng, 8, 4200), block=b, gamma=b)
        elif kind == "draft":
            n = rng.choice([1, 1, 2, 3, 5, 8, 11, 16])
            c = _case(kind, rng.choice(["mid", "7b", "33b"]), seqs=n, ctx=_loguniform(rng, 8, 2100), ctx_hi=_loguniform(rng, 8, 2100))
        elif kind == "verify":
            pair = rng.choice(["mid", "7b", "13b", "33b"])
            n = rng.choice([1, 1, 1, 2, 3, 6, 11, 16])
            hi = 4200 if n == 1 else 2100
            c = _case(kind, pair, layers=rng.randint(2, 12) if pair == "mid" else rng.randint(1, 4), seqs=n,
                      ctx=_loguniform(rng, 8, hi), ctx_hi=_loguniform(rng, 8, hi), gamma=rng.randint(1, 20))
        elif kind == "prompt":
            c = _case(kind, rng.choice(["mid", "7b", "13b"]), layers=rng.randint(1, 4), ctx=_loguniform(rng, 2, 4100))
        elif kind == "accept":
            c = _case(kind, "7b", gamma=rng.randint(1, 31), sample=rng.random() < 0.6)
        else:
            b = rng.choice([1, 2, 4])
            c = _case(kind, "tiny", layers=rng.randint(1, 4), ctx=_loguniform(rng, 4, 900), gamma=b, block=b, sample=False)
        w = work(c)
        if w["flops"] <= cap[0] and w["bytes"] <= cap[1]:
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _shape(t, layers=None):
    d, h, hd, f, v, n = t
    return dict(n_layers=n if layers is None else layers, d_model=d, n_heads=h, head_dim=hd, d_ffn=f, vocab=v, rope_theta=THETA, rms_eps=EPS)


def _lengths(case):
    """Committed tokens of each sequence, spread over [ctx, ctx_hi]."""
    n, lo, hi = case["seqs"], case["ctx"], case["ctx_hi"]
    return [lo + (hi - lo) * ((7 * i + 3) % n) // max(1, n - 1) for i in range(n)] if n > 1 else [lo]


def _gammas(case):
    """Drafts verified for each sequence: the whole window alone, windows of one to four quarters of it in a batch."""
    n, g = case["seqs"], case["gamma"]
    return [g] if n == 1 else [max(1, g * (1, 2, 3, 1, 4, 2, 3, 1, 2, 3, 1, 2, 4, 1, 2, 3)[i % 16] // 4) for i in range(n)]


def _bf16(case):
    return case["pair"] != "tiny"


class _Weights:
    """Seeded weights, made on the GPU in the order they are asked for."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
        self.store = torch.bfloat16 if _bf16(case) else torch.float32
        ts, ds = _shape(TARGETS[case["pair"]], case["layers"]), _shape(DRAFTS[case["pair"]])
        share = case["pair"] in ("mid", "tiny")
        self.target = self.lm(ts)
        self.draft = self.lm(ds, self.target if share else None)
        d = ds["d_model"]
        pe = torch.randn((32, d), generator=self.g, device="cuda") * 0.02
        pe[0] = 0
        self.mb = dict(layer=self.layer(ds), final_norm=self.gain(d), cls=torch.randn((2, d), generator=self.g, device="cuda") * 1.5 / (2 * d) ** 0.5,
                       posemb=pe)

    def mat(self, n, k):
        return torch.empty((n, k), dtype=self.store, device="cuda").normal_(0.0, 0.02, generator=self.g)

    def gain(self, d):
        return 1 + 0.1 * torch.randn(d, generator=self.g, device="cuda")

    def layer(self, s):
        d, f = s["d_model"], s["d_ffn"]
        return dict(attn_norm=self.gain(d), wq=self.mat(d, d), wk=self.mat(d, d), wv=self.mat(d, d), wo=self.mat(d, d), ffn_norm=self.gain(d),
                    wg=self.mat(f, d), wu=self.mat(f, d), wd=self.mat(d, f))

    def lm(self, s, share=None):
        w = dict(layers=[self.layer(s) for _ in range(s["n_layers"])])
        w["embed"], w["head"] = (share["embed"], share["head"]) if share else (self.mat(s["vocab"], s["d_model"]), self.mat(s["vocab"], s["d_model"]))
        w["final_norm"] = self.gain(s["d_model"])
        return w


def _tokens(case, seed):
    """Prompts (one list of ids per sequence) and draft ids."""
    r = np.random.default_rng(seed * 104729 + 5)
    v = TARGETS[case["pair"]][4]
    return [r.integers(0, v, n).astype(np.int32) for n in _lengths(case)], [r.integers(0, v, 32).astype(np.int32) for _ in range(case["seqs"])]


def _accept_inputs(case, seed):
    """Draft and target logits of a window, and the drafts: the two models agree in part, as in speculative decoding."""
    g = torch.Generator(device="cuda").manual_seed(seed * 6007 + 1)
    v, k = TARGETS[case["pair"]][4], case["gamma"]
    ld = torch.randn((k + 1, v), generator=g, device="cuda") * 1.5
    lt = ld + 0.3 * torch.randn((k + 1, v), generator=g, device="cuda")
    y = (ld[:k] - torch.log(-torch.log(torch.rand((k, v), generator=g, device="cuda").clamp_(1e-30, 1 - 1e-7)))) if case["sample"] else ld[:k]
    return lt, ld, y.argmax(1).to(torch.int32)


def prepare(case, seed):
    if case["kind"] == "accept":
        lt, ld, y = _accept_inputs(case, seed)
        return dict(case=case, lt=lt, ld=ld, y=y, n=torch.zeros(1, dtype=torch.int32, device="cuda"), z=torch.zeros(1, dtype=torch.int32, device="cuda"),
                    stream=torch.cuda.current_stream().cuda_stream)
    w = _Weights(case, seed)
    block = case["block"]
    gmax = max(1, max(_gammas(case)), case["gamma"])
    gmax = min(31 // block, -(-gmax // block)) * block
    desc = dict(target=_shape(TARGETS[case["pair"]]), draft=_shape(DRAFTS[case["pair"]]), dtype="bf16" if _bf16(case) else "f32", block=block,
                gamma_max=gmax, beta=3.0, t0=0.5, rho=1.05)
    w.mb["posemb"] = w.mb["posemb"][:gmax + 1]
    prompts, drafts = _tokens(case, seed)
    s = Session(desc, w.target, w.draft, w.mb, max_seq=max(map(len, prompts)) + gmax + 40, max_batch=case["seqs"])
    del w
    prompts = [torch.from_numpy(p).cuda() for p in prompts]
    ids = list(range(case["seqs"]))
    if case["kind"] != "prompt":
        for i, p in zip(ids, prompts):
            B.pacer_prefill(s.ctx, i, p)
    if case["kind"] == "verify":
        # windows of drafts with ids made from the seed
        for i in ids:
            B.pacer_begin_step(s.ctx, i)
        for _ in range(max(_gammas(case))):
            B.pacer_draft_step(s.ctx, ids, B.GREEDY, 0, 0)
        for i, y in zip(ids, drafts):
            t = s.draft_tokens(i)
            t.copy_(torch.from_numpy(y[:t.numel()]).cuda())
    torch.cuda.synchronize()
    return dict(case=case, s=s, prompts=prompts, ids=ids, gammas=_gammas(case), mode=B.SAMPLE if case["sample"] else B.GREEDY)


# ---------------------------------------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind, b = case["kind"], case["block"]
    if kind == "accept":
        B.pacer_accept_noalloc(state["lt"], state["ld"], state["y"], case["gamma"], True, state["lt"].shape[1], B.SAMPLE if case["sample"] else B.GREEDY, 0.0,
                               RNG_SEED, STEP, 0, state["n"], state["z"], state["stream"])
        return state["n"], state["z"]
    s, ids, mode = state["s"], state["ids"], state["mode"]
    if kind == "verify":
        B.pacer_verify(s.ctx, ids, state["gammas"], s.logits)
        return [s.logits[i, :g + 1] for i, g in zip(ids, state["gammas"])]
    if kind == "prompt":
        B.pacer_prefill(s.ctx, 0, state["prompts"][0])
    for i in ids:
        B.pacer_begin_step(s.ctx, i)
    if kind == "draft":
        B.pacer_draft_step(s.ctx, ids, mode, RNG_SEED, STEP)
        return [(s.draft_logits(i)[0], s.draft_hidden(i)[0], s.draft_tokens(i)[:1]) for i in ids]
    for _ in range(b):
        B.pacer_draft_step(s.ctx, ids, mode, RNG_SEED, STEP)
    B.pacer_preverify_block(s.ctx, ids, s.alpha, s.stop)
    B.pacer_wait_stop(s.ctx, ids)
    out = [s.draft_logits(0)[:b], s.draft_hidden(0)[:b], s.draft_tokens(0)[:b], s.alpha[0]]
    if kind in ("prompt", "step"):
        B.pacer_verify(s.ctx, ids, None, s.logits)
        out.append(s.logits[0, :b + 1])
    return out


# ---------------------------------------------------------------------------------------------- bounds
def _pass_work(t, layers, rows, keys, wb, head_rows, kv_only_last=False):
    """Bytes and flops of one forward: weights once, the keys and values that the rows look at, the logits."""
    d, _, _, f, v, _ = t
    per = 4 * d * d + 3 * d * f
    p = layers * per - ((d * d + 3 * d * f + d * d) if kv_only_last else 0)
    kvs = sum(a for a, _ in keys)
    pairs = sum(a * r for a, r in keys)
    byt = wb * p + 2 * wb * d * layers * kvs + (wb * v * d + 4 * v * head_rows if head_rows else 0)
    return byt, 2.0 * p * rows + 4.0 * d * layers * pairs + (2.0 * v * d * head_rows)


def work(case):
    kind, g = case["kind"], case["gamma"]
    t, dr = TARGETS[case["pair"]], DRAFTS[case["pair"]]
    wb = 2 if _bf16(case) else 4
    lens = _lengths(case)
    if kind == "accept":
        return dict(bytes=8.0 * (g + 1) * t[4], flops=10.0 * (g + 1) * t[4])
    parts = []
    if kind == "verify":
        gs = _gammas(case)
        parts.append(_pass_work(t, case["layers"], sum(gs) + len(gs), [(n + k, k + 1) for n, k in zip(lens, gs)], wb, sum(gs) + len(gs)))
    elif kind == "draft":
        parts.append(_pass_work(dr, dr[5], len(lens), [(n, 1) for n in lens], wb, len(lens)))
    else:
        n, b = lens[0], case["block"]
        if kind == "prompt" and n > 1:
            causal = [(n - 1, (n - 1) / 2)]
            parts.append(_pass_work(t, case["layers"], n - 1, causal, wb, 0, True))
            parts.append(_pass_work(dr, dr[5], n - 1, causal, wb, 0))
            parts.append((wb * 2 * dr[0] ** 2, 4.0 * (n - 1) * dr[0] ** 2))
        parts += [_pass_work(dr, dr[5], 1, [(n + j, 1)], wb, 1) for j in range(b)]
        parts.append(_pass_work(dr, 1, b, [(n + b - 1, b)], wb, 0))
        if kind in ("prompt", "step"):
            parts.append(_pass_work(t, case["layers"], b + 1, [(n + b, b + 1)], wb, b + 1))
    return dict(bytes=float(sum(p[0] for p in parts)), flops=float(sum(p[1] for p in parts)))


def tolerance(case):
    """Four times the distance from exact() that the f16 operands and caches give: 2-norm 0.0005..0.0016 at up to 12
    layers, 0.002..0.0034 for the 24- and 32-layer models; the f32 pair 2.5e-7."""
    if case["kind"] == "accept":
        return "exact"
    if not _bf16(case):
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    deep = case["pair"] == "33b" or case["layers"] > 12
    return {"rel": 1.2e-2 if deep else 6e-3, "max": 1.2e-1 if deep else 6e-2, "differ": 0.01}


# ---------------------------------------------------------------------------------------------- the same in 64 bits
def _philox(seed, seq, step, row, purpose, n):
    """Philox-4x32-10 (Salmon et al. 2011): n uniforms in (0, 1) keyed by the seed, counter (id / 4, row, step, purpose + 256 seq)."""
    m32 = np.uint64(0xFFFFFFFF)
    k = -(-n // 4)
    c = [np.arange(k, dtype=np.uint64), np.full(k, row, np.uint64), np.full(k, step, np.uint64), np.full(k, purpose | (seq << 8), np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & m32, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    bits = np.stack(c, 1).reshape(-1)[:n]
    return torch.from_numpy(((bits >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23).cuda()


def _gumbel(u):
    return -torch.log(-torch.log(u))


def _norm(x, g):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def _rope(x, pos, hd):
    half = hd // 2
    ang = pos[:, None].double() * THETA ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / hd)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _layer(x, w, h, hd, cache):
    """One decoder layer on new rows x at the positions after those in `cache` (a dict that keeps K and V)."""
    n, d = x.shape
    past = cache["k"].shape[0] if cache else 0
    pos = torch.arange(past, past + n, device="cuda")
    y = _norm(x, w["attn_norm"])
    q, k, v = [(y @ w[m].double().T).view(n, h, hd) for m in ("wq", "wk", "wv")]
    q, k = _rope(q, pos, hd), _rope(k, pos, hd)
    if past:
        k, v = torch.cat([cache["k"], k]), torch.cat([cache["v"], v])
    cache["k"], cache["v"] = k, v
    mask = torch.arange(past + n, device="cuda")[None] > pos[:, None]
    o = torch.empty_like(q)
    for i in range(h):
        sc = (q[:, i] @ k[:, i].T.contiguous() / math.sqrt(hd)).masked_fill_(mask, -math.inf)
        o[:, i] = torch.softmax(sc, -1) @ v[:, i].contiguous()
    x = x + o.view(n, d) @ w["wo"].double().T
    y = _norm(x, w["ffn_norm"])
    return x + (torch.nn.functional.silu(y @ w["wg"].double().T) * (y @ w["wu"].double().T)) @ w["wd"].double().T


class _Ref:
    """A model in 64 bits with its cache; rows() returns the final-norm output of the new rows."""

    def __init__(self, w, t):
        self.w, self.h, self.hd = w, t[1], t[2]
        self.caches = [dict() for _ in w["layers"]]

    def rows(self, ids):
        x = self.w["embed"][torch.as_tensor(ids, device="cuda").long()].double()
        for w, c in zip(self.w["layers"], self.caches):
            x = _layer(x, w, self.h, self.hd, c)
        return _norm(x, self.w["final_norm"])

    def logits(self, hid):
        return hid @ self.w["head"].double().T


def _exact_accept(case, seed):
    lt, ld, y = _accept_inputs(case, seed)
    lt, ld, k = lt.double(), ld.double(), case["gamma"]
    n = k
    if case["sample"]:
        lp, lq = torch.log_softmax(lt, 1), torch.log_softmax(ld, 1)
        for i in range(k):
            if float(_philox(RNG_SEED, 0, STEP, i + 1, 1, 1)[0]) > float((lp[i, y[i]] - lq[i, y[i]]).exp()):
                n = i
                break
        gum = _gumbel(_philox(RNG_SEED, 0, STEP, n + 1, 2, lt.shape[1]))
        res = (lp[n].exp() - lq[n].exp()).clamp_min(0) if n < k else lp[n].exp()
        z = int((torch.log(res) + gum).argmax())
    else:
        best = lt.argmax(1)
        n = next((i for i in range(k) if int(best[i]) != int(y[i])), k)
        z = int(best[n])
    one = lambda v: torch.tensor([v], dtype=torch.int32, device="cuda")
    return one(n), one(z)


def exact(case, seed):
    if case["kind"] == "accept":
        return _exact_accept(case, seed)
    w = _Weights(case, seed)
    t, dr = TARGETS[case["pair"]], DRAFTS[case["pair"]]
    prompts, drafts = _tokens(case, seed)
    kind, b = case["kind"], case["block"]
    if kind == "verify":
        out = []
        for p, y, g in zip(prompts, drafts, _gammas(case)):
            m = _Ref(w.target, t)
            out.append(m.logits(m.rows(np.concatenate([p, y[:g]]))[-(g + 1):]))
        return out

    def pick(lg, seq, j):
        return int((lg + _gumbel(_philox(RNG_SEED, seq, STEP, j + 1, 0, lg.shape[0])) if case["sample"] else lg).argmax())

    if kind == "draft":
        out = []
        for i, p in enumerate(prompts):
            m = _Ref(w.draft, dr)
            hid = m.rows(p)[-1]
            lg = m.logits(hid)
            out.append((lg, hid, torch.tensor([pick(lg, i, 0)], dtype=torch.int32, device="cuda")))
        return out
    p = prompts[0]
    m = _Ref(w.draft, dr)
    hids, toks, lgs = m.rows(p), [], []
    for j in range(b):
        lgs.append(m.logits(hids[-1]))
        toks.append(pick(lgs[-1], 0, j))
        if j + 1 < b:
            hids = torch.cat([hids, m.rows(np.array([toks[-1]]))])
    x = hids.clone()
    x[-b:] += w.mb["posemb"][1:b + 1].double()
    z = _norm(_layer(x, w.mb["layer"], dr[1], dr[2], {})[-b:], w.mb["final_norm"]) @ w.mb["cls"].double().T
    out = [torch.stack(lgs), hids[-b:], torch.tensor(toks, dtype=torch.int32, device="cuda"), torch.sigmoid(z[:, 1] - z[:, 0])]
    if kind in ("prompt", "step"):
        m = _Ref(w.target, t)
        out.append(m.logits(m.rows(np.concatenate([p, np.array(toks, dtype=np.int32)]))[-(b + 1):]))
    return out
