"""Performance cases of the drafter step, through the library's entry points.

A case is a dict of plain values.  Its "kind" names the call sequence:

  round           one chained drafter round (``carryover_round``), as a serving
                  loop issues it: the slots' committed lengths are set, then
                  route, projection and attention run in one call
  prefill         the prompt's rows projected and committed in one call each
                  (``carryover_route`` + ``carryover_project_kv``)
  attend          the block attention alone, with the extras of
                  ``drafter_block_attention_ext``: the block's own rows as a
                  third segment and the carried rows' attention mass
  train_forward   the training-shaped second pass: F(E) folded, every recorded
                  position projected and committed, every anchored block's
                  window projected, then the shared-prefix attention
  train_backward  its backward: the attention backward, then the projection
                  backward of both projection calls
  verify          stochastic (T = 1) verification of a batch of windows

Weights are N(0, 0.02^2), target states N(0, 1); committed keys and values and
the queries carry the statistics that such weights give (logits of unit
standard deviation), as everywhere else in this repository.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2609_14717_amd as co

PAGE = 16
VOCAB = 1000                       # token ids of the greedy verification
SIGMA_W = 0.02
EPS = 1e-6                         # of the RMS norms


# ------------------------------------------------------------------ the cases

def _widths(Dcat, d, L, Hq, Hkv, hd, theta, dtype="bf16"):
    return dict(Dcat=Dcat, d=d, L=L, Hq=Hq, Hkv=Hkv, hd=hd, theta=theta, dtype=dtype)


def _small(dtype="bf16"):
    return _widths(768, 256, 1, 4, 2, 64, 1e4, dtype)


def _large(L=1):
    return _widths(20480, 4096, L, 32, 8, 128, 1e6)


def _round(name, S, B, lo, hi, reject, widths, z_norm=False, k_norm=False):
    c = dict(name=name, kind="round", S=S, B=B, ctx_lo=lo, ctx_hi=hi, reject=reject, **widths)
    return dict(c, z_norm=z_norm, k_norm=k_norm)


def listed():
    return [
        # one short fp32 stream: the smallest round, all launches and latency
        _round("round_f32_tiny", 1, 8, 128, 128, 0.25, _small("f32")),
        # a full-precision run of a small drafter over a batch of ragged streams
        _round("round_f32_batch8", 8, 16, 100, 4000, 0.25, _widths(2560, 1024, 2, 8, 4, 64, 1e4, "f32")),
        # one interactive stream of a large drafter: weights stream from memory
        _round("round_batch1_8b", 1, 16, 2048, 2048, 0.25, _large()),
        # the serving batch of a small drafter: 32 ragged contexts
        _round("round_batch32", 32, 16, 512, 8192, 0.25, _small()),
        # the serving batch of a large drafter
        _round("round_batch32_8b", 32, 16, 512, 8192, 0.25, _large()),
        # long contexts and five drafter layers: the most memory traffic
        _round("round_long_5layer", 16, 16, 16384, 32768, 0.3, _large(5)),
        # odd sizes: a 7-row window, three query heads per KV head, short ragged
        # contexts, the normalised drafter
        _round("round_odd_norm", 11, 7, 37, 1500, 0.2, _widths(1920, 640, 2, 12, 4, 128, 1e6),
               z_norm=True, k_norm=True),
        # a prompt of 2048 tokens for a large drafter: compute-bound projection
        dict(name="prefill_8b", kind="prefill", S=1, n=2048, **_large()),
        # the drafter's attention with its own block rows and the carry diagnostic
        dict(name="attend_self_batch32_8b", kind="attend", S=32, B=16, ctx_lo=512, ctx_hi=8192,
             reject=0.25, self_rows=True, mass=True, **_large()),
        # the training step's two directions: 8 recorded responses of 4096
        # positions, 256 anchored blocks each
        dict(name="train_forward", kind="train_forward", S=8, n=4096, A=256, B=16, **_small()),
        dict(name="train_backward", kind="train_backward", S=8, n=4096, A=256, B=16, **_small()),
        # T = 1 verification of the serving batch over a large vocabulary
        dict(name="verify_batch32", kind="verify", S=32, B=16, V=128000),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_widths(rng, B, dtype):
    hd = rng.choice((64, 128))
    Hkv = rng.choice((1, 2, 4, 8))
    G = rng.choice([g for g in (1, 2, 3, 4, 6, 8) if B * g <= 64])
    Dcat = 64 * _log(rng, 4, 320 if dtype == "bf16" else 40)
    d = 64 * _log(rng, 2, 64 if dtype == "bf16" else 16)
    return _widths(Dcat, d, rng.choice((1, 1, 2, 3, 5)), G * Hkv, Hkv, hd, rng.choice((1e4, 1e6)),
                   dtype)


def _context(rng, c, most_bytes):
    """Ragged context bounds whose keys and values stay under ``most_bytes``."""
    row = 2 * c["L"] * c["Hkv"] * c["hd"] * _eb(c)
    cap = max(64, min(32768, int(most_bytes / (row * c["S"]))))
    hi = _log(rng, 64, cap)
    return dict(ctx_lo=rng.randint(1, hi), ctx_hi=hi)


def draw(rng):
    kind = rng.choice(("round",) * 6 + ("prefill", "prefill", "attend", "attend", "train_forward",
                                        "train_backward", "verify"))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    if kind in ("round", "attend"):
        B = rng.choice((16, 16, 16, 8, rng.randint(1, 32)))
        c = dict(kind=kind, S=_log(rng, 1, 48 if dtype == "bf16" else 12), B=B,
                 reject=round(rng.uniform(0.05, 0.5), 2), **_draw_widths(rng, B, dtype))
        c.update(_context(rng, c, 4e9 if dtype == "bf16" else 6e7))
        if kind == "round":
            c.update(z_norm=rng.random() < 0.2, k_norm=rng.random() < 0.2)
        else:
            c.update(self_rows=rng.random() < 0.8, mass=rng.random() < 0.5)
        return c
    if kind == "prefill":
        S, w = _log(rng, 1, 8), _draw_widths(rng, 16, dtype)
        per_row = 2 * w["d"] * (w["Dcat"] + 2 * w["L"] * w["Hkv"] * w["hd"])
        most = min(4096, 4e11 / per_row) if dtype == "bf16" else 512
        return dict(kind=kind, S=S, n=_log(rng, 17, int(most) // S), **w)
    if kind in ("train_forward", "train_backward"):
        B, hd = rng.choice((8, 16)), 64
        Hkv, G = rng.choice((1, 2, 4)), rng.choice([g for g in (1, 2, 4) if B * g <= 32])
        S, n = _log(rng, 1, 8), _log(rng, 200, 4096)
        return dict(kind=kind, S=S, n=n, A=_log(rng, 3, min(256 // Hkv, n // 2)), B=B,
                    **_widths(64 * _log(rng, 4, 16), rng.choice((128, 256, 320)), 1, G * Hkv, Hkv,
                              hd, 1e4))
    return dict(kind="verify", S=_log(rng, 1, 48), B=rng.choice((4, 8, 16, rng.randint(1, 24))),
                V=_log(rng, 1000, 160000))


# ------------------------------------------------------------- common pieces

def _eb(c):
    return 2 if c["dtype"] == "bf16" else 4


def _dt(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _sigma_kv(c):
    """Standard deviation of a projected key or value entry."""
    return SIGMA_W ** 2 * math.sqrt(c["Dcat"] * c["d"])


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(g, shape, dtype, sigma):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, sigma, generator=g)


def _weights(c, g):
    """The drafter's weights, and co_weights over them (F(E) folded once, as a
    program does when it loads them)."""
    z_norm, k_norm = c.get("z_norm", False), c.get("k_norm", False)
    n_kv = 2 * c["L"] * c["Hkv"] * c["hd"]
    w = dict(wf=_randn(g, (c["d"], c["Dcat"]), _dt(c), SIGMA_W),
             wkv=_randn(g, (n_kv, c["d"]), _dt(c), SIGMA_W),
             e=_randn(g, (c["Dcat"],), _dt(c), SIGMA_W), z_gain=None, k_gain=None, f_e=None)
    if z_norm:
        w["z_gain"] = SIGMA_W * math.sqrt(c["Dcat"]) * (1 + _randn(g, (c["d"],), torch.float32, 0.1))
    if k_norm:
        w["k_gain"] = _sigma_kv(c) * (1 + _randn(g, (c["L"], c["hd"]), torch.float32, 0.1))
    if c["dtype"] == "bf16":
        w["f_e"] = torch.empty(c["d"], dtype=torch.float32, device="cuda")
    w["co"] = co.weights(w["wf"], w["wkv"], w["e"], w["f_e"], None, w["z_gain"], w["k_gain"])
    return w


def _dims(c, S, B, max_pages, num_pages):
    return co.make_dims(S, B, c["Dcat"], c["d"], c["L"], c["Hq"], c["Hkv"], c["hd"], max_pages,
                        num_pages, c["dtype"], c["theta"])


def _workspace(dims, which):
    return torch.zeros(max(256, co.workspace_bytes(dims, which)), dtype=torch.uint8, device="cuda")


def _lengths(c, seed):
    """Committed lengths: spread evenly over the case's range, in a seeded order."""
    S, lo, hi = c["S"], c["ctx_lo"], c["ctx_hi"]
    n = [hi if S == 1 else lo + (hi - lo) * i // (S - 1) for i in range(S)]
    random.Random(seed).shuffle(n)
    return n


def _accepted(c, seed, count):
    """Accepted prefix lengths: every position rejected with probability ``reject``."""
    r = random.Random(seed + 1)
    return [next((j for j in range(c["B"]) if r.random() < c["reject"]), c["B"])
            for _ in range(count)]


def _tokens(m, B, g):
    """(draft, target) whose longest common prefix is m[s] in every row."""
    m = torch.as_tensor(m, dtype=torch.int32, device="cuda")[:, None]
    S = len(m)
    target = torch.randint(0, VOCAB, (S, B), generator=g, device="cuda", dtype=torch.int32)
    other = torch.randint(0, VOCAB, (S, B), generator=g, device="cuda", dtype=torch.int32)
    j = torch.arange(B, device="cuda", dtype=torch.int32)[None]
    draft = torch.where(j < m, target, torch.where(j == m, (target + 1) % VOCAB, other))
    return draft.contiguous(), target


def _page_table(pages, max_pages, g):
    """Rows of distinct pages in a random order; unused entries 0."""
    total = sum(pages)
    ids = torch.randperm(total, generator=g, device="cuda").to(torch.int32)
    pt = torch.zeros((len(pages), max_pages), dtype=torch.int32, device="cuda")
    at = 0
    for s, n in enumerate(pages):
        pt[s, :n] = ids[at:at + n]
        at += n
    return pt, total


def _batch_state(c, seed, g):
    """(dims, state, committed lengths on the device) of a batch of ragged
    sequences whose pages hold keys and values of earlier rounds."""
    n = _lengths(c, seed)
    pages = [-(-(x + 2 * c["B"]) // PAGE) for x in n]
    max_pages = -(-(c["ctx_hi"] + 4 * c["B"]) // PAGE)
    pt, total = _page_table(pages, max_pages, g)
    dims = _dims(c, c["S"], c["B"], max_pages, total)
    st = co.alloc_state(dims, pt)
    st["k_cache"].normal_(0.0, _sigma_kv(c), generator=g)
    st["v_cache"].normal_(0.0, _sigma_kv(c), generator=g)
    ctx = torch.tensor(n, dtype=torch.int32, device="cuda")
    st["ctx_len"].copy_(ctx)
    return dims, st, ctx


# ----------------------------------------------------------------- prepare

def prepare(case, seed):
    return {"round": _prepare_round, "prefill": _prepare_prefill, "attend": _prepare_attend,
            "train_forward": _prepare_train, "train_backward": _prepare_train_backward,
            "verify": _prepare_verify}[case["kind"]](case, seed)


def _prepare_round(c, seed):
    g = _gen(seed)
    S, B = c["S"], c["B"]
    dims, st, ctx = _batch_state(c, seed, g)
    w = _weights(c, g)
    if w["f_e"] is not None:
        co.carryover_fold_e(dims, w["co"], w["f_e"])
    draft, target = _tokens(_accepted(c, seed, S), B, g)
    q = _randn(g, (c["L"], S, B, c["Hq"], c["hd"]), _dt(c), 1 / _sigma_kv(c))
    return dict(case=c, dims=dims, st=st, ctx0=ctx, w=w, draft=draft, target=target, q=q,
                hidden=_randn(g, (S, B, c["Dcat"]), _dt(c), 1.0), rt=co.alloc_route(S, B),
                out=torch.empty_like(q), lse=torch.empty(q.shape[:-1], device="cuda"),
                ws=_workspace(dims, co.CO_WS_ROUND))


def _prepare_prefill(c, seed):
    g = _gen(seed)
    S, n = c["S"], c["n"]
    P = -(-(n + 4 * PAGE) // PAGE)
    pt, total = _page_table([P] * S, P, g)
    dims = _dims(c, S, n, P, total)
    w = _weights(c, g)
    if w["f_e"] is not None:
        co.carryover_fold_e(dims, w["co"], w["f_e"])
    return dict(case=c, dims=dims, st=co.alloc_state(dims, pt), w=w, rt=co.alloc_route(S, n),
                hidden=_randn(g, (S, n, c["Dcat"]), _dt(c), 1.0),
                ws=_workspace(dims, co.CO_WS_PROJECT))


def _prepare_attend(c, seed):
    g = _gen(seed)
    S, B = c["S"], c["B"]
    dims, st, _ = _batch_state(c, seed, g)
    st["k_carry"].normal_(0.0, _sigma_kv(c), generator=g)
    st["v_carry"].normal_(0.0, _sigma_kv(c), generator=g)
    st["carry_len"].copy_(B - torch.tensor(_accepted(c, seed, S), dtype=torch.int32))
    q = _randn(g, (c["L"], S, B, c["Hq"], c["hd"]), _dt(c), 1 / _sigma_kv(c))
    own = [None, None]
    if c["self_rows"]:
        own = [_randn(g, (c["L"], S, B, c["Hkv"], c["hd"]), _dt(c), _sigma_kv(c)) for _ in range(2)]
    return dict(case=c, dims=dims, st=st, q=q, k_self=own[0], v_self=own[1],
                out=torch.empty_like(q), lse=torch.empty(q.shape[:-1], device="cuda"),
                mass=torch.empty(q.shape[:-1], device="cuda") if c["mass"] else None,
                ws=_workspace(dims, co.CO_WS_ATTENTION))


def _prepare_train(c, seed):
    """S recorded responses of n positions; A sorted anchors in each, whose
    windows start at a + 1 and leave u rejected rows, so that the block's
    queries sit at a' = a + (B - u) + 1 and see the response up to there."""
    g = _gen(seed)
    S, n, A, B = c["S"], c["n"], c["A"], c["B"]
    V, P = S * A, -(-c["n"] // PAGE)
    pt, total = _page_table([P] * S, P, g)
    dims, vdims = _dims(c, S, n, P, total), _dims(c, V, B, P, total)
    st = co.alloc_state(dims, pt)
    w = _weights(c, g)
    r = random.Random(seed)
    anchors = torch.tensor([a for _ in range(S) for a in sorted(r.sample(range(n - 2 * B), A))])
    u = torch.tensor([r.randint(0, B) for _ in range(V)])
    vctx = (anchors + 1).to(torch.int32).cuda()
    carry = co.alloc_state(_dims(c, V, B, P, 1), pt.repeat_interleave(A, 0))
    vst = dict(carry, k_cache=st["k_cache"], v_cache=st["v_cache"])
    draft, target = _tokens((B - u).tolist(), B, g)
    q = _randn(g, (c["L"], V, B, c["Hq"], c["hd"]), _dt(c), 1 / _sigma_kv(c))
    ws = torch.zeros(max(256, co.workspace_bytes(dims, co.CO_WS_PROJECT),
                         co.workspace_bytes(vdims, co.CO_WS_ROUND)), dtype=torch.uint8,
                     device="cuda")
    return dict(case=c, dims=dims, vdims=vdims, st=st, vst=vst, w=w, vctx=vctx,
                draft=draft, target=target, q=q, rt=co.alloc_route(S, n), vrt=co.alloc_route(V, B),
                h=_randn(g, (S, n, c["Dcat"]), _dt(c), 1.0),
                vh=_randn(g, (V, B, c["Dcat"]), _dt(c), 1.0),
                out=torch.empty_like(q), lse=torch.empty(q.shape[:-1], device="cuda"), ws=ws)


def _prepare_train_backward(c, seed):
    s = _prepare_train(c, seed)
    _run_train_forward(s)
    st, vst, w = s["st"], s["vst"], s["w"]
    like = lambda t: torch.zeros(t.shape, dtype=torch.float32, device="cuda")  # noqa: E731
    s.update(d_out=_randn(_gen(seed + 1), s["q"].shape, _dt(c), 1.0), dq=like(s["q"]),
             dk=like(st["k_cache"]), dv=like(st["v_cache"]), dkc=like(vst["k_carry"]),
             dvc=like(vst["v_carry"]), dwf=like(w["wf"]), dwkv=like(w["wkv"]), de=like(w["e"]),
             aws=_workspace(s["vdims"], co.CO_WS_ATTENTION_BACKWARD),
             pws=torch.zeros(max(co.workspace_bytes(s["dims"], co.CO_WS_PROJECT_BACKWARD),
                                 co.workspace_bytes(s["vdims"], co.CO_WS_PROJECT_BACKWARD), 256),
                             dtype=torch.uint8, device="cuda"))
    return s


def _prepare_verify(c, seed):
    """Target and drafter distributions that disagree as a drafter and its
    target do, the drafter's proposals drawn from its own."""
    g = _gen(seed)
    S, B, V = c["S"], c["B"], c["V"]
    logits = _randn(g, (S, B + 1, V), torch.float32, 2.0)
    q = torch.softmax(logits[:, :B] + _randn(g, (S, B, V), torch.float32, 1.0), -1)
    noise = torch.empty_like(q).exponential_(generator=g)
    draft = (q / noise).argmax(-1).to(torch.int32)
    words = torch.randint(-2 ** 31, 2 ** 31, (S, B + 1), generator=g, device="cuda").to(torch.int32)
    new = lambda *shape: torch.zeros(shape, dtype=torch.int32, device="cuda")  # noqa: E731
    return dict(case=c, dims=co.make_dims(S, B, 64, 64, 1, 1, 1, 64, 1, 1, "bf16", 1e4),
                draft=draft, p=torch.softmax(logits, -1), q=q, words=words, bits=new(S, B),
                m=new(S), tok=new(S), status=new(1))


# --------------------------------------------------------------------- run

def run(state):
    return {"round": _run_round, "prefill": _run_prefill, "attend": _run_attend,
            "train_forward": _run_train_forward, "train_backward": _run_train_backward,
            "verify": _run_verify}[state["case"]["kind"]](state)


def _cache(st):
    return {k: st[k] for k in ("k_cache", "v_cache", "k_carry", "v_carry", "status")}


def _run_round(s):
    st, rt = s["st"], s["rt"]
    st["ctx_len"].copy_(s["ctx0"])
    co.carryover_round(s["dims"], s["w"]["co"], s["hidden"], s["draft"], s["target"], s["q"], st,
                       rt, s["out"], s["lse"], 0, s["ws"])
    return dict(_cache(st), out=s["out"], lse=s["lse"], ctx_len=st["ctx_len"],
                carry_len=st["carry_len"], **rt)


def _run_prefill(s):
    st, rt = s["st"], s["rt"]
    st["ctx_len"].zero_()
    co.carryover_route(s["dims"], None, None, co.CO_ROUTE_ACCEPT_ALL, st, rt)
    co.carryover_project_kv(s["dims"], s["w"]["co"], s["hidden"], rt, st, s["ws"])
    return dict(k_cache=st["k_cache"], v_cache=st["v_cache"], status=st["status"],
                ctx_len=st["ctx_len"], **rt)


def _run_attend(s):
    co.drafter_block_attention_ext(s["dims"], 0, s["case"]["L"], s["q"], s["k_self"], s["v_self"],
                                   s["st"], s["out"], s["lse"], s["mass"], 0, s["ws"])
    return dict(out=s["out"], lse=s["lse"], mass=s["mass"], status=s["st"]["status"])


def _run_train_forward(s):
    st, vst, w = s["st"], s["vst"], s["w"]["co"]
    co.carryover_fold_e(s["dims"], w, s["w"]["f_e"])     # the weights change every step
    st["ctx_len"].zero_()
    co.carryover_route(s["dims"], None, None, co.CO_ROUTE_ACCEPT_ALL, st, s["rt"])
    co.carryover_project_kv(s["dims"], w, s["h"], s["rt"], st, s["ws"])
    vst["ctx_len"].copy_(s["vctx"])
    co.carryover_route(s["vdims"], s["draft"], s["target"], co.CO_ROUTE_CARRY_ONLY, vst, s["vrt"])
    co.carryover_project_kv(s["vdims"], w, s["vh"], s["vrt"], vst, s["ws"])
    co.drafter_block_attention(s["vdims"], 0, s["case"]["L"], s["q"], vst, s["out"], s["lse"],
                               co.CO_ATTN_SHARED_PREFIX, s["ws"])
    return dict(_cache(vst), out=s["out"], lse=s["lse"], f_e=s["w"]["f_e"],
                ctx_len=vst["ctx_len"], carry_len=vst["carry_len"])


def _run_train_backward(s):
    vst, w = s["vst"], s["w"]["co"]
    for k in ("dk", "dv", "dwf", "dwkv", "de"):          # a step's gradients start from zero
        s[k].zero_()
    co.drafter_block_attention_backward(s["vdims"], 0, s["case"]["L"], s["q"], vst, s["out"],
                                        s["lse"], s["d_out"], s["case"]["A"], s["dq"], s["dk"],
                                        s["dv"], s["dkc"], s["dvc"], s["aws"])
    co.carryover_project_kv_backward(s["dims"], w, s["h"], s["rt"], s["dk"], s["dv"], s["dkc"],
                                     s["dvc"], s["dwf"], s["dwkv"], s["de"], s["pws"])
    co.carryover_project_kv_backward(s["vdims"], w, s["vh"], s["vrt"], s["dk"], s["dv"], s["dkc"],
                                     s["dvc"], s["dwf"], s["dwkv"], s["de"], s["pws"])
    return dict({k: s[k] for k in ("dq", "dk", "dv", "dkc", "dvc", "dwf", "dwkv", "de")},
                status=vst["status"])


def _run_verify(s):
    co.carryover_verify_sample(s["dims"], s["case"]["V"], s["draft"], s["p"], s["q"], s["words"],
                               s["bits"], s["m"], s["tok"], s["status"])
    return {k: s[k] for k in ("bits", "m", "tok", "status")}


# -------------------------------------------------------------------- work

def work(c):
    if c["kind"] == "verify":
        # the proposals' probabilities, then one row of p and (unless every
        # proposal was accepted) of q
        S, B, V = c["S"], c["B"], c["V"]
        return {"bytes": 4.0 * S * (5 * B + 2 * V + 3), "flops": 0.0}
    es, S, L = _eb(c), c["S"], c["L"]
    n_kv = 2 * L * c["Hkv"] * c["hd"]
    weights = (c["d"] * c["Dcat"] + n_kv * c["d"] + c["Dcat"]) * es
    per_row = 2.0 * (c["Dcat"] * c["d"] + c["d"] * n_kv)
    row_bytes = (c["Dcat"] + n_kv) * es                  # a row's state in, its keys and values out
    if c["kind"] == "prefill":
        M = S * c["n"]
        return {"bytes": float(weights + M * row_bytes), "flops": M * per_row}
    B, qd = c["B"], c["Hq"] * c["hd"]
    if c["kind"] in ("round", "attend"):
        own = c["kind"] == "attend"
        # expected accepted and carried rows; keys seen by every query
        m = sum((1 - c["reject"]) ** j for j in range(1, B + 1))
        ctx = (c["ctx_lo"] + c["ctx_hi"]) / 2 if S > 1 else c["ctx_hi"]
        keys = S * (ctx + ((B - m) if own else B) + (B if own and c["self_rows"] else 0))
        q_bytes = L * S * B * (2 * qd * es + 4 * c["Hq"] * (2 if own and c["mass"] else 1))
        bytes_ = keys * n_kv * es + q_bytes
        flops = 4.0 * keys * L * B * qd
        if not own:
            bytes_ += weights + S * B * row_bytes
            flops += S * B * per_row
        return {"bytes": float(bytes_), "flops": flops}
    # training: half of the response is seen by an average block, half of the
    # blocks' rows are carried
    V, n, A = S * c["A"], c["n"], c["A"]
    rows, carried = S * n, V * B / 2
    keys = V * (n / 2 + B / 2)                           # (block, key) pairs of every query row
    attn = 4.0 * keys * L * B * qd
    kv_bytes = (rows + carried) * n_kv
    q_el = L * V * B * qd
    if c["kind"] == "train_forward":
        return {"bytes": float(weights + (rows + carried) * c["Dcat"] * es + kv_bytes * es
                               + q_el * 2 * es + 4 * L * V * B * c["Hq"]),
                "flops": (rows + carried) * per_row + attn + 2.0 * c["d"] * c["Dcat"]}
    grads = 4 * (c["d"] * c["Dcat"] + n_kv * c["d"] + c["Dcat"])
    return {"bytes": float(weights + grads + (rows + carried) * c["Dcat"] * es + kv_bytes * (es + 4)
                           + q_el * (3 * es + 4) + 4 * L * V * B * c["Hq"]),
            "flops": 2.5 * attn + 2 * (rows + carried) * per_row}


def tolerance(c):
    if c["kind"] == "verify":
        return "exact"                                   # decisions and tokens
    if c["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4}                # fp32 sums in another order: 4e-7 from 64 bits
    if c["kind"] == "train_backward":
        return {"rel": 1.4e-2}                           # P, dS and dJ rounded to bf16: 3.4e-3 from 64 bits
    return {"rel": 1e-2}                                 # bf16 Z, K/V, P and O: 2.3-4e-3 from 64 bits


# ------------------------------------------------- the same results in 64 bits

def exact(case, seed):
    if case["kind"] == "verify":
        return None                                      # whole numbers only
    s = prepare(case, seed)
    return {"round": _exact_round, "prefill": _exact_prefill, "attend": _exact_attend,
            "train_forward": _exact_train, "train_backward": _exact_backward}[case["kind"]](s)


def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain


def _rotate(x, pos, theta, sign=1.0):
    """Rotate-half pairs (i, i + hd/2) of x [..., hd] at pos (broadcast over x's leading dims)."""
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    ang = sign * pos.double()[..., None] * inv
    cs, sn = torch.cos(ang), torch.sin(ang)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat((lo * cs - hi * sn, hi * cs + lo * sn), -1)


def _project(c, w, x, pos):
    """Rows x [M][Dcat] at positions pos -> rotated keys and values [M][L][Hkv][hd]."""
    z = x @ w["wf"].double().T
    if w["z_gain"] is not None:
        z = _rms(z, w["z_gain"].double())
    kv = (z @ w["wkv"].double().T).view(-1, c["L"], 2, c["Hkv"], c["hd"])
    k = kv[:, :, 0]
    if w["k_gain"] is not None:
        k = _rms(k, w["k_gain"].double()[:, None, :])
    return _rotate(k, pos[:, None, None], c["theta"]), kv[:, :, 1]


def _prefix(draft, target):
    return torch.cumprod((draft == target).int(), 1).sum(1)


def _put(K, V, page, slot, k, v):
    """Rows k, v [n][L][Hkv][hd] into pages of K [L][pages][Hkv][16][hd], V [L][pages][Hkv][hd][16]."""
    K.permute(1, 3, 0, 2, 4)[page, slot] = k
    V.permute(1, 4, 0, 2, 3)[page, slot] = v


def _get(st, layer, s, n, K, V):
    """Committed keys and values [Hkv][n][hd] of sequence s."""
    page = st["page_table"][s, :-(-n // PAGE)].long()
    hkv, hd = K.shape[2], K.shape[4]
    k = K[layer][page].transpose(0, 1).reshape(hkv, -1, hd)[:, :n]
    v = V[layer][page].permute(1, 0, 3, 2).reshape(hkv, -1, hd)[:, :n]
    return k.double(), v.double()


def _attend(c, q, pos, k, v):
    """q [B][Hq][hd] at positions pos over k, v [Hkv][T][hd] -> out [B][Hq][hd], lse and weights."""
    B, G = q.shape[0], c["Hq"] // c["Hkv"]
    qr = _rotate(q.double(), pos[:, None], c["theta"]) / math.sqrt(c["hd"])
    qr = qr.view(B, c["Hkv"], G, c["hd"]).permute(1, 0, 2, 3).reshape(c["Hkv"], B * G, c["hd"])
    x = qr @ k.transpose(1, 2)
    lse = torch.logsumexp(x, -1)
    p = torch.exp(x - lse[..., None])
    back = lambda t: t.view(c["Hkv"], B, G, -1).permute(1, 0, 2, 3).reshape(B, c["Hq"], -1)  # noqa: E731
    return back(p @ v), back(lse[..., None])[..., 0], p, back


def _exact_route(s):
    """Accepted lengths, positions and destinations of a batch's window rows."""
    c, st = s["case"], s["st"]
    B, ctx0 = c["B"], s["ctx0"].long()
    m = _prefix(s["draft"], s["target"]).long()
    j = torch.arange(B, device="cuda")[None]
    pos = ctx0[:, None] + j
    return m, pos, st["page_table"].gather(1, pos // PAGE).long()


def _exact_round(s):
    c, st, w = s["case"], s["st"], s["w"]
    B, S, L = c["B"], c["S"], c["L"]
    m, pos, page = _exact_route(s)
    carried = torch.arange(B, device="cuda")[None] >= m[:, None]
    x = s["hidden"].double() + carried[..., None] * w["e"].double()
    k, v = _project(c, w, x.view(S * B, -1), pos.view(-1))
    K, V = st["k_cache"].double(), st["v_cache"].double()
    Kc, Vc = st["k_carry"].double(), st["v_carry"].double()
    keep = ~carried.view(-1)
    _put(K, V, page.view(-1)[keep], (pos % PAGE).view(-1)[keep], k[keep], v[keep])
    k, v = (t.view(S, B, L, c["Hkv"], c["hd"]) for t in (k, v))
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(out.shape[:-1], dtype=torch.float64, device="cuda")
    for i in range(S):
        mi = int(m[i])
        n, r = int(s["ctx0"][i]) + mi, torch.arange(B - mi, device="cuda")
        _put(Kc[:, i], Vc[:, i], r // PAGE, r % PAGE, k[i, mi:], v[i, mi:])
        for layer in range(L):
            kk, vv = _get(st, layer, i, n, K, V)
            kk = torch.cat((kk, k[i, mi:, layer].transpose(0, 1)), 1)
            vv = torch.cat((vv, v[i, mi:, layer].transpose(0, 1)), 1)
            qpos = n + torch.arange(B, device="cuda")
            out[layer, i], lse[layer, i], _, _ = _attend(c, s["q"][layer, i], qpos, kk, vv)
    return dict(k_cache=K, v_cache=V, k_carry=Kc, v_carry=Vc, out=out, lse=lse, status=None,
                ctx_len=None, carry_len=None, accept_len=None, row_pos=None, row_dst=None)


def _exact_prefill(s):
    c, st = s["case"], s["st"]
    S, n = c["S"], c["n"]
    K, V = st["k_cache"].double(), st["v_cache"].double()
    pos = torch.arange(n, device="cuda")
    for i in range(S):
        k, v = _project(c, s["w"], s["hidden"][i].double(), pos)
        _put(K, V, st["page_table"][i].long()[pos // PAGE], pos % PAGE, k, v)
    return dict(k_cache=K, v_cache=V, status=None, ctx_len=None, accept_len=None, row_pos=None,
                row_dst=None)


def _exact_attend(s):
    c, st = s["case"], s["st"]
    B = c["B"]
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(out.shape[:-1], dtype=torch.float64, device="cuda")
    mass = torch.empty_like(lse)
    for i in range(c["S"]):
        n, u = int(st["ctx_len"][i]), int(st["carry_len"][i])
        qpos, r = n + torch.arange(B, device="cuda"), torch.arange(u, device="cuda")
        for layer in range(c["L"]):
            k, v = _get(st, layer, i, n, st["k_cache"], st["v_cache"])
            kc = st["k_carry"][layer, i].double()[r // PAGE, :, r % PAGE]
            vc = st["v_carry"][layer, i].double()[r // PAGE, :, :, r % PAGE]
            k, v = torch.cat((k, kc.transpose(0, 1)), 1), torch.cat((v, vc.transpose(0, 1)), 1)
            if c["self_rows"]:
                own = _rotate(s["k_self"][layer, i].double(), qpos[:, None], c["theta"])
                k = torch.cat((k, own.transpose(0, 1)), 1)
                v = torch.cat((v, s["v_self"][layer, i].double().transpose(0, 1)), 1)
            out[layer, i], lse[layer, i], p, back = _attend(c, s["q"][layer, i], qpos, k, v)
            mass[layer, i] = back(p[..., n:n + u].sum(-1, keepdim=True)
                                  / p[..., :n + u].sum(-1, keepdim=True))[..., 0]
    return dict(out=out, lse=lse, mass=mass if c["mass"] else None, status=None)


def _blocks(c, s, vctx):
    """Accepted lengths, shifted anchors, window positions and carried rows of every block."""
    m = _prefix(s["draft"], s["target"]).long()
    j = torch.arange(c["B"], device="cuda")
    pos = vctx.long()[:, None] + j
    return m, vctx.long() + m, pos, j[None] >= m[:, None]


def _exact_train(s):
    c, st, vst, w = s["case"], s["st"], s["vst"], s["w"]
    S, n, A, B, L = c["S"], c["n"], c["A"], c["B"], c["L"]
    K, V = st["k_cache"].double(), st["v_cache"].double()
    Kc, Vc = vst["k_carry"].double(), vst["v_carry"].double()
    pos = torch.arange(n, device="cuda")
    m, a2, bpos, carried = _blocks(c, s, s["vctx"])
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(out.shape[:-1], dtype=torch.float64, device="cuda")
    e = w["e"].double()
    for i in range(S):
        k, v = _project(c, w, s["h"][i].double(), pos)
        _put(K, V, st["page_table"][i].long()[pos // PAGE], pos % PAGE, k, v)
        b = slice(i * A, (i + 1) * A)
        kb, vb = _project(c, w, (s["vh"][b].double() + e).view(A * B, -1), bpos[b].reshape(-1))
        blk, row = carried[b].nonzero(as_tuple=True)
        dst = row - m[b][blk]
        at = blk * B + row
        for full, part in ((Kc[:, b].permute(1, 2, 4, 0, 3, 5), kb),
                           (Vc[:, b].permute(1, 2, 5, 0, 3, 4), vb)):
            full[blk, dst // PAGE, dst % PAGE] = part[at]
        for layer in range(L):
            o, z, *_ = _block_attention(c, s["q"][layer, b], a2[b], m[b], k[:, layer], v[:, layer],
                                        Kc[layer, b], Vc[layer, b])
            out[layer, b], lse[layer, b] = o, z
    return dict(k_cache=K, v_cache=V, k_carry=Kc, v_carry=Vc, out=out, lse=lse, f_e=w["wf"].double() @ e,
                status=None, ctx_len=None, carry_len=None)


def _block_attention(c, q, a2, m, k, v, Kc, Vc):
    """A blocks q [A][B][Hq][hd] over a response's k, v [n][Hkv][hd] up to a2 and
    their own carried rows (pages Kc [A][CP][Hkv][16][hd], Vc [A][CP][Hkv][hd][16])."""
    A, B, H, G, hd = q.shape[0], c["B"], c["Hkv"], c["Hq"] // c["Hkv"], c["hd"]
    qpos = a2[:, None] + torch.arange(B, device="cuda")
    qr = _rotate(q.double(), qpos[:, :, None], c["theta"]) / math.sqrt(hd)
    qr = qr.view(A, B, H, G, hd).permute(2, 0, 1, 3, 4).reshape(H, A, B * G, hd)
    kc = Kc.permute(2, 0, 1, 3, 4).reshape(H, A, -1, hd)
    vc = Vc.permute(2, 0, 1, 4, 3).reshape(H, A, -1, hd)
    n, cp = k.shape[0], kc.shape[2]
    ks, vs = k.permute(1, 0, 2).contiguous(), v.permute(1, 0, 2).contiguous()
    x = torch.cat(((qr.reshape(H, A * B * G, hd) @ ks.transpose(1, 2)).view(H, A, B * G, n),
                   qr @ kc.transpose(2, 3).contiguous()), -1)
    hide = torch.cat((torch.arange(n, device="cuda")[None] >= a2[:, None],
                      torch.arange(cp, device="cuda")[None] >= (B - m)[:, None]), 1)
    x.masked_fill_(hide[None, :, None, :], -math.inf)
    z = torch.logsumexp(x, -1)
    p = torch.exp(x - z[..., None])
    o = (p[..., :n].reshape(H, A * B * G, n) @ vs).view(H, A, B * G, hd) + p[..., n:] @ vc
    back = lambda t: t.view(H, A, B, G, -1).permute(1, 2, 0, 3, 4).reshape(A, B, H * G, -1)  # noqa: E731
    return back(o), back(z[..., None])[..., 0], p, qr, ks, vs, kc, vc, back


def _exact_backward(s):
    c, st, vst, w = s["case"], s["st"], s["vst"], s["w"]
    S, n, A, B, L, H, hd = (c[k] for k in ("S", "n", "A", "B", "L", "Hkv", "hd"))
    G, CP = c["Hq"] // H, -(-B // PAGE)
    m, a2, bpos, carried = _blocks(c, s, s["vctx"])
    pos, scale = torch.arange(n, device="cuda"), 1 / math.sqrt(hd)
    g = {k: torch.zeros(s[k].shape, dtype=torch.float64, device="cuda")
         for k in ("dq", "dk", "dv", "dkc", "dvc", "dwf", "dwkv", "de")}
    wf, wkv, e = w["wf"].double(), w["wkv"].double(), w["e"].double()

    def project_back(x, dk, dv, rpos, on):
        """Adds the weight gradients of rows x whose rotated-key and value gradients are dk, dv."""
        dj = torch.stack((_rotate(dk, rpos[:, None, None], c["theta"], -1.0), dv), 2)
        dj = dj.reshape(len(x), -1)
        xe = x + on[:, None] * e
        dz = dj @ wkv
        g["dwkv"] += dj.T @ (xe @ wf.T)
        g["dwf"] += dz.T @ xe
        g["de"] += (dz * on[:, None]).sum(0) @ wf

    for i in range(S):
        b = slice(i * A, (i + 1) * A)
        dkr = torch.zeros((n, L, H, hd), dtype=torch.float64, device="cuda")
        dvr = torch.zeros_like(dkr)
        for layer in range(L):
            k, v = (t.transpose(0, 1) for t in _get(st, layer, i, n, st["k_cache"], st["v_cache"]))
            o, z, p, qr, ks, vs, kc, vc, back = _block_attention(
                c, s["q"][layer, b], a2[b], m[b], k, v, vst["k_carry"][layer, b].double(),
                vst["v_carry"][layer, b].double())
            split = lambda t: (t.double().view(A, B, H, G, hd).permute(2, 0, 1, 3, 4)  # noqa: E731
                               .reshape(H, A, B * G, hd))
            do = split(s["d_out"][layer, b])
            flat = lambda t: t.reshape(H, A * B * G, t.shape[-1])  # noqa: E731
            dp = torch.cat(((flat(do) @ vs.transpose(1, 2)).view(H, A, B * G, n),
                            do @ vc.transpose(2, 3).contiguous()), -1)
            ds = p * (dp - (do * split(o)).sum(-1, keepdim=True))
            dqr = (flat(ds[..., :n]) @ ks).view(H, A, B * G, hd) + ds[..., n:] @ kc
            qpos = a2[b][:, None] + torch.arange(B, device="cuda")
            g["dq"][layer, b] = _rotate(back(dqr) * scale, qpos[:, :, None], c["theta"], -1.0)
            dkr[:, layer] = (flat(ds[..., :n]).transpose(1, 2).contiguous() @ flat(qr)).transpose(0, 1)
            dvr[:, layer] = (flat(p[..., :n]).transpose(1, 2).contiguous() @ flat(do)).transpose(0, 1)
            pages = lambda t: t.view(H, A, CP, PAGE, hd).permute(1, 2, 0, 3, 4)  # noqa: E731
            g["dkc"][layer, b] = pages(ds[..., n:].transpose(2, 3).contiguous() @ qr)
            g["dvc"][layer, b] = pages(p[..., n:].transpose(2, 3).contiguous() @ do).transpose(3, 4)
        page = st["page_table"][i].long()[pos // PAGE]
        _put(g["dk"], g["dv"], page, pos % PAGE, dkr, dvr)
        project_back(s["h"][i].double(), dkr, dvr, pos, torch.zeros(n, device="cuda").double())
        blk, row = carried[b].nonzero(as_tuple=True)
        dst, at = row - m[b][blk], slice(i * A, (i + 1) * A)
        rows = (g["dkc"][:, at].permute(1, 2, 4, 0, 3, 5)[blk, dst // PAGE, dst % PAGE],
                g["dvc"][:, at].permute(1, 2, 5, 0, 3, 4)[blk, dst // PAGE, dst % PAGE])
        project_back(s["vh"][b].double()[blk, row], *rows, bpos[b][blk, row],
                     torch.ones(len(blk), device="cuda").double())
    return dict(g, status=None)
