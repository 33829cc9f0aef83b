"""GPU parity of the attention backward (the training side of the second
drafter pass, Algorithm 2) through the C ABI, against the fp64 oracle's
reverse mode (itself pinned by finite differences):

* the training layout: the anchored blocks of each recorded response share its
  committed pages (one group per response), so a committed key's gradient is
  the sum over every block that sees it; carry keys belong to one block;
* a serving layout (one sequence per group) after carryover rounds: ragged
  contexts, an empty sequence, a sequence with carry rows only, padded query
  rows (8 block rows x 2 heads) and a layer sub-range.

Gradients are compared per head vector at 2e-2, the bf16 rule of the forward,
with the denominator floored at a fraction of the largest reference vector of
the same (layer, KV head) slab: err = ||g - r||_inf / max(||r||_inf,
floor * max_slab ||r||_inf).  Vectors above the floor are held to the plain
per-vector rule; below it the rule is absolute.  A gradient vector is a sum of
terms of both signs whose magnitudes follow the slab's scale (dS = P (dP - D)
cancels, and so do the sums over queries), so the absolute error of a small
vector is set by its terms, not by its cancelled sum.

* The attention backward on its own (every key and value drawn directly by
  the seeded generator, so that both sides read the same bf16 values): floor
  1/8.  Its own rounding points are the bf16 rotated queries, the bf16 forward
  output in D, and P and dS rounded to bf16 before the three products.
* The whole path (keys and values projected by the GPU, rounded to bf16 twice
  -- F's output and the stored rows -- against the oracle's exact
  projection): floor 1, i.e. within 2e-2 of the slab's largest vector.  A
  logit moves by q . dk when a stored key moves by dk, and the softmax
  derivative turns that into relative errors of P that the cancelling sums of
  dV, dK and dq do not average away; the unit test above separates the
  backward's own error from this inherited one.
"""
import numpy as np
import pytest

import oracle
from synth import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from helpers import OracleRun, host, seq_block, to_np  # noqa: E402

GTOL = 2e-2
FLOOR_UNIT = 1.0 / 8      # the attention backward on identical bf16 inputs
FLOOR_PATH = 1.0          # gradients of the whole path (inputs projected on each side)
CARRY_T0 = wl.TCAP // 2   # logical positions of directly drawn carry rows (past any context)

TRAIN_SMALL = wl.TRAIN_FWD.replace(name="bwd_train_small", S=2, seq_len=512, anchors=10,
                                   seed=0x5EED30)
SERVE = wl.RAGGED32.replace(name="bwd_serve", S=6, B=8, L=2, ctx_lo=40, ctx_hi=700, rounds=4,
                            accept=("geom", 0.3), seed=0x5EED31)


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    return co


WORST = []


def slab_close(g, r, what, tol=GTOL, floor=FLOOR_PATH):
    """g, r [n][hd] of one (layer, KV head): every head vector within tol,
    relative to max(its own reference norm, floor x the slab's largest)."""
    g = np.asarray(g, np.float64)
    r = np.asarray(r, np.float64)
    assert np.all(np.isfinite(g)), f"{what}: non-finite GPU values"
    if r.size == 0:
        return 0.0
    num = np.abs(g - r).max(axis=-1)
    ref = np.abs(r).max(axis=-1)
    top = max(float(ref.max()), 1e-30)
    e = float((num / np.maximum(ref, floor * top)).max())
    for f in SPREAD:                        # the same rule at other floors, for the record
        SPREAD[f] = max(SPREAD[f], float((num / np.maximum(ref, f * top)).max()))
    WORST.append((e, what))
    assert e <= tol, f"{what}: max head-vector error {e:.3e} > {tol} (floor {floor} of the slab)"
    return e


SPREAD = {1.0: 0.0, 0.5: 0.0, 0.25: 0.0, 1 / 8: 0.0, 1 / 16: 0.0, 1 / 64: 0.0}


def oracle_grads(st, Q, dO, Hq, theta, seqs, group_of):
    """Reverse mode of attend_state: dq [L][S][B][Hq][hd] and, per group, the
    committed keys' gradients summed over the group's sequences
    ({grp: (dK, dV)} with [L][n][Hkv][hd]), and per sequence the carry keys'."""
    L, S, B, _, hd = Q.shape
    Hkv = st.Hkv
    G = Hq // Hkv
    ctx = st.ctx_len()
    dq = np.zeros(Q.shape)
    com, car = {}, {}
    for s in seqs:
        nc = int(ctx[s])
        nu = st.uk[s].shape[1]
        grp = group_of(s)
        if grp not in com:
            com[grp] = [np.zeros((L, 0, Hkv, hd)), np.zeros((L, 0, Hkv, hd))]
        for i in range(2):   # grow to this sequence's committed length
            have = com[grp][i].shape[1]
            if have < nc:
                com[grp][i] = np.concatenate([com[grp][i], np.zeros((L, nc - have, Hkv, hd))], 1)
        car[s] = [np.zeros((L, nu, Hkv, hd)), np.zeros((L, nu, Hkv, hd))]
        for layer in range(L):
            for g in range(Hkv):
                k, v = st.context(s, layer, g)
                heads = list(range(g * G, (g + 1) * G))
                q = Q[layer, s][:, heads].reshape(B * G, hd)
                do = dO[layer, s][:, heads].reshape(B * G, hd)
                qpos = np.repeat(nc + np.arange(B), G)
                gq, gk, gv = oracle.attend_backward(q, qpos, k, v, do, theta)
                dq[layer, s][:, heads] = gq.reshape(B, G, hd)
                com[grp][0][layer, :nc, g] += gk[:nc]
                com[grp][1][layer, :nc, g] += gv[:nc]
                car[s][0][layer, :, g] = gk[nc:]
                car[s][1][layer, :, g] = gv[nc:]
    return dq, com, car


def grad_buffers(st):
    z = lambda t: torch.zeros(t.shape, dtype=torch.float32, device=t.device)
    return z(st["k_cache"]), z(st["v_cache"]), z(st["k_carry"]), z(st["v_carry"])


def gather_grad_committed(dk, dv, pt_row, layer, n):
    pos = torch.arange(n, device=dk.device)
    pages = pt_row[pos // 16].long()
    slots = (pos % 16).long()
    return to_np(dk[layer][pages, :, slots, :]), to_np(dv[layer][pages, :, :, slots])


def gather_grad_carry(dk, dv, s, layer, n):
    r = torch.arange(n, device=dk.device)
    return (to_np(dk[layer, s][r // 16, :, r % 16, :]), to_np(dv[layer, s][r // 16, :, :, r % 16]))


def check(co, dims, st, q, out, lse, dO_dev, group, orc_st, Q, dO, w, seqs, group_of, leaders,
          layer_begin=0, layer_count=None, tag="", floor=FLOOR_PATH):
    layer_count = w.L if layer_count is None else layer_count
    dk, dv, dkc, dvc = grad_buffers(st)
    dq = torch.zeros((layer_count,) + tuple(q.shape[1:]), dtype=torch.float32, device="cuda")
    ws = torch.zeros(co.workspace_bytes(dims, co.CO_WS_ATTENTION_BACKWARD) + 256,
                     dtype=torch.uint8, device="cuda")
    co.drafter_block_attention_backward(dims, layer_begin, layer_count,
                                        q[layer_begin:layer_begin + layer_count], st, out, lse,
                                        dO_dev, group, dq, dk, dv, dkc, dvc, ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(st) == 0
    rq, rcom, rcar = oracle_grads(orc_st, Q, dO, w.Hq, w.theta, seqs, group_of)
    gq = to_np(dq)
    G = w.Hq // w.Hkv
    errs = []
    for s in seqs:
        for li, layer in enumerate(range(layer_begin, layer_begin + layer_count)):
            for g in range(w.Hkv):
                heads = list(range(g * G, (g + 1) * G))
                errs.append(slab_close(gq[li, s][:, heads].reshape(-1, w.hd),
                                       rq[layer, s][:, heads].reshape(-1, w.hd),
                                       f"{tag} dq s{s} l{layer} g{g}", floor=floor))
        nu = orc_st.uk[s].shape[1]
        if nu:
            for layer in range(layer_begin, layer_begin + layer_count):
                gk, gv = gather_grad_carry(dkc, dvc, s, layer, nu)
                for g in range(w.Hkv):
                    errs.append(slab_close(gk[:, g], rcar[s][0][layer, :, g],
                                           f"{tag} dk carry s{s} g{g}", floor=floor))
                    errs.append(slab_close(gv[:, g], rcar[s][1][layer, :, g],
                                           f"{tag} dv carry s{s} g{g}", floor=floor))
    pt = st["page_table"]
    for grp, (rk, rv) in rcom.items():
        n = rk.shape[1]
        if n == 0:
            continue
        for layer in range(layer_begin, layer_begin + layer_count):
            gk, gv = gather_grad_committed(dk, dv, pt[leaders[grp]], layer, n)
            for g in range(w.Hkv):
                errs.append(slab_close(gk[:, g], rk[layer, :, g], f"{tag} dk group {grp} g{g}",
                                   floor=floor))
                errs.append(slab_close(gv[:, g], rv[layer, :, g], f"{tag} dv group {grp} g{g}",
                                   floor=floor))
    print(f"[backward] {tag}: max head-vector error {max(errs):.3e} over {len(errs)} slabs; "
          "worst: " + ", ".join(f"{n} {e:.2e}" for e, n in sorted(WORST)[-3:])
          + "; at other floors: " + ", ".join(f"{f:g}: {e:.2e}" for f, e in SPREAD.items()),
          flush=True)
    WORST.clear()
    for f in SPREAD:
        SPREAD[f] = 0.0
    return errs


def test_backward_train_layout():
    co = _gpu()
    from helpers import OracleTrain
    from synth.scenario import TrainScenario
    from synth import device as sdev
    w = TRAIN_SMALL
    V, A = w.S * w.anchors, w.anchors
    print(f"[backward] workload={w.name} blocks={V}", flush=True)
    sc = TrainScenario(w)
    out, lse = sc.forward(shared_prefix=True)
    dO_dev = sdev.materialise(w, wl.spec_dout(w, S=V), "cuda")
    torch.cuda.synchronize()
    orc = OracleTrain(w, range(V))
    Q = seq_block(w, wl.spec_q(w, 0, S=V), 1, range(V))
    dO = host(w, wl.spec_dout(w, S=V))
    check(co, sc.vdims, sc.vst, sc.q, out, lse, dO_dev, A, orc.st, Q, dO, w, list(range(V)),
          lambda v: v // A, {r: r * A for r in range(w.S)}, tag="train")


def test_backward_train_full_size_sampled():
    """The training layout at full size (8 responses x 4096 positions, 2048
    anchored blocks), as the bench runs it: every block of response 0 against
    the oracle, including the sums over its 256 blocks of the shared keys."""
    co = _gpu()
    from helpers import OracleTrain
    from synth.scenario import TrainScenario
    from synth import device as sdev
    w = wl.TRAIN_FWD
    V, A = w.S * w.anchors, w.anchors
    print(f"[backward] workload={w.name} blocks={V}, response 0 checked", flush=True)
    sc = TrainScenario(w)
    out, lse = sc.forward(shared_prefix=True)
    dO_dev = sdev.materialise(w, wl.spec_dout(w, S=V), "cuda")
    torch.cuda.synchronize()
    sample = list(range(A))
    orc = OracleTrain(w, sample)
    Q = seq_block(w, wl.spec_q(w, 0, S=V), 1, sample)
    dO = seq_block(w, wl.spec_dout(w, S=V), 1, sample)
    check(co, sc.vdims, sc.vst, sc.q, out, lse, dO_dev, A, orc.st, Q, dO, w, sample,
          lambda v: v // A, {0: 0}, tag="train full")


def test_backward_serving_layout():
    co = _gpu()
    from synth.scenario import Scenario
    from synth import device as sdev
    w = SERVE
    sc, orc = Scenario(w), OracleRun(w)
    # sequence 4 empty, sequence 5 carry rows only
    for r in range(3):
        hidden, q, draft, target, m = sc.round_inputs(r)
        out, lse = sc.new_output()
        co.carryover_round(sc.dims, sc.W, hidden, draft, target, q, sc.st, sc.rt, out, lse, 0,
                           sc.ws)
        orc.round(r, attend=False)
    torch.cuda.synchronize()
    # one sequence without keys, and one with carry rows only
    sc.st["ctx_len"][4] = 0
    sc.st["carry_len"][4] = 0
    orc.st.ck[4] = orc.st.ck[4][:, :0]
    orc.st.cv[4] = orc.st.cv[4][:, :0]
    orc.st.uk[4] = orc.st.uk[4][:, :0]
    orc.st.uv[4] = orc.st.uv[4][:, :0]
    with_carry = [s for s in range(w.S) if s != 4 and orc.st.uk[s].shape[1] > 0]
    if with_carry:
        sc_only = with_carry[-1]
        sc.st["ctx_len"][sc_only] = 0
        orc.st.ck[sc_only] = orc.st.ck[sc_only][:, :0]
        orc.st.cv[sc_only] = orc.st.cv[sc_only][:, :0]
    _, q, _, _, _ = sc.round_inputs(3)
    out, lse = sc.new_output()
    co.drafter_block_attention(sc.dims, 0, w.L, q, sc.st, out, lse, 0, sc.ws)
    dO_dev = sdev.materialise(w, wl.spec_dout(w), "cuda")
    torch.cuda.synchronize()
    Q = host(w, wl.spec_q(w, 3))
    dO = host(w, wl.spec_dout(w))
    seqs = list(range(w.S))
    print(f"[backward] workload={w.name} layers 0..{w.L - 1}", flush=True)
    check(co, sc.dims, sc.st, q, out, lse, dO_dev, 1, orc.st, Q, dO, w, seqs, lambda s: s,
          {s: s for s in seqs}, tag="serve")
    # the second layer alone: its forward output and LSE are the slices of layer 1
    print(f"[backward] workload={w.name} layer 1 alone", flush=True)
    Q1 = Q.copy()
    dO1 = dO.copy()
    dO1[0] = 0.0
    check(co, sc.dims, sc.st, q, out[1:], lse[1:], dO_dev[1:], 1, orc.st, Q1, dO1, w, seqs,
          lambda s: s, {s: s for s in seqs}, layer_begin=1, layer_count=1, tag="serve l1")


def test_backward_group_mismatch_sets_status():
    """Sequences declared as one group whose page rows differ: CO_ERR_GROUP."""
    co = _gpu()
    from synth.scenario import Scenario
    w = SERVE.replace(name="bwd_group", S=4, L=1, rounds=2, seed=0x5EED32)
    sc = Scenario(w)
    _, q, _, _, _ = sc.round_inputs(0)
    out, lse = sc.new_output()
    co.drafter_block_attention(sc.dims, 0, w.L, q, sc.st, out, lse, 0, sc.ws)
    dk, dv, dkc, dvc = grad_buffers(sc.st)
    dq = torch.zeros(q.shape, dtype=torch.float32, device="cuda")
    ws = torch.zeros(co.workspace_bytes(sc.dims, co.CO_WS_ATTENTION_BACKWARD) + 256,
                     dtype=torch.uint8, device="cuda")
    co.drafter_block_attention_backward(sc.dims, 0, w.L, q, sc.st, out, lse, out, 2, dq, dk, dv,
                                        dkc, dvc, ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.st) == co.CO_ERR_GROUP


def test_projection_backward_train_layout():
    """The whole training backward of the second pass: attention backward,
    then the projection backward of the forward's two projection calls (the
    recorded responses' committed rows, then the blocks' carried rows), summed
    into dW_F, dW_KV and dE_carry; against the oracle's reverse modes."""
    co = _gpu()
    from helpers import OracleTrain
    from synth.scenario import TrainScenario
    from synth import device as sdev
    w = TRAIN_SMALL
    V, A = w.S * w.anchors, w.anchors
    print(f"[backward] projection, workload={w.name} blocks={V}", flush=True)
    sc = TrainScenario(w)
    out, lse = sc.forward(shared_prefix=True)
    dO_dev = sdev.materialise(w, wl.spec_dout(w, S=V), "cuda")
    dk, dv, dkc, dvc = grad_buffers(sc.vst)
    dq = torch.zeros(tuple(sc.q.shape), dtype=torch.float32, device="cuda")
    ws = torch.zeros(co.workspace_bytes(sc.vdims, co.CO_WS_ATTENTION_BACKWARD) + 256,
                     dtype=torch.uint8, device="cuda")
    co.drafter_block_attention_backward(sc.vdims, 0, w.L, sc.q, sc.vst, out, lse, dO_dev, A, dq,
                                        dk, dv, dkc, dvc, ws)
    n_kv = 2 * w.L * w.Hkv * w.hd
    dwf = torch.zeros((w.d, w.Dcat), dtype=torch.float32, device="cuda")
    dwkv = torch.zeros((n_kv, w.d), dtype=torch.float32, device="cuda")
    de = torch.zeros(w.Dcat, dtype=torch.float32, device="cuda")
    for dims, hidden, rt in ((sc.dims, sc.h_committed, sc.crt), (sc.vdims, sc.hidden, sc.vrt)):
        pws = torch.zeros(co.workspace_bytes(dims, co.CO_WS_PROJECT_BACKWARD) + 256,
                          dtype=torch.uint8, device="cuda")
        co.carryover_project_kv_backward(dims, sc.W, hidden, rt, dk, dv, dkc, dvc, dwf, dwkv, de,
                                         pws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.vst) == 0

    orc = OracleTrain(w, range(V))
    Q = seq_block(w, wl.spec_q(w, 0, S=V), 1, range(V))
    dO = host(w, wl.spec_dout(w, S=V))
    _, com, car = oracle_grads(orc.st, Q, dO, w.Hq, w.theta, range(V), lambda v: v // A)
    ref = [np.zeros((w.d, w.Dcat)), np.zeros((n_kv, w.d)), np.zeros(w.Dcat)]

    def add(grads):
        for i in range(3):
            ref[i] += grads[i]

    shape = (w.seq_len, w.L, w.Hkv, w.hd)
    for s in range(w.S):   # committed rows of every response, positions 0..seq_len-1
        h = host(w, wl.spec_hctx(w, s, 0, w.seq_len))
        gk, gv = np.zeros(shape), np.zeros(shape)
        n = com[s][0].shape[1]
        gk[:n] = com[s][0].transpose(1, 0, 2, 3)
        gv[:n] = com[s][1].transpose(1, 0, 2, 3)
        add(oracle.project_backward(h, orc.E, np.zeros(w.seq_len, bool), orc.WF, orc.WKV,
                                    np.arange(w.seq_len), w.L, w.Hkv, w.hd, w.theta, gk, gv))
    H = host(w, wl.spec_h(w, 0, S=V))   # [V][B][Dcat]
    rows, pos, gk, gv = [], [], [], []
    for v in range(V):                  # carried rows of every block
        for j in range(w.B):
            dst = int(orc.rr["row_dst"][v][j])
            if dst < 0 and dst != oracle.SKIP:
                c = -1 - dst
                rows.append(H[v, j])
                pos.append(int(orc.rr["row_pos"][v][j]))
                gk.append(car[v][0][:, c])
                gv.append(car[v][1][:, c])
    add(oracle.project_backward(np.array(rows), orc.E, np.ones(len(rows), bool), orc.WF, orc.WKV,
                                np.array(pos), w.L, w.Hkv, w.hd, w.theta, np.array(gk),
                                np.array(gv)))
    for name, g, r in (("dW_F", dwf, ref[0]), ("dW_KV", dwkv, ref[1]), ("dE", de, ref[2])):
        e = slab_close(to_np(g).reshape(1, -1), r.reshape(1, -1), name)
        print(f"[backward] {name}: error {e:.3e} of the largest reference value", flush=True)


# ------------------------------------------- the attention backward on its own

def _all_rows_spec(w, which, n_seqs, n_rows):
    """Directly drawn rows [n_seqs][L][Hkv][n_rows][hd] at logical positions
    CARRY_T0.. of every sequence: element (s, l, g, r, :) is the element
    (l, g, r, :) of spec_kv_direct(w, which, s, CARRY_T0, n_rows)."""
    st_, shape, strides, base, sigma = wl.spec_kv_direct(w, which, 0, CARRY_T0, n_rows)
    per_seq = w.L * w.Hkv * wl.TCAP * w.hd
    return st_, (n_seqs,) + shape, (per_seq,) + strides, base, sigma


def _direct_carry(w, st, n_seqs, n_rows):
    """Fill rows 0..n_rows-1 of every sequence's carry segment with directly
    drawn keys and values (device side)."""
    from synth import device as sdev
    k = sdev.materialise(w, _all_rows_spec(w, "k", n_seqs, n_rows), "cuda")   # [S][L][Hkv][n][hd]
    v = sdev.materialise(w, _all_rows_spec(w, "v", n_seqs, n_rows), "cuda")
    r = torch.arange(n_rows, device="cuda")
    # k_carry [L][S][CP][Hkv][16][hd], v_carry [L][S][CP][Hkv][hd][16]
    st["k_carry"][:, :, r // 16, :, r % 16, :] = k.permute(3, 1, 0, 2, 4)
    st["v_carry"][:, :, r // 16, :, :, r % 16] = v.permute(3, 1, 0, 2, 4)


def _oracle_carry(w, orc_st, s, nu):
    """The same carry rows of sequence s on the host: [L][nu][Hkv][hd]."""
    k = host(w, wl.spec_kv_direct(w, "k", s, CARRY_T0, nu)).transpose(0, 2, 1, 3)
    v = host(w, wl.spec_kv_direct(w, "v", s, CARRY_T0, nu)).transpose(0, 2, 1, 3)
    orc_st.uk[s] = k
    orc_st.uv[s] = v


def test_backward_direct_kv_serving():
    """The attention backward alone, serving layout (one sequence per group):
    committed and carry keys and values drawn directly, so the GPU and the
    oracle read identical bf16 inputs.  Ragged contexts, a full carry block,
    an empty sequence, a carry-only sequence, padded query rows (8 block rows
    x 2 heads), two layers; per head vector at 2e-2 with the floor at 1/8 of
    the slab."""
    co = _gpu()
    from synth.scenario import Scenario
    from synth import device as sdev
    w = SERVE.replace(name="bwd_direct_serve", seed=0x5EED33)
    print(f"[backward] direct K/V, workload={w.name}", flush=True)
    sc = Scenario(w)
    orc = OracleRun(w)
    carry = np.array([w.B, 0, 3, 1, 0, 5], np.int32)[:w.S]
    ctx = wl.initial_ctx(w).astype(np.int32).copy()
    ctx[4] = 0                                  # no keys at all
    ctx[5] = 0                                  # carry rows only
    _direct_carry(w, sc.st, w.S, w.B)
    sc.st["ctx_len"].copy_(torch.from_numpy(ctx))
    sc.st["carry_len"].copy_(torch.from_numpy(carry))
    for s in range(w.S):
        orc.st.ck[s] = orc.st.ck[s][:, :ctx[s]]
        orc.st.cv[s] = orc.st.cv[s][:, :ctx[s]]
        _oracle_carry(w, orc.st, s, int(carry[s]))
    q = sdev.materialise(w, wl.spec_q(w, 0), "cuda")
    out, lse = sc.new_output()
    co.drafter_block_attention(sc.dims, 0, w.L, q, sc.st, out, lse, 0, sc.ws)
    dO_dev = sdev.materialise(w, wl.spec_dout(w), "cuda")
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.st) == 0
    Q = host(w, wl.spec_q(w, 0))
    dO = host(w, wl.spec_dout(w))
    seqs = list(range(w.S))
    check(co, sc.dims, sc.st, q, out, lse, dO_dev, 1, orc.st, Q, dO, w, seqs, lambda s: s,
          {s: s for s in seqs}, tag="direct serve", floor=FLOOR_UNIT)


def test_backward_direct_kv_train_full_size():
    """The attention backward alone in the training layout at full size (8
    responses x 4096 positions, 2048 anchored blocks sharing their response's
    pages, one group per response): every key and value drawn directly; the
    256 blocks of response 2 against the oracle, including the sums over
    those blocks of the shared keys' gradients; per head vector at 2e-2 with
    the floor at 1/8 of the slab."""
    co = _gpu()
    from synth import device as sdev
    w = wl.TRAIN_FWD
    S, A, B = w.S, w.anchors, w.B
    V = S * A
    R = 2                                       # the response checked
    print(f"[backward] direct K/V, workload={w.name} blocks={V}, response {R} checked",
          flush=True)
    pt = wl.page_table(w)
    P = w.max_pages_per_seq
    dims = co.make_dims(S, w.seq_len, w.Dcat, w.d, w.L, w.Hq, w.Hkv, w.hd, P, pt.size, w.dtype,
                        w.theta)
    st = co.alloc_state(dims, pt, "cuda")
    for s in range(S):
        k = sdev.materialise(w, wl.spec_kv_direct(w, "k", s, 0, w.seq_len), "cuda")
        v = sdev.materialise(w, wl.spec_kv_direct(w, "v", s, 0, w.seq_len), "cuda")
        co.carryover_import_kv(dims, s, 0, k, v, st)
        del k, v
    a, u, a2 = wl.anchors(w)
    vdims = co.make_dims(V, B, w.Dcat, w.d, w.L, w.Hq, w.Hkv, w.hd, P, pt.size, w.dtype,
                         w.theta)
    vst = co.alloc_state(vdims, np.repeat(pt, A, axis=0), "cuda")
    vst["k_cache"], vst["v_cache"] = st["k_cache"], st["v_cache"]
    vst["ctx_len"].copy_(torch.from_numpy(a2.ravel().astype(np.int32)))
    vst["carry_len"].copy_(torch.from_numpy(u.ravel().astype(np.int32)))
    _direct_carry(w, vst, V, B)
    q = sdev.materialise(w, wl.spec_q(w, 0, S=V), "cuda")
    out = torch.empty((w.L, V, B, w.Hq, w.hd), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((w.L, V, B, w.Hq), dtype=torch.float32, device="cuda")
    ws = torch.zeros(max(co.workspace_bytes(vdims, co.CO_WS_ROUND), 256), dtype=torch.uint8,
                     device="cuda")
    co.drafter_block_attention(vdims, 0, w.L, q, vst, out, lse, co.CO_ATTN_SHARED_PREFIX, ws)
    dO_dev = sdev.materialise(w, wl.spec_dout(w, S=V), "cuda")
    torch.cuda.synchronize()
    assert co.carryover_read_status(vst) == 0

    sample = list(range(R * A, (R + 1) * A))
    ost = oracle.State(V, w.L, w.Hkv, w.hd)
    kr = host(w, wl.spec_kv_direct(w, "k", R, 0, w.seq_len)).transpose(0, 2, 1, 3)
    vr = host(w, wl.spec_kv_direct(w, "v", R, 0, w.seq_len)).transpose(0, 2, 1, 3)
    a2f, uf = a2.ravel(), u.ravel()
    for vv in sample:
        ost.set_committed(vv, kr[:, :a2f[vv]], vr[:, :a2f[vv]])
        _oracle_carry(w, ost, vv, int(uf[vv]))
    Q = seq_block(w, wl.spec_q(w, 0, S=V), 1, sample)
    dO = seq_block(w, wl.spec_dout(w, S=V), 1, sample)
    check(co, vdims, vst, q, out, lse, dO_dev, A, ost, Q, dO, w, sample, lambda v: v // A,
          {R: R * A}, tag="direct train", floor=FLOOR_UNIT)


# (S, B, Dcat, d, L, Hkv, hd): row counts around the staged 64, one and several
# row ranges, a Dcat that ends half a tile in, both head widths, several layers;
# the last takes the per-row products (few rows against wide weights)
PB_CASES = [(1, 1, 64, 64, 1, 1, 64), (3, 21, 320, 128, 1, 1, 64), (5, 13, 448, 192, 2, 1, 128),
            (1, 700, 256, 320, 1, 4, 64), (40, 16, 768, 256, 1, 2, 64), (9, 200, 1024, 64, 3, 2, 128),
            (2, 16, 4096, 2048, 1, 8, 64)]


@pytest.mark.parametrize("c", PB_CASES, ids=lambda c: "-".join(map(str, c)))
def test_projection_backward_products(c):
    """dW_F, dW_KV and dE against 64-bit products for rows that are committed,
    carried, skipped or point outside the caches, added to what the outputs
    hold.  dJ, and on the per-row path z and dz, are rounded to bf16: at most
    three relative errors of 2^-9 in every term."""
    import paper_2609_14717_amd as co
    S, B, Dcat, d, L, Hkv, hd = c
    print(f"[backward] projection products {c}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(S * 1000 + B)
    rnd = lambda *s, dt=torch.float32: torch.randn(s, generator=g, device="cuda").to(dt)  # noqa: E731
    M, CP, P = S * B, (B + 15) // 16, (S * B + 15) // 16 + 3
    n_kv = 2 * L * Hkv * hd
    dims = co.make_dims(S, B, Dcat, d, L, Hkv, Hkv, hd, P, P, "bf16", 1e4)
    wf, wkv, e = (rnd(*s, dt=torch.bfloat16) for s in ((d, Dcat), (n_kv, d), (Dcat,)))
    h = rnd(S, B, Dcat, dt=torch.bfloat16)
    dk, dv = rnd(L, P, Hkv, 16, hd), rnd(L, P, Hkv, hd, 16)
    dkc, dvc = rnd(L, S, CP, Hkv, 16, hd), rnd(L, S, CP, Hkv, hd, 16)
    kind = torch.randint(0, 4, (M,), generator=g, device="cuda")   # 0, 1 committed, 2 carried, 3 skipped
    r, j = torch.arange(M, device="cuda"), torch.arange(M, device="cuda") % B
    slot = torch.randperm(P * 16, generator=g, device="cuda")[:M]
    dst = torch.where(kind < 2, slot, torch.where(kind == 2, -1 - j, torch.full_like(r, co.SKIP)))
    if M > 8:
        dst[3], dst[7] = P * 16 + 5, -1 - CP * 16              # outside the caches: no gradient
    pos = torch.randint(0, 30000, (M,), generator=g, device="cuda")
    rt = dict(accept_len=torch.zeros(S, dtype=torch.int32, device="cuda"),
              row_pos=pos.to(torch.int32).view(S, B).contiguous(),
              row_dst=dst.to(torch.int32).view(S, B).contiguous())
    outs = [rnd(d, Dcat), rnd(n_kv, d), rnd(Dcat)]
    want = [o.double().clone() for o in outs]
    ws = torch.full((max(256, co.workspace_bytes(dims, co.CO_WS_PROJECT_BACKWARD)),), 255,
                    dtype=torch.uint8, device="cuda")          # NaN patterns
    co.carryover_project_kv_backward(dims, co.weights(wf, wkv, e), h, rt, dk, dv, dkc, dvc, *outs, ws)
    torch.cuda.synchronize()

    com, car = (dst >= 0) & (dst < P * 16), (dst < 0) & (dst >= -CP * 16)
    gk, gv = (torch.zeros((M, L, Hkv, hd), dtype=torch.float64, device="cuda") for _ in range(2))
    at = dst[com]
    gk[com] = dk[:, at // 16, :, at % 16].double()
    gv[com] = dv.permute(0, 1, 2, 4, 3)[:, at // 16, :, at % 16].double()
    at, s = -1 - dst[car], r[car] // B
    gk[car] = dkc[:, s, at // 16, :, at % 16].double()
    gv[car] = dvc.permute(0, 1, 2, 3, 5, 4)[:, s, at // 16, :, at % 16].double()
    i = torch.arange(hd // 2, device="cuda", dtype=torch.float64)
    ang = pos.double()[:, None] * 1e4 ** (-2 * i / hd)
    cs, sn = torch.cos(ang)[:, None, None], torch.sin(ang)[:, None, None]
    lo, hi = gk[..., :hd // 2], gk[..., hd // 2:]
    gk = torch.cat((lo * cs + hi * sn, hi * cs - lo * sn), -1)
    dj = torch.stack((gk, gv), 2).reshape(M, n_kv)
    carried = ((dst < 0) & (dst != co.SKIP)).double()[:, None]
    x = h.view(M, Dcat).double() + carried * e.double()
    G = dj.T @ x
    add = [wkv.double().T @ G, G @ wf.double().T, ((carried * dj).sum(0) @ wkv.double()) @ wf.double()]
    for name, o, w0, a in zip(("dW_F", "dW_KV", "dE"), outs, want, add):
        err = float((o.double() - w0 - a).norm() / (a.norm() + 1e-30)) if float(a.norm()) else 0.0
        print(f"  {name}: {err:.2e}", flush=True)
        assert err <= 3 * 2.0 ** -9, (name, err)
