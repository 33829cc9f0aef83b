"""GPU parity of the bf16 attention at the edges of its split and dispatch: parts of
one segment merged in a workgroup, left as records and whole; the even split
where segments are too many or too uneven; one sequence per lane (64) and
several (65 and more); one and two query tiles; empty sequences; and, per case,
the extras of drafter_block_attention_ext against the stand-alone calls; and the
path that each case takes."""
import numpy as np
import pytest

from synth import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from helpers import OracleRun, compare_round  # noqa: E402
from test_gpu_edge import SHAPES  # noqa: E402

BASE = wl.RAGGED32.replace(Dcat=256, d=128, hd=128, theta=1e6, rounds=3, accept=("geom", 0.25))
STREAMS, PERSISTENT = 1, 0   # as the attn_wave override
CASES = [
    # S, B, L, Hq, Hkv, contexts, head_dim, page table (0: as wide as the contexts), path
    (1, 16, 1, 8, 2, 2100, 2100, 128, 0, STREAMS),    # 64 rows: parts of 3 tiles, one record each
    (1, 7, 1, 6, 2, 2100, 2100, 128, 0, STREAMS),     # 21 rows: the parts of a workgroup merged
    (2, 1, 1, 1, 1, 1, 130, 128, 0, STREAMS),         # one query row; whole segments
    (3, 16, 2, 2, 1, 33, 600, 128, 0, STREAMS),       # 32 rows exactly, several layers
    (5, 11, 1, 3, 1, 100, 9000, 128, 0, STREAMS),     # 33 rows: two tiles, the second one row; uneven lengths
    (64, 4, 1, 8, 8, 1, 40, 128, 0, STREAMS),         # one sequence per lane
    (65, 4, 1, 8, 8, 1, 40, 128, 0, STREAMS),         # two per lane: the even split
    (130, 16, 1, 4, 1, 1, 300, 128, 0, STREAMS),      # three per lane, 64 rows, more pieces than streams
    # head_dim 64: more than 32 query rows
    (7, 16, 2, 8, 2, 1, 900, 64, 0, STREAMS),         # 64 rows
    (3, 13, 1, 3, 1, 100, 700, 64, 0, STREAMS),       # 39 rows
    (70, 16, 1, 4, 1, 1, 90, 64, 0, STREAMS),         # two sequences per lane, 64 rows
    # the persistent kernel, its records merged by one wavefront an item or by four
    (1, 16, 1, 4, 2, 4000, 4000, 64, 0, PERSISTENT),  # two segments, over a hundred records each
    (6, 5, 1, 4, 2, 1, 700, 64, 0, PERSISTENT),       # 10 rows: items past the last in the last workgroup
    (12, 3, 1, 4, 4, 1, 300, 64, 0, PERSISTENT),      # 48 segments, and one more row of them
    (13, 3, 1, 4, 4, 1, 300, 64, 0, PERSISTENT),
    (3, 16, 1, 6, 2, 30, 192, 64, 0, PERSISTENT),     # 48 rows: a table of 16 pages, one of 17,
    (3, 16, 1, 6, 2, 30, 193, 64, 0, STREAMS),        # and one of 400 over the same contexts
    (3, 16, 1, 6, 2, 30, 192, 64, 400, STREAMS),
    (3, 16, 1, 8, 2, 30, 192, 64, 0, STREAMS),        # 64 rows: any table
    # head_dim 128, up to 16 rows: 255 and 256 segments, tables of 131072 pages in all
    # and just under it, whatever the contexts
    (51, 16, 1, 5, 5, 1, 200, 128, 520, STREAMS),
    (32, 16, 1, 8, 8, 1, 200, 128, 512, PERSISTENT),
    (32, 16, 1, 8, 8, 1, 200, 128, 511, STREAMS),
    (32, 9, 1, 16, 8, 1, 200, 128, 512, STREAMS),     # 18 rows: any table
    # few and short segments in a wide table: whole workgroups to a segment, places
    # left free in them, segments of one tile, two rows of jobs out of four
    (4, 16, 1, 8, 8, 1, 16, 128, 300, STREAMS),
    (4, 15, 1, 16, 8, 20, 60, 128, 300, STREAMS),
    (17, 15, 1, 8, 4, 80, 140, 128, 300, STREAMS),
    (3, 16, 1, 2, 1, 33, 600, 128, 300, STREAMS),
]


def widen(co, sc, pages):
    """The scenario's sequences in a page table of ``pages`` columns."""
    w, pt = sc.w, sc.st["page_table"]
    more = torch.zeros((w.S, pages - pt.shape[1]), dtype=torch.int32, device="cuda")
    sc.st["page_table"] = torch.cat((pt, more), 1).contiguous()
    sc.dims = co.make_dims(w.S, w.B, w.Dcat, w.d, w.L, w.Hq, w.Hkv, w.hd, pages, sc.dims.num_pages,
                           w.dtype, w.theta)
    sc.ws = torch.zeros(co.workspace_bytes(sc.dims, co.CO_WS_ROUND), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("c", CASES, ids=lambda c: "-".join(map(str, c)))
def test_stream_split_edges(c, tune):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    from synth.scenario import Scenario
    S, B, L, Hq, Hkv, lo, hi, hd, pages, path = c
    w = BASE.replace(name="streams", S=S, B=B, L=L, Hq=Hq, Hkv=Hkv, hd=hd, ctx_lo=lo, ctx_hi=hi,
                     seed=0x5EED40 + S + B)
    print(f"[streams] {c}", flush=True)
    sc, orc = Scenario(w), OracleRun(w)
    if pages:
        widen(co, sc, pages)
    for r, m in enumerate((None, [0, B] * (S // 2) + [B] * (S % 2))):
        hidden, q, draft, target, m = sc.round_inputs(r, m)
        out, lse = sc.new_output()
        co.carryover_round(sc.dims, sc.W, hidden, draft, target, q, sc.st, sc.rt, out, lse, 0, sc.ws)
        torch.cuda.synchronize()
        assert co.carryover_read_status(sc.st) == 0
        rr, O, LSE = orc.round(r, m=m)
        compare_round(sc, orc, rr, O, LSE, out, lse, sc.rt, orc.seqs, f"streams {c} r{r}")
    def taken(wave):
        """The call's output and the path it took: the streams' header in the workspace
        is 2 S + 4 words, the persistent kernel's goes on with its slices' starts."""
        tune("attn_wave", wave)
        x, z = sc.new_output()
        ws = torch.full((co.workspace_bytes(sc.dims, co.CO_WS_ATTENTION),), 255, dtype=torch.uint8, device="cuda")
        co.drafter_block_attention(sc.dims, 0, L, q, sc.st, x, z, 0, ws)
        word = int(ws[:4 * (2 * S + 5)].view(torch.int32)[2 * S + 4])
        return x, z, STREAMS if word == -1 else PERSISTENT

    both = {}
    for wave in (PERSISTENT, STREAMS):
        x, z, by = both[wave] = taken(wave)
        assert by == wave
        torch.testing.assert_close(x.float(), out.float(), rtol=2e-2, atol=2e-2 * float(out.float().abs().max()))
        torch.testing.assert_close(z, lse, rtol=1e-5, atol=1e-3)
    x, z, by = taken(-1)
    assert by == path and torch.equal(x, out) and torch.equal(x, both[path][0]) and torch.equal(z, both[path][1])
    # sequences without keys among the others: O = 0, LSE = -inf
    sc.st["ctx_len"][::3] = 0
    sc.st["carry_len"][::3] = 0
    ws = torch.zeros(co.workspace_bytes(sc.dims, co.CO_WS_ATTENTION), dtype=torch.uint8, device="cuda")
    before = out.clone()
    co.drafter_block_attention(sc.dims, 0, L, q, sc.st, out, lse, 0, ws)
    assert co.carryover_read_status(sc.st) == 0
    assert not out[:, ::3].any() and bool((lse[:, ::3] == -np.inf).all())
    keep = [s for s in range(S) if s % 3]
    torch.testing.assert_close(out[:, keep].float(), before[:, keep].float(), rtol=2e-2, atol=2e-2 * float(
        before.float().abs().max()))
    # the extras: mass and self segment in the call, and as calls of their own
    mk = lambda: (torch.randn(L, S, B, Hkv, hd, device="cuda") * 0.05).to(torch.bfloat16)  # noqa: E731
    k_self, v_self, mass, mass2 = mk(), mk(), torch.empty_like(lse), torch.empty_like(lse)
    co.drafter_carry_mass(sc.dims, 0, L, q, sc.st, lse, mass2)
    co.drafter_self_merge(sc.dims, 0, L, q, k_self, v_self, sc.st, out, lse)
    out2, lse2 = torch.empty_like(out), torch.empty_like(lse)
    co.drafter_block_attention_ext(sc.dims, 0, L, q, k_self, v_self, sc.st, out2, lse2, mass, 0, ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.st) == 0
    torch.testing.assert_close(lse2, lse, rtol=1e-2, atol=1e-2)
    torch.testing.assert_close(mass, mass2, rtol=2e-2, atol=2e-3)
    torch.testing.assert_close(out2.float(), out.float(), rtol=2e-2, atol=2e-2 * float(
        out.float().abs().max()))


def attend64(dims, st, q, k_self=None, v_self=None):
    """The attention over [C;U(;S)] of the state's stored keys and values in 64 bits:
    out, lse and the mass on U of every query."""
    L, S, B, Hq, hd = q.shape
    H, G, half = dims.num_kv_heads, Hq // dims.num_kv_heads, hd // 2
    inv = dims.rope_theta ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half)

    def rotate(x, pos):   # x [n][heads][hd] at positions pos [n]
        ang = pos.double()[:, None, None] * inv
        cs, sn, lo, hi = torch.cos(ang), torch.sin(ang), x[..., :half], x[..., half:]
        return torch.cat((lo * cs - hi * sn, hi * cs + lo * sn), -1)

    def rows(K, V, n):    # pages K [p][H][16][hd], V [p][H][hd][16] -> [H][n][hd]
        return (K.transpose(0, 1).reshape(H, -1, hd)[:, :n].double(),
                V.permute(1, 0, 3, 2).reshape(H, -1, hd)[:, :n].double())

    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    lse, mass = (torch.zeros(q.shape[:-1], dtype=torch.float64, device="cuda") for _ in range(2))
    for s in range(S):
        n, u = int(st["ctx_len"][s]), int(st["carry_len"][s])
        pages, pos = st["page_table"][s, :-(-n // 16)].long(), n + torch.arange(B, device="cuda")
        for i in range(L):
            kv = [rows(st["k_cache"][i][pages], st["v_cache"][i][pages], n),
                  rows(st["k_carry"][i, s], st["v_carry"][i, s], u)]
            if k_self is not None:
                kv.append((rotate(k_self[i, s].double(), pos).transpose(0, 1),
                           v_self[i, s].double().transpose(0, 1)))
            k, v = (torch.cat([x[j] for x in kv], 1) for j in range(2))
            qr = rotate(q[i, s].double(), pos).view(B, H, G, hd).transpose(0, 1).reshape(H, B * G, hd)
            x = (qr @ k.transpose(1, 2).contiguous()) / hd ** 0.5
            z = torch.logsumexp(x, -1)
            p = torch.exp(x - z[..., None])
            m = p[..., n:n + u].sum(-1) / p[..., :n + u].sum(-1)
            back = lambda t: t.view(H, B, G, -1).transpose(0, 1).reshape(B, Hq, -1)  # noqa: E731
            out[i, s], lse[i, s], mass[i, s] = back(p @ v), back(z)[..., 0], back(m)[..., 0]
    return out, lse, mass


def random_state(S, B, G, hd, lo, hi, seed, scale=1.0, max_pages=None, Hkv=2, L=1):
    """(dims, state, q, own rows) of ragged sequences; logits of deviation ``scale``."""
    import paper_2609_14717_amd as co
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    n = [hi if S == 1 else lo + (hi - lo) * i // (S - 1) for i in range(S)]
    P = max(-(-(hi + 4 * B) // 16), 1)
    pt = torch.randperm(S * P, generator=g, device="cuda").to(torch.int32).view(S, P)
    if max_pages:
        pt = torch.cat((pt, torch.zeros((S, max_pages - P), dtype=torch.int32, device="cuda")), 1)
    dims = co.make_dims(S, B, 64, 64, L, Hkv * G, Hkv, hd, pt.shape[1], S * P, "bf16", 1e4)
    st = co.alloc_state(dims, pt.contiguous())
    for k in ("k_cache", "v_cache", "k_carry", "v_carry"):
        st[k].copy_(rnd(*st[k].shape))
    st["ctx_len"].copy_(torch.tensor(n, dtype=torch.int32))
    st["carry_len"].copy_(torch.tensor([(3 * s + 1) % (B + 1) for s in range(S)], dtype=torch.int32))
    q = (rnd(L, S, B, Hkv * G, hd).float() * scale).to(torch.bfloat16)
    own = rnd(L, S, B, Hkv, hd), rnd(L, S, B, Hkv, hd)
    return dims, st, q, own


@pytest.mark.parametrize("scale", [0.5, 1.0])
@pytest.mark.parametrize("B,G,hd", [(7, 1, 128), (16, 1, 128), (7, 3, 128), (16, 2, 128), (11, 3, 128), (16, 3, 128),
                                    (11, 3, 64), (16, 3, 64), (16, 4, 64)])
def test_stream_error(B, G, hd, scale, tune):
    """Where the streams take the persistent kernel's place their output is no further
    from 64 bits (1 %: the samples are some 10^4 and more independent values).
    Above 32 rows the weights keep 16 bits, which leaves two roundings to bf16: of the
    output, and of the queries, whose logits of deviation ``scale`` take ``scale``
    times its relative error.  That is 2^-8 / sqrt(3) of the binade, 0.7355 of it
    relative to values spread evenly over the logarithm: 1.66e-3 (and 5 %: the
    samples, and the block's own keys, rounded once rotated)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    dims, st, q, own = random_state(6, B, G, hd, 300, 1500, 100 * B + G + hd, scale)
    ws = torch.zeros(co.workspace_bytes(dims, co.CO_WS_ATTENTION), dtype=torch.uint8, device="cuda")
    print(f"[streams] error B={B} G={G} hd={hd} scale={scale}", flush=True)
    for extras in (False, True):
        ks, vs = own if extras else (None, None)
        O, LSE, MASS = attend64(dims, st, q, ks, vs)
        err = {}
        for path in (STREAMS, PERSISTENT):
            tune("attn_wave", path)
            out, lse = torch.empty_like(q), torch.empty(q.shape[:-1], device="cuda")
            mass = torch.empty_like(lse) if extras else None
            co.drafter_block_attention_ext(dims, 0, 1, q, ks, vs, st, out, lse, mass, 0, ws)
            torch.cuda.synchronize()
            assert co.carryover_read_status(st) == 0
            err[path] = float((out.double() - O).norm() / O.norm())
            torch.testing.assert_close(lse.double(), LSE, rtol=0, atol=1e-2)
            if extras:
                torch.testing.assert_close(mass.double(), MASS, rtol=2e-2, atol=1e-4)
        print(f"  extras={extras}: {err[STREAMS]:.3e} persistent {err[PERSISTENT]:.3e}", flush=True)
        assert err[STREAMS] <= 1.01 * err[PERSISTENT], err
        if B * G > 32:
            assert err[STREAMS] <= 1.05 * (1 + scale ** 2) ** 0.5 * 0.7355 * 2 ** -8 / 3 ** 0.5, err


MORE_SHAPES = [   # what SHAPES leaves to the parity suite: 32 rows at 64, 64 rows at 128
    SHAPES[0].replace(name="nt2_hd64", Hq=4, seed=0x5EED2B),
    SHAPES[3].replace(name="nt4_hd128", Hq=8, seed=0x5EED2C),
]


@pytest.mark.parametrize("wave", [PERSISTENT, STREAMS])
@pytest.mark.parametrize("w", SHAPES + MORE_SHAPES, ids=lambda w: w.name)
def test_every_instantiation(w, wave, tune):
    """Every query tile count of both paths, whichever the default takes, against the
    oracle; its extras (instantiations of their own) against the stand-alone calls."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    from synth.scenario import Scenario
    print(f"[streams] {w.name} attn_wave={wave}", flush=True)
    tune("attn_wave", wave)
    sc, orc = Scenario(w), OracleRun(w)
    hidden, q, draft, target, m = sc.round_inputs(0)
    out, lse = sc.new_output()
    co.carryover_round(sc.dims, sc.W, hidden, draft, target, q, sc.st, sc.rt, out, lse, 0, sc.ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.st) == 0
    rr, O, LSE = orc.round(0)
    compare_round(sc, orc, rr, O, LSE, out, lse, sc.rt, orc.seqs, f"{w.name} {wave}")
    k_self, v_self = sc.self_kv(0)
    mass, mass2 = torch.empty_like(lse), torch.empty_like(lse)
    co.drafter_carry_mass(sc.dims, 0, w.L, q, sc.st, lse, mass2)
    co.drafter_self_merge(sc.dims, 0, w.L, q, k_self, v_self, sc.st, out, lse)
    ws = torch.zeros(co.workspace_bytes(sc.dims, co.CO_WS_ATTENTION), dtype=torch.uint8, device="cuda")
    out2, lse2 = torch.empty_like(out), torch.empty_like(lse)
    co.drafter_block_attention_ext(sc.dims, 0, w.L, q, k_self, v_self, sc.st, out2, lse2, mass, 0, ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(sc.st) == 0
    torch.testing.assert_close(lse2, lse, rtol=1e-2, atol=1e-2)
    torch.testing.assert_close(mass, mass2, rtol=2e-2, atol=2e-3)
    torch.testing.assert_close(out2.float(), out.float(), rtol=2e-2, atol=2e-2 * float(
        out.float().abs().max()))


RAMPS = {"rising": (-300.0, 300.0), "falling": (300.0, -300.0), "low": (-260.0, -250.0),
         "small": (-2.0, 2.0), "edge": (-9.0, 9.0), "high": (250.0, 260.0)}


@pytest.mark.parametrize("hd,Hq,shared", [(64, 2, True), (64, 4, True), (64, 2, False), (128, 2, False),
                                          (128, 4, False), (128, 2, True)])
@pytest.mark.parametrize("ramp", list(RAMPS))
def test_softmax_reference(ramp, hd, Hq, shared):
    """Scores that rise, fall or stay far from 0 along the keys: the running
    reference is the first tile's maximum and follows later ones.
    Against 64 bits on the same bf16 inputs; P and O are rounded to bf16 (2^-8
    each at most, relative to the largest output of the row)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    S, B, n = 5, 16, 700
    print(f"[streams] reference {ramp} hd={hd} Hq={Hq} shared={shared}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(hd + Hq)
    P = n // 16 + 2
    pt = torch.arange(P, dtype=torch.int32, device="cuda").repeat(S, 1)
    dims = co.make_dims(S, B, 64, 64, 1, Hq, 1, hd, P, P, "bf16", 1e4)
    st = co.alloc_state(dims, pt)
    lo, hi = RAMPS[ramp]
    key = torch.zeros(P * 16, hd, device="cuda")
    key[:, 0] = torch.linspace(lo, hi, P * 16, device="cuda")   # the score, with q = sqrt(hd) e_0
    val = torch.randn(P * 16, hd, generator=g, device="cuda")
    key, val = key.to(torch.bfloat16), val.to(torch.bfloat16)
    st["k_cache"].copy_(key.view(1, P, 1, 16, hd))
    st["v_cache"].copy_(val.view(1, P, 1, 16, hd).transpose(3, 4))
    lens = [n, n - 1, 333, 31, 1]
    st["ctx_len"].copy_(torch.tensor(lens, dtype=torch.int32))
    q = torch.zeros(1, S, B, Hq, hd, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = (hd ** 0.5 * torch.linspace(0.5, 1.0, B * Hq, device="cuda")).view(B, Hq).to(torch.bfloat16)
    out, lse = torch.empty_like(q), torch.empty(q.shape[:-1], device="cuda")
    ws = torch.zeros(co.workspace_bytes(dims, co.CO_WS_ATTENTION), dtype=torch.uint8, device="cuda")
    co.drafter_block_attention(dims, 0, 1, q, st, out, lse, co.CO_Q_PREROTATED |
                               (co.CO_ATTN_SHARED_PREFIX if shared else 0), ws)
    torch.cuda.synchronize()
    assert co.carryover_read_status(st) == 0
    # the kernels scale the queries into log2 units and round them to bf16
    scale = torch.tensor(hd ** -0.5 * np.log2(np.e), dtype=torch.float32, device="cuda")
    qs = (q.float() * scale).to(torch.bfloat16).double() * np.log(2.0)
    for s, m in enumerate(lens):
        x = qs[0, s].reshape(B * Hq, hd) @ key[:m].double().T
        ref = torch.softmax(x, -1) @ val[:m].double()
        got = out[0, s].reshape(B * Hq, hd).double()
        err = (got - ref).abs().amax(-1) / ref.abs().amax(-1)
        assert float(err.max()) <= 2 * 2.0 ** -8, (s, float(err.max()))
        torch.testing.assert_close(lse[0, s].reshape(-1).double(), torch.logsumexp(x, -1), rtol=1e-5, atol=1e-3)
