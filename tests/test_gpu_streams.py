"""GPU parity of the head_dim 128 attention at the edges of its split: parts of
one segment merged in a workgroup, left as records and whole; the even split
where segments are too many or too uneven; one sequence per lane (64) and
several (65 and more); one and two query tiles; empty sequences; and, per case,
the extras of drafter_block_attention_ext against the stand-alone calls."""
import numpy as np
import pytest

from synth import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from helpers import OracleRun, compare_round  # noqa: E402

BASE = wl.RAGGED32.replace(Dcat=256, d=128, hd=128, theta=1e6, rounds=3, accept=("geom", 0.25))
CASES = [
    # S, B, L, Hq, Hkv, contexts
    (1, 16, 1, 8, 2, 2100, 2100),     # 64 rows: parts of 4 tiles, one record each
    (1, 7, 1, 6, 2, 2100, 2100),      # 21 rows: the parts of a workgroup merged
    (2, 1, 1, 1, 1, 1, 130),          # one query row; whole segments
    (3, 16, 2, 2, 1, 33, 600),        # 32 rows exactly, several layers
    (5, 11, 1, 3, 1, 100, 9000),      # 33 rows: two tiles, the second one row; uneven lengths
    (64, 4, 1, 8, 8, 1, 40),          # one sequence per lane
    (65, 4, 1, 8, 8, 1, 40),          # two per lane: the even split
    (130, 16, 1, 4, 1, 1, 300),       # three per lane, 64 rows, more pieces than streams
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "-".join(map(str, c)))
def test_stream_split_edges(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    from synth.scenario import Scenario
    S, B, L, Hq, Hkv, lo, hi = c
    w = BASE.replace(name="streams", S=S, B=B, L=L, Hq=Hq, Hkv=Hkv, ctx_lo=lo, ctx_hi=hi,
                     seed=0x5EED40 + S + B)
    print(f"[streams] {c}", flush=True)
    sc, orc = Scenario(w), OracleRun(w)
    for r, m in enumerate((None, [0, B] * (S // 2) + [B] * (S % 2))):
        hidden, q, draft, target, m = sc.round_inputs(r, m)
        out, lse = sc.new_output()
        co.carryover_round(sc.dims, sc.W, hidden, draft, target, q, sc.st, sc.rt, out, lse, 0, sc.ws)
        torch.cuda.synchronize()
        assert co.carryover_read_status(sc.st) == 0
        rr, O, LSE = orc.round(r, m=m)
        compare_round(sc, orc, rr, O, LSE, out, lse, sc.rt, orc.seqs, f"streams {c} r{r}")
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
    mk = lambda: (torch.randn(L, S, B, Hkv, 128, device="cuda") * 0.05).to(torch.bfloat16)  # noqa: E731
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
