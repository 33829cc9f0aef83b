"""GPU parity of the full-precision round at the edges of its kernels: row tiles
of 32, K split over sixteen wavefronts (fewer steps than wavefronts included),
E staged and read where it is used, windows within and past one ballot, one and two
query tiles, segments of one chunk (256 keys, finished in place) and
of several (records and the merge)."""
import pytest

from synth import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from helpers import OracleRun, compare_round  # noqa: E402

BASE = wl.RAGGED32.replace(dtype="f32", L=1, rounds=3, accept=("geom", 0.25))
CASES = [
    # B, S, Dcat, d, Hq, Hkv, hd, contexts
    (1, 1, 64, 64, 1, 1, 64, 1, 1),            # one row, eight K steps, one key
    (8, 4, 192, 64, 4, 1, 64, 200, 247),       # 32 query rows; one chunk, its last pages
    (11, 3, 448, 192, 3, 1, 64, 230, 300),     # 33 rows, 33 query rows; one chunk and two
    (16, 2, 1088, 128, 4, 1, 64, 1000, 1100),  # 64 query rows
    (7, 5, 256, 320, 6, 2, 128, 5, 520),       # 21 query rows at head_dim 128
    (16, 2, 256, 128, 8, 2, 128, 15, 700),     # 64 query rows at head_dim 128
    (31, 1, 128, 64, 2, 1, 64, 17000, 17000),  # more than 64 chunks of 256 keys
    (5, 7, 4160, 64, 2, 1, 64, 10, 60),        # more E than is staged in LDS
    (16, 2, 4096, 64, 2, 1, 64, 10, 60),       # as much as is
    (33, 3, 256, 128, 1, 1, 64, 20, 300),      # windows one ballot of a row tile reaches back over,
    (34, 3, 256, 128, 1, 1, 64, 20, 300),      # and longer ones: every row reads its own tokens
    (64, 2, 4160, 64, 1, 1, 128, 20, 300),     # both
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "-".join(map(str, c)))
def test_f32_round_edges(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    from synth.scenario import Scenario
    B, S, Dcat, d, Hq, Hkv, hd, lo, hi = c
    w = BASE.replace(name="f32_edge", S=S, B=B, Dcat=Dcat, d=d, Hq=Hq, Hkv=Hkv, hd=hd, ctx_lo=lo,
                     ctx_hi=hi, seed=0x5EED30 + B + S)
    print(f"[f32] {c}", flush=True)
    sc, orc = Scenario(w), OracleRun(w)
    for r in range(2):
        hidden, q, draft, target, m = sc.round_inputs(r)
        out, lse = sc.new_output()
        co.carryover_round(sc.dims, sc.W, hidden, draft, target, q, sc.st, sc.rt, out, lse, 0, sc.ws)
        torch.cuda.synchronize()
        assert co.carryover_read_status(sc.st) == 0
        rr, O, LSE = orc.round(r)
        compare_round(sc, orc, rr, O, LSE, out, lse, sc.rt, orc.seqs, f"f32 {c} r{r}")
