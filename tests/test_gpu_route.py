"""GPU parity of the route step over wide windows (more rows than one
wavefront takes at a time): descriptors, lengths and status bit-exact against
the oracle, in every mode and with every error."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODES = {"carry": 0, "baseline": 1, "accept_all": 2, "carry_only": 4}


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("B", [64, 65, 127, 128, 1023, 1024, 1025, 2500])
def test_wide_window_route(B, mode):
    """First, middle and last rows of a workgroup's pass rejected, none
    rejected, a negative length, no capacity and page ids out of range."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14717_amd as co
    rng = np.random.default_rng(B)
    m = [0, 1, 63, 64, B // 2, B - 1, B, B, 5, B]
    m = [min(x, B) for x in m]
    S, P = len(m), (B + 40) // 16 + 1
    page = rng.permutation(S * P).astype(np.int32).reshape(S, P)
    ctx = rng.integers(0, 30, S).astype(np.int32)
    ctx[7] = -3                                           # CO_ERR_LENGTH
    ctx[8] = P * 16 - B + 1                               # CO_ERR_CAPACITY
    codes = [oracle.ERR_LENGTH, oracle.ERR_CAPACITY]
    page[9, (ctx[9] + B - 1) // 16] = S * P               # the last accepted row's page
    for bits in ((False,) if mode == "accept_all" else (False, True)):
        print(f"[route] B={B} {mode} bits={bits}", flush=True)
        target = rng.integers(0, 50, (S, B)).astype(np.int32)
        j = np.arange(B)[None]
        mm = np.array(m)[:, None]
        draft = np.where(j < mm, target, np.where(j == mm, target + 1, rng.integers(0, 50, (S, B))))
        if bits:
            draft = np.where(j < mm, 1, np.where(j == mm, 0, rng.integers(0, 2, (S, B))))
        draft = np.ascontiguousarray(draft.astype(np.int32))
        want = oracle.route(draft, target, ctx, np.full(S, 7), page, S * P, mode,
                            "bits" if bits else "tokens")
        dims = co.make_dims(S, B, 64, 64, 1, 1, 1, 64, P, S * P, "bf16", 1e4)
        st = co.alloc_state(dims, torch.from_numpy(page).cuda())
        st["ctx_len"].copy_(torch.from_numpy(ctx))
        st["carry_len"].fill_(7)
        rt = co.alloc_route(S, B)
        co.carryover_route(dims, torch.from_numpy(draft).cuda(), torch.from_numpy(target).cuda(),
                           MODES[mode] | (co.CO_ROUTE_ACCEPT_BITS if bits else 0), st, rt)
        torch.cuda.synchronize()
        for k in ("accept_len", "row_pos", "row_dst"):
            np.testing.assert_array_equal(rt[k].cpu().numpy(), want[k], err_msg=k)
        for k in ("ctx_len", "carry_len"):
            np.testing.assert_array_equal(st[k].cpu().numpy(), want[k], err_msg=k)
        bad = {int(x) for x in want["status"]} - {oracle.OK}
        assert set(codes) <= bad and co.carryover_read_status(st) in bad
