"""The lane-per-token encoding kernel (kept counts of 16, 32 and 48) byte for
byte against the oracle, where it can go wrong: scores that tie at every cut,
candidates in every order, forced strategies of every group and block size,
truncated bitmaps, E4M3 values, both packing routes."""
import pytest
import torch

from _parity import assert_state_equal, oracle_pairs, params_pair
import paper_2607_00760_amd as M
from workloads import gen

pytestmark = pytest.mark.gpu

SMALL = dict(ctx=(1000, 64, 129), hkv=2)
CASES = {
    # rounded to few levels and unrotated: nearly every cut is a tie
    "ties_search": (dict(rotate=False, **SMALL), {}, 2.0),
    "ties_search_bf16": (dict(rotate=False, dtype="bf16", **SMALL), {}, 4.0),
    "ties_forced_g1": (dict(rotate=False, **SMALL), dict(force_default=True, default=(48, 1, 16)), 2.0),
    "ties_forced_g2": (dict(rotate=False, **SMALL), dict(force_default=True, default=(16, 2, 4)), 2.0),
    "ties_forced_g4": (dict(rotate=False, **SMALL), dict(force_default=True, default=(32, 4, 8)), 2.0),
    "ties_truncated": (dict(rotate=False, **SMALL), dict(trunc=96), 2.0),
    "zeros": (dict(rotate=False, **SMALL), {}, 0.0),
    # candidates in other orders, thresholds that reach the last of each list
    "order_large_first": (SMALL, dict(keep_cand=(48, 32, 16), group_cand=(1, 2, 4), block_cand=(4, 8, 16)), None),
    "order_mixed": (SMALL, dict(keep_cand=(32, 16, 48), group_cand=(2, 1, 4), block_cand=(8, 4, 16), tau_channel=0.15), None),
    "repeated": (SMALL, dict(keep_cand=(32, 32, 32), group_cand=(2, 2, 2), block_cand=(8, 8, 8)), None),
    "never_passes": (SMALL, dict(tau_channel=0.0, tau_block=0.0), None),
    "always_passes": (SMALL, dict(tau_channel=1e9, tau_block=1e9), None),
    "all_kept_t32": (SMALL, dict(trunc=32, keep_cand=(16, 32, 32), tau_channel=0.2), None),
    "fp8_truncated_32": (SMALL, dict(fp8=True, trunc=32, keep_cand=(16, 32, 16), tau_channel=0.5), None),
    "fp8_g4": (SMALL, dict(fp8=True, force_default=True, default=(16, 4, 4)), None),
    "many_windows": (dict(rot_window=128, **SMALL), {}, None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_encode_matches_oracle(name):
    over, extra, levels = CASES[name]
    spec = gen.spec("c2", **over)
    cap = spec.max_ctx + 70
    lay = gen.make_layer(spec, 0, capacity=cap)
    if levels is not None:
        for which in ("k", "v"):                               # a few magnitudes, both signs, signed zeros
            x = (lay[which].float() * levels).round().clamp(-3, 3)
            x[..., ::7] = -0.0
            lay[which] = x.to(lay[which].dtype)
    lp, op = params_pair(spec, **extra)
    ops = oracle_pairs(op, spec, lay, cap)
    for single in (True, False):
        c = M.MosaicCache(lp, spec.num_seqs, cap, rotated=spec.rotate, device="cuda")
        rk = lay["rot_k"].cuda() if spec.rotate else None
        rv = lay["rot_v"].cuda() if spec.rotate else None
        c.compress(lay["k"].cuda(), lay["v"].cuda(), lay["ctx_lens"], rk, rv, single_pass=single)
        torch.cuda.synchronize()
        for p in range(spec.num_seqs * spec.hkv):
            assert_state_equal(c, p, ops[p], where=f"{name} single={single}")
