"""Decode parity where the split plan, the scoring grid and the combine change
form: the three plans (fixed on the host for caches of one window, in registers
for up to 128 pairs of up to 16 windows, general beyond, and both of these for
one-window batches too uneven for the fixed one), one to three windows (fused
and two-kernel combine, for two windows of eight heads by the number of pairs), selections of a few blocks, every block size with all
channels kept, and update buffers of 1 to 31 tokens.  Scores and selections bit for bit, outputs against the fp64 oracle
within the bound of the parity tests."""
import numpy as np
import pytest
import torch

from _parity import assert_close, gpu_cache, gpu_scores_sel, oracle_decode_all, oracle_pairs, params_pair, scale_of
from workloads import gen

pytestmark = pytest.mark.gpu

MANY = tuple(70 + 37 * (i % 9) for i in range(33))              # 132 pairs of 4 kv heads
CASES = {
    # three windows: the general plan, whose loops take the pairs 128 at a time, and the register plan's last
    "many_pairs": (dict(ctx=MANY, hkv=4, rot_window=128), {}),
    "at_128_pairs": (dict(ctx=MANY[:32], hkv=4, group=8, rot_window=128), {}),
    "one_window_132_pairs": (dict(ctx=MANY, hkv=4), {}),
    "one_window_128_pairs": (dict(ctx=MANY[:32], hkv=4, group=8), {}),
    # a fixed plan would need more than four places for every workgroup the chip holds
    "uneven_128_pairs": (dict(ctx=(6000,) + (70,) * 127, hkv=1), dict(select=(1, 1))),
    "uneven_160_pairs": (dict(ctx=(70,) * 100 + (6000,) + (81,) * 59, hkv=1), dict(select=(1, 1))),
    "windows_1": (dict(ctx=(1000, 500), hkv=2, rot_window=4096), {}),
    "windows_2": (dict(ctx=(1000, 500), hkv=2, rot_window=640), {}),
    "windows_2_g8_64_pairs": (dict(ctx=tuple(60 + 11 * i for i in range(16)), hkv=4, group=8, rot_window=128), {}),
    "windows_2_g8_68_pairs": (dict(ctx=tuple(60 + 11 * i for i in range(17)), hkv=4, group=7, rot_window=128), {}),
    "windows_3": (dict(ctx=(1300, 500), hkv=2, rot_window=512), {}),
    "windows_16": (dict(ctx=(1000, 70), hkv=2, rot_window=64), dict(select=(1, 3))),
    "windows_17": (dict(ctx=(1080, 70), hkv=2, rot_window=64), dict(select=(1, 3))),
    "windows_64": (dict(ctx=(4092, 70), hkv=1, rot_window=64), dict(select=(1, 3))),
    "windows_70_mostly_empty": (dict(ctx=(300, 4476, 33), hkv=1, group=8, rot_window=64), {}),
    "buffers": (dict(ctx=(1, 31, 33, 63, 65, 95, 97, 127), hkv=1, group=7, dtype="bf16"), {}),
    "few_blocks_b16": (dict(ctx=(9000, 129), hkv=1), dict(force_default=True, default=(32, 1, 16))),
    "all_selected_b4": (dict(ctx=(4000, 33), hkv=1), dict(force_default=True, default=(16, 2, 4), select=(1, 1))),
    "quest_b8": (dict(ctx=(3000, 801, 40), hkv=2, rotate=False), dict(force_default=True, default=(128, 1, 8))),
    "quest_b4_g8": (dict(ctx=(3000, 801, 40), hkv=1, group=8, dtype="bf16", rotate=False),
                    dict(force_default=True, default=(128, 1, 4), select=(1, 2))),
    "quest_b16_rotated": (dict(ctx=(5000, 64), hkv=1, dtype="bf16"), dict(force_default=True, default=(128, 1, 16))),
    # the fused front kernel: its longest contexts (2048 blocks of 4, of 16), its most pairs, mixed and
    # truncated records, both group paddings, appended halves
    "front_b4_last": (dict(ctx=(8191, 8100), hkv=1), dict(force_default=True, default=(32, 1, 4))),
    "front_b16_last": (dict(ctx=(32767, 100), hkv=1, dtype="bf16"), dict(force_default=True, default=(32, 2, 16), block_cand=(16, 16, 16))),
    "front_first_past": (dict(ctx=(8256, 100), hkv=1), dict(force_default=True, default=(32, 1, 4))),
    "front_256_pairs": (dict(ctx=tuple(40 + 3 * i for i in range(64)), hkv=4), {}),
    "front_past_256_pairs": (dict(ctx=tuple(40 + 3 * i for i in range(65)), hkv=4), {}),
    "front_mixed_g7": (dict(ctx=(3000, 32, 64, 97), hkv=2, group=7, kind="outlier_random", dtype="bf16"), dict(tau_channel=0.2)),
    "front_trunc_g8": (dict(ctx=(2000, 1033), hkv=1, group=8), dict(trunc=96)),
    "front_trunc_b4_g7": (dict(ctx=(8100, 33), hkv=1, group=7, dtype="bf16"), dict(force_default=True, default=(16, 1, 4), trunc=96)),
    "front_trunc_32": (dict(ctx=(2500, 64), hkv=2), dict(trunc=32, keep_cand=(16, 32, 32), tau_channel=0.2)),
    "front_unrotated": (dict(ctx=(1500, 33), hkv=1, group=1, rotate=False), dict(fp8=True)),
    "some_keep_all": (dict(ctx=(1500, 900), hkv=2), dict(keep_cand=(16, 64, 128), default=(128, 1, 8), tau_channel=0.01)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_decode_plan(name):
    over, extra = CASES[name]
    spec = gen.spec("c1", **over)
    cap = spec.max_ctx + 4
    lay = gen.make_layer(spec, 0, capacity=cap)
    lp, op = params_pair(spec, **extra)
    ops = oracle_pairs(op, spec, lay, cap)
    c = gpu_cache(lp, spec, lay, cap)
    q = gen.make_queries(spec, 0)
    c.workspace.zero_()
    out = c.decode(q.cuda(), scale_of())
    torch.cuda.synchronize()
    # the plans made on the GPU leave their blocks per split behind the list header, the fixed one nothing
    nw = c.layout.num_windows
    planned = int(c.ws_region("wsel", 0, 4 * (nw + 3)).cpu().numpy().view(np.int32)[nw + 2]) > 0
    assert planned == (nw > 1 or name.startswith("uneven")), f"{name}: another split plan than the case is for"
    want, sels, scores = oracle_decode_all(ops, spec, q, scale_of())
    for p in range(spec.num_seqs * spec.hkv):
        nb = ops[p].info().nblk
        gs, gsel, _ = gpu_scores_sel(c, p, nb)
        assert np.array_equal(gs.view(np.uint32), scores[p].view(np.uint32)), f"{name} pair {p}: block scores"
        assert np.array_equal(gsel, sels[p]), f"{name} pair {p}: selected blocks"
    assert_close(out.cpu().numpy(), want, name)
