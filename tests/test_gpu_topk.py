"""Selections at the edges of the single-workgroup top-k's forms (1, 4 and 16
waves of 4 keys per thread, then 8, 16 and 32 keys), in the fused front kernel
(every sequence at most 2048 blocks) and in the top-k kernel, against the
oracle, bit for bit: distinct scores, a few levels (ties at the threshold, some
of them taken), all equal."""
import numpy as np
import pytest
import torch

from _parity import gpu_cache, gpu_scores_sel, oracle_decode_all, oracle_pairs, params_pair, scale_of
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("select", [(1, 10), (1, 2)])
@pytest.mark.parametrize("blocks", [(16, 256, 272, 1008, 1024, 1040), (16, 256, 272, 1024, 4112), (1040, 4096, 4112), (8192, 8208), (16384, 16400)])
def test_topk_edges(blocks, select):
    ctx = tuple(4 * b for b in blocks)
    spec = gen.spec("c1", ctx=ctx, hkv=1, rotate=False)
    lay = gen.make_layer(spec, 0, capacity=spec.max_ctx)
    lp, op = params_pair(spec, force_default=True, default=(16, 1, 4), select=select)
    few = {w: (lay[w].float() * 0.5).round().clamp(-1, 1).to(lay[w].dtype) for w in ("k", "v")}
    few["k"] = few["k"][:, :, ::4].repeat_interleave(4, 2)[:, :, :spec.max_ctx]      # a block's tokens alike
    for name, data in (("distinct", lay), ("levels", {**lay, **few})):
        ops = oracle_pairs(op, spec, data, spec.max_ctx)
        c = gpu_cache(lp, spec, data, spec.max_ctx)
        q = gen.make_queries(spec, 0)
        if name == "levels":
            q = q.round()
        for which, qq in (("q", q), ("zero", torch.zeros_like(q))):
            print(f"[topk] {blocks} {select} {name} {which}", flush=True)
            c.decode(qq.cuda(), scale_of())
            torch.cuda.synchronize()
            _, sels, scores = oracle_decode_all(ops, spec, qq, scale_of())
            for p in range(spec.num_seqs):
                gs, gsel, _ = gpu_scores_sel(c, p, blocks[p])
                assert np.array_equal(gs.view(np.uint32), scores[p].view(np.uint32)), f"{name} {which} pair {p}: scores"
                assert np.array_equal(gsel, sels[p]), f"{name} {which} pair {p}: selected blocks"
