"""Dense decode attention at the edges of its 32-token steps, its 128-token
rounds and its 1024-token runs, for every width of the group's padding,
against the fp64 oracle.  Logits and sums are fp32 over exact 16-bit products
and the weights carry 22 or 24 bits, so 2e-6 relative covers them with the
exponential's error (a few ulp of logits below 2^4)."""
import numpy as np
import pytest
import torch

from _parity import bits, scale_of
import paper_2607_00760_amd as M
from oracle import oracle as O
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("G", [1, 4, 5, 8])
def test_dense_edges(dtype, G):
    lens = (1, 31, 32, 33, 127, 129, 1023, 1024, 1025, 1153, 2048, 0)
    spec = gen.spec("c1", ctx=lens, hkv=1, group=G, dtype=dtype, rotate=False)
    lay = gen.make_layer(spec, 0)
    q = gen.make_queries(spec, 0).cuda()
    ctx = torch.tensor(lens, dtype=torch.int32, device="cuda")
    out = M.dense_decode(q, lay["k"].cuda(), lay["v"].cuda(), ctx, scale_of(), spec.max_ctx, G).cpu().numpy()
    for b, L in enumerate(lens):
        got = out[b].astype(np.float64)
        if L == 0:
            assert not got.any()
            continue
        want = O.dense_attention(bits(q)[b], bits(lay["k"])[b, 0, :L], bits(lay["v"])[b, 0, :L], np.float32(scale_of()), dtype)
        rel = np.linalg.norm(got - want) / np.linalg.norm(want)
        assert rel < 2e-6, f"L={L} G={G} {dtype}: rel {rel:.2e}"
