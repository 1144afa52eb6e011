"""Dense decode attention at the edges of its 32-token steps, its 128-token
rounds and its 1024-token runs, for every width of the group's padding,
against the fp64 oracle.  Logits and sums are fp32 over exact 16-bit products
and the weights carry 24 bits, so 2e-6 relative covers them with the
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


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("G", [4, 8])
def test_dense_weights_keep_24_bits(dtype, G):
    """Sequences of two tokens: weights 1 and w = exp(-x), w in (1/2, 1).  With
    V = a in the first token and -1 in the second, a the 16-bit value nearest to
    w, the output (a - w') / (1 + w) gives the weight w' that took part to
    2^-33, as a - w' is below 2^-8 and the output has 24 bits.  An fp32 weight
    in (1/2, 1) is a multiple of 2^-24, an odd one half of the time; two fp16
    parts leave an even one wherever the second part is 2^-13 or more (its last
    place is then 2^-23 or more), and two bf16 parts lose more still."""
    S, dt = 64, torch.float16 if dtype == "fp16" else torch.bfloat16
    rng = np.random.RandomState(3)
    q = torch.zeros(S, G, 128)
    q[:, :, 0] = torch.from_numpy(rng.randint(64, 128, (S, G)) / 128.0)      # exact in both types
    k, v = torch.zeros(S, 1, 2, 128), torch.zeros(S, 1, 2, 128)
    k[:, 0, 1, 0] = -torch.from_numpy(rng.randint(16, 88, S) / 128.0)
    z = (q[:, :, 0] * k[:, 0, 1, :1]).double().numpy()                       # [S][G]
    a = torch.from_numpy(np.exp(z)).to(dt)
    v[:, 0, 0, :G], v[:, 0, 1] = a.float(), -1.0
    out = M.dense_decode(q.to(dt).cuda(), k.to(dt).cuda(), v.to(dt).cuda(), torch.full((S,), 2, dtype=torch.int32, device="cuda"),
                         1.0, 2, G).cpu().double()
    got = torch.diagonal(out[:, :, :G], dim1=1, dim2=2).numpy()              # head h's channel h
    a = a.double().numpy()
    w = np.exp(z)
    for _ in range(3):
        w = a - got * (1.0 + w)
    assert np.abs(w / np.exp(z) - 1.0).max() < 4 * 2.0 ** -23                # the exponential's own error
    n = w * 2.0 ** 24
    assert np.abs(n - np.round(n)).max() < 0.05
    wide = np.abs(w - a) >= 2.0 ** -13
    odd = np.round(n).astype(np.int64)[wide] % 2
    assert wide.sum() > 64 and odd.mean() > 0.25, f"{odd.sum()} odd of {wide.sum()}"


def _softmax64(q, k, v):
    """[G][128], fp64: attention of q [G][128] over k, v [n][128], scale 1 / sqrt(128)."""
    z = q.double() @ k.double().T * float(scale_of())
    return (torch.softmax(z, 1) @ v.double()).numpy()


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("G", [4, 7])
def test_dense_masked_tokens(dtype, G):
    """Tokens masked through their keys, to a logit of -inf or to the type's
    lowest value: whole 32-token steps, a wave's first steps, whole 1024-token
    runs, all but the last token.  They take no part, so the result is the
    attention over the others (bound as above)."""
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    masks = [(0, 32), (0, 64), (0, 300), (32, 160), (0, 1024), (0, 1100), (1024, 2048), (0, 2499), (1, 2500)]
    S, n = len(masks), 2500
    g = torch.Generator().manual_seed(7)
    q, k, v = (torch.randn(*sh, 128, generator=g).to(dt) for sh in ((S, G), (S, 1, n), (S, 1, n)))
    q[:, :, 0] = 1.0
    lens = torch.full((S,), n, dtype=torch.int32, device="cuda")
    for mask in (-float("inf"), torch.finfo(dt).min):
        kk = k.clone()
        for s, (a, b) in enumerate(masks):
            kk[s, 0, a:b, 0] = mask
        out = M.dense_decode(q.cuda(), kk.cuda(), v.cuda(), lens, scale_of(), n, G).cpu().double().numpy()
        for s, (a, b) in enumerate(masks):
            keep = [t for t in range(n) if not a <= t < b]
            want = _softmax64(q[s], k[s, 0, keep], v[s, 0, keep])
            rel = np.linalg.norm(out[s] - want) / np.linalg.norm(want)
            assert rel < 2e-6, f"{dtype} G={G} mask {mask} of {a}..{b}: rel {rel:.2e}"


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_dense_infinite_values(dtype, G):
    """An infinite element of V gives its infinity in its column (every weight
    here is positive), two of opposite signs or a NaN give NaN, and the other
    columns stay as they are (bound as above): at the first and last token, in
    steps that the context ends in, in one of several runs."""
    dt, inf = torch.float16 if dtype == "fp16" else torch.bfloat16, float("inf")
    cases = [(1, {(0, 3): inf}), (33, {(32, 0): -inf}), (33, {(0, 127): inf, (31, 5): -inf}), (300, {(17, 9): inf, (299, 9): -inf}),
             (300, {(299, 64): inf}), (2500, {(1500, 1): inf, (2499, 2): -inf}), (2500, {(3, 7): float("nan")}), (2500, {})]
    S, n = len(cases), 2500
    g = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn(*sh, 128, generator=g).to(dt) for sh in ((S, G), (S, 1, n), (S, 1, n)))
    for s, (_, at) in enumerate(cases):
        for (t, c), x in at.items():
            v[s, 0, t, c] = x
    lens = torch.tensor([L for L, _ in cases], dtype=torch.int32, device="cuda")
    out = M.dense_decode(q.cuda(), k.cuda(), v.cuda(), lens, scale_of(), n, G).cpu().double().numpy()
    for s, (L, at) in enumerate(cases):
        want = _softmax64(q[s], k[s, 0, :L], v[s, 0, :L])
        fin = np.isfinite(want)
        assert (~fin).any(0).sum() == len({c for _, c in at})                # the reference itself: those columns only
        where = f"{dtype} G={G} L={L} {at}"
        assert np.array_equal(out[s][~fin], want[~fin], equal_nan=True), where
        rel = np.linalg.norm(out[s][fin] - want[fin]) / np.linalg.norm(want[fin])
        assert rel < 2e-6, f"{where}: rel {rel:.2e}"


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_dense_long_runs(dtype):
    """512 pairs of up to 4096 tokens: more than 1024 chunks, so runs of two, at
    the edges of a run (bound as above)."""
    dt, S, H, G, n = (torch.float16 if dtype == "fp16" else torch.bfloat16), 64, 8, 4, 4096
    lens = [(2047, 2048, 2049, 4096, 0, 1, 3000, 4095)[s % 8] for s in range(S)]
    g = torch.Generator(device="cuda").manual_seed(5)
    k = torch.randn(S, H, n, 128, generator=g, device="cuda", dtype=torch.float32).to(dt)
    v = torch.randn(S, H, n, 128, generator=g, device="cuda", dtype=torch.float32).to(dt)
    q = torch.randn(S, H * G, 128, generator=g, device="cuda").to(dt)
    out = M.dense_decode(q, k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"), scale_of(), n, G).cpu().double().numpy()
    for s, L in enumerate(lens):
        for h in range(0, H, 3):
            got = out[s, h * G: (h + 1) * G]
            if L == 0:
                assert not got.any()
                continue
            want = _softmax64(q[s, h * G: (h + 1) * G].cpu(), k[s, h, :L].cpu(), v[s, h, :L].cpu())
            rel = np.linalg.norm(got - want) / np.linalg.norm(want)
            assert rel < 2e-6, f"{dtype} sequence {s} head {h} L={L}: rel {rel:.2e}"
