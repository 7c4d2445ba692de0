"""fp32 attention at the edges of its 32-row tiles and of its head-dim classes, against the oracle.

Bound: scores are fp32 sums of d products with |s| <= a few units at these inputs, so exp(s) carries about (d + 8) 2^-24
times |s|; contractions over s rows add (s + 4) 2^-24 of their absolute sums.  4 (d + s + 32) 2^-24 of a tensor's largest
entry covers both with the magnitudes used here (N(0, 1) operands)."""

import numpy as np
import pytest
import torch

from paper_2308_15762_amd import hanayo as hn
from helpers import dev, host, nerr

pytestmark = pytest.mark.gpu


def reference(qkv, vl, dc, heads, d, causal):
    b, s, _ = qkv.shape
    q, k, v = (t.reshape(b, s, heads, d).transpose(0, 2, 1, 3) for t in np.split(qkv.astype(np.float64), 3, -1))
    sc = q @ k.transpose(0, 1, 3, 2) / np.sqrt(d)
    ok = np.ones((b, 1, s, s), bool)
    if causal:
        ok &= np.tril(np.ones((s, s), bool))
    if vl is not None:
        ok &= (np.arange(s)[None, :] < vl[:, None])[:, None, None, :]
    sc = np.where(ok, sc, -np.inf)
    mx = sc.max(-1, keepdims=True)
    e = np.exp(sc - mx)
    lse = (mx + np.log(e.sum(-1, keepdims=True)))[..., 0]
    p = e / e.sum(-1, keepdims=True)
    g = dc.astype(np.float64).reshape(b, s, heads, d).transpose(0, 2, 1, 3)
    c = p @ v
    dp = g @ v.transpose(0, 1, 3, 2)
    ds = p * (dp - (g * c).sum(-1, keepdims=True)) / np.sqrt(d)
    back = lambda t: t.transpose(0, 2, 1, 3).reshape(b, s, heads * d)
    return back(c), lse, np.concatenate([back(ds @ k), back(ds.transpose(0, 1, 3, 2) @ q), back(p.transpose(0, 1, 3, 2) @ g)], -1)


@pytest.mark.parametrize("b,s,heads,d,causal,padded", [
    (1, 1, 1, 8, True, False), (2, 31, 3, 32, True, False), (1, 33, 2, 40, False, True), (2, 160, 2, 64, True, True), (1, 97, 2, 72, False, False),
    (1, 129, 2, 96, True, False), (2, 65, 1, 104, True, True), (1, 256, 2, 128, False, True), (3, 128, 4, 64, True, False)])
def test_attention_fp32(b, s, heads, d, causal, padded):
    rng = np.random.default_rng(s * 131 + d)
    H = heads * d
    qkv, dc = rng.normal(size=(b, s, 3 * H)).astype(np.float32), rng.normal(size=(b, s, H)).astype(np.float32)
    vl = rng.integers(1, s + 1, size=b).astype(np.int32) if padded else None
    ctx_ref, lse_ref, dqkv_ref = reference(qkv, vl, dc, heads, d, causal)
    qd, dcd = dev(qkv, "fp32"), dev(dc, "fp32")
    vd = None if vl is None else torch.from_numpy(vl).cuda()
    ctx, lse = torch.empty((b, s, H), device="cuda"), torch.empty((b, heads, s), device="cuda")
    dqkv, delta = torch.full((b, s, 3 * H), 7.0, device="cuda"), torch.empty((b, heads, s), device="cuda")
    hn.hanayo_op_attention_forward(hn.FP32, qd, vd, ctx, lse, b, s, heads, d, causal)
    hn.hanayo_op_attention_backward(hn.FP32, qd, vd, ctx, lse, dcd, dqkv, delta, b, s, heads, d, causal)
    torch.cuda.synchronize()
    tol = 4 * (d + s + 32) * 2.0 ** -24
    assert nerr(host(ctx), ctx_ref) <= tol
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= tol * max(1.0, np.abs(lse_ref).max())
    for i, name in enumerate(("dq", "dk", "dv")):
        got, ref = host(dqkv)[..., i * H:(i + 1) * H], dqkv_ref[..., i * H:(i + 1) * H]
        assert np.abs(got - ref).max() <= tol * max(np.abs(ref).max(), 1.0), name


def run(qkv, vl, dc, heads, d, causal, ctx=None, lse=None):
    b, s, _ = qkv.shape
    H = heads * d
    qd, vd = dev(qkv, "fp32"), None if vl is None else torch.from_numpy(vl).cuda()
    if ctx is None:
        ctx, lse = torch.full((b, s, H), 7.0, device="cuda"), torch.full((b, heads, s), 7.0, device="cuda")
        hn.hanayo_op_attention_forward(hn.FP32, qd, vd, ctx, lse, b, s, heads, d, causal)
    dqkv, delta = torch.full((b, s, 3 * H), 7.0, device="cuda"), torch.empty((b, heads, s), device="cuda")
    hn.hanayo_op_attention_backward(hn.FP32, qd, vd, ctx, lse, dev(dc, "fp32"), dqkv, delta, b, s, heads, d, causal)
    torch.cuda.synchronize()
    return ctx, lse, host(dqkv)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("s,heads,d", [(40, 1, 24), (97, 2, 64), (161, 1, 96), (130, 2, 128)])
def test_masked_rows_may_hold_anything(s, heads, d, bad):
    """Keys behind valid_len and, under the causal mask, later tokens have probability zero: what their rows hold reaches no
    result that the mask keeps from them."""
    rng = np.random.default_rng(s + d)
    H, b = heads * d, 2
    qkv, dc = rng.normal(size=(b, s, 3 * H)).astype(np.float32), rng.normal(size=(b, s, H)).astype(np.float32)
    tol = 4 * (d + s + 32) * 2.0 ** -24
    close = lambda got, ref: np.abs(got - ref).max() <= tol * max(np.abs(ref).max(), 1.0)
    # keys and values of padding
    vl = np.array([s - 9, 1], np.int32)
    for n in range(b):
        qkv[n, vl[n]:, H:] = 0.0
    ref = reference(qkv, vl, dc, heads, d, False)
    for n in range(b):
        qkv[n, vl[n]:, H:] = bad
    ctx, lse, dqkv = run(qkv, vl, dc, heads, d, False)
    assert close(host(ctx), ref[0]) and close(lse.cpu().numpy(), ref[1]) and close(dqkv, ref[2])
    # token j and those after it, as seen by the tokens before it
    qkv, j = rng.normal(size=(b, s, 3 * H)).astype(np.float32), s - 21
    clean = reference(qkv, None, dc, heads, d, True)
    poisoned = qkv.copy()
    poisoned[:, j] = bad
    ctx, lse, dqkv = run(poisoned, None, dc, heads, d, True)
    assert close(host(ctx)[:, :j], clean[0][:, :j]) and close(lse.cpu().numpy()[:, :, :j], clean[1][:, :, :j])
    assert close(dqkv[:, :j, :H], clean[2][:, :j, :H])
    assert np.isnan(host(ctx)[:, j:]).any(axis=-1).all()            # and those that see it do not come out clean
    # a query and its upstream gradient, as seen by the keys behind it
    ctx, lse, _ = run(qkv, None, dc, heads, d, True)
    poisoned, dcp = qkv.copy(), dc.copy()
    poisoned[:, j, :H] = bad
    dcp[:, j] = bad
    _, _, dqkv = run(poisoned, None, dcp, heads, d, True, ctx, lse)
    assert close(dqkv[:, j + 1:], clean[2][:, j + 1:])
    assert close(dqkv[:, :j, :H], clean[2][:, :j, :H])
    assert not np.isfinite(dqkv[:, :j + 1, H:]).any()
