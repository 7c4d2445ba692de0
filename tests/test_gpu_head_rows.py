"""The head's work on the labelled rows only: how many of them there are stays on the device, so the row count is tried at
the edges of the GEMM tiles, with few and with all rows labelled, with a vocabulary that is cut into slices (from 4096 on)
and one that is not.  fp32 results are sums of at most vocab or rows products: 4 sqrt(8192) 2^-24 < 3e-5 of the largest
entry covers their rounding; bf16 rounds logits, probabilities and hidden states once each, 4 x 2^-8."""

import numpy as np
import pytest
import torch

from oracle import ends as OE
from paper_2308_15762_amd import hanayo as hn
from paper_2308_15762_amd import synth
from helpers import dev, dev_bytes, host, perr

pytestmark = pytest.mark.gpu
TOL = {"fp32": 3e-5, "bf16": 4 * 2.0 ** -8}


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("seq,mb,hidden,vocab,picked", [
    (7, 1, 64, 72, 1), (65, 3, 128, 520, 64), (129, 2, 136, 1000, 257), (256, 2, 256, 4096, 1), (300, 2, 256, 5128, 65), (128, 4, 320, 8200, 512)])
@pytest.mark.parametrize("final_ln", [False, True])
def test_head_on_labelled_rows(dtype, seq, mb, hidden, vocab, picked, final_ln):
    wl = synth.WORKLOADS["bert_1024_bf16"].scaled(dtype=dtype, hidden=hidden, heads=hidden // 8, ffn=hidden, seq=seq, mb=mb, vocab=vocab, n_blocks=1)
    rng = np.random.default_rng(seq + vocab)
    T = seq * mb
    labels = np.full(T, -1, np.int32)
    at = np.sort(rng.permutation(T)[:min(picked, T)])
    labels[at] = rng.integers(0, vocab, size=at.size)
    labels[at[-1]] = vocab - 1
    other = np.setdiff1d(np.arange(T), at)
    if other.size:
        labels[other[0]] = vocab                               # outside the vocabulary: not counted
    labels = labels.reshape(mb, seq)
    p = synth.ends_params(wl, ln_random=True)
    lnf = (p["lnf"] or (1.0 + 0.1 * rng.normal(size=hidden), 0.1 * rng.normal(size=hidden)))
    lnf = tuple(synth._finish(np.asarray(a), dtype) for a in lnf)
    head, y = synth.untied_head(wl), synth.forward_input(wl, 0, 0)
    d, e = hn.desc_for(wl), hn.EndsDesc(vocab, seq, int(final_ln))
    f32 = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    loss, d_head, d_lnf, yd = f32(1), f32(vocab, hidden), f32(2 * hidden), dev(y, dtype)
    dy = torch.full_like(yd, 7.0)
    work = dev_bytes(hn.hanayo_head_workspace_bytes(d, e))
    work.fill_(255)                                            # NaNs: nothing past the counted rows may be used
    hn.hanayo_head_loss(d, e, dev(np.concatenate(lnf), dtype) if final_ln else None, dev(head, dtype), yd, torch.from_numpy(labels).cuda(), 0.5,
                        loss, dy, d_lnf if final_ln else None, d_head, work)
    torch.cuda.synchronize()
    f = lambda a: np.asarray(a, dtype=np.float64)
    w_loss, w_dy, w_head, w_lnf = OE.head_loss(f(y), np.where(labels < vocab, labels, -1), f(head), tuple(map(f, lnf)) if final_ln else None, 1e-5, 0.5)
    assert abs(float(loss) - w_loss) <= TOL[dtype] * w_loss
    assert perr(host(dy), w_dy) <= TOL[dtype] and perr(host(d_head), w_head) <= TOL[dtype]
    assert not host(dy).reshape(T, hidden)[other].any()
    if final_ln:
        assert perr(host(d_lnf), np.concatenate(w_lnf)) <= TOL[dtype]


@pytest.mark.parametrize("config", [0, 1, 7, 9, 10, 11])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_head_under_a_forced_gemm_kernel(config, dtype):
    """A kernel is forced only where it takes the problem: the direct-to-LDS ones take no fp32, whose results are then those of
    the automatic choice, bit for bit."""
    d, e = hn.make_desc(1, 64, 1, 64, 65, 3, hn.PRE_LN, hn.MASK_CAUSAL, hn.BF16 if dtype == "bf16" else hn.FP32), hn.EndsDesc(4104, 65, 0)
    g = torch.Generator().manual_seed(3)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    y, head = torch.randn((3, 65, 64), generator=g).to(t), (0.02 * torch.randn((4104, 64), generator=g)).to(t)
    labels = torch.randint(-2000, 4104, (3, 65), generator=g, dtype=torch.int32)

    def run(config):
        loss, d_head, dy = torch.zeros(1, device="cuda"), torch.zeros((4104, 64), device="cuda"), torch.empty_like(y, device="cuda")
        hn.hanayo_op_gemm_config(config)
        try:
            hn.hanayo_head_loss(d, e, None, head.cuda(), y.cuda(), labels.cuda(), 1.0, loss, dy, None, d_head, dev_bytes(hn.hanayo_head_workspace_bytes(d, e)))
        finally:
            hn.hanayo_op_gemm_config(-1)
        torch.cuda.synchronize()
        return host(loss), host(dy), host(d_head)

    got, auto = run(config), run(-1)
    f = lambda a: a.double().numpy()
    want = OE.head_loss(f(y), np.where(labels.numpy() < 0, -1, labels.numpy()), f(head), None, 1e-5, 1.0)
    for a, b, w in zip(got, auto, want):
        assert perr(a, w) <= TOL[dtype]
        if dtype == "fp32" and config > 1:
            assert (a == b).all()


@pytest.mark.parametrize("dtype,vocab", [("bf16", (1 << 22) - 8), ("bf16", 1 << 22), ("fp32", 1 << 23)])
def test_head_with_a_very_large_vocabulary(dtype, vocab):
    """The last vocabulary whose contraction is cut into slices, the first that is not, and one whose rows are too long for the
    32-bit offsets of the matrix-instruction kernels.  fp32: the contraction over the vocabulary runs in sums of 65536 terms,
    4 sqrt(65536) 2^-24 < 6.2e-5, by the rule above."""
    tol = 6.2e-5 if dtype == "fp32" else TOL[dtype]
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    d, e = hn.make_desc(1, 8, 1, 8, 3, 1, hn.PRE_LN, hn.MASK_CAUSAL, hn.BF16 if dtype == "bf16" else hn.FP32), hn.EndsDesc(vocab, 3, 0)
    g = torch.Generator().manual_seed(11)
    y, head = torch.randn((1, 3, 8), generator=g).to(t), torch.randn((vocab, 8), generator=g).to(t)
    labels = torch.tensor([[vocab - 1, -1, 5]], dtype=torch.int32)
    loss, d_head, dy = torch.zeros(1, device="cuda"), torch.zeros((vocab, 8), device="cuda"), torch.full_like(y, 7.0, device="cuda")
    hn.hanayo_head_loss(d, e, None, head.cuda(), y.cuda(), labels.cuda(), 1.0, loss, dy, None, d_head, dev_bytes(hn.hanayo_head_workspace_bytes(d, e)))
    torch.cuda.synchronize()
    w_loss, w_dy, w_head, _ = OE.head_loss(y.double().numpy(), labels.numpy(), head.double().numpy(), None, 1e-5, 1.0)
    assert abs(float(loss) - w_loss) <= tol * w_loss
    assert perr(host(dy), w_dy) <= tol and perr(host(d_head), w_head) <= tol
    assert not host(dy)[0, 1].any()
