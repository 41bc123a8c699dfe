"""LayerNorm and causal attention kernels vs the oracle's definitions
(fp64 on the same bf16-rounded inputs).  Bars: bf16 outputs 4e-3 (one bf16 rounding on fp32
arithmetic; attention 8e-3 / 1e-2: probabilities are rounded to bf16 before the second
product), fp32 outputs 1e-5; each normwise and element by element (util.close)."""
import numpy as np
import pytest
import torch

from oracle import blocks
from paper_2401_01728_amd.inputs import gen
from util import bf16_normal, close, host64, dev

pytestmark = pytest.mark.gpu


# the last three rows: 8192 rows and more take the four-rows-per-wave forward (seven and four column
# groups), 1792 is the widest row of the two-register-set forward
@pytest.mark.parametrize("T,d", [(64, 128), (100, 1024), (37, 1600), (16, 2048), (8, 4096), (5, 64),
                                 (8203, 1600), (8197, 1024), (23, 1792)])
def test_layernorm_forward_backward(T, d):
    from paper_2401_01728_amd import kernels as k
    eps = 1e-5
    x32 = gen.normal_f32(1, 0, T * d, mean=0.3, std=2.0).reshape(T, d)
    g, g64 = bf16_normal(1, 1, (d,), mean=1.0, std=0.1)
    b, b64 = bf16_normal(1, 2, (d,), std=0.1)
    y, mean, rstd = k.layernorm_fwd(dev(x32), g, b, eps)
    ref, (xh, r) = blocks.layernorm_fwd(x32.astype(np.float64), g64, b64, eps)
    close(host64(y), ref, 4e-3, "k", group="LayerNorm / column sum / attention kernels, bar 4e-3")
    close(host64(mean), x32.astype(np.float64).mean(-1), 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")
    close(host64(rstd), r[:, 0], 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")
    # bf16 input variant also emits the widened copy
    xb, xb64 = bf16_normal(1, 3, (T, d), std=1.5)
    xc = torch.empty(T, d, dtype=torch.float32, device="cuda")
    y2, _, _ = k.layernorm_fwd(xb, g, b, eps, xcopy=xc)
    assert np.array_equal(host64(xc), xb64)
    close(host64(y2), blocks.layernorm_fwd(xb64, g64, b64, eps)[0], 4e-3, "k", group="LayerNorm / column sum / attention kernels, bar 4e-3")
    # backward joined with the residual branch
    dy, dy64 = bf16_normal(1, 4, (T, d), std=1e-2)
    dres32 = gen.normal_f32(1, 5, T * d, std=1e-2).reshape(T, d)
    dx, dx16, dg, db, dbias = k.layernorm_bwd(dy, dev(x32), mean, rstd, g, dev(dres32))
    rdx, rdg, rdb = blocks.layernorm_bwd(dy64, g64, (xh, r))
    rdx = rdx + dres32
    close(host64(dx), rdx, 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")
    close(host64(dx16), rdx, 4e-3, "k", group="LayerNorm / column sum / attention kernels, bar 4e-3")
    close(host64(dg), rdg, 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")
    close(host64(db), rdb, 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")
    close(host64(dbias), rdx.sum(0), 1e-5, "k", group="LayerNorm / column sum / attention kernels, bar 1e-5")


# the LayerNorm that adds a product's pieces: every register layout (up to 1024, 2048, 4096 columns), odd rows and widths
@pytest.mark.parametrize("T,d,S,rows", [(5, 64, 2, 2), (37, 1024, 4, 4), (16, 1028, 8, 2), (9, 2048, 2, 8), (3, 2052, 4, 2), (6, 4096, 8, 16)])
def test_layernorm_of_parts(T, d, S, rows):
    from paper_2401_01728_amd import kernels as k
    eps, grp = 1e-5, "LayerNorm / column sum / attention kernels, bar "
    part32 = gen.normal_f32(4, 0, S * T * d, std=0.7).reshape(S, T, d)
    res32 = gen.normal_f32(4, 1, T * d, mean=0.3, std=2.0).reshape(T, d)
    (bias, bias64), (g, g64), (b, b64) = bf16_normal(4, 2, (d,)), bf16_normal(4, 3, (d,), mean=1.0, std=0.1), bf16_normal(4, 4, (d,))
    x64 = part32.astype(np.float64).sum(0) + bias64 + res32
    xsum, y, mean, rstd = k.layernorm_fwd_parts(dev(part32), bias, dev(res32), g, b, eps)
    ref, (xh, r) = blocks.layernorm_fwd(x64, g64, b64, eps)
    for got, want, tol in ((xsum, x64, 1e-5), (mean, x64.mean(-1), 1e-5), (rstd, r[:, 0], 1e-5), (y, ref, 4e-3)):
        close(host64(got), want, tol, "k", group=grp + "%.0e" % tol)
    x2, out16 = k.layernorm_fwd_parts(dev(part32), bias, dev(res32), None, None, eps)
    assert torch.equal(x2, xsum) and torch.equal(out16, xsum.to(torch.bfloat16))
    dyp32 = gen.normal_f32(4, 5, S * T * d, std=1e-2).reshape(S, T, d)
    dres32 = gen.normal_f32(4, 6, T * d, std=1e-2).reshape(T, d)
    dx, dx16, part = k.layernorm_bwd_parts(dev(dyp32), xsum, mean, rstd, g, dev(dres32), rows)
    dx64, dg, db = blocks.layernorm_bwd(dyp32.astype(np.float64).sum(0), g64, (xh, r))
    dx64 = dx64 + dres32
    assert torch.equal(dx16, dx.to(torch.bfloat16))
    for got, want in zip((host64(dx), *host64(part).sum(0)), (dx64, dg, db, dx64.sum(0))):
        close(got, want, 1e-5, "k", group=grp + "1e-05")


def _heads(t64, mb, S, H, dh):
    return t64.reshape(mb, S, H, dh).transpose(0, 2, 1, 3)


def _unheads(t):
    mb, H, S, dh = t.shape
    return t.transpose(0, 2, 1, 3).reshape(mb * S, H * dh)


@pytest.mark.parametrize("mb,S,H,dh", [(2, 128, 2, 64), (1, 192, 3, 64), (1, 256, 2, 128), (2, 512, 2, 64),
                                        (1, 64, 1, 64), (1, 320, 1, 128)])
def test_attention_forward_backward(mb, S, H, dh):
    from paper_2401_01728_amd import kernels as k
    d = H * dh
    qkv, qkv64 = bf16_normal(3, 0, (mb * S, 3 * d), std=1.0)
    q, kk, v = (_heads(qkv64[:, i * d:(i + 1) * d], mb, S, H, dh) for i in range(3))
    ref, prob = blocks.causal_attention_fwd(q, kk, v)
    out, lse2 = k.attention_fwd(qkv, mb, S, d, H)
    close(host64(out), _unheads(ref), 8e-3, "k", group="LayerNorm / column sum / attention kernels, bar 8e-3")
    # log-sum-exp (base 2, scaled domain) against the definition
    s = np.einsum("bhid,bhjd->bhij", q, kk) / np.sqrt(dh)
    s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
    mx = s.max(-1)
    lse_ref = (mx + np.log(np.exp(s - mx[..., None]).sum(-1))) / np.log(2.0)
    assert np.abs(host64(lse2).reshape(mb, H, S) - lse_ref).max() < 1e-3
    dout, dout64 = bf16_normal(3, 1, (mb * S, d), std=1e-2)
    dq, dk, dv = blocks.causal_attention_bwd(_heads(dout64, mb, S, H, dh), q, kk, v, prob)
    # the kernel's D = rowsum(dO * O) uses its own bf16 output, as the stage does
    dqkv = host64(k.attention_bwd(qkv, out, dout, lse2, mb, S, d, H))
    close(dqkv[:, :d], _unheads(dq), 1e-2, "k", group="LayerNorm / column sum / attention kernels, bar 1e-2")
    close(dqkv[:, d:2 * d], _unheads(dk), 1e-2, "k", group="LayerNorm / column sum / attention kernels, bar 1e-2")
    close(dqkv[:, 2 * d:], _unheads(dv), 8e-3, "k", group="LayerNorm / column sum / attention kernels, bar 8e-3")


# row blocks at and beyond the number up to which both parts of the backward share a launch, sequences whose
# last row block is half empty
@pytest.mark.parametrize("mb,S,H,dh", [(32, 64, 16, 64), (33, 64, 16, 64), (9, 192, 30, 64), (16, 64, 16, 128),
                                        (17, 64, 16, 128), (5, 192, 26, 128)])
def test_attention_many_row_blocks(mb, S, H, dh):
    test_attention_forward_backward(mb, S, H, dh)


# two groups of waves to a workgroup, sequences of 384 and more: odd numbers of tiles, a half-empty last row block, the most row
# blocks the rules take (256 forward, 128 backward) and a few more
@pytest.mark.parametrize("mb,S,H,dh", [(1, 384, 1, 64), (2, 448, 3, 64), (1, 576, 2, 128), (8, 512, 4, 64), (16, 512, 4, 64), (13, 576, 4, 64),
                                        (8, 448, 8, 128)])
def test_attention_of_few_row_blocks(mb, S, H, dh):
    test_attention_forward_backward(mb, S, H, dh)


# 2048 rows and more: two rows to a wave; one row less: a workgroup to each row
@pytest.mark.parametrize("T,d", [(2051, 1024), (2049, 1792), (2047, 64)])
def test_layernorm_around_two_rows_a_wave(T, d):
    test_layernorm_forward_backward(T, d)


def test_attention_rejects_unsupported_shapes():
    from paper_2401_01728_amd import kernels as k
    import paper_2401_01728_amd as rv
    qkv = torch.zeros(100, 3 * 96, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rv.RvError):
        k.attention_fwd(qkv, 1, 100, 96, 1)        # head size 96, seq 100
