"""bf16 MFMA matrix products vs numpy fp64 on the same bf16-rounded operands.

Bar: bf16 outputs carry one bf16 rounding (2^-9 relative) on top of fp32 accumulation:
4e-3 (well inside the 2e-2 stage bar); fp32 outputs 1e-5; each normwise and element by element
(util.close).
"""
import numpy as np
import pytest
import torch

from oracle import blocks
from util import bf16_normal, close, host64, dev

pytestmark = pytest.mark.gpu

GROUP = {4e-3: "matrix product kernels, bf16 outputs", 1e-5: "matrix product kernels, fp32 outputs"}


def _out(shape, dtype):
    return torch.full(shape, float("nan"), dtype=dtype, device="cuda")


SHAPES = [(256, 256, 64), (128, 128, 128), (512, 384, 192), (200, 320, 256), (1024, 1024, 512), (64, 64, 64),
          (776, 1600, 320)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tile", [2128, 2192, 2256, 5256])
def test_forward_product_and_epilogues(M, N, K, tile):
    from paper_2401_01728_amd import kernels as k
    x, x64 = bf16_normal(1, 0, (M, K))
    w, w64 = bf16_normal(1, 1, (K, N), std=0.05)
    b, b64 = bf16_normal(1, 2, (N,), std=0.5)
    r64 = np.random.default_rng(0).normal(size=(M, N)).astype(np.float32)
    r = dev(r64)
    ref = x64 @ w64 + b64
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS, o, bias=b, tile=tile)
    close(host64(o), ref, 4e-3, "gemm", group=GROUP[4e-3])
    o32 = _out((M, N), torch.float32); o16 = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_F32_BIAS_RESID_BF16, o32, out2=o16, bias=b, resid=r, tile=tile)
    close(host64(o32), ref + r64, 1e-5, "gemm", group=GROUP[1e-5])
    close(host64(o16), ref + r64, 4e-3, "gemm", group=GROUP[4e-3])
    o32b = _out((M, N), torch.float32)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_F32_BIAS_RESID, o32b, bias=b, resid=r, tile=tile)
    assert torch.equal(o32, o32b)
    z = _out((M, N), torch.bfloat16); g = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS_GELU, z, out2=g, bias=b, tile=tile)
    close(host64(z), ref, 4e-3, "gemm", group=GROUP[4e-3])
    close(host64(g), blocks.gelu(ref), 4e-3, "gemm", group=GROUP[4e-3])


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tile", [2128, 2192, 2256, 5256])
def test_input_gradient_product(M, N, K, tile):
    """dx[M, N] = dy[M, K] W^T with W stored [N, K] (its rows are the output columns)."""
    from paper_2401_01728_amd import kernels as k
    dy, dy64 = bf16_normal(2, 0, (M, K))
    w, w64 = bf16_normal(2, 1, (N, K), std=0.05)
    z, z64 = bf16_normal(2, 2, (M, N))
    ref = dy64 @ w64.T
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(dy, 0, w, 0, M, N, K, k.EPI_BF16, o, tile=tile)
    close(host64(o), ref, 4e-3, "gemm", group=GROUP[4e-3])
    o2 = _out((M, N), torch.bfloat16)
    k.gemm_bf16(dy, 0, w, 0, M, N, K, k.EPI_BF16_DGELU, o2, zin=z, tile=tile)
    close(host64(o2), ref * blocks.gelu_grad(z64), 4e-3, "gemm", group=GROUP[4e-3])


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tile", [2128, 2192, 2256, 5256])
def test_weight_gradient_product(M, N, K, tile):
    """dW[M, N] = x^T dy with x [K, M] and dy [K, N]: contraction over the slow dimension."""
    from paper_2401_01728_amd import kernels as k
    x, x64 = bf16_normal(3, 0, (K, M))
    dy, dy64 = bf16_normal(3, 1, (K, N))
    o = _out((M, N), torch.float32)
    k.gemm_bf16(x, 1, dy, 1, M, N, K, k.EPI_F32, o, tile=tile)
    close(host64(o), x64.T @ dy64, 1e-5, "gemm", group=GROUP[1e-5])


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 384, 448, 576])
def test_ring_depths_of_the_256_tile(K):
    """The 256x256 tile walks K through a four-slot ring of 32-deep tiles (K/32 = 2 .. 18 tiles:
    fewer tiles than slots, exactly as many, one more, and a few turns of the ring), each layout,
    on a ragged output (two tile rows, two tile columns, the last of each partly filled)."""
    from paper_2401_01728_amd import kernels as k
    M, N = 328, 456
    x, x64 = bf16_normal(11, 0, (M, K)); w, w64 = bf16_normal(11, 1, (K, N), std=0.05)
    b, b64 = bf16_normal(11, 2, (N,), std=0.5)
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS, o, bias=b, tile=5256)            # forward layout
    close(host64(o), x64 @ w64 + b64, 4e-3, "gemm", group=GROUP[4e-3])
    wt, wt64 = bf16_normal(11, 3, (N, K), std=0.05)
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, wt, 0, M, N, K, k.EPI_BF16, o, tile=5256)                         # input-gradient layout
    close(host64(o), x64 @ wt64.T, 4e-3, "gemm", group=GROUP[4e-3])
    xt, xt64 = bf16_normal(11, 4, (K, M)); dy, dy64 = bf16_normal(11, 5, (K, N), std=1e-2)
    o32 = _out((M, N), torch.float32)
    k.gemm_bf16(xt, 1, dy, 1, M, N, K, k.EPI_F32, o32, tile=5256)                       # weight-gradient layout
    close(host64(o32), xt64.T @ dy64, 1e-5, "gemm", group=GROUP[1e-5])
    g32 = _out((M, N), torch.float32)
    k.gemm_wgrad_grouped([xt], [dy], [g32])
    assert torch.equal(g32, o32)


# the other tiles on the same ring, of three or four slots: fewer 32-deep tiles than slots, exactly as many, more
@pytest.mark.parametrize("tile", [2128, 2192, 2256])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 576])
def test_ring_depths_of_the_other_tiles(K, tile):
    """The bars of test_ring_depths_of_the_256_tile, on an output ragged for each of the tiles, one wave of which has nothing to
    multiply."""
    from paper_2401_01728_amd import kernels as k
    M, N = 328, 328
    x, x64 = bf16_normal(12, 0, (M, K)); w, w64 = bf16_normal(12, 1, (K, N), std=0.05)
    b, b64 = bf16_normal(12, 2, (N,), std=0.5)
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS, o, bias=b, tile=tile)
    close(host64(o), x64 @ w64 + b64, 4e-3, "gemm", group=GROUP[4e-3])
    wt, wt64 = bf16_normal(12, 3, (N, K), std=0.05)
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, wt, 0, M, N, K, k.EPI_BF16, o, tile=tile)
    close(host64(o), x64 @ wt64.T, 4e-3, "gemm", group=GROUP[4e-3])
    xt, xt64 = bf16_normal(12, 4, (K, M)); dy, dy64 = bf16_normal(12, 5, (K, N), std=1e-2)
    o32 = _out((M, N), torch.float32)
    k.gemm_bf16(xt, 1, dy, 1, M, N, K, k.EPI_F32, o32, tile=tile)
    close(host64(o32), xt64.T @ dy64, 1e-5, "gemm", group=GROUP[1e-5])


def test_strided_operands_and_rejects():
    """Operands that are column blocks of wider matrices (pitch > width), as q|k|v are."""
    from paper_2401_01728_amd import kernels as k
    import paper_2401_01728_amd as rv
    M, N, K = 256, 192, 128
    big, big64 = bf16_normal(4, 0, (M, 3 * K))
    w, w64 = bf16_normal(4, 1, (K, N), std=0.05)
    b, b64 = bf16_normal(4, 2, (N,))
    x = big[:, K:2 * K]
    o = _out((M, N), torch.bfloat16)
    k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS, o, bias=b)
    close(host64(o), big64[:, K:2 * K] @ w64 + b64, 4e-3, "gemm", group=GROUP[4e-3])
    with pytest.raises(rv.RvError):
        k.gemm_bf16(x, 0, w, 1, M, N, 100, k.EPI_BF16_BIAS, o, bias=b)       # K % 64
    with pytest.raises(rv.RvError):
        k.gemm_bf16(x, 1, w, 0, M, N, K, k.EPI_BF16, o)                      # unsupported layout pair
    wide = _out((M, N + 4), torch.bfloat16)
    with pytest.raises(rv.RvError):
        k.gemm_bf16(x, 0, w, 1, M, N, K, k.EPI_BF16_BIAS, wide[:, :N], bias=b)   # bf16 output pitch % 8


def test_grouped_weight_gradient_products():
    """Four products of different widths in one launch equal the single launches bit for bit."""
    from paper_2401_01728_amd import kernels as k
    K = 320
    dims = [(192, 256), (64, 64), (136, 512), (512, 72)]
    xs, dys, outs, refs = [], [], [], []
    for i, (M, N) in enumerate(dims):
        x, x64 = bf16_normal(9, 2 * i, (K, M)); dy, dy64 = bf16_normal(9, 2 * i + 1, (K, N), std=1e-2)
        xs.append(x); dys.append(dy); outs.append(_out((M, N), torch.float32)); refs.append(x64.T @ dy64)
    k.gemm_wgrad_grouped(xs, dys, outs)
    for i, (M, N) in enumerate(dims):
        close(host64(outs[i]), refs[i], 1e-5, "gemm", group=GROUP[1e-5])
        single = _out((M, N), torch.float32)
        k.gemm_bf16(xs[i], 1, dys[i], 1, M, N, K, k.EPI_F32, single, tile=5256)
        assert torch.equal(single, outs[i])
    import paper_2401_01728_amd as rv
    with pytest.raises(rv.RvError):
        k.gemm_wgrad_grouped(xs * 2, dys * 2, outs * 2)      # more than four


# K / 32 = 2, 8, 10, 62 k-tiles (fewer than the split form's eight ring slots, as many, two more, several turns);
# 64 k-tiles are 2048 tokens, where the in-order form takes over
@pytest.mark.parametrize("K,tile", [(64, 1128), (256, 1128), (320, 1128), (1984, 1128), (2048, 5256)])
def test_grouped_weight_gradients_with_their_update(K, tile):
    """The launch of a decoder stage: gradients against fp64 and bit for bit against single launches of the same tile,
    the updated masters and versions bit for bit against rv_block_update with that gradient, with and without the
    gradient stored."""
    from paper_2401_01728_amd import kernels as k
    import paper_2401_01728_amd as rv
    eta = 0.05
    dims = [(192, 256), (64, 64), (136, 512), (512, 72)]
    xs, dys, ws, refs = [], [], [], []
    for i, (M, N) in enumerate(dims):
        x, x64 = bf16_normal(12, 3 * i, (K, M)); dy, dy64 = bf16_normal(12, 3 * i + 1, (K, N), std=1e-2)
        xs.append(x); dys.append(dy); refs.append(x64.T @ dy64)
        ws.append(torch.randn(M, N, device="cuda"))
    single = [_out(s, torch.float32) for s in dims]
    for i, (M, N) in enumerate(dims):
        k.gemm_bf16(xs[i], 1, dys[i], 1, M, N, K, k.EPI_F32, single[i], tile=tile)
        close(host64(single[i]), refs[i], 1e-5, "gemm", group=GROUP[1e-5])
    outs = [_out(s, torch.float32) for s in dims]
    k.gemm_wgrad_update(xs, dys, outs)
    assert all(torch.equal(a, b) for a, b in zip(outs, single))
    new, ver = [w.clone() for w in ws], [_out(s, torch.bfloat16) for s in dims]
    for i in range(4):
        rv.block_update(new[i].view(-1), single[i].view(-1), eta, bf16_out=ver[i].view(-1))
    for store in (True, False):
        w, v, outs = [w.clone() for w in ws], [_out(s, torch.bfloat16) for s in dims], [_out(s, torch.float32) for s in dims]
        k.gemm_wgrad_update(xs, dys, outs if store else None, w, v, eta)
        assert all(torch.equal(a, b) for a, b in zip(w, new)) and all(torch.equal(a, b) for a, b in zip(v, ver))
        assert not store or all(torch.equal(a, b) for a, b in zip(outs, single))
    with pytest.raises(rv.RvError):
        k.gemm_wgrad_update(xs, dys, None, None, None, eta)      # nothing to write
    with pytest.raises(rv.RvError):
        k.gemm_wgrad_update(xs, dys, outs, ws, None, eta)        # masters without versions


# an eighth of a tile, one tile exactly, a ragged second tile; K = 2, 4, 10 and 34 tiles of 32 (fewer than a
# workgroup's groups, as many, a partly filled turn, several turns of every ring)
@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (64, 64, 128), (136, 200, 320), (40, 136, 1088), (264, 72, 64)])
@pytest.mark.parametrize("tile", [1032, 1064, 1065, 1128])
def test_split_contraction(M, N, K, tile):
    """Tiles whose contraction is split over groups of waves: every layout and epilogue (bars as above)."""
    test_forward_product_and_epilogues(M, N, K, tile)
    test_input_gradient_product(M, N, K, tile)
    if tile != 1032:
        test_weight_gradient_product(M, N, K, tile)


@pytest.mark.parametrize("kind,M,N,K", [("dx", 8192, 1280, 3840), ("resid", 8192, 1280, 5120), ("dx", 8192, 1280, 1280),
                                        ("bias", 2048, 4608, 1536)])
def test_automatic_tile_is_among_the_fast_ones(kind, M, N, K):
    """A launch alone against the same launch with each tile forced.  Bar 1.15: the fastest of six timings of 20
    launches repeats within 2 %, and with the wrong one of the three these take 1.25 to 1.4 times as long."""
    from paper_2401_01728_amd import kernels as k
    bf = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    A, b, r = bf(M, K), bf(N), torch.randn(M, N, device="cuda")
    B = bf(N, K) if kind == "dx" else bf(K, N)
    o = _out((M, N), torch.float32 if kind == "resid" else torch.bfloat16)

    def launch(tile):
        if kind == "dx":
            k.gemm_bf16(A, 0, B, 0, M, N, K, k.EPI_BF16, o, tile=tile)
        elif kind == "bias":
            k.gemm_bf16(A, 0, B, 1, M, N, K, k.EPI_BF16_BIAS, o, bias=b, tile=tile)
        else:
            k.gemm_bf16(A, 0, B, 1, M, N, K, k.EPI_F32_BIAS_RESID, o, bias=b, resid=r, tile=tile)

    times = {}
    for _ in range(6):
        for tile in (0, 5256, 2192, 2128):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            launch(tile)
            e0.record()
            for _ in range(20):
                launch(tile)
            e1.record(); torch.cuda.synchronize()
            times[tile] = min(times.get(tile, 1e9), e0.elapsed_time(e1))
    assert times[0] <= 1.15 * min(v for t, v in times.items() if t), times


# Products cut into stretches of the contraction: more stretches than a form has groups of waves get k-tiles (K = 64 in two), uneven
# stretches (K/32 = 10 in 3, 4 and 8), ragged tiles, fewer tiles than XCDs and more than one band of tile rows
@pytest.mark.parametrize("M,N,K,parts", [(8, 8, 64, 2), (40, 72, 320, 4), (128, 200, 320, 3), (648, 136, 1024, 8), (256, 448, 1792, 8)])
@pytest.mark.parametrize("tile", [1032, 1064, 1065, 1128])
def test_product_in_stretches(M, N, K, parts, tile):
    from paper_2401_01728_amd import kernels as k
    x, x64 = bf16_normal(9, 0, (M, K))
    edges = [32 * (K // 32 * i // parts) for i in range(parts + 1)]
    for b_kmajor in (0, 1):
        w, w64 = bf16_normal(9, 1 + b_kmajor, (K, N) if b_kmajor else (N, K), std=0.05)
        got = host64(k.gemm_part(x, w, b_kmajor, M, N, K, tile, parts))
        w64 = w64 if b_kmajor else w64.T
        for i in range(parts):
            lo, hi = edges[i], edges[i + 1]
            close(got[i], x64[:, lo:hi] @ w64[lo:hi], 1e-5, "part %d" % i, group=GROUP[1e-5])


def test_product_in_stretches_refuses():
    import paper_2401_01728_amd as rv
    from paper_2401_01728_amd import kernels as k
    x = torch.zeros(64, 64, dtype=torch.bfloat16, device="cuda")
    for tile, parts in ((1032, 3), (1032, 0), (5256, 2), (0, 2)):      # K / 32 = 2 stretches at most; the split forms only
        with pytest.raises(rv.RvError):
            k.gemm_part(x, x, 0, 64, 64, 64, tile, parts)


def _blocks(t):
    """[R, C] -> the same memory size, blocks of 32 columns, each a run of R rows of 32."""
    return t.view(t.shape[0], -1, 32).transpose(0, 1).contiguous()


# Operands and results in blocks of 32 columns, the layout of a stage's versions and operand activations: bit for bit what rows
# give, in every tile form, ragged in both directions (a last tile of one block of columns, of eight rows), one k-tile and more
@pytest.mark.parametrize("M,N,K", [(40, 96, 64), (200, 352, 256), (264, 288, 128), (776, 1600, 320)])
@pytest.mark.parametrize("tile", [2128, 2192, 2256, 5256, 1128, 1065, 1064, 1032])
def test_operands_in_blocks_of_columns(M, N, K, tile):
    from paper_2401_01728_amd import kernels as k
    x, _ = bf16_normal(10, 0, (M, K))
    w, _ = bf16_normal(10, 1, (K, N), std=0.05)
    wt, z = w.t().contiguous(), bf16_normal(10, 2, (M, N))[0]
    b, r = bf16_normal(10, 3, (N,), std=0.5)[0], torch.randn(M, N, device="cuda")
    bf, f32 = torch.bfloat16, torch.float32
    for xb, wb in ((0, 1), (1, 0), (1, 1)):
        X, W, WT = _blocks(x) if xb else x, _blocks(w) if wb else w, _blocks(wt) if wb else wt
        for epi, dt, kw in ((k.EPI_BF16_BIAS, bf, dict(bias=b)), (k.EPI_F32_BIAS_RESID, f32, dict(bias=b, resid=r)),
                            (k.EPI_F32_BIAS_RESID_BF16, f32, dict(bias=b, resid=r)), (k.EPI_BF16_BIAS_GELU, bf, dict(bias=b))):
            want, got = _out((M, N), dt), _out((M, N), dt)
            two = epi in (k.EPI_F32_BIAS_RESID_BF16, k.EPI_BF16_BIAS_GELU)
            want2, got2 = (_out((M, N), bf) if two else None for _ in range(2))
            k.gemm_bf16(x, 0, w, 1, M, N, K, epi, want, out2=want2, tile=tile, **kw)
            gb = epi == k.EPI_BF16_BIAS_GELU
            k.gemm_bf16_blocks(X, xb, 0, W, wb, 1, M, N, K, epi, got, got2, gb, tile=tile, **kw)
            assert torch.equal(got, want) and (not two or torch.equal(got2.flatten(), (_blocks(want2) if gb else want2).flatten()))
        for epi, zin in ((k.EPI_BF16, None), (k.EPI_BF16_DGELU, z)):
            want, got = _out((M, N), bf), _out((M, N), bf)
            k.gemm_bf16(x, 0, wt, 0, M, N, K, epi, want, zin=zin, tile=tile)
            k.gemm_bf16_blocks(X, xb, 0, WT, wb, 0, M, N, K, epi, got, None, zin is not None, zin=zin, tile=tile)
            assert torch.equal(got.flatten(), (want if zin is None else _blocks(want)).flatten())
        if tile < 2000:
            for parts in (2, min(8, K // 32)):
                for km, w_rows, w_form in ((1, w, W), (0, wt, WT)):
                    got = torch.full((parts, M, N), float("nan"), device="cuda")
                    k.gemm_bf16_blocks(X, xb, 0, w_form, wb, km, M, N, K, 0, got, tile=tile, parts=parts)
                    assert torch.equal(got, k.gemm_part(x, w_rows, km, M, N, K, tile, parts))
    if tile != 1032:                       # both operands k-major: their columns in blocks
        Mw = (M + 31) // 32 * 32
        xt, _ = bf16_normal(10, 4, (K, Mw))
        want, got = _out((Mw, N), f32), _out((Mw, N), f32)
        k.gemm_bf16(xt, 1, w, 1, Mw, N, K, k.EPI_F32, want, tile=tile)
        k.gemm_bf16_blocks(_blocks(xt), 1, 1, _blocks(w), 1, 1, Mw, N, K, k.EPI_F32, got, tile=tile)
        assert torch.equal(got, want)


def test_blocks_of_columns_are_whole():
    import paper_2401_01728_amd as rv
    from paper_2401_01728_amd import kernels as k
    x = torch.zeros(64, 72, dtype=torch.bfloat16, device="cuda")
    o = torch.zeros(72, 72, dtype=torch.float32, device="cuda")
    for args in ((x, 1, 1, x, 0, 1, 72, 72, 64, k.EPI_F32), (x, 0, 1, x, 1, 1, 72, 72, 64, k.EPI_F32)):      # 72 columns
        with pytest.raises(rv.RvError):
            k.gemm_bf16_blocks(*args, o)
    with pytest.raises(rv.RvError):        # a result that is never in blocks
        k.gemm_bf16_blocks(x, 0, 1, x, 0, 1, 72, 72, 64, k.EPI_F32, o, None, 1)
