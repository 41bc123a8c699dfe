"""fp32 MLP stage vs the oracle: the tiny 2-stage chain (tau = 1 then tau = 0), MSE in the
harness; stash / version / delayed-update semantics of paper Alg. 1 + Eq. 2 end to end.

Bar (fp32 products, K <= 128): normwise 1e-5 per tensor; the update itself 1e-6 against
w_old - eta * g_gpu in fp64.
"""
import numpy as np
import pytest
import torch

from oracle import blocks, stage as ostage
from paper_2401_01728_amd.inputs import gen
from util import close, dev, host64, rel_l2

pytestmark = pytest.mark.gpu


def kaiming_uniform_flat(seed, dims):
    """W ~ U(+-sqrt(6/fan_in)), b ~ U(+-1/sqrt(fan_in)), canonical flat order."""
    parts = []
    for i in range(len(dims) - 1):
        fan_in = dims[i]
        bw = np.sqrt(6.0 / fan_in); bb = 1.0 / np.sqrt(fan_in)
        parts.append(gen.uniform_f32(seed, 2 * i, dims[i] * dims[i + 1], -bw, bw))
        parts.append(gen.uniform_f32(seed, 2 * i + 1, dims[i + 1], -bb, bb))
    return np.concatenate(parts).astype(np.float32)


def test_two_stage_chain_config1():
    import paper_2401_01728_amd as rv
    dims, mb, n_mb, eta = [64, 128, 64], 8, 16, 0.01
    taus = [1, 0]                      # staleness falls to zero at the last peer
    w0 = [kaiming_uniform_flat(1 + s, dims) for s in range(2)]
    g_st = [rv.Stage.mlp(dims, mb, taus[s], eta) for s in range(2)]
    o_st = [ostage.Stage("mlp", taus[s], eta, w0[s], dims=dims) for s in range(2)]
    for s in range(2):
        assert g_st[s].num_params == 16576
        g_st[s].set_params(dev(w0[s]))
    xs = [gen.normal_f32(1, 100 + t, mb * 64).reshape(mb, 64) for t in range(n_mb)]
    ts = [gen.normal_f32(1, 200 + t, mb * 64).reshape(mb, 64) for t in range(n_mb)]
    # pipeline order: stage 0 forwards mb t, stage 1 forwards + backwards it at once (tau=0),
    # its input gradient reaches stage 0 one step later (tau=1).
    pending = {}
    worst = 0.0
    for t in range(n_mb + 1):
        if t < n_mb:
            h_g = g_st[0].forward(t, dev(xs[t])); h_o = o_st[0].forward(t, xs[t])
            close(host64(h_g), h_o, 1e-5, "t", group="MLP stage, bar 1e-5")
            y_g = g_st[1].forward(t, h_g); y_o = o_st[1].forward(t, h_o)
            close(host64(y_g), y_o, 1e-5, "t", group="MLP stage, bar 1e-5")
            dy_g = (2.0 / y_g.numel()) * (y_g - dev(ts[t]))          # harness: MSE gradient
            dy_o = 2.0 * (y_o - ts[t]) / y_o.size
            w_old = host64(g_st[1].get_params())
            dh_g = g_st[1].backward(t, dy_g.contiguous()); dh_o = o_st[1].backward(t, dy_o)
            close(host64(dh_g), dh_o, 2e-5, "t", group="MLP stage, bar 2e-5")
            gg = host64(g_st[1].last_grad())
            close(gg, o_st[1].last_grad, 2e-5, "t", group="MLP stage, bar 2e-5")
            w_new = host64(g_st[1].get_params())
            assert np.all(np.abs(w_new - (w_old - np.float64(np.float32(eta)) * gg)) <= 1e-6 * (np.abs(w_old) + eta * np.abs(gg)))
            pending[t] = (dh_g, dh_o)
        j = t - 1
        if j >= 0:
            dh_g, dh_o = pending.pop(j)
            dx_g = g_st[0].backward(j, dh_g); dx_o = o_st[0].backward(j, dh_o)
            assert o_st[0].last_staleness == min(j, 1)
            close(host64(dx_g), dx_o, 5e-5, "t", group="MLP stage, bar 5e-5")
            close(host64(g_st[0].last_grad()), o_st[0].last_grad, 5e-5, "t", group="MLP stage, bar 5e-5")
    for s in range(2):
        close(host64(g_st[s].get_params()), o_st[s].w, 1e-6, "t", group="MLP stage, bar 1e-6")
        assert g_st[s].in_flight == 0


@pytest.mark.parametrize("dims,mb,tau", [([5, 7, 3], 3, 2), ([33, 17, 65, 9], 19, 3), ([4, 4], 1, 0)])
def test_general_shapes_and_fifo_schedule(dims, mb, tau):
    import paper_2401_01728_amd as rv
    eta = 0.05
    w0 = kaiming_uniform_flat(5, dims)
    g = rv.Stage.mlp(dims, mb, tau, eta); g.set_params(dev(w0))
    o = ostage.Stage("mlp", tau, eta, w0, dims=dims)
    n = 7
    xs = [gen.normal_f32(5, 10 + t, mb * dims[0]).reshape(mb, dims[0]) for t in range(n)]
    dys = [gen.normal_f32(5, 50 + t, mb * dims[-1]).reshape(mb, dims[-1]) for t in range(n)]
    for t in range(n + tau):
        if t < n:
            close(host64(g.forward(t, dev(xs[t]))), o.forward(t, xs[t]), 1e-5, "t", group="MLP stage, bar 1e-5")
            assert g.in_flight == len(o.live)
        j = t - tau
        if j >= 0:
            dx = g.backward(j, dev(dys[j])); dxo = o.backward(j, dys[j])
            close(host64(dx), dxo, 1e-5, "t", group="MLP stage, bar 1e-5")
            close(host64(g.last_grad()), o.last_grad, 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.get_params()), o.w, 1e-6, "t", group="MLP stage, bar 1e-6")


def test_out_of_order_backward_keeps_versions_apart():
    """Any in-flight id may be backwarded; each must see the weights of ITS forward."""
    import paper_2401_01728_amd as rv
    dims, mb, tau, eta = [6, 9, 4], 4, 2, 0.1
    w0 = kaiming_uniform_flat(6, dims)
    g = rv.Stage.mlp(dims, mb, tau, eta); g.set_params(dev(w0))
    o = ostage.Stage("mlp", tau, eta, w0, dims=dims)
    x = lambda t: gen.normal_f32(6, 10 + t, mb * 6).reshape(mb, 6)
    dy = lambda t: gen.normal_f32(6, 50 + t, mb * 4).reshape(mb, 4)
    order = [("f", 0), ("f", 1), ("b", 1), ("f", 2), ("b", 2), ("f", 3), ("b", 3), ("f", 4), ("b", 0), ("b", 4)]
    for op, t in order:
        if op == "f":
            close(host64(g.forward(t, dev(x(t)))), o.forward(t, x(t)), 1e-5, "t", group="MLP stage, bar 1e-5")
        else:
            close(host64(g.backward(t, dev(dy(t)))), o.backward(t, dy(t)), 1e-5, "t", group="MLP stage, bar 1e-5")
            close(host64(g.last_grad()), o.last_grad, 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.get_params()), o.w, 1e-6, "t", group="MLP stage, bar 1e-6")


def test_error_paths_leave_state_unchanged():
    import paper_2401_01728_amd as rv
    dims, mb, tau = [4, 5, 3], 2, 1
    g = rv.Stage.mlp(dims, mb, tau, 0.1)
    w0 = kaiming_uniform_flat(7, dims); g.set_params(dev(w0))
    x = torch.zeros(mb, 4, device="cuda"); dy = torch.ones(mb, 3, device="cuda")
    g.forward(10, x); g.forward(11, x)
    for bad, code in [(lambda: g.forward(12, x), rv.api.RV_E_STASH_FULL),
                      (lambda: g.backward(99, dy), rv.api.RV_E_UNKNOWN_MB)]:
        with pytest.raises(rv.RvError) as e:
            bad()
        assert e.value.status == code
    g.backward(10, dy)
    with pytest.raises(rv.RvError) as e:
        g.forward(11, x)
    assert e.value.status == rv.api.RV_E_DUP_MB
    with pytest.raises(rv.RvError):
        g.set_params(dev(w0))                      # a microbatch is still in flight
    assert g.in_flight == 1
    g.backward(11, dy)
    assert g.in_flight == 0


def test_stage_with_momentum_and_weight_decay():
    """Stale-gradient schedule with the section 4.1 optimiser (momentum 0.9, weight decay 5e-4)."""
    import paper_2401_01728_amd as rv
    dims, mb, tau, eta = [33, 17, 9], 6, 2, 0.05
    w0 = kaiming_uniform_flat(8, dims)
    g = rv.Stage.mlp(dims, mb, tau, eta); g.set_params(dev(w0)); g.set_optimizer(0.9, 5e-4)
    o = ostage.Stage("mlp", tau, eta, w0, dims=dims, momentum=0.9, weight_decay=5e-4)
    n = 8
    for t in range(n + tau):
        if t < n:
            x = gen.normal_f32(8, 10 + t, mb * dims[0]).reshape(mb, dims[0])
            close(host64(g.forward(t, dev(x))), o.forward(t, x), 1e-5, "t", group="MLP stage, bar 1e-5")
        j = t - tau
        if j >= 0:
            dy = gen.normal_f32(8, 50 + j, mb * dims[-1]).reshape(mb, dims[-1])
            close(host64(g.backward(j, dev(dy))), o.backward(j, dy), 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.get_params()) - w0, o.w - w0, 1e-4, "t", group="MLP stage, bar 1e-4")
    with pytest.raises(rv.RvError):
        g.set_optimizer(-1.0, 0.0)


@pytest.mark.parametrize("A,momentum", [(3, 0.0), (2, 0.9)])
def test_stage_with_gradient_accumulation(A, momentum):
    """Section 4.2: the gradients of A microbatches are summed before one update; the parameters
    stay put in between and the staleness is counted in updates."""
    import paper_2401_01728_amd as rv
    dims, mb, tau, eta = [33, 17, 9], 6, 1, 0.05
    w0 = kaiming_uniform_flat(8, dims)
    g = rv.Stage.mlp(dims, mb, tau, eta); g.set_params(dev(w0)); g.set_accumulation(A)
    o = ostage.Stage("mlp", tau, eta, w0, dims=dims, accumulate=A, momentum=momentum)
    if momentum:
        g.set_optimizer(momentum, 0.0)
    n = 3 * A + 1                                            # ends inside a group
    for t in range(n + tau):
        if t < n:
            x = gen.normal_f32(8, 10 + t, mb * dims[0]).reshape(mb, dims[0])
            close(host64(g.forward(t, dev(x))), o.forward(t, x), 1e-5, "t", group="MLP stage, bar 1e-5")
        j = t - tau
        if j >= 0:
            dy = gen.normal_f32(8, 50 + j, mb * dims[-1]).reshape(mb, dims[-1])
            before = g.get_params().clone()
            close(host64(g.backward(j, dev(dy))), o.backward(j, dy), 1e-5, "t", group="MLP stage, bar 1e-5")
            close(host64(g.last_grad()), o.last_grad, 1e-5, "t", group="MLP stage, bar 1e-5")
            moved = not torch.equal(before, g.get_params())
            assert moved == ((j + 1) % A == 0)
    close(host64(g.get_params()) - w0, o.w - w0, 1e-4, "t", group="MLP stage, bar 1e-4")
    with pytest.raises(rv.RvError):
        g.set_accumulation(0)


@pytest.mark.parametrize("dims,mb,momentum", [
    # one launch per direction: 16 / 32 / 64 rows, one to four layers, widest rows, contractions of one piece,
    # of exactly one request and of more than one
    ([1, 1], 1, 0.0), ([16, 128, 16], 16, 0.9), ([17, 129, 15], 17, 0.0), ([256, 13, 256], 33, 0.0),
    ([250, 40, 31, 7], 64, 0.9), ([120, 256, 20], 16, 0.0), ([40, 64, 3, 33, 128], 48, 0.0),
    # the same with more than 32 rows: up to 64 wide
    ([64, 13, 64], 33, 0.0), ([60, 40, 31, 7], 64, 0.9), ([40, 64, 3, 33, 64], 48, 0.0),
    # a 32 x 32 tile per workgroup: just past the widths / rows / layers of the form above
    ([257, 64, 31], 8, 0.9), ([64, 100, 64], 65, 0.0), ([8, 9, 10, 11, 12, 13], 5, 0.9), ([520, 40], 33, 0.0),
    # LDS tiles of 64 and of 128 with ragged edges (one layer: no gate, so no gate can fall the other
    # way); contractions of less than a tile, of one, of two and a bit
    ([1030, 2052], 2051, 0.0), ([2052, 2060], 2049, 0.9), ([31, 4100], 600, 0.0), ([32, 1037], 1030, 0.9), ([65, 2048], 2048, 0.0),
    # an input of several turns of the workgroups that copy it, with a piece and a float left over
    ([4099, 9], 2051, 0.0),
])
def test_product_forms_at_their_edges(dims, mb, momentum):
    """Two microbatches against the oracle.  Bar: sums of K <= 4100 fp32 products with random signs, in any order,
    stay within about sqrt(K) * 2^-24 = 3.8e-6 normwise; 1e-5 leaves a factor of 2.6."""
    import paper_2401_01728_amd as rv
    eta, wd = 1e-3, 1e-3 if momentum else 0.0
    w0 = kaiming_uniform_flat(61, dims)
    g = rv.Stage.mlp(dims, mb, 1, eta); g.set_params(dev(w0))
    if momentum:
        g.set_optimizer(momentum, wd)
    o = ostage.Stage("mlp", 1, eta, w0, dims=dims, momentum=momentum, weight_decay=wd)
    x = [gen.normal_f32(61, 10 + t, mb * dims[0]).reshape(mb, dims[0]) for t in range(2)]
    dy = [gen.normal_f32(61, 50 + t, mb * dims[-1], std=0.1).reshape(mb, dims[-1]) for t in range(2)]
    grp = "MLP product forms, bar 1e-5"
    for t in range(2):
        close(host64(g.forward(t, dev(x[t]))), o.forward(t, x[t]), 1e-5, "t", group=grp)
    for t in range(2):
        close(host64(g.backward(t, dev(dy[t]))), o.backward(t, dy[t]), 1e-5, "t", group=grp)
        close(host64(g.last_grad()), o.last_grad, 1e-5, "t", group=grp)
    # two updates: each rounds the weight once (2^-24 of it), and eta times a gradient off by 1e-5 is less than 1e-7 of
    # the weights' norm
    close(host64(g.get_params()), o.w, 1e-6, "t", group="MLP product forms: parameters, bar 1e-6")


@pytest.mark.parametrize("momentum", [0.0, 0.9])
@pytest.mark.parametrize("dims,mb", [([24, 24], 9), ([24, 40, 24], 9), ([300, 40, 300], 9), ([300, 300], 40), ([64, 64], 2000),
                                     ([1100, 1100], 1030)])
def test_output_may_share_the_input_buffer(dims, mb, momentum):
    import paper_2401_01728_amd as rv
    w0 = kaiming_uniform_flat(62, dims)
    g = rv.Stage.mlp(dims, mb, 0, 0.05); g.set_params(dev(w0))
    if momentum:
        g.set_optimizer(momentum, 1e-3)
    o = ostage.Stage("mlp", 0, 0.05, w0, dims=dims, momentum=momentum, weight_decay=1e-3 if momentum else 0.0)
    x = gen.normal_f32(62, 1, mb * dims[0]).reshape(mb, dims[0])
    b = dev(x)
    g.forward(0, b, b)
    close(host64(b), o.forward(0, x), 1e-5, "t", group="MLP stage, bar 1e-5")
    dy = dev(x)
    g.backward(0, dy, dy)
    dxo = o.backward(0, x)
    close(host64(dy), dxo, 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.last_grad()), o.last_grad, 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.get_params()) - w0, o.w - w0, 1e-4, "t", group="MLP stage, bar 1e-4")


def _same(got, ref, tol, grp):
    """Infinities and NaN in the same places, the rest within the bar."""
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref)
    close(got[ok], ref[ok], tol, "t", group=grp)


# one launch per direction (16, 32 and 64 rows), split contraction, LDS tiles; widths and row counts that are no
# multiple of a piece, so that the last weight row and the last activation row are what clamped indexes read
_ODD = [([20, 7], 5), ([20, 24, 7], 13), ([17, 33, 9], 29), ([131, 30, 33], 45), ([61, 30, 33], 45), ([300, 21, 9], 13), ([301, 1030], 1030)]


@pytest.mark.parametrize("where,dims,mb", [("first weight row",) + c for c in _ODD + [([18, 21, 19, 5], 50)]] +
                         [("last weight row",) + c for c in _ODD if len(c[0]) == 3] + [("activation",) + c for c in _ODD])
@pytest.mark.filterwarnings("ignore::RuntimeWarning")
def test_an_infinity_stays_where_it_belongs(where, dims, mb):
    """One infinite weight in the last row of the first or last layer, or one infinite activation in the last row
    of the microbatch, against the oracle.  (Two layers for the last two: the unit in front of the last layer's
    infinity has its gate open, and no hidden unit sums infinities of both signs - there the oracle's product with
    the gate and its maximum give NaN.)"""
    import paper_2401_01728_amd as rv
    w0 = kaiming_uniform_flat(63, dims)
    x = gen.normal_f32(63, 1, mb * dims[0]).reshape(mb, dims[0])
    dy = gen.normal_f32(63, 2, mb * dims[-1], std=0.1).reshape(mb, dims[-1])
    if where == "activation":
        x[mb - 1, dims[0] - 1] = np.inf
    elif where == "first weight row":
        w0[(dims[0] - 1) * dims[1] + dims[1] // 2] = np.inf
    else:
        last = dims[0] * dims[1] + dims[1]
        w0[last - 1] = 100.0
        w0[last + (dims[1] - 1) * dims[2] + dims[2] // 2] = np.inf
    g = rv.Stage.mlp(dims, mb, 0, 0.05); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 0.05, w0, dims=dims)
    grp = "MLP stage, bar 1e-5"
    _same(host64(g.forward(0, dev(x))), o.forward(0, x), 1e-5, grp)
    dx, dxo = g.backward(0, dev(dy)), o.backward(0, dy)
    _same(host64(dx), dxo, 1e-5, grp)
    _same(host64(g.last_grad()), o.last_grad, 1e-5, grp)
    _same(host64(g.get_params()), o.w, 1e-6, "MLP stage, bar 1e-6")


@pytest.mark.parametrize("dims,mb,momentum", [
    # results of at most 32 rows or columns and thousands the other way: a tile per wave up to a contraction of 128,
    # split beyond, in both gradients at once and each beside the other forms; one row more takes LDS tiles
    ([128, 8200], 8, 0.0), ([129, 8200], 8, 0.9), ([8, 33000], 32, 0.9), ([33000, 7], 8, 0.0), ([8, 5], 33000, 0.9), ([5, 8200], 33, 0.0),
    ([3, 33000], 64, 0.0), ([3, 33000], 65, 0.0), ([8200, 200], 16, 0.9), ([130, 40], 8200, 0.0),
])
def test_thin_products(dims, mb, momentum):
    """As above.  Bar: contractions up to K = 33000, sqrt(K) * 2^-24 = 1.1e-5 in the worst order of additions; 3e-5
    leaves a factor of 2.8.  (One layer: no gate.)"""
    import paper_2401_01728_amd as rv
    eta, wd = 1e-3, 1e-3 if momentum else 0.0
    w0 = kaiming_uniform_flat(64, dims)
    g = rv.Stage.mlp(dims, mb, 0, eta); g.set_params(dev(w0))
    if momentum:
        g.set_optimizer(momentum, wd)
    o = ostage.Stage("mlp", 0, eta, w0, dims=dims, momentum=momentum, weight_decay=wd)
    x = gen.normal_f32(64, 10, mb * dims[0]).reshape(mb, dims[0])
    dy = gen.normal_f32(64, 50, mb * dims[-1], std=0.1).reshape(mb, dims[-1])
    grp = "MLP thin products, bar 3e-5"
    close(host64(g.forward(0, dev(x))), o.forward(0, x), 3e-5, "t", group=grp)
    close(host64(g.backward(0, dev(dy))), o.backward(0, dy), 3e-5, "t", group=grp)
    close(host64(g.last_grad()), o.last_grad, 3e-5, "t", group=grp)
    close(host64(g.get_params()), o.w, 1e-6, "t", group="MLP product forms: parameters, bar 1e-6")


def test_more_version_slots_than_one_launch_clears():
    """tau = 70: 72 version slots, each bound to a microbatch in turn.  Contractions are no multiple of 16, so the
    kernels read the zero behind every slot's parameters; the memory the slots may get held NaN before."""
    import paper_2401_01728_amd as rv
    dims, mb, tau, eta = [20, 24, 7], 5, 70, 1e-3
    junk = [torch.full((1 << 19,), float("nan"), device="cuda") for _ in range(64)]
    torch.cuda.synchronize(); del junk; torch.cuda.empty_cache()
    w0 = kaiming_uniform_flat(65, dims)
    g = rv.Stage.mlp(dims, mb, tau, eta); g.set_params(dev(w0))
    o = ostage.Stage("mlp", tau, eta, w0, dims=dims)
    for t in range(2 * tau + 10):
        x = gen.normal_f32(65, 10 + t, mb * dims[0]).reshape(mb, dims[0])
        close(host64(g.forward(t, dev(x))), o.forward(t, x), 1e-5, "t", group="MLP stage, bar 1e-5")
        if t >= tau:
            dy = gen.normal_f32(65, 500 + t, mb * dims[-1], std=0.1).reshape(mb, dims[-1])
            close(host64(g.backward(t - tau, dev(dy))), o.backward(t - tau, dy), 1e-5, "t", group="MLP stage, bar 1e-5")
    close(host64(g.get_params()), o.w, 1e-6, "t", group="MLP stage, bar 1e-6")


# 64x64 weight-gradient tiles two to a workgroup: an odd number of them, ragged or whole, contractions of one and two tile depths
@pytest.mark.parametrize("dims,mb,momentum", [([700, 830], 40, 0.9), ([704, 832], 32, 0.0), ([704, 832], 64, 0.9)] +
                         # the split walk: one set of requests exactly, a second one begun, full, a third and a fourth begun
                         [([K, 40], 9, 0.0) for K in (256, 264, 512, 513, 769, 1030)])
def test_two_tiles_a_workgroup_and_the_split_walk(dims, mb, momentum):
    test_product_forms_at_their_edges(dims, mb, momentum)


# LDS tiles walked in three bf16 planes, steps of 16 in k.  Tiles of 128: up to five steps are loaded by the general form, from six on
# whole steps by pieces (one less where a row is no multiple of a piece).  Tiles of 64: the same at 10 steps; from 80 in
# k on by two halves of a workgroup, an even or odd number of steps.  The last ones: input gradient tiles of 64 two to a workgroup beside
# split weight gradients, an odd and an even number of them, on each side of the rule.
@pytest.mark.parametrize("dims,mb", [([K, 4100], 1030) for K in (95, 96, 97, 113, 130)] + [([96, 4101], 1030)] +
                         [([K, 700], 900) for K in (79, 80, 81, 96, 97, 255, 256, 257, 288, 576, 577)] + [([600, 701], 900), ([592, 702], 900)] +
                         [([832, 24], 700), ([700, 110], 660), ([700, 111], 660)])
def test_products_in_three_planes(dims, mb):
    """Bar: sums of K products with random signs in fp32 stay within sqrt(K) * 2^-24 normwise in any order; the pieces left out
    are together at most 2^-24 of a product."""
    import paper_2401_01728_amd as rv
    w0 = kaiming_uniform_flat(66, dims)
    g = rv.Stage.mlp(dims, mb, 0, 1e-3); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 1e-3, w0, dims=dims)
    x = gen.normal_f32(66, 1, mb * dims[0]).reshape(mb, dims[0])
    dy = gen.normal_f32(66, 2, mb * dims[1], std=0.1).reshape(mb, dims[1])
    bar = lambda k: float(np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24)
    close(host64(g.forward(0, dev(x))), o.forward(0, x), bar(dims[0]), "t", group="MLP in three planes: out")
    close(host64(g.backward(0, dev(dy))), o.backward(0, dy), bar(dims[1]), "t", group="MLP in three planes: grad_in")
    close(host64(g.last_grad()), o.last_grad, bar(mb), "t", group="MLP in three planes: gradient")


@pytest.mark.parametrize("where", ["first weight row", "activation"])
@pytest.mark.filterwarnings("ignore::RuntimeWarning")
def test_an_infinity_in_a_large_tile(where):
    test_an_infinity_stays_where_it_belongs(where, [301, 4100], 1030)


@pytest.mark.parametrize("dims,mb,what,at", [
    # forward by two halves of a workgroup: in the first half's part of the contraction, in the second one's, in both operands' last element
    ([300, 700], 900, "weight", (5, 350)), ([300, 700], 900, "weight", (299, 699)), ([300, 700], 900, "activation", (899, 5)),
    ([300, 700], 900, "activation", (450, 299)),
    # 64x64 tiles two to a workgroup, an odd number of them: weight gradient (activation, gradient), input gradient (weight, gradient)
    ([700, 830], 40, "activation", (39, 699)), ([700, 830], 40, "activation", (0, 0)), ([700, 830], 40, "gradient", (20, 829)),
    ([832, 24], 700, "weight", (831, 23)), ([832, 24], 700, "gradient", (699, 0)),
])
@pytest.mark.filterwarnings("ignore::RuntimeWarning")
def test_an_infinity_in_tiles_that_share_a_workgroup(dims, mb, what, at):
    """As test_an_infinity_stays_where_it_belongs: both tiles, or both halves of one, walk again together."""
    import paper_2401_01728_amd as rv
    K, N = dims
    w0 = kaiming_uniform_flat(70, dims)
    x = gen.normal_f32(70, 1, mb * K).reshape(mb, K)
    dy = gen.normal_f32(70, 2, mb * N, std=0.1).reshape(mb, N)
    if what == "weight": w0[at[0] * N + at[1]] = np.inf
    else: (x if what == "activation" else dy)[at] = np.inf
    g = rv.Stage.mlp(dims, mb, 0, 0.05); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 0.05, w0, dims=dims)
    grp = "MLP stage, bar 1e-5"
    _same(host64(g.forward(0, dev(x))), o.forward(0, x), 1e-5, grp)
    dx, dxo = g.backward(0, dev(dy)), o.backward(0, dy)
    _same(host64(dx), dxo, 1e-5, grp)
    _same(host64(g.last_grad()), o.last_grad, 1e-5, grp)


@pytest.mark.parametrize("scale", [1e-26, 1e-31, 1e-34])
def test_gradients_near_the_smallest_numbers(scale):
    """The third piece of 1e-33 is no bf16 number unless the operands are scaled.  Bar: sums of fp32 products as above; of
    results down to 1e-37 the smallest number's half, 7e-46, is far below 2^-24."""
    import paper_2401_01728_amd as rv
    dims, mb = [1500, 4100], 1030
    w0 = kaiming_uniform_flat(67, dims)
    g = rv.Stage.mlp(dims, mb, 0, 1e-3); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 1e-3, w0, dims=dims)
    x = gen.normal_f32(67, 1, mb * dims[0]).reshape(mb, dims[0])
    dy = gen.normal_f32(67, 2, mb * dims[1]).reshape(mb, dims[1]) * np.float32(scale)
    g.forward(0, dev(x)); o.forward(0, x)
    dx, dxo = host64(g.backward(0, dev(dy))), o.backward(0, dy)
    up = 1.0 / scale                       # (the comparison's own squares would underflow)
    close(dx * up, dxo * up, 1e-5, "t", group="MLP near the smallest numbers, bar 1e-5")
    close(host64(g.last_grad()) * up, o.last_grad * up, 1e-5, "t", group="MLP near the smallest numbers, bar 1e-5")


# forward / input gradient / weight gradient: tiles of 128 / 64 / 128; by two halves of a workgroup / split / split; split / split /
# 64x64 tiles two to a workgroup, an odd number of them
_PLANES = [([1500, 4100], 1030), ([300, 700], 900), ([700, 830], 40)]


@pytest.mark.parametrize("small", ["rows", "columns", "weights", "gradient"])
@pytest.mark.parametrize("dims,mb", _PLANES)
def test_small_operands_beside_ordinary_ones(dims, mb, small):
    """Every row and column against its own scale: every other row of x and of the other rows of dy at 1e-36; the first 64 columns
    of W and of dy, which are tiles of their own beside ordinary ones; weights of few bits near 1e-42 under activations and
    gradients of 1e8; a gradient of 1e-41 with activations of 1e8.  Bar as test_products_in_three_planes."""
    import paper_2401_01728_amd as rv
    K, N = dims
    s = {"weights": 1e-41, "gradient": 1e-41}.get(small, 1e-36)
    one = lambda n: np.ones(n)
    xr, wc, dr, dc = one(mb), one(N), one(mb), one(N)      # scales of x's rows, W's columns, dy's rows and columns
    if small == "rows": xr[::2] = s; dr[1::2] = s
    if small == "columns": wc[:64] = s; dc[:64] = s
    if small == "weights": wc[:] = s; xr[:] = 1e8; dr[:] = 1e8
    if small == "gradient": dr[:] = s; xr[:] = 1e8
    w0 = kaiming_uniform_flat(68, dims)
    w0[K * N:] = 0.0
    w0[:K * N] = (w0[:K * N].reshape(K, N) * wc).astype(np.float32).ravel()
    x = (gen.normal_f32(68, 1, mb * K).reshape(mb, K) * xr[:, None]).astype(np.float32)
    dy = (gen.normal_f32(68, 2, mb * N).reshape(mb, N) * dr[:, None] * dc).astype(np.float32)
    g = rv.Stage.mlp(dims, mb, 0, 0.0); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 0.0, w0, dims=dims)
    bar = lambda k: float(np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24)
    grp = "MLP, small operands: "
    up = 1.0 / (xr[:, None] * wc)
    close(host64(g.forward(0, dev(x))) * up, o.forward(0, x) * up, bar(K), "t", group=grp + "out")
    dx, dxo = host64(g.backward(0, dev(dy))), o.backward(0, dy)
    if small != "gradient":                # (there the input gradient is as small as the gradient: nothing of 24 bits)
        up = 1.0 / (dr[:, None] * wc.max())
        close(dx * up, dxo * up, bar(N), "t", group=grp + "grad_in")
    up = 1.0 / ((xr * dr).max() * dc)      # (rows: each of the products has one small operand)
    gr, gro = host64(g.last_grad())[:K * N].reshape(K, N), o.last_grad[:K * N].reshape(K, N)
    close(gr * up, gro * up, bar(mb), "t", group=grp + "gradient")


@pytest.mark.parametrize("xs,ws,ds", [(1e18, 1e14, 1e17), (1e35, 1e-2, 1e-3), (1e-3, 1e36, 1e-2), (1e-2, 1e-3, 1e35)])
@pytest.mark.parametrize("dims,mb", _PLANES)
def test_large_operands(dims, mb, xs, ws, ds):
    """Results past 2^96, operands past 2^112: such tiles leave the range of the scaled sums or pieces and are walked again; the
    results are ordinary floats.  Bar as test_products_in_three_planes."""
    import paper_2401_01728_amd as rv
    K, N = dims
    w0 = (kaiming_uniform_flat(71, dims) * np.float32(ws)).astype(np.float32)
    x = gen.normal_f32(71, 1, mb * K).reshape(mb, K) * np.float32(xs)
    dy = gen.normal_f32(71, 2, mb * N).reshape(mb, N) * np.float32(ds)
    g = rv.Stage.mlp(dims, mb, 0, 0.0); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 0.0, w0, dims=dims)
    bar = lambda k: float(np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24)
    grp = "MLP, large operands: "
    close(host64(g.forward(0, dev(x))), o.forward(0, x), bar(K), "t", group=grp + "out")
    close(host64(g.backward(0, dev(dy))), o.backward(0, dy), bar(N), "t", group=grp + "grad_in")
    close(host64(g.last_grad()), o.last_grad, bar(mb), "t", group=grp + "gradient")


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("dims,mb", [([4096, 1024], 512), ([16384, 1024], 512), ([256, 16384], 2100), ([512, 1100], 16400)])
def test_sums_of_one_sign(dims, mb, sign):
    """Uniform operands without cancellation (the weights' sign times `sign`): nothing is lost to one side.  In k: 4096 and 16384 by two
    halves of a workgroup, an input gradient of 16384, a weight gradient of 16400 rows.  Bars: normwise as
    test_products_in_three_planes; the mean error 2^-22 of the result, four roundings - a sum that lost half a unit in its last
    place every 16 in k would be off by K / 16 * 2^-26 or more, 3.8e-6 at 4096."""
    import paper_2401_01728_amd as rv
    K, N = dims
    w0 = np.concatenate([gen.uniform_f32(69, 0, K * N, 0.0, 1.0) * np.float32(sign), np.zeros(N, np.float32)]).astype(np.float32)
    x = gen.uniform_f32(69, 1, mb * K, 0.0, 1.0).reshape(mb, K)
    dy = gen.uniform_f32(69, 2, mb * N, 0.0, 1.0).reshape(mb, N)
    g = rv.Stage.mlp(dims, mb, 0, 0.0); g.set_params(dev(w0))
    o = ostage.Stage("mlp", 0, 0.0, w0, dims=dims)

    def check(got, ref, k, what):
        close(got, ref, float(np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24), "t", group="MLP, sums of one sign: " + what)
        assert abs((got - ref).mean()) <= 2.0 ** -22 * np.abs(ref).mean(), (what, (got - ref).mean() / np.abs(ref).mean())

    check(host64(g.forward(0, dev(x))), o.forward(0, x), K, "out")
    check(host64(g.backward(0, dev(dy))), o.backward(0, dy), N, "grad_in")
    check(host64(g.last_grad())[:K * N], o.last_grad[:K * N], mb, "gradient")


# 32x16 tiles: contractions of less than a group of 16, exactly one per wave, one more, both sets of requests exactly, a third begun; the
# last row and column counts on each side of a tile's edge; forward and input gradient at the limits of the rule and one past them
@pytest.mark.parametrize("dims,mb", [([K, 40], 33) for K in (7, 128, 129, 1024, 1025)] + [([300, 17], 32), ([300, 16], 65), ([31, 600], 70),
                                     ([40, 4096], 17), ([2048, 300], 9), ([2049, 300], 9), ([300, 4097], 9),
                                     # forward tiles and copying workgroups together as many as the CUs; input gradients of a contraction
                                     # of 256 and one less, longer than the weight gradient's and not; one turn of the CUs more
                                     ([40, 4080], 17), ([300, 256], 20), ([300, 255], 20), ([64, 260], 259), ([64, 260], 260), ([1900, 600], 20)])
def test_slim_tiles(dims, mb):
    """Bar as test_product_forms_at_their_edges."""
    test_product_forms_at_their_edges(dims, mb, 0.0)
    test_product_forms_at_their_edges(dims, mb, 0.9)
