"""Decoder stage vs the oracle: the stage step of paper Alg. 1 with the stale-gradient
update of Eq. 2 (forward(t), backward(t - tau) at the stashed weight version, update).

Both sides receive the same values: fp32 master weights; activations and upstream
gradients already rounded to bf16.  Bars (bf16 products, fp32 accumulation): for outputs,
input gradients and every parameter-gradient tensor 2e-2 normwise AND element by element
|got - ref| <= 2e-2 * (|ref| + rms(ref)) (util.close; achieved errors are printed at the end
of the run); the update itself 1e-6 against w_old - eta * g_gpu in fp64.
"""
import numpy as np
import pytest
import torch

from oracle import blocks, stage as ostage
from paper_2401_01728_amd.inputs import gen
from util import bf16_normal, close, dev, host64, rel_l2

pytestmark = pytest.mark.gpu

TOL = 2e-2


def decoder_params_host(seed, L, d, f):
    """weights, biases, LN beta ~ N(0, 0.02); LN gamma ~ 1 + N(0, 0.02); canonical order."""
    per = 4 * d * d + 2 * d * f + 9 * d + f
    w = gen.normal_f32(seed, 0, L * per, 0.0, 0.02)
    for l in range(L):
        base = l * per
        w[base:base + d] += np.float32(1.0)
        o2 = base + 2 * d + 3 * d * d + 3 * d + d * d + d
        w[o2:o2 + d] += np.float32(1.0)
    return w


def check_tensors(got_flat, ref_flat, shapes, tol=TOL, what="", group=None):
    """Every parameter-gradient tensor on its own (got_flat may be fp32: widened per tensor)."""
    got = blocks.unflatten(got_flat, shapes); ref = blocks.unflatten(ref_flat, shapes)
    grp = group or what.split(" step")[0] + " param grads"
    for name, _ in shapes:
        close(got[name], ref[name], tol, "%s %s" % (what, name), group=grp)


def check_update(w_new, w_old, gg, eta):
    """Eq. 2 in isolation: the new master against w_old - eta * (the GPU's own gradient) in fp64."""
    e = np.float64(np.float32(eta))
    for lo in range(0, w_new.size, 1 << 24):
        sl = slice(lo, lo + (1 << 24))
        wn, wo, g = (np.asarray(a[sl], dtype=np.float64) for a in (w_new, w_old, gg))
        assert np.all(np.abs(wn - (wo - e * g)) <= 1e-6 * (np.abs(wo) + eta * np.abs(g)))


def run_schedule(L, d, H, f, S, mb, tau, n_mb, seed, eta=1e-3, grad_std=1e-3, fused_step=False):
    import paper_2401_01728_amd as rv
    shapes = blocks.decoder_param_shapes(L, d, f)
    w0 = decoder_params_host(seed, L, d, f)
    g = rv.Stage.decoder(L, d, H, f, S, mb, tau, eta, keep_grad=True)
    assert g.num_params == w0.size
    g.set_params(dev(w0))
    o = ostage.Stage("decoder", tau, eta, w0, n_blocks=L, d=d, h=H, f=f)
    tag = "decoder L%d d%d S%d tau%d" % (L, d, S, tau)
    for t in range(n_mb + tau):
        j = t - tau
        both = fused_step and t < n_mb and j >= 0
        if t < n_mb:
            x, x64 = bf16_normal(seed, 1000 + t, (mb, S, d))
        if j >= 0:
            dy, dy64 = bf16_normal(seed, 2000 + j, (mb, S, d), std=grad_std)
            w_old = host64(g.get_params())
        if both:                        # rv_stage_step: the two halves overlap on two streams
            y, dx = g.step(t, x, j, dy)
        if t < n_mb:
            if not both:
                y = g.forward(t, x)
            close(host64(y), o.forward(t, x64), TOL, "out %d" % t, group=tag + " out")
        if j >= 0:
            if not both:
                dx = g.backward(j, dy)
            dxo = o.backward(j, dy64)
            assert o.last_staleness == min(j, tau)
            close(host64(dx), dxo, TOL, "grad_in %d" % j, group=tag + " grad_in")
            gg = host64(g.last_grad())
            check_tensors(gg, o.last_grad, shapes, what="grad step %d" % j, group=tag + " param grads")
            check_update(host64(g.get_params()), w_old, gg, eta)
    assert g.in_flight == 0
    # after n_mb stale updates the two parameter vectors still agree to the gradient bar times eta
    assert rel_l2(host64(g.get_params()) - w0, o.w - w0) < TOL
    return g, o


@pytest.mark.parametrize("L,d,H,f,S,mb,tau", [
    (2, 128, 2, 256, 128, 2, 2),       # dh = 64, several tiles per product
    (1, 256, 2, 512, 192, 1, 1),       # dh = 128, seq not a multiple of 128
    (3, 192, 3, 320, 64, 3, 0),        # tau = 0: sequential SGD; widths that are not multiples of 128
])
def test_small_stage_schedules(L, d, H, f, S, mb, tau):
    run_schedule(L, d, H, f, S, mb, tau, n_mb=2 * tau + 2, seed=20 + L)


# LayerNorm backward by 2, 4 and 8 rows per workgroup for widths up to 1024 and beyond (16: the full-size stages)
@pytest.mark.parametrize("d,H,S,mb", [(128, 2, 512, 1), (128, 2, 512, 2), (128, 2, 512, 4),
                                      (1088, 17, 64, 1), (1088, 17, 512, 2), (1088, 17, 512, 4), (2304, 18, 64, 1)])
def test_stage_of_few_or_many_tokens(d, H, S, mb):
    run_schedule(1, d, H, 64, S, mb, 0, n_mb=1, seed=60 + mb)


@pytest.mark.parametrize("L,d,H,f,S,mb,tau", [(2, 128, 2, 256, 128, 2, 2), (2, 256, 2, 512, 128, 1, 0),
                                               (3, 192, 3, 320, 64, 3, 1)])
def test_fused_step_equals_forward_then_backward(L, d, H, f, S, mb, tau):
    """rv_stage_step must give what forward(t); backward(t - tau) gives (oracle order F, B)."""
    run_schedule(L, d, H, f, S, mb, tau, n_mb=2 * tau + 4, seed=40 + L, fused_step=True)


def test_fused_step_is_bitwise_the_two_calls():
    """... and the update applied inside the gradient kernels (the default) gives, bit for bit, the
    parameters of the variant that also keeps the gradient; only the latter can be read back."""
    import paper_2401_01728_amd as rv
    L, d, H, f, S, mb, tau = 2, 128, 2, 256, 128, 2, 2
    w0 = dev(decoder_params_host(9, L, d, f))
    res = []
    for fused, keep in ((False, False), (True, False), (True, True)):
        g = rv.Stage.decoder(L, d, H, f, S, mb, tau, 1e-3, keep_grad=keep); g.set_params(w0)
        outs = []
        for t in range(8 + tau):
            j = t - tau
            x, _ = bf16_normal(9, 1000 + t, (mb, S, d)); dy, _ = bf16_normal(9, 2000 + max(j, 0), (mb, S, d), std=1e-3)
            if fused and t < 8 and j >= 0:
                y, dx = g.step(t, x, j, dy); outs += [y, dx]
            else:
                if t < 8:
                    outs.append(g.forward(t, x))
                if j >= 0:
                    outs.append(g.backward(j, dy))
        outs.append(g.get_params())
        torch.cuda.synchronize()
        res.append([o.clone() for o in outs])
        if keep:
            assert torch.isfinite(g.last_grad()).all()
        else:
            with pytest.raises(rv.RvError):
                g.last_grad()
    for other in res[1:]:
        assert len(other) == len(res[0])
        for a, b in zip(res[0], other):
            assert torch.equal(a, b)


def test_deep_staleness_reduced_shape():
    """The deep-staleness stage's whole run of 64 interleaved microbatches (4 warm-up forwards, 60
    steady steps through rv_stage_step, 4 draining backwards; 12 blocks, tau = 4, 5 stash slots
    and weight versions) at reduced widths: d = 448 with 7 heads of 64 (1600 / 4 = 400 is not a
    multiple of the head size), ffn 1792, seq 128, microbatch 2."""
    run_schedule(12, 448, 7, 1792, 128, 2, 4, n_mb=64, seed=5, fused_step=True)


def test_backward_uses_the_stashed_version_not_the_current_one():
    """With the configs' learning rate one update moves a weight by less than bf16 resolves, so a
    backward at the wrong version would pass every other test.  Here eta is chosen so that one
    update displaces the parameters by about 10 % of their norm: the stage must still match the
    oracle, and an oracle with the mistake planted in it (backward at the CURRENT parameters)
    must be far outside the bar, else this test could not tell the difference."""
    import paper_2401_01728_amd as rv
    L, d, H, f, S, mb, tau, seed, n = 2, 128, 2, 256, 128, 2, 2, 77, 5
    shapes = blocks.decoder_param_shapes(L, d, f)
    w0 = decoder_params_host(seed, L, d, f)
    xs = [bf16_normal(seed, 1000 + t, (mb, S, d)) for t in range(n)]
    dys = [bf16_normal(seed, 2000 + t, (mb, S, d), std=1e-3) for t in range(n)]
    _, g0 = blocks.decoder_backward(w0.astype(np.float64), L, d, H, f, 1e-5, xs[0][1], dys[0][1])
    eta = float(np.float32(0.1 * np.linalg.norm(w0) / np.linalg.norm(g0)))

    class CurrentWeightsStage(ostage.Stage):           # the planted mistake
        def backward(self, mb_id, dy, defer=False):
            _, x, k = self.live[mb_id]
            self.live[mb_id] = (self.w.copy(), x, k)
            return super().backward(mb_id, dy, defer)

    g = rv.Stage.decoder(L, d, H, f, S, mb, tau, eta, keep_grad=True); g.set_params(dev(w0))
    o = ostage.Stage("decoder", tau, eta, w0, n_blocks=L, d=d, h=H, f=f)
    bad = CurrentWeightsStage("decoder", tau, eta, w0, n_blocks=L, d=d, h=H, f=f)
    told_apart = 0.0
    for t in range(n + tau):
        j = t - tau
        if t < n and j >= 0:
            y, dx = g.step(t, xs[t][0], j, dys[j][0])
        elif t < n:
            y = g.forward(t, xs[t][0])
        else:
            dx = g.backward(j, dys[j][0])
        if t < n:
            close(host64(y), o.forward(t, xs[t][1]), TOL, "out %d" % t, group="large-step stage out")
            bad.forward(t, xs[t][1])
        if j >= 0:
            close(host64(dx), o.backward(j, dys[j][1]), TOL, "grad_in %d" % j, group="large-step stage grad_in")
            check_tensors(host64(g.last_grad()), o.last_grad, shapes, what="grad step %d" % j,
                          group="large-step stage param grads")
            bad.backward(j, dys[j][1])
            if o.last_staleness > 0:
                told_apart = max(told_apart, rel_l2(bad.last_grad, o.last_grad))
    assert told_apart > 5 * TOL, told_apart


def test_decoder_error_paths():
    import paper_2401_01728_amd as rv
    with pytest.raises(rv.RvError):
        rv.Stage.decoder(1, 100, 1, 256, 64, 1, 0, 1e-3)          # d % 64
    with pytest.raises(rv.RvError):
        rv.Stage.decoder(1, 192, 2, 256, 64, 1, 0, 1e-3)          # head size 96
    with pytest.raises(rv.RvError):
        rv.Stage.decoder(1, 128, 2, 256, 100, 1, 0, 1e-3)         # seq % 64
    g = rv.Stage.decoder(1, 128, 2, 256, 64, 1, 1, 1e-3)
    x = torch.zeros(1, 64, 128, dtype=torch.bfloat16, device="cuda")
    g.forward(0, x); g.forward(1, x)
    with pytest.raises(rv.RvError) as e:
        g.forward(2, x)
    assert e.value.status == rv.api.RV_E_STASH_FULL
    with pytest.raises(rv.RvError) as e:
        g.backward(5, x)
    assert e.value.status == rv.api.RV_E_UNKNOWN_MB
    g.backward(1, x); g.backward(0, x)
    assert g.in_flight == 0


@pytest.mark.parametrize("A,momentum,wd", [(2, 0.0, 0.0), (1, 0.9, 5e-4), (2, 0.9, 5e-4)])
def test_decoder_stage_with_accumulation_in_fused_steps(A, momentum, wd, L=2):
    """Gradient accumulation (section 4.2) and the momentum / weight-decay optimiser (section 4.1)
    through rv_stage_step: block-wise accumulate / update on the side stream, forwards bound to
    a version that only every A-th backward replaces."""
    import paper_2401_01728_amd as rv
    d, H, f, S, mb, tau, eta = 128, 2, 256, 128, 2, 2, 1e-2
    shapes = blocks.decoder_param_shapes(L, d, f)
    w0 = decoder_params_host(31, L, d, f)
    g = rv.Stage.decoder(L, d, H, f, S, mb, tau, eta); g.set_params(dev(w0)); g.set_accumulation(A)
    if momentum or wd:
        g.set_optimizer(momentum, wd)
    o = ostage.Stage("decoder", tau, eta, w0, n_blocks=L, d=d, h=H, f=f, accumulate=A, momentum=momentum,
                     weight_decay=wd)
    n = 7
    for t in range(n + tau):
        j = t - tau
        if t < n:
            x, x64 = bf16_normal(31, 1000 + t, (mb, S, d))
        if j >= 0:
            dy, dy64 = bf16_normal(31, 2000 + j, (mb, S, d), std=1e-3)
        if t < n and j >= 0:
            y, dx = g.step(t, x, j, dy)
        elif t < n:
            y = g.forward(t, x)
        else:
            dx = g.backward(j, dy)
        tag = "decoder accumulate"
        if t < n:
            close(host64(y), o.forward(t, x64), TOL, "out %d" % t, group=tag + " out")
        if j >= 0:
            close(host64(dx), o.backward(j, dy64), TOL, "grad_in %d" % j, group=tag + " grad_in")
            check_tensors(host64(g.last_grad()), o.last_grad, shapes, what="grad step %d" % j, group=tag + " param grads")
    assert o.k == n // A
    assert rel_l2(host64(g.get_params()) - w0, o.w - w0) < TOL


# Six blocks, whose gradients leave four and two at a time, and with them the ranges the update kernels are given; a block's 132480
# parameters are no multiple of the 1024 of a workgroup, which then holds the end of one block and the beginning of the next
@pytest.mark.parametrize("A,momentum,wd", [(2, 0.0, 0.0), (1, 0.9, 5e-4), (2, 0.9, 5e-4)])
def test_updates_of_several_blocks_at_once(A, momentum, wd):
    test_decoder_stage_with_accumulation_in_fused_steps(A, momentum, wd, 6)


@pytest.mark.parametrize("A,momentum", [(2, 0.0), (1, 0.9)])
def test_versions_after_updates_of_several_blocks(A, momentum):
    """As test_versions_hold_the_masters, for blocks that share an update's workgroup."""
    import paper_2401_01728_amd as rv
    st = [rv.Stage.decoder(6, 128, 2, 256, 64, 2, 0, 1e-2) for _ in range(2)]
    st[0].set_accumulation(A)
    st[0].set_optimizer(momentum)
    st[0].set_params(dev(decoder_params_host(83, 6, 128, 256)))
    for t in range(2):
        st[0].forward(t, bf16_normal(84, 2 * t, st[0].in_shape)[0])
        st[0].backward(t, bf16_normal(84, 2 * t + 1, st[0].in_shape, std=1e-2)[0])
    st[1].set_params(st[0].get_params())
    x = bf16_normal(84, 9, st[0].in_shape)[0]
    assert torch.equal(st[0].forward(9, x), st[1].forward(9, x))


@pytest.mark.parametrize("L,d,H,f,S,mb,tau,step", [(1, 128, 2, 2048, 256, 4, 0, False), (2, 256, 2, 1024, 128, 3, 1, True),
                                                   (4, 128, 2, 512, 64, 2, 2, True), (1, 2048, 16, 8192, 64, 1, 0, False)])
def test_grad_in_may_share_the_buffer_of_grad_out(L, d, H, f, S, mb, tau, step):
    """Bit for bit as with two buffers: one block (whose dW2 reads the gradient that its own input gradient replaces) and
    more, the weight-gradient products leaving early (d 2048, ffn 8192) and not, alone and inside a stage step."""
    import paper_2401_01728_amd as rv
    w0 = dev(decoder_params_host(71, L, d, f))
    res = []
    for shared in (False, True):
        g = rv.Stage.decoder(L, d, H, f, S, mb, tau, 1e-2, keep_grad=True)
        g.set_params(w0)
        outs = []
        for t in range(tau + 3):
            x, _ = bf16_normal(71, 10 + t, (mb, S, d))
            dy, _ = bf16_normal(71, 50 + t, (mb, S, d), std=1e-2)
            dx = dy if shared else torch.empty_like(dy)
            y = torch.empty_like(x)
            if t < tau:
                g.forward(t, x, y)
            elif step:
                g.step(t, x, t - tau, dy, y, dx)
            else:
                g.forward(t, x, y); g.backward(t - tau, dy, dx)
            outs += [y] + ([dx, g.last_grad()] if t >= tau else [])
        res.append(outs + [g.get_params()])
    assert all(torch.equal(a, b) for a, b in zip(*res))


def torch_block_grads(w0, L, d, H, f, x, dy):
    """out, grad_in and parameter gradient of the stage in fp32 torch on the GPU, from the bf16-rounded parameters."""
    import torch.nn.functional as F
    p = dev(w0).to(torch.bfloat16).float().requires_grad_(True)
    xin = x.float().requires_grad_(True)
    dh, h, S = d // H, xin, x.shape[1]
    mask = torch.full((S, S), float("-inf"), device="cuda").triu(1)
    for l in range(L):
        q = {n: t.reshape(s) for (n, s), t in zip(blocks.decoder_param_shapes(1, d, f), p.view(L, -1)[l].split(
            [int(np.prod(s)) for _, s in blocks.decoder_param_shapes(1, d, f)]))}
        g1, b1, wqkv, bqkv, wo, bo, g2, b2, w1, c1, w2, c2 = q.values()
        qkv = F.layer_norm(h, (d,), g1, b1) @ wqkv + bqkv
        qh, kh, vh = (t.reshape(-1, S, H, dh).transpose(1, 2).contiguous() for t in qkv.split(d, dim=-1))
        a = torch.softmax(torch.matmul(qh, kh.transpose(2, 3).contiguous()) * dh ** -0.5 + mask, -1)
        h = h + torch.matmul(a, vh).transpose(1, 2).reshape(h.shape) @ wo + bo
        h = h + F.gelu(F.layer_norm(h, (d,), g2, b2) @ w1 + c1) @ w2 + c2
    gx, gp = torch.autograd.grad(h, (xin, p), dy.float())
    return h.detach(), gx, gp


# How the side work of a backward leaves: every block with buffers of its own and four, two or one block to a launch
# (with a remainder, and with the feed-forward products ahead of the rest), or two alternating sets of buffers
# (more than 512 MiB for all blocks).
@pytest.mark.parametrize("L,d,H,f,S,mb", [(6, 128, 2, 256, 64, 2), (5, 320, 5, 1280, 64, 3), (2, 768, 12, 3072, 128, 1),
                                          (2, 2048, 16, 8192, 64, 1), (8, 128, 2, 256, 64, 512)])
def test_side_work_schedules(L, d, H, f, S, mb):
    import paper_2401_01728_amd as rv
    shapes = blocks.decoder_param_shapes(L, d, f)
    w0 = decoder_params_host(70 + L, L, d, f)
    g = rv.Stage.decoder(L, d, H, f, S, mb, 1, 1e-3, keep_grad=True)
    g.set_params(dev(w0))
    (x, _), (dy, _) = bf16_normal(71, 0, (mb, S, d)), bf16_normal(71, 1, (mb, S, d), std=1e-3)
    ref = torch_block_grads(w0, L, d, H, f, x, dy)
    y = g.forward(0, x)
    y1, dx = g.step(1, x, 0, dy)                 # both halves at once, at the same weights
    tag = "side work, %d blocks of d %d on %d tokens" % (L, d, mb * S)
    for what, a, b in (("out", y, ref[0]), ("out of the step", y1, ref[0]), ("grad_in", dx, ref[1])):
        close(host64(a), host64(b), TOL, what, group=tag)
    gg = host64(g.last_grad())
    check_tensors(gg, host64(ref[2]), shapes, what="grad", group=tag)
    check_update(host64(g.get_params()), w0, gg, 1e-3)
    g.backward(1, dy)                            # and the halves apart (fp32 column sums per tile row, whose height may differ)
    close(host64(g.last_grad()), gg, 1e-5, "grad, apart", group=tag + ", apart")


# Whichever kernel published a version - the gradient products' epilogue, the update with its momentum form, an averaging over
# stages of one shape or of two - holds the bf16 rounding of the masters: a fresh stage given those masters answers bit for bit alike
@pytest.mark.parametrize("how", ["fused", "split tiles", "accumulate", "momentum", "average", "average of two shapes"])
def test_versions_hold_the_masters(how):
    import paper_2401_01728_amd as rv
    d, f, mb, S = (2048, 4096, 1, 64) if how == "fused" else (192, 320, 3, 64)
    make = lambda L, d, f: rv.Stage.decoder(L, d, d // 64, f, S, mb, 0, 1e-2)
    st = [make(2, d, f)]
    if how == "accumulate":
        st[0].set_accumulation(2)
    if how == "momentum":
        st[0].set_optimizer(0.9, 5e-4)
    if how == "average":
        st.append(make(2, d, f))
    if how == "average of two shapes":     # of as many parameters each
        st = [make(1, 64, 768), make(1, 128, 192)]
        assert st[0].num_params == st[1].num_params
    for k, s in enumerate(st):
        s.set_params(dev(decoder_params_host(80 + k, 2, d, f)[:s.num_params]) if "two" not in how else
                     torch.randn(s.num_params, device="cuda") * 0.02)
        for t in range(2):
            x, dy = bf16_normal(81, 2 * t, s.in_shape)[0], bf16_normal(81, 2 * t + 1, s.in_shape, std=1e-2)[0]
            s.forward(t, x)
            s.backward(t, dy)
    if len(st) > 1:
        rv.api.cluster_sync(st, 3)
    for s in st:
        fresh = make(1 if "two" in how else 2, s.dims[0], s.dims[2])
        fresh.set_params(s.get_params())
        x = bf16_normal(82, 0, s.in_shape)[0]
        assert torch.equal(s.forward(9, x), fresh.forward(9, x))


# The feed-forward pair of a block's gradient products leaves in a launch of its own where the block is the stage's first one; there
# as elsewhere the block decides how they are summed.  Blocks of which the pair alone would be split: on 2048 tokens, and on few
@pytest.mark.parametrize("d,H,f,S,mb", [(512, 8, 3328, 64, 32), (1536, 24, 5376, 64, 2)])
def test_gradients_do_not_depend_on_the_launch_they_leave_in(d, H, f, S, mb):
    import paper_2401_01728_amd as rv
    block = decoder_params_host(73, 1, d, f)
    passing = block.copy()              # a block whose two branches add nothing: Wo, bo, W2, b2 zero
    shapes = blocks.decoder_param_shapes(1, d, f)
    for name, v in blocks.unflatten(passing, shapes).items():
        if name.split(".")[1] in ("Wo", "bo", "W2", "b2"):
            v[...] = 0.0
    (x, _), (dy, _) = bf16_normal(73, 0, (mb, S, d)), bf16_normal(73, 1, (mb, S, d), std=1e-2)
    res = []
    for w in ([block], [passing, block]):
        g = rv.Stage.decoder(len(w), d, H, f, S, mb, 0, 1e-2, keep_grad=True)
        g.set_params(dev(np.concatenate(w)))
        y = g.forward(0, x)
        g.backward(0, dy)
        gb = blocks.unflatten(g.last_grad()[-block.size:].cpu().numpy(), shapes)
        res.append((y.float().cpu().numpy(), gb["blk0.W1"], gb["blk0.W2"]))
    assert all(np.array_equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("tau", [0, 2])
def test_refused_backward_changes_nothing(tau):
    """An arriving gradient that does not begin at 16 bytes is refused before anything is admitted or enqueued, by the step
    and by the backward alone: microbatches in flight, results and parameters are those of a stage that never saw it."""
    import paper_2401_01728_amd as rv
    L, d, H, f, S, mb = 2, 128, 2, 256, 64, 2
    w0 = dev(decoder_params_host(72, L, d, f))
    res = []
    for disturbed in (False, True):
        g = rv.Stage.decoder(L, d, H, f, S, mb, tau, 1e-2, keep_grad=True)
        g.set_params(w0)
        outs = []
        for t in range(tau + 3):
            x, _ = bf16_normal(72, 10 + t, (mb, S, d))
            dy, _ = bf16_normal(72, 50 + t, (mb, S, d), std=1e-2)
            if t < tau:
                g.forward(t, x)
                continue
            if disturbed:
                odd = torch.empty(dy.numel() + 1, dtype=dy.dtype, device="cuda")[1:].view(dy.shape)
                odd.copy_(dy)
                calls = [lambda: g.step(t, x, t - tau, odd)] + ([lambda: g.backward(t - tau, odd)] if tau else [])
                for call in calls:
                    with pytest.raises(rv.RvError) as e:
                        call()
                    assert e.value.status == rv.api.RV_E_INVAL and g.in_flight == tau
                with pytest.raises(rv.RvError) as e:
                    g.backward(t, dy)              # the refused step's forward is not in flight
                assert e.value.status == rv.api.RV_E_UNKNOWN_MB
            outs += [*g.step(t, x, t - tau, dy), g.last_grad()]
        res.append(outs + [g.get_params()])
    assert all(torch.equal(a, b) for a, b in zip(*res))


# The work buffer that creation falls back to: two alternating sets where every block had one of its own (four, two or one block to
# a launch; the feed-forward products ahead of the rest), all results bit for bit the same
@pytest.mark.parametrize("L,d,H,f,mb,A,momentum", [(6, 128, 2, 256, 2, 1, 0.0), (5, 320, 5, 1280, 3, 1, 0.9), (3, 2048, 16, 8192, 1, 1, 0.0),
                                                   (4, 512, 8, 3328, 4, 2, 0.0)])
def test_smaller_work_buffer(L, d, H, f, mb, A, momentum):
    import paper_2401_01728_amd as rv
    from paper_2401_01728_amd import kernels as k
    w0 = dev(decoder_params_host(85, L, d, f))
    res = []
    for less in (False, True):
        g = rv.Stage.decoder(L, d, H, f, 64, mb, 1, 1e-2, keep_grad=True)
        g.set_accumulation(A)
        if momentum:
            g.set_optimizer(momentum)
        g.set_params(w0)
        outs = []
        for t in range(4):
            if less and t == 2:                        # between two uses of the stage; once only, and only when idle
                with pytest.raises(rv.RvError):
                    k.stage_less_work(g)
                outs += [g.backward(1, dy), g.last_grad()]
                k.stage_less_work(g)
                with pytest.raises(rv.RvError):
                    k.stage_less_work(g)
            elif t == 2:
                outs += [g.backward(1, dy), g.last_grad()]
            x, dy = bf16_normal(85, 2 * t, g.in_shape)[0], bf16_normal(85, 2 * t + 1, g.in_shape, std=1e-2)[0]
            outs += [g.forward(t, x)] if t % 2 == 0 else [*g.step(t, x, t - 1, dy), g.last_grad()]
        res.append(outs + [g.backward(3, dy), g.last_grad(), g.get_params()])
    assert all(torch.equal(a, b) for a, b in zip(*res))


def test_smaller_work_buffer_is_refused():
    import paper_2401_01728_amd as rv
    from paper_2401_01728_amd import kernels as k
    for g in (rv.Stage.decoder(2, 128, 2, 256, 64, 2, 0, 1e-2), rv.Stage.mlp([8, 8], 4, 0, 0.1)):   # two sets are more than two blocks need
        with pytest.raises(rv.RvError) as e:
            k.stage_less_work(g)
        assert e.value.status == rv.api.RV_E_INVAL
