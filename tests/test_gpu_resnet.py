"""GPU parity of the convolution stages: the three 3x3-convolution products against NumPy fp64, then
whole PipeMare training runs of ResNet-shaped CNNs against the fp64 oracle (slots and step counters
bit-exact, master weights within 1e-5 (fp32) / 2e-3 (bf16) max-relative per unit)."""
import numpy as np
import pytest

import workloads as wl
from oracle import pipemare_oracle as po
from oracle import resnet_oracle as ro
from pm_testutil import make_gpu, make_oracle, max_rel_err

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-3}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(2, 8, 8, 16, 16, 1), (2, 8, 8, 16, 32, 2), (1, 12, 12, 32, 32, 1), (2, 8, 8, 64, 64, 1),
                                   (2, 8, 8, 32, 64, 2), (3, 6, 6, 3, 16, 1), (5, 16, 16, 16, 16, 1), (2, 10, 6, 48, 16, 1)])
def test_conv_primitives_against_numpy(torch_cuda, dtype, shape):
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    B, H, W, Cin, Cout, stride = shape
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(sum(shape))
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1

    def dev(a):
        return torch.from_numpy(a.astype(np.float32)).cuda().to(tdt).contiguous()

    def host(t):
        return t.float().cpu().numpy().astype(np.float64)

    x = dev(rng.standard_normal((B, H, W, Cin)))
    params = dev(np.concatenate([(rng.standard_normal((Cout, 9 * Cin)) / np.sqrt(9 * Cin)).ravel(),
                                 1.0 + 0.2 * rng.standard_normal(Cout), 0.2 * rng.standard_normal(Cout)]))
    dz = dev(rng.standard_normal((B, Ho, Wo, Cout)))
    z = torch.empty(B, Ho, Wo, Cout, dtype=tdt, device="cuda")
    y = torch.empty_like(z)
    dx = torch.empty(B, H, W, Cin, dtype=tdt, device="cuda")
    dW = torch.full((Cout, 9 * Cin), 7.0, dtype=torch.float32, device="cuda")       # must be overwritten
    st = torch.cuda.current_stream().cuda_stream
    pm.pm_conv3x3_fwd(st, dtype, B, H, W, Cin, Cout, stride, x.data_ptr(), params.data_ptr(), z.data_ptr(), y.data_ptr())
    pm.pm_conv3x3_bwd_data(st, dtype, B, H, W, Cin, Cout, stride, dz.data_ptr(), params.data_ptr(), dx.data_ptr())
    nscr = pm.pm_conv3x3_bwd_weight_scratch(dtype, B, H, W, Cin, Cout, stride)
    scr = torch.empty(max(nscr, 4), dtype=torch.uint8, device="cuda")
    pm.pm_conv3x3_bwd_weight(st, dtype, B, H, W, Cin, Cout, stride, dz.data_ptr(), x.data_ptr(), dW.data_ptr(),
                             scr.data_ptr(), nscr)
    torch.cuda.synchronize()
    X, P, DZ = host(x), host(params), host(dz)
    Wm, sc, sh = P[:Cout * 9 * Cin].reshape(Cout, 9 * Cin), P[Cout * 9 * Cin:Cout * 9 * Cin + Cout], P[Cout * 9 * Cin + Cout:]
    cols = ro._im2col(X, stride)
    z_ref = cols @ Wm.T
    y_ref = np.maximum(z_ref * sc + sh, 0.0)
    dx_ref = ro._col2im((DZ.reshape(-1, Cout) @ Wm).reshape(cols.shape), X.shape, stride)
    dW_ref = DZ.reshape(-1, Cout).T @ cols.reshape(-1, 9 * Cin)
    out_tol = 2.0 ** -8 if dtype == "bf16" else 3e-6
    for got, ref, tol, name in ((host(z), z_ref, out_tol, "z"), (host(y), y_ref, out_tol * 1.5, "y"),
                                (host(dx), dx_ref, out_tol, "dx"), (host(dW), dW_ref, 3e-6, "dW")):
        err = np.max(np.abs(got - ref.reshape(got.shape))) / np.max(np.abs(ref))
        assert err <= tol, (name, err)


def run_pair(torch, w, steps, tau=None, N=1, gpu_kw=None, check_tables=True, **kw):
    params = wl.init_params(w)
    tf, tb = tau if tau is not None else po.pipeline_delays(w.P, N)
    stream = wl.ImageStream(w)
    o = make_oracle(w, params, tf, tb, N=N, **kw)
    g = make_gpu(w, params, tf, tb, N=N, **dict(kw, **(gpu_kw or {})))
    losses = []
    for k in range(steps):
        mbs = [stream.batch(k * N + j) for j in range(N)]
        lo = o.step(mbs if N > 1 else mbs[0])
        lg = 0.0
        for x, y in mbs:
            lg += g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True) / N
        losses.append((lo, lg))
        if check_tables:
            t_used, fs, bs, ws, lrs = g.step_table()
            assert t_used == k
            for u, L in enumerate(w.layers):
                R = tf[L.stage - 1] + 1
                vf, vb = o.last_versions[u]
                assert (fs[u], bs[u], ws[u]) == (vf % R, vb % R, (k + 1) % R)
                assert lrs[u] == pytest.approx(o.last_lr[u], rel=2e-7)
    return g, o, losses


@pytest.mark.parametrize("batch,image,blocks,N,segment", [(1, 4, 1, 1, 0), (5, 12, 2, 2, 0), (3, 20, 2, 1, 3), (51, 36, 1, 1, 0)])
def test_bf16_backward_chain_edges(torch_cuda, batch, image, blocks, N, segment):
    """The data gradients that carry the affine backward of the unit below, and the grouped weight gradients: maps of
    one pixel, pixel counts that are no multiple of a wave's 32 or a block's 128 (720, 1200, 66096 pixels; one and four
    waves per block), microbatches that accumulate, recomputation that overwrites the outputs between them.
    Odd channels are shifted far above and even ones far below zero and the kernels are small, so that no rounding
    flips a ReLU; what is left is 2^-9 per stored tensor and weight, two of them in each of up to 13 convolutions,
    2^-9 sqrt(26) = 1 % of a part's norm.  The bound is three times that.  (What it leaves open - a few pixels of a large
    map, the mask - the two tests below cover.)"""
    torch = torch_cuda
    w = wl.resnet(blocks, batch, dtype="bf16", image=image)
    params = wl.init_params(w)
    for p, L in zip(params[:-1], w.layers[:-1]):
        nw = L.n_out * 9 * L.n_in
        p[:nw] *= 0.1
        p[nw + L.n_out:] = np.where(np.arange(L.n_out) % 2, 4.0, -4.0)
    kw = dict(opt="sgdm", lr=0.02, beta=0.9, D=0.5, K=6)
    tf, tb = po.pipeline_delays(w.P, N)
    if segment:
        kw.update(tau_recomp=po.recompute_delays(w.P, segment, N, tb), segment=segment)
    o = make_oracle(w, params, tf, tb, N=N, **kw)
    g = make_gpu(w, params, tf, tb, N=N, **kw)
    stream = wl.ImageStream(w)
    mbs = [stream.batch(j) for j in range(N)]
    o.step(mbs if N > 1 else mbs[0])
    for x, y in mbs:
        g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True)
    for u, L in enumerate(w.layers[:-1]):
        nw = L.n_out * 9 * L.n_in
        for name, part in (("W", slice(0, nw)), ("scale", slice(nw, nw + L.n_out)), ("shift", slice(nw + L.n_out, None))):
            # the library keeps the sum over the microbatches and averages in the update
            a, b = g.state(4, u)[part].astype(np.float64) / N, o.last_grads[u][part]
            err = float(np.linalg.norm(a - b) / np.linalg.norm(b))
            assert err <= 3e-2, (u, name, err)
    g.close()


def _conv_affine(m, u, p, f):
    """Pre-activation of unit u without its shift: scale * z (+ shortcut)."""
    ci, co, _ = m.specs[u]
    nw = co * 9 * ci
    a = m._conv_forward(u, p, f.__getitem__)[f"z{u}"] * p[nw:nw + co]
    if u >= 2 and (u - 1) % 2 == 1:
        a = a + ro._shortcut(f[m._in_name(u - 1)], co, m.specs[u - 1][2])
    return a


def _check_gradients(torch, w, params, x, y, bound):
    """All convolutions' gradients of one step against the oracle, per part and by norm."""
    kw = dict(opt="sgdm", lr=0.02, beta=0.9, D=0.5, K=6)
    tf, tb = po.pipeline_delays(w.P, 1)
    o, g = make_oracle(w, params, tf, tb, **kw), make_gpu(w, params, tf, tb, **kw)
    o.step((x, y))
    g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True)
    for u, L in enumerate(w.layers[:-1]):
        nw = L.n_out * 9 * L.n_in
        for name, part in (("W", slice(0, nw)), ("scale", slice(nw, nw + L.n_out)), ("shift", slice(nw + L.n_out, None))):
            a, b = g.state(4, u)[part].astype(np.float64), o.last_grads[u][part]
            err = float(np.linalg.norm(a - b) / np.linalg.norm(b))
            assert err <= bound, (u, name, err)
    g.close()


@pytest.mark.parametrize("batch,image,seed", [(3, 8, 6), (4, 4, 1), (2, 12, 16)])
def test_bf16_backward_chain_where_the_mask_changes_from_pixel_to_pixel(torch_cuda, batch, image, seed):
    """The ReLU mask of the fused data gradient, half of the pixels on in every channel: images of +-1, kernels that mostly
    pass one channel through, and each channel's shift in the middle of the widest gap between its pre-activations, so
    that no rounding moves one across zero (at least 3 % of their spread away, seven convolutions of about 2^-9 each).  A
    mask taken from another pixel changes a gradient by its own size; the bound is that of the test above."""
    rng = np.random.default_rng(seed)
    w = wl.resnet(1, batch, dtype="bf16", image=image)
    params = wl.init_params(w)
    m = ro.ResNetModel(1, 10, image)
    x = (rng.choice([-1, 1], (batch, 3, image, image)) * rng.uniform(1, 1.1, (batch, 3, image, image))).astype(np.float32)
    f = {"img": x.transpose(0, 2, 3, 1).astype(np.float64)}
    for u, (ci, co, _) in enumerate(m.specs):
        nw = co * 9 * ci
        W = 0.03 * rng.standard_normal((co, 9, ci))
        W[np.arange(co), 4, rng.permutation(co) % ci] += rng.choice([-1, 1], co)
        p = params[u]
        p[:nw], p[nw:nw + co], p[nw + co:] = W.ravel(), rng.uniform(0.8, 1.2, co), 0
        a = _conv_affine(m, u, p.astype(np.float64), f).reshape(-1, co)
        for c in range(co):
            v = np.sort(a[:, c])
            lo, hi = len(v) // 5, max(len(v) - len(v) // 5, len(v) // 5 + 2)
            i = lo + int(np.argmax(np.diff(v[lo:hi])))
            p[nw + co + c] = -(v[i] + v[i + 1]) / 2
            assert (v[i + 1] - v[i]) / 2 >= 0.03 * np.std(v)
        f.update(m._conv_forward(u, p.astype(np.float64), f.__getitem__))
    y = rng.integers(0, 10, batch).astype(np.int32)
    _check_gradients(torch_cuda, w, params, x, y, 3e-2)


@pytest.mark.parametrize("batch,image,blocks,segment", [(51, 36, 1, 0), (33, 32, 2, 0), (5, 12, 2, 3), (37, 28, 1, 0)])
def test_bf16_gradients_do_not_depend_on_where_an_image_lies(torch_cuda, batch, image, blocks, segment):
    """A batch and the same batch rotated: every pixel's values are the same bits wherever its image lies, so the gradients of
    all convolutions differ by the order of their fp32 sums, 1e-5 of the norm at most.  What a block's edge loses, doubles
    or takes from elsewhere does not rotate with the images: the last block of 51 x 36 x 36 pixels has 48 of 66096, a
    norm of 2.7 % of the whole."""
    torch = torch_cuda
    w = wl.resnet(blocks, batch, dtype="bf16", image=image)
    params = wl.init_params(w)
    tf, tb = po.pipeline_delays(w.P, 1)
    kw = dict(opt="sgdm", lr=0.02, beta=0.9, D=0.5, K=6)
    if segment:
        kw.update(tau_recomp=po.recompute_delays(w.P, segment, 1, tb), segment=segment)
    x, y = wl.ImageStream(w).batch(0)

    def gradients(by):
        g = make_gpu(w, params, tf, tb, **kw)
        g.step(torch.from_numpy(np.roll(x, by, 0)).cuda(), torch.from_numpy(np.roll(y, by)).cuda(), want_loss=True)
        out = [g.state(4, u).astype(np.float64) for u in range(len(w.layers) - 1)]
        g.close()
        return out

    want = gradients(0)
    for by in (1, batch // 2, batch - 1):
        for u, (a, b) in enumerate(zip(gradients(by), want)):
            nw = w.layers[u].n_out * 9 * w.layers[u].n_in
            for part in (slice(0, nw), slice(nw, None)):
                assert np.linalg.norm(a[part] - b[part]) <= 1e-5 * np.linalg.norm(b[part]), (by, u, part)


@pytest.mark.parametrize("shape", [(1, 1, 1, 16, 16, 1), (3, 7, 5, 32, 16, 2), (9, 31, 33, 16, 32, 1), (2, 200, 180, 16, 16, 1),
                                   (40, 16, 16, 48, 64, 1), (130, 16, 16, 64, 64, 1), (9, 61, 60, 48, 48, 1), (35, 64, 61, 16, 16, 1)])
def test_conv_primitives_at_tile_edges(torch_cuda, shape):
    """Pixel counts around a wave's 32 and a block's 128, several chunks per wave in the weight gradient, four waves
    per block in the forward product (with 64 and 48 channels: both channel tiles in one wave), the most blocks of a
    weight gradient by itself (4270 chunks); references and tolerances as above."""
    test_conv_primitives_against_numpy(torch_cuda, "bf16", shape)


@pytest.mark.parametrize("case", ["pipemare_f32", "pipemare_bf16", "t2_off", "pipedream", "gpipe", "adamw_clip",
                                  "microbatches", "two_blocks_bf16"])
def test_small_resnet_modes(torch_cuda, case):
    dtype = "bf16" if case.endswith("bf16") else "f32"
    nb = 2 if case == "two_blocks_bf16" else 1
    w = wl.resnet(nb, 6, dtype=dtype, image=8)
    kw = dict(opt="sgdm", lr=0.02, beta=0.9, D=0.5, K=6)
    tau, N = None, 1
    if case == "t2_off":
        kw["t2"] = False
    elif case == "pipedream":
        tau = po.pipeline_delays(w.P, 1, "pipedream")
    elif case == "gpipe":
        tau = po.pipeline_delays(w.P, 1, "gpipe")
    elif case == "adamw_clip":
        kw = dict(opt="adamw", lr=1e-3, beta=0.9, beta2=0.98, weight_decay=0.01, clip_norm=0.5, D=0.3, K=6)
    elif case == "microbatches":
        N = 2
    g, o, losses = run_pair(torch_cuda, w, 12, tau=tau, N=N, **kw)
    for lo, lg in losses:
        assert lg == pytest.approx(lo, rel=3e-2 if dtype == "bf16" else 1e-4)
    err, errs = max_rel_err(g.weights(), o.weights())
    print(case, "max-rel", err)
    assert err <= TOL[dtype], errs
    g.close()


@pytest.mark.parametrize("batch", [126, 128, 130, 511, 1025])
def test_channel_sums_of_many_partials(torch_cuda, batch):
    """Scale and shift gradients of the image layer in fp32, whose 32 sums come from 63, 64, 65, 256 and 513 partials: the reduction
    changes its walk from 64 on, in whole and partial turns of 32 slices and eight loads.  A ReLU whose input
    rounds across zero (one in 10^6) moves a sum by one of its up to 65600 terms, 2e-5 of it; the bound is ten of those, a
    partial left out is ten times the bound."""
    torch = torch_cuda
    w = wl.resnet(1, batch, dtype="f32", image=8)
    params = wl.init_params(w)
    kw = dict(opt="sgdm", lr=0.02, beta=0.9, D=0.5, K=6)
    tf, tb = po.pipeline_delays(w.P, 1)
    o, g = make_oracle(w, params, tf, tb, **kw), make_gpu(w, params, tf, tb, **kw)
    x, y = wl.ImageStream(w).batch(0)
    o.step((x, y))
    g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True)
    nw = w.layers[0].n_out * 9 * w.layers[0].n_in
    for part in (slice(nw, nw + 16), slice(nw + 16, None)):
        a, b = g.state(4, 0)[part].astype(np.float64), o.last_grads[0][part]
        err = float(np.max(np.abs(a - b)) / np.max(np.abs(b)))
        assert err <= 2e-4, err
    g.close()
