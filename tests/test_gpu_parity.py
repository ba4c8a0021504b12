"""GPU parity: the HIP path (through the C ABI) against the fp64 CPU oracle on the same seeded inputs.

Tolerances (stated by the task for this method): ring-slot indices and step counters bit-exact;
master weights after N steps within max-relative error 1e-5 (fp32 contexts) / 2e-3 (bf16 compute,
fp32 master), where the error of a unit is ||w_gpu - w_oracle||_inf / ||w_oracle||_inf and the
maximum is taken over units.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import pipemare_oracle as po
from pm_testutil import GivenGrads, make_gpu, make_oracle, max_rel_err

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-3}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch


def run_pair(torch, w, steps, tau=None, check_tables=False, N=1, gpu_kw=None, free_running=False, **kw):
    """Step oracle and GPU side by side; returns (gpu ctx, oracle, losses).  free_running: no
    per-step read-backs, so consecutive steps really overlap on the device."""
    params = wl.init_params(w)
    tf, tb = tau if tau is not None else po.pipeline_delays(w.P, N)
    stream = wl.BatchStream(w)
    o = make_oracle(w, params, tf, tb, N=N, **kw)
    g = make_gpu(w, params, tf, tb, N=N, **dict(kw, **(gpu_kw or {})))
    losses = []
    for k in range(steps):
        mbs = [stream.batch(k * N + j) for j in range(N)]
        lo = o.step(mbs if N > 1 else mbs[0])
        lg = 0.0
        for x, y in mbs:
            xd = torch.from_numpy(x).cuda()
            yd = torch.from_numpy(y).cuda()
            if free_running and k + 1 < steps:
                g.step(xd, yd)
                lg = lo
            else:
                lg += g.step(xd, yd, want_loss=True) / N
        losses.append((lo, lg))
        if check_tables:
            t_used, fs, bs, ws, lrs = g.step_table()
            assert t_used == k
            for u, L in enumerate(w.layers):
                R = tf[L.stage - 1] + 1
                vf, vb = o.last_versions[u]
                assert (fs[u], bs[u], ws[u]) == (vf % R, vb % R, (k + 1) % R)      # bit-exact integers
                assert lrs[u] == pytest.approx(o.last_lr[u], rel=2e-7)
    return g, o, losses


# ------------------------------------------------------------------------------- the update pass alone
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opt", ["sgdm", "adamw"])
def test_fused_update_alone_matches_oracle(torch_cuda, dtype, opt):
    """T1 + optimizer + delta + write-back on given gradients, several tiles and ragged unit sizes."""
    layers = (wl.Layer("linear", 40, 70, "relu", 1), wl.Layer("linear", 70, 33, "relu", 2),
              wl.Layer("linear", 33, 129, "relu", 2), wl.Layer("linear", 129, 5, "none", 3))
    w = wl.Workload("upd", layers, 3, 1, "mse", dtype, 4, 5)
    params = wl.init_params(w, 11)
    tf, tb = [5, 2, 1], [0, 1, 1]                      # corrected, corrected with tau_bkwd>0, uncorrected
    kw = dict(opt=opt, lr=0.02 if opt == "sgdm" else 3e-3, beta=0.9, weight_decay=0.01, D=0.3, K=6)
    o = make_oracle(w, params, tf, tb, model=GivenGrads(), keep_history=True, **kw)
    g = make_gpu(w, params, tf, tb, **kw)
    rng = np.random.default_rng(0)
    for k in range(9):
        grads = [rng.standard_normal(p.size).astype(np.float32) * 0.1 for p in params]
        o.step(tuple(grads))
        g.set_grads(grads)
        g.apply_update()
        t_used, fs, bs, ws, lrs = g.step_table()
        assert t_used == k
    err, _ = max_rel_err(g.weights(), o.weights())
    assert err < 2e-6                                                   # fp32 master in both modes
    for u in range(len(layers)):
        d = g.state(1, u)
        assert np.max(np.abs(d - o.delta[u])) <= 2e-6 * np.max(np.abs(o.delta[u])) + 1e-9 + 1e-7 * np.max(np.abs(o.weights(u)))
        # corrected backward weights for the next step: w_{t+1-tau_b} - (tau_f - tau_b) * delta_{t+1}
        st = layers[u].stage - 1
        if tf[st] > tb[st]:
            base = o.hist[u][max(o.t - tb[st], 0)]
            want = base - (tf[st] - tb[st]) * o.delta[u]
            got = g.state(3, u)
            tol = 1e-5 if dtype == "f32" else 2.0 ** -7   # two bf16 roundings (stored version, result)
            assert np.max(np.abs(got - want)) <= tol * np.max(np.abs(want))
    g.close()


def test_update_chunk_boundaries_large_unit(torch_cuda):
    """One unit spanning many 2048-element chunks plus a ragged tail; every element checked."""
    layers = (wl.Layer("linear", 1000, 77, "none", 1),)
    w = wl.Workload("big", layers, 1, 1, "mse", "bf16", 4, 77)
    params = wl.init_params(w, 3)
    o = make_oracle(w, params, [3], [0], model=GivenGrads(), lr=0.05, D=0.5, K=0)
    g = make_gpu(w, params, [3], [0], lr=0.05, D=0.5, K=0)
    rng = np.random.default_rng(1)
    for k in range(5):
        grads = [rng.standard_normal(params[0].size).astype(np.float32)]
        o.step(tuple(grads))
        g.set_grads(grads)
        g.apply_update()
    assert np.max(np.abs(g.weights(0) - o.weights(0))) < 1e-5
    g.close()


@pytest.mark.parametrize("opt", ["sgdm", "adamw"])
def test_update_large_streams_variant_every_element(torch_cuda, opt):
    """Parameter streams beyond 1 GiB per pass take the update kernel's other access variant (non-temporal,
    one group of four elements per thread, two blocks per chunk), otherwise reached only by the 12-layer
    Transformer: 50 M parameters in three units (corrected with tau_bkwd = 0, corrected from a stored ring
    version, uncorrected), 3 steps on given gradients, EVERY element of weights, delta and corrected weights
    against the oracle."""
    layers = (wl.Layer("linear", 4096, 4096, "relu", 1), wl.Layer("linear", 4096, 4097, "relu", 2),
              wl.Layer("linear", 4097, 4096, "none", 3))
    w = wl.Workload("upd_big", layers, 3, 1, "mse", "bf16", 4, 4096)
    rng = np.random.default_rng(5)
    params = [rng.uniform(-0.05, 0.05, size=wl.n_params(L)).astype(np.float32) for L in layers]
    assert sum(p.size for p in params) * 32 > 1 << 30
    tf, tb = [4, 2, 1], [0, 1, 1]
    kw = dict(opt=opt, lr=0.02 if opt == "sgdm" else 3e-3, beta=0.9, weight_decay=0.01, D=0.3, K=4)
    o = make_oracle(w, params, tf, tb, model=GivenGrads(), keep_history=True, **kw)
    g = make_gpu(w, params, tf, tb, **kw)
    for k in range(3):
        grads = [(rng.standard_normal(p.size, dtype=np.float32) * 0.1) for p in params]
        o.step(tuple(grads))
        g.set_grads(grads)
        g.apply_update()
    err, errs = max_rel_err(g.weights(), o.weights())
    assert err < 2e-6, errs
    for u in range(len(layers)):
        d = g.state(1, u)
        assert np.max(np.abs(d - o.delta[u])) <= 2e-6 * np.max(np.abs(o.delta[u])) + 1e-7 * np.max(np.abs(o.weights(u)))
        st = layers[u].stage - 1
        if tf[st] > tb[st]:
            want = o.hist[u][max(o.t - tb[st], 0)] - (tf[st] - tb[st]) * o.delta[u]
            assert np.max(np.abs(g.state(3, u) - want)) <= 2.0 ** -7 * np.max(np.abs(want))
    # the newest ring slot is what the next forward of a tau = 1 stage reads: compare through the step table
    t_used, fs, bs, ws, lrs = g.step_table()
    assert t_used == 2 and list(ws) == [3 % 5, 3 % 3, 3 % 2]
    g.close()


# ------------------------------------------------------------------------------- chained launches
CHAIN_CASES = {
    # name: (widths, acts, stages, loss, M, steps, extra)
    "w64_m32": ([64, 64, 64, 64, 64, 10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 32, 16, {}),
    "w128_m128_relu": ([128] * 7 + [10], ["relu"] * 6 + ["none"], [1, 2, 3, 4, 5, 6, 6], "xent", 128, 16, {}),
    "mixed_widths_m64": ([64, 128, 64, 256, 192, 64, 5], ["gelu", "relu", "gelu", "none", "gelu", "none"], [1, 2, 3, 4, 5, 6], "xent", 64, 16, {}),
    "mse_head_in_the_chain_m96": ([128, 64, 128, 64], ["gelu", "gelu", "none"], [1, 2, 3], "mse", 96, 16, {}),
    "k2048_two_slices_per_wave": ([64, 2048, 2048, 64, 10], ["gelu", "gelu", "gelu", "none"], [1, 2, 3, 4], "xent", 128, 8, {}),
    "n4096_more_tiles_than_blocks": ([64, 4096, 64, 64, 10], ["gelu", "gelu", "gelu", "none"], [1, 2, 3, 4], "xent", 128, 8, {}),
    "graph": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 16, dict(_gpu=dict(use_graph=True))),
    "microbatches": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 10, dict(_N=2)),
    "pipedream": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 14, dict(_method="pipedream")),
    "t2_off": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 14, dict(t2=False)),
    # (Adam turns sub-noise-floor gradient entries into full steps: a step size at which 14 of them stay inside the band)
    "adamw": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 14, dict(opt="adamw", lr=2e-5)),
    "stochastic": ([128] * 5 + [10], ["gelu"] * 4 + ["none"], [1, 2, 3, 4, 4], "xent", 64, 14, dict(stochastic=dict(tau_max=6, seed=3))),
}


@pytest.mark.parametrize("name", list(CHAIN_CASES))
def test_chained_launches_match_oracle_and_the_launch_per_product_path(torch_cuda, name):
    """bf16 chains run with the persistent forward / data-gradient launches (an option): weights against the
    oracle (2e-3), and activations-driven state against the same run with one launch per product (both
    round to bf16 at the same places; only the order of the fp32 partial sums differs)."""
    widths, acts, stages, loss, M, steps, extra = CHAIN_CASES[name]
    extra = dict(extra)
    gpu_kw = extra.pop("_gpu", None)
    N = extra.pop("_N", 1)
    method = extra.pop("_method", "pipemare")
    layers = tuple(wl.Layer("linear", widths[j], widths[j + 1], acts[j], stages[j]) for j in range(len(acts)))
    w = wl.Workload("chain_" + name, layers, max(stages), N, loss, "bf16", M, widths[-1], init="he")
    tau = po.pipeline_delays(w.P, N, method)
    kw = dict(lr=0.002, beta=0.9, D=0.5, K=6)
    kw.update(extra)
    side = torch_cuda.cuda.Stream()
    with torch_cuda.cuda.stream(side):
        g, o, losses = run_pair(torch_cuda, w, steps, tau=tau, N=N, gpu_kw=dict(stream=side, chained_launches=True, **(gpu_kw or {})),
                                check_tables=extra.get("stochastic") is None, **kw)
        # the chained launches did run: forward every unit but the head (it writes fp32 logits for the loss); backward
        # the data gradient of every unit, the head's included only where its width allows
        L = len(layers)
        assert g.chained_units() == (L - 1, L - 1 if widths[-1] % 64 == 0 else L - 2), g.chained_units()
        for lo, lg in losses:
            assert lg == pytest.approx(lo, rel=3e-2, abs=1e-5)
        err, errs = max_rel_err(g.weights(), o.weights())
        print(name, "max-rel vs oracle", err)
        assert err <= 2e-3, errs
        # the same run with one launch per product
        params = wl.init_params(w)
        h = make_gpu(w, params, tau[0], tau[1], N=N, stream=side, **dict(kw, **(gpu_kw or {})))
        assert h.chained_units() == (0, 0)
        stream = wl.BatchStream(w)
        for k in range(steps):
            for j in range(N):
                x, y = stream.batch(k * N + j)
                h.step(torch_cuda.from_numpy(x).cuda(), torch_cuda.from_numpy(y).cuda())
        d, ds = max_rel_err(g.weights(), [v.astype(np.float64) for v in h.weights()])
        print(name, "max-rel vs launch-per-product", d)
        assert d <= 1e-3, ds
        h.close()
        g.close()


def test_chained_launches_are_left_out_where_the_shapes_do_not_qualify(torch_cuda):
    """The option asks, the shapes decide: rows not a multiple of 32, fp32, a width that is no multiple of 64."""
    def units(widths, M, dtype):
        layers = tuple(wl.Layer("linear", widths[j], widths[j + 1], "gelu" if j + 2 < len(widths) else "none", j + 1)
                       for j in range(len(widths) - 1))
        w = wl.Workload("chain_probe", layers, len(layers), 1, "xent", dtype, M, widths[-1], init="he")
        tau = po.pipeline_delays(w.P, 1, "pipemare")
        g = make_gpu(w, wl.init_params(w), tau[0], tau[1], chained_launches=True)
        u = g.chained_units()
        g.close()
        return u
    assert units([64, 64, 64, 64, 10], 32, "bf16") == (3, 2)
    assert units([64, 64, 64, 64, 10], 48, "bf16") == (0, 0)
    assert units([64, 64, 64, 64, 10], 32, "f32") == (0, 0)
    assert units([64, 64, 64, 64, 10], 160, "bf16") == (0, 0)
    fwd, bwd = units([64, 64, 96, 64, 64, 10], 32, "bf16")      # unit 2 reads 96 columns: the forward chain stops before it
    assert fwd == 2 and bwd == 0, (fwd, bwd)


# ------------------------------------------------------------------------------- linear primitives
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(128, 1024, 1024), (48, 72, 200), (300, 264, 136), (128, 1024, 16), (16, 64, 64),
                                   (2048, 512, 2048), (4096, 1024, 4096), (4000, 1000, 4040), (8192, 512, 1024),
                                   (8192, 1024, 1024), (8192, 4096, 1024)])     # the last two: 256 x 128 / 128 x 256 blocks
def test_linear_primitives_against_numpy(torch_cuda, dtype, shape):
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    M, n_in, n_out = shape
    rng = np.random.default_rng(M + n_in)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def dev(a):
        return torch.from_numpy(a.astype(np.float32)).cuda().to(tdt).contiguous()

    def host(t):
        return t.float().cpu().numpy().astype(np.float64)

    x, W = dev(rng.standard_normal((M, n_in))), dev(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in))
    b, dz = dev(rng.standard_normal(n_out) * 0.1), dev(rng.standard_normal((M, n_out)))
    zprev = dev(rng.standard_normal((M, n_in)))
    z = torch.empty(M, n_out, dtype=tdt, device="cuda")
    a = torch.empty_like(z)
    dzp = torch.empty(M, n_in, dtype=tdt, device="cuda")
    dW = torch.empty(n_out, n_in, dtype=torch.float32, device="cuda")
    db = torch.empty(n_out, dtype=torch.float32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    pm.pm_linear_fwd(st, dtype, M, n_in, n_out, x.data_ptr(), W.data_ptr(), b.data_ptr(), "gelu", z.data_ptr(), a.data_ptr())
    pm.pm_linear_bwd_data(st, dtype, M, n_in, n_out, dz.data_ptr(), W.data_ptr(), zprev.data_ptr(), "gelu", dzp.data_ptr())
    pm.pm_linear_bwd_weight(st, dtype, M, n_in, n_out, dz.data_ptr(), x.data_ptr(), dW.data_ptr(), db.data_ptr())
    torch.cuda.synchronize()
    X, Wh, B, DZ, ZP = host(x), host(W), host(b), host(dz), host(zprev)
    z_ref = X @ Wh.T + B
    a_ref = po._act(z_ref, "gelu")
    dzp_ref = (DZ @ Wh) * po._act_grad(ZP, "gelu")
    dW_ref, db_ref = DZ.T @ X, DZ.sum(0)
    # Relative to the largest output: one output rounding for bf16 outputs (2^-8), and for every product the
    # fp32 accumulation over its K terms - rounding errors of 2^-24 per addition that add up like a random walk
    # over terms of similar size: 1.5 sqrt(K) 2^-24 (measured 0.7 of that at K = 8192).  A dropped or doubled
    # term changes an output by about 1 / sqrt(K) of its size, a thousand times more.
    def acc_tol(K):
        return 1.5 * np.sqrt(K) * 2.0 ** -24
    out_tol = 2.0 ** -8 if dtype == "bf16" else 0.0
    for got, ref, tol in ((host(z), z_ref, out_tol + acc_tol(n_in)), (host(a), a_ref, out_tol + acc_tol(n_in)),
                          (host(dzp), dzp_ref, out_tol + acc_tol(n_out)), (host(dW), dW_ref, acc_tol(M)),
                          (host(db), db_ref, acc_tol(M))):
        scale = np.max(np.abs(ref))
        assert np.max(np.abs(got - ref)) <= tol * scale
    acc_tol = acc_tol(M)
    # accumulate flag adds on top
    pm.pm_linear_bwd_weight(st, dtype, M, n_in, n_out, dz.data_ptr(), x.data_ptr(), dW.data_ptr(), db.data_ptr(), True)
    torch.cuda.synchronize()
    assert np.max(np.abs(host(dW) - 2 * dW_ref)) <= 2 * acc_tol * np.max(np.abs(dW_ref)) * 2
    assert np.max(np.abs(host(db) - 2 * db_ref)) <= 2 * acc_tol * np.max(np.abs(db_ref)) * 2


# ------------------------------------------------------------------------------- whole step, small cases
def test_config1_fp32_mlp_50_steps(torch_cuda):
    """The smallest configuration of the task (config 1): 4-stage fp32 MLP, tau_fwd = (7,5,3,1), tau_bkwd = 0, momentum 0.9, lr 0.01, D 0.9."""
    w = wl.config(1)
    o_ = w.opt
    g, o, losses = run_pair(torch_cuda, w, w.steps, check_tables=True, lr=o_["lr"], beta=o_["beta"], D=o_["D"], K=o_["K"])
    assert po.pipeline_delays(w.P, 1)[0] == [7, 5, 3, 1]
    err, errs = max_rel_err(g.weights(), o.weights())
    print("config1 max-rel", err, errs)
    assert err <= TOL["f32"]
    for lo, lg in losses:
        assert lg == pytest.approx(lo, rel=1e-4, abs=1e-6)
    assert g.stats()["t"] == w.steps
    g.close()


@pytest.mark.parametrize("case", ["pipemare", "t2_off", "pipedream", "gpipe", "adamw_clip", "microbatches", "graph",
                                  "gamma_override", "ragged_bf16", "sync_warmup", "sync_warmup_bf16",
                                  "overlap", "overlap_free", "overlap_gpipe", "overlap_warmup", "overlap_clip_f32"])
def test_modes_small(torch_cuda, case):
    """Every mode of the step on a small MLP (several stages share units; odd widths hit the
    non-MFMA kernel, multiples of 8 the MFMA kernel)."""
    dtype = "bf16" if case in ("ragged_bf16", "graph", "pipemare", "sync_warmup_bf16", "overlap", "overlap_free",
                               "overlap_gpipe", "overlap_warmup") else "f32"
    width = 72 if case != "ragged_bf16" else 50
    w = wl.small_mlp(width, 5, 6, "gelu", "xent", dtype, 24, layers_per_stage=2)
    # bf16 contexts: at the fp32 cases' step (0.02) the 10-class head moves by 55 % of its largest entry in
    # these 14 steps, and bf16's relative error on that movement (activations, ring and corrected weights are
    # stored in bf16) comes to 3.8e-3 of max|w| (measured); at 0.005 the head moves 14 % and the error is 1.1e-3
    kw = dict(lr=0.02 if dtype == "f32" else 0.005, beta=0.9, D=0.5, K=8)
    tau, N, gpu_kw = None, 1, {}
    if case == "t2_off":
        kw["t2"] = False
    elif case == "pipedream":
        tau = po.pipeline_delays(w.P, 1, "pipedream")
    elif case == "gpipe":
        tau = po.pipeline_delays(w.P, 1, "gpipe")
    elif case == "adamw_clip":
        kw = dict(opt="adamw", lr=2e-3, beta=0.9, beta2=0.98, weight_decay=0.01, clip_norm=0.5, D=0.3, K=8,
                  sched=dict(kind="warmup_invsqrt", base=2e-3, init=1e-5, warmup=6))
    elif case == "microbatches":
        N = 2
    elif case == "graph":
        gpu_kw = dict(use_graph=True)
    elif case == "gamma_override":
        kw["gamma_override"] = [0.9, 0.8, 0.7]
    elif case.startswith("sync_warmup"):
        kw["sync_warmup"] = 5            # PipeMareW: 5 synchronous steps, then 9 asynchronous ones
    free = False
    if case.startswith("overlap"):
        # update of step t on the library's second stream, concurrent with the forward of step t+1
        gpu_kw = dict(overlap_update=True)
        free = case != "overlap"
        if case == "overlap_gpipe":
            tau = po.pipeline_delays(w.P, 1, "gpipe")       # zero delays: the forward must wait for the update
        elif case == "overlap_warmup":
            kw["sync_warmup"] = 5
        elif case == "overlap_clip_f32":
            kw = dict(opt="adamw", lr=2e-3, beta=0.9, beta2=0.98, weight_decay=0.01, clip_norm=0.5, D=0.3, K=8)
    steps = 14
    if case == "graph":
        # a captured graph is bound to the batch buffers: feed every step through the same two tensors
        torch = torch_cuda
        params = wl.init_params(w)
        tf, tb = po.pipeline_delays(w.P, 1)
        stream = wl.BatchStream(w)
        o = make_oracle(w, params, tf, tb, **kw)
        side = torch.cuda.Stream()                           # capture needs a non-default stream
        with torch.cuda.stream(side):
            g = make_gpu(w, params, tf, tb, use_graph=True, stream=side, **kw)
            x0, y0 = stream.batch(0)
            xd, yd = torch.from_numpy(x0).cuda(), torch.from_numpy(y0).cuda()
            for k in range(steps):
                x, y = stream.batch(k)
                xd.copy_(torch.from_numpy(x))
                yd.copy_(torch.from_numpy(y))
                o.step((x, y))
                lg = g.step(xd, yd, want_loss=(k % 3 == 0))     # eager work and syncs between replays
                t_used, fs, bs, ws, lrs = g.step_table()
                assert t_used == k
                for u, L in enumerate(w.layers):
                    R = tf[L.stage - 1] + 1
                    assert (fs[u], ws[u]) == (o.last_versions[u][0] % R, (k + 1) % R)
    else:
        g, o, losses = run_pair(torch_cuda, w, steps, tau=tau, check_tables=not free, N=N, gpu_kw=gpu_kw,
                                free_running=free, **kw)
        for lo, lg in losses:
            assert lg == pytest.approx(lo, rel=3e-2 if dtype == "bf16" else 1e-4)
    err, errs = max_rel_err(g.weights(), o.weights())
    print(case, "max-rel", err)
    assert err <= TOL[dtype]
    g.close()


def test_t2_changes_the_result_and_first_unit_is_insensitive(torch_cuda):
    """Guards against a backward that silently reads the forward weights: with T2 on/off the
    trajectories must differ (units >= 2 see the corrected weights), each matching its oracle."""
    w = wl.small_mlp(64, 3, 4, "relu", "mse", "f32", 16)
    ga, oa, _ = run_pair(torch_cuda, w, 12, lr=0.05, beta=0.9, D=0.5, K=0, t2=True)
    gb, ob, _ = run_pair(torch_cuda, w, 12, lr=0.05, beta=0.9, D=0.5, K=0, t2=False)
    assert max_rel_err(ga.weights(), oa.weights())[0] <= TOL["f32"]
    assert max_rel_err(gb.weights(), ob.weights())[0] <= TOL["f32"]
    diff = max(np.max(np.abs(a - b)) for a, b in zip(ga.weights(), gb.weights()))
    assert diff > 1e-4
    ga.close()
    gb.close()


def test_divergence_is_reported_not_fatal(torch_cuda):
    """A step size far above the stability threshold (Sec. 3.1) must end in PM_EDIVERGED, not a crash."""
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    w = wl.small_mlp(32, 2, 1, "none", "mse", "f32", 8)
    params = wl.init_params(w)
    tf, tb = po.pipeline_delays(w.P, 1)
    g = make_gpu(w, params, tf, tb, lr=1e4, beta=0.9, D=0.5, K=0)
    stream = wl.BatchStream(w)
    with pytest.raises(pm.PmError) as e:
        for k in range(200):
            x, y = stream.batch(k)
            g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True)
    assert e.value.name == "PM_EDIVERGED"
    g.close()


@pytest.mark.parametrize("M,n_in,n_out", [(1, 1, 1), (3, 5, 7), (16, 64, 1), (17, 16, 33), (100, 784, 512), (65, 129, 30), (33, 48, 34),
                                          (511, 260, 515), (256, 31, 512), (600, 512, 2000), (2048, 20, 1030)])
def test_fp32_linear_primitives_every_tile_choice(torch_cuda, M, n_in, n_out):
    """fp32 products on blocks of 16, 32 and 64 outputs, with vector and with single accesses, contractions of no, one
    and several whole 16-deep pieces and a remainder.  Bound per element: each of the K products and K additions rounds
    by at most 2^-24, so |error| <= 2 K 2^-24 sum |a b| (and the activation adds one rounding of its own)."""
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    rng = np.random.default_rng(M * 7 + n_in * 3 + n_out)
    x, W, dz, zp = (rng.standard_normal(s).astype(np.float32) for s in ((M, n_in), (n_out, n_in), (M, n_out), (M, n_in)))
    b = rng.standard_normal(n_out).astype(np.float32)
    g0, b0 = rng.standard_normal((n_out, n_in)).astype(np.float32), rng.standard_normal(n_out).astype(np.float32)
    x_d, W_d, dz_d, zp_d, b_d = (torch.from_numpy(v).cuda() for v in (x, W, dz, zp, b))
    st = torch.cuda.current_stream().cuda_stream
    x64, W64, dz64 = x.astype(np.float64), W.astype(np.float64), dz.astype(np.float64)

    def check(got, want, terms, K):
        got = got.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= (2 * K + 4) * 2.0 ** -24 * terms), np.max(np.abs(got - want) / terms)

    z, a = torch.full((M, n_out), np.nan, device="cuda"), torch.full((M, n_out), np.nan, device="cuda")
    pm.pm_linear_fwd(st, "f32", M, n_in, n_out, x_d.data_ptr(), W_d.data_ptr(), b_d.data_ptr(), "relu", z.data_ptr(), a.data_ptr())
    zw, terms = x64 @ W64.T + b, np.abs(x64) @ np.abs(W64).T + np.abs(b)
    check(z, zw, terms, n_in)
    check(a, np.maximum(zw, 0), terms, n_in)
    dp = torch.full((M, n_in), np.nan, device="cuda")
    pm.pm_linear_bwd_data(st, "f32", M, n_in, n_out, dz_d.data_ptr(), W_d.data_ptr(), zp_d.data_ptr(), "relu", dp.data_ptr())
    check(dp, (dz64 @ W64) * (zp > 0), np.abs(dz64) @ np.abs(W64), n_out)
    for acc in (0, 1):
        dW, db = torch.from_numpy(g0).cuda(), torch.from_numpy(b0).cuda()
        pm.pm_linear_bwd_weight(st, "f32", M, n_in, n_out, dz_d.data_ptr(), x_d.data_ptr(), dW.data_ptr(), db.data_ptr(), acc)
        check(dW, dz64.T @ x64 + acc * g0, np.abs(dz64).T @ np.abs(x64) + acc * np.abs(g0), M)
        check(db, dz64.sum(0) + acc * b0, np.abs(dz64).sum(0) + acc * np.abs(b0), M)


def _fma_chain(a, b, start=None):
    """C[i, j] = chain of fp32 fused multiply-adds over k of a[i, k] b[j, k], one rounding each (the 64-bit significand of
    the extended type holds a product exactly, so rounding the sum to fp32 is a fused multiply-add but for a double
    rounding of one in 2^40)."""
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision on this machine")
    c = np.zeros((a.shape[0], b.shape[0]), dtype=np.float32) if start is None else start
    for k in range(a.shape[1]):
        c = (np.multiply.outer(a[:, k].astype(np.longdouble), b[:, k].astype(np.longdouble)) + c).astype(np.float32)
    return c


@pytest.mark.parametrize("M,n_in,n_out", [(1, 1, 1), (3, 5, 7), (16, 64, 16), (17, 16, 33), (65, 129, 30), (33, 48, 34), (100, 203, 96),
                                          (260, 31, 512), (300, 64, 1040)])
def test_fp32_products_sum_in_index_order(torch_cuda, M, n_in, n_out):
    """Every fp32 product is one chain of fused multiply-adds in the order of the contraction index, for all tile
    choices: bit for bit.  (A ReLU network turns one rounding next to zero into another gradient, so the order of the
    sums is part of the result.)  The bias gradient: rows m, m + 4, ... in four chains, added in order."""
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    rng = np.random.default_rng(M * 5 + n_in * 3 + n_out)
    x, W, dz = (rng.standard_normal(s).astype(np.float32) for s in ((M, n_in), (n_out, n_in), (M, n_out)))
    b = rng.standard_normal(n_out).astype(np.float32)
    x_d, W_d, dz_d, b_d = (torch.from_numpy(v).cuda() for v in (x, W, dz, b))
    st = torch.cuda.current_stream().cuda_stream
    z = torch.full((M, n_out), np.nan, device="cuda")
    pm.pm_linear_fwd(st, "f32", M, n_in, n_out, x_d.data_ptr(), W_d.data_ptr(), b_d.data_ptr(), "none", z.data_ptr(), 0)
    assert np.array_equal(z.cpu().numpy(), _fma_chain(x, W) + b)
    dp = torch.full((M, n_in), np.nan, device="cuda")
    pm.pm_linear_bwd_data(st, "f32", M, n_in, n_out, dz_d.data_ptr(), W_d.data_ptr(), x_d.data_ptr(), "none", dp.data_ptr())
    assert np.array_equal(dp.cpu().numpy(), _fma_chain(dz, np.ascontiguousarray(W.T)))
    dW, db = torch.zeros((n_out, n_in), device="cuda"), torch.zeros(n_out, device="cuda")
    pm.pm_linear_bwd_weight(st, "f32", M, n_in, n_out, dz_d.data_ptr(), x_d.data_ptr(), dW.data_ptr(), db.data_ptr(), 0)
    assert np.array_equal(dW.cpu().numpy(), _fma_chain(np.ascontiguousarray(dz.T), np.ascontiguousarray(x.T)))
    chains = [np.zeros(n_out, dtype=np.float32) for _ in range(4)]
    for m in range(M):
        chains[m % 4] = chains[m % 4] + dz[m]
    assert np.array_equal(db.cpu().numpy(), ((chains[0] + chains[1]) + chains[2]) + chains[3])


@pytest.mark.parametrize("rows,widths,N", [(129, (64, 64), 1), (200, (72, 136, 200, 40), 2), (255, (24, 520, 8), 1),
                                           (200, (1000,) * 9, 1), (1000, (1000,) * 9, 1), (131, (1024,) * 9, 2)])
def test_bf16_chain_weight_gradients_of_many_rows(torch_cuda, rows, widths, N):
    """More than 128 rows: the weight and bias gradients of all units in one pipelined launch, on tiles of 64 and (eight
    units of 1000 or 1024) of 128, ragged in every extent.  Weights with at most one entry of +-1 per row and
    column, integer inputs and no activation keep every activation and data gradient exact (a data gradient is a rounded
    value of the loss passed on), so what is left are the fp32 sums: |error| <= 2 K 2^-24 sum |dz a|."""
    from workloads import Layer, Workload
    torch = torch_cuda
    rng = np.random.default_rng(rows + len(widths))
    L = len(widths) - 1
    w = Workload(name="chain", layers=tuple(Layer("linear", widths[l], widths[l + 1], "none", l + 1) for l in range(L)), P=L, N=N,
                 loss="mse", dtype="bf16", microbatch=rows, n_classes=widths[-1])
    Ws, params = [], []
    for a, b in zip(widths, widths[1:]):
        n = min(a, b)
        W = np.zeros((b, a), dtype=np.float32)
        W[rng.permutation(b)[:n], rng.permutation(a)[:n]] = rng.choice([-1, 1], n)
        Ws.append(W)
        params.append(np.concatenate([W.ravel(), np.zeros(b, dtype=np.float32)]))
    g = make_gpu(w, params, *po.pipeline_delays(L, N), N=N, opt="sgdm", lr=0.0, K=6)
    want = [(0.0, 0.0, 0.0, 0.0)] * L
    for _ in range(N):
        x = rng.integers(-4, 5, (rows, widths[0])).astype(np.float32)
        y = rng.integers(-4, 5, (rows, widths[-1])).astype(np.float32)
        g.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), want_loss=True)
        acts = [x]
        for W in Ws:
            acts.append(acts[-1] @ W.T)
        inv = np.float32(1) / (np.float32(rows) * np.float32(widths[-1]))
        dz = torch.from_numpy(np.float32(2) * (acts[-1] - y) * inv).bfloat16().float().numpy()
        for l in range(L - 1, -1, -1):
            dz64, a64 = dz.astype(np.float64), acts[l].astype(np.float64)
            want[l] = tuple(p + q for p, q in zip(want[l], (dz64.T @ a64, np.abs(dz64).T @ np.abs(a64), dz64.sum(0), np.abs(dz64).sum(0))))
            dz = dz @ Ws[l]
    tol = 2 * N * rows * 2.0 ** -24
    for l in range(L):
        got = g.state(4, l).astype(np.float64)
        dW, W_terms, db, b_terms = want[l]
        assert np.all(np.abs(got[:dW.size].reshape(dW.shape) - dW) <= tol * W_terms), l
        assert np.all(np.abs(got[dW.size:] - db) <= tol * b_terms), l
    g.close()


@pytest.mark.parametrize("M,n_in,n_out", [(1, 24, 8), (33, 40, 1032), (31, 1024, 72), (130, 1032, 200), (300, 1288, 200), (129, 72, 1000),
                                          (700, 776, 776), (1500, 328, 1288), (2000, 200, 520), (1300, 1000, 2056), (3000, 1032, 1032),
                                          (4097, 264, 2056), (8200, 264, 4104), (8192, 256, 4096)])
def test_bf16_products_at_the_edges_of_every_block_shape(torch_cuda, M, n_in, n_out):
    """Forward and data gradient for every block shape of the dispatch, with rows, columns and contractions that end inside a
    tile and inside a slab.  A row of NaN stays in its row, whatever lies around the operands (NaN here) stays out, and
    nothing behind the outputs is written.  Bound per output: one bf16 rounding, and K fp32 additions of terms whose absolute
    values sum to S: (K + 4) 2^-24 S."""
    import paper_1910_05124_amd as pm
    torch = torch_cuda
    gen = torch.Generator(device="cuda").manual_seed(M * 7 + n_in * 3 + n_out)

    def guarded(rows, cols, fill=None):
        buf = torch.full((rows * cols + 4096,), float("nan"), device="cuda", dtype=torch.bfloat16)
        t = buf[2048:2048 + rows * cols].view(rows, cols)
        if fill is None:
            t.copy_(torch.randn(rows, cols, device="cuda", generator=gen))
        return buf, t

    _, x = guarded(M, n_in)
    _, W = guarded(n_out, n_in)
    _, b = guarded(1, n_out)
    _, dz = guarded(M, n_out)
    _, zp = guarded(M, n_in)
    bad = M // 2 if M > 1 else None
    if bad is not None:
        x[bad] = float("nan")
        dz[bad] = float("nan")
    st = torch.cuda.current_stream().cuda_stream
    zbuf, z = guarded(M, n_out, "nan")
    abuf, a = guarded(M, n_out, "nan")
    dbuf, dp = guarded(M, n_in, "nan")
    pm.pm_linear_fwd(st, "bf16", M, n_in, n_out, x.data_ptr(), W.data_ptr(), b.data_ptr(), "relu", z.data_ptr(), a.data_ptr())
    pm.pm_linear_bwd_data(st, "bf16", M, n_in, n_out, dz.data_ptr(), W.data_ptr(), zp.data_ptr(), "relu", dp.data_ptr())
    torch.cuda.synchronize()
    keep = [m for m in range(M) if m != bad]
    Wd = W.double()
    for got, ref, S, K in ((z, x.double() @ Wd.T + b.double(), x.double().abs() @ Wd.abs().T + b.double().abs(), n_in),
                           (dp, (dz.double() @ Wd) * (zp.double() > 0), dz.double().abs() @ Wd.abs(), n_out)):
        tol = 2.0 ** -8 * ref.abs() + (K + 4) * 2.0 ** -24 * S
        assert bool(((got.double() - ref).abs() <= tol)[keep].all())
        if bad is not None and got is z:
            assert bool(torch.isnan(got[bad]).all())
    assert torch.equal(a[keep], torch.relu(z[keep]))
    for buf, t in ((zbuf, z), (abuf, a), (dbuf, dp)):
        assert bool(torch.isnan(buf[:2048]).all()) and bool(torch.isnan(buf[2048 + t.numel():]).all())
