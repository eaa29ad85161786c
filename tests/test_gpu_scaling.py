"""GPU checks of the dynamic adjoint scaling state machine (paper Algorithm 2: initial scale,
halve-and-retry on overflow, failure after k_max attempts, growth) and of the unscaled-safe
variant, against the CPU oracle; plus degenerate inputs.  Scale histories and retry counts are
powers of two and integers: they must match exactly."""
import numpy as np
import pytest
import torch

from paper_2510_23498_amd import binding as rb
from paper_2510_23498_amd import workloads as wl
from oracle import rampde_oracle as orc

import parity as par

pytestmark = pytest.mark.gpu
PATHS = pytest.mark.parametrize("flags", [0, rb.PER_LAYER_KERNELS], ids=["tile", "layer"])


def _linear_case(N):
    """One linear layer with gain 128 and no time input: the cotangent W^T lambda overflows fp16
    at the initial scale (|lambda| ~ 2^11 times 2^7), so the scale has to be halved."""
    d = 4
    theta = np.concatenate([(np.eye(d) * 128.0).ravel(), np.zeros(d)]).astype(np.float32)
    y0 = np.full((2, d), 0.001, dtype=np.float32)
    tg = np.arange(N + 1, dtype=np.float64) * 2.0 ** -10
    aN = np.full((2, d), 1.5, dtype=np.float32)
    return d, theta, y0, tg, aN


def _gpu_linear(d, theta, y0, tg, aN, scaling, k_max, flags, tabname="euler", grad_t=None):
    dev = torch.device("cuda:0")
    vel = rb.Velocity.mlp((d, d), time_input=False)
    t = wl.TABLEAUX[tabname]
    tab = rb.Tableau(t.A, t.b, t.c)
    pol = rb.Policy(low="f16", scaling=scaling, k_max=k_max, flags=flags)
    th = torch.from_numpy(theta).to(dev)
    yN, ck = rb.rampde_odeint_fwd(vel, th, torch.from_numpy(y0).to(dev), tg, tab, pol)
    return rb.rampde_odeint_bwd(vel, th, tg, tab, pol, ck, torch.from_numpy(aN).to(dev), grad_t=grad_t), ck


def _oracle_linear(d, theta, y0, tg, aN, scaling, k_max, tabname="euler"):
    vel = orc.MLPVelocity((d, d), time_input=False, activation="identity")
    pol = orc.Policy(low="f16", scaling=scaling, k_max=k_max)
    tab = wl.TABLEAUX[tabname]
    yN, ck = orc.odeint_fwd(vel, theta.astype(np.float64), y0, tg, tab, pol)
    return orc.odeint_bwd(vel, theta.astype(np.float64), tg, tab, pol, ck, aN)


@PATHS
@pytest.mark.parametrize("N,tabname", [(1, "euler"), (5, "euler"), (4, "rk4")])
def test_overflow_halves_scale_and_retries(N, tabname, flags):
    case = _linear_case(N)
    print(f"[case] overflow retry N={N} {tabname} flags={flags}", flush=True)
    (gy0, gth, info), _ = _gpu_linear(*case, "dynamic", 16, flags, tabname)
    ref = _oracle_linear(*case, "dynamic", 16, tabname)
    assert ref.status == "ok" and ref.retries >= 1
    assert info.status == 0 and info.retries == ref.retries
    np.testing.assert_array_equal(info.scale_hist.astype(np.float64), ref.scale_hist)
    assert par.rel_err(gy0.cpu().numpy(), ref.grad_y0) <= par.TOL_EMUL
    assert par.rel_err(gth.cpu().numpy(), ref.grad_theta) <= par.TOL_EMUL
    assert info.s_min == ref.scale_hist.min() and info.s_max == ref.scale_hist.max()


@PATHS
def test_scaling_fails_after_k_max_attempts(flags):
    case = _linear_case(3)
    ref = _oracle_linear(*case, "dynamic", 1)
    assert ref.status == "scale_failed"
    with pytest.raises(rb.RampdeError) as ei:
        _gpu_linear(*case, "dynamic", 1, flags)
    assert ei.value.code == rb.ESCALE
    assert ei.value.stats.failed_step == ref.failed_step == 2
    assert ei.value.stats.status == 2


@PATHS
def test_unscaled_safe_returns_infinite_gradients(flags):
    d, theta, y0, tg, aN = _linear_case(2)
    ref = _oracle_linear(d, theta, y0, tg, aN * 1000.0, "none_safe", 1)
    assert ref.status == "overflow_inf"
    (gy0, gth, info), _ = _gpu_linear(d, theta, y0, tg, aN * 1000.0, "none_safe", 1, flags)
    assert info.status == 1 and info.failed_step == ref.failed_step
    assert torch.isinf(gth).all() and torch.isinf(gy0).all()
    # without an overflow the safe variant equals the unscaled one
    (gy0s, gths, infos), _ = _gpu_linear(d, theta, y0, tg, aN * 1e-3, "none_safe", 1, flags)
    (gy0n, gthn, _), _ = _gpu_linear(d, theta, y0, tg, aN * 1e-3, "none", 1, flags)
    assert infos.status == 0
    assert torch.equal(gy0s, gy0n) and par.rel_err(gths.cpu().numpy(), gthn.cpu().numpy()) < 1e-6


@PATHS
def test_nonfinite_terminal_gradient_is_reported_at_step_N(flags):
    d, theta, y0, tg, aN = _linear_case(3)
    aN = aN.copy()
    aN[1, 2] = np.inf
    with pytest.raises(rb.RampdeError) as ei:
        _gpu_linear(d, theta, y0, tg, aN, "dynamic", 16, flags)
    assert ei.value.code == rb.ESCALE and ei.value.stats.failed_step == 3


@PATHS
def test_zero_terminal_gradient_gives_unit_scale_and_zero_gradients(flags):
    d, theta, y0, tg, aN = _linear_case(3)
    (gy0, gth, info), _ = _gpu_linear(d, theta, y0, tg, np.zeros_like(aN), "dynamic", 16, flags)
    assert info.status == 0 and info.scale_hist[3] == 1.0
    assert not gy0.any() and not gth.any()


@PATHS
def test_scale_grows_when_the_adjoint_decays(flags):
    # contracting linear dynamics: |a| shrinks going backward, so the scale must double (growth rule)
    d = 4
    theta = np.concatenate([(-np.eye(d) * 64.0).ravel(), np.zeros(d)]).astype(np.float32)
    y0 = np.full((3, d), 0.25, dtype=np.float32)
    tg = np.linspace(0.0, 12 * 2.0 ** -8, 13)
    aN = np.full((3, d), 3.0, dtype=np.float32)
    (gy0, gth, info), _ = _gpu_linear(d, theta, y0, tg, aN, "dynamic", 16, flags)
    ref = _oracle_linear(d, theta, y0, tg, aN, "dynamic", 16)
    assert ref.scale_hist[0] > ref.scale_hist[-1]
    np.testing.assert_array_equal(info.scale_hist.astype(np.float64), ref.scale_hist)
    assert info.retries == ref.retries
    assert par.rel_err(gy0.cpu().numpy(), ref.grad_y0) <= par.TOL_EMUL
    assert par.rel_err(gth.cpu().numpy(), ref.grad_theta) <= par.TOL_EMUL


@PATHS
def test_literal_policy_flags(flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="lit", B=40, N=6)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    for gflag, okw in ((rb.ROUND_INCREMENT, {"round_increment": True}), (rb.GROW_RAW_NORM, {"grow_raw_norm": True})):
        gpu = par.run_gpu(cfg, theta, y0, target, flags=flags | gflag)
        emu = par.run_oracle(cfg, theta, y0, target, "emul", flags=okw)
        par.compare(cfg, gpu, emu, par.TOL_EMUL, f"emulation oracle {okw}")
        np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


@PATHS
def test_single_sample_single_step(flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="one", B=1, N=1, widths=(3, 16, 3), tableau="euler")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.2)
    gpu = par.run_gpu(cfg, theta, y0, target, flags=flags)
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")


def test_gradient_is_accumulated_into_the_callers_vector():
    # g starts at the caller's dL/dtheta (Algorithm 2, initialisation)
    cfg = wl.CONFIGS["cfg1"].with_(name="acc", B=32, N=3)
    theta, y0, target = par.make_inputs(cfg)
    vel, tab, pol = par.gpu_descriptors(cfg)
    dev = torch.device("cuda:0")
    th = torch.from_numpy(theta).to(dev)
    yN, ck = rb.rampde_odeint_fwd(vel, th, torch.from_numpy(y0).to(dev), cfg.tgrid(), tab, pol)
    gyN = (yN - torch.from_numpy(target).to(dev)).contiguous()
    _, g0, _ = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, gyN)
    init = torch.full_like(g0, 0.5)
    _, g1, _ = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, gyN, grad_theta=init.clone())
    assert par.rel_err((g1 - 0.5).cpu().numpy(), g0.cpu().numpy()) < 1e-5



@PATHS
@pytest.mark.parametrize("N,tabname", [(5, "euler"), (4, "rk4")])
def test_time_grid_gradient_counts_a_retried_step_once(N, tabname, flags):
    # the sums of a step whose cotangent chain overflowed are discarded before the step is redone
    case = _linear_case(N)
    print(f"[case] dL/dt with overflow retry N={N} {tabname}", flush=True)
    gt = torch.full((N + 1,), 0.25, dtype=torch.float32, device="cuda:0")   # accumulated into
    (gy0, gth, info), _ = _gpu_linear(*case, "dynamic", 16, flags, tabname, grad_t=gt)
    ref = _oracle_linear(*case, "dynamic", 16, tabname)
    assert ref.retries >= 1 and info.retries == ref.retries
    assert par.rel_err(gt.cpu().numpy() - 0.25, ref.grad_t) <= par.TOL_EMUL, (gt.cpu().numpy() - 0.25, ref.grad_t)
    assert par.rel_err(gy0.cpu().numpy(), ref.grad_y0) <= par.TOL_EMUL


# ------------------------------------------------------------------ the state machine at multi-workgroup sizes
def _gain_case(base, **kw):
    """A workload whose LAST weight tensor is multiplied by `gain`: the cotangent chain then amplifies
    the scaled adjoint beyond the fp16 range at the initial scale, and the adjoint itself grows from
    step to step going backward, so that the scale has to be halved again in the middle of the pass."""
    gain = kw.pop("gain")
    cfg = wl.CONFIGS[base].with_(**{"low": "f16", **kw})
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    name, shp, off = [x for x in wl.theta_layout(cfg) if x[0].startswith("W")][-1]
    theta = theta.copy()
    theta[off:off + int(np.prod(shp))] *= gain
    return cfg, theta, y0, target


MULTI_WG = [
    # the 8-wavefront adjoint kernel (wide network), several row tiles and a ragged tail
    ("cfg3", dict(name="retry512", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic")),
    # the register-resident kernels (all steps in one launch)
    ("cfg2", dict(name="retry256", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic")),
    # the 4-wavefront adjoint kernel with the parameter gradients on the helper stream (stages that are not a chain)
    ("cfg2", dict(name="retry256k", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic", tableau="kutta3")),
    # the convolution path (per-layer kernels)
    ("cfg4", dict(name="retryconv", B=2, N=4, C=8, H=8, W=16, t1=0.02, gain=256.0, scaling="dynamic")),
]


@pytest.mark.parametrize("base,kw", MULTI_WG, ids=[k["name"] for _, k in MULTI_WG])
@pytest.mark.parametrize("flags,row_tile,wgrad_tile,step_group",
                         [(0, 0, 0, 0), (rb.PER_LAYER_KERNELS, 0, 0, 0), (0, 64, 0, 0), (0, 64, 256, 0), (0, 64, 256, 3),
                          (0, 64, 256, 1)],
                         ids=["tile", "layer", "wide", "wide-groups-of-4", "wide-groups-of-3", "wide-groups-of-1"])
def test_retry_in_the_middle_of_the_pass_many_workgroups(base, kw, flags, row_tile, wgrad_tile, step_group):
    # (wgrad_tile = 256: the parameter gradients of a group of accepted steps are one launch; a rejected
    # step cuts its group short and the next group starts with it)
    if base == "cfg4" and (flags or row_tile):
        pytest.skip("the convolution has one path")
    if base == "cfg2" and row_tile:
        pytest.skip("the 64-row-tile kernels are for 512-wide networks")
    cfg, theta, y0, target = _gain_case(base, **dict(kw))
    print(f"[case] mid-pass retry {cfg.name} B={cfg.B} flags={flags}", flush=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    hist = emu["scale_hist"]
    assert emu["status"] == "ok" and emu["retries"] >= 3
    assert np.sum(hist[:-1] < hist[1:]) >= 2, "the scale must drop at more than one step"
    gpu = par.run_gpu(cfg, theta, y0, target, flags=flags, row_tile=row_tile, wgrad_tile=wgrad_tile, step_group=step_group)
    assert gpu["status"] == 0
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), hist)
    assert gpu["retries"] == emu["retries"]
    # (the scale decisions above are exact; the values are compared at the fp64 tolerance: a last layer
    # with gain 256 magnifies every difference in fp32 summation order by that gain, here and in the
    # forward pass, so these deliberately ill-conditioned networks do not reach 1e-3)
    errs = par.compare(cfg, gpu, emu, par.TOL_F64[cfg.low], "emulation oracle (amplifying network)")
    print("  vs emul:", {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)


@pytest.mark.parametrize("step_group", [2, 3, 5])
def test_retry_in_the_middle_of_a_group_of_convolution_steps(step_group):
    # stages of a group recomputed in one launch, its parameter gradients in one that leaves the rejected step and those
    # behind it out; tiles that exchange lines
    cfg, theta, y0, target = _gain_case("cfg4", name="retryconvgroup", B=2, N=5, C=8, H=24, W=20, t1=0.025, gain=256.0, scaling="dynamic")
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    assert emu["status"] == "ok" and emu["retries"] >= 2
    gpu = par.run_gpu(cfg, theta, y0, target, step_group=step_group)
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    assert gpu["status"] == 0 and gpu["retries"] == emu["retries"]
    par.compare(cfg, gpu, emu, par.TOL_F64[cfg.low], "emulation oracle (amplifying network)")


@pytest.mark.parametrize("C,H,B", [(64, 16, 64), (64, 8, 64)])
def test_weight_gradients_with_a_running_cost_use_the_whole_device(C, H, B):
    # the steps go one by one then: a step's contraction is dealt out as where a group is one step.  With the chunks of a
    # step in a full group they took 4 to 16 times as long; the bound leaves 2 for the noise of short launches
    cfg = wl.CONFIGS["cfg4"].with_(name="convgys", B=B, N=32, C=C, H=H, W=H, tableau="heun", low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    th, y = (torch.from_numpy(x).to("cuda:0") for x in (theta, y0))
    gys = torch.zeros((cfg.N + 1,) + tuple(cfg.state_shape), device="cuda:0")
    ms = {}
    for group in (0, 1):
        vel, tab, pol = par.gpu_descriptors(cfg, "none", step_group=group)
        yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
        for _ in range(3):
            rb.rampde_timing_enable(True)
            rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, yN, grad_ys=gys)
            t, launches, _ = rb.rampde_timing_read(rb.K_WGRAD_GEMM)
            rb.rampde_timing_enable(False)
            assert launches == cfg.N
            ms[group] = min(t, ms.get(group, t))
    assert ms[0] <= 2 * ms[1]


@pytest.mark.parametrize("scaling", ["dynamic", "none"])
def test_fewer_convolution_steps_at_once_on_a_smaller_workspace(scaling):
    # the queried workspace holds the stages of all five steps; one with room for fewer takes fewer at once: the bits of a
    # call that asks for as many
    cfg, theta, y0, _ = _gain_case("cfg4", name="fewersets", B=6, N=5, C=8, H=24, W=20, t1=0.025, gain=1.0, scaling=scaling)
    vel, tab, pol = par.gpu_descriptors(cfg, scaling)
    th, y = (torch.from_numpy(x).to("cuda:0") for x in (theta, y0))
    yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
    gyN = 2 / yN.numel() * yN

    def backward(policy, size):
        gy0, gth, info = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, policy, ck, gyN, workspace=ws[:size])
        assert info.status == 0
        return gy0, gth

    asked = {g: par.gpu_descriptors(cfg, scaling, step_group=g)[2] for g in (5, 2, 1)}
    sizes = {g: rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, a, True) for g, a in asked.items()}
    assert sizes[5] > sizes[2] > sizes[1]
    ws = rb.alloc_workspace(vel, cfg.B, cfg.N, tab, pol, True)
    for g, a in asked.items():
        want, got = backward(a, sizes[5]), backward(pol, sizes[g])
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("flags", [0, rb.NO_WAITS])
@pytest.mark.parametrize("C,H,W", [(40, 20, 16), (24, 9, 12)])
def test_overflow_of_a_convolution_under_a_fixed_scale_leaves_its_infinity(C, H, W, flags):
    # a hidden cotangent overflows around one pixel (2e4 / 2 x 10 > 65504) and with it, all weights being positive, the
    # cotangents of the stage before: db_1 and db_2 are infinite, as sums of +infinity and finite terms.  The pad channels
    # (infinity times their zero weights) must not make them NaN
    cfg = wl.CONFIGS["cfg4"].with_(name="convinf", B=1, N=1, C=C, H=H, W=W, tableau="heun", low="f16")
    theta = np.zeros(cfg.n_params, dtype=np.float32)
    slices = {n: (slice(o, o + int(np.prod(shp))), shp) for n, shp, o in wl.theta_layout(cfg)}
    for n in ("W1", "W2"):
        theta[slices[n][0]].reshape(slices[n][1])[:, :C] = 10.0  # (not the time's)
    vel, tab, pol = par.gpu_descriptors(cfg, "none", flags=flags)
    th, y0 = torch.from_numpy(theta).to("cuda:0"), torch.zeros((1, C, H, W), device="cuda:0")
    _, ckpt = rb.rampde_odeint_fwd(vel, th, y0, cfg.tgrid(), tab, pol)
    gyN = torch.zeros_like(y0)
    gyN[0, 3, H // 2, W // 2] = 2e4
    _, gth, _ = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ckpt, gyN)
    for n in ("b1", "b2"):
        assert bool(torch.isposinf(gth[slices[n][0]]).all())


@pytest.mark.parametrize("base,kw", MULTI_WG, ids=[k["name"] for _, k in MULTI_WG])
def test_scaling_failure_many_workgroups(base, kw):
    cfg, theta, y0, target = _gain_case(base, **dict(kw))
    emu = par.run_oracle(cfg, theta, y0, target, "emul", k_max=1)
    assert emu["status"] == "scale_failed"
    print(f"[case] scaling failure {cfg.name}: oracle fails at step {emu['failed_step']}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, k_max=1, expect_error=True)
    assert gpu.get("error") == rb.ESCALE
    assert gpu["info"].failed_step == emu["failed_step"] and gpu["info"].status == 2


@pytest.mark.parametrize("base,kw", MULTI_WG, ids=[k["name"] for _, k in MULTI_WG])
def test_unscaled_safe_many_workgroups(base, kw):
    # a loss gradient of order 1e3 overflows the unscaled fp16 chain of these amplifying networks
    kw = dict(kw)
    kw["scaling"] = "none_safe"
    cfg, theta, y0, target = _gain_case(base, **kw)
    cfg = cfg.with_(grad_scale=1e3 if cfg.loss == "half_sse" else 1e3 * cfg.B * cfg.d)
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    assert emu["status"] == "overflow_inf"
    print(f"[case] unscaled-safe overflow {cfg.name}: oracle overflows at step {emu['failed_step']}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target)
    assert gpu["status"] == 1 and gpu["failed_step"] == emu["failed_step"]
    assert np.all(np.isinf(gpu["grad_theta"])) and np.all(np.isinf(gpu["grad_y0"]))


# Kernels that run several adjoint steps in a launch and take the accept / grow decisions themselves
GROUPED = [
    ("cfg2", dict(name="retry256", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic")),
    ("cfg2", dict(name="retry128", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(30, 100, 100, 100, 30))),
    # one hidden layer, activations from memory and from LDS; flows, whose trace row adds sums of every accepted step
    ("cfg2", dict(name="retry1h", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(64, 600, 64))),
    ("cfg2", dict(name="retry1h2", B=40, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(128, 512, 128))),
    ("cnf", dict(name="retrycnf", B=100, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(20, 200, 20))),
    ("cnf", dict(name="retrycnfw", B=40, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(15, 600, 15))),
    # workgroups that share row tiles (groups of two steps and up; one step per group and dL/dt: the row-tile kernels)
    ("cfg2", dict(name="retrycl512", B=70, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(128, 512, 512, 128))),
    ("cfg2", dict(name="retrycl768", B=40, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(128, 700, 128))),
]


def _compare_amplifying(cfg, theta, y0, target, gpu, emu, flags=None, want_grad_t=False):
    """Every tensor within the fp64 tolerance or four times the oracle's own response to weights that are perturbed by
    3e-7 relative (a couple of fp32 roundings; the largest of three draws), where that is more: a network whose last layer
    has gain 256 turns one flipped 16-bit rounding into up to 5 % of the early gradients."""
    rng = np.random.default_rng(7)
    errs, sens = {}, {}
    outs = {"yN": lambda r: r["yN"], "grad_y0": lambda r: r["grad_y0"], "grad_theta": lambda r: r["grad_theta"]}
    if want_grad_t:
        outs["grad_t"] = lambda r: r["grad_t"]
    for name, sl in par.layer_slices(cfg):
        outs["grad_" + name] = lambda r, sl=sl: r["grad_theta"][sl]
    alts = [par.run_oracle(cfg, (theta * (1.0 + 3e-7 * rng.standard_normal(theta.shape))).astype(np.float32), y0, target, "emul",
                           flags=flags) for _ in range(3)]
    for k, get in outs.items():
        errs[k] = par.rel_err(get(gpu), get(emu))
        sens[k] = max(par.rel_err(get(a), get(emu)) for a in alts)
    print("  vs emul / oracle's response:", {k: f"{errs[k]:.1e} / {sens[k]:.1e}" for k in errs}, flush=True)
    bad = {k: (errs[k], sens[k]) for k in errs if not errs[k] <= max(par.TOL_F64[cfg.low], 4.0 * sens[k])}
    assert not bad, bad


@pytest.mark.parametrize("base,kw", GROUPED, ids=[k["name"] for _, k in GROUPED])
@pytest.mark.parametrize("step_group,want_grad_t", [(0, False), (1, False), (2, False), (4, False), (2, True), (0, True)])
def test_retry_inside_and_across_groups_of_steps(base, kw, step_group, want_grad_t):
    # a rejected step ends its launch; the pass goes on from the adjoint that this launch wrote (its own buffer, or
    # dL/dy_0 if it was the last group), and what the rejected run added to dL/dt is replaced
    cfg, theta, y0, target = _gain_case(base, **dict(kw))
    print(f"[case] retry in groups of {step_group}: {cfg.name} grad_t={want_grad_t}", flush=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    hist = emu["scale_hist"]
    assert emu["status"] == "ok" and emu["retries"] >= 3
    assert np.sum(hist[:-1] < hist[1:]) >= 3, "the scale must drop at several steps"
    gpu = par.run_gpu(cfg, theta, y0, target, step_group=step_group, want_grad_t=want_grad_t)
    assert gpu["status"] == 0 and gpu["retries"] == emu["retries"]
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), hist)
    _compare_amplifying(cfg, theta, y0, target, gpu, emu, want_grad_t=want_grad_t)


LEAST = GROUPED + [("cfg2", dict(name="retry4l", B=300, N=6, t1=0.09, gain=256.0, scaling="dynamic", widths=(64, 256, 256, 256, 64)))]


@pytest.mark.parametrize("base,kw", LEAST, ids=[k["name"] for _, k in LEAST])
@pytest.mark.parametrize("want_grad_t", [False, True])
def test_retries_on_the_least_workspace(base, kw, want_grad_t):
    # the smallest workspace that the pass accepts (kernels that need less than those of the queried size): the same
    # decisions, and nothing written behind it
    cfg, theta, y0, target = _gain_case(base, **dict(kw))
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    vel, tab, pol = par.gpu_descriptors(cfg)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
    gyN = torch.from_numpy(np.ascontiguousarray(wl.loss_and_grad(cfg, yN.cpu().numpy(), target)[1])).to(dev)
    ws = rb.alloc_workspace(vel, cfg.B, cfg.N, tab, pol, True)

    def run(size):
        gt = torch.zeros(cfg.N + 1, device=dev) if want_grad_t else None
        ws[size:] = 77
        gy0, gth, info = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, gyN, workspace=ws[:size], grad_t=gt)
        assert bool((ws[size:] == 77).all())
        return dict(yN=yN.cpu().numpy(), grad_y0=gy0.cpu().numpy(), grad_theta=gth.cpu().numpy(), retries=info.retries,
                    scale_hist=info.scale_hist, grad_t=gt.cpu().numpy() if want_grad_t else None)

    refused, size, gpu = 0, ws.numel(), run(ws.numel())
    while size - refused > 256:
        mid = (refused + size) // 512 * 256
        try:
            gpu, size = run(mid), mid
        except rb.RampdeError as e:
            assert e.code == rb.EWORKSPACE
            refused = mid
    print(f"[case] {cfg.name}: {size} of {ws.numel()} bytes", flush=True)
    assert gpu["retries"] == emu["retries"]
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    _compare_amplifying(cfg, theta, y0, target, gpu, emu, want_grad_t=want_grad_t)


@pytest.mark.parametrize("base,kw", GROUPED[1:], ids=[k["name"] for _, k in GROUPED[1:]])
def test_failure_overflow_and_scale_groups_with_grouped_steps(base, kw):
    cfg, theta, y0, target = _gain_case(base, **dict(kw))
    print(f"[case] failure, unscaled-safe overflow, scale groups: {cfg.name}", flush=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", k_max=1)
    gpu = par.run_gpu(cfg, theta, y0, target, k_max=1, expect_error=True, step_group=4)
    assert emu["status"] == "scale_failed" and gpu.get("error") == rb.ESCALE
    assert gpu["info"].failed_step == emu["failed_step"] and gpu["info"].status == 2
    big = cfg.with_(scaling="none_safe", grad_scale=1e3 if cfg.loss == "half_sse" else 1e3 * cfg.B * cfg.d)
    emu = par.run_oracle(big, theta, y0, target, "emul")
    gpu = par.run_gpu(big, theta, y0, target, step_group=4)
    assert emu["status"] == "overflow_inf" and gpu["status"] == 1 and gpu["failed_step"] == emu["failed_step"]
    assert np.all(np.isposinf(gpu["grad_y0"])) and np.all(np.isposinf(gpu["grad_theta"]))
    # two scale groups, each with its own retries (G times the state width is a multiple of 8)
    G = (cfg.B // 2 + 8) // 8 * 8
    emu = par.run_oracle(cfg, theta, y0, target, "emul", flags={"scale_group": G})
    gpu = par.run_gpu(cfg, theta, y0, target, scale_group=G, step_group=4)
    assert emu["status"] == "ok" and gpu["status"] == 0 and gpu["retries"] == emu["retries"] >= 4
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    _compare_amplifying(cfg, theta, y0, target, gpu, emu, flags={"scale_group": G})


@PATHS
@pytest.mark.parametrize("want_info", [True, False])
def test_unscaled_variant_propagates_a_nonfinite_loss_gradient(flags, want_info):
    # the plain unscaled variant has no range checks (paper Sec. 5): an inf in dL/dy_N is not an
    # error and must come back as non-finite gradients, with or without the statistics block
    cfg = wl.CONFIGS["cfg1"].with_(name="infgrad", B=40, N=5, widths=(6, 32, 6))
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    vel, tab, pol = par.gpu_descriptors(cfg, scaling="none", flags=flags)
    dev = torch.device("cuda:0")
    th = torch.from_numpy(theta).to(dev)
    yN, ck = rb.rampde_odeint_fwd(vel, th, torch.from_numpy(y0).to(dev), cfg.tgrid(), tab, pol)
    gyN = torch.ones_like(yN)
    gyN[3, 2] = float("inf")
    gy0 = torch.zeros_like(yN)
    gth = torch.zeros(rb.rampde_num_params(vel), dtype=torch.float32, device=dev)
    _, _, info = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, gyN, grad_y0=gy0, grad_theta=gth,
                                      want_info=want_info)
    torch.cuda.synchronize()
    assert not torch.isfinite(gy0).all() and not torch.isfinite(gth).all()
    if want_info:
        assert info.status == 0


def _constant_adjoint_case(N):
    """Zero velocity: the adjoint stays at 1.5 in every entry, nothing in the chain can overflow
    except lambda = Q(S a) itself.  S_N = 2^10 (S_N * 1.5 = 1536 lies in (1024, 2048])."""
    d = 4
    theta = np.zeros(d * d + d, dtype=np.float32)
    y0 = np.full((2, d), 0.5, dtype=np.float32)
    tg = np.arange(N + 1, dtype=np.float64) / N
    aN = np.full((2, d), 1.5, dtype=np.float32)
    return d, theta, y0, tg, aN


@PATHS
def test_raw_norm_growth_rule_differs_from_the_default(flags):
    # default rule: S ||a|| = 1536 > 1/(2 u) = 1024, the scale never grows: 2^10 throughout.
    # literal rule (||a|| = 1.5 <= 1024 at every clean step): the scale doubles after every clean
    # step, so step i is entered with 2^(10 + N-1-i), until lambda = 2^16 * 1.5 overflows fp16; that
    # step halves back to 2^15 (one retry, and no growth after a retried step), the next one is
    # entered with 2^15, is clean and doubles, the one after overflows again, and so on.
    N = 10
    d, theta, y0, tg, aN = _constant_adjoint_case(N)
    expect_default = np.full(N + 1, 2.0 ** 10)
    expect_raw = np.array([2.0 ** min(10 + (N - 1 - i), 15) for i in range(N)] + [2.0 ** 10])
    first_overflow = N - 1 - 6
    expect_retries = {0: 0, rb.GROW_RAW_NORM: (first_overflow + 2) // 2}
    for gflag, want in ((0, expect_default), (rb.GROW_RAW_NORM, expect_raw)):
        (gy0, gth, info), _ = _gpu_linear(d, theta, y0, tg, aN, "dynamic", 16, flags | gflag)
        np.testing.assert_array_equal(info.scale_hist.astype(np.float64), want)
        assert info.status == 0 and info.retries == expect_retries[gflag]
        assert torch.equal(gy0.cpu(), torch.from_numpy(aN))


# ------------------------------------------------------------------ scale groups (policy.scale_group)
def _group_inputs(cfg, spread):
    """Inputs whose loss gradient differs from sample to sample by powers of two up to 2^-spread, so that
    the groups start from different scales: the running-cost cotangents of sample b (added to the adjoint
    at every step) are scaled by 2^-(b * spread // B); the terminal-cost gradient, which weighs all
    samples alike, is made negligible beside them (the caller passes a cfg with a tiny grad_scale)."""
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    shape = (cfg.N + 1,) + tuple(np.shape(y0))
    u = wl.uniforms(cfg.seed + 29, f"{cfg.name}.scale_groups.gys", int(np.prod(shape))).reshape(shape)
    w = 2.0 ** -(np.arange(cfg.B) * spread // cfg.B)
    gys = (0.05 * (u - 0.5) * w.reshape((1, cfg.B) + (1,) * (len(shape) - 2))).astype(np.float32)
    return theta, y0, target, gys


GROUP_CASES = [
    # (workload, overrides, G, flags, row_tile): a group size that does not divide the batch; groups of one
    # 64-row tile of the wide kernels; the per-layer kernels; the convolution path with one sample per group
    ("cfg1", dict(name="groups_cfg1", B=70), 32, 0, 0),
    ("cfg3", dict(name="groups_cfg3", B=200, N=4), 64, 0, 64),
    ("cfg3", dict(name="groups_cfg3_tile", B=100, N=3), 48, 0, 16),
    ("cfg2", dict(name="groups_cfg2_layer", B=90, N=4, low="f16", scaling="dynamic"), 40, 4, 0),
    ("cfg4", dict(name="groups_conv", B=3, N=3, C=8, H=8, W=16), 1, 0, 0),
]


@pytest.mark.parametrize("base,kw,G,flags,row_tile", GROUP_CASES, ids=[c[1]["name"] for c in GROUP_CASES])
def test_scale_groups_match_the_oracle_with_the_same_groups(base, kw, G, flags, row_tile):
    cfg = wl.CONFIGS[base].with_(grad_scale=1e-12, **kw)
    theta, y0, target, gys = _group_inputs(cfg, spread=24)
    print(f"[case] scale groups {cfg.name} B={cfg.B} G={G} flags={flags} row_tile={row_tile}", flush=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", flags={"scale_group": G}, grad_ys=gys)
    assert emu["status"] == "ok"
    groups = -(-cfg.B // G)
    assert emu["scale_hist"].shape == (groups, cfg.N + 1)
    assert len({tuple(r) for r in emu["scale_hist"]}) > 1, "the groups must not all share one scale history"
    gpu = par.run_gpu(cfg, theta, y0, target, flags=flags, row_tile=row_tile, grad_ys=gys, scale_group=G,
                      want_grad_t=True)
    assert gpu["status"] == 0
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    assert gpu["retries"] == emu["retries"]
    errs = par.compare(cfg, gpu, emu, par.TOL_EMUL, f"emulation oracle (scale groups of {G})")
    errs["grad_t"] = par.rel_err(gpu["grad_t"], emu["grad_t"])
    print("  vs emul:", {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)
    assert errs["grad_t"] <= 5 * par.TOL_EMUL
    # one scale for the whole batch: the small samples' cotangents sink towards the subnormals and the
    # result moves away from the fp64 gradient, which the grouped one stays close to
    f64 = par.run_oracle(cfg, theta, y0, target, "f64", grad_ys=gys)
    last = slice(-(cfg.B - (groups - 1) * G), None)
    e_grp = par.rel_err(gpu["grad_y0"][last], f64["grad_y0"][last])
    one = par.run_gpu(cfg, theta, y0, target, flags=flags, row_tile=row_tile, grad_ys=gys)
    e_one = par.rel_err(one["grad_y0"][last], f64["grad_y0"][last])
    print(f"  last group's dL/dy_0 vs fp64: own scale {e_grp:.2e}, batch-wide scale {e_one:.2e}", flush=True)
    assert e_grp <= par.TOL_F64[cfg.low] and e_grp <= e_one * 1.5


def test_scale_groups_retry_failure_and_overflow_are_per_group():
    # the amplifying network of the mid-pass retry tests, two groups; every group retries on its own
    cfg, theta, y0, target = _gain_case("cfg3", name="groups_retry", B=150, N=5, t1=0.09, gain=256.0, scaling="dynamic")
    G = 80
    print(f"[case] scale groups with retries {cfg.name} B={cfg.B} G={G}", flush=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", flags={"scale_group": G})
    assert emu["status"] == "ok" and emu["retries"] >= 4 and emu["scale_hist"].shape == (2, cfg.N + 1)
    gpu = par.run_gpu(cfg, theta, y0, target, scale_group=G)
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    assert gpu["retries"] == emu["retries"] and gpu["status"] == 0
    par.compare(cfg, gpu, emu, par.TOL_F64[cfg.low], "emulation oracle (amplifying network, scale groups)")
    # k_max = 1: the first group fails
    emu1 = par.run_oracle(cfg, theta, y0, target, "emul", k_max=1, flags={"scale_group": G})
    gpu1 = par.run_gpu(cfg, theta, y0, target, k_max=1, expect_error=True, scale_group=G)
    assert emu1["status"] == "scale_failed" and gpu1.get("error") == rb.ESCALE
    assert gpu1["info"].failed_step == emu1["failed_step"] and gpu1["info"].status == 2
    # unscaled-safe: an overflow in a group leaves +inf in ALL of dL/dy_0 and dL/dtheta
    big = cfg.with_(grad_scale=1e3 * cfg.B * cfg.d, scaling="none_safe")
    emu2 = par.run_oracle(big, theta, y0, target, "emul", flags={"scale_group": G})
    gpu2 = par.run_gpu(big, theta, y0, target, scale_group=G)
    assert emu2["status"] == "overflow_inf" and gpu2["status"] == 1
    assert np.all(np.isposinf(gpu2["grad_y0"])) and np.all(np.isposinf(gpu2["grad_theta"]))


def test_scale_group_sizes_that_cover_the_batch_are_the_default_path():
    cfg = wl.CONFIGS["cfg1"].with_(name="groups_whole", B=40)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    base = par.run_gpu(cfg, theta, y0, target)
    for G in (40, 1000):
        got = par.run_gpu(cfg, theta, y0, target, scale_group=G)
        assert got["scale_hist"].shape == (cfg.N + 1,)
        np.testing.assert_array_equal(got["grad_theta"], base["grad_theta"])
        np.testing.assert_array_equal(got["grad_y0"], base["grad_y0"])


@pytest.mark.parametrize("row_tile", [16, 0], ids=["row-tiles", "clusters"])
def test_backward_pass_beside_a_long_forward_pass_on_another_stream(row_tile):
    # row tiles: the forward pass (about 100 ms) holds a quarter of the compute units, so that the 256 workgroups of the
    # backward launch, which exchange the adjoint scale, cannot all run: the launch gives up and the pass is redone step by
    # step long before the forward pass ends.  Clusters: the forward pass holds the whole device in launches of about 3 ms,
    # the backward kernels run between them or beside one whose workgroups then cannot all run, so that it is redone by row
    # tiles: its results are those of the pass alone, or of the row tiles
    long = wl.CONFIGS["cfg5"].with_(name="beside", N=1024)
    cfg = wl.CONFIGS["cfg2"].with_(name="beside", low="f16", N=8)
    dev = torch.device("cuda:0")

    def tensors(c):
        theta, y0, _ = par.make_inputs(c)
        return torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)

    lvel, ltab, lpol = par.gpu_descriptors(long, row_tile=row_tile)
    lth, ly0 = tensors(long)
    lws = rb.alloc_workspace(lvel, long.B, long.N, ltab, lpol, False)
    lyN, lck = torch.empty_like(ly0), torch.empty(lvel.ckpt_shape(long.B, long.N), dtype=torch.float16, device=dev)
    vel, tab, pol = par.gpu_descriptors(cfg)
    th, y0 = tensors(cfg)
    yN, ck = rb.rampde_odeint_fwd(vel, th, y0, cfg.tgrid(), tab, pol)
    ws = rb.alloc_workspace(vel, cfg.B, cfg.N, tab, pol, True)
    alone = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, yN, workspace=ws)
    undisturbed = [rb.rampde_odeint_fwd(lvel, lth, ly0, long.tgrid(), ltab, q)[0] for q in (lpol, par.gpu_descriptors(long, row_tile=16)[2])]
    mark = torch.zeros(1, device=dev)
    for _ in range(8):  # (a stream may share its hardware queue with the current one: nothing runs side by side then)
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        rb.rampde_odeint_fwd(lvel, lth, ly0, long.tgrid(), ltab, lpol, ckpt=lck, yN=lyN, workspace=lws, stream=side)
        ended = torch.cuda.Event()
        ended.record(side)
        mark.add_(1.0)
        torch.cuda.current_stream().synchronize()
        if not ended.query():
            break
    else:
        pytest.skip("no stream whose kernels run beside those of the current one")
    beside = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, yN, workspace=ws)
    waited = ended.query()
    torch.cuda.synchronize()
    assert not waited or row_tile == 0, "the backward pass must not wait for the other stream's forward pass"
    np.testing.assert_array_equal(beside[2].scale_hist, alone[2].scale_hist)
    for a, b in zip(beside[:2], alone[:2]):
        assert par.rel_err(a.cpu().numpy(), b.cpu().numpy()) <= par.TOL_EMUL
    assert any(torch.equal(lyN, ref) for ref in undisturbed)


@pytest.mark.parametrize("widths,B,N,low,tab,gain", [
    ((128, 512, 512, 128), 1, 5, "f16", "rk4", 1.0),            # one row: a tile nearly empty; a group cut by the grid's end
    ((128, 512, 512, 128), 65, 7, "bf16", "heun", 1.0),         # fixed scale: all steps of a group in one launch
    ((200, 1024, 1024, 200), 33, 9, "f16", "euler", 1.0),       # the 32-row tile of the widest networks, odd batch
    ((70, 300, 190, 70), 130, 6, "f16", "rk4", 1.0),            # run-time widths
    ((128, 512, 512, 512, 128), 300, 6, "f16", "rk4", 256.0),   # rejected steps inside a group
    ((128, 512, 512, 128), 4096, 3, "f16", "rk4", 1.0),         # several groups of whole rounds
    # both sides of the line where groups under a fixed scale recompute inside instead: 32-row tiles that fill three quarters
    # of a round, 16-row tiles of one 1024-wide layer past nine sixteenths
    ((64, 512, 512, 64), 6112, 3, "bf16", "euler", 1.0),
    ((64, 512, 512, 64), 6113, 3, "bf16", "euler", 1.0),
    ((128, 1000, 128), 2304, 3, "bf16", "heun", 1.0),
    ((128, 1000, 128), 2305, 3, "bf16", "heun", 1.0),
    # and under detection: groups of two steps from 6913 rows on, of none with two 512-wide layers
    ((128, 512, 512, 512, 128), 6913, 4, "f16", "euler", 1.0),
    ((64, 512, 512, 64), 8192, 4, "f16", "euler", 1.0),
])
def test_stages_recomputed_ahead_equal_those_recomputed_inside(widths, B, N, low, tab, gain):
    # one step per group recomputes inside the adjoint kernel.  The contractions sum in the same order in both: in bf16
    # the cotangents agree bit for bit.  In fp16 the compiler rounds fp32 -> fp16 with the multiply-add in front of it in
    # one instruction (v_fma_mixlo_f16, one rounding) in some places of a kernel and in two in others: a value whose
    # fp32 rounding meets a tie of the fp16 one (2^-13 of them) moves by one unit 2^-10, 1.1e-5 in the norm of a tensor;
    # eight such tensors in a row stay below 1e-4.  The parameter gradients are also summed in another fp32 order.
    # (With a gain of 256 in the last layer such a flip grows from step to step: the bound of this workload against the
    # oracle.)
    cfg, theta, y0, target = _gain_case("cfg3", name="ahead", widths=widths, B=B, N=N, t1=0.015 * N, low=low, tableau=tab,
                                        gain=gain, scaling="dynamic" if low == "f16" else "none")
    # (row_tile: the row-tile kernels, not the clusters of cluster.hpp)
    row_tile = 16 if B <= 2048 else 0
    one = par.run_gpu(cfg, theta, y0, target, step_group=1, row_tile=row_tile)
    for group in (0, 2):
        got = par.run_gpu(cfg, theta, y0, target, step_group=group, row_tile=row_tile)
        assert got["retries"] == one["retries"] and (gain == 1.0 or one["retries"] > 0)
        np.testing.assert_array_equal(got["scale_hist"], one["scale_hist"])
        if low == "bf16":
            np.testing.assert_array_equal(got["grad_y0"], one["grad_y0"])
        tol = 1e-4 if gain == 1.0 else par.TOL_EMUL
        assert par.rel_err(got["grad_y0"], one["grad_y0"]) <= tol
        assert par.rel_err(got["grad_theta"], one["grad_theta"]) <= tol


@pytest.mark.parametrize("widths,B,low,tab", [
    ((64, 256, 256, 64), 300, "f16", "rk4"),         # scale changes in mid-group: the first stage of a step is redone
    ((30, 128, 100, 90, 30), 17, "f16", "heun"),
    ((7, 33, 7), 1, "bf16", "euler"),
    ((64, 256, 256, 200, 64), 4113, "bf16", "rk4"),  # 32-row tiles, the last one with one row
])
def test_stages_recomputed_ahead_of_the_register_resident_chain(widths, B, low, tab):
    # one step per group runs in one kernel; the same sums in the same order, gradients of the time grid included
    cfg, theta, y0, target = _gain_case("cfg2", name="ahead_res", widths=widths, B=B, N=9, t1=0.135, low=low, tableau=tab,
                                        gain=64.0, scaling="dynamic" if low == "f16" else "none")
    for want_t in (False, True):
        one = par.run_gpu(cfg, theta, y0, target, step_group=1, want_grad_t=want_t)
        for group in (0, 4):
            got = par.run_gpu(cfg, theta, y0, target, step_group=group, want_grad_t=want_t)
            assert got["retries"] == one["retries"]
            np.testing.assert_array_equal(got["scale_hist"], one["scale_hist"])
            # (fp16: see test_stages_recomputed_ahead_equal_those_recomputed_inside)
            for key in ("grad_y0", "grad_theta") + (("grad_t",) if want_t else ()):
                assert par.rel_err(got[key], one[key]) <= (1e-5 if low == "bf16" else par.TOL_EMUL), key
    if B == 300:
        assert one["retries"] > 0


def test_scale_that_grows_within_a_launch_of_the_register_resident_chain():
    # v = -32 tanh(y) per component, close to y = 0: the adjoint shrinks by a constant factor from step to step, so the scale
    # that a step starts with is often the one before its doubling, and its first stage is redone
    cfg = wl.CONFIGS["cfg1"].with_(name="shrink", widths=(16, 64, 16), B=40, N=12, t1=12.0 / 64, low="f16", scaling="dynamic", loss="mse")
    theta, y0, target = par.make_inputs(cfg)
    theta = np.zeros_like(theta)
    for name, shp, off in wl.theta_layout(cfg):
        if name == "W1":
            theta[off:off + 64 * 17].reshape(64, 17)[:, :16] = np.tile(np.eye(16), (4, 1))
        elif name == "W2":
            theta[off:off + 16 * 64].reshape(16, 64)[:] = -8.0 * np.tile(np.eye(16), (1, 4))
    gpu = par.run_gpu(cfg, theta, y0 * 0.01, target)
    emu = par.run_oracle(cfg, theta, y0 * 0.01, target, "emul")
    assert emu["scale_hist"][0] >= 16 * emu["scale_hist"][-1]
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
