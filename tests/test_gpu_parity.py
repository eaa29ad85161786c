"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by element
in the norm-wise sense, on seeded inputs with the shapes of the five workloads.

Tolerances: relative 2-norm error <= 1e-3 against the rounding-emulation oracle and
<= 2e-2 (fp16) / 5e-2 (bf16) against the fp64 oracle, for y_N, the stored trajectory,
dL/dy_0 and dL/dtheta (overall and per parameter tensor).  The adjoint scale history and
the retry count are compared exactly: they are powers of two and integers.
"""
import numpy as np
import pytest
import torch

from paper_2510_23498_amd import workloads as wl

import parity as par

pytestmark = pytest.mark.gpu


PER_LAYER = 4  # policy flag: one kernel per layer instead of the row-tile-persistent kernels
PATHS = pytest.mark.parametrize("flags", [0, PER_LAYER], ids=["tile", "layer"])


def _both(cfg, bias_std=0.0, scaling=None, tol_emul=par.TOL_EMUL, flags=0, row_tile=0, grad_ys=None, wgrad_tile=0):
    theta, y0, target = par.make_inputs(cfg, bias_std=bias_std)
    print(f"[case] {cfg.name} kind={cfg.kind} B={cfg.B} N={cfg.N} low={cfg.low} tab={cfg.tableau} flags={flags} "
          f"row_tile={row_tile} wgrad_tile={wgrad_tile}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=flags, row_tile=row_tile, grad_ys=grad_ys,
                      wgrad_tile=wgrad_tile)
    if grad_ys is not None:
        emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling=scaling, grad_ys=grad_ys.astype(np.float64))
        par.compare(cfg, gpu, emu, tol_emul, "emulation oracle")
        return gpu, emu, None
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling=scaling)
    f64 = par.run_oracle(cfg, theta, y0, target, "f64")
    e1 = par.compare(cfg, gpu, emu, tol_emul, "emulation oracle", tol_max=par.TOL_EMUL_MAX[cfg.low])
    e2 = par.compare(cfg, gpu, f64, par.TOL_F64[cfg.low], "fp64 oracle", check_ckpt=False)
    print("  vs emul:", {k: f"{v:.2e}" for k, v in e1.items()}, flush=True)
    print("  vs f64 :", {k: f"{v:.2e}" for k, v in e2.items()}, flush=True)
    assert gpu["status"] == 0 and emu["status"] == "ok"
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    assert gpu["retries"] == emu["retries"]
    return gpu, emu, f64


@PATHS
def test_cfg1_tiny_mlp_full_size(flags):
    _both(wl.CONFIGS["cfg1"], flags=flags)


@PATHS
def test_cfg1_nonzero_bias_and_ragged_batch(flags):
    _both(wl.CONFIGS["cfg1"].with_(name="cfg1r", B=77, N=5), bias_std=0.3, flags=flags)


@PATHS
@pytest.mark.parametrize("tab", ["euler", "heun", "rk4", "kutta3"])
def test_small_mlp_all_tableaux(tab, flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="tabs", B=130, N=6, widths=(5, 40, 24, 5), tableau=tab)
    _both(cfg, bias_std=0.2, flags=flags)


@PATHS
def test_mlp_odd_widths_many_layers(flags):
    # widths that pad to 64/128/192/320 columns: every column-group size of the tile kernels
    cfg = wl.CONFIGS["cfg1"].with_(name="odd", B=50, N=3, widths=(70, 130, 300, 190, 70), tableau="heun")
    _both(cfg, bias_std=0.1, flags=flags)


@PATHS
def test_cfg2_shape_reduced_batch(flags):
    # widths of the bf16 workload; batch spans several row tiles and a ragged tail
    _both(wl.CONFIGS["cfg2"].with_(name="cfg2s", B=300, N=6), bias_std=0.1, flags=flags)


@PATHS
def test_cfg3_shape_reduced_needs_dynamic_scaling(flags):
    cfg = wl.CONFIGS["cfg3"].with_(name="cfg3s", B=200, N=6)
    gpu, emu, f64 = _both(cfg, flags=flags)
    assert gpu["scale_hist"][cfg.N] > 2.0 ** 20  # the 1e-6 loss gradient needs a large scale
    # negative control: without scaling the fp16 cotangents underflow and the gradient is lost
    theta, y0, target = par.make_inputs(cfg)
    raw = par.run_gpu(cfg, theta, y0, target, scaling="none", flags=flags)
    e_raw = par.rel_err(raw["grad_theta"], f64["grad_theta"])
    e_dyn = par.rel_err(gpu["grad_theta"], f64["grad_theta"])
    assert e_raw > par.TOL_F64["f16"] and e_raw > 10 * e_dyn, (e_raw, e_dyn)


@PATHS
def test_unscaled_fp16_cotangents_in_the_subnormal_range_match_the_emulation(flags):
    # With the 1e-6 loss gradient and NO scaling most cotangents are a few units of the smallest fp16
    # subnormal (2^-24).  The oracle keeps gradual underflow; so must every conversion and matrix
    # instruction of the device path, or the two would differ by O(1) here (the fp64 comparison in
    # test_cfg3_shape_reduced_needs_dynamic_scaling only shows that the unscaled result is useless, not
    # that both sides agree on HOW it is useless).
    # ONE step of a network with ONE hidden layer: beyond that this regime is chaotic with respect to
    # rounding -- every cotangent is the rounding of a value of about one unit, so the first entry that
    # rounds the other way (the two sides sum their fp32 accumulators in different orders) moves a whole
    # row of the next layer by a sizeable fraction of a unit, and so on.  Measured on both kernel paths
    # alike: one RK4 step of 128-512-128 agrees to 7e-6 (one Euler step bit for bit); one step of the
    # four-layer cfg3 network to 3e-4 in dL/dy_0 but only 1e-2 in the first layer's gradient; 6 steps 5e-2.
    cfg = wl.CONFIGS["cfg3"].with_(name="cfg3sub", B=200, N=1, t1=2.0 / 64, widths=(128, 512, 128))
    theta, y0, target = par.make_inputs(cfg)
    print(f"[case] {cfg.name} scaling=none flags={flags}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling="none", flags=flags)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling="none")
    step = np.abs(emu["grad_y0"] - emu["grad_yN"])
    assert 0 < np.median(step[step > 0]) < 2.0 ** -20, "the case must exercise subnormal cotangents"
    # max-norm bound: a hidden cotangent here carries two or three significant bits, so ONE entry that
    # rounds the other way moves that sample's term of a first-layer gradient entry by up to half of
    # itself; the bound allows a handful of such entries (measured 4e-3), the 2-norm bound stays 1e-3.
    errs = par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle (unscaled)", tol_max=1e-2)
    print("  vs emul:", {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)
    # the adjoint increment itself (not hidden behind the much larger dL/dy_N), in units of 2^-24: it is
    # built from those two-or-three-bit cotangents alone, so the bound is 5 * TOL_EMUL (measured 1.2e-3);
    # flushing subnormals anywhere on the way would leave O(1) here
    inc_gpu = (gpu["grad_y0"].astype(np.float64) - gpu["grad_yN"]) * 2.0 ** 24
    inc_emu = (emu["grad_y0"] - emu["grad_yN"]) * 2.0 ** 24
    assert par.rel_err(inc_gpu, inc_emu) <= 5 * par.TOL_EMUL


# ------------------------------------------------------------------ 64-row-tile kernels of 512-wide networks
@pytest.mark.parametrize("B", [200, 64, 65, 1])
def test_wide_kernels_cfg3_shape(B):
    # the kernels the full-size cfg3 runs on, requested explicitly at a batch the oracle handles:
    # several tiles and a ragged tail, exactly one tile, one tile plus one row, a single row
    _both(wl.CONFIGS["cfg3"].with_(name=f"wide{B}", B=B, N=5), bias_std=0.1, row_tile=64)


@pytest.mark.parametrize("tab,low,widths", [("heun", "f16", (128, 512, 128)), ("kutta3", "f16", (128, 512, 512, 128)),
                                            ("euler", "f16", (128, 400, 512, 300, 500, 128)),
                                            ("rk4", "bf16", (128, 512, 512, 512, 128))])
def test_wide_kernels_depths_tableaux_precisions(tab, low, widths):
    # 2 to 5 layers (hidden widths that pad to 512), every tableau; bf16 under dynamic scaling so that
    # the adjoint also takes these kernels (with a fixed scale it runs groups of steps on the others)
    cfg = wl.CONFIGS["cfg3"].with_(name=f"wide{tab}{low}", B=150, N=4, tableau=tab, low=low, widths=widths,
                                   scaling="dynamic", grad_scale=1.0 if low == "bf16" else 1e-6)
    # bf16 at contraction length 512: the device sums 512 products in fp32, the oracle in fp64 with one
    # rounding; the two land on different sides of a bf16 rounding boundary (spacing 2^-8) often enough
    # that 16 stage evaluations of 4 layers accumulate to about 1e-3 in the 2-norm.  The 16-, 32- and
    # 64-row kernels give bit-identical results on this case, so it is not a property of one kernel.
    _both(cfg, bias_std=0.1, row_tile=64, tol_emul=2e-3 if low == "bf16" else par.TOL_EMUL)


# ------------------------------------------------------------------ parameter gradients: 128 x 128 block per wavefront
@pytest.mark.parametrize("B", [200, 65, 1])
def test_slab_parameter_gradient_kernel_cfg3_shape(B):
    # the kernel that the full-size cfg3 takes by its contraction length, requested at batches the oracle
    # handles: K-chunks shorter than its ring of k-steps, a ragged tail, a single row
    _both(wl.CONFIGS["cfg3"].with_(name=f"slab{B}", B=B, N=3), bias_std=0.1, row_tile=64, wgrad_tile=256)


@pytest.mark.parametrize("tab,low,widths,row_tile", [
    ("heun", "f16", (128, 512, 128), 64), ("kutta3", "bf16", (128, 512, 512, 128), 64),
    ("euler", "f16", (128, 400, 512, 300, 500, 128), 64),      # hidden widths that are no multiple of 128
    ("rk4", "f16", (64, 1024, 1024, 64), 0), ("rk4", "f16", (38, 302, 700, 38), 0)])  # 8-wave row-tile kernels; widths that are no multiple of 4
def test_slab_parameter_gradient_kernel_shapes(tab, low, widths, row_tile):
    # every arrangement of the four wavefronts (2 x 2, 4 x 1, 1 x 4), masked feature groups, rows with
    # and without a time column, both precisions
    cfg = wl.CONFIGS["cfg3"].with_(name=f"slab{tab}{low}{len(widths)}", B=150, N=3, tableau=tab, low=low, widths=widths,
                                   scaling="dynamic", grad_scale=1.0 if low == "bf16" else 1e-6)
    _both(cfg, bias_std=0.1, row_tile=row_tile, wgrad_tile=256, tol_emul=2e-3 if low == "bf16" else par.TOL_EMUL)


def test_slab_parameter_gradient_kernel_by_contraction_length():
    # chosen without being asked for: 4 stages x 2048 rows = 8192 k
    cfg = wl.CONFIGS["cfg3"].with_(name="slabauto", B=2048, N=2)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, row_tile=64)
    emu = par.run_oracle(cfg, theta, y0, target, "emul")
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle", tol_max=par.TOL_EMUL_MAX[cfg.low])
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    small = par.run_gpu(cfg, theta, y0, target, row_tile=64, wgrad_tile=128)
    assert par.rel_err(gpu["grad_theta"], small["grad_theta"]) < 1e-5


def test_wide_kernels_running_cost_and_literal_flags():
    cfg = wl.CONFIGS["cfg3"].with_(name="widerun", B=100, N=4)
    gys = wl.normals(3, "widerun.gys", (cfg.N + 1, cfg.B, 128), 1e-7)
    _both(cfg, bias_std=0.1, row_tile=64, grad_ys=gys)
    # rounded increment + naive low-precision state (the forward pass takes the 64-row kernels)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling="none", flags=1 | 8, row_tile=64)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling="none",
                         flags=dict(round_increment=True, naive_state=True))
    for k in ("yN", "ckpt"):
        assert par.rel_err(gpu[k].reshape(emu[k].shape), emu[k]) <= par.TOL_EMUL, k


def test_cfg4_conv_shape_reduced():
    _both(wl.CONFIGS["cfg4"].with_(name="cfg4s", B=3, N=3), bias_std=0.1)


@pytest.mark.parametrize("C,H,W,B", [(96, 4, 8, 4), (8, 8, 16, 2), (70, 2, 64, 1), (8, 16, 24, 1), (16, 8, 40, 2)])
def test_conv_weight_gradient_all_taps_kernel(C, H, W, B):
    # image lines of 8 k pixels: the convolution weight gradient runs in the kernel that handles all
    # nine taps per workgroup (several channel blocks, a halo wider than the k-step, one-line images,
    # lines of 24 and 40 pixels: a k-step of 128 pixels then starts at a different column each time)
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convw{C}x{H}x{W}", B=B, N=2, C=C, H=H, W=W, tableau="kutta3")
    _both(cfg, bias_std=0.1)


@pytest.mark.parametrize("H,W,B,wgrad_tile", [(16, 16, 3, 0), (8, 64, 2, 0), (20, 32, 3, 0), (32, 32, 2, 64)])
def test_conv_weight_gradient_64_channels_transposing_reads(H, W, B, wgrad_tile):
    # 64 channels and 16 / 32 / 64 pixels per line: the weight gradient (with the bias and time-channel sums) takes
    # the kernel built on transposing LDS reads -- K-chunks that start and end inside images (20 lines per image),
    # stage boundaries inside a chunk; policy.wgrad_tile = 64 keeps the kernel that transposes in registers
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convtr{H}x{W}", B=B, N=2, C=64, H=H, W=W, tableau="kutta3")
    _both(cfg, bias_std=0.1, wgrad_tile=wgrad_tile)


def test_conv_weight_gradient_64_channels_transposing_reads_bf16():
    cfg = wl.CONFIGS["cfg4"].with_(name="convtrbf16", B=3, N=2, C=64, H=16, W=32, tableau="kutta3", low="bf16")
    # bf16 at contraction length 9 * 65: the device sums the products in fp32, the oracle in fp64 with one rounding,
    # and the two land on different sides of a bf16 rounding boundary often enough for 1e-3 (grad_y0, which no
    # weight-gradient kernel touches, is the largest: 1.9e-3); same bound as for the 512-wide bf16 networks above
    gpu, _, _ = _both(cfg, bias_std=0.1, tol_emul=2e-3)
    # the two weight-gradient kernels contract the same rounded operands: they agree to fp32 summation order
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    old = par.run_gpu(cfg, theta, y0, target, wgrad_tile=64)
    assert par.rel_err(gpu["grad_theta"], old["grad_theta"]) <= 1e-5
    np.testing.assert_array_equal(gpu["grad_y0"], old["grad_y0"])


@pytest.mark.parametrize("C,H,W,B,low", [(64, 3, 1, 5, "f16"), (24, 1, 15, 3, "f16"), (64, 14, 14, 2, "f16"), (20, 5, 17, 2, "bf16"),
                                         (24, 28, 28, 2, "f16"), (64, 2, 31, 9, "f16"), (8, 7, 33, 2, "f16"), (64, 3, 63, 2, "f16"),
                                         (32, 8, 8, 3, "f16"), (64, 8, 8, 342, "bf16")])
def test_conv_weight_gradient_ragged_image_lines(C, H, W, B, low):
    # image lines padded to 16, 32 or 64 pixels in LDS (one pixel, one less and one more than a padded line, odd pixels
    # counts per stage), against the generic contraction of the same rounded operands: fp32 summation order only
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convrag{C}x{H}x{W}", B=B, N=2, C=C, H=H, W=W, tableau="kutta3", low=low)
    gpu, _, _ = _both(cfg, bias_std=0.1, tol_emul=2e-3 if low == "bf16" else par.TOL_EMUL)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    old = par.run_gpu(cfg, theta, y0, target, wgrad_tile=64)
    assert par.rel_err(gpu["grad_theta"], old["grad_theta"]) <= 1e-5


@pytest.mark.parametrize("C,H,W,B", [(64, 5, 1, 2), (33, 9, 20, 2), (64, 30, 30, 3), (40, 70, 2, 2), (3, 15, 15, 260), (32, 3, 64, 3)])
def test_conv_tiles_of_whole_lines(C, H, W, B):
    # tiles of lines that do not fill the pixel blocks, a last tile with fewer lines, one and two wavefronts per pixel
    # block, 33 channels (two output blocks), several tiles per workgroup
    _both(wl.CONFIGS["cfg4"].with_(name=f"convtile{C}x{H}x{W}", B=B, N=1, C=C, H=H, W=W, tableau="heun"), bias_std=0.1)


@pytest.mark.parametrize("C,H,W,few,many", [(64, 32, 32, 2, 128), (24, 28, 28, 1, 128), (64, 14, 14, 2, 256), (64, 9, 64, 1, 60), (64, 32, 32, 2, 400),
                                            (32, 33, 30, 1, 90), (64, 40, 13, 2, 100)])
def test_conv_tiles_of_other_heights_give_the_same_bits(C, H, W, few, many):
    # the height of a tile follows from the number of images: from one or two lines to the most that a workgroup
    # multiplies, in one round of workgroups and in several.  A pixel's sums are the same ones in every tile, so an image's
    # trajectory and adjoint are too
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convheight{C}x{H}x{W}", B=many, N=1, C=C, H=H, W=W, tableau="heun", low="bf16", loss="half_sse")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    a = par.run_gpu(cfg, theta, y0, target)
    b = par.run_gpu(cfg.with_(B=few), theta, y0[-few:].copy(), target[-few:].copy())
    np.testing.assert_array_equal(a["yN"][-few:], b["yN"])
    np.testing.assert_array_equal(a["ckpt"][:, -few:], b["ckpt"])
    np.testing.assert_array_equal(a["grad_y0"][-few:], b["grad_y0"])


@pytest.mark.parametrize("C,H,W,B,N,low,tab,group", [(64, 24, 32, 2, 3, "bf16", "rk4", 2), (16, 13, 12, 3, 5, "f16", "heun", 0),
                                                     (40, 9, 17, 2, 4, "bf16", "euler", 3), (8, 7, 64, 1, 3, "f16", "rk4", 1),
                                                     (64, 5, 5, 2, 7, "bf16", "heun", 0)])
def test_conv_steps_in_one_launch(C, H, W, B, N, low, tab, group):
    # tiles that exchange lines (whole and cut short) and images of one tile; groups of steps that do not divide N, a group of
    # one; unequal steps; the running cost's cotangents, which go step by step
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convsteps{C}x{H}x{W}", B=B, N=N, C=C, H=H, W=W, tableau=tab, low=low)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    tgrid = _nonuniform_grid(N, seed=6)
    tol = 2e-3 if low == "bf16" else par.TOL_EMUL  # (bf16: see test_conv_weight_gradient_64_channels_transposing_reads_bf16)
    for gys in (None, wl.normals(7, "convsteps.gys", (N + 1,) + tuple(cfg.state_shape), 0.1)):
        gpu = par.run_gpu(cfg, theta, y0, target, tgrid=tgrid, step_group=group, grad_ys=gys)
        emu = par.run_oracle(cfg, theta, y0, target, "emul", tgrid=tgrid, grad_ys=None if gys is None else gys.astype(np.float64))
        par.compare(cfg, gpu, emu, tol, "emulation oracle", tol_max=par.TOL_EMUL_MAX[low])
        np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


@pytest.mark.parametrize("low,scaling", [("bf16", "none"), ("f16", "dynamic")])
def test_conv_launches_that_are_given_up(low, scaling):
    # no workgroup waits for its neighbours: the launches behind do the work again, under overflow detection the host does.
    # The same sums in the same order; in bf16 that gives the same bits.  (In f16 the compiler may round a fused
    # multiply-add to 16 bits directly in one kernel and by way of 32 bits in the other: a flipped rounding here and there,
    # 2^-11 of a value, as between the library and the oracle.)
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="convredo", B=3, N=3, C=40, H=19, W=20, tableau="rk4", low=low)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    a = par.run_gpu(cfg, theta, y0, target, scaling=scaling)
    b = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=rb.NO_WAITS)
    np.testing.assert_array_equal(a["scale_hist"], b["scale_hist"])
    for k in ("yN", "ckpt", "grad_y0", "grad_theta"):
        if low == "bf16":
            np.testing.assert_array_equal(a[k], b[k])
        assert par.rel_err(b[k], a[k]) <= par.TOL_EMUL


def _conv_pass(cfg, theta, y0, **kw):
    """A training pass on workspaces of its own -> (results, launches redone behind the forward pass and behind the
    backward pass: a word of the control block at the head of a workspace, launches of the evaluations in all)."""
    from paper_2510_23498_amd import binding as rb
    grad_ys = kw.pop("grad_ys", None)
    vel, tab, pol = par.gpu_descriptors(cfg, **kw)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    gys = None if grad_ys is None else torch.from_numpy(grad_ys).to(dev)
    ws = [rb.alloc_workspace(vel, cfg.B, cfg.N, tab, pol, b) for b in (False, True)]
    rb.rampde_timing_enable(True)
    yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol, workspace=ws[0])
    gy0, gth, info = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, yN / yN.numel(), grad_ys=gys, workspace=ws[1])
    torch.cuda.synchronize()
    launches = rb.rampde_timing_read(rb.K_VELOCITY_GEMM)[1]
    rb.rampde_timing_enable(False)
    out = dict(yN=yN, ckpt=ck.float(), grad_y0=gy0, grad_theta=gth)
    return {k: v.cpu().numpy() for k, v in out.items()}, [int(w[:64].view(torch.int32)[13]) for w in ws], launches


def _same_conv_pass(cfg, got, undisturbed, grad_theta_bits):
    # (bits: see test_conv_launches_that_are_given_up)
    for k in ("yN", "ckpt", "grad_y0", "grad_theta"):
        if cfg.low == "bf16" and (k != "grad_theta" or grad_theta_bits):
            np.testing.assert_array_equal(got[k], undisturbed[k])
        assert par.rel_err(got[k], undisturbed[k]) <= par.TOL_EMUL


@pytest.mark.parametrize("low,scaling,running_cost", [("bf16", "none", False), ("bf16", "none", True), ("f16", "none", False), ("bf16", "dynamic", False),
                                                      ("f16", "dynamic", True)])
@pytest.mark.parametrize("after", [9, 20, 26, 40, 50, 85])
def test_conv_launches_given_up_in_mid_pass(low, scaling, running_cost, after):
    # three groups of two steps, each 14 exchanges of recomputation (two rounds over the images) and 16 of the chains: given
    # up in the recomputation's second round, in both steps of a chain behind a whole recomputation, in later groups, and
    # with a running cost's cotangents (steps one by one, 7 and 8 exchanges); in the forward pass in four of its steps
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="convmid", B=3, N=6, C=40, H=19, W=20, tableau="rk4", low=low)
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    gys = (np.random.default_rng(5).standard_normal((cfg.N + 1,) + cfg.state_shape) * 0.01 / y0.size).astype(np.float32) if running_cost else None
    a, redone, launches = _conv_pass(cfg, theta, y0, scaling=scaling, step_group=2, grad_ys=gys)
    assert redone == [0, 0]
    b, redone, more = _conv_pass(cfg, theta, y0, scaling=scaling, step_group=2, grad_ys=gys, flags=rb.no_waits_after(after))
    assert redone[0] == (1 if after < 48 else 0)
    assert redone[1] >= 1 if scaling == "none" else more > launches
    _same_conv_pass(cfg, b, a, scaling == "none")


@pytest.mark.parametrize("running_cost,groups", [(False, 3), (True, 6)])
@pytest.mark.parametrize("after", [0, 9, 20, 50])
def test_conv_groups_behind_one_that_is_given_up(running_cost, groups, after):
    # only the launches that gave up are done again (0: each group's; else one): those behind them run as ever
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="convgroups", B=3, N=6, C=40, H=19, W=20, tableau="rk4", low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    gys = np.full((cfg.N + 1,) + cfg.state_shape, 0.01 / y0.size, np.float32) if running_cost else None
    _, redone, _ = _conv_pass(cfg, theta, y0, scaling="none", step_group=2, grad_ys=gys, flags=rb.no_waits_after(after))
    assert redone[1] == (1 if after else groups)


@pytest.mark.parametrize("C", [40, 21])
def test_conv_work_of_the_launches(C):
    # whole steps per launch and single evaluations alike: the recomputation leaves out a step's last slope
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="convwork", B=3, N=5, C=C, H=19, W=20, tableau="rk4", low="f16")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    rb.rampde_timing_enable(True)
    par.run_gpu(cfg, theta, y0, target, step_group=2)
    work = rb.rampde_timing_read(rb.K_VELOCITY_GEMM)[2]
    rb.rampde_timing_enable(False)
    assert work == cfg.N * (8 + 7 + 8) * 2.0 * 3 * 19 * 20 * 64 * 9 * 64


@pytest.mark.parametrize("scaling", ["dynamic", "none_safe", "none"])
def test_conv_parameter_gradients_of_a_pass_that_is_redone(scaling):
    # image lines that are no multiple of 8 pixels on the generic contraction, which adds to the caller's gradient step by
    # step: each step's share is in it once
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="convonce", B=3, N=6, C=40, H=19, W=20, tableau="rk4", low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    a, b = (_conv_pass(cfg, theta, y0, scaling=scaling, step_group=2, wgrad_tile=64, flags=flags)[0] for flags in (0, rb.no_waits_after(40)))
    np.testing.assert_array_equal(a["grad_y0"], b["grad_y0"])
    assert par.rel_err(b["grad_theta"], a["grad_theta"]) <= 1e-5  # (fp32 atomics: about 10^4 terms in any order, 2^-24 each)


@pytest.mark.parametrize("C,H,W,B,N,tab,after", [(40, 19, 20, 3, 30, "rk4", 100),   # the first of two launches of a forward pass
                                                 (40, 19, 20, 3, 30, "rk4", 200),   # ... the second
                                                 (8, 16, 64, 150, 3, "euler", 8)])  # the second of two rounds over the images
def test_conv_forward_launches_given_up_in_mid_pass(C, H, W, B, N, tab, after):
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convpieces{C}", B=B, N=N, C=C, H=H, W=W, tableau=tab, low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    a, redone, _ = _conv_pass(cfg, theta, y0, scaling="none")
    assert redone == [0, 0]
    b, redone, _ = _conv_pass(cfg, theta, y0, scaling="none", flags=rb.no_waits_after(after))
    assert redone[0] == 1
    _same_conv_pass(cfg, b, a, True)


@pytest.mark.parametrize("C,H,W,B,low,scaling", [(40, 19, 20, 3, "bf16", "none"), (64, 20, 33, 2, "f16", "dynamic"), (24, 8, 8, 3, "bf16", "dynamic"),
                                                 (16, 7, 9, 2, "f16", "none"), (21, 12, 10, 2, "bf16", "dynamic")])
def test_conv_time_weight_that_rounds_to_infinity(C, H, W, B, low, scaling):
    # a tap outside the image leaves its time weight out of the sum, also an infinite one: images of several tiles and of
    # one, kernels that run whole steps and (21 channels) single evaluations.  Bits as with a finite weight behind which
    # tanh is +-1 as well; f16: see test_conv_launches_that_are_given_up
    cfg = wl.CONFIGS["cfg4"].with_(name=f"convinf{C}x{H}x{W}", B=B, N=2, C=C, H=H, W=W, tableau="heun", low=low)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    offs = {n: o for n, _, o in wl.theta_layout(cfg)}
    tgrid = np.linspace(0.5, 1.0, 3)
    huge, large = (3.4e38, 1e38) if low == "bf16" else (1e6, 6e4)

    def with_weight(layer, value, taps=((1, 0, 0, 1.0), (3, 2, 1, -1.0), (C - 1, 1, 2, 1.0))):
        th = theta.copy()
        for co, ky, kx, sign in taps:  # (the last input channel is the time)
            th[offs[layer] + ((co * (C + 1) + C) * 3 + ky) * 3 + kx] = sign * value
        return th

    same = np.testing.assert_array_equal if low == "bf16" else lambda a, b: np.testing.assert_array_less(par.rel_err(a, b), par.TOL_EMUL)
    a, b = (par.run_gpu(cfg, with_weight("W1", v), y0, target, scaling=scaling, tgrid=tgrid) for v in (huge, large))
    for k in ("yN", "ckpt", "grad_y0", "grad_theta"):
        assert np.isfinite(b[k]).all()
        if k != "grad_theta":
            same(a[k], b[k])
    # (the redone pass deals the contraction out in other chunks: fp32 sums of about 1000 terms in another order, 2^-24 each)
    assert par.rel_err(a["grad_theta"], b["grad_theta"]) <= (1e-5 if low == "bf16" else par.TOL_EMUL)
    # behind the second convolution: +-infinity where the tap is inside, and nothing elsewhere (one step of one evaluation)
    one = cfg.with_(N=1, tableau="euler")
    a, b = (par.run_gpu(one, with_weight("W2", v), y0, target, scaling="none", tgrid=tgrid[:2]) for v in (huge, 0.0))
    inside = np.zeros((C, H, W), dtype=bool)
    inside[1, 1:, 1:] = inside[3, :-1, :] = inside[C - 1, :, :-1] = True
    assert (np.isposinf(a["yN"]) | np.isneginf(a["yN"]))[:, inside].all()
    same(a["yN"][:, ~inside], b["yN"][:, ~inside])


def test_conv_small_odd_geometry():
    cfg = wl.CONFIGS["cfg4"].with_(name="convodd", B=2, N=2, C=5, H=7, W=6, tableau="kutta3")
    _both(cfg, bias_std=0.1)


@pytest.mark.parametrize("widths,low", [((40, 250, 200, 40), "bf16"), ((64, 256, 64), "f16"), ((7, 100, 128, 128, 7), "f16")])
def test_forward_tiles_of_four_eight_and_sixteen_rows_give_the_same_bits(widths, low):
    # up to 1024 rows in tiles of 4, up to 2048 in tiles of 8 (256 compute units): the rows' sums are the same ones
    cfg = wl.CONFIGS["cfg1"].with_(name="fwdcopies", B=2049, N=2, widths=widths, low=low)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    from paper_2510_23498_amd import binding as rb
    vel, tab, pol = par.gpu_descriptors(cfg)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    yN, ckpt = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
    for B in (1, 3, 5, 17, 1023, 1024, 1025, 2047, 2048):
        print(f"[case] {widths} rows {B}", flush=True)
        part, ck = rb.rampde_odeint_fwd(vel, th, y[-B:].clone(), cfg.tgrid(), tab, pol)
        assert torch.equal(part, yN[-B:]) and torch.equal(ck, ckpt[:, -B:])


@pytest.mark.parametrize("base,widths,low,overflow", [("cfg1", (30, 600, 30), "bf16", False), ("cfg1", (64, 300, 64), "f16", False),
                                                      ("cfg1", (50, 1000, 50), "f16", True), ("cnf", (20, 900, 20), "f16", False)])
def test_one_hidden_layer_forward_tiles_give_the_same_bits(base, widths, low, overflow):
    # as above: the copies of a row in a tile share the tanh arithmetic and nothing else, so that the recomputation, which
    # has tiles of 16 rows only, forms the forward pass's stages.  An output weight that rounds to infinity makes its own
    # output infinite, at every batch size
    cfg = wl.CONFIGS[base].with_(name="fwdshallow", B=2049, N=1 if overflow else 2, widths=widths, low=low, tableau="euler" if overflow else "rk4")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    if overflow:
        theta[wl.theta_layout(cfg)[2][2] + 37] = 1e6
    from paper_2510_23498_amd import binding as rb
    vel, tab, pol = par.gpu_descriptors(cfg)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    yN, ckpt = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
    assert bool(torch.isinf(ckpt[1, :, 0]).any()) == overflow
    for B in (1, 5, 1024, 1025, 2048):
        print(f"[case] {widths} rows {B}", flush=True)
        part, ck = rb.rampde_odeint_fwd(vel, th, y[-B:].clone(), cfg.tgrid(), tab, pol)
        np.testing.assert_array_equal(part.cpu().numpy(), yN[-B:].cpu().numpy())
        np.testing.assert_array_equal(ck.float().cpu().numpy(), ckpt[:, -B:].float().cpu().numpy())


@pytest.mark.parametrize("B,low", [(3, "f16"), (1030, "bf16")])
def test_one_hidden_layer_forward_tiles_of_four_and_eight_rows(B, low):
    _both(wl.CONFIGS["cfg2"].with_(name=f"shallowrows{B}", B=B, N=2, widths=(30, 600, 30), low=low), bias_std=0.1,
          tol_emul=2e-3 if low == "bf16" else par.TOL_EMUL)


@PATHS
@pytest.mark.parametrize("tab", ["rk4", "heun", "euler"])
def test_cfg5_shape_reduced(tab, flags):
    _both(wl.CONFIGS["cfg5"].with_(name="cfg5s", B=96, N=5, tableau=tab), flags=flags)


@PATHS
def test_running_cost_cotangents(flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="run", B=64, N=4, widths=(6, 32, 6))
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gys = wl.normals(3, "run.gys", (cfg.N + 1, cfg.B, 6), 0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, grad_ys=gys, flags=flags)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", grad_ys=gys.astype(np.float64))
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")


@pytest.mark.parametrize("group", [2, 3, 64])
@pytest.mark.parametrize("low", ["bf16", "f16"])
def test_fixed_scale_runs_groups_of_steps_per_launch(group, low):
    # Without overflow detection (scaling "none") the adjoint kernel runs several steps per launch and
    # their parameter gradients are one contraction; groups of 2 / 3 (ragged last group) / all steps, ragged batch (rows padded inside the contraction), running-cost cotangents.
    # (group 3 on a 7-step grid: groups of 3, 3 and 1 steps)
    cfg = wl.CONFIGS["cfg2"].with_(name=f"grp{group}{low}", B=200, N=7 if group == 3 else 8,
                                   widths=(24, 256, 256, 24), low=low,
                                   tableau="kutta3" if group == 3 else "rk4")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gys = wl.normals(5, "grp.gys", (cfg.N + 1, cfg.B, 24), 1e-3)
    print(f"[case] {cfg.name}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling="none", grad_ys=gys, step_group=group)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling="none", grad_ys=gys.astype(np.float64))
    e = par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
    print("  vs emul:", {k: f"{v:.2e}" for k, v in e.items()}, flush=True)
    assert gpu["status"] == 0
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


# ------------------------------------------------------------------ time-grid gradient dL/dt
def _time_grid_case(cfg, scaling=None, bias_std=0.1, grad_ys=None, flags=0, step_group=0):
    theta, y0, target = par.make_inputs(cfg, bias_std=bias_std)
    print(f"[case] dL/dt {cfg.name} B={cfg.B} N={cfg.N} low={cfg.low} tab={cfg.tableau} flags={flags}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling=scaling, grad_ys=grad_ys, want_grad_t=True, flags=flags,
                      step_group=step_group)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling=scaling,
                         grad_ys=None if grad_ys is None else grad_ys.astype(np.float64))
    f64 = par.run_oracle(cfg, theta, y0, target, "f64", grad_ys=None if grad_ys is None else grad_ys.astype(np.float64))
    e_emu = par.rel_err(gpu["grad_t"], emu["grad_t"])
    e_f64 = par.rel_err(gpu["grad_t"], f64["grad_t"])
    print(f"  dL/dt vs emul {e_emu:.2e}  vs f64 {e_f64:.2e}", flush=True)
    assert e_emu <= par.TOL_EMUL, (e_emu, gpu["grad_t"], emu["grad_t"])
    assert e_f64 <= par.TOL_F64[cfg.low], e_f64
    # the other outputs are those of the plain backward pass
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])
    return gpu, emu


@PATHS
@pytest.mark.parametrize("tab", ["euler", "heun", "rk4", "kutta3"])
def test_time_grid_gradient_small_mlp_all_tableaux(tab, flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="dt" + tab, B=130, N=6, widths=(5, 40, 24, 5), tableau=tab)
    _time_grid_case(cfg, flags=flags)


@pytest.mark.parametrize("C,H,W,B,tab", [(64, 32, 32, 2, "rk4"), (64, 16, 16, 3, "heun"), (64, 4, 64, 2, "kutta3"),
                                          (5, 7, 6, 2, "kutta3"), (70, 4, 8, 4, "heun"),
                                          (70, 4, 8, 3, "heun"), (8, 16, 24, 1, "kutta3"), (24, 9, 28, 2, "rk4"), (64, 3, 33, 1, "heun")])
def test_time_grid_gradient_conv(C, H, W, B, tab):
    # both convolutions carry a time channel; all-taps weight-gradient kernel and the generic one (W = 6)
    cfg = wl.CONFIGS["cfg4"].with_(name=f"dtconv{C}x{H}x{W}", B=B, N=2, C=C, H=H, W=W, tableau=tab)
    _time_grid_case(cfg)


@pytest.mark.parametrize("kind", ["mlp", "mlp_per_layer", "conv"])
def test_time_grid_gradient_is_reproducible_bit_for_bit(kind):
    # the batch sums of dL/dt are folded from per-workgroup slots in a fixed order (no floating-point atomics): two
    # runs on the same inputs give the same bits, with hundreds of workgroups adding to every step's sums
    if kind == "conv":
        cfg = wl.CONFIGS["cfg4"].with_(name="dtrep_conv", B=4, N=3, C=64, H=32, W=32)
        flags = 0
    else:
        cfg = wl.CONFIGS["cfg2"].with_(name="dtrep_mlp", B=4000, N=4)
        flags = 4 if kind == "mlp_per_layer" else 0
    theta, y0, target = par.make_inputs(cfg)
    a = par.run_gpu(cfg, theta, y0, target, want_grad_t=True, flags=flags)
    b = par.run_gpu(cfg, theta, y0, target, want_grad_t=True, flags=flags)
    assert np.all(np.isfinite(a["grad_t"])) and np.linalg.norm(a["grad_t"]) > 0
    np.testing.assert_array_equal(a["grad_t"], b["grad_t"])


def test_time_grid_gradient_cfg1_and_running_cost():
    _time_grid_case(wl.CONFIGS["cfg1"])
    cfg = wl.CONFIGS["cfg1"].with_(name="dtrun", B=64, N=4, widths=(6, 32, 6))
    _time_grid_case(cfg, grad_ys=wl.normals(3, "dtrun.gys", (cfg.N + 1, cfg.B, 6), 0.1))


@pytest.mark.parametrize("group", [3, 64])
def test_time_grid_gradient_fixed_scale_step_groups(group):
    cfg = wl.CONFIGS["cfg2"].with_(name=f"dtgrp{group}", B=200, N=7, widths=(24, 256, 256, 24))
    _time_grid_case(cfg, scaling="none", step_group=group)


def test_time_grid_gradient_wide_and_single_layer_networks():
    _time_grid_case(wl.CONFIGS["cfg5"].with_(name="dt5", B=96, N=4))
    _time_grid_case(wl.CONFIGS["cfg3"].with_(name="dt3", B=300, N=3))
    _time_grid_case(wl.CONFIGS["cfg1"].with_(name="dtlin", B=40, N=5, widths=(12, 12)))


# ------------------------------------------------------------------ naive low-precision baseline (Table 5)
NAIVE = 8  # policy flag: state and adjoint kept in low precision (no fp32 accumulators)


@PATHS
@pytest.mark.parametrize("low", ["f16", "bf16"])
def test_naive_state_baseline_matches_oracle(low, flags):
    cfg = wl.CONFIGS["cfg1"].with_(name="naive" + low, B=70, N=12, widths=(6, 40, 6), low=low)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    print(f"[case] naive baseline {low} flags={flags}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling="none", flags=flags | NAIVE)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling="none", flags=dict(naive_state=True))
    tol = par.TOL_EMUL
    for k in ("yN", "ckpt", "grad_y0", "grad_theta"):
        e = par.rel_err(gpu[k].reshape(emu[k].shape), emu[k])
        print(f"  {k}: {e:.2e}", flush=True)
        assert e <= tol, (k, e)
    # and it is a different computation from the scheme's
    good = par.run_gpu(cfg, theta, y0, target, scaling="none", flags=flags)
    assert par.rel_err(good["yN"], gpu["yN"]) > 0


def test_fp32_accumulator_beats_naive_low_precision_state_on_the_gpu():
    # many small steps of a contractive linear problem: rounding the state after every step loses the
    # increments (paper Sec. 4 discussion of Table 5); the scheme's fp32 accumulator does not
    import torch
    from paper_2510_23498_amd import binding as rb
    from oracle import rampde_oracle as orc
    rng = np.random.default_rng(11)
    d, B, N = 8, 4, 1000
    M = rng.normal(size=(d, d))
    A = -(M @ M.T) / d
    theta = np.concatenate([A.ravel(), np.zeros(d)])
    y0 = rng.normal(size=(B, d))
    rho = np.max(np.abs(np.linalg.eigvalsh(A)))
    tg = np.arange(N + 1) * (0.5 * 2.0 / rho) * 0.05
    t = wl.TABLEAUX["euler"]
    ref = orc.odeint_fwd(orc.MLPVelocity((d, d), time_input=False, activation="identity"), theta, y0, tg, t,
                         orc.Policy(low="f64"))[0]
    dev = torch.device("cuda:0")
    vel = rb.Velocity.mlp((d, d), time_input=False)
    tab = rb.Tableau(t.A, t.b, t.c)
    th = torch.from_numpy(theta.astype(np.float32)).to(dev)
    y0d = torch.from_numpy(y0.astype(np.float32)).to(dev)
    for low in ("f16", "bf16"):
        errs = {}
        for name, fl in (("scheme", 0), ("naive", NAIVE)):
            yN, _ = rb.rampde_odeint_fwd(vel, th, y0d, tg, tab, rb.Policy(low=low, scaling="none", flags=fl))
            torch.cuda.synchronize()
            errs[name] = par.rel_err(yN.cpu().numpy(), ref)
        print(f"[case] naive vs scheme {low}: {errs}", flush=True)
        assert errs["naive"] > 10.0 * errs["scheme"], (low, errs)


# ------------------------------------------------------------------ non-uniform time grids
def _nonuniform_grid(N, t0=0.0, t1=1.0, seed=3):
    w = 0.25 + wl.normals(seed, "grid", (N,), 1.0) ** 2       # step lengths differing by up to ~20x
    return t0 + (t1 - t0) * np.concatenate([[0.0], np.cumsum(w) / np.sum(w)])


@PATHS
@pytest.mark.parametrize("low,scaling,group", [("f16", "dynamic", 0), ("bf16", "none", 64), ("bf16", "none", 3)])
def test_nonuniform_time_grid(low, scaling, group, flags):
    # every step has its own h (and, with fixed scale, the groups-of-steps contraction rescales its
    # running sums by h_i / h_{i+1} at the step boundaries); dL/dt rides along
    cfg = wl.CONFIGS["cfg2"].with_(name=f"nonuni{low}{group}", B=150, N=10, widths=(20, 256, 256, 20), low=low)
    tg = _nonuniform_grid(cfg.N)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    print(f"[case] non-uniform grid {low} {scaling} group={group} flags={flags} h in [{np.diff(tg).min():.3f}, "
          f"{np.diff(tg).max():.3f}]", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=flags, tgrid=tg, want_grad_t=True,
                      step_group=group)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling=scaling, tgrid=tg)
    e = par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
    et = par.rel_err(gpu["grad_t"], emu["grad_t"])
    print("  vs emul:", {k: f"{v:.2e}" for k, v in e.items()}, f"dL/dt {et:.2e}", flush=True)
    assert et <= par.TOL_EMUL
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


def test_nonuniform_time_grid_conv():
    cfg = wl.CONFIGS["cfg4"].with_(name="nonuniconv", B=2, N=4)
    tg = _nonuniform_grid(cfg.N, seed=4)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, tgrid=tg)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", tgrid=tg)
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


def test_fixed_scale_many_steps_default_group_length():
    # 130 steps without an environment override: groups of 64, 64 and 2 steps
    cfg = wl.CONFIGS["cfg2"].with_(name="grp130", B=48, N=130, widths=(8, 256, 256, 8), tableau="heun")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    print(f"[case] {cfg.name}", flush=True)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling="none", want_grad_t=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling="none")
    e = par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle")
    et = par.rel_err(gpu["grad_t"], emu["grad_t"])
    print("  vs emul:", {k: f"{v:.2e}" for k, v in e.items()}, f"dL/dt {et:.2e}", flush=True)
    assert et <= par.TOL_EMUL
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


@pytest.mark.parametrize("group", [1, 2, 4])
def test_slab_parameter_gradient_groups_of_steps_nonuniform_grid(group):
    # 7 steps in groups of 1, 2 and 4 (the last group is cut short at step 0); on a non-uniform grid h_i / S_i
    # differs from step to step, so the rescaling of the running sums at step boundaries is exercised
    cfg = wl.CONFIGS["cfg3"].with_(name=f"slabgrp{group}", B=100, N=7)
    tg = _nonuniform_grid(cfg.N, t1=2.0, seed=5)
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, row_tile=64, wgrad_tile=256, step_group=group, tgrid=tg, want_grad_t=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", tgrid=tg)
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle", tol_max=par.TOL_EMUL_MAX[cfg.low])
    assert par.rel_err(gpu["grad_t"], emu["grad_t"]) <= par.TOL_EMUL
    np.testing.assert_array_equal(gpu["scale_hist"].astype(np.float64), emu["scale_hist"])


@pytest.mark.parametrize("B", [4097, 8193])
def test_row_tile_rule_just_past_one_round_of_workgroups(B):
    # one row more than 256 tiles of 16 / 32 rows: 32-row tiles, and the 64-row-tile kernels under a fixed scale; the
    # last tile holds one row, and 63 rows of every stage are padding of the parameter-gradient contraction
    _both(wl.CONFIGS["cfg3"].with_(name=f"round{B}", B=B, N=1, t1=2.0 / 64, tableau="heun", low="bf16", scaling="none"))


@pytest.mark.parametrize("scaling", ["none", "dynamic"])
@pytest.mark.parametrize("widths,B,low", [
    ((7, 33, 7), 1, "f16"),                      # two layers, width 64: one row, odd state width
    ((64, 20, 64, 64), 17, "bf16"),              # three layers of 64, a tile and a row
    ((30, 65, 128, 100, 30), 70, "f16"),         # four layers of 128: the transposed slices are loaded per phase
    ((48, 129, 48), 257, "bf16"),                # two layers of 256
    ((64, 256, 130, 256, 64), 33, "f16"),        # four layers of 256
    ((16, 200, 180, 16), 4113, "f16"),           # 32-row tiles, the last one ragged, 63 rows of padding
])
def test_register_resident_kernels(widths, B, low, scaling):
    widths = widths if widths[0] == widths[-1] else widths + (widths[0],)
    # (N = 4: with h = 1/3 the fp32 values that are rounded to bf16 tie often, and the oracle's order of operations then
    # rounds 1.5 % of the cotangents the other way, 5e-4 of dL/dy_0 and up to 1.8e-3 of db_1, on every kernel path alike)
    cfg = wl.CONFIGS["cfg1"].with_(name="res" + "_".join(map(str, widths)), B=B, N=4, widths=widths, low=low,
                                   tableau="rk4", loss="mse")
    _both(cfg, bias_std=0.1, scaling=scaling)


@pytest.mark.parametrize("widths", [(64, 256, 256, 64), (64, 300, 64)])
def test_redone_pass_after_a_wait_that_ran_out(widths):
    # workgroups that do not wait for each other's words give the launch up: the step-by-step kernels redo the pass, seen
    # as their launches (one per step) beside the one that gave up; gradients are added to the caller's once
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg2"].with_(name="nowait", B=1000, N=4, low="f16", widths=widths)
    launches = {}
    for flags in (0, rb.NO_WAITS):
        rb.rampde_timing_enable(True)
        _both(cfg, bias_std=0.1, scaling="dynamic", flags=flags)
        launches[flags] = rb.rampde_timing_read(rb.K_FUSED_ADJOINT_STEP)[1]
        rb.rampde_timing_enable(False)
    assert launches == {0: 1, rb.NO_WAITS: 1 + cfg.N}


@pytest.mark.parametrize("scaling", ["none", "dynamic"])
@pytest.mark.parametrize("d,H,B,low", [(64, 257, 40, "f16"), (5, 1024, 17, "bf16"), (65, 200, 35, "f16"), (128, 512, 16, "bf16")])
def test_one_hidden_layer_kernels(d, H, B, low, scaling):
    cfg = wl.CONFIGS["cfg1"].with_(name=f"shallow{d}_{H}", B=B, N=4, widths=(d, H, d), low=low, loss="mse")
    _both(cfg, bias_std=0.1, scaling=scaling)


@pytest.mark.parametrize("widths,B,row_tile", [((128, 512, 128), 70, 64), ((128, 512, 128), 70, 32), ((64, 256, 256, 64), 70, 64),
                                               ((64, 200, 200, 64), 40, 32), ((20, 60, 20), 33, 32), ((128, 256, 128), 6964, 0)])
def test_row_tiles_of_networks_with_kernels_of_their_own(widths, B, row_tile):
    # a row tile that only the streaming kernels have, and a batch that fills their round (forward)
    cfg = wl.CONFIGS["cfg1"].with_(name=f"rows{row_tile}_" + "_".join(map(str, widths)), B=B, N=2, widths=widths, low="f16", loss="mse")
    _both(cfg, bias_std=0.1, scaling="dynamic", row_tile=row_tile)


@pytest.mark.parametrize("scaling", ["none", "dynamic"])
def test_time_grid_gradient_of_one_hidden_layer_with_row_tile_64(scaling):
    # dL/dt and everything else come from different kernels here; the workspace that the query names holds either
    cfg = wl.CONFIGS["cfg1"].with_(name="tgrid128_512", B=100, N=4, widths=(128, 512, 128), low="f16", loss="mse")
    theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
    gpu = par.run_gpu(cfg, theta, y0, target, scaling=scaling, row_tile=64, want_grad_t=True)
    emu = par.run_oracle(cfg, theta, y0, target, "emul", scaling=scaling)
    par.compare(cfg, gpu, emu, par.TOL_EMUL, "emulation oracle", tol_max=par.TOL_EMUL_MAX[cfg.low])
    assert par.rel_err(gpu["grad_t"], emu["grad_t"]) <= par.TOL_EMUL


def test_time_grid_gradient_of_more_row_tiles_than_slots():
    # a launch of the narrow-network kernels writes a slot per 16 rows; past 2^19 of them the 32-row kernels form dL/dt
    from paper_2510_23498_amd import binding as rb
    rows = 16 * (1 << 19) + 16
    cfg = wl.CONFIGS["cfg1"].with_(name="slots", B=rows, N=1, tableau="euler", low="bf16", scaling="none")
    vel, tab, pol = par.gpu_descriptors(cfg)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    theta = torch.randn(rb.rampde_num_params(vel), generator=gen, device="cuda") * 0.3
    y0 = torch.randn((rows, 2), generator=gen, device="cuda")
    gyN = torch.rand((rows, 2), generator=gen, device="cuda") * 1e-6

    def backward(sl):
        y, g = y0[sl].contiguous(), gyN[sl].contiguous()
        _, ck = rb.rampde_odeint_fwd(vel, theta, y, cfg.tgrid(), tab, pol)
        return rb.rampde_odeint_bwd_tgrid(vel, theta, cfg.tgrid(), tab, pol, ck, g)

    whole = backward(slice(0, rows))
    halves = [backward(slice(0, rows // 2)), backward(slice(rows // 2, rows))]
    # (fp32 sums of a few thousand terms per slot and of the slots, in another order: 1e-4 of sums without cancellation)
    for i, join in ((0, lambda a, b: torch.cat([a, b])), (1, torch.add), (2, torch.add)):
        ref = join(halves[0][i], halves[1][i])
        assert par.rel_err(whole[i].cpu().numpy(), ref.cpu().numpy()) <= par.TOL_EMUL


@pytest.mark.parametrize("widths,B,low,scaling,tab", [
    ((256, 1024, 1024, 256), 70, "f16", "dynamic", "rk4"),       # 32 rows per cluster, the last one ragged
    ((200, 1024, 900, 200), 513, "bf16", "none", "heun"),        # 64 rows per cluster, the last one holds one row
    ((128, 1000, 128), 33, "f16", "dynamic", "rk4"),             # one hidden layer
    ((128, 1000, 128), 1024, "bf16", "none", "euler"),           # ... at the largest batch: 64 rows per cluster
    ((200, 900, 200), 1024, "f16", "dynamic", "euler"),
    ((200, 1000, 200), 513, "f16", "dynamic", "heun"),           # ... the last cluster holds one row
    ((128, 700, 128), 700, "bf16", "none", "heun"),              # 12 workgroups per cluster; 21 row tiles of 32 run at once
    ((200, 768, 200), 1001, "f16", "dynamic", "euler"),
    ((140, 1024, 140), 1024, "bf16", "none", "euler"),           # (a state that pads to 192 columns: no cluster kernels)
    ((100, 1024, 800, 100), 1, "f16", "none_safe", "heun"),      # one row
    ((128, 512, 512, 512, 128), 1030, "f16", "dynamic", "heun"),
    ((128, 512, 400, 300, 128), 2048, "bf16", "none", "euler"),  # ... at the largest batch
    ((50, 300, 512, 50), 41, "f16", "dynamic", "rk4"),
    ((64, 512, 512, 512, 64), 1025, "bf16", "none", "euler"),
    ((256, 1024, 1024, 256), 1100, "f16", "dynamic", "euler"),   # 128 rows per cluster, the last one ends past the padding
    ((128, 1000, 1024, 128), 2048, "bf16", "none", "euler"),
    ((200, 600, 768, 200), 1025, "bf16", "none", "heun"),        # 12 workgroups per cluster
    ((128, 700, 128), 35, "f16", "dynamic", "rk4"),
    ((100, 768, 700, 100), 513, "f16", "dynamic", "euler"),
])
def test_cluster_kernels(widths, B, low, scaling, tab):
    # (as many steps as a forward pass on clusters takes at least)
    cfg = wl.CONFIGS["cfg1"].with_(name="cl" + "_".join(map(str, widths)), B=B, N={"euler": 16, "heun": 8, "rk4": 4}[tab], widths=widths,
                                   low=low, tableau=tab, loss="mse")
    # (the exchange buffers of the clusters are part of the forward workspace, and row_tile keeps to the row-tile kernels)
    from paper_2510_23498_amd import binding as rb
    size = []
    for row_tile in (0, 16):
        vel, t, pol = par.gpu_descriptors(cfg, scaling=scaling, row_tile=row_tile)
        size.append(rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, t, pol, False))
    assert (size[0] > size[1]) == (not 128 < widths[0] <= 192)
    _both(cfg, bias_std=0.1, scaling=scaling)


@pytest.mark.parametrize("widths,B", [((256, 1024, 1024, 256), 70), ((128, 512, 512, 512, 128), 1030)])
def test_cluster_launches_that_were_given_up(widths, B):
    # the row-tile kernels redo them: forward and under a fixed scale behind them on the stream, else by way of the host.
    # In bf16 the row-tile kernels agree bit for bit among themselves, but not with the clusters' order of sums
    from paper_2510_23498_amd import binding as rb
    for low, scaling in (("bf16", "none"), ("f16", "dynamic")):
        cfg = wl.CONFIGS["cfg1"].with_(name="given_up", B=B, N=5, widths=widths, low=low, loss="mse")
        theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
        got = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=rb.NO_WAITS)
        rows = par.run_gpu(cfg, theta, y0, target, scaling=scaling, row_tile=16)
        clusters = par.run_gpu(cfg, theta, y0, target, scaling=scaling)
        par.compare(cfg, got, clusters, par.TOL_EMUL, "the cluster kernels")
        par.compare(cfg, got, rows, par.TOL_EMUL, "the row-tile kernels")
        if low == "bf16":
            for key in ("yN", "ckpt", "grad_y0"):
                np.testing.assert_array_equal(got[key], rows[key])
            assert np.any(got["yN"] != clusters["yN"])


@pytest.mark.parametrize("widths,B", [((128, 512, 512, 128), 70), ((128, 700, 128), 600), ((256, 1024, 1024, 256), 1100)])
@pytest.mark.parametrize("after", [3, 10, 26])
def test_cluster_launches_given_up_in_mid_pass(widths, B, after):
    # with part of the results written: the one forward launch (28 evaluations), and of four groups of adjoint steps
    # (8, 8, 8 and 4 evaluations) the first, the second and the last one.  The forward pass is redone from y0; under a fixed
    # scale the group is redone from the adjoint that its predecessor left, under detection the whole pass
    from paper_2510_23498_amd import binding as rb
    for low, scaling in (("bf16", "none"), ("f16", "dynamic")):
        cfg = wl.CONFIGS["cfg1"].with_(name="mid_pass", B=B, N=7, widths=widths, low=low, loss="mse")
        theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
        gys = (np.random.default_rng(5).standard_normal((cfg.N + 1,) + cfg.state_shape) * 0.01 / y0.size).astype(np.float32)
        got = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=rb.no_waits_after(after), step_group=2, grad_ys=gys)
        rows = par.run_gpu(cfg, theta, y0, target, scaling=scaling, row_tile=16, grad_ys=gys)
        par.compare(cfg, got, rows, par.TOL_EMUL, "the row-tile kernels")
        np.testing.assert_array_equal(got["scale_hist"], rows["scale_hist"])
        if low == "bf16":
            for key in ("yN", "ckpt"):
                np.testing.assert_array_equal(got[key], rows[key])


@pytest.mark.parametrize("after", [5, 300, 799])
def test_later_launch_of_a_forward_pass_on_clusters_is_given_up(after):
    # 200 RK4 steps are three launches of 268 evaluations; yN holds the state between them
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg1"].with_(name="pieces", B=40, N=200, widths=(128, 512, 512, 128), low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    out = []
    for kw in (dict(flags=rb.no_waits_after(after)), dict(row_tile=16), {}):
        vel, tab, pol = par.gpu_descriptors(cfg, **kw)
        out.append(rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert not torch.equal(out[2][1], out[1][1])  # (undisturbed: another order of sums)


@pytest.mark.parametrize("widths,B,tab,N", [
    ((64, 512, 512, 64), 300, "euler", 40),      # one contraction over a long group of short steps
    ((100, 300, 300, 100), 2048, "heun", 9),     # ... of longer ones
    ((256, 700, 700, 256), 760, "rk4", 3),       # on both sides of 3e9 multiplications a step: 760 rows pad to 768, 3.02e9
    ((256, 700, 700, 256), 700, "rk4", 3),       # 704, 2.77e9
])
def test_parameter_gradients_of_groups_on_clusters(widths, B, tab, N):
    # by either kernel the same sums, in another order in 32 bits
    for low, scaling in (("bf16", "none"), ("f16", "dynamic")):
        cfg = wl.CONFIGS["cfg1"].with_(name="clgrads", B=B, N=N, widths=widths, low=low, tableau=tab, loss="mse")
        theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
        got = [par.run_gpu(cfg, theta, y0, target, scaling=scaling, wgrad_tile=t) for t in (0, 128, 256)]
        for other in got[1:]:
            np.testing.assert_array_equal(got[0]["grad_y0"], other["grad_y0"])
            assert par.rel_err(got[0]["grad_theta"], other["grad_theta"]) <= 1e-5
        rows = par.run_gpu(cfg, theta, y0, target, scaling=scaling, row_tile=16)
        par.compare(cfg, got[0], rows, par.TOL_EMUL, "the row-tile kernels")


@pytest.mark.parametrize("widths,B", [((128, 512, 512, 128), 65), ((200, 1000, 200), 33)])
@pytest.mark.parametrize("N,in_place", [(7, False), (8, False), (7, True), (8, True)])
def test_groups_of_steps_on_clusters_under_a_fixed_scale(widths, B, N, in_place):
    # the adjoint goes from group to group through two buffers in turn, an even and an odd number of them, the last group
    # short or full; running cost; dL/dy_0 in the place of dL/dy_N
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg1"].with_(name="clgroups", B=B, N=N, widths=widths, low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    gys = torch.randn(N + 1, B, widths[0], generator=torch.Generator().manual_seed(3)).to(dev)
    out = []
    for kw in (dict(step_group=2), dict(row_tile=16)):
        vel, tab, pol = par.gpu_descriptors(cfg, **kw)
        yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol)
        g = yN.clone()
        gy0, gth, _ = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, g, grad_ys=gys,
                                           grad_y0=g if in_place and "step_group" in kw else None)
        out.append((gy0.cpu().numpy(), gth.cpu().numpy()))
    for a, b in zip(*out):
        assert par.rel_err(a, b) <= par.TOL_EMUL


@pytest.mark.parametrize("widths,B", [((256, 1024, 1024, 256), 70), ((256, 1024, 1024, 256), 300), ((128, 512, 512, 512, 128), 1030)])
def test_workgroups_that_are_not_spread_evenly_over_the_dies(widths, B):
    # one XCD has more workgroups of a launch than its share, so that a cluster elsewhere has none and nobody waits for it
    # (70 rows: 3 clusters on 8 XCDs, 300 rows: 10): its rows are computed all the same, by the row-tile kernels
    from paper_2510_23498_amd import binding as rb
    for low, scaling in (("bf16", "none"), ("f16", "dynamic")):
        cfg = wl.CONFIGS["cfg1"].with_(name="skewed", B=B, N=3, widths=widths, low=low, loss="mse")
        theta, y0, target = par.make_inputs(cfg, bias_std=0.1)
        got = par.run_gpu(cfg, theta, y0, target, scaling=scaling, flags=rb.SKEWED_CLUSTERS)
        rows = par.run_gpu(cfg, theta, y0, target, scaling=scaling, row_tile=16)
        par.compare(cfg, got, rows, par.TOL_EMUL, "the row-tile kernels")
        np.testing.assert_array_equal(got["scale_hist"], rows["scale_hist"])
        if low == "bf16":
            for key in ("yN", "ckpt", "grad_y0"):
                np.testing.assert_array_equal(got[key], rows[key])


@pytest.mark.parametrize("widths,B,low,tab", [
    ((64, 256, 256, 64), 1, "f16", "rk4"), ((30, 200, 130, 256, 30), 4, "bf16", "heun"), ((7, 100, 7), 3, "f16", "euler"),
    ((64, 256, 256, 64), 5, "f16", "rk4"),  # one row more: the ordinary tile
])
def test_forward_of_a_handful_of_rows(widths, B, low, tab):
    # every row by itself gives the same bits as the batch (samples are independent, the order of sums does not depend on B)
    cfg = wl.CONFIGS["cfg1"].with_(name="few", B=B, N=5, widths=widths, low=low, tableau=tab, loss="mse")
    _both(cfg, bias_std=0.1)
    from paper_2510_23498_amd import binding as rb
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    vel, t, pol = par.gpu_descriptors(cfg)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    wide = torch.cat([y] * 5)[:17].contiguous()  # (17 rows: two ordinary tiles)
    ref, ref_ck = rb.rampde_odeint_fwd(vel, th, wide, cfg.tgrid(), t, pol)
    yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), t, pol)
    # (fp16: see test_stages_recomputed_ahead_equal_those_recomputed_inside)
    assert par.rel_err(yN.cpu().numpy(), ref[:B].cpu().numpy()) <= (1e-4 if low == "f16" else 0.0)
    assert par.rel_err(ck.float().cpu().numpy(), ref_ck[:, :B].float().cpu().numpy()) <= (2e-3 if low == "f16" else 0.0)


@pytest.mark.parametrize("C,H,W,B,low,tab", [(8, 9, 13, 3, "f16", "rk4"), (24, 28, 28, 2, "bf16", "heun"), (64, 7, 64, 2, "f16", "rk4"),
                                             (40, 16, 16, 3, "bf16", "rk4"), (20, 8, 8, 2, "f16", "rk4"), (16, 8, 16, 2, "f16", "kutta3")])
def test_stage_inputs_formed_by_the_convolution(C, H, W, B, low, tab):
    # pad channels, tiles cut short and full, rows that are not whole 16-byte groups (20 channels) and stages that are not a
    # chain (kutta3: kernels of their own form the stage inputs there); two steps, so that the update forms one too
    cfg = wl.CONFIGS["cfg4"].with_(name="stagein", C=C, H=H, W=W, B=B, N=2, t1=0.25, low=low, tableau=tab)
    _both(cfg, bias_std=0.1, scaling="dynamic" if low == "f16" else "none")


@pytest.mark.parametrize("widths,B,row_tile", [
    ((64, 600, 64), 100, 32), ((128, 256, 128), 16384, 0), ((64, 256, 256, 64), 70, 64), ((140, 300, 140), 33, 0),
    ((256, 1024, 1024, 256), 70, 0), ((128, 512, 512, 512, 128), 300, 0),  # (not by the clusters in place)
])
def test_forward_pass_in_place(widths, B, row_tile):
    # yN = y0, on exactly the queried workspace: the bits of the call out of place, on the same kernels (for the cluster
    # networks those of row tiles, which agree bit for bit among themselves in bf16)
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg1"].with_(name="in_place", B=B, N=3, widths=widths, low="bf16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    vel, tab, pol = par.gpu_descriptors(cfg, row_tile=row_tile)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    if widths[1] >= 512 and len(widths) > 3:
        ref_pol = par.gpu_descriptors(cfg, row_tile=16)[2]
    else:
        ref_pol = pol
    ref, ref_ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, ref_pol)
    got, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol, yN=y)
    assert got.data_ptr() == y.data_ptr() and torch.equal(got, ref) and torch.equal(ck, ref_ck)


@pytest.mark.parametrize("base,widths,low,tabname,N,large,B", [
    ("cfg1", (64, 512, 512, 64), "bf16", "heun", 16, 654, 588),           # no clusters; groups of steps under a fixed scale
    ("cfg1", (128, 300, 300, 300, 128), "f16", "heun", 64, 2247, 1123),   # ... under detection: a step per launch
    ("cfg1", (2, 1000, 1000, 2), "f16", "rk4", 64, 1071, 535),            # stages not recomputed ahead
    ("cfg1", (2, 128, 128, 128, 2), "f16", "heun", 64, 7558, 3779),       # adjoint of a group in one launch, slopes not kept
    ("cnf", (63, 1024, 63), "bf16", "heun", 4, 1109, 998),                # ... of a flow
])
def test_smaller_batch_on_the_workspace_of_a_larger_one(base, widths, low, tabname, N, large, B):
    # it is smaller than what the batch would take of its own: the same results (32-bit sums in another order) by the
    # kernels that need less
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS[base].with_(name="last_batch", B=B, N=N, widths=widths, low=low, tableau=tabname, loss="mse")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    vel, tab, pol = par.gpu_descriptors(cfg, scaling="dynamic" if low == "f16" else "none")
    own = [rb.alloc_workspace(vel, B, N, tab, pol, b) for b in (False, True)]
    less = [rb.alloc_workspace(vel, large, N, tab, pol, b) for b in (False, True)]
    assert less[1].numel() < own[1].numel()
    out = []
    for ws in (own, less):
        yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), tab, pol, workspace=ws[0])
        for want_t in (False, True):
            gt = torch.zeros(N + 1, device=dev) if want_t else None
            kw = {"grad_t": gt} if want_t else {}
            gy0, gth, info = rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), tab, pol, ck, yN, workspace=ws[1], **kw)
            out.append([yN, ck, gy0, gth] + ([gt] if want_t else []))
    for k in (0, 1):
        for a, b in zip(out[k], out[k + 2]):
            assert par.rel_err(a.float().cpu().numpy(), b.float().cpu().numpy()) <= par.TOL_EMUL


@pytest.mark.parametrize("C,H,W,tab,wgrad_tile,large,B", [(8, 7, 9, "kutta3", 0, 200, 190), (21, 8, 8, "rk4", 0, 200, 190),
                                                          (21, 8, 8, "heun", 64, 3, 2), (64, 8, 8, "euler", 64, 3, 2)])
def test_smaller_batch_of_images_on_the_workspace_of_a_larger_one(C, H, W, tab, wgrad_tile, large, B):
    # fewer private copies of the weight gradients, or none: the same results (32-bit sums in another order)
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="last_images", B=B, N=3, C=C, H=H, W=W, tableau=tab, low="f16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    dev = torch.device("cuda:0")
    th, y = torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev)
    vel, t, pol = par.gpu_descriptors(cfg, scaling="dynamic", wgrad_tile=wgrad_tile)
    own, less = (rb.alloc_workspace(vel, b, cfg.N, t, pol, True) for b in (B, large))
    assert less.numel() < own.numel()
    yN, ck = rb.rampde_odeint_fwd(vel, th, y, cfg.tgrid(), t, pol)
    a, b = (rb.rampde_odeint_bwd(vel, th, cfg.tgrid(), t, pol, ck, yN, workspace=ws)[:2] for ws in (own, less))
    for x, ref in zip(b, a):
        assert par.rel_err(x.cpu().numpy(), ref.cpu().numpy()) <= par.TOL_EMUL


def test_infinite_slope_that_no_stage_uses():
    # stages that do not build on one another: the second one starts from the stored state although the first one's slope
    # has left the range of 16 bits
    from paper_2510_23498_amd import binding as rb
    cfg = wl.CONFIGS["cfg4"].with_(name="apart", C=16, H=8, W=8, B=2, N=1, low="f16")
    theta, y0, _ = par.make_inputs(cfg, bias_std=0.1)
    name, shape, off = [x for x in wl.theta_layout(cfg) if x[0].startswith("b")][-1]
    theta[off:off + int(np.prod(shape))] = 7e4
    vel, _, pol = par.gpu_descriptors(cfg)
    tab = rb.Tableau([[0.0, 0.0], [0.0, 0.0]], [0.5, 0.5], [0.0, 0.5])
    dev = torch.device("cuda:0")
    yN, _ = rb.rampde_odeint_fwd(vel, torch.from_numpy(theta).to(dev), torch.from_numpy(y0).to(dev), cfg.tgrid(), tab, pol)
    assert bool(torch.isposinf(yN).all())
