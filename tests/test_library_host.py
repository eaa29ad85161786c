"""Host-side checks of the C-ABI library that need no GPU: the built library loads, exports every
symbol the header declares, sizes parameters and workspaces consistently, and rejects bad
arguments before anything is launched (paper Sec. 3 / Algorithms 1-2 define the arguments:
time partition, tableau, precision and scaling policy)."""
import ctypes as C
import itertools
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_2510_23498_amd import binding as rb
from paper_2510_23498_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _header_functions():
    text = open(os.path.join(ROOT, "include", "rampde.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rampde_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = rb.load_library()
    names = _header_functions()
    assert {"rampde_odeint_fwd", "rampde_odeint_bwd", "rampde_workspace_bytes", "rampde_num_params",
            "rampde_strerror", "rampde_version"} <= set(names)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in include/rampde.h but not exported"
    assert set(rb.EXPORTS) <= set(names)
    assert rb.rampde_version() >= 100


def _descr(cfg, **kw):
    if cfg.kind == "mlp":
        vel = rb.Velocity.mlp(cfg.widths)
    elif cfg.kind == "cnf":
        vel = rb.Velocity.cnf(cfg.widths[0], cfg.widths[1])
    elif cfg.kind == "parabolic":
        vel = rb.Velocity.parabolic(cfg.C, cfg.H, cfg.W, n_intervals=cfg.n_intervals)
    else:
        vel = rb.Velocity.conv2(cfg.C, cfg.H, cfg.W)
    t = wl.TABLEAUX[cfg.tableau]
    return vel, rb.Tableau(t.A, t.b, t.c), rb.Policy(low=cfg.low, **kw)


@pytest.mark.parametrize("name", sorted(wl.CONFIGS))
def test_parameter_count_and_workspace_sizes(name):
    cfg = wl.CONFIGS[name]
    vel, tab, pol = _descr(cfg)
    assert rb.rampde_num_params(vel) == wl.n_params(cfg) == cfg.n_params
    wf = rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, pol, False)
    wb = rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, pol, True)
    assert 0 < wf < wb < 8 << 30
    # the per-layer path is a valid plan too
    pl = rb.Policy(low=cfg.low, flags=rb.PER_LAYER_KERNELS)
    assert rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, pl, True) > 0
    # with one step per launch the query is monotone in the batch size (the default plan gives the
    # parameter-gradient kernel shorter groups of steps at a larger batch, so its buffers need not grow)
    p1 = rb.Policy(low=cfg.low, step_group=1)
    assert (rb.rampde_workspace_bytes(vel, 2 * cfg.B, cfg.N, tab, p1, True)
            > rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, p1, True))


@pytest.mark.parametrize("C", [64, 20])
def test_weight_gradient_of_eight_pixel_lines_pads_only_short_contractions(C):
    # 256 images of 8 x 8: the default plan is that of wgrad_tile = 64 (conv_wgrad), not the one that pads lines to 16
    # pixels, which stays for shorter contractions; the two cut the contraction differently, so their private gradient
    # copies tell them apart
    cfg = wl.CONFIGS["cfg4"].with_(C=C, H=8, W=8)
    vel, tab, pol = _descr(cfg)
    blocks = rb.Policy(low=cfg.low, wgrad_tile=64)
    same = [rb.rampde_workspace_bytes(vel, B, cfg.N, tab, pol, True) == rb.rampde_workspace_bytes(vel, B, cfg.N, tab, blocks, True)
            for B in (128, 256, 1024)]
    assert same == [False, True, True]


@pytest.mark.parametrize("base,kw", [
    ("cfg2", dict(low="f16", B=4096, N=64)),
    ("cfg2", dict(low="f16", B=4096, N=64, widths=(128, 512, 128))),
    ("cnf", dict(B=4000, N=64)),
    ("cfg2", dict(low="f16", B=8192, N=64, widths=(64, 64, 64))),  # (the slopes that dL/dt needs are part of a step's buffers)
])
def test_workspace_of_grouped_steps_under_detection(base, kw):
    # include/rampde.h: about 1 GiB of per-step buffers (and what else a pass keeps); fewer with a smaller step_group
    cfg = wl.CONFIGS[base].with_(**kw)
    vel, tab, pol = _descr(cfg)
    size = rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, pol, True)
    assert size <= (1 << 30) + (200 << 20)
    small = rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, rb.Policy(low=cfg.low, step_group=2), True)
    assert small <= 200 << 20


@pytest.mark.parametrize("N,asked,even", [(5, 4, 3), (9, 8, 5), (7, 3, 3), (33, 0, 17)])
def test_groups_of_convolution_steps_are_even(N, asked, even):
    # the last group of a pass is no shorter than it has to be (33 steps: at most 32 at once)
    cfg = wl.CONFIGS["cfg4"].with_(C=8, H=16, W=16, B=4, N=N)
    vel, tab, _ = _descr(cfg)
    size = {g: rb.rampde_workspace_bytes(vel, cfg.B, N, tab, rb.Policy(low=cfg.low, step_group=g), True) for g in (asked, even, even - 1)}
    assert size[asked] == size[even] > size[even - 1]


@pytest.mark.parametrize("widths,B", [((256, 1024, 1024, 256), 1024), ((256, 1024, 1024, 256), 512), ((100, 1000, 1000, 100), 941),
                                      ((128, 512, 512, 512, 128), 2000), ((128, 512, 512, 128), 2048), ((100, 600, 100), 1024)])
def test_workspace_of_clusters_under_detection(widths, B):
    # include/rampde.h: about 640 MiB of per-step buffers, and what else a pass keeps
    cfg = wl.CONFIGS["cfg5"].with_(widths=widths, low="f16", B=B, N=256)
    vel, tab, pol = _descr(cfg)
    assert rb.rampde_workspace_bytes(vel, B, cfg.N, tab, pol, True) <= (640 << 20) + (120 << 20)


def test_row_tile_that_only_the_streaming_kernels_have_selects_them():
    # what tells the plans apart: the 64-row kernels keep sum_j b_j k_j of every row in the forward workspace, the
    # streaming kernels their slopes, the kernels for narrow networks and one hidden layer neither
    cfg = wl.CONFIGS["cfg2"].with_(B=4096, low="f16")

    def forward_bytes(widths, row_tile):
        vel, tab, _ = _descr(cfg.with_(widths=widths))
        return rb.rampde_workspace_bytes(vel, cfg.B, cfg.N, tab, rb.Policy(low="f16", row_tile=row_tile), False)

    wide, slopes = cfg.B * 128 * 4, 4 * cfg.B * 64 * 2
    assert forward_bytes((128, 512, 128), 64) >= forward_bytes((128, 512, 128), 0) + wide
    for widths, tiles in (((64, 256, 256, 64), (32,)), ((64, 100, 100, 64), ()), ((64, 600, 64), ())):
        auto = forward_bytes(widths, 0)
        assert forward_bytes(widths, 16) == auto
        for rows in (32, 64):
            got = forward_bytes(widths, rows)
            assert (got == auto) if rows in tiles else (got > auto + slopes // 2)


def test_forward_rule_of_one_hidden_layer_at_the_edges_of_a_round():
    # 128 -> 256 -> 128: streaming kernels (slopes in the workspace) where their tiles fill at least 85 % of the rounds
    cfg = wl.CONFIGS["cfg2"].with_(widths=(128, 256, 128))
    vel, tab, pol = _descr(cfg)
    for B, streaming in ((4096, False), (6963, False), (6964, True), (8192, True), (12000, False), (16384, True), (20000, False),
                         (60000, True)):
        assert (rb.rampde_workspace_bytes(vel, B, cfg.N, tab, pol, False) > 4 * B * 128 * 2) == streaming, B


@pytest.mark.parametrize("widths,B,ahead", [
    ((64, 512, 512, 64), 4096, True), ((64, 512, 512, 64), 7000, False), ((64, 512, 512, 64), 8192, False),
    ((128, 300, 300, 128), 8192, False), ((64, 512, 512, 512, 64), 7400, False), ((64, 512, 512, 512, 64), 8192, True),
    ((128, 512, 512, 512, 128), 6912, False), ((128, 512, 512, 512, 128), 6913, True), ((200, 256, 256, 200), 8192, True),
])
def test_recomputation_ahead_under_detection(widths, B, ahead):
    # as many buffer sets as steps are recomputed ahead: more than the one of a plan with one step per group
    cfg = wl.CONFIGS["cfg2"].with_(widths=widths, low="f16")
    vel, tab, _ = _descr(cfg)
    size = [rb.rampde_workspace_bytes(vel, B, 8, tab, rb.Policy(low="f16", step_group=g, wgrad_tile=256), True) for g in (0, 1)]
    assert (size[0] > size[1]) == ahead


@pytest.mark.parametrize("widths,B,least", [
    ((64, 512, 512, 64), 20, 4), ((64, 512, 512, 64), 1024, 6), ((64, 512, 512, 64), 1025, 16), ((128, 300, 300, 128), 2048, 11),
    ((128, 512, 512, 512, 128), 1024, 2), ((128, 512, 512, 512, 128), 2048, 6), ((128, 700, 128), 500, 4), ((128, 700, 128), 1024, 7),
    ((100, 700, 700, 100), 2048, 7), ((128, 1000, 128), 1024, 16), ((256, 1024, 1024, 256), 1024, 1), ((256, 1024, 1024, 256), 2048, 2),
])
def test_forward_passes_of_few_evaluations_are_not_on_clusters(widths, B, least):
    # the exchange buffers are part of the forward workspace; row_tile keeps to the row-tile kernels
    cfg = wl.CONFIGS["cfg1"].with_(widths=widths, tableau="euler")
    vel, tab, _ = _descr(cfg)
    for N in (1, least - 1, least, 100):
        if N < 1:
            continue
        size = [rb.rampde_workspace_bytes(vel, B, N, tab, rb.Policy(low="f16", row_tile=r), False) for r in (0, 16)]
        assert (size[0] > size[1]) == (N >= least), N


def test_checkpoint_store_is_half_of_fp32():
    # only the low-precision states are kept (paper Sec. 3): (N+1) * n * 2 bytes
    for cfg in wl.CONFIGS.values():
        vel, _, pol = _descr(cfg)
        n = int(np.prod(vel.ckpt_shape(cfg.B, cfg.N)))
        assert n == (cfg.N + 1) * cfg.B * cfg.d
        assert n * 2 * 2 == n * 4


def _call_fwd(vel, tab, pol, tgrid, B=4, theta=1, y0=1, ckpt=1, yN=1, ws=1, ws_bytes=1 << 40):
    """Call rampde_odeint_fwd with dummy non-null pointers: every case below must be rejected
    by the host-side checks, before any pointer is used."""
    lib = rb.load_library()
    tg = np.ascontiguousarray(np.asarray(tgrid, dtype=np.float64))
    pc = pol.c
    p = lambda x: C.c_void_p(int(0x1000 * x)) if x else None
    return lib.rampde_odeint_fwd(C.byref(vel.c), p(theta), p(y0), B, tg.ctypes.data_as(C.POINTER(C.c_double)),
                                 len(tg) - 1, C.byref(tab.c), C.byref(pc), p(ckpt), p(yN), p(ws), ws_bytes, None)


def test_forward_rejects_bad_arguments_without_touching_the_device():
    cfg = wl.CONFIGS["cfg1"]
    vel, tab, pol = _descr(cfg)
    grid = cfg.tgrid()
    assert _call_fwd(vel, tab, pol, grid, theta=0) == rb.EINVAL           # null pointer
    assert _call_fwd(vel, tab, pol, grid, ws=0) == rb.EINVAL
    assert _call_fwd(vel, tab, pol, grid, B=0) == rb.EINVAL
    assert _call_fwd(vel, tab, pol, grid, y0=1.001) == rb.EINVAL          # device pointer not 16-byte aligned
    assert _call_fwd(vel, tab, pol, grid, ckpt=1.002) == rb.EINVAL
    assert _call_fwd(vel, tab, pol, grid[::-1]) == rb.EINVAL              # decreasing grid
    assert _call_fwd(vel, tab, pol, [0.0, 0.5, 0.5, 1.0]) == rb.EINVAL    # not strictly increasing
    assert _call_fwd(vel, tab, pol, [0.0, np.nan, 1.0]) == rb.EINVAL
    assert _call_fwd(vel, tab, pol, [0.0]) == rb.EINVAL                   # N < 1
    bad_tab = rb.Tableau([[0.0, 0.5], [0.5, 0.0]], [0.5, 0.5], [0.0, 1.0])  # entry above the diagonal
    assert _call_fwd(vel, bad_tab, pol, grid) == rb.EINVAL
    implicit = rb.Tableau([[0.5]], [1.0], [0.5])                          # diagonal entry: implicit scheme
    assert _call_fwd(vel, implicit, pol, grid) == rb.EINVAL
    assert _call_fwd(vel, tab, rb.Policy(low="f32"), grid) == rb.EUNSUPPORTED
    nine = rb.Tableau(np.tril(np.ones((9, 9)), -1), np.ones(9) / 9, np.linspace(0, 1, 9))
    assert _call_fwd(vel, nine, pol, grid) == rb.EUNSUPPORTED             # more stages than supported
    assert _call_fwd(vel, tab, pol, grid, ws_bytes=16) == rb.EWORKSPACE   # too small
    bad_vel = rb.Velocity.mlp((4, 8, 5))                                  # output width != state width
    assert _call_fwd(bad_vel, tab, pol, grid) == rb.EINVAL
    assert rb.rampde_num_params(bad_vel) == 0
    assert rb.rampde_workspace_bytes(bad_vel, 4, 3, tab, pol, True) == 0


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="the pointers are dummies: only where no device can follow them")
def test_queried_workspace_is_enough_for_every_call_in_place_too():
    # the size that the query names is never refused: forward and backward, with yN = y0 and grad_y0 = grad_yN, over
    # widths on both sides of every choice of kernels (there is no device here: the calls end at their first launch)
    lib = rb.load_library()
    p = lambda x: C.c_void_p(0x100000 * x)
    N = 4
    tg = np.linspace(0.0, 1.0, N + 1)
    tgp = tg.ctypes.data_as(C.POINTER(C.c_double))
    for widths in ((64, 600, 64), (30, 768, 30), (2, 1024, 2), (64, 256, 64), (128, 256, 128), (128, 512, 128), (128, 1000, 128),
                   (64, 256, 256, 64), (50, 300, 512, 50), (128, 512, 512, 512, 128), (256, 1024, 1024, 256), (140, 300, 140)):
        for row_tile in (0, 16, 32, 64):
            for low, tabname in (("f16", "rk4"), ("bf16", "euler"), ("bf16", "kutta3")):
                cfg = wl.CONFIGS["cfg1"].with_(widths=widths, tableau=tabname)
                vel, tab, _ = _descr(cfg)
                pol = rb.Policy(low=low, row_tile=row_tile)
                pc = pol.c
                for B in (1, 100, 1000, 4096, 16384, 60000):
                    qf = rb.rampde_workspace_bytes(vel, B, N, tab, pol, False)
                    qb = rb.rampde_workspace_bytes(vel, B, N, tab, pol, True)
                    for yN in (4, 2):
                        rc = lib.rampde_odeint_fwd(C.byref(vel.c), p(1), p(2), B, tgp, N, C.byref(tab.c), C.byref(pc), p(3), p(yN),
                                                   p(5), qf, None)
                        assert rc == rb.EHIP, (widths, row_tile, low, tabname, B, yN, rc)
                        rc = lib.rampde_odeint_bwd(C.byref(vel.c), p(1), B, tgp, N, C.byref(tab.c), C.byref(pc), p(3), p(2), None,
                                                   p(yN), p(7), None, None, p(5), qb, None)
                        assert rc == rb.EHIP, (widths, row_tile, low, tabname, B, yN, rc)


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="the pointers are dummies: only where no device can follow them")
def test_workspace_of_a_larger_batch_serves_smaller_ones():
    # the last batch of an epoch, or inference on fewer samples: kernels that would need more than the larger batch's
    # workspace (clusters and their exchange buffers, stages of more steps at once, slopes, gradient copies) give way
    lib = rb.load_library()
    p = lambda x: C.c_void_p(0x100000 * x)

    def codes(cfg, low, N, size_f, size_b, B):
        vel, tab, _ = _descr(cfg)
        pc = rb.Policy(low=low).c
        tgp = np.linspace(0.0, 1.0, N + 1).ctypes.data_as(C.POINTER(C.c_double))
        out = [lib.rampde_odeint_fwd(C.byref(vel.c), p(1), p(2), B, tgp, N, C.byref(tab.c), C.byref(pc), p(3), p(4), p(5), size_f, None)]
        for grad_t in (None, p(9)):
            out.append(lib.rampde_odeint_bwd_tgrid(C.byref(vel.c), p(1), B, tgp, N, C.byref(tab.c), C.byref(pc), p(3), p(2), None, p(4),
                                                   p(7), grad_t, None, None, p(5), size_b, None))
        return out

    def sizes(cfg, low, N, B):
        vel, tab, _ = _descr(cfg)
        return [rb.rampde_workspace_bytes(vel, B, N, tab, rb.Policy(low=low), b) for b in (False, True)]

    for widths in ((2, 32, 2), (64, 600, 64), (128, 1000, 128), (64, 256, 256, 64), (100, 300, 300, 100),
                   (128, 512, 512, 512, 128), (200, 700, 700, 200), (256, 1024, 1024, 256)):
        for low, tabname in (("f16", "rk4"), ("bf16", "heun")):
            cfg = wl.CONFIGS["cfg1"].with_(widths=widths, tableau=tabname)
            for B in (100, 1024, 1025, 2049, 4096, 6000, 20000):
                size_f, _ = sizes(cfg, low, 16, B)
                for part in (0.95, 0.7, 0.5, 0.3, 0.1, 0.02):
                    small = max(1, int(B * part))
                    assert codes(cfg, low, 16, size_f, 1 << 40, small) == [rb.EHIP] * 3, (widths, low, B, small)
    for base, widths, low, tabname, N, B, small in (
            ("cfg1", (64, 512, 512, 64), "bf16", "heun", 16, 654, 588), ("cfg1", (128, 300, 300, 300, 128), "f16", "heun", 64, 2247, 1123),
            ("cfg1", (2, 1000, 1000, 2), "f16", "rk4", 64, 1071, 535), ("cfg1", (2, 128, 128, 128, 2), "f16", "heun", 64, 7558, 3779),
            ("cfg1", (256, 1000, 1000, 256), "f16", "heun", 16, 15439, 1543), ("cnf", (63, 1024, 63), "bf16", "heun", 4, 1109, 998)):
        cfg = wl.CONFIGS[base].with_(widths=widths, tableau=tabname)
        size_f, size_b = sizes(cfg, low, N, B)
        assert size_b < sizes(cfg, low, N, small)[1]  # (what the smaller batch would take of a workspace of its own)
        assert codes(cfg, low, N, size_f, size_b, small) == [rb.EHIP] * 3, (widths, low, B, small)


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="the pointers are dummies: only where no device can follow them")
@pytest.mark.parametrize("shape", [(8, 7, 9), (21, 8, 8), (24, 28, 28), (64, 32, 32), (64, 8, 8), (32, 5, 70), (128, 16, 16)])
def test_workspace_of_a_larger_batch_of_images_serves_smaller_ones(shape):
    # (fewer chunks of a larger batch's weight-gradient contraction, or none where its pixels do not divide)
    lib = rb.load_library()
    p = lambda x: C.c_void_p(0x100000 * x)
    for tabname, N, wgrad_tile, scaling in itertools.product(("euler", "rk4", "kutta3"), (1, 5, 33), (0, 64), ("none", "dynamic")):
        cfg = wl.CONFIGS["cfg4"].with_(C=shape[0], H=shape[1], W=shape[2], tableau=tabname)
        vel, tab, _ = _descr(cfg)
        pol = rb.Policy(low="f16", scaling=scaling, wgrad_tile=wgrad_tile)
        tgp = np.linspace(0.0, 1.0, N + 1).ctypes.data_as(C.POINTER(C.c_double))
        for B in (1, 3, 20, 200):
            size = [rb.rampde_workspace_bytes(vel, B, N, tab, pol, b) for b in (False, True)]
            for part in (1.0, 0.99, 0.95, 0.7, 0.5, 0.02):
                small = max(1, int(B * part))
                for yN in (4, 2):  # (not in place and in place)
                    rc = [lib.rampde_odeint_fwd(C.byref(vel.c), p(1), p(2), small, tgp, N, C.byref(tab.c), C.byref(pol.c), p(3), p(yN), p(5),
                                                size[0], None)]
                    for grad_t in (None, p(9)):
                        rc.append(lib.rampde_odeint_bwd_tgrid(C.byref(vel.c), p(1), small, tgp, N, C.byref(tab.c), C.byref(pol.c), p(3), p(2),
                                                              None, p(yN), p(7), grad_t, None, None, p(5), size[1], None))
                    assert rc == [rb.EHIP] * 3, (tabname, N, wgrad_tile, scaling, B, small, yN, rc)


def test_backward_rejects_bad_arguments_without_touching_the_device():
    lib = rb.load_library()
    cfg = wl.CONFIGS["cfg1"]
    vel, tab, pol = _descr(cfg)
    tg = np.ascontiguousarray(cfg.tgrid())
    pc = pol.c
    p = lambda x: C.c_void_p(int(0x1000 * x)) if x else None

    def call(theta=1, ckpt=1, gyN=1, gy0=1, gth=1, ws=1, ws_bytes=1 << 40, N=cfg.N, B=4, pc=pc):
        return lib.rampde_odeint_bwd(C.byref(vel.c), p(theta), B, tg.ctypes.data_as(C.POINTER(C.c_double)), N,
                                     C.byref(tab.c), C.byref(pc), p(ckpt), p(gyN), None, p(gy0), p(gth), None, None,
                                     p(ws), ws_bytes, None)

    assert call(theta=0) == rb.EINVAL
    assert call(ckpt=0) == rb.EINVAL
    assert call(gth=0) == rb.EINVAL
    assert call(N=0) == rb.EINVAL
    assert call(ws_bytes=64) == rb.EWORKSPACE
    assert call(gyN=1.001) == rb.EINVAL                                   # not 16-byte aligned
    assert call(gy0=1.003) == rb.EINVAL
    # scale groups: negative size; a group whose slice of the buffers would not start 16-byte aligned
    # (cfg1 has 2 state elements per sample: 3 samples are 6 elements)
    assert call(B=8, pc=rb.Policy(low="f16", scaling="dynamic", scale_group=-1).c) == rb.EINVAL
    assert call(B=8, pc=rb.Policy(low="f16", scaling="dynamic", scale_group=3).c) == rb.EINVAL


def test_error_strings():
    for code in (rb.OK, rb.EINVAL, rb.EUNSUPPORTED, rb.EWORKSPACE, rb.ESCALE, rb.EHIP, 99):
        msg = rb.rampde_strerror(code)
        assert isinstance(msg, str) and msg
    assert "scaling" in rb.rampde_strerror(rb.ESCALE)


def test_timing_interface_rejects_bad_class():
    lib = rb.load_library()
    assert lib.rampde_timing_read(99, None) == rb.EINVAL


def test_bench_refuses_more_than_one_gpu():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode != 0
    assert "ONE GPU" in res.stderr
