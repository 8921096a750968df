"""The single-launch kernels that take groups of channels (small planes): group sizes, runs that end in a shared vector,
a last group of fewer channels, every block size, both directions -- each against the oracle and, where x holds
infinities and NaNs outside S, against the streaming kernels."""
import numpy as np
import pytest
import torch

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, NS, Workload
from parity import assert_parity, oracle_reference

pytestmark = pytest.mark.gpu


def _forced(wl, inp, variant, channels):
    opts = {"path": 2, "grouped": variant, "grouped_channels": channels}
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        res = bns.run_workload(wl, inp)
        took = (bns.bns_get_option("last_fused_forward"), bns.bns_get_option("last_fused_backward"))
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)
    return res, took


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,variant,channels", [
    ((5, 7, 2, 4), 1, 64),          # planes of one vector (bf16) or two, all channels in one group
    ((64, 20, 7, 7), 1, 8),         # whole vectors per run; the last group has 4 channels
    ((64, 19, 7, 7), 1, 3),         # runs that end in a shared vector; one channel left for the last group
    ((9, 33, 3, 3), 3, 5),          # planes of nine elements: a vector spans two channels almost everywhere
    ((40, 6, 14, 14), 5, 1),        # 512 threads, 8 vectors
    ((100, 3, 15, 13), 6, 2),       # 512 threads, 16 vectors, more rows than one pass takes
    ((1, 65, 5, 5), 4, 64),         # one sample
    ((33, 130, 4, 4), 1, 0),        # the planner's own group
])
def test_groups_of_channels(shape, variant, channels, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 3)), dict(mode=FS, patch_h=max(1, H - 1), patch_w=max(1, W // 2)),
             dict(mode=FS, patch_h=1, patch_w=W, fs_per_channel=1)]
    if N >= 4:
        modes += [dict(mode=FS, patch_h=1, patch_w=2, n_v=2, mix_beta=0.3), dict(mode=NS, n_s=1, n_v=1)]
    for i, mkw in enumerate(modes):
        wl = Workload(name="grouped", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=40 + i, sampling_seed=17, layer_id=i,
                      epoch=2, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] grouped {shape} {dtype} {mkw} variant {variant} channels {channels}", flush=True)
        res, took = _forced(wl, inp, variant, channels)
        assert took == (3, 4)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"grouped {shape} {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_what_lies_outside_s_does_not_reach_the_statistics(dtype):
    """Infinities and NaNs outside S: the statistics, and y and dx of the other elements, are those of the streaming
    kernels (which never read x outside S for them)."""
    wl = Workload(name="grouped_nan", N=12, C=21, H=7, W=7, dtype=dtype, mode=FS, patch_h=3, patch_w=4, data_seed=3,
                  sampling_seed=5, layer_id=1)
    inp = workloads.make_inputs(wl)
    box = bns.bns_sample_index(bns.make_shape(wl.N, wl.C, wl.H, wl.W), bns.make_spec(FS, 0, 3, 4, 0, 1, 0), 5)[0]
    outside = np.ones((wl.H, wl.W), dtype=bool)
    outside[box[2]:box[2] + box[3], box[4]:box[4] + box[5]] = False
    h, w = np.argwhere(outside)[0], np.argwhere(outside)[-1]
    inp["x"][:, 0::2, h[0], h[1]] = np.nan
    inp["x"][:, 1::4, w[0], w[1]] = np.inf
    got, took = _forced(wl, inp, 1, 8)
    assert took == (3, 4)
    bns.bns_set_option("path", 1)
    try:
        want = bns.run_workload(wl, inp)
    finally:
        bns.bns_set_option("path", 0)
    assert np.isfinite(got["save_mean"]).all() and np.isfinite(got["save_invstd"]).all()
    for k in ("y", "dx", "dgamma", "dbeta", "save_mean", "save_invstd"):
        assert (np.isfinite(got[k]) == np.isfinite(want[k])).all(), k
        ok = np.isfinite(want[k])
        # the same numbers up to the order of a few hundred 32-bit additions, and one rounding to 8 bits for bf16
        tol = 2e-5 if dtype == "f32" or k not in ("y", "dx") else 1e-2
        assert np.allclose(got[k][ok], want[k][ok], rtol=tol, atol=tol), k


@pytest.mark.parametrize("shape,dtype,mode,want", [
    ((62, 200, 7, 7), "f32", FULL, (False, True)),         # forward: 806 vectors in a group
    ((120, 200, 7, 7), "f32", FULL, (True, True)),         # 1560
    ((12, 600, 11, 9), "f32", FS, (False, True)),          # a patch: 900 vectors in three channels
    ((14, 600, 11, 9), "f32", FS, (True, True)),           # 1050
    ((2, 528, 10, 10), "bf16", BS, (False, False)),        # backward: 26 vectors to a channel, one wave each
    ((8, 528, 10, 10), "bf16", BS, (False, True)),         # 104
    ((21, 200, 14, 14), "f32", BS, (False, False)),        # 1029 vectors to a channel in 3.3 MB
    ((26, 200, 14, 14), "f32", BS, (False, True)),         # in 4.1 MB
    ((4, 852, 17, 17), "f32", NS, (False, True)),          # 289 lanes, but four channels: backward only
    # more blocks than compute units, 16 vectors per thread: two of them share a unit forward
    ((20, 272, 32, 32), "f32", FS, (True, True)),          # 272 blocks; backward, planes that begin on cache lines
    ((40, 272, 32, 32), "bf16", FS, (True, False)),        # bf16: a last round of 16 blocks
    ((40, 400, 32, 32), "bf16", FS, (True, True)),         # ... of 144
    ((20, 272, 28, 28), "f32", FS, (False, False)),        # planes that begin anywhere: a last round of 16 blocks
    ((20, 336, 28, 28), "f32", FS, (False, True)),         # ... of 80
    ((20, 272, 28, 28), "f32", FULL, (False, False)),      # all points: the other kernels hold a channel per block in one round
    ((34, 64, 23, 20), "bf16", FULL, (False, False)),      # few channels
    ((9, 16, 40, 40), "bf16", FULL, (False, False)),
    ((6, 130, 33, 33), "f32", FS, (False, False)),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_default_choice_on_both_sides_of_its_lines(shape, dtype, mode, want):
    """want: whether forward and backward take groups of channels."""
    N, C_, H, W = shape
    kw = dict(patch_h=max(1, H // 2), patch_w=max(1, W // 2)) if mode == FS else dict(n_s=1) if mode in (BS, NS) else {}
    wl = Workload(name="grouped_lines", N=N, C=C_, H=H, W=W, dtype=dtype, mode=mode, data_seed=45, sampling_seed=9, layer_id=3, **kw)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] grouped or not by default, {shape} {dtype} {mode}", flush=True)
    res = bns.run_workload(wl, inp)
    took = bns.bns_get_option("last_fused_forward"), bns.bns_get_option("last_fused_backward")
    assert (took[0] == 3, took[1] == 4) == want, took
    assert_parity(res, oracle_reference(wl, inp), wl, what=f"grouped or not {shape} {dtype} {mode}", inp=inp)


def test_default_choice_where_the_other_kernels_take_several_rounds():
    """Forward, planes of whole vectors: the planner turns to groups of channels when a channel per block means several
    rounds, and keeps to the other kernels when the groups would, too."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for C_, N, want in ((4 * units, 64, 3), (4 * units, 96, 1)):        # groups of four channels; of one, four rounds of blocks
        side = 14 if want == 3 else 20
        wl = Workload(name="grouped_rounds", N=N, C=C_, H=side, W=side, dtype="bf16", mode=BS, n_s=8, data_seed=44, sampling_seed=9,
                      layer_id=2)
        x = torch.randn(N, C_, side, side, device="cuda").to(torch.bfloat16)
        shape, spec = bns.make_shape(N, C_, side, side, "bf16"), bns.make_spec(BS, 8, 0, 0, 0, 2, 0)
        vec = [torch.rand(C_, device="cuda") for _ in range(6)]
        y = torch.empty_like(x)
        ws = torch.empty(bns.bns_workspace_bytes(shape, spec), dtype=torch.uint8, device="cuda")
        print(f"[gpu-case] grouped or not, {wl.shape}", flush=True)
        bns.bns_forward(shape, spec, 9, x, vec[0], vec[1], 1e-5, 0.1, y, vec[2], vec[3], vec[4], vec[5], ws)
        path, kind = bns.bns_get_option("last_path_forward"), bns.bns_get_option("last_fused_forward")
        assert (path, kind) == (2, 3) if want == 3 else path == 1
        n0 = int(bns.bns_sample_index(shape, spec, 9)[0][0])
        s = x[n0:n0 + 8].double()
        mean, var = s.mean(dim=(0, 2, 3)), s.var(dim=(0, 2, 3), unbiased=False)
        assert torch.allclose(vec[2].double(), mean, rtol=0, atol=1e-5)     # 1600 and more terms of size one: some 1e-6 in 32 bits
        want_y = (x.double() - mean[None, :, None, None]) * (vec[0].double() / torch.sqrt(var + 1e-5))[None, :, None, None]
        want_y += vec[1].double()[None, :, None, None]
        assert float((y.double() - want_y).abs().max()) <= 2 ** -8 * float(want_y.abs().max()) + 1e-3    # one rounding to 8 bits
