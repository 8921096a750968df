"""Planes that are no whole number of vectors, in the streaming kernels and in the single-launch kernels of every block
size: planes of a vector and a few elements, one row, long odd planes; the last vector of a plane is shared with the one
before it and must count once.  And the kernels that such planes get by default, on both sides of each line of the rule."""
import numpy as np
import pytest

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, NS, Workload
from parity import assert_parity, oracle_reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(5, 6, 3, 3), (7, 5, 1, 11), (3, 9, 5, 3), (12, 20, 2, 6), (9, 70, 13, 15), (20, 3, 45, 47),
                                   (2, 65, 31, 1), (33, 40, 10, 10)], ids=lambda s: "x".join(map(str, s)))
def test_odd_planes(shape, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 2)), dict(mode=FS, patch_h=max(1, H // 2), patch_w=max(1, W - 1)),
             dict(mode=FS, patch_h=1, patch_w=1, fs_per_channel=1)]
    if N >= 3:
        modes.append(dict(mode=NS, n_s=1, n_v=2, mix_beta=0.4))
    for i, mkw in enumerate(modes):
        wl = Workload(name="odd", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=70 + i, sampling_seed=19, layer_id=i, epoch=3, **mkw)
        inp = workloads.make_inputs(wl)
        ref = oracle_reference(wl, inp)
        for opts in ({"path": 1}, {"path": 1, "split_statistics": 1, "splits_reduce": 3, "norm_unroll": 4, "dx_unroll": 4},
                     {"grouped": 2}, {"path": 2, "fused_variant": 2}, {"path": 2, "fused_variant": 4},
                     {"path": 2, "fused_variant": 4, "fused_keep_x": 1}, {"path": 2, "fused_variant": 7}):
            print(f"[gpu-case] odd planes {shape} {dtype} {mkw} {opts}", flush=True)
            try:
                for k, v in opts.items():
                    bns.bns_set_option(k, v)
                res = bns.run_workload(wl, inp)
            except bns.BnsError as e:               # a variant that is not built for Eq. 4
                assert e.status == bns.BNS_EUNSUPPORTED and opts.get("path") == 2 and "n_v" in mkw
                continue
            finally:
                for k in opts:
                    bns.bns_set_option(k, 0)
            assert_parity(res, ref, wl, what=f"odd {shape} {dtype} {mkw} {opts}", inp=inp)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 5, 45, 45),                 # 2025 elements per channel: one element per access
    (1, 5, 29, 71),                 # 2059: vectors, one block
    (1, 1100, 47, 47),              # more channels than (512, 8) blocks fit at once
    (7, 20, 61, 61),                # teams of (512, 8) blocks
    (2, 600, 67, 67),               # several rounds of them
    (2, 530, 45, 45),               # fp32: 4050 elements per channel, more channels than blocks of vectors at once
    (12, 3, 101, 99),               # few channels: the default's share of a block in bf16
], ids=lambda s: "x".join(map(str, s)))
def test_default_kernels_for_odd_planes(shape, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 2)), dict(mode=FS, patch_h=max(1, H // 3), patch_w=max(1, W // 2))]
    if N >= 3:
        modes.append(dict(mode=FS, patch_h=2, patch_w=3, n_v=2, mix_beta=0.4))
    for i, mkw in enumerate(modes):
        wl = Workload(name="odd_default", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=75 + i, sampling_seed=20, layer_id=i, epoch=1,
                      **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] odd planes, default kernels {shape} {dtype} {mkw}", flush=True)
        res = bns.run_workload(wl, inp)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"odd, default {shape} {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("shape,dtype", [
    ((3, 100, 41, 42), "f32"),      # 2.07 MB, below the line of the streaming passes: one element per access
    ((3, 100, 43, 45), "f32"),      # 2.3 MB: vectors
    ((5, 100, 45, 47), "bf16"),     # 2.1 MB, vectors of eight
    ((9, 139, 58, 58), "bf16"),     # 8.4 MB and planes of 420.5 vectors: eight elements, below the line (64-bit accesses) four
    ((9, 138, 58, 58), "bf16"),
    ((60, 95, 3, 63), "f32"),       # 4.3 MB, vectors in the reduction, too; 47.25 of them per plane
], ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else s)
def test_odd_planes_in_the_streaming_kernels(shape, dtype):
    N, C_, H, W = shape
    for i, mkw in enumerate((dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 3)), dict(mode=FS, patch_h=H // 2, patch_w=W // 2),
                             dict(mode=FS, patch_h=2, patch_w=2, n_v=1, mix_beta=0.3))):
        wl = Workload(name="odd_streaming", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=80 + i, sampling_seed=21, layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        ref = oracle_reference(wl, inp)
        for opts in ({"path": 1}, {"path": 1, "split_statistics": 1, "splits_reduce": 3, "norm_unroll": 4, "dx_unroll": 4}):
            print(f"[gpu-case] odd planes, streaming {shape} {dtype} {mkw} {opts}", flush=True)
            try:
                for k, v in opts.items():
                    bns.bns_set_option(k, v)
                res = bns.run_workload(wl, inp)
            finally:
                for k in opts:
                    bns.bns_set_option(k, 0)
            assert_parity(res, ref, wl, what=f"odd, streaming {shape} {dtype} {mkw} {opts}", inp=inp)


def test_odd_planes_in_the_bf16_reduction():
    """34 MB: the sums of Eq. 5 from vectors of eight elements."""
    wl = Workload(name="odd_reduce", N=17, C=100, H=99, W=101, dtype="bf16", mode=BS, n_s=4, data_seed=86, sampling_seed=22, layer_id=5)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] odd planes, streaming reduction {wl.shape} bf16", flush=True)
    bns.bns_set_option("path", 1)
    try:
        res = bns.run_workload(wl, inp)
    finally:
        bns.bns_set_option("path", 0)
    assert_parity(res, oracle_reference(wl, inp), wl, what="odd, bf16 reduction", inp=inp)


@pytest.mark.parametrize("shape,mkw", [((57, 144, 31, 31), dict(mode=FS, patch_h=7, patch_w=7)),
                                       ((9, 848, 23, 23), dict(mode=BS, n_s=2))], ids=["streaming_statistics", "single_launch"])
def test_odd_planes_lose_no_precision_by_fewer_blocks(shape, mkw):
    """Error of the mean over all channels.  One rounding to fp32 is 3.4e-8 of a value (2^-24 / sqrt(3)); the sums within a wave
    add about as much again.  Adding the waves in fp32 made it 1.4e-7 and 1.2e-7."""
    N, C_, H, W = shape
    wl = Workload(name="odd_mean", N=N, C=C_, H=H, W=W, dtype="f32", data_seed=90, sampling_seed=23, layer_id=6, **mkw)
    inp = workloads.make_inputs(wl)
    rng = np.random.default_rng(91)
    mu, sigma = rng.uniform(-1, 1, (1, C_, 1, 1)), rng.uniform(0.5, 2, (1, C_, 1, 1))
    inp["x"] = (rng.standard_normal(shape) * sigma + mu).astype(inp["x"].dtype)
    ref = oracle_reference(wl, inp)
    print(f"[gpu-case] odd planes, error of the mean {shape} {mkw}", flush=True)
    res = bns.run_workload(wl, inp)
    assert_parity(res, ref, wl, what=f"odd, mean {shape}", inp=inp)
    got, want = res["save_mean"].astype(np.float64), ref["save_mean"]
    error = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"error of the mean {error:.2e}", flush=True)
    assert error < 8e-8
