"""The single-launch kernels of one block per compute unit (large N x C x H x W tensors), forced on small ones: teams of one and
of several blocks, one round and more, shares that end in the middle of a block's vectors, more sampled vectors per thread
than the on-chip store holds, planes and rows that are no whole number of vectors -- against the oracle."""
import numpy as np
import pytest
import torch

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, NS, Workload
from parity import assert_parity, oracle_reference

pytestmark = pytest.mark.gpu


def _forced(wl, inp, resident, again=False):
    opts = {"path": 2, "grouped": 2, "resident": resident}
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        res = bns.run_workload(wl, inp)
        took = (bns.bns_get_option("last_fused_forward"), bns.bns_get_option("last_fused_backward"))
        return res, took, bns.run_workload(wl, inp) if again else None
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)


# resident: 3 dy alone stays on chip, 4 x beside it
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 1, 2, 4),               # a plane of one vector (bf16) or two; hardly a thread with work
    (2, 300, 4, 4),             # more channels than blocks: two rounds of teams of one
    (32, 4, 28, 28),            # bf16: 3136 vectors, 7 of 49 per thread
    (64, 3, 56, 56),            # bf16: 49 vectors per thread to the last; fp32: two blocks
    (65, 2, 56, 56),            # one sample more: another block per team, its share mostly empty
    (40, 130, 56, 56),          # several rounds of teams
    (33, 5, 45, 47),            # planes and rows of odd length
    (50, 3, 30, 30),            # bf16: planes of 112.5 vectors; rows that cross vectors in both types
    (3, 2, 112, 112),
], ids=lambda s: "x".join(map(str, s)))
def test_resident_kernels(shape, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 8)), dict(mode=NS, n_s=max(1, N - 1)),
             dict(mode=FS, patch_h=max(1, H // 4), patch_w=max(1, W // 4)),
             dict(mode=FS, patch_h=H, patch_w=max(1, W // 6), fs_per_channel=1), dict(mode=FS, patch_h=1, patch_w=W)]
    if N * C_ * H * W > 10000000:
        modes = modes[1::2]
    if N >= 4:
        modes.append(dict(mode=FS, patch_h=max(1, H // 4), patch_w=max(1, W // 4), n_v=2, mix_beta=0.3))
    for i, mkw in enumerate(modes):
        wl = Workload(name="resident", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=90 + i, sampling_seed=23, layer_id=i, epoch=4,
                      **mkw)
        inp = workloads.make_inputs(wl)
        ref = oracle_reference(wl, inp)
        for resident in (3, 4):
            print(f"[gpu-case] resident {shape} {dtype} {mkw} {resident}", flush=True)
            res, took, again = _forced(wl, inp, resident, again=True)
            assert took[1] == 5 and (wl.n_v or took[0] == 4)
            assert_parity(res, ref, wl, what=f"resident {resident} {shape} {dtype} {mkw}", inp=inp)
            for k in res:
                assert (res[k] == again[k]).all(), f"{k}: not bit-identical from run to run"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hw", [(14, 16), (15, 13)])
def test_what_lies_outside_s_does_not_reach_the_statistics(dtype, hw):
    """Infinities and NaNs outside S: the statistics and y on S are those of the streaming kernels."""
    H, W = hw
    wl = Workload(name="resident_nan", N=30, C=9, H=H, W=W, dtype=dtype, mode=FS, patch_h=3, patch_w=4, data_seed=3,
                  sampling_seed=5, layer_id=1)
    inp = workloads.make_inputs(wl)
    outs = []
    for opts in ({"path": 1}, {"path": 2, "grouped": 2, "resident": 3}):
        b = bns.Buffers(wl, inp)
        box = bns.bns_sample_index(b.shape, b.spec, b.seed)[0]
        inside = torch.zeros(H, W, dtype=torch.bool, device=b.x.device)
        inside[box[2]:box[2] + box[3], box[4]:box[4] + box[5]] = True
        b.x[:, :, ~inside] = float("nan")
        b.x[0, :, ~inside] = float("inf")
        try:
            for k, v in opts.items():
                bns.bns_set_option(k, v)
            b.forward()
        finally:
            for k in opts:
                bns.bns_set_option(k, 0)
        outs.append((b.results(), inside.cpu().numpy()))
    (want, inside), (got, _) = outs
    for k in ("save_mean", "save_invstd", "running_mean", "running_var"):
        assert np.isfinite(got[k]).all()
        assert np.allclose(got[k], want[k], rtol=1e-5, atol=1e-6), k
    tol = 1e-5 if dtype == "f32" else 1e-2
    assert np.allclose(got["y"][:, :, inside], want["y"][:, :, inside], rtol=tol, atol=tol)
    assert not np.isfinite(got["y"][:, :, ~inside]).any()


def test_a_team_mate_that_never_publishes_ends_in_nan():
    wl = Workload(name="resident_mute", N=40, C=6, H=56, W=56, dtype="f32", mode=BS, n_s=4, data_seed=8, sampling_seed=1)
    inp = workloads.make_inputs(wl)
    opts = {"path": 2, "resident": 4, "test_mute_exchange": 1, "test_spin_limit": 64}
    b = bns.Buffers(wl, inp)
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        b.backward()
        res = b.results()
        assert bns.bns_get_option("last_fused_backward") == 5
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)
    assert np.isnan(res["dbeta"]).all() and np.isnan(res["dgamma"]).all()
    assert bns.bns_expired_waits(b.workspace) > 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_team_mate_that_never_publishes_leaves_the_moving_averages_alone(dtype):
    wl = Workload(name="resident_mute_forward", N=90, C=6, H=56, W=56, dtype=dtype, mode=BS, n_s=4, data_seed=8, sampling_seed=1)
    inp = workloads.make_inputs(wl)
    opts = {"path": 2, "resident": 1, "test_mute_exchange": 1, "test_spin_limit": 64}
    b = bns.Buffers(wl, inp)
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        b.forward()
        res = b.results()
        assert bns.bns_get_option("last_fused_forward") == 4
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)
    assert np.isnan(res["save_mean"]).all() and np.isnan(res["save_invstd"]).all() and np.isnan(res["y"]).all()
    assert (res["running_mean"] == inp["running_mean"]).all() and (res["running_var"] == inp["running_var"]).all()
    assert bns.bns_expired_waits(b.workspace) > 0
