"""Which of the single-launch N x C x H x W kernels a call takes, on both sides of the planner's lines; each call against the oracle."""
import pytest
import torch

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, Workload
from parity import assert_parity, oracle_reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,dtype,opts,took", [
    # (512, 16) blocks of whole vectors that read patch elements on their own: a second one on a unit where one does not hold all channels
    ((2, 240, 108, 108), "f32", {}, (2, 1)),
    ((2, 288, 108, 108), "f32", {}, (2, 1)),
    ((2, 520, 108, 108), "f32", {}, (1, None)),             # nor do two
    ((52, 384, 20, 20), "f32", {}, (2, 3)),                 # groups of channels come before two
    ((2, 288, 107, 107), "f32", {}, (1, None)),             # element-aligned vectors take one
    # 265 members of eight vectors per thread: more than one per unit, all the same
    ((65, 1, 259, 257), "f32", {"path": 2, "fused_variant": 4}, (2, 1)),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) and len(v) == 4 else None)
def test_blocks_per_unit_of_a_patch(shape, dtype, opts, took):
    N, C_, H, W = shape
    wl = Workload(name="patch_blocks", N=N, C=C_, H=H, W=W, dtype=dtype, mode=FS, patch_h=H // 2, patch_w=W // 3, data_seed=95, sampling_seed=25,
                  layer_id=8)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] blocks per unit of a patch {shape} {dtype} {opts}", flush=True)
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        res = bns.run_workload(wl, inp)
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)
    assert bns.bns_get_option("last_path_forward") == took[0]
    assert took[1] is None or bns.bns_get_option("last_fused_forward") == took[1]
    assert_parity(res, oracle_reference(wl, inp), wl, what=f"blocks per unit {shape}", inp=inp)


# (kernel, block size, blocks that share a channel) forward and backward; kernels as in "last_fused_forward" / "last_fused_backward", block sizes as in
# "fused_variant" (0: kernels that have none); None: not looked at.  For 256 compute units.
@pytest.mark.parametrize("shape,dtype,mode,forward,backward", [
    # teams of (512, 8) blocks, if there is one for every second unit: 2 x 64 of them, 6 x 24; not 3 x 24, 2 x 16
    ((34, 64, 23, 20), "bf16", FULL, (1, 4, 2), (2, 4, 2)),
    ((24, 24, 48, 48), "f32", BS, (1, 4, 6), (1, 4, 6)),
    ((12, 24, 48, 48), "f32", BS, (1, 2, 27), (1, 2, 27)),
    ((9, 16, 64, 64), "bf16", FULL, (1, 2, 18), (2, 2, 18)),
    ((9, 16, 40, 40), "bf16", FULL, (1, 4, 1), (2, 4, 1)),     # one block that holds its channel comes first
    # teams of small blocks, more than four to a unit: 22 x 46 of 128 threads are not, 22 x 48 are
    ((7, 46, 56, 56), "f32", BS, (1, 2, 22), (1, 2, 22)),
    ((7, 48, 56, 56), "f32", BS, (1, 3, 6), (1, 3, 6)),
    # a patch, one block per unit: 130 blocks of element-aligned vectors, 256 of twice as many
    ((6, 130, 33, 33), "f32", FS, (1, 4, 1), (2, 4, 2)),
    ((3, 256, 86, 84), "f32", FS, (1, 5, 1), (2, 4, 2)),
    # the pipelined kernel from 800 vectors to a channel on (here 720 and 1008, 768 and 896); not for 10
    ((5, 1264, 24, 24), "f32", BS, None, (4, 0, 1)),
    ((7, 1264, 24, 24), "f32", BS, None, (3, 0, None)),
    ((6, 1264, 32, 32), "bf16", BS, None, (4, 0, 1)),
    ((7, 1264, 32, 32), "bf16", BS, None, (3, 0, None)),
    ((5, 1808, 4, 4), "bf16", BS, (1, 1, 1), (1, 1, 1)),
    # so many blocks of groups that those come before one small block per channel
    ((48, 816, 10, 10), "bf16", FULL, (3, 0, 1), (4, 0, 1)),
    ((26, 1584, 12, 12), "bf16", BS, (3, 0, 1), (4, 0, 1)),    # 1584 channels in 12 MB
    ((13, 1584, 12, 12), "bf16", BS, (1, 2, 1), (4, 0, 1)),    # in 6 MB
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) and len(v) == 4 else None)
def test_block_size_and_team(shape, dtype, mode, forward, backward):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expected choices are those of 256 compute units")
    N, C_, H, W = shape
    kw = dict(patch_h=H // 2, patch_w=W // 2) if mode == FS else dict(n_s=1) if mode == BS else {}
    wl = Workload(name="choice", N=N, C=C_, H=H, W=W, dtype=dtype, mode=mode, data_seed=96, sampling_seed=26, layer_id=9, **kw)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] block size and team {shape} {dtype} {mode}", flush=True)
    res = bns.run_workload(wl, inp)
    for direction, want in (("forward", forward), ("backward", backward)):
        if want is not None:
            got = tuple(bns.bns_get_option(f"last_{what}_{direction}") for what in ("fused", "variant", "team"))
            assert bns.bns_get_option(f"last_path_{direction}") == 2
            assert got[:2] == want[:2] and want[2] in (None, got[2]), (direction, got)
    assert_parity(res, oracle_reference(wl, inp), wl, what=f"block size and team {shape} {dtype} {mode}", inp=inp)
