"""Which of the single-launch N x C x H x W kernels a call takes, on both sides of the planner's lines; each call against the oracle."""
import pytest

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import FS, Workload
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
