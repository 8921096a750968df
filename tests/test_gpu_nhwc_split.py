"""The N x H x W x C backward whose reduction goes through the rows front to back and writes dx outside S as it goes, forced on small
tensors: less than a chunk of rows, a chunk and a row, several chunks per block, idle column lanes, several column tiles, S at
either end, in runs, and all rows."""
import numpy as np
import pytest

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, NS, VDN, Workload
from parity import assert_parity, oracle_boxes, oracle_reference

pytestmark = pytest.mark.gpu


def _run(wl, inp, **options):
    try:
        for k, v in options.items():
            bns.bns_set_option(k, v)
        res = bns.run_workload(wl, inp)
        return res, bns.bns_get_option("last_path_backward")
    finally:
        for k in options:
            bns.bns_set_option(k, 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,blocks", [
    ((2, 8, 1, 1), 0),              # two rows
    ((5, 256, 4, 4), 1),            # 80 rows: five chunks (f32), walked by one block
    ((3, 64, 11, 31), 2),           # 1023 rows: the last chunk one row short
    ((5, 64, 5, 41), 2),            # 1025 rows: a chunk of one row
    ((9, 40, 13, 17), 3),           # idle lanes, odd count of chunks per block
    ((7, 520, 9, 9), 0),            # f32: three column tiles, the last with two lanes at work; bf16: two, the last with one
    ((40, 16, 30, 30), 8192),       # more blocks asked for than chunks
], ids=str)
def test_backward_front_to_back(shape, blocks, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 4)), dict(mode=NS, n_s=N - 1), dict(mode=VDN, n_s=1),
             dict(mode=FS, patch_h=max(1, H // 2), patch_w=max(1, W // 3)), dict(mode=FS, patch_h=1, patch_w=W)]
    for i, mkw in enumerate(modes):
        wl = Workload(name="split", N=N, C=C_, H=H, W=W, dtype=dtype, layout="nhwc", data_seed=70 + i, sampling_seed=11, layer_id=i,
                      epoch=2, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] front to back {shape} {dtype} {mkw}", flush=True)
        res, path = _run(wl, inp, nhwc_fused=2, nhwc_split_ordered=1, nhwc_blocks=blocks)
        assert path == 4
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"front to back {shape} {dtype} {mkw}", inp=inp)
        stages, path = _run(wl, inp, path=1, nhwc_fused=2, nhwc_blocks=blocks)
        assert path == 1
        # Eq. 6 outside S has no sum in it: there the bits are those of the one-kernel dx pass
        b = oracle_boxes(wl)[0]
        outside = np.ones((N, 1, H, W), bool)
        outside[b[0]:b[0] + b[1], :, b[2]:b[2] + b[3], b[4]:b[4] + b[5]] = False
        outside = np.broadcast_to(outside, (N, C_, H, W))
        assert (res["dx"][outside] == stages["dx"][outside]).all()


@pytest.mark.parametrize("kw,want", [
    (dict(N=32, C=256, H=28, W=28, n_s=8), 4),          # a quarter of the rows, 26 MB
    (dict(N=32, C=256, H=28, W=28, n_s=9), 1),          # more of them
    (dict(N=32, C=200, H=32, W=28, n_s=8), 1),          # 50 of 64 lanes
    (dict(N=32, C=256, H=16, W=28, n_s=8), 1),          # 15 MB
    (dict(N=32, C=150, H=40, W=40, n_s=8), 1),          # no 16-byte accesses
])
def test_rule_of_the_default(kw, want):
    wl = Workload(name="split_rule", mode=BS, dtype="f32", layout="nhwc", data_seed=7, sampling_seed=8, layer_id=1, **kw)
    inp = workloads.make_inputs(wl)
    assert _run(wl, inp, nhwc_fused=2)[1] == want
    assert _run(wl, inp, nhwc_fused=2, nhwc_split_ordered=2)[1] == 1 and _run(wl, inp, nhwc_fused=2, nhwc_split_dx=2)[1] == 1
    assert _run(wl, inp, path=1)[1] == 1


@pytest.mark.parametrize("kw,want", [
    (dict(C=1024, dtype="f32", mode=BS, n_s=8), 4),                             # four column tiles of 64 lanes
    (dict(C=1024, dtype="f32", mode=FS, patch_h=7, patch_w=7), 4),
    (dict(C=768, dtype="f32", mode=BS, n_s=8), 4),                              # three, no lane idle, S contiguous
    (dict(C=768, dtype="f32", mode=FS, patch_h=7, patch_w=7), 1),
    (dict(C=736, dtype="f32", mode=BS, n_s=8), 1),                              # 184 of 192 lanes
    (dict(C=1536, dtype="bf16", mode=BS, n_s=8), 1),
    (dict(C=2048, dtype="f32", mode=FS, patch_h=7, patch_w=7), 4),              # eight
    (dict(C=1792, dtype="f32", mode=FS, patch_h=7, patch_w=7), 1),              # seven
    (dict(C=484, dtype="f32", mode=BS, n_s=8), 4),                              # two, rows that start anywhere
    (dict(C=484, dtype="f32", mode=FS, patch_h=7, patch_w=7), 1),
    (dict(C=764, dtype="f32", mode=BS, n_s=8), 1),                              # three of them
], ids=str)
def test_rule_of_column_tiles_and_segments(kw, want):
    wl = Workload(name="split_tiles", N=64, H=14, W=14, layout="nhwc", data_seed=7, sampling_seed=8, layer_id=1, **kw)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] tiles {kw}", flush=True)
    res, path = _run(wl, inp, nhwc_fused=2)
    assert path == want
    assert_parity(res, oracle_reference(wl, inp), wl, what=f"tiles {kw}", inp=inp)
