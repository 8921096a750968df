"""The single-launch kernels of the N x H x W x C layout: column tiles whose last vector is shared, fewer channels than a
vector, every number of rows per thread, rows that do not fit the registers, Eq. 4 -- each against the oracle; the
give-up path of their exchange; and that they stay out of HIP graphs."""
import numpy as np
import pytest
import torch

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import BS, FS, FULL, NS, Workload
from parity import assert_parity, oracle_reference

pytestmark = pytest.mark.gpu


def _with(opts, call):
    try:
        for k, v in opts.items():
            bns.bns_set_option(k, v)
        return call()
    finally:
        for k in opts:
            bns.bns_set_option(k, 0)


def _paths():
    return bns.bns_get_option("last_path_forward"), bns.bns_get_option("last_path_backward")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,lanes", [
    ((3, 3, 9, 9), 0),              # fewer channels than a vector
    ((4, 9, 20, 20), 0),            # a vector and a channel: the second vector shares seven (three) channels with the first
    ((4, 41, 20, 20), 5),           # a last tile of one lane is avoided
    ((2, 150, 19, 19), 8),          # tiles of unequal width, rows at odd multiples of two bytes
    ((7, 64, 33, 31), 4),           # many members per tile, a ragged last share of the rows
    ((30, 520, 12, 12), 0),         # more tiles than fit a row of lanes
    ((1, 8, 1, 70), 0),             # hardly more rows than row lanes
])
def test_single_launch_nhwc(shape, lanes, dtype):
    N, C_, H, W = shape
    modes = [dict(mode=FULL), dict(mode=BS, n_s=max(1, N // 3)), dict(mode=FS, patch_h=max(1, H // 2), patch_w=max(1, W - 3))]
    if N >= 3:
        modes += [dict(mode=FS, patch_h=1, patch_w=2, n_v=2, mix_beta=0.3), dict(mode=NS, n_s=1, n_v=1)]
    for i, mkw in enumerate(modes):
        wl = Workload(name="nhwc_fused", N=N, C=C_, H=H, W=W, dtype=dtype, layout="nhwc", data_seed=50 + i, sampling_seed=18,
                      layer_id=i, epoch=1, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch {shape} {dtype} {mkw} lanes {lanes}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": lanes}, lambda: bns.run_workload(wl, inp))
        assert _paths() in ((2, 2), (3, 3))                 # (3: so few rows that one block takes them all)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"nhwc fused {shape} {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rounds", [5, 9, 17, 45])
def test_rows_per_thread(rounds, dtype):
    """5, 9: the next larger number of kept rows; 17: x is no longer kept; 45: rows that do not fit the registers."""
    V = 4 if dtype == "f32" else 8
    C_ = 128 * V                                            # 16 tiles of 8 lanes on 256 compute units: 16 members of 64 rows
    units = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 64 * (units // 16) * (rounds - 1) + 37
    for i, mkw in enumerate((dict(mode=FULL), dict(mode=BS, n_s=1), dict(mode=FS, patch_h=1, patch_w=5, n_v=1))):
        wl = Workload(name="rows", N=3, C=C_, H=1, W=rows // 3, dtype=dtype, layout="nhwc", data_seed=60 + i, sampling_seed=3,
                      layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch, {rounds} rows per thread {wl.shape} {dtype} {mkw}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": 8}, lambda: bns.run_workload(wl, inp))
        assert _paths() == (2, 2)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"{rounds} rows per thread {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("C_,lanes,members", [
    (8, 2, 33),                 # 64 threads per channel, one member each, as many as there are rows of 256
    (32, 8, 15),                # 16 threads per channel: one member each, no multiple of eight
    (128, 32, 31),              # four threads per channel: eight members each, all polled at once
    (128, 32, 33),              # nine each: five at a time
    (128, 32, 70),              # eighteen each: six at a time
], ids=str)
def test_members_of_a_tile(C_, lanes, members):
    """Blocks that share a tile's rows: how many of them a thread polls, and what is left over."""
    rows = members * (2 if members * C_ <= 4096 else 4) * (512 // lanes) - 5        # rows per thread, by the pairs of sums that a block reads
    for i, mkw in enumerate((dict(mode=FULL), dict(mode=FS, patch_h=1, patch_w=5, n_v=1))):
        wl = Workload(name="members", N=3, C=C_, H=1, W=rows // 3, dtype="f32", layout="nhwc", data_seed=70 + i, sampling_seed=3,
                      layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch, {members} members {wl.shape} {mkw}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": lanes}, lambda: bns.run_workload(wl, inp))
        assert _paths() == (2, 2)
        assert (bns.bns_get_option("last_team_forward"), bns.bns_get_option("last_team_backward")) == (members, members)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"{members} members {mkw}", inp=inp)


@pytest.mark.parametrize("dtype,C_,rounds", [
    ("f32", 1250, 3), ("f32", 1250, 13),        # both directions without the hint, x kept and not
    ("f32", 1250, 19), ("f32", 1252, 45),       # forward: all loads first; rows read twice, whole vectors
    ("bf16", 2484, 3), ("bf16", 2489, 13), ("bf16", 2489, 20), ("bf16", 2489, 41),     # 41: rows in LDS
    ("bf16", 2496, 5),                          # rows on 64 bytes: with the hint
], ids=str)
def test_lines_shared_between_tiles(dtype, C_, rounds):
    """Rows that begin on no 64 bytes, in several tiles: blocks of two tiles write parts of one line, with plain stores."""
    V = 4 if dtype == "f32" else 8
    tiles = -(-(-(-C_ // V)) // 8)
    members = torch.cuda.get_device_properties(0).multi_processor_count // tiles
    rows = 64 * members * (rounds - 1) + 41
    for i, mkw in enumerate((dict(mode=BS, n_s=1), dict(mode=FS, patch_h=1, patch_w=9))):
        wl = Workload(name="lines", N=3, C=C_, H=1, W=rows // 3, dtype=dtype, layout="nhwc", data_seed=90 + i, sampling_seed=4,
                      layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch, shared lines, {rounds} rows per thread {wl.shape} {dtype} {mkw}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": 8}, lambda: bns.run_workload(wl, inp))
        assert _paths() == (2, 2)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"shared lines, {rounds} rows {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("path", [0, 1], ids=["default", "streaming"])
def test_inverse_deviation_at_its_ends(layout, path):
    """1 / sqrt(Var + eps): a constant channel without and with eps, a spread near the ends of fp32, an infinity."""
    N, C_, H, W = 4, 8, 9, 9
    dev, scale = torch.device("cuda:0"), [0.0, 0.0, 1e-18, 1e18, 1.0, 3e-5, 1e4, 1.0]
    z = torch.randn(N, C_, H, W, generator=torch.Generator().manual_seed(7), dtype=torch.float64)
    x = (z * torch.tensor(scale, dtype=torch.float64)[None, :, None, None]).float()
    x[0, 7, 0, 0] = float("inf")
    stored = (x.permute(0, 2, 3, 1) if layout == "nhwc" else x).contiguous().to(dev)
    shape, spec = bns.make_shape(N, C_, H, W, "f32", layout), bns.make_spec(FULL)
    out = lambda: torch.empty(C_, device=dev)               # noqa: E731
    ws = torch.zeros(bns.bns_workspace_bytes(shape, spec), dtype=torch.uint8, device=dev)
    for eps in (0.0, 1e-5):
        mean, invstd = out(), out()
        _with({"path": path}, lambda: bns.bns_forward(shape, spec, 1, stored, torch.ones(C_, device=dev), torch.zeros(C_, device=dev),
                                                      eps, 0.1, torch.empty_like(stored), mean, invstd, None, None, ws))
        got, d = invstd.cpu().double(), x.double()
        want = 1.0 / torch.sqrt(d.var(dim=(0, 2, 3), unbiased=False) + float(np.float32(eps)))
        print(f"[gpu-case] inverse deviation {layout} path {path} eps {eps}: {got.tolist()}", flush=True)
        assert torch.equal(got[:2], want[:2].float().double())                  # (infinity without eps)
        # a single-precision sum of 324 squares is off by no more than 324 * 2^-24, its square root by half of that; the squares are
        # those of x - pivot, whose mean (at most 3 deviations from the first element here) is taken off again
        m1 = (d.mean(dim=(0, 2, 3)) - d[0, :, 0, 0])[2:7]
        assert (m1.square() < 9 * d.var(dim=(0, 2, 3), unbiased=False)[2:7]).all()
        assert (((got - want) / want)[2:7].abs() < 162 * 2.0 ** -24 * (1.0 + m1.square() / d.var(dim=(0, 2, 3), unbiased=False)[2:7])).all()
        assert torch.isnan(got[7])


@pytest.mark.parametrize("shape,dtype,want", [
    ((13, 137, 7, 7), "bf16", (3, 1)),          # ragged rows, 175 KB: not in waiting kernels
    ((30, 137, 12, 12), "bf16", (2, 2)),        # the same rows, 1.2 MB
    ((52, 349, 4, 4), "f32", (3, 2)),           # seven rows per thread: one block takes them forward, a team backward
    ((4, 349, 4, 4), "f32", (3, 3)),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_default_choice_on_both_sides_of_its_lines(shape, dtype, want):
    N, C_, H, W = shape
    for i, mkw in enumerate((dict(mode=FULL), dict(mode=BS, n_s=2), dict(mode=FS, patch_h=2, patch_w=3))):
        wl = Workload(name="nhwc_default", N=N, C=C_, H=H, W=W, dtype=dtype, layout="nhwc", data_seed=65 + i, sampling_seed=4,
                      layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc default kernels {shape} {dtype} {mkw}", flush=True)
        res = bns.run_workload(wl, inp)
        assert _paths() == want
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"nhwc default {shape} {dtype} {mkw}", inp=inp)


def test_missing_team_mate_and_what_comes_after():
    wl = Workload(name="nhwc_give_up", N=9, C=70, H=40, W=40, dtype="f32", layout="nhwc", mode=BS, n_s=3, data_seed=5,
                  sampling_seed=6, layer_id=1)
    inp = workloads.make_inputs(wl)
    buf = bns.Buffers(wl, inp)
    print("[gpu-case] nhwc single launch, give-up path", flush=True)

    def both():
        buf.forward()
        buf.backward()
        assert _paths() == (2, 2)
        return buf.results(), bns.bns_expired_waits(buf.workspace)

    bad, expired_bad = _with({"nhwc_fused": 1, "test_spin_limit": 64, "test_mute_exchange": 1}, both)
    good, expired_good = _with({"nhwc_fused": 1}, both)
    for k in ("y", "save_mean", "save_invstd", "dx", "dgamma", "dbeta"):
        assert np.isnan(bad[k]).all(), f"{k}: finite values after a wait that expired"
    for k in ("running_mean", "running_var"):
        assert np.array_equal(bad[k], inp[k].astype(np.float32)), k
    assert expired_bad > 0 and expired_good == 0
    assert_parity(good, oracle_reference(wl, inp), wl, what="after the give-up run", inp=inp)


def test_a_wait_that_runs_out_concerns_its_channel_only():
    """One channel of a tile is not published: its results are NaN and its moving averages stay, every other channel of
    the tile is right, its moving averages (Eq. 8) included."""
    wl = Workload(name="nhwc_one_channel", N=9, C=70, H=40, W=40, dtype="f32", layout="nhwc", mode=BS, n_s=3, data_seed=5,
                  sampling_seed=6, layer_id=1)
    inp = workloads.make_inputs(wl)
    buf = bns.Buffers(wl, inp)
    print("[gpu-case] nhwc single launch, one channel not published", flush=True)
    _with({"nhwc_fused": 1, "test_spin_limit": 64, "test_mute_channel": 6}, buf.forward)
    assert _paths()[0] == 2
    got, ref = buf.results(), oracle_reference(wl, inp)
    assert bns.bns_expired_waits(buf.workspace) > 0
    rest = np.arange(wl.C) != 5
    for k in ("y", "save_mean", "save_invstd"):
        bad = np.moveaxis(got[k], 1, 0)[5] if k == "y" else got[k][5]
        assert np.isnan(bad).all(), k
    for k in ("running_mean", "running_var"):
        assert got[k][5] == inp[k][5], k
        # one fp32 rounding of each term of Eq. 8 and of the statistic itself
        np.testing.assert_allclose(got[k][rest], ref[k][rest], rtol=1e-5, atol=1e-6, err_msg=k)
    y, want = got["y"][:, rest], ref["y"][:, rest]
    assert np.abs(y - want).max() <= 1e-5 * np.abs(want).max()


def test_sums_left_by_the_streaming_kernels_are_not_taken_for_a_team_mates():
    """The exchange takes any slot word that carries the launch's stamp.  Streaming calls on constant tensors leave zeros
    as partial sums in the workspace; the next stamp is then set to zero, which is what those words would carry
    if they lay in the slots."""
    wl = Workload(name="nhwc_left_over", N=9, C=70, H=40, W=40, dtype="f32", layout="nhwc", mode=BS, n_s=3, data_seed=5,
                  sampling_seed=6, layer_id=1)
    inp = workloads.make_inputs(wl)
    flat = dict(inp, x=np.full_like(inp["x"], 2.0), dy=np.zeros_like(inp["dy"]))
    buf, left = bns.Buffers(wl, inp), bns.Buffers(wl, flat)
    left.workspace = buf.workspace
    header = torch.tensor([0x626E7301 << 32, 0], dtype=torch.int64, device="cuda").view(torch.uint8)     # magic | stamp 0, counts 0
    print("[gpu-case] nhwc single launch after streaming calls in the same workspace", flush=True)

    def streaming():
        buf.workspace.fill_(0xA5)                           # (no zeros, and no stamps used before, in the slots themselves)
        left.forward()
        left.backward()
        assert _paths() == (1, 1)
        buf.workspace[:16].copy_(header)

    _with({"nhwc_fused": 2}, streaming)
    _with({"nhwc_fused": 1}, buf.forward)
    assert _paths()[0] == 2
    _with({"nhwc_fused": 2}, streaming)
    _with({"nhwc_fused": 1}, buf.backward)
    assert _paths()[1] == 2
    assert bns.bns_expired_waits(buf.workspace) == 0
    assert_parity(buf.results(), oracle_reference(wl, inp), wl, what="after streaming calls", inp=inp)


def test_sums_of_many_channels_in_the_other_layout_are_not_taken_for_a_team_mates():
    """As above for the widest exchange (452 KiB of slots), after N x C x H x W calls of 3840 channels, whose workspace has the
    least room for slots."""
    wl = Workload(name="nhwc_wide", N=9, C=256, H=40, W=40, dtype="bf16", layout="nhwc", mode=BS, n_s=3, data_seed=7,
                  sampling_seed=8, layer_id=1)
    before = Workload(name="nchw_many", N=9, C=3840, H=8, W=8, dtype="f32", mode=BS, n_s=3, data_seed=9, sampling_seed=10)
    inp, flat = workloads.make_inputs(wl), workloads.make_inputs(before)
    flat.update(x=np.full_like(flat["x"], 2.0), dy=np.zeros_like(flat["dy"]))
    buf, left = bns.Buffers(wl, inp), bns.Buffers(before, flat)
    assert left.workspace.numel() >= buf.workspace.numel()
    buf.workspace = left.workspace
    header = torch.tensor([0x626E7301 << 32, 0], dtype=torch.int64, device="cuda").view(torch.uint8)
    print("[gpu-case] nhwc single launch after nchw streaming calls of 3840 channels in the same workspace", flush=True)

    def streaming():
        buf.workspace.fill_(0xA5)
        left.forward()
        left.backward()
        assert _paths() == (1, 1)
        buf.workspace[:16].copy_(header)

    many, wide = {"path": 1, "splits_stats": 64, "splits_reduce": 64}, {"nhwc_fused": 1, "nhwc_fused_lanes": 16}
    _with(many, streaming)
    _with(wide, buf.forward)
    assert _paths()[0] == 2
    _with(many, streaming)
    _with(wide, buf.backward)
    assert _paths()[1] == 2
    assert bns.bns_expired_waits(buf.workspace) == 0
    assert_parity(buf.results(), oracle_reference(wl, inp), wl, what="after streaming calls", inp=inp)
    res = _with(many, lambda: bns.run_workload(before, workloads.make_inputs(before)))        # blocks per channel bounded
    assert_parity(res, oracle_reference(before, workloads.make_inputs(before)), before, what="3840 channels, 64 splits",
                  inp=workloads.make_inputs(before))


def test_a_captured_call_takes_the_streaming_kernels():
    wl = Workload(name="nhwc_graph", N=20, C=64, H=40, W=40, dtype="f32", layout="nhwc", mode=BS, n_s=4, data_seed=7,
                  sampling_seed=8, layer_id=2)
    inp = workloads.make_inputs(wl)
    ref = oracle_reference(wl, inp)
    buf = bns.Buffers(wl, inp)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        buf.forward()
        buf.backward()
        assert _paths() == (2, 2)                           # (8 MB: single launch outside a graph)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        buf.forward()
        buf.backward()
    assert _paths() == (1, 1)
    for _ in range(3):
        buf.running_mean.copy_(torch.from_numpy(inp["running_mean"]))
        buf.running_var.copy_(torch.from_numpy(inp["running_var"]))
        buf.y.fill_(float("nan"))
        buf.dx.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        assert_parity(buf.results(), ref, wl, what="replay", inp=inp)


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_a_call_beside_a_capture_leaves_the_capture_alone(layout):
    """A stream that carried a kernel whose blocks wait is captured; a call on another stream meanwhile cannot be ordered behind
    that kernel without recording on the captured stream.  It takes the streaming kernels, runs at once, and the graph
    holds what was captured."""
    wl = Workload(name="beside_capture", N=32, C=96, H=28, W=28, dtype="f32", layout=layout, mode=BS, n_s=4, data_seed=9,
                  sampling_seed=11, layer_id=3)
    inp = workloads.make_inputs(wl)
    ref = oracle_reference(wl, inp)
    a, b = bns.Buffers(wl, inp), bns.Buffers(wl, inp)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print(f"[gpu-case] a call beside a capture, {layout}", flush=True)

    def capture():
        with torch.cuda.stream(side):
            a.forward()
            a.backward()
        assert _paths() == (2, 2)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            a.forward()
            with torch.cuda.stream(other):
                b.forward()
                b.backward()
            beside = _paths()
            a.backward()
        return beside

    beside = _with({"fused_variant": 3}, capture)
    assert beside == (1, 1)
    other.synchronize()
    assert_parity(b.results(), ref, wl, what="beside the capture", inp=inp)
    for _ in range(3):
        a.running_mean.copy_(torch.from_numpy(inp["running_mean"]))
        a.running_var.copy_(torch.from_numpy(inp["running_var"]))
        a.y.fill_(float("nan"))
        a.dx.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        assert_parity(a.results(), ref, wl, what="replay", inp=inp)


@pytest.mark.parametrize("dtype,rounds", [("f32", 24), ("f32", 25), ("f32", 54), ("f32", 55), ("bf16", 25), ("bf16", 49), ("bf16", 50), ("bf16", 51)])
def test_rows_in_registers_and_lds(dtype, rounds):
    """The last number of rows that a variant holds and the first that it does not: registers alone (24), registers and LDS (backward 54
    in fp32, 49 in bf16; forward 54 and 50), a row that is read again."""
    V = 4 if dtype == "f32" else 8
    units = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 64 * (units // 16) * (rounds - 1) + 37
    for i, mkw in enumerate((dict(mode=FULL), dict(mode=BS, n_s=1))):
        wl = Workload(name="rows_lds", N=3, C=128 * V, H=1, W=rows // 3, dtype=dtype, layout="nhwc", data_seed=64 + i, sampling_seed=4,
                      layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch, {rounds} rows per thread {wl.shape} {dtype} {mkw}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": 8}, lambda: bns.run_workload(wl, inp))
        assert _paths() == (2, 2)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"{rounds} rows per thread {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("kw", [
    dict(N=101, C=16, H=14, W=14, dtype="bf16"),            # 633 KB, 19796 rows
    dict(N=43, C=24, H=14, W=14, dtype="f32"),              # 809 KB, 8428 rows
    dict(N=33, C=10, H=16, W=16, dtype="bf16"),             # 8448 rows, columns that are no whole number of vectors
    dict(N=16, C=63, H=32, W=32, dtype="f32"),              # 4 MiB less 64 KiB
], ids=lambda kw: "{N}x{C}x{H}x{W}-{dtype}".format(**kw))
def test_many_rows_in_up_to_4_mib_carry_the_bits_of_the_stage_calls(kw):
    """More than 8192 rows, up to 4 MiB: a whole call has the bits of its stage calls, and a captured one those of an eager one."""
    wl = Workload(name="nhwc_band", layout="nhwc", mode=FS, patch_h=5, patch_w=7, data_seed=17, sampling_seed=8, layer_id=4, **kw)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] many rows in up to 4 MiB {wl.shape} {wl.dtype}", flush=True)
    whole = bns.run_workload(wl, inp)
    assert _paths() == (1, 1)
    buf = bns.Buffers(wl, inp)
    bns.bns_forward_stats(buf.shape, buf.spec, buf.seed, buf.x, wl.eps, wl.momentum, buf.save_mean, buf.save_invstd,
                          buf.running_mean, buf.running_var, buf.workspace)
    bns.bns_forward_normalize(buf.shape, buf.x, buf.gamma, buf.beta, buf.save_mean, buf.save_invstd, buf.y)
    bns.bns_backward_reduce(buf.shape, buf.x, buf.dy, buf.save_mean, buf.save_invstd, buf.dgamma, buf.dbeta, buf.workspace)
    bns.bns_backward_dx(buf.shape, buf.spec, buf.seed, buf.x, buf.dy, buf.gamma, buf.save_mean, buf.save_invstd, buf.dgamma,
                        buf.dbeta, buf.dx)
    stages = buf.results()
    buf = bns.Buffers(wl, inp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        buf.forward()
        buf.backward()
    for _ in range(3):
        buf.running_mean.copy_(torch.from_numpy(inp["running_mean"]))
        buf.running_var.copy_(torch.from_numpy(inp["running_var"]))
        buf.y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
    replay = buf.results()
    for k in whole:
        assert (whole[k] == stages[k]).all() and (whole[k] == replay[k]).all(), k


@pytest.mark.parametrize("shape", [(2, 131072, 2, 2), (5, 9000000, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_few_rows_of_very_many_channels(shape):
    """Rows so long that the offsets of rows past the end, which the kernel walks over, approach (first shape) or pass (second)
    32 bits: one launch without waits, the results of the streaming kernels."""
    N, C_, H, W = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    rand = lambda *s: torch.rand(*s, generator=gen, device="cuda")                  # noqa: E731
    sh, sp = bns.make_shape(N, C_, H, W, "f32", "nhwc"), bns.make_spec(BS, N - 1, 0, 0, 0, 3, 0)
    x, dy, gamma, beta = rand(N, H, W, C_) - 0.3, rand(N, H, W, C_) - 0.5, rand(C_) + 0.5, rand(C_)
    ws = torch.empty(bns.bns_workspace_bytes(sh, sp), dtype=torch.uint8, device="cuda")
    print(f"[gpu-case] few rows of very many channels {shape}", flush=True)

    def step():
        out = dict(y=torch.empty_like(x), dx=torch.empty_like(x), rm=torch.zeros(C_, device="cuda"), rv=torch.ones(C_, device="cuda"))
        out.update({k: torch.empty(C_, device="cuda") for k in ("mean", "invstd", "dgamma", "dbeta")})
        bns.bns_forward(sh, sp, 7, x, gamma, beta, 1e-3, 0.1, out["y"], out["mean"], out["invstd"], out["rm"], out["rv"], ws)
        bns.bns_backward(sh, sp, 7, x, dy, gamma, out["mean"], out["invstd"], out["dx"], out["dgamma"], out["dbeta"], ws)
        return out

    got = step()
    assert _paths() == (3, 3)
    want = _with({"nhwc_fused": 2}, step)
    assert _paths() == (1, 1)
    for k in got:
        assert torch.allclose(got[k], want[k], rtol=1e-5, atol=1e-5 * float(want[k].abs().max())), k


@pytest.mark.parametrize("dtype,rounds,ragged", [
    ("f32", 20, False), ("f32", 28, True), ("f32", 33, False), ("f32", 41, True),         # 41, ragged: a row that is read again
    ("bf16", 17, True), ("bf16", 29, False), ("bf16", 36, True), ("bf16", 37, True),      # 36: the last with all loads first, 37: LDS
])
def test_rows_between_the_steps(dtype, rounds, ragged):
    """Every step of the rows that registers hold beyond 16, rows that begin on no 64 bytes (forward requests all of them first), Eq. 4."""
    V = 4 if dtype == "f32" else 8
    units = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 64 * (units // 16) * (rounds - 1) + 37
    for i, mkw in enumerate((dict(mode=BS, n_s=1), dict(mode=FS, patch_h=1, patch_w=rows // 7, n_v=1, mix_beta=0.4))):
        wl = Workload(name="rows_steps", N=3, C=128 * V - (3 if ragged else 0), H=1, W=rows // 3, dtype=dtype, layout="nhwc", data_seed=74 + i,
                      sampling_seed=5, layer_id=i, **mkw)
        inp = workloads.make_inputs(wl)
        print(f"[gpu-case] nhwc single launch, {rounds} rows per thread {wl.shape} {dtype} {mkw}", flush=True)
        res = _with({"nhwc_fused": 1, "nhwc_fused_lanes": 8}, lambda: bns.run_workload(wl, inp))
        assert _paths() == (2, 2)
        assert_parity(res, oracle_reference(wl, inp), wl, what=f"{rounds} rows per thread {dtype} {mkw}", inp=inp)


@pytest.mark.parametrize("kw,want", [
    (dict(N=8, C=28, H=23, W=23, mode=BS, n_s=2), (2, 2)),          # 237 KB, streaming's accesses 64 bits
    (dict(N=5, C=28, H=23, W=23, mode=BS, n_s=2), (1, 1)),          # 148 KB
    (dict(N=8, C=29, H=23, W=23, mode=BS, n_s=2), (1, 1)),          # 245 KB, single elements
    (dict(N=8, C=29, H=23, W=23, mode=FULL), (2, 1)),
    (dict(N=14, C=29, H=23, W=23, mode=BS, n_s=2), (2, 2)),         # 430 KB
], ids=str)
def test_ragged_bf16_rows_of_small_tensors(kw, want):
    wl = Workload(name="ragged_small", dtype="bf16", layout="nhwc", data_seed=3, sampling_seed=4, layer_id=2, **kw)
    inp = workloads.make_inputs(wl)
    print(f"[gpu-case] ragged {kw}", flush=True)
    res = bns.run_workload(wl, inp)
    assert (bns.bns_get_option("last_path_forward"), bns.bns_get_option("last_path_backward")) == want
    assert_parity(res, oracle_reference(wl, inp), wl, what=f"ragged {kw}", inp=inp)
