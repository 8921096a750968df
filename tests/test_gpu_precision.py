"""Precision of what the statistics are made of, against 64 bits.

Sums over a channel in the single-launch N x C x H x W kernels.  Both sums are made to dwarf what they are taken of: the pivot (the first sampled element) lies far from a channel's mean, dy far from
zero.  A value rounded to fp32 is off by 2^-24 / sqrt(3) of itself at most, as a root mean square; additions within a thread, of which each
holds a small part of the sum, hardly count, and every addition across lanes, waves and blocks that is made in fp32 counts in full."""
import numpy as np
import pytest
import torch

from paper_1810_10962_amd import bns, workloads
from paper_1810_10962_amd.workloads import Workload
from parity import oracle_reference

FULL, NS, VDN = bns.BNS_FULL, bns.BNS_NS, bns.BNS_VDN
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]
ROUNDING = 2.0 ** -24 / np.sqrt(3.0)


@pytest.mark.parametrize("shape,dtype,mkw,threads,roundings,blocks", [
    # threads that hold sampled elements, roundings in each (elements, and the first addition across lanes), blocks that share a channel
    ((9, 320, 11, 11), "f32", dict(mode=NS, n_s=1), 31, 5, 1),
    ((40, 144, 9, 9), "f32", dict(mode=VDN, n_s=2), 42, 5, 1),
    ((11, 112, 18, 19), "f32", dict(mode=NS, n_s=1), 86, 5, 1),
    ((34, 64, 23, 20), "bf16", dict(mode=FULL), 1900, 9, 4),
    ((58, 96, 12, 12), "f32", dict(mode=FULL), 1000, 9, 2),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v.get("mode") if isinstance(v, dict) else str(v))
def test_sums_across_lanes_and_waves_are_not_rounded(shape, dtype, mkw, threads, roundings, blocks):
    N, C_, H, W = shape
    wl = Workload(name="rounding", N=N, C=C_, H=H, W=W, dtype=dtype, data_seed=92, sampling_seed=24, layer_id=7, **mkw)
    inp = workloads.make_inputs(wl)
    rng = np.random.default_rng(93)
    x, dy = rng.standard_normal(shape), rng.standard_normal(shape) + 8.0
    x[0, :, 0, 0] = 8.0
    exact = (lambda a: workloads.round_to_bf16(a.astype(np.float32))) if dtype == "bf16" else (lambda a: a.astype(np.float32))
    inp["x"], inp["dy"] = exact(x), exact(dy)
    print(f"[gpu-case] rounding of the sums {shape} {dtype} {mkw}", flush=True)
    res, ref = bns.run_workload(wl, inp), oracle_reference(wl, inp)
    inside = np.sqrt(roundings / threads + (1.0 / blocks if blocks > 1 else 0.0))       # (a block's share is handed on as fp32)
    rms = lambda name, scale: float(np.sqrt(np.mean(((res[name] - ref[name]) / scale) ** 2)))       # noqa: E731
    shift = np.abs(ref["save_mean"] - 8.0)                  # the sums are of x - pivot
    mean, dbeta = rms("save_mean", shift), rms("dbeta", ref["dbeta"])
    print(f"mean {mean / ROUNDING:.2f} ({inside:.2f}), dbeta {dbeta / ROUNDING:.2f} roundings", flush=True)
    assert mean < ROUNDING * inside
    # dy, whose sums every point takes part in, and the rounding of the result
    assert dbeta < ROUNDING * np.sqrt(1.0 + inside ** 2)


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("kernels,options", [("single launch", {"grouped": 2, "nhwc_fused": 1}), ("grouped", {"grouped": 1}),
                                             ("streaming", {"path": 1, "nhwc_fused": 2})], ids=["single_launch", "grouped", "streaming"])
def test_inverse_square_root(layout, kernels, options):
    """Bit for bit the value in 64 bits, rounded once: an fp64 result two units off lies on the other side of an fp32 rounding boundary
    once in 2^28 values, the hardware's estimate of 23 bits in every second one."""
    N, C_, H, W = 4, 16, 12, 12
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(94)
    x = torch.tensor(rng.integers(1, 16, C_).astype(np.float32) / 8, device=dev)    # (few bits: the mean of some rows is exact, too)
    x = (x if layout == "nhwc" else x[:, None, None]).expand((N, H, W, C_) if layout == "nhwc" else (N, C_, H, W)).contiguous()
    shape, spec = bns.make_shape(N, C_, H, W, "f32", layout), bns.make_spec(FULL)
    one, zero, y = torch.ones(C_, device=dev), torch.zeros(C_, device=dev), torch.empty_like(x)
    ws = torch.zeros(bns.bns_workspace_bytes(shape, spec), dtype=torch.uint8, device=dev)
    values = np.ldexp(rng.uniform(1.0, 4.0, 400), 2 * rng.integers(-62, 62, 400)).astype(np.float32)    # every mantissa, odd and even powers
    mean, got = torch.empty(C_, device=dev), torch.empty(len(values), C_, device=dev)
    print(f"[gpu-case] inverse square root {layout} {kernels}", flush=True)
    try:
        for k, v in options.items():
            bns.bns_set_option(k, v)
        for i, eps in enumerate(values):
            bns.bns_forward(shape, spec, 1, x, one, zero, float(eps), 0.1, y, mean, got[i], None, None, ws)
        took = bns.bns_get_option("last_path_forward"), bns.bns_get_option("last_fused_forward")
    finally:
        for k in options:
            bns.bns_set_option(k, 0)
    assert (took[0] == 1) == (kernels == "streaming")
    if layout == "nchw" and kernels != "streaming":
        assert (took[1] == 3) == (kernels == "grouped")
    want = (1.0 / np.sqrt(values.astype(np.float64))).astype(np.float32)
    assert np.array_equal(got.cpu().numpy(), np.repeat(want[:, None], C_, 1))
