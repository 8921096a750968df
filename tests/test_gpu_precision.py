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
