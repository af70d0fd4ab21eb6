"""Shared helpers for the GPU tests: run the HIP library through the C ABI on
seeded inputs and compare with the oracle."""

from __future__ import annotations

import functools

import numpy as np

import azgen
import oracle
from oracle import az_oracle as O

TOL = {  # max |dP| elementwise, max |dV|
    "bf16": (1e-2, 2e-2),
    "int8": (3e-2, 5e-2),
    "fp8": (3e-2, 5e-2),
}


def gpu_eval(spec_shape, blob, dtype, planes, legal, w_scales=None, act_scales=None, tiling=0,
             max_batch=None, repeat=1):
    """Evaluates through az_net_load / az_eval_batch; returns numpy (P, V) (a list of
    (P, V) when repeat > 1)."""
    import torch

    import paper_2609_37447_amd as az
    B = planes.shape[0]
    spec = az.spec_from_shape(spec_shape, max_batch or max(B, 1))
    net = az.az_net_load(spec, blob, dtype, w_scales, act_scales)
    try:
        if tiling:
            az.az_net_set_tiling(net, tiling)
        dev = torch.device("cuda:0")
        pl = torch.from_numpy(np.ascontiguousarray(planes, dtype=np.float32)).to(dev)
        lg = torch.from_numpy(np.ascontiguousarray(legal, dtype=np.uint8)).to(dev)
        outs = []
        for _ in range(repeat):
            pol = torch.full((B, legal.shape[1]), float("nan"), device=dev)
            val = torch.full((B,), float("nan"), device=dev)
            az.eval_tensors(net, pl, lg, pol, val)
            torch.cuda.synchronize()
            outs.append((pol.cpu().numpy().astype(np.float64), val.cpu().numpy().astype(np.float64)))
    finally:
        az.az_net_free(net)
    return outs[0] if repeat == 1 else outs


def launched_grids(call):
    """Workgroups (first grid dimension) of each kernel of this library that call
    launches, from the profiler's trace."""
    import json
    import os
    import tempfile

    import torch
    from torch.profiler import ProfilerActivity, profile
    for _ in range(3):  # a trace without any kernel says nothing about the call
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
            call()
            torch.cuda.synchronize()
        with tempfile.TemporaryDirectory() as d:
            path = os.path.join(d, "trace.json")
            prof.export_chrome_trace(path)
            with open(path) as f:
                events = json.load(f)["traceEvents"]
        grids = [e["args"]["grid"][0] for e in events if e.get("cat") == "kernel" and "az_" in e.get("name", "")]
        if grids:
            break
    return grids


def check_grids(spec, n_moves, blob, dtype, scales, sizes, boards, tilings):
    """The launched grid of every forced tiling and the automatic choice (0) is that of
    the tiling az_net_tiling_for names; boards: its boards per workgroup."""
    import torch

    import paper_2609_37447_amd as az
    net = az.az_net_load(spec, blob, dtype, *scales)
    try:
        for B in sizes:
            pl = torch.zeros((B, spec.in_planes, 8, 8), device="cuda")
            lg = torch.ones((B, n_moves), dtype=torch.uint8, device="cuda")
            pol, val = torch.empty((B, n_moves), device="cuda"), torch.empty((B,), device="cuda")
            for t in (0,) + tilings:
                az.az_net_set_tiling(net, t)
                told = az.az_net_tiling_for(net, B)
                assert t in (0, told)
                assert launched_grids(lambda: az.eval_tensors(net, pl, lg, pol, val)) == [-(-B // boards[told])], (B, t)
    finally:
        az.az_net_free(net)


@functools.lru_cache(maxsize=8)
def quant_scales(wname: str, fmt: str, alpha_fold: bool = True):
    """(weight scales, activation scales) by absmax calibration on the workload's
    512 seeded calibration positions, computed by the oracle."""
    w = azgen.WORKLOADS[wname]
    blob = azgen.workload_weights(w, alpha_fold)
    amax = _absmax(wname, alpha_fold)
    return O.weight_scales(w.shape, blob, fmt), O.act_scales_from_absmax(amax, fmt)


@functools.lru_cache(maxsize=8)
def _absmax(wname: str, alpha_fold: bool):
    w = azgen.WORKLOADS[wname]
    blob = azgen.workload_weights(w, alpha_fold)
    return O.calibrate_absmax(w.shape, blob, azgen.make_calibration_planes(w))


def oracle_eval(shape, blob, dtype, planes, legal, w_scales=None, act_scales=None, chunk=128, progress=None):
    """Oracle outputs (float64 network for f32 / bf16, the quantised definition
    for int8 / fp8), in chunks of rows; progress(msg) is called per chunk."""
    P, V = [], []
    for s in range(0, planes.shape[0], chunk):
        pl, lg = planes[s:s + chunk], legal[s:s + chunk]
        if dtype in ("f32", "bf16"):
            p, v = oracle.forward(shape, blob, pl, lg)
        else:
            p, v = oracle.forward_quant(shape, blob, w_scales, act_scales, dtype, pl, lg)
        P.append(p)
        V.append(v)
        if progress is not None:
            progress(f"  oracle rows {s}..{s + pl.shape[0] - 1}")
    return np.concatenate(P), np.concatenate(V)


def assert_policy_structure(P, legal, atol_sum=1e-5):
    """Illegal cells exactly 0, legal rows sum to 1, rows without legal cells all zero."""
    m = legal != 0
    assert np.all(P[~m] == 0.0), "nonzero prior on an illegal move"
    assert np.all(np.isfinite(P))
    has = m.any(axis=1)
    sums = P.sum(axis=1)
    assert np.all(np.abs(sums[has] - 1.0) <= atol_sum), np.abs(sums[has] - 1.0).max()
    assert np.all(sums[~has] == 0.0)


def compare(Pg, Vg, Pr, Vr, dtype):
    tp, tv = TOL[dtype]
    dp = float(np.abs(Pg - Pr).max())
    dv = float(np.abs(Vg - Vr).max())
    assert dp <= tp and dv <= tv, f"{dtype}: max|dP| {dp:.3g} (tol {tp}), max|dV| {dv:.3g} (tol {tv})"
    return dp, dv


def compare_f32(Pg, Vg, Pr, Vr):
    """fp32 gate: per row max|dP| <= 1e-4 * max P*, |dV| <= 1e-4 * max(|V*|, 1e-2)."""
    rowmax = Pr.max(axis=1)
    dp = np.abs(Pg - Pr).max(axis=1)
    assert np.all(dp <= 1e-4 * rowmax), float((dp / np.maximum(rowmax, 1e-300)).max())
    dv = np.abs(Vg - Vr)
    assert np.all(dv <= 1e-4 * np.maximum(np.abs(Vr), 1e-2)), float(dv.max())


def top1_agreement(Pa, Pb, legal):
    m = legal != 0
    has = m.any(axis=1)
    a = np.where(m, Pa, -1.0).argmax(axis=1)
    b = np.where(m, Pb, -1.0).argmax(axis=1)
    return float(np.mean(a[has] == b[has]))
