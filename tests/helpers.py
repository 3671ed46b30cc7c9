"""Comparison helpers shared by the GPU parity tests."""
import ctypes

import numpy as np
import torch

from oracle import isopo_oracle as orc
from paper_2512_23353_amd import workloads as wl

TOL = {"f32": 1e-4, "bf16": 2e-2}   # relative tolerances the benchmark definition states


def rel_err(got, ref) -> float:
    """Norm-wise relative error ||got - ref||_F / ||ref||_F."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    den = np.linalg.norm(ref)
    return float(np.linalg.norm(got - ref) / den) if den > 0 else float(np.linalg.norm(got))


def assert_K_close(K, K_ref, tol, what=""):
    K = np.asarray(K, dtype=np.float64)
    assert np.array_equal(K, K.T), f"{what}: K not bit-symmetric"
    assert rel_err(K, K_ref) <= tol, f"{what}: K rel err {rel_err(K, K_ref):.3e} > {tol}"
    d = np.sqrt(np.clip(np.diag(K_ref), 0, None))
    guard = tol * np.outer(d, d)
    bad = np.abs(K - K_ref) > guard + 1e-300
    assert not bad.any(), f"{what}: |dK_ij| above tol*sqrt(K_ii K_jj) at {np.argwhere(bad)[:4].tolist()}"


def assert_c_close(c, c_ref, tol, what=""):
    c = np.asarray(c, dtype=np.float64)
    assert rel_err(c, c_ref) <= tol, f"{what}: c rel err {rel_err(c, c_ref):.3e} > {tol}"
    assert np.max(np.abs(c - c_ref)) <= tol * np.max(np.abs(c_ref)) + 1e-300, f"{what}: c element guard"


def assert_dW_close(dW, dW_ref, tol, what="", dW_abs=None):
    """Norm-wise tolerance plus an element guard.  Rounding of the terms of
    dW = sum_i c_i G_i (bf16 stash, bf16 pre-scaled Delta) is relative to the
    terms, not to their possibly cancelling sum, and X has outlier channels 20x
    the rest, so the guard is tol * (sum_i |c_i G_i| + its mean) where the
    oracle provides that scale, else 8 tol rms(dW)."""
    dW = np.asarray(dW, dtype=np.float64)
    assert rel_err(dW, dW_ref) <= tol, f"{what}: dW rel err {rel_err(dW, dW_ref):.3e} > {tol}"
    if dW_abs is not None:
        guard = tol * (dW_abs + dW_abs.mean())
    else:
        guard = 8 * tol * np.sqrt(np.mean(dW_ref ** 2))
    bad = np.abs(dW - dW_ref) > guard + 1e-300
    assert not bad.any(), f"{what}: dW element guard at {np.argwhere(bad)[:4].tolist()}"


def oracle_step(prob, variant, lam, reg_mode=0, chunk_rows=None, dW_in=None, beta=0.0):
    return orc.layer_step(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets, prob.A, variant, lam,
                          reg_mode, dW_in=dW_in, beta=beta, chunk_rows=chunk_rows)


def to_device(prob, device):
    from paper_2512_23353_amd import isopo
    X, D = prob.X.to(device), prob.Delta.to(device)
    layer = isopo.Layer(X, D, prob.seq_offsets)
    A = torch.from_numpy(prob.A).to(device)
    return layer, A


class SplitPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tile", "groups", "n_chunks", "chunk_tokens", "longest_first")]


def split_plan(d_in, d_out, lengths, per_sequence):
    """Launch plan of the fp32 contraction (host arithmetic; the library's internal C++ function)."""
    from paper_2512_23353_amd import isopo
    fn = isopo.load()._ZN5isopo22plan_split_contractionEiiiiPKib
    fn.restype = SplitPlan
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return fn(ctypes.c_int(d_out), ctypes.c_int(d_in), ctypes.c_int(int(off[-1])), ctypes.c_int(len(lengths)),
              off.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), ctypes.c_bool(per_sequence))


class ContractionPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tile", "occupancy", "tiles_m", "tiles_n", "n_chunks", "chunk_tokens",
                                            "whole_tiles")] + [("xcd_start", ctypes.c_int * 9), ("blocks", ctypes.c_longlong)]


def bf16_plan(d_in, d_out, lengths, per_sequence, weighted=False, budget=False):
    """Launch plan of the bf16 contraction, also for the weighted sum and a launch with a budget of compute units, which
    isopo_contraction_plan does not describe."""
    from paper_2512_23353_amd import isopo
    fn = isopo.load()._ZN5isopo16plan_contractionEiiiiPKibbb
    fn.restype = ContractionPlan
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return fn(ctypes.c_int(d_out), ctypes.c_int(d_in), ctypes.c_int(int(off[-1])), ctypes.c_int(len(lengths)),
              off.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), ctypes.c_bool(per_sequence), ctypes.c_bool(weighted),
              ctypes.c_bool(budget))


class WalkPlan(ctypes.Structure):
    _fields_ = [("per_xcd", ctypes.c_int), ("kind", ctypes.c_int), ("first", ctypes.c_int * 9), ("alone", ctypes.c_int * 8)]


def walk_plan(d_in, d_out, lengths, budget=0):
    """How the workgroups of a per-sequence bf16 launch share its (sequence, tile) pairs, and the order of the sequences."""
    from paper_2512_23353_amd import isopo
    fn = isopo.load()._ZN5isopo9plan_walkEiiiiPKiiPt
    fn.restype = WalkPlan
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    order = np.zeros(len(lengths), dtype=np.uint16)
    tile = bf16_plan(d_in, d_out, lengths, True, budget=budget > 0).tile
    plan = fn(ctypes.c_int(tile), ctypes.c_int(d_out), ctypes.c_int(d_in), ctypes.c_int(len(lengths)),
              off.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), ctypes.c_int(budget if tile == 256 else 0),
              order.ctypes.data_as(ctypes.POINTER(ctypes.c_uint16)))
    return plan, order
