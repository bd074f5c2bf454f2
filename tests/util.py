"""Helpers shared by the GPU parity tests: build the library's inputs from a
seeded workload, and compare against the CPU oracle with the stated tolerances."""
import sys

import numpy as np
import torch

import oracle
import paper_2411_11217_amd as M
from moe_workloads import MoEConfig, make_inputs, oracle_view

# Tolerances of the parity bar.  bf16 storage with fp32 accumulation: max |err| <= 2e-2
# and relative RMS <= 1e-2.  float32 (outputs of the tiny workload are ~0.02, so the absolute
# bound says nothing): relative RMS <= 1e-5 and max |err| <= 1e-5 * max|ref| * 10.
BF16_MAX_ABS, BF16_REL_RMS = 2e-2, 1e-2
F32_REL_RMS = 1e-5
NEAR_TIE = 1e-4


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def shape_of(cfg: MoEConfig) -> M.MoEShape:
    return M.make_shape(cfg.T, cfg.H, cfg.F, cfg.E, cfg.k, cfg.dtype, cfg.page_bytes)


def rel_rms(got: np.ndarray, ref: np.ndarray) -> float:
    den = np.sqrt(np.mean(ref.astype(np.float64) ** 2))
    num = np.sqrt(np.mean((got.astype(np.float64) - ref.astype(np.float64)) ** 2))
    return float(num / max(den, 1e-300))


def assert_close(got, ref, dtype: str, what: str):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (what, got.shape, ref.shape)
    if got.size == 0:
        return
    assert np.isfinite(got).all(), what + ": non-finite values"
    err = np.abs(got - ref).max()
    rr = rel_rms(got, ref)
    say(f"    {what}: max|err|={err:.3e} rel-rms={rr:.3e} (ref rms {np.sqrt(np.mean(ref**2)):.3e})")
    if dtype == "bf16":
        assert err <= BF16_MAX_ABS, f"{what}: max abs err {err} > {BF16_MAX_ABS}"
        assert rr <= BF16_REL_RMS, f"{what}: rel rms {rr} > {BF16_REL_RMS}"
    else:
        assert rr <= F32_REL_RMS, f"{what}: rel rms {rr} > {F32_REL_RMS}"
        assert err <= 10 * F32_REL_RMS * max(np.abs(ref).max(), 1e-30), f"{what}: max abs err {err}"


def assert_h_close(got, ref, dtype: str, what: str):
    """The SwiGLU product h is a ROUNDED intermediate (storage type dt).  The GPU forms it from
    float32 accumulators, the oracle from doubles, so a value that sits near a rounding boundary
    may land on the neighbouring representable number: allow one unit in the last place of the
    storage type on fewer than 5 in a thousand elements (observed: about 6 in ten thousand), plus 1e-4 absolute for values near zero (where
    the float32 accumulation error of g and u, ~1e-5, exceeds the spacing of the type), and hold
    the whole array to the relative-RMS bound."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape and np.isfinite(got).all(), what
    mant = 7 if dtype == "bf16" else 23
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(ref), 2.0 ** -100))) - mant)
    diff = np.abs(got - ref)
    flips = float((diff > 0).mean())
    rr = rel_rms(got, ref)
    say(f"    {what}: unequal share={flips:.2e} max|err|={float(diff.max()):.3e} rel-rms={rr:.3e}")
    if dtype == "bf16":
        assert (diff <= 1.001 * ulp + 1e-4).all(), what + ": more than one ulp off"
        assert flips < 5e-3, what + ": too many elements differ"
        assert rr <= BF16_REL_RMS
    else:
        assert rr <= F32_REL_RMS, what


def linear_takes_rows_kernel(T, K, N):
    """The rule of that name in csrc/moe_host.h, so that a test of one of the linear map's kernels can say that its shape reaches it."""
    return (N // 64) * -(-T // 128) <= 256 or (K <= 1536 and T <= 32) or (T > 128 and -(-T // 64) * (N // 128) <= 256)


def row_tiles(counts):
    """Row tiles of 256 rows that the experts' rows make; a remainder of up to 32 rows per full tile rides along."""
    n = 0
    for c in counts:
        q, r = divmod(int(c), 256)
        n += q if q and 0 < r <= 32 * q else q + (r > 0)
    return n


def bf16_launches(counts, H, F, down_cols=0):
    """What launch_expert_ffn_bf16 (csrc/moe_ffn_bf16.hip) takes for gate/up and for down beyond the kernel for few rows, and the
    number of tiles per XCD that stay together, by its own formulas."""
    E, each = len(counts), int(sum(counts)) // len(counts)
    assert each > 80, "the kernel for few rows"
    tiles, dt = E * max(1, (each - 32 + 255) // 256), H // 128

    def half(n):
        return 0 < n % 256 <= 128

    if down_cols == 1 or (down_cols == 0 and tiles * dt <= 256):
        down = "128 columns, halves" if tiles * dt <= 128 else "128 columns"
    else:
        down = "256 columns, halves" if half(tiles * ((dt + 1) // 2)) else "256 columns"
    return "halves" if half(tiles * (F // 128)) else "whole", down, 32 if each > 256 else 8 if each > 128 else 0


class Case:
    """A workload on both sides: CPU tensors + oracle views, device tensors + paged weights."""

    def __init__(self, cfg: MoEConfig, shuffle_pages: bool = False, extra_pages: int = 0,
                 identical_experts: bool = False, pin_pages: bool = False, to_device: bool = True, inputs=None):
        self.cfg = cfg
        self.shape = shape_of(cfg)
        self.inp = inputs if inputs is not None else make_inputs(cfg, threads=16, identical_experts=identical_experts)
        self.view = {k: oracle_view(v) for k, v in self.inp.items() if k != "bias"}
        self.bias_np = None if self.inp["bias"] is None else self.inp["bias"].numpy().astype(np.float64)
        order = torch.Generator().manual_seed(1234) if shuffle_pages else None
        self.pw = M.PagedWeights(self.shape, self.inp["W1"], self.inp["W3"], self.inp["W2"], order=order,
                                 extra_pages=extra_pages, pin=pin_pages)
        if to_device:
            self.x = self.inp["x"].cuda()
            self.Wr = self.inp["Wr"].cuda()
            self.bias = None if self.inp["bias"] is None else self.inp["bias"].cuda()
            if not pin_pages:
                self.pw.to_device()

    def oracle_route(self):
        v = self.view
        return oracle.route(v["x"], v["Wr"], self.cfg.k, self.cfg.dtype_code, bias=self.bias_np)

    def oracle_layer(self, tokens=None):
        v = self.view
        return oracle.layer(v["x"], v["Wr"], v["W1"], v["W3"], v["W2"], self.cfg.k, self.cfg.dtype_code,
                            bias=self.bias_np, tokens=tokens)


def compare_routing(cfg, ids_gpu, w_gpu, rt, what="route"):
    """Bit-exact expert sets and order, except tokens the oracle flags as near ties
    (set decided by < 1e-4: excluded, counted; order decided by < 1e-4: compared as sets).
    Returns the boolean mask of tokens whose expert SET matches the oracle's."""
    ids_gpu = np.asarray(ids_gpu)
    w_gpu = np.asarray(w_gpu, dtype=np.float64)
    set_tie = rt["gap_next"] < NEAR_TIE
    order_tie = rt["gap_inner"] < NEAR_TIE
    exact = (ids_gpu == rt["ids"]).all(axis=1)
    same_set = (np.sort(ids_gpu, axis=1) == np.sort(rt["ids"], axis=1)).all(axis=1)
    say(f"    {what}: tokens={ids_gpu.shape[0]} near-tie(set)={int(set_tie.sum())} near-tie(order)={int(order_tie.sum())} "
        f"exact={int(exact.sum())} same-set={int(same_set.sum())}")
    bad = ~exact & ~set_tie & ~order_tie
    assert not bad.any(), f"{what}: {int(bad.sum())} tokens differ without a near tie, first {np.nonzero(bad)[0][:5]}"
    assert (same_set | set_tie).all(), what + ": expert set differs without a near tie"
    # gate weights: compare per expert id on tokens with the same set
    if same_set.any():
        og = np.argsort(ids_gpu[same_set], axis=1)
        oo = np.argsort(rt["ids"][same_set], axis=1)
        wg = np.take_along_axis(w_gpu[same_set], og, axis=1)
        wo = np.take_along_axis(rt["w"][same_set], oo, axis=1)
        err = np.abs(wg - wo).max()
        say(f"    {what}: gate weight max|err|={err:.3e}")
        assert err <= 2e-5, what + ": gate weights differ"
    np.testing.assert_allclose(w_gpu.sum(axis=1), 1.0, atol=1e-5)
    return same_set


def check_permutation_valid(ids: np.ndarray, E: int, k: int, pm: dict):
    """Properties that define the permutation for ANY ids (used at full size)."""
    flat = ids.reshape(-1)
    R = flat.shape[0]
    counts, offsets, row_src, row_of = (np.asarray(pm[n]) for n in ("counts", "offsets", "row_src", "row_of"))
    assert np.array_equal(counts, np.bincount(flat, minlength=E))
    assert counts.sum() == R and offsets[0] == 0 and offsets[E] == R
    assert np.array_equal(offsets[1:], np.cumsum(counts))
    assert np.array_equal(row_src, np.argsort(flat, kind="stable"))
    assert np.array_equal(row_of[row_src], np.arange(R))


def assert_status_clean(status):
    """Status words: [0] error bits and [1] (unused) must be zero; [2], [3] carry the shader clock a block of the
    bf16 GEMM launches saw (diagnostic, any value)."""
    st = [int(v) for v in status]
    assert st[0] == 0 and st[1] == 0, st
    return st
