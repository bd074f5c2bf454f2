"""GPU parity: every stage of the HIP path against the CPU oracle, element by
element, on the same seeded inputs, through the C ABI.  Stage tests feed each
GPU stage the ORACLE's upstream results so that a near tie in the router cannot
cascade; the layer test runs the fused call end to end."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2411_11217_amd as M
from moe_workloads import CONFIGS, MoEConfig, make_inputs, scaled
from util import (F32_REL_RMS, Case, assert_close, assert_h_close, assert_status_clean, bf16_launches, check_permutation_valid, compare_routing, rel_rms, row_tiles, say,
                  shape_of)

pytestmark = pytest.mark.gpu

C1 = CONFIGS["c1_tiny_f32"]
# reduced bf16 cases: several row tiles of 256 with ragged tails, several column tiles,
# an odd number of 128-wide column tiles in the down projection (H = 384), k in {1,2,4}
MED = {
    "bf16_two_experts_ragged": MoEConfig("m1", "bf16", T=700, H=256, F=384, E=2, k=1, page_bytes=64 * 1024, seed=21),
    "bf16_top2_of_4": MoEConfig("m2", "bf16", T=333, H=384, F=512, E=4, k=2, page_bytes=48 * 1024, seed=22),
    "bf16_top4_of_16": MoEConfig("m3", "bf16", T=200, H=256, F=256, E=16, k=4, page_bytes=32 * 1024, seed=23),
    "bf16_top4_of_16_more_rows": MoEConfig("m6", "bf16", T=420, H=256, F=256, E=16, k=4, page_bytes=32 * 1024, seed=26),   # beyond the kernel for few rows
    "f32_top2_of_5": MoEConfig("m4", "f32", T=150, H=128, F=256, E=5, k=2, page_bytes=96 * 1024, seed=24),
    # launches whose tiles are all whole, three column tiles, one expert with several row tiles: short search (chunks off), chunks of 8, chunks of 32
    "bf16_single_groups": MoEConfig("m7", "bf16", T=2200, H=384, F=384, E=44, k=2, page_bytes=48 * 1024, seed=27, bias=((3, 0.5), (9, 0.25))),
    "bf16_chunks_of_8": MoEConfig("m8", "bf16", T=3300, H=384, F=384, E=44, k=2, page_bytes=48 * 1024, seed=28, bias=((3, 0.5), (9, 0.25))),
    "bf16_chunks_of_32": MoEConfig("m9", "bf16", T=6200, H=384, F=384, E=44, k=2, page_bytes=48 * 1024, seed=29, bias=((3, 0.4), (9, 0.2))),
    "bf16_skewed": MoEConfig("m5", "bf16", T=600, H=256, F=256, E=8, k=2, page_bytes=64 * 1024, seed=25,
                             bias=((0, 3.0), (7, -3.0))),
}


def _dev_i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _dev_f32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def run_stagewise(case: Case):
    cfg, s = case.cfg, case.shape
    ref = case.oracle_layer()
    # ---- a1 route
    ids, w, logits = M.moe_route(s, case.x, case.Wr, bias=case.bias, want_logits=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(logits.cpu().numpy(), ref["logits"], rtol=0, atol=2e-5 * max(1.0, np.abs(ref["logits"]).max()))
    compare_routing(cfg, ids.cpu().numpy(), w.cpu().numpy(), ref)
    # ---- a2 permute on the oracle's ids: bit exact
    pm = M.moe_permute(s, _dev_i32(ref["ids"]), x=case.x, topk_w=_dev_f32(ref["w"]))
    torch.cuda.synchronize()
    for name in ("counts", "offsets", "row_src", "row_of"):
        assert np.array_equal(pm[name].cpu().numpy(), ref[name]), name
    xp = pm["x_perm"].cpu()
    xp_bits = xp.view(torch.int16).numpy().view(np.uint16) if cfg.dtype == "bf16" else xp.numpy()
    assert np.array_equal(xp_bits, ref["x_perm"]), "x_perm"
    assert np.array_equal(pm["row_w"].cpu().numpy(), ref["w"].astype(np.float32).reshape(-1)[ref["row_src"]])
    # ---- a3 expert FFN on the oracle's permuted rows
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(ref["x_perm"], ref["offsets"], v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    xperm_dev = case.x[torch.from_numpy(ref["row_src"] // cfg.k).long().cuda()].contiguous()
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    h, out = M.moe_expert_ffn(s, xperm_dev, _dev_i32(ref["offsets"]), case.pw.table_dev, case.pw.pages_dev, status=status)
    torch.cuda.synchronize()
    assert_status_clean(status.cpu().tolist())
    assert_h_close(h.float().cpu().numpy(), h_ref, cfg.dtype, "h")
    assert_close(out.cpu().numpy(), o_ref, cfg.dtype, "expert out")
    # with the gate weight fused into the epilogue
    rw = ref["w"].reshape(-1)[ref["row_src"]]
    _, out_w = M.moe_expert_ffn(s, xperm_dev, _dev_i32(ref["offsets"]), case.pw.table_dev, case.pw.pages_dev,
                                row_w=_dev_f32(rw))
    assert_close(out_w.cpu().numpy(), o_ref * rw[:, None], cfg.dtype, "expert out * w")
    # ---- a4 combine on the oracle's expert outputs
    o_dev = _dev_f32(o_ref)
    y = M.moe_combine(s, o_dev, _dev_i32(ref["row_of"]), topk_w=_dev_f32(ref["w"]))
    y_ref = oracle.combine(o_dev.cpu().numpy().astype(np.float64), ref["row_of"], cfg.k, w=ref["w"].astype(np.float32))
    assert_close(y.cpu().numpy(), y_ref, "f32", "combine")
    y1 = M.moe_combine(s, o_dev, _dev_i32(ref["row_of"]), topk_w=None)
    assert_close(y1.cpu().numpy(), oracle.combine(o_dev.cpu().numpy().astype(np.float64), ref["row_of"], cfg.k), "f32",
                 "combine (unweighted)")
    return ref


def run_layer(case: Case, ref=None):
    cfg, s = case.cfg, case.shape
    ref = ref or case.oracle_layer()
    y, ws = M.moe_layer(s, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, bias=case.bias)
    torch.cuda.synchronize()
    assert_status_clean(ws.view("status").cpu().tolist())
    ids = ws.view("topk_ids").cpu().numpy()
    same = compare_routing(cfg, ids, ws.view("topk_w").cpu().numpy(), ref, "layer route")
    pm = {n: ws.view(n).cpu().numpy() for n in ("counts", "offsets", "row_src", "row_of")}
    check_permutation_valid(ids, cfg.E, cfg.k, pm)               # valid for the ids the GPU chose
    if same.all() and (ids == ref["ids"]).all():
        for n in pm:
            assert np.array_equal(pm[n], ref[n]), n
    assert (np.abs(pm["counts"].astype(np.int64) - ref["counts"]).sum()) <= 2 * int((~same).sum())
    assert_close(y.cpu().numpy()[same], ref["y"][same], cfg.dtype, "layer y")
    return y, ws


@pytest.mark.parametrize("down_cols,H,down", [(0, 256, "128 columns, halves"), (1, 256, "128 columns, halves"), (2, 256, "256 columns, halves"), (1, 1024, "128 columns"), (0, 1024, "256 columns")])
def test_expert_ffn_row_counts_across_the_tile_variants(down_cols, H, down):
    """Segments of 1 .. 300 rows, one per expert, on both sides of every threshold of the bf16 kernel's row-tile
    variants (32, 64, 128, 192 rows, the 256-row tile boundary, tiles that take a remainder of up to 32 rows along) and an
    empty one, against the oracle row by row; with the tall tiles switched off every bit stays the same.  In each of the four down
    launches (H = 256: all tiles of the only round in halves)."""
    counts = [1, 16, 17, 32, 33, 0, 64, 65, 127, 128, 129, 160, 192, 193, 255, 256, 257, 300, 31, 449, 272, 273, 288, 289, 532,
              544, 576, 577, 800, 863, 865, 1061]
    E, F = len(counts), 384
    assert bf16_launches(counts, H, F, down_cols) == ("whole", down, 32)
    cfg = MoEConfig("rows", "bf16", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=64 * 1024, seed=77)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    x_bits = v["x"]                                     # [T, H] in the oracle's storage form; k = 1: rows are tokens
    h_ref, o_ref = oracle.expert_ffn(x_bits, offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    M.set_option("down_cols", down_cols)
    try:
        status = torch.zeros(4, dtype=torch.int32, device="cuda")
        h, out = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, status=status)
        torch.cuda.synchronize()
    finally:
        M.set_option("down_cols", 0)
    assert_status_clean(status.cpu().tolist())
    M.set_option("down_cols", down_cols)
    M.set_option("tall_tiles", 0)
    try:
        h0, out0 = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, status=status)
        torch.cuda.synchronize()
    finally:
        M.set_option("down_cols", 0)
        M.set_option("tall_tiles", 1)
    assert torch.equal(h0, h) and torch.equal(out0, out)
    for e, c in enumerate(counts):
        if c == 0:
            continue
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        assert_h_close(h.float().cpu().numpy()[lo:hi], h_ref[lo:hi], "bf16", f"h, expert {e} with {c} rows")
        assert_close(out.cpu().numpy()[lo:hi], o_ref[lo:hi], "bf16", f"out, expert {e} with {c} rows")


@pytest.mark.parametrize("counts,H,F,down,tiles", [
    ([90, 100, 33, 257, 129, 64, 0, 193, 81, 288, 65, 120, 97, 1, 140, 88], 4480, 128, "256 columns, halves", 15 * 18),    # an odd number of page tiles
    ([90, 257, 150, 193, 33, 280, 64, 256], 128, 4608, "128 columns, halves", 8),               # gate/up: 36 x 8 tiles
    ([90, 257, 150, 193, 33, 280, 64, 289], 640, 128, "128 columns, halves", 9 * 5),             # all of them in halves
    ([800, 20, 20, 280], 4096, 128, "128 columns, halves", 6 * 32),                              # 24 per XCD: all of them whole
    ([4608] + [1] * 15, 1024, 128, "128 columns, halves", 33 * 8),                               # 33 per XCD: 32 whole, one in halves
    ([800, 600, 20, 700], 4096, 128, "128 columns", 10 * 32),
])
def test_bf16_tiles_of_a_last_round_in_halves(counts, H, F, down, tiles):
    """A last round of at most half a round of tiles, which are computed in halves of their columns, of every height (`tiles`: those of the
    down launch); the tiles dealt to the XCDs and evened out, or neither: the same bits."""
    gate, launch, _ = bf16_launches(counts, H, F)
    assert gate == "halves" and launch == down and tiles == row_tiles(counts) * (H // 128 if down.startswith("128") else (H // 128 + 1) // 2)
    E = len(counts)
    cfg = MoEConfig("halves", "bf16", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=64 * 1024, seed=83)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(v["x"], offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    w = np.random.default_rng(1).random(cfg.T, dtype=np.float32) + 0.5

    def run():
        res = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w))
        torch.cuda.synchronize()
        return res

    h, out = run()
    assert_h_close(h.float().cpu().numpy(), h_ref, "bf16", "h")
    assert_close(out.cpu().numpy(), o_ref * w[:, None], "bf16", "out")
    for option in ("balance", "xcd_remap"):
        M.set_option(option, 0)
        try:
            h0, out0 = run()
        finally:
            M.set_option(option, 1)
        assert torch.equal(h0, h) and torch.equal(out0, out), option


@pytest.mark.parametrize("counts,H,F", [
    ([1, 16, 17, 31, 32, 33, 0, 48, 63, 64, 65, 128, 129], 256, 384),       # 48 rows on average: 128-row blocks
    ([1, 15, 0, 33, 64, 65, 100, 17], 128, 640),                              # 36 rows: 64-row blocks, two and ten k-steps
    ([95, 96, 97, 112, 113, 127, 40, 1, 60], 128, 256),                      # 82 rows: beyond the kernel for few rows
    ([95, 96, 97, 112, 113, 127, 40, 1, 34], 384, 128),                      # 79 rows
    ([300, 3, 0, 1], 256, 256),                                               # 76 rows, three row tiles of one expert
    ([130, 161, 176, 191, 145, 0], 256, 384),                                 # 133 rows: five and six row tiles per wavefront
])
def test_bf16_expert_ffn_with_few_rows_per_expert(counts, H, F):
    """Segments on both sides of the 16-row MFMA tiles, the row-tile pairs and the blocks of the kernel for few rows per expert."""
    E = len(counts)
    cfg = MoEConfig("few", "bf16", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=48 * 1024, seed=79)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(v["x"], offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    w = np.random.default_rng(1).random(cfg.T, dtype=np.float32) + 0.5
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    h, out = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w), status=status)
    torch.cuda.synchronize()
    assert_status_clean(status.cpu().tolist())
    for e, c in enumerate(counts):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if c:
            assert_h_close(h.float().cpu().numpy()[lo:hi], h_ref[lo:hi], "bf16", f"h, expert {e} with {c} rows")
            assert_close(out.cpu().numpy()[lo:hi], o_ref[lo:hi] * w[lo:hi, None], "bf16", f"out, expert {e} with {c} rows")
    run_layer(case)


@pytest.mark.parametrize("counts,H,F", [
    ([1, 15, 16, 17, 31, 32, 33, 0, 64, 70], 128, 256),          # 27 rows on average: k split over the wavefronts, two k-steps for four of them
    ([5, 0, 40], 384, 640),                                        # the same with 6 and 10 k-steps
    ([1, 15, 16, 17, 31, 32, 33, 0, 65, 160], 128, 256),         # 37 rows on average: columns split over the wavefronts
    ([200, 97, 0], 384, 640),
])
def test_f32_expert_ffn_row_counts_across_the_kernels(counts, H, F):
    """Segments on both sides of the 16-row MFMA tiles and the 32-row blocks of the two float32 kernels, against the oracle; the layer
    leaves the permuted rows in its workspace whether or not its GEMM gathers them."""
    E = len(counts)
    cfg = MoEConfig("rows32", "f32", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=96 * 1024, seed=78)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(v["x"], offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    w = np.random.default_rng(1).random(cfg.T, dtype=np.float32) + 0.5
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    h, out = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w), status=status)
    torch.cuda.synchronize()
    assert_status_clean(status.cpu().tolist())
    assert_h_close(h.cpu().numpy(), h_ref, "f32", "h")
    assert_close(out.cpu().numpy(), o_ref * w[:, None], "f32", "out * w")
    ws = M.Workspace(case.shape)
    ws.buf.fill_(0xFF)                                             # NaN everywhere
    y, _ = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws)
    assert torch.equal(ws.view("x_perm"), case.x[ws.view("row_src").long()])
    M.set_option("fuse_gather", 0)
    try:
        y0, _ = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev)
    finally:
        M.set_option("fuse_gather", 1)
    assert torch.equal(y0, y)


@pytest.mark.parametrize("dtype,T", [("bf16", 1), ("bf16", 3), ("bf16", 16), ("bf16", 17), ("f32", 1), ("f32", 8), ("f32", 9), ("f32", 31),
                                     ("f32", 32), ("f32", 63), ("f32", 64), ("f32", 65)])
@pytest.mark.parametrize("E,k", [(1, 1), (5, 2), (8, 8), (16, 3), (17, 17), (33, 4), (64, 64), (64, 8)])
def test_layer_places_the_rows_of_a_handful_of_tokens(dtype, T, E, k):
    """With few tokens (bf16: 16, f32: 512 over the padded number of experts) the router's block also does the permutation: what
    the layer leaves in its workspace is what the two calls give, bit by bit, and its output that of the stages."""
    cfg = MoEConfig("place", dtype, T=T, H=256, F=128, E=E, k=k, page_bytes=32 * 1024, seed=83)
    case = Case(cfg)
    s = case.shape
    ids, w, _ = M.moe_route(s, case.x, case.Wr)
    pm = M.moe_permute(s, ids, x=case.x, topk_w=w)
    h, out = M.moe_expert_ffn(s, pm["x_perm"], pm["offsets"], case.pw.table_dev, case.pw.pages_dev, row_w=pm["row_w"])
    y_ref = M.moe_combine(s, out, pm["row_of"])
    ws = M.Workspace(s)
    ws.buf.fill_(0xFF)
    y, _ = M.moe_layer(s, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(ws.view("topk_ids").reshape(-1), ids.reshape(-1)) and torch.equal(ws.view("topk_w").reshape(-1), w.reshape(-1))
    for name in ("counts", "offsets", "row_src", "row_of", "row_w"):
        assert torch.equal(ws.view(name).reshape(-1), pm[name].reshape(-1)), name
    assert_status_clean(ws.view("status").tolist())
    assert torch.equal(y, y_ref)


@pytest.mark.parametrize("counts,H,F", [
    ([1, 0, 3], 128, 128),                     # two k-steps each way
    ([16], 512, 640),                            # as many k-steps as are under way, and two more
    ([0, 7, 2, 0, 1], 1024, 1152),               # twice as many, and two more
    ([2, 13, 0], 1536, 384),
])
def test_bf16_handful_of_tokens(counts, H, F):
    """The kernel for at most 16 tokens against the oracle, and bit by bit against the kernel that takes over with more; one expert
    may have more rows than a tile when the offsets do not come from a routing."""
    E, T = len(counts), sum(counts)
    cfg = MoEConfig("thin", "bf16", T=T + 17, H=H, F=F, E=E, k=1, page_bytes=48 * 1024, seed=81)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    few = M.make_shape(T, H, F, E, 1, "bf16", cfg.page_bytes)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(v["x"][:T], offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    x = case.x[:T].contiguous()
    w = np.random.default_rng(2).random(T, dtype=np.float32) + 0.5
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    h, out = M.moe_expert_ffn(few, x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w), status=status)
    torch.cuda.synchronize()
    assert_status_clean(status.cpu().tolist())
    assert_h_close(h.float().cpu().numpy(), h_ref, "bf16", "h")
    assert_close(out.cpu().numpy(), o_ref * w[:, None], "bf16", "out * w")
    more = offsets.copy()
    more[-1] += 17                                       # 17 rows more behind those of the last expert: beyond this kernel
    w2 = np.concatenate([w, np.ones(17, np.float32)])
    h2, out2 = M.moe_expert_ffn(case.shape, case.x, _dev_i32(more), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w2))
    assert torch.equal(h2[:T], h) and torch.equal(out2[:T], out)
    if T * 2 > 16:                                       # all rows of two per token on one expert: two row tiles
        twice = M.make_shape(T, H, F, E, min(E, 2), "bf16", cfg.page_bytes)
        R = twice.R
        one = np.zeros(E + 1, np.int32)
        one[1:] = R
        h3, out3 = M.moe_expert_ffn(twice, case.x[:R].contiguous(), _dev_i32(one), case.pw.table_dev, case.pw.pages_dev)
        h4, out4 = M.moe_expert_ffn(M.make_shape(R + 17, H, F, E, 1, "bf16", cfg.page_bytes), torch.cat([case.x[:R], case.x[:17]]),
                                    _dev_i32(np.concatenate([[0], np.full(E, R + 17, np.int32)]).astype(np.int32)), case.pw.table_dev, case.pw.pages_dev)
        assert torch.equal(h4[:R], h3) and torch.equal(out4[:R], out3)


@pytest.mark.parametrize("T", [1, 4])
def test_bf16_handful_of_tokens_with_weights_beyond_the_last_level_cache(T):
    """403 MB of expert weights: the kernel for a handful of tokens loads them with the non-temporal hint, in both launches."""
    cfg = MoEConfig("thin_stream", "bf16", T=T, H=2048, F=4096, E=8, k=2, page_bytes=1 << 20, seed=86)
    case = Case(cfg, shuffle_pages=True)
    ws = M.Workspace(case.shape)
    ws.buf.fill_(0xFF)
    y = torch.full((T, cfg.H), float("nan"), device="cuda")
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
    torch.cuda.synchronize()
    assert_status_clean(ws.view("status").tolist())
    ids, w = ws.view("topk_ids").cpu().numpy(), ws.view("topk_w").cpu().numpy()
    same = compare_routing(cfg, ids, w, case.oracle_route())
    ref = case.oracle_layer()
    assert_close(y.cpu().numpy()[same], ref["y"][same], "bf16", "y")


@pytest.mark.parametrize("counts,H,F", [
    ([1, 16, 17, 33, 64, 65, 96, 97, 128, 129, 300, 0], 128, 256),    # the split kernel's row tiles and loops; two and four k-steps
    ([260, 31, 111], 384, 640),                                         # six and ten k-steps, three row tiles of an expert
    ([100, 40, 70, 0, 33, 64, 128, 129], 128, 1024),                    # column blocks for more than a round of 32 rows, for less of 64
    ([20] * 63 + [70], 128, 256),                                       # few rows, but column blocks for every compute unit: gate/up alone
    ([36, 20, 70, 1, 64, 33, 65, 0], 128, 4224),                        # column blocks for more than a round, at most 48 rows on average
    ([150, 40, 9, 260], 256, 4224),                                     # 264 column blocks: the blocks of 128 rows
])
def test_f32_split_products(counts, H, F):
    """The float32 kernel on the bf16 matrix cores against the oracle.  Its sums over k take one float32 rounding (2^-24) per 32 k
    at the size of the result and six at the size of 32 terms: below 1e-6 relative RMS with up to 132 such steps."""
    E = len(counts)
    cfg = MoEConfig("split32", "f32", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=96 * 1024, seed=79)
    case = Case(cfg, shuffle_pages=True, extra_pages=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = case.view
    h_ref, o_ref = oracle.expert_ffn(v["x"], offsets, v["W1"], v["W3"], v["W2"], cfg.dtype_code)
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    h, out = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, status=status)
    torch.cuda.synchronize()
    assert_status_clean(status.cpu().tolist())
    assert rel_rms(h.cpu().numpy(), h_ref) < 1e-6
    assert rel_rms(out.cpu().numpy(), o_ref) < 1e-6
    for e, c in enumerate(counts):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if c:
            assert_close(out.cpu().numpy()[lo:hi], o_ref[lo:hi], "f32", f"out, expert {e} with {c} rows")


@pytest.mark.parametrize("counts,H,F", [([100, 40], 128, 256), ([100, 40, 70, 33, 64, 1, 128, 129], 128, 1024),
                                         ([36, 20, 70, 1, 64, 33, 65, 2], 128, 4224), ([150, 40, 9, 260], 256, 4224)])       # every kernel of gate/up
def test_f32_split_products_of_extreme_values(counts, H, F):
    """Infinities, NaN, values that bf16 rounds to infinity and rows so small that their sums are formed again: h and out as the
    float32 products give them, row by row, and nothing of it in other rows.  2e-6: a chain of F / 4 = 1056 float32 roundings at
    most, 2^-24 * sqrt(1056 / 3) if they are random."""
    T, E = sum(counts), len(counts)
    cfg = MoEConfig("extreme32", "f32", T=T, H=H, F=F, E=E, k=1, page_bytes=96 * 1024, seed=80)
    case = Case(cfg)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    x = case.x.clone()
    x[3, 5] = float("inf")
    x[20, 7] = float("-inf")
    x[21, 8] = float("nan")
    x[40, 9], x[40, 10] = 3.4e38, -3.4e38
    x[60] *= 2.0 ** -52                               # h about 2^-106, sums of the down launch below their limit
    x[61] *= 2.0 ** -58                               # h about 2^-118
    x[110, 100] = float("inf")
    w = torch.rand(T, generator=torch.Generator().manual_seed(4)) + 0.5
    h, out = M.moe_expert_ffn(case.shape, x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=w.cuda())
    h, out, x = h.cpu(), out.cpu(), x.cpu()
    h_ref, o_ref = torch.empty_like(h), torch.empty_like(out)
    h64, o64 = torch.empty_like(h, dtype=torch.float64), torch.empty_like(out, dtype=torch.float64)
    for e in range(E):
        r = slice(int(offsets[e]), int(offsets[e + 1]))
        W1, W3, W2 = (case.inp[n][e] for n in ("W1", "W3", "W2"))
        g, u = x[r] @ W1.T, x[r] @ W3.T
        h_ref[r], o_ref[r] = g / (1 + torch.exp(-g)) * u, h[r] @ W2.T * w[r, None]
        g, u = x[r].double() @ W1.T.double(), x[r].double() @ W3.T.double()
        h64[r], o64[r] = g / (1 + torch.exp(-g)) * u, h[r].double() @ W2.T.double() * w[r, None].double()
    for got, ref in ((h, h_ref), (out, o_ref)):
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
        assert torch.equal(torch.sign(got[torch.isinf(got)]), torch.sign(ref[torch.isinf(ref)]))
    assert not torch.isfinite(out[[3, 20, 21, 110]]).any()
    plain = [i for i in range(T) if i not in (3, 20, 21, 40, 60, 61, 110)]
    assert torch.isfinite(h[plain]).all() and torch.isfinite(out[plain]).all()
    for rows in (plain, [60], [61]):
        assert rel_rms(h[rows].numpy(), h64[rows].numpy()) < 2e-6 and rel_rms(out[rows].numpy(), o64[rows].numpy()) < 2e-6, rows
    assert rel_rms(h[40][torch.isfinite(h_ref[40])].numpy(), h_ref[40][torch.isfinite(h_ref[40])].numpy()) < F32_REL_RMS


@pytest.mark.parametrize("counts,H,F", [([100, 40], 128, 256), ([100, 40, 70, 33, 64, 1, 128, 129], 128, 1024),
                                         ([36, 20, 70, 1, 64, 33, 65, 2], 128, 4224), ([150, 40, 9, 260], 256, 4224)])       # every kernel of gate/up
@pytest.mark.parametrize("sx,s1,s3,s2", [
    (-118, 50, 118, 0),                        # x: third parts below the last bit of a bf16 subnormal; sums of 2^-68 and of 1
    (-136, 120, 120, 0),                       # x: float32 subnormals, most of them no bf16 at all
    (50, -118, 0, 0),                          # W1
    (-59, 0, 0, 118),                          # h, in the down launch
    (-68, 0, 0, 120),                          # h: float32 subnormals
])
def test_f32_split_products_of_small_operands(counts, H, F, sx, s1, s3, s2):
    """Operands whose low parts no bf16 holds, against factors that make their sums ordinary numbers: as accurate as float32
    products.  Relative RMS below 2e-6: a chain of F / 4 = 1056 float32 roundings at most, 2^-24 * sqrt(1056 / 3) if they are
    random."""
    E = len(counts)
    cfg = MoEConfig("small32", "f32", T=sum(counts), H=H, F=F, E=E, k=1, page_bytes=96 * 1024, seed=84)
    inp = make_inputs(cfg, threads=16)
    for name, e in (("x", sx), ("W1", s1), ("W3", s3), ("W2", s2)):
        inp[name] = inp[name] * 2.0 ** e
    case = Case(cfg, inputs=inp)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    w = np.random.default_rng(3).random(cfg.T, dtype=np.float32) + 0.5
    h, out = M.moe_expert_ffn(case.shape, case.x, _dev_i32(offsets), case.pw.table_dev, case.pw.pages_dev, row_w=_dev_f32(w))
    h, out = h.cpu(), out.cpu()
    for e in range(E):
        r = slice(int(offsets[e]), int(offsets[e + 1]))
        g, u = inp["x"][r].double() @ inp["W1"][e].T.double(), inp["x"][r].double() @ inp["W3"][e].T.double()
        h_ref = g / (1 + torch.exp(-g)) * u
        o_ref = (h[r].double() @ inp["W2"][e].T.double()) * torch.from_numpy(w[r]).double()[:, None]
        h_rms = float(h_ref.square().mean().sqrt())
        # h itself may be a float32 subnormal: one unit of those, for the rounding of silu(g) and of the product
        assert float((h[r].double() - h_ref).square().mean().sqrt()) < 2e-6 * h_rms + 2.0 ** -149, f"h, expert {e}"
        assert rel_rms(out[r].numpy(), o_ref.numpy()) < 2e-6, f"out, expert {e}"


@pytest.mark.parametrize("counts,H,F", [([100, 40], 128, 256), ([100, 40, 70, 33, 64, 1, 128, 129], 128, 1024),
                                         ([36, 20, 70, 1, 64, 33, 65, 2], 128, 4224), ([150, 40, 9, 260], 256, 4224)])       # every kernel of gate/up
@pytest.mark.parametrize("scale", [float("inf"), float("nan"), 2.0 ** -45, 2.0 ** -100])
def test_f32_rows_do_not_depend_on_their_neighbours(counts, H, F, scale):
    """Rows of infinities, NaN or tiny values (2^-45: sums of the down launch alone) change no bit of h and out of any other row."""
    cfg = MoEConfig("neighbours32", "f32", T=sum(counts), H=H, F=F, E=len(counts), k=1, page_bytes=96 * 1024, seed=85)
    case = Case(cfg)
    offsets = _dev_i32(np.concatenate([[0], np.cumsum(counts)]))
    h0, out0 = M.moe_expert_ffn(case.shape, case.x, offsets, case.pw.table_dev, case.pw.pages_dev)
    rows = torch.tensor([3, 20, 21, 60, counts[0] + 1, sum(counts) - 1])
    x = case.x.clone()
    x[rows] *= scale
    h, out = M.moe_expert_ffn(case.shape, x, offsets, case.pw.table_dev, case.pw.pages_dev)
    others = torch.ones(sum(counts), dtype=torch.bool)
    others[rows] = False
    assert torch.equal(h.cpu()[others], h0.cpu()[others]) and torch.equal(out.cpu()[others], out0.cpu()[others])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,H,E,k", [(1, 128, 1, 1), (17, 128, 3, 3), (100, 384, 16, 4), (33, 1024, 17, 2), (250, 256, 32, 8),
                                     (47, 640, 33, 5), (130, 2048, 64, 64), (2000, 512, 8, 2)])
def test_router_shapes(T, H, E, k, dtype):
    # token counts off the 16-token blocks, fewer 64-element units than wavefronts, every expert-padding bound, a bias
    bias = ((0, 0.5), (E - 1, -0.25)) if E > 1 else ((0, 1.0),)
    cfg = MoEConfig("route", dtype, T=T, H=H, F=128, E=E, k=k, page_bytes=64 * 1024, seed=40 + E, bias=bias)
    case = Case(cfg)
    ref = case.oracle_route()
    ids, w, logits = M.moe_route(case.shape, case.x, case.Wr, bias=case.bias, want_logits=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(logits.cpu().numpy(), ref["logits"], rtol=0, atol=2e-5 * max(1.0, np.abs(ref["logits"]).max()))
    compare_routing(cfg, ids.cpu().numpy(), w.cpu().numpy(), ref)


@pytest.mark.parametrize("T", [256, 257, 511, 513, 1025, 2047, 3841, 4097])
@pytest.mark.parametrize("E,k", [(8, 2), (17, 3), (64, 8)])
def test_router_tokens_per_block(T, E, k):
    """Batches on both sides of one to sixteen tokens per block: against the oracle, and a token's logits, experts and weights are the
    bits that a batch of its first 100 tokens gives."""
    cfg = MoEConfig("tpb", "bf16", T=T, H=256, F=128, E=E, k=k, page_bytes=64 * 1024, seed=60 + E)
    case = Case(cfg)
    ref = case.oracle_route()
    ids, w, logits = M.moe_route(case.shape, case.x, case.Wr, want_logits=True)
    few = M.make_shape(100, 256, 128, E, k, "bf16", 64 * 1024)
    for at in (0, T - 100):
        sub = M.moe_route(few, case.x[at:at + 100].contiguous(), case.Wr, want_logits=True)
        torch.cuda.synchronize()
        for a, b in zip((ids, w, logits), sub):
            assert torch.equal(a[at:at + 100], b)
    np.testing.assert_allclose(logits.cpu().numpy(), ref["logits"], rtol=0, atol=2e-5 * max(1.0, np.abs(ref["logits"]).max()))
    compare_routing(cfg, ids.cpu().numpy(), w.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("E,k", [(1, 1), (5, 5), (8, 3), (17, 4), (64, 8)])
def test_router_selects_like_a_scan_with_ties_infinities_and_nan(E, k, dtype):
    """The selected experts are those of k scans over the logits that keep the first free one and replace it by what compares
    greater: the lower index of equal logits (repeated router rows), infinities, NaN only when no free expert precedes it."""
    T, H = 35, 128
    g = torch.Generator().manual_seed(E)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Wr = torch.randn(((E + 1) // 2, H), generator=g).to(dt).repeat(2, 1)[:E].contiguous()      # every logit twice
    x = torch.randn((T, H), generator=g).to(dt)
    bias = torch.zeros(E)
    for e, v in ((1, float("inf")), (3, float("-inf")), (4, float("nan")), (E - 1, float("-inf"))):
        if e < E:
            bias[e] = v
    s = M.make_shape(T, H, 128, E, k, dtype, 65536)
    for b in (None, bias, bias.roll(1), torch.full((E,), float("nan"))):
        ids, w, logits = M.moe_route(s, x.cuda(), Wr.cuda(), bias=None if b is None else b.cuda(), want_logits=True)
        lg, ids = logits.cpu().tolist(), ids.cpu().tolist()
        for t in range(T):
            free, want = list(range(E)), []
            for _ in range(k):
                best = free[0]
                for e in free:
                    if lg[t][e] > lg[t][best]:
                        best = e
                free.remove(best)
                want.append(best)
            assert ids[t] == want, (t, lg[t])
        if b is None:
            sel = torch.softmax(torch.gather(logits.cpu().double(), 1, torch.tensor(ids)), 1)
            assert (w.cpu().double() - sel).abs().max() <= 2e-6      # __expf and a reciprocal: a few units of 2^-23


@pytest.mark.parametrize("E", [1, 2, 5, 33, 64])
def test_permutation_leaves_out_ids_that_are_no_experts(E):
    k = min(E, 2)
    for T in (40, 1500, 9000):                                         # one block, blocks that count in place, a count launch
        rng = np.random.default_rng(T)
        ids = rng.integers(-2, E + 2, size=(T, k)).astype(np.int32)
        ids.reshape(-1)[:4] = (-1, 64, E, -2147483648)                 # the last three: the bits of experts in other ids
        pm = M.moe_permute(M.MoEShape(T, 128, 128, E, k, M.DTYPE_BF16, 16384), _dev_i32(ids))
        flat = ids.reshape(-1)
        ok = (flat >= 0) & (flat < E)
        counts = np.bincount(flat[ok], minlength=E)
        assert np.array_equal(pm["counts"].cpu().numpy(), counts)
        assert np.array_equal(pm["offsets"].cpu().numpy(), np.r_[0, np.cumsum(counts)])
        order = np.flatnonzero(ok)[np.argsort(flat[ok], kind="stable")]
        assert np.array_equal(pm["row_src"].cpu().numpy()[:ok.sum()], order)


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (1000, 1, 1), (512, 3, 2), (513, 3, 2), (4096, 8, 2), (16384, 64, 1),
                                   (5000, 16, 4), (40000, 64, 2), (131072, 8, 2), (140000, 5, 2)])
def test_permutation_block_counts(T, E, k):
    # one block (no count kernel), up to 256 blocks (each placing block sums the block counts), more (scan kernel)
    rng = np.random.default_rng(T + E)
    skew = rng.random(E) ** 3 + 1e-3                      # some experts rare, some popular
    ids = np.stack([rng.choice(E, size=k, replace=False, p=skew / skew.sum()) for _ in range(T)]).astype(np.int32)
    w = rng.random((T, k), dtype=np.float32)
    ref = oracle.permute(ids, E)
    s = M.MoEShape(T, 128, 128, E, k, M.DTYPE_BF16, 16384)
    pm = M.moe_permute(s, _dev_i32(ids), topk_w=_dev_f32(w))
    torch.cuda.synchronize()
    for name in ("counts", "offsets", "row_src", "row_of"):
        assert np.array_equal(pm[name].cpu().numpy(), ref[name]), name
    assert np.array_equal(pm["row_w"].cpu().numpy(), w.reshape(-1)[ref["row_src"]])


@pytest.mark.parametrize("T,E,k", [(300, 8, 2), (2500, 16, 4), (8192, 8, 2), (2048, 64, 8), (20000, 8, 2)])
def test_permutation_may_put_row_of_over_the_ids(T, E, k):
    rng = np.random.default_rng(T)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    ref = oracle.permute(ids, E)
    s = M.MoEShape(T, 128, 128, E, k, M.DTYPE_BF16, 16384)
    lib = M.binding._lib()
    both = _dev_i32(ids)
    counts, offsets, row_src = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E + 1, T * k))
    ws = torch.empty(max(M.workspace_layout(s).permute_bytes, 16), dtype=torch.uint8, device="cuda")
    rc = lib.moe_permute(ctypes.byref(s), both.data_ptr(), None, None, counts.data_ptr(), offsets.data_ptr(), row_src.data_ptr(), both.data_ptr(),
                         None, None, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0
    for name, t in (("counts", counts), ("offsets", offsets), ("row_src", row_src), ("row_of", both.reshape(-1))):
        assert np.array_equal(t.cpu().numpy(), ref[name]), name


def test_c1_stagewise_and_layer():
    case = Case(C1)
    ref = run_stagewise(case)
    run_layer(case, ref)


@pytest.mark.parametrize("name", list(MED))
@pytest.mark.parametrize("down_cols", [2, 1, 0])
def test_reduced_cases_stagewise_and_layer(name, down_cols):
    # 256- and 128-wide column tiles of the down projection (0: chosen by grid size)
    say(f"  case {name} down_cols {down_cols}")
    M.set_option("down_cols", down_cols)
    try:
        case = Case(MED[name], shuffle_pages=True, extra_pages=3)
        ref = run_stagewise(case)
        if name == "bf16_single_groups" and down_cols == 0:
            counts = ref["counts"].tolist()
            assert bf16_launches(counts, case.cfg.H, case.cfg.F) == ("whole", "128 columns", 0) and max(counts) > 512 and any(c > 256 and c % 256 <= 32 for c in counts)
        run_layer(case, ref)
    finally:
        M.set_option("down_cols", 0)


@pytest.mark.parametrize("name", ["bf16_top2_of_4", "bf16_two_experts_ragged", "f32_top2_of_5", "bf16_chunks_of_8", "bf16_chunks_of_32"])
@pytest.mark.parametrize("option,default,other", [("xcd_remap", 1, 0), ("fuse_gather", 1, 0), ("half_tiles", 1, 0), ("tall_tiles", 1, 0),
                                                  ("down_cols", 0, 1), ("down_cols", 0, 2), ("chunked", 32, 0), ("chunked", 32, 8),
                                                  ("tall_first", 1, 0), ("balance", 1, 0)])
def test_kernel_options_give_identical_bits(option, default, other, name):
    # which block computes which tile, the tile variant, and who gathers the rows of x do not change any arithmetic
    case = Case(MED[name])
    y1, ws = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, bias=case.bias)
    if name.startswith("bf16_chunks"):
        counts = ws.view("counts").cpu().tolist()
        whole, down, chunk = bf16_launches(counts, case.cfg.H, case.cfg.F)
        assert whole == "whole" and "halves" not in down and name.endswith("of_%d" % chunk) and max(counts) > 512
    M.set_option(option, other)
    try:
        y0, _ = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, bias=case.bias)
    finally:
        M.set_option(option, default)
    assert torch.equal(y0, y1)


@pytest.mark.parametrize("seed", range(8))
def test_random_shapes_and_routings_against_the_oracle(seed):
    # seeded random layer shapes with a random router bias (uneven segments of every length up to a few row tiles)
    rng = np.random.default_rng(1000 + seed)
    E = int(rng.integers(1, 13))
    k = int(rng.integers(1, min(E, 4) + 1))
    T = int(rng.integers(1, 1400))
    H = int(rng.choice([128, 256, 384]))
    F = int(rng.choice([128, 256, 640]))
    bias = tuple((e, float(rng.normal(0.0, 0.35))) for e in range(E)) if E > 1 else ()
    cfg = MoEConfig(f"rand{seed}", "bf16", T=T, H=H, F=F, E=E, k=k, page_bytes=int(rng.choice([16384, 49152, 65536])),
                    seed=50 + seed, bias=bias)
    say(f"    T={T} H={H} F={F} E={E} k={k} page={cfg.page_bytes}")
    case = Case(cfg, shuffle_pages=bool(seed & 1), extra_pages=seed % 3)
    y, ws = run_layer(case)
    say(f"    counts: {ws.view('counts').cpu().tolist()}")


def test_page_indirection_is_invisible():
    """Shuffling the physical page slots (table updated with them) leaves every bit of the output unchanged."""
    cfg = MED["bf16_top2_of_4"]
    a = Case(cfg)
    b = Case(cfg, shuffle_pages=True, extra_pages=7, inputs=a.inp)
    ya, _ = M.moe_layer(a.shape, a.x, a.Wr, a.pw.table_dev, a.pw.pages_dev)
    yb, _ = M.moe_layer(b.shape, b.x, b.Wr, b.pw.table_dev, b.pw.pages_dev)
    assert not torch.equal(a.pw.table_dev, b.pw.table_dev)
    assert torch.equal(ya, yb)
    # run-to-run bit identity (no order-dependent atomics anywhere on the path)
    ya2, ws = M.moe_layer(a.shape, a.x, a.Wr, a.pw.table_dev, a.pw.pages_dev)
    assert torch.equal(ya, ya2)


def test_non_resident_page_is_flagged_not_followed():
    cfg = MED["bf16_top2_of_4"]
    case = Case(cfg)
    table = case.pw.table_host.clone()
    table[1, 2] = -1
    with pytest.raises(M.MoEError) as ei:
        M.page_table_validate(case.shape, table, case.pw.pool_pages)
    assert ei.value.status == -4
    # the kernels guard the entry themselves: no fault, status bit set
    y, ws = M.moe_layer(case.shape, case.x, case.Wr, table.cuda(), case.pw.pages_dev)
    torch.cuda.synchronize()
    assert ws.view("status").cpu()[0].item() & 1 == 1
    table[1, 2] = case.pw.pool_pages + 5
    y, ws = M.moe_layer(case.shape, case.x, case.Wr, table.cuda(), case.pw.pages_dev)
    torch.cuda.synchronize()
    assert ws.view("status").cpu()[0].item() & 1 == 1


@pytest.mark.parametrize("kw", [
    dict(T=1), dict(T=5, k=1), dict(T=64, E=4, k=4), dict(T=257, E=1, k=1), dict(T=255, E=3, k=2),
    dict(T=513, E=2, k=2), dict(T=40, E=64, k=8, H=128, F=128),
], ids=lambda kw: "-".join(f"{a}{b}" for a, b in kw.items()))
def test_edge_shapes(kw):
    base = dict(T=64, H=256, F=256, E=8, k=2)
    base.update(kw)
    cfg = MoEConfig("edge", "bf16", page_bytes=64 * 1024, seed=31, **base)
    case = Case(cfg)
    ref = run_stagewise(case)
    run_layer(case, ref)


def test_empty_batch_is_a_noop():
    cfg = MoEConfig("empty", "bf16", T=0, H=128, F=128, E=4, k=2, page_bytes=16384, seed=1)
    s = shape_of(cfg)
    x = torch.empty((0, 128), dtype=torch.bfloat16, device="cuda")
    Wr = torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda")
    ids, w, _ = M.moe_route(s, x, Wr)
    assert ids.shape == (0, 2)
    pm = M.moe_permute(s, ids, x=x, topk_w=w)
    torch.cuda.synchronize()
    assert pm["counts"].cpu().tolist() == [0, 0, 0, 0] and pm["offsets"].cpu().tolist() == [0] * 5


def test_all_tokens_to_one_expert_and_empty_experts():
    cfg = MoEConfig("one", "bf16", T=300, H=256, F=256, E=4, k=1, page_bytes=64 * 1024, seed=33, bias=((2, 50.0),))
    case = Case(cfg)
    ref = run_stagewise(case)
    assert ref["counts"].tolist() == [0, 0, 300, 0]
    run_layer(case, ref)


def test_expert_with_more_row_tiles_than_the_tile_order_cuts_into_row_blocks():
    # 70000 of 70400 rows go to one expert: 273 row tiles, beyond the 256 up to which the tile order cuts an expert into row
    # blocks (it falls back to single column-tile groups there), next to experts with a handful of rows; the XCDs' shares
    # of such a launch differ, so blocks take tiles of other XCDs
    cfg = MoEConfig("tallest", "bf16", T=70400, H=128, F=128, E=4, k=1, page_bytes=16384, seed=35, bias=((1, 0.8),))
    case = Case(cfg)
    ref = run_stagewise(case)
    counts = ref["counts"].tolist()
    assert counts[1] > 256 * 256 and sum(counts) == 70400 and 0 < min(counts) < 2000, counts
    run_layer(case, ref)


def test_identical_experts_and_single_expert_invariants():
    """With identical experts the output does not depend on routing; with one expert the layer is a dense SwiGLU FFN."""
    cfg = MED["bf16_top2_of_4"]
    case = Case(cfg, identical_experts=True)
    y, _ = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev)
    Wr2 = torch.randn(case.Wr.shape, generator=torch.Generator().manual_seed(7)).to(torch.bfloat16).cuda()
    y2, ws2 = M.moe_layer(case.shape, case.x, Wr2, case.pw.table_dev, case.pw.pages_dev)
    dense_cfg = scaled(cfg, E=1, k=1)
    inp1 = {k: (v[:1].contiguous() if k in ("W1", "W3", "W2", "Wr") else v) for k, v in case.inp.items()}
    dense = Case(dense_cfg, inputs=inp1)
    yd, _ = M.moe_layer(dense.shape, dense.x, dense.Wr, dense.pw.table_dev, dense.pw.pages_dev)
    ref = dense.oracle_layer()
    assert_close(yd.cpu().numpy(), ref["y"], "bf16", "dense (E=1)")
    assert_close(y.cpu().numpy(), ref["y"], "bf16", "identical experts vs dense")
    assert_close(y2.cpu().numpy(), ref["y"], "bf16", "identical experts, other router")
    w = ws2.view("topk_w").cpu().numpy()
    np.testing.assert_allclose(w.sum(axis=1), 1.0, atol=1e-5)
    assert ws2.view("counts").cpu().numpy().sum() == cfg.T * cfg.k


@pytest.mark.parametrize("name,T", [("bf16_top4_of_16", 300),              # 75 rows per expert: the kernel for few rows
                                    ("bf16_top4_of_16_more_rows", 420),    # 105: the 256-row blocks
                                    ("f32_top2_of_5", 150),                # 60: the float32 kernel that splits the columns
                                    ("f32_top2_of_5", 40)])                # 16: the one that splits k
def test_streamed_pages_match_resident_pages_bitwise(name, T):
    cfg = scaled(MED[name], T=T)
    res = Case(cfg)
    y_res, ws_res = M.moe_layer(res.shape, res.x, res.Wr, res.pw.table_dev, res.pw.pages_dev)
    torch.cuda.synchronize()
    host = M.PagedWeights(res.shape, res.inp["W1"], res.inp["W3"], res.inp["W2"],
                          order=torch.Generator().manual_seed(3), extra_pages=4, pin=True)
    st = M.Streamer(res.shape, host.pages_host, host.table_host)
    try:
        for _ in range(2):          # the second call reuses slots that the first one filled
            ws_st = M.Workspace(res.shape)
            ws_st.buf.fill_(0xFF)                                             # NaN everywhere
            y_st, _ = M.moe_layer_streamed(st, res.x, res.Wr, workspace=ws_st)
            torch.cuda.synchronize()
            assert_status_clean(ws_st.view("status").cpu().tolist())
            assert torch.equal(y_st, y_res)
            if cfg.dtype == "f32":                                            # every expert's launch writes its rows of x_perm
                assert torch.equal(ws_st.view("x_perm"), res.x[ws_st.view("row_src").long() // cfg.k])
        x_perm = res.x[ws_res.view("row_src").long() // cfg.k].contiguous()   # moe_layer gathered inside its GEMM
        h, out = M.moe_expert_ffn_streamed(st, x_perm, ws_res.view("offsets"), row_w=ws_res.view("row_w"))
        torch.cuda.synchronize()
        assert torch.equal(out, ws_res.view("out")) and torch.equal(h, ws_res.view("h"))
    finally:
        st.close()
    ref = res.oracle_layer()
    assert_close(y_res.cpu().numpy(), ref["y"], cfg.dtype, "streamed case vs oracle")


@pytest.mark.parametrize("resident", ["none", "some", "all"])
@pytest.mark.parametrize("tokens", [96, 200])              # 48 and 100 rows per expert: either bf16 kernel
def test_multi_layer_weight_paging_matches_resident_layers_bitwise(resident, tokens):
    """Three layers, four micro-batches, two passes (the second starts with the first layer already
    prefetched): every output equals moe_layer on that layer's resident pages, bit for bit."""
    base = scaled(MED["bf16_top2_of_4"], T=tokens)
    s = shape_of(base)
    gu, d = M.pages_required(s)
    ppe = gu + d
    n_res = {"none": 0, "some": gu // 2 + 1, "all": ppe}[resident]
    L, n = 3, 4
    cases = [Case(scaled(base, seed=base.seed + 10 * l)) for l in range(L)]
    hosts = [M.PagedWeights(s, c.inp["W1"], c.inp["W3"], c.inp["W2"], order=torch.Generator().manual_seed(40 + l),
                            extra_pages=2, pin=True) for l, c in enumerate(cases)]
    g = torch.Generator().manual_seed(77)
    x_host = [[torch.randn((s.T, s.H), generator=g).to(torch.bfloat16).pin_memory() for _ in range(n)] for _ in range(L)]
    want = [[M.moe_layer(s, x_host[l][j].cuda(), cases[l].Wr, cases[l].pw.table_dev, cases[l].pw.pages_dev)[0]
             for j in range(n)] for l in range(L)]
    torch.cuda.synchronize()
    pipe = M.Pipeline(s, [(h.pages_host, h.table_host) for h in hosts], n_res, max_micro_batches=n)
    try:
        for rep in range(2):
            y = [[torch.zeros((s.T, s.H), dtype=torch.float32, device="cuda") for _ in range(n)] for _ in range(L)]
            ws = pipe.run(x_host, [c.Wr for c in cases], y)
            torch.cuda.synchronize()
            assert_status_clean(ws.view("status").cpu().tolist())
            for l in range(L):
                for j in range(n):
                    assert torch.equal(y[l][j], want[l][j]), (resident, rep, l, j)
    finally:
        pipe.close()
    ref = cases[0].oracle_layer()
    y0, _ = M.moe_layer(s, cases[0].x, cases[0].Wr, cases[0].pw.table_dev, cases[0].pw.pages_dev)
    assert_close(y0.cpu().numpy(), ref["y"], "bf16", "paging case, layer 0 vs oracle")


def test_layer_can_be_captured_in_a_hip_graph_and_replayed():
    """The layer call only launches kernels (status words are cleared by a kernel, not a memset), so it can be
    captured; every replay, with eager work in between, equals the eager result."""
    case = Case(MED["bf16_top2_of_4"])
    s = case.shape
    ws = M.Workspace(s)
    y = torch.empty((s.T, s.H), dtype=torch.float32, device="cuda")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        M.moe_layer(s, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y, stream=st)
        st.synchronize()
        want = y.clone()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            M.moe_layer(s, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y, stream=st)
        for rep in range(4):
            y.zero_()
            ws.buf.zero_()
            (case.x.float() @ case.x.float().T).sum().item()       # eager work and a synchronisation between replays
            g.replay()
            st.synchronize()
            assert torch.equal(y, want), rep


@pytest.mark.parametrize("non_temporal", [False, True])
@pytest.mark.parametrize("n16,blocks", [(1, 1), (1, 7), (1023, 1), (1025, 1), (4099, 3), (100000, 64)])
def test_stream_probe_reads_every_word_once(n16, blocks, non_temporal):
    # the probe folds what it reads into one word per lane and reports a single value: put it at the ends and around the unrolled stretch
    lib = M.binding._lib()
    fn = lib.moe_probe_stream_read_nt if non_temporal else lib.moe_probe_stream_read
    buf = torch.zeros(n16 * 4, dtype=torch.int32, device="cuda")
    sink = torch.zeros(1, dtype=torch.int32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for at in sorted({0, n16 // 2, n16 - 1, min(1024, n16 - 1)}):
        buf.zero_()
        sink.zero_()
        assert fn(buf.data_ptr(), n16 * 16, blocks, sink.data_ptr(), st) == 0
        assert sink.item() == 0
        buf[at * 4 + at % 4] = 0x5EEDF00D
        assert fn(buf.data_ptr(), n16 * 16, blocks, sink.data_ptr(), st) == 0
        assert sink.item() == 1
    assert fn(buf.data_ptr(), 8, blocks, None, st) == -1 and fn(buf.data_ptr() + 4, 16, 1, None, st) == -1
