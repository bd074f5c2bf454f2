"""GPU parity at the full workload sizes, in the launch configuration the
benchmark times (the fused moe_layer call).  Routing and permutation are compared
in full (they are cheap).  The expert FFN and the output are compared with the
oracle in full on the 256-token workload, and on the larger ones on at least 1024
tokens taken at a stride over the micro-batch plus the rows that make sure every
(expert, row tile) pair is covered: the first and the last row of every row
tile, of a tall row tile also the first of its rows beyond 256, and every row of
an expert with fewer than 256 rows.  Outputs and intermediates are filled with NaN before the call, so a tile
that was never written cannot pass as stale finite data."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2411_11217_amd as M
from moe_workloads import CONFIGS, prompt_lengths, scaled
from util import Case, assert_close, assert_h_close, check_permutation_valid, compare_routing, say, shape_of, assert_status_clean

pytestmark = pytest.mark.gpu

ROW_TILE, TALL = 256, 32


def row_tiles(n):
    """(first row, rows) of the row tiles the expert GEMMs cut a segment of n rows into, as include/moe.h documents it
    for the option "tall_tiles": q full tiles of 256 rows and a remainder r; when 0 < r <= 32 q the remainder rides along
    with the last m tiles (each 256 + r / m rows high, the first r % m of them one more), m = ceil(r / 16) if there are
    that many tiles, else ceil(r / 32); otherwise it is a tile of its own.  Only used to aim the sample, never to
    compute a value."""
    q, r = divmod(n, ROW_TILE)
    if not M.get_option("tall_tiles") or q == 0 or r == 0 or r > TALL * q:
        return [(a, min(ROW_TILE, n - a)) for a in range(0, n, ROW_TILE)]
    m = (r + 15) // 16
    if m > q:
        m = (r + TALL - 1) // TALL
    base, more = ROW_TILE + r // m, r % m
    tiles = [(i * ROW_TILE, ROW_TILE) for i in range(q - m)]
    a = (q - m) * ROW_TILE
    for i in range(m):
        rows = base + (1 if i < more else 0)
        tiles.append((a, rows))
        a += rows
    assert a == n
    return tiles


def sample_rows_of_tiles(ref_pm, E):
    """For every (expert, row tile): its first and last row, and of a tall tile also the first row beyond 256.
    An expert with fewer than 256 rows gives all its rows.  -> (rows, set of (expert, tile index, part))"""
    offsets = ref_pm["offsets"]
    rows, wanted = [], set()
    for e in range(E):
        lo, n = int(offsets[e]), int(offsets[e + 1]) - int(offsets[e])
        if 0 < n < ROW_TILE:
            rows.extend(range(lo, lo + n))
        for i, (a, cnt) in enumerate(row_tiles(n)):
            rows.extend([lo + a, lo + a + cnt - 1])
            wanted.add((e, i, "body"))
            if cnt > ROW_TILE:
                rows.extend([lo + a + ROW_TILE, lo + a + cnt - 1])
                wanted.add((e, i, "extra rows"))
    return np.array(sorted(set(rows)), dtype=np.int64), wanted


def covered_tiles(rows, ref_pm, E):
    """The (expert, tile index, part) triples that the compared rows fall into."""
    offsets = ref_pm["offsets"]
    got = set()
    for e in range(E):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        mine = rows[(rows >= lo) & (rows < hi)] - lo
        for i, (a, cnt) in enumerate(row_tiles(hi - lo)):
            inside = mine[(mine >= a) & (mine < a + cnt)] - a
            if (inside < ROW_TILE).any():
                got.add((e, i, "body"))
            if (inside >= ROW_TILE).any():
                got.add((e, i, "extra rows"))
    return got


def sample_tokens(cfg, ref_pm, min_tokens=1024):
    """Token indices to compare: all of them up to min_tokens; beyond, a stride over T giving at least min_tokens, plus
    the tokens behind the rows of sample_rows_of_tiles."""
    T, k = cfg.T, cfg.k
    if T <= min_tokens:
        return np.arange(T, dtype=np.int32)
    toks = set(range(0, T, max(1, T // min_tokens)))
    toks.add(T - 1)
    rows, _ = sample_rows_of_tiles(ref_pm, cfg.E)
    toks.update((ref_pm["row_src"][rows] // k).tolist())
    return np.array(sorted(toks), dtype=np.int32)


def nan_filled_outputs(case: Case):
    """A workspace whose intermediates h and out, and an output y, all hold NaN."""
    cfg = case.cfg
    ws = M.Workspace(case.shape)
    ws.view("h").fill_(float("nan"))
    ws.view("out").fill_(float("nan"))
    y = torch.full((cfg.T, cfg.H), float("nan"), dtype=torch.float32, device="cuda")
    return ws, y


def check_full(case: Case, y: torch.Tensor, ws, label: str):
    cfg = case.cfg
    t0 = time.time()
    rt = case.oracle_route()
    say(f"    oracle route: {time.time() - t0:.1f}s")
    ids = ws.view("topk_ids").cpu().numpy()
    w = ws.view("topk_w").cpu().numpy()
    same = compare_routing(cfg, ids, w, rt, label + " route")
    pm_gpu = {n: ws.view(n).cpu().numpy() for n in ("counts", "offsets", "row_src", "row_of")}
    check_permutation_valid(ids, cfg.E, cfg.k, pm_gpu)
    pm_ref = oracle.permute(ids, cfg.E)                    # the oracle's permutation of the ids the GPU chose
    for n in pm_ref:
        assert np.array_equal(pm_gpu[n], pm_ref[n]), n
    say(f"    counts: {pm_gpu['counts'].tolist()}")
    assert pm_gpu["counts"].sum() == cfg.T * cfg.k
    assert_status_clean(ws.view("status").cpu().tolist())
    # every element of the output and of both intermediates was written (they held NaN before the call)
    assert not bool(torch.isnan(y).any()), label + ": y has elements the layer never wrote"
    assert not bool(torch.isnan(ws.view("out")).any()), label + ": out has rows the down GEMM never wrote"
    assert not bool(torch.isnan(ws.view("h")).any()), label + ": h has elements the gate/up GEMM never wrote"
    yh = y.cpu().numpy()
    assert np.isfinite(yh).all()

    toks = sample_tokens(cfg, pm_ref)
    n_sampled = len(toks)
    toks = toks[same[toks]]                                # near-tie tokens are reported above, not compared
    t0 = time.time()
    v = case.view
    flat = (toks[:, None].astype(np.int64) * cfg.k + np.arange(cfg.k)[None, :]).reshape(-1)
    rows = pm_ref["row_of"][flat]
    # coverage of the sample: every (expert, row tile) pair has a compared row, a tall tile also among its extra rows
    _, wanted = sample_rows_of_tiles(pm_ref, cfg.E)
    missing = wanted - covered_tiles(rows, pm_ref, cfg.E)
    assert len(missing) <= 2 * int((~same).sum()), sorted(missing)[:5]      # only a near-tie token may take a tile's row away
    xp = oracle.gather_rows(v["x"], pm_ref["row_src"], cfg.k, cfg.dtype_code)
    h_ref, o_ref = oracle.expert_ffn(xp, pm_ref["offsets"], v["W1"], v["W3"], v["W2"], cfg.dtype_code, sel=rows)
    # gate weights of the sampled tokens in the GPU's slot order (same expert set as the oracle's)
    w_ref = np.zeros((len(toks), cfg.k))
    for i, t in enumerate(toks):
        lookup = {int(e): rt["w"][t, s] for s, e in enumerate(rt["ids"][t])}
        w_ref[i] = [lookup[int(e)] for e in ids[t]]
    y_ref = oracle.combine(o_ref, np.arange(rows.shape[0], dtype=np.int32), cfg.k, w=w_ref)
    say(f"    oracle FFN on {len(toks)} of {n_sampled} sampled tokens ({rows.shape[0]} rows covering {len(wanted)} (expert, row tile) "
        f"parts): {time.time() - t0:.1f}s")
    rows_t = torch.from_numpy(rows.astype(np.int64)).cuda()
    if not M.get_option("fuse_gather"):                    # else the gate/up GEMM gathers the rows, and h below covers them
        assert_close(ws.view("x_perm")[rows_t].float().cpu().numpy(),
                     torch.from_numpy(xp[rows].view(np.int16)).view(torch.bfloat16).float().numpy(), "f32", label + " x_perm rows")
    assert_h_close(ws.view("h")[rows_t].float().cpu().numpy(), h_ref, cfg.dtype, label + " h rows")
    rw = ws.view("row_w")[rows_t].cpu().numpy().astype(np.float64)
    assert_close(ws.view("out")[rows_t].cpu().numpy(), o_ref * rw[:, None], cfg.dtype, label + " out rows")
    assert_close(yh[toks], y_ref, cfg.dtype, label + " y (sampled tokens)")


@pytest.mark.parametrize("name", ["c2_mixtral8x7b_t256", "c3_mixtral8x7b_t4096"])
def test_mixtral_8x7b_shapes(name):
    # the two workloads share the layer shape; they differ in seed and token count
    cfg = CONFIGS[name]
    t0 = time.time()
    case = Case(cfg)
    say(f"    inputs + pages ready: {time.time() - t0:.1f}s")
    ws, y = nan_filled_outputs(case)
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
    torch.cuda.synchronize()
    check_full(case, y, ws, name)


def test_mixtral_8x7b_t256_with_the_row_copy():
    # the layer with x_perm written by the permutation step and read by the gate/up GEMM
    cfg = CONFIGS["c2_mixtral8x7b_t256"]
    case = Case(cfg)
    M.set_option("fuse_gather", 0)
    try:
        ws, y = nan_filled_outputs(case)
        M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
        torch.cuda.synchronize()
        check_full(case, y, ws, cfg.name + " fuse_gather=0")
    finally:
        M.set_option("fuse_gather", 1)


@pytest.mark.parametrize("T", [512, 1024, 1536, 2048])
def test_mixtral_8x7b_around_the_ridge(T):
    # micro-batch sizes on both sides of the point where a kernel execution turns compute bound (about 1000 tokens
    # for this shape): the down launch takes its narrow column tiles up to 1024 tokens and the wide ones beyond, the
    # experts have one to three row tiles, some of them tall, and the tile order switches its chunks on
    cfg = scaled(CONFIGS["c3_mixtral8x7b_t4096"], name=f"ridge_t{T}", T=T)
    case = Case(cfg)
    ws, y = nan_filled_outputs(case)
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
    torch.cuda.synchronize()
    check_full(case, y, ws, cfg.name)


@pytest.fixture(scope="module")
def mixtral_8x7b_t700():
    return Case(scaled(CONFIGS["c3_mixtral8x7b_t4096"], name="few_rows", T=700))


@pytest.mark.parametrize("T", [4, 100, 160, 400, 580, 700])
def test_mixtral_8x7b_with_one_row_tile_per_expert(mixtral_8x7b_t700, T):
    # the weights exceed the last-level cache and the experts have one row tile each: the kernels' loops with non-temporal
    # weight loads.  1, 25 and 40 rows per expert on average: the blocks of 64 rows of the kernel for few rows, with one and
    # two pairs of row tiles; 100, 145 and 175: the short loops of the 256-row blocks with four, five and six row tiles
    import copy
    case = copy.copy(mixtral_8x7b_t700)
    case.cfg = scaled(case.cfg, name=f"few_rows_t{T}", T=T)
    case.shape = shape_of(case.cfg)
    case.x = case.x[:T].contiguous()
    case.view = dict(case.view, x=case.view["x"][:T])
    ws, y = nan_filled_outputs(case)
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
    torch.cuda.synchronize()
    check_full(case, y, ws, case.cfg.name)


def test_mixtral_8x7b_prefill_micro_batch():
    # a prefill micro-batch as the request batching forms it from a seeded prompt-length mix (average 77, maximum
    # 418, 128 requests per micro-batch): a token count that none of the tile sizes divides
    from paper_2411_11217_amd.batching import Request, batch_requests
    lens = prompt_lengths(1024, seed=2)
    mbs, aborted = batch_requests([Request(i, int(v)) for i, v in enumerate(lens)], 8, 128, gen_len=128, cache_size=1 << 40)
    assert not aborted and len(mbs) == 8
    tokens = [mb.prompt_tokens for mb in mbs]
    assert max(tokens) - min(tokens) <= 418 and sum(tokens) == int(lens.sum())
    T = next(t for t in tokens if t % 256 != 0)
    cfg = scaled(CONFIGS["c3_mixtral8x7b_t4096"], name="prefill_micro_batch", T=T)
    say(f"    micro-batch tokens: {tokens}, running T={T}")
    case = Case(cfg)
    ws, y = nan_filled_outputs(case)
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, workspace=ws, y=y)
    torch.cuda.synchronize()
    check_full(case, y, ws, cfg.name)


def test_mixtral_8x22b_skewed():
    cfg = CONFIGS["c4_mixtral8x22b_t8192_skew"]
    t0 = time.time()
    case = Case(cfg)
    say(f"    inputs + pages ready: {time.time() - t0:.1f}s")
    ws, y = nan_filled_outputs(case)
    M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev, bias=case.bias, workspace=ws, y=y)
    torch.cuda.synchronize()
    share = ws.view("counts").cpu().numpy() / float(cfg.R)
    assert 0.38 <= share[0] <= 0.42 and 0 < share[7] < 0.02, share
    check_full(case, y, ws, cfg.name)


def test_dbrx_streamed_from_pinned_host():
    cfg = CONFIGS["c5_dbrx_t16384_streamed"]
    t0 = time.time()
    case = Case(cfg, pin_pages=True)
    say(f"    inputs + pinned pages ready: {time.time() - t0:.1f}s")
    st = M.Streamer(case.shape, case.pw.pages_host, case.pw.table_host)
    try:
        ws, y = nan_filled_outputs(case)
        M.moe_layer_streamed(st, case.x, case.Wr, workspace=ws, y=y)
        torch.cuda.synchronize()
        check_full(case, y, ws, cfg.name)
        # the same layer with every page resident gives the same bits
        case.pw.to_device(keep_host=True)
        y_res, _ = M.moe_layer(case.shape, case.x, case.Wr, case.pw.table_dev, case.pw.pages_dev)
        torch.cuda.synchronize()
        assert torch.equal(y, y_res)
    finally:
        st.close()
