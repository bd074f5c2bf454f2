// a3, bf16 operands: which kernel a launch of the expert FFN or of the dense linear map takes.
#include "moe_ffn_gemm_bf16.h"

namespace moe {

int launch_expert_ffn_bf16(const moe_shape& s, const Geom& g, const FfnArgs& a, hipStream_t st) {
    const int R = s.T * s.k;
    const int n_exp = a.e_end - a.e_begin;
    GemmParams p{};
    fill_common(p, s, g, a);
    fill_gate_up(p, s, g, a);
    const int64_t rows_each = R / s.E;
    const bool streams = rows_each <= kStreamRows && (int64_t)s.E * 3 * s.H * s.F * 2 > kStreamBytes;
    p.stream = !streams ? 0 : s.F >= 6144 && s.E * g.dt >= kComputeUnits ? 2 : 1;       // 2: h of every expert past the L2 as well
    if (rows_kernel_takes((int)rows_each)) {
        int rc = thin_takes_gate_up(s) ? launch_gate_up_thin_bf16(p, s.F, R, n_exp, st) : launch_gate_up_rows_bf16(p, s.F, R, (int)rows_each, n_exp, st);
        if (rc != MOE_OK) return rc;
        if (a.mid_event) MOE_HIP_TRY(hipEventRecord(a.mid_event, st));
        fill_down(p, s, g, a);
        return thin_takes_down(s) ? launch_down_thin_bf16(p, s.H, R, n_exp, st) : launch_down_rows_bf16(p, s.H, R, (int)rows_each, n_exp, st);
    }
    const int64_t row_tiles_each = std::max<int64_t>(1, (rows_each - p.tall_rows + BM - 1) / BM);
    // A last round that is at most half full, by the tiles that an even split of the rows over the experts would give: its tiles are
    // computed in halves (the kernel goes by the tiles there are).  us for the launch, whole tiles / halves: DBRX shape 600 tokens gate/up (5.25 rounds) 711 / 698, down
    // (1.5) 416 / 393, 900 tokens 879 / 868 and 495 / 464; Mixtral-8x22B shape 1500 tokens down (1.5) 706 / 653, 3000 (2.25) 1035 / 957; 1024 x 2816, 6000 tokens gate/up
    // (4.1) 145 / 139; Mixtral-8x7B shape 1000 tokens gate/up (3.5) 402 / 404: on half of the compute units whole tiles get the memory, and
    // the power, of the others, and where the weights stream that is all that halves could win.
    auto half_round = [&]() {
        const int64_t last = n_exp * row_tiles_each * p.NT % kComputeUnits;
        return last != 0 && last <= kComputeUnits / 2;
    };
    const int rc = half_round() ? launch_gate_up_halves_bf16(p, R, n_exp, st) : launch_stages<0, 2>(p, R, n_exp, st);
    if (rc != MOE_OK) return rc;
    if (a.mid_event) MOE_HIP_TRY(hipEventRecord(a.mid_event, st));
    fill_down(p, s, g, a);
    // Down projection with few row tiles: 256-wide column tiles would leave compute units without a block, so the columns are cut
    // into 128-wide tiles as long as these make no more than one round.  The routing result is not known here; the choice
    // goes by the row tiles an even split of the rows over the experts would give (the grid is sized by the
    // upper bound as ever).  us for the launch, narrow / wide: Mixtral-8x7B shape 1000 tokens (256 narrow tiles) 247 / 312, 1200 (512) 453 / 367;
    // Mixtral-8x22B shape 600 tokens (384) 384 / 295, 1000: 472 / 377; 2048 x 4096 1500 tokens (256) 74 / 92, 2500 (384) 108 / 95; 1024 x 2816
    // 2000 tokens (128) 55 / 69; DBRX shape 600 tokens (768) 435 / 405.
    // down_cols: 0 = this rule, 1 / 2 = force 128 / 256 columns.
    const int opt = get_opt(OPT_DOWN_COLS);
    const int64_t narrow_tiles = n_exp * row_tiles_each * (int64_t)g.dt;
    // Where even these are at most half a round: 64-wide ones, as long as the tiles that the routing makes are at most half a round
    // (an expert with 40 % of the rows: 2048 x 4096, 1024 tokens 208 tiles, 65 us whole and 82 if halved).  us for the launch, 128 / 64 wide: 2048 x 4096 500 tokens (128
    // tiles) 52 / 44, 1024: 73 / 65; 1024 x 2816 500 tokens (64) 30 / 25, 1024: 41 / 35, 1500 (128): 36 / 32; more tiles, halved all the same: 2048 x 4096 1400 tokens (256) 60 / 80.
    if (opt == 1 || (opt == 0 && narrow_tiles <= kComputeUnits)) {
        p.NT = (int32_t)g.dt;
        if (narrow_tiles <= kComputeUnits / 2) return launch_down_narrow_halves_bf16(p, R, n_exp, st);
        return launch_stages<1, 1>(p, R, n_exp, st);
    }
    return half_round() ? launch_down_halves_bf16(p, R, n_exp, st) : launch_stages<1, 2>(p, R, n_exp, st);
}

// y = x W^T for a dense weight matrix held as pages: one of the two down-projection kernels (linear_takes_rows_kernel in
// moe_host.h) with one "expert" that owns all T rows and no row weight.
int launch_linear_bf16(const LinearArgs& a, hipStream_t st) {
    GemmParams p{};
    p.A = (const char*)a.x;
    p.lda_bytes = (int64_t)a.K * 2;
    p.dense_rows = a.T;
    p.table = a.page_table;
    p.pool = a.pool;
    p.page_bytes = a.page_bytes;
    p.tile_bytes = (int64_t)kTileN * kTileK * 2;
    p.pool_pages = (int32_t)std::min<int64_t>(a.pool_pages, 0x7fffffff);
    p.tpp = (int32_t)(a.page_bytes / p.tile_bytes);
    p.ppe = (int32_t)a.pages;
    p.group_base = 0;
    p.KT = a.K / kTileK;
    p.n_page_tiles = a.N / kTileN;
    p.e_begin = 0;
    p.e_end = 1;
    p.table_row_mod = 0;
    p.out = a.out;
    p.ldo = a.N;
    p.n_cols = a.N;
    p.row_w = nullptr;
    p.status = a.status;
    p.xcd_remap = get_opt(OPT_XCD_REMAP);
    p.half_tiles = get_opt(OPT_HALF_TILES);
    p.tall_rows = get_opt(OPT_TALL_TILES) ? 32 : 0;
    p.tall_first = get_opt(OPT_TALL_FIRST);
    p.balance = get_opt(OPT_BALANCE);
    p.chunked = std::min(std::max(get_opt(OPT_CHUNKED), 0), 32);
    if (linear_takes_rows_kernel(a.T, a.K, a.N)) {
        p.out16 = a.out16;
        return launch_linear_rows_bf16(p, a.N, a.T, st);
    }
    const int wide_tiles = (p.n_page_tiles + 1) / 2;
    int rc;
    if ((int64_t)(a.T / BM + 1) * wide_tiles < 2 * kComputeUnits) {       // too few 256-wide tiles to fill the chip
        p.NT = p.n_page_tiles;
        // Row tiles of 128 as long as they make one round: a tile of 256 rows x 128 columns is a chain of some 0.6 us per k-step
        // whatever else the chip does, one of 128 rows 0.4.  us for the pre-attention task, 256 / 128 rows: 4096 x 6144 512
        // tokens (192 tiles of 128) 56 / 46; 6144 x 9216 256 tokens (144) 72 / 57; 2048 x 3072 700 tokens (144) 38 / 34,
        // 1000 (192) 40 / 34.  With up to 160 rows, a short tile of 256, they read the weights twice to have twice the blocks, which wide
        // matrices with a long k do not win back: 129 rows, 4096 x 13312 (208 tiles of 128) 37 / 34, 4096 x 14336 (224) 37 / 37, 4096 x 15360 (240) 37 / 38, 4096 x
        // 16384 (256) 35 / 40, 6144 x 13312 50 / 50, 6144 x 16384 47 / 55, but 2048 x 16384 21.4 / 20.4; 161 rows 4096 x 16384 39 / 36.
        // Not for the experts' down launch, whose experts are a tile each and would read their weights twice: 2048 x 4096 1024
        // tokens 70 us for the launch, 86 with tiles of 128.
        const int64_t half_tiles = (int64_t)((a.T + 127) / 128) * p.NT;
        if (p.half_tiles && a.T > 128 && half_tiles <= kComputeUnits && (a.T > 160 || half_tiles <= 224 || p.KT <= 32)) {
            p.tall_rows = 0;
            rc = launch_stages<1, 1, 128>(p, a.T, 1, st);
        } else {
            rc = launch_stages<1, 1>(p, a.T, 1, st);
        }
    } else {
        p.NT = wide_tiles;
        rc = launch_stages<1, 2>(p, a.T, 1, st);
    }
    if (rc != MOE_OK || !a.out16) return rc;
    return launch_cast_bf16((int64_t)a.T * a.N, a.out, a.out16, st);
}


}  // namespace moe
