// a3 and the dense linear map for launches with few rows per expert, bf16 operands, fp32 accumulation, on
// v_mfma_f32_16x16x32_bf16.  The launch is bound by reading every weight once, and what counts is how many bytes are under
// way and how short a block's way to its first load is.
//
// A block owns a row tile (16 * RT rows) x 16 * CW * FC columns (MODE 0: features, gate and up).  The CW wavefronts split the
// columns; a wavefront's 16 weight rows of a half-tile are 1 KiB in a row in the page, exactly one 16-byte load per lane and
// exactly its MFMA operand, so the weights go from the page straight into registers, D k-steps ahead (p.stream: with the
// non-temporal hint).  The activations, which all wavefronts share, are loaded as far ahead into registers and pass through a
// double-buffered LDS stage (one k-step, 128-byte rows, the chunk swizzle of moe_ffn_gemm_bf16.h), one barrier per k-step.
// All loads are the compiler's own, in one order, so its counted waits keep D - 1 k-steps under way across the barriers.
// Rows beyond the tile's last pair of 16-row MFMA tiles are neither loaded nor multiplied (a copy of the loop per pair:
// branches inside it would put an LDS latency in front of every MFMA).  Few registers and little LDS: two or more blocks share
// a compute unit and cover each other's start and end.
//
// FC = 1 in the linear map: a block's groups of 16 columns need not be a page tile's, every wavefront walks the tile of its own.
// RG > 1 (linear map): RG groups of CW wavefronts share the columns and split the row tiles.  Every output is the same chain of
// MFMAs along k as in moe_ffn_gemm_bf16.h: the same bits.
#include "moe_ffn_common.h"

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kComputeUnits = 256;                   // MI355X
constexpr int kHalfTileBytes = 128 * 64;             // 32 k of a page tile
constexpr int kTileBytes = 2 * kHalfTileBytes;

template <int N>
struct Num {
    static constexpr int value = N;
};

// FC: fragments of 16 columns per wavefront (MODE 0: of 16 features, gate and up)
template <int MODE, int RT, int CW, int FC, int RG, int D>
__global__ __launch_bounds__(64 * CW * RG) void ffn_rows_bf16(const GemmParams p) {
    constexpr int BM = 16 * RT, NB = MODE == 0 ? 2 * FC : FC, kCols = 16 * CW * FC;
    constexpr int kPass = 8 * CW * RG;               // rows that one load instruction per thread fetches
    constexpr int AJ = (BM + kPass - 1) / kPass, kStage = AJ * kPass * 128;
    static_assert(RT % 2 == 0 && RT <= 8 && (128 % kCols == 0 || (MODE == 1 && FC == 1)) && (kPass <= BM || RG == 1 || kPass >= 16 * RG), "");
    constexpr int kOutRow = kCols * 2 + 16;          // MODE 0: bytes of a row of h in LDS, 16 of padding
    constexpr int kSmem = MODE == 0 && BM * kOutRow > 2 * kStage ? BM * kOutRow : 2 * kStage;
    static_assert(MODE == 1 || RG == 1, "the row groups are the linear map's");
    __shared__ __attribute__((aligned(1024))) char smem[kSmem];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = RG == 1 ? wave : wave % CW, rg = RG == 1 ? 0 : wave / CW;
    const int r = lane & 15, g = lane >> 4;

    RowsTile tc;
    if (!locate_rows_tile<BM>(p, tc)) return;
    // diagnostic: some blocks report the shader clock they saw, as in moe_ffn_gemm_bf16.h
    const bool clock_probe = p.status && (blockIdx.x & 511) == 256 && threadIdx.x == 0;
    long long probe_c = 0, probe_w = 0;
    if (clock_probe) {
        probe_c = clock64();
        probe_w = wall_clock64();
    }
    const int nt = tc.nt, row0 = tc.row0, rows_here = tc.rows_here;
    const int32_t* trow = p.table + (size_t)(p.table_row_mod ? tc.e % p.table_row_mod : tc.e) * p.ppe + p.group_base;

    // activations: 16 bytes of rows tid / 8 + kPass * j
    uint32_t a_off[AJ];
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
        const int row = min(j * kPass + (tid >> 3), rows_here - 1);
        const int src = p.a_gather ? min(max(p.a_gather[row0 + row] / p.a_div, 0), p.a_rows - 1) : row;
        a_off[j] = (uint32_t)src * (uint32_t)p.lda_bytes + (tid & 7) * 16;
    }
    const char* a_base = p.a_gather ? p.A : p.A + (int64_t)row0 * p.lda_bytes;
    const int a_wr0 = (tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 4) & 7)) << 4);
    auto a_wr = [&](int j) __attribute__((always_inline)) { return (kPass % 16 ? a_wr0 ^ ((j & 1) << 6) : a_wr0) + j * kPass * 128; };     // kPass / 2 is 4 modulo 8 or 0
    const int a_rd[2] = {r * 128 + ((g ^ ((r >> 1) & 7)) << 4), r * 128 + (((4 + g) ^ ((r >> 1) & 7)) << 4)};

    // weights: one page tile is walked along k, MODE 0 two (the W1 and the W3 tile of the same features)
    int bad = 0, page, within, page1 = 0, within1 = 0;
    const char* tile[MODE == 0 ? 2 : 1];
    auto page_addr = [&](int pg) __attribute__((always_inline)) -> const char* {
        int slot = __builtin_amdgcn_readfirstlane(trow[pg]);
        if ((unsigned)slot >= (unsigned)p.pool_pages) {   // never follow an entry outside the pool
            bad = 1;
            slot = 0;
        }
        return p.pool + (int64_t)slot * p.page_bytes;
    };
    // MODE 1 with FC = 1: each wavefront has the page tile of its own 16 columns (a block may begin in one and end in the next)
    constexpr bool kOwn = MODE == 1 && FC == 1;
    constexpr int kColTiles = kOwn ? 1 : 128 / kCols;     // blocks per page tile along the columns
    const int group = kOwn ? min(nt * CW + cw, p.n_cols / 16 - 1) : 0;       // the last block may have wavefronts too many
    {
        const int t0 = kOwn ? (group >> 3) * p.KT : (nt / kColTiles) * (MODE == 0 ? 2 : 1) * p.KT;
        page = t0 / p.tpp;
        within = t0 - page * p.tpp;
        tile[0] = page_addr(page) + (int64_t)within * kTileBytes;
        if (MODE == 0) {
            page1 = (t0 + p.KT) / p.tpp;
            within1 = t0 + p.KT - page1 * p.tpp;
            tile[MODE == 0] = page_addr(page1) + (int64_t)within1 * kTileBytes;
        }
    }
    auto advance = [&]() __attribute__((always_inline)) {
        tile[0] += kTileBytes;
        if (++within == p.tpp) {
            within = 0;
            tile[0] = page_addr(++page);
        }
        if (MODE == 0) {
            tile[MODE == 0] += kTileBytes;
            if (++within1 == p.tpp) {
                within1 = 0;
                tile[MODE == 0] = page_addr(++page1);
            }
        }
    };
    const uint32_t b_off = ((kOwn ? (group & 7) * 16 : (nt % kColTiles) * kCols + cw * 16 * FC) + r) * 64 + ((g ^ ((r >> 2) & 2)) << 4);

    // row group rg: row tiles rg * (NRT / RG) ..
    constexpr int TPW = (RT + RG - 1) / RG;
    f32x4 acc[TPW][NB];
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    int tile0 = 0, tiles_mine = TPW;                 // this wavefront's first row tile and their number

    // the loop for NRT row tiles: rows beyond them are neither loaded nor multiplied
    auto main_loop = [&](auto stream_c, auto nrt_c) __attribute__((always_inline)) {
        constexpr bool STREAM = decltype(stream_c)::value;
        constexpr int NRT = decltype(nrt_c)::value, NA = (16 * NRT + kPass - 1) / kPass, NT = (NRT + RG - 1) / RG;
        static_assert(RG * NT * 16 <= AJ * kPass, "every row tile that is multiplied lies inside the stage");
        tile0 = rg * NT;
        tiles_mine = NT;
        i32x4 areg[D][NA], breg[D][2][NB];
        int kt_load = 0;                             // k-step that the next load_b fetches
        auto load_a = [&](int s, int slot) __attribute__((always_inline)) {
            const char* base = a_base + (int64_t)min(s, p.KT - 1) * 128;
#pragma unroll
            for (int j = 0; j < NA; ++j) areg[slot][j] = *(const i32x4*)(base + a_off[j]);
        };
        auto load_b = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const i32x4* src = (const i32x4*)(tile[MODE == 0 ? b / FC : 0] + (MODE == 0 ? b % FC : b) * 1024 + hp * kHalfTileBytes + b_off);
                    if constexpr (STREAM) breg[slot][hp][b] = __builtin_nontemporal_load(src);
                    else breg[slot][hp][b] = *src;
                }
            if (++kt_load < p.KT) advance();
        };
        int buf = 0;
        auto step = [&](int s, int slot, bool more) __attribute__((always_inline)) {     // slot: known at compile time
            char* st = smem + buf;
#pragma unroll
            for (int j = 0; j < NA; ++j) *(i32x4*)(st + a_wr(j)) = areg[slot][j];
            __syncthreads();
            if (more) load_a(s + D, slot);
            i32x4 a[2][NT];
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int i = 0; i < NT; ++i) a[hp][i] = *(const i32x4*)(st + a_rd[hp] + (tile0 + i) * 2048);
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[hp][i]), __builtin_bit_cast(bf16x8, breg[slot][hp][b]), acc[i][b], 0, 0, 0);
            if (more) load_b(slot);
            buf ^= kStage;
        };
#pragma unroll
        for (int u = 0; u < D; ++u) {
            load_a(u, u);
            load_b(u);
        }
        int s = 0;
        for (; s + 2 * D <= p.KT; s += D)
#pragma unroll
            for (int u = 0; u < D; ++u) step(s + u, u, true);
#pragma unroll
        for (int u = 0; u < 2 * D - 1; ++u)
            if (s + u < p.KT) step(s + u, u % D, s + u + D < p.KT);
    };
    auto run = [&](auto stream_c) __attribute__((always_inline)) {
        if (RT > 6 && rows_here > 96) main_loop(stream_c, Num<RT>{});
        else if (RT > 4 && rows_here > 64) main_loop(stream_c, Num<RT < 6 ? RT : 6>{});
        else if (RT > 2 && rows_here > 32) main_loop(stream_c, Num<RT < 4 ? RT : 4>{});
        else main_loop(stream_c, Num<2>{});
    };
    if (RG == 1 && p.stream && tc.mtiles == 1) run(Num<RG == 1>{});        // RG > 1: the linear map, never streamed
    else run(Num<0>{});

    if constexpr (MODE == 0) {
        // h leaves through LDS in whole lines, 16 bytes a lane, in part past the L2 (see kStreamRows)
        __syncthreads();                             // everyone has read the last stage
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i * 16 < rows_here)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int f = 0; f < FC; ++f)
                        *(__bf16*)(smem + (i * 16 + g * 4 + v) * kOutRow + (cw * 16 * FC + f * 16 + r) * 2) = (__bf16)silu_mul_bf16(acc[i][f][v], acc[i][NB - FC + f][v]);
        __syncthreads();
        constexpr int kChunks = kCols / 8;           // 16-byte chunks of a row
        char* o = (char*)p.out + ((int64_t)row0 * p.ldo + nt * kCols) * 2;
        auto store_rows = [&](auto past_l2) __attribute__((always_inline)) {
            for (int c = tid; c < rows_here * kChunks; c += 64 * CW * RG) {
                const int row = c / kChunks, ch = c % kChunks;
                const i32x4 hv = *(const i32x4*)(smem + row * kOutRow + ch * 16);
                i32x4* dst = (i32x4*)(o + (int64_t)row * p.ldo * 2 + ch * 16);
                if constexpr (decltype(past_l2)::value) {
                    __builtin_nontemporal_store(hv, dst);
                    asm volatile("" ::: "memory");       // else the compiler makes one store of this one and the plain one
                } else {
                    *dst = hv;
                }
            }
        };
        if (p.stream > 1 || (p.stream && tc.mtiles == 1)) store_rows(Num<1>{});
        else store_rows(Num<0>{});
    } else {
        const int col = nt * kCols + cw * 16 * FC + r;
        const bool mine = !kOwn || group == nt * CW + cw;
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = (tile0 + i) * 16 + g * 4 + v;
                if (row >= rows_here || !mine || (RG > 1 && i >= tiles_mine)) continue;
                const int64_t o = (int64_t)(row0 + row) * p.ldo + col;
                const float wgt = p.row_w ? p.row_w[row0 + row] : 1.0f;
#pragma unroll
                for (int f = 0; f < FC; ++f) {
                    const float y = acc[i][f][v] * wgt;
                    ((float*)p.out)[o + f * 16] = y;
                    if (p.out16) p.out16[o + f * 16] = (uint16_t)f32_to_bf16_bits(y);
                }
            }
    }
    if (clock_probe) {
        const long long dc = clock64() - probe_c, dw = wall_clock64() - probe_w;
        if (dw > 0) p.status[2 + MODE] = (int32_t)(dc * 100 / dw);       // MHz
    }
    if (bad && lane == 0 && p.status) atomicOr(p.status, 1);
}

template <int MODE, int RT, int CW, int FC, int RG, int D>
int launch_rows(GemmParams& p, int cols, int R, int n_exp, hipStream_t st) {
    p.NT = (cols / 16 + CW * FC - 1) / (CW * FC);
    hipLaunchKernelGGL((ffn_rows_bf16<MODE, RT, CW, FC, RG, D>), dim3(rows_grid(p.NT, R, 16 * RT, n_exp)), dim3(64 * CW * RG), 0, st, p);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

}  // namespace

// Where the expert GEMMs take this kernel: up to 80 rows per expert on average (of all experts: the launches of a streamed
// layer take what the resident layer's single launch takes).  us for the layer, moe_ffn_gemm_bf16.h's kernel / this one:
// Mixtral-8x7B shape (2 of 8 experts) 1 token 196 / 165, 4: 364 / 355, 16: 469 / 455, 64: 477 / 466, 150: 485 / 478, 256 (64
// rows each): 522 / 511, 288: 532 / 520, 400 (100 rows): 552 / 560; 64 experts of 2048 x 1024, 8 per token, 20 tokens 192 /
// 183, 400: 241 / 235, 600 (75 rows): 252 / 247, 777 (97 rows): 259 / 262; DBRX shape 120 tokens 1089 / 1036, 250: 1129 / 1096.
// What is left is the weights' way from HBM: with 4, 36 and 256 tokens of the Mixtral-8x7B shape 6.5, 6.7 and 5.8 TB/s in the
// gate/up launch, 6.2, 6.6 and 5.9 in the down launch, whatever the depth and the block.
// The average is all the host knows.  An expert with more rows than a block reads its weights once per row tile, 1.1 to 2.3 times
// over the fabric.  Skewed routing (40 % of the rows on one expert, or one expert with every token) is still 2 - 25 % faster this
// way; with every token on the same k experts two of the shapes lose, all other experts being empty: DBRX shape 80 tokens 395 /
// 439, 130: 452 / 534, 176: 470 / 563, 256: 521 / 539, 300: 674 / 649; Mixtral-8x22B shape 130 tokens 365 / 465, 200 and more: within 4 %
// (8x7B shape 130 tokens 284 / 265, 300: 382 / 320).
constexpr int kRowsKernelMax = 80;
// Up to here 64-row blocks with half the columns; 45 .. 72 rows need two of them per expert for some experts, and the second
// one reads the weights again (176 tokens of the Mixtral-8x7B shape, 44 rows: 489 against 503 with 128-row blocks).
constexpr int kRows64Max = 44;

bool rows_kernel_takes(int rows_each) { return rows_each <= kRowsKernelMax; }

int launch_gate_up_rows_bf16(GemmParams& p, int F, int R, int rows_each, int n_exp, hipStream_t st) {
    if (rows_each <= kRows64Max) return launch_rows<0, 4, 4, 1, 1, 4>(p, F, R, n_exp, st);
    return launch_rows<0, 8, 8, 1, 1, 2>(p, F, R, n_exp, st);
}

int launch_down_rows_bf16(GemmParams& p, int H, int R, int rows_each, int n_exp, hipStream_t st) {
    if (rows_each <= kRows64Max) return launch_rows<1, 4, 4, 2, 1, 4>(p, H, R, n_exp, st);
    return launch_rows<1, 8, 8, 1, 1, 4>(p, H, R, n_exp, st);
}

// The dense linear map (moe_host.h: linear_takes_rows_kernel says when it comes here, linear_rows_block with which blocks).  A compute unit has some 110 lines under way; a line from HBM holds its place for about
// 0.55 us, one from the L2 for 0.13, so a compute unit brings 25 GB/s of the one or 110 GB/s of the other, and the launch wants every
// compute unit to take an equal share.  With one and two groups the wavefronts split the rows too (their weights meet in the L1); three
// groups with two row groups each lost 1 - 2 us with weights from HBM (4096 x 6144 100 tokens 22.8 / 24.0).  More groups with row groups: 20 - 40 % slower.
// us for the launch, the blocks before (32 columns, or 64, or 128 rows x 64 columns) / these, weights where the call before left them | from HBM: 4096 x 4096
// 36 tokens 16.7 / 15.7 | 18.1 / 17.1, 100: 20.1 / 16.9 | 21.8 / 18.5; 4096 x 6144 160: 27.6 / 22.2 | 29.3 / 24.5, 256: 28.2 / 24.0 | 38.3 / 30.1; 6144 x 9216 100: 38.7 / 31.9 | 52.3 /
// 37.7; 2048 x 3072 100: 12.3 / 10.3 | 12.9 / 10.7, 400: 17.0 / 14.7 | 17.0 / 14.9; 4096 x 512 4000: 46.2 / 27.2; 512 x 512 300: 6.6 / 5.0; equal where the blocks are what they
// were (4096 x 6144 100: 64 columns).  Up to 64 rows four groups are the most: more
// columns per block only leave compute units idle (6144 x 9216 40 tokens 29.1 / 27.4).
// Temporal loads, us without / with the non-temporal hint, weights where the call before left them (one matrix fits the 256 MiB
// last-level cache) | weights from HBM: 4096 x 6144 64 tokens 17 / 21 | 21 / 22; 6144 x 9216 64 tokens 30 / 35 | 38 / 37, 128: 40 /
// 59 | 58 / 60 (with the blocks before).
// Groups of wavefronts that split k change the order of the sums, which the O projection hands on to a rounding and the router: left out.  So are
// two k-steps behind one barrier: within 5 % either way, the barriers are not what the launch waits for.
int launch_linear_rows_bf16(GemmParams& p, int N, int T, hipStream_t st) {
    const LinearBlock b = linear_rows_block(T, p.KT * kTileK, N);
    if (b.rows == 128) return launch_rows<1, 8, 4, 1, 2, 4>(p, N, T, 1, st);
    if (b.rows == 32) return b.groups == 1 ? launch_rows<1, 2, 1, 1, 2, 8>(p, N, T, 1, st) : launch_rows<1, 2, 2, 1, 2, 8>(p, N, T, 1, st);
    switch (b.groups) {
        case 1: return launch_rows<1, 4, 1, 1, 4, 8>(p, N, T, 1, st);
        case 2: return launch_rows<1, 4, 2, 1, 2, 6>(p, N, T, 1, st);
        case 4: return launch_rows<1, 4, 4, 1, 1, 4>(p, N, T, 1, st);
        case 5: return launch_rows<1, 4, 5, 1, 1, 4>(p, N, T, 1, st);
        case 6: return launch_rows<1, 4, 6, 1, 1, 4>(p, N, T, 1, st);
        default: return launch_rows<1, 4, 8, 1, 1, 4>(p, N, T, 1, st);
    }
}

}  // namespace moe
