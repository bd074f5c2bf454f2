// a3 for float32 storage: the same grouped SwiGLU FFN over the same page format, on v_mfma_f32_16x16x4_f32 (256 FLOP per
// clock and compute unit, a sixteenth of the bf16 rate: with more than a few rows per expert the matrix cores are the bound,
// 157 TFLOP/s nominal; with fewer it is the weights' way from HBM).
//
// In both kernels a lane's share of an operand is a 16-byte chunk (four consecutive k of one row): lane l holds chunk
// 4q + l / 16 of row l % 16, and four MFMAs take one element of the four each, so that MFMA j adds the k = 16q + 4g + j
// (g = 0 .. 3).  Activations and weights use the same map, so no element needs to move between lanes.  The weight chunks go
// from the page straight into registers: a weight element is used by one wavefront alone, LDS would only cost a round trip.
//
//   ffn_rows_f32: a block owns 32 rows x 64 columns (MODE 0: 64 features, gate and up).  The four wavefronts split the
//     columns and share the activations, which go through LDS (two stages of one 64-wide k-step; the registers hold the
//     next one), one barrier per k-step.  17 KiB of LDS and few registers: four and more blocks share a compute unit, hide
//     each other's latency and keep the end of a launch short (a k-step is 64 MFMAs of 32 cycles per wavefront in MODE 0).
//     Blocks of 64 rows read the weights half as often and were slower up to thousands of tokens, 32 / 64 rows, us for the
//     layer of 1024 x 2816 (8 experts, 2 per token): 260 tokens 175 / 216, 500: 241 / 287, 1000: 396 / 424, 2000: 685 / 734,
//     8000: 2441 / 2396 (113 / 116 TFLOP/s for the layer).  The MFMAs of a row tile run in a row: with those of the two row
//     tiles alternating (longer distance between two on one accumulator) 1000 tokens took 427.
//   ffn_few_rows_f32: at most 32 rows x 16 columns (MODE 0: 16 features), the wavefronts split k instead: every fourth
//     k-step each, activations straight from memory, no barrier until the four partial tiles are added through LDS in a
//     fixed order.  Four times the blocks, each a quarter as long: with a few rows per expert the launch is latency.  The order
//     of the sums differs from ffn_rows_f32's, so a row's last bits depend on the rows per expert of the call.  The same four
//     partial sums in ffn_rows_f32 would make them equal and cost it 4 - 10 % (in registers three instead of four wavefronts fit a
//     SIMD, in LDS as much: 1024 x 2816, 700 tokens 282 / 301, 4000 tokens 1248 / 1361 us for the layer).
//
// Against one kernel with 64-row x 256-column blocks and both operands staged through LDS behind a barrier each way: 256 x
// 512, 64 tokens: both launches 94 -> 16 us, the layer 116 -> 30 us; 1024 x 2816, 700 tokens: 782 -> 270 us, 812 -> 296 us.
#include "moe_ffn_common.h"

namespace moe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kTileBytes = 128 * 64 * 4;             // a page tile: 128 rows of 256 bytes
constexpr int kRows = 32;                            // rows of a block, of either kernel
// Up to this many rows per expert on average the blocks of ffn_few_rows_f32 take the launch, us for the layer, ffn_few_rows
// / ffn_rows: 256 x 512 (8 experts, 2 per token) 64 tokens 30 / 43, 130 tokens 35 / 44, 260 tokens (65 rows) 42 / 45, 500
// tokens 51 / 50; 1024 x 2816 8 tokens 83 / 119, 100 tokens 112 / 147, 130 tokens 158 / 153, 260 tokens 203 / 175: beyond 32
// rows an expert's weights are read once per row tile by either, and the activations once per 16 columns instead of 64.
constexpr int kFewRows = 32;

// The tiles of one column tile along k, `step` tiles at a time; a page-table look-up only where a page begins.  An entry
// outside the pool is never followed: slot 0 is read instead and *bad is raised.
struct TileWalk {
    int page, within;
    const char* tile;
    __device__ __forceinline__ void locate(const GemmParams& p, const int32_t* trow, int& bad) {
        int slot = __builtin_amdgcn_readfirstlane(trow[page]);
        if ((unsigned)slot >= (unsigned)p.pool_pages) {
            bad = 1;
            slot = 0;
        }
        tile = p.pool + (int64_t)slot * p.page_bytes + (int64_t)within * kTileBytes;
    }
    __device__ __forceinline__ void start(const GemmParams& p, const int32_t* trow, int first, int& bad) {
        page = first / p.tpp;
        within = first - page * p.tpp;
        locate(p, trow, bad);
    }
    __device__ __forceinline__ void next(const GemmParams& p, const int32_t* trow, int step, int& bad) {
        within += step;
        tile += (int64_t)step * kTileBytes;
        if (within >= p.tpp) {
            do {
                within -= p.tpp;
                ++page;
            } while (within >= p.tpp);
            locate(p, trow, bad);
        }
    }
};

// chunk 4q + g of row n of a page tile: byte offset for q & 1 = 0, 1; q >> 1 adds 128 (the page format of moe.h)
__device__ __forceinline__ int chunk_offset(int n, int q, int g) { return n * 256 + (((q * 4 + g) ^ ((n >> 1) & 7)) << 4); }

// row of the matrix at A that row r (of this launch's row order) reads
__device__ __forceinline__ int64_t source_row(const GemmParams& p, int r) {
    return p.a_gather ? (int64_t)min(max(p.a_gather[r] / p.a_div, 0), p.a_rows - 1) : (int64_t)r;
}

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

// NB weight fragments per wavefront: MODE 0 the gate rows and the up rows of 16 features, MODE 1 16 columns
template <int MODE>
__global__ __launch_bounds__(kThreads) void ffn_rows_f32(const GemmParams p) {
    constexpr int RT = kRows / 16, NB = MODE == 0 ? 2 : 1;
    constexpr int kStride = 68;                      // floats per LDS row (64 + pad, 16-byte aligned)
    __shared__ __attribute__((aligned(16))) float sA[2][kRows * kStride];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    const TileCoord tc = locate_tile<kRows>(p);
    if (!tc.valid) return;
    const int nt = tc.nt, row0 = tc.row0, rows_here = tc.rows_here;
    const int nrt = (rows_here + 15) >> 4;           // row tiles with rows
    const int32_t* trow = p.table + (size_t)(p.table_row_mod ? tc.e % p.table_row_mod : tc.e) * p.ppe + p.group_base;
    int bad = 0;
    TileWalk w[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) w[b].start(p, trow, ((nt >> 1) * NB + b) * p.KT, bad);
    const int n = (nt & 1) * 64 + wave * 16 + r;
    const int boff[2] = {chunk_offset(n, 0, g), chunk_offset(n, 1, g)};

    const char* asrc[RT];                            // this thread's 16 bytes of rows tid / 16 + 16 j of the stage
#pragma unroll
    for (int j = 0; j < RT; ++j)
        asrc[j] = p.A + source_row(p, row0 + min(j * 16 + (tid >> 4), rows_here - 1)) * p.lda_bytes + (tid & 15) * 16;
    const int a_wr = (tid >> 4) * kStride + (tid & 15) * 4;

    f32x4 areg[RT], breg[2][NB][4], acc[RT][NB];
    auto load = [&](int kt, int set) __attribute__((always_inline)) {        // k-step kt: activations, and weights into set
#pragma unroll
        for (int j = 0; j < RT; ++j) areg[j] = *(const f32x4*)(asrc[j] + (int64_t)kt * 256);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) breg[set][b][q] = *(const f32x4*)(w[b].tile + boff[q & 1] + (q >> 1) * 128);
    };
    const bool copy = p.a_copy && nt == 0;           // the first column tile's blocks write the rows out as well
    auto store_a = [&](int kt, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < RT; ++j) *(f32x4*)(&sA[set][j * 16 * kStride + a_wr]) = areg[j];
        if (copy) {
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                const int row = j * 16 + (tid >> 4);
                if (row < rows_here) *(f32x4*)((char*)p.a_copy + (int64_t)(row0 + row) * p.lda_bytes + (int64_t)kt * 256 + (tid & 15) * 16) = areg[j];
            }
        }
    };
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int kt, int set) __attribute__((always_inline)) {        // set = kt & 1, known at compile time
        if (kt + 1 < p.KT) {
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b].next(p, trow, 1, bad);
            load(kt + 1, set ^ 1);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < RT; ++i)
                if (i < nrt) {
                    const f32x4 a = *(const f32x4*)(&sA[set][(i * 16 + r) * kStride + (q * 4 + g) * 4]);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], breg[set][b][q][j], acc[i][b], 0, 0, 0);
                }
        if (kt + 1 < p.KT) {
            store_a(kt + 1, set ^ 1);                // last read in step kt - 1: everyone has passed the barrier behind it
            __syncthreads();
        }
    };
    load(0, 0);
    store_a(0, 0);
    __syncthreads();
    for (int kt = 0; kt < p.KT; kt += 2) {           // KT is even (H and F are multiples of 128)
        step(kt, 0);
        step(kt + 1, 1);
    }

    // register v of lane (r, g): row i * 16 + g * 4 + v, column r
    const int col = nt * 64 + wave * 16 + r;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = i * 16 + g * 4 + v;
            if (row >= rows_here) continue;
            float* o = (float*)p.out + (int64_t)(row0 + row) * p.ldo + col;
            if (MODE == 0) *o = silu_mul(acc[i][0][v], acc[i][NB - 1][v]);
            else *o = acc[i][0][v] * (p.row_w ? p.row_w[row0 + row] : 1.0f);
        }
    if (bad && tid == 0 && p.status) atomicOr(p.status, 1);
}

template <int MODE>
__global__ __launch_bounds__(kThreads) void ffn_few_rows_f32(const GemmParams p) {
    constexpr int RT = kRows / 16, NB = MODE == 0 ? 2 : 1, W = kThreads / 64;
    __shared__ float part[W][RT][NB][4][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    const TileCoord tc = locate_tile<kRows>(p);
    if (!tc.valid) return;
    const int nt = tc.nt, row0 = tc.row0, rows_here = tc.rows_here;
    const bool two = rows_here > 16;
    const bool copy = p.a_copy && nt == 0;           // the first column tile's blocks write the rows out as well
    const int32_t* trow = p.table + (size_t)(p.table_row_mod ? tc.e % p.table_row_mod : tc.e) * p.ppe + p.group_base;
    int bad = 0;
    f32x4 acc[RT][NB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave < p.KT) {
        TileWalk w[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) w[b].start(p, trow, ((nt >> 3) * NB + b) * p.KT + wave, bad);
        const int n = (nt & 7) * 16 + r;
        const int boff[2] = {chunk_offset(n, 0, g), chunk_offset(n, 1, g)};
        const char* asrc[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i)
            asrc[i] = p.A + source_row(p, row0 + min(i * 16 + r, rows_here - 1)) * p.lda_bytes + g * 16;
        f32x4 areg[2][RT][4], breg[2][NB][4];
        auto load = [&](int kt, int set) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) breg[set][b][q] = *(const f32x4*)(w[b].tile + boff[q & 1] + (q >> 1) * 128);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) areg[set][i][q] = *(const f32x4*)(asrc[i] + (int64_t)kt * 256 + q * 64);
        };
        auto step = [&](int kt, int set) __attribute__((always_inline)) {    // set: known at compile time
            if (kt + W < p.KT) {
#pragma unroll
                for (int b = 0; b < NB; ++b) w[b].next(p, trow, W, bad);
                load(kt + W, set ^ 1);
            }
#pragma unroll
            for (int i = 0; i < RT; ++i)
                if (i == 0 || two) {
                    if (copy && i * 16 + r < rows_here) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *(f32x4*)((char*)p.a_copy + (int64_t)(row0 + i * 16 + r) * p.lda_bytes + (int64_t)kt * 256 + q * 64 + g * 16) = areg[set][i][q];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int b = 0; b < NB; ++b)
                                acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(areg[set][i][q][j], breg[set][b][q][j], acc[i][b], 0, 0, 0);
                }
        };
        load(wave, 0);
        for (int kt = wave; kt < p.KT; kt += 2 * W) {
            step(kt, 0);
            if (kt + W < p.KT) step(kt + W, 1);
        }
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[wave][i][b][v][lane] = acc[i][b][v];
    __syncthreads();
    // wavefront v adds up register v of every lane
    const int v = wave;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int row = i * 16 + g * 4 + v;
        if (row >= rows_here) continue;
        float sum[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) sum[b] = (part[0][i][b][v][lane] + part[1][i][b][v][lane]) + (part[2][i][b][v][lane] + part[3][i][b][v][lane]);
        float* o = (float*)p.out + (int64_t)(row0 + row) * p.ldo + nt * 16 + r;
        if (MODE == 0) *o = silu_mul(sum[0], sum[NB - 1]);
        else *o = sum[0] * (p.row_w ? p.row_w[row0 + row] : 1.0f);
    }
    if (bad && lane == 0 && p.status) atomicOr(p.status, 1);
}

// cols: output columns (MODE 0: features) of the launch; rows_each: rows per expert on average (of all experts, so that the
// experts of a streamed layer, one launch each, take the same kernel as the resident layer's single launch)
template <int MODE>
int launch_mode(GemmParams& p, int cols, int R, int rows_each, int n_exp, hipStream_t st) {
    const bool few = rows_each <= kFewRows;
    p.NT = cols / (few ? 16 : 64);
    const dim3 grid(gemm_grid(p.NT, R, kRows, n_exp, p.chunked)), block(kThreads);
    if (few) hipLaunchKernelGGL((ffn_few_rows_f32<MODE>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((ffn_rows_f32<MODE>), grid, block, 0, st, p);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

}  // namespace

int launch_expert_ffn_f32(const moe_shape& s, const Geom& g, const FfnArgs& a, hipStream_t st) {
    const int R = s.T * s.k, n_exp = a.e_end - a.e_begin;
    GemmParams p{};
    fill_common(p, s, g, a);
    fill_gate_up(p, s, g, a);
    int rc = launch_mode<0>(p, s.F, R, R / s.E, n_exp, st);
    if (rc != MOE_OK) return rc;
    if (a.mid_event) MOE_HIP_TRY(hipEventRecord(a.mid_event, st));
    fill_down(p, s, g, a);
    return launch_mode<1>(p, s.H, R, R / s.E, n_exp, st);
}

int launch_expert_ffn(const moe_shape& s, const FfnArgs& a, hipStream_t st) {
    const Geom g = geometry(s);
    if (s.dtype == MOE_DTYPE_BF16) return launch_expert_ffn_bf16(s, g, a, st);
    return launch_expert_ffn_f32(s, g, a, st);
}

}  // namespace moe
