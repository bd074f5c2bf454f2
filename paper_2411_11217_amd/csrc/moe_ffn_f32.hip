// a3 for float32 storage: the same grouped SwiGLU FFN over the same page format.  With more than a few rows per expert the
// matrix cores are the bound, with fewer it is the weights' way from HBM.
//
//   ffn_split_f32: float32 products on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, 16 times the rate of the float32 MFMA).
//     Every value is a sum of three bf16, x = x0 + x1 + x2 with 24 bits together, and a product is the six partial products
//     x2 y0 + x0 y2 + x1 y1 + x1 y0 + x0 y1 + x0 y0; what is left out, x1 y2 and x2 y1, is below 2^-24 of it.  The six MFMAs of 32 k add up in
//     registers of their own, from zero, and a float32 addition takes the sum over: with all six on the accumulator itself
//     every MFMA rounds at the size of the accumulator.  Relative error against float64 of h / of out for a given h: float32 MFMA 8.7e-7 / 9.5e-7,
//     six MFMAs on the accumulator 7.3e-7 / 5.8e-7, this way 1.8e-7 / 1.5e-7 (1024 x 2816; 256 x 512: 4.2e-7 / 4.1e-7, 3.4e-7 /
//     2.4e-7, 1.1e-7 / 0.8e-7).
//     What the parts cannot hold: infinities and values that bf16 rounds to one give NaN (inf - inf), and of a value below
//     2^-110 up to 2^-134 is lost, half the last bit of a bf16 subnormal (neither the conversion nor the MFMA flushes them).  A sum of K
//     products loses at most K 2^-134 (X + W) of that, with X and W the largest magnitudes of its row and its column, which the threads
//     note as they split (a v_max3 for two values: 2 - 3 % of the layer), and less than K 2^-146 in products that underflow.  A sum that
//     is not finite, or below 2^26 times these with neither its row nor its column zero, is replaced by that of the float32 MFMA, operands straight from
//     memory: a wavefront does that for the row tiles of 16 that hold such a sum, and stores those sums alone.  With X = W = 1 and K = 1024
//     the limit is 2^-97; ordinary sums meet it when they cancel to 0 exactly, one in some 30 million.
//     A block owns 16 RT rows x 64 columns (MODE 0: 64 features, gate and up).  The four wavefronts split the columns; a
//     weight element is used by one wavefront alone and goes from the page straight into registers, where it is split.
//     The activations are split once per block and pass through LDS (two stages; the registers hold the next step or two), one
//     barrier per step of 32 k.  Splitting eight values takes 44 vector instructions, as long as 11 MFMAs: the more rows
//     a block has, the more MFMAs share the split of its weights, and blocks of other wavefronts on the same SIMD fill
//     the matrix cores meanwhile (three per SIMD).  Few columns (MODE 1) or few blocks: KG = 2, two groups of four wavefronts with 32 k of a step each.
//     1024 x 2816, 700 tokens, against the float32 MFMA with blocks of 32 rows: gate/up 186 / 132 us, down 110 / 93, layer 285 / 210;
//     3000 tokens 954 / 657; 256 x 512, 1100 tokens 66 / 49.  700 tokens: matrix cores busy 0.52 and 0.38 of the launches' cycles,
//     vector instructions 0.66 and 0.62.
//   ffn_few_rows_f32: at most 32 rows x 16 columns (MODE 0: 16 features) on v_mfma_f32_16x16x4_f32, the wavefronts split k instead: every fourth
//     k-step each, activations straight from memory, no barrier until the four partial tiles are added through LDS in a
//     fixed order.  A lane's share of an operand is a 16-byte chunk (four consecutive k of one row): lane l holds chunk 4q +
//     l / 16 of row l % 16, and four MFMAs take one element of the four each, so that MFMA j adds the k = 16q + 4g + j (g = 0 .. 3);
//     activations and weights use the same map, so no element needs to move between lanes.  Four times the
//     blocks, each a quarter as long: with a few rows per expert the launch is latency.
// The two kernels add in different orders, so a row's last bits depend on the rows per expert of the call.
#include <mutex>
#include <type_traits>

#include "moe_ffn_common.h"

namespace moe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kComputeUnits = 256;                   // MI355X
constexpr int kTileBytes = 128 * 64 * 4;             // a page tile: 128 rows of 256 bytes
constexpr int kFewRows = 32;                         // rows of a block of ffn_few_rows_f32

// Where ffn_split_f32 takes a launch: with more than 32 rows per expert on average (beyond, an expert's weights are read once per row
// tile by the other kernel, and its activations once per 16 columns), and with more than 16 where its blocks of 64 columns
// make a round on the 256 compute units.  us for the launch, ffn_few_rows / ffn_split with 128 rows (gate/up): gate/up of 1024 x 2816 (8 experts, 2 per
// token; 352 blocks) 50 tokens 53 / 55, 70: 61 / 55, 110: 69 / 55, 128: 86 / 59; its down launch (128 blocks) 70: 34 / 46, 110: 40 / 48,
// 128: 55 / 49; 256 x 512 (64 and 32 blocks) 110 tokens 13 / 16 and 11 / 16.
inline bool split_takes(int rows_each, int64_t column_blocks) {
    return rows_each > kFewRows || (rows_each > kFewRows / 2 && column_blocks >= kComputeUnits);
}

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

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int pack_bf16(float a, float b) {          // both rounded to nearest even
    int v = 0;
#ifdef __HIP_DEVICE_COMPILE__
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(v) : "v"(a), "v"(b));
#endif
    return v;
}

// the largest of m, |a| and |b|; a NaN among them does not matter here
__device__ __forceinline__ void raise_to(float& m, float a, float b) {
#ifdef __HIP_DEVICE_COMPILE__
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
#endif
}

// eight values, each as a sum of three bf16: part[0] + part[1] + part[2]; top: raised to the largest magnitude among them
__device__ __forceinline__ void split_bf16(const f32x4& lo, const f32x4& hi, i32x4 (&part)[3], float& top) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = j < 2 ? lo[2 * j] : hi[2 * j - 4], b = j < 2 ? lo[2 * j + 1] : hi[2 * j - 3];
        raise_to(top, a, b);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int v = pack_bf16(a, b);
            part[q][j] = v;
            a -= __builtin_bit_cast(float, v << 16);
            b -= __builtin_bit_cast(float, v & (int)0xffff0000);
        }
    }
}

// RT: row tiles of 16; KG: groups of four wavefronts, each takes 32 k of a step
template <int MODE, int RT, int KG>
__global__ __launch_bounds__(kThreads * KG, KG == 1 ? 3 : 4) void ffn_split_f32(const GemmParams p) {
    constexpr int NB = MODE == 0 ? 2 : 1, BM = 16 * RT, AJ = (BM + 63) / 64;
    constexpr int kPlane = BM * 64, kSplitStage = 3 * kPlane;     // LDS bytes of one part of 32 k: rows of 32 bf16; of all three
    constexpr int D = MODE == 0 ? 1 : 2;             // steps whose loads are under way
    constexpr int kStage = KG * kSplitStage;
    extern __shared__ __attribute__((aligned(1024))) char smem[];      // two stages
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3), kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);
    const int r = lane & 15, g = lane >> 4;

    RowsTile tc;
    if (!locate_rows_tile<BM, true>(p, tc)) return;
    const int nt = tc.nt, row0 = tc.row0, rows_here = tc.rows_here;
    const int32_t* trow = p.table + (size_t)(p.table_row_mod ? tc.e % p.table_row_mod : tc.e) * p.ppe + p.group_base;
    int bad = 0;
    TileWalk w[NB];
    auto weights_start = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b) w[b].start(p, trow, ((nt >> 1) * NB + b) * p.KT, bad);
    };
    weights_start();
    const int n = (nt & 1) * 64 + wave * 16 + r;
    const int boff = chunk_offset(n, 0, g);          // the next chunk: bit 6 the other way; half a k-step on: 128 bytes more

    // this thread's chunks, a 64-byte piece apart, of rows tid / 4 and 64 + tid / 4 (KG = 2: the second group the other 32 k)
    const int a_row = (tid >> 2) & 63, a_ch = tid & 3;
    const char* asrc[AJ];
#pragma unroll
    for (int j = 0; j < AJ; ++j)
        asrc[j] = p.A + source_row(p, row0 + min(j * 64 + a_row, rows_here - 1)) * p.lda_bytes + a_ch * 16 + kg * 128;
    const int a_wr = kg * kSplitStage + a_row * 64 + ((a_ch ^ ((a_row >> 2) & 2)) << 4);
    const int a_rd = kg * kSplitStage + r * 64 + ((g ^ ((r >> 2) & 2)) << 4);
    const bool copy = p.a_copy && nt == 0;           // the first column tile's blocks write the rows out as well

    f32x4 acc[RT][NB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float a_top[AJ], w_top[NB];                      // largest magnitudes of this thread's activations (by row) and weights
#pragma unroll
    for (int j = 0; j < AJ; ++j) a_top[j] = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b) w_top[b] = 0.f;

    // NRT: row tiles that are loaded and multiplied.  A step is 32 * KG k.
    auto main_loop = [&](auto nrt_c) __attribute__((always_inline)) {
        constexpr int NRT = decltype(nrt_c)::value, NA = NRT > 4 ? 2 : 1;
        const int steps = 2 * p.KT / KG;             // even: KT is
        f32x4 areg[D][NA][2], breg[D][NB][2];
        i32x4 bpart[1][NB][3];
        auto load = [&](int s, int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NA; ++j)
#pragma unroll
                for (int c = 0; c < 2; ++c) areg[slot][j][c] = *(const f32x4*)(asrc[j] + (int64_t)s * (128 * KG) + c * 64);
            if (s > 0 && (KG == 2 || !(s & 1))) {
#pragma unroll
                for (int b = 0; b < NB; ++b) w[b].next(p, trow, 1, bad);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                int o = boff;
                asm("" : "+v"(o) : "s"(s));          // both offsets are formed here, and not kept through the loop
#pragma unroll
                for (int c = 0; c < 2; ++c) breg[slot][b][c] = *(const f32x4*)(w[b].tile + (o ^ (c * 64)) + (KG == 2 ? kg : s & 1) * 128);
            }
        };
        auto copy_rows = [&](int s, int slot) __attribute__((always_inline)) {
            char* dst = (char*)p.a_copy + (int64_t)row0 * p.lda_bytes + (int64_t)s * (128 * KG);
            int first = a_row;
            asm("" : "+v"(first) : "s"(s));          // as above
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                const int row = j * 64 + first;
                const uint32_t o = (uint32_t)row * (uint32_t)p.lda_bytes + a_ch * 16 + kg * 128;
                if (row < rows_here) {
                    *(f32x4*)(dst + o) = areg[slot][j][0];
                    *(f32x4*)(dst + o + 64) = areg[slot][j][1];
                }
            }
        };
        auto split = [&](int slot, char* st, i32x4 (&bp)[NB][3]) __attribute__((always_inline)) {   // a step's loads: activations to st, weights to bp
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                i32x4 part[3];
                split_bf16(areg[slot][j][0], areg[slot][j][1], part, a_top[j]);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (BM % 64 == 0 || j * 64 + a_row < BM) *(i32x4*)(st + q * kPlane + j * 4096 + a_wr) = part[q];
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                split_bf16(breg[slot][b][0], breg[slot][b][1], bp[b], w_top[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto multiply = [&](const char* st, const i32x4 (&bp)[NB][3]) __attribute__((always_inline)) {
            constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};      // the small products first
            constexpr int G = MODE == 0 ? 1 : 2;     // row tiles at a time: four independent chains, or two
            i32x4 a[2][G][3];
            auto fetch = [&](int i, int set) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < G; ++t)
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[set][t][q] = *(const i32x4*)(st + q * kPlane + (i + t) * 1024 + a_rd);
            };
            f32x4 sum[2][G][NB];
            auto add = [&](int i, int set) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < G; ++t)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        acc[i + t][b] += sum[set][t][b];
                        asm volatile("" : "+v"(acc[i + t][b]));      // here, and not behind the loop with all sums kept until there
                    }
            };
            fetch(0, 0);
#pragma unroll
            for (int i = 0; i < NRT; i += G) {
                const int set = (i / G) & 1;
                if (i + G < NRT) fetch(i + G, set ^ 1);
#pragma unroll
                for (int pr = 0; pr < 6; ++pr)
#pragma unroll
                    for (int t = 0; t < G; ++t)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            sum[set][t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[set][t][pa[pr]]), __builtin_bit_cast(bf16x8, bp[b][pb[pr]]), pr == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[set][t][b], 0, 0, 0);
                if (i > 0) add(i - G, set ^ 1);      // behind the MFMAs of the next row tiles: their latency has passed
                __builtin_amdgcn_sched_barrier(0);
            }
            add(NRT - G, (NRT / G - 1) & 1);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
        if (copy) copy_rows(0, 0);
        split(0, smem, bpart[0]);
        if (D < steps) load(D, 0);
        __syncthreads();
        for (int s = 0; s < steps; s += 2) {
            multiply(smem, bpart[0]);
            if (copy) copy_rows(s + 1, D - 1);
            split(D - 1, smem + kStage, bpart[0]);   // last read in step s - 1: everyone has passed the barrier behind it
            if (s + 1 + D < steps) load(s + 1 + D, D - 1);
            __syncthreads();
            multiply(smem + kStage, bpart[0]);
            if (s + 2 < steps) {
                if (copy) copy_rows(s + 2, 0);
                split(0, smem, bpart[0]);
                if (s + 2 + D < steps) load(s + 2 + D, 0);
                __syncthreads();
            }
        }
    };
    if (RT > 6 && rows_here > 96) main_loop(std::integral_constant<int, RT>{});
    else if (RT > 4 && rows_here > 64) main_loop(std::integral_constant<int, RT < 6 ? RT : 6>{});
    else if (RT > 2 && rows_here > 32) main_loop(std::integral_constant<int, RT < 4 ? RT : 4>{});
    else main_loop(std::integral_constant<int, 2>{});
    // the thread's coordinates once more: kept through the loop they would take registers that it does not have
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63, r_e = lane_e & 15, g_e = lane_e >> 4, row_e = (tid_e >> 2) & 63;
    // what the four threads of a row, the four lanes of a column and the two groups have seen; stage 0 was last read before
    // the last barrier of the loop, with KG = 2 the second group's sums lie there
    float* s_top = (float*)(smem + (KG == 2 ? RT * NB * 4096 : 0));          // [KG][BM] rows, KG = 2: [NB][256] weights of the second group
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
        a_top[j] = fmaxf(a_top[j], __shfl_xor(a_top[j], 1, 64));
        a_top[j] = fmaxf(a_top[j], __shfl_xor(a_top[j], 2, 64));
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        w_top[b] = fmaxf(w_top[b], __shfl_xor(w_top[b], 16, 64));
        w_top[b] = fmaxf(w_top[b], __shfl_xor(w_top[b], 32, 64));
    }
    if (KG == 2) __syncthreads();
#pragma unroll
    for (int j = 0; j < AJ; ++j)
        if ((tid_e & 3) == 0 && (BM % 64 == 0 || j * 64 + row_e < BM)) s_top[kg * BM + j * 64 + row_e] = j * 64 + row_e < rows_here ? a_top[j] : 0.f;
    if constexpr (KG == 2) {                         // the second group's sums are added to the first's
        f32x4* part = (f32x4*)smem + (tid_e & 255);
        if (kg == 1) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b) part[(i * NB + b) * 256] = acc[i][b];
#pragma unroll
            for (int b = 0; b < NB; ++b) s_top[KG * BM + b * 256 + (tid_e & 255)] = w_top[b];
        }
        __syncthreads();
        if (kg == 1) {
            if (bad && lane_e == 0 && p.status) atomicOr(p.status, 1);
            return;
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[i][b] += part[(i * NB + b) * 256];
#pragma unroll
        for (int b = 0; b < NB; ++b) w_top[b] = fmaxf(w_top[b], s_top[KG * BM + b * 256 + tid_e]);
    } else {
        __syncthreads();
    }

    // register v: row i * 16 + g_e * 4 + v, column r_e
    const int col = nt * 64 + wave * 16 + r_e;
    auto store = [&](int i, const f32x4 (&a)[NB], uint32_t rows) __attribute__((always_inline)) {       // rows: bit v for register v
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = i * 16 + g_e * 4 + v;
            if (row >= rows_here || !((rows >> v) & 1)) continue;
            float* o = (float*)p.out + (int64_t)(row0 + row) * p.ldo + col;
            if (MODE == 0) *o = silu_mul(a[0][v], a[NB - 1][v]);
            else *o = a[0][v] * (p.row_w ? p.row_w[row0 + row] : 1.0f);
        }
    };
#pragma unroll
    for (int i = 0; i < RT; ++i) store(i, acc[i], 15);
    // Odd: a sum that is not finite, or below the limit where what the parts of its operands and its products lost may show (see
    // the top of the file; nothing is lost where the row or the column is zero).  Only these are replaced, so that a row's bits depend on
    // its own values alone and not on what else is in its tile.
    const float per_unit = (float)p.KT * 64.f * 0x1p-108f;
    float w_limit[NB], least = INFINITY, finite = 0.f;        // least: a sum's distance from its limit; finite: 0, or NaN
#pragma unroll
    for (int b = 0; b < NB; ++b) w_limit[b] = w_top[b] == 0.f ? -INFINITY : per_unit * (w_top[b] + 0x1p-12f);
    auto row_limits = [&](int i) __attribute__((always_inline)) {
        f32x4 t = *(const f32x4*)(s_top + i * 16 + g_e * 4);
        if (KG == 2) {
            const f32x4 u = *(const f32x4*)(s_top + BM + i * 16 + g_e * 4);
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = fmaxf(t[v], u[v]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] = t[v] == 0.f ? -INFINITY : per_unit * t[v];
        return t;
    };
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const f32x4 limit = row_limits(i);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                least = fminf(least, fabsf(acc[i][b][v]) - (limit[v] + w_limit[b]));
                finite = fmaf(acc[i][b][v], 0.f, finite);
            }
    }
    if (__builtin_expect(__ballot(least < 0.f || finite != 0.f) != 0, 0)) {
        uint32_t odd = 0;                            // bit 4 i + v: register v of row tile i
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const f32x4 limit = row_limits(i);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const float m = fabsf(acc[i][b][v]);
                    odd |= (uint32_t)(!(m < INFINITY) || m - (limit[v] + w_limit[b]) < 0.f) << (4 * i + v);
                }
        }
        for (int i = 0; i * 16 < rows_here; ++i) {
            const uint32_t mine = (odd >> (4 * i)) & 15;
            if (!__ballot(mine != 0)) continue;
            const char* arow = p.A + source_row(p, row0 + min(i * 16 + r_e, rows_here - 1)) * p.lda_bytes + g_e * 16;
            const int n_e = (nt & 1) * 64 + wave * 16 + r_e, boff_e[2] = {chunk_offset(n_e, 0, g_e), chunk_offset(n_e, 1, g_e)};
            f32x4 sum[NB], a[2][4], wt[2][NB][4];
#pragma unroll
            for (int b = 0; b < NB; ++b) sum[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            weights_start();
            auto load = [&](int kt, int slot) __attribute__((always_inline)) {
                if (kt > 0) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) w[b].next(p, trow, 1, bad);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[slot][q] = *(const f32x4*)(arow + (int64_t)kt * 256 + q * 64);
#pragma unroll
                    for (int b = 0; b < NB; ++b) wt[slot][b][q] = *(const f32x4*)(w[b].tile + boff_e[q & 1] + (q >> 1) * 128);
                }
            };
            auto multiply = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int b = 0; b < NB; ++b) sum[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[slot][q][j], wt[slot][b][q][j], sum[b], 0, 0, 0);
            };
            load(0, 0);
            for (int kt = 0; kt < p.KT; kt += 2) {   // KT is even
                load(kt + 1, 1);
                multiply(0);
                if (kt + 2 < p.KT) load(kt + 2, 0);
                multiply(1);
            }
            store(i, sum, mine);
        }
    }
    if (bad && lane_e == 0 && p.status) atomicOr(p.status, 1);
}

template <int MODE>
__global__ __launch_bounds__(kThreads) void ffn_few_rows_f32(const GemmParams p) {
    constexpr int RT = kFewRows / 16, NB = MODE == 0 ? 2 : 1, W = kThreads / 64;
    __shared__ float part[W][RT][NB][4][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    // the order of locate_tile costs every block a microsecond or more; us for the layer with it / with this one: 256 x 512, 64 tokens 25.5 / 22.3, 20: 22.6 / 19.4;
    // 1024 x 2816, 30 tokens 76.5 / 71.3, 100 (the down launch) 86.9 / 84.9
    RowsTile tc;
    if (!locate_rows_tile<kFewRows>(p, tc)) return;
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

template <int MODE, int RT, int KG>
int launch_split(GemmParams& p, int cols, int R, int n_exp, hipStream_t st) {
    constexpr int lds = 2 * KG * 3 * RT * 16 * 64;
    p.NT = cols / 64;
    const int grid = rows_grid(p.NT, R, 16 * RT, n_exp);
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute((const void*)ffn_split_f32<MODE, RT, KG>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    MOE_HIP_TRY(attr_err);
    hipLaunchKernelGGL((ffn_split_f32<MODE, RT, KG>), dim3(grid), dim3(kThreads * KG), lds, st, p);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

// cols: output columns (MODE 0: features) of the launch.  The rules go by the rows per expert on average (of all experts, so
// that the experts of a streamed layer, one launch each, take the same kernel as the resident layer's single launch).
template <int MODE>
int launch_mode(GemmParams& p, int cols, int R, int E, int n_exp, hipStream_t st) {
    const int rows_each = R / E;
    const int64_t column_blocks = (int64_t)(cols / 64) * E;
    if (split_takes(rows_each, column_blocks)) {
        // us for the launch of 1024 x 2816, 64 rows and KG = 2 / 128 rows and KG = 2 / 64 rows and KG = 1: 150 tokens 50 / 52 / 78, 700:
        // 76 / 78 / 91, 1000: 113 / 134 / 110, 4000: 318 / 385 / 311
        if constexpr (MODE == 1) {
            return launch_split<1, 4, 2>(p, cols, R, n_exp, st);
        } else {
            // Blocks of 32 rows with KG = 2 as long as they make one round: with fewer blocks than compute units the chain along k is all that
            // counts, and these have half of it.  us for the layer, 64 rows and KG = 1 / these (before both: 32 rows on the float32 MFMA): 512 x 128, 8
            // experts, 100 rows each (64 blocks of 32 rows) 44 / 37 (40), 400 rows (208) 51 / 45; 2048 x 128, 4 experts, 50 rows (16) 88 / 61 (79); 8192 x
            // 512, 4 experts, 35 rows (64) 294 / 186 (286), 250 rows (256) 380 / 349; 256 x 512, 8 experts, 125 rows (256) 41.6 / 41.4; beyond,
            // 128 x 512, 8 experts, 200 rows (448) 38.8 / 39.7; 128 x 4096, 2 experts, 100 rows (512) 82.4 / 82.8.
            if (column_blocks * ((rows_each + 31) / 32) <= kComputeUnits) return launch_split<0, 2, 2>(p, cols, R, n_exp, st);
            // With up to 48 rows on average blocks of 64 rows with KG = 2 are the better ones where the rows are shared out unevenly, and as good where
            // they are not.  us for the layer, 128 rows and KG = 1 / these: 2048 x 1024, 16 experts, 2 per token, 300 tokens 146 / 129, 40 % of the rows on
            // one expert 179 / 156, all on two 158 / 100; 1024 x 2816, 8 experts, 70 tokens, likewise 90 / 87, 99 / 96, 95 / 75; 170 tokens 113 / 114;
            // 64 rows on average 1024 x 1024, 32 experts 174 / 190, 512 x 8192, 4 experts 172 / 181.
            if (rows_each <= 48) return launch_split<0, 4, 2>(p, cols, R, n_exp, st);
            // 128 rows halve what a block spends on splitting weights, 64 make more blocks: 1024 x 2816 (352 blocks for up to 128 rows
            // each) 300 tokens 78 / 77, 700: 110 / 114, 4000: 449 / 474; 256 x 512, 300 tokens (64 blocks) 23 / 18, 1000: 26 / 21
            if (column_blocks * ((rows_each + 127) / 128) >= kComputeUnits) return launch_split<0, 8, 1>(p, cols, R, n_exp, st);
            return launch_split<0, 4, 1>(p, cols, R, n_exp, st);
        }
    }
    p.NT = cols / 16;
    hipLaunchKernelGGL((ffn_few_rows_f32<MODE>), dim3(rows_grid(p.NT, R, kFewRows, n_exp)), dim3(kThreads), 0, st, p);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

}  // namespace

int launch_expert_ffn_f32(const moe_shape& s, const Geom& g, const FfnArgs& a, hipStream_t st) {
    const int R = s.T * s.k, n_exp = a.e_end - a.e_begin;
    GemmParams p{};
    fill_common(p, s, g, a);
    fill_gate_up(p, s, g, a);
    int rc = launch_mode<0>(p, s.F, R, s.E, n_exp, st);
    if (rc != MOE_OK) return rc;
    if (a.mid_event) MOE_HIP_TRY(hipEventRecord(a.mid_event, st));
    fill_down(p, s, g, a);
    return launch_mode<1>(p, s.H, R, s.E, n_exp, st);
}

int launch_expert_ffn(const moe_shape& s, const FfnArgs& a, hipStream_t st) {
    const Geom g = geometry(s);
    if (s.dtype == MOE_DTYPE_BF16) return launch_expert_ffn_bf16(s, g, a, st);
    return launch_expert_ffn_f32(s, g, a, st);
}

}  // namespace moe
