// a3 for a handful of tokens, bf16 operands, fp32 accumulation, on v_mfma_f32_16x16x32_bf16.  Few experts have rows then, and
// a block of moe_ffn_rows_bf16.hip with its 64 or 128 columns leaves compute units without weights to stream (one token of
// the Mixtral-8x7B shape: 64 blocks in the down launch, 82 us for 235 MB).
//
// Here a wavefront is on its own: 16 columns (MODE 0: 16 features, gate and up), one row tile, no LDS and no barrier.  Its weights
// (1 KiB in a row per half-tile, one MFMA operand) and its activations (16 rows x 64 bytes, from the L2 after the first
// wavefront) go straight into registers, D k-steps ahead, all loads the compiler's own and in one order.  With at most 16 tokens an
// expert has at most 16 rows (others, from offsets that no routing made, take several row tiles).  us for the launch, D = 8 / 12 / 16:
// down of the Mixtral-8x7B shape, one token 45 / 46 / 45 (rows kernel 82), two tokens 74 / 79 / - (96); four wavefronts to a block
// instead of one 55.  Every output is the same chain of MFMAs along k as in the other bf16 kernels: the same bits.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "moe_ffn_common.h"

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kHalfTileBytes = 128 * 64;             // 32 k of a page tile
constexpr int kTileBytes = 2 * kHalfTileBytes;

// CW: wavefronts of a block, side by side along the columns
template <int MODE, int CW>
__global__ __launch_bounds__(64 * CW) void ffn_thin_bf16(const GemmParams p) {
    constexpr int D = 8;                             // k-steps under way
    constexpr int BM = 16, NB = MODE == 0 ? 2 : 1, kCols = 16 * CW, kColTiles = 128 / kCols;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;

    RowsTile tc;
    if (!locate_rows_tile<BM>(p, tc)) return;
    const int nt = tc.nt, row0 = tc.row0, rows_here = tc.rows_here, KT = p.KT;
    const int32_t* trow = p.table + (size_t)(p.table_row_mod ? tc.e % p.table_row_mod : tc.e) * p.ppe + p.group_base;
    int bad = 0, page[NB], within[NB];
    const char* tile[NB];
    auto page_addr = [&](int pg) __attribute__((always_inline)) -> const char* {
        int slot = __builtin_amdgcn_readfirstlane(trow[pg]);
        if ((unsigned)slot >= (unsigned)p.pool_pages) {   // never follow an entry outside the pool
            bad = 1;
            slot = 0;
        }
        return p.pool + (int64_t)slot * p.page_bytes;
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int t0 = ((nt / kColTiles) * NB + b) * KT;
        page[b] = t0 / p.tpp;
        within[b] = t0 - page[b] * p.tpp;
        tile[b] = page_addr(page[b]) + (int64_t)within[b] * kTileBytes;
    }
    const uint32_t b_off = ((nt % kColTiles) * kCols + wave * 16 + r) * 64 + ((g ^ ((r >> 2) & 2)) << 4);
    const int row = min(r, rows_here - 1);
    const int src = p.a_gather ? min(max(p.a_gather[row0 + row] / p.a_div, 0), p.a_rows - 1) : row;
    const uint32_t a_off = (uint32_t)src * (uint32_t)p.lda_bytes + g * 16;
    const char* a_base = p.a_gather ? p.A : p.A + (int64_t)row0 * p.lda_bytes;

    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto main_loop = [&](auto stream_c) __attribute__((always_inline)) {
        i32x4 areg[D][2], breg[D][2][NB];
        auto load = [&](int s, int slot) __attribute__((always_inline)) {        // k-step s, s in order
#pragma unroll
            for (int hp = 0; hp < 2; ++hp) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const i32x4* src = (const i32x4*)(tile[b] + hp * kHalfTileBytes + b_off);
                    if constexpr (decltype(stream_c)::value) breg[slot][hp][b] = __builtin_nontemporal_load(src);
                    else breg[slot][hp][b] = *src;
                }
                areg[slot][hp] = *(const i32x4*)(a_base + (int64_t)s * 128 + hp * 64 + a_off);
            }
            if (s + 1 < KT) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    tile[b] += kTileBytes;
                    if (__builtin_expect(++within[b] == p.tpp, 0)) {
                        within[b] = 0;
                        tile[b] = page_addr(++page[b]);
                    }
                }
            }
        };
        auto multiply = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, areg[slot][hp]), __builtin_bit_cast(bf16x8, breg[slot][hp][b]), acc[b], 0, 0, 0);
        };
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < KT) load(u, u);
        int s = 0;
        for (; s + 2 * D <= KT; s += D)
#pragma unroll
            for (int u = 0; u < D; ++u) {
                multiply(u);
                load(s + u + D, u);
            }
        // fewer than 2 D k-steps are left, the next D of them loaded
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (s + u < KT) {
                multiply(u);
                if (s + u + D < KT) load(s + u + D, u);
            }
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (s + u + D < KT) multiply(u);
    };
    if (p.stream && tc.mtiles == 1) main_loop(std::true_type{});
    else main_loop(std::false_type{});

    const int col = nt * kCols + wave * 16 + r;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int orow = g * 4 + v;
        if (orow >= rows_here) continue;
        const int64_t o = (int64_t)(row0 + orow) * p.ldo + col;
        if constexpr (MODE == 0) ((__bf16*)p.out)[o] = (__bf16)silu_mul_bf16(acc[0][v], acc[1][v]);
        else ((float*)p.out)[o] = acc[0][v] * (p.row_w ? p.row_w[row0 + orow] : 1.0f);
    }
    if (bad && lane == 0 && p.status) atomicOr(p.status, 1);
}

template <int MODE, int CW>
int launch_thin(GemmParams& p, int cols, int R, int n_exp, hipStream_t st) {
    p.NT = cols / (16 * CW);
    hipLaunchKernelGGL((ffn_thin_bf16<MODE, CW>), dim3(rows_grid(p.NT, R, 16, n_exp)), dim3(64 * CW), 0, st, p);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

}  // namespace

// experts with rows, on average over routings that favour none, and the standard deviation
static double experts_with_rows(const moe_shape& s, double* deviation = nullptr) {
    const double E = s.E, none = std::pow(1.0 - s.k / E, s.T);                      // an expert, two experts without a row
    const double neither = s.E > 1 ? std::pow((E - s.k) * (E - s.k - 1.0) / (E * (E - 1.0)), s.T) : none;
    if (deviation) *deviation = std::sqrt(std::max(0.0, E * none * (1.0 - none) + E * (E - 1.0) * (neither - none * none)));
    return E * (1.0 - none);
}

// Where the launches of at most 16 tokens come here, by the blocks that moe_ffn_rows_bf16.hip would keep busy.
// Gate/up: up to about one and a half blocks of 64 features per compute unit.  us, that kernel / this one: 1024 x 2816 (8 experts, 2
// per token) 1 token (88 blocks) 13 / 11, 16 tokens (348) 25 / 22; 2048 x 4096 1 token (128) 22 / 18, 4 tokens (350) 34 / 31, 16 tokens (506)
// 47 / 46; 64 experts of 2048 x 1024, 8 per token, 3 tokens (337) 40 / 36, 8 tokens (671) 61 / 63; Mixtral-8x7B shape 1 token (448) 76 / 79.
bool thin_takes_gate_up(const moe_shape& s) { return s.T <= 16 && experts_with_rows(s) * (s.F / 64) <= 440; }
// Down: with clearly fewer blocks of 128 columns than compute units, or with between one and one and a half per compute unit, which share
// out unevenly; here 384 blocks' worth of wavefronts, twelve per compute unit, are the most that run at once.  us for both
// launches, by experts with rows (blocks), that kernel / this one:
//   k of 14336 (4096 x 14336) 2 experts (64) 153 / 114, 4 (128) 233 / 214, 6 (192) 326 / 321, 8 (256) 416 / 416, 9 (288) 515 / 468, 12 (384) 625 / 615,
//   13 (416) 668 / 691; 10752 (6144 x 10752) 3 (144) 205 / 199, 4 (192) 254 / 253, 5 (240) 321 / 329, 6 (288) 405 / 374, 9 (432) 522 / 538;
//   8192 (5120 x 8192) 2 (80) 100 / 85, 3 (120) 133 / 126, 5 (200) 196 / 204, 7 (280) 299 / 282, 10 (400) 378 / 416; (3072 x 8192) 6 (144) 150 / 153, 8
//   (192) 186 / 199; 4096 (4096 x 4096) 5 (160) 91 / 89, 6 (192) 96 / 100;
//   2048 (2048 x 2048) 8 (128) 40 / 37, 11 (176) 50 / 50, 15 (240) 64 / 66, (4096 x 2048) 9 (288) 90 / 81, 13 (416) 108 / 109, 15 (480) 119 / 118.
// The routing is not known here.  The lower range goes by the average; the upper one by the average plus the deviation, or all experts, and where
// k is not long by the average less half the deviation (routings that fill one round or less lose as much there as the others gain; with a long
// k they lose little: 6144 x 16384, 8 experts, 4 tokens, 262 blocks on average, layer 522 / 502 over sixteen routings).
bool thin_takes_down(const moe_shape& s) {
    if (s.T > 16) return false;
    const double per_expert = s.H / 128;
    double deviation;
    const double blocks = experts_with_rows(s, &deviation) * per_expert;
    if (s.F <= 2048) return blocks < 190 || (blocks > 256 && blocks < 500);
    const bool long_k = s.F > 10240;
    if (blocks < (long_k ? 190 : 130)) return true;
    return blocks - (long_k ? 0.0 : 0.5 * deviation * per_expert) > 256 && std::min(blocks + deviation * per_expert, s.E * per_expert) <= 384;
}

int launch_gate_up_thin_bf16(GemmParams& p, int F, int R, int n_exp, hipStream_t st) { return launch_thin<0, 2>(p, F, R, n_exp, st); }

int launch_down_thin_bf16(GemmParams& p, int H, int R, int n_exp, hipStream_t st) { return launch_thin<1, 1>(p, H, R, n_exp, st); }

}  // namespace moe
