// a1. Router: logits = x Wr^T (+bias), top-k by descending logit (ties to the
// lower expert index), softmax over the k selected logits.
//
// The product is a tall-skinny contraction (E <= 64 outputs per token), bound
// by reading x from HBM once.
//
// bf16 (route_mfma_kernel): a block of 16 wavefronts (8 beyond 32 experts) owns up to 16 tokens.  The
// reduction over H is cut into units of 64 elements (one 128-byte line per
// token), dealt round robin to the wavefronts; for a unit, lane (r = lane % 16,
// g = lane / 16) loads bytes g*16 .. g*16+15 of both halves of token r's line and
// of expert row r's line (zero for rows >= E), and two 16x16x32 MFMAs add the
// unit to a 16 x 16 f32 tile per 16 experts.  Which element of the line meets
// which k index of the MFMA does not matter as long as x and Wr use the same
// mapping.  Several units' loads are issued before their MFMAs to cover the
// HBM latency; with 16 wavefronts a row of 4096 elements is a single such batch
// per wavefront.  The wavefronts' tiles are added through LDS.
//
// f32 (route_kernel): on the vector ALUs.  A block of four wavefronts owns
// TPB = 64 / EP tokens (EP = experts padded to 8, 16, 32 or 64) and splits the
// reduction over its 256 lanes: every lane takes 8 consecutive elements per
// step and keeps TPB * EP = 64 float partial sums, folded over the lanes of a
// wavefront with a halving butterfly (63 cross-lane moves: lane j ends up with
// the sum of value j) and over the four wavefronts through LDS.
//
// In both, the selection and the softmax are done by one lane per (token, expert).
//
// With at most 16 tokens of bf16 data one block has all of them, and in moe_layer it does the permutation too, with the
// counting sort of moe_permute.hip on the ids that it has in LDS: a launch less, which is 4 to 5 us of a call that can
// be as short as 30.  With f32 data the same is done for short rows (route_place_f32_kernel).
#include <algorithm>

#include "moe_place.h"

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void load8(const float* base, size_t elem, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(base + elem);
    const float4 b = *reinterpret_cast<const float4*>(base + elem + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// The maximum over groups of EP lanes (a power of two), in all their lanes.  Inside rows of 16 lanes with data-parallel moves, which
// answer at once where a shuffle goes through LDS.
template <int CTRL>
__device__ __forceinline__ float max_dpp(float v) {
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false)));
}
template <int EP>
__device__ __forceinline__ float group_max(float v) {
    static_assert(EP >= 8, "");
    v = max_dpp<0xB1>(v);                            // lane ^ 1
    v = max_dpp<0x4E>(v);                            // lane ^ 2
    v = max_dpp<0x141>(v);                           // the mirror lane of eight
    if (EP >= 16) v = max_dpp<0x140>(v);             // the mirror lane of sixteen
    if (EP >= 32) v = fmaxf(v, __shfl_xor(v, 16, 64));
    if (EP >= 64) v = fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)));
    return v;
}

// Top-k of lg[0 .. E) by descending value (the lower index keeps a tie) and the softmax over the selected values, for token
// tok, by EP lanes of one wavefront (EP = experts padded to a power of two; lane `le` of the group holds expert le): k rounds
// of a maximum over the lanes and a ballot for its first holder.  One lane per token took k * E steps of LDS latency
// each: with 64 experts, 8 per token, 777 tokens the launch took 34 us, then 17, and 15.6 with the maximum by data-parallel moves instead of shuffles (the f32 kernel with 16384 and more tokens of a power
// of two of elements loses 2 - 5 %, 65536 tokens of 4096, 8 experts: 201 / 212; with fewer it gains as much).  A NaN is selected only when no free expert precedes it, as
// a scan that keeps the first and replaces it by what compares greater would do.  Every lane of the wavefront calls this; `live`: the token exists.
template <int EP>
__device__ __forceinline__ void select_top_k(const float* lg, int E, int k, int tok, bool live, int32_t* __restrict__ ids,
                                             float* __restrict__ w, int32_t* s_ids = nullptr, float* s_w = nullptr) {
    const int lane = threadIdx.x & 63, le = lane & (EP - 1);
    auto group = [&](uint64_t m) __attribute__((always_inline)) {    // this group's bits of a ballot
        return EP == 64 ? m : (m >> (lane - le)) & ((1ull << (EP & 63)) - 1);
    };
    const float v = le < E ? lg[le] : 0.f;
    const bool nan = v != v;
    const uint64_t nans = group(__ballot(nan));
    bool free_e = le < E;
    float first = 0.f, den = 0.f, my_p = 0.f;
    int my_id = 0;
    for (int s = 0; s < k; ++s) {
        const int f0 = __ffsll((long long)group(__ballot(free_e))) - 1;      // s < k <= E: there is one
        float bv = free_e && !nan ? v : -INFINITY;
        bv = group_max<EP>(bv);
        const int top = __ffsll((long long)group(__ballot(free_e && !nan && v == bv))) - 1;
        const bool take_nan = (nans >> f0) & 1;
        const int best = take_nan ? f0 : top;
        if (take_nan) bv = NAN;
        free_e = free_e && le != best;
        if (s == 0) first = bv;
        const float p = __expf(bv - first);
        den += p;
        if (le == s) {
            my_id = best;
            my_p = p;
        }
    }
    const float inv = 1.0f / den;
    if (live && le < k) {
        ids[(size_t)tok * k + le] = my_id;
        w[(size_t)tok * k + le] = my_p * inv;
        if (s_ids) {
            s_ids[tok * k + le] = my_id;
            s_w[tok * k + le] = my_p * inv;
        }
    }
}

// The permutation of R <= 1024 rows by one block of NW wavefronts that has their ids and weights in LDS.  cnt: 16 x
// MOE_MAX_EXPERTS words of LDS, start: MOE_MAX_EXPERTS.  Starts and ends its use of them behind barriers of its own.
template <int NW>
__device__ __forceinline__ void place_rows(const int32_t* s_ids, const float* s_w, int R, int E, int32_t (*cnt)[MOE_MAX_EXPERTS],
                                           int32_t* start, const PlaceOut& o) {
    constexpr int P = 16 / NW;                               // wavefront passes: 16 of them cover the rows
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    for (int i = threadIdx.x; i < 16 * MOE_MAX_EXPERTS; i += NW * 64) cnt[0][i] = 0;
    if (o.status && threadIdx.x < 4) o.status[threadIdx.x] = 0;
    __syncthreads();
    int my_id[P], my_rank[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = (p * NW + wave) * 64 + lane;
        my_id[p] = i < R ? s_ids[i] : -1;
        const uint64_t m = same_expert(my_id[p], E);
        my_rank[p] = lanes_below(m, lane);
        if (m && my_rank[p] == 0) cnt[p * NW + wave][my_id[p]] = __popcll(m);
    }
    __syncthreads();
    if (wave == 0) {
        int run = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int c = cnt[j][lane];                      // zero beyond the experts
            cnt[j][lane] = run;
            run += c;
        }
        int incl = run;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(incl, d, 64);
            if (lane >= d) incl += u;
        }
        start[lane] = incl - run;
        if (lane < E) {
            o.offsets[lane] = incl - run;
            o.counts[lane] = run;
        }
        if (lane == E - 1) o.offsets[E] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = (p * NW + wave) * 64 + lane, e = my_id[p];
        if (e >= 0) {
            const int r = start[e] + cnt[p * NW + wave][e] + my_rank[p];
            o.row_of[i] = r;
            o.row_src[r] = i;
            o.row_w[r] = s_w[i];
        }
    }
}

// NE: 16-expert tiles (experts padded to 16, 32 or 64); NW: wavefronts of a block; PLACE: the one block of the launch places
// the rows as well.
template <int NE, int NW, bool PLACE>
__device__ __forceinline__ void route_mfma(const char* __restrict__ x, const char* __restrict__ Wr, const float* __restrict__ bias,
                                           int32_t* __restrict__ ids, float* __restrict__ w, float* __restrict__ logits,
                                           int T, int H, int E, int k, int tpb, const PlaceOut& place) {
    constexpr int EP = NE * 16;
    // Units whose loads are in flight together.  Beyond 32 experts two: with four a wavefront needs 193 registers and only one
    // block fits a compute unit; 65536 tokens of 2048, 64 experts, 8 per token: 251 us with four, 156 with two, 777 tokens 17
    // either way; 65536 tokens, 33 experts, 5 per token: 172 and 105.
    constexpr int UB = NE <= 2 ? 4 : 2;
    __shared__ float s_part[NW][16][EP];
    __shared__ float s_logit[16][EP];
    __shared__ int32_t s_ids[PLACE ? 16 * MOE_MAX_EXPERTS : 1];
    __shared__ float s_w[PLACE ? 16 * MOE_MAX_EXPERTS : 1];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * tpb;
    const int r = lane & 15, g = lane >> 4;
    const size_t row_bytes = (size_t)H * 2;
    const char* xa = x + (size_t)min(t0 + min(r, tpb - 1), T - 1) * row_bytes + g * 16;      // rows past the block's tokens repeat the last one
    const char* wb[NE];
    bool wv[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        const int e = n * 16 + r;
        wv[n] = e < E;
        wb[n] = Wr + (size_t)min(e, E - 1) * row_bytes + g * 16;
    }
    f32x4 acc[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    const int units = H >> 6;
    for (int ub = wave; ub < units; ub += NW * UB) {
        bf16x8 a[UB][2], b[NE][UB][2];
#pragma unroll
        for (int j = 0; j < UB; ++j) {
            const int u = ub + NW * j;
            const bool ok = u < units;                         // the same for the whole wavefront
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const size_t off = (size_t)u * 128 + h * 64;
                a[j][h] = ok ? *reinterpret_cast<const bf16x8*>(xa + off) : zero;
#pragma unroll
                for (int n = 0; n < NE; ++n) b[n][j][h] = (ok && wv[n]) ? *reinterpret_cast<const bf16x8*>(wb[n] + off) : zero;
            }
        }
#pragma unroll
        for (int j = 0; j < UB; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int n = 0; n < NE; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][h], b[n][j][h], acc[n], 0, 0, 0);
    }
    // lane (r, g) holds tokens g*4 .. g*4+3 of expert n*16 + r
#pragma unroll
    for (int n = 0; n < NE; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) s_part[wave][g * 4 + i][n * 16 + r] = acc[n][i];
    __syncthreads();
    for (int v = threadIdx.x; v < tpb * EP; v += NW * 64) {
        const int t = v / EP, e = v % EP;
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) sum += s_part[q][t][e];
        if (bias != nullptr && e < E) sum += bias[e];
        s_logit[t][e] = sum;
        if (logits && e < E && t0 + t < T) logits[(size_t)(t0 + t) * E + e] = sum;
    }
    __syncthreads();
    constexpr int TW = 64 / EP;                              // tokens a wavefront selects for at a time
    const int live = min(tpb, T - t0);
    for (int t = wave * TW; t < live; t += NW * TW)          // the whole wavefront, as long as its first token exists
        select_top_k<EP>(s_logit[t + lane / EP], E, k, t0 + t + lane / EP, t + lane / EP < live, ids, w, PLACE ? s_ids : nullptr, PLACE ? s_w : nullptr);
    if constexpr (PLACE) {
        static_assert(sizeof(s_part) >= 16 * MOE_MAX_EXPERTS * 4 && sizeof(s_logit) >= MOE_MAX_EXPERTS * 4, "");
        place_rows<NW>(s_ids, s_w, T * k, E, (int32_t(*)[MOE_MAX_EXPERTS])s_part, (int32_t*)s_logit, place);
    }
}

template <int NE, int NW>
__global__ __launch_bounds__(NW * 64) void route_mfma_kernel(const char* __restrict__ x, const char* __restrict__ Wr, const float* __restrict__ bias,
                                                             int32_t* __restrict__ ids, float* __restrict__ w, float* __restrict__ logits,
                                                             int T, int H, int E, int k, int tpb) {
    route_mfma<NE, NW, false>(x, Wr, bias, ids, w, logits, T, H, E, k, tpb, PlaceOut{});
}

template <int NE, int NW>
__global__ __launch_bounds__(NW * 64) void route_place_kernel(const char* __restrict__ x, const char* __restrict__ Wr, const float* __restrict__ bias,
                                                              int32_t* __restrict__ ids, float* __restrict__ w, int T, int H, int E, int k,
                                                              const PlaceOut place) {
    route_mfma<NE, NW, true>(x, Wr, bias, ids, w, nullptr, T, H, E, k, 16, place);
}

// EP: experts padded to a compile-time bound (a power of two, 8..64).  The logits of the 64 / EP tokens from t0 on, over the chunks
// of eight elements first, first + step, ..: lane j of a wavefront gets the sum of value j = token * EP + expert over its lanes.
template <int EP>
__device__ __forceinline__ float partial_logits(const float* __restrict__ x, const float* __restrict__ Wr, int t0, int T, int H, int E,
                                                int first, int step) {
    constexpr int TPB = 64 / EP;                      // tokens
    const int lane = threadIdx.x & 63;
    float acc[64];                                    // value v = t * EP + e
#pragma unroll
    for (int v = 0; v < 64; ++v) acc[v] = 0.f;

    const int chunks = H >> 3;
    for (int c = first; c < chunks; c += step) {
        float xv[TPB][8];
#pragma unroll
        for (int t = 0; t < TPB; ++t) {
            const int tt = min(t0 + t, T - 1);           // rows past the end repeat the last token
            load8(x, (size_t)tt * H + (size_t)c * 8, xv[t]);
        }
#pragma unroll
        for (int e = 0; e < EP; ++e) {
            if (e < E) {
                float wv[8];
                load8(Wr, (size_t)e * H + (size_t)c * 8, wv);
#pragma unroll
                for (int t = 0; t < TPB; ++t)
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc[t * EP + e] = fmaf(xv[t][i], wv[i], acc[t * EP + e]);
            }
        }
    }
    // halving butterfly over the lanes: in the step with mask m a lane keeps the half of its
    // values that its bit m selects and receives the partner's sums for that half
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const bool upper = (lane & m) != 0;
#pragma unroll
        for (int i = 0; i < m; ++i) {
            const float keep = upper ? acc[i + m] : acc[i];
            const float give = upper ? acc[i] : acc[i + m];
            acc[i] = keep + __shfl_xor(give, m, 64);
        }
    }
    return acc[0];
}

template <int EP>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ x, const float* __restrict__ Wr,
                                                    const float* __restrict__ bias, int32_t* __restrict__ ids,
                                                    float* __restrict__ w, float* __restrict__ logits,
                                                    int T, int H, int E, int k) {
    constexpr int TPB = 64 / EP;                      // tokens per block
    __shared__ float s_part[4][64];
    __shared__ float s_logit[64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * TPB;
    s_part[wave][lane] = partial_logits<EP>(x, Wr, t0, T, H, E, threadIdx.x, 256);
    __syncthreads();
    if (threadIdx.x < 64) {
        const int v = threadIdx.x, t = v / EP, e = v % EP;
        float sum = (s_part[0][v] + s_part[1][v]) + (s_part[2][v] + s_part[3][v]);
        if (bias != nullptr && e < E) sum += bias[e];
        s_logit[v] = sum;
        if (logits && e < E && t0 + t < T) logits[(size_t)(t0 + t) * E + e] = sum;
    }
    __syncthreads();
    if (wave == 0) select_top_k<EP>(s_logit + lane / EP * EP, E, k, t0 + lane / EP, t0 + lane / EP < T, ids, w);
}

// Few tokens of a short row: a row has one chunk of eight elements per lane at most, so a wavefront of the kernel above has all the
// work of its block.  Here it is one of the kPlaceWaves of the only block, which then places the rows as well.  The same bits.
// 16 wavefronts would take twice the tokens, but one block of them is slower than the launch it saves, us for the layer of 256 x 512 (8
// experts, 2 per token), 8 / 16 wavefronts: 64 tokens 25 / 27, 65 (two launches / one) 26 / 28, 128: 30 / 35.
constexpr int kPlaceWaves = 8, kPlaceElements = 512;
constexpr int experts_padded(int E) { return E <= 8 ? 8 : E <= 16 ? 16 : E <= 32 ? 32 : 64; }

template <int EP>
__global__ __launch_bounds__(kPlaceWaves * 64) void route_place_f32_kernel(const float* __restrict__ x, const float* __restrict__ Wr,
                                                                          const float* __restrict__ bias, int32_t* __restrict__ ids,
                                                                          float* __restrict__ w, int T, int H, int E, int k, const PlaceOut place) {
    constexpr int TPB = 64 / EP;                      // tokens per wavefront
    __shared__ float s_logit[kPlaceWaves][64];
    __shared__ int32_t s_ids[kPlaceWaves * TPB * EP];  // k <= E <= EP
    __shared__ float s_w[kPlaceWaves * TPB * EP];
    __shared__ int32_t s_cnt[16][MOE_MAX_EXPERTS], s_start[MOE_MAX_EXPERTS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = wave * TPB;
    if (t0 < T) {
        const int e = lane % EP;
        float sum = partial_logits<EP>(x, Wr, t0, T, H, E, lane, 64);
        if (bias != nullptr && e < E) sum += bias[e];
        s_logit[wave][lane] = sum;                    // read by this wavefront alone
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        select_top_k<EP>(s_logit[wave] + lane / EP * EP, E, k, t0 + lane / EP, t0 + lane / EP < T, ids, w, s_ids, s_w);
    }
    place_rows<kPlaceWaves>(s_ids, s_w, T * k, E, s_cnt, s_start, place);
}

template <int EP>
int launch_f32(const moe_shape& s, const void* x, const void* Wr, const float* bias, int32_t* ids, float* w,
               float* logits, hipStream_t st, const PlaceOut* place) {
    if (place) {
        hipLaunchKernelGGL((route_place_f32_kernel<EP>), dim3(1), dim3(kPlaceWaves * 64), 0, st, (const float*)x, (const float*)Wr, bias, ids, w,
                           s.T, s.H, s.E, s.k, *place);
        MOE_HIP_TRY(hipGetLastError());
        return MOE_OK;
    }
    constexpr int tokens_per_block = 64 / EP;
    const dim3 grid((s.T + tokens_per_block - 1) / tokens_per_block), block(256);
    hipLaunchKernelGGL((route_kernel<EP>), grid, block, 0, st, (const float*)x, (const float*)Wr, bias, ids, w, logits, s.T,
                       s.H, s.E, s.k);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

template <int NE, int NW>
int launch_bf16(const moe_shape& s, const void* x, const void* Wr, const float* bias, int32_t* ids, float* w,
                float* logits, hipStream_t st, const PlaceOut* place) {
    // Tokens of a block: as few as give every compute unit one, 16 at most (the rows of the MFMA beyond them repeat the last token: no more
    // memory, the same sums).  Blocks of 16 tokens left most compute units idle below 4096 tokens, and one brings only about 25 GB/s from
    // HBM.  us for the launch with 16 / this many, x and Wr from HBM: Mixtral-8x7B shape 36 tokens 8.6 / 6.3, 256: 9.1 / 6.4, 1000: 9.8 / 7.4, 3000: 10.4 / 9.9; DBRX shape
    // 600 tokens 16.8 / 11.9; 64 experts of 2048, 8 per token, 777 tokens 17.5 / 13.8.  Fewer than a round of blocks needs is slower: 1000 tokens by 2: 11.8.
    constexpr int kComputeUnits = 256;               // MI355X
    const int tpb = std::min(16, (s.T - 1) / kComputeUnits + 1);
    const dim3 grid((s.T + tpb - 1) / tpb), block(NW * 64);
    if (place)
        hipLaunchKernelGGL((route_place_kernel<NE, NW>), dim3(1), block, 0, st, (const char*)x, (const char*)Wr, bias, ids, w, s.T, s.H, s.E,
                           s.k, *place);
    else
        hipLaunchKernelGGL((route_mfma_kernel<NE, NW>), grid, block, 0, st, (const char*)x, (const char*)Wr, bias, ids, w, logits, s.T, s.H,
                           s.E, s.k, tpb);
    MOE_HIP_TRY(hipGetLastError());
    return MOE_OK;
}

}  // namespace

bool route_places(const moe_shape& s) {
    if (s.T <= 0) return false;
    if (s.dtype == MOE_DTYPE_BF16) return s.T <= 16;
    return s.H <= kPlaceElements && s.T <= kPlaceWaves * 64 / experts_padded(s.E);
}

int launch_route(const moe_shape& s, const void* x, const void* Wr, const float* bias, int32_t* ids, float* w,
                 float* logits, hipStream_t st, const PlaceOut* place) {
    if (s.T == 0) return MOE_OK;
    if (place && (!route_places(s) || logits)) return MOE_ERR_INVALID_ARG;
    if (s.dtype == MOE_DTYPE_BF16) {
        if (s.E <= 16) return launch_bf16<1, 16>(s, x, Wr, bias, ids, w, logits, st, place);
        if (s.E <= 32) return launch_bf16<2, 16>(s, x, Wr, bias, ids, w, logits, st, place);
        return launch_bf16<4, 8>(s, x, Wr, bias, ids, w, logits, st, place);
    }
    if (s.E <= 8) return launch_f32<8>(s, x, Wr, bias, ids, w, logits, st, place);
    if (s.E <= 16) return launch_f32<16>(s, x, Wr, bias, ids, w, logits, st, place);
    if (s.E <= 32) return launch_f32<32>(s, x, Wr, bias, ids, w, logits, st, place);
    return launch_f32<64>(s, x, Wr, bias, ids, w, logits, st, place);
}

}  // namespace moe
