// a2. Permutation of routed rows by expert: a stable counting sort of the flat
// indices i = t*k + slot by expert id, in two small kernels plus a row copy.
//
//   place   : every block owns kChunk consecutive flat indices.  Lanes of a wavefront pass with the same expert find each
//             other with a ballot per bit of the id (six for 64 experts); the mask gives an entry's rank among them and
//             their number, staged in LDS per pass.  Up to kCountInPlace blocks, every block also counts the ids of all the others itself
//             (integer sums in LDS): those before its own chunk give its base inside every expert, all of them give
//             counts[], whose scan over the lanes is offsets[] (block 0 writes both).  The rank of an entry inside its
//             expert is offsets[e] + base + (entries of earlier wavefront passes of the block) + its rank in its pass.
//   count   : with more blocks, or when row_of takes the memory of the ids, a launch of its own counts every block's chunk
//             (block_counts[block][E]) and the placing blocks add these up; with more than kScanInPlace blocks a
//             one-block scan kernel does the sums once instead (block_base, counts, offsets).
//             The placement is a pure function of the input, hence stable (ascending flat index inside an
//             expert) and reproducible.
//   gather  : x_perm[row] = x[row_src[row] / k], 16 bytes per lane, one block per row.
#include "moe_place.h"

namespace moe {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kPasses = 4;
constexpr int kChunk = kThreads * kPasses;   // flat indices per block
// Up to this many blocks the placing blocks read all ids instead of a count launch (4.7 us and more).
constexpr int kCountInPlace = 16;
constexpr int kScanInPlace = 256;            // up to this many blocks every placing block sums the block counts itself

// cnt[pass * kWaves + wave][e] = entries for expert e of every wavefront pass of this block's chunk, and each entry's
// rank among those of its pass.  Ends with a barrier.
__device__ __forceinline__ void count_chunk(const int (&my_id)[kPasses], int E, int32_t (*cnt)[MOE_MAX_EXPERTS], int (&my_rank)[kPasses]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kPasses * kWaves * MOE_MAX_EXPERTS; i += kThreads) cnt[0][i] = 0;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const uint64_t m = same_expert(my_id[p], E);
        my_rank[p] = lanes_below(m, lane);
        if (m && my_rank[p] == 0) cnt[p * kWaves + wave][my_id[p]] = __popcll(m);
    }
    __syncthreads();
}

__global__ __launch_bounds__(kThreads) void count_kernel(const int32_t* __restrict__ ids, int R, int E,
                                                         int32_t* __restrict__ block_counts) {
    __shared__ int32_t cnt[kPasses * kWaves][MOE_MAX_EXPERTS];
    const int base = blockIdx.x * kChunk;
    int my_id[kPasses], my_rank[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {               // all loads under way at once
        const int i = base + p * kThreads + threadIdx.x;
        my_id[p] = i < R ? ids[i] : -1;
    }
    count_chunk(my_id, E, cnt, my_rank);
    for (int e = threadIdx.x; e < E; e += kThreads) {
        int sum = 0;
#pragma unroll
        for (int j = 0; j < kPasses * kWaves; ++j) sum += cnt[j][e];
        block_counts[(size_t)blockIdx.x * E + e] = sum;
    }
}

__global__ __launch_bounds__(64) void scan_kernel(const int32_t* __restrict__ block_counts, int nblocks, int E,
                                                  int32_t* __restrict__ block_base, int32_t* __restrict__ counts,
                                                  int32_t* __restrict__ offsets, int32_t* __restrict__ status) {
    __shared__ int32_t total[MOE_MAX_EXPERTS];
    const int e = threadIdx.x;
    if (status && threadIdx.x < 4) status[threadIdx.x] = 0;
    if (e < E) {
        int run = 0;
        for (int b = 0; b < nblocks; ++b) {
            const int c = block_counts[(size_t)b * E + e];
            block_base[(size_t)b * E + e] = run;
            run += c;
        }
        total[e] = run;
        counts[e] = run;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int j = 0; j < E; ++j) {
            offsets[j] = run;
            run += total[j];
        }
        offsets[E] = run;
    }
}

// block_base != null: the scan kernel has run (block_base, counts, offsets are inputs).  Else they are formed here, from
// block_counts[nblocks][E] or, when that is null, from the ids themselves, and block 0 writes counts[], offsets[] and clears
// status[0..3] when status is not null.
__global__ __launch_bounds__(kThreads) void place_kernel(const int32_t* __restrict__ ids,
                                                         const float* __restrict__ topk_w, int R, int E,
                                                         const int32_t* __restrict__ block_counts, int nblocks,
                                                         const int32_t* __restrict__ block_base,
                                                         int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                         int32_t* __restrict__ row_src, int32_t* __restrict__ row_of,
                                                         float* __restrict__ row_w, int32_t* __restrict__ status) {
    __shared__ int32_t cnt[kPasses * kWaves][MOE_MAX_EXPERTS];
    __shared__ int32_t start[MOE_MAX_EXPERTS];
    __shared__ int32_t others[kWaves][2][MOE_MAX_EXPERTS];     // ids of the chunks before / behind this block's, per wavefront
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = blockIdx.x * kChunk;
    const bool count_ids = !block_base && !block_counts && nblocks > 1;
    // sums over the other blocks' counts (loads under way during the ballots below)
    int before = 0, all = 0;
    if (threadIdx.x < E) {
        const int e = threadIdx.x;
        if (block_base) {
            before = offsets[e] + block_base[(size_t)blockIdx.x * E + e];
        } else if (block_counts) {
            for (int b = 0; b < nblocks; ++b) {
                const int c = block_counts[(size_t)b * E + e];
                all += c;
                if (b < (int)blockIdx.x) before += c;
            }
        }
    }
    if (!block_base && status && blockIdx.x == 0 && threadIdx.x < 4) status[threadIdx.x] = 0;
    int my_id[kPasses], my_rank[kPasses];
    float my_w[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {               // all loads under way at once
        const int i = base + p * kThreads + threadIdx.x;
        my_id[p] = i < R ? ids[i] : -1;
        my_w[p] = (row_w && i < R) ? topk_w[i] : 0.f;
    }
    if (count_ids) {
        for (int i = threadIdx.x; i < kWaves * 2 * MOE_MAX_EXPERTS; i += kThreads) others[0][0][i] = 0;
        __syncthreads();
        for (int b = 0; b < nblocks; ++b) {
            if (b == (int)blockIdx.x) continue;
            int id[kPasses];
#pragma unroll
            for (int p = 0; p < kPasses; ++p) {
                const int i = b * kChunk + p * kThreads + threadIdx.x;
                id[p] = i < R ? ids[i] : -1;
            }
#pragma unroll
            for (int p = 0; p < kPasses; ++p)
                if (id[p] >= 0 && id[p] < E) atomicAdd(&others[wave][b > (int)blockIdx.x][id[p]], 1);
        }
    }
    count_chunk(my_id, E, cnt, my_rank);
    // exclusive running sum over the (pass, wavefront) order in which flat indices grow; then the experts' starts
    if (wave == 0) {
        int run = 0;
        if (lane < E) {
            int c[kPasses * kWaves];
#pragma unroll
            for (int j = 0; j < kPasses * kWaves; ++j) c[j] = cnt[j][lane];
#pragma unroll
            for (int j = 0; j < kPasses * kWaves; ++j) {
                cnt[j][lane] = run;
                run += c[j];
            }
        }
        if (!block_base) {
            int total = block_counts ? all : run;
            if (count_ids && lane < E) {
#pragma unroll
                for (int q = 0; q < kWaves; ++q) before += others[q][0][lane];
                total += before;
#pragma unroll
                for (int q = 0; q < kWaves; ++q) total += others[q][1][lane];
            }
            int incl = total;                            // lanes beyond the experts add zeros
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int u = __shfl_up(incl, d, 64);
                if (lane >= d) incl += u;
            }
            before += incl - total;
            if (blockIdx.x == 0) {
                if (lane < E) {
                    offsets[lane] = incl - total;
                    counts[lane] = total;
                }
                if (lane == E - 1) offsets[E] = incl;
            }
        }
        start[lane] = before;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const int i = base + p * kThreads + threadIdx.x;
        const int e = my_id[p];
        if (i < R && e >= 0 && e < E) {                      // ids outside [0,E) are left unplaced
            const int r = start[e] + cnt[p * kWaves + wave][e] + my_rank[p];
            row_of[i] = r;
            row_src[r] = i;
            if (row_w) row_w[r] = my_w[p];
        }
    }
}

__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ x, const int32_t* __restrict__ row_src,
                                                          int k, int T, int row_vec, uint4* __restrict__ x_perm) {
    const int r = blockIdx.x;
    const int t = min(max(row_src[r] / k, 0), T - 1);   // stays in bounds even if ids were invalid
    const uint4* src = x + (size_t)t * row_vec;
    uint4* dst = x_perm + (size_t)r * row_vec;
    for (int c = threadIdx.x; c < row_vec; c += 256) dst[c] = src[c];
}

}  // namespace

size_t permute_workspace_bytes(const moe_shape& s) {
    const size_t R = (size_t)s.T * s.k;
    const size_t nblocks = (R + kChunk - 1) / kChunk;
    return 2 * std::max<size_t>(nblocks, 1) * s.E * sizeof(int32_t);
}

int launch_permute(const moe_shape& s, const int32_t* ids, const float* topk_w, const void* x, int32_t* counts,
                   int32_t* offsets, int32_t* row_src, int32_t* row_of, float* row_w, void* x_perm, void* ws,
                   int32_t* status_to_clear, hipStream_t st) {
    const int R = s.T * s.k;
    const int nblocks = std::max((R + kChunk - 1) / kChunk, 1);      // R == 0: one block writes the zero counts
    int32_t* block_counts = nullptr;
    int32_t* block_base = nullptr;
    // Blocks that count all ids themselves read them while others write row_of: a row_of in the memory of the ids gets the
    // count launch, behind which a block reads its own chunk alone, before it writes it.
    const bool same_memory = overlap(ids, (int64_t)R * 4, row_of, (int64_t)R * 4);
    if (nblocks > kCountInPlace || (nblocks > 1 && same_memory)) {
        block_counts = (int32_t*)ws;
        hipLaunchKernelGGL(count_kernel, dim3(nblocks), dim3(kThreads), 0, st, ids, R, s.E, block_counts);
        MOE_HIP_TRY(hipGetLastError());
    }
    if (nblocks > kScanInPlace) {
        block_base = block_counts + (size_t)nblocks * s.E;
        hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(64), 0, st, block_counts, nblocks, s.E, block_base, counts, offsets,
                           status_to_clear);
        MOE_HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(place_kernel, dim3(nblocks), dim3(kThreads), 0, st, ids, topk_w, R, s.E, block_counts, nblocks,
                       block_base, counts, offsets, row_src, row_of, row_w, status_to_clear);
    MOE_HIP_TRY(hipGetLastError());
    if (R > 0) {
        if (x && x_perm) {
            const int row_vec = s.H * (s.dtype == MOE_DTYPE_BF16 ? 2 : 4) / 16;
            hipLaunchKernelGGL(gather_rows_kernel, dim3(R), dim3(256), 0, st, (const uint4*)x, row_src, s.k, s.T, row_vec,
                               (uint4*)x_perm);
            MOE_HIP_TRY(hipGetLastError());
        }
    }
    return MOE_OK;
}

}  // namespace moe
