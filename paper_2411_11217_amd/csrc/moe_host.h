// Declarations of the host-only part of the library (shape checks, page geometry, the weight packer): no GPU
// types, so plain C++ translation units can include it.  Nothing here is part of the C ABI (that is include/moe.h).
#pragma once

#include <stdint.h>

#include "moe.h"

namespace moe {

// Weight tile: 128 output features x 64 reduction elements (see the page
// format in moe.h).  A bf16 tile is stored as two half-tiles of 32 reduction
// elements each.
constexpr int kTileN = 128;
constexpr int kTileK = 64;

struct Geom {
    int esize;            // bytes per element of dtype
    int64_t tile_bytes;   // kTileN * kTileK * esize
    int64_t tpp;          // tiles per page
    int64_t kt_gu;        // H / 64  : k-tiles of the gate/up product
    int64_t ft;           // F / 128 : f-tiles (each has a W1 and a W3 tile row)
    int64_t tiles_gu;     // 2 * ft * kt_gu
    int64_t kt_d;         // F / 64  : k-tiles of the down product
    int64_t dt;           // H / 128 : d-tiles
    int64_t tiles_d;      // dt * kt_d
    int64_t pages_gu, pages_d, ppe;   // pages per expert: GU group, D group, both
};

int validate_shape(const moe_shape* s);          // MOE_OK or error
Geom geometry(const moe_shape& s);               // shape must be valid

// MOE_OK, MOE_ERR_PAGE_NOT_RESIDENT (an entry outside [0, pool_pages)) or, with need_distinct,
// MOE_ERR_INVALID_ARG when two entries name the same slot.  table: host int32[E][ppe].
int check_table_host(const moe_shape& s, const Geom& g, const int32_t* table, int64_t pool_pages, bool need_distinct);

// Copies one 128 x 64 weight tile between a dense row-major matrix (leading dimension ld elements)
// and its page image.
void copy_tile(char* page_tile, char* dense, int64_t ld, int esize, bool to_page);

// Whether two buffers of na and nb bytes share any of them.
inline bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
    const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
    return p < q ? q - p < (uintptr_t)na : p - q < (uintptr_t)nb;
}

// Dense paged matrices (moe_linear): MOE_OK or an error; pages of one matrix (shape must be valid).
int validate_linear(const moe_linear_shape* s);
int64_t linear_pages(const moe_linear_shape& s);

// Where the dense linear map takes the kernel for few rows (csrc/moe_ffn_rows_bf16.hip): as long as blocks of 64 columns and 128
// rows, or with more than 128 rows of 128 columns and 64 rows, make one round on the 256 compute units (which blocks it has
// then is linear_rows_block's choice), and with a short k and few rows.
//   One matrix alone has too few columns to fill the chip with 256-row blocks (moe_ffn_gemm_bf16.h).  us, those blocks / this
// kernel, weights where the call before left them | weights from HBM (copies that exceed the last-level cache in turn): 4096 x
// 6144 (K x N) 1 token - | 45 / 15, 100: - | 47 / 30; 6144 x 9216 16 tokens 33 / 21 | 48 / 29, 100: 41 / 39 | 59 / 50;
// 4096 x 16384 (one full round) 16 tokens 25 / 22 | 42 / 27, 64: 31 / 24 | 40 / 30, 128: 32 / 32 | 46 / 42; 8192 x 1024 600
// tokens 75 / 47 | 76 / 50 (36 with the blocks of 64 rows x 64 columns that it has now up to 256 of them).
//   Beyond one round a block's way through all of k is paid for twice: 4096 x 18432 16 tokens 26 / 33 | 38 / 39, 128: 33 / 51 | 48
// / 73; 4096 x 32000 64 tokens 44 / 46 | 50 / 55, 100: 47 / 64 | 53 / 75; 4096 x 128256 128 tokens 224 / 304.
//   A short way makes the other kernel's blocks (one per compute unit, set-up and tile search of 2 us) the longer ones again:
// 1024 x 65536 32 tokens 28 / 25 | 33 / 29, 64: 31 / 30 | 36 / 36, 128: 34 / 36 | 39 / 50; 1024 x 18432 32 tokens 12 / 12 | 17 / 14;
// 1536 x 18432 32 tokens 14 / 15 | 21 / 19, 1536 x 65536: 37 / 33 | 44 / 41; 2048 x 32768 32 tokens 24 / 23 | 28 / 27, but 2048 x 18432: 16
// / 19 | 22 / 23.
//   With more than 128 rows and blocks of 64 rows x 128 columns: us, row tiles of 128 or 256 / this kernel, 4096 x
// 6144 300 tokens 35 / 26 | 41 / 34; 6144 x 9216 140: 44 / 35 | 53 / 43; 4096 x 10880 192: 37 / 28 | 43 / 37; 2048 x 6144 300: 23 / 16 | 27 / 20; 4096 x 4096 450: 29 / 25 | 32
// / 29.
inline bool linear_takes_rows_kernel(int T, int K, int N) {
    constexpr int64_t kComputeUnits = 256;           // MI355X
    return (int64_t)(N / 64) * (((int64_t)T + 127) / 128) <= kComputeUnits || (K <= 1536 && T <= 32) || (T > 128 && (((int64_t)T + 63) / 64) * (N / 128) <= kComputeUnits);
}

// Its blocks: `rows` rows and `groups` groups of 16 columns.  64 rows, and the fewest groups with which all blocks make one round; with up to
// 64 rows four groups are the most.
//   With up to 32 rows and one or two groups 32 rows: the blocks of 64 have four (two) groups of wavefronts for the rows, and those without any load the weights all the
// same.  us, 64 rows / 32, weights where the call before left them | from HBM: 4096 x 4096 1 token 13.2 / 12.6 | 14.2 / 12.9, 32: 13.8 / 13.0 | 14.6 / 13.6; 14336 x 4096 8: 38.2 /
// 37.1 | 39.5 / 37.7; 512 x 512 16: 4.5 / 4.3; 1024 x 6144 1: 5.4 / 5.2 | 7.0 / 6.2; 8192 x 4224 1: 22.0 / 22.2 | 24.8 / 24.4.
//   Up to eight column tiles of a row tile run on as many XCDs, each of which fetches the rows for itself.  More than 216 blocks of one or two groups then ask for
// more of them than arrive, and half as many have it done sooner, except with a short k.  us, one / two / four groups: 4096 x 128 1700 tokens (216 blocks of one) 21.0 / 17.9 /
// 21.2, 2000: 23.2 / 18.1 / 21.1, 3300 (208 of two) - / 20.8 / 21.5, 4000: - / 24.0 / 21.7; 2048 x 256 1700 (216 of two) - / 13.0 / 13.0, 2000: - / 14.4 / 13.3; 8192 x 128 4000: - / 52 / 41;
// 1152 x 128 4000: - / 9.6 / 10.2.  The line is late by 5 to 15 % for some k (2048 x 128 2500: - / 13.0 / 12.5, 3000: - / 14.7 / 12.8;
// 8192 x 256 1600: - / 36.1 / 34.8) and early for none by as much.
//   With an odd number of row tiles of 64 the blocks of eight groups leave more compute units idle than blocks of 128 rows x 64 columns do, and
// weights from HBM, which a program with more than one layer has, come at the rate of the compute units that ask for them.  us, 128 x 64 /
// 64 x 128, weights where the call before left them | from HBM: 4096 x 5120 300 tokens 27.8 / 24.5 | 29.9 / 32.7; 4096 x 8192 192: 28.4 / 25.5 | 31.4 / 35.0;
// 14336 x 5120 320: 85 / 71 | 92 / 99; 2048 x 3072 576: 17.2 / 15.6 | 18.0 / 19.0; 3072 x 1920 960: 24.4 / 23.9 | 24.9 / 25.8.  Not with at most 24 rows in the last of
// them (4096 x 5120 264: 27.4 / 24.2 | 29.7 / 29.5; 8192 x 8192 150: 51 / 42 | 60 / 55; 4096 x 3072 530: 28.3 / 24.5 | 29.5 / 29.0), a short k (1536 x 5120 300: 14.2 / 12.9 | 15.5 / 15.9, 1536 x 3072 576: 14.2 / 12.8 |
// 14.8 / 14.2, 2048 x 1920 960: 17.7 / 15.8 | 17.7 / 15.9), many row tiles, where one more or less is nothing (4096 x 512 4000: 42.8 / 26.2 | 42.8 / 26.9), or an even number (4096 x 16384 100: 32 / 29 | 39 / 37).
//   Where the two sides differ, weights from HBM decide: 65 to 96 rows with six groups lose where a matrix of 80 MB and more is in the last-level cache (the second row
// tile's blocks, with 32 rows at most, run ahead of the first one's and read the weights again), 128 x 64 / six / eight groups: 4096 x 12288 72 tokens 26.5 / 32.8 / 24.3 | 34.4 / 28.4 / 32.5, 8192 x
// 12288 65: 47.8 / 58.8 / 41.8 | 60.6 / 53.8 / 56.0, 1024 x 12288 65: 9.9 / 10.3 / 9.7 | 12.4 / 11.5 / 12.2.
//   Up to 96 rows and a short k have the blocks of 128 rows in place of five, six and eight groups too: the set-up of the second row tile's blocks is what
// counts.  us, 128 x 64 / 64 rows: 128 x 9216 72 tokens 5.6 / 6.0 | 6.4 / 6.6, 128 x 16384 65: 5.8 / 6.2 | 6.6 / 7.2; 512 x 12288 65: 7.3 / 7.7 | 8.9 / 8.9, 96: 7.9 / 7.9 | 9.4 / 9.1; but
// 256 x 16384 100: 7.1 / 7.0 | 8.1 / 7.9, 512 x 16384 100: 9.2 / 8.9 | 10.6 / 10.2, 1024 x 12288 65: 9.9 / 10.4 | 12.5 / 11.5.
struct LinearBlock {
    int rows, groups;
};
inline LinearBlock linear_rows_block(int T, int K, int N) {
    constexpr int64_t kComputeUnits = 256;
    const int64_t groups = N / 16, row_tiles = ((int64_t)T + 63) / 64;
    auto one_round = [&](int g) { return row_tiles * ((groups + g - 1) / g) <= kComputeUnits; };
    const int rows = T <= 32 ? 32 : 64;
    auto crowded = [&](int g) { return K >= 1536 && groups <= 8 * g && row_tiles * ((groups + g - 1) / g) > 216; };
    if (one_round(1) && !crowded(1)) return {rows, 1};
    if (one_round(2) && !crowded(2)) return {rows, 2};
    if (T <= 64 || one_round(4)) return {64, 4};
    const bool tall_one_round = (N / 64) * (((int64_t)T + 127) / 128) <= kComputeUnits;
    if (tall_one_round && T <= 96 && K <= 512) return {128, 4};
    if (one_round(5)) return {64, 5};
    if (one_round(6)) return {64, 6};
    if (tall_one_round && row_tiles % 2 && row_tiles < 32 && (T - 1) % 64 >= 24 && K >= (row_tiles < 10 ? 2048 : 3072)) return {128, 4};
    return {64, 8};
}

}  // namespace moe
