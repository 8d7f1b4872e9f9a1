// Products of packed codes on the matrix cores (gfx950).
//
// A batch of vectors turns the product into a contraction, so it runs on the matrix cores
// straight from the matrix entries, packed to 2 bits (ternary) or 1 bit (binary), whatever
// the kind of the handle (but for matrices of few rows, see use_packed); the redundancy a block of
// rows has is worth less there than the vectors that share one decoded weight.  The dense kind, the comparison point without any
// preprocessing beyond packing (the role the paper gives its low-bit multiplier baseline in
// Benchmarking Results), multiplies a single vector this way too.  Kernels:
//   few    16 rows x up to 4 vectors per wave, for 1 to 4 vectors; tall: 32 or 64 rows, on tall matrices, or 16 long ones
//   split  16 to 64 rows x 16 or 32 vectors per workgroup, the columns dealt to its eight waves; bound
//          by the latency of its loads (4096 x 14336, 16 bf16 vectors: 10.3 us; as 16 products of one
//          vector 78 us; with 32 vectors per workgroup, half of them padding, 14.4)
//   tile   128 rows x 128 vectors per workgroup of four or eight waves; bound by the matrix cores and
//          the decoding (4096 x 14336, 2048 bf16 vectors: 211 us = 1.14 PFLOP/s, 8.2 ms as single
//          products; a library product of 8192^3 reaches 1.21 PFLOP/s on the same card)
//   table  up to 256 columns and many rows: v stays in registers or LDS, waves go through the rows
// Tiles and workgroups of 32 vectors use v_mfma_f32_32x32x16_bf16 (measured 15.1 ns per instruction and SIMD against
// 12.7 for v_mfma_f32_16x16x32_bf16, which does half the work), the others the smaller one.
//
// Layout: [row group of 16][tile of 256 columns][lane][2 * BITS dwords], one load of 16
// (8) bytes per lane and tile.  Lane l holds row l%16 and the column slices 8*(l/16).. of the
// tile's eight 32-column steps.  A ternary dword d feeds steps 2d and 2d+1; pair slot p (0..7)
// has its even column in bits 14-2p.. and its odd column in bits 30-2p.., two's complement.  A
// binary dword d feeds steps 4d..4d+3; every step owns one bit of each of the eight nibbles.
//
// Decoding: after one AND (and a shift) every nibble of a dword is the 4-bit float of one
// entry (0100 = 2.0, 1100 = -2.0), and v_cvt_scalef32_pk_bf16_fp4 turns a byte, that is two
// entries, into two bf16: 11 instructions for 16 ternary entries of a lane where shifting and
// masking pairs into place took 15.  The nibbles come out in the order 4 0 5 1 6 2 7 3 of a
// slice's eight columns; v is brought into the same order when it is staged.
//
// float32 vectors are split exactly into three bf16 planes (top, middle and bottom 8
// significant bits) that take one MFMA each, so integer-valued inputs stay exact and nothing
// is lost against float32 inputs (elements below 2^-109 excepted, whose last bits a bf16 cannot
// hold).  Accumulation is float32 throughout and the order of the sums is fixed.  In split and tile,
// and up to four vectors, where every plane is a row of its own, the top plane has sums of its
// own: its products have few bits, so they add up almost exactly, and the other planes' rounding is
// 2^-8 of what it would be on top of them (14336 x 4096, 700 vectors, relative error against float64
// 4.6e-8, with all planes in one sum 5.6e-7).  The tables of up to 256 columns with more vectors add all
// planes into one: sums that short do not need it (at most 1.6e-7; the block patterns 1.6e-7 and more).
#include <cstdio>

#include "rsr_internal.h"

namespace rsr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// rows of v start anywhere: 16 bytes at the alignment of an element (the hardware takes any)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));

constexpr int kTileCols = kDenseTileCols;  // 256: eight 32-column steps
constexpr int kTileSteps = kTileCols / 32;
constexpr int kCUs = 256;

// ---- packing ---------------------------------------------------------------------------------
// Puts the code of column e (0..7) of a lane's slice in 32-column step st into the lane's dwords.
template <int BITS>
__device__ __forceinline__ void put_code(uint32_t (&word)[2 * BITS], int st, int e, uint32_t code) {
    if (BITS == 2) {
        const int p = 4 * (st & 1) + (e >> 1);
        word[st >> 1] |= code << ((e & 1 ? 30 : 14) - 2 * p);
    } else {
        constexpr int bit_of[4] = {2, 1, 0, 3};
        const int nibble = e < 4 ? 2 * e + 1 : 2 * (e - 4);
        word[st >> 2] |= code << (4 * nibble + bit_of[st & 3]);
    }
}

// One thread per (row group, tile, lane): eight loads of eight entries each.
template <int BITS>
__global__ __launch_bounds__(256) void k_pack_codes(const int8_t *__restrict__ M, int64_t rows, int64_t cols,
                                                    int64_t ntiles, uint32_t *__restrict__ tiled,
                                                    int *__restrict__ err_flag) {
    const int64_t ngroups = (rows + kDenseRows - 1) / kDenseRows;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= ngroups * ntiles * 64) return;
    const int lane = (int)(gid & 63);
    const int64_t gt = gid >> 6, G = gt / ntiles, t = gt - G * ntiles;
    const int64_t i = G * kDenseRows + (lane & 15);
    const int64_t j0 = t * kTileCols + 8 * (lane >> 4);
    uint32_t word[2 * BITS];
#pragma unroll
    for (int d = 0; d < 2 * BITS; ++d) word[d] = 0;
    uint32_t bad = 0;
    if (i < rows) {
        const int8_t *row = M + i * cols;
#pragma unroll
        for (int st = 0; st < kTileSteps; ++st) {
            const int64_t j = j0 + 32 * st;
            uint32_t x[2] = {0, 0};
            if (j + 8 <= cols) {
                const u32x2 y = *reinterpret_cast<const u32x2_any *>(row + j);
                x[0] = y.x;
                x[1] = y.y;
            } else {
                for (int e = 0; e < 8 && j + e < cols; ++e)
                    x[e >> 2] |= (uint32_t)(uint8_t)row[j + e] << (8 * (e & 3));
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // entries outside the alphabet: bits 2..7 not all equal to bit 1, or the code 10
                const uint32_t s = (x[h] >> 1) & 0x01010101u, o = x[h] & 0x01010101u;
                bad |= BITS == 2 ? ((x[h] ^ (s * 255u)) & 0xfcfcfcfcu) | (s & ~o) : x[h] & 0xfefefefeu;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                put_code<BITS>(word, st, e, (x[e >> 2] >> (8 * (e & 3))) & (BITS == 2 ? 3u : 1u));
            }
        }
    }
    if (bad) atomicOr(err_flag, 1);
#pragma unroll
    for (int d = 0; d < 2 * BITS; ++d) tiled[gid * 2 * BITS + d] = word[d];
}

// The same codes from the canonical artifacts (a handle made from bytes has no matrix), one workgroup
// per row group: LDS holds one word per column, the codes of the group's 16 rows, and every block that
// has rows in the group puts its digits there, a thread per pattern code.  The artifacts may be damaged:
// whatever they hold, no access leaves the block or LDS, and *err_flag |= 4 unless every pi is a
// permutation, the boundaries rise from 0 to the number of columns, no code has digits in rows that
// do not exist and no entry is in M+ and M- both.  The matrix itself is never
// formed: its rows x cols bytes can be more than all else that loading allocates.  (Loading 1024 x 1024
// binary 130 us, 4096 x 14336 fused k = 8 1.6 ms, with the matrix formed, packed and freed 180 us and
// 2.0 ms; few row groups of a wide matrix are bound by the latency of their chains: 40 x 32000 192 us.)
constexpr uint32_t kLongColumns = 128, kPieceColumns = 512;  // longer groups are cut up and dealt to the waves
constexpr __host__ __device__ int long_pieces(int cols) { return cols / (int)kLongColumns + 1; }  // the most there are

// Codes of the rows that digits [lo, hi) of pattern code c stand for, the first of them row `at` of the
// group.  Digits 0, 1, 2 are 0, +1, -1; pass 1 is M-.
template <int BITS>
__device__ __forceinline__ uint32_t row_bits(uint32_t c, int base, int pass, int lo, int hi, int at) {
    uint32_t bits = 0;
    if (base == 2) {
        c = (c >> lo) & ((1u << (hi - lo)) - 1u);
        if (BITS == 1) return c << at;
        c = (c | c << 8) & 0x00ff00ffu;
        c = (c | c << 4) & 0x0f0f0f0fu;
        c = (c | c << 2) & 0x33333333u;
        c = (c | c << 1) & 0x55555555u;
        return (pass ? 3u * c : c) << (2 * at);
    }
    for (int r = 0; r < hi; ++r, c /= 3u) {
        const uint32_t d = c % 3u;
        if (r >= lo && d) bits |= (d == 1 ? 1u : 3u) << (2 * (at + r - lo));
    }
    return bits;
}

struct RestorePass {
    const uint16_t *pi;
    const uint32_t *off;
};

template <int BITS>
__global__ __launch_bounds__(1024) void k_restore_codes(const RestorePass p0, const RestorePass p1, int npass,
                                                        int64_t rows, int cols, int k, int base, int64_t P,
                                                        int64_t ngroups, uint32_t *__restrict__ tiled,
                                                        int *__restrict__ err_flag) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint32_t *column = reinterpret_cast<uint32_t *>(smem);
    uint32_t *longs = column + cols;  // count, then {first position, length, codes} of the pieces of long groups
    const int tid = threadIdx.x, NT = blockDim.x;
    uint32_t *seen = longs + 1 + 3 * long_pieces(cols);  // a bit per column
    const int ntiles = (cols + kTileCols - 1) / kTileCols;
    bool bad = false;
    for (int64_t G = blockIdx.x; G < ngroups; G += gridDim.x) {
        for (int j = tid; j < cols; j += NT) column[j] = 0;
        const int64_t r0 = G * kDenseRows, r1 = min(r0 + kDenseRows, rows);
        for (int64_t b = r0 / k; b * k < r1; ++b) {
            const int lo = (int)max((int64_t)0, r0 - b * k), hi = (int)min((int64_t)k, r1 - b * k);
            const int at = (int)(b * k + lo - r0);  // row of the group that digit `lo` belongs to
            for (int ps = 0; ps < npass; ++ps) {
                const uint16_t *pib = (ps ? p1.pi : p0.pi) + b * cols;
                const uint32_t *ob = (ps ? p1.off : p0.off) + b * (P + 1);
                __syncthreads();
                if (tid == 0) longs[0] = 0;
                if (b * k >= r0)
                    for (int i = tid; i < (cols + 31) / 32; i += NT) seen[i] = 0;
                __syncthreads();
                if (b * k >= r0) {  // checked by the group its first row is in: a permutation, and all of it
                    for (int t = tid; t < cols; t += NT) {
                        const uint32_t j = pib[t], bit = 1u << (j & 31);
                        if (j >= (uint32_t)cols || (atomicOr(&seen[j >> 5], bit) & bit)) bad = true;
                    }
                    if (tid == 0 && (ob[0] != 0 || ob[1] > (uint32_t)cols || ob[P] != (uint32_t)cols)) bad = true;
                }
                auto put = [&](int j, uint32_t bits) {
                    // (a row of the column that M+ has set already cannot be in M- too)
                    if (j < cols && (atomicOr(&column[j], bits) & bits & (BITS == 1 ? 0xffffu : 0x55555555u))) bad = true;
                };
                // codes from here on have digits in rows behind the last one
                uint32_t code_end = 1;
                for (int64_t r = b * k; r < min((b + 1) * k, rows); ++r) code_end *= (uint32_t)base;
                for (int64_t c0 = 1 + tid; c0 < P; c0 += 4 * NT) {
                    uint32_t first[4], end[4];  // four codes in flight, and the first column of each
                    int column0[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int64_t c = min(c0 + i * NT, P - 1);
                        first[i] = ob[c];
                        end[i] = ob[c + 1];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) column0[i] = pib[min(first[i], (uint32_t)cols - 1u)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (c0 + i * NT >= P) continue;
                        const uint32_t s = first[i], e = min(end[i], (uint32_t)cols);
                        if (end[i] < s || end[i] > (uint32_t)cols) bad = true;
                        if (s >= e) continue;
                        if (c0 + i * NT >= code_end) bad = true;
                        const uint32_t bits = row_bits<BITS>((uint32_t)(c0 + i * NT), base, ps, lo, hi, at);
                        if (e - s >= kLongColumns) {
                            const uint32_t pieces = (e - s + kPieceColumns - 1) / kPieceColumns;
                            const uint32_t n = atomicAdd(&longs[0], pieces);
                            for (uint32_t q = 0; q < pieces; ++q) {
                                // (there is room, unless the boundaries are damaged)
                                if (n + q >= (uint32_t)long_pieces(cols)) break;
                                uint32_t *l = longs + 1 + 3 * (n + q);
                                l[0] = s + q * kPieceColumns;
                                l[1] = min((q + 1) * kPieceColumns, e - s) - q * kPieceColumns;
                                l[2] = bits;
                            }
                            continue;
                        }
                        put(column0[i], bits);
                        for (uint32_t t = s + 1; t < e; t += 4) {
                            int col[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q) col[q] = pib[min(t + q, e - 1)];
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (t + q < e) put(col[q], bits);
                        }
                    }
                }
                __syncthreads();
                const uint32_t n = min(longs[0], (uint32_t)long_pieces(cols));
                for (uint32_t i = tid >> 6; i < n; i += NT >> 6) {  // a wave per piece
                    const uint32_t *l = longs + 1 + 3 * i;
                    for (uint32_t t = tid & 63; t < l[1]; t += 64) put(pib[l[0] + t], l[2]);
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < ntiles * 64; i += NT) {
            const int lane = i & 63, j0 = (i >> 6) * kTileCols + 8 * (lane >> 4);
            uint32_t word[2 * BITS];
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) word[d] = 0;
#pragma unroll
            for (int st = 0; st < kTileSteps; ++st)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int j = j0 + 32 * st + e;
                    const uint32_t x = j < cols ? column[j] : 0u;
                    put_code<BITS>(word, st, e, (x >> (BITS * (lane & 15))) & (BITS == 2 ? 3u : 1u));
                }
            uint32_t *to = tiled + (G * ntiles * 64 + i) * (2 * BITS);
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) to[d] = word[d];
        }
        __syncthreads();
    }
    if (bad) atomicOr(err_flag, 4);
}

// ---- decoding --------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t two_bf16(uint32_t nibbles, int byte) {
    // scale 0.5: the nibbles are 0, 2.0 and -2.0
    switch (byte) {
        case 0: return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(nibbles, 0.5f, 0));
        case 1: return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(nibbles, 0.5f, 1));
        case 2: return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(nibbles, 0.5f, 2));
        default: return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(nibbles, 0.5f, 3));
    }
}

// The eight entries of a lane for 32-column step st of a tile.
template <int BITS>
__device__ __forceinline__ bf16x8 decode(const uint32_t (&w)[2 * BITS], int st) {
    u32x4 a;
    if (BITS == 2) {
        const uint32_t d = w[st >> 1];
        const uint32_t hi = d & 0xccccccccu, lo = (d << 2) & 0xccccccccu;
        const int b = st & 1 ? 0 : 1;
        a.x = two_bf16(hi, b);
        a.y = two_bf16(hi, b + 2);
        a.z = two_bf16(lo, b);
        a.w = two_bf16(lo, b + 2);
    } else {
        const uint32_t d = w[st >> 2];
        const int j = st & 3;
        const uint32_t t = (j == 0 ? d : j == 1 ? d << 1 : j == 2 ? d << 2 : d >> 1) & 0x44444444u;
        a.x = two_bf16(t, 0);
        a.y = two_bf16(t, 1);
        a.z = two_bf16(t, 2);
        a.w = two_bf16(t, 3);
    }
    return __builtin_bit_cast(bf16x8, a);
}

template <int BITS>
__device__ __forceinline__ void load_codes(const uint32_t *__restrict__ p, uint32_t (&w)[2 * BITS]) {
    if (BITS == 2) {
        const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        w[0] = x.x; w[1] = x.y; w[2 * BITS - 2] = x.z; w[2 * BITS - 1] = x.w;
    } else {
        const u32x2 x = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p));
        w[0] = x.x; w[1] = x.y;
    }
}

// Two row groups for the 32-row MFMA: afterwards `a` holds, lane rows 0..3, slice 0 of group a,
// slice 0 of group b, slice 2 of a, slice 2 of b, and `b` the slices 1 and 3: with the MFMA's
// lane = 32 * (half of the columns) + row, `a` is one 16-column operand and `b` the next.
template <int N>
__device__ __forceinline__ void pair_groups(uint32_t (&a)[N], uint32_t (&b)[N]) {
#pragma unroll
    for (int d = 0; d < N; ++d) {
        const auto r = __builtin_amdgcn_permlane16_swap(a[d], b[d], false, false);
        a[d] = r[0];
        b[d] = r[1];
    }
}

// ---- vectors ---------------------------------------------------------------------------------
// Eight consecutive elements of a vector, as loaded (col past the end: zeros).
template <typename VT>
struct Piece {
    u32x4 q[sizeof(VT) / 2];
};

// The piece of `row` at column `col`, which lies wholly before or wholly behind `end`.
template <typename VT>
__device__ __forceinline__ Piece<VT> load_piece(const VT *__restrict__ row, int col, int end) {
    Piece<VT> p = {};
    if (col + 8 <= end) {
#pragma unroll
        for (int i = 0; i < (int)sizeof(VT) / 2; ++i)
            p.q[i] = *reinterpret_cast<const u32x4_any *>(reinterpret_cast<const unsigned char *>(row + col) + 16 * i);
    }
    return p;
}

// Element by element what load_piece leaves out: a piece that straddles `end`.
template <typename VT>
__device__ __forceinline__ void finish_piece(Piece<VT> &p, const VT *__restrict__ row, int col, int end) {
    if (col >= end || col + 8 <= end) return;
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        e[i] = 0;
        if (col + i < end)
            e[i] = sizeof(VT) == 4 ? reinterpret_cast<const uint32_t *>(row)[col + i]
                                   : reinterpret_cast<const uint16_t *>(row)[col + i];
    }
    if (sizeof(VT) == 4) {
        p.q[0] = u32x4{e[0], e[1], e[2], e[3]};
        p.q[sizeof(VT) / 2 - 1] = u32x4{e[4], e[5], e[6], e[7]};
    } else {
        p.q[0] = u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
    }
}

// One staging step's pieces, row[j] at column col0 + piece_col.  (The branch on a whole step
// costs nothing where a mask per load made large batches 3 % slower.)
template <typename VT, int N>
__device__ __forceinline__ void load_pieces(Piece<VT> (&p)[N], const VT *const (&row)[N], int col0, int cols,
                                            int piece_col, int end) {
    if (col0 + cols <= end) {
#pragma unroll
        for (int j = 0; j < N; ++j) p[j] = load_piece<VT>(row[j], piece_col + col0, 0x7fffffff);
        return;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) p[j] = load_piece<VT>(row[j], col0 + piece_col, end);
    if (end & 7) {
#pragma unroll
        for (int j = 0; j < N; ++j) finish_piece<VT>(p[j], row[j], col0 + piece_col, end);
    }
}

// low halves of (a, b): a in the low half of the result; and the high halves
__device__ __forceinline__ uint32_t low_halves(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t high_halves(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// Writes the piece to LDS, in the order 4 0 5 1 6 2 7 3 of its elements: one plane for bf16,
// three (`plane` bytes apart) for float32.
__device__ __forceinline__ void store_piece(unsigned char *at, int plane, const Piece<uint16_t> &p) {
    (void)plane;
    const u32x4 q = p.q[0];
    *reinterpret_cast<u32x4 *>(at) = u32x4{low_halves(q.z, q.x), high_halves(q.z, q.x), low_halves(q.w, q.y),
                                           high_halves(q.w, q.y)};
}
__device__ __forceinline__ void store_piece(unsigned char *at, int plane, const Piece<float> &p) {
    uint32_t x[8] = {p.q[0].x, p.q[0].y, p.q[0].z, p.q[0].w, p.q[1].x, p.q[1].y, p.q[1].z, p.q[1].w};
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
        // x = top + rest exactly: each plane keeps 8 of the 24 significant bits
        *reinterpret_cast<u32x4 *>(at + pl * plane) = u32x4{high_halves(x[4], x[0]), high_halves(x[5], x[1]),
                                                            high_halves(x[6], x[2]), high_halves(x[7], x[3])};
        if (pl < 2) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[i] = __float_as_uint(__uint_as_float(x[i]) - __uint_as_float(x[i] & 0xffff0000u));
        }
    }
}

__device__ __forceinline__ bf16x8 lds_operand(const unsigned char *at) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(at));
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 v, bf16x8 w, f32x16 acc) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, w, acc, 0, 0, 0);
}

// Vector (row of the MFMA result) of accumulator register i in lane half h.
__device__ __forceinline__ int acc_vector(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// ---- infinities and NaN ------------------------------------------------------------------------
// 0 x inf is NaN, so one infinite or NaN element of v makes all rows of its vector NaN on the matrix
// cores, and the float32 planes of an infinity (inf, then inf - inf) do the same to the rows that it is in.
// The block patterns leave columns without a row out, and so do the products here (`skip_zeros`: the
// kinds that have block patterns; the dense kind multiplies every entry): a result that is not
// finite is summed again over the entries that are not zero.  A finite one says that all its elements
// were, so nothing is looked at before.
__device__ __forceinline__ bool finite(float x) { return __builtin_fabsf(x) <= 3.402823466e38f; }
__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }

// (Functions of their own, called where nothing else is left to do: inlined, they changed the order of
// the instructions of the kernels around them, 2 % for 1 to 16 vectors and 15 % for bf16 tiles.)
// row: of the codes; n: vector.
template <typename VT, int BITS>
__device__ __forceinline__ float nonzeros(const uint32_t *codes, int ntiles, const VT *v, long long ldv, long long row,
                                          int n) {
    const uint32_t *group = codes + (row / kDenseRows) * ntiles * 128 * BITS;
    const int r = (int)(row % kDenseRows);
    const VT *x = v + n * ldv;
    float sum = 0.0f;
#pragma unroll 1
    for (int i = 0; i < ntiles * 4 * kTileSteps; ++i) {  // (tile, step, slice)
        const int t = i >> 5, st = (i >> 2) & 7, slice = i & 3;
        const uint32_t *lane = group + ((long long)t * 64 + 16 * slice + r) * (2 * BITS);
        const uint32_t word = lane[BITS == 2 ? st >> 1 : st >> 2];
        const VT *at = x + t * kTileCols + 32 * st + 8 * slice;
#pragma unroll 1
        for (int e = 0; e < 8; ++e) {
            int shift;
            if (BITS == 2) {
                shift = (e & 1 ? 30 : 14) - 2 * (4 * (st & 1) + (e >> 1));
            } else {
                const int j = st & 3;
                shift = 4 * (e < 4 ? 2 * e + 1 : 2 * (e - 4)) + (j == 3 ? 3 : 2 - j);
            }
            const uint32_t code = (word >> shift) & (BITS == 2 ? 3u : 1u);
            if (code) sum += code & 2u ? -widen(at[e]) : widen(at[e]);  // (columns past the end have code 0)
        }
    }
    return sum;
}

template <typename VT, int BITS>
__device__ __attribute__((noinline)) float sum_of_nonzeros(const uint32_t *codes, int ntiles, const VT *v,
                                                           long long ldv, long long row, int n) {
    return nonzeros<VT, BITS>(codes, ntiles, v, ldv, row, n);
}

// A wave's results of `vectors` x `rows`, which it has stored: out is the first, of row `row` of the codes and
// of the vector at v.
template <typename VT, int BITS>
__device__ __attribute__((noinline)) void sum_again(const uint32_t *codes, int ntiles, const VT *v, long long ldv,
                                                    long long row, float *out, long long ldo, int rows, int vectors,
                                                    float scale) {
    __threadfence();
    for (int n = 0; n < vectors; ++n)
        for (int i = threadIdx.x & 63; i < rows; i += 64) {
            float *at = out + n * ldo + i;
            if (!finite(*at)) *at = scale * nonzeros<VT, BITS>(codes, ntiles, v, ldv, row + i, n);
        }
}

// ---- few: up to four vectors -----------------------------------------------------------------
// A wave takes 16 rows and a share of the columns; `wk` waves of a workgroup share the columns of
// a row group and add their partial results at the end, the only place where waves wait for each
// other.  Every wave stages its own columns of v in LDS of its own, so a wave starts on its codes
// as soon as they and its part of v are there.  The vectors are the rows of the MFMA: vector q
// sits in rows 4q.. (float32: its three planes in rows 4q, 4q+1, 4q+2), so that lane 16 q + r of
// the result holds everything about (vector q, row r), and one MFMA serves all planes.
constexpr int few_waves(int wk) { return wk < 4 ? 4 : wk; }

// Tiles of columns that a wave stages at a time.
template <typename VT, int NV>
constexpr int few_tiles = NV == 1 ? 4 : sizeof(VT) == 4 ? 1 : 2;
template <typename VT, int NV, int TILES = few_tiles<VT, NV>>
struct Few {
    static constexpr int planes = sizeof(VT) == 4 ? 3 : 1;
    static constexpr int tiles = TILES;
    static constexpr int cols = tiles * kTileCols;
    static constexpr int pieces = cols / 8;
    static constexpr int loads = NV * pieces / 64;
    static constexpr int stride = cols * 2 + 16;  // bytes between slots: an odd number of 16-byte units
    static constexpr int wave_bytes = NV * planes * stride;
};

template <typename VT, int BITS, int NV, int WK>
__global__ __launch_bounds__(few_waves(WK) * 64) void k_packed_few(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ntiles, int ngroups, int n_in, int n_out,
    long long ldv, int nv, float scale, float *__restrict__ out, long long ldo, int skip_zeros,
    const LayerTable layers) {
    using S = Few<VT, NV>;
    constexpr int WR = few_waves(WK) / WK;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wr = w / WK, wk = w % WK;
    const int g = min((int)blockIdx.x * WR + wr, ngroups - 1);
    const int t0 = ntiles * wk / WK, t1 = ntiles * (wk + 1) / WK;
    const int end = min(n_in, t1 * kTileCols);
    const uint32_t *c0 = codes + ((long long)g * ntiles * 64 + lane) * (2 * BITS);
    unsigned char *mine = smem + w * S::wave_bytes;

    Piece<VT> p[S::loads];
    auto request_v = [&](int t) {
        const int col0 = t * kTileCols;
#pragma unroll
        for (int j = 0; j < S::loads; ++j) {
            const int i = j * 64 + lane, n = NV == 1 ? 0 : min(i / S::pieces, nv - 1);
            p[j] = load_piece<VT>(v + n * ldv, col0 + 8 * (i % S::pieces), end);
        }
        if ((end & 7) && end <= col0 + S::cols) {
#pragma unroll
            for (int j = 0; j < S::loads; ++j) {
                const int i = j * 64 + lane, n = NV == 1 ? 0 : min(i / S::pieces, nv - 1);
                finish_piece<VT>(p[j], v + n * ldv, col0 + 8 * (i % S::pieces), end);
            }
        }
    };
    uint32_t c[S::tiles][2 * BITS];
    auto request_codes = [&](int t) {
#pragma unroll
        for (int i = 0; i < S::tiles; ++i)
            if (t + i < t1) load_codes<BITS>(c0 + (long long)(t + i) * 128 * BITS, c[i]);
    };
    // the MFMA row of this lane: vector m/4, float32 plane m%4
    const int m = lane & 15;
    const int slot = (NV == 1 ? 0 : m >> 2) * S::planes + (S::planes == 3 ? min(m & 3, 2) : 0);
    const unsigned char *operand = mine + slot * S::stride + (lane >> 4) * 16;
    f32x4 acc0 = {}, acc1 = {};
    if (t0 < t1) {
        request_v(t0);
        request_codes(t0);
    }
    for (int t = t0; t < t1; t += S::tiles) {
#pragma unroll
        for (int j = 0; j < S::loads; ++j) {
            const int i = j * 64 + lane;
            store_piece(mine + (i / S::pieces) * S::planes * S::stride + 16 * (i % S::pieces), S::stride, p[j]);
        }
        if (t + S::tiles < t1) request_v(t + S::tiles);
        // the wave's LDS operations execute in order: no barrier inside a wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < S::tiles; ++i) {
            if (t + i >= t1) break;
#pragma unroll
            for (int st = 0; st < kTileSteps; st += 2) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_operand(operand + i * 512 + st * 64),
                                                               decode<BITS>(c[i], st), acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_operand(operand + i * 512 + st * 64 + 64),
                                                               decode<BITS>(c[i], st + 1), acc1, 0, 0, 0);
            }
        }
        if (t + S::tiles < t1) request_codes(t + S::tiles);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    float sum = acc0.x + acc1.x;
    if (S::planes == 3) sum += (acc0.y + acc1.y) + (acc0.z + acc1.z);
    int group = (int)blockIdx.x * WR + wr;
    if (WK > 1) {
        float *red = reinterpret_cast<float *>(smem + few_waves(WK) * S::wave_bytes);
        red[w * 64 + lane] = sum;
        __syncthreads();
        if (tid >= WR * 64) return;
        sum = 0.0f;
#pragma unroll
        for (int i = 0; i < WK; ++i) sum += red[(w * WK + i) * 64 + lane];
        group = (int)blockIdx.x * WR + w;
    }
    const int q = lane >> 4;
    const long long row = (long long)group * kDenseRows + m;
    auto store = [&](float x) {
        if (layers.n == 0) {
            if (q < nv && row < n_out) out[q * ldo + row] = scale * x;
        } else if (q == 0 && group < ngroups) {
            // stacked handle: the group belongs to one layer (layers start on group boundaries)
            int s = 0;
#pragma unroll
            for (int i = 1; i < kMaxLayers; ++i)
                if (i < layers.n && group >= layers.first[i]) s = i;
            const int local = (group - layers.first[s]) * kDenseRows + m;
            if (local < layers.rows[s]) layers.out[s][local] = layers.scale[s] * x;
        }
    };
    store(sum);
    if (__builtin_expect(!finite(sum), 0)) {
        if (skip_zeros && q < nv && group < ngroups)
            store(sum_of_nonzeros<VT, BITS>(codes, ntiles, v, ldv, row, q));
    }
}

// Two or four row groups (G) per wave, on tall matrices: v is staged, and read as an operand, once for all of them; or one
// row group with more tiles staged at a time.  A kernel of its own, not the same template with k_packed_few: written as
// loops over G = 1, that one took 3 % longer with the same registers where a wave has all of a row (binary, one bf16 vector,
// 100000 x 256 3.61 -> 3.72 us, 139000 x 256 4.08 -> 4.20).
template <typename VT, int BITS, int NV, int WK, int G, int TILES>
__global__ __launch_bounds__(few_waves(WK) * 64) void k_packed_tall(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ntiles, int ngroups, int n_in, int n_out,
    long long ldv, int nv, float scale, float *__restrict__ out, long long ldo, int skip_zeros,
    const LayerTable layers) {
    using S = Few<VT, NV, TILES>;
    constexpr int W = few_waves(WK), WR = W / WK;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wr = w / WK, wk = w % WK;
    const int t0 = ntiles * wk / WK, t1 = ntiles * (wk + 1) / WK;
    const int end = min(n_in, t1 * kTileCols);
    const uint32_t *c0[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
        c0[g] = codes + ((long long)min(((int)blockIdx.x * WR + wr) * G + g, ngroups - 1) * ntiles * 64 + lane) * (2 * BITS);
    unsigned char *mine = smem + w * S::wave_bytes;

    Piece<VT> p[S::loads];
    auto request_v = [&](int t) {
        const int col0 = t * kTileCols;
#pragma unroll
        for (int j = 0; j < S::loads; ++j) {
            const int i = j * 64 + lane, n = NV == 1 ? 0 : min(i / S::pieces, nv - 1);
            p[j] = load_piece<VT>(v + n * ldv, col0 + 8 * (i % S::pieces), end);
        }
        if ((end & 7) && end <= col0 + S::cols) {
#pragma unroll
            for (int j = 0; j < S::loads; ++j) {
                const int i = j * 64 + lane, n = NV == 1 ? 0 : min(i / S::pieces, nv - 1);
                finish_piece<VT>(p[j], v + n * ldv, col0 + 8 * (i % S::pieces), end);
            }
        }
    };
    uint32_t c[G][S::tiles][2 * BITS];
    auto request_codes = [&](int t) {
#pragma unroll
        for (int i = 0; i < S::tiles; ++i)
            if (t + i < t1) {
#pragma unroll
                for (int g = 0; g < G; ++g) load_codes<BITS>(c0[g] + (long long)(t + i) * 128 * BITS, c[g][i]);
            }
    };
    // the MFMA row of this lane: vector m/4, float32 plane m%4
    const int m = lane & 15;
    const int slot = (NV == 1 ? 0 : m >> 2) * S::planes + (S::planes == 3 ? min(m & 3, 2) : 0);
    const unsigned char *operand = mine + slot * S::stride + (lane >> 4) * 16;
    f32x4 acc0[G] = {}, acc1[G] = {};
    if (t0 < t1) {
        request_v(t0);
        request_codes(t0);
    }
    for (int t = t0; t < t1; t += S::tiles) {
#pragma unroll
        for (int j = 0; j < S::loads; ++j) {
            const int i = j * 64 + lane;
            store_piece(mine + (i / S::pieces) * S::planes * S::stride + 16 * (i % S::pieces), S::stride, p[j]);
        }
        if (t + S::tiles < t1) request_v(t + S::tiles);
        // the wave's LDS operations execute in order: no barrier inside a wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < S::tiles; ++i) {
            if (t + i >= t1) break;
#pragma unroll
            for (int st = 0; st < kTileSteps; st += 2) {
                const bf16x8 x0 = lds_operand(operand + i * 512 + st * 64);
#pragma unroll
                for (int g = 0; g < G; ++g)
                    acc0[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, decode<BITS>(c[g][i], st), acc0[g], 0, 0, 0);
                const bf16x8 x1 = lds_operand(operand + i * 512 + st * 64 + 64);
#pragma unroll
                for (int g = 0; g < G; ++g)
                    acc1[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, decode<BITS>(c[g][i], st + 1), acc1[g], 0, 0, 0);
            }
        }
        if (t + S::tiles < t1) request_codes(t + S::tiles);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    const int q = lane >> 4;
    auto put = [&](int group, float sum) {
        const long long row = (long long)group * kDenseRows + m;
        auto store = [&](float x) {
            if (layers.n == 0) {
                if (q < nv && row < n_out) out[q * ldo + row] = scale * x;
            } else if (q == 0 && group < ngroups) {
                // stacked handle: the group belongs to one layer (layers start on group boundaries)
                int s = 0;
#pragma unroll
                for (int i = 1; i < kMaxLayers; ++i)
                    if (i < layers.n && group >= layers.first[i]) s = i;
                const int local = (group - layers.first[s]) * kDenseRows + m;
                if (local < layers.rows[s]) layers.out[s][local] = layers.scale[s] * x;
            }
        };
        store(sum);
        if (__builtin_expect(!finite(sum), 0)) {
            if (skip_zeros && q < nv && group < ngroups)
                store(sum_of_nonzeros<VT, BITS>(codes, ntiles, v, ldv, row, q));
        }
    };
    float sum[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        sum[g] = acc0[g].x + acc1[g].x;
        if (S::planes == 3) sum[g] += (acc0[g].y + acc1[g].y) + (acc0[g].z + acc1[g].z);
    }
    const int group0 = (int)blockIdx.x * WR * G;
    float *red = reinterpret_cast<float *>(smem + W * S::wave_bytes);  // [group][wave][lane]
#pragma unroll
    for (int g = 0; g < G; ++g) red[(g * W + w) * 64 + lane] = sum[g];
    __syncthreads();
    static_assert(WK > 1 && WR * G <= W, "a wave per row group of the workgroup");
    if (w >= WR * G) return;
    const float *part = red + ((w % G) * W + w / G * WK) * 64 + lane;
    float x = 0.0f;
#pragma unroll
    for (int k = 0; k < WK; ++k) x += part[k * 64];
    put(group0 + w, x);
}

// ---- split: 16 to 64 rows x 16 or 32 vectors, the columns dealt to the waves -------------------
// For batches too small to fill the chip with tiles of 128 x 128.  2^wk_log2 of the eight waves of a
// workgroup share the columns of 16 G rows (ROWS: fewer than all eight).  Every wave works through its own share of the tiles and
// stages its own columns of the 16 NT vectors in LDS of its own: nothing in the loop waits for
// another wave, the partial results are added at the end.
template <typename VT, int NT>
struct Split {
    static constexpr int planes = sizeof(VT) == 4 ? 3 : 1;
    static constexpr int vectors = 16 * NT;
    static constexpr int cols = sizeof(VT) == 4 ? 64 : 128;  // columns staged at a time
    static constexpr int pieces = cols / 8;
    static constexpr int loads = vectors * pieces / 64;
    static constexpr int stride = cols * 2 + 16;  // bytes between vectors: an odd number of 16-byte units
    static constexpr int plane = vectors * stride;
    static constexpr int wave_bytes = planes * plane;
    static constexpr int stages = kTileCols / cols;
};
constexpr int kSplitWaves = 8;

template <typename VT, int BITS, int NT, int G, bool ROWS>
__global__ __launch_bounds__(kSplitWaves * 64) void k_packed_split(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ntiles, int ngroups, int n_in, int n_out,
    long long ldv, int batch, float *__restrict__ out, long long ldo, float scale, int wk_log2_rows, int skip_zeros) {
    using S = Split<VT, NT>;
    const int wk_log2 = ROWS ? wk_log2_rows : 3;  // (shifts that are known: 0.3 us less for the smallest products)
    constexpr bool kPairs = NT == 2;              // 32 x 32 MFMAs over two row groups
    constexpr int kAcc = G * NT * 4;              // result registers of a lane
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wr = w >> wk_log2, kpart = w - (wr << wk_log2);
    const int vec0 = blockIdx.y * S::vectors;
    const int row_sets = kSplitWaves >> wk_log2;  // of 16 G rows
    const int group0 = ((int)blockIdx.x * row_sets + wr) * G;
    const int t0 = ntiles * kpart >> wk_log2, t1 = ntiles * (kpart + 1) >> wk_log2;
    unsigned char *mine = smem + w * S::wave_bytes;

    const VT *row[S::loads];
    int at[S::loads];
#pragma unroll
    for (int j = 0; j < S::loads; ++j) {
        const int n = (j * 64 + lane) / S::pieces;
        row[j] = v + (long long)min(vec0 + n, batch - 1) * ldv;
        at[j] = n * S::stride;
    }
    const int piece_col = 8 * (lane % S::pieces);
    const uint32_t *code[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
        code[g] = codes + ((long long)min(group0 + g, ngroups - 1) * ntiles * 64 + lane) * (2 * BITS);

    Piece<VT> p[S::loads];
    auto request = [&](int col0) { load_pieces<VT>(p, row, col0, S::cols, piece_col, n_in); };
    constexpr int kSums = S::planes == 3 ? 2 : 1;  // the top plane, and the others
    f32x4 acc[kSums][kPairs ? 1 : G] = {};
    f32x16 pair_acc[kSums][kPairs ? G / 2 : 1] = {};
    uint32_t c[G][2 * BITS];
    if (t0 < t1) {
#pragma unroll
        for (int g = 0; g < G; ++g) load_codes<BITS>(code[g] + (long long)t0 * 128 * BITS, c[g]);
        request(t0 * kTileCols);
    }
    for (int t = t0; t < t1; ++t) {
        uint32_t cn[G][2 * BITS];
        const long long next = (long long)min(t + 1, t1 - 1) * 128 * BITS;
#pragma unroll
        for (int g = 0; g < G; ++g) load_codes<BITS>(code[g] + next, cn[g]);
        if constexpr (kPairs) {
#pragma unroll
            for (int g = 0; g < G; g += 2) pair_groups(c[g], c[g + 1]);
        }
#pragma unroll
        for (int s = 0; s < S::stages; ++s) {
#pragma unroll
            for (int j = 0; j < S::loads; ++j) store_piece(mine + at[j] + piece_col * 2, S::plane, p[j]);
            const int ahead = t * kTileCols + (s + 1) * S::cols;
            if (ahead < t1 * kTileCols) request(ahead);
            // the wave's LDS operations execute in order: no barrier inside a wave
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < S::cols / 32; ++k) {
                const int st = s * (S::cols / 32) + k;
                if constexpr (kPairs) {
                    const unsigned char *x = mine + (lane & 31) * S::stride + (4 * k + 2 * half) * 16;
#pragma unroll
                    for (int xy = 0; xy < 2; ++xy) {
                        bf16x8 o[S::planes];
#pragma unroll
                        for (int pl = 0; pl < S::planes; ++pl) o[pl] = lds_operand(x + pl * S::plane + 16 * xy);
#pragma unroll
                        for (int g = 0; g < G; g += 2) {
                            const bf16x8 y = decode<BITS>(c[g + xy], st);
#pragma unroll
                            for (int pl = 0; pl < S::planes; ++pl) {
                                f32x16 &to = pair_acc[pl ? kSums - 1 : 0][g / 2];
                                to = mfma32(o[pl], y, to);
                            }
                        }
                    }
                } else {
                    const unsigned char *x = mine + (lane & 15) * S::stride + (4 * k + (lane >> 4)) * 16;
                    bf16x8 o[S::planes];
#pragma unroll
                    for (int pl = 0; pl < S::planes; ++pl) o[pl] = lds_operand(x + pl * S::plane);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const bf16x8 y = decode<BITS>(c[g], st);
#pragma unroll
                        for (int pl = 0; pl < S::planes; ++pl) {
                            f32x4 &to = acc[pl ? kSums - 1 : 0][g];
                            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o[pl], y, to, 0, 0, 0);
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) c[g][d] = cn[g][d];
    }
    __syncthreads();  // the staging areas become the partial results [wave][register][lane]
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < kAcc; ++i) {
        float sum = kPairs ? pair_acc[0][i >> 4][i & 15] : acc[0][i >> 2][i & 3];
        if (kSums == 2) sum += kPairs ? pair_acc[1][i >> 4][i & 15] : acc[1][i >> 2][i & 3];
        red[(w * kAcc + i) * 64 + lane] = sum;
    }
    __syncthreads();
    for (int e = tid; e < row_sets * kAcc * 64; e += kSplitWaves * 64) {
        const int i = (e >> 6) % kAcc, r = (e >> 6) / kAcc;
        const float *part = red + ((r << wk_log2) * kAcc + i) * 64 + lane;
        float sum = 0.0f;
        if (!ROWS) {
#pragma unroll
            for (int k = 0; k < kSplitWaves; ++k) sum += part[k * kAcc * 64];
        } else {
            for (int k = 0; k < 1 << wk_log2; ++k) sum += part[k * kAcc * 64];
        }
        const long long first = (long long)(((int)blockIdx.x * row_sets + r) * G) * kDenseRows;
        const long long rr = first + (kPairs ? 32 * (i >> 4) + (lane & 31) : 16 * (i >> 2) + (lane & 15));
        const int n = vec0 + (kPairs ? acc_vector(i & 15, half) : 4 * (lane >> 4) + (i & 3));
        if (n < batch && rr < n_out) {
            out[(long long)n * ldo + rr] = scale * sum;
            if (__builtin_expect(!finite(sum), 0)) {
                if (skip_zeros)
                    out[(long long)n * ldo + rr] = scale * sum_of_nonzeros<VT, BITS>(codes, ntiles, v, ldv, rr, n);
            }
        }
    }
}

// ---- tile: 128 rows x 128 vectors, four or eight waves ------------------------------------------
// A wave owns RB x VB blocks of 32 rows x 32 vectors: 64 x 64 or 32 x 128.  KW = 2: two sets of four
// waves, one multiplies the even 16-column operands and one the odd ones; they add up at the end.
// The vectors are staged in LDS, double buffered, one barrier per stage, float32 two (four with
// eight waves) stages ahead, as far as the registers reach; bf16, with a quarter of the load
// instructions per MFMA, gains nothing from more than one; the codes come straight from memory, every wave those of its
// own rows.
template <typename VT>
struct Tile {
    static constexpr int planes = sizeof(VT) == 4 ? 3 : 1;
    static constexpr int cols = sizeof(VT) == 4 ? 32 : 64;
    static constexpr int pieces = cols / 8;
    static constexpr int stride = cols * 2 + 16;
    static constexpr int plane = 128 * stride;
    static constexpr int buffer = planes * plane;
    static constexpr int stages = kTileCols / cols;
    static constexpr int ahead = sizeof(VT) == 4 ? 2 : 1;  // stages of v in registers, on their way (KW = 1)
};

template <typename VT, int BITS, int KW, int RB>
__global__ __launch_bounds__(256 * KW, 2) void k_packed_tile(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ntiles, int ngroups, int n_in, int n_out,
    long long ldv, int batch, float *__restrict__ out, long long ldo, float scale, int row_tiles, int vec_tiles,
    int skip_zeros) {
    using S = Tile<VT>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kw = w >> 2;
    constexpr int NT = 256 * KW;
    constexpr int VB = 4 / RB, RW = 4 / RB;       // blocks of 32 vectors of a wave; waves beside each other in rows
    const int wr = w & (RW - 1), wn = (w & 3) / RW;
    // consecutive workgroups go to the eight XCDs in turn: each XCD gets a contiguous run of
    // tiles, eight row tiles for every vector tile, so that its L2 sees the same vectors again
    const int all = row_tiles * vec_tiles, per = (all + 7) / 8;
    const int lin = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || lin >= all) return;
    const int band = lin / (8 * vec_tiles), in_band = lin - band * 8 * vec_tiles;
    const int band_rows = min(8, row_tiles - band * 8);
    const int rt = band * 8 + in_band % band_rows, vt = in_band / band_rows;
    const int vec0 = vt * 128;
    constexpr int kLoads = 128 * S::pieces / NT;

    const VT *row[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j)
        row[j] = v + (long long)min(vec0 + (j * NT + tid) / S::pieces, batch - 1) * ldv;
    const int piece_col = 8 * (tid % S::pieces);
    unsigned char *put = smem + (tid / S::pieces) * S::stride + piece_col * 2;
    const uint32_t *code[2 * RB];
#pragma unroll
    for (int g = 0; g < 2 * RB; ++g)
        code[g] = codes + ((long long)min(rt * 8 + wr * 2 * RB + g, ngroups - 1) * ntiles * 64 + lane) * (2 * BITS);

    constexpr int kAhead = S::planes == 3 ? S::ahead * KW : S::ahead;
    static_assert(S::stages % kAhead == 0, "a stage's registers are known when the code is compiled");
    Piece<VT> p[kAhead][kLoads];  // stage s of a tile in p[s % ahead]
    auto request = [&](int slot, int col0) { load_pieces<VT>(p[slot], row, col0, S::cols, piece_col, n_in); };
    auto stage = [&](int buf, int slot) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
            store_piece(put + buf * S::buffer + j * (NT / S::pieces) * S::stride, S::plane, p[slot][j]);
    };
    constexpr int kSums = S::planes == 3 ? 2 : 1;  // the top plane, and the others
    f32x16 sums[kSums][RB][VB] = {};
    auto &acc = sums[0];
    uint32_t c[2 * RB][2 * BITS];
#pragma unroll
    for (int g = 0; g < 2 * RB; ++g) load_codes<BITS>(code[g], c[g]);
#pragma unroll
    for (int s = 0; s < kAhead; ++s) request(s, s * S::cols);
    stage(0, 0);
    const int end = ntiles * kTileCols;
    if (kAhead * S::cols < end) request(0, kAhead * S::cols);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
        uint32_t cn[2 * RB][2 * BITS];
        const long long next = (long long)min(t + 1, ntiles - 1) * 128 * BITS;
#pragma unroll
        for (int g = 0; g < 2 * RB; ++g) load_codes<BITS>(code[g] + next, cn[g]);
#pragma unroll
        for (int r = 0; r < RB; ++r) pair_groups(c[2 * r], c[2 * r + 1]);
        if (KW == 2 && kw == 1) {  // this wave multiplies the odd 16-column operands
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d)
#pragma unroll
                for (int r = 0; r < RB; ++r) c[2 * r][d] = c[2 * r + 1][d];
        }
#pragma unroll
        for (int s = 0; s < S::stages; ++s) {
            const unsigned char *buf = smem + (s & 1) * S::buffer + (wn * 32 * VB + (lane & 31)) * S::stride + 32 * half;
#pragma unroll
            for (int k = 0; k < S::cols / 32; ++k) {
                const int st = s * (S::cols / 32) + k;
#pragma unroll
                for (int half_step = 0; half_step < 2 / KW; ++half_step) {
                    const int xy = KW == 2 ? kw : half_step;
                    bf16x8 x[RB];
#pragma unroll
                    for (int r = 0; r < RB; ++r) x[r] = decode<BITS>(c[2 * r + (KW == 2 ? 0 : xy)], st);
#pragma unroll
                    for (int pl = 0; pl < S::planes; ++pl)
#pragma unroll
                        for (int n = 0; n < VB; ++n) {
                            const bf16x8 o = lds_operand(buf + pl * S::plane + 64 * k + 16 * xy + n * 32 * S::stride);
#pragma unroll
                            for (int r = 0; r < RB; ++r) {
                                f32x16 &to = sums[pl ? kSums - 1 : 0][r][n];
                                to = mfma32(o, x[r], to);
                            }
                        }
                }
            }
            // the next stage goes to the other buffer, which nobody reads any more
            stage((s + 1) & 1, (s + 1) % kAhead);
            const int ahead = t * kTileCols + (s + 1 + kAhead) * S::cols;
            if (ahead < end) request((s + 1) % kAhead, ahead);
            __syncthreads();
        }
#pragma unroll
        for (int g = 0; g < 2 * RB; ++g)
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) c[g][d] = cn[g][d];
    }
    // The codes requested last are not used.  They are waited for here (vmcnt = 0): if one of their
    // registers comes to hold an address or a result below, every store gets a wait for all that is on its
    // way, the stores before it among them (6912 x 2560 x 512 bf16 vectors: 30.0 instead of 25.3 us).
    __builtin_amdgcn_s_waitcnt(0x0f70);
    if constexpr (kSums == 2) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int n = 0; n < VB; ++n) acc[r][n] += sums[1][r][n];
    }
    if constexpr (KW == 2) {
        // the second four waves hand over their sums, half of them at a time (the last stage's barrier
        // is behind every read of the buffers)
        float *red = reinterpret_cast<float *>(smem) + (w & 3) * 2048 + lane;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            if (kw == 1) {
#pragma unroll
                for (int i = 0; i < 32; ++i) red[i * 64] = acc[(2 * part + i / 16) / VB][(2 * part + i / 16) % VB][i & 15];
            }
            __syncthreads();
            if (kw == 0) {
#pragma unroll
                for (int i = 0; i < 32; ++i) acc[(2 * part + i / 16) / VB][(2 * part + i / 16) % VB][i & 15] += red[i * 64];
            }
            __syncthreads();
        }
        if (kw == 1) return;
    }
    float check = 0.0f;  // NaN if a result is not finite
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) check += 0.0f * acc[r][b][i];
    const bool again = __ballot(check != check) != 0;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int row_out = rt * 128 + (wr * RB + r) * 32 + (lane & 31);
#pragma unroll
        for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int n = vec0 + (wn * VB + b) * 32 + acc_vector(i, half);
                if (n < batch && row_out < n_out) out[(long long)n * ldo + row_out] = scale * acc[r][b][i];
            }
    }
    if (__builtin_expect(again, 0)) {
        const int row0 = rt * 128 + wr * RB * 32, n0 = vec0 + wn * VB * 32;
        if (skip_zeros && row0 < n_out && n0 < batch)
            sum_again<VT, BITS>(codes, ntiles, v + n0 * ldv, ldv, row0, out + n0 * ldo + row0, ldo,
                                min(RB * 32, n_out - row0), min(VB * 32, batch - n0), scale);
    }
}

// ---- tables: up to 256 columns -----------------------------------------------------------------
// One tile of columns: all of a vector fits the registers (or the LDS) of a wave, so it is brought
// into operand order once and the wave then works through many row groups, with nothing but their
// codes to wait for.  1048576 x 256 binary, float32 vectors, before (a wave stages v for every 512
// bytes of codes; tiles of 128 vectors) and now: 1 vector 24.7 -> 14.3 us with bf16 operands, 7.9 with digits (4.2 TB/s; a
// plain read of the codes takes 6.6; with sixteen such tables in turn, whose codes come from HBM, 15.6 and 8.8), 16 vectors
// 171 -> 32, 64 vectors 201 -> 100 (3.0 TB/s, of which the 268 MB of results take two thirds).

// table_few: up to 16 vectors.  The operands of the eight 32-column steps stay in registers; for up
// to four vectors the float32 planes are rows of the MFMA as in k_packed_few, beyond that every
// plane is an MFMA of its own.  One vector: digits, below.
constexpr int kTableWaves = 4;
template <typename VT, int NV>
struct TableFew {
    static constexpr int planes = sizeof(VT) == 4 ? 3 : 1;
    static constexpr int operands = NV == 16 ? planes : 1;
    static constexpr int occupancy = operands == 3 ? 2 : 4;  // waves per SIMD
    static constexpr int stride = kTileCols * 2 + 16;  // bytes between slots: an odd number of 16-byte units
};

// One vector: the 16 rows of the MFMA are free for its digits.  With 2^E <= max |v| < 2^(E+1) an element
// is the sum of d_p 2^(E-3-5p), p = 0..15, d_p whole numbers from -16 to 16.  Those are exact in the 8-bit float
// format, and the nibbles of the codes are 4-bit floats as they are, so v_mfma_scale_f32_16x16x128_f8f6f4
// takes both: per row group 2 MFMAs of 14.6 ns where the bf16 operands took 8 of 7.7, and one AND for eight
// entries where they took an AND and four conversions.  Every row of the result is a sum of whole
// numbers below 2^13 in units of its own plane, which is exact (the instruction cuts off what lies 2^-15
// and more below its largest term: 14 binades in one sum were measured to be wrong by 4e-5 of it), so
// the only roundings are those of the final sum over the planes.  Elements that reach below the last digit (nonzero and
// smaller than 2^(E-55)) go into further sets of digits, each with the exponent 56 below the one before (float32 needs
// five at most): two more MFMAs per row group and set, exact too.  1048576 x 256 binary, float32, with one set 7.9 us, with a
// second one for an element at 2^-70 10.6, with all five 14.9 (14.3 with bf16 operands, 15.1 after digits that turned out not to
// hold the vector); 241000 x 256 two-bit codes, launches not in a graph, 5.7, with a second set 6.6 (6.2, 7.7).
// Not taken, by the whole workgroup, where an element is not finite.
constexpr int kDigits = 16;
constexpr int kDigitStride = kTileCols + 16;  // bytes between planes
constexpr int kDigitExponents = 56;                       // of the elements in one set
constexpr int kDigitSetBytes = kDigits * kDigitStride;
constexpr int kDigitSets = (127 + 149) / kDigitExponents + 1;
constexpr int kTableOneLds = kDigitSets * kDigitSetBytes + 2 * kTableWaves * 4;  // digits; two words per wave
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Where the digit of a column stands among the 256 of its plane, [half][lane quarter][dword][nibble] of the weights'
// operand; `weight`: what an entry of 1 is as a 4-bit float there.
template <int BITS>
__device__ __forceinline__ int digit_place(int col, float *weight) {
    const int st = col >> 5, q = (col >> 3) & 3, e = col & 7;
    if (BITS == 1) {
        const int j = st & 3;
        *weight = j == 1 ? 1.0f : j == 2 ? 0.5f : 2.0f;
        return 128 * (st >> 2) + 32 * q + 8 * j + (e < 4 ? 2 * e + 1 : 2 * (e - 4));
    }
    const int bit = (e & 1 ? 30 : 14) - 2 * (4 * (st & 1) + (e >> 1));
    *weight = 2.0f;
    return 128 * (st >> 2) + 32 * q + 16 * ((st >> 1) & 1) + (bit & 2 ? 0 : 8) + (bit >> 2);
}

// The weights' operand of half h of the columns.
template <int BITS>
__device__ __forceinline__ i32x8 nibbles(const uint32_t (&w)[2 * BITS], int h) {
    i32x4 x;
    if (BITS == 1) {
        x = i32x4{(int)(w[h] & 0x44444444u), (int)(w[h] & 0x22222222u), (int)(w[h] & 0x11111111u),
                  (int)((w[h] >> 1) & 0x44444444u)};
    } else {
        const uint32_t a = w[2 * h * (BITS - 1)], b = w[2 * h * (BITS - 1) + 1];
        x = i32x4{(int)(a & 0xccccccccu), (int)((a << 2) & 0xccccccccu), (int)(b & 0xccccccccu),
                  (int)((b << 2) & 0xccccccccu)};
    }
    return __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1);
}

// The largest of the wave's values, none of them negative, in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max(float x) {
    return __builtin_fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, false)));
}
__device__ __forceinline__ float wave_max(float x) {
    x = dpp_max<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8
    x = dpp_max<0x112, 0xf>(x);
    x = dpp_max<0x114, 0xf>(x);
    x = dpp_max<0x118, 0xf>(x);
    x = dpp_max<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    return dpp_max<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
}

// Writes the digits of v to LDS, a thread per column, and returns the number of sets; 0 (for the whole workgroup) if an
// element is not finite.  *exponent: of the unit of plane 0 of the first set.  `most`: two words per wave.
template <typename VT, int BITS>
__device__ __forceinline__ int table_digits(const VT *__restrict__ v, int n_in, unsigned char *digits, float *most,
                                            int *exponent) {
    const int col = threadIdx.x;
    const float x = col < n_in ? widen(v[col]) : 0.0f;
    float top = wave_max(__builtin_fabsf(x));  // (a NaN is lost by the maximum and found below)
    if ((col & 63) == 63) most[col >> 6] = top;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTableWaves; ++i) top = __builtin_fmaxf(top, most[i]);
    const int E = top > 0.0f ? (int)__builtin_amdgcn_frexp_expf(top) - 1 : 0;
    // (nothing of this means anything beside an element that is not finite, but it stays in range)
    const int below = x != 0.0f ? E - ((int)__builtin_amdgcn_frexp_expf(x) - 1) : 0;
    int set = 0;
    const bool far = __ballot(below >= kDigitExponents) != 0;
    if (__builtin_expect(far, 0)) set = min(max(below, 0) / kDigitExponents, kDigitSets - 1);
    float weight;
    unsigned char *at = digits + digit_place<BITS>(col, &weight);
    const float unit = 1.0f / weight;
    float rest = __builtin_amdgcn_ldexpf(x, 3 - E + set * kDigitExponents);
    unsigned char *mine = at + set * kDigitSetBytes;
#pragma unroll
    for (int p = 0; p < kDigits; p += 2) {
        const float d0 = __builtin_rintf(rest);
        rest = (rest - d0) * 32.0f;
        const float d1 = __builtin_rintf(rest);
        rest = (rest - d1) * 32.0f;
        const int two = __builtin_amdgcn_cvt_pk_fp8_f32(d0 * unit, d1 * unit, 0, false);
        mine[p * kDigitStride] = (unsigned char)two;
        mine[(p + 1) * kDigitStride] = (unsigned char)(two >> 8);
    }
    // the column has no digits in the other sets
    auto none_in = [&](int other) {
        if (other == set) return;
#pragma unroll
        for (int p = 0; p < kDigits; ++p) at[other * kDigitSetBytes + p * kDigitStride] = 0;
    };
    if (__builtin_expect(far, 0)) none_in(0);
    *exponent = E - 3;
    int sets = 1;
    if (__ballot(!finite(x)))
        sets = kDigitSets + 1;
    else
        while (__ballot(set >= sets)) ++sets;
    int *need = reinterpret_cast<int *>(most + kTableWaves);
    if ((col & 63) == 0) need[col >> 6] = sets;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTableWaves; ++i) sets = max(sets, need[i]);
    sets = __builtin_amdgcn_readfirstlane(sets);
    if (sets > kDigitSets) return 0;
    if (__builtin_expect(sets > 1, 0)) {
        for (int s = 1; s < sets; ++s) none_in(s);
        __syncthreads();
    }
    return sets;
}

// The row groups [g0, g1) of a wave with the digits in LDS; c: the codes of the first ones.  MANY: more than one set.
template <int BITS, int U, bool MANY>
__device__ __forceinline__ void table_by_digits(const uint32_t *__restrict__ c0, uint32_t (&c)[U][2 * BITS],
                                                const unsigned char *digits, int sets, int exponent, int g0, int g1,
                                                int n_out, float scale, float *__restrict__ out, const LayerTable &layers) {
    const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
    // row m: plane m; bytes 0..15 and 16..31: columns 16 q and 64 + 16 q of a half
    auto operand = [&](int set, int h) {
        const unsigned char *at = digits + set * kDigitSetBytes + m * kDigitStride + 128 * h + 16 * q;
        const i32x4 lo = *reinterpret_cast<const i32x4 *>(at), hi = *reinterpret_cast<const i32x4 *>(at + 64);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    i32x8 op0, op1;
    auto load_set = [&](int set) {
        op0 = operand(set, 0);
        op1 = operand(set, 1);
    };
    if (!MANY) load_set(0);
    const int plane_scale = 127 - 5 * m;  // a power of two, biased by 127
    // x[i]: of row group 4 i + q, row m
    auto product = [&](int exponent, float (&x)[U / 4]) {
        f32x4 acc[U];
#pragma unroll
        for (int i = 0; i < U; ++i)
            acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(op0, nibbles<BITS>(c[i], 0), f32x4{}, 0, 4, 0,
                                                                      plane_scale, 0, 127);
#pragma unroll
        for (int i = 0; i < U; ++i)
            acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(op1, nibbles<BITS>(c[i], 1), acc[i], 0, 4, 0,
                                                                      plane_scale, 0, 127);
        float sum[U];  // lane quarter q: planes 4 q .. 4 q + 3
#pragma unroll
        for (int i = 0; i < U; ++i) sum[i] = ((acc[i].w + acc[i].z) + acc[i].y) + acc[i].x;
#pragma unroll
        for (int i = 0; i < U; i += 4) {
            // sums over the four lane quarters; quarter q gets that of the q-th of four row groups
            auto add = [](auto r) { return __uint_as_float(r[0]) + __uint_as_float(r[1]); };
            const float a = add(__builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i]), __float_as_uint(sum[i + 2]), false, false));
            const float b = add(__builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i + 1]), __float_as_uint(sum[i + 3]), false, false));
            x[i / 4] = __builtin_amdgcn_ldexpf(
                add(__builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)), exponent);
        }
    };
    for (int g = g0; g < g1; g += U) {
        uint32_t next[U][2 * BITS];
#pragma unroll
        for (int i = 0; i < U; ++i)
            if (g + U + i < g1) load_codes<BITS>(c0 + (long long)(g + U + i) * 128 * BITS, next[i]);
        float x[U / 4];
        if constexpr (MANY) {  // the smallest first
            load_set(sets - 1);
            product(exponent - (sets - 1) * kDigitExponents, x);
            for (int s = sets - 2; s >= 0; --s) {
                load_set(s);
                float y[U / 4];
                product(exponent - s * kDigitExponents, y);
#pragma unroll
                for (int i = 0; i < U / 4; ++i) x[i] += y[i];
            }
        } else {
            product(exponent, x);
        }
#pragma unroll
        for (int i = 0; i < U; i += 4) {
            if (g + i + q >= g1) continue;
            if (layers.n == 0) {
                const long long row = (long long)(g + i) * kDenseRows + lane;
                if (row < n_out) out[row] = scale * x[i / 4];
            } else {
                int s = 0;
#pragma unroll
                for (int l = 1; l < kMaxLayers; ++l)
                    if (l < layers.n && g + i + q >= layers.first[l]) s = l;
                const int local = (g + i + q - layers.first[s]) * kDenseRows + m;
                if (local < layers.rows[s]) layers.out[s][local] = layers.scale[s] * x[i / 4];
            }
        }
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) c[i][d] = next[i][d];
    }
}

template <typename VT, int BITS, int NV>
__global__ __launch_bounds__(kTableWaves * 64, (TableFew<VT, NV>::occupancy)) void k_table_few(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ngroups, int per, int n_in, int n_out,
    long long ldv, int nv, float scale, float *__restrict__ out, long long ldo, int skip_zeros,
    const LayerTable layers) {
    using S = TableFew<VT, NV>;
    constexpr int U = 8 / BITS;  // row groups at a time: 4 KiB of codes
    const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int kBytes = NV * S::planes * S::stride;
    __shared__ __attribute__((aligned(16))) unsigned char smem[NV == 1 ? kTableOneLds : kBytes];
    const int g0 = (int)min((long long)ngroups, ((long long)blockIdx.x * kTableWaves + w) * per);
    const int g1 = (int)min((long long)ngroups, (long long)g0 + per);

    const uint32_t *c0 = codes + lane * (2 * BITS);
    uint32_t c[U][2 * BITS];
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (g0 + i < g1) load_codes<BITS>(c0 + (long long)(g0 + i) * 128 * BITS, c[i]);
    if constexpr (NV == 1) {
        static_assert(kTableWaves * 64 == kTileCols && kBytes <= kDigitSetBytes, "a thread per column");
        int exponent;
        const int sets = table_digits<VT, BITS>(v, n_in, smem, reinterpret_cast<float *>(smem + kDigitSets * kDigitSetBytes), &exponent);
        if (__builtin_expect(sets == 1, 1)) {
            table_by_digits<BITS, U, false>(c0, c, smem, 1, exponent, g0, g1, n_out, scale, out, layers);
            return;
        }
        if (sets > 1) {
            // (four row groups at a time: the operands change with the set, and more do not fit the registers)
            uint32_t four[4][2 * BITS];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int d = 0; d < 2 * BITS; ++d) four[i][d] = c[i][d];
            table_by_digits<BITS, 4, true>(c0, four, smem, sets, exponent, g0, g1, n_out, scale, out, layers);
            return;
        }
        __syncthreads();  // (the flags have been read)
    }
    constexpr int pieces = kTileCols / 8;
    for (int i = threadIdx.x; i < NV * pieces; i += kTableWaves * 64) {
        const int n = i / pieces, col = 8 * (i % pieces);
        const VT *row = v + min(n, nv - 1) * ldv;
        Piece<VT> p = load_piece<VT>(row, col, n_in);
        if (n_in & 7) finish_piece<VT>(p, row, col, n_in);
        store_piece(smem + n * S::planes * S::stride + col * 2, S::stride, p);
    }
    __syncthreads();
    bf16x8 op[S::operands][kTileSteps];
    {
        const int n = NV == 1 ? 0 : NV == 4 ? m >> 2 : m;
        const int plane = NV < 16 && S::planes == 3 ? min(m & 3, 2) : 0;
#pragma unroll
        for (int o = 0; o < S::operands; ++o)
#pragma unroll
            for (int st = 0; st < kTileSteps; ++st)
                op[o][st] = lds_operand(smem + (n * S::planes + plane + o) * S::stride + 64 * st + 16 * q);
    }
    uint64_t again = 0;  // lanes with results that are not finite
    for (int g = g0; g < g1; g += U) {
        uint32_t next[U][2 * BITS];
#pragma unroll
        for (int i = 0; i < U; ++i)
            if (g + U + i < g1) load_codes<BITS>(c0 + (long long)(g + U + i) * 128 * BITS, next[i]);
        f32x4 acc[U] = {};
#pragma unroll
        for (int i0 = 0; i0 < U; i0 += 2) {
            if (g + i0 >= g1) break;
#pragma unroll
            for (int st = 0; st < kTileSteps; ++st)
#pragma unroll
                for (int i = i0; i < i0 + 2; ++i) {
                    const bf16x8 x = decode<BITS>(c[i], st);
#pragma unroll
                    for (int o = 0; o < S::operands; ++o)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[o][st], x, acc[i], 0, 0, 0);
                }
        }
        float check = 0.0f;  // NaN if one of them is not finite
        if (NV == 16) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const long long row = (long long)(g + i) * kDenseRows + m;
                if (g + i >= g1 || row >= n_out) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (4 * q + e < nv) out[(4 * q + e) * ldo + row] = scale * acc[i][e];
                    check += 0.0f * acc[i][e];
                }
            }
        } else {
            float sum[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                sum[i] = S::planes == 3 ? acc[i].x + (acc[i].y + acc[i].z) : acc[i].x;
                check += 0.0f * sum[i];  // (behind g1: some finite weights, whatever the registers hold)
            }
            if (layers.n) {
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    if (q || g + i >= g1) continue;
                    int s = 0;
#pragma unroll
                    for (int l = 1; l < kMaxLayers; ++l)
                        if (l < layers.n && g + i >= layers.first[l]) s = l;
                    const int local = (g + i - layers.first[s]) * kDenseRows + m;
                    if (local < layers.rows[s]) layers.out[s][local] = layers.scale[s] * sum[i];
                }
            } else if (NV == 1) {
                // all rows of the MFMA are the one vector: lane quarter q stores the q-th of four groups
#pragma unroll
                for (int i = 0; i < U; i += 4) {
                    const float x = q == 0 ? sum[i] : q == 1 ? sum[i + 1] : q == 2 ? sum[i + 2] : sum[i + 3];
                    const long long row = (long long)(g + i) * kDenseRows + lane;
                    if (g + i + q < g1 && row < n_out) out[row] = scale * x;
                }
            } else {
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const long long row = (long long)(g + i) * kDenseRows + m;
                    if (g + i < g1 && row < n_out && q < nv) out[q * ldo + row] = scale * sum[i];
                }
            }
        }
        again |= __ballot(check != check);
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) c[i][d] = next[i][d];
    }
    if (__builtin_expect(again != 0, 0)) {
        if (!skip_zeros) return;
        const long long row0 = (long long)g0 * kDenseRows;
        const int rows = (int)min((long long)(g1 - g0) * kDenseRows, (long long)n_out - row0);
        if (layers.n == 0) {
            sum_again<VT, BITS>(codes, 1, v, ldv, row0, out + row0, ldo, rows, nv, scale);
            return;
        }
        for (int s = 0; s < layers.n; ++s) {  // the part of the wave's rows that is in layer s
            const long long start = (long long)layers.first[s] * kDenseRows;
            const long long from = max(row0, start);
            const long long to = min((long long)g1 * kDenseRows, start + layers.rows[s]);
            if (from < to)
                sum_again<VT, BITS>(codes, 1, v, 0, from, layers.out[s] + (from - start), 0, (int)(to - from), 1,
                                    layers.scale[s]);
        }
    }
}

// table_many: 32 NT vectors per workgroup, in LDS in operand order with all planes; a wave takes
// 64 rows at a time, so an operand read from LDS serves two MFMAs.
constexpr int kManyWaves = 8;
constexpr int kManyStride = kTileCols * 2 + 16;  // bytes between vectors: an odd number of 16-byte units
template <typename VT, int NT>
struct TableMany {
    static constexpr int planes = sizeof(VT) == 4 ? 3 : 1;
    static constexpr int plane = 32 * NT * kManyStride;
    static constexpr int lds = planes * plane;
};

template <typename VT, int BITS, int NT>
__global__ __launch_bounds__(kManyWaves * 64, (NT == 1 ? 4 : 2)) void k_table_many(
    const uint32_t *__restrict__ codes, const VT *__restrict__ v, int ngroups, int n_in, int n_out, long long ldv,
    int batch, float scale, float *__restrict__ out, long long ldo, int skip_zeros) {
    using S = TableMany<VT, NT>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int vec0 = blockIdx.y * 32 * NT;
    const int sets = (ngroups + 3) / 4, stride = gridDim.x * kManyWaves;
    const uint32_t *c0 = codes + lane * (2 * BITS);
    uint32_t c[4][2 * BITS];
    int set = blockIdx.x * kManyWaves + w;
#pragma unroll
    for (int i = 0; i < 4; ++i) load_codes<BITS>(c0 + (long long)min(set * 4 + i, ngroups - 1) * 128 * BITS, c[i]);
    for (int i = tid; i < 32 * NT * (kTileCols / 8); i += kManyWaves * 64) {
        const int n = i / (kTileCols / 8), col = 8 * (i % (kTileCols / 8));
        const VT *row = v + (long long)min(vec0 + n, batch - 1) * ldv;
        Piece<VT> p = load_piece<VT>(row, col, n_in);
        if (n_in & 7) finish_piece<VT>(p, row, col, n_in);
        store_piece(smem + n * kManyStride + col * 2, S::plane, p);
    }
    __syncthreads();
    const unsigned char *x = smem + (lane & 31) * kManyStride + 32 * half;
    uint64_t again = 0;  // lanes with results that are not finite
    for (; set < sets; set += stride) {
        uint32_t next[4][2 * BITS];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            load_codes<BITS>(c0 + (long long)min((set + stride) * 4LL + i, ngroups - 1LL) * 128 * BITS, next[i]);
        pair_groups(c[0], c[1]);
        pair_groups(c[2], c[3]);
        f32x16 acc[2][NT] = {};
#pragma unroll
        for (int st = 0; st < kTileSteps; ++st) {
            if (32 * st >= n_in) break;
#pragma unroll
            for (int xy = 0; xy < 2; ++xy) {
                const bf16x8 w0 = decode<BITS>(c[xy], st), w1 = decode<BITS>(c[2 + xy], st);
#pragma unroll
                for (int pl = 0; pl < S::planes; ++pl)
#pragma unroll
                    for (int ng = 0; ng < NT; ++ng) {
                        const bf16x8 o =
                            lds_operand(x + pl * S::plane + ng * 32 * kManyStride + 64 * st + 16 * xy);
                        acc[0][ng] = mfma32(o, w0, acc[0][ng]);
                        acc[1][ng] = mfma32(o, w1, acc[1][ng]);
                    }
            }
        }
        float check = 0.0f;  // NaN if one of them is not finite
#pragma unroll
        for (int ng = 0; ng < NT; ++ng)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int n = vec0 + ng * 32 + acc_vector(i, half);
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) {
                    const long long r = (long long)set * 64 + rg * 32 + (lane & 31);
                    if (n < batch && r < n_out)
                        out[(long long)n * ldo + r] = scale * acc[rg][ng][i];
                    check += 0.0f * acc[rg][ng][i];
                }
            }
        again |= __ballot(check != check);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int d = 0; d < 2 * BITS; ++d) c[i][d] = next[i][d];
    }
    if (__builtin_expect(again != 0, 0)) {
        if (!skip_zeros || vec0 >= batch) return;
        for (set = blockIdx.x * kManyWaves + w; set < sets; set += stride) {
            const long long row0 = (long long)set * 64;
            sum_again<VT, BITS>(codes, 1, v + vec0 * ldv, ldv, row0, out + vec0 * ldo + row0, ldo,
                                (int)min(64LL, n_out - row0), min(32 * NT, batch - vec0), scale);
        }
    }
}

struct Args {
    const uint32_t *codes;
    const void *v;
    int ntiles, ngroups, n_in, n_out, batch, device, skip_zeros;
    long long ldv, ldo;
    float *out;
    float scale;
    hipStream_t stream;
    LayerTable layers;
    char *name;  // not null: write the name of the kernel there instead of launching it
    size_t name_len;
};

// The instantiation as a profiler prints it.
template <typename VT, typename... Number>
hipError_t put_name(const Args &x, const char *kernel, const char *numbers, Number... n) {
    const int at = std::snprintf(x.name, x.name_len, "%s<%s, ", kernel, sizeof(VT) == 4 ? "float" : "unsigned short");
    if (at > 0 && (size_t)at < x.name_len) std::snprintf(x.name + at, x.name_len - at, numbers, n...);
    return hipSuccess;
}

// G = 0: k_packed_few; else k_packed_tall.
template <typename VT, int BITS, int NV, int WK, int G, int TILES = few_tiles<VT, NV>>
hipError_t launch_few_groups(const Args &x) {
    static std::atomic<size_t> enabled[kMaxDevices];
    auto kern = [] {
        if constexpr (G == 0)
            return k_packed_few<VT, BITS, NV, WK>;
        else
            return k_packed_tall<VT, BITS, NV, WK, G, TILES>;
    }();
    if (x.name) {
        if (G == 0) return put_name<VT>(x, "k_packed_few", "%d, %d, %d>", BITS, NV, WK);
        return put_name<VT>(x, "k_packed_tall", "%d, %d, %d, %d, %d>", BITS, NV, WK, G, TILES);
    }
    constexpr int each = G == 0 ? 1 : G;
    constexpr size_t lds = (size_t)few_waves(WK) * (Few<VT, NV, TILES>::wave_bytes + each * 64 * 4);
    static_assert(lds <= (size_t)kLdsBytes, "every wave stages columns of its own");
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, x.device, enabled)) return e;
    constexpr int groups = few_waves(WK) / WK * each;
    hipLaunchKernelGGL(kern, dim3((unsigned)((x.ngroups + groups - 1) / groups)), dim3(few_waves(WK) * 64), lds, x.stream,
                       x.codes, static_cast<const VT *>(x.v), x.ntiles, x.ngroups, x.n_in, x.n_out, x.ldv, x.batch,
                       x.scale, x.out, x.ldo, x.skip_zeros, x.layers);
    return hipGetLastError();
}

// Row groups of a wave, G = 0 for k_packed_few, and tiles staged at a time.  Two or four groups save the staging of v and
// the reads of its operands, which is most of the work for float32 vectors (three planes) and for several; they pay once the
// workgroups of one row group are too many for the chip, that is 256 of sixteen waves or 512 of eight.  One bf16 vector is
// staged in no time (13824 x 2560 4.3 us, with two groups 4.7).  Measured with 1 / 2 / 4 groups:
//   float32, 1 vector    6000 x 8000 7.4 / 5.8 / 12.0 us (4000 rows 4.9 / 5.6), 10000 x 2500 7.2 / 5.6 / 6.1, 14336 x 4096 6.9 /
//                        6.0 / 6.4 (8192 rows 4.8 / 4.8), 40000 x 500 6.1 / 5.0 / 5.4 (20000 4.1 / 4.3), 14336 x 1000 3.8 / 3.7
//   float32, 3 vectors   6000 x 8000 9.4 / 6.9 / 8.9, 10000 x 8000 13.2 / 11.5 / 9.1, 14336 x 4096 8.8 / 7.0 / 6.3
//                        (8192 rows 5.7 / 5.5 / 5.9), 40000 x 1000 6.4 / 5.1 / 5.2
//   bf16, 4 vectors      14336 x 2500 7.6 / 6.5 / 6.4, 14336 x 1000 4.1 / 3.7 (8192 rows 3.3 / 3.3);
//                        with two tiles of columns to a wave 14336 x 4096 6.0 / 5.9, but in two rounds 20000 x 4096 7.1 / 7.3
// The limits, with one / two (/ four) groups: eight waves, 4 float32 vectors of 2560 (ten tiles to eight waves), 513 groups 5.3 /
// 5.2 / 5.8 and 1024 7.8 / 5.9 / 6.0, of 4096, 513 6.3 / 5.7 / 6.0, 640 6.9 / 6.7 / 6.0, with one-bit codes and more than
// 16 tiles 3 vectors of 4461, 700 groups 7.2 / 7.1 / 7.4; sixteen waves, 1 float32 vector of 14336, 520
// groups 2 to 4 % slower with two.  Four waves, 1 float32 vector: five workgroups of one row group share a CU, so 1281 is where
// their second round begins (of 1280, 780 groups 3.8 / 3.8, 1400 4.9 / 4.2, 1700 5.3 / 5.6; of 1792, 2500 groups 7.2 /
// 7.5); with two-bit codes three of two row groups, whose second round begins at 1537: of 1020, 1536 groups
// 4.63 / 4.00, 1600 4.82 / 5.16, 1800 5.13 / 5.36, 1920 5.33 / 5.35); several: 770 groups of 1280 6 % slower, of 1024 9 % faster,
// from 900 on all faster.  Two waves, 4 bf16 vectors: two tiles, 900 groups 3.3 / 3.2; three, of 700, 1300 4.9 / 5.5, 1700 5.8 / 5.6.
// One float32 vector, eight waves: that is 512 workgroups of two-bit codes (86 registers), but 768 of one-bit codes (78), three to
// a CU; k_packed_tall (94) has two either way, 1024 row groups in a round.  One-bit, of 2560, 640 groups 4.28 / 4.89, 768 4.42 /
// 5.06, 820 5.40 / 5.05, 1024 5.58 / 4.93, 1100 6.22 / 6.76, 1536 7.35 / 7.75, 1800 9.09 / 8.34; between 1024 and 1536, both being in their
// second round, two pay on 2048 (1300 6.31 / 5.85) and long rows (of 5120, 1100 7.51 / 8.07, 1300 8.61 / 8.28, 1536 9.26 / 8.52).
// Sixteen waves and several bf16 vectors: a CU holds two workgroups of k_packed_few (60 registers, 70 KB of LDS) and one of
// k_packed_tall (66 registers and more), so a round is 512 row groups for either, and two groups pay where the last round is
// more than half full: with one / two groups, 4 vectors of 8192 elements, 4160 rows 5.8 / 5.2, 8192 6.5 / 5.9, 8320 8.1 /
// 8.3, 12480 9.9 / 8.9, 16384 11.7 / 9.6, 17600 12.7 / 12.1, 24576 16.0 / 13.5.  Four tiles staged at a time take one step
// instead of two where most waves have three or four (4 vectors of 14336, 4096 rows 6.9 -> 6.2, two groups, 6144 rows
// 9.2 -> 8.3), and otherwise only LDS: 4 vectors of 8192, 4096 rows 4.6 -> 5.0, of 20480, 2048 rows 8.2 -> 8.3.
struct FewShape {
    int G, tiles;
};
template <typename VT, int BITS, int NV>
FewShape few_shape(int ntiles, int ngroups, int wk) {
    const bool wide = sizeof(VT) == 4;
    const int tiles = few_tiles<VT, NV>;
    if ((!wide && NV == 1) || wk == 1) return {0, tiles};
    if (wk == 16 && !wide) {
        const bool four = ntiles >= 36 && ntiles <= 64;
        if (ngroups <= 256) return {four ? 1 : 0, four ? 4 : tiles};
        if ((ngroups - 1) % 512 < 256 || (four && ngroups > 1024)) return {0, tiles};
        return {2, four ? 4 : tiles};
    }
    if (wk == 16 && NV == 1 && ntiles > 44 && ngroups > 512 && ngroups <= 768) return {0, tiles};
    if (wk == 16) return {ngroups <= 256 ? 0 : NV == 4 && ngroups > 512 ? 4 : 2, tiles};
    if (wk == 8 && wide && NV == 1 && BITS == 1) {
        const bool two = ngroups > 1024 && ngroups <= 1536 ? ntiles == 8 || (ntiles >= 16 && ngroups > 1280) : ngroups > 768;
        return {two ? 2 : 0, tiles};
    }
    if (wk == 8 && wide) return {ngroups <= 512 ? 0 : NV == 4 && ngroups > ((BITS == 1 ? ntiles == 16 : ntiles >= 16) ? 576 : 768) ? 4 : 2, tiles};
    if (wk == 8) return {ngroups > 768 && (ntiles <= 12 || ngroups <= 1024) ? 2 : 0, tiles};
    if (wk == 4 && NV == 1 && BITS == 2 && ntiles == 4 && ngroups > 1536 && ngroups <= 1856) return {0, tiles};
    if (wk == 4 && NV == 1) return {(ntiles == 4 ? ngroups > 768 : ngroups > 1280 && ngroups <= 1536) ? 2 : 0, tiles};
    if (wk == 4) return {ngroups > (ntiles == 4 ? 768 : 896) ? 2 : 0, tiles};
    return {ngroups > (wide ? 2048 : ntiles == 2 ? 768 : 1536) ? 2 : 0, tiles};
}

template <typename VT, int BITS, int NV, int WK>
hipError_t launch_few_wk(const Args &x) {
    const FewShape s = few_shape<VT, BITS, NV>(x.ntiles, x.ngroups, WK);
    if constexpr (sizeof(VT) == 4 && NV == 4 && WK >= 8) {
        if (s.G == 4) return launch_few_groups<VT, BITS, NV, WK, 4>(x);
    }
    if constexpr (sizeof(VT) == 2 && NV == 4 && WK == 16) {
        if (s.tiles == 4) return s.G == 1 ? launch_few_groups<VT, BITS, NV, WK, 1, 4>(x) : launch_few_groups<VT, BITS, NV, WK, 2, 4>(x);
    }
    if constexpr ((sizeof(VT) == 4 || NV == 4) && WK > 1) {
        if (s.G == 2) return launch_few_groups<VT, BITS, NV, WK, 2>(x);
    }
    return launch_few_groups<VT, BITS, NV, WK, 0>(x);
}

// Waves that share the columns of a row group: one per tile of columns up to eight, so that all
// loads of a product leave at once; from 24 tiles on sixteen waves, whose loads, decoding and MFMAs
// overlap better.  Measured with 4 / 8 / 16 waves, one bf16 vector: 4096 x 14336 (56 tiles) 7.9 /
// 5.9 / 5.4 us, 2560 x 6912 (27) 4.6 / 3.7 / 3.6, 4096 x 4096 (16) 3.3 / 3.0 / 3.2, 14336 x 4096
// 5.3 / 4.9 / 6.1; 100000 x 256 (one tile) 3.3 with one wave, 4.3 with two.
int few_wk(int ntiles) {
    return ntiles >= 24 ? 16 : ntiles >= 8 ? 8 : ntiles >= 4 ? 4 : ntiles >= 2 ? 2 : 1;
}

template <typename VT, int BITS, int NV>
hipError_t launch_few(const Args &x) {
    switch (few_wk(x.ntiles)) {
        case 16: return launch_few_wk<VT, BITS, NV, 16>(x);
        case 8: return launch_few_wk<VT, BITS, NV, 8>(x);
        case 4: return launch_few_wk<VT, BITS, NV, 4>(x);
        case 2: return launch_few_wk<VT, BITS, NV, 2>(x);
        default: return launch_few_wk<VT, BITS, NV, 1>(x);
    }
}

// Consecutive row groups every wave gets: so many that `waves` waves, which just fill the chip, do
// them all.
int table_groups_per_wave(int64_t groups, int waves) {
    const int64_t per = (groups + waves - 1) / waves;
    return (int)(per > 4 ? (per + 3) / 4 * 4 : per);
}

template <typename VT, int BITS, int NV>
hipError_t launch_table_few(const Args &x) {
    if (x.name) return put_name<VT>(x, "k_table_few", "%d, %d>", BITS, NV);
    constexpr int waves = kCUs * 4 * TableFew<VT, NV>::occupancy;
    const int per = table_groups_per_wave(x.ngroups, waves);
    const unsigned grid = (unsigned)((x.ngroups + (long long)per * kTableWaves - 1) / ((long long)per * kTableWaves));
    hipLaunchKernelGGL((k_table_few<VT, BITS, NV>), dim3(grid), dim3(kTableWaves * 64), 0, x.stream, x.codes,
                       static_cast<const VT *>(x.v), x.ngroups, per, x.n_in, x.n_out, x.ldv, x.batch, x.scale, x.out,
                       x.ldo, x.skip_zeros, x.layers);
    return hipGetLastError();
}

template <typename VT, int BITS, int NT>
hipError_t launch_table_many(const Args &x) {
    if (x.name) return put_name<VT>(x, "k_table_many", "%d, %d>", BITS, NT);
    static std::atomic<size_t> enabled[kMaxDevices];
    auto kern = k_table_many<VT, BITS, NT>;
    constexpr size_t lds = TableMany<VT, NT>::lds;
    static_assert(lds <= (size_t)kLdsBytes, "all vectors of a workgroup are staged at once");
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, x.device, enabled)) return e;
    const int sets = (x.ngroups + 3) / 4, chunks = (x.batch + 32 * NT - 1) / (32 * NT);
    int grid = (sets + kManyWaves - 1) / kManyWaves;
    const int room = kCUs * (NT == 1 ? 2 : 1) / chunks;  // of the workgroups that the chip holds
    if (grid > room) grid = room;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid, (unsigned)chunks), dim3(kManyWaves * 64), lds, x.stream, x.codes,
                       static_cast<const VT *>(x.v), x.ngroups, x.n_in, x.n_out, x.ldv, x.batch, x.scale, x.out,
                       x.ldo, x.skip_zeros);
    return hipGetLastError();
}

// Shape of the split kernel: vectors (16 NT) and row groups (G) of a workgroup, waves that share a row
// group's columns.  Up to 16 vectors take the 16 x 16 MFMA and no padding.  More rows per workgroup
// read v less often, fewer give more workgroups: measured with 1 / 2 / 4 row groups, 16 float32
// vectors: 4096 rows (x 14336) 22.8 / 23.4 / 28.7 us, 6912 (x 2560) 10.0 / 8.3 / 9.7, 14336 (x 4096)
// 20.9 / 13.8 / 11.8.  From 512 row groups on two of them are more than one workgroup per CU, which costs most where
// columns are many: 9000 rows with 2 / 4, 16 float32 vectors, x 8000 23.2 / 19.4, x 4096 13.6 / 11.1, x 2400 10.9 / 10.7,
// x 1000 6.2 / 6.5; 16 bf16 x 4096 7.9 / 6.7, 6 bf16 x 8000 10.9 / 10.8, x 2400 6.1 / 6.6.  Where the limits lie (codes in the L2;
// from the Infinity Cache two groups lose a few per cent more): float32 x 2900 (12 tiles), 9 vectors, 513 groups 10.3 / 10.4, 540
// 10.7 / 10.4, x 3300, 513 11.0 / 10.5; bf16 x 3300, 9 vectors, 513 6.5 / 7.2, 540 7.0 / 7.3, 600 7.3 / 7.3, 16 vectors,
// 513 6.7 / 7.4, 540 8.0 / 7.5.  32 vectors with 2 / 4: a workgroup of four row groups takes about 1.3 times as
// long (24 float32 vectors, 6912 x 2560: 12.4 / 15.0), so four pay where they save a round of
// workgroups (14336 x 4096: 24.0 / 16.8), for bf16 where they fit in one round (4096 x 14336, 100
// vectors: 30.4 / 21.5; 6912 x 2560, 432 workgroups: 13.7 / 14.5).  Waves without columns take
// other rows where there are workgroups enough (60000 x 300, 24 float32 vectors: 31 / 19 / 13.5 us
// with 4 / 2 / 2 waves on a row group and 2 / 2 / 4 row groups).
struct SplitShape {
    int NT, G, wk_log2;
};
SplitShape split_shape(int ntiles, int ngroups, int batch, bool wide) {
    SplitShape s = {batch <= 16 ? 1 : 2, 1, 3};
    const long long units = (long long)ngroups * ((batch + 16 * s.NT - 1) / (16 * s.NT));
    if (s.NT == 1) {
        const int four = wide && ntiles >= 13 ? 512 : (wide && ntiles == 12) || (ntiles >= 13 && batch > 8) ? 536 : 640;
        s.G = units > four ? 4 : units > 320 ? 2 : 1;
    } else {
        const long long two = (units / 2 + kCUs - 1) / kCUs, four = (units / 4 + kCUs - 1) / kCUs;  // rounds
        s.G = 13 * four < 10 * two && (wide || four <= 1) ? 4 : 2;
    }
    const long long room = s.NT == 2 && !wide ? 2 * kCUs : kCUs;
    while (s.wk_log2 > 0 && 1 << s.wk_log2 > ntiles && (units / s.G << s.wk_log2) / kSplitWaves > room) --s.wk_log2;
    return s;
}

template <typename VT, int BITS, int NT, int G, bool ROWS>
hipError_t launch_split_rows(const Args &x, int wk_log2) {
    if (x.name) return put_name<VT>(x, "k_packed_split", "%d, %d, %d, %s>", BITS, NT, G, ROWS ? "true" : "false");
    static std::atomic<size_t> enabled[kMaxDevices];
    auto kern = k_packed_split<VT, BITS, NT, G, ROWS>;
    constexpr size_t lds = (size_t)kSplitWaves * Split<VT, NT>::wave_bytes;
    static_assert(lds >= (size_t)kSplitWaves * G * NT * 1024 && lds <= (size_t)kLdsBytes,
                  "partial results share the staging area");
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, x.device, enabled)) return e;
    const int groups = (kSplitWaves >> wk_log2) * G;  // of a workgroup
    const dim3 grid((unsigned)((x.ngroups + groups - 1) / groups), (unsigned)((x.batch + 16 * NT - 1) / (16 * NT)));
    hipLaunchKernelGGL(kern, grid, dim3(kSplitWaves * 64), lds, x.stream, x.codes, static_cast<const VT *>(x.v),
                       x.ntiles, x.ngroups, x.n_in, x.n_out, x.ldv, x.batch, x.out, x.ldo, x.scale, wk_log2,
                       x.skip_zeros);
    return hipGetLastError();
}

template <typename VT, int BITS, int NT, int G>
hipError_t launch_split_g(const Args &x, int wk_log2) {
    return wk_log2 == 3 ? launch_split_rows<VT, BITS, NT, G, false>(x, 3)
                        : launch_split_rows<VT, BITS, NT, G, true>(x, wk_log2);
}

template <typename VT, int BITS>
hipError_t launch_split(const Args &x) {
    const SplitShape sh = split_shape(x.ntiles, x.ngroups, x.batch, sizeof(VT) == 4);
    switch (sh.NT * 10 + sh.G) {
        case 24: return launch_split_g<VT, BITS, 2, 4>(x, sh.wk_log2);
        case 22: return launch_split_g<VT, BITS, 2, 2>(x, sh.wk_log2);
        case 14: return launch_split_g<VT, BITS, 1, 4>(x, sh.wk_log2);
        case 12: return launch_split_g<VT, BITS, 1, 2>(x, sh.wk_log2);
        default: return launch_split_g<VT, BITS, 1, 1>(x, sh.wk_log2);
    }
}

template <typename VT, int BITS, int KW, int RB>
hipError_t launch_tile_kw(const Args &x) {
    if (x.name) return put_name<VT>(x, "k_packed_tile", "%d, %d, %d>", BITS, KW, RB);
    static std::atomic<size_t> enabled[kMaxDevices];
    auto kern = k_packed_tile<VT, BITS, KW, RB>;
    constexpr size_t lds = 2 * (size_t)Tile<VT>::buffer;
    static_assert(lds >= 4 * 2048 * sizeof(float), "partial results share the staging buffers");
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, x.device, enabled)) return e;
    const int row_tiles = (x.n_out + 127) / 128, vec_tiles = (x.batch + 127) / 128;
    const int per = (row_tiles * vec_tiles + 7) / 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(per * 8)), dim3(256 * KW), lds, x.stream, x.codes,
                       static_cast<const VT *>(x.v), x.ntiles, x.ngroups, x.n_in, x.n_out, x.ldv, x.batch, x.out,
                       x.ldo, x.scale, row_tiles, vec_tiles, x.skip_zeros);
    return hipGetLastError();
}

// Up to 256 workgroups a CU has one, and eight waves do better than four: 4096 x 14336 x 512 bf16
// vectors 118 -> 108 us, 6912 x 2560 x 300 float32 71 -> 53; beyond, two workgroups share a CU and four
// waves each are faster (6912 x 2560 x 700: bf16 37.8 against 38.8, float32 95 against 106), until, from
// 500 workgroups on, the two meet (4096 x 4096 x 2048 float32 172 / 175; 14336 x 4096 x 700 260 / 244).
// With eight waves bf16 is bound by decoding, so a wave takes 32 rows and all vectors (every code
// decoded by one wave instead of two: 120 -> 105); float32 reads its three planes of v too often then
// (252 -> 259).
template <typename VT, int BITS>
hipError_t launch_tile(const Args &x) {
    if ((long long)((x.n_out + 127) / 128) * ((x.batch + 127) / 128) > kCUs) return launch_tile_kw<VT, BITS, 1, 2>(x);
    return launch_tile_kw<VT, BITS, 2, sizeof(VT) == 4 ? 2 : 1>(x);
}

// Tiles of 128 x 128 need enough workgroups to be worth their size, tiles / columns split over waves:
// bf16 4096 x 4096 x 512 vectors (128 workgroups) 33.7 / 36.2 us, 4096 x 14336 x 512 108 / 119,
// 14336 x 4096 x 100 (112) 31.6 / 27.3; float32 14336 x 4096 x 100 (112) 76 / 60, 4096 x 4096 x 512 (128)
// 80 / 64, x 600 (160) 82 / 78, 6912 x 2560 x 300 (162) 53 / 69.  Up to 32 vectors a tile is mostly padding (60000 x 300, 24 float32 vectors:
// 24.3 / 13.5).
bool use_tile(const Args &x, bool wide) {
    const long long workgroups = (long long)((x.n_out + 127) / 128) * ((x.batch + 127) / 128);
    return workgroups >= (wide ? 160 : 128) && x.batch > 32;
}

// Up to 256 columns: vectors per workgroup of the table kernels, 0 where the others are faster.
// Waves that work through many row groups pay for bringing v into registers first and win only
// when there are rows enough, measured (table kernel / other, 200 ternary columns):
//   1 float32 vector   120000 rows 4.7 / 4.9 us (binary 5.3 / 4.8), 160000 4.9 / 5.8 (binary 5.3 / 5.7)
//   1 bf16 vector      160000 rows 4.9 / 4.7 (binary 5.3 / 4.6), 240000 5.3 / 5.8 (binary 5.6 / 5.7; with an element that needs a
//                      second set of digits 6.5 / 5.8 and 5.8 / 5.7, 400000 7.7 / 8.1)
//   4 bf16 vectors     20000 rows 3.3 / 3.1, 100000 4.1 / 5.0
//   5 to 16            500 rows 3.3 / 3.6 (bf16), 20000 rows 4.6 / 14.7 (float32): always
//   up to 64, float32  3000 rows 10.9 / 6.0, 12000 11.7 / 15.1
//   up to 64, bf16     12000 rows 7.4 / 6.3, 20000 7.7 / 8.8
// From more than 128 vectors on the tile kernel has little padding left (100000 rows, 200 float32
// vectors: 49.9 / 53.5; 20000 rows, 512 bf16 vectors 18.4 / 13.7).
int table_vectors(int ntiles, int64_t rows, int batch, bool wide) {
    if (ntiles != 1) return 0;
    if (batch == 1) return rows >= (wide ? 140000 : 240000) ? 1 : 0;
    if (batch <= 4) return rows >= 65536 ? 4 : 0;
    if (batch <= 16) return 16;
    if (batch > 128 || rows < (wide ? 10000 : 16384)) return 0;
    return batch <= 32 ? 32 : 64;
}

template <typename VT, int BITS>
hipError_t launch(const Args &x) {
    switch (table_vectors(x.ntiles, x.n_out, x.batch, sizeof(VT) == 4)) {
        case 1: return launch_table_few<VT, BITS, 1>(x);
        case 4: return launch_table_few<VT, BITS, 4>(x);
        case 16: return launch_table_few<VT, BITS, 16>(x);
        case 32: return launch_table_many<VT, BITS, 1>(x);
        case 64: return launch_table_many<VT, BITS, 2>(x);
        default: break;
    }
    if (x.batch == 1) return launch_few<VT, BITS, 1>(x);
    if (x.batch <= 4) return launch_few<VT, BITS, 4>(x);
    return use_tile(x, sizeof(VT) == 4) ? launch_tile<VT, BITS>(x) : launch_split<VT, BITS>(x);
}

}  // namespace

int64_t packed_bytes(int64_t groups, int64_t cols, int bits) {
    return groups * ((cols + kTileCols - 1) / kTileCols) * 512 * bits;
}

hipError_t launch_pack_codes(const int8_t *M, int64_t rows, int64_t cols, int bits, void *packed, int *err_flag) {
    const int64_t ntiles = (cols + kTileCols - 1) / kTileCols;
    // (a launch holds fewer than 2^32 threads: so many row groups at a time)
    const int64_t band = (((int64_t)1 << 31) / (64 * ntiles)) * kDenseRows;
    uint32_t *to = static_cast<uint32_t *>(packed);
    for (int64_t r = 0; r < rows; r += band) {
        const int64_t n = rows - r < band ? rows - r : band;
        const int64_t total = row_groups(n) * ntiles * 64;
        const dim3 grid((unsigned)((total + 255) / 256));
        if (bits == 1)
            hipLaunchKernelGGL(k_pack_codes<1>, grid, dim3(256), 0, 0, M + r * cols, n, cols, ntiles, to, err_flag);
        else
            hipLaunchKernelGGL(k_pack_codes<2>, grid, dim3(256), 0, 0, M + r * cols, n, cols, ntiles, to, err_flag);
        if (hipError_t e = hipGetLastError()) return e;
        to += total * 2 * bits;
    }
    return hipSuccess;
}

namespace {

template <int BITS>
hipError_t launch_restore(const rsr_handle_s *h, int *err_flag) {
    static std::atomic<size_t> enabled[kMaxDevices];
    auto kern = k_restore_codes<BITS>;
    const size_t lds = ((size_t)h->cols + 1 + 3 * long_pieces((int)h->cols) + (h->cols + 31) / 32) * 4;
    static_assert((kMaxCols + 1 + 3 * long_pieces(kMaxCols) + (kMaxCols + 31) / 32) * 4 <= kLdsBytes,
                  "a word and a bit per column, three words per piece");
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, h->device, enabled)) return e;
    RestorePass p[2];
    for (int i = 0; i < 2; ++i) {
        const PassData &pd = h->pass[i < h->npass ? i : 0];
        p[i] = {pd.pi, pd.off};
    }
    const int64_t grid = h->code_groups < 65536 ? h->code_groups : 65536;
    const int64_t wide = h->cols > h->P ? h->cols : h->P;
    const int threads = wide <= 1024 ? 256 : wide <= 8192 ? 512 : 1024;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds, 0, p[0], p[1], h->npass, h->rows, (int)h->cols,
                       h->k, h->base, h->P, h->code_groups, reinterpret_cast<uint32_t *>(h->packed), err_flag);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_restore_codes(const rsr_handle_s *h, int *err_flag) {
    return h->code_bits == 1 ? launch_restore<1>(h, err_flag) : launch_restore<2>(h, err_flag);
}

namespace {

void set_sizes(const rsr_handle_s *h, int batch, Args *x) {
    x->codes = reinterpret_cast<const uint32_t *>(h->packed);
    x->ntiles = (int)((h->cols + kTileCols - 1) / kTileCols);
    x->ngroups = (int)h->code_groups;
    x->n_in = (int)h->cols;
    x->n_out = (int)h->rows;
    x->batch = batch;
    x->device = h->device;
    x->skip_zeros = h->kind != RSR_DENSE_TERNARY_P2;
}

hipError_t launch_any(const rsr_handle_s *h, int v_dtype, const Args &x) {
    if (h->code_bits == 1) return v_dtype == RSR_BF16 ? launch<uint16_t, 1>(x) : launch<float, 1>(x);
    return v_dtype == RSR_BF16 ? launch<uint16_t, 2>(x) : launch<float, 2>(x);
}

}  // namespace

hipError_t launch_packed(const rsr_handle_s *h, const void *v, int v_dtype, float scale, float *out, int batch,
                         int64_t ldv, int64_t ldo, hipStream_t stream, const LayerTable *layers) {
    Args x;
    set_sizes(h, batch, &x);
    x.v = v;
    x.ldv = ldv;
    x.ldo = ldo;
    x.out = out;
    x.scale = scale;
    x.stream = stream;
    if (layers)
        x.layers = *layers;
    else
        x.layers.n = 0;
    x.name = nullptr;
    return launch_any(h, v_dtype, x);
}

void packed_kernel_name(const rsr_handle_s *h, int v_dtype, int batch, char *buf, size_t len) {
    Args x = {};
    set_sizes(h, batch, &x);
    x.name = buf;
    x.name_len = len;
    (void)launch_any(h, v_dtype, x);
}

// Flat in the number of rows as long as every CU has at most one workgroup, linear in the column tiles
// that a wave goes through: least squares over measured products of up to 512 rows (5 % in the mean).
float packed_few_rows_us(const rsr_handle_s *h, bool wide, int batch) {
    const float tiles = (float)((h->cols + kTileCols - 1) / kTileCols);
    if (batch <= 4) return 3.2f + (wide ? 0.066f : 0.042f) * tiles;
    if (batch <= 16) return wide ? 3.4f + 0.25f * tiles : 2.9f + 0.078f * tiles;
    return wide ? 5.0f + 0.49f * tiles : 4.0f + 0.157f * tiles;
}

void packed_launch_shape(const rsr_handle_s *h, int v_dtype, int *workgroups, int *threads, int *lds_bytes) {
    const int ntiles = (int)((h->cols + kTileCols - 1) / kTileCols);
    const bool wide = v_dtype != RSR_BF16;
    if (table_vectors(ntiles, h->rows, 1, wide)) {
        const int64_t per = kTableWaves * (int64_t)table_groups_per_wave(h->code_groups, kCUs * 4 * 4);
        *workgroups = (int)((h->code_groups + per - 1) / per);
        *threads = kTableWaves * 64;
        *lds_bytes = kTableOneLds;
        return;
    }
    const int wk = few_wk(ntiles), waves = few_waves(wk);
    const int ngroups = (int)h->code_groups;
    const int G = !wide ? 0 : h->code_bits == 1 ? few_shape<float, 1, 1>(ntiles, ngroups, wk).G : few_shape<float, 2, 1>(ntiles, ngroups, wk).G;
    const int groups = G ? G : 1, rows = waves / wk * groups;
    const int wave_bytes = wide ? Few<float, 1>::wave_bytes : Few<uint16_t, 1>::wave_bytes;
    *workgroups = (int)((h->code_groups + rows - 1) / rows);
    *threads = waves * 64;
    *lds_bytes = waves * (wave_bytes + groups * 64 * 4);
}

}  // namespace rsr
