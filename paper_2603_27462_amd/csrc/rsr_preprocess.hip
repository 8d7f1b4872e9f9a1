// One-time preprocessing kernels of librsr (paper, System Overview, "Algorithm
// overview", and Kernels Implementation), one workgroup per block of k rows:
//   k_sort_columns  pattern codes of the block's columns, a stable counting sort of the
//                   columns by code, the group boundaries over all P codes, and what the
//                   host needs to choose the layout of the stream
//   k_build_stream  the compact stream the multiply kernel reads: 16-bit entries,
//                   zero-contribution group dropped, one tail flag per group, columns of a
//                   group in an order that suits the LDS banks, laid out for coalesced
//                   per-lane strips; and the small tables of the multiply kernel
// Everything between the matrix and these results stays in LDS.  Both are bound by the latency
// and the instruction count of their LDS steps, not by memory (4096 x 4096, fused, k = 8: 40 and
// 46 us, 15 of them for spreading the columns over the banks; as seven kernels with their
// intermediates in memory and the placement of whole runs 430 us).
#include <type_traits>

#include "rsr_internal.h"

namespace rsr {

namespace {

constexpr int kThreads = 256;  // workgroup size of the element-wise kernels

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive scan of one value per thread over the workgroup; *total gets the sum.
// wsum: one word of LDS per wave.  Contains two barriers.
__device__ __forceinline__ uint32_t wg_exclusive_scan(uint32_t x, uint32_t *wsum, int waves, uint32_t *total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_scan(x);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int i = 0; i < waves; ++i) {
        const uint32_t t = wsum[i];
        if (i < w) before += t;
        all += t;
    }
    __syncthreads();
    *total = all;
    return before + incl - x;
}

// ---- codes, sort, boundaries -----------------------------------------------------------------
typedef uint32_t u32_any __attribute__((aligned(1)));

// Digits of four entries (one per byte) for an encode mode, one per byte; bad != 0: an entry
// outside the alphabet.
__device__ __forceinline__ uint32_t digits4(uint32_t x, int mode, uint32_t *bad) {
    const uint32_t one = x & 0x01010101u, neg = (x >> 7) & 0x01010101u;
    if (mode == MODE_BINARY) {
        *bad |= x & 0xfefefefeu;
        return one;
    }
    // 0, 1 and 255: all bits alike but for the lowest, and that one set where the others are
    *bad |= ((x ^ (neg * 255u)) & 0xfefefefeu) | (neg & ~one);
    if (mode == MODE_POS) return one & ~neg;
    if (mode == MODE_NEG) return neg;
    return one + neg;
}

constexpr int kDigitBits = 5;  // most bits of the code one sorting step looks at
// Codes without columns whose boundaries the next column's thread writes by itself; of more in a row it is the
// wave (4096 x 4096 binary, k = 12, where the codes of a random matrix crowd together: 140 -> 36 us; where gaps are
// short nothing changes, while a search per code takes 45 -> 50 us for fused, k = 8).
constexpr int kShortGap = 8;

// Stable sort of the columns of each block by pattern code: digit by digit of the code's bits,
// every step a counting sort over at most 32 buckets.  A wave owns a contiguous run of positions and
// takes it 64 at a time; lanes with equal digits find each other with one ballot per bit, so
// their ranks keep the order.  WIDE: more columns than LDS holds as (code, column) pairs: only
// the columns are moved and the codes are looked up in `codes`, [nb][n].
// stats[0] = max over blocks of the columns outside group 0; stats[1] = the same plus one
// placeholder per empty group among codes 1..P-1; stats[2] = most non-empty groups among
// codes 1..P-1.  The caller zeroes stats.
template <int NT, bool WIDE>
__global__ __launch_bounds__(NT) void k_sort_columns(const int8_t *__restrict__ M, int64_t rows, int n, int k,
                                                     int base, int mode, int64_t nb, int64_t P, int bits,
                                                     uint16_t *__restrict__ codes, uint16_t *__restrict__ pi,
                                                     uint32_t *__restrict__ off, uint32_t *__restrict__ stats,
                                                     int *__restrict__ err_flag) {
    constexpr int W = NT / 64;
    typedef typename std::conditional<WIDE, uint16_t, uint32_t>::type Item;  // column, or code << 16 | column
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int npad = (n + 7) & ~7;
    Item *A = reinterpret_cast<Item *>(smem), *B = A + npad;
    uint32_t *cnt = reinterpret_cast<uint32_t *>(B + npad);  // [digit][wave]
    uint32_t *sums = cnt + (W << kDigitBits);                 // groups, columns outside group 0
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int seg = (n + NT - 1) / NT * 64;
    const int lo = min(n, w * seg), hi = min(n, lo + seg);
    const int steps = (bits + kDigitBits - 1) / kDigitBits, step_bits = (bits + steps - 1) / steps;

    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        uint16_t *cb = WIDE ? codes + b * n : nullptr;
        if (tid < 2) sums[tid] = 0;
        // codes of four columns at a time, two per register: c = c * base + digit, last row first
        uint32_t bad = 0;
        for (int j = 4 * tid; j < n; j += 4 * NT) {
            uint32_t even = 0, odd = 0;
            const int valid = (int)min((int64_t)k, rows - b * k);
            const int8_t *col = M + b * k * n + j;
            for (int r0 = (valid - 1) & ~3; r0 >= 0; r0 -= 4) {
                uint32_t x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[i] = 0;
                    if (r0 + i >= valid) continue;
                    const int8_t *at = col + (int64_t)(r0 + i) * n;
                    if (j + 4 <= n) {
                        x[i] = *reinterpret_cast<const u32_any *>(at);
                    } else {
                        for (int e = 0; j + e < n; ++e) x[i] |= (uint32_t)(uint8_t)at[e] << (8 * e);
                    }
                }
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const uint32_t d = digits4(x[i], mode, &bad);
                    even = even * base + (d & 0x00ff00ffu);
                    odd = odd * base + ((d >> 8) & 0x00ff00ffu);
                }
            }
            const uint32_t c[4] = {even & 0xffffu, odd & 0xffffu, even >> 16, odd >> 16};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < n) {
                    if (WIDE) {
                        cb[j + e] = (uint16_t)c[e];
                        A[j + e] = (Item)(j + e);
                    } else {
                        A[j + e] = (Item)(c[e] << 16 | (uint32_t)(j + e));
                    }
                }
        }
        if (bad) atomicOr(err_flag, 1);
        auto code_of = [&](Item x) -> uint32_t { return WIDE ? (uint32_t)cb[x] : (uint32_t)x >> 16; };
        for (int shift = 0; shift < bits; shift += step_bits) {
            const int nbits = min(step_bits, bits - shift);
            for (int i = tid; i < (W << nbits); i += NT) cnt[i] = 0;
            __syncthreads();
            // lanes of the wave with the same digit
            auto peers = [&](uint32_t digit, bool valid) {
                uint64_t m = __ballot(valid);
                for (int i = 0; i < nbits; ++i) {
                    const bool set = (digit >> i) & 1u;
                    const uint64_t ones = __ballot(set);
                    m &= set ? ones : ~ones;
                }
                return m;
            };
            const uint32_t mask = (1u << nbits) - 1u;
            for (int t = lo + lane; t < hi; t += 64)  // count
                atomicAdd(&cnt[((code_of(A[t]) >> shift) & mask) * W + w], 1u);
            __syncthreads();
            if (w == 0) {  // exclusive scan over [digit][wave]
                const int each = ((W << nbits) + 63) / 64;
                uint32_t sum = 0;
                for (int i = 0; i < each; ++i)
                    if (lane * each + i < (W << nbits)) sum += cnt[lane * each + i];
                uint32_t run = wave_inclusive_scan(sum) - sum;
                for (int i = 0; i < each; ++i)
                    if (lane * each + i < (W << nbits)) {
                        const uint32_t x = cnt[lane * each + i];
                        cnt[lane * each + i] = run;
                        run += x;
                    }
            }
            __syncthreads();
            for (int t0 = lo; t0 < hi; t0 += 64) {  // stable placement
                const int t = t0 + lane;
                const bool valid = t < hi;
                const Item x = valid ? A[t] : Item(0);
                const uint32_t digit = valid ? (code_of(x) >> shift) & mask : 0u;
                const uint64_t m = peers(digit, valid);
                const uint32_t rank =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (valid) {
                    const uint32_t first = cnt[digit * W + w];
                    B[first + rank] = x;
                    // the wave's LDS operations execute in order: everybody has read it, and the next
                    // 64 positions read it after this
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    if (rank == 0) cnt[digit * W + w] = first + (uint32_t)__popcll(m);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            Item *tmp = A; A = B; B = tmp;
        }
        // A is pi_b.  Group boundaries: off[c] = first position whose code >= c.
        uint16_t *pib = pi + b * n;
        uint32_t *ob = off + b * (P + 1);
        uint32_t groups = 0;
        for (int t0 = 64 * w; t0 < n; t0 += NT) {
            const int t = t0 + lane;
            int cur = 0, prev = 0;
            if (t < n) {
                const Item x = A[t];
                pib[t] = (uint16_t)x;
                cur = (int)code_of(x);
                prev = t ? (int)code_of(A[t - 1]) : -1;
                for (int c = prev + 1; c <= min(cur, prev + kShortGap); ++c) ob[c] = (uint32_t)t;
                if (cur != prev && cur > 0) {
                    ++groups;
                    if (prev <= 0) sums[1] = (uint32_t)(n - t);
                }
            }
            // many empty groups in a row: the wave writes them together
            for (uint64_t wide = __ballot(cur - prev > kShortGap); wide; wide &= wide - 1) {
                const int l = __builtin_ctzll(wide);
                const int to = __builtin_amdgcn_readlane(cur, l);
                for (int c = __builtin_amdgcn_readlane(prev, l) + 1 + kShortGap + lane; c <= to; c += 64)
                    ob[c] = (uint32_t)(t0 + l);
            }
        }
        for (int c = (int)code_of(A[n - 1]) + 1 + tid; c <= (int)P; c += NT) ob[c] = (uint32_t)n;
        if (groups) atomicAdd(&sums[0], groups);
        __syncthreads();
        if (tid < 3) {  // (one thread for all three took three times the latency, 4 us of a block's 45)
            const uint32_t some = sums[0], real = sums[1];
            const uint32_t mine = tid == 0 ? real : tid == 1 ? real + (uint32_t)(P - 1) - some : some;
            if (mine > __hip_atomic_load(&stats[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&stats[tid], mine);
        }
        __syncthreads();
    }
}

// ---- the stream of the multiply kernel -------------------------------------------------------
// Slabs wave w owns when S slabs are dealt to W waves, the longer shares first.
__device__ __forceinline__ void wave_share(int S, int W, int w, int *first, int *count) {
    const int per = S / W, rem = S - per * W;
    *first = w * per + min(w, rem);
    *count = per + (w < rem ? 1 : 0);
}

// Sign of digit r of code c as a 2-bit two's complement field (00: 0, 01: +1, 11: -1).
template <int BASE>
__device__ __forceinline__ uint32_t sign2_of(uint32_t c, int r) {
    for (int i = 0; i < r; ++i) c /= (uint32_t)BASE;
    const uint32_t d = c % (uint32_t)BASE;
    return d == 0 ? 0u : d == 1 ? 1u : 3u;
}
template <int BASE>
__device__ __forceinline__ int sign_of(uint32_t c, int r) {
    const uint32_t s = sign2_of<BASE>(c, r);
    return s == 3u ? -1 : (int)s;
}

// Reorders the stream inside its groups so that the LDS gathers of the multiply kernel collide
// less.  Gather instruction i of a wave reads entry i of all 64 strips of the wave; the LDS serves
// the two half-waves side by side and needs one cycle per distinct dword that falls on the same
// of its 32 banks.  The order of the columns inside a group is free for the kernel (sums commute
// up to rounding; the canonical pi is not touched), so neighbours of one group inside a strip change places
// where that lowers the loads of their banks, the other entries of the two slots of the half-wave being what they
// are -- counted for both vector types the kernel serves: bank
// (col / 2) mod 32 for 2-byte elements and col mod 32 for 4-byte elements.  One wave per wave of the
// multiply kernel, or per two of them if their strips have at most 16 entries: lane = (wave, half-wave, slot).
// A sweep looks at the even or at the odd pairs of slots, in turn, so that columns move along
// their group; neighbouring lanes are a pair, so an element's partner and its share of the gain come through DPP, a lane
// needs the loads of its own slot only, and writes are rare.  Four strips at a time, which do not see
// each other's changes.  Bound by vector instructions, 30 per strip and sweep; one lane placing up to four
// columns at a time took 220 (4096 x 4096, fused, k = 8: the whole kernel 112 -> 46 us; the product is the same,
// 7.35 -> 7.31 us for the metric workload, and 3 % slower with the streams left as sorted.  Four sweeps give another
// 0.5 % and cost 17 us).  Strips of more than 32 entries are left as they are.
constexpr int kSpreadSweeps = 2;
constexpr int kSpreadTogether = 4;                     // strips
constexpr int kSpreadRow = 2 * 32 + 4;                 // loads of a slot: a byte per bank of either kind; padding
constexpr int kSpreadWaveBytes = 64 * kSpreadRow;

// x of the other lane of the pair (2 i, 2 i + 1)
__device__ __forceinline__ int pair_lane(int x) {
    return __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, true);  // quad_perm: 1, 0, 3, 2
}

// part: of the stream, 64 strips of epl entries; slots: 16 or 32 lanes per half-wave of the part; loads: of the wave.
__device__ __forceinline__ void spread_banks(uint16_t *part, int epl, int slots, uint8_t *loads) {
    const int lane = threadIdx.x & 63, half = slots == 16 ? (lane >> 4) & 1 : lane >> 5, own = lane & (slots - 1);
    uint32_t *words = reinterpret_cast<uint32_t *>(loads + lane * kSpreadRow);
    for (int i = 0; i < kSpreadRow / 4; ++i) words[i] = 0;
    if (own < epl) {
        const uint16_t *at = part + 32 * half * epl + own;
#pragma unroll 8
        for (int l = 0; l < 32; ++l) {
            const uint32_t x = at[l * epl] >> 1;
            atomicAdd(&words[(x >> 3) & 7], 1u << (8 * ((x >> 1) & 3)));
            atomicAdd(&words[8 + ((x >> 2) & 7)], 1u << (8 * (x & 3)));
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int sweep = 0; sweep < kSpreadSweeps; ++sweep) {
        const int odd = sweep & 1, upper = lane & 1, slot = own + odd;  // pairs (0, 1), (2, 3), .. or (1, 2), ..
        const bool pair = slot - upper + 1 < epl;
        uint8_t *load2 = loads + (pair ? lane + odd : lane) * kSpreadRow, *load4 = load2 + 32;
        words = reinterpret_cast<uint32_t *>(load2);
        uint16_t *first = part + 32 * half * epl + (pair ? slot : 0);
        for (int l0 = 0; l0 < 32; l0 += kSpreadTogether) {
            uint16_t *at = first + l0 * epl;
            uint32_t entry[kSpreadTogether], other[kSpreadTogether];
            int gain[kSpreadTogether];
#pragma unroll
            for (int l = 0; l < kSpreadTogether; ++l) entry[l] = at[l * epl];
#pragma unroll
            for (int l = 0; l < kSpreadTogether; ++l) {
                other[l] = (uint32_t)pair_lane((int)entry[l]);
                const uint32_t b2 = (entry[l] >> 2) & 31, b4 = (entry[l] >> 1) & 31;
                const uint32_t o2 = (other[l] >> 2) & 31, o4 = (other[l] >> 1) & 31;
                // what changes in this slot: the partner's column joins its banks, this one has left
                gain[l] = (b2 == o2 ? 0 : (int)load2[o2] - (int)load2[b2] + 1) +
                          (b4 == o4 ? 0 : (int)load4[o4] - (int)load4[b4] + 1);
            }
#pragma unroll
            for (int l = 0; l < kSpreadTogether; ++l) {
                // (columns may pass each other unless a group ends between them)
                const bool open = pair && !((upper ? other[l] : entry[l]) & 1u);
                if (open && gain[l] + pair_lane(gain[l]) < 0) {
                    const uint32_t x = entry[l] >> 1, y = other[l] >> 1;
                    atomicSub(&words[(x >> 3) & 7], 1u << (8 * ((x >> 1) & 3)));
                    atomicAdd(&words[(y >> 3) & 7], 1u << (8 * ((y >> 1) & 3)));
                    atomicSub(&words[8 + ((x >> 2) & 7)], 1u << (8 * (x & 3)));
                    atomicAdd(&words[8 + ((y >> 2) & 7)], 1u << (8 * (y & 3)));
                    at[l * epl] = (uint16_t)((other[l] & ~1u) | (entry[l] & 1u));
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

struct StreamArgs {
    const uint16_t *pi;
    const uint32_t *off;
    int64_t block0;  // of workgroup 0
    int64_t nb, P, slots;
    int n, S, W, k, enc, by_rank, fw, spread;  // spread: the strips are short enough to be spread
    uint16_t *entries, *start;
    void *sgn;
    uint32_t *gword, *gcount;
    int *err_flag;
};

constexpr int kLongGroup = 64;  // groups from here on are copied by the whole workgroup

// LDS of k_build_stream, byte offsets.
struct StreamLds {
    int gcode, start, loads, longs, wsum, holes, total;
};
inline __host__ __device__ StreamLds stream_lds(int n, int64_t P, int S, int W, int64_t slots, int by_rank,
                                              int spread) {
    StreamLds o;
    o.gcode = S * kSlab * 2;                                              // the stream comes first
    o.start = o.gcode + (by_rank ? (int)((slots * 2 + 15) & ~(int64_t)15) : 0);
    o.loads = o.start + ((W * 64 + 1) * 2 + 15) / 16 * 16;
    o.longs = o.loads + (spread ? W * kSpreadWaveBytes : 0);
    o.wsum = o.longs + (n / kLongGroup + 2) * 12;
    o.holes = o.wsum + 16 * 4;
    o.total = o.holes + (int)(P / 64 + 16) * 4;
    return o;
}

// Stream of block b (L = 512 S entries): for code c = 1..P-1 in order, the columns of group c
// (entry = column<<1, last one |1).  Indexed by code: an empty group contributes one placeholder
// entry (zero slot = index n, tail bit set), so that every code owns exactly one tail.  Indexed by
// rank: empty groups contribute nothing and gcode[rank] records the code of every non-empty group
// (rank 1.., gcode[0] = 0), gcount[b] their number.  Filler entries (zero slot, no tail) up to L.
// Then the columns are spread over the banks, every strip gets the slot of the first tail at or
// after its start (1 + tails before it), the entries go to their slabs (see PassData), and the signs
// of the strips and the weights of the slots follow from the codes.
template <int BASE>
__global__ __launch_bounds__(1024) void k_build_stream(const StreamArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const StreamLds at = stream_lds(a.n, a.P, a.S, a.W, a.slots, a.by_rank, a.spread);
    uint16_t *stream = reinterpret_cast<uint16_t *>(smem);
    uint16_t *gcode = reinterpret_cast<uint16_t *>(smem + at.gcode);
    uint16_t *first_slot = reinterpret_cast<uint16_t *>(smem + at.start);
    uint32_t *longs = reinterpret_cast<uint32_t *>(smem + at.longs);  // count, -, -, then {from, to, length}
    uint32_t *wsum = reinterpret_cast<uint32_t *>(smem + at.wsum);
    uint32_t *holes = reinterpret_cast<uint32_t *>(smem + at.holes);  // [round][wave]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, NT = blockDim.x, waves = NT >> 6;
    const int L = a.S * kSlab, strips = a.W * 64;
    const uint16_t zero_entry = (uint16_t)(a.n << 1);
    const int64_t b = a.block0 + blockIdx.x;
    const uint16_t *pib = a.pi + b * a.n;
    const uint32_t *ob = a.off + b * (a.P + 1);
    const uint32_t off1 = ob[1];
    if (tid == 0) longs[0] = 0;

    // ---- logical order: rounds of NT codes; empty groups are counted per (round, wave) first ------
    const int rounds = (int)((a.P - 1 + NT - 1) / NT);
#pragma unroll 8
    for (int r = 0; r < rounds; ++r) {
        const int64_t c = 1 + (int64_t)r * NT + tid;
        const uint64_t none = __ballot(c < a.P && ob[min(c, a.P - 1)] == ob[min(c + 1, a.P)]);
        if (lane == 0) holes[r * waves + w] = (uint32_t)__popcll(none);
    }
    __syncthreads();
    uint32_t empties = 0;
    for (int i0 = 0; i0 < rounds * waves; i0 += NT) {
        const uint32_t x = i0 + tid < rounds * waves ? holes[i0 + tid] : 0u;
        uint32_t sum;
        const uint32_t ex = empties + wg_exclusive_scan(x, wsum, waves, &sum);
        if (i0 + tid < rounds * waves) holes[i0 + tid] = ex;
        empties += sum;
    }
    __syncthreads();
    // (two rounds ahead the boundaries, one round ahead the first four columns of the groups are on their way:
    // 4096 x 4096 fused, k = 8: 55 -> 52 us)
    auto bounds = [&](int r, uint32_t *from, uint32_t *to) {
        const int64_t c = 1 + (int64_t)r * NT + tid;
        *from = ob[min(c, a.P - 1)];
        *to = ob[min(c + 1, a.P)];
    };
    auto columns = [&](uint32_t from, uint32_t to, uint32_t (&col)[4]) {
        const uint32_t last = min(max(to, from + 1) - 1, (uint32_t)a.n - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) col[i] = pib[min(from + i, last)];
    };
    uint32_t s, e, s1, e1, col[4];
    bounds(0, &s, &e);
    bounds(1, &s1, &e1);
    columns(s, e, col);
    for (int r = 0; r < rounds; ++r) {
        const int64_t c = 1 + (int64_t)r * NT + tid;
        uint32_t s2, e2, next[4];
        bounds(r + 2, &s2, &e2);
        columns(s1, e1, next);
        const uint64_t none = __ballot(c < a.P && s == e);
        const uint32_t eb = holes[r * waves + w] +  // empty groups before code c
            __builtin_amdgcn_mbcnt_hi((uint32_t)(none >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)none, 0u));
        const uint32_t to = s - off1 + (a.by_rank ? 0u : eb);
        if (c >= a.P) {
        } else if (s == e) {
            if (!a.by_rank) stream[to] = zero_entry | 1;
        } else {
            if (a.by_rank) gcode[c - eb] = (uint16_t)c;
            if (e - s >= kLongGroup) {
                uint32_t *l = longs + 3 + 3 * atomicAdd(&longs[0], 1u);
                l[0] = s; l[1] = to; l[2] = e - s;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (s + i < e) stream[to + i] = (uint16_t)(col[i] << 1 | (s + i + 1 == e ? 1u : 0u));
                for (uint32_t t = s + 4; t < e; t += 4) {  // four columns in flight
                    uint32_t more[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) more[i] = pib[min(t + i, e - 1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (t + i < e) stream[to + (t + i - s)] = (uint16_t)(more[i] << 1 | (t + i + 1 == e ? 1u : 0u));
                }
            }
        }
        s = s1; e = e1; s1 = s2; e1 = e2;
#pragma unroll
        for (int i = 0; i < 4; ++i) col[i] = next[i];
    }
    const int len = (int)(a.n - off1) + (a.by_rank ? 0 : (int)empties);
    for (int t = len + tid; t < L; t += NT) stream[t] = zero_entry;
    const int64_t count = a.P - 1 - empties;
    if (a.by_rank && tid == 0) { a.gcount[b] = (uint32_t)count; gcode[0] = 0; }
    __syncthreads();
    for (uint32_t i = 0; i < longs[0]; ++i) {
        const uint32_t s = longs[3 + 3 * i], to = longs[4 + 3 * i], m = longs[5 + 3 * i];
        for (uint32_t t = tid; t < m; t += NT) stream[to + t] = (uint16_t)((pib[s + t] << 1) | (t + 1 == m ? 1 : 0));
    }
    __syncthreads();

    // ---- banks ---------------------------------------------------------------------------------
    int first = 0, slabs = 0;  // of this wave
    if (w < a.W) wave_share(a.S, a.W, w, &first, &slabs);
    const int epl = 8 * slabs;
    if (a.spread) {
        // (the first wave's strips are the longest)
        const bool two = 8 * ((a.S + a.W - 1) / a.W) <= 16;
        const int v = two ? 2 * w + (lane >> 5) : w;
        int from, count;
        wave_share(a.S, a.W, min(v, a.W - 1), &from, &count);
        if (v >= a.W) count = 0;
        if (two ? 2 * w < a.W : w < a.W && 8 * count <= 32)
            spread_banks(stream + from * kSlab, 8 * count, two ? 16 : 32, smem + at.loads + w * kSpreadWaveBytes);
    }
    __syncthreads();

    // ---- strips --------------------------------------------------------------------------------
    const uint4 *strip = reinterpret_cast<const uint4 *>(stream + first * kSlab + lane * epl);
    uint32_t tails = 0;
    for (int h = 0; h < slabs; ++h) {
        const uint4 d = strip[h];
        tails += __popc(d.x & 0x00010001u) + __popc(d.y & 0x00010001u) + __popc(d.z & 0x00010001u) +
                 __popc(d.w & 0x00010001u);
    }
    uint32_t total;
    const uint32_t slot = 1 + wg_exclusive_scan(tails, wsum, waves, &total);
    if (w < a.W) {
        a.start[(b * a.W + w) * 64 + lane] = (uint16_t)slot;
        first_slot[w * 64 + lane] = (uint16_t)slot;
        uint4 *to = reinterpret_cast<uint4 *>(a.entries) + (b * a.S + first) * 64 + lane;
        for (int h = 0; h < slabs; ++h) {
            uint4 d = strip[h];
            if (a.enc == kEncSmall) {
                d.x = ((d.x & 0x00010001u) << 15) | (d.x & 0xfffefffeu);
                d.y = ((d.y & 0x00010001u) << 15) | (d.y & 0xfffefffeu);
                d.z = ((d.z & 0x00010001u) << 15) | (d.z & 0xfffefffeu);
                d.w = ((d.w & 0x00010001u) << 15) | (d.w & 0xfffefffeu);
            }
            to[h * 64] = d;
        }
    }
    // every block holds exactly P - 1 (by code) or `count` (by rank) tails
    if (tid == 0 && (int64_t)total != (a.by_rank ? count : a.P - 1)) atomicOr(a.err_flag, 2);
    __syncthreads();

    // ---- signs of the strips: digits of the first group closed at or after the start of the next
    // strip, if there is one -----------------------------------------------------------------------
    if (!a.by_rank) {
        // word (b, r, l): row r at bits 2w for strip (w, l); 16-bit words when W <= 8
        for (int i = tid; i < a.k * 64; i += NT) {
            const int r = i >> 6, l = i & 63;
            uint32_t word = 0;
            for (int v = 0; v < a.W; ++v) {
                const int g = v * 64 + l + 1;
                const uint32_t c = g < strips ? first_slot[g] : 0xffffffffu;
                if (c < a.P) word |= sign2_of<BASE>(c, r) << (2 * v);
            }
            const int64_t to = (b * a.k) * 64 + i;
            if (a.W <= 8)
                static_cast<uint16_t *>(a.sgn)[to] = (uint16_t)word;
            else
                static_cast<uint32_t *>(a.sgn)[to] = word;
        }
        return;
    }
    // word (b, w, l): strip (w, l), row r at bits 2r
    for (int g = tid; g < strips; g += NT) {
        uint32_t word = 0;
        const uint32_t next = g + 1 < strips ? first_slot[g + 1] : 0xffffffffu;
        if (next <= count) {
            const uint32_t c = gcode[next];
            for (int r = 0; r < a.k; ++r) word |= sign2_of<BASE>(c, r) << (2 * r);
        }
        static_cast<uint32_t *>(a.sgn)[b * strips + g] = word;
    }
    // weights of the slots: field r (fw bits, two's complement) = sgn_r(code of rank s) -
    // sgn_r(code of rank s+1), the second term 0 behind the last group; 0 for s = 0 and behind it
    for (int64_t s = tid; s < a.slots; s += NT) {
        uint32_t word = 0;
        if (s >= 1 && s <= count) {
            const uint32_t c = gcode[s], next = s < count ? gcode[s + 1] : 0u;
            for (int r = 0; r < a.k; ++r) {
                const int wgt = sign_of<BASE>(c, r) - sign_of<BASE>(next, r);
                word |= ((uint32_t)wgt & ((1u << a.fw) - 1u)) << (a.fw * r);
            }
        }
        a.gword[b * a.slots + s] = word;
    }
}

// Plain fill (used instead of a memset node so that callers may capture the sequence).
__global__ __launch_bounds__(kThreads) void k_fill_u32(uint32_t *__restrict__ p, uint32_t value,
                                                       int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < count) p[i] = value;
}

// T[j][i] = M[i][j] through 64 x 64 tiles in LDS (coalesced on both sides).
__global__ __launch_bounds__(256) void k_transpose_i8(const int8_t *__restrict__ M, int64_t rows,
                                                      int64_t cols, int8_t *__restrict__ T) {
    __shared__ int8_t tile[64][65];
    const int64_t tiles_x = (cols + 63) / 64;
    const int64_t ti = blockIdx.x / tiles_x, tj = blockIdx.x % tiles_x;
    const int x = threadIdx.x & 63, y0 = threadIdx.x >> 6;
    for (int y = y0; y < 64; y += 4) {
        const int64_t i = ti * 64 + y, j = tj * 64 + x;
        tile[y][x] = (i < rows && j < cols) ? M[i * cols + j] : (int8_t)0;
    }
    __syncthreads();
    for (int y = y0; y < 64; y += 4) {
        const int64_t j = tj * 64 + y, i = ti * 64 + x;
        if (i < rows && j < cols) T[j * rows + i] = tile[x][y];
    }
}

// Columns a block can have if it is sorted as (code, column) pairs, and from which on its LDS is more than half a CU's.
constexpr int kPairColumns = 18 * 1024;
constexpr int kAloneColumns = 10 * 1024;

template <int NT, bool WIDE>
hipError_t launch_sort(const int8_t *M, int64_t rows, int64_t cols, int k, int base, int mode, int64_t P,
                       uint16_t *codes, uint16_t *pi, uint32_t *off, uint32_t *stats, int *err_flag) {
    static std::atomic<size_t> enabled[kMaxDevices];
    const int64_t nb = (rows + k - 1) / k;
    const int64_t npad = (cols + 7) & ~(int64_t)7;
    const size_t lds = (size_t)npad * (WIDE ? 4 : 8) + (((NT / 64) << kDigitBits) + 2) * 4;
    int bits = 1, device = 0;
    while (((int64_t)1 << bits) < P) ++bits;
    if (hipError_t e = hipGetDevice(&device)) return e;
    auto kern = k_sort_columns<NT, WIDE>;
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, device, enabled)) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(nb < 65536 ? nb : 65536)), dim3(NT), lds, 0, M, rows, (int)cols, k, base,
                       mode, nb, P, bits, codes, pi, off, stats, err_flag);
    return hipGetLastError();
}

// A launch holds fewer than 2^32 threads; the runtime takes a larger grid without an error and runs
// a part of it.  More blocks than kLaunchBlocks (of up to 1024 threads) take several launches.
constexpr int64_t kLaunchBlocks = (int64_t)1 << 21;

template <int BASE>
hipError_t launch_stream(StreamArgs a, int threads, size_t lds) {
    static std::atomic<size_t> enabled[kMaxDevices];
    int device = 0;
    if (hipError_t e = hipGetDevice(&device)) return e;
    auto kern = k_build_stream<BASE>;
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, device, enabled)) return e;
    for (a.block0 = 0; a.block0 < a.nb; a.block0 += kLaunchBlocks) {
        const int64_t left = a.nb - a.block0;
        hipLaunchKernelGGL(kern, dim3((unsigned)(left < kLaunchBlocks ? left : kLaunchBlocks)), dim3(threads), lds, 0,
                           a);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

}  // namespace

bool sort_needs_codes(int64_t cols) { return cols > kPairColumns; }

hipError_t launch_sort_columns(const int8_t *M, int64_t rows, int64_t cols, int k, int base, int mode, int64_t P,
                               uint16_t *codes, uint16_t *pi, uint32_t *off, uint32_t *stats, int *err_flag) {
    if (sort_needs_codes(cols))
        return launch_sort<512, true>(M, rows, cols, k, base, mode, P, codes, pi, off, stats, err_flag);
    // Workgroups of 1024 threads do not share a CU (512 blocks of 4096 columns sort 2.3 times slower with them), so they
    // are for blocks that have one to themselves: because of their LDS (4096 x 14336 fused k = 8 144 -> 114 us, 1500 x
    // 18000 k = 4 110 -> 85), or because there are no more blocks than CUs (1500 x 10200 55 -> 46, 500 x 8000 30 -> 25,
    // 2040 x 3000 28 -> 25; 2000 x 2000 the same, 500 x 600 9 -> 11).
    if (cols > kAloneColumns || (cols > 2560 && (rows + k - 1) / k <= 256))
        return launch_sort<1024, false>(M, rows, cols, k, base, mode, P, codes, pi, off, stats, err_flag);
    return cols > 512 ? launch_sort<512, false>(M, rows, cols, k, base, mode, P, codes, pi, off, stats, err_flag)
                      : launch_sort<256, false>(M, rows, cols, k, base, mode, P, codes, pi, off, stats, err_flag);
}

hipError_t launch_transpose(const int8_t *M, int64_t rows, int64_t cols, int8_t *T) {
    const int64_t tiles = ((rows + 63) / 64) * ((cols + 63) / 64);
    hipLaunchKernelGGL(k_transpose_i8, dim3((unsigned)tiles), dim3(256), 0, 0, M, rows, cols, T);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t value, int64_t count) {
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((count + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, 0, p, value, count);
    return hipGetLastError();
}

hipError_t launch_pack_pass(const rsr_handle_s *h, int pass, int *err_flag) {
    const PassData &pd = h->pass[pass];
    StreamArgs a;
    a.pi = pd.pi;
    a.off = pd.off;
    a.nb = h->nb;
    a.P = h->P;
    a.slots = h->slots;
    a.n = (int)h->cols;
    a.S = (int)pd.S;
    a.W = h->W;
    a.k = h->k;
    a.enc = h->enc;
    a.by_rank = h->by_rank;
    a.fw = gword_field_bits(h->base);
    a.spread = a.S / a.W <= 4;
    a.entries = pd.entries;
    a.start = pd.start;
    a.sgn = pd.sgn;
    a.gword = pd.gword;
    a.gcount = pd.gcount;
    a.err_flag = err_flag;
    // (what the multiply kernel's LDS holds, 4 (columns + slots) bytes and more, bounds this to 158.1 KiB: 32302 columns, E by
    // rank)
    const StreamLds lds = stream_lds(a.n, a.P, a.S, a.W, a.slots, a.by_rank, a.spread);
    if (lds.total > kLdsBytes) return hipErrorInvalidValue;
    const int threads = a.W * 64 > 512 ? a.W * 64 : 512;
    return h->base == 2 ? launch_stream<2>(a, threads, (size_t)lds.total)
                        : launch_stream<3>(a, threads, (size_t)lds.total);
}

}  // namespace rsr
