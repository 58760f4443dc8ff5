// fp32 contractions on the bf16 matrix cores at fp32 accuracy: what the score pass (sfb_forward_split.hip) and the
// reconstruction (sfb_reconstruct_split.hip) share.
//
// gfx950 multiplies bf16 sixteen times faster than fp32 on its matrix cores.  Every fp32 operand is split EXACTLY into
// three bf16 terms, x = h + m + l (h = bf16(x), m = bf16(x - h), l = bf16(x - h - m): 3 x 8 significand bits cover
// fp32's 24, and both differences are exact in fp32; below 2^-109 l runs out of bf16's exponents: sums of operands of 2^-118
// are off by 3e-7, of 2^-120 by 1e-6, of 2^-125 by 3e-5, where the fp32 instruction keeps 1e-7), and a product a * b is taken as the six term products whose
// weight is at least 2^-16 of the leading one:
//     a_h b_h  +  (a_h b_m + a_m b_h)  +  (a_h b_l + a_l b_h + a_m b_m).
// Each is exact in the fp32 accumulator's input (8 x 8 bits).  What is left out (a_m b_l + a_l b_m + a_l b_l) is below
// 2^-24 of |a b| and unbiased, the size of ONE fp32 rounding of one product; a matrix instruction adds 16 products
// per rounding where the fp32 one adds two, so a sum of K products is rounded 6 K / 16 times instead of K / 2 times.
//
// A workgroup is eight wavefronts, two per SIMD: four take k 0..15 of every chunk of 32 k, four k 16..31, each group
// as 2 x 2 over the tile.  Everything a chunk needs is spread over the chunks before it, so that a wavefront never
// stops between its matrix instructions: while it multiplies chunk c from registers, it reads its fragments of chunk
// c + 1 from LDS, splits its share of chunk c + 2 into the other LDS buffer (the vector instructions go into the
// shadow of the matrix instructions, about four each: measured free up to four, 5 % at six), and requests its share
// of chunk c + 4 (c + 6 in the small tiles, which have registers left and are the ones that wait for memory).  One barrier per chunk, two LDS buffers of three planes [row][32 k] (rows of the A tile, then B).
#pragma once
#include <type_traits>

#include "sfb_device.h"

namespace sfb {

typedef __bf16 sp_bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t sp_u32x4 __attribute__((ext_vector_type(4)));
typedef float sp_f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // a 16-byte access at any 4-byte address

constexpr int kSpChunk = 32;       // k per chunk
constexpr int kSplitThreads = 512;

// every wavefront of the workgroup; this wavefront's LDS writes are visible and its LDS reads done
__device__ __forceinline__ void split_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ f32x16 split_mfma(sp_u32x4 a, sp_u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sp_bf16x8, a), __builtin_bit_cast(sp_bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 split_mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

template <int FIRST, int LAST, class F>
__device__ __forceinline__ void split_for(F f) {
    if constexpr (FIRST < LAST) {
        f(std::integral_constant<int, FIRST>{});
        split_for<FIRST + 1, LAST>(f);
    }
}

// The exact split of two pairs of fp32 values (a0 a1, b0 b1) in four parts of four to six vector instructions, the two
// pairs side by side so that neighbours do not depend on each other: a wavefront alone on its SIMD then needs no more
// than a matrix instruction's 32 cycles for a part (one pair at a time: about 45, every instruction waiting for the last)
struct SplitQuad {
    float a0, a1, b0, b1, ta, tb, ua, ub;
    uint32_t ha, hb, ma, mb, la, lb;
    template <int P>
    __device__ __forceinline__ void part(float xa0, float xa1, float xb0, float xb1) {
        if constexpr (P == 0) {
            ha = cvt_pk_bf16(xa0, xa1);
            hb = cvt_pk_bf16(xb0, xb1);
            ta = __uint_as_float(ha << 16); tb = __uint_as_float(hb << 16);
            ua = __uint_as_float(ha & 0xffff0000u); ub = __uint_as_float(hb & 0xffff0000u);
        } else if constexpr (P == 1) {
            a0 = xa0 - ta; b0 = xb0 - tb; a1 = xa1 - ua; b1 = xb1 - ub;
            ma = cvt_pk_bf16(a0, a1);
            mb = cvt_pk_bf16(b0, b1);
        } else if constexpr (P == 2) {
            ta = __uint_as_float(ma << 16); tb = __uint_as_float(mb << 16);
            ua = __uint_as_float(ma & 0xffff0000u); ub = __uint_as_float(mb & 0xffff0000u);
            a0 -= ta; b0 -= tb;
        } else {
            a1 -= ua; b1 -= ub;
            la = cvt_pk_bf16(a0, a1);
            lb = cvt_pk_bf16(b0, b1);
        }
    }
};

// The multiplying side.  Tile (WM MT x 32) x (WN NT x 32), four wavefronts as WM x WN, each MT x NT blocks of 32 x 32.
// PITCH: bytes from one LDS row to the next; SWZ: 16-byte item c of row r sits at c ^ f(r) instead of c.
// APART: the five smaller term products have sums of their own, so that the leading ones' running sum is rounded once for
// every sixteen k instead of six times (error of a sum of 4096 products 1.4e-7 instead of 2.5e-7, of 512 1.3e-7 instead of
// 2.4e-7; the fp32 instruction 5.8e-7 and 2.9e-7): for callers who chose these products for their accuracy (sfb_set_plan).
// No time of its own, but 64 x 64 blocks of a wavefront have no registers left for it.
template <int MT, int NT, int PITCH, bool SWZ, bool APART, int WM = 2>
struct SplitTile {
    static constexpr int WN = 4 / WM, BM = 32 * WM * MT, BN = 32 * WN * NT, ROWS = BM + BN;
    static constexpr int PLANE = ROWS * PITCH, BYTES = 3 * PLANE;      // one group's buffer
    static constexpr int XCHG = 8 * MT * NT * 8 * 64 * 4;               // exchange of partial sums at the end
    static constexpr int LDS = 2 * BYTES > XCHG ? 2 * BYTES : XCHG;

    // Among eight consecutive rows any one item falls into eight different 16-byte bank groups of 128 bytes, among
    // sixteen into sixteen of 256; of four consecutive rows (from a multiple of four) half a row each, too.
    static __device__ __forceinline__ int swz(int r) { return SWZ ? (((r >> 2) & 1) | ((((r >> 1) ^ (r >> 3)) & 1) << 1)) : 0; }

    struct Frag { sp_u32x4 a[3][MT], b[3][NT]; };
    static_assert(!APART || MT * NT <= 2, "registers");
    f32x16 acc[MT][NT], rest[APART ? MT : 1][APART ? NT : 1];
    int a_base, b_base;            // byte offset of this lane's item in the A and the B part

    __device__ __forceinline__ void init(int wave, int lane) {
        const int wm = (wave & 3) / WN, wn = wave % WN, l32 = lane & 31, half = lane >> 5;
        // every row this lane reads is l32 modulo 32
        const int item = 16 * ((2 * (wave >> 2) + half) ^ swz(l32));
        a_base = (wm * 32 * MT + l32) * PITCH + item;
        b_base = (BM + wn * 32 * NT + l32) * PITCH + item;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    acc[i][j][e] = 0.f;
                    if constexpr (APART) rest[i][j][e] = 0.f;
                }
    }
    // fragment read Q of the 3 (MT + NT): plane by plane, A blocks then B blocks
    static constexpr int READS = 3 * (MT + NT), MFMAS = 6 * MT * NT;
    template <int Q>
    __device__ __forceinline__ void read(Frag& f, const unsigned char* buf) {
        constexpr int P = Q / (MT + NT), B = Q % (MT + NT);
        if constexpr (B < MT) f.a[P][B] = *reinterpret_cast<const sp_u32x4*>(buf + a_base + P * PLANE + B * 32 * PITCH);
        else f.b[P][B - MT] = *reinterpret_cast<const sp_u32x4*>(buf + b_base + P * PLANE + (B - MT) * 32 * PITCH);
    }
    // matrix instruction Q: the six term products, smallest first; the blocks innermost, so that none waits for the one before
    template <int Q>
    __device__ __forceinline__ void mma(const Frag& f) {
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
        constexpr int T = Q / (MT * NT), I = Q / NT % MT, J = Q % NT;
        if constexpr (APART && T < 5) rest[I][J] = split_mfma(f.a[PA[T]][I], f.b[PB[T]][J], rest[I][J]);
        else acc[I][J] = split_mfma(f.a[PA[T]][I], f.b[PB[T]][J], acc[I][J]);
    }
    // fetch(raw, c): requests this lane's raw words of chunk c (c may be past the end: anything valid).
    // prep(raw, c):  what has to happen to them before they are split, branches included.
    // park(part, raw, state, buf): part 0 .. PARTS - 1 of splitting them into an LDS buffer.
    // DEPTH (2 or 4): chunks whose raw words are in flight.
    template <class Raw, class State, int PARTS, bool BEHIND_FIRST, int DEPTH, class Fetch, class Prep, class Park>
    __device__ __forceinline__ void run(int n_chunks, unsigned char* lds, Fetch fetch, Prep prep, Park park) {
        unsigned char* const buf0 = lds;
        unsigned char* const buf1 = lds + BYTES;
        static_assert(DEPTH == 2 || DEPTH == 4, "raw sets");
        Raw r[DEPTH];
        State st;
        Frag f0, f1;
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) fetch(r[d], d);
        prep(r[0], 0);
        split_for<0, PARTS>([&](auto p) { park(p, r[0], st, buf0); });
        fetch(r[0], DEPTH);
        split_barrier();
        split_for<0, READS>([&](auto q) { read<decltype(q)::value>(f0, buf0); });
        prep(r[1], 1);
        split_for<0, PARTS>([&](auto p) { park(p, r[1], st, buf1); });
        fetch(r[1], DEPTH + 1);
        auto step = [&](int c, Frag& now, Frag& next, const unsigned char* from, Raw& raw, unsigned char* to) {
            prep(raw, c + 2);
            // Slot q: one matrix instruction, then its share of the reads and of the parts.  The barrier (everybody has
            // parked chunk c + 1 and read chunk c) stands LEAD matrix instructions into the step, the LDS work after it.
            constexpr int LEAD = MFMAS / 6, R_SLOTS = MFMAS / 2, P_SLOTS = MFMAS - LEAD;
            split_for<0, MFMAS>([&](auto qc) {
                constexpr int q = decltype(qc)::value, w = q - LEAD;
                __builtin_amdgcn_sched_barrier(0);
                // the wavefront that is behind goes first: otherwise one of the two on a SIMD runs ahead to the barrier and
                // leaves the other alone on the matrix pipe
                if constexpr (BEHIND_FIRST && q % (MFMAS / 4) == 0) __builtin_amdgcn_s_setprio(3 - q / (MFMAS / 4));
                mma<q>(now);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (w == -1) split_barrier();
                if constexpr (w >= 0) {
                    constexpr int R0 = w * READS / R_SLOTS, R1 = (w + 1) * READS / R_SLOTS;
                    split_for<(R0 < READS ? R0 : READS), (R1 < READS ? R1 : READS)>([&](auto r) { read<decltype(r)::value>(next, from); });
                    split_for<w * PARTS / P_SLOTS, (w + 1) * PARTS / P_SLOTS>([&](auto p) { park(p, raw, st, to); });
                }
            });
            __builtin_amdgcn_sched_barrier(0);
            fetch(raw, c + 2 + DEPTH);
        };
        // (left in the middle, so that every path into a step has the other raw sets' loads behind it)
        for (int c = 0;;) {
            step(c, f0, f1, buf1, r[2 % DEPTH], buf0);
            if (++c >= n_chunks) break;
            step(c, f1, f0, buf0, r[3 % DEPTH], buf1);
            if (++c >= n_chunks) break;
            if constexpr (DEPTH == 4) {
                step(c, f0, f1, buf1, r[0], buf0);
                if (++c >= n_chunks) break;
                step(c, f1, f0, buf0, r[1], buf1);
                if (++c >= n_chunks) break;
            }
        }
    }
    // Adds the sums of the two halves of every chunk.  Afterwards sum[i][j][t] holds entry e = 8 g + t of block (i, j),
    // g = wave / 4: this wavefront finishes half of the entries of its blocks, its partner in the other group the other
    // half.  (k 0..15) + (k 16..31): one fixed order.
    __device__ __forceinline__ void exchange(int wave, int lane, unsigned char* lds, float (&sum)[MT][NT][8]) {
        if constexpr (APART) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] += rest[i][j][e];
        }
        const int g = wave >> 2;
        split_barrier();                                 // everybody is done with the buffers
        float* x = reinterpret_cast<float*>(lds);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    x[((wave * MT * NT + i * NT + j) * 8 + t) * 64 + lane] = g == 0 ? acc[i][j][8 + t] : acc[i][j][t];
        split_barrier();
        const int partner = wave ^ 4;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float other = x[((partner * MT * NT + i * NT + j) * 8 + t) * 64 + lane];
                    sum[i][j][t] = g == 0 ? acc[i][j][t] + other : other + acc[i][j][8 + t];
                }
    }
    // An infinity (or a finite value beyond bf16's largest, 3.39e38: it rounds to one) leaves NaN in its second term, and six
    // term products may overflow where their sum does not.  All of that ends in a sum that is not finite, so such sums, and
    // no others, are replaced by form(i, j): block (i, j) of this wavefront by the fp32 instruction from the operands as they
    // are (a wavefront and its partner both form the whole block).  1000 x 4096, 512 samples: scores 34 us, 71 with one class
    // at minus infinity, 140 with half of them; update 31 us, 111 with one infinite feature (a lane summing each such entry by
    // itself: 740, 3770 and 2470).
    template <class Form>
    __device__ __forceinline__ void mend(int wave, float (&sum)[MT][NT][8], Form form) {
        const int g = wave >> 2;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                bool finite = true;
#pragma unroll
                for (int t = 0; t < 8; ++t) finite &= __builtin_isfinite(sum[i][j][t]);
                if (__all(finite)) continue;
                const f32x16 x = form(i, j);
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (!__builtin_isfinite(sum[i][j][t])) sum[i][j][t] = g == 0 ? x[t] : x[8 + t];
            }
    }
    // row of entry 8 g + t inside its block (the column is lane % 32)
    static __device__ __forceinline__ int entry_row(int g, int t, int lane) {
        const int e = 8 * g + t;
        return 8 * (e / 4) + 4 * (lane >> 5) + (e % 4);
    }
};

}  // namespace sfb
