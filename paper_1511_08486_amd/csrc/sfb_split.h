// fp32 contractions on the 16-bit matrix cores at fp32 accuracy: what the score pass (sfb_forward_split.hip) and the
// reconstruction (sfb_reconstruct_split.hip) share.
//
// gfx950 multiplies 16-bit operands sixteen times faster than fp32 on its matrix cores.  Every fp32 operand is split into terms of 16 bits
// and a product is taken as its leading term products, each exact in the fp32 accumulator's input:
//   Three bf16 terms, x = h + m + l (h = bf16(x), m = bf16(x - h), l = bf16(x - h - m)): EXACT, 3 x 8 significand bits cover
//     fp32's 24, and both differences are exact in fp32 (below 2^-109 l runs out of bf16's exponents: sums of operands of 2^-118
//     are off by 3e-7, of 2^-120 by 1e-6, of 2^-125 by 3e-5, where the fp32 instruction keeps 1e-7).  Six products, those whose
//     weight is at least 2^-16 of the leading one; what is left out is below 2^-24 of |a b| and unbiased.
//   Two fp16 terms of the scaled value, s x = h + l / 2048 (h = fp16(s x), l = fp16(2048 (s x - h))): 22 significand bits and a sign, three
//     quarters of all fp32 values exactly, the others 2^-24 off.  Three products; left out: a_l b_l, below 2^-22 and unbiased.  Half the matrix
//     instructions and two thirds of the LDS traffic.  fp16 has few exponents, so a workgroup takes one power of two s per operand, from its
//     first 64 k.  l is kept 2048 times as large, in sums of its own, and so has the exponents of h: every value between 2^-12 and 2^15
//     scaled keeps its 22 bits, below it is at most 2^-36 scaled off.  (With l as it is, values lost bits from 2^-2 scaled on: samples
//     or classes 2^-15 of their neighbours were 1e-6 of their own norm off, now 2e-7 at any factor.)  Every group of four values is looked
//     at: none beyond 2^15 scaled, and none whose largest is below 2^-12 but not zero, so that a value is at most 2^-24 of its group's largest
//     off.  From the first chunk with a group outside on, the rest of the sum is taken in three terms.  s puts the first 64 k in the middle of that
//     window: softmax factors of 3326 classes are 3e-4 in most blocks until a label comes, and 1 then (update with 532 pairs: with 2^6 above the
//     first values and 2^21 below 21.2 us, with the window's middle 18.4).  Softmax factors of logits of deviation 3.5 stay in two terms (1000 x
//     4096 with 512 pairs 23.4 us), of 4 and more are refused at the first look (27.5; three terms throughout 26.6; before two terms 29.5).
// Sums of 256 products and more are closer to fp64 with two terms than with the three terms in one running sum that they replace; of the norm,
// operands of mixed signs (then -> two terms here): scores 1000 x 4096, 512 samples 2.5e-7 -> 1.8e-7, update 2.4e-7 -> 1.7e-7;
// 600 x 4096 with 1024: 2.9e-7 -> 1.9e-7 and 2.4e-7 -> 1.7e-7.  Three terms here: 1.4e-7 and 1.3e-7 (1000 x 4096).  Either way the smaller
// products have sums of their own, so that the leading ones' running sum is rounded once for every 32 k, and long walks add theirs in two
// halves (4096 positive products: 2.7e-7 before, 3.0e-7 in one running sum, 1.6e-7 in halves).
//
// A workgroup has two kinds of wavefronts.  Splitting ones (eight, two a SIMD) request raw words three chunks of 32 k ahead, through
// descriptors whose base moves by scalar instructions, split them and park the terms in LDS; multiplying ones (one or two a SIMD) read
// fragments and do nothing but matrix instructions, so neither kind stands in the other's instruction stream.  One barrier a chunk; two terms
// have three LDS buffers (a fragment is read one phase of products before its use, across the barrier too), three terms two.
// 128 x 128 tiles, a chunk: 0.76 us for scores and 0.88 for the update (1.04 where every wavefront did both in turns, with three terms); in cycles, of
// then 1600: matrix instructions alone 770, 966 with the barrier, LDS reads, writes and loads without either 1500, splits alone 1027 (of
// 17 vector instructions for four values; 21 with the second term's scale).
#pragma once
#include <type_traits>

#include "sfb_device.h"

namespace sfb {

typedef __bf16 sp_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 sp_f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t sp_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint32_t sp_lds_u32;             // (a flat load would wait for every load on its way)
typedef float sp_f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // a 16-byte access at any 4-byte address

constexpr int kSpChunk = 32;       // k per chunk
constexpr int kSpTopExp = 14;      // two terms: values stay below 2^15 scaled,
constexpr int kSpLeastExp = -12;   // the largest of a group of four above 2^-12 (or it is zero),
constexpr int kSpTopExpLeast = 2;  // and the first chunks' largest is above 2^2
constexpr int kSpBlankExp = 4;     // the scale's exponent where they are all zero
constexpr int kSpLowExp = 11;      // the second term is kept 2^11 times as large

// every wavefront of the workgroup; this wavefront's LDS writes are visible and its LDS reads done
__device__ __forceinline__ void split_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ f32x16 split_mfma(sp_u32x4 a, sp_u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sp_bf16x8, a), __builtin_bit_cast(sp_bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 split_mfma16_f16(sp_u32x4 a, sp_u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(sp_f16x8, a), __builtin_bit_cast(sp_f16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 split_mfma16(sp_u32x4 a, sp_u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sp_bf16x8, a), __builtin_bit_cast(sp_bf16x8, b), c, 0, 0, 0);
}

// four k: one of this lane's quarter each
__device__ __forceinline__ f32x4 split_mfma16_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f32x16 split_mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

template <int FIRST, int LAST, class F>
__device__ __forceinline__ void split_for(F f) {
    if constexpr (FIRST < LAST) {
        f(std::integral_constant<int, FIRST>{});
        split_for<FIRST + 1, LAST>(f);
    }
}

// The exact split of two pairs of fp32 values (a0 a1, b0 b1) in four parts of four to six vector instructions, the two
// pairs side by side so that neighbours do not depend on each other (an instruction that waits for the last takes eight cycles, not four)
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

// Two fp16 terms of two scaled values each, packed: h = fp16(s x), l = fp16(2^11 (s x - h)); s is a power of two, the difference is exact.
// s_low = 2^11 s.  Eight vector instructions of four cycles (v_fma_mixlo_f16, which gives either term in one, takes twice as long).
struct SplitPair {
    uint32_t h, l;
    __device__ __forceinline__ SplitPair(float x0, float x1, float s, float s_low) {
        const float minus = -(float)(1 << kSpLowExp);
        float r0, r1;
        asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(h) : "v"(x0 * s), "v"(x1 * s));
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(h), "s"(minus), "v"(x0 * s_low));
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(h), "s"(minus), "v"(x1 * s_low));
        asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(l) : "v"(r0), "v"(r1));
    }
};
// largest magnitude of four
__device__ __forceinline__ float split_most4(f32x4 x) {
    float m;
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(x[0]), "v"(x[1]), "v"(x[2]));
    asm("v_max_f32 %0, |%1|, %0" : "+v"(m) : "v"(x[3]));
    return m;
}

// Scale of one operand and the bounds that its values keep (magnitudes as their bit patterns)
struct SplitScale {
    float s, s_low;
    int e;                         // s = 2^e, s_low = 2^(e + 11)
    uint32_t most, least_m1;       // largest allowed magnitude; smallest one of a group that is not all zero, minus one
    // m: largest magnitude of the first chunks, low_m1: smallest largest of a group of them that is not all zero, minus one.  What they
    // leave of the window lies half above them and half below.  false: no such scale, the three-term products take the tile.
    __device__ __forceinline__ bool set(uint32_t m, uint32_t low_m1) {
        const int x = (int)(m >> 23), span = x - (int)((low_m1 + 1u) >> 23);
        e = m == 0 ? kSpBlankExp : max(kSpTopExp - (kSpTopExp - kSpLeastExp - span) / 2, kSpTopExpLeast) + 127 - x;
        s = __uint_as_float((uint32_t)(127 + e) << 23);
        s_low = __uint_as_float((uint32_t)(127 + e + kSpLowExp) << 23);
        most = (uint32_t)min(127 + kSpTopExp + 1 - e, 254) << 23;
        least_m1 = ((uint32_t)(127 + kSpLeastExp - e) << 23) - 1u;
        return m == 0 || (x >= 28 && x < 255 && span <= kSpTopExp - kSpLeastExp);
    }
};

// largest of sixteen lanes, in each of them
__device__ __forceinline__ uint32_t split_max16(uint32_t x) {
    auto step = [](uint32_t v, auto ctrl) { return max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, decltype(ctrl)::value, 0xf, 0xf, true)); };
    x = step(x, std::integral_constant<int, 0xb1>{});                    // quad_perm 1,0,3,2
    x = step(x, std::integral_constant<int, 0x4e>{});                    // quad_perm 2,3,0,1
    x = step(x, std::integral_constant<int, 0x141>{});                   // row_half_mirror
    return step(x, std::integral_constant<int, 0x140>{});                // row_mirror
}

// One workgroup's contraction: a tile of BM x BN by WM x WN multiplying wavefronts, each MB x NB blocks of 16 x 16, and SPLITTERS
// splitting ones.  An LDS row is 32 k of one row of the tile (BM of the A operand, then BN of B), 64 bytes a plane; 16-byte item c of row r
// sits at c ^ swz(r).
// EXACT: three-term products throughout, for callers who chose them (sfb_set_plan).
template <int BM_, int BN_, int WM_, int WN_, int SPLITTERS, bool EXACT>
struct SplitTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, MB = BM / (16 * WM), NB = BN / (16 * WN), ROWS = BM + BN;
    static constexpr int MULTIPLIERS = WM * WN, THREADS = 64 * (MULTIPLIERS + SPLITTERS);
    static constexpr int PLANE = ROWS * 64;
    static constexpr int CTL = 6 * PLANE;                               // three buffers of two planes or two of three; control words; first halves
    static constexpr int HALF = CTL + 32, LDS = HALF + 64 * MULTIPLIERS * 4 * (4 * MB * NB - 1);
    static_assert(LDS <= 160 * 1024, "LDS");

    // Among eight consecutive rows any one item falls into eight different 16-byte bank groups of 128 bytes, among
    // sixteen into sixteen of 256; of four consecutive rows (from a multiple of four) half a row each, too.
    static __device__ __forceinline__ int swz(int r) { return ((r >> 2) & 1) | ((((r >> 1) ^ (r >> 3)) & 1) << 1); }

    // Control words: [0] chunks from this number on are not taken in two terms; [4 ..] what the splitting wavefronts saw in the first
    // two chunks: of each operand the largest magnitude, and the smallest largest of a group that is not all zero, minus one (complement).
    static __device__ __forceinline__ uint32_t stop_word(unsigned char* lds) { return *(volatile sp_lds_u32*)(lds + CTL); }
    static __device__ __forceinline__ bool scales(const unsigned char* lds, SplitScale (&sc)[2]) {
        const uint4 all = *reinterpret_cast<const uint4*>(lds + CTL + 16);
        auto uniform = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
        const bool a = sc[0].set(uniform(all.x), ~uniform(all.y)), b = sc[1].set(uniform(all.z), ~uniform(all.w));
        return a && b;
    }

    static __device__ __forceinline__ int threes(int n) { return n > 0 ? n / 3 * 3 : 0; }   // of n, in whole threes

    // ---- the multiplying wavefronts ----
    static constexpr bool REST = MB * NB <= 8;                          // the smaller products have sums of their own (registers)
    static_assert(REST || EXACT, "two terms: the smaller products are on another scale");
    // Two terms: leading products of even and odd chunks apart where there are registers for it (all-positive operands, 600 x 4096, 1024 pairs:
    // 1.8e-7 of the norm in one sum, 0.9e-7 in two)
    static constexpr int SUMS = ROWS > 128 && ROWS < 256 && !EXACT ? 2 : 1;
    f32x4 acc[MB][NB], rest[REST ? MB : 1][REST ? NB : 1], odd[SUMS == 2 ? MB : 1][SUMS == 2 ? NB : 1];
    float kept;                    // of the first half's sums: the one that LDS has no room for (128 x 128: 160 KB but 2016 bytes)
    bool halved;                   // the others are there (uniform)
    int a_base, b_base;            // byte offset of this lane's item in the A and the B part

    __device__ __forceinline__ void init(int wave, int lane) {
        const int wm = wave / WN, wn = wave % WN, l16 = lane & 15;
        const int item = 16 * ((lane >> 4) ^ swz(l16));                  // every row this lane reads is l16 modulo 16
        a_base = (wm * 16 * MB + l16) * 64 + item;
        b_base = (BM + wn * 16 * NB + l16) * 64 + item;
        halved = false;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (REST) rest[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (SUMS == 2) odd[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    }
    // The leading sums so far wait in LDS (a lane's own words), new ones start at zero: half as many roundings of sums half as large
    __device__ __forceinline__ void set_aside(unsigned char* lds) {
        split_for<0, MB * NB>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            f32x4& sum = acc[q / NB][q % NB];
            if constexpr (q + 1 < MB * NB) {
                *reinterpret_cast<f32x4*>(lds + HALF + (q * 64 * MULTIPLIERS + (int)threadIdx.x) * 16) = sum;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    *reinterpret_cast<float*>(lds + HALF + q * 64 * MULTIPLIERS * 16 + (e * 64 * MULTIPLIERS + (int)threadIdx.x) * 4) = sum[e];
                kept = sum[3];
            }
            sum = f32x4{0.f, 0.f, 0.f, 0.f};
        });
        halved = true;
    }
    __device__ __forceinline__ void add_halves(const unsigned char* lds) {
        if (!halved) return;
        split_for<0, MB * NB>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            f32x4& sum = acc[q / NB][q % NB];
            if constexpr (q + 1 < MB * NB) {
                sum += *reinterpret_cast<const f32x4*>(lds + HALF + (q * 64 * MULTIPLIERS + (int)threadIdx.x) * 16);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    sum[e] += *reinterpret_cast<const float*>(lds + HALF + q * 64 * MULTIPLIERS * 16 + (e * 64 * MULTIPLIERS + (int)threadIdx.x) * 4);
                sum[3] += kept;
            }
        });
        halved = false;
    }
    __device__ __forceinline__ sp_u32x4 item_a(const unsigned char* buf, int plane, int i) const {
        return *reinterpret_cast<const sp_u32x4*>(buf + a_base + plane * PLANE + i * 16 * 64);
    }
    __device__ __forceinline__ sp_u32x4 item_b(const unsigned char* buf, int plane, int j) const {
        return *reinterpret_cast<const sp_u32x4*>(buf + b_base + plane * PLANE + j * 16 * 64);
    }
    // All blocks' products of one plane of A and one of B, with COUNT reads spread over the first of them (two a matrix instruction at most
    // in small tiles, every other instruction in large ones).
    template <int T, bool LEADING, int COUNT, bool ODD = false, class Read>
    __device__ __forceinline__ void phase(const sp_u32x4 (&a)[MB], const sp_u32x4 (&b)[NB], Read read) {
        split_for<0, MB * NB>([&](auto qc) {
            constexpr int q = decltype(qc)::value, i = q / NB, j = q % NB;
            __builtin_amdgcn_sched_barrier(0);
            f32x4& to = REST && !LEADING ? rest[REST ? i : 0][REST ? j : 0] : ODD ? odd[SUMS == 2 ? i : 0][SUMS == 2 ? j : 0] : acc[i][j];
            if constexpr (T == 2) to = split_mfma16_f16(a[i], b[j], to);
            else to = split_mfma16(a[i], b[j], to);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int OVER = COUNT > 0 ? (MB * NB > COUNT ? COUNT : MB * NB) : 1;
            if constexpr (q < OVER) split_for<q * COUNT / OVER, (q + 1) * COUNT / OVER>(read);
        });
        __builtin_amdgcn_sched_barrier(0);
    }
    // Two terms (planes h, l), chunks 0 .. n - 1; returns the first that was not taken.  A fragment is read into the registers that it takes
    // over one phase of products ahead of its use.
    __device__ __forceinline__ int multiply2(int n, int half, unsigned char* lds) {
        constexpr int BUF = 2 * PLANE;
        sp_u32x4 ah[MB], al[MB], bh[NB], bl[NB];
        int at = 0, c = 0, end = SUMS == 1 && half > 0 ? half : n;
        bool go;
#pragma unroll
        for (int i = 0; i < MB; ++i) ah[i] = item_a(lds, 0, i);
#pragma unroll
        for (int j = 0; j < NB; ++j) bl[j] = item_b(lds, 1, j);
        auto step = [&](auto is_odd) {
            const unsigned char* const now = lds + at;
            at = at == 2 * BUF ? 0 : at + BUF;
            const unsigned char* const next = lds + at;
            const uint32_t stop = stop_word(lds);
            phase<2, false, NB + MB>(ah, bl, [&](auto rc) {
                constexpr int r = decltype(rc)::value;
                if constexpr (r < NB) bh[r] = item_b(now, 0, r);
                else al[r - NB] = item_a(now, 1, r - NB);
            });
            phase<2, true, NB, decltype(is_odd)::value>(ah, bh, [&](auto rc) { bl[decltype(rc)::value] = item_b(next, 1, decltype(rc)::value); });
            phase<2, false, MB>(al, bh, [&](auto rc) { ah[decltype(rc)::value] = item_a(next, 0, decltype(rc)::value); });
            asm volatile("s_barrier" ::: "memory");                      // (its reads of the buffer that is written next are used up)
            ++c;
            go = (uint32_t)__builtin_amdgcn_readfirstlane((int)stop) > (uint32_t)c;
            return go && c < end;
        };
        for (;;) {
            while (step(std::false_type{}))
                if (SUMS == 2 && !step(std::bool_constant<SUMS == 2>{})) break;
            if (SUMS == 2 || !go || c == n) break;
            set_aside(lds);                                              // (c == half; not in the loop, whose registers it would take)
            end = n;
        }
        // (the splitting wavefronts see it behind three steps, or at the end)
        const int whole = threes(n - 2);
        for (int b = c; b < n && (b > whole || b % 3 != 0); ++b) asm volatile("s_barrier" ::: "memory");
        return c;
    }
    // Three terms (planes h, m, l), chunks c0 .. n - 1.  The first products wait for two planes' fragments only, every other plane is read over
    // the products before its use, into the registers that are free by then.
    __device__ __forceinline__ void multiply3(int c0, int n, int half, unsigned char* lds) {
        constexpr int BUF = 3 * PLANE;
        for (int c = c0, at = 0; c < n; ++c, at = BUF - at) {
            const unsigned char* const now = lds + at;
            if (c == half) set_aside(lds);
            sp_u32x4 ah[MB], a1[MB], bh[NB], b1[NB];
            split_for<0, (MB > NB ? MB : NB)>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                if constexpr (r < MB) ah[r] = item_a(now, 0, r);
                if constexpr (r < NB) bh[r] = item_b(now, 0, r);
            });
            phase<3, true, NB>(ah, bh, [&](auto rc) { b1[decltype(rc)::value] = item_b(now, 1, decltype(rc)::value); });
            phase<3, false, MB>(ah, b1, [&](auto rc) { a1[decltype(rc)::value] = item_a(now, 1, decltype(rc)::value); });
            phase<3, false, 0>(a1, b1, [](auto) {});
            phase<3, false, NB>(a1, bh, [&](auto rc) { b1[decltype(rc)::value] = item_b(now, 2, decltype(rc)::value); });
            phase<3, false, MB>(ah, b1, [&](auto rc) { a1[decltype(rc)::value] = item_a(now, 2, decltype(rc)::value); });
            phase<3, false, 0>(a1, bh, [](auto) {});
            asm volatile("s_barrier" ::: "memory");
        }
    }
    // halves: walks of so many chunks and more are summed in two halves, the second from the middle on or from where the split changes
    __device__ __forceinline__ void multiply(int n, int halves, unsigned char* lds) {
        int done = 0;
        const int half = n >= halves ? n / 2 : -1;
        auto merge = [&](int e, float rest_scale) {
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if constexpr (SUMS == 2) {
                            acc[i][j][q] += odd[i][j][q];
                            odd[i][j][q] = 0.f;
                        }
                        if constexpr (REST) {
                            acc[i][j][q] = __builtin_fmaf(rest[i][j][q], rest_scale, acc[i][j][q]);
                            rest[i][j][q] = 0.f;
                        }
                        acc[i][j][q] = __builtin_amdgcn_ldexpf(acc[i][j][q], e);
                    }
        };
        if constexpr (!EXACT) {
            if (threadIdx.x < 8) *(volatile sp_lds_u32*)(lds + CTL + 4 * threadIdx.x) = threadIdx.x == 0 ? 0xffffffffu : 0u;   // wavefront 0
            split_barrier();
            split_barrier();
            SplitScale sc[2];
            if (scales(lds, sc)) {
                split_barrier();
                done = multiply2(n, half, lds);
                add_halves(lds);
                merge(-(sc[0].e + sc[1].e), 1.0f / (1 << kSpLowExp));
            }
            if (done >= n) return;
        }
        split_barrier();
        multiply3(done, n, half < 0 || done == 0 ? half : done, lds);
        add_halves(lds);
        merge(0, 1.f);
    }

    // ---- the splitting wavefronts ----
    // ITEMS groups of four values a lane and chunk, in slots of the same operand: where(c, first) says where chunk c is (c may be past the end:
    // then there is nothing to move; first: compile time, chunk 0 may be only there), load(raw, place, u, first) requests unit u of its raw
    // words (as many units as pairs of groups), prep(raw, c, first) does what has to happen to them before they are split, take(raw, i) is
    // group i, put(buf, plane, i, words) parks four terms of it.  Raw words of three chunks are in flight.
    // A unit is requested as soon as its words are used up, one behind every pair of groups (LAG pairs later): in one burst behind a chunk the
    // requests of four wavefronts took 900 cycles to be accepted, and nothing was split meanwhile.
    // Slot slot(i): operand second[slot], parked only where on[slot] (both uniform).
    // split_in: chunks c0 .. n - 1 in T terms; r[0] holds the raw words of chunk c0.  ready (two terms: always): prepared (and r[1] those of the next).
    template <int T, class Raw, int ITEMS, int SLOTS, int LAG, class Slot, class Where, class Load, class Prep, class Take, class Put>
    static __device__ __forceinline__ int split_in(int c0, int n, unsigned char* lds, Raw (&r)[3], bool ready, const SplitScale (&sc)[2],
                                            const bool (&second)[SLOTS], const bool (&on)[SLOTS], Slot slot, Where where, Load load, Prep prep,
                                            Take take, Put put) {
        constexpr int LEAD = T == 2 ? 2 : 1, BUF = T * PLANE, UNITS = (ITEMS + 1) / 2;
        float s[SLOTS], s_low[SLOTS];
        uint32_t most[SLOTS], least[SLOTS];
        if constexpr (T == 2) {
#pragma unroll
            for (int q = 0; q < SLOTS; ++q) {
                s[q] = second[q] ? sc[1].s : sc[0].s;
                s_low[q] = second[q] ? sc[1].s_low : sc[0].s_low;
                most[q] = second[q] ? sc[1].most : sc[0].most;
                least[q] = second[q] ? sc[1].least_m1 : sc[0].least_m1;
            }
        }
        auto park = [&](const Raw& raw, int c, int at, auto after) {
            uint32_t mx[SLOTS], mn[SLOTS];
#pragma unroll
            for (int q = 0; q < SLOTS; ++q) { mx[q] = 0u; mn[q] = 0xffffffffu; }
            split_for<0, UNITS>([&](auto uc) {
                split_for<2 * decltype(uc)::value, (2 * decltype(uc)::value + 2 < ITEMS ? 2 * decltype(uc)::value + 2 : ITEMS)>([&](auto ic) {
                    constexpr int q = decltype(slot(ic))::value;
                    const f32x4 x = take(raw, ic);
                    constexpr std::integral_constant<int, 0> p0{};
                    constexpr std::integral_constant<int, 1> p1{};
                    constexpr std::integral_constant<int, 2> p2{};
                    if constexpr (T == 2) {
                        const SplitPair a(x[0], x[1], s[q], s_low[q]), b(x[2], x[3], s[q], s_low[q]);
                        const uint32_t m = __float_as_uint(split_most4(x));
                        mx[q] = max(mx[q], m);
                        mn[q] = min(mn[q], m - 1u);
                        if (on[q]) {
                            put(lds + at, p0, ic, make_uint2(a.h, b.h));
                            put(lds + at, p1, ic, make_uint2(a.l, b.l));
                        }
                    } else {
                        SplitQuad quad;
                        split_for<0, 4>([&](auto p) { quad.template part<decltype(p)::value>(x[0], x[1], x[2], x[3]); });
                        if (on[q]) {
                            put(lds + at, p0, ic, make_uint2(quad.ha, quad.hb));
                            put(lds + at, p1, ic, make_uint2(quad.ma, quad.mb));
                            put(lds + at, p2, ic, make_uint2(quad.la, quad.lb));
                        }
                    }
                });
                __builtin_amdgcn_sched_barrier(6);                       // (vector and scalar instructions may pass)
                after(uc);
                __builtin_amdgcn_sched_barrier(6);
            });
            if constexpr (T == 2) {
                bool bad = false;
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) bad |= on[q] && (mx[q] > most[q] || mn[q] < least[q]);
                if (bad) __hip_atomic_fetch_min(reinterpret_cast<uint32_t*>(lds + CTL), (uint32_t)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        constexpr std::false_type later{};
        auto fetch = [&](Raw& raw, int c, auto units) {                  // the first so many units
            const auto place = where(c, later);
            split_for<0, decltype(units)::value>([&](auto u) { load(raw, place, u, later); });
        };
        constexpr std::integral_constant<int, UNITS> all{};
        constexpr std::integral_constant<int, UNITS - LAG> early{};
        static_assert(LAG <= UNITS, "units");
        int at = LEAD * BUF;
        if constexpr (T == 2) {
            // (the third set's words are requested behind the first's, not before: the first's are not held up)
            const auto third = where(c0 + 2, later), fourth = where(c0 + 3, later);
            park(r[0], c0, 0, [&](auto uc) { load(r[2], third, uc, later); });
            park(r[1], c0 + 1, BUF, [&](auto uc) { load(r[0], fourth, uc, later); });
            fetch(r[1], c0 + 4, early);
        } else {
            fetch(r[1], c0 + 1, all);
            fetch(r[2], c0 + 2, all);
            if (!ready) prep(r[0], c0, std::true_type{});
            park(r[0], c0, 0, [](auto) {});
            fetch(r[0], c0 + 3, early);
        }
        split_barrier();
        int c = c0;
        auto step = [&](Raw& raw, auto after) {
            prep(raw, c + LEAD, later);
            park(raw, c + LEAD, at, after);
            at = at == (T == 2 ? 2 : 1) * BUF ? 0 : at + BUF;
            split_barrier();
            ++c;
        };
        auto full_step = [&](Raw& before, Raw& raw) {
            const auto last = where(c + LEAD + 2, later), next = where(c + LEAD + 3, later);
            step(raw, [&](auto uc) {
                constexpr int u = decltype(uc)::value;
                if constexpr (u < LAG) load(before, last, std::integral_constant<int, UNITS - LAG + u>{}, later);
                else load(raw, next, std::integral_constant<int, u - LAG>{}, later);
            });
        };
        // Whole rounds of the three raw sets, then what is left of them.  The loop is left behind three steps only: an exit between
        // steps meets the loop's own back edge in the generated code, where the wait for a raw set is then one for whatever
        // any of the paths has on its way (the first of three steps waited for every load).
        const int whole = c0 + threes(n - c0 - LEAD);
        uint32_t stop = 0xffffffffu;
        while (c < whole && stop > (uint32_t)c) {
            full_step(r[LEAD - 1], r[LEAD]);
            full_step(r[LEAD], r[(LEAD + 1) % 3]);
            full_step(r[(LEAD + 1) % 3], r[LEAD - 1]);
            if (T == 2) stop = (uint32_t)__builtin_amdgcn_readfirstlane((int)stop_word(lds));
        }
        if (stop <= (uint32_t)c) return (int)stop;
        if (c + LEAD < n) step(r[LEAD], [](auto) {});
        if (c + LEAD < n) step(r[(LEAD + 1) % 3], [](auto) {});
        for (; c < n; ++c) split_barrier();
        return T == 2 ? (int)min((uint32_t)n, (uint32_t)__builtin_amdgcn_readfirstlane((int)stop_word(lds))) : n;
    }
    template <class Raw, int ITEMS, int SLOTS, int LAG, class Slot, class Where, class Load, class Prep, class Take, class Put>
    static __device__ __forceinline__ void split(int n, unsigned char* lds, const bool (&second)[SLOTS], const bool (&on)[SLOTS], Slot slot,
                                          Where where, Load load, Prep prep, Take take, Put put) {
        Raw r[3];
        SplitScale sc[2];
        auto fetch = [&](Raw& raw, int c, auto first) {
            const auto place = where(c, first);
            split_for<0, (ITEMS + 1) / 2>([&](auto u) { load(raw, place, u, first); });
        };
        int done = 0;
        bool ready = false;
        fetch(r[0], 0, std::true_type{});
        if constexpr (!EXACT) {
            fetch(r[1], 1, std::false_type{});
            split_barrier();                                             // the control words are clear
            prep(r[0], 0, std::true_type{});
            prep(r[1], 1, std::false_type{});
            uint32_t words[4] = {0u, 0u, 0u, 0u};                        // (smallest as the largest complement)
            split_for<0, ITEMS>([&](auto ic) {
                constexpr int q = decltype(slot(ic))::value;
                const uint32_t x = __float_as_uint(split_most4(take(r[0], ic))), y = __float_as_uint(split_most4(take(r[1], ic)));
                const uint32_t m = on[q] ? max(x, y) : 0u, l = on[q] ? max(~(x - 1u), ~(y - 1u)) : 0u;
                words[0] = max(words[0], second[q] ? 0u : m);
                words[1] = max(words[1], second[q] ? 0u : l);
                words[2] = max(words[2], second[q] ? m : 0u);
                words[3] = max(words[3], second[q] ? l : 0u);
            });
#pragma unroll
            for (int i = 0; i < 4; ++i) words[i] = split_max16(words[i]);
            const int i = threadIdx.x & 15;                              // lanes 0 .. 3 of every sixteen: a word each
            const uint32_t word = i == 0 ? words[0] : i == 1 ? words[1] : i == 2 ? words[2] : words[3];
            // (as an atomic of the language it becomes a loop over the lanes: four of them took 1000 cycles)
            if (i < 4) asm volatile("ds_max_u32 %0, %1" ::"v"((uint32_t)(uintptr_t)(sp_lds_u32*)(lds + CTL + 16) + 4u * i), "v"(word) : "memory");
            split_barrier();
            ready = !scales(lds, sc);                                    // (then three terms begin with the words that are there)
            if (!ready) {
                done = split_in<2, Raw, ITEMS, SLOTS, LAG>(0, n, lds, r, true, sc, second, on, slot, where, load, prep, take, put);
                if (done >= n) return;
                fetch(r[0], done, std::true_type{});
            }
        }
        split_in<3, Raw, ITEMS, SLOTS, LAG>(done, n, lds, r, ready, sc, second, on, slot, where, load, prep, take, put);
    }

    // An infinity (or a finite value beyond bf16's largest, 3.39e38: it rounds to one) leaves NaN in its second term, and six
    // term products may overflow where their sum does not.  All of that ends in a sum that is not finite, so such sums, and
    // no others, are replaced by form(i, j): block (i, j) of this wavefront by the fp32 instruction from the operands as they
    // are (never a lane summing such an entry by itself: with half of the classes at minus infinity that took a hundred times the time).
    template <class Form>
    __device__ __forceinline__ void mend(Form form) {
        float zero[4] = {0.f, 0.f, 0.f, 0.f};                            // stays so unless an entry is not finite
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) zero[e] = __builtin_fmaf(acc[i][j][e], 0.f, zero[e]);
        if (__all((zero[0] + zero[1]) + (zero[2] + zero[3]) == 0.f)) return;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const f32x4 x = form(i, j);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!__builtin_isfinite(acc[i][j][e])) acc[i][j][e] = x[e];
            }
    }
};

// Entry e of a lane's block is its row 4 (lane / 16) + e and column lane % 16.  Which row of a matrix LDS row r holds: with split_row64 (16) four
// (two) neighbouring blocks of a lane are neighbouring rows (columns of the result: one access); with split_row32 a lane's
// rows are uniform ones plus its own 16 ((lane / 16) % 2) + lane / 32, and BM needs to be a multiple of 32 only.
__device__ __forceinline__ int split_row64(int r) { return (r & ~63) + 4 * (r & 15) + ((r >> 4) & 3); }
__device__ __forceinline__ int split_row32(int r) { return (r & ~31) + 4 * (r & 7) + ((r >> 3) & 3); }
__device__ __forceinline__ int split_row16(int r) { return (r & ~31) + 2 * (r & 15) + ((r >> 4) & 1); }

// All bits while c < n, none from there on.  (Left to the compiler as a choice between two constants, it ended in a vector register, and
// every load that takes its descriptor's size from it in a loop over the lanes.)
__device__ __forceinline__ uint32_t split_while(int c, int n) {
    int all;
    asm("s_sub_i32 %0, %1, %2\n\ts_ashr_i32 %0, %0, 31" : "=&s"(all) : "s"(c), "s"(n) : "scc");
    return (uint32_t)all;
}

// Descriptor of raw words from p on: `bytes` of them, none where they are not wanted (such loads return zero and move nothing)
// (p and bytes are uniform; said so, or the compiler puts a loop over the lanes' descriptors around every load)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t split_words(const void* p, uint32_t bytes) {
    const uint64_t at = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), (short)0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}
typedef float sp_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ sp_f32x2 split_load2(__amdgpu_buffer_rsrc_t words, uint32_t offset) {
    return __builtin_bit_cast(sp_f32x2, __builtin_amdgcn_raw_buffer_load_b64(words, (int)offset, 0, 0));
}
__device__ __forceinline__ f32x4 split_load4(__amdgpu_buffer_rsrc_t words, uint32_t offset) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(words, (int)offset, 0, 0));
}

}  // namespace sfb
