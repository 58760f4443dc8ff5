// Scores (Section 2, z = W a) for fp32 features on the 16-bit matrix cores at fp32 accuracy: Z[n][j] = sum_d A[n][d] *
// W[j][d] with every operand split into terms (sfb_split.h: the arithmetic, its error, and the two kinds of wavefronts).
//
// Both operands are contiguous along the contraction.  A splitting lane loads 16 bytes (four k) of a row of A or W, eight lanes to
// a 128-byte line, splits them and writes 8 bytes per plane, so W is never copied and A passes through
// once more only to be stored as V.  Rows beyond the matrix repeat the last row (their scores are not stored); a partial
// chunk of D is taken first, before the loop, with the words beyond D replaced by zero in both operands.  Accesses are 16 bytes wide at
// 4-byte alignment: any leading dimension is taken.  DIFF: the operand is x_i - y_i (metric learning).
// us, every wavefront splitting and multiplying in three terms -> here: 1000 x 4096, 512 samples 28.6 -> 22.9; 600 x 4096, 1024 pairs of points 37.6 ->
// 29.5; 1000 x 4096, 4096 samples 176 -> 125.
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

template <int BM, int BN, bool EXACT>
using ScoreTile = SplitTile<BM, BN, BM == 128 && BN == 128 ? 4 : 2, 2, 8, EXACT>;

template <int NB>
__device__ __forceinline__ int ss_row(int r) { return NB == 4 ? split_row64(r) : split_row16(r); }

template <int BM, int BN, bool DIFF, bool EXACT>
__global__ __launch_bounds__((ScoreTile<BM, BN, EXACT>::THREADS), BM + BN == 256 ? 4 : BM + BN == 192 || DIFF ? 3 : 6) void scores_split_kernel(
    const float* __restrict__ A, const float* __restrict__ A2, int64_t lda, const float* __restrict__ W, int64_t ldw,
    float* __restrict__ Z, int64_t ldz, int64_t zstride, float* __restrict__ Vout, int64_t ldv, int M, int N, int K,
    int k_slice, int halves, int n_mb, int n_nb, int total) {
    using Tile = ScoreTile<BM, BN, EXACT>;
    constexpr int STEP = 64;                                             // rows that the splitting lanes take at a time, eight lanes a row
    constexpr int A_IT = BM / STEP, IT = (BM + BN) / STEP;               // 16-byte items per splitting lane and chunk: of A, of A and W
    extern __shared__ __attribute__((aligned(16))) unsigned char ss_lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // consecutive ids share the class block (its W rows then sit in one die's L2)
    int id = xcd_contiguous_id(blockIdx.x, total);
    const int mb = id % n_mb;
    id /= n_mb;
    const int nb = id % n_nb, ks = id / n_nb;
    const int m0 = mb * BM, n0 = nb * BN;
    const int k_begin = ks * k_slice, k_end = min(K, k_begin + k_slice);
    const int n_chunks = (k_end - k_begin + kSpChunk - 1) / kSpChunk;

    if (wave >= Tile::MULTIPLIERS) {
        const bool ragged = (K & 31) != 0 && k_end == K;                 // the last chunk is partial: it is taken first
        // item i of a lane: LDS row r0 + STEP i (A's rows in order, then W's by ss_row), k 4 c0 .. 4 c0 + 3 of the chunk
        const int tid = threadIdx.x - 64 * Tile::MULTIPLIERS, r0 = tid >> 3, c0 = tid & 7;
        uint32_t off[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i)
            off[i] = (i < A_IT ? (uint32_t)min(r0 + STEP * i, M - 1 - m0) * (uint32_t)lda
                               : (uint32_t)min(ss_row<Tile::NB>(r0 + STEP * (i - A_IT)), N - 1 - n0) * (uint32_t)ldw) * 4u + 16u * c0;
        const int last_k = k_begin + (n_chunks - 1) * kSpChunk + 4 * c0; // of the partial chunk: its words are read from the last four of
        const uint32_t last_off = (uint32_t)min(last_k, K - 4) * 4u - 16u * c0;   // the row (host: K >= 4) and moved into place by prep
        const int sh = max(0, last_k - (K - 4));
        const int lds_item = r0 * 64 + 16 * ((c0 >> 1) ^ Tile::swz(r0)) + 8 * (c0 & 1);   // rows r0 + STEP i share the swizzle

        struct Raw { f32x4 x[IT], y[DIFF ? A_IT : 1]; };
        struct Place { __amdgpu_buffer_rsrc_t a, a2, w; uint32_t more; };
        auto where = [&](int c, auto first) {
            const bool partial = decltype(first)::value && ragged && c == 0;
            const int k = partial ? 0 : k_begin + (c - (ragged ? 1 : 0)) * kSpChunk;
            const uint32_t bytes = split_while(c, n_chunks);
            return Place{split_words(A + (int64_t)m0 * lda + k, bytes), split_words(DIFF ? A2 + (int64_t)m0 * lda + k : nullptr, bytes),
                         split_words(W + (int64_t)n0 * ldw + k, bytes), partial ? last_off : 0u};
        };
        auto load = [&](Raw& raw, const Place& at, auto uc, auto first) {
#pragma unroll
            for (int i = 2 * decltype(uc)::value; i < 2 * decltype(uc)::value + 2 && i < IT; ++i) {
                const uint32_t o = decltype(first)::value ? off[i] + at.more : off[i];
                raw.x[i] = split_load4(i < A_IT ? at.a : at.w, o);
                if (DIFF && i < A_IT) raw.y[i] = split_load4(at.a2, o);
            }
        };
        // the class blocks share the copy of A (or X - Y) into V: block nb takes every n_nb-th chunk
        int v_next = Vout != nullptr ? nb : -1;
        auto prep = [&](Raw& raw, int c, auto first) {
            const bool partial = decltype(first)::value && ragged && c == 0;
            if constexpr (DIFF) {
#pragma unroll
                for (int i = 0; i < A_IT; ++i) raw.x[i] -= raw.y[i];
            }
            if (decltype(first)::value && partial) {                     // words read early move up, zeros beyond D
#pragma unroll
                for (int i = 0; i < IT; ++i) {
                    f32x4& x = raw.x[i];
                    if (sh & 1) x = f32x4{x[1], x[2], x[3], 0.f};
                    if (sh & 2) x = f32x4{x[2], x[3], 0.f, 0.f};
                    if (sh >= 4) x = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            if (c == v_next && c < n_chunks) {                           // v_i = a_i (or x_i - y_i)
                v_next += n_nb;
                const int k = partial ? last_k : k_begin + (c - (ragged ? 1 : 0)) * kSpChunk + 4 * c0;
#pragma unroll
                for (int i = 0; i < A_IT; ++i) {
                    if (m0 + r0 + STEP * i >= M) continue;
                    float* out = Vout + (int64_t)(m0 + r0 + STEP * i) * ldv + k;
                    if (!decltype(first)::value || !partial || k + 4 <= K) {
                        *reinterpret_cast<sp_f32x4u*>(out) = raw.x[i];
                    } else {
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            if (k + e < K) out[e] = raw.x[i][e];
                    }
                }
            }
        };
        auto take = [](const Raw& raw, auto ic) -> f32x4 { return raw.x[decltype(ic)::value]; };
        auto put = [&](unsigned char* buf, auto plane, auto ic, uint2 words) {
            *reinterpret_cast<uint2*>(buf + lds_item + decltype(plane)::value * Tile::PLANE + decltype(ic)::value * STEP * 64) = words;
        };
        const bool second[2] = {false, true}, on[2] = {true, true};
        Tile::template split<Raw, IT, 2, 0>(n_chunks, ss_lds, second, on,
                                               [](auto ic) { return std::integral_constant<int, (decltype(ic)::value >= A_IT)>{}; }, where, load, prep,
                                               take, put);
        return;
    }

    Tile t;
    t.init(wave, lane);
    t.multiply(n_chunks, halves, ss_lds);
    const int wm = wave / Tile::WN, wn = wave % Tile::WN, l16 = lane & 15, quarter = lane >> 4;
    t.mend([&](int i, int j) {
        const int64_t row = min(m0 + (wm * Tile::MB + i) * 16 + l16, M - 1), col = min(n0 + ss_row<Tile::NB>((wn * Tile::NB + j) * 16 + l16), N - 1);
        const float *a = A + row * lda, *a2 = DIFF ? A2 + row * lda : nullptr, *w = W + col * ldw;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        int k = k_begin;
        for (; k + kSpChunk <= k_end; k += kSpChunk) {                   // any order of k will do: four for each quarter of the lanes
            f32x4 p[2], q[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int o = k + 16 * c + 4 * quarter;
                p[c] = *reinterpret_cast<const sp_f32x4u*>(a + o);
                if (DIFF) p[c] -= *reinterpret_cast<const sp_f32x4u*>(a2 + o);
                q[c] = *reinterpret_cast<const sp_f32x4u*>(w + o);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) x = split_mfma16_f32(p[c][e], q[c][e], x);
        }
        for (; k < k_end; k += 4) {
            const int o = min(k + quarter, k_end - 1);
            const bool on = k + quarter < k_end;
            x = split_mfma16_f32(on ? (DIFF ? a[o] - a2[o] : a[o]) : 0.f, on ? w[o] : 0.f, x);
        }
        return x;
    });
    // The blocks of a lane are that many neighbouring classes: one access a row.  (Rows of Z are as long as there are classes: twelve of
    // them pass 2^32 bytes from 89 million on, so a lane's rows are 64-bit offsets.)
    constexpr int WIDE = Tile::NB;
    typedef float f32_wide __attribute__((ext_vector_type(WIDE), aligned(4)));
    const int lane_row = m0 + wm * Tile::MB * 16 + 4 * quarter, col = n0 + wn * 16 * WIDE + WIDE * l16;
    float* const zout = Z + (int64_t)ks * zstride + (int64_t)lane_row * ldz + col;
    auto store = [&](auto all) {
#pragma unroll
        for (int i = 0; i < Tile::MB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = i * 16 + e;
                float* const at = zout + (int64_t)row * ldz;
                f32_wide x;
#pragma unroll
                for (int j = 0; j < WIDE; ++j) x[j] = t.acc[i][j][e];
                if (decltype(all)::value) {
                    *reinterpret_cast<f32_wide*>(at) = x;
                } else if (lane_row + row < M && col < N) {              // (rows of Z are whole fours: what lies past N is nobody's)
                    *reinterpret_cast<f32_wide*>(at) = x;
                }
            }
    };
    if (m0 + BM <= M && n0 + BN <= N) store(std::true_type{});
    else store(std::false_type{});
}

bool forward_split_ok(const FwdArgs& a) {
    // lane offsets (up to 128 rows of 4-byte words) stay below 2^32
    return !a.bf16 && a.D >= 4 && a.lda < (1 << 22) && a.ldw < (1 << 22);
}

template <int BM, int BN, bool DIFF, bool EXACT>
static hipError_t launch_split(const FwdArgs& a, const FwdPlan& p, hipStream_t s) {
    using Tile = ScoreTile<BM, BN, EXACT>;
    constexpr size_t lds_bytes = Tile::LDS;
    static std::atomic<bool> raised{false};
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)scores_split_kernel<BM, BN, DIFF, EXACT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int n_mb = (a.n_rows + Tile::BM - 1) / Tile::BM, n_nb = (a.J + Tile::BN - 1) / Tile::BN;
    const int total = n_mb * n_nb * p.split_k;
    SFB_LAUNCH((scores_split_kernel<BM, BN, DIFF, EXACT>), dim3(total), dim3(Tile::THREADS), lds_bytes, s, (const float*)a.a,
               (const float*)a.a2, a.lda, a.w, a.ldw, a.zp, a.ldz, a.zstride, (float*)a.v, a.ldv, a.n_rows, a.J, a.D,
               p.k_slice, p.halves, n_mb, n_nb, total);
    return hipGetLastError();
}

template <bool DIFF>
static hipError_t launch_split_tile(const FwdArgs& a, const FwdPlan& p, hipStream_t s) {
    auto with = [&](auto exact) {
        constexpr bool X = decltype(exact)::value;
        if (p.bm == 128 && p.bn == 128) return launch_split<128, 128, DIFF, X>(a, p, s);
        if (p.bm == 128 && p.bn == 64) return launch_split<128, 64, DIFF, X>(a, p, s);
        if (p.bm == 64 && p.bn == 128) return launch_split<64, 128, DIFF, X>(a, p, s);
        if (p.bm == 64 && p.bn == 64) return launch_split<64, 64, DIFF, X>(a, p, s);
        return hipErrorInvalidValue;
    };
    return p.exact ? with(std::true_type{}) : with(std::false_type{});
}

// Tile, slices of D and terms, by a cost in microseconds fitted to 22 shapes (J = 40 to 4000, D = 300 to 8192, N = 128 to 11200, every
// tile in two and three terms, one MI355X).  A chunk of 32 columns costs a compute unit (two terms / three) 0.74 / 1.08 us with 256 rows
// staged, 0.58 / 0.78 with 192 and 0.36 / 0.47 with 128 (two 64 x 64 workgroups share a unit; one alone 0.40 / 0.48), every further
// round of 256 workgroups restarts for 1.7 us, and a slice's partial scores are written and read back at about 1.9 TB/s together, one plane after
// the other: 0.1 us more each (3 classes x 3072, 976 samples: 20 slices instead of 27, 14.9 -> 13.0 us; 20 x 5504: 18.7 -> 16.7).
// Two terms start 1 to 2 us later and win from 4 (large tiles) to 16 chunks a workgroup on (over many magnitudes, where they are refused, 1000 x 4096
// with 512 samples takes 33 us with the factor kernel and 27 in two terms).  On 150 shapes the choices are 1.7 % over the best on average; costs
// fitted anew gain 0.4 %, and lose 4 % at 1000 x 4096 with 512.  Below eight chunks (256 columns) they are also the less exact ones:
// products are 7e-8 of the norm off, 8 chunks' running sums 1e-7.
// `most` bounds the bytes of partial scores (the caller's room for them); one slice is always allowed.  exact: three terms; halves: see FwdPlan.
FwdPlan plan_forward_split(int64_t n_rows, int64_t J, int64_t D, size_t most, bool exact, int halves) {
    static const struct { int bm, bn, resident, terms; double start_us, chunk_us, lone_us; } tiles[8] = {
        {128, 128, 1, 2, 8.5, 0.74, 0.74}, {64, 128, 1, 2, 7.4, 0.58, 0.58}, {128, 64, 1, 2, 7.4, 0.58, 0.58}, {64, 64, 2, 2, 7.2, 0.36, 0.40},
        {128, 128, 1, 3, 7.5, 1.08, 1.08}, {64, 128, 1, 3, 5.9, 0.78, 0.78}, {128, 64, 1, 3, 5.9, 0.78, 0.78}, {64, 64, 2, 3, 5.4, 0.47, 0.48}};
    FwdPlan p{};
    p.dma = false;
    p.halves = halves;
    double best = 1e300;
    const int64_t chunks = (D + kSpChunk - 1) / kSpChunk;
    const double plane = (double)n_rows * (double)((J + 3) / 4 * 4) * 4.0;
    for (const auto& t : tiles) {
        if (exact && t.terms == 2) continue;
        const int64_t n = ((n_rows + t.bm - 1) / t.bm) * ((J + t.bn - 1) / t.bn);
        for (int64_t s = 1; s <= 32; ++s) {
            if (s > 1 && (s * 2 > chunks || (double)s * plane > (double)most)) break;
            const int64_t per = (chunks + s - 1) / s, slices = (chunks + per - 1) / per;
            if (slices != s || (t.terms == 2 && per < 8)) continue;
            const double rounds = (double)((n * s + 255) / 256);
            const double deep = (double)((n * s + 256 * t.resident - 1) / (256 * t.resident));
            const double a = t.lone_us * deep, b = t.chunk_us * rounds;
            const double us = t.start_us + (double)per * (a > b ? a : b) + (t.resident == 1 ? 1.7 * (rounds - 1.0) : 0.0) + (double)s * (plane / 1.9e6 + 0.1);
            if (us < best * (1.0 - 1e-9)) {
                best = us;
                p.bm = t.bm; p.bn = t.bn; p.split_k = (int)s;
                p.k_slice = (int)(per * kSpChunk);
                p.grid = (int)(n * s);
                p.exact = t.terms == 3;
            }
        }
    }
    return p;
}

// k_slice of the plan is a multiple of 32.
hipError_t launch_forward_split(const FwdArgs& a, const FwdPlan& p, hipStream_t s) {
    return a.diff ? launch_split_tile<true>(a, p, s) : launch_split_tile<false>(a, p, s);
}

}  // namespace sfb
