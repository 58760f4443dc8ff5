// Scores (Section 2, z = W a) for fp32 features on the bf16 matrix cores at fp32 accuracy: Z[n][j] = sum_d A[n][d] *
// W[j][d] with every operand split exactly into three bf16 terms (sfb_split.h: the arithmetic, its error, and how the
// two groups of wavefronts take turns).
//
// Both operands are contiguous along the contraction.  A lane loads 16 bytes (four k) of a row of A or W, eight lanes to
// a 128-byte line, splits them and writes 8 bytes per plane, so W is never copied and A passes through
// once more only to be stored as V.  Rows beyond the matrix repeat the last row (their scores are not stored); in the
// last, partial chunk of D the words beyond D are replaced by zero in both operands.  Accesses are 16 bytes wide at
// 4-byte alignment: any leading dimension is taken.  DIFF: the operand is x_i - y_i (metric learning).
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

template <int MT, int NT, bool DIFF, bool APART>
__global__ __launch_bounds__(kSplitThreads, 2) void scores_split_kernel(
    const float* __restrict__ A, const float* __restrict__ A2, int64_t lda, const float* __restrict__ W, int64_t ldw,
    float* __restrict__ Z, int64_t ldz, int64_t zstride, float* __restrict__ Vout, int64_t ldv, int M, int N, int K,
    int k_slice, int n_mb, int n_nb, int total) {
    using Tile = SplitTile<MT, NT, 64, true, APART>;
    constexpr int BM = Tile::BM, BN = Tile::BN;
    constexpr int A_IT = BM / 64, IT = (BM + BN) / 64;                   // 16-byte items per lane and chunk: of A, of A and W
    extern __shared__ __attribute__((aligned(16))) unsigned char ss_lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // consecutive ids share the class block (its W rows then sit in one die's L2)
    int id = xcd_contiguous_id(blockIdx.x, total);
    const int mb = id % n_mb;
    id /= n_mb;
    const int nb = id % n_nb, ks = id / n_nb;
    const int m0 = mb * BM, n0 = nb * BN;
    const int k_begin = ks * k_slice, k_end = min(K, k_begin + k_slice);
    const int n_chunks = (k_end - k_begin + kSpChunk - 1) / kSpChunk;
    const bool ragged = (K & 31) != 0 && k_end == K;                     // the last chunk is partial

    // item i of a lane: row r0 + 64 i of the A rows followed by the W rows, k 4 c0 .. 4 c0 + 3 of the chunk
    const int r0 = tid >> 3, c0 = tid & 7;
    const unsigned char* const a_base = reinterpret_cast<const unsigned char*>(A + (int64_t)m0 * lda);
    const unsigned char* const a2_base = DIFF ? reinterpret_cast<const unsigned char*>(A2 + (int64_t)m0 * lda) : nullptr;
    const unsigned char* const w_base = reinterpret_cast<const unsigned char*>(W + (int64_t)n0 * ldw);
    uint32_t off[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i)
        off[i] = i < A_IT ? (uint32_t)min(r0 + 64 * i, M - 1 - m0) * (uint32_t)lda * 4u
                          : (uint32_t)min(r0 + 64 * i - BM, N - 1 - n0) * (uint32_t)ldw * 4u;
    // rows r0 + 64 i share the swizzle
    const int lds_item = r0 * 64 + 16 * ((c0 >> 1) ^ Tile::swz(r0)) + 8 * (c0 & 1);

    struct Raw { f32x4 x[IT], y[DIFF ? A_IT : 1]; };
    auto ld = [](const unsigned char* p) -> f32x4 { return *reinterpret_cast<const sp_f32x4u*>(p); };
    auto fetch = [&](Raw& raw, int c) {
        // in a partial chunk the words are read from the last four of the row and moved into place by prep (host: K >= 4)
        const uint32_t o = (uint32_t)min(k_begin + min(c, n_chunks - 1) * kSpChunk + 4 * c0, K - 4) * 4u;
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            raw.x[i] = ld((i < A_IT ? a_base : w_base) + (off[i] + o));
            if (DIFF && i < A_IT) raw.y[i] = ld(a2_base + (off[i] + o));
        }
    };
    // the class blocks share the copy of A (or X - Y) into V: block nb takes the chunks c with c % n_nb == nb
    const bool write_v = Vout != nullptr;
    auto prep = [&](Raw& raw, int c) {
        const int k0 = k_begin + c * kSpChunk + 4 * c0;
        const bool last = ragged && c == n_chunks - 1;
        if (DIFF) {
#pragma unroll
            for (int i = 0; i < A_IT; ++i) raw.x[i] -= raw.y[i];
        }
        if (last) {                                                      // words read early move up, zeros beyond D
            const int sh = max(0, k0 - (K - 4));
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                f32x4& x = raw.x[i];
                if (sh & 1) x = f32x4{x[1], x[2], x[3], 0.f};
                if (sh & 2) x = f32x4{x[2], x[3], 0.f, 0.f};
                if (sh >= 4) x = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        if (write_v && (c % n_nb) == nb && c < n_chunks) {               // v_i = a_i (or x_i - y_i)
#pragma unroll
            for (int i = 0; i < A_IT; ++i) {
                if (m0 + r0 + 64 * i >= M) continue;
                float* out = Vout + (int64_t)(m0 + r0 + 64 * i) * ldv + k0;
                if (!last || k0 + 4 <= K) {
                    *reinterpret_cast<sp_f32x4u*>(out) = raw.x[i];
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (k0 + e < K) out[e] = raw.x[i][e];
                }
            }
        }
    };
    struct State { SplitQuad s; };
    auto park = [&](auto part, const Raw& raw, State& st, unsigned char* buf) {
        constexpr int p = decltype(part)::value, i = p / 4;                          // item
        st.s.template part<p % 4>(raw.x[i][0], raw.x[i][1], raw.x[i][2], raw.x[i][3]);
        if constexpr (p % 4 == 3) {
            unsigned char* o = buf + lds_item + i * 64 * 64;
            *reinterpret_cast<uint2*>(o) = make_uint2(st.s.ha, st.s.hb);
            *reinterpret_cast<uint2*>(o + Tile::PLANE) = make_uint2(st.s.ma, st.s.mb);
            *reinterpret_cast<uint2*>(o + 2 * Tile::PLANE) = make_uint2(st.s.la, st.s.lb);
        }
    };

    Tile t;
    t.init(wave, lane);
    t.template run<Raw, State, 4 * IT, true, (IT <= 3 && !DIFF) || IT == 2 ? 4 : 2>(n_chunks, ss_lds, fetch, prep, park);

    float sum[MT][NT][8];
    t.exchange(wave, lane, ss_lds, sum);
    const int wm = (wave & 3) >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
    t.mend(wave, sum, [&](int i, int j) {
        const int64_t row = min(m0 + (wm * MT + i) * 32 + l32, M - 1), col = min(n0 + (wn * NT + j) * 32 + l32, N - 1);
        const float *a = A + row * lda, *a2 = DIFF ? A2 + row * lda : nullptr, *w = W + col * ldw;
        f32x16 x;
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = 0.f;
        int k = k_begin;
        for (; k + kSpChunk <= k_end; k += kSpChunk) {                   // any order of k will do: four for each half of the lanes
            f32x4 p[4], q[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int o = k + 8 * c + 4 * half;
                p[c] = *reinterpret_cast<const sp_f32x4u*>(a + o);
                if (DIFF) p[c] -= *reinterpret_cast<const sp_f32x4u*>(a2 + o);
                q[c] = *reinterpret_cast<const sp_f32x4u*>(w + o);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) x = split_mfma_f32(p[c][e], q[c][e], x);
        }
        for (; k < k_end; k += 2) {
            const int o = min(k + half, k_end - 1);
            const bool on = k + half < k_end;
            x = split_mfma_f32(on ? (DIFF ? a[o] - a2[o] : a[o]) : 0.f, on ? w[o] : 0.f, x);
        }
        return x;
    });
    float* zout = Z + (int64_t)ks * zstride;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int col = n0 + (wn * NT + j) * 32 + l32;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int row = m0 + (wm * MT + i) * 32 + Tile::entry_row(wave >> 2, q, lane);
                if (row < M && col < N) zout[(int64_t)row * ldz + col] = sum[i][j][q];
            }
    }
}

bool forward_split_ok(const FwdArgs& a) {
    // lane offsets (up to 128 rows of 4-byte words) stay below 2^32
    return !a.bf16 && a.D >= 4 && a.lda < (1 << 22) && a.ldw < (1 << 22);
}

template <int MT, int NT, bool DIFF, bool APART>
static hipError_t launch_split(const FwdArgs& a, const FwdPlan& p, hipStream_t s) {
    using Tile = SplitTile<MT, NT, 64, true, APART>;
    constexpr size_t lds_bytes = Tile::LDS;
    static std::atomic<bool> raised{false};
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)scores_split_kernel<MT, NT, DIFF, APART>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int n_mb = (a.n_rows + Tile::BM - 1) / Tile::BM, n_nb = (a.J + Tile::BN - 1) / Tile::BN;
    const int total = n_mb * n_nb * p.split_k;
    SFB_LAUNCH((scores_split_kernel<MT, NT, DIFF, APART>), dim3(total), dim3(kSplitThreads), lds_bytes, s, (const float*)a.a,
               (const float*)a.a2, a.lda, a.w, a.ldw, a.zp, a.ldz, a.zstride, (float*)a.v, a.ldv, a.n_rows, a.J, a.D,
               p.k_slice, n_mb, n_nb, total);
    return hipGetLastError();
}

template <bool DIFF>
static hipError_t launch_split_tile(const FwdArgs& a, const FwdPlan& p, hipStream_t s) {
    if (p.apart) {
        if (p.bm == 64 && p.bn == 128) return launch_split<1, 2, DIFF, true>(a, p, s);
        if (p.bm == 64 && p.bn == 64) return launch_split<1, 1, DIFF, true>(a, p, s);
        return hipErrorInvalidValue;
    }
    if (p.bm == 128 && p.bn == 128) return launch_split<2, 2, DIFF, false>(a, p, s);
    if (p.bm == 128 && p.bn == 64) return launch_split<2, 1, DIFF, false>(a, p, s);
    if (p.bm == 64 && p.bn == 128) return launch_split<1, 2, DIFF, false>(a, p, s);
    if (p.bm == 64 && p.bn == 64) return launch_split<1, 1, DIFF, false>(a, p, s);
    return hipErrorInvalidValue;
}

// Tile and slices of D, by a cost in microseconds fitted to 202 shapes (J = 32 to 2000, D = 256 to 8192, N = 64 to 4096,
// four tiles, up to three slice counts each, one MI355X; the choice is within 2 % of the best measured one on average):
// a chunk of 32 columns costs a compute unit 1.10 / 0.72 / 0.40 us with 256 / 192 / 128 rows staged (the small tiles
// pay more LDS traffic per product), three 64 x 64 workgroups share a unit, every further round of 256 workgroups
// restarts for 1.7 us, and a slice's partial scores are written and read back at about 2.2 TB/s together, one plane after
// the other: 0.1 us more each (3 classes x 3072, 976 samples: 20 slices instead of 27, 14.9 -> 13.0 us; 20 x 5504: 18.7 -> 16.7).
// `most` bounds the bytes of partial scores (the caller's room for them); one slice is always allowed.  apart: the tiles of
// 64 samples (the smaller products' sums apart).
FwdPlan plan_forward_split(int64_t n_rows, int64_t J, int64_t D, size_t most, bool apart) {
    static const struct { int bm, bn, resident; double chunk_us, lone_us; } tiles[4] = {
        {128, 128, 1, 1.10, 1.10}, {64, 128, 1, 0.72, 0.72}, {128, 64, 1, 0.72, 0.72}, {64, 64, 3, 0.40, 0.44}};
    FwdPlan p{};
    p.dma = false;
    double best = 1e300;
    const int64_t chunks = (D + kSpChunk - 1) / kSpChunk;
    const double plane = (double)n_rows * (double)((J + 3) / 4 * 4) * 4.0;
    p.apart = apart;
    for (const auto& t : tiles) {
        if (apart && t.bm != 64) continue;
        const int64_t n = ((n_rows + t.bm - 1) / t.bm) * ((J + t.bn - 1) / t.bn);
        for (int64_t s = 1; s <= 32; ++s) {
            if (s > 1 && (s * 2 > chunks || (double)s * plane > (double)most)) break;
            const int64_t per = (chunks + s - 1) / s, slices = (chunks + per - 1) / per;
            if (slices != s) continue;
            const double rounds = (double)((n * s + 255) / 256);
            const double deep = (double)((n * s + 256 * t.resident - 1) / (256 * t.resident));
            const double a = t.lone_us * deep, b = t.chunk_us * rounds;
            const double us = (double)per * (a > b ? a : b) + (t.resident == 1 ? 1.7 * (rounds - 1.0) : 0.0) + (double)s * (plane / 2.2e6 + 0.1);
            if (us < best * (1.0 - 1e-9)) {
                best = us;
                p.bm = t.bm; p.bn = t.bn; p.split_k = (int)s;
                p.k_slice = (int)(per * kSpChunk);
                p.grid = (int)(n * s);
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
