// Reconstruction + update (Section 3, Section 2.1) for fp32 factors on the bf16 matrix cores at fp32 accuracy:
//     W[j][d] <- W[j][d] + alpha * sum_n U[n][j] * V[n][d]
// with every operand split exactly into three bf16 terms (sfb_split.h: the arithmetic, its error, and how the two
// groups of wavefronts take turns).
//
// The contraction runs over the factor pairs (the rows of U and V), the slow index of both operands in memory, while
// the matrix instruction wants eight consecutive k per lane.  A lane therefore loads a block of 4 pairs x 4 columns
// (four 16-byte loads, eight lanes to a 128-byte line), and writes per plane four 8-byte items "one column, four
// consecutive pairs".  Two LDS layouts keep the writes of sixteen consecutive lanes and the fragment reads of eight
// off each other's banks: rows of 80 bytes, one per column in order; and, where a wavefront owns two column blocks,
// rows of 64 bytes with a swizzle, column 4 b + e of every 64 in row 16 e + b.  In the second a lane's two blocks
// hold columns two apart and the lane sixteen further the ones between: one v_permlane16_swap per pair of sums and
// a lane has two neighbouring columns of W, 32 lanes 256 contiguous bytes.
// Columns beyond J or D repeat the last four (they feed entries of W that are not stored); pairs beyond N and pairs
// of dead workers are replaced by zero on the way into LDS.  Accesses are 16 (W: 8 or 4) bytes wide at 4-byte
// alignment: any leading dimension is taken.
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

typedef float rs_f32x2u __attribute__((ext_vector_type(2), aligned(4)));

// (three blocks: a strip of 96 rows by one wavefront's 32 columns)
template <int MT, int NT, bool APART>
using ReconTile = SplitTile<MT, NT, NT == 2 ? 64 : 80, NT == 2, APART, MT == 3 ? 1 : 2>;

// column of the tile's A or B part that LDS row r holds
template <int NT>
__device__ __forceinline__ int rs_column(int r) {
    return NT == 2 ? (r & ~63) + 4 * (r & 15) + ((r >> 4) & 3) : r;
}

// PLANES: the workgroups of slice k contract over k_chunks chunks of pairs and store their bare sums in plane k of W
// (a workspace then); apply_partials_kernel adds the planes up.
template <int MT, int NT, bool PLANES, bool APART>
__global__ __launch_bounds__(kSplitThreads, 2) void reconstruct_split_kernel(
    float* __restrict__ W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V,
    int64_t ldv, int J, int D, int N, float alpha, int n_jb, int tiles, int total, int k_chunks, bool halves, int prox_kind, float prox_a,
    uint64_t live_mask, uint32_t inv_b) {
    using Tile = ReconTile<MT, NT, APART>;
    constexpr int BM = Tile::BM, BN = Tile::BN;
    constexpr bool PAIRS = NT == 2;                                      // the permuted layout: two columns of W per lane
    extern __shared__ __attribute__((aligned(16))) unsigned char rs_lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int id = xcd_contiguous_id(blockIdx.x, total);
    const int slice = PLANES ? id / tiles : 0, tile = PLANES ? id % tiles : id;
    const int jb = tile % n_jb, db = tile / n_jb;
    const int j0 = jb * BM, d0 = db * BN;
    const int n_chunks = (N + kSpChunk - 1) / kSpChunk;
    int c_begin = PLANES ? slice * k_chunks : 0;                         // host: no slice is empty
    const int c_end = PLANES ? min(n_chunks, c_begin + k_chunks) : n_chunks;
    const int n_begin = c_begin * kSpChunk, n_end = min(N, c_end * kSpChunk);

    // lane block: pairs 4 kb .. 4 kb + 3, columns 4 rb .. 4 rb + 3 of the BM columns of U and BN of V side by side
    // (four consecutive lanes read 64 contiguous bytes: with lanes of different rows side by side, rows a multiple of 32
    // bytes apart took the loads of a 64 x 64 tile from 24.5 to 33 us at 1024 pairs)
    const int kb = (tid >> 2) & 7, rb = (tid >> 6) * 8 + ((tid >> 5) & 1) * 4 + (tid & 3);
    const bool stages = (BM + BN) * 2 == kSplitThreads || __builtin_amdgcn_readfirstlane(rb) < (BM + BN) / 4;   // by wavefronts
    const bool is_v = __builtin_amdgcn_readfirstlane(rb) >= BM / 4;      // the same for a whole wavefront
    const int ncols = is_v ? D : J;
    const int col = is_v ? d0 + 4 * rb - BM : j0 + 4 * rb;
    const int col_ok = min(col, ncols - 4);                              // host: J, D >= 4
    const int shift = col - col_ok;                                      // 1..3: the words move down by that many columns
    const bool edge = ((J & 3) != 0 && j0 + BM > J) || ((D & 3) != 0 && d0 + BN > D);   // uniform
    const int64_t ld = is_v ? ldv : ldu;
    const unsigned char* src = reinterpret_cast<const unsigned char*>(is_v ? V : U);     // uniform base + 32-bit lane offset
    const uint32_t pitch = (uint32_t)ld * 4u;                            // host: N rows of it stay below 2^32 bytes
    const uint32_t off = (uint32_t)(4 * kb) * pitch + (uint32_t)col_ok * 4u;
    const uint32_t off_last = (uint32_t)(N - 1) * pitch + (uint32_t)col_ok * 4u;
    const int row0 = PAIRS ? (rb >> 4) * 64 + (rb & 15) : 4 * rb;        // LDS row of the first column; the others follow every ROW_STEP
    constexpr int ROW_STEP = PAIRS ? 16 * 64 : 80;
    const int lds_block = PAIRS ? row0 * 64 + 16 * ((kb >> 1) ^ Tile::swz(row0)) + 8 * (kb & 1) : row0 * 80 + 8 * kb;

    struct Raw { f32x4 x[4]; };
    auto fetch = [&](Raw& raw, int c) {
        const uint32_t o = (uint32_t)min(c_begin + c, n_chunks - 1) * (32u * pitch) + off;
#pragma unroll
        for (int i = 0; i < 4; ++i)                                      // pairs beyond N repeat the last one
            raw.x[i] = *reinterpret_cast<const sp_f32x4u*>(src + min(o + i * pitch, off_last));
    };
    auto prep = [&](Raw& raw, int local) {
        const int c = c_begin + local, n0 = c * kSpChunk + 4 * kb;
        if (inv_b != 0) {                                                // some workers are dead (uniform)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t p = __umulhi((uint32_t)min(n0 + i, N - 1), inv_b);
                if (!((live_mask >> p) & 1ull)) raw.x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        if (c * kSpChunk + kSpChunk > N) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n0 + i >= N) raw.x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (edge) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4& x = raw.x[i];
                if (shift & 1) x = f32x4{x[1], x[2], x[3], x[3]};
                if (shift & 2) x = f32x4{x[2], x[3], x[3], x[3]};
            }
        }
    };
    struct State { SplitQuad s; };
    auto park = [&](auto part, const Raw& raw, State& st, unsigned char* buf) {
        constexpr int p = decltype(part)::value, e = p / 4;                          // column
        st.s.template part<p % 4>(raw.x[0][e], raw.x[1][e], raw.x[2][e], raw.x[3][e]);
        if constexpr (p % 4 == 3) {
            if (!stages) return;
            unsigned char* o = buf + lds_block + e * ROW_STEP;
            *reinterpret_cast<uint2*>(o) = make_uint2(st.s.ha, st.s.hb);
            *reinterpret_cast<uint2*>(o + Tile::PLANE) = make_uint2(st.s.ma, st.s.mb);
            *reinterpret_cast<uint2*>(o + 2 * Tile::PLANE) = make_uint2(st.s.la, st.s.lb);
        }
    };

    Tile t;
    t.init(wave, lane);
    // halves: the first half's sums wait in LDS behind the buffers while the second half's start anew
    float* const first = reinterpret_cast<float*>(rs_lds + Tile::LDS) + wave * (MT * NT * 8 * 64) + lane;
    float sum[MT][NT][8];
    if (!PLANES && halves) {
        t.template run<Raw, State, 16, false, 2>(n_chunks / 2, rs_lds, fetch, prep, park);
        c_begin = n_chunks / 2;
        t.exchange(wave, lane, rs_lds, sum);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 8; ++q) first[((i * NT + j) * 8 + q) * 64] = sum[i][j][q];
        split_barrier();                                                 // (the second half's first chunk goes where others still read)
        t.init(wave, lane);
    }
    t.template run<Raw, State, 16, false, 2>(c_end - c_begin, rs_lds, fetch, prep, park);

    // the entries of W this wavefront finishes: requested before the exchange, used after it (requested before the
    // contraction they stand in front of its loads in the in-order queue: 0.3 to 0.8 us slower)
    const int wm = (wave & 3) / Tile::WN, wn = wave % Tile::WN, l32 = lane & 31;
    auto w_row = [&](int i, int q) { return j0 + rs_column<NT>((wm * MT + i) * 32 + Tile::entry_row(wave >> 2, q, lane)); };
    // one column per block, or (PAIRS) the first of two neighbours
    const int dcol = PAIRS ? d0 + wn * 64 + 4 * (l32 & 15) + 2 * (l32 >> 4) : d0 + wn * 32 + l32;
    float w[MT][NT][8];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float* row = W + (int64_t)min(w_row(i, q), J - 1) * ldw;
            if constexpr (PLANES) {
                w[i][0][q] = w[i][NT - 1][q] = 0.f;
            } else if constexpr (PAIRS) {
                const rs_f32x2u x = *reinterpret_cast<const rs_f32x2u*>(row + min(dcol, D - 2));
                w[i][0][q] = dcol > D - 2 ? x.y : x.x;
                w[i][1][q] = x.y;
            } else {
                w[i][0][q] = row[min(dcol, D - 1)];
            }
        }
    t.exchange(wave, lane, rs_lds, sum);
    if (!PLANES && halves) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 8; ++q) sum[i][j][q] += first[((i * NT + j) * 8 + q) * 64];
    }
    t.mend(wave, sum, [&](int i, int j) {
        const int half = lane >> 5;
        const float* u = U + min(j0 + rs_column<NT>((wm * MT + i) * 32 + l32), J - 1);
        const float* v = V + min(d0 + rs_column<NT>((wn * NT + j) * 32 + l32), D - 1);
        f32x16 x;
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = 0.f;
        for (int n0 = n_begin; n0 < n_end; n0 += 16) {
            float p[8], q[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int n = n0 + 2 * c + half;
                const int64_t o = min(n, n_end - 1);
                const bool on = n < n_end && (inv_b == 0 || ((live_mask >> __umulhi((uint32_t)o, inv_b)) & 1ull));
                p[c] = u[o * ldu];
                q[c] = v[o * ldv];
                if (!on) p[c] = q[c] = 0.f;
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) x = split_mfma_f32(p[c], q[c], x);
        }
        return x;
    });
    float* const w_out = W + (PLANES ? (int64_t)slice * J * ldw : 0);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int row = w_row(i, q);
            float* out = w_out + (int64_t)row * ldw + dcol;
            if constexpr (PAIRS) {
                // lanes 16..31 (48..63) give their first block's sum for the second block's of lanes 0..15 (32..47)
                asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(sum[i][0][q]), "+v"(sum[i][1][q]));
                rs_f32x2u x;
                x.x = PLANES ? sum[i][0][q] : prox_entry(w[i][0][q] + alpha * sum[i][0][q], prox_kind, prox_a);
                x.y = PLANES ? sum[i][1][q] : prox_entry(w[i][1][q] + alpha * sum[i][1][q], prox_kind, prox_a);
                if (row < J) {
                    if (dcol + 1 < D) *reinterpret_cast<rs_f32x2u*>(out) = x;
                    else if (dcol < D) *out = x.x;
                }
            } else {
                const float x = PLANES ? sum[i][0][q] : prox_entry(w[i][0][q] + alpha * sum[i][0][q], prox_kind, prox_a);
                if (row < J && dcol < D) *out = x;
            }
        }
}

bool reconstruct_split_ok(const ReconArgs& a) {
    // 32-bit byte offsets into U and V;
    // a masked call finds the worker of a pair with a 32-bit reciprocal of B: exact while N * B < 2^32
    return !a.bf16 && a.J >= 4 && a.D >= 4 && ((int64_t)a.N + 64) * (a.ldu > a.ldv ? a.ldu : a.ldv) < (1LL << 30) &&
           (!a.use_mask || (a.B > 1 && (int64_t)a.N * a.B < (1LL << 32)));
}

template <int MT, int NT, bool PLANES, bool APART>
static hipError_t launch_split(const ReconArgs& a, int slices, bool halves, hipStream_t s) {
    using Tile = ReconTile<MT, NT, APART>;
    constexpr size_t most = Tile::LDS + (PLANES ? 0 : Tile::XCHG);
    static_assert(most <= 160 * 1024, "LDS");
    const size_t lds_bytes = halves ? most : (size_t)Tile::LDS;
    static std::atomic<bool> raised{false};
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)reconstruct_split_kernel<MT, NT, PLANES, APART>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int n_jb = (a.J + Tile::BM - 1) / Tile::BM, n_db = (a.D + Tile::BN - 1) / Tile::BN;
    const int tiles = n_jb * n_db, chunks = (a.N + kSpChunk - 1) / kSpChunk;
    const int k_chunks = (chunks + slices - 1) / slices;
    const uint32_t inv_b = a.use_mask ? (uint32_t)(((1ull << 32) + a.B - 1) / a.B) : 0;
    SFB_LAUNCH((reconstruct_split_kernel<MT, NT, PLANES, APART>), dim3(tiles * slices), dim3(kSplitThreads), lds_bytes, s,
               PLANES ? a.partial : a.w, PLANES ? (int64_t)a.D : a.ldw, a.u, a.ldu, (const float*)a.v, a.ldv, a.J, a.D, a.N,
               a.alpha, n_jb, tiles, tiles * slices, k_chunks, halves, a.prox_kind, a.prox_a, a.live_mask, inv_b);
    return hipGetLastError();
}

// Tile, slices of the pairs and microseconds (the other kernels': reconstruct_fp32_us), fitted to 202 shapes
// (J = 32 to 2000, D = 256 to 8192, N = 64 to 4096) on one MI355X.  A chunk of 32 pairs costs 1.04 / 0.63 us per round
// of 256 tiles of 128 x 128 / 64 x 128 and 0.42 us with 64 x 64 tiles (three share a compute unit), on top of 5.6 us,
// W's trip at 7 TB/s and 2.8 us per further round.  1000 x 4096 (fp32 instruction -> here): 23.1 -> 19.2 us at 256 pairs,
// 40 -> 29.5 at 512, 255 -> 169 at 4096; 600 x 784 with 1024: 32.6 -> 17.5.
// 96 x 128 tiles (0.88 us a chunk) are for the J whose 128-row tiles leave compute units idle or just pass a round of 256: 600 x 4096
// with 1024 pairs 43.0 -> 40.9 us (160 -> 224 workgroups), 576 rows 42.4 -> 38.4, 1001 x 4100 with 488 in place of 64 x 64 tiles 46.6 ->
// 42.7; below 16 chunks they save 2 us at most, and in walks of more than 64 the chip's power sets the pace, not its idle units (2894 x
// 512, 6912 pairs in two slices: 2 % slower).
// Where the tiles leave compute units idle the pairs are cut into slices, at most 64 and as many as `room` bytes hold
// planes of J x D sums for; adding those up is a second kernel.
static SplitReconPlan plan_part(int64_t J, int64_t D, int64_t N, size_t room, bool apart, bool alone) {
    static const struct { int bm, bn, resident; double chunk_us, lone_us; } tiles[4] = {
        {128, 128, 1, 1.04, 1.04}, {96, 128, 1, 0.88, 0.88}, {64, 128, 1, 0.63, 0.63}, {64, 64, 3, 0.42, 0.38}};
    const int64_t chunks = (N + kSpChunk - 1) / kSpChunk;
    SplitReconPlan best{0, 0, 1, apart, 1e300, 0, 0, 0, 0, 1};
    for (const auto& t : tiles) {
        if (apart && t.bm != 64) continue;                                        // (the smaller products' sums apart)
        if (t.bm == 96 && chunks < 16) continue;
        const int64_t n = ((J + t.bm - 1) / t.bm) * ((D + t.bn - 1) / t.bn);
        auto cost = [&](int64_t rows, int64_t cols, int64_t s, int64_t per) {
            const int64_t wgs = ((rows + t.bm - 1) / t.bm) * ((cols + t.bn - 1) / t.bn) * s;
            const double w_mb = 8e-6 * (double)rows * (double)cols, rounds = (double)((wgs + 255) / 256);
            const double deep = (double)((wgs + 256 * t.resident - 1) / (256 * t.resident));
            const double a = t.lone_us * deep, b = t.chunk_us * rounds;
            return 5.6 + (double)per * (a > b ? a : b) + (t.resident == 1 ? 2.8 * (rounds - 1.0) : 0.0) +
                   (s == 1 ? 0.14 * w_mb : 3.5 + 0.1 * (double)s * w_mb);         // planes written and read, W read and written
        };
        for (int64_t s = 1; s <= 64 && (s == 1 || ((size_t)(s * J * D) * sizeof(float) <= room && chunks >= 2 * s && n * s <= 1536)); ++s) {
            const int64_t per = (chunks + s - 1) / s;
            if ((chunks + per - 1) / per != s) continue;                          // the same cut as a smaller count, or an empty slice
            if (t.bm == 96 && per > 64) continue;
            const double us = cost(J, D, s, per);
            if (us < best.us) best = SplitReconPlan{t.bm, t.bn, (int)s, apart, us, 0, 0, 0, 0, 1};
        }
        if (!alone || t.resident != 1 || (t.bm == 96 && chunks > 64)) continue;
        const int64_t rows = (J - 4) / t.bm * t.bm, cols = (D - 4) / t.bn * t.bn; // (a launch takes four rows and columns and more)
        if (cols > 0 && (((J + t.bm - 1) / t.bm) * (cols / t.bn) + 255) / 256 < (n + 255) / 256) {
            const SplitReconPlan rest = plan_part(J, D - cols, N, room, apart, false);
            const double us = cost(J, cols, 1, chunks) + rest.us;
            if (us < 0.97 * best.us) best = SplitReconPlan{t.bm, t.bn, 1, apart, us, 0, (int)cols, rest.bm, rest.bn, rest.slices};
        }
        if (rows > 0 && ((rows / t.bm) * ((D + t.bn - 1) / t.bn) + 255) / 256 < (n + 255) / 256) {
            const SplitReconPlan rest = plan_part(J - rows, D, N, room, apart, false);
            const double us = cost(rows, D, 1, chunks) + rest.us;
            if (us < 0.97 * best.us) best = SplitReconPlan{t.bm, t.bn, 1, apart, us, (int)rows, 0, rest.bm, rest.bn, rest.slices};
        }
    }
    return best;
}
// Where the last row or column of tiles is what begins another round of 256, it is a second, smaller launch with a plan of its
// own (1001 x 4100, 488 pairs: 256 tiles of 128 x 128 and four columns, 42.7 -> 39.3 us; 1001 x 4129, 1000: 88.6 -> 59.7).
SplitReconPlan reconstruct_split_plan(int64_t J, int64_t D, int64_t N, size_t room, bool apart) { return plan_part(J, D, N, room, apart, true); }

template <int MT, int NT, bool APART>
static hipError_t launch_tile(const ReconArgs& a, int slices, bool halves, hipStream_t s) {
    if (slices == 1) return launch_split<MT, NT, false, APART>(a, 1, halves, s);
    const hipError_t e = launch_split<MT, NT, true, APART>(a, slices, false, s);
    return e != hipSuccess ? e : launch_apply_partials(a, slices, a.D, s);
}

static hipError_t launch_part(const ReconArgs& a, int bm, int bn, int slices, bool apart, bool halves, hipStream_t s) {
    if (slices < 1 || (slices > 1 && a.partial == nullptr)) return hipErrorInvalidValue;
    if (apart) {
        if (bm == 64 && bn == 128) return launch_tile<1, 2, true>(a, slices, halves, s);
        if (bm == 64 && bn == 64) return launch_tile<1, 1, true>(a, slices, halves, s);
        return hipErrorInvalidValue;
    }
    if (bm == 128 && bn == 128) return launch_tile<2, 2, false>(a, slices, halves, s);
    if (bm == 96 && bn == 128) return launch_tile<3, 1, false>(a, slices, halves, s);
    if (bm == 64 && bn == 128) return launch_tile<1, 2, false>(a, slices, halves, s);
    if (bm == 64 && bn == 64) return launch_tile<1, 1, false>(a, slices, halves, s);
    return hipErrorInvalidValue;
}

// plan.slices > 1 (or rest_slices): a.partial holds that many planes of J x D (of the rest's rows and columns) floats
hipError_t launch_reconstruct_split(const ReconArgs& a, const SplitReconPlan& p, bool halves, hipStream_t s) {
    halves = halves && a.N > 4 * kSpChunk;                               // two chunks or more in each
    if (p.main_rows == 0 && p.main_cols == 0) return launch_part(a, p.bm, p.bn, p.slices, p.apart, halves, s);
    ReconArgs b = a;
    if (p.main_rows > 0) b.J = p.main_rows;
    else b.D = p.main_cols;
    const hipError_t e = launch_part(b, p.bm, p.bn, p.slices, p.apart, halves, s);
    if (e != hipSuccess) return e;
    const LaunchEvents main = launch_events();                           // the launch that is reported as the family's
    b = a;
    b.w += (int64_t)p.main_rows * a.ldw + p.main_cols;
    b.u += p.main_rows;
    b.v = (const float*)a.v + p.main_cols;
    b.J -= p.main_rows;
    b.D -= p.main_cols;
    const hipError_t e2 = launch_part(b, p.rest_bm, p.rest_bn, p.rest_slices, p.apart, halves && p.rest_slices == 1, s);
    launch_events().name = main.name;
    launch_events().blocks = main.blocks;
    return e2;
}

}  // namespace sfb
