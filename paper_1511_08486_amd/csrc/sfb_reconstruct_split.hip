// Reconstruction + update (Section 3, Section 2.1) for fp32 factors on the 16-bit matrix cores at fp32 accuracy:
//     W[j][d] <- W[j][d] + alpha * sum_n U[n][j] * V[n][d]
// with every operand split into terms (sfb_split.h: the arithmetic, its error, and the two kinds of wavefronts).
//
// The contraction runs over the factor pairs (the rows of U and V), the slow index of both operands in memory, while
// the matrix instruction wants eight consecutive k per lane.  A splitting lane therefore loads a block of 4 pairs x 4 (2) columns
// and writes per plane four (two) 8-byte items "one column, four consecutive pairs".  Column 4 b + e of every 64 sits in LDS row 16 e + b (2 b
// + e of every 32 in row 16 e + b, where blocks are two columns wide): the writes of sixteen lanes and the fragment reads of eight stay
// off each other's banks, and a multiplying lane's blocks hold neighbouring columns of W, which it reads and writes in one 16- or 8-byte access.
// Columns beyond J or D repeat the last ones (they feed entries of W that are not stored); pairs beyond N lie behind the end of the
// descriptors and read as zero, pairs of dead workers are replaced by zero on the way into LDS.  Any alignment and leading dimension is taken.
// us, every wavefront splitting and multiplying in three terms -> here: 1000 x 4096, 512 pairs 31.3 -> 24.5; 600 x 4096, 1024 43.7 -> 31.1; 1000 x 4096, 4096
// 169 -> 115; refused by two terms 29.5 -> 27.5, 169 -> 167.
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

// SPLITTERS: eight, or four in 64 x 64 tiles of which several share a compute unit (first measured at 800 x 2500, 200 pairs, 520 tiles: 15.2 us, 19.0
// with eight; 333 x 1001 with 228, 96 tiles: 11.6 and 9.4)
template <int BM, int BN, int SPLITTERS, bool EXACT>
using ReconTile = SplitTile<BM, BN, BM == 128 ? 4 : 2, BM == 96 ? 4 : 2, SPLITTERS, EXACT>;

// column of the tile's A part (U) and of its B part (V) that LDS row r holds; CB: columns of a splitting lane's block
template <int BM, int CB>
__device__ __forceinline__ int rs_u(int r) { return CB == 2 ? split_row16(r) : BM % 64 == 0 ? split_row64(r) : split_row32(r); }
template <int CB>
__device__ __forceinline__ int rs_v(int r) { return CB == 2 ? split_row16(r) : split_row64(r); }

// PLANES: the workgroups of slice k contract over k_chunks chunks of pairs and store their bare sums in plane k of W
// (a workspace then); apply_partials_kernel adds the planes up.
template <int BM, int BN, int SPLITTERS, bool PLANES, bool EXACT>
__global__ __launch_bounds__((ReconTile<BM, BN, SPLITTERS, EXACT>::THREADS), BM + BN == 128 ? (SPLITTERS == 8 ? 6 : 4) : BM + BN == 192 ? 3 : 4) void reconstruct_split_kernel(
    float* __restrict__ W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V,
    int64_t ldv, int J, int D, int N, float alpha, int n_jb, int tiles, int total, int k_chunks, int halves, int prox_kind, float prox_a,
    uint64_t live_mask, uint32_t inv_b) {
    using Tile = ReconTile<BM, BN, SPLITTERS, EXACT>;
    constexpr int CB = BM + BN == 128 && SPLITTERS == 8 ? 2 : 4;         // columns of a splitting lane's block
    extern __shared__ __attribute__((aligned(16))) unsigned char rs_lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int id = xcd_contiguous_id(blockIdx.x, total);
    const int slice = PLANES ? id / tiles : 0, tile = PLANES ? id % tiles : id;
    const int jb = tile % n_jb, db = tile / n_jb;
    const int j0 = jb * BM, d0 = db * BN;
    const int all_chunks = (N + kSpChunk - 1) / kSpChunk;
    const int c_begin = PLANES ? slice * k_chunks : 0;                   // host: no slice is empty
    const int c_end = PLANES ? min(all_chunks, c_begin + k_chunks) : all_chunks, n_chunks = c_end - c_begin;
    const int n_begin = c_begin * kSpChunk, n_end = min(N, c_end * kSpChunk);

    if (wave >= Tile::MULTIPLIERS) {
        // Lane block: pairs 4 kb .. 4 kb + 3, columns c0 .. c0 + CB - 1 of the BM columns of U and BN of V side by side; consecutive lanes
        // read 64 contiguous bytes (with lanes of different rows side by side, rows a multiple of 32
        // bytes apart took the loads of a 64 x 64 tile from 24.5 to 33 us at 1024 pairs).
        const int tid = threadIdx.x - 64 * Tile::MULTIPLIERS, first = 8 * CB * (wave - Tile::MULTIPLIERS);
        const int kb = CB == 4 ? (tid >> 2) & 7 : (tid >> 3) & 7;
        const int c0 = first + (CB == 4 ? 16 * ((tid >> 5) & 1) + 4 * (tid & 3) : 2 * (tid & 7));
        const bool edge = ((J & (CB - 1)) != 0 && j0 + BM > J) || ((D & (CB - 1)) != 0 && d0 + BN > D);   // uniform
        const bool on[1] = {first < BM + BN}, is_v[1] = {first >= BM};   // the same for a whole wavefront
        const int ncols = is_v[0] ? D : J;
        const int col = is_v[0] ? d0 + c0 - BM : j0 + c0;
        const int col_ok = min(col, ncols - CB);                         // host: J, D >= 4
        const int shift = col - col_ok;                                  // up to CB - 1: the words move down by that many columns
        const uint32_t pitch = (uint32_t)(is_v[0] ? ldv : ldu) * 4u;     // host: N rows of it stay below 2^32 bytes
        const unsigned char* const src = reinterpret_cast<const unsigned char*>(is_v[0] ? V : U) + (uint64_t)n_begin * pitch;
        const uint32_t bytes = (uint32_t)(N - 1 - n_begin) * pitch + (uint32_t)ncols * 4u;   // pairs beyond N read as zero
        uint32_t off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) off[i] = (uint32_t)(4 * kb + i) * pitch + (uint32_t)col_ok * 4u;
        int lds_at[CB];
#pragma unroll
        for (int e = 0; e < CB; ++e) {                                   // the LDS row of column c: the inverse of rs_u and rs_v
            const int c = c0 + e - (is_v[0] ? BM : 0);
            const int by = CB == 2 ? (c & ~31) + 16 * (c & 1) + ((c & 31) >> 1)
                                   : is_v[0] || BM % 64 == 0 ? (c & ~63) + 16 * (c & 3) + ((c & 63) >> 2) : (c & ~31) + 8 * (c & 3) + ((c & 31) >> 2);
            const int row = by + (is_v[0] ? BM : 0);
            lds_at[e] = row * 64 + 16 * ((kb >> 1) ^ Tile::swz(row)) + 8 * (kb & 1);
        }

        typedef float f32_cb __attribute__((ext_vector_type(CB)));
        struct Raw { f32_cb x[4]; };
        auto where = [&](int c, auto) {
            const uint32_t gone = (uint32_t)c * (32u * pitch);
            return split_words(src + gone, on[0] ? (bytes - gone) & split_while(c, n_chunks) : 0u);
        };
        auto load = [&](Raw& raw, const __amdgpu_buffer_rsrc_t& words, auto uc, auto) {
            if constexpr (CB == 4) {
                constexpr int i = 2 * decltype(uc)::value;
                raw.x[i] = split_load4(words, off[i]);
                raw.x[i + 1] = split_load4(words, off[i + 1]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) raw.x[i] = split_load2(words, off[i]);
            }
        };
        auto prep = [&](Raw& raw, int c, auto) {
            if (inv_b != 0) {                                            // some workers are dead (uniform)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t p = __umulhi((uint32_t)min(n_begin + c * kSpChunk + 4 * kb + i, N - 1), inv_b);
                    if (!((live_mask >> p) & 1ull)) raw.x[i] = f32_cb(0.f);
                }
            }
            if (edge) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f32_cb& x = raw.x[i];
                    if constexpr (CB == 4) {
                        if (shift & 1) x = f32x4{x[1], x[2], x[3], x[3]};
                        if (shift & 2) x = f32x4{x[2], x[3], x[3], x[3]};
                    } else {
                        if (shift & 1) x[0] = x[1];
                    }
                }
            }
        };
        auto take = [](const Raw& raw, auto ic) -> f32x4 {               // column by column
            constexpr int e = decltype(ic)::value;
            return f32x4{raw.x[0][e], raw.x[1][e], raw.x[2][e], raw.x[3][e]};
        };
        auto put = [&](unsigned char* buf, auto plane, auto ic, uint2 words) {
            *reinterpret_cast<uint2*>(buf + lds_at[decltype(ic)::value] + decltype(plane)::value * Tile::PLANE) = words;
        };
        Tile::template split<Raw, CB, 1, (CB == 4 ? 2 : 0)>(n_chunks, rs_lds, is_v, on, [](auto) { return std::integral_constant<int, 0>{}; }, where, load,
                                              prep, take, put);
        return;
    }

    Tile t;
    t.init(wave, lane);
    t.multiply(n_chunks, halves, rs_lds);

    // The entries of W this wavefront finishes: four (two) neighbouring columns a row.  A scalar address a row and one lane offset (host: 50
    // rows of W below 2^32 bytes) where the tile is whole.
    constexpr int WIDE = Tile::NB < 4 ? Tile::NB : 4;
    typedef float f32_wide __attribute__((ext_vector_type(WIDE), aligned(4)));
    const int wm = wave / Tile::WN, wn = wave % Tile::WN, l16 = lane & 15, quarter = lane >> 4;
    const int lane_row = CB == 2 ? 8 * quarter : BM % 64 == 0 ? 16 * quarter : 16 * (quarter & 1) + (quarter >> 1);
    auto row_of = [&](int i, int e) { return rs_u<BM, CB>((wm * Tile::MB + i) * 16 + e); };           // + lane_row
    // (two blocks of a wavefront in rows by split_row64: every other pair of columns is its neighbour's)
    constexpr bool EVERY_OTHER = WIDE == 2 && CB == 4;
    const int lane_col = EVERY_OTHER ? 4 * l16 + 2 * (wn & 1) : WIDE * l16;
    const int first_col = d0 + (EVERY_OTHER ? (wn >> 1) * 64 : wn * 16 * WIDE), col = first_col + lane_col;
    static_assert(Tile::NB <= 4, "columns");
    const bool inside = j0 + BM <= J && d0 + BN <= D, whole = col + WIDE <= D;   // of the tile, of this lane's columns
    const uint32_t w_lane = (uint32_t)lane_row * (uint32_t)ldw * 4u + (uint32_t)lane_col * 4u;
    float* const w_out = W + (PLANES ? (int64_t)slice * J * ldw : 0);
    auto w_at = [&](int i, int e) {
        float* base = w_out + (int64_t)(j0 + row_of(i, e)) * ldw + first_col;
        return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + w_lane);
    };
    // (a tile that is not: no load under a condition, which would be waited for before the next.  Rows beyond J read an earlier
    // one, columns beyond D the row's last words: 36 x 541, 192 pairs 7.8 us, entry by entry 7.9)
    f32_wide w[Tile::MB][4];
    const bool part = !inside && d0 + BN > D && D % WIDE != 0;               // some lane's columns end within its words (uniform)
    if constexpr (!PLANES) {
        const int col_ok = min(col, D - WIDE);                               // host: D >= 4
        const uint32_t col_bytes = (uint32_t)col_ok * 4u, lane_bytes = (uint32_t)lane_row * (uint32_t)ldw * 4u + col_bytes;
#pragma unroll
        for (int i = 0; i < Tile::MB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* base = W + (int64_t)min(j0 + row_of(i, e), J - 1) * ldw;
                const uint32_t bytes = j0 + row_of(i, e) + lane_row < J ? lane_bytes : col_bytes;
                if (inside) w[i][e] = *reinterpret_cast<const f32_wide*>(w_at(i, e));
                else w[i][e] = *reinterpret_cast<const f32_wide*>(reinterpret_cast<const char*>(base) + bytes);
            }
        if (part) {
            const int early = col - col_ok;                                  // the words come down by that many
#pragma unroll
            for (int i = 0; i < Tile::MB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f32_wide& x = w[i][e];
                    if (early & 1) {
#pragma unroll
                        for (int j = 0; j + 1 < WIDE; ++j) x[j] = x[j + 1];
                    }
                    if constexpr (WIDE == 4)
                        if (early & 2) x[0] = x[2], x[1] = x[3];
                }
        }
    }
    t.mend([&](int i, int j) {
        const float* u = U + min(j0 + rs_u<BM, CB>((wm * Tile::MB + i) * 16 + l16), J - 1);
        const float* v = V + min(d0 + rs_v<CB>((wn * Tile::NB + j) * 16 + l16), D - 1);
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        for (int n0 = n_begin; n0 < n_end; n0 += 16) {
            float p[4], q[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int n = n0 + 4 * c + quarter;
                const int64_t o = min(n, n_end - 1);
                const bool on = n < n_end && (inv_b == 0 || ((live_mask >> __umulhi((uint32_t)o, inv_b)) & 1ull));
                p[c] = u[o * ldu];
                q[c] = v[o * ldv];
                if (!on) p[c] = q[c] = 0.f;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) x = split_mfma16_f32(p[c], q[c], x);
        }
        return x;
    });
    auto store = [&](auto all) {
#pragma unroll
        for (int i = 0; i < Tile::MB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f32_wide x;
#pragma unroll
                for (int j = 0; j < WIDE; ++j)
                    x[j] = PLANES ? t.acc[i][j][e] : prox_entry(w[i][e][j] + alpha * t.acc[i][j][e], prox_kind, prox_a);
                if (decltype(all)::value) {
                    *reinterpret_cast<f32_wide*>(w_at(i, e)) = x;
                } else if (j0 + row_of(i, e) + lane_row < J) {
                    if (whole) *reinterpret_cast<f32_wide*>(w_at(i, e)) = x;
                    if (part && !whole) {
#pragma unroll
                        for (int j = 0; j + 1 < WIDE; ++j)
                            if (col + j < D) w_at(i, e)[j] = x[j];
                    }
                }
            }
    };
    if (inside) store(std::true_type{});
    else store(std::false_type{});
}

bool reconstruct_split_ok(const ReconArgs& a) {
    // 32-bit byte offsets into U and V;
    // a masked call finds the worker of a pair with a 32-bit reciprocal of B: exact while N * B < 2^32
    return !a.bf16 && a.J >= 4 && a.D >= 4 && a.ldw < (1 << 24) && ((int64_t)a.N + 64) * (a.ldu > a.ldv ? a.ldu : a.ldv) < (1LL << 30) &&
           (!a.use_mask || (a.B > 1 && (int64_t)a.N * a.B < (1LL << 32)));
}

template <int BM, int BN, int SPLITTERS, bool PLANES, bool EXACT>
static hipError_t launch_split(const ReconArgs& a, int slices, int halves, hipStream_t s) {
    using Tile = ReconTile<BM, BN, SPLITTERS, EXACT>;
    constexpr size_t lds_bytes = Tile::LDS;
    static std::atomic<bool> raised{false};
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)reconstruct_split_kernel<BM, BN, SPLITTERS, PLANES, EXACT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int n_jb = (a.J + Tile::BM - 1) / Tile::BM, n_db = (a.D + Tile::BN - 1) / Tile::BN;
    const int tiles = n_jb * n_db, chunks = (a.N + kSpChunk - 1) / kSpChunk;
    const int k_chunks = (chunks + slices - 1) / slices;
    const uint32_t inv_b = a.use_mask ? (uint32_t)(((1ull << 32) + a.B - 1) / a.B) : 0;
    SFB_LAUNCH((reconstruct_split_kernel<BM, BN, SPLITTERS, PLANES, EXACT>), dim3(tiles * slices), dim3(Tile::THREADS), lds_bytes, s,
               PLANES ? a.partial : a.w, PLANES ? (int64_t)a.D : a.ldw, a.u, a.ldu, (const float*)a.v, a.ldv, a.J, a.D, a.N,
               a.alpha, n_jb, tiles, tiles * slices, k_chunks, halves, a.prox_kind, a.prox_a, a.live_mask, inv_b);
    return hipGetLastError();
}

// Tile, slices of the pairs, terms and microseconds (the other kernels': reconstruct_fp32_us), fitted to 150 shapes (J = 6 to 4000, D = 50
// to 8192, N = 66 to 12000, every tile in two and three terms with up to ten counts of slices) on one MI355X: 1.8 % over the best of them on average.
// A chunk of 32 pairs costs (two terms / three) 0.88 / 1.02 us per round of 256 tiles of 128 x 128, 0.76 / 0.91 with 96 x 128, 0.68 / 0.82 with 64 x
// 128 and 0.34 / 0.39 with 64 x 64 tiles where two share a compute unit (0.44 / 0.46 alone), on top of 5 to 6.5 us, W's trip (0.12 us a MB, read and
// written) and up to 1.8 us per further round.  1000 x 4096 (fp32 instruction -> here): 22.5 -> 16.9 us at 256 pairs, 39.8 -> 24.5 at 512; 600 x 780
// with 1024: 32.1 -> 15.8; 2000 x 8192 with 80: 67 -> 40.
// Two terms win from 4 (64 x 64: 13) chunks a workgroup on (1000 x 4096 with 512 pairs 24.5 against 26.6 us); below four chunks (128 pairs) they are
// also the less exact ones.
// 96 x 128 tiles are for the J whose 128-row tiles leave compute units idle or just pass a round of 256 (600 x 4096 with 1024 pairs: 160 -> 224
// workgroups); below 16 chunks they save 2 us at most, and in walks of more than 64 the chip's power sets the pace, not its
// idle units (2894 x 512, 6912 pairs in two slices: 2 % slower).
// Where the tiles leave compute units idle the pairs are cut into slices, at most 64 and as many as `room` bytes hold
// planes of J x D sums for; adding those up is a second kernel, 1.3 us and its traffic, and what the next score pass waits longer for W then: D / 1500 us, 2.4 at
// most (steps of 40 x 7383 with 322 pairs 24.8 us in one piece and 27.4 in two slices, updates 10.3 both; 193 x 1473 with 476: 23.2 and 23.3, 11.5 and 10.7;
// 216 x 268 with 384: 18.9 and, in four, 17.4, 10.2 and 8.6).
static SplitReconPlan plan_part(int64_t J, int64_t D, int64_t N, size_t room, bool exact, bool alone) {
    static const struct { int bm, bn, resident, terms; double start_us, chunk_us, lone_us, round_us; } tiles[8] = {
        {128, 128, 1, 2, 6.4, 0.88, 0.88, 0.4}, {96, 128, 1, 2, 6.5, 0.76, 0.76, 1.5}, {64, 128, 1, 2, 6.2, 0.68, 0.68, 1.4}, {64, 64, 2, 2, 5.4, 0.34, 0.44, 0.9},
        {128, 128, 1, 3, 5.4, 1.02, 1.02, 1.0}, {96, 128, 1, 3, 5.4, 0.91, 0.91, 1.8}, {64, 128, 1, 3, 5.0, 0.82, 0.82, 0.9}, {64, 64, 2, 3, 4.8, 0.39, 0.46, 0.7}};
    const int64_t chunks = (N + kSpChunk - 1) / kSpChunk;
    SplitReconPlan best{0, 0, 1, true, 1e300, 0, 0, 0, 0, 1, true, 0};
    for (const auto& t : tiles) {
        if (exact && t.terms == 2) continue;
        if (t.bm == 96 && chunks < 16) continue;
        const bool ex = t.terms == 3;
        const int64_t n = ((J + t.bm - 1) / t.bm) * ((D + t.bn - 1) / t.bn);
        auto cost = [&](int64_t rows, int64_t cols, int64_t s, int64_t per) {
            const int64_t wgs = ((rows + t.bm - 1) / t.bm) * ((cols + t.bn - 1) / t.bn) * s;
            const double w_mb = 8e-6 * (double)rows * (double)cols, rounds = (double)((wgs + 255) / 256);
            const double deep = (double)((wgs + 256 * t.resident - 1) / (256 * t.resident));
            const double more = t.resident == 1 ? rounds - 1.0 : deep - (rounds > 1.0 ? 0.0 : 1.0);
            return t.start_us + (double)per * (rounds > 1.0 ? t.chunk_us * rounds : t.lone_us) + t.round_us * more +
                   (s == 1 ? 0.12 * w_mb                                          // W read and written
                           : 1.3 + 0.27 * (double)s * w_mb + (cols < 3600 ? (double)cols / 1500.0 : 2.4));   // planes written and read; a later W
        };
        for (int64_t s = 1; s <= 64 && (s == 1 || ((size_t)(s * J * D) * sizeof(float) <= room && chunks >= 2 * s && n * s <= 1536)); ++s) {
            const int64_t per = (chunks + s - 1) / s;
            if ((chunks + per - 1) / per != s) continue;                          // the same cut as a smaller count, or an empty slice
            if ((t.bm == 96 && per > 64) || (!ex && per < 4)) continue;
            const double us = cost(J, D, s, per);
            if (us < best.us) best = SplitReconPlan{t.bm, t.bn, (int)s, ex, us, 0, 0, 0, 0, 1, true, 0};
        }
        if (!alone || t.resident != 1 || (t.bm == 96 && chunks > 64) || (!ex && chunks < 4)) continue;
        const int64_t rows = (J - 4) / t.bm * t.bm, cols = (D - 4) / t.bn * t.bn; // (a launch takes four rows and columns and more)
        if (cols > 0 && (((J + t.bm - 1) / t.bm) * (cols / t.bn) + 255) / 256 < (n + 255) / 256) {
            const SplitReconPlan rest = plan_part(J, D - cols, N, room, exact, false);
            const double us = cost(J, cols, 1, chunks) + rest.us;
            if (us < best.us) best = SplitReconPlan{t.bm, t.bn, 1, ex, us, 0, (int)cols, rest.bm, rest.bn, rest.slices, rest.exact, 0};
        }
        if (rows > 0 && ((rows / t.bm) * ((D + t.bn - 1) / t.bn) + 255) / 256 < (n + 255) / 256) {
            const SplitReconPlan rest = plan_part(J - rows, D, N, room, exact, false);
            const double us = cost(rows, D, 1, chunks) + rest.us;
            if (us < best.us) best = SplitReconPlan{t.bm, t.bn, 1, ex, us, (int)rows, 0, rest.bm, rest.bn, rest.slices, rest.exact, 0};
        }
    }
    return best;
}
// Where the last row or column of tiles is what begins another round of 256, it is a second, smaller launch with a plan of its
// own: 1001 x 4100, 384 to 2048 pairs: 256 tiles of 128 x 128 and four columns 30 to 83 us, 34 to 103 in one; 2049 x 4096 with 384 46.8 and 52.2; 1412 x 4395
// with 1536 94.3 and 97.8.
SplitReconPlan reconstruct_split_plan(int64_t J, int64_t D, int64_t N, size_t room, bool exact, int halves) {
    SplitReconPlan p = plan_part(J, D, N, room, exact, true);
    p.halves = halves;
    return p;
}

template <int BM, int BN, int SPLITTERS, bool EXACT>
static hipError_t launch_tile(const ReconArgs& a, int slices, int halves, hipStream_t s) {
    if (slices == 1) return launch_split<BM, BN, SPLITTERS, false, EXACT>(a, 1, halves, s);
    const hipError_t e = launch_split<BM, BN, SPLITTERS, true, EXACT>(a, slices, halves, s);
    return e != hipSuccess ? e : launch_apply_partials(a, slices, a.D, s);
}

static hipError_t launch_part(const ReconArgs& a, int bm, int bn, int slices, bool exact, int halves, hipStream_t s) {
    if (slices < 1 || (slices > 1 && a.partial == nullptr)) return hipErrorInvalidValue;
    auto with = [&](auto ex) {
        constexpr bool X = decltype(ex)::value;
        if (bm == 128 && bn == 128) return launch_tile<128, 128, 8, X>(a, slices, halves, s);
        if (bm == 96 && bn == 128) return launch_tile<96, 128, 8, X>(a, slices, halves, s);
        if (bm == 64 && bn == 128) return launch_tile<64, 128, 8, X>(a, slices, halves, s);
        const int64_t small = (int64_t)((a.J + 63) / 64) * ((a.D + 63) / 64) * slices;
        if (bm == 64 && bn == 64) return small <= 256 ? launch_tile<64, 64, 8, X>(a, slices, halves, s) : launch_tile<64, 64, 4, X>(a, slices, halves, s);
        return hipErrorInvalidValue;
    };
    return exact ? with(std::true_type{}) : with(std::false_type{});
}

// plan.slices > 1 (or rest_slices): a.partial holds that many planes of J x D (of the rest's rows and columns) floats
hipError_t launch_reconstruct_split(const ReconArgs& a, const SplitReconPlan& p, hipStream_t s) {
    if (p.main_rows == 0 && p.main_cols == 0) return launch_part(a, p.bm, p.bn, p.slices, p.exact, p.halves, s);
    ReconArgs b = a;
    if (p.main_rows > 0) b.J = p.main_rows;
    else b.D = p.main_cols;
    const hipError_t e = launch_part(b, p.bm, p.bn, p.slices, p.exact, p.halves, s);
    if (e != hipSuccess) return e;
    const LaunchEvents main = launch_events();                           // the launch that is reported as the family's
    b = a;
    b.w += (int64_t)p.main_rows * a.ldw + p.main_cols;
    b.u += p.main_rows;
    b.v = (const float*)a.v + p.main_cols;
    b.J -= p.main_rows;
    b.D -= p.main_cols;
    const hipError_t e2 = launch_part(b, p.rest_bm, p.rest_bn, p.rest_slices, p.rest_exact, p.halves, s);
    launch_events().name = main.name;
    launch_events().blocks = main.blocks;
    return e2;
}

}  // namespace sfb
