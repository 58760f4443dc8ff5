// bf16 features, W of any shape: scores and update in tiles sized for the shape at hand (sfb_bf16.hip streams matrices of
// hundreds of MB in tiles of 256 rows, which leave most compute units idle where W is small).
//
// scores_bf16_kernel: Z[n][j] = sum_d A[n][d] * W[j][d], partial sums per slice of D.  Both operands are contiguous along the
// contraction; a lane loads 16 bytes of a row of A or W two chunks ahead, rounds or splits W's words on their way into LDS,
// and passes A's on to V.  TERMS = 1: W rounded to bf16.  TERMS = 3: W split exactly into three bf16 terms (sfb_split.h), the
// features being bf16 already: the products are fp32's, three matrix instructions instead of one.
//
// update_bf16_kernel: W[j][d] += sum_n bf16(alpha * U[n][j]) * V[n][d], straight from the received factors.  The contraction
// runs over the pairs, the slow index of both operands in memory; the rows go to LDS as they come (U rounded to bf16 on
// the way) and gfx950's transposing LDS read hands every lane four pairs of its column: no transposed copy, no launch for it.
//
// Both: four wavefronts as 2 x 2 over the tile (128 x 128: eight as 2 x 4), two LDS buffers, one barrier per chunk, chunks requested two
// ahead in registers.  Rows are taken at any alignment (16-byte accesses at the element's own alignment).
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

typedef uint32_t bt_u32x4u __attribute__((ext_vector_type(4), aligned(2)));   // a 16-byte access at any bf16's address
typedef short bt_s16x4 __attribute__((ext_vector_type(4)));

// 16-byte item c of an LDS row of ITEMS items sits at c ^ f(row): sixteen consecutive rows, sixteen different bank groups
template <int ITEMS>
__device__ __forceinline__ int bt_swz(int r) { return ITEMS == 8 ? (r & 7) ^ ((r >> 3) & 1) : (r >> 2) & 3; }

// Rows of pairs: 32-byte piece p of row r sits at p ^ bt_turn(r), so that the four rows of a transposing read, and the next
// sixteen columns' beside them, fall on different banks
template <int COLS>
__device__ __forceinline__ int bt_turn(int r) { return COLS == 64 ? r & 3 : 2 * (r & 3); }

// eight bf16 (four floats) moved down by sh places, zeros behind them
__device__ __forceinline__ sp_u32x4 bt_down8(sp_u32x4 x, int sh) {
    if (sh & 4) x = sp_u32x4{x[2], x[3], 0u, 0u};
    if (sh & 2) x = sp_u32x4{x[1], x[2], x[3], 0u};
    if (sh & 1) x = sp_u32x4{(x[0] >> 16) | (x[1] << 16), (x[1] >> 16) | (x[2] << 16), (x[2] >> 16) | (x[3] << 16), x[3] >> 16};
    if (sh >= 8) x = sp_u32x4{0u, 0u, 0u, 0u};
    return x;
}
__device__ __forceinline__ f32x4 bt_down4(f32x4 x, int sh) {
    if (sh & 1) x = f32x4{x[1], x[2], x[3], 0.f};
    if (sh & 2) x = f32x4{x[2], x[3], 0.f, 0.f};
    if (sh >= 4) x = f32x4{0.f, 0.f, 0.f, 0.f};
    return x;
}
// elements c .. c + 7 (+ 3) of a row of n, one by one, zeros beyond it
__device__ __forceinline__ sp_u32x4 bt_each8(const bf16_t* row, int c, int n) {
    sp_u32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t lo = row[min(c + 2 * e, n - 1)], hi = row[min(c + 2 * e + 1, n - 1)];
        x[e] = (c + 2 * e < n ? lo : 0u) | (c + 2 * e + 1 < n ? hi << 16 : 0u);
    }
    return x;
}
__device__ __forceinline__ f32x4 bt_each4(const float* row, int c, int n) {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float v = row[min(c + e, n - 1)];
        x[e] = c + e < n ? v : 0.f;
    }
    return x;
}

// The walk through the chunks: while a wavefront multiplies chunk c from registers it reads its fragments of chunk c + 1 from
// LDS, parks its share of chunk c + 2 in the other LDS buffer and then requests chunk c + 4, all of it between the matrix
// instructions; one barrier per chunk.  (A first form that read, multiplied and parked in turns took 0.75 us a chunk of 64 x 128,
// most of it waiting for its own LDS reads.)
//   fetch(raw, c): requests chunk c's words (c may be past the end: anything valid).   prep(raw, c): what has to happen to
//   them first, branches included.   park<p>(raw, buf): part p of PARTS.   read<q>(frag, buf): fragment read q of READS.
//   mma<q>(frag): matrix instruction q of MFMAS.   tail(): called before the last chunk but one (or the last) is multiplied.
template <class Raw, class Frag, int MFMAS, int READS, int PARTS, class Fetch, class Prep, class Park, class Read, class Mma, class Tail>
__device__ __forceinline__ void bt_run(int n_chunks, unsigned char* buf0, unsigned char* buf1, Fetch fetch, Prep prep, Park park, Read read,
                                       Mma mma, Tail tail) {
    Raw r0, r1;
    Frag f0, f1;
    auto park_all = [&](Raw& raw, unsigned char* buf) { split_for<0, PARTS>([&](auto p) { park(p, raw, buf); }); };
    auto read_all = [&](Frag& f, const unsigned char* buf) { split_for<0, READS>([&](auto q) { read(q, f, buf); }); };
    fetch(r0, 0);
    fetch(r1, 1);
    prep(r0, 0);
    park_all(r0, buf0);
    fetch(r0, 2);
    split_barrier();
    read_all(f0, buf0);
    prep(r1, 1);
    park_all(r1, buf1);
    fetch(r1, 3);
    // multiplies `now`; AHEAD >= 1: reads the next chunk from `from`; AHEAD == 2: parks the one after it in `to`
    auto multiply = [&](auto ahead, Frag& now, Frag& next, const unsigned char* from, Raw& raw, unsigned char* to) {
        constexpr int AHEAD = decltype(ahead)::value, R_SLOTS = MFMAS >= 2 ? MFMAS / 2 : 1;
        if constexpr (AHEAD >= 1) split_barrier();                       // the next chunk is parked, this one read by everybody
        split_for<0, MFMAS>([&](auto qc) {
            constexpr int q = decltype(qc)::value, R0 = q * READS / R_SLOTS, R1 = (q + 1) * READS / R_SLOTS;
            if constexpr (AHEAD >= 1)
                split_for<(R0 < READS ? R0 : READS), (R1 < READS ? R1 : READS)>([&](auto r) { read(r, next, from); });
            __builtin_amdgcn_sched_barrier(0);
            mma(qc, now);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (AHEAD == 2) split_for<q * PARTS / MFMAS, (q + 1) * PARTS / MFMAS>([&](auto p) { park(p, raw, to); });
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> NONE{};
    constexpr std::integral_constant<int, 1> ONE{};
    constexpr std::integral_constant<int, 2> TWO{};
    auto step = [&](int c, Frag& now, Frag& next, const unsigned char* from, Raw& raw, unsigned char* to) {
        prep(raw, c + 2);
        multiply(TWO, now, next, from, raw, to);
        fetch(raw, c + 4);
    };
    int c = 0;
    for (; c + 3 < n_chunks; c += 2) {
        step(c, f0, f1, buf1, r0, buf0);
        step(c + 1, f1, f0, buf0, r1, buf1);
    }
    // one to three chunks are left: the first is in f0, the second parked in buf1, the third on its way in r0
    const int left = n_chunks - c;
    if (left == 3) {
        prep(r0, c + 2);
        multiply(TWO, f0, f1, buf1, r0, buf0);
        tail();
        multiply(ONE, f1, f0, buf0, r0, buf0);
        multiply(NONE, f0, f0, buf0, r0, buf0);
    } else {
        tail();
        if (left == 2) {
            multiply(ONE, f0, f1, buf1, r0, buf0);
            multiply(NONE, f1, f1, buf1, r0, buf0);
        } else {
            multiply(NONE, f0, f0, buf1, r0, buf0);
        }
    }
}

// NARROW: rows of fewer than eight columns, element by element.
template <int BM, int BN, int WGM, int WGN, int TERMS, bool NARROW>
__global__ __launch_bounds__(WGM * WGN * 64, 2) void scores_bf16_kernel(
    const bf16_t* __restrict__ A, int64_t lda, const float* __restrict__ W, int64_t ldw, float* __restrict__ Z, int64_t ldz,
    int64_t zstride, bf16_t* __restrict__ Vout, int64_t ldv, int M, int N, int K, int k_slice, int n_mb, int n_nb, int total) {
    constexpr int kBtThreads = WGM * WGN * 64;
    constexpr int BK = kBfTileChunk<TERMS>, IA = BK / 8, IW = BK / 4, ROW = 2 * BK;      // items per row of A and W; bytes of an LDS row
    constexpr int A_LD = BM * IA / kBtThreads, W_LD = BN * IW / kBtThreads;
    constexpr int MT = BM / (32 * WGM), NT = BN / (32 * WGN), STEPS = BK / 16;
    constexpr int W_PLANE = BN * ROW, BUF = BM * ROW + TERMS * W_PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char bt_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, wm = wave / WGN, wn = wave % WGN;

    // consecutive ids share the class block (its W rows then sit in one die's L2)
    int id = xcd_contiguous_id(blockIdx.x, total);
    const int mb = id % n_mb;
    id /= n_mb;
    const int nb = id % n_nb, ks = id / n_nb;
    const int m0 = mb * BM, n0 = nb * BN;
    const int k_begin = ks * k_slice, k_end = min(K, k_begin + k_slice);
    const int n_chunks = (k_end - k_begin + BK - 1) / BK;
    const bool ragged = (K % BK) != 0 && k_end == K;                     // the last chunk is partial

    const int ra = tid / IA, ca = tid % IA, rw = tid / IW, cw = tid % IW;
    // uniform bases + 32-bit lane offsets (host: 128 rows of A and W below 2^32 bytes)
    const unsigned char* const a_base = reinterpret_cast<const unsigned char*>(A + (int64_t)m0 * lda);
    const unsigned char* const w_base = reinterpret_cast<const unsigned char*>(W + (int64_t)n0 * ldw);
    uint32_t a_off[A_LD], w_off[W_LD];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) a_off[i] = (uint32_t)min(ra + i * (kBtThreads / IA), M - 1 - m0) * (uint32_t)lda * 2u;
#pragma unroll
    for (int i = 0; i < W_LD; ++i) w_off[i] = (uint32_t)min(rw + i * (kBtThreads / IW), N - 1 - n0) * (uint32_t)ldw * 4u;

    struct Raw { sp_u32x4 a[A_LD]; f32x4 w[W_LD]; };
    auto fetch = [&](Raw& raw, int c) {
        const int k0 = k_begin + min(c, n_chunks - 1) * BK;
        if constexpr (NARROW) {
#pragma unroll
            for (int i = 0; i < A_LD; ++i) raw.a[i] = bt_each8(reinterpret_cast<const bf16_t*>(a_base + a_off[i]), k0 + 8 * ca, K);
#pragma unroll
            for (int i = 0; i < W_LD; ++i) raw.w[i] = bt_each4(reinterpret_cast<const float*>(w_base + w_off[i]), k0 + 4 * cw, K);
        } else {
            // in a partial chunk the words are read from the last ones of the row and moved into place by prep
            const uint32_t oa = (uint32_t)min(k0 + 8 * ca, K - 8) * 2u, ow = (uint32_t)min(k0 + 4 * cw, K - 4) * 4u;
#pragma unroll
            for (int i = 0; i < A_LD; ++i) raw.a[i] = *reinterpret_cast<const bt_u32x4u*>(a_base + (a_off[i] + oa));
#pragma unroll
            for (int i = 0; i < W_LD; ++i) raw.w[i] = *reinterpret_cast<const sp_f32x4u*>(w_base + (w_off[i] + ow));
        }
    };
    // the class blocks share the copy of A into V: block nb takes the chunks c with c % n_nb == nb
    const bool write_v = Vout != nullptr;
    auto prep = [&](Raw& raw, int c) {
        const int k0 = k_begin + c * BK;
        const bool last = ragged && c == n_chunks - 1;
        if (!NARROW && last) {
            const int sa = max(0, k0 + 8 * ca - (K - 8)), sw = max(0, k0 + 4 * cw - (K - 4));
#pragma unroll
            for (int i = 0; i < A_LD; ++i) raw.a[i] = bt_down8(raw.a[i], sa);
#pragma unroll
            for (int i = 0; i < W_LD; ++i) raw.w[i] = bt_down4(raw.w[i], sw);
        }
        if (write_v && (c % n_nb) == nb && c < n_chunks) {               // v_i = a_i
            const int k = k0 + 8 * ca;
#pragma unroll
            for (int i = 0; i < A_LD; ++i) {
                const int row = m0 + ra + i * (kBtThreads / IA);
                if (row >= M) continue;
                bf16_t* out = Vout + (int64_t)row * ldv + k;
                if (!last || k + 8 <= K) {
                    *reinterpret_cast<bt_u32x4u*>(out) = raw.a[i];
                } else {
#pragma unroll
                    for (int e = 0; e < 7; ++e)
                        if (k + e < K) out[e] = (bf16_t)(raw.a[i][e / 2] >> (16 * (e & 1)));
                }
            }
        }
    };
    const int a_item = ra * ROW + 16 * (ca ^ bt_swz<IA>(ra)), w_item = BM * ROW + rw * ROW + 16 * ((cw >> 1) ^ bt_swz<IA>(rw)) + 8 * (cw & 1);
    SplitQuad quad;
    constexpr int W_PARTS = TERMS == 1 ? 1 : 4;
    auto park = [&](auto part, const Raw& raw, unsigned char* buf) {
        constexpr int p = decltype(part)::value;
        if constexpr (p < A_LD) {
            *reinterpret_cast<sp_u32x4*>(buf + a_item + p * (kBtThreads / IA) * ROW) = raw.a[p];
        } else {
            constexpr int i = (p - A_LD) / W_PARTS, q = (p - A_LD) % W_PARTS;
            unsigned char* o = buf + w_item + i * (kBtThreads / IW) * ROW;
            const f32x4 x = raw.w[i];
            if constexpr (TERMS == 1) {
                *reinterpret_cast<uint2*>(o) = make_uint2(cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3]));
            } else {
                quad.template part<q>(x[0], x[1], x[2], x[3]);
                if constexpr (q == 3) {
                    *reinterpret_cast<uint2*>(o) = make_uint2(quad.ha, quad.hb);
                    *reinterpret_cast<uint2*>(o + W_PLANE) = make_uint2(quad.ma, quad.mb);
                    *reinterpret_cast<uint2*>(o + 2 * W_PLANE) = make_uint2(quad.la, quad.lb);
                }
            }
        }
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // every row this lane reads is l32 modulo 32
    const int a_at = (wm * 32 * MT + l32) * ROW, w_at = BM * ROW + (wn * 32 * NT + l32) * ROW, sz = bt_swz<IA>(l32);
    struct Frag { sp_u32x4 a[STEPS][MT], w[STEPS][TERMS][NT]; };
    constexpr int PER = MT + TERMS * NT;                                 // fragments of sixteen k
    auto read = [&](auto rd, Frag& f, const unsigned char* buf) {
        constexpr int q = decltype(rd)::value, s = q / PER, r = q % PER;
        const unsigned char* at = buf + 16 * ((2 * s + half) ^ sz);
        if constexpr (r < MT) f.a[s][r] = *reinterpret_cast<const sp_u32x4*>(at + a_at + r * 32 * ROW);
        else f.w[s][(r - MT) / NT][(r - MT) % NT] = *reinterpret_cast<const sp_u32x4*>(at + w_at + (r - MT) / NT * W_PLANE + (r - MT) % NT * 32 * ROW);
    };
    auto mma = [&](auto mm, const Frag& f) {                             // smallest terms first, blocks innermost
        constexpr int q = decltype(mm)::value, s = q / (TERMS * MT * NT), t = TERMS - 1 - q / (MT * NT) % TERMS, i = q / NT % MT, j = q % NT;
        acc[i][j] = split_mfma(f.a[s][i], f.w[s][t][j], acc[i][j]);
    };
    bt_run<Raw, Frag, STEPS * TERMS * MT * NT, STEPS * PER, A_LD + W_PARTS * W_LD>(n_chunks, bt_lds, bt_lds + BUF, fetch, prep, park, read, mma, [] {});

    float sum[MT][NT][16];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[i][j][e] = acc[i][j][e];
    if constexpr (TERMS == 3) {
        // values without a three-term split (infinities, and what rounds to one) end in sums that are not finite: those are
        // formed again by the fp32 instruction
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                bool finite = true;
#pragma unroll
                for (int e = 0; e < 16; ++e) finite &= __builtin_isfinite(sum[i][j][e]);
                if (__all(finite)) continue;
                const bf16_t* a = A + (int64_t)min(m0 + (wm * MT + i) * 32 + l32, M - 1) * lda;
                const float* w = W + (int64_t)min(n0 + (wn * NT + j) * 32 + l32, N - 1) * ldw;
                f32x16 x;
#pragma unroll
                for (int e = 0; e < 16; ++e) x[e] = 0.f;
#pragma unroll 1
                for (int k = k_begin; k < k_end; k += 8) {
                    float p[4], q[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int o = k + 2 * t + half, at = min(o, k_end - 1);
                        p[t] = o < k_end ? bf16_to_f32(a[at]) : 0.f;
                        q[t] = o < k_end ? w[at] : 0.f;
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) x = split_mfma_f32(p[t], q[t], x);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (!__builtin_isfinite(sum[i][j][e])) sum[i][j][e] = x[e];
            }
    }
    float* zout = Z + (int64_t)ks * zstride;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = n0 + (wn * NT + j) * 32 + l32;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = m0 + (wm * MT + i) * 32 + 8 * (e / 4) + 4 * half + (e % 4);
                if (row < M && col < N) zout[(int64_t)row * ldz + col] = sum[i][j][e];
            }
        }
}

// PLANES: the workgroups of slice k contract over k_chunks chunks of pairs and store their bare sums in plane k of W (a
// workspace then); apply_partials_kernel adds the planes up.  NARROW: fewer than four classes or eight columns.
template <int BM, int BN, int WGM, int WGN, bool PLANES, bool NARROW>
__global__ __launch_bounds__(WGM * WGN * 64, 2) void update_bf16_kernel(
    float* __restrict__ W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const bf16_t* __restrict__ V, int64_t ldv, int J,
    int D, int N, float alpha, int n_jb, int tiles, int total, int k_chunks, int prox_kind, float prox_a, uint64_t live_mask,
    uint32_t inv_b) {
    constexpr int kBtThreads = WGM * WGN * 64;
    constexpr int KC = kBfUpdateChunk, IU = BM / 4, IV = BN / 8;         // pairs per chunk; items per row of U and V
    constexpr int U_LD = KC * IU / kBtThreads, V_LD = KC * IV / kBtThreads, U_STEP = kBtThreads / IU, V_STEP = kBtThreads / IV;
    constexpr int U_ROW = 2 * BM, V_ROW = 2 * BN, BUF = KC * (U_ROW + V_ROW);
    constexpr int MT = BM / (32 * WGM), NT = BN / (32 * WGN);
    extern __shared__ __attribute__((aligned(16))) unsigned char bt_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, wm = wave / WGN, wn = wave % WGN;
    const int id = xcd_contiguous_id(blockIdx.x, total);
    const int slice = PLANES ? id / tiles : 0, tile = PLANES ? id % tiles : id;
    const int jb = tile % n_jb, db = tile / n_jb, j0 = jb * BM, d0 = db * BN;
    const int all_chunks = (N + KC - 1) / KC, c_begin = PLANES ? slice * k_chunks : 0;   // host: no slice is empty
    const int n_chunks = (PLANES ? min(all_chunks, c_begin + k_chunks) : all_chunks) - c_begin;

    const int ru = tid / IU, cu = j0 + 4 * (tid % IU), rv = tid / IV, cv = d0 + 8 * (tid % IV);
    // columns beyond the last four (eight) repeat them, moved into place by park
    const int cu_ok = NARROW ? cu : min(cu, J - 4), cv_ok = NARROW ? cv : min(cv, D - 8);
    const bool edge_u = !NARROW && j0 + BM > J && (J & 3) != 0, edge_v = !NARROW && d0 + BN > D && (D & 7) != 0;   // uniform

    struct Raw { f32x4 u[U_LD]; sp_u32x4 v[V_LD]; };
    auto fetch = [&](Raw& raw, int c) {                                  // host: 64 rows of U and V below 2^32 bytes
        const int p0 = (c_begin + min(c, n_chunks - 1)) * KC, left = N - 1 - p0;   // pairs beyond N repeat the last one
        const unsigned char* const u_base = reinterpret_cast<const unsigned char*>(U + (int64_t)p0 * ldu);
        const unsigned char* const v_base = reinterpret_cast<const unsigned char*>(V + (int64_t)p0 * ldv);
#pragma unroll
        for (int i = 0; i < U_LD; ++i) {
            const uint32_t off = (uint32_t)min(ru + i * U_STEP, left) * ((uint32_t)ldu * 4u);
            if constexpr (NARROW) raw.u[i] = bt_each4(reinterpret_cast<const float*>(u_base + off), cu, J);
            else raw.u[i] = *reinterpret_cast<const sp_f32x4u*>(u_base + (off + (uint32_t)cu_ok * 4u));
        }
#pragma unroll
        for (int i = 0; i < V_LD; ++i) {
            const uint32_t off = (uint32_t)min(rv + i * V_STEP, left) * ((uint32_t)ldv * 2u);
            if constexpr (NARROW) raw.v[i] = bt_each8(reinterpret_cast<const bf16_t*>(v_base + off), cv, D);
            else raw.v[i] = *reinterpret_cast<const bt_u32x4u*>(v_base + (off + (uint32_t)cv_ok * 2u));
        }
    };
    // all ones for a pair that counts, zero for pairs beyond N and of dead workers
    auto keep = [&](int n) -> uint32_t {
        const uint32_t p = __umulhi((uint32_t)n, inv_b);                 // worker (no mask: inv_b is 0 and every bit is set)
        return n < N ? 0u - (uint32_t)((live_mask >> (p & 63u)) & 1ull) : 0u;
    };
    auto prep = [&](Raw& raw, int c) {
        const int p0 = (c_begin + c) * KC;
        if (inv_b != 0 || p0 + KC > N) {
#pragma unroll
            for (int i = 0; i < U_LD; ++i) {
                const uint32_t on = keep(p0 + ru + i * U_STEP);
#pragma unroll
                for (int e = 0; e < 4; ++e) raw.u[i][e] = __uint_as_float(__float_as_uint(raw.u[i][e]) & on);
            }
#pragma unroll
            for (int i = 0; i < V_LD; ++i) raw.v[i] &= keep(p0 + rv + i * V_STEP);
        }
        if (edge_u) {
#pragma unroll
            for (int i = 0; i < U_LD; ++i) raw.u[i] = bt_down4(raw.u[i], cu - cu_ok);
        }
        if (edge_v) {
#pragma unroll
            for (int i = 0; i < V_LD; ++i) raw.v[i] = bt_down8(raw.v[i], cv - cv_ok);
        }
    };
    const int u_item = ru * U_ROW + 32 * ((tid % IU >> 2) ^ bt_turn<BM>(ru)) + 8 * (tid & 3);
    const int v_item = KC * U_ROW + rv * V_ROW + 32 * ((tid % IV >> 1) ^ bt_turn<BN>(rv)) + 16 * (tid & 1);
    auto park = [&](auto part, const Raw& raw, unsigned char* buf) {
        constexpr int p = decltype(part)::value;
        if constexpr (p < U_LD) {
            const f32x4 x = raw.u[p] * alpha;
            *reinterpret_cast<uint2*>(buf + u_item + p * U_STEP * U_ROW) = make_uint2(cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3]));
        } else {
            *reinterpret_cast<sp_u32x4*>(buf + v_item + (p - U_LD) * V_STEP * V_ROW) = raw.v[p - U_LD];
        }
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // Sixteen lanes read four pairs (rows) of sixteen columns, a quarter of a row each; lane i is handed column i of the
    // four rows.  Lanes 0..15 and 16..31 take the two halves of a block's columns, lanes 32.. the pairs eight further.
    const int g = lane >> 4, l16 = lane & 15, pair = 8 * (g >> 1) + (l16 >> 2);
    int u_at[MT], v_at[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) u_at[i] = pair * U_ROW + 32 * ((2 * (wm * MT + i) + (g & 1)) ^ bt_turn<BM>(pair)) + 8 * (l16 & 3);
#pragma unroll
    for (int j = 0; j < NT; ++j) v_at[j] = KC * U_ROW + pair * V_ROW + 32 * ((2 * (wn * NT + j) + (g & 1)) ^ bt_turn<BN>(pair)) + 8 * (l16 & 3);
    auto read_tr = [&](const unsigned char* p, int row) -> sp_u32x4 {
        typedef __attribute__((address_space(3))) bt_s16x4* lds_ptr;
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p));
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * row)));
        return sp_u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    constexpr int STEPS = KC / 16;
    struct Frag { sp_u32x4 u[STEPS][MT], v[STEPS][NT]; };
    auto read = [&](auto rd, Frag& f, const unsigned char* buf) {
        constexpr int q = decltype(rd)::value, s = q / (MT + NT), r = q % (MT + NT);
        if constexpr (r < MT) f.u[s][r] = read_tr(buf + u_at[r] + 16 * s * U_ROW, U_ROW);
        else f.v[s][r - MT] = read_tr(buf + v_at[r - MT] + 16 * s * V_ROW, V_ROW);
    };
    auto mma = [&](auto mm, const Frag& f) {
        constexpr int q = decltype(mm)::value, s = q / (MT * NT), i = q / NT % MT, j = q % NT;
        acc[i][j] = split_mfma(f.u[s][i], f.v[s][j], acc[i][j]);
    };

    float* const w_out = W + (PLANES ? (int64_t)slice * J * ldw : 0);
    const int jw = j0 + wm * 32 * MT, dw = d0 + wn * 32 * NT;
    const bool inside = jw + 32 * MT <= J && dw + 32 * NT <= D;          // by wavefronts
    // entry e of block (i, j): a uniform address plus this lane's offset
    const uint32_t w_lane = ((uint32_t)(4 * half) * (uint32_t)ldw + (uint32_t)l32) * 4u;   // host: 8 rows of W below 2^32 bytes
    auto w_at = [&](int i, int j, int e) -> float* {
        float* base = w_out + (int64_t)(jw + 32 * i + 8 * (e / 4) + (e % 4)) * ldw + dw + 32 * j;
        return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + w_lane);
    };

    // W's entries are requested behind the words of the last chunk (before them they would stand in front of them in the queue)
    float w[MT][NT][16];
    auto ask_w = [&]() {
        if constexpr (PLANES) return;
        if (inside) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e)
#pragma unroll
                    for (int j = 0; j < NT; ++j) w[i][j][e] = *w_at(i, j, e);
        } else {                                                         // addresses clamped into the matrix
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float* row = w_out + (int64_t)min(jw + 32 * i + 8 * (e / 4) + 4 * half + (e % 4), J - 1) * ldw;
#pragma unroll
                    for (int j = 0; j < NT; ++j) w[i][j][e] = row[min(dw + 32 * j + l32, D - 1)];
                }
        }
    };
    bt_run<Raw, Frag, STEPS * MT * NT, STEPS * (MT + NT), U_LD + V_LD>(n_chunks, bt_lds, bt_lds + BUF, fetch, prep, park, read, mma, ask_w);

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = jw + 32 * i + 8 * (e / 4) + 4 * half + (e % 4);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const float x = PLANES ? acc[i][j][e] : prox_entry(w[i][j][e] + acc[i][j][e], prox_kind, prox_a);
                if (inside || (row < J && dw + 32 * j + l32 < D)) *w_at(i, j, e) = x;
            }
        }
}

template <int BM, int BN, int WGM, int WGN, int TERMS, bool NARROW>
static hipError_t launch_scores(const FwdArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    constexpr int BK = kBfTileChunk<TERMS>;
    constexpr size_t lds_bytes = 2 * (size_t)(BM + TERMS * BN) * BK * 2;
    static_assert(lds_bytes <= 64 * 1024, "what a launch may ask for without hipFuncSetAttribute");
    const int n_mb = (a.n_rows + BM - 1) / BM, n_nb = (a.J + BN - 1) / BN, total = n_mb * n_nb * p.slices;
    SFB_LAUNCH((scores_bf16_kernel<BM, BN, WGM, WGN, TERMS, NARROW>), dim3(total), dim3(WGM * WGN * 64), lds_bytes, s, (const bf16_t*)a.a, a.lda,
               a.w, a.ldw, a.zp, a.ldz, a.zstride, (bf16_t*)a.v, a.ldv, a.n_rows, a.J, a.D, p.per_slice, n_mb, n_nb, total);
    return hipGetLastError();
}

template <int TERMS>
static hipError_t launch_scores(const FwdArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    if (p.bm == 128 && p.bn == 128) return launch_scores<128, 128, 2, 4, TERMS, false>(a, p, s);
    if (p.bm == 128 && p.bn == 64) return launch_scores<128, 64, 2, 2, TERMS, false>(a, p, s);
    if (p.bm == 64 && p.bn == 128) return launch_scores<64, 128, 2, 2, TERMS, false>(a, p, s);
    if (p.bm == 64 && p.bn == 64) return launch_scores<64, 64, 2, 2, TERMS, false>(a, p, s);
    return hipErrorInvalidValue;
}

hipError_t launch_scores_bf16(const FwdArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    if (a.D < 8) return launch_scores<64, 64, 2, 2, 3, true>(a, p, s);
    return p.terms == 1 ? launch_scores<1>(a, p, s) : launch_scores<3>(a, p, s);
}

template <int BM, int BN, int WGM, int WGN, bool PLANES, bool NARROW>
static hipError_t launch_update(const ReconArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    constexpr size_t lds_bytes = 2 * (size_t)kBfUpdateChunk * 2 * (BM + BN);
    static_assert(lds_bytes <= 64 * 1024, "what a launch may ask for without hipFuncSetAttribute");
    const int n_jb = (a.J + BM - 1) / BM, n_db = (a.D + BN - 1) / BN, tiles = n_jb * n_db;
    const uint32_t inv_b = a.use_mask ? (uint32_t)(((1ull << 32) + a.B - 1) / a.B) : 0;
    SFB_LAUNCH((update_bf16_kernel<BM, BN, WGM, WGN, PLANES, NARROW>), dim3(tiles * p.slices), dim3(WGM * WGN * 64), lds_bytes, s,
               PLANES ? a.partial : a.w, PLANES ? (int64_t)a.D : a.ldw, a.u, a.ldu, (const bf16_t*)a.v, a.ldv, a.J, a.D, a.N,
               a.alpha, n_jb, tiles, tiles * p.slices, p.per_slice, a.prox_kind, a.prox_a,
               a.live_mask, inv_b);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, bool NARROW>
static hipError_t launch_update(const ReconArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    if (p.slices == 1) return launch_update<BM, BN, WGM, WGN, false, NARROW>(a, p, s);
    const hipError_t e = launch_update<BM, BN, WGM, WGN, true, NARROW>(a, p, s);
    if (e != hipSuccess) return e;
    ReconArgs b = a;
    b.alpha = 1.0f;                                                      // it is in the factors already
    return launch_apply_partials(b, p.slices, a.D, s);
}

bool update_bf16_ok(const ReconArgs& a) {
    // 32-bit byte offsets inside a chunk of pairs and a block of rows of W; a masked call finds the worker of a pair with a
    // 32-bit reciprocal of B: exact while N * B < 2^32
    return a.ldu < (1 << 23) && a.ldv < (1 << 24) && a.ldw < (1 << 27) && (!a.use_mask || (a.B > 1 && (int64_t)a.N * a.B < (1LL << 32)));
}
bool scores_bf16_ok(const FwdArgs& a) { return a.lda < (1 << 23) && a.ldw < (1 << 22); }

// plan.slices > 1: a.partial holds that many planes of J x D floats
hipError_t launch_update_bf16(const ReconArgs& a, const Bf16TilePlan& p, hipStream_t s) {
    if (p.slices < 1 || (p.slices > 1 && a.partial == nullptr)) return hipErrorInvalidValue;
    if (a.J < 4 || a.D < 8) return launch_update<64, 64, 2, 2, true>(a, p, s);
    if (p.bm == 128 && p.bn == 128) return launch_update<128, 128, 2, 4, false>(a, p, s);
    if (p.bm == 64 && p.bn == 128) return launch_update<64, 128, 2, 2, false>(a, p, s);
    if (p.bm == 64 && p.bn == 64) return launch_update<64, 64, 2, 2, false>(a, p, s);
    return hipErrorInvalidValue;
}

// Tile and slices of D, by a cost in microseconds of the pass and the factor kernel behind it, fitted to 200 shapes (J = 20 to
// 10000, D = 64 to 20928, N = 30 to 11000, four tiles, up to ten slice counts each, one MI355X; the choice is within 1 % (TERMS
// = 1) and 2 % (TERMS = 3) of the best measured one on average).  A chunk costs a lone workgroup and a compute unit full of them
// what the table says; a slice's partial scores are written and read at about 2 TB/s.  No unit is full: counters of 1000 x 4096 with
// 512, thousands of cycles a compute unit, scores and update: busy 28.3 and 30.6; vector cache (64 bytes a clock) 9.6 and 10.0, the
// largest share, and waiting for misses 11.5 and 16.0; LDS 6.1 and 5.1, no conflicts; matrix pipe 4.1 and 4.1; vector unit 3.9 and
// 6.5.  By the costs below 6.9 of the scores' 13.3 us and 6.7 of the update's 15.5 are chunks; the others are start, first loads, W's
// trip and write-back.
// Against the 256 x 256 tiles of sfb_bf16.hip: 192 x 1600, N = 1280: 21.8 -> 10.6 us; 1000 x 4096, 512: 25.7 -> 18.
Bf16TilePlan plan_scores_bf16(int64_t n_rows, int64_t J, int64_t D, int terms, size_t most) {
    static const struct { int bm, bn, resident; double lone_us[2], full_us[2]; } tiles[4] = {
        {128, 128, 1, {0.68, 0.69}, {0.70, 0.64}}, {64, 128, 2, {0.56, 0.60}, {0.49, 0.48}},
        {128, 64, 2, {0.51, 0.50}, {0.43, 0.42}}, {64, 64, 3, {0.34, 0.38}, {0.29, 0.28}}};
    const int exact = terms == 3, bk = exact ? kBfTileChunk<3> : kBfTileChunk<1>;
    const int64_t chunks = (D + bk - 1) / bk;
    const double plane = (double)n_rows * (double)((J + 3) / 4 * 4) * 4.0;
    Bf16TilePlan best{0, 0, 1, 0, terms, 1e300};
    for (const auto& t : tiles) {
        const int64_t n = ((n_rows + t.bm - 1) / t.bm) * ((J + t.bn - 1) / t.bn);
        for (int64_t s = 1; s <= 32 && s <= chunks && n * s < (1LL << 30); ++s) {
            if (s > 1 && (double)s * plane > (double)most) break;
            const int64_t per = (chunks + s - 1) / s;
            if ((chunks + per - 1) / per != s) continue;                          // the same cut as a smaller count
            const double lone = t.lone_us[exact] * (double)((n * s + 256 * t.resident - 1) / (256 * t.resident));
            const double full = t.full_us[exact] * (double)((n * s + 255) / 256);
            const double us = 7.4 + (double)per * (lone > full ? lone : full) + (double)s * (plane * (exact ? 0.57e-6 : 0.46e-6) + 0.05);
            if (us < best.us * (1.0 - 1e-9)) best = Bf16TilePlan{t.bm, t.bn, (int)s, (int)(per * bk), terms, us};
        }
    }
    return best;
}

// The same for the update, fitted to 196 shapes (within 2.5 % of the best on average).  Where tiles leave compute units idle the
// pairs are cut into slices, as many as `room` bytes hold planes of J x D sums for; adding those up is a second kernel.  Against the
// 256 x 128 tiles of sfb_bf16.hip and their packing kernel: 192 x 1600, N = 1280: 37.6 -> 10.3 us; 1000 x 4096, 512: 30.4 -> 15.1.
Bf16TilePlan plan_update_bf16(int64_t J, int64_t D, int64_t N, size_t room) {
    static const struct { int bm, bn, resident; double lone_us, full_us; } tiles[3] = {
        {128, 128, 1, 0.80, 0.84}, {64, 128, 2, 0.60, 0.48}, {64, 64, 3, 0.38, 0.36}};
    const int64_t chunks = (N + kBfUpdateChunk - 1) / kBfUpdateChunk;
    const double plane = (double)J * (double)D * 4.0;
    Bf16TilePlan best{0, 0, 1, 0, 1, 1e300};
    for (const auto& t : tiles) {
        const int64_t n = ((J + t.bm - 1) / t.bm) * ((D + t.bn - 1) / t.bn);
        for (int64_t s = 1; s <= 64 && s <= chunks && n * s < (1LL << 30); ++s) {
            if (s > 1 && ((double)s * plane > (double)room || plane >= 4.0 * (double)(1LL << 31))) break;
            const int64_t per = (chunks + s - 1) / s;
            if ((chunks + per - 1) / per != s) continue;
            const double deep = (double)((n * s + 256 * t.resident - 1) / (256 * t.resident));
            const double lone = t.lone_us * deep, full = t.full_us * (double)((n * s + 255) / 256);
            const double us = 5.1 + (double)per * (lone > full ? lone : full) + 0.63 * (deep - 1.0) +
                              (s == 1 ? plane * 0.385e-6 : 1.95 + (double)s * plane * 0.42e-6);
            if (us < best.us * (1.0 - 1e-9)) best = Bf16TilePlan{t.bm, t.bn, (int)s, (int)per, 1, us};
        }
    }
    return best;
}

}  // namespace sfb
