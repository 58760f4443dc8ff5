// Reconstruction + update with few factor pairs (one worker's batch and less), fp32:
//     W[j][d] <- W[j][d] + alpha * sum_n U[n][j] * V[n][d]
// Bound by W's trip through memory: 64 pairs on 1000 x 4096 are 0.5 GFLOP against 33 MB, which nothing but a read and a
// write of every entry takes 7.1 us for.  So: small tiles, four workgroups of 64 x 64 per compute unit; the tile's columns
// of all pairs go to LDS in one piece, by copies requested before W's entries, so that the products (fp32 instruction) are
// formed while those are on their way; workgroups in the order of W's rows, not dealt out to the dies in ranges; and W
// loaded and stored as data that is not used again (nontemporal: 10.3 us per call against 11.2 without).
// W's addresses are a scalar base an entry and one lane offset: formed per lane they were a third of the vector instructions (1000 x
// 4096, 64 pairs 10.7 -> 10.1 us; 2000 x 8192: 35.9 -> 32.5).
// Against the kernels that stage tiles, 1000 x 4096: 14.9 -> 7.4 us with 8 pairs, 12.0 -> 10.1 with 64; 2000 x 8192: 61 -> 25 and 45 -> 32.5 (one
// W over and over; in a replayed chain over eight 7.2, 9.2, 25.3 and 31.0).
// Larger tiles (128 x 64, 128 x 128) halve the copies into LDS and were 3 % slower: fewer workgroups to overlap.
#include "sfb_kernels.h"
#include "sfb_split.h"

namespace sfb {

constexpr int kThinStage = 16;                                           // pairs per stage

// (W is not __restrict__: its loads have to stay between the copies into LDS and the wait that counts them.)
// STAGES: all of them are requested up front, so N <= STAGES * kThinStage.  WIDE: 16-byte rows of U and V, four columns and
// four pairs per copy instruction and lane; single words otherwise.
template <int STAGES, bool MASK, bool WIDE>
struct ThinFp32 {
static constexpr int THREADS = 256, WAVES = STAGES > 4 ? 2 : 4;          // per workgroup; wavefronts per SIMD
static __device__ __forceinline__ void run(
    float* W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V, int64_t ldv,
    int J, int D, int N, int B, float alpha, int n_db, int prox_kind, float prox_a, uint64_t live_mask, uint32_t) {
    constexpr int PAIRS = kThinStage * STAGES;
    __shared__ float rt_lds[2 * PAIRS * 64];                             // [U, V][pair][64 columns]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int jw = (int)(blockIdx.x / n_db) * 64, dw = (int)(blockIdx.x % n_db) * 64;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)rt_lds;
    // pairs beyond N repeat the last one, columns beyond J or D the last (four)
    if constexpr (WIDE) {
        const float* u = U + min(jw + 4 * (lane & 15), J - 4);
        const float* v = V + min(dw + 4 * (lane & 15), D - 4);
#pragma unroll
        for (int i = 0; i < PAIRS / 16; ++i) {
            const int n = 4 * (wave + 4 * i);
            const int64_t row = min(n + (lane >> 4), N - 1);
            lds_dma16(u + row * ldu, lds0 + n * 256);
            lds_dma16(v + row * ldv, lds0 + (PAIRS + n) * 256);
        }
    } else {
        const float* u = U + min(jw + lane, J - 1);
        const float* v = V + min(dw + lane, D - 1);
#pragma unroll
        for (int i = 0; i < PAIRS / 4; ++i) {
            const int n = wave + 4 * i;
            const int64_t row = min(n, N - 1);
            lds_dma4(u + row * ldu, lds0 + n * 256);
            lds_dma4(v + row * ldv, lds0 + (PAIRS + n) * 256);
        }
    }
    const int j0 = jw + (wave >> 1) * 32, d0 = dw + (wave & 1) * 32, col = d0 + l32;
    auto row_of = [&](int e) { return 8 * (e / 4) + 4 * half + (e % 4); };
    // W: a uniform address an entry plus this lane's offset (host: 8 rows of W below 2^32 bytes)
    const bool inside = j0 + 32 <= J && d0 + 32 <= D;                    // by wavefronts
    const uint32_t w_lane = ((uint32_t)(4 * half) * (uint32_t)ldw + (uint32_t)l32) * 4u;
    auto w_at = [&](int e) -> float* {
        float* base = W + (int64_t)(j0 + 8 * (e / 4) + (e % 4)) * ldw + d0;
        return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + w_lane);
    };
    float w[16];
    if (inside) {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = __builtin_nontemporal_load(w_at(e));
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = __builtin_nontemporal_load(W + (int64_t)min(j0 + row_of(e), J - 1) * ldw + min(col, D - 1));
    }
    wait_vmcnt<16>();                                                    // loads return in order: W's entries are still on their way
    __builtin_amdgcn_s_barrier();
    const float* a_at = rt_lds + half * 64 + (wave >> 1) * 32 + l32;
    const float* b_at = rt_lds + (PAIRS + half) * 64 + (wave & 1) * 32 + l32;
    // Running sums: two, as in the 128 x 128 kernel that this one mostly stands in for, four where there are registers for them
    // (of the norm, 64 pairs: 1.07e-7, one sum 1.44e-7; 128: 1.1e-7 and 2.0e-7; the same time)
    constexpr int SUMS = STAGES > 4 ? 4 : 2;
    f32x16 acc[SUMS];
#pragma unroll
    for (int p = 0; p < SUMS; ++p)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[p][e] = 0.f;
    // a stage's fragments are read while the products of the one before are formed
    struct Frags { float a[kThinStage / 2], b[kThinStage / 2]; } fr[2];
    auto read = [&](Frags& f, int c) {
#pragma unroll
        for (int i = 0; i < kThinStage / 2; ++i) {
            f.a[i] = a_at[(c * kThinStage + 2 * i) * 64];
            f.b[i] = b_at[(c * kThinStage + 2 * i) * 64];
        }
    };
    read(fr[0], 0);
#pragma unroll
    for (int c = 0; c < STAGES; ++c) {
        Frags& f = fr[c & 1];
        if (c + 1 < STAGES) read(fr[(c + 1) & 1], c + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kThinStage / 2; ++i) {
            float x = f.a[i], y = f.b[i];
            if (MASK || c >= STAGES - (STAGES > 4 ? 2 : 1)) {            // pairs beyond N and of dead workers count as zero
                const int n = c * kThinStage + 2 * i + half;
                const bool on = n < N && (!MASK || ((live_mask >> (min(n, N - 1) / B)) & 1ull));
                x = on ? x : 0.f;
                y = on ? y : 0.f;
            }
            acc[i % SUMS] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc[i % SUMS], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        float sum = acc[0][e] + acc[1][e];
        if constexpr (SUMS == 4) sum += acc[2][e] + acc[3][e];
        w[e] += alpha * sum;
    }
    if (prox_kind != 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = prox_entry(w[e], prox_kind, prox_a);
    }
    if (inside) {
#pragma unroll
        for (int e = 0; e < 16; ++e) __builtin_nontemporal_store(w[e], w_at(e));
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (j0 + row_of(e) < J && col < D) W[(int64_t)(j0 + row_of(e)) * ldw + col] = w[e];
    }
}
};

// 17 to 64 pairs: the products on the bf16 matrix cores, every operand split exactly into three bf16 terms (sfb_split.h).  All
// workgroups start together and multiply at the same time, so the fp32 instruction's products (64 pairs of 1000 x 4096: 8192
// cycles of every matrix pipe, 3.9 us) stand between W's way in and its way out; these take 3072.
// Tile of 64 x 128, eight wavefronts as 2 x 4, two workgroups per compute unit.  Loads of U and V (a thread: four pairs of KP /
// 32 columns of U and KP / 16 of V, four lanes side by side), then of W; splits into LDS, [plane][column][pairs], sixteen-byte
// items turned so that neither the writes of sixteen lanes nor the reads of eight meet on a bank; then one barrier and the products.
// The leading products have a running sum of their own: of the norm, 64 pairs: 0.5e-7 (fp32 instruction in two sums 1.07e-7).
typedef float rt_f32x2u __attribute__((ext_vector_type(2), aligned(4)));

template <int KP>
struct ThinSplit {
static constexpr int THREADS = 512, WAVES = 4;
static __device__ __forceinline__ void run(
    float* W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V, int64_t ldv,
    int J, int D, int N, int, float alpha, int n_db, int prox_kind, float prox_a, uint64_t live_mask, uint32_t inv_b) {
    constexpr int BM = 64, BN = 128, UC = KP / 32, VC = KP / 16, ROW = 2 * KP, ITEMS = KP / 8, PLANE = (BM + BN) * ROW;
    __shared__ __attribute__((aligned(16))) unsigned char rt_split_lds[3 * PLANE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, wm = wave >> 2, wn = wave & 3;
    const int j0 = (int)(blockIdx.x / n_db) * BM, d0 = (int)(blockIdx.x % n_db) * BN;
    auto turn = [](int r) { return ITEMS == 8 ? (r >> 1) & 7 : (r >> 2) & 3; };

    // pairs 4 kb .. 4 kb + 3 of columns UC c .. of U's block and VC c .. of V's
    const int kb = (tid >> 2) & (KP / 4 - 1), c = (tid & 3) + 4 * (tid / KP);
    const int cu = j0 + UC * c, cv = d0 + VC * c;
    const int cu_ok = min(cu, J - UC), cv_ok = min(cv, D - VC);          // columns beyond the last repeat it, moved into place below
    float u[4][UC], v[4][VC];
    // 32-bit offsets (host: 64 rows of U and V below 2^32 bytes); pairs beyond N repeat the last one
    const uint32_t pu = (uint32_t)ldu * 4u, pv = (uint32_t)ldv * 4u;
    const uint32_t ou = (uint32_t)(4 * kb) * pu + (uint32_t)cu_ok * 4u, ov = (uint32_t)(4 * kb) * pv + (uint32_t)cv_ok * 4u;
    const uint32_t lu = (uint32_t)(N - 1) * pu + (uint32_t)cu_ok * 4u, lv = (uint32_t)(N - 1) * pv + (uint32_t)cv_ok * 4u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const char* up = reinterpret_cast<const char*>(U) + min(ou + i * pu, lu);
        if constexpr (UC == 2) {
            const rt_f32x2u x = *reinterpret_cast<const rt_f32x2u*>(up);
            u[i][0] = x.x;
            u[i][1] = x.y;
        } else {
            u[i][0] = *reinterpret_cast<const float*>(up);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const char* vp = reinterpret_cast<const char*>(V) + min(ov + i * pv, lv);
        if constexpr (VC == 4) {
            const f32x4 x = *reinterpret_cast<const sp_f32x4u*>(vp);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i][e] = x[e];
        } else {
            const rt_f32x2u x = *reinterpret_cast<const rt_f32x2u*>(vp);
            v[i][0] = x.x;
            v[i][1] = x.y;
        }
    }
    // W: a uniform address an entry plus this lane's offset (host: 8 rows of W below 2^32 bytes)
    const int jw = j0 + 32 * wm, dw = d0 + 32 * wn, col = dw + l32;
    const bool inside = jw + 32 <= J && dw + 32 <= D;                    // by wavefronts
    const uint32_t w_lane = ((uint32_t)(4 * half) * (uint32_t)ldw + (uint32_t)l32) * 4u;
    auto row_of = [&](int e) { return jw + 8 * (e / 4) + 4 * half + (e % 4); };
    auto w_at = [&](int e) -> float* {
        float* base = W + (int64_t)(jw + 8 * (e / 4) + (e % 4)) * ldw + dw;
        return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + w_lane);
    };
    float w[16];
    if (inside) {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = __builtin_nontemporal_load(w_at(e));
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = W[(int64_t)min(row_of(e), J - 1) * ldw + min(col, D - 1)];
    }
    __builtin_amdgcn_sched_barrier(0);

    if (inv_b != 0 || N < KP) {                                          // pairs beyond N and of dead workers count as zero
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = 4 * kb + i;
            const bool on = n < N && ((live_mask >> (__umulhi((uint32_t)n, inv_b) & 63u)) & 1ull);
#pragma unroll
            for (int e = 0; e < UC; ++e) u[i][e] = on ? u[i][e] : 0.f;
#pragma unroll
            for (int e = 0; e < VC; ++e) v[i][e] = on ? v[i][e] : 0.f;
        }
    }
    if (cu > cu_ok) {                                                    // (columns beyond the matrix feed entries that are not stored)
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i][0] = u[i][UC - 1];
    }
    if (VC == 4 && cv > cv_ok && cv < D) {
        const int sh = cv - cv_ok;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i][0] = sh == 1 ? v[i][1] : sh == 2 ? v[i][VC / 2] : v[i][VC - 1];
            v[i][1] = sh == 1 ? v[i][VC / 2] : v[i][VC - 1];
            v[i][VC / 2] = v[i][VC - 1];
        }
    } else if (VC == 2 && cv > cv_ok) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i][0] = v[i][1];
    }
    auto park = [&](float x0, float x1, float x2, float x3, int row) {
        SplitQuad s;
        s.template part<0>(x0, x1, x2, x3);
        s.template part<1>(x0, x1, x2, x3);
        s.template part<2>(x0, x1, x2, x3);
        s.template part<3>(x0, x1, x2, x3);
        unsigned char* o = rt_split_lds + row * ROW + 16 * ((kb >> 1) ^ turn(row)) + 8 * (kb & 1);
        *reinterpret_cast<uint2*>(o) = make_uint2(s.ha, s.hb);
        *reinterpret_cast<uint2*>(o + PLANE) = make_uint2(s.ma, s.mb);
        *reinterpret_cast<uint2*>(o + 2 * PLANE) = make_uint2(s.la, s.lb);
    };
#pragma unroll
    for (int e = 0; e < UC; ++e) park(u[0][e], u[1][e], u[2][e], u[3][e], UC * c + e);
#pragma unroll
    for (int e = 0; e < VC; ++e) park(v[0][e], v[1][e], v[2][e], v[3][e], BM + VC * c + e);
    split_barrier();

    f32x16 acc, rest;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = rest[e] = 0.f;
    struct Frag { sp_u32x4 a[3], b[3]; } f[2];
    auto read = [&](Frag& g, int s) {
        const unsigned char* at = rt_split_lds + l32 * ROW + 16 * ((2 * s + half) ^ turn(l32));   // every row it reads is l32 modulo 32
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            g.a[p] = *reinterpret_cast<const sp_u32x4*>(at + p * PLANE + 32 * wm * ROW);
            g.b[p] = *reinterpret_cast<const sp_u32x4*>(at + p * PLANE + (BM + 32 * wn) * ROW);
        }
    };
    read(f[0], 0);
#pragma unroll
    for (int s = 0; s < KP / 16; ++s) {
        const Frag& g = f[s & 1];
        if (s + 1 < KP / 16) read(f[(s + 1) & 1], s + 1);
        __builtin_amdgcn_sched_barrier(0);
        rest = split_mfma(g.a[2], g.b[0], rest);
        acc = split_mfma(g.a[0], g.b[0], acc);
        rest = split_mfma(g.a[0], g.b[2], rest);
        rest = split_mfma(g.a[1], g.b[1], rest);
        rest = split_mfma(g.a[1], g.b[0], rest);
        rest = split_mfma(g.a[0], g.b[1], rest);
        __builtin_amdgcn_sched_barrier(0);
    }
    float sum[16];
    bool finite = true;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        sum[e] = acc[e] + rest[e];
        finite &= __builtin_isfinite(sum[e]);
    }
    if (!__all(finite)) {                                                // infinities, and what rounds to one: by the fp32 instruction
        const float* ur = U + min(jw + l32, J - 1);
        const float* vr = V + min(col, D - 1);
        f32x16 x;
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = 0.f;
#pragma unroll 1
        for (int n0 = 0; n0 < N; n0 += 2) {
            const int n = min(n0 + half, N - 1);
            const bool on = n0 + half < N && ((live_mask >> (__umulhi((uint32_t)n, inv_b) & 63u)) & 1ull);
            const float p = ur[(int64_t)n * ldu], q = vr[(int64_t)n * ldv];
            x = split_mfma_f32(on ? p : 0.f, on ? q : 0.f, x);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[e] = __builtin_isfinite(sum[e]) ? sum[e] : x[e];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] += alpha * sum[e];
    if (prox_kind != 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = prox_entry(w[e], prox_kind, prox_a);
    }
    if (inside) {
#pragma unroll
        for (int e = 0; e < 16; ++e) __builtin_nontemporal_store(w[e], w_at(e));
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (row_of(e) < J && col < D) W[(int64_t)row_of(e) * ldw + col] = w[e];
    }
}
};

template <class Form>
__global__ __launch_bounds__(Form::THREADS, Form::WAVES) void reconstruct_thin_kernel(
    float* W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V, int64_t ldv, int J, int D, int N, int B,
    float alpha, int n_db, int prox_kind, float prox_a, uint64_t live_mask, uint32_t inv_b) {
    Form::run(W, ldw, U, ldu, V, ldv, J, D, N, B, alpha, n_db, prox_kind, prox_a, live_mask, inv_b);
}

template <class Form>
static hipError_t launch_form(const ReconArgs& a, int cols, hipStream_t s) {
    const int n_db = (a.D + cols - 1) / cols, total = (a.J + 63) / 64 * n_db;
    const uint32_t inv_b = a.use_mask && a.B > 1 ? (uint32_t)(((1ull << 32) + a.B - 1) / a.B) : 0;   // worker of a pair, exact: N <= 64
    SFB_LAUNCH((reconstruct_thin_kernel<Form>), dim3(total), dim3(Form::THREADS), 0, s, a.w, a.ldw, a.u, a.ldu, (const float*)a.v,
               a.ldv, a.J, a.D, a.N, a.B, a.alpha, n_db, a.prox_kind, a.prox_a, a.live_mask, inv_b);
    return hipGetLastError();
}
static bool thin_wide(const ReconArgs& a) {
    auto wide = [](const void* p, int64_t ld, int n) { return ((uintptr_t)p % 16) == 0 && ld % 4 == 0 && n % 4 == 0; };
    return !a.use_mask && wide(a.u, a.ldu, a.J) && wide(a.v, a.ldv, a.D);
}
template <int STAGES>
static hipError_t launch_thin(const ReconArgs& a, hipStream_t s) {
    if (a.use_mask) return launch_form<ThinFp32<STAGES, true, false>>(a, 64, s);
    if (thin_wide(a)) return launch_form<ThinFp32<STAGES, false, true>>(a, 64, s);
    return launch_form<ThinFp32<STAGES, false, false>>(a, 64, s);
}

// Split products: 17 to 64 pairs on a W large enough for its products to show (instruction -> split below, us; "cold": eight W in turn,
// "hot": seven updates of each in a row, W mostly in the caches).
// Where the instruction's copies into LDS go word by word (unaligned rows, masks): from 256 tiles of 64 x 64 on (224, 401 x 2000: 32 pairs 3.9 -> 4.5, 64:
// 4.6 -> 5.1; 320, 601 x 2001: 6.2 -> 5.2 and 7.2 -> 5.9; 1001 x 4099: 13.3 -> 9.5 and 15.0 -> 11.2; cold and hot alike).
// Elsewhere with more than 48 pairs: beyond 768 tiles (64 pairs, 640 x 4096: cold 6.7 -> 8.1, hot 6.8 -> 7.3; 768 x 4096: 7.3 -> 8.3 and 7.0 ->
// 7.6; 832 x 4096: 8.6 -> 8.4 and 8.6 -> 7.7; 1000 x 4096: 9.2 -> 8.8 and 9.3 -> 8.3; 4000 x 8192: 59.5 -> 57.5 and 58.9 -> 48.5): up to there every
// compute unit has three of the instruction's workgroups at most and one or two of these, whose chain of loads, splits and
// products is the longer one.  With up to 48, beyond 1536 tiles, for a W that is hot, as it is behind the score pass of a step or under several
// workers' updates (2000 x 4096: 20 pairs 13.9 -> 12.5, 48: 14.8 -> 14.7; 4000 x 8192: 48.4 -> 41.5 and 51.2 -> 47.9; cold 13.7 -> 14.4, 14.7 -> 16.2, 48.9 -> 48.8,
// 51.0 -> 54.1; 1200 x 4096, 32 pairs, 9.1 -> 9.3 hot).
static bool thin_split_wins(const ReconArgs& a) {
    const int64_t tiles = (int64_t)((a.J + 63) / 64) * ((a.D + 63) / 64);
    return a.N > 16 && a.N <= 64 && a.J >= 4 && a.D >= 4 && (!a.use_mask || a.B > 1) && a.ldu < (1 << 23) && a.ldv < (1 << 23) &&
           tiles > (!thin_wide(a) ? 256 : a.N > 48 ? 768 : 1536);
}

// Up to 64 pairs always (against the kernels that stage tiles: the figures at the head); up to 128 while W is small enough for
// the matrix pipe's share not to show (4000 x 700 with 128: 15.0 against 16.8; 1000 x 4096: 17.5 against 16.1).
// Not with a mask, which looks up the worker of every pair (256 x 1024 with 128: 10.6 against 6.8 by split products; 64 x 64: 10.2, 6.4).
bool reconstruct_thin_ok(const ReconArgs& a) {
    const int64_t tiles = (int64_t)((a.J + 63) / 64) * ((a.D + 63) / 64);
    return !a.bf16 && tiles < (1LL << 31) && a.ldw < (1 << 27) && (a.N <= 64 || (a.N <= 128 && tiles <= 768 && !a.use_mask));
}

hipError_t launch_reconstruct_thin(const ReconArgs& a, hipStream_t s) {
    if (thin_split_wins(a)) return a.N <= 32 ? launch_form<ThinSplit<32>>(a, 128, s) : launch_form<ThinSplit<64>>(a, 128, s);
    switch ((a.N + kThinStage - 1) / kThinStage) {
        case 1: return launch_thin<1>(a, s);
        case 2: return launch_thin<2>(a, s);
        case 3: return launch_thin<3>(a, s);
        case 4: return launch_thin<4>(a, s);
        case 5:
        case 6: return launch_thin<6>(a, s);
        case 7:
        case 8: return launch_thin<8>(a, s);
    }
    return hipErrorNotSupported;
}

}  // namespace sfb
