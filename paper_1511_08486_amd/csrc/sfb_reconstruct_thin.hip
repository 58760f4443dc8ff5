// Reconstruction + update with few factor pairs (one worker's batch and less), fp32:
//     W[j][d] <- W[j][d] + alpha * sum_n U[n][j] * V[n][d]
// Bound by W's trip through memory: 64 pairs on 1000 x 4096 are 0.5 GFLOP against 33 MB, which nothing but a read and a
// write of every entry takes 7.1 us for.  So: small tiles, four workgroups of 64 x 64 per compute unit; the tile's columns
// of all pairs go to LDS in one piece, by copies requested before W's entries, so that the products (fp32 instruction) are
// formed while those are on their way; workgroups in the order of W's rows, not dealt out to the dies in ranges; and W
// loaded and stored as data that is not used again (nontemporal: 10.3 us per call against 11.2 without).
// 1000 x 4096: 14.9 -> 7.9 us with 8 pairs, 12.0 -> 10.3 with 64; 2000 x 8192: 61 -> 25 and 45 -> 36.
// Larger tiles (128 x 64, 128 x 128) halve the copies into LDS and were 3 % slower: fewer workgroups to overlap.
#include "sfb_device.h"
#include "sfb_kernels.h"

namespace sfb {

constexpr int kThinStage = 16;                                           // pairs per stage

// (W is not __restrict__: its loads have to stay between the copies into LDS and the wait that counts them.)
// STAGES: all of them are requested up front, so N <= STAGES * kThinStage.  WIDE: 16-byte rows of U and V, four columns and
// four pairs per copy instruction and lane; single words otherwise.
template <int STAGES, bool MASK, bool WIDE>
__global__ __launch_bounds__(256, STAGES > 4 ? 2 : 4) void reconstruct_thin_kernel(
    float* W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const float* __restrict__ V, int64_t ldv,
    int J, int D, int N, int B, float alpha, int n_db, int prox_kind, float prox_a, uint64_t live_mask) {
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
    float* w_at = W + min(col, D - 1);
    float w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] = __builtin_nontemporal_load(w_at + (int64_t)min(j0 + row_of(e), J - 1) * ldw);
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
    if (j0 + 32 <= J && d0 + 32 <= D) {
#pragma unroll
        for (int e = 0; e < 16; ++e) __builtin_nontemporal_store(w[e], w_at + (int64_t)(j0 + row_of(e)) * ldw);
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (j0 + row_of(e) < J && col < D) w_at[(int64_t)(j0 + row_of(e)) * ldw] = w[e];
    }
}

template <int STAGES, bool MASK, bool WIDE>
static hipError_t launch_thin(const ReconArgs& a, hipStream_t s) {
    const int n_db = (a.D + 63) / 64, total = (a.J + 63) / 64 * n_db;
    SFB_LAUNCH((reconstruct_thin_kernel<STAGES, MASK, WIDE>), dim3(total), dim3(256), 0, s, a.w, a.ldw, a.u, a.ldu,
               (const float*)a.v, a.ldv, a.J, a.D, a.N, a.B, a.alpha, n_db, a.prox_kind, a.prox_a, a.live_mask);
    return hipGetLastError();
}
template <int STAGES>
static hipError_t launch_thin(const ReconArgs& a, hipStream_t s) {
    auto wide = [](const void* p, int64_t ld, int n) { return ((uintptr_t)p % 16) == 0 && ld % 4 == 0 && n % 4 == 0; };
    if (a.use_mask) return launch_thin<STAGES, true, false>(a, s);
    if (wide(a.u, a.ldu, a.J) && wide(a.v, a.ldv, a.D)) return launch_thin<STAGES, false, true>(a, s);
    return launch_thin<STAGES, false, false>(a, s);
}

// Up to 64 pairs always (1000 x 4096: 7.9 us with 8 pairs, 10.6 with 64, against 14.9 and 12.0 with the kernels that stage
// tiles; 2000 x 8192: 25 and 36 against 61 and 45; 300 x 1000: one launch, 5.6); up to 128 while W is small enough for
// the matrix pipe's share not to show (4000 x 700 with 128: 15.0 against 16.8; 1000 x 4096: 17.5 against 16.1).
// Not with a mask, which looks up the worker of every pair (256 x 1024 with 128: 10.6 against 6.8 by split products; 64 x 64: 10.2, 6.4).
bool reconstruct_thin_ok(const ReconArgs& a) {
    const int64_t tiles = (int64_t)((a.J + 63) / 64) * ((a.D + 63) / 64);
    return !a.bf16 && tiles < (1LL << 31) && (a.N <= 64 || (a.N <= 128 && tiles <= 768 && !a.use_mask));
}

hipError_t launch_reconstruct_thin(const ReconArgs& a, hipStream_t s) {
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
