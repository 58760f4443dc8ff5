// Whole steps of models with few classes (J <= 32): one pass over the features.
//
// A small W leaves the separate kernels nothing to do but move the batch: scores read A and write V, the update reads V
// again (ragged rows through a padded copy of it: twice more), and each is a launch of its own.  Here a workgroup keeps
// its samples' feature rows in LDS from the first byte to the last use: load (and store V on the way, or, of a large batch,
// during the products), scores, factor u, and its share of U^T V.
//   scores   v_mfma_f32_16x16x4_f32: 16 samples x 16 classes; lane l reads four consecutive columns of row l % 16 with
//            one 16-byte LDS read (rows Dp + 4 floats apart, Dp the columns in whole sixteens: conflict-free) and feeds
//            four instructions (the contraction index is a dummy); the wavefronts cut D into slices, whose sums meet
//            in LDS and are added in slice order.
//   factor   16 lanes to a sample (32 for more than 16 classes): softmax residual or the pair models' coefficient.
//   update   the same instruction with classes as rows, columns of V as columns and samples as the contraction; lane l
//            reads columns 4 (l % 16) .. + 3 of a sample's row and feeds four blocks, so it ends with four consecutive
//            entries of rows of W.
// With one workgroup (N rows fit in LDS) the sums go straight into W.  Otherwise every workgroup stores its J x D sums
// as a plane of the workspace and few_apply_kernel adds the planes in order: the same bits every time.
// Ten classes x 784 columns, 12000 samples: 75 MB to move, 74 us as five kernels.
#include <type_traits>

#include "sfb_device.h"
#include "sfb_kernels.h"

namespace sfb {

constexpr int kFewThreads = 1024, kFewWaves = kFewThreads / 64;
typedef float few_f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 few_mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// four consecutive entries of a row of `cols`, zero beyond it
__device__ __forceinline__ f32x4 few_load4(const float* __restrict__ row, int col, int cols) {
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
    if (col + 4 <= cols) return *reinterpret_cast<const few_f32x4u*>(row + col);
#pragma unroll
    for (int e = 0; e < 3; ++e)
        if (col + e < cols) r[e] = row[col + e];
    return r;
}
__device__ __forceinline__ f32x4 few_load4(const bf16_t* __restrict__ row, int col, int cols) { return load4(row, col, cols); }
__device__ __forceinline__ void few_store4(float* __restrict__ row, int col, int cols, f32x4 v) {
    if (col + 4 <= cols) {
        *reinterpret_cast<few_f32x4u*>(row + col) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (col + e < cols) row[col + e] = v[e];
    }
}
__device__ __forceinline__ void few_store4(bf16_t* __restrict__ row, int col, int cols, f32x4 v) { store4(row, col, cols, v); }

// The four entries without a branch around the load, so that waiting for one load is not waiting for all of them:
// few_peek4 reads the row's last four where the end is near (rows hold four columns or more), few_settle4 moves them.
__device__ __forceinline__ f32x4 few_peek4(const float* __restrict__ row, int col, int cols) {
    return *reinterpret_cast<const few_f32x4u*>(row + min(col, cols - 4));
}
__device__ __forceinline__ f32x4 few_settle4(f32x4 x, int col, int cols) {
    const int past = col - (cols - 4);                                     // 4 and more: nothing of the row is left
    if (past > 0)
        x = f32x4{past == 1 ? x[1] : past == 2 ? x[2] : past == 3 ? x[3] : 0.f, past == 1 ? x[2] : past == 2 ? x[3] : 0.f,
                  past == 1 ? x[3] : 0.f, 0.f};
    return x;
}
// to memory past the caches
__device__ __forceinline__ void few_store4_past(float* __restrict__ row, int col, int cols, f32x4 v) {
    if (col + 4 <= cols)
        __builtin_nontemporal_store(v, reinterpret_cast<few_f32x4u*>(row + col));
    else
        few_store4(row, col, cols, v);
}

// a thread's items of four columns: row r, columns 4 c .. 4 c + 3
struct FewItem {
    int r, c;
    __device__ __forceinline__ FewItem(int i, int items) : r(i / items), c(i - i / items * items) {}
    __device__ __forceinline__ void step(const FewItem& by, int items) {
        r += by.r, c += by.c;
        if (c >= items) c -= items, ++r;
    }
};

// NJ: class blocks of 16.  UPDATE: 0 factors only, 1 sums into plane blockIdx.x of `planes`, 2 straight into W (one workgroup).
// LATE: V leaves from LDS, a piece at a time between the matrix instructions, instead of between the loads (see few_late).
// Between the loads every wait for a load was one for the stores before it as well.
template <typename TIn, bool DIFF, int NJ, int UPDATE, bool LATE>
__global__ __launch_bounds__(kFewThreads) void few_step_kernel(FewArgs a, int rows_per_wg, int Dp, int k_slices, int groups) {
    constexpr int JP = 16 * NJ;
    extern __shared__ __attribute__((aligned(16))) float few_lds[];      // feature rows, then slices of scores; u overlays those
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int pitch = Dp + 4;
    const int row0 = blockIdx.x * rows_per_wg, rows = min(rows_per_wg, a.n_rows - row0);
    float* const feat = few_lds;
    float* const zp = few_lds + (int64_t)rows_per_wg * pitch;             // [k_slices][row blocks * 16][JP]
    const int row_blocks = (rows + 15) / 16, zrows = (rows_per_wg + 15) / 16 * 16;

    // features -> LDS (zeros up to Dp columns), and on to V
    const int items = Dp / 4;
    const FewItem first(tid, items), stride(kFewThreads, items);
    FewItem out = first;                                                   // what this thread stores of V next
    auto store_late = [&]() {
        if constexpr (LATE) {
            if (out.r < rows) {
                few_store4_past((float*)a.v + (row0 + out.r) * (int64_t)a.ldv, 4 * out.c, a.D,
                                *reinterpret_cast<const f32x4*>(&feat[out.r * pitch + 4 * out.c]));
                out.step(stride, items);
            }
        }
    };
    if constexpr (LATE) {
        constexpr int BATCH = DIFF ? 5 : 10;
        const float* A = (const float*)a.a + (int64_t)row0 * a.lda;
        const float* A2 = DIFF ? (const float*)a.a2 + (int64_t)row0 * a.lda : nullptr;
        for (FewItem at = first, to = first; to.r < rows;) {
            f32x4 x[BATCH], x2[DIFF ? BATCH : 1];
#pragma unroll
            for (int q = 0; q < BATCH; ++q) {
                if (at.r < rows) {
                    x[q] = few_peek4(A + (int64_t)at.r * a.lda, 4 * at.c, a.D);
                    if (DIFF) x2[q] = few_peek4(A2 + (int64_t)at.r * a.lda, 4 * at.c, a.D);
                }
                at.step(stride, items);
            }
#pragma unroll
            for (int q = 0; q < BATCH; ++q) {
                if (to.r < rows) {
                    if (DIFF) x[q] -= x2[q];
                    *reinterpret_cast<f32x4*>(&feat[to.r * pitch + 4 * to.c]) = few_settle4(x[q], 4 * to.c, a.D);
                }
                to.step(stride, items);
            }
        }
    } else {
        const int total = rows * items;
        const TIn* A = (const TIn*)a.a + (int64_t)row0 * a.lda;
        const TIn* A2 = DIFF ? (const TIn*)a.a2 + (int64_t)row0 * a.lda : nullptr;
        TIn* V = (TIn*)a.v + (int64_t)row0 * a.ldv;
        for (int i0 = 0; i0 < total; i0 += 4 * kFewThreads) {
            f32x4 x[4];
            int r[4], c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = min(i0 + q * kFewThreads + tid, total - 1);
                r[q] = i / items;
                c[q] = 4 * (i - r[q] * items);
                x[q] = few_load4(A + (int64_t)r[q] * a.lda, c[q], a.D);
                if (DIFF) x[q] -= few_load4(A2 + (int64_t)r[q] * a.lda, c[q], a.D);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (i0 + q * kFewThreads + tid < total) {
                    *reinterpret_cast<f32x4*>(&feat[r[q] * pitch + c[q]]) = x[q];
                    few_store4(V + (int64_t)r[q] * a.ldv, c[q], a.D, x[q]);
                }
            }
        }
    }
    __syncthreads();

    // (asked for before the late stores: a wait for a load waits for the stores before it as well)
    const int label0 = LATE ? a.y[row0 + min(tid / JP, rows - 1)] : 0;

    // scores: wavefront = (row block, slice of D)
    for (int job = wave; job < row_blocks * k_slices; job += kFewWaves) {
        const int rb = job % row_blocks, ks = job / row_blocks;
        const int steps = Dp / 16, per = (steps + k_slices - 1) / k_slices;
        const int s0 = ks * per, s1 = min(steps, s0 + per);
        f32x4 acc[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const float* fr = feat + min(rb * 16 + l16, rows - 1) * pitch + 4 * quad;
        const float* wr[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) wr[j] = a.w + (int64_t)min(16 * j + l16, a.J - 1) * a.ldw;
        constexpr int AHEAD = 4;
        f32x4 w[AHEAD][NJ];
#pragma unroll
        for (int p = 0; p < AHEAD; ++p)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (s0 + p < s1) w[p][j] = few_load4(wr[j], 16 * (s0 + p) + 4 * quad, a.D);
        for (int s = s0; s < s1; s += AHEAD) {
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) {
                if (s + p >= s1) break;
                const f32x4 f = *reinterpret_cast<const f32x4*>(fr + 16 * (s + p));
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j] = few_mfma(f[e], w[p][j][e], acc[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    if (s + p + AHEAD < s1) w[p][j] = few_load4(wr[j], 16 * (s + p + AHEAD) + 4 * quad, a.D);
                if ((p & 1) != 0) store_late();
            }
        }
        // lane: class 16 j + l16 of samples 16 rb + 4 quad + e
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) zp[(ks * zrows + rb * 16 + 4 * quad + e) * JP + 16 * j + l16] = acc[j][e];
    }
    if (UPDATE == 0 || a.use_mask) {                                       // (the rows of dead workers are cleared below)
        while (LATE && out.r < rows) store_late();
    }
    __syncthreads();

    // factor u: JP lanes to a sample
    constexpr int PER = kFewThreads / JP;                                 // samples at a time
    const int jl = tid % JP;
    float* const us = zp;                                                 // u of sample r at [r][JP]: slice 0's scores of that sample
    for (int r0 = 0; r0 < rows; r0 += PER) {
        const int r = r0 + tid / JP;
        const bool live = r < rows;
        const int rr = live ? r : rows - 1;
        float z = 0.f;
        for (int ks = 0; ks < k_slices; ++ks) z += zp[(ks * zrows + rr) * JP + jl];
        const int label = LATE && r0 == 0 ? label0 : a.y[row0 + rr];
        auto sum = [](float v) {
#pragma unroll
            for (int o = JP / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            return v;
        };
        float u, f;
        if (!DIFF) {                                                      // logistic: softmax - e_y
            float m = jl < a.J ? z : -INFINITY;
#pragma unroll
            for (int o = JP / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
            const float ex = jl < a.J ? __expf(z - m) : 0.f;
            const float total = sum(ex), zy = sum(jl == label && jl < a.J ? z : 0.f);
            u = ex * (1.0f / total) - (jl == label ? 1.0f : 0.0f);
            f = m + __logf(total) - zy;
        } else {                                                          // pairs: |z|^2 or the hinge
            const float q = sum(jl < a.J ? z * z : 0.f);
            u = z * (label != 0 ? 2.0f : (q < 1.0f ? -2.0f : 0.0f));
            f = label != 0 ? q : fmaxf(0.f, 1.0f - q);
        }
        if (live) {
            if (jl < a.J) a.u[(int64_t)(row0 + r) * a.ldu + jl] = u;
            if (a.loss != nullptr && jl == 0) a.loss[row0 + r] = f;
            if (UPDATE != 0) {
                bool on = jl < a.J;
                if (a.use_mask && !((a.live_mask >> ((row0 + r) / a.B)) & 1ull)) {
                    on = false;                                           // a dead worker's rows count as zero whatever they hold
                    for (int c = jl; c < Dp; c += JP) feat[r * pitch + c] = 0.f;
                }
                us[r * JP + jl] = on ? u : 0.f;                           // (its slice 0 score was read by this thread)
            }
        }
    }
    if constexpr (UPDATE == 0) return;
    // (the rows behind the last sample, up to whole sixteens, count as zero: u here, the features where they are read)
    __syncthreads();
    for (int i = rows * JP + tid; i < row_blocks * 16 * JP; i += kFewThreads) us[i] = 0.f;
    __syncthreads();

    // update: wavefront = groups of 64 columns
    for (int gi = wave; gi < groups; gi += kFewWaves) {
        const int d0 = 64 * gi, dc = d0 + 4 * l16;
        f32x4 acc[NJ][4];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 wold[NJ][4];
        if constexpr (UPDATE == 2) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    wold[j][e] = few_load4(a.w + (int64_t)min(16 * j + 4 * quad + e, a.J - 1) * a.ldw, min(dc, Dp), a.D);
        }
        const int col = min(dc, Dp - 4);
        for (int n = 0; n < row_blocks * 4; ++n) {                        // samples 4 n + quad
            store_late();
            f32x4 v = *reinterpret_cast<const f32x4*>(feat + min(4 * n + quad, rows - 1) * pitch + col);
            if (4 * n + 3 >= rows && 4 * n + quad >= rows) v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float u = us[(4 * n + quad) * JP + 16 * j + l16];
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[j][t] = few_mfma(u, v[t], acc[j][t]);
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * j + 4 * quad + e;
                const f32x4 s = {acc[j][0][e], acc[j][1][e], acc[j][2][e], acc[j][3][e]};
                if (row < a.J && dc < a.D) {
                    if constexpr (UPDATE == 2)
                        few_store4(a.w + (int64_t)row * a.ldw, dc, a.D, prox_entry4(wold[j][e] + a.alpha * s, a.prox_kind, a.prox_a));
                    else
                        *reinterpret_cast<f32x4*>(a.planes + ((int64_t)blockIdx.x * a.J + row) * Dp + dc) = s;
                }
            }
    }
    while (LATE && out.r < rows) store_late();
}

// W += alpha * (the planes' sums in plane order): four columns of a row to sixteen threads, each of which adds a
// sixteenth of the planes
constexpr int kFewApplyThreads = 256;
__global__ __launch_bounds__(kFewApplyThreads) void few_apply_kernel(float* __restrict__ W, int64_t ldw, const float* __restrict__ planes,
                                                                     int n_planes, int J, int D, int Dp, float alpha, int prox_kind,
                                                                     float prox_a) {
    __shared__ f32x4 part[16][16];
    const int c = threadIdx.x & 15, p = threadIdx.x >> 4;
    const int items = Dp / 4, i = blockIdx.x * 16 + c;
    const bool in = i < J * items;
    const int row = in ? i / items : 0, col = in ? 4 * (i - row * items) : 0;
    const int per = (n_planes + 15) / 16, p0 = p * per, p1 = min(n_planes, p0 + per);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    const float* src = planes + (int64_t)row * Dp + col;
#pragma unroll 8
    for (int k = p0; k < p1; ++k) s += *reinterpret_cast<const f32x4*>(src + (int64_t)k * J * Dp);
    part[p][c] = s;
    __syncthreads();
    if (p == 0 && in && col < D) {
        f32x4 t = part[0][c];
#pragma unroll
        for (int k = 1; k < 16; ++k) t += part[k][c];
        float* wrow = W + (int64_t)row * ldw;
        const f32x4 w = few_load4(wrow, col, D);
        few_store4(wrow, col, D, prox_entry4(w + alpha * t, prox_kind, prox_a));
    }
}

static int few_dp(int64_t D) { return (int)((D + 15) / 16 * 16); }

// Rows per workgroup (0: the shape does not fit): as many workgroups as compute units where there are samples for it,
// 16 rows or more where the 160 KB of LDS hold them (features and slices of scores), never less than 8.
static int few_rows(int64_t N, int64_t J, int64_t D, int* k_slices, size_t* lds) {
    const int dp = few_dp(D), jp = J > 16 ? 32 : 16;
    auto need = [&](int64_t rows, int ks) {
        return ((size_t)rows * (dp + 4) + (size_t)ks * ((rows + 15) / 16 * 16) * jp) * sizeof(float);
    };
    auto slices = [&](int64_t rows) {
        int ks = (int)(kFewWaves / ((rows + 15) / 16));
        if (ks < 1) ks = 1;
        if (ks > dp / 16) ks = dp / 16;
        while (ks > 1 && need(rows, ks) > 160 * 1024) --ks;
        return ks;
    };
    auto fits = [&](int64_t rows) { return need(rows, 1) <= 160 * 1024; };
    // one workgroup up to 64 samples (beyond, its serial parts cost more than the second kernel: 128 columns x 216
    // samples 16 us in one, 10 in fourteen)
    int64_t rows = N;
    if (!fits(rows) || N > 64) {
        rows = (N + 255) / 256;
        if (rows < 16) rows = 16;
        while (rows > 8 && !fits(rows)) --rows;
        if (!fits(rows)) return 0;
    }
    *k_slices = slices(rows);
    *lds = need(rows, *k_slices);
    return *lds <= 160 * 1024 ? (int)rows : 0;
}

// Long rows leave too few workgroups, each with too much to load (2944 columns of pairs, 768 samples: 40 us against 24
// for the separate kernels; 1664 columns, 144 samples: 15 against 19).
bool few_ok(int64_t N, int64_t J, int64_t D, bool diff) {
    int ks;
    size_t lds;
    return J <= 32 && D >= 4 && D <= (diff ? 1024 : 2048) && few_rows(N, J, D, &ks, &lds) > 0;
}

size_t few_workspace(int64_t N, int64_t J, int64_t D) {
    int ks;
    size_t lds;
    const int rows = few_rows(N, J, D, &ks, &lds);
    const int64_t n = rows > 0 ? (N + rows - 1) / rows : 0;
    return n > 1 ? (size_t)n * J * few_dp(D) * sizeof(float) : 0;
}

// Late stores are for batches that, with their V, are more than the L2s hold: the loads come first at the rate of memory,
// and the stores, which take as long again, run under the products; past the caches, so that the kernel's end has nothing
// to write back.  Steps of fp32, us, one batch again and again / a ring of batches of 1.2 to 2 GB: ten classes x 784 columns, 12000 samples 27.5 -> 24.6 /
// 32.9 -> 26.4, 8000 samples 22.0 -> 20.5 / 25.7 -> 22.8; thirteen classes x 1000, 9000 samples 30.6 -> 27.9 / 36.7 -> 29.8, pairs 36.5 -> 31.6 / 44.1 -> 34.0.
// Smaller batches have a piece or two to a thread and lose (256 columns x 512 samples 6.6 -> 7.7), bf16 rows too (12000
// samples 23.4 -> 24.7).  Batches of more than 256 workgroups gain where they are new and lose where they are not (thirteen classes x 1664, 7208 samples
// 71.9 -> 73.9 / 80.0 -> 78.6).  With two class blocks the products bound the kernel where a workgroup has hundreds of rows (twenty classes, 246 rows of 128 columns:
// 63.5 -> 66.6; 129 rows of 256: 32.5 -> 30.7) or follows another (twenty-four x 1280, 9368 samples 82.0 -> 86.4 / 90.4 -> 91.3; pairs gain there too).
static bool few_late(const FewArgs& a, int rows) {
    return !a.bf16 && (int64_t)a.n_rows * a.D * 4 >= (int64_t)22 << 20 && (a.J <= 16 || (rows <= 192 && (a.diff || (a.n_rows + rows - 1) / rows <= 256)));
}

template <typename TIn, bool DIFF, int NJ, int UPDATE, bool LATE>
static hipError_t launch_few_t(const FewArgs& a, int rows, int k_slices, size_t lds, hipStream_t s) {
    static std::atomic<bool> raised{false};
    if (lds > 64 * 1024 && !raised) {
        hipError_t e = hipFuncSetAttribute((const void*)few_step_kernel<TIn, DIFF, NJ, UPDATE, LATE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised = true;
    }
    SFB_LAUNCH((few_step_kernel<TIn, DIFF, NJ, UPDATE, LATE>), dim3((a.n_rows + rows - 1) / rows), dim3(kFewThreads), lds, s, a, rows,
               few_dp(a.D), k_slices, (a.D + 63) / 64);
    return hipGetLastError();
}

template <typename TIn, bool DIFF, int NJ>
static hipError_t launch_few_u(const FewArgs& a, int rows, int ks, size_t lds, int update, hipStream_t s) {
    if constexpr (sizeof(TIn) == 4) {
        if (few_late(a, rows)) return update == 0 ? launch_few_t<TIn, DIFF, NJ, 0, true>(a, rows, ks, lds, s)
                                            : launch_few_t<TIn, DIFF, NJ, 1, true>(a, rows, ks, lds, s);
    }
    if (update == 0) return launch_few_t<TIn, DIFF, NJ, 0, false>(a, rows, ks, lds, s);
    if (update == 1) return launch_few_t<TIn, DIFF, NJ, 1, false>(a, rows, ks, lds, s);
    return launch_few_t<TIn, DIFF, NJ, 2, false>(a, rows, ks, lds, s);
}

template <typename TIn, bool DIFF>
static hipError_t launch_few_j(const FewArgs& a, int rows, int ks, size_t lds, int update, hipStream_t s) {
    return a.J <= 16 ? launch_few_u<TIn, DIFF, 1>(a, rows, ks, lds, update, s) : launch_few_u<TIn, DIFF, 2>(a, rows, ks, lds, update, s);
}

hipError_t launch_few(const FewArgs& a, bool update, hipStream_t s) {
    int ks;
    size_t lds;
    const int rows = few_rows(a.n_rows, a.J, a.D, &ks, &lds);
    if (rows <= 0) return hipErrorInvalidValue;
    const int n = (a.n_rows + rows - 1) / rows, mode = !update ? 0 : n == 1 ? 2 : 1;
    hipError_t e = a.bf16 ? launch_few_j<bf16_t, false>(a, rows, ks, lds, mode, s)
                   : a.diff ? launch_few_j<float, true>(a, rows, ks, lds, mode, s)
                            : launch_few_j<float, false>(a, rows, ks, lds, mode, s);
    if (e != hipSuccess || mode != 1) return e;
    hipLaunchKernelGGL(few_apply_kernel, dim3((a.J * (few_dp(a.D) / 4) + 15) / 16), dim3(kFewApplyThreads), 0, s, a.w, a.ldw, a.planes,
                       n, a.J, a.D, few_dp(a.D), a.alpha, a.prox_kind, a.prox_a);
    return hipGetLastError();
}

}  // namespace sfb
