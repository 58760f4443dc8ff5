// Reconstruction + update (Section 3, Section 2.1) for sparse features:
//     W[j][d] <- W[j][d] + alpha * sum over the stored entries (i, d) of U[i][j] * v
// The dense contraction multiplies every pair by every column; at a few stored entries per hundred nearly all of that is
// multiplication by zero.  Two kernels instead:
//
// column_lists_kernel turns the dense rows V of the live workers (already written, repeated entries already added up) into
// lists of the non-zero entries per column, rows ascending, grouped by blocks of 32 columns.  One workgroup per block; lanes run
// along a row's 32 columns (128 contiguous bytes), every thread owns one column of 32 rows in registers: count, prefix
// sum over (column, part of the rows), write.  A block takes its place in the
// entry array with one atomic add: where a block lies depends on timing, what it holds does not.  The array holds the stored
// entries of the batch; row pointers that overlap make more non-zeros of them, and a block that finds no room then leaves no
// list but a mark (kNoList): its columns take every pair from V.
//
// sparse_update_kernel: a workgroup parks U[all pairs][32 classes] in LDS (128 KB at 1024 pairs) and walks its share
// of the column blocks, a wavefront per half block.  Sixteen lanes take a column, two classes each: every entry is one
// 8-byte LDS read per lane at the entry's row (the sixteen lanes read 128 contiguous bytes: no bank conflicts whatever
// the rows) and two multiply-adds; row and value are broadcast inside the sixteen lanes by the instruction's own
// lane operand (row_newbcast), so an entry costs three vector instructions and one LDS read for four columns at once.
// The sums of half a block turn through LDS into rows of W, which were requested before the walk.  The sum over a
// column runs over ascending rows: the same bits every time.  A class with a factor that is not finite takes every pair
// of its columns from V instead, as the dense contraction does: infinity times a zero that is not stored is NaN.
#include <type_traits>

#include "sfb_device.h"
#include "sfb_kernels.h"

namespace sfb {

constexpr int kClThreads = 1024, kClRows = 32;                           // 32 parts of 32 rows: at most 1024 pairs
constexpr int kSuThreads = 1024, kSuWaves = kSuThreads / 64, kSuClasses = 32;
constexpr int kSuTile = 16 * 32;                                          // sums of half a block, floats
constexpr uint32_t kNoList = 0x80000000u;                                // in place of a block's bounds: empty lists, take V

__global__ __launch_bounds__(kClThreads) void column_lists_kernel(const float* __restrict__ V, int64_t ldv, int N, int D,
                                                                  uint32_t* __restrict__ counter, uint32_t* __restrict__ starts,
                                                                  uint2* __restrict__ entries, uint32_t room, int B, uint64_t live_mask,
                                                                  int use_mask) {
    __shared__ uint32_t cnt[32 * 33];
    __shared__ uint32_t wsum[16], base_s;
    const int tid = threadIdx.x, c = tid & 31, part = tid >> 5;            // part: a contiguous range of rows
    const int d = blockIdx.x * 32 + c;
    const int r0 = part * kClRows;
    const float* at_row = V + (int64_t)min(r0, N - 1) * ldv + min(d, D - 1);
    float v[kClRows];                                                      // all loads in flight at once
#pragma unroll
    for (int r = 0; r < kClRows; ++r) {
        v[r] = *at_row;
        if (r0 + r + 1 < N) at_row += ldv;
    }
    // bit r: row r0 + r counts (a dead worker's rows count as zero whatever they hold: an infinity of theirs would leave NaN
    // against the zeros in place of their factors)
    uint32_t rows = d >= D || r0 >= N ? 0u : N - r0 >= kClRows ? ~0u : (1u << (N - r0)) - 1u;
    if (use_mask) {
        int p = r0 / B, left = B - (r0 - p * B);                           // worker of the row, its rows from here on
#pragma unroll 1
        for (int r = 0; r < kClRows && r0 + r < N; ++r) {
            if (!((live_mask >> p) & 1ull)) rows &= ~(1u << r);
            if (--left == 0) {
                left = B;
                ++p;
            }
        }
    }
    uint32_t n = 0;
#pragma unroll
    for (int r = 0; r < kClRows; ++r) {
        v[r] = ((rows >> r) & 1u) ? v[r] : 0.f;
        n += v[r] != 0.f;
    }
    // exclusive prefix sum in the order (column, part): thread tid handles position tid of that order
    cnt[c * 33 + part] = n;
    __syncthreads();
    const int oc = tid >> 5, op = tid & 31;                                // position tid = column oc, part op
    uint32_t x = cnt[oc * 33 + op], inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if ((tid & 63) >= o) inc += y;
    }
    if ((tid & 63) == 63) wsum[tid >> 6] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < (tid >> 6)) before += wsum[w];
        total += wsum[w];
    }
    if (tid == 0) base_s = atomicAdd(counter, total);
    cnt[oc * 33 + op] = before + inc - x;
    __syncthreads();
    const uint32_t base = base_s;                                          // (host: N * D below 2^32, the counter cannot wrap)
    const bool fits = (uint64_t)base + total <= room;
    uint32_t* st = starts + (int64_t)blockIdx.x * 33;
    if (tid < 32) st[tid] = fits ? base + cnt[tid * 33] : kNoList;
    if (tid == 32) st[32] = fits ? base + total : kNoList;
    uint32_t at = base + cnt[c * 33 + part];
    if (n != 0 && fits) {
#pragma unroll
        for (int r = 0; r < kClRows; ++r)
            if (v[r] != 0.f) entries[at++] = make_uint2((uint32_t)(r0 + r), __float_as_uint(v[r]));
    }
}

template <int N>
__device__ __forceinline__ uint32_t bcast16(uint32_t x) {   // lane N of every sixteen to all of them
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + N, 0xf, 0xf, false);
}
// a += (v of lane N of every sixteen) * u (s_nop: v may have been written by the vector instruction right before)
template <int N>
__device__ __forceinline__ void fmac_bcast16(float& a0, float& a1, float v, float2 u) {
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+&v"(a0), "+&v"(a1) : "v"(v), "v"(u.x), "v"(u.y), "n"(N));
}
template <int FIRST, int LAST, class F>
__device__ __forceinline__ void lane_loop(F f) {
    if constexpr (FIRST < LAST) {
        f(std::integral_constant<int, FIRST>{});
        lane_loop<FIRST + 1, LAST>(f);
    }
}

__global__ __launch_bounds__(kSuThreads) void sparse_update_kernel(
    float* __restrict__ W, int64_t ldw, const float* __restrict__ U, int64_t ldu, const uint32_t* __restrict__ starts,
    const uint2* __restrict__ entries, int N, int J, int D, int B, float alpha, uint64_t live_mask, int use_mask, int n_jb,
    int n_blocks, int splits, int prox_kind, float prox_a, const float* __restrict__ V, int64_t ldv) {
    extern __shared__ __attribute__((aligned(16))) float su_lds[];          // U [N][32], then a 32 x 32 tile per wavefront
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int id = xcd_contiguous_id(blockIdx.x, n_jb * splits);
    const int jb = id % n_jb, sp = id / n_jb;
    const int j0 = jb * kSuClasses;

    // U: eight lanes to a row; a bit per class for factors that are not finite (kept where the first tile will be: 1024 pairs
    // and the tiles fill the LDS)
    uint32_t* const bad_at = reinterpret_cast<uint32_t*>(su_lds + (int64_t)N * kSuClasses);
    uint32_t bad = 0;
    if (tid == 0) *bad_at = 0;
    for (int r = tid >> 3; r < N; r += kSuThreads / 8) {
        const int j = j0 + 4 * (tid & 7);
        bool live = true;
        if (use_mask) live = (live_mask >> (r / B)) & 1ull;
        f32x4 u = {0.f, 0.f, 0.f, 0.f};
        if (live && j < J) u = load4(U + (int64_t)r * ldu, j, J);
        *reinterpret_cast<f32x4*>(&su_lds[r * kSuClasses + 4 * (tid & 7)]) = u;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (!(fabsf(u[k]) < INFINITY)) bad |= 1u << (4 * (tid & 7) + k);
    }
    __syncthreads();
    if (bad != 0) atomicOr(bad_at, bad);
    __syncthreads();
    bad = __builtin_amdgcn_readfirstlane(*bad_at);
    __syncthreads();

    float* const tile = su_lds + (int64_t)N * kSuClasses + wave * kSuTile;
    const unsigned char* const slab = reinterpret_cast<const unsigned char*>(su_lds);
    const int g = lane >> 4, l16 = lane & 15;                              // group of sixteen = column, lane = two classes
    const uint32_t lane_off = 8u * l16;
    const int per = (n_blocks + splits - 1) / splits;
    const int b_end = min(n_blocks, (sp + 1) * per);
    const int wr = lane >> 2, wc = 4 * (lane & 3);                         // W rows wr, wr + 16, columns wc .. wc + 3 of the half

    // half blocks of 16 columns, a wavefront each
    for (int h = 2 * sp * per + wave; h < 2 * b_end; h += kSuWaves) {
        const int d0 = h * 16;
        f32x4 w[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = j0 + wr + 16 * t;
            w[t] = row < J ? load4(W + (int64_t)row * ldw, d0 + wc, D) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const uint32_t* st = starts + (int64_t)(h >> 1) * 33 + 16 * (h & 1);
        // columns 4 q + g: four at a time, all four rounds' bounds first
        int beg[4], len[4];
        uint32_t no_list = 0;                                               // the same in every lane: the whole block's
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t b = st[4 * q + g];
            no_list = b & kNoList;
            beg[q] = (int)(b & ~kNoList);
            len[q] = (int)(st[4 * q + g + 1] - b);
        }
        uint2 e = entries[beg[0] + min(l16, max(len[0] - 1, 0))];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float a0 = 0.f, a1 = 0.f;
            const int longest = max(max(__builtin_amdgcn_readlane(len[q], 0), __builtin_amdgcn_readlane(len[q], 16)),
                                    max(__builtin_amdgcn_readlane(len[q], 32), __builtin_amdgcn_readlane(len[q], 48)));
            for (int e0 = 0;; e0 += 16) {
                // lanes past the column's end: row 0, value 0
                const bool in = e0 + l16 < len[q];
                const uint32_t off = in ? e.x * (kSuClasses * 4u) : 0u;
                const float val = in ? __uint_as_float(e.y) : 0.f;
                // request the next sixteen entries, of this column or the first of the next round's
                constexpr int kLast = 3;
                const int qn = q < kLast ? q + 1 : q;
                if (e0 + 16 < longest) e = entries[beg[q] + min(e0 + 16 + l16, max(len[q] - 1, 0))];
                else if (q < kLast) e = entries[beg[qn] + min(l16, max(len[qn] - 1, 0))];
                // straight-line code per count of four entries: all rows of U requested, then multiplied as they arrive
                const int left = longest - e0;                              // uniform
                auto walk = [&](auto count) {
                    constexpr int C = decltype(count)::value;
                    float2 u[C];
                    lane_loop<0, C>([&](auto n) {
                        constexpr int F = decltype(n)::value;
                        u[F] = *reinterpret_cast<const float2*>(slab + (bcast16<F>(off) + lane_off));
                    });
                    lane_loop<0, C>([&](auto n) {
                        constexpr int F = decltype(n)::value;
                        fmac_bcast16<F>(a0, a1, val, u[F]);
                    });
                };
                if (left > 12) walk(std::integral_constant<int, 16>{});
                else if (left > 8) walk(std::integral_constant<int, 12>{});
                else if (left > 4) walk(std::integral_constant<int, 8>{});
                else if (left > 0) walk(std::integral_constant<int, 4>{});
                if (left <= 16) break;
            }
            // sums of column 4 q + g: [column][class], classes XORed with the column's quad so that the rows read back
            // below fall on different banks
            *reinterpret_cast<float2*>(&tile[(4 * q + g) * 32 + ((2 * l16) ^ (8 * q))]) = make_float2(a0, a1);
        }
        // (one wavefront's own tile: its LDS operations are in order)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = j0 + wr + 16 * t;
            f32x4 s;
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] = tile[(wc + k) * 32 + ((wr + 16 * t) ^ (2 * wc))];
            if (no_list != 0 || (bad != 0 && ((bad >> (wr + 16 * t)) & 1u))) {
                s = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int r = 0; r < N; ++r) {
                    if (use_mask && !((live_mask >> (r / B)) & 1ull)) continue;
                    const float u = su_lds[r * kSuClasses + wr + 16 * t];
#pragma unroll
                    for (int k = 0; k < 4; ++k) s[k] += u * V[(int64_t)r * ldv + min(d0 + wc + k, D - 1)];
                }
            }
            if (row < J) store4(W + (int64_t)row * ldw, d0 + wc, D, prox_entry4(w[t] + alpha * s, prox_kind, prox_a));
        }
    }
}

// bytes of workspace for `stored` entries of D columns: the counter, 33 bounds per block of 32 columns, the entries
static size_t lists_head(int64_t D) { return 256 + ((size_t)((D + 31) / 32) * 33 * sizeof(int32_t) + 255) / 256 * 256; }
// (the walk may look at one entry behind the last list)
size_t sparse_update_workspace(int64_t D, int64_t stored) { return lists_head(D) + (size_t)(stored + 1) * sizeof(uint2); }

// U of 32 classes and the wavefronts' tiles have to fit in LDS; entry numbers are below kNoList, and V can hold no more
// non-zeros than the lists' 32-bit counter counts
bool sparse_update_ok(int64_t N, int64_t D, int64_t stored) {
    return ((size_t)N * kSuClasses + kSuWaves * kSuTile) * sizeof(float) <= 160 * 1024 && N * D < (1LL << 32) &&
           stored < (int64_t)kNoList - 1;
}

static int sparse_update_splits(int64_t J, int64_t D) {
    const int64_t n_blocks = (D + 31) / 32, n_jb = (J + kSuClasses - 1) / kSuClasses;
    int64_t s = 256 / n_jb;                                                // one round of workgroups, one per compute unit
    if (s < 1) s = 1;
    return (int)(s < n_blocks ? s : n_blocks);
}

// Microseconds on one MI355X: the lists at 3.3 TB/s of V, then per workgroup 1.12 ns an entry of its columns (or W at
// 4 TB/s).  2000 x 8192, 1024 pairs: 65 us at 2 % stored against 150 for the dense contraction (which wins from about 5 %).
double sparse_update_us(int64_t N, int64_t J, int64_t D, int64_t stored) {
    const double n_jb = (double)((J + kSuClasses - 1) / kSuClasses), splits = (double)sparse_update_splits(J, D);
    const double rounds = (double)(int64_t)((n_jb * splits + 255.0) / 256.0);
    const double walk = rounds * 1.12e-3 * (double)stored / splits, w_us = 2e-6 * (double)J * (double)D;
    return 6.0 + 1.2e-6 * (double)N * (double)D + 7.0 + (walk > w_us ? walk : w_us);
}

hipError_t launch_sparse_update(const ReconArgs& a, int64_t stored, void* workspace, hipStream_t s) {
    const int n_blocks = (a.D + 31) / 32, n_jb = (a.J + kSuClasses - 1) / kSuClasses;
    uint32_t* counter = (uint32_t*)workspace;                              // zero: csr_densify_kernel of this step cleared it
    uint32_t* starts = (uint32_t*)((char*)workspace + 256);
    uint2* entries = (uint2*)((char*)workspace + lists_head(a.D));
    hipLaunchKernelGGL(column_lists_kernel, dim3(n_blocks), dim3(kClThreads), 0, s, (const float*)a.v, a.ldv, a.N, a.D,
                       counter, starts, entries, (uint32_t)stored, a.B, a.live_mask, a.use_mask ? 1 : 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds_bytes = ((size_t)a.N * kSuClasses + kSuWaves * kSuTile) * sizeof(float);
    static std::atomic<bool> raised{false};
    if (lds_bytes > 64 * 1024 && !raised) {
        e = hipFuncSetAttribute((const void*)sparse_update_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int splits = sparse_update_splits(a.J, a.D);
    SFB_LAUNCH(sparse_update_kernel, dim3(n_jb * splits), dim3(kSuThreads), lds_bytes, s, a.w, a.ldw, a.u, a.ldu, starts, entries,
               a.N, a.J, a.D, a.B, a.alpha, a.live_mask, a.use_mask ? 1 : 0, n_jb, n_blocks, splits, a.prox_kind, a.prox_a,
               (const float*)a.v, a.ldv);
    return hipGetLastError();
}

}  // namespace sfb
