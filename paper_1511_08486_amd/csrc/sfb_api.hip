// C ABI of the SFB library (see include/sfb.h): argument validation, launch plans,
// and the order of kernel launches for one bulk-synchronous SFB iteration.
// Host code only; every step of the computation runs in the kernels.
#include "../../include/sfb.h"

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <new>
#include <vector>

#include "sfb_kernels.h"

using namespace sfb;

namespace {
constexpr int kFamilies = 6;  // 0 scores, 1 factor u, 2 reconstruct-apply, 3 sparse helpers, 4 proximal step, 5 one-pass update + next scores
struct EventPair { hipEvent_t a, b; };
struct LastKernel { const char* name; uint32_t grid; };   // what SFB_LAUNCH left

// Scratch of the entry point that allocates nothing (sfb_step_noalloc): device memory that belongs
// to the library's code object, one copy per GPU the library is loaded on, held until the process
// ends.  It plays the role of the registered workspace (split-K partial scores, packed bf16
// factors), every byte of which a step writes before reading it, so nothing has to be cleared
// between calls.  In host code the array's NAME is only a handle for hipGetSymbolAddress; kernels
// are given the device address kept in static_scratch_ptr.
constexpr size_t kStaticScratchBytes = SFB_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::atomic<void*> static_scratch_ptr[kMaxDevices];     // zero-initialised: not resolved yet

// Device address of `scratch` on the current device, resolved once per device.
hipError_t resolve_static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* p = static_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        static_scratch_ptr[dev].store(p, std::memory_order_release);   // every thread resolves the same address
    }
    *out = p;
    return hipSuccess;
}
}  // namespace

namespace sfb {
LaunchEvents& launch_events() {
    static thread_local LaunchEvents le{nullptr, nullptr, false, nullptr, 0};
    return le;
}
}  // namespace sfb

struct sfb_ctx {
    sfb_model model;
    int64_t J, D;
    int32_t P, B;
    sfb_dtype dtype;
    hipStream_t stream;
    FwdPlan fwd_all, fwd_worker;   // scores of all N rows / of one worker's B rows
    FwdPlan fwd_bf16;              // all N rows on the bf16 matrix cores (bf16 contexts)
    Bf16TilePlan tile_scores[2][2];   // bf16 contexts: scores in tiles, all rows or one worker's, W rounded or exact
    Bf16TilePlan tile_update[2];   // bf16 contexts: update in tiles, all pairs or one worker's
    bool tile_bf16_scores, tile_bf16_update;   // take them (a score tile or an update of the caller's choice is about the 256-row kernels)
    FwdPlan fwd_split, fwd_split_worker;   // the same on the 16-bit matrix cores, fp32 operands split into terms
    bool split_scores;             // use them where the shape allows
    int split_recon;               // reconstruction with split products: 1 where the shape allows, 0 never, -1 where it is the cheaper one
    SplitReconPlan split_plans[2][2];      // its tile and slices: all pairs or one worker's, without or with a workspace
    ReconPlan recon;
    ReconPlan recon_padded;        // the plan of the padded shape (ragged fp32 contexts: see padded_factors)
    bool padded_factors;           // fp32 and J, D or P*B not what the LDS-DMA reconstructions take as they are
    FusedPlan fused;               // update fused with the next scores (bf16 contexts whose shape it covers)
    bool fused_ok, use_fused;
    void* ws;
    size_t ws_bytes;
    int last_hip;
    bool timing;
    bool few;                      // at most 32 classes: whole steps in one pass over the features (sfb_few.hip)
    void* lists;                   // L2SVM: where in the workspace this step's column lists may go (null: no room), and
    int64_t lists_stored;          //   the number of stored entries of its batch
    bool sparse_forward;           // L2SVM: scores from the CSR entries when W rows fit in LDS and that is the cheaper pass
    bool sparse_always;            //   ... whenever they fit (no cost comparison)
    bool lists_always;             // L2SVM: the update from the column lists wherever they fit (no cost comparison)
    LastKernel last[kFamilies];    // main kernel of every family's last launch (name null: none yet)
    std::vector<EventPair> used[kFamilies], spare;
};

namespace {

inline int64_t round_up4(int64_t x) { return (x + 3) / 4 * 4; }

// Bytes of split-K partial scores (the first region of the workspace), rounded to 256.
size_t scores_need(const sfb_ctx* c) {
    const int64_t ldz = round_up4(c->J);
    const bool split = c->split_scores && c->D >= 4;
    size_t need = (size_t)(split ? c->fwd_split : c->fwd_all).split_k * (size_t)c->P * c->B * ldz * sizeof(float);
    const size_t one = (size_t)(split ? c->fwd_split_worker : c->fwd_worker).split_k * (size_t)c->B * ldz * sizeof(float);
    if (one > need) need = one;
    if (c->dtype == SFB_BF16) {
        const size_t bf = (size_t)c->fwd_bf16.split_k * (size_t)c->P * c->B * ldz * sizeof(float);
        if (bf > need) need = bf;
    }
    if (c->fused_ok) {
        const size_t fu = (size_t)c->fused.slices * (size_t)c->P * c->B * ldz * sizeof(float);
        if (fu > need) need = fu;
    }
    return (need + 255) / 256 * 256;
}

// bf16 contexts append the transposed bf16 factors of the reconstruction.
size_t workspace_need(const sfb_ctx* c) {
    size_t need = scores_need(c);
    if (c->dtype == SFB_BF16) need += bf16_recon_workspace(c->J, c->D, (int64_t)c->P * c->B);
    if (c->fused_ok) need += fused_extra_workspace(c->D, (int64_t)c->P * c->B);   // staged next features, last
    // ragged fp32 shapes: padded copies of the factors, made and used inside one reconstruction, when the
    // partial scores (consumed by the factor kernel of the same call that wrote them) are dead: same bytes
    // few tiles and many factor pairs: planes of partial sums behind those copies (or behind the masked copy of U)
    if (c->padded_factors) {
        const size_t pad = conform_workspace(c->J, c->D, (int64_t)c->P * c->B) +
                           reconstruct_small_split_workspace(c->recon_padded.n_split, c->J, conform_cols(c->D));
        if (pad > need) need = pad;
    } else if (c->dtype == SFB_F32 && c->recon.n_split > 1) {
        const size_t sp = masked_workspace(c->J, (int64_t)c->P * c->B) +
                          reconstruct_small_split_workspace(c->recon.n_split, c->J, c->D);
        if (sp > need) need = sp;
    }
    // few classes: planes of sums, one per workgroup (sfb_create has made sure that they stay within bounds)
    if (c->few) {
        const size_t planes = few_workspace((int64_t)c->P * c->B, c->J, c->D);
        if (planes > need) need = planes;
    }
    // sparse features: lists of the stored entries per column behind the scores, for one entry in twelve or as many as the
    // bytes that sfb_step_noalloc has leave room for
    if (c->model == SFB_L2SVM) {
        const size_t n = (size_t)c->P * c->B;
        size_t at = (n * round_up4(c->J) * sizeof(float) + 255) / 256 * 256 + sparse_update_workspace(c->D, (int64_t)(n * c->D / 12));
        if (at > SFB_NOALLOC_SCRATCH_BYTES) at = SFB_NOALLOC_SCRATCH_BYTES;
        if (at > need && sparse_update_ok((int64_t)n, c->D, (int64_t)(n * c->D / 12))) need = at;
    }
    // the column projection of the proximal step reuses the front of the buffer between steps
    const size_t prox = prox_workspace(c->J, c->D);
    return need > prox ? need : prox;
}

// The split products' plans.  exact: three terms an operand throughout, where the caller chose them (sfb_set_plan) or features are sparse: a sum of
// a few products has the error of its products, and those of two terms are the rougher ones (2 % stored: 8e-8 of the norm against 4e-8).
// chosen: ... and sums in two halves however short, which has half the error of a long one (by default only walks of 48 chunks and more, where
// it is below the fp32 instruction's and costs nothing that shows: positive operands, 4096 of them, 3.0e-7 of the norm in one sum, 1.5e-7 in two).
constexpr int kSplitHalves = 48, kSplitHalvesChosen = 4;
void plan_split_scores(sfb_ctx* c, bool exact, bool chosen) {
    const int halves = chosen ? kSplitHalvesChosen : kSplitHalves;
    const int64_t N = (int64_t)c->P * c->B;
    // room for the partial scores: what ragged contexts reserve for their padded factor copies anyway, or a few MiB; the
    // others the 16 MiB that sfb_step_noalloc has; or what the fp32 instruction's plan would take, where that is more
    size_t most = SFB_NOALLOC_SCRATCH_BYTES;
    if (c->padded_factors) {
        most = conform_workspace(c->J, c->D, N);
        if (most < ((size_t)4 << 20)) most = (size_t)4 << 20;
    }
    const size_t f32_need = (size_t)c->fwd_all.split_k * (size_t)N * (size_t)round_up4(c->J) * sizeof(float);
    if (f32_need > most) most = f32_need;
    c->fwd_split = plan_forward_split(N, c->J, c->D, most, exact, halves);
    c->fwd_split_worker = plan_forward_split(c->B, c->J, c->D, (size_t)c->fwd_split.split_k * (size_t)N * (size_t)round_up4(c->J) * sizeof(float), exact, halves);
}
void plan_split_recon(sfb_ctx* c, bool exact, bool chosen) {
    if (c->dtype != SFB_F32) return;
    for (int one = 0; one < 2; ++one)
        for (int with_ws = 0; with_ws < 2; ++with_ws)
            c->split_plans[one][with_ws] = reconstruct_split_plan(c->J, c->D, one ? c->B : (int64_t)c->P * c->B, with_ws ? workspace_need(c) : 0, exact,
                                                                  chosen ? kSplitHalvesChosen : kSplitHalves);
}

// The tiles' slices are cut to the bytes the context asks for: to be planned again whenever those change (sfb_set_plan).
void plan_bf16_tiles(sfb_ctx* c) {
    if (c->dtype != SFB_BF16) return;
    for (int one = 0; one < 2; ++one) {
        const int64_t N = one ? c->B : (int64_t)c->P * c->B;
        for (int exact = 0; exact < 2; ++exact) c->tile_scores[one][exact] = plan_scores_bf16(N, c->J, c->D, exact ? 3 : 1, scores_need(c));
        c->tile_update[one] = plan_update_bf16(c->J, c->D, N, workspace_need(c));
    }
}

sfb_status hip_fail(sfb_ctx* c, hipError_t e) {
    c->last_hip = (int)e;
    return SFB_EHIP;
}

// Arms a pair of events for the next kernel launch when timing is on (see SFB_LAUNCH), and notes the last kernel
// launched in its scope as the family's.
struct Timed {
    sfb_ctx* c;
    int fam;
    EventPair ev;
    bool on;
    Timed(sfb_ctx* ctx, int family) : c(ctx), fam(family), on(ctx->timing) {
        launch_events().name = nullptr;
        if (!on) return;
        if (!c->spare.empty()) {
            ev = c->spare.back();
            c->spare.pop_back();
        } else {
            hipError_t e = hipEventCreate(&ev.a);
            if (e == hipSuccess) {
                e = hipEventCreate(&ev.b);
                if (e != hipSuccess) (void)hipEventDestroy(ev.a);
            }
            if (e != hipSuccess) {          // this launch goes untimed; the caller can see why
                c->last_hip = (int)e;
                on = false;
                return;
            }
        }
        LaunchEvents& le = launch_events();
        le.start = ev.a;
        le.stop = ev.b;
        le.armed = true;
    }
    ~Timed() {
        LaunchEvents& le = launch_events();
        if (le.name) c->last[fam] = LastKernel{le.name, le.blocks};
        if (!on) return;
        if (le.armed) {             // nothing was launched: the events hold no timestamps
            le.armed = false;
            c->spare.push_back(ev);
        } else {
            c->used[fam].push_back(ev);
        }
    }
};

sfb_status check_common(const sfb_ctx* c, const float* W, int64_t ldw, const float* U, int64_t ldu,
                        const void* V, int64_t ldv) {
    if (!c || !W || !U || !V) return SFB_EINVAL;
    if (ldw < c->D || ldu < c->J || ldv < c->D) return SFB_ESHAPE;
    return SFB_OK;
}

sfb_status check_batch(const sfb_ctx* c, const sfb_batch* b, const int32_t* y) {
    if (!b || !y) return SFB_EINVAL;
    if (c->model == SFB_L2SVM) {
        if (!b->csr_rowptr || (b->nnz > 0 && (!b->csr_col || !b->csr_val))) return SFB_EINVAL;
        if (b->nnz < 0) return SFB_ESHAPE;
    } else {
        if (!b->a) return SFB_EINVAL;
        if (c->model == SFB_DML && !b->a2) return SFB_EINVAL;
        if (b->lda < c->D) return SFB_ESHAPE;
    }
    return SFB_OK;
}

// Factor u (and the loss) of `n_rows` samples from the `split_k` partial scores at the front of the workspace.
sfb_status factor_rows(sfb_ctx* c, int split_k, int64_t zstride, const int32_t* y, int64_t row0, int n_rows, float* U,
                       int64_t ldu, float* loss, const sfb_sdca* sdca) {
    FactorArgs g{};
    g.zp = (const float*)c->ws; g.ldz = round_up4(c->J); g.zstride = zstride; g.split_k = split_k;
    g.y = y; g.u = U + row0 * ldu; g.ldu = ldu; g.loss = loss ? loss + row0 : nullptr;
    g.n_rows = n_rows; g.J = (int)c->J; g.model = (Model)c->model;
    if (sdca) {
        g.sdca = SdcaDev{sdca->sample, sdca->dual, sdca->ld_dual, sdca->conj, sdca->s};
    }
    Timed t(c, 1);
    hipError_t e = launch_factor(g, c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

uint64_t live_workers(const sfb_ctx* c, const uint8_t* active, bool* use_mask) {
    *use_mask = false;
    if (!active) return ~0ull;
    uint64_t m = 0;
    for (int p = 0; p < c->P; ++p) {
        if (active[p]) m |= (1ull << p); else *use_mask = true;
    }
    return m;
}

// At most 32 classes, dense features: the factors of `n_rows` samples (outputs from row `row0` on) and, with `update`, the
// update of W by them, in one pass over the features.
sfb_status few_rows(sfb_ctx* c, float* W, int64_t ldw, const sfb_batch* b, const int32_t* y, int64_t row0, int n_rows, float* U,
                    int64_t ldu, void* V, int64_t ldv, float* loss, bool update, float alpha = 0.f, const uint8_t* active = nullptr,
                    int prox_kind = 0, float prox_a = 0.f) {
    if (c->ws == nullptr || c->ws_bytes < workspace_need(c)) return SFB_EWORKSPACE;
    FewArgs f{};
    f.bf16 = c->dtype == SFB_BF16;
    f.diff = c->model == SFB_DML;
    f.a = b->a; f.a2 = f.diff ? b->a2 : nullptr; f.lda = b->lda;
    f.w = W; f.ldw = ldw; f.y = y;
    f.u = U + row0 * ldu; f.ldu = ldu;
    f.v = (char*)V + (size_t)row0 * ldv * (f.bf16 ? 2 : 4); f.ldv = ldv;
    f.loss = loss ? loss + row0 : nullptr;
    f.planes = (float*)c->ws;
    f.n_rows = n_rows; f.J = (int)c->J; f.D = (int)c->D; f.B = c->B;
    f.alpha = alpha;
    f.live_mask = live_workers(c, active, &f.use_mask);
    f.prox_kind = prox_kind; f.prox_a = prox_a;
    {
        Timed t(c, 0);
        hipError_t e = launch_few(f, update, c->stream);
        if (e != hipSuccess) return hip_fail(c, e);
    }
    c->last[1] = c->last[0];                                     // one kernel is all of the step, or of its factors
    if (update) c->last[2] = c->last[0];
    return SFB_OK;
}

// Factors of `n_rows` samples whose outputs start at row `row0` of U, V, loss.
sfb_status factors_rows(sfb_ctx* c, const FwdPlan& plan, const float* W, int64_t ldw, const sfb_batch* b,
                        const int32_t* y, int64_t row0, int n_rows, float* U, int64_t ldu, void* V,
                        int64_t ldv, float* loss, const sfb_sdca* sdca = nullptr) {
    if (c->ws == nullptr || c->ws_bytes < workspace_need(c)) return SFB_EWORKSPACE;
    c->lists = nullptr;
    if (c->few && !sdca && few_ok(n_rows, c->J, c->D, c->model == SFB_DML))
        return few_rows(c, const_cast<float*>(W), ldw, b, y, row0, n_rows, U, ldu, V, ldv, loss, false);
    const bool bf16 = c->dtype == SFB_BF16;
    const size_t vsz = bf16 ? 2 : 4;
    void* v_rows = (char*)V + (size_t)row0 * ldv * vsz;
    const int64_t ldz = round_up4(c->J);

    FwdArgs f{};
    f.w = W; f.ldw = ldw;
    f.zp = (float*)c->ws; f.ldz = ldz; f.zstride = (int64_t)n_rows * ldz;
    f.n_rows = n_rows; f.J = (int)c->J; f.D = (int)c->D;
    f.bf16 = bf16;
    bool sparse_scores = false;
    if (c->model == SFB_L2SVM) {
        // scores from the stored entries only (2*nnz*J flops), or the dense contraction on the densified rows
        sparse_scores = c->sparse_forward && csr_scores_ok((int)c->D) && b->nnz <= (1LL << 30) - 1024 &&
                        (c->sparse_always || csr_scores_wins(n_rows, c->J, c->D, b->nnz));
        // the update of the same step may want lists of the entries per column, behind the planes of scores: where the bytes
        // that the context asks for hold them, so that sfb_step and sfb_step_noalloc, which differ in the bytes they have,
        // take the same kernel (contexts that ask for more than the latter's array are refused there and may use what they got)
        if (n_rows == c->P * c->B && sparse_update_ok(n_rows, c->D, b->nnz)) {
            const int planes = sparse_scores ? 1 : c->split_scores && c->D >= 4 ? c->fwd_split.split_k : plan.split_k;
            const size_t at = ((size_t)planes * n_rows * ldz * sizeof(float) + 255) / 256 * 256;
            const size_t asked = workspace_need(c), room = asked <= SFB_NOALLOC_SCRATCH_BYTES ? asked : c->ws_bytes;
            if (at + sparse_update_workspace(c->D, b->nnz) <= room) {
                c->lists = (char*)c->ws + at;
                c->lists_stored = b->nnz;
            }
        }
        // v_i first: the dense rows are what the reconstruction multiplies
        DensifyArgs d{b->csr_rowptr, b->csr_col, b->csr_val, (float*)v_rows, ldv, n_rows, (int)c->D, b->nnz, (uint32_t*)c->lists};
        {
            Timed t(c, 3);
            hipError_t e = launch_csr_densify(d, c->stream);
            if (e != hipSuccess) return hip_fail(c, e);
        }
        if (sparse_scores) {
            Timed t(c, 0);
            hipError_t e = launch_csr_scores(d, W, ldw, (float*)c->ws, ldz, (int)c->J, c->stream);
            if (e != hipSuccess) return hip_fail(c, e);
        } else {
            f.a = v_rows; f.a2 = nullptr; f.lda = ldv; f.v = nullptr; f.ldv = 0; f.diff = false;
        }
    } else {
        f.a = b->a; f.a2 = (c->model == SFB_DML) ? b->a2 : nullptr; f.lda = b->lda;
        f.v = v_rows; f.ldv = ldv; f.diff = (c->model == SFB_DML);
    }
    // bf16 features, full batch, aligned: the bf16 matrix-core kernel with its own plan
    const bool on_bf16_cores = bf16 && n_rows == c->P * c->B && n_rows >= 128 && forward_bf16_ok(f);
    // W is rounded to bf16 where that kernel would, and taken exactly in all other bf16 calls
    const Bf16TilePlan& tiles = c->tile_scores[n_rows != c->P * c->B][!on_bf16_cores];
    const size_t tile_planes = (size_t)tiles.slices * (size_t)n_rows * (size_t)ldz * sizeof(float);
    if (bf16 && c->tile_bf16_scores && scores_bf16_ok(f) && tiles.bm > 0 && tile_planes <= scores_need(c) &&
        !(on_bf16_cores && forward_bf16_wins(c->fwd_bf16, n_rows, c->J, c->D, tiles.us))) {
        {
            Timed t(c, 0);
            hipError_t e = launch_scores_bf16(f, tiles, c->stream);
            if (e != hipSuccess) return hip_fail(c, e);
        }
        return factor_rows(c, tiles.slices, f.zstride, y, row0, n_rows, U, ldu, loss, sdca);
    }
    // fp32 features: split-bf16 products, unless the caller chose the fp32 matrix instruction (sfb_set_plan).  Leading
    // dimensions beyond its 32-bit offsets take the fp32 kernels, whose plan may cut D into more slices than there is room for
    const bool all_rows = n_rows == c->P * c->B;
    const bool on_split = !sparse_scores && !bf16 && c->split_scores && forward_split_ok(f);
    FwdPlan used = on_bf16_cores ? c->fwd_bf16 : on_split ? (all_rows ? c->fwd_split : c->fwd_split_worker) : plan;
    if (!sparse_scores && !on_split && !on_bf16_cores) {
        const int64_t fit = (int64_t)(scores_need(c) / ((size_t)n_rows * ldz * sizeof(float)));
        if (used.split_k > fit) {
            used.split_k = (int)fit;
            finish_forward_plan(&used, n_rows, c->J, c->D);
        }
    }
    if (!sparse_scores) {
        Timed t(c, 0);
        hipError_t e = on_bf16_cores ? launch_forward_bf16(f, used, c->stream)
                       : on_split    ? launch_forward_split(f, used, c->stream)
                                     : launch_forward(f, used, c->stream);
        if (e != hipSuccess) return hip_fail(c, e);
    }
    return factor_rows(c, sparse_scores ? 1 : used.split_k, f.zstride, y, row0, n_rows, U, ldu, loss, sdca);
}

sfb_status check_sdca(const sfb_ctx* c, const sfb_sdca* d) {
    if (!d || !d->dual || !d->sample || d->n_data < 1) return SFB_EINVAL;
    if (!std::isfinite(d->lam) || !(d->lam > 0.f) || !std::isfinite(d->s) || !(d->s > 0.f) || d->s > 1.f)
        return SFB_EINVAL;
    if (d->ld_dual < c->J) return SFB_ESHAPE;
    if (c->model != SFB_MLR) return SFB_EUNSUPPORTED;
    return SFB_OK;
}

sfb_status check_recon(const sfb_ctx* c, float eta, float scale, const uint8_t* active) {
    if (!std::isfinite(eta) || !std::isfinite(scale)) return SFB_EINVAL;
    if (active && c->P > 64) return SFB_EUNSUPPORTED;
    return SFB_OK;
}

// n_rows: factor pairs to contract over (0 = all P*B; a single worker's B otherwise, no mask)
// same_step: U, V are what factors_rows has just left (the column lists it made room for may be used)
sfb_status recon_launch(sfb_ctx* c, float* W, int64_t ldw, const float* U, int64_t ldu, const void* V,
                        int64_t ldv, float eta, float scale, const uint8_t* active, int n_rows = 0,
                        int prox_kind = 0, float prox_a = 0.f, bool same_step = false) {
    ReconArgs r{};
    r.w = W; r.ldw = ldw; r.u = U; r.ldu = ldu; r.v = V; r.ldv = ldv;
    r.J = (int)c->J; r.D = (int)c->D; r.N = n_rows > 0 ? n_rows : c->P * c->B; r.B = c->B;
    r.alpha = -eta * scale;
    r.bf16 = c->dtype == SFB_BF16;
    r.live_mask = live_workers(c, active, &r.use_mask);
    r.prox_kind = prox_kind; r.prox_a = prox_a;
    Timed t(c, 2);
    hipError_t e;
    if (r.bf16) {
        if (c->ws == nullptr || c->ws_bytes < workspace_need(c)) return SFB_EWORKSPACE;
        const Bf16TilePlan& tiles = c->tile_update[n_rows > 0];
        const size_t planes = tiles.slices > 1 ? (size_t)tiles.slices * (size_t)c->J * (size_t)c->D * sizeof(float) : 0;
        if (c->tile_bf16_update && update_bf16_ok(r) && tiles.bm > 0 && planes <= workspace_need(c) && tiles.us < reconstruct_bf16_us(c->J, c->D, r.N)) {
            r.partial = tiles.slices > 1 ? (float*)c->ws : nullptr;      // (the partial scores are dead)
            e = launch_update_bf16(r, tiles, c->stream);
        } else {
            e = launch_reconstruct_bf16(r, (char*)c->ws + scores_need(c), c->stream);
        }
        if (e != hipSuccess) return hip_fail(c, e);
        return SFB_OK;
    }
    bool on_split = false, on_lists = false, on_thin = false;
    const bool have_ws = c->ws != nullptr && c->ws_bytes >= workspace_need(c);
    const SplitReconPlan* sp = nullptr;
    const bool whole = reconstruct_takes_dma(r, c->recon);
    // (ragged calls included, down to the smallest: 37 x 203 with 15 pairs 5.2 us, 8.8 by a copy and a kernel)
    if (c->split_recon < 0) on_thin = reconstruct_thin_ok(r);
    if (c->split_recon != 0 && !on_thin) {
        // what the fp32 kernels would take, copies of ragged, misaligned or masked factors included
        // (a call that needs no copy in a context that keeps room for them has no planes for slices of the pairs: 100 x 192
        // with 2048 pairs walks them in six workgroups, 41 us)
        double us = c->padded_factors && have_ws && !whole
                        ? reconstruct_fp32_us(c->recon_padded, c->J, c->D, conform_rows(r.N), true)
                        : reconstruct_fp32_us(c->recon, c->J, c->D, r.N, have_ws && !c->padded_factors);
        if (!whole) us += 3.5 + 1.6e-6 * (double)r.N * (double)(c->J + c->D);
        if (reconstruct_split_ok(r)) {
            sp = &c->split_plans[n_rows > 0][have_ws];
            const size_t planes = sp->slices > 1 ? (size_t)sp->slices : sp->main_rows + sp->main_cols > 0 && sp->rest_slices > 1 ? (size_t)sp->rest_slices : 0;
            const size_t rows = (size_t)(c->J - sp->main_rows), cols = (size_t)(c->D - sp->main_cols);
            if (planes * rows * cols * sizeof(float) > workspace_need(c)) sp = &c->split_plans[n_rows > 0][0];
            on_split = c->split_recon == 1 || sp->us < us;
            if (on_split) us = sp->us;
        }
        on_lists = same_step && c->lists != nullptr && c->split_recon < 0 &&
                   sparse_update_us(r.N, c->J, c->D, c->lists_stored) < us;
    }
    if (c->lists_always && same_step && c->lists != nullptr) {
        on_lists = true;
        on_thin = false;
    }
    if (on_thin) {
        e = launch_reconstruct_thin(r, c->stream);
    } else if (on_lists) {
        e = launch_sparse_update(r, c->lists_stored, c->lists, c->stream);
    } else if (on_split) {
        r.partial = have_ws ? (float*)c->ws : nullptr;                   // (plans without a workspace have no slices)
        e = launch_reconstruct_split(r, *sp, c->stream);
    } else {
        // calls that would end in the register-staged kernel first try a copy of the factors that the LDS-DMA
        // kernels accept: padded ones for ragged shapes, U with a dead worker's rows zeroed for a masked call
        // (N x ceil4(J) floats: never more than the partial scores, whose bytes it takes)
        e = hipErrorNotSupported;
        const int64_t n_all = (int64_t)c->P * c->B;
        if (have_ws && !whole) {
            if (c->padded_factors && conformed_variant_ok(c->recon_padded.variant)) {
                if (c->recon_padded.n_split > 1) r.partial = (float*)((char*)c->ws + conform_workspace(c->J, c->D, n_all));
                e = launch_reconstruct_conformed(r, c->recon_padded, c->ws, c->stream);
                r.partial = nullptr;
            } else if (r.use_mask && masked_workspace(c->J, r.N) <= scores_need(c)) {
                if (!c->padded_factors && c->recon.n_split > 1) r.partial = (float*)((char*)c->ws + masked_workspace(c->J, n_all));
                e = launch_reconstruct_masked(r, c->recon, c->ws, c->stream);
                r.partial = nullptr;
            }
        }
        if (e == hipErrorNotSupported) {
            if (have_ws && !c->padded_factors && c->recon.n_split > 1)
                r.partial = (float*)((char*)c->ws + masked_workspace(c->J, n_all));
            e = launch_reconstruct(r, c->recon, c->stream);
        }
    }
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

}  // namespace

extern "C" {

sfb_status sfb_create(sfb_ctx** out, sfb_model m, int64_t J, int64_t D, int32_t P, int32_t B,
                      sfb_dtype input_dtype, void* hip_stream) {
    if (!out) return SFB_EINVAL;
    *out = nullptr;
    if (J <= 0 || D <= 0 || P <= 0 || B <= 0) return SFB_EINVAL;
    if (m != SFB_MLR && m != SFB_DML && m != SFB_L2SVM) return SFB_EINVAL;
    if (input_dtype != SFB_F32 && input_dtype != SFB_BF16) return SFB_EDTYPE;
    if (input_dtype == SFB_BF16 && m != SFB_MLR) return SFB_EUNSUPPORTED;
    // kernels index rows and columns with 32-bit ints
    if (J > (1 << 30) || D > (1 << 30) || (int64_t)P * B > (1 << 30)) return SFB_EUNSUPPORTED;
    sfb_ctx* c = new (std::nothrow) sfb_ctx();
    if (!c) return SFB_EINVAL;
    c->model = m; c->J = J; c->D = D; c->P = P; c->B = B; c->dtype = input_dtype;
    c->stream = (hipStream_t)hip_stream;
    c->fwd_all = plan_forward((int64_t)P * B, J, D);
    c->fwd_worker = plan_forward(B, J, D);
    c->fwd_bf16 = plan_forward_bf16((int64_t)P * B, J, D);
    // Small products are all latency: splitting operands into LDS takes longer to start than the fp32 instruction's copies.
    // 128 x 1152: 9.0 us (fp32) against 9.8 with 72 samples, 11.8 against 12.5 with 976; 320 x 2304, 384 samples: 14.0
    // against 14.7; even at 320 x 3072, 384, and 64 x 3072, 1800; 320 x 2304, 976: 22.4 against 21.9; longer rows (128 x
    // 5504, 72: 13.9 against 13.1) and rows that those copies do not take (D not in chunks of 32) are faster split.
    c->split_scores = input_dtype == SFB_F32 &&
                      !(m != SFB_DML && (D % 32) == 0 && D <= 3072 && (double)P * B * (double)J * (double)D < 3e8);
    c->split_recon = -1;
    c->recon = plan_reconstruct(J, D, (int64_t)P * B);
    {
        const int64_t N = (int64_t)P * B;
        c->padded_factors = input_dtype == SFB_F32 &&
                            !((J % 4) == 0 && J >= 4 && (D % 128) == 0 && (N % 32) == 0 && N >= 32);
        c->recon_padded = plan_reconstruct_padded(J, D, N, -1);
    }
    plan_split_scores(c, m == SFB_L2SVM, false);
    c->fused_ok = input_dtype == SFB_BF16 && m == SFB_MLR && fused_shape_ok(J, D, (int64_t)P * B);
    c->use_fused = true;
    c->fused = c->fused_ok ? plan_fused(J, D, (int64_t)P * B) : FusedPlan{};
    c->few = false;
    if (m != SFB_L2SVM && few_ok((int64_t)P * B, J, D, m == SFB_DML)) {
        // (contexts that sfb_step_noalloc could hold stay that way)
        const size_t planes = few_workspace((int64_t)P * B, J, D);
        c->few = planes <= SFB_NOALLOC_SCRATCH_BYTES || planes <= workspace_need(c);
    }
    plan_split_recon(c, m == SFB_L2SVM, false);
    c->tile_bf16_scores = c->tile_bf16_update = true;
    plan_bf16_tiles(c);
    c->ws = nullptr; c->ws_bytes = 0; c->lists = nullptr; c->lists_stored = 0; c->last_hip = 0; c->timing = false; c->sparse_forward = true; c->sparse_always = false;
    c->lists_always = false;
    for (LastKernel& k : c->last) k = LastKernel{nullptr, 0};
    // Set-up for sfb_step_noalloc on the device that is current now: resolve the address of the
    // library's scratch array, so that the entry point itself only reads it.  On a machine without a
    // GPU this fails; the context is still good for everything that can be checked on the host, and
    // the entry point tries again (and reports SFB_EHIP if it still cannot).
    {
        void* unused = nullptr;
        if (resolve_static_scratch(&unused) != hipSuccess) (void)hipGetLastError();
    }
    *out = c;
    return SFB_OK;
}

void sfb_destroy(sfb_ctx* c) {
    if (!c) return;
    for (int f = 0; f < kFamilies; ++f)
        for (auto& e : c->used[f]) { (void)hipEventDestroy(e.a); (void)hipEventDestroy(e.b); }
    for (auto& e : c->spare) { (void)hipEventDestroy(e.a); (void)hipEventDestroy(e.b); }
    delete c;
}

sfb_status sfb_workspace_bytes(const sfb_ctx* c, size_t* bytes) {
    if (!c || !bytes) return SFB_EINVAL;
    *bytes = workspace_need(c);
    return SFB_OK;
}

sfb_status sfb_set_workspace(sfb_ctx* c, void* dev, size_t bytes) {
    if (!c || !dev) return SFB_EINVAL;
    if (((uintptr_t)dev % 256) != 0) return SFB_EINVAL;
    if (bytes < workspace_need(c)) return SFB_EWORKSPACE;
    c->ws = dev; c->ws_bytes = bytes;
    return SFB_OK;
}

sfb_status sfb_compute_factors(sfb_ctx* c, const float* W, int64_t ldw, const sfb_batch* batch,
                               const int32_t* y, float* U, int64_t ldu, void* V, int64_t ldv, float* loss) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch, y);
    if (s != SFB_OK) return s;
    return factors_rows(c, c->fwd_all, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss);
}

sfb_status sfb_compute_factors_worker(sfb_ctx* c, const float* W, int64_t ldw, const sfb_batch* batch_p,
                                      const int32_t* y_p, int32_t p, float* U, int64_t ldu, void* V,
                                      int64_t ldv, float* loss) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch_p, y_p);
    if (s != SFB_OK) return s;
    if (p < 0 || p >= c->P) return SFB_ESHAPE;
    return factors_rows(c, c->fwd_worker, W, ldw, batch_p, y_p, (int64_t)p * c->B, c->B, U, ldu, V, ldv, loss);
}

sfb_status sfb_reconstruct_apply(sfb_ctx* c, float* W, int64_t ldw, const float* U, int64_t ldu,
                                 const void* V, int64_t ldv, float eta, float scale, const uint8_t* active) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    return recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active);
}

sfb_status sfb_reconstruct_apply_worker(sfb_ctx* c, float* W, int64_t ldw, const float* U, int64_t ldu,
                                        const void* V, int64_t ldv, int32_t p, float eta, float scale) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_recon(c, eta, scale, nullptr);
    if (s != SFB_OK) return s;
    if (p < 0 || p >= c->P) return SFB_ESHAPE;
    const size_t vsz = c->dtype == SFB_BF16 ? 2 : 4;
    return recon_launch(c, W, ldw, U + (int64_t)p * c->B * ldu, ldu,
                        (const char*)V + (size_t)p * c->B * (size_t)ldv * vsz, ldv, eta, scale, nullptr, c->B);
}

sfb_status sfb_step(sfb_ctx* c, float* W, int64_t ldw, const sfb_batch* batch, const int32_t* y, float* U,
                    int64_t ldu, void* V, int64_t ldv, float* loss, float eta, const uint8_t* active) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch, y);
    if (s != SFB_OK) return s;
    float scale;                              // mini-batch mean inside a worker (Section 3)
    (void)sfb_default_scale(c, &scale);
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    if (c->few) return few_rows(c, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss, true, -eta * scale, active);
    s = factors_rows(c, c->fwd_all, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss);
    if (s != SFB_OK) return s;
    return recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active, 0, 0, 0.f, true);
}

sfb_status sfb_step_pipelined(sfb_ctx* c, float* W, int64_t ldw, float* U, int64_t ldu, void* V, int64_t ldv,
                              const sfb_batch* next_batch, const int32_t* next_y, float* loss, float eta,
                              const uint8_t* active) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, next_batch, next_y);
    if (s != SFB_OK) return s;
    float scale;
    (void)sfb_default_scale(c, &scale);
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    if (c->ws == nullptr || c->ws_bytes < workspace_need(c)) return SFB_EWORKSPACE;
    const int N = c->P * c->B;
    if (c->fused_ok && c->use_fused) {
        FusedArgs f{};
        f.w = W; f.ldw = ldw; f.u = U; f.ldu = ldu; f.v = V; f.ldv = ldv;
        f.a_next = next_batch->a; f.lda = next_batch->lda;
        f.zp = (float*)c->ws; f.ldz = round_up4(c->J); f.zstride = (int64_t)N * f.ldz;
        f.J = (int)c->J; f.D = (int)c->D; f.N = N; f.B = c->B;
        f.alpha = -eta * scale;
        f.live_mask = live_workers(c, active, &f.use_mask);
        if (fused_call_ok(f)) {
            char* ws_factors = (char*)c->ws + scores_need(c);
            char* ws_next = ws_factors + bf16_recon_workspace(c->J, c->D, N);
            {
                Timed t(c, 5);
                hipError_t e = launch_fused(f, c->fused, ws_factors, ws_next, c->stream);
                if (e != hipSuccess) return hip_fail(c, e);
            }
            return factor_rows(c, c->fused.slices, f.zstride, next_y, 0, N, U, ldu, loss, nullptr);
        }
    }
    // the same two steps as separate passes over W
    s = recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active);
    if (s != SFB_OK) return s;
    return factors_rows(c, c->fwd_all, W, ldw, next_batch, next_y, 0, N, U, ldu, V, ldv, loss);
}

sfb_status sfb_pipeline_info(const sfb_ctx* c, int32_t* fused, int32_t* grid, int32_t* slices) {
    if (!c) return SFB_EINVAL;
    const bool on = c->fused_ok && c->use_fused;
    if (fused) *fused = on ? 1 : 0;
    if (grid) *grid = on ? c->fused.grid : 0;
    if (slices) *slices = on ? c->fused.slices : 0;
    return SFB_OK;
}

sfb_status sfb_step_noalloc(sfb_ctx* c, float* W, int64_t ldw, const sfb_batch* batch, const int32_t* y, float* U,
                            int64_t ldu, void* V, int64_t ldv, float* loss, float eta, const uint8_t* active) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch, y);
    if (s != SFB_OK) return s;
    float scale;
    (void)sfb_default_scale(c, &scale);
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    if (workspace_need(c) > kStaticScratchBytes) return SFB_ESCRATCH;
    void* ptr = nullptr;
    hipError_t e = resolve_static_scratch(&ptr);     // a table read after sfb_create on this device
    if (e != hipSuccess) return hip_fail(c, e);
    // the kernels take the scratch address where they take the registered workspace in sfb_step
    void* const ws = c->ws;
    const size_t ws_bytes = c->ws_bytes;
    c->ws = ptr; c->ws_bytes = kStaticScratchBytes;
    if (c->few) s = few_rows(c, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss, true, -eta * scale, active);
    else s = factors_rows(c, c->fwd_all, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss);
    if (s == SFB_OK && !c->few) s = recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active, 0, 0, 0.f, true);
    c->ws = ws; c->ws_bytes = ws_bytes;
    return s;
}

sfb_status sfb_sdca_compute_factors(sfb_ctx* c, const float* W, int64_t ldw, const sfb_batch* batch,
                                    const int32_t* y, const sfb_sdca* sdca, float* U, int64_t ldu, void* V,
                                    int64_t ldv, float* loss) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch, y);
    if (s != SFB_OK) return s;
    s = check_sdca(c, sdca);
    if (s != SFB_OK) return s;
    return factors_rows(c, c->fwd_all, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss, sdca);
}

sfb_status sfb_sdca_step(sfb_ctx* c, float* W, int64_t ldw, const sfb_batch* batch, const int32_t* y,
                         const sfb_sdca* sdca, float* U, int64_t ldu, void* V, int64_t ldv, float* loss) {
    if (!c || !sdca) return SFB_EINVAL;
    // Z <- Z - (1/n_data) sum delta u a^T and W = Z / lam, folded into one scale (Section 2.1)
    const float scale = (float)(1.0 / ((double)sdca->lam * (double)sdca->n_data));
    if (!std::isfinite(scale)) return SFB_EINVAL;
    sfb_status s = sfb_sdca_compute_factors(c, W, ldw, batch, y, sdca, U, ldu, V, ldv, loss);
    if (s != SFB_OK) return s;
    return recon_launch(c, W, ldw, U, ldu, V, ldv, 1.0f, scale, nullptr);
}

// kind and parameters of a proximal step; the workspace only matters for the column projection
static sfb_status check_prox(const sfb_ctx* c, sfb_prox_kind kind, float eta, float param, bool need_workspace) {
    if ((int)kind < SFB_PROX_NONE || (int)kind > SFB_PROX_COLUMN_BALL) return SFB_EINVAL;
    if (!std::isfinite(eta) || !std::isfinite(param) || eta < 0.f || param < 0.f) return SFB_EINVAL;
    if (kind == SFB_PROX_COLUMN_BALL && !(param > 0.f)) return SFB_EINVAL;
    if (need_workspace && kind == SFB_PROX_COLUMN_BALL && (c->ws == nullptr || c->ws_bytes < workspace_need(c)))
        return SFB_EWORKSPACE;
    return SFB_OK;
}

sfb_status sfb_prox(sfb_ctx* c, float* W, int64_t ldw, sfb_prox_kind kind, float eta, float param) {
    if (!c || !W) return SFB_EINVAL;
    sfb_status s = check_prox(c, kind, eta, param, false);
    if (s != SFB_OK) return s;
    if (ldw < c->D) return SFB_ESHAPE;
    if (kind == SFB_PROX_NONE) return SFB_OK;
    s = check_prox(c, kind, eta, param, true);
    if (s != SFB_OK) return s;
    ProxArgs a{W, ldw, (int)c->J, (int)c->D, (int)kind, eta, param};
    Timed t(c, 4);
    hipError_t e = launch_prox(a, c->ws, c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

// The proximal step after an update: the entrywise kinds ride in the reconstruction's epilogue
// (no extra pass over W), the column projection runs as its own kernels afterwards.
static sfb_status recon_then_prox(sfb_ctx* c, float* W, int64_t ldw, const float* U, int64_t ldu, const void* V,
                                  int64_t ldv, float eta, float scale, const uint8_t* active, sfb_prox_kind kind,
                                  float param, bool same_step) {
    if (kind == SFB_PROX_L2SQ)
        return recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active, 0, 1, 1.0f / (1.0f + eta * param), same_step);
    if (kind == SFB_PROX_L1) return recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active, 0, 2, eta * param, same_step);
    sfb_status s = recon_launch(c, W, ldw, U, ldu, V, ldv, eta, scale, active, 0, 0, 0.f, same_step);
    if (s != SFB_OK || kind == SFB_PROX_NONE) return s;
    return sfb_prox(c, W, ldw, kind, eta, param);
}

sfb_status sfb_reconstruct_apply_prox(sfb_ctx* c, float* W, int64_t ldw, const float* U, int64_t ldu, const void* V,
                                      int64_t ldv, float eta, float scale, const uint8_t* active,
                                      sfb_prox_kind kind, float param) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    s = check_prox(c, kind, eta, param, true);
    if (s != SFB_OK) return s;
    return recon_then_prox(c, W, ldw, U, ldu, V, ldv, eta, scale, active, kind, param, false);
}

sfb_status sfb_step_prox(sfb_ctx* c, float* W, int64_t ldw, const sfb_batch* batch, const int32_t* y, float* U,
                         int64_t ldu, void* V, int64_t ldv, float* loss, float eta, const uint8_t* active,
                         sfb_prox_kind kind, float param) {
    sfb_status s = check_common(c, W, ldw, U, ldu, V, ldv);
    if (s != SFB_OK) return s;
    s = check_batch(c, batch, y);
    if (s != SFB_OK) return s;
    float scale;
    (void)sfb_default_scale(c, &scale);
    s = check_recon(c, eta, scale, active);
    if (s != SFB_OK) return s;
    s = check_prox(c, kind, eta, param, true);
    if (s != SFB_OK) return s;
    if (c->few) {
        const int entry = kind == SFB_PROX_L2SQ ? 1 : kind == SFB_PROX_L1 ? 2 : 0;      // entrywise kinds ride along
        s = few_rows(c, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss, true, -eta * scale, active, entry,
                     entry == 1 ? 1.0f / (1.0f + eta * param) : eta * param);
        if (s != SFB_OK || kind != SFB_PROX_COLUMN_BALL) return s;
        return sfb_prox(c, W, ldw, kind, eta, param);
    }
    s = factors_rows(c, c->fwd_all, W, ldw, batch, y, 0, c->P * c->B, U, ldu, V, ldv, loss);
    if (s != SFB_OK) return s;
    return recon_then_prox(c, W, ldw, U, ldu, V, ldv, eta, scale, active, kind, param, true);
}

sfb_status sfb_shape(const sfb_ctx* c, int64_t* J, int64_t* D, int32_t* P, int32_t* B, int32_t* input_dtype) {
    if (!c) return SFB_EINVAL;
    if (J) *J = c->J;
    if (D) *D = c->D;
    if (P) *P = c->P;
    if (B) *B = c->B;
    if (input_dtype) *input_dtype = (int32_t)c->dtype;
    return SFB_OK;
}

sfb_status sfb_default_scale(const sfb_ctx* c, float* scale) {
    if (!c || !scale) return SFB_EINVAL;
    *scale = 1.0f / (float)c->B;
    return SFB_OK;
}

sfb_status sfb_sync(sfb_ctx* c) {
    if (!c) return SFB_EINVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

const char* sfb_strerror(sfb_status s) {
    switch (s) {
        case SFB_OK: return "ok";
        case SFB_EINVAL: return "invalid argument (null pointer, non-positive size, non-finite eta or scale)";
        case SFB_ESHAPE: return "shape mismatch (leading dimension shorter than the row, negative nnz, worker index out of range)";
        case SFB_EDTYPE: return "unknown dtype";
        case SFB_EWORKSPACE: return "workspace missing or too small";
        case SFB_EUNSUPPORTED: return "unsupported model/dtype combination or size";
        case SFB_EHIP: return "HIP runtime error";
        case SFB_ESCRATCH: return "the context needs more scratch than the library's fixed array holds (use sfb_step with a registered workspace)";
    }
    return "unknown status";
}

int sfb_last_hip_error(const sfb_ctx* c) { return c ? c->last_hip : 0; }

sfb_status sfb_plan_info(const sfb_ctx* c, int32_t* fwd_split_k, int32_t* fwd_grid, int32_t* recon_grid) {
    if (!c) return SFB_EINVAL;
    const FwdPlan& f = c->dtype == SFB_BF16 ? c->fwd_bf16 : c->split_scores && c->D >= 4 ? c->fwd_split : c->fwd_all;
    if (fwd_split_k) *fwd_split_k = f.split_k;
    if (fwd_grid) *fwd_grid = f.grid;
    bool tile_update = false;
    if (c->dtype == SFB_BF16) {                                  // as the calls on aligned operands choose (factors_rows, recon_launch)
        const int64_t N = (int64_t)c->P * c->B;
        const bool rounded = N >= 128 && c->D % 32 == 0;
        const Bf16TilePlan& t = c->tile_scores[0][!rounded];
        if (c->tile_bf16_scores && t.bm > 0 && !(rounded && forward_bf16_wins(c->fwd_bf16, N, c->J, c->D, t.us))) {
            if (fwd_split_k) *fwd_split_k = t.slices;
            if (fwd_grid) *fwd_grid = (int32_t)(((N + t.bm - 1) / t.bm) * ((c->J + t.bn - 1) / t.bn) * t.slices);
        }
        const Bf16TilePlan& u = c->tile_update[0];
        tile_update = c->tile_bf16_update && u.bm > 0 && u.us < reconstruct_bf16_us(c->J, c->D, N);
        if (recon_grid && tile_update)
            *recon_grid = (int32_t)(((c->J + u.bm - 1) / u.bm) * ((c->D + u.bn - 1) / u.bn) * u.slices);
    }
    if (recon_grid && !tile_update) {
        // ragged fp32 shapes run the padded shape's plan once a workspace is registered (recon_launch)
        const bool padded = c->padded_factors && conformed_variant_ok(c->recon_padded.variant) && c->ws != nullptr &&
                            c->ws_bytes >= workspace_need(c);
        *recon_grid = c->dtype == SFB_BF16 ? (int32_t)bf16_recon_grid(c->J, c->D) : padded ? c->recon_padded.grid : c->recon.grid;
    }
    return SFB_OK;
}

sfb_status sfb_last_kernel(const sfb_ctx* c, int32_t which, char* name, size_t bytes, int32_t* grid) {
    if (!c || which < 0 || which >= kFamilies || (name && bytes == 0)) return SFB_EINVAL;
    if (name) {                                                  // as it stands at the launch, up to its template arguments
        const char* k = c->last[which].name ? c->last[which].name : "";
        if (*k == '(') ++k;
        size_t n = 0;
        while (n + 1 < bytes && k[n] != '\0' && k[n] != '<') ++n;
        for (size_t i = 0; i < n; ++i) name[i] = k[i];
        name[n] = '\0';
    }
    if (grid) *grid = (int32_t)c->last[which].grid;
    return SFB_OK;
}

sfb_status sfb_set_plan(sfb_ctx* c, int32_t fwd_bm, int32_t fwd_bn, int32_t fwd_split_k, int32_t recon_variant,
                        int32_t fwd_dma) {
    if (!c) return SFB_EINVAL;
    if ((fwd_bm > 0 && fwd_bm != 64 && fwd_bm != 128) || (fwd_bn > 0 && fwd_bn != 64 && fwd_bn != 128))
        return SFB_EINVAL;
    if (recon_variant >= num_reconstruct_variants() || fwd_split_k > 64) return SFB_EINVAL;
    if (fwd_bm <= 0 && fwd_bn <= 0 && fwd_split_k <= 0 && recon_variant < 0 && fwd_dma < 0) return SFB_OK;   // keep everything
    c->few = false;                                              // a plan of the caller's is about the separate kernels
    FwdPlan p = c->fwd_all;
    if (fwd_bm > 0) p.bm = fwd_bm;
    if (fwd_bn > 0) p.bn = fwd_bn;
    if (fwd_split_k > 0) p.split_k = fwd_split_k;
    if (fwd_dma >= 0) p.dma = (fwd_dma & 1) != 0;
    if (fwd_dma >= 0) c->sparse_forward = (fwd_dma & 2) == 0;   // bit 1 set: dense scores for CSR input
    if (fwd_dma >= 0) c->sparse_always = (fwd_dma & 32) != 0;   // bit 5 set: from the entries whenever the kernel can take them
    // bit 2 set: fp32 scores as split-bf16 products; a tile or slice count of its own means the fp32 instruction's kernels
    if (fwd_dma >= 0) c->split_scores = (fwd_dma & 4) != 0 && c->dtype == SFB_F32;
    else if (fwd_bm > 0 || fwd_bn > 0 || fwd_split_k > 0) c->split_scores = false;
    if (fwd_dma >= 0) c->split_recon = (fwd_dma & 8) != 0;      // bit 3 set: the reconstruction likewise
    else if (recon_variant >= 0) c->split_recon = 0;
    if (fwd_dma >= 0) c->lists_always = (fwd_dma & 64) != 0;    // bit 6 set: L2SVM steps update from the column lists wherever they fit
    if (fwd_dma >= 0) c->use_fused = (fwd_dma & 16) == 0;       // bit 4 set: sfb_step_pipelined runs two separate passes
    finish_forward_plan(&p, (int64_t)c->P * c->B, c->J, c->D);
    if (fwd_dma >= 0 && c->split_scores) plan_split_scores(c, true, true);
    c->fwd_all = p;
    if (fwd_bm > 0 || fwd_bn > 0 || fwd_split_k > 0) c->tile_bf16_scores = false;
    if (recon_variant >= 0) {
        c->tile_bf16_update = false;
        c->recon = plan_reconstruct_variant(c->J, c->D, recon_variant);
        c->recon_padded = plan_reconstruct_padded(c->J, c->D, (int64_t)c->P * c->B, recon_variant);
    }
    if (fwd_dma >= 0 && c->split_recon == 1) plan_split_recon(c, true, true);
    plan_bf16_tiles(c);                                          // (the choice may have changed the workspace, either way)
    return SFB_OK;
}

sfb_status sfb_stream_copy(sfb_ctx* c, void* dst, const void* src, size_t bytes) {
    if (!c || !dst || !src) return SFB_EINVAL;
    if (((uintptr_t)dst % 16) != 0 || ((uintptr_t)src % 16) != 0 || (bytes % 16) != 0) return SFB_EINVAL;
    if (bytes == 0) return SFB_OK;
    Timed t(c, 3);
    hipError_t e = launch_stream_copy(src, dst, (int64_t)bytes, c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

sfb_status sfb_probe(sfb_ctx* c, sfb_probe_kind kind, float* W, int64_t ldw, int32_t param) {
    if (!c) return SFB_EINVAL;
    if (c->ws == nullptr || c->ws_bytes < 256) return SFB_EWORKSPACE;      // 64 floats of sink
    hipError_t e;
    switch (kind) {
        case SFB_PROBE_W_STREAM: {
            if (!W || (param != 1 && param != 2)) return SFB_EINVAL;
            if (ldw < c->D) return SFB_ESHAPE;
            if (((uintptr_t)W % 16) != 0 || (ldw % 4) != 0 || (c->D % 32) != 0) return SFB_EUNSUPPORTED;
            Timed t(c, 3);
            e = launch_probe_w_stream(W, ldw, (int)c->J, (int)c->D, c->fwd_bf16.k_slice, param, (float*)c->ws, c->stream);
            break;
        }
        case SFB_PROBE_W_RMW: {
            if (!W) return SFB_EINVAL;
            if (ldw < c->D) return SFB_ESHAPE;
            Timed t(c, 3);
            e = launch_probe_w_rmw(W, ldw, (int)c->J, (int)c->D, 0.0f, c->stream);
            break;
        }
        case SFB_PROBE_MFMA_F32:
        case SFB_PROBE_MFMA_BF16: {
            if (param != 1 && param != 2) return SFB_EINVAL;
            Timed t(c, 3);
            e = launch_probe_mfma(kind == SFB_PROBE_MFMA_BF16, param, SFB_PROBE_MFMA_ITERS, (float*)c->ws, c->stream);
            break;
        }
        case SFB_PROBE_EMPTY: {
            Timed t(c, 3);
            e = launch_probe_empty(c->stream);
            break;
        }
        case SFB_PROBE_FUSED_TRAFFIC: {
            if (!W) return SFB_EINVAL;
            if (ldw < c->D) return SFB_ESHAPE;
            // the shapes and operands the one-pass kernel takes, and its packed-operand areas of the workspace
            const int N = c->P * c->B;
            if (!c->fused_ok || (int64_t)c->J * ldw >= (1LL << 31) || ((uintptr_t)W % 16) != 0 || (ldw % 4) != 0)
                return SFB_EUNSUPPORTED;
            if (c->ws_bytes < workspace_need(c)) return SFB_EWORKSPACE;
            char* ws_factors = (char*)c->ws + scores_need(c);
            char* ws_next = ws_factors + bf16_recon_workspace(c->J, c->D, N);
            Timed t(c, 3);
            e = launch_probe_fused_traffic(W, ldw, (int)c->J, (int)c->D, N, c->fused, ws_factors, ws_next, c->stream);
            break;
        }
        default: return SFB_EINVAL;
    }
    if (e != hipSuccess) return hip_fail(c, e);
    return SFB_OK;
}

sfb_status sfb_enable_timing(sfb_ctx* c, int enable) {
    if (!c) return SFB_EINVAL;
    c->timing = enable != 0;
    return SFB_OK;
}

sfb_status sfb_kernel_time_ms(sfb_ctx* c, int which, double* ms, int64_t* launches) {
    if (!c || which < 0 || which >= kFamilies || !ms) return SFB_EINVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    double total = 0.0;
    for (auto& p : c->used[which]) {
        float t = 0.f;
        e = hipEventElapsedTime(&t, p.a, p.b);
        if (e != hipSuccess) return hip_fail(c, e);
        total += t;
    }
    *ms = total;
    if (launches) *launches = (int64_t)c->used[which].size();
    return SFB_OK;
}

sfb_status sfb_reset_timing(sfb_ctx* c) {
    if (!c) return SFB_EINVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(c, e);
    for (int f = 0; f < kFamilies; ++f) {
        for (auto& p : c->used[f]) c->spare.push_back(p);
        c->used[f].clear();
    }
    return SFB_OK;
}

}  // extern "C"
