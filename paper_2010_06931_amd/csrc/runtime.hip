// Host runtime behind the C ABI (include/octmc.h): contexts, pair ingest and
// pyramid, the evaluation sequence of the hot path, the L-BFGS level loop and
// the merge.  All vectors stay in device memory; only float64 scalars cross
// to the host (objective and directional derivative per line-search trial,
// one set of dot products per L-BFGS iteration).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <deque>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "octmc_internal.h"

using namespace octmc;

namespace {
thread_local std::string g_err;
}  // namespace

int octmc::fail(int code, const std::string& msg)
{
    g_err = msg;
    return code;
}

namespace {

size_t esize(octmc_dtype dt) { return dt == OCTMC_F32 ? 4 : 2; }

// ---------------------------------------------------------------------------
// Scratch of octmc_eval_noalloc: one file-scope device array (each GPU the
// library runs on holds its own copy until the process ends), laid out as the
// per-A-scan partials [na][8] float32, the displacement-sum block rows
// [256][4] float64 and the combination block rows [nblk][8] float64, for at
// most kNoAllocMaxAscans A-scans.  Host code never uses the array's name as
// an address: octmc_create resolves the device address once per device
// (hipGetSymbolAddress, with that device current) and every launch takes it.
// Every kernel writes the whole part of the array it later reads, so nothing
// has to start at zero.
constexpr size_t kNoAllocPart = (size_t)OCTMC_NOALLOC_MAX_ASCANS * 8 * 4;
constexpr size_t kNoAllocSum = 256 * 4 * 8;
constexpr size_t kNoAllocComb = ((size_t)OCTMC_NOALLOC_MAX_ASCANS + 255) / 256 * 8 * 8;
constexpr size_t kNoAllocBytes = kNoAllocPart + kNoAllocSum + kNoAllocComb;
static_assert(kNoAllocPart % 256 == 0 && kNoAllocSum % 256 == 0, "sub-buffers stay 256-byte aligned");
static_assert(kNoAllocBytes == OCTMC_NOALLOC_SCRATCH_BYTES, "the size the header states");

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

// The device address of `scratch` on the current device `device`, resolved
// on the first call for that device.
int scratch_address(int device, void** out)
{
    if (device < 0 || device >= kMaxDevices) return fail(OCTMC_E_INVALID, "device ordinal out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(OCTMC_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_addr[device] = p;
    }
    *out = g_scratch_addr[device];
    return OCTMC_OK;
}

}  // namespace

#include "runtime_types.h"

namespace {

constexpr int kSumBlocks = 256;
// The count of finished combination blocks lies in the last row of the
// displacement-sum partials, which few A-scans do not use; the structural launch
// of each evaluation clears it.
constexpr size_t kTicketAt = kSumBlocks * 4 - 1;
// The rows of few A-scans are more than of many; they lie where the dot products'
// rows do (an evaluation and a pass of dot products follow each other).
static_assert(512 * (kMaxDots + 1) >= kFewMaxAscans / kFewAscans * 8, "they fit there");
static_assert((size_t)kFewMaxAscans / kFewAscans * 64 <= kNoAllocComb, "and in the static scratch");

int nblk_combine(int na) { return (na + kRedBlock - 1) / kRedBlock; }

// ---------------------------------------------------------------------------
// hot path: one grouped evaluation over up to kMaxJobs pairs at one level

}  // namespace

int octmc::eval_group(const EvalArgs* ea, int n, hipStream_t s, hipEvent_t* ev, bool with_struct)
{
    SumJobs sj{};
    StructJobs tj{};
    CombineJobs cj{};
    tj.n = cj.n = n;
    // one skip flag for the grouped launch (a solver enqueued ahead of its decisions)
    sj.skip = tj.skip = cj.skip = ea[0].skip;
    for (int q = 1; q < n; ++q)
        if (ea[q].skip != ea[0].skip) return fail(OCTMC_E_INVALID, "grouped evaluations must share their skip flag");
    int sb = 0;
    bool axial = true;
    for (int q = 0; q < n; ++q) axial &= ea[q].axial;
    const bool fold = with_struct && !axial && !ev;
    EvalView views[kMaxJobs];
    for (int q = 0; q < n; ++q) {
        if (ea[q].view) {
            views[q] = *ea[q].view;
        } else {
            octmc_pair* P = ea[q].pair;
            EvalView& v = views[q];
            v.L = P->lev[ea[q].level];
            v.dtype = P->dtype;
            v.params = &P->params;
            v.part = P->part;
            v.sum_blk = P->sum_blk;
            v.comb_blk = few_ascans(v.L.na) ? P->dot_blk : P->comb_blk;
            v.ticket = P->ticket;
            v.eta = P->eta + ea[q].level;
            v.orient = P->orient;
        }
    }
    const octmc_dtype dt = views[0].dtype;
    bool any_eta = false;
    for (int q = 0; q < n; ++q) {
        const EvalView& V = views[q];
        const Level& L = V.L;
        any_eta |= ea[q].eta_mode == 0;
        const octmc_params& pr = *V.params;
        if (V.dtype != dt) return fail(OCTMC_E_DTYPE, "batched pairs must share the storage type");
        const int nsum = few_ascans(L.na) ? 0 : std::min(kSumBlocks, (2 * L.na + kRedBlock - 1) / kRedBlock);
        const float* dy = ea[q].disp_y ? ea[q].disp_y : ea[q].disp + (size_t)L.na * 3;
        if (with_struct && dy != ea[q].disp + (size_t)L.na * 3)
            return fail(OCTMC_E_INVALID, "the structural kernels read both slots' fields as one [2][na][3] array");
        // the sums go with the structural launch where that can take them (not between
        // the events that time the two apart)
        if (nsum && !fold) sj.j[sj.n++] = SumJob{{ea[q].disp, dy}, V.sum_blk, L.na, sb, nsum};
        sb += nsum;
        tj.j[q] = StructJob{L.sx, L.sy, ea[q].disp, V.part, L.w, L.h, L.d, L.na, 0, L.vol_bytes,
                            (float)pr.eps_huber, L.dp, V.sum_blk, fold ? nsum : 0, 0,
                            few_ascans(L.na) ? V.ticket : nullptr};
        const int blen = L.w;  // square scans: every B-scan has w A-scans
        const double f = std::floor(pr.flyback_frac * blen + 0.5);
        CombineJob c{};
        c.part = V.part;
        c.disp[0] = ea[q].disp;
        c.disp[1] = dy;
        c.grad = ea[q].grad;
        c.grad64 = ea[q].grad64;
        c.ax = L.ax;
        c.ay = L.ay;
        c.vx = L.vx;
        c.vy = L.vy;
        c.sum_blk = V.sum_blk;
        c.nsum = nsum;
        c.eta = V.eta;
        c.p = ea[q].p;
        c.blk = V.comb_blk;
        c.ticket = V.ticket;
        c.terms = ea[q].terms;
        c.w = L.w;
        c.h = L.h;
        c.d = L.d;
        c.na = L.na;
        c.mode = 1;
        c.orient = V.orient;
        c.delta0 = pr.delta0;
        c.eps_h = pr.eps_huber;
        c.eps_r = pr.eps_reg;
        constexpr double most = std::numeric_limits<double>::max();
        c.ieps_h = std::min(1.0 / pr.eps_huber, most);
        c.ieps_r = std::min(1.0 / pr.eps_reg, most);
        c.alpha = pr.alpha;
        c.gamma = pr.mean_weight;
        c.wfb = 1.0 / std::sqrt(1.0 + f);
        cj.j[q] = c;
    }
    if (ev) HIP_TRY(hipEventRecord(ev[0], s));
    if (sj.n) HIP_TRY(launch_sum(sj, sb, s));
    if (ev) HIP_TRY(hipEventRecord(ev[1], s));
    if (with_struct) HIP_TRY(launch_struct(tj, dt, s, axial));
    if (ev) HIP_TRY(hipEventRecord(ev[2], s));
    if (any_eta) {  // eta of the jobs that ask for it, before their evaluation
        CombineJobs c0{};
        c0.skip = cj.skip;
        for (int q = 0; q < n; ++q) {
            if (ea[q].eta_mode != 0) continue;
            CombineJob c = cj.j[q];
            c.mode = 0;
            c.grad = nullptr;
            c.grad64 = nullptr;
            c.p = nullptr;
            c0.j[c0.n++] = c;
        }
        HIP_TRY(launch_combine(c0, s));
    }
    HIP_TRY(launch_combine(cj, s));
    if (ev) HIP_TRY(hipEventRecord(ev[3], s));
    return OCTMC_OK;
}

namespace {

int check_level(const octmc_pair* P, int level)
{
    if (!P) return fail(OCTMC_E_INVALID, "pair is NULL");
    if (level < 0 || level >= P->nlev) return fail(OCTMC_E_INVALID, "level out of range");
    return OCTMC_OK;
}

}  // namespace

namespace {

bool finite_param(double v) { return std::isfinite(v); }


}  // namespace

// Evaluation scratch of a pair whose finest level has na A-scans; eta = 1
// at every level.
int octmc::pair_alloc_scratch(octmc_pair* P, size_t na, hipStream_t s)
{
    HIP_TRY(P->alloc(&P->part, na * 8 * 4));
    HIP_TRY(P->alloc(&P->sum_blk, kSumBlocks * 4 * 8));
    P->ticket = reinterpret_cast<unsigned*>(P->sum_blk + kTicketAt);
    HIP_TRY(P->alloc(&P->comb_blk, (size_t)nblk_combine((int)na) * 8 * 8));
    HIP_TRY(P->alloc(&P->eta, OCTMC_MAX_LEVELS * 8));
    HIP_TRY(P->alloc(&P->terms, OCTMC_NTERMS * 8));
    HIP_TRY(P->alloc(&P->dot_blk, (size_t)512 * (kMaxDots + 1) * 8));
    HIP_TRY(P->alloc(&P->dot_out, (kMaxDots + 1) * 8));
    HIP_TRY(P->alloc(&P->lb, sizeof(LbState)));
    static const std::vector<double> ones(OCTMC_MAX_LEVELS, 1.0);
    HIP_TRY(hipMemcpyAsync(P->eta, ones.data(), OCTMC_MAX_LEVELS * 8, hipMemcpyHostToDevice, s));
    return OCTMC_OK;
}

octmc_dtype octmc::pair_dtype(const octmc_pair* pair) { return pair->dtype; }
int octmc::pair_level_ascans(const octmc_pair* pair, int level) { return pair->lev[level].na; }
int octmc::pair_nlev(const octmc_pair* pair) { return pair->nlev; }
const octmc_params& octmc::pair_params(const octmc_pair* pair) { return pair->params; }
int octmc::pair_device(const octmc_pair* pair) { return pair->ctx->device; }
const std::vector<double>& octmc::pair_theta(const octmc_pair* pair) { return pair->theta; }

int octmc::ctx_device(const octmc_ctx* ctx) { return ctx->device; }
void octmc::ctx_trim(octmc_ctx* ctx) { ctx->cache->trim(); }

octmc_params octmc::resolve_levels(const octmc_params& p, const octmc_shape& shape)
{
    octmc_params r = p;
    if (p.levels != 0) return r;
    int wl = shape.w, dl = shape.d, L = 1;
    while (L < OCTMC_MAX_LEVELS && wl > kAutoCoarsest) {
        const int nw = (wl + 1) / 2, nd = (dl + 1) / 2;
        if (nw < 4 || nd < 4) break;
        wl = nw;
        dl = nd;
        ++L;
    }
    r.levels = L;
    return r;
}

int octmc::validate_params(const octmc_params* p)
{
    if (!p) return fail(OCTMC_E_INVALID, "params is NULL");
    const double vals[] = {p->alpha, p->delta0,  p->eps_huber,   p->eps_reg,  p->flyback_frac, p->mean_weight,
                           p->c1,    p->c2,      p->merge_kappa, p->merge_tau, p->gamma_tilt};
    for (double v : vals)
        if (!finite_param(v)) return fail(OCTMC_E_INVALID, "parameters must be finite");
    if (p->alpha < 0) return fail(OCTMC_E_INVALID, "alpha must be >= 0");
    if (p->delta0 < 0 || p->delta0 > 1) return fail(OCTMC_E_INVALID, "delta0 must lie in [0, 1]");
    if (!(p->eps_huber > 0) || !(p->eps_reg > 0)) return fail(OCTMC_E_INVALID, "eps_huber and eps_reg must be > 0");
    if (p->flyback_frac < 0 || p->mean_weight < 0) return fail(OCTMC_E_INVALID, "negative flyback or mean weight");
    if (p->levels < 1 || p->levels > OCTMC_MAX_LEVELS) return fail(OCTMC_E_INVALID, "levels must lie in [1, 8]");
    if (p->iters_per_level < 0) return fail(OCTMC_E_INVALID, "iters_per_level must be >= 0");
    if (p->lbfgs_m < 1 || p->lbfgs_m > 8) return fail(OCTMC_E_INVALID, "lbfgs_m must lie in [1, 8]");
    if (p->ls_max_evals < 1) return fail(OCTMC_E_INVALID, "ls_max_evals must be >= 1");
    if (!(p->c1 > 0 && p->c1 < p->c2 && p->c2 < 1)) return fail(OCTMC_E_INVALID, "need 0 < c1 < c2 < 1");
    if (p->prealign_iters < 0) return fail(OCTMC_E_INVALID, "prealign_iters must be >= 0");
    if (p->gamma_tilt < 0) return fail(OCTMC_E_INVALID, "gamma_tilt must be >= 0");
    if (p->flags & ~(OCTMC_CHECK_NAN | OCTMC_DETECT_INVALID | OCTMC_ENFACE_PROJECT | OCTMC_PREALIGN |
                     OCTMC_MULTI_PAIRWISE | OCTMC_HOST_LINE_SEARCH))
        return fail(OCTMC_E_INVALID, "unknown flags");
    return OCTMC_OK;
}

int octmc::validate_shape(const octmc_params* params, const octmc_shape* shape)
{
    if (!shape) return fail(OCTMC_E_INVALID, "shape is NULL");
    const int w = shape->w, h = shape->h, d = shape->d;
    if (shape->dtype != OCTMC_F32 && shape->dtype != OCTMC_BF16 && shape->dtype != OCTMC_F16)
        return fail(OCTMC_E_DTYPE, "unknown storage type");
    if (shape->mem != OCTMC_MEM_HOST && shape->mem != OCTMC_MEM_DEVICE)
        return fail(OCTMC_E_INVALID, "unknown memory kind");
    if (w != h) return fail(OCTMC_E_SHAPE, "only square scans (w == h) are supported");
    if (w < 4 || d < 4) return fail(OCTMC_E_SHAPE, "scans must be at least 4 x 4 x 4");
    if ((size_t)w * h * d * 4 >= (1ull << 31)) return fail(OCTMC_E_SHAPE, "volume larger than 2^31 bytes");
    int wl = w, dl = d;
    for (int l = 1; l < params->levels; ++l) {
        wl = (wl + 1) / 2;
        dl = (dl + 1) / 2;
    }
    if (wl < 4 || dl < 4) return fail(OCTMC_E_SHAPE, "too many pyramid levels for this size");
    return OCTMC_OK;
}

// Every device allocation pair_create_impl, register_impl and merge_impl make
// for one pair whose inputs are on the host, each rounded up to the slab alignment.
// Structural inputs on the device are read where they are: the room of their copies
// is reserved too and stays free.
size_t octmc::pair_footprint(const octmc_params& pr, const octmc_shape& sh, bool have_octa, bool have_enface,
                             bool have_valid, bool merged)
{
    const size_t w = sh.w, h = sh.h, d = sh.d, na = w * h, nv = na * d;
    const size_t es = esize(sh.dtype);
    size_t t = 0;
    t += 2 * slab_bytes(nv * 4);  // float32 copies of the inputs
    t += slab_bytes(64);          // counters
    t += 2 * slab_bytes(na * 4);  // en face
    if (have_octa) {
        const bool detect = !have_valid && (pr.flags & OCTMC_DETECT_INVALID);
        t += 2 * slab_bytes(nv * 4);
        if (have_valid || detect) t += slab_bytes(h * 4) + slab_bytes(w * 4);  // substitution tables
        if (detect) t += slab_bytes(h * 8) + slab_bytes(w * 8);                // B-scan means
        if (!have_enface && (pr.flags & OCTMC_ENFACE_PROJECT)) t += slab_bytes(enface_scratch_bytes(sh.w, sh.h, sh.d));
    }
    t += slab_bytes(h * 4) + slab_bytes(w * 4);  // validity
    size_t lw = w, lh = h, ld = d;
    for (int l = 0; l < pr.levels; ++l) {
        if (l == 0 || sh.dtype != OCTMC_F32)  // a coarser level's float32 volume is its storage
            t += 2 * slab_bytes(lw * lh * (size_t)storage_pitch((int)ld, sh.dtype) * es);  // at its pitch
        if (l + 1 < pr.levels) {
            const size_t w2 = (lw + 1) / 2, h2 = (lh + 1) / 2, d2 = (ld + 1) / 2;
            t += 2 * slab_bytes(w2 * h2 * d2 * 4) + 2 * slab_bytes(w2 * h2 * 4) + slab_bytes(h2 * 4) +
                 slab_bytes(w2 * 4);
            lw = w2;
            lh = h2;
            ld = d2;
        }
    }
    t += slab_bytes(na * 8 * 4) + slab_bytes(kSumBlocks * 4 * 8) +
         slab_bytes((size_t)nblk_combine((int)na) * 8 * 8) + slab_bytes(OCTMC_MAX_LEVELS * 8) +
         slab_bytes(OCTMC_NTERMS * 8) + slab_bytes((size_t)512 * (kMaxDots + 1) * 8) +
         slab_bytes((kMaxDots + 1) * 8) + slab_bytes(sizeof(LbState));
    const size_t n0 = 6 * na;
    t += (size_t)(8 + 2 * pr.lbfgs_m) * slab_bytes(n0 * 8) + slab_bytes(n0 * 4);  // solver
    if (merged) t += slab_bytes(2 * na * 8) + slab_bytes(na * 16);                 // merge
    return t;
}

// ===========================================================================
// C ABI

extern "C" {

const char* octmc_version(void) { return "octmc 0.1 (gfx950)"; }

const char* octmc_last_error(void) { return g_err.c_str(); }

int octmc_params_default(octmc_params* out)
{
    if (!out) return fail(OCTMC_E_INVALID, "out is NULL");
    octmc_params p{};
    p.alpha = 1.0;
    p.delta0 = 0.5;
    p.eps_huber = 1e-3;
    p.eps_reg = 0.1;
    p.flyback_frac = 0.25;
    p.mean_weight = 1.0;
    p.levels = 0;  // automatic: the coarsest level at most kAutoCoarsest A-scans wide
    p.iters_per_level = 100;
    p.lbfgs_m = 5;
    p.ls_max_evals = 20;
    p.c1 = 1e-4;
    p.c2 = 0.9;
    p.merge_kappa = 1.0;
    p.merge_tau = 0.05;
    p.flags = 0;
    p.prealign_iters = 100;
    p.gamma_tilt = 1.0;
    *out = p;
    return OCTMC_OK;
}

int octmc_create(int device_ordinal, octmc_ctx** out)
{
    if (!out) return fail(OCTMC_E_INVALID, "out is NULL");
    int n = 0;
    HIP_TRY(hipGetDeviceCount(&n));
    if (device_ordinal < 0 || device_ordinal >= n) return fail(OCTMC_E_INVALID, "no such device");
    HIP_TRY(hipSetDevice(device_ordinal));
    void* scr = nullptr;
    OCTMC_TRY(scratch_address(device_ordinal, &scr));
    *out = new octmc_ctx{device_ordinal, scr, BlockCache::of(device_ordinal)};
    return OCTMC_OK;
}

int octmc_destroy(octmc_ctx* ctx)
{
    delete ctx;
    return OCTMC_OK;
}

int octmc_trim(octmc_ctx* ctx)
{
    if (!ctx) return fail(OCTMC_E_INVALID, "ctx is NULL");
    HIP_TRY(hipSetDevice(ctx->device));
    ctx_trim(ctx);
    return OCTMC_OK;
}

}  // extern "C"

// Stage 1 before ingest (Fig. 1): a structural-only pair (delta0 = 0, no en
// face images) of float32 device copies of the inputs carries the stage-1
// solve; both structural volumes and the OCTA volumes are then resampled
// axially with its field, and the pair is created from the prealigned
// volumes with the remaining flags.
int octmc::prealign_create(octmc_ctx* ctx, const octmc_params* params, const octmc_shape* shape,
                           const float* oct_x, const float* oct_y, const float* octa_x, const float* octa_y,
                           const float* enface_x, const float* enface_y, const float* valid_x,
                           const float* valid_y, hipStream_t s, octmc_pair** out)
{
    const int w = shape->w, h = shape->h, d = shape->d;
    const size_t na = (size_t)w * h, nv = na * d;
    const bool host = shape->mem == OCTMC_MEM_HOST;
    const hipMemcpyKind kind = host ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    const bool have_octa = octa_x && octa_y;
    Blocks tmp(ctx->cache);
    auto dalloc = [&](size_t bytes) { return static_cast<float*>(tmp.get(bytes)); };
    const int nvol = have_octa ? 4 : 2;
    const float* src[4] = {oct_x, oct_y, octa_x, octa_y};
    const float* in[4] = {nullptr, nullptr, nullptr, nullptr};
    float* pre[4] = {nullptr, nullptr, nullptr, nullptr};
    for (int q = 0; q < nvol; ++q) {
        float* copy = host ? dalloc(nv * 4) : nullptr;  // device inputs are read where they are
        pre[q] = dalloc(nv * 4);
        if ((host && !copy) || !pre[q]) return fail(OCTMC_E_OOM, "out of device memory (prealignment)");
        if (host) HIP_TRY(hipMemcpyAsync(copy, src[q], nv * 4, kind, s));
        in[q] = host ? copy : src[q];
    }
    float* zero = dalloc(na * 4);
    float* dz = dalloc(2 * na * 4);
    double* th_d = (double*)dalloc(2 * (size_t)(w + h) * 8);
    if (!zero || !dz || !th_d) return fail(OCTMC_E_OOM, "out of device memory (prealignment)");
    HIP_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(zero), 0u, na, s));
    octmc_params p1 = *params;
    p1.flags &= OCTMC_CHECK_NAN | OCTMC_HOST_LINE_SEARCH;
    p1.delta0 = 0.0;  // the en face OCTA data is not used in this stage (Sec. 2.4)
    octmc_shape sh1 = *shape;
    sh1.mem = OCTMC_MEM_DEVICE;
    std::vector<double> th;
    {
        octmc_pair* P1 = nullptr;
        OCTMC_TRY(pair_create_impl(ctx, &p1, &sh1, in[0], in[1], nullptr, nullptr, zero, zero, nullptr, nullptr, s,
                                   nullptr, &P1));
        std::unique_ptr<octmc_pair> g1(P1);
        OCTMC_TRY(prealign_solve(P1, params->gamma_tilt, params->prealign_iters, th, nullptr, s));
        HIP_TRY(P1->mem.settle(s));
    }
    HIP_TRY(hipMemcpyAsync(th_d, th.data(), th.size() * 8, hipMemcpyHostToDevice, s));
    HIP_TRY(launch_tilt_expand(th_d, w, h, nullptr, dz, s));
    for (int q = 0; q < nvol; ++q) HIP_TRY(launch_resample_z(in[q], dz + (q & 1) * na, na, d, pre[q], s));
    // en face images (depth projections, unchanged by axial shifts) and
    // validity vectors as given, on the device
    float* enf[2] = {nullptr, nullptr};
    float* val[2] = {nullptr, nullptr};
    if (enface_x && enface_y) {
        enf[0] = dalloc(na * 4);
        enf[1] = dalloc(na * 4);
        if (!enf[0] || !enf[1]) return fail(OCTMC_E_OOM, "out of device memory (prealignment)");
        HIP_TRY(hipMemcpyAsync(enf[0], enface_x, na * 4, kind, s));
        HIP_TRY(hipMemcpyAsync(enf[1], enface_y, na * 4, kind, s));
    }
    if (valid_x && valid_y) {
        val[0] = dalloc((size_t)h * 4);
        val[1] = dalloc((size_t)w * 4);
        if (!val[0] || !val[1]) return fail(OCTMC_E_OOM, "out of device memory (prealignment)");
        HIP_TRY(hipMemcpyAsync(val[0], valid_x, (size_t)h * 4, kind, s));
        HIP_TRY(hipMemcpyAsync(val[1], valid_y, (size_t)w * 4, kind, s));
    }
    octmc_params p2 = *params;
    p2.flags &= ~OCTMC_PREALIGN;
    octmc_pair* P = nullptr;
    OCTMC_TRY(pair_create_impl(ctx, &p2, &sh1, pre[0], pre[1], have_octa ? pre[2] : nullptr,
                               have_octa ? pre[3] : nullptr, enf[0], enf[1], val[0], val[1], s, nullptr, &P));
    P->theta = th;
    *out = P;
    tmp.idle = true;  // pair_create_impl has waited for the stream
    return OCTMC_OK;
}

int octmc::pair_create_impl(octmc_ctx* ctx, const octmc_params* params, const octmc_shape* shape,
                            const float* oct_x, const float* oct_y, const float* octa_x, const float* octa_y,
                            const float* enface_x, const float* enface_y, const float* valid_x, const float* valid_y,
                            hipStream_t s, Slab* slab, octmc_pair** out)
{
    if (!ctx || !shape || !out || !oct_x || !oct_y) return fail(OCTMC_E_INVALID, "NULL argument");
    OCTMC_TRY(validate_params(params));
    OCTMC_TRY(validate_shape(params, shape));
    const int w = shape->w, h = shape->h, d = shape->d;
    const bool have_octa = octa_x && octa_y;
    const bool have_enface = enface_x && enface_y;
    const bool detect = have_octa && !valid_x && (params->flags & OCTMC_DETECT_INVALID);
    const bool project = have_octa && !have_enface && (params->flags & OCTMC_ENFACE_PROJECT);
    void* pscratch = nullptr;
    if (!have_octa && !have_enface) return fail(OCTMC_E_INVALID, "need both OCTA volumes or both en face images");
    if (project && (w > enface_max_bscan() || h > enface_max_bscan()))
        return fail(OCTMC_E_SHAPE, "B-scans longer than 8192 A-scans for the projection");
    if ((octa_x != nullptr) != (octa_y != nullptr) || (enface_x != nullptr) != (enface_y != nullptr))
        return fail(OCTMC_E_INVALID, "OCTA inputs must be given for both scans");
    if ((valid_x != nullptr) != (valid_y != nullptr)) return fail(OCTMC_E_INVALID, "give both validity vectors or none");
    HIP_TRY(hipSetDevice(ctx->device));
    if (params->flags & OCTMC_PREALIGN) {
        if (slab) return fail(OCTMC_E_INVALID, "OCTMC_PREALIGN is not available for served requests");
        return prealign_create(ctx, params, shape, oct_x, oct_y, octa_x, octa_y, enface_x, enface_y, valid_x, valid_y,
                               s, out);
    }
    auto* P = new octmc_pair();
    std::unique_ptr<octmc_pair> guard(P);
    P->slab = slab;
    P->ctx = ctx;
    P->mem.cache = ctx->cache;
    P->params = *params;
    P->dtype = shape->dtype;
    P->nlev = params->levels;
    const size_t na = (size_t)w * h, nv = na * d;
    const bool host = shape->mem == OCTMC_MEM_HOST;
    const hipMemcpyKind kind = host ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    Blocks tmp(ctx->cache);
    auto talloc = [&](size_t bytes) -> void* {
        // temporaries stay in the slab until the pair is released
        return slab ? slab->take(bytes) : tmp.get(bytes);
    };
    // the structural inputs on the device: those that are there are only read,
    // and this call returns after its last reader
    const float* f32[2] = {oct_x, oct_y};
    for (int V = 0; host && V < 2; ++V) {
        float* copy = (float*)talloc(nv * 4);
        if (!copy) return fail(OCTMC_E_OOM, "out of device memory (input staging)");
        HIP_TRY(hipMemcpyAsync(copy, f32[V], nv * 4, kind, s));
        f32[V] = copy;
    }
    unsigned* ctr = nullptr;
    HIP_TRY(P->alloc(&ctr, 64));
    HIP_TRY(launch_fill_u32(ctr, 0u, 16, s));
    P->counters = ctr;
    if (params->flags & OCTMC_CHECK_NAN) {
        HIP_TRY(launch_count_nonfinite(f32[0], nv, ctr + 8, s));
        HIP_TRY(launch_count_nonfinite(f32[1], nv, ctr + 8, s));
        unsigned bad = 0;
        HIP_TRY(hipMemcpyAsync(&bad, ctr + 8, 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        if (bad) return fail(OCTMC_E_NAN, "non-finite values in the structural volumes");
    }
    // validity: as given, from the OCTA volumes below, or all valid
    float* cval[2] = {nullptr, nullptr};
    const int nval[2] = {h, w};
    const float* valid[2] = {valid_x, valid_y};
    for (int V = 0; V < 2; ++V) {
        HIP_TRY(P->alloc(&cval[V], nval[V] * 4));
        if (valid_x) HIP_TRY(hipMemcpyAsync(cval[V], valid[V], nval[V] * 4, kind, s));
        else if (!detect) HIP_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(cval[V]), 0x3F800000u, nval[V], s));
    }
    // OCTA volumes: keep for the merge, replace invalid B-scans by their
    // nearest valid neighbour (Sec. 2.3, 2.5), then project
    float* enf[2] = {nullptr, nullptr};
    HIP_TRY(P->alloc(&enf[0], na * 4));
    HIP_TRY(P->alloc(&enf[1], na * 4));
    if (have_octa) {
        const float* src[2] = {octa_x, octa_y};
        for (int V = 0; V < 2; ++V) {
            HIP_TRY(P->alloc(&P->octa[V], nv * 4));
            if (host) {
                HIP_TRY(hipMemcpyAsync(P->octa[V], src[V], nv * 4, kind, s));
                src[V] = P->octa[V];
            }
            if (detect) {  // B-scan validity from the OCTA volume (Sec. 2.2)
                double* means = (double*)talloc(nval[V] * 8);
                if (!means) return fail(OCTMC_E_OOM, "out of device memory (validity)");
                HIP_TRY(launch_validity(src[V], w, h, d, V, means, cval[V], s));
            }
            if (project) {  // Sec. 2.3, from the OCTA volume before substitution
                if (!pscratch) pscratch = talloc(enface_scratch_bytes(w, h, d));
                if (!pscratch) return fail(OCTMC_E_OOM, "out of device memory (projection)");
                HIP_TRY(launch_enface_project(f32[V], src[V], w, h, d, V, cval[V], nullptr, enf[V], nullptr, nullptr,
                                              pscratch, s));
            }
            int* from = nullptr;
            if (valid_x || detect) {
                from = (int*)talloc(nval[V] * 4);
                if (!from) return fail(OCTMC_E_OOM, "out of device memory");
                HIP_TRY(launch_nearest_valid(cval[V], nval[V], from, s));
            }
            const bool mean = !have_enface && !project;
            if (!host || from || mean)
                HIP_TRY(launch_take_octa(src[V], P->octa[V], w, h, d, from, V, mean ? enf[V] : nullptr, s));
        }
    }
    if (have_enface) {
        HIP_TRY(hipMemcpyAsync(enf[0], enface_x, na * 4, kind, s));
        HIP_TRY(hipMemcpyAsync(enf[1], enface_y, na * 4, kind, s));
    }
    // pyramid: float32 at every level, stored in the storage type
    const float* cur[2] = {f32[0], f32[1]};
    float* cen[2] = {enf[0], enf[1]};
    int lw = w, lh = h, ld = d;
    for (int l = 0; l < P->nlev; ++l) {
        Level& L = P->lev[l];
        L.w = lw;
        L.h = lh;
        L.d = ld;
        L.na = lw * lh;
        // 16-bit storage of an odd depth gets one padding sample per A-scan, so
        // that the two-samples-per-lane structural kernel serves every level
        L.dp = storage_pitch(ld, P->dtype);
        const size_t lnv = (size_t)L.na * L.dp;
        L.vol_bytes = (uint32_t)(lnv * esize(P->dtype));
        LevelJob job;
        job.nvol = 2;
        job.w = lw;
        job.h = lh;
        job.d = ld;
        job.dp = L.dp;
        const bool more = l + 1 < P->nlev, as_is = P->dtype == OCTMC_F32;
        const int w2 = (lw + 1) / 2, h2 = (lh + 1) / 2, d2 = (ld + 1) / 2;
        void* st[2];
        float *ne[2], *nval2[2];
        for (int V = 0; V < 2; ++V) {
            job.in[V] = cur[V];
            job.image[V] = cen[V];
            job.valid[V] = cval[V];
            job.nvalid[V] = V == 0 ? lh : lw;
            if (as_is && l > 0) {  // the level's float32 volume is its storage
                st[V] = const_cast<float*>(cur[V]);
            } else {
                HIP_TRY(P->alloc(&st[V], lnv * esize(P->dtype)));
                job.store[V] = st[V];
            }
            if (more) {
                const size_t bytes = (size_t)w2 * h2 * d2 * 4;
                if (as_is) HIP_TRY(P->alloc(&job.next[V], bytes));
                else job.next[V] = (float*)talloc(bytes);
                if (!job.next[V]) return fail(OCTMC_E_OOM, "out of device memory (pyramid)");
                HIP_TRY(P->alloc(&ne[V], (size_t)w2 * h2 * 4));
                HIP_TRY(P->alloc(&nval2[V], (V == 0 ? h2 : w2) * 4));
                job.next_image[V] = ne[V];
                job.next_valid[V] = nval2[V];
            }
        }
        if (job.store[0] || more) HIP_TRY(launch_level(job, P->dtype, s));
        L.sx = st[0];
        L.sy = st[1];
        L.ax = cen[0];
        L.ay = cen[1];
        L.vx = cval[0];
        L.vy = cval[1];
        if (more) {
            for (int V = 0; V < 2; ++V) {
                cur[V] = job.next[V];
                cen[V] = ne[V];
                cval[V] = nval2[V];
            }
            lw = w2;
            lh = h2;
            ld = d2;
        }
    }
    OCTMC_TRY(pair_alloc_scratch(P, na, s));
    HIP_TRY(tmp.settle(s));
    *out = guard.release();
    return OCTMC_OK;
}

extern "C" {

int octmc_pair_create(octmc_ctx* ctx, const octmc_params* params, const octmc_shape* shape, const float* oct_x,
                      const float* oct_y, const float* octa_x, const float* octa_y, const float* enface_x,
                      const float* enface_y, const float* valid_x, const float* valid_y, void* stream,
                      octmc_pair** out)
{
    octmc_params pr{};
    if (params && shape) pr = resolve_levels(*params, *shape);
    return pair_create_impl(ctx, params && shape ? &pr : params, shape, oct_x, oct_y, octa_x, octa_y, enface_x,
                            enface_y, valid_x, valid_y, static_cast<hipStream_t>(stream), nullptr, out);
}

int octmc_validity_from_octa(octmc_ctx* ctx, const octmc_shape* shape, const float* octa, int32_t scan,
                             float* valid_out, void* stream)
{
    if (!ctx || !shape || !octa || !valid_out) return fail(OCTMC_E_INVALID, "NULL argument");
    if (scan != 0 && scan != 1) return fail(OCTMC_E_INVALID, "scan must be 0 (X-fast) or 1 (Y-fast)");
    if (shape->mem != OCTMC_MEM_HOST && shape->mem != OCTMC_MEM_DEVICE)
        return fail(OCTMC_E_INVALID, "unknown memory kind");
    const int w = shape->w, h = shape->h, d = shape->d;
    if (w < 1 || h < 1 || d < 1) return fail(OCTMC_E_SHAPE, "empty volume");
    const size_t nv = (size_t)w * h * d;
    if (nv * 4 >= (1ull << 31)) return fail(OCTMC_E_SHAPE, "volume larger than 2^31 bytes");
    HIP_TRY(hipSetDevice(ctx->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    Blocks tmp(ctx->cache);
    const float* vol = octa;
    if (shape->mem == OCTMC_MEM_HOST) {
        void* q = tmp.get(nv * 4);
        HIP_TRY(q ? hipSuccess : tmp.err);
        HIP_TRY(hipMemcpyAsync(q, octa, nv * 4, hipMemcpyHostToDevice, s));
        vol = static_cast<const float*>(q);
    }
    void* means = tmp.get((size_t)(scan == 0 ? h : w) * 8);
    HIP_TRY(means ? hipSuccess : tmp.err);
    HIP_TRY(launch_validity(vol, w, h, d, scan, static_cast<double*>(means), valid_out, s));
    HIP_TRY(tmp.settle(s));
    return OCTMC_OK;
}

int octmc_enface_workspace_size(int32_t w, int32_t h, int32_t d, uint64_t* bytes)
{
    if (!bytes) return fail(OCTMC_E_INVALID, "NULL argument");
    if (w < 1 || h < 1 || d < 1) return fail(OCTMC_E_SHAPE, "empty volume");
    *bytes = enface_scratch_bytes(w, h, d);
    return OCTMC_OK;
}

int octmc_enface_project(octmc_ctx* ctx, const octmc_shape* shape, const float* oct, const float* octa,
                         int32_t scan, const float* valid, const double* fixed, float* enface_out,
                         int32_t* count_out, double* stats_out, void* workspace, uint64_t workspace_bytes,
                         void* stream)
{
    if (!ctx || !shape || !oct || !octa || !enface_out) return fail(OCTMC_E_INVALID, "NULL argument");
    if (scan != 0 && scan != 1) return fail(OCTMC_E_INVALID, "scan must be 0 (X-fast) or 1 (Y-fast)");
    if (shape->mem != OCTMC_MEM_HOST && shape->mem != OCTMC_MEM_DEVICE)
        return fail(OCTMC_E_INVALID, "unknown memory kind");
    const int w = shape->w, h = shape->h, d = shape->d;
    if (w < 1 || h < 1 || d < 1) return fail(OCTMC_E_SHAPE, "empty volume");
    if (w > enface_max_bscan() || h > enface_max_bscan()) return fail(OCTMC_E_SHAPE, "B-scans longer than 8192 A-scans");
    const size_t nv = (size_t)w * h * d, nb = scan == 0 ? h : w;
    if (nv * 4 >= (1ull << 31)) return fail(OCTMC_E_SHAPE, "volume larger than 2^31 bytes");
    if (fixed && !(fixed[0] == fixed[0] && fixed[1] == fixed[1])) return fail(OCTMC_E_INVALID, "fixed mapping is NaN");
    HIP_TRY(hipSetDevice(ctx->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    Blocks tmp(ctx->cache);
    auto dalloc = [&](size_t bytes) { return tmp.get(bytes); };
    if (workspace && workspace_bytes < enface_scratch_bytes(w, h, d))
        return fail(OCTMC_E_INVALID, "workspace smaller than octmc_enface_workspace_size");
    void* scratch = workspace ? workspace : dalloc(enface_scratch_bytes(w, h, d));
    if (!scratch) return fail(OCTMC_E_OOM, "out of device memory (projection scratch)");
    const float *o = oct, *a = octa, *v = valid;
    if (shape->mem == OCTMC_MEM_HOST) {
        float* q = (float*)dalloc(2 * nv * 4 + nb * 4);
        if (!q) return fail(OCTMC_E_OOM, "out of device memory (input copies)");
        HIP_TRY(hipMemcpyAsync(q, oct, nv * 4, hipMemcpyHostToDevice, s));
        HIP_TRY(hipMemcpyAsync(q + nv, octa, nv * 4, hipMemcpyHostToDevice, s));
        o = q;
        a = q + nv;
        if (valid) {
            HIP_TRY(hipMemcpyAsync(q + 2 * nv, valid, nb * 4, hipMemcpyHostToDevice, s));
            v = q + 2 * nv;
        }
    }
    HIP_TRY(launch_enface_project(o, a, w, h, d, scan, v, fixed, enface_out, count_out, stats_out, scratch, s));
    if (!tmp.dev.empty() || stats_out) HIP_TRY(tmp.settle(s));
    return OCTMC_OK;
}

int octmc_pair_destroy(octmc_pair* pair)
{
    if (pair && !pair->slab) {  // a slab's owner orders its release after the pair's work
        (void)hipSetDevice(pair->ctx->device);
        pair->mem.idle = hipDeviceSynchronize() == hipSuccess;
    }
    delete pair;
    return OCTMC_OK;
}

int octmc_pair_levels(const octmc_pair* pair, int32_t* levels)
{
    if (!pair || !levels) return fail(OCTMC_E_INVALID, "NULL argument");
    *levels = pair->nlev;
    return OCTMC_OK;
}

int octmc_pair_level_shape(const octmc_pair* pair, int32_t level, int32_t* w, int32_t* h, int32_t* d)
{
    OCTMC_TRY(check_level(pair, level));
    if (w) *w = pair->lev[level].w;
    if (h) *h = pair->lev[level].h;
    if (d) *d = pair->lev[level].d;
    return OCTMC_OK;
}

int octmc_eval(octmc_pair* pair, int32_t level, const float* disp, double* terms, float* grad, int32_t eta_mode,
               void* stream)
{
    OCTMC_TRY(check_level(pair, level));
    if (!disp || !terms) return fail(OCTMC_E_INVALID, "disp and terms are required");
    if (eta_mode != 0 && eta_mode != 1) return fail(OCTMC_E_INVALID, "eta_mode must be 0 or 1");
    HIP_TRY(hipSetDevice(pair->ctx->device));
    EvalArgs ea{pair, disp, terms, grad, nullptr, nullptr, level, eta_mode};
    return eval_group(&ea, 1, static_cast<hipStream_t>(stream));
}

int octmc_eval_noalloc(octmc_ctx* ctx, const octmc_params* params, const octmc_shape* shape, const void* sx,
                       const void* sy, const float* ax, const float* ay, const float* vx, const float* vy,
                       const float* disp, double* eta, double* terms, float* grad, int32_t eta_mode, void* stream)
{
    if (!ctx || !params || !shape) return fail(OCTMC_E_INVALID, "ctx, params and shape are required");
    if (!sx || !sy || !ax || !ay || !vx || !vy || !disp || !eta || !terms)
        return fail(OCTMC_E_INVALID, "volumes, en face images, validity, disp, eta and terms are required");
    if (eta_mode != 0 && eta_mode != 1) return fail(OCTMC_E_INVALID, "eta_mode must be 0 or 1");
    octmc_params pr = *params;
    pr.levels = 1;  // one level: the pyramid depth plays no part here
    OCTMC_TRY(validate_params(&pr));
    if (shape->mem != OCTMC_MEM_DEVICE) return fail(OCTMC_E_INVALID, "octmc_eval_noalloc takes device inputs");
    OCTMC_TRY(validate_shape(&pr, shape));
    const int w = shape->w, h = shape->h, d = shape->d;
    const size_t na = (size_t)w * h;
    if (na > (size_t)OCTMC_NOALLOC_MAX_ASCANS)
        return fail(OCTMC_E_SHAPE, "w * h exceeds OCTMC_NOALLOC_MAX_ASCANS (the static scratch of octmc_eval_noalloc)");
    if (!ctx->noalloc_scratch) return fail(OCTMC_E_DEVICE, "the context holds no scratch address");
    HIP_TRY(hipSetDevice(ctx->device));
    EvalView v;
    v.L.w = w;
    v.L.h = h;
    v.L.d = d;
    v.L.na = (int)na;
    v.L.dp = d;  // the caller's volumes: [h][w][d]
    v.L.sx = const_cast<void*>(sx);  // read only
    v.L.sy = const_cast<void*>(sy);
    v.L.ax = const_cast<float*>(ax);
    v.L.ay = const_cast<float*>(ay);
    v.L.vx = const_cast<float*>(vx);
    v.L.vy = const_cast<float*>(vy);
    v.L.vol_bytes = (uint32_t)(na * d * esize(shape->dtype));
    v.dtype = shape->dtype;
    v.params = &pr;
    char* base = static_cast<char*>(ctx->noalloc_scratch);
    v.part = reinterpret_cast<float*>(base);
    v.sum_blk = reinterpret_cast<double*>(base + kNoAllocPart);
    v.comb_blk = reinterpret_cast<double*>(base + kNoAllocPart + kNoAllocSum);
    v.ticket = reinterpret_cast<unsigned*>(v.sum_blk + kTicketAt);
    v.eta = eta;
    v.orient = 2;
    EvalArgs ea{nullptr, disp, terms, grad, nullptr, nullptr, 0, eta_mode};
    ea.view = &v;
    return eval_group(&ea, 1, static_cast<hipStream_t>(stream));
}

int octmc_eval_profile(octmc_pair* pair, int32_t level, const float* disp, double* terms, float* grad,
                       int32_t eta_mode, float* stage_ms, void* stream)
{
    OCTMC_TRY(check_level(pair, level));
    if (!disp || !terms || !stage_ms) return fail(OCTMC_E_INVALID, "disp, terms and stage_ms are required");
    if (eta_mode != 0 && eta_mode != 1) return fail(OCTMC_E_INVALID, "eta_mode must be 0 or 1");
    HIP_TRY(hipSetDevice(pair->ctx->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t ev[4] = {};
    for (auto& e : ev) HIP_TRY(hipEventCreate(&e));
    struct Ev {
        hipEvent_t* e;
        ~Ev()
        {
            for (int k = 0; k < 4; ++k) (void)hipEventDestroy(e[k]);
        }
    } guard{ev};
    EvalArgs ea{pair, disp, terms, grad, nullptr, nullptr, level, eta_mode};
    OCTMC_TRY(eval_group(&ea, 1, s, ev));
    HIP_TRY(hipEventSynchronize(ev[3]));
    for (int k = 0; k < 3; ++k) HIP_TRY(hipEventElapsedTime(stage_ms + k, ev[k], ev[k + 1]));
    return OCTMC_OK;
}

int octmc_eval_batched(octmc_pair* const* pairs, int32_t npairs, int32_t level, const float* disp, double* terms,
                       float* grad, int32_t eta_mode, void* stream)
{
    if (!pairs || npairs < 1 || !disp || !terms) return fail(OCTMC_E_INVALID, "bad batched arguments");
    if (eta_mode != 0 && eta_mode != 1) return fail(OCTMC_E_INVALID, "eta_mode must be 0 or 1");
    for (int q = 0; q < npairs; ++q) {
        OCTMC_TRY(check_level(pairs[q], level));
        for (int r = 0; r < q; ++r)
            if (pairs[r] == pairs[q]) return fail(OCTMC_E_INVALID, "a pair appears twice in the batch");
    }
    const Level& L0 = pairs[0]->lev[level];
    for (int q = 1; q < npairs; ++q) {
        const Level& L = pairs[q]->lev[level];
        if (L.w != L0.w || L.h != L0.h || L.d != L0.d) return fail(OCTMC_E_SHAPE, "batched pairs differ in shape");
    }
    HIP_TRY(hipSetDevice(pairs[0]->ctx->device));
    const size_t nd = (size_t)2 * L0.na * 3;
    for (int q0 = 0; q0 < npairs; q0 += kMaxJobs) {
        const int cnt = std::min(kMaxJobs, npairs - q0);
        EvalArgs ea[kMaxJobs];
        for (int q = 0; q < cnt; ++q)
            ea[q] = EvalArgs{pairs[q0 + q], disp + (q0 + q) * nd, terms + (size_t)(q0 + q) * OCTMC_NTERMS,
                             grad ? grad + (q0 + q) * nd : nullptr, nullptr, nullptr, level, eta_mode};
        OCTMC_TRY(eval_group(ea, cnt, static_cast<hipStream_t>(stream)));
    }
    return OCTMC_OK;
}

}  // extern "C"

int octmc::merge_impl(octmc_pair* pair, const float* disp, float* merged_oct, float* merged_octa, hipStream_t s,
                      Slab* slab)
{
    if (!pair || !disp || !merged_oct) return fail(OCTMC_E_INVALID, "NULL argument");
    if (merged_octa && !pair->octa[0]) return fail(OCTMC_E_INVALID, "no OCTA volumes were given at creation");
    HIP_TRY(hipSetDevice(pair->ctx->device));
    const Level& L = pair->lev[0];
    Blocks tmp(pair->ctx->cache);
    unsigned long long* grid = nullptr;
    float4* wts = nullptr;
    if (slab) {
        grid = static_cast<unsigned long long*>(slab->take((size_t)2 * L.na * 8));
        wts = static_cast<float4*>(slab->take((size_t)L.na * 16));
        if (!grid || !wts) return fail(OCTMC_E_OOM, "slab exhausted (merge)");
    } else {
        grid = static_cast<unsigned long long*>(tmp.get((size_t)2 * L.na * 8));
        wts = static_cast<float4*>(tmp.get((size_t)L.na * 16));
        HIP_TRY(grid && wts ? hipSuccess : tmp.err);
    }
    HIP_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(grid), 0u, (size_t)4 * L.na, s));
    HIP_TRY(launch_density(disp, L.w, L.h, grid, s));
    HIP_TRY(launch_merge_weights(disp, L.w, L.h, grid, merged_octa ? L.vx : nullptr, merged_octa ? L.vy : nullptr,
                                 pair->params.merge_kappa, pair->params.merge_tau, wts, s));
    HIP_TRY(launch_merge_volume(L.sx, L.sy, pair->dtype, disp, wts, 0, L.w, L.h, L.d, L.dp, merged_oct, s));
    if (merged_octa)
        HIP_TRY(launch_merge_volume(pair->octa[0], pair->octa[1], OCTMC_F32, disp, wts, 1, L.w, L.h, L.d, L.d,
                                    merged_octa, s));
    HIP_TRY(tmp.settle(s));
    return OCTMC_OK;
}

int octmc::register_impl(octmc_pair* pair, float* disp_out, float* merged_oct, float* merged_octa, octmc_report* rep,
                         hipStream_t s, Evaluator* ev, Slab* slab, double* h_terms_in, double* h_dots_in)
{
    if (!pair || !disp_out) return fail(OCTMC_E_INVALID, "NULL argument");
    if (merged_octa && !pair->octa[0]) return fail(OCTMC_E_INVALID, "no OCTA volumes were given at creation");
    int idle = 0;
    if (!pair->busy.compare_exchange_strong(idle, 1)) return fail(OCTMC_E_BUSY, "pair is in use");
    struct Unbusy {
        octmc_pair* p;
        ~Unbusy() { p->busy.store(0); }
    } ub{pair};
    HIP_TRY(hipSetDevice(pair->ctx->device));
    DirectEvaluator direct;
    if (!ev) ev = &direct;
    const octmc_params& pr = pair->params;
    const size_t n0 = (size_t)6 * pair->lev[0].na;
    Solver sv;
    sv.m = pr.lbfgs_m;
    Blocks mem(pair->ctx->cache);
    auto dalloc = [&](double** p) -> int {
        if (slab) {
            *p = static_cast<double*>(slab->take(n0 * 8));
            if (!*p) return fail(OCTMC_E_OOM, "slab exhausted (solver)");
            return OCTMC_OK;
        }
        *p = static_cast<double*>(mem.get(n0 * 8));
        HIP_TRY(*p ? hipSuccess : mem.err);
        return OCTMC_OK;
    };
    OCTMC_TRY(dalloc(&sv.x));
    OCTMC_TRY(dalloc(&sv.g));
    OCTMC_TRY(dalloc(&sv.p));
    OCTMC_TRY(dalloc(&sv.xt));
    OCTMC_TRY(dalloc(&sv.xprev));
    OCTMC_TRY(dalloc(&sv.sc));
    OCTMC_TRY(dalloc(&sv.gt));
    OCTMC_TRY(dalloc(&sv.yc));
    for (int k = 0; k < sv.m; ++k) {
        OCTMC_TRY(dalloc(&sv.S[k]));
        OCTMC_TRY(dalloc(&sv.Y[k]));
    }
    if (slab) {
        sv.xt32 = static_cast<float*>(slab->take(n0 * 4));
        if (!sv.xt32) return fail(OCTMC_E_OOM, "slab exhausted (solver)");
    } else {
        sv.xt32 = static_cast<float*>(mem.get(n0 * 4));
        HIP_TRY(sv.xt32 ? hipSuccess : mem.err);
    }
    double *h_terms = h_terms_in, *h_dots = h_dots_in;
    if (!h_terms) h_terms = mem.get_host(OCTMC_NTERMS);
    if (!h_dots) h_dots = mem.get_host(kMaxDots + 1);
    HIP_TRY(h_terms && h_dots ? hipSuccess : mem.err);
    if (rep) {
        std::memset(rep, 0, sizeof(*rep));
        rep->nlevels = pair->nlev;
    }
    // the iteration's decisions on the device when the evaluator only
    // enqueues work and the history fits one keyed dot-product pass
    const bool device_ls = ev->enqueue_only() && !(pr.flags & OCTMC_HOST_LINE_SEARCH) && sv.m <= kLbMaxM;
    for (int l = pair->nlev - 1; l >= 0; --l) {
        const Level& L = pair->lev[l];
        const size_t n = (size_t)6 * L.na;
        if (l == pair->nlev - 1) {
            HIP_TRY(hipMemsetAsync(sv.x, 0, n * 8, s));
        } else {
            const Level& C = pair->lev[l + 1];
            HIP_TRY(hipMemcpyAsync(sv.xprev, sv.x, (size_t)6 * C.na * 8, hipMemcpyDeviceToDevice, s));
            HIP_TRY(launch_upsample(sv.xprev, C.w, C.h, sv.x, L.w, L.h, s));
        }
        sv.n = n;
        LevelRun run{pair, l, &sv, s, n, h_terms, h_dots, ev};
        LevelStats st;
        if (device_ls)
            OCTMC_TRY(run.run_device(pr, st));
        else
            OCTMC_TRY(run.run(pr, st));
        if (rep) {
            const int r = pair->nlev - 1 - l;
            rep->iters[r] = st.iters;
            rep->evals[r] = st.evals;
            rep->ls_fail[r] = st.ls_fail;
            rep->f_start[r] = st.f_start;
            rep->f_end[r] = st.f_end;
            HIP_TRY(hipMemcpyAsync(h_terms, pair->eta + l, 8, hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            rep->eta[r] = h_terms[0];
        }
    }
    HIP_TRY(launch_to_f32(sv.x, disp_out, n0, s));
    if (merged_oct) OCTMC_TRY(merge_impl(pair, disp_out, merged_oct, merged_octa, s, slab));
    HIP_TRY(mem.settle(s));
    return OCTMC_OK;
}

extern "C" {

int octmc_merge(octmc_pair* pair, const float* disp, float* merged_oct, float* merged_octa, void* stream)
{
    return merge_impl(pair, disp, merged_oct, merged_octa, static_cast<hipStream_t>(stream), nullptr);
}

int octmc_register(octmc_pair* pair, float* disp_out, float* merged_oct, float* merged_octa, octmc_report* rep,
                   void* stream)
{
    return register_impl(pair, disp_out, merged_oct, merged_octa, rep, static_cast<hipStream_t>(stream), nullptr,
                         nullptr, nullptr, nullptr);
}

}  // extern "C"
