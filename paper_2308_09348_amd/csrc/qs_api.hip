// qs_api.hip -- host side of the C ABI declared in include/qscatter.h.
//
// The host validates arguments, derives the scalar constants of the problem
// (Sec. 2 eq. a0eff; Sec. 4 eq. dpdtRR; Sec. 3 eq. PWCRR) and enqueues
// kernels; all per-sample arithmetic runs on the device.
#include "qscatter.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "qs_internal.h"

namespace {
// What a tuning choice is kept for: launches that agree on these run alike.
struct TuneKey {
    int32_t n_steps, rr, amp, dep, prec, hist_words, lg_total, lg_shots;
    bool operator==(const TuneKey &o) const { return std::memcmp(this, &o, sizeof(*this)) == 0; }
};
struct TuneEntry {
    TuneKey key;
    int32_t dep_tile, phase_cap, dep_cap;
};
// A captured forward launch sequence and the launch arguments it was
// captured with (it is replayed only for byte-identical arguments).
struct GraphEntry {
    std::vector<unsigned char> sig;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};
constexpr size_t kMaxGraphs = 8;
}  // namespace

constexpr int kStageSlots = 4;  // pinned staging blocks of the shot tables
constexpr int kStatusWords = 32;  // qs_sync_status calls that read through pinned words at once
constexpr int kTimingRing = 64;  // event sets of profiled calls kept for qs_timings_sum

struct qs_ctx {
    int device = -1;
    float *rad32 = nullptr;
    double *rad64 = nullptr;
    float *rad32d = nullptr;   // derivative tables (adjoint)
    double *rad64d = nullptr;
    double *phtab = nullptr;   // LCFA photon number CDF
    // per-call device scratch (grow-only)
    float *env32 = nullptr;
    double *env64 = nullptr;
    size_t env32_cap = 0, env64_cap = 0;
    unsigned long long *accum = nullptr;  // [2 + histogram words]: chimax, flags, hist
    size_t accum_cap = 0;
    double *partials = nullptr;
    size_t part_cap = 0;
    double *shadow = nullptr;  // outputs of the FP64-shadow view passes (photons, adjoint)
    size_t shadow_cap = 0;
    unsigned char *states = nullptr;  // per-sample final states (SampleState arrays)
    size_t states_cap = 0;
    uint16_t *order = nullptr;  // chi order of the samples (passes with FP64 steps)
    size_t order_cap = 0;
    // per-shot tables too large for the set-up kernel's argument: pinned staging
    // on the host, a device copy.  Calls take the staging blocks in turn, so the
    // host can stage a call while the copies of the kStageSlots - 1 calls before
    // it still wait on the stream; a block is reused once its own copy has run.
    unsigned char *stage[kStageSlots] = {};
    size_t stage_cap[kStageSlots] = {};
    hipEvent_t stage_done[kStageSlots] = {};  // the last copy out of each block
    bool stage_pending[kStageSlots] = {};
    int stage_next = 0;
    unsigned char *shot_tab = nullptr;
    size_t shot_tab_cap = 0;
    int *eval_flags = nullptr;
    // kernel timing: a ring of event sets, one set per profiled call, so
    // that many calls can be enqueued before any of them is read
    bool profiling = false;
    bool profiled_call = false;
    hipEvent_t ev[kTimingRing][6] = {};
    int ev_next = 0;   // the set the next profiled call records into
    int ev_last = 0;   // the set of the last profiled call
    int ev_count = 0;  // profiled calls since profiling was switched on
    // launch tuning (qs_tune): choices by launch class, and a forced choice
    // while tuning
    std::vector<TuneEntry> tunes;
    bool tune_forced = false;
    TuneEntry forced{};
    // forward launch graphs (qs_set_graphs)
    bool graphs = false;
    hipStream_t cap_stream = nullptr;
    std::vector<GraphEntry> graph_cache;
    // qs_forward_noalloc: the device address of this device's `scratch` array
    unsigned char *na_scratch = nullptr;
    // pinned words that qs_sync_status reads status words through, each claimed
    // by one call at a time (bits of status_used)
    int32_t *status_host = nullptr;
    std::atomic<uint32_t> status_used{0};
    char last_error[512] = {0};
};

// ---- scratch of qs_forward_noalloc -----------------------------------------
// The entry point for callers that cannot allocate takes all of its device
// scratch from one file-scope array (each GPU holds its own copy from the
// library's load until the process ends).  Layout, each part 256-byte aligned:
// the per-sample final states (6 double arrays and 1 float array of
// QS_NOALLOC_MAX_SAMPLES), the FP64 and FP32 envelope tables (2 n_steps + 1
// points at the largest n_steps), the accumulators (work counters, the status
// flags, the histogram words of the largest bins), the moment partials, the chi
// order of the samples and the device copy of the shot table.
namespace na {
constexpr size_t r256(size_t n) { return (n + 255) / 256 * 256; }
constexpr size_t kSamples = QS_NOALLOC_MAX_SAMPLES;
constexpr size_t kEnvPoints = 2 * 65536 + 1;
constexpr size_t kAccumWords = 2 + 1 + 3 * 4096 + 4 + 1;
// (rows of kMomRow samples below kDepItems items of kDepTile, else of kMomTile)
constexpr size_t kPartWords =
    std::max((kSamples + qs::kMomTile - 1) / qs::kMomTile,
             (size_t)qs::kDepItems * qs::kDepTile / qs::kMomRow) * qs::kPartials;
constexpr size_t kArr = r256(kSamples * 8), kArrf = r256(kSamples * 4);
constexpr size_t kStatesOff = 0;
constexpr size_t kEnv64Off = kStatesOff + 6 * kArr + kArrf;
constexpr size_t kEnv32Off = kEnv64Off + r256(kEnvPoints * 8);
constexpr size_t kAccumOff = kEnv32Off + r256(kEnvPoints * 4);
constexpr size_t kPartOff = kAccumOff + r256(kAccumWords * 8);
constexpr size_t kOrderOff = kPartOff + r256(kPartWords * 8);
constexpr size_t kTabOff = kOrderOff + r256(kSamples * sizeof(uint16_t));
constexpr size_t kTabBytes = r256(sizeof(qs::ShotParams) + sizeof(qs::ShotOut));
constexpr size_t kBytes = kTabOff + kTabBytes;
static_assert(kBytes < ((size_t)56 << 20), "the no-allocation scratch stays under 56 MiB");
}  // namespace na

static __device__ __align__(256) unsigned char scratch[na::kBytes];

namespace {

// CODATA 2018
constexpr double kPi = 3.14159265358979323846;
constexpr double kAlpha = 7.2973525693e-3;
constexpr double kLambdaBarC_um = 3.8615926796e-7;
constexpr double kC_um_per_fs = 0.299792458;

void set_err(qs_ctx *c, const char *msg) {
    if (c) std::snprintf(c->last_error, sizeof(c->last_error), "%s", msg);
}

qs_status hip_fail(qs_ctx *c, hipError_t e, const char *where) {
    if (c)
        std::snprintf(c->last_error, sizeof(c->last_error), "%s: %s", where, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? QS_ENOMEM : QS_EDEVICE;
}

// Device address of `scratch` on each device: looked up once per device, by
// the first qs_create on it, with that device current.  In host code the
// array's name is only a host-side stand-in; kernels get this address.
std::mutex g_scratch_mutex;
std::vector<unsigned char *> g_scratch_addr;

hipError_t scratch_address(int device, unsigned char **out) {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if ((size_t)device >= g_scratch_addr.size()) g_scratch_addr.resize((size_t)device + 1, nullptr);
    if (!g_scratch_addr[device]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_addr[device] = static_cast<unsigned char *>(ptr);
    }
    *out = g_scratch_addr[device];
    return hipSuccess;
}

class DeviceGuard {
   public:
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev_) != hipSuccess) prev_ = -1;
        if (prev_ != dev) (void)hipSetDevice(dev);
        dev_ = dev;
    }
    ~DeviceGuard() {
        if (prev_ >= 0 && prev_ != dev_) (void)hipSetDevice(prev_);
    }

   private:
    int prev_ = -1, dev_ = -1;
};

bool fin(double v) { return std::isfinite(v); }

// Peak over the focal plane of a transverse mode's amplitude (QS_MODE_*):
// HG m, n: max_s |H_m(s)| e^(-s^2/2) times the same for n (separable, s =
// sqrt2 x / W0); LG p, l: max_t t^(|l|/2) |L_p^|l|(t)| e^(-t/2), t = 2 rho^2 / W0^2.
// A scan at 1/4096 of the lobe scale, then golden-section search on the
// best bracket.
double hermite_fn(int m, double s) {
    double h0 = 1.0, h1 = 2.0 * s;
    if (m == 0) return std::exp(-0.5 * s * s);
    for (int k = 1; k < m; ++k) {
        const double h2 = 2.0 * s * h1 - 2.0 * k * h0;
        h0 = h1;
        h1 = h2;
    }
    return std::fabs(h1) * std::exp(-0.5 * s * s);
}

double laguerre_fn(int p, int l, double t) {
    double L0 = 1.0, L1 = 1.0 + l - t, Lp = p >= 1 ? L1 : L0;
    for (int k = 1; k < p; ++k) {
        const double L2 = ((2.0 * k + 1 + l - t) * L1 - (k + l) * L0) / (k + 1);
        L0 = L1;
        L1 = L2;
        Lp = L2;
    }
    return std::pow(t, 0.5 * l) * std::fabs(Lp) * std::exp(-0.5 * t);
}

template <class F>
double scan_max(F f, double hi) {
    const int n = 1 << 16;
    int best = 0;
    double fb = f(0.0);
    for (int k = 1; k <= n; ++k) {
        const double v = f(hi * k / n);
        if (v > fb) fb = v, best = k;
    }
    double a = hi * std::max(best - 1, 0) / n, b = hi * std::min(best + 1, n) / n;
    const double g = 0.5 * (std::sqrt(5.0) - 1.0);
    for (int it = 0; it < 100; ++it) {
        const double c = b - g * (b - a), d = a + g * (b - a);
        if (f(c) > f(d))
            b = d;
        else
            a = c;
    }
    return std::max(fb, f(0.5 * (a + b)));
}

double mode_peak(int mode, int m, int n) {
    if (mode == QS_MODE_HG) {
        auto peak1 = [](int k) {
            return scan_max([k](double s) { return hermite_fn(k, s); }, std::sqrt(2.0 * k + 1) + 4);
        };
        return peak1(m) * peak1(n);
    }
    if (mode == QS_MODE_LG) {
        const int l = std::abs(n);
        return scan_max([m, l](double t) { return laguerre_fn(m, l, t); }, 4.0 * m + 2.0 * l + 30);
    }
    return 1.0;
}

qs_status validate_shot(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_bins *H,
                        int64_t n_samples) {
    if (!L || !B || !H) return set_err(c, "null argument"), QS_EINVAL;
    const double vals[] = {L->a0, L->lambda_um, L->w0_um, L->tau_fs, L->x_off_um, L->y_off_um,
                           L->delay_fs, B->gamma0, B->sigma_gamma, B->sigma_r_um, B->sigma_z_um,
                           B->div_mrad, H->e_lo, H->e_hi, H->th_lo_mrad, H->th_hi_mrad};
    for (double v : vals)
        if (!fin(v)) return set_err(c, "non-finite parameter"), QS_EINVAL;
    if (!(L->a0 >= 0) || !(L->lambda_um > 0) || !(L->w0_um >= 0) || !(L->tau_fs > 0))
        return set_err(c, "laser parameter out of range"), QS_EINVAL;
    if (L->envelope != QS_ENV_GAUSS && L->envelope != QS_ENV_SIN2)
        return set_err(c, "unknown envelope"), QS_EINVAL;
    if (L->mode != QS_MODE_GAUSS && L->mode != QS_MODE_HG && L->mode != QS_MODE_LG)
        return set_err(c, "unknown transverse mode"), QS_EINVAL;
    if (L->mode == QS_MODE_HG && (L->mode_m < 0 || L->mode_m > 8 || L->mode_n < 0 || L->mode_n > 8))
        return set_err(c, "Hermite-Gauss orders must be in [0, 8]"), QS_EINVAL;
    if (L->mode == QS_MODE_LG && (L->mode_m < 0 || L->mode_m > 8 || L->mode_n < -8 || L->mode_n > 8))
        return set_err(c, "Laguerre-Gauss indices: p in [0, 8], l in [-8, 8]"), QS_EINVAL;
    if (!(B->gamma0 > 1) || !(B->sigma_gamma >= 0) || !(B->sigma_r_um >= 0) ||
        !(B->sigma_z_um >= 0) || !(B->div_mrad >= 0))
        return set_err(c, "beam parameter out of range"), QS_EINVAL;
    if ((B->transverse != QS_PROFILE_GAUSS && B->transverse != QS_PROFILE_FLAT) ||
        (B->longitudinal != QS_PROFILE_GAUSS && B->longitudinal != QS_PROFILE_FLAT))
        return set_err(c, "unknown beam profile"), QS_EINVAL;
    if (n_samples < 1 || n_samples > (int64_t)1 << 32)
        return set_err(c, "n_samples must be in [1, 2^32]"), QS_EINVAL;
    if (H->n_e < 1 || H->n_e > 4096 || H->n_th < 1 || H->n_th > 4096 || H->n_a < 1 ||
        H->n_a > 4096)
        return set_err(c, "bin counts must be in [1, 4096]"), QS_EINVAL;
    if (!(H->e_hi > H->e_lo) || !(H->th_hi_mrad > H->th_lo_mrad))
        return set_err(c, "histogram window must have hi > lo"), QS_EINVAL;
    return QS_OK;
}

qs_status validate_outputs(qs_ctx *c, const qs_outputs *O) {
    if (!O) return set_err(c, "null argument"), QS_EINVAL;
    if (!O->energy_hist || !O->angle_hist || !O->a0eff_hist || !O->moments || !O->status)
        return set_err(c, "null output pointer"), QS_EINVAL;
    if (O->samples && (O->sample_stride < 1 || O->n_sample_records < 0))
        return set_err(c, "sample records need stride >= 1"), QS_EINVAL;
    return QS_OK;
}

qs_status validate_outputs(qs_ctx *c, const qs_grad_outputs *O) {
    if (!O) return set_err(c, "null argument"), QS_EINVAL;
    if (!O->grad) return set_err(c, "null gradient pointer"), QS_EINVAL;
    if (!O->d_energy_hist && !O->d_angle_hist && !O->d_moments)
        return set_err(c, "no upstream weights"), QS_EINVAL;
    if (O->d_moments && !O->moments)
        return set_err(c, "d_moments needs the forward moments"), QS_EINVAL;
    return QS_OK;
}

qs_status validate_numerics(qs_ctx *c, const qs_numerics *N) {
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    const double vals[] = {N->window_fwhm, N->kernel_sigma_bins, N->chi_fp64, N->c_theta};
    for (double v : vals)
        if (!fin(v)) return set_err(c, "non-finite parameter"), QS_EINVAL;
    if (N->n_steps < 1 || N->n_steps > 65536)
        return set_err(c, "n_steps must be in [1, 65536]"), QS_EINVAL;
    if (N->shot < 0) return set_err(c, "shot must be >= 0"), QS_EINVAL;
    if (!(N->window_fwhm > 0) || !(N->kernel_sigma_bins >= 0) || !(N->c_theta >= 0))
        return set_err(c, "numerics parameter out of range"), QS_EINVAL;
    if (N->rr_model != QS_RR_CLASSICAL && N->rr_model != QS_RR_QUANTUM)
        return set_err(c, "unknown rr_model"), QS_EINVAL;
    if (N->amp_mode != QS_AMP_A0EFF && N->amp_mode != QS_AMP_LOCAL)
        return set_err(c, "unknown amp_mode"), QS_EINVAL;
    if (N->deposit < QS_DEP_POINT || N->deposit > QS_DEP_GAUSS)
        return set_err(c, "unknown deposit"), QS_EINVAL;
    if (N->precision != QS_PREC_FP32 && N->precision != QS_PREC_FP64)
        return set_err(c, "unknown precision"), QS_EINVAL;
    if ((N->flags & ~QS_VALIDATE_FP64) != 0) return set_err(c, "unknown flags"), QS_EINVAL;
    if (N->shadow_stride < 0 || N->shadow_stride > (1 << 20))
        return set_err(c, "shadow_stride must be in [0, 2^20]"), QS_EINVAL;
    return QS_OK;
}

template <class T>
qs_status grow(qs_ctx *c, T **p, size_t *cap, size_t n, const char *what) {
    if (*cap >= n) return QS_OK;
    if (*p) {
        // earlier work queued on any stream may still read the old buffer
        (void)hipDeviceSynchronize();
        (void)hipFree(*p);
    }
    *p = nullptr;
    *cap = 0;
    hipError_t e = hipMalloc(reinterpret_cast<void **>(p), n * sizeof(T));
    if (e != hipSuccess) return hip_fail(c, e, what);
    *cap = n;
    return QS_OK;
}

qs_status grow_pinned(qs_ctx *c, int slot, size_t n) {
    if (c->stage_cap[slot] >= n) return QS_OK;
    if (c->stage[slot]) {
        if (c->stage_pending[slot]) (void)hipEventSynchronize(c->stage_done[slot]);
        c->stage_pending[slot] = false;
        (void)hipHostFree(c->stage[slot]);
    }
    c->stage[slot] = nullptr;
    c->stage_cap[slot] = 0;
    hipError_t e =
        hipHostMalloc(reinterpret_cast<void **>(&c->stage[slot]), n, hipHostMallocDefault);
    if (e != hipSuccess) return hip_fail(c, e, "pinned staging");
    c->stage_cap[slot] = n;
    return QS_OK;
}

// A view pass of the FP64 shadow: every stride-th sample of each shot (the
// n_samples of the call are the view's); the FP64 view pass (report) writes
// the error report, its outputs sitting `span` doubles after the FP32 view's.
struct View {
    int32_t stride;
    int64_t span;
    bool report;
};

qs_status forward_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                       const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                       const qs_outputs *O, double *tape, hipStream_t s, bool noalloc = false);
qs_status backward_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                        const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                        const qs_grad_outputs *O, const double *tape, hipStream_t s,
                        const View *view = nullptr);
qs_status photons_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                       const int64_t *n_samples, const qs_numerics *N, const qs_photon_bins *PB,
                       const qs_photon_outputs *PO, hipStream_t s, const View *view = nullptr);
qs_status factor_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                      const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                      const qs_node_grid *G, const qs_outputs *O, hipStream_t s);
qs_status tune_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                    const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                    const char *path, qs_tuning *out, hipStream_t s);

}  // namespace

extern "C" {

int qs_abi_version(void) { return QS_ABI_VERSION; }

// SHA-256 of the sources and flags this library was built from, stamped by
// the build script.
#ifndef QS_BUILD_ID
#define QS_BUILD_ID "unknown"
#endif
const char *qs_build_id(void) { return QS_BUILD_ID; }

const char *qs_strerror(qs_status s) {
    switch (s) {
        case QS_OK: return "ok";
        case QS_EINVAL: return "invalid argument";
        case QS_ENOMEM: return "out of device memory";
        case QS_EDEVICE: return "HIP runtime error";
        case QS_ENONFINITE: return "non-finite sample state";
        case QS_EUNSUPPORTED: return "unsupported";
        case QS_ERANGE: return "chi beyond the tabulated range";
    }
    return "unknown status";
}

const char *qs_last_error(qs_ctx *ctx) { return ctx ? ctx->last_error : ""; }

qs_status qs_create(qs_ctx **out, int device) {
    if (!out) return QS_EINVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return QS_EINVAL;
    qs_ctx *c = new (std::nothrow) qs_ctx;
    if (!c) return QS_ENOMEM;
    c->device = device;
    DeviceGuard g(device);
    hipError_t e;
    double *work = nullptr;
    const size_t wd = std::max(qs::radiation_work_doubles(), qs::photon_work_doubles());
    if ((e = hipMalloc(&c->rad32, sizeof(float) * qs::kCells32 * qs::kCellVals)) != hipSuccess ||
        (e = hipMalloc(&c->rad64, sizeof(double) * qs::kCells64 * qs::kCellVals)) != hipSuccess ||
        (e = hipMalloc(&c->rad32d, sizeof(float) * qs::kCells32 * 4 * qs::kDerivFuncs)) !=
            hipSuccess ||
        (e = hipMalloc(&c->rad64d, sizeof(double) * qs::kCells64 * 4 * qs::kDerivFuncs)) !=
            hipSuccess ||
        (e = hipMalloc(&c->phtab, qs::kPhTabBytes)) !=
            hipSuccess ||
        (e = hipMalloc(&c->eval_flags, sizeof(int))) != hipSuccess ||
        (e = hipMalloc(&work, sizeof(double) * wd)) != hipSuccess ||
        (e = hipMemset(c->eval_flags, 0, sizeof(int))) != hipSuccess) {
        qs_status st = hip_fail(c, e, "qs_create allocation");
        if (work) (void)hipFree(work);
        qs_destroy(c);
        return st;
    }
    e = qs::build_radiation_tables(c->rad32, c->rad64, c->rad32d, c->rad64d, work, wd, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = qs::build_photon_table(c->phtab, work, wd, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    (void)hipFree(work);
    if (e != hipSuccess) {
        qs_status st = hip_fail(c, e, "radiation tables");
        qs_destroy(c);
        return st;
    }
    // this device's scratch address (qs_forward_noalloc), the status words' block
    if ((e = scratch_address(device, &c->na_scratch)) != hipSuccess ||
        (e = hipHostMalloc(reinterpret_cast<void **>(&c->status_host),
                           kStatusWords * sizeof(int32_t), hipHostMallocDefault)) != hipSuccess) {
        qs_status st = hip_fail(c, e, "scratch set-up");
        qs_destroy(c);
        return st;
    }
    *out = c;
    return QS_OK;
}

void qs_destroy(qs_ctx *c) {
    if (!c) return;
    {
        DeviceGuard g(c->device);
        (void)hipDeviceSynchronize();
        (void)hipFree(c->rad32);
        (void)hipFree(c->rad64);
        (void)hipFree(c->rad32d);
        (void)hipFree(c->rad64d);
        (void)hipFree(c->phtab);
        (void)hipFree(c->env32);
        (void)hipFree(c->env64);
        (void)hipFree(c->accum);
        (void)hipFree(c->partials);
        (void)hipFree(c->shadow);
        (void)hipFree(c->states);
        (void)hipFree(c->order);
        (void)hipFree(c->shot_tab);
        for (int k = 0; k < kStageSlots; ++k) {
            if (c->stage[k]) (void)hipHostFree(c->stage[k]);
            if (c->stage_done[k]) (void)hipEventDestroy(c->stage_done[k]);
        }
        if (c->status_host) (void)hipHostFree(c->status_host);
        (void)hipFree(c->eval_flags);
        for (auto &set : c->ev)
            for (hipEvent_t &e : set)
                if (e) (void)hipEventDestroy(e);
        for (GraphEntry &g : c->graph_cache) {
            if (g.exec) (void)hipGraphExecDestroy(g.exec);
            if (g.graph) (void)hipGraphDestroy(g.graph);
        }
        if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    }
    delete c;
}

qs_status qs_forward(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_numerics *N,
                     const qs_bins *H, const qs_outputs *O, void *stream) {
    if (!c) return QS_EINVAL;
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return forward_impl(c, 1, L, B, &n, N, H, O, nullptr, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_forward_noalloc(qs_ctx *c, const qs_laser *L, const qs_beam *B,
                             const qs_numerics *N, const qs_bins *H, const qs_outputs *O,
                             void *stream) {
    if (!c) return QS_EINVAL;
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    if (N->n_samples > (int64_t)QS_NOALLOC_MAX_SAMPLES)
        return set_err(c, "qs_forward_noalloc: n_samples above QS_NOALLOC_MAX_SAMPLES"),
               QS_EINVAL;
    if (N->flags & QS_VALIDATE_FP64)
        return set_err(c, "qs_forward_noalloc: no FP64 shadow (QS_VALIDATE_FP64)"),
               QS_EUNSUPPORTED;
    const int64_t n = N->n_samples;
    return forward_impl(c, 1, L, B, &n, N, H, O, nullptr, reinterpret_cast<hipStream_t>(stream),
                        true);
}

qs_status qs_forward_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                             const qs_beam *beams, const int64_t *n_samples,
                             const qs_numerics *num, const qs_bins *bins, const qs_outputs *outs,
                             void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins || !outs)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return forward_impl(c, n_shots, lasers, beams, n_samples, num, bins, outs, nullptr,
                        reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_forward_factorised(qs_ctx *c, const qs_laser *L, const qs_beam *B,
                                const qs_numerics *N, const qs_bins *H, const qs_node_grid *G,
                                const qs_outputs *O, void *stream) {
    if (!c) return QS_EINVAL;
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return factor_impl(c, 1, L, B, &n, N, H, G, O, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_forward_factorised_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                                        const qs_beam *beams, const int64_t *n_samples,
                                        const qs_numerics *num, const qs_bins *bins,
                                        const qs_node_grid *grids, const qs_outputs *outs,
                                        void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins ||
        !grids || !outs)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return factor_impl(c, n_shots, lasers, beams, n_samples, num, bins, grids, outs,
                       reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_radiation_eval(qs_ctx *c, int32_t precision, int64_t n, const double *chi,
                            double *out, void *stream) {
    if (!c) return QS_EINVAL;
    if (n < 0 || (n > 0 && (!chi || !out)) ||
        (precision != QS_PREC_FP32 && precision != QS_PREC_FP64))
        return set_err(c, "invalid radiation_eval arguments"), QS_EINVAL;
    DeviceGuard guard(c->device);
    hipError_t e = qs::launch_radiation_eval(c->rad32, c->rad64, precision, n, chi, out,
                                             c->eval_flags, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(c, e, "radiation_eval kernel");
    return QS_OK;
}

qs_status qs_backward(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_numerics *N,
                      const qs_bins *H, const qs_grad_outputs *O, void *stream) {
    if (!c) return QS_EINVAL;
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return backward_impl(c, 1, L, B, &n, N, H, O, nullptr, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_backward_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                              const qs_beam *beams, const int64_t *n_samples,
                              const qs_numerics *num, const qs_bins *bins,
                              const qs_grad_outputs *outs, void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins || !outs)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return backward_impl(c, n_shots, lasers, beams, n_samples, num, bins, outs, nullptr,
                         reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_forward_tape(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_numerics *N,
                          const qs_bins *H, const qs_outputs *O, double *tape, void *stream) {
    if (!c) return QS_EINVAL;
    if (!N || !tape) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return forward_impl(c, 1, L, B, &n, N, H, O, tape, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_forward_tape_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                                  const qs_beam *beams, const int64_t *n_samples,
                                  const qs_numerics *num, const qs_bins *bins,
                                  const qs_outputs *outs, double *tape, void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins || !outs ||
        !tape)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return forward_impl(c, n_shots, lasers, beams, n_samples, num, bins, outs, tape,
                        reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_backward_tape(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_numerics *N,
                           const qs_bins *H, const qs_grad_outputs *O, const double *tape,
                           void *stream) {
    if (!c) return QS_EINVAL;
    if (!N || !tape) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return backward_impl(c, 1, L, B, &n, N, H, O, tape, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_backward_tape_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                                   const qs_beam *beams, const int64_t *n_samples,
                                   const qs_numerics *num, const qs_bins *bins,
                                   const qs_grad_outputs *outs, const double *tape,
                                   void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins || !outs ||
        !tape)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return backward_impl(c, n_shots, lasers, beams, n_samples, num, bins, outs, tape,
                         reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_photons(qs_ctx *c, const qs_laser *L, const qs_beam *B, const qs_numerics *N,
                     const qs_photon_bins *PB, const qs_photon_outputs *PO, void *stream) {
    if (!c) return QS_EINVAL;
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    const int64_t n = N->n_samples;
    return photons_impl(c, 1, L, B, &n, N, PB, PO, reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_photons_batched(qs_ctx *c, int32_t n_shots, const qs_laser *lasers,
                             const qs_beam *beams, const int64_t *n_samples,
                             const qs_numerics *num, const qs_photon_bins *bins,
                             const qs_photon_outputs *outs, void *stream) {
    if (!c) return QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20) || !lasers || !beams || !n_samples || !bins || !outs)
        return set_err(c, "invalid batch arguments"), QS_EINVAL;
    return photons_impl(c, n_shots, lasers, beams, n_samples, num, bins, outs,
                        reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_photon_cdf(qs_ctx *c, int64_t n, const double *chi, const double *xi, double *out,
                        void *stream) {
    if (!c) return QS_EINVAL;
    if (n < 0 || (n > 0 && (!chi || !xi || !out)))
        return set_err(c, "invalid photon_cdf arguments"), QS_EINVAL;
    DeviceGuard guard(c->device);
    hipError_t e = qs::launch_photon_cdf(c->phtab, n, chi, xi, out,
                                         reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(c, e, "photon_cdf kernel");
    return QS_OK;
}

qs_status qs_radiation_derivs(qs_ctx *c, int32_t precision, int64_t n, const double *chi,
                              double *out, void *stream) {
    if (!c) return QS_EINVAL;
    if (n < 0 || (n > 0 && (!chi || !out)) ||
        (precision != QS_PREC_FP32 && precision != QS_PREC_FP64))
        return set_err(c, "invalid radiation_derivs arguments"), QS_EINVAL;
    DeviceGuard guard(c->device);
    hipError_t e = qs::launch_radiation_derivs(c->rad32d, c->rad64d, precision, n, chi, out,
                                               c->eval_flags,
                                               reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(c, e, "radiation_derivs kernel");
    return QS_OK;
}

qs_status qs_tune(qs_ctx *c, int32_t n_shots, const qs_laser *lasers, const qs_beam *beams,
                  const int64_t *n_samples, const qs_numerics *N, const qs_bins *bins,
                  const char *cache_path, qs_tuning *out, void *stream) {
    if (!c || !lasers || !beams || !n_samples || !N || !bins)
        return set_err(c, "null argument"), QS_EINVAL;
    if (n_shots < 1 || n_shots > (1 << 20)) return set_err(c, "n_shots out of range"), QS_EINVAL;
    DeviceGuard guard(c->device);
    return tune_impl(c, n_shots, lasers, beams, n_samples, N, bins, cache_path, out,
                     reinterpret_cast<hipStream_t>(stream));
}

qs_status qs_set_graphs(qs_ctx *c, int on) {
    if (!c) return QS_EINVAL;
    c->graphs = on != 0;
    return QS_OK;
}

qs_status qs_set_profiling(qs_ctx *c, int on) {
    if (!c) return QS_EINVAL;
    DeviceGuard guard(c->device);
    if (on && !c->ev[kTimingRing - 1][5]) {
        for (auto &set : c->ev)
            for (hipEvent_t &ev : set) {
                if (ev) continue;
                hipError_t e = hipEventCreate(&ev);
                if (e != hipSuccess) return hip_fail(c, e, "event create");
            }
    }
    c->profiling = on != 0;
    c->profiled_call = false;
    c->ev_count = 0;
    return QS_OK;
}

// a profiled call has been enqueued into the set c->ev[c->ev_next]
static void advance_timing_ring(qs_ctx *c) {
    c->ev_last = c->ev_next;
    c->ev_next = (c->ev_next + 1) % kTimingRing;
    c->ev_count = std::min(c->ev_count + 1, kTimingRing);
}

// kernel durations of one event set, after its last event
static qs_status read_timing_set(qs_ctx *c, int set, double *ms) {
    hipError_t e = hipEventSynchronize(c->ev[set][5]);
    if (e != hipSuccess) return hip_fail(c, e, "event synchronize");
    for (int k = 0; k < 5; ++k) {
        float t = 0.0f;
        e = hipEventElapsedTime(&t, c->ev[set][k], c->ev[set][k + 1]);
        if (e != hipSuccess) return hip_fail(c, e, "event elapsed");
        ms[k] = t;
    }
    return QS_OK;
}

qs_status qs_last_timings(qs_ctx *c, double *ms) {
    if (!c || !ms) return QS_EINVAL;
    if (!c->profiling || !c->profiled_call)
        return set_err(c, "no profiled call"), QS_EINVAL;
    DeviceGuard guard(c->device);
    return read_timing_set(c, c->ev_last, ms);
}

qs_status qs_timings_sum(qs_ctx *c, int32_t *n_calls, double *ms) {
    if (!c || !n_calls || !ms) return QS_EINVAL;
    if (!c->profiling || c->ev_count == 0)
        return set_err(c, "no profiled call"), QS_EINVAL;
    DeviceGuard guard(c->device);
    for (int k = 0; k < 5; ++k) ms[k] = 0.0;
    for (int i = 0; i < c->ev_count; ++i) {
        const int set = (c->ev_last - i + kTimingRing) % kTimingRing;
        double one[5];
        const qs_status st = read_timing_set(c, set, one);
        if (st != QS_OK) return st;
        for (int k = 0; k < 5; ++k) ms[k] += one[k];
    }
    *n_calls = c->ev_count;
    return QS_OK;
}

qs_status qs_sync_status(qs_ctx *c, const int32_t *status, void *stream) {
    if (!c || !status) return QS_EINVAL;
    DeviceGuard guard(c->device);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // the word follows the stream's work into pinned memory, one wait for both
    // (the wait and a blocking copy after it: 21 us on an idle stream, now 12)
    uint32_t used = c->status_used.load(), bit = 0;
    do {
        bit = ~used & (used + 1);  // the lowest free word
    } while (bit && !c->status_used.compare_exchange_weak(used, used | bit));
    if (bit) {
        int32_t *w = c->status_host + __builtin_ctz(bit);
        const hipError_t copied = hipMemcpyAsync(w, status, sizeof(*w), hipMemcpyDeviceToHost, s);
        const hipError_t e = hipStreamSynchronize(s);
        const int32_t v = *w;
        c->status_used.fetch_and(~bit);
        if (e != hipSuccess) return hip_fail(c, e, "stream synchronize");
        if (copied == hipSuccess) return (qs_status)v;
    }
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(c, e, "stream synchronize");
    int32_t v = 0;
    e = hipMemcpy(&v, status, sizeof(v), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(c, e, "status copy");
    return (qs_status)v;
}

}  // extern "C"

namespace {

// Shared set-up of a batch: validation of the shots, the constants of the
// shared phase grid (Sec. 2 eq. a0eff, Sec. 4 eq. dpdtRR) and the per-shot
// table, built on the host as [ShotParams x n][OutT x n].
struct Batch {
    qs::BatchParams bp{};
    double psi_max = 0, h = 0, omega_tau = 0;
    int prec = qs::PREC_F32;
    int max_nh = 0;       // largest histogram word count of a shot
    int64_t total = 0;    // samples over all shots
    int64_t hist_words = 0;
    Batch() = default;
    Batch(const Batch &) = delete;  // (stage may point into it)
    size_t tab_bytes = 0;
    bool direct = false;             // the shot table goes with the set-up kernel
    qs::SetupTab small{};            // direct: the table
    unsigned char *stage = nullptr;  // the table: `small` or a pinned staging buffer
    int slot = 0;                    // its block in the context's ring (not direct)
    qs::ShotParams *sp = nullptr;   // in the table
    unsigned char *outs = nullptr;  // in the table, after the ShotParams
};

int ilog2(int64_t v) {
    int r = 0;
    while (v > 1) {
        v >>= 1;
        ++r;
    }
    return r;
}

TuneKey tune_key(const qs_numerics *N, int prec, int hist_words, int64_t total, int32_t n_shots) {
    TuneKey k;
    std::memset(&k, 0, sizeof(k));
    k.n_steps = N->n_steps;
    k.rr = N->rr_model;
    k.amp = N->amp_mode;
    k.dep = N->deposit;
    k.prec = prec;
    k.hist_words = hist_words;
    k.lg_total = ilog2(total);
    k.lg_shots = ilog2(n_shots);
    return k;
}

const TuneEntry *find_tune(const qs_ctx *c, const TuneKey &k) {
    if (c->tune_forced) return &c->forced;
    for (const TuneEntry &t : c->tunes)
        if (t.key == k) return &t;
    return nullptr;
}

// The deposit work item of launches without a tuned choice or tuned to kDepTile:
// 1024 samples, and for small launches as few as leave about 512 items, so that
// they spread over the device (256 CUs).  Measured on focused laws, items of 256 / 512 / 1024 /
// 4096 samples: 5003 samples 39 / 68 / 120 / 441 us, 50,001 51 / 71 / 121 / 445 us,
// 2^18 123 / 104 / 132 / 443 us, 2^20 364 / 260 / 215 / 449 us, 2^22 1329 / 772 /
// 592 / 684 us, 128 shots of 2^12 .. 2^18 1205 / 1129 / 1175 / 1439 us, 1500 shots
// 14.0 / 12.5 / 12.0 / 12.1 ms.
int default_dep_tile(int64_t total) {
    int tile = qs::kDepTile;
    while (tile > qs::kMomRow && total / tile < qs::kDepItems) tile >>= 1;
    return tile;
}

qs_status prepare_batch(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                        const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                        size_t out_size, Batch &b, bool noalloc = false,
                        int32_t draw_stride = 1) {
    qs_status st = validate_numerics(c, N);
    if (st != QS_OK) return st;
    for (int k = 0; k < n_shots; ++k) {
        if ((st = validate_shot(c, &L[k], &B[k], &H[k], n_samples[k])) != QS_OK) return st;
        if (L[k].lambda_um != L[0].lambda_um || L[k].tau_fs != L[0].tau_fs ||
            L[k].envelope != L[0].envelope)
            return set_err(c, "the shots of a batch must share wavelength, duration and envelope"),
                   QS_EUNSUPPORTED;
        b.max_nh = std::max(b.max_nh, H[k].n_e + 2 + H[k].n_th + 2 + H[k].n_a);
        b.total += n_samples[k];
        if (b.total > ((int64_t)1 << 36))
            return set_err(c, "a batch holds at most 2^36 samples"), QS_EINVAL;
    }

    // ---- shared constants ----
    const qs_laser &L0 = L[0];
    const double omega0 = 2.0 * kPi * kC_um_per_fs / L0.lambda_um;  // rad / fs
    const double aS = L0.lambda_um / (2.0 * kPi * kLambdaBarC_um);
    b.omega_tau = omega0 * L0.tau_fs;
    b.psi_max = L0.envelope == QS_ENV_GAUSS ? N->window_fwhm * b.omega_tau : b.omega_tau;
    b.h = 2.0 * b.psi_max / (double)N->n_steps;
    if (N->precision == QS_PREC_FP64)
        b.prec = qs::PREC_F64;
    else if (N->rr_model == QS_RR_QUANTUM && N->chi_fp64 > 0)
        b.prec = qs::PREC_F32MIX;

    qs::BatchParams &bp = b.bp;
    bp.ell_per_psi = L0.lambda_um / (4.0 * kPi);
    bp.two_over_aS = 2.0 / aS;
    bp.K = 4.0 * kAlpha / (3.0 * aS);
    bp.CD = 55.0 / (6.0 * std::sqrt(3.0)) * kAlpha / (aS * aS);
    bp.psi_max = b.psi_max;
    bp.h = b.h;
    bp.ellf = (float)bp.ell_per_psi;
    bp.two_over_aSf = (float)bp.two_over_aS;
    bp.Kf = (float)bp.K;
    bp.CDf = (float)bp.CD;
    bp.psi0f = (float)(-b.psi_max);
    bp.hf = (float)b.h;
    bp.chi_fp64 = (float)N->chi_fp64;
    bp.n_steps = N->n_steps;
    bp.n_shots = n_shots;
    bp.deposit = N->deposit;
    bp.quantum = N->rr_model == QS_RR_QUANTUM;
    bp.key0 = (uint32_t)N->seed;
    bp.key1 = (uint32_t)(N->seed >> 32);
    bp.ksig_bins = N->kernel_sigma_bins;
    bp.c_theta = N->c_theta;
    // launch choices of this launch class (qs_tune), else the defaults
    const TuneEntry *tune = find_tune(c, tune_key(N, b.prec, b.max_nh, b.total, n_shots));
    bp.dep_tile = tune && tune->dep_tile != qs::kDepTile ? tune->dep_tile : default_dep_tile(b.total);
    bp.mom_row = bp.dep_tile < qs::kMomTile ? qs::kMomRow : qs::kMomTile;
    bp.phase_cap = tune ? tune->phase_cap : 0;
    bp.dep_cap = tune ? tune->dep_cap : 0;

    // ---- per-shot table ----
    b.tab_bytes = ((sizeof(qs::ShotParams) + out_size) * n_shots + 255) / 256 * 256;
    unsigned char *stage = nullptr;
    // small tables go to the device by value with the set-up kernel (one shot; the
    // launches of a graph take theirs from the copy before each replay)
    static_assert(na::kTabBytes <= sizeof(qs::SetupTab), "one shot's table");
    b.direct = b.tab_bytes <= sizeof(qs::SetupTab) && (noalloc || !c->graphs);
    if (b.direct) {
        stage = reinterpret_cast<unsigned char *>(b.small.w);
    } else {
        const int slot = c->stage_next;
        if (c->stage_pending[slot]) {
            // the copy out of this block, kStageSlots calls ago
            hipError_t e = hipEventSynchronize(c->stage_done[slot]);
            if (e != hipSuccess) return hip_fail(c, e, "staging event");
            c->stage_pending[slot] = false;
        }
        if ((st = grow_pinned(c, slot, b.tab_bytes)) != QS_OK) return st;
        stage = c->stage[slot];
        b.slot = slot;
    }
    b.stage = stage;
    b.sp = reinterpret_cast<qs::ShotParams *>(stage);
    b.outs = stage + sizeof(qs::ShotParams) * n_shots;
    int64_t item = 0, ditem = 0, mtile = 0, gitem = 0, off = 0, hoff = 0;
    for (int k = 0; k < n_shots; ++k) {
        const qs_laser &l = L[k];
        const qs_beam &bm = B[k];
        const qs_bins &hb = H[k];
        qs::ShotParams &p = b.sp[k];
        p = qs::ShotParams{};
        const bool plane_wave = l.w0_um == 0.0;
        p.a0 = l.a0;
        p.inv_w0sq = plane_wave ? 0.0 : 1.0 / (l.w0_um * l.w0_um);
        p.inv_zR = plane_wave ? 0.0 : l.lambda_um / (kPi * l.w0_um * l.w0_um);
        // a focus so small that these overflow has no spatial factor (0 times them
        // is no number, which the FP64 factor's clamps would take for 0): an
        // amplitude that is none either, so that every sample is reported
        if (!std::isfinite(p.inv_w0sq) || !std::isfinite(p.inv_zR))
            p.a0 = std::numeric_limits<double>::quiet_NaN();
        p.x_off = l.x_off_um;
        p.y_off = l.y_off_um;
        p.z_delay = 0.5 * kC_um_per_fs * l.delay_fs;
        p.gamma0 = bm.gamma0;
        p.sigma_gamma = bm.sigma_gamma;
        p.sigma_r = bm.sigma_r_um;
        p.sigma_z = bm.sigma_z_um;
        p.profile = (bm.transverse == QS_PROFILE_FLAT ? qs::kFlatR : 0) |
                    (bm.longitudinal == QS_PROFILE_FLAT ? qs::kFlatZ : 0);
        p.div_rad = 1e-3 * bm.div_mrad;
        p.a0f = (float)p.a0;
        p.inv_w0sqf = (float)p.inv_w0sq;
        p.inv_zRf = (float)p.inv_zR;
        p.plane_wave = plane_wave ? 1 : 0;
        {
            // the quadratic midpoint of the spatial factor is used only when one
            // phase step moves a sample much less than the focal scales: its
            // error is S''' d^3 / 16 for a step of length d, and the third
            // derivative of the Gaussian focus's factor along the axis is at
            // most about 135 / zR^3 of its peak, so below 3e-3 of the scale the
            // midpoint amplitude is within 2.3e-7 of the peak (about four FP32
            // roundings of it, a few 1e-7 of the energy loss at most)
            const double step_um = b.h * bp.ell_per_psi;
            // (a mode of order k varies on W0 / sqrt(1 + k))
            const int order = l.mode == QS_MODE_HG   ? std::max(l.mode_m, l.mode_n)
                              : l.mode == QS_MODE_LG ? 2 * l.mode_m + std::abs(l.mode_n)
                                                     : 0;
            const double scale = plane_wave ? 0.0
                                            : std::fmax(p.inv_zR, 6.0 * p.div_rad / l.w0_um) *
                                                  std::sqrt(1.0 + order);
            p.mid_interp = step_um * scale < 3e-3 ? 1 : 0;
        }
        p.mode = plane_wave ? QS_MODE_GAUSS : l.mode;
        p.mode_m = l.mode_m;
        p.mode_n = l.mode_n;
        p.mode_inv_norm = p.mode == QS_MODE_GAUSS ? 1.0 : 1.0 / mode_peak(l.mode, l.mode_m, l.mode_n);
        p.mode_inv_normf = (float)p.mode_inv_norm;
        if (p.mode != QS_MODE_GAUSS) bp.any_mode = 1;
        p.shot_word = N->shot + k;
        p.draw_stride = draw_stride;
        p.n_samples = n_samples[k];
        p.state_off = off;
        p.item0 = item;
        p.ditem0 = ditem;
        p.mtile0 = mtile;
        p.gitem0 = gitem;
        p.hist_off = hoff;
        p.n_e = hb.n_e;
        p.n_th = hb.n_th;
        p.n_a = hb.n_a;
        p.e_lo = hb.e_lo;
        p.e_w = (hb.e_hi - hb.e_lo) / hb.n_e;
        p.th_lo = hb.th_lo_mrad;
        p.th_w = (hb.th_hi_mrad - hb.th_lo_mrad) / hb.n_th;
        off += n_samples[k];
        item += (n_samples[k] + qs::kPhaseBlock - 1) / qs::kPhaseBlock;
        ditem += (n_samples[k] + bp.dep_tile - 1) / bp.dep_tile;
        mtile += (n_samples[k] + bp.mom_row - 1) / bp.mom_row;
        gitem += (n_samples[k] + qs::kChiGroup - 1) / qs::kChiGroup;
        hoff += hb.n_e + 2 + hb.n_th + 2 + hb.n_a;
    }
    bp.n_items = item;
    bp.n_ditems = ditem;
    bp.n_mtiles = mtile;
    bp.n_gitems = gitem;
    bp.prec = b.prec;
    b.hist_words = hoff;
    return QS_OK;
}

// Copy the staged shot table to the device and record the staging event (unless
// the set-up kernel takes it along).
qs_status upload_batch(qs_ctx *c, const Batch &b, hipStream_t s) {
    if (b.direct) return QS_OK;
    const int slot = b.slot;
    if (!c->stage_done[slot]) {
        hipError_t e = hipEventCreateWithFlags(&c->stage_done[slot], hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(c, e, "event create");
    }
    hipError_t e = hipMemcpyAsync(c->shot_tab, b.stage, b.tab_bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(c, e, "shot table copy");
    if ((e = hipEventRecord(c->stage_done[slot], s)) != hipSuccess)
        return hip_fail(c, e, "event record");
    c->stage_pending[slot] = true;
    c->stage_next = (slot + 1) % kStageSlots;
    return QS_OK;
}

// First device work of a call: the shot table (by value, or copied before this),
// the envelope table, the clear of the accumulators.
hipError_t launch_setup(const Batch &b, const qs_numerics *N, int envelope,
                        unsigned char *shot_tab, unsigned long long *accum, size_t words,
                        float *env32, double *env64, hipStream_t s) {
    return qs::launch_setup(b.direct ? &b.small : nullptr, b.direct ? b.tab_bytes : 0, shot_tab,
                            accum, words, b.psi_max, b.h, N->n_steps, envelope, b.omega_tau, env32,
                            env64, s);
}

qs_status forward_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                       const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                       const qs_outputs *O, double *tape, hipStream_t s, bool noalloc) {
    qs_status st;
    for (int k = 0; k < n_shots; ++k)
        if ((st = validate_outputs(c, &O[k])) != QS_OK) return st;
    if (tape && L)
        for (int k = 0; k < n_shots; ++k)
            if (L[k].mode != QS_MODE_GAUSS)
                return set_err(c, "derivatives are for the Gaussian mode only"), QS_EUNSUPPORTED;
    // FP64 shadow of an FP32 pass: a second view of the shot table (after the
    // outputs) integrates every shadow_stride-th sample in FP64
    const bool shadow = N && (N->flags & QS_VALIDATE_FP64) && N->precision == QS_PREC_FP32 &&
                        !tape;
    Batch b;
    if ((st = prepare_batch(c, n_shots, L, B, n_samples, N, H,
                            sizeof(qs::ShotOut) + (shadow ? sizeof(qs::ShotParams) : 0), b,
                            noalloc)) != QS_OK)
        return st;
    if (qs::deposit_lds_bytes(b.max_nh) > 160 * 1024)
        return set_err(c, "histograms exceed the LDS budget"), QS_EINVAL;
    DeviceGuard guard(c->device);
    qs::BatchParams &bp = b.bp;
    qs::ShotOut *so = reinterpret_cast<qs::ShotOut *>(b.outs);
    qs::ShotParams *sv = reinterpret_cast<qs::ShotParams *>(b.outs + sizeof(qs::ShotOut) * n_shots);
    static_assert(qs::kMoments == QS_M_N, "moment count");
    int64_t sh_total = 0, sh_items = 0, shd_words = 0;
    if (shadow) {
        const int stride = N->shadow_stride > 0 ? N->shadow_stride : 64;
        for (int k = 0; k < n_shots; ++k) {
            qs::ShotParams &p = b.sp[k];
            const int64_t ns = (n_samples[k] + stride - 1) / stride;
            p.shadow_stride = stride;
            p.shadow_off = sh_total;
            p.shd_off = shd_words;
            shd_words += (int64_t)H[k].n_e + 2 + H[k].n_th + 2;
            sv[k] = p;
            sv[k].draw_stride = stride;
            sv[k].n_samples = ns;
            sv[k].src_off = p.state_off;
            sv[k].state_off = sh_total;
            sv[k].item0 = sh_items;
            sh_total += ns;
            sh_items += (ns + qs::kPhaseBlock - 1) / qs::kPhaseBlock;
        }
    }
    for (int k = 0; k < n_shots; ++k) {
        const qs_outputs &o = O[k];
        so[k] = qs::ShotOut{};
        so[k].energy_hist = o.energy_hist;
        so[k].angle_hist = o.angle_hist;
        so[k].a0eff_hist = o.a0eff_hist;
        so[k].moments = o.moments;
        so[k].status = o.status;
        so[k].samples = o.samples;
        so[k].rec_stride = o.samples ? o.sample_stride : 1;
        so[k].rec_n = o.samples ? o.n_sample_records : 0;
    }

    // ---- device scratch ----
    const size_t nenv = (size_t)2 * N->n_steps + 1;
    const size_t arr = ((size_t)b.total * 8 + 255) / 256 * 256;
    const size_t arrf = ((size_t)b.total * 4 + 255) / 256 * 256;
    const size_t sarr = ((size_t)sh_total * 8 + 255) / 256 * 256;
    const size_t sarrf = ((size_t)sh_total * 4 + 255) / 256 * 256;
    const size_t flag_words = ((size_t)n_shots + 1) / 2;
    // work counters (phase, deposit, shadow phase, unused), flags, histograms,
    // FP64-shadow law differences, FP64 wave-steps per shot (forward passes)
    const size_t count_words = tape ? 0 : (size_t)n_shots;
    const size_t accum_words =
        2 + flag_words + (size_t)b.hist_words + (size_t)shd_words + count_words;
    float *env32 = nullptr;
    double *env64 = nullptr;
    unsigned long long *accum = nullptr;
    double *partials = nullptr;
    uint16_t *order = nullptr;
    unsigned char *states = nullptr, *shot_tab = nullptr;
    // samples in chi order: with FP64 steps where chi is high the wavefronts
    // step alike; in FP64 passes (the same results in any order) their lanes
    // read fewer distinct table cells, which pays from two wavefronts a SIMD
    // on (2^20 samples x 512 steps 6.2 -> 4.9 ms, 200,001 x 1024 3.2 -> 2.9 ms,
    // 5000 x 512 0.56 -> 0.61 ms)
    const bool ordered =
        b.prec == qs::PREC_F32MIX ||
        (b.prec == qs::PREC_F64 && N->rr_model == QS_RR_QUANTUM && !tape && b.total > 65536);
    if (noalloc) {
        // one shot, no shadow, no tape: every part fits its slot of `scratch`
        // (the sizes were validated; these checks keep the carve honest)
        if (n_shots != 1 || shadow || tape || (size_t)b.total > na::kSamples ||
            nenv > na::kEnvPoints || accum_words > na::kAccumWords ||
            (size_t)bp.n_mtiles * qs::kPartials > na::kPartWords || b.tab_bytes > na::kTabBytes ||
            arr > na::kArr || arrf > na::kArrf)
            return set_err(c, "qs_forward_noalloc: the call exceeds the static scratch"), QS_EINVAL;
        unsigned char *base = c->na_scratch;
        env64 = reinterpret_cast<double *>(base + na::kEnv64Off);
        env32 = reinterpret_cast<float *>(base + na::kEnv32Off);
        accum = reinterpret_cast<unsigned long long *>(base + na::kAccumOff);
        partials = reinterpret_cast<double *>(base + na::kPartOff);
        order = reinterpret_cast<uint16_t *>(base + na::kOrderOff);
        states = base + na::kStatesOff;
        shot_tab = base + na::kTabOff;
    } else {
        if ((st = grow(c, &c->env32, &c->env32_cap, nenv, "envelope table")) != QS_OK) return st;
        if ((st = grow(c, &c->env64, &c->env64_cap, nenv, "envelope table")) != QS_OK) return st;
        if ((st = grow(c, &c->accum, &c->accum_cap, accum_words, "accumulators")) != QS_OK)
            return st;
        if ((st = grow(c, &c->partials, &c->part_cap, (size_t)bp.n_mtiles * qs::kPartials,
                       "moment partials")) != QS_OK)
            return st;
        if ((st = grow(c, &c->states, &c->states_cap, 6 * arr + arrf + 6 * sarr + sarrf,
                       "sample states")) != QS_OK)
            return st;
        if (ordered && (st = grow(c, &c->order, &c->order_cap, (size_t)b.total, "chi order")) != QS_OK)
            return st;
        if ((st = grow(c, &c->shot_tab, &c->shot_tab_cap, b.tab_bytes, "shot table")) != QS_OK)
            return st;
        order = c->order;
        env32 = c->env32;
        env64 = c->env64;
        accum = c->accum;
        partials = c->partials;
        states = c->states;
        shot_tab = c->shot_tab;
    }
    bp.shots = reinterpret_cast<const qs::ShotParams *>(shot_tab);
    bp.outs = reinterpret_cast<const qs::ShotOut *>(shot_tab + sizeof(qs::ShotParams) * n_shots);
    bp.rad32 = c->rad32;
    bp.rad64 = c->rad64;
    bp.rad32d = c->rad32d;
    bp.rad64d = c->rad64d;
    bp.order = ordered ? order : nullptr;
    bp.st.mu = reinterpret_cast<double *>(states);
    bp.st.s2 = reinterpret_cast<double *>(states + arr);
    bp.st.S0 = reinterpret_cast<double *>(states + 2 * arr);
    bp.st.g0 = reinterpret_cast<double *>(states + 3 * arr);
    bp.st.thx = reinterpret_cast<double *>(states + 4 * arr);
    bp.st.thy = reinterpret_cast<double *>(states + 5 * arr);
    bp.st.cmx = reinterpret_cast<float *>(states + 6 * arr);
    if (shadow) {
        unsigned char *base = states + 6 * arr + arrf;
        bp.sst.mu = reinterpret_cast<double *>(base);
        bp.sst.s2 = reinterpret_cast<double *>(base + sarr);
        bp.sst.S0 = reinterpret_cast<double *>(base + 2 * sarr);
        bp.sst.g0 = reinterpret_cast<double *>(base + 3 * sarr);
        bp.sst.thx = reinterpret_cast<double *>(base + 4 * sarr);
        bp.sst.thy = reinterpret_cast<double *>(base + 5 * sarr);
        bp.sst.cmx = reinterpret_cast<float *>(base + 6 * sarr);
    }
    bp.queue = reinterpret_cast<unsigned int *>(accum);
    bp.flags = reinterpret_cast<int *>(accum + 2);
    bp.hist = accum + 2 + flag_words;
    bp.shdiff = shadow ? bp.hist + b.hist_words : nullptr;
    bp.fp64_steps = count_words ? bp.hist + b.hist_words + shd_words : nullptr;
    bp.prec = b.prec;
    bp.partials = partials;
    bp.tape = tape;
    bp.tape_n = b.total;

    // ---- enqueue ----
    const bool prof = c->profiling && !noalloc;
    if ((st = upload_batch(c, b, s)) != QS_OK) return st;
    // the device work after the shot-table copy: set-up (envelope, clear), phase
    // (or tangent), deposit, finalize; with events between them when profiling
    auto enqueue = [&](hipStream_t q, bool marks) -> qs_status {
        hipError_t e;
        auto mark = [&](int k) {
            return marks ? hipEventRecord(c->ev[c->ev_next][k], q) : hipSuccess;
        };
        if ((e = mark(0)) != hipSuccess) return hip_fail(c, e, "event record");
        if ((e = launch_setup(b, N, L[0].envelope, shot_tab, accum, accum_words, env32, env64,
                              q)) != hipSuccess)
            return hip_fail(c, e, "set-up kernel");
        if ((e = mark(1)) != hipSuccess) return hip_fail(c, e, "event record");
        if ((e = mark(2)) != hipSuccess) return hip_fail(c, e, "event record");
        if (ordered && (e = qs::launch_order(bp, q)) != hipSuccess)
            return hip_fail(c, e, "order kernel");
        if (tape) {
            // the forward pass that also records the parameter derivatives
            if ((e = qs::launch_tangent(bp, env32, env64, b.prec, N->rr_model, N->amp_mode,
                                        true, q)) != hipSuccess)
                return hip_fail(c, e, "tangent kernel");
        } else if ((e = qs::launch_phase(bp, env32, env64, b.prec, N->rr_model,
                                         N->amp_mode, q)) != hipSuccess) {
            return hip_fail(c, e, "phase kernel");
        }
        if (shadow && sh_items > 0) {
            // the shadowed samples again in FP64 (their own work counter)
            qs::BatchParams bs = bp;
            bs.shots = reinterpret_cast<const qs::ShotParams *>(
                shot_tab + (sizeof(qs::ShotParams) + sizeof(qs::ShotOut)) * n_shots);
            bs.n_items = sh_items;
            bs.order = nullptr;  // (of the whole shots)
            bs.st = bp.sst;
            bs.queue = bp.queue + 2;
            if ((e = qs::launch_phase(bs, env32, env64, qs::PREC_F64, N->rr_model,
                                      N->amp_mode, q)) != hipSuccess)
                return hip_fail(c, e, "shadow phase kernel");
            // the two states' laws of every shadowed sample, bin by bin
            qs::BatchParams bd = bp;
            bd.shots = bs.shots;
            if ((e = qs::launch_shadow_diff(bd, sh_items, b.max_nh, q)) != hipSuccess)
                return hip_fail(c, e, "shadow difference kernel");
        }
        if ((e = mark(3)) != hipSuccess) return hip_fail(c, e, "event record");
        if ((e = qs::launch_deposit(bp, b.max_nh, false, q)) != hipSuccess)
            return hip_fail(c, e, "deposit kernel");
        if ((e = mark(4)) != hipSuccess) return hip_fail(c, e, "event record");
        if ((e = qs::launch_finalize(bp, q)) != hipSuccess) return hip_fail(c, e, "finalize kernel");
        if ((e = mark(5)) != hipSuccess) return hip_fail(c, e, "event record");
        return QS_OK;
    };
    if (c->graphs && !prof && !tape && !noalloc) {
        // everything the captured launches depend on besides the device shot
        // table (copied before every replay) and the tables built at creation
        struct Sig {
            qs::BatchParams bp;
            double psi_max, h, omega_tau;
            const void *env32, *env64, *accum;
            int64_t accum_words;
            // the FP64 shadow's launches take these by value
            int64_t sh_items, sh_total;
            int32_t shadow;
            int32_t n_steps, envelope, prec, rr, amp, max_nh;
        } sig;
        std::memset(&sig, 0, sizeof(sig));
        sig.bp = bp;
        sig.psi_max = b.psi_max;
        sig.h = b.h;
        sig.omega_tau = b.omega_tau;
        sig.env32 = env32;
        sig.env64 = env64;
        sig.accum = accum;
        sig.accum_words = (int64_t)accum_words;
        sig.sh_items = sh_items;
        sig.sh_total = sh_total;
        sig.shadow = shadow ? 1 : 0;
        sig.n_steps = N->n_steps;
        sig.envelope = L[0].envelope;
        sig.prec = b.prec;
        sig.rr = N->rr_model;
        sig.amp = N->amp_mode;
        sig.max_nh = b.max_nh;
        const unsigned char *sb = reinterpret_cast<const unsigned char *>(&sig);
        std::vector<unsigned char> key(sb, sb + sizeof(sig));
        hipError_t e;
        for (const GraphEntry &g : c->graph_cache) {
            if (g.sig == key) {
                if ((e = hipGraphLaunch(g.exec, s)) != hipSuccess)
                    return hip_fail(c, e, "graph launch");
                c->profiled_call = false;
                c->last_error[0] = 0;
                return QS_OK;
            }
        }
        if (!c->cap_stream &&
            (e = hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking)) != hipSuccess)
            return hip_fail(c, e, "capture stream");
        GraphEntry g;
        g.sig = std::move(key);
        if ((e = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed)) != hipSuccess)
            return hip_fail(c, e, "graph capture");
        const qs_status cs = enqueue(c->cap_stream, false);
        e = hipStreamEndCapture(c->cap_stream, &g.graph);
        if (cs != QS_OK) {
            if (g.graph) (void)hipGraphDestroy(g.graph);
            return cs;
        }
        if (e != hipSuccess) return hip_fail(c, e, "graph capture");
        if ((e = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0)) != hipSuccess) {
            (void)hipGraphDestroy(g.graph);
            return hip_fail(c, e, "graph instantiate");
        }
        if (c->graph_cache.size() >= kMaxGraphs) {
            (void)hipGraphExecDestroy(c->graph_cache.front().exec);
            (void)hipGraphDestroy(c->graph_cache.front().graph);
            c->graph_cache.erase(c->graph_cache.begin());
        }
        c->graph_cache.push_back(std::move(g));
        if ((e = hipGraphLaunch(c->graph_cache.back().exec, s)) != hipSuccess)
            return hip_fail(c, e, "graph launch");
        c->profiled_call = false;
        c->last_error[0] = 0;
        return QS_OK;
    }
    if ((st = enqueue(s, prof)) != QS_OK) return st;
    if (prof) advance_timing_ring(c);
    c->profiled_call = prof;
    c->last_error[0] = 0;
    return QS_OK;
}

qs_status backward_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                        const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                        const qs_grad_outputs *O, const double *tape, hipStream_t s,
                        const View *view) {
    qs_status st;
    for (int k = 0; k < n_shots; ++k)
        if ((st = validate_outputs(c, &O[k])) != QS_OK) return st;
    if (L)
        for (int k = 0; k < n_shots; ++k)
            if (L[k].mode != QS_MODE_GAUSS)
                return set_err(c, "derivatives are for the Gaussian mode only"), QS_EUNSUPPORTED;
    bool want_err = false;
    for (int k = 0; k < n_shots; ++k) want_err = want_err || O[k].errors;
    // FP64 shadow of an FP32 adjoint: two view passes after this one
    const bool shadow = !view && want_err && N && (N->flags & QS_VALIDATE_FP64) &&
                        N->precision == QS_PREC_FP32;
    Batch b;
    if ((st = prepare_batch(c, n_shots, L, B, n_samples, N, H, sizeof(qs::ShotGrad), b, false,
                            view ? view->stride : 1)) != QS_OK)
        return st;
    DeviceGuard guard(c->device);
    qs::BatchParams &bp = b.bp;
    qs::ShotGrad *so = reinterpret_cast<qs::ShotGrad *>(b.outs);
    for (int k = 0; k < n_shots; ++k) {
        so[k].d_energy = O[k].d_energy_hist;
        so[k].grad = O[k].grad;
        so[k].status = O[k].status;
        so[k].d_angle = O[k].d_angle_hist;
        so[k].d_moments = O[k].d_moments;
        so[k].moments = O[k].moments;
        so[k].errors = shadow ? nullptr : O[k].errors;
    }
    const size_t nenv = (size_t)2 * N->n_steps + 1;
    const size_t flag_words = ((size_t)n_shots + 1) / 2;
    const size_t accum_words = 1 + flag_words;
    if ((st = grow(c, &c->env32, &c->env32_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->env64, &c->env64_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->accum, &c->accum_cap, accum_words, "accumulators")) != QS_OK) return st;
    if ((st = grow(c, &c->partials, &c->part_cap, (size_t)bp.n_items * qs::kGradRows * qs::kGradParams, "gradient partials")) != QS_OK)
        return st;
    const bool ordered = b.prec == qs::PREC_F32MIX;  // FP64 steps: samples in chi order
    if (ordered && (st = grow(c, &c->order, &c->order_cap, (size_t)b.total, "chi order")) != QS_OK)
        return st;
    if ((st = grow(c, &c->shot_tab, &c->shot_tab_cap, b.tab_bytes, "shot table")) != QS_OK)
        return st;
    bp.shots = reinterpret_cast<const qs::ShotParams *>(c->shot_tab);
    bp.gouts =
        reinterpret_cast<const qs::ShotGrad *>(c->shot_tab + sizeof(qs::ShotParams) * n_shots);
    bp.rad32 = c->rad32;
    bp.rad64 = c->rad64;
    bp.rad32d = c->rad32d;
    bp.rad64d = c->rad64d;
    bp.queue = reinterpret_cast<unsigned int *>(c->accum);
    bp.flags = reinterpret_cast<int *>(c->accum + 1);
    bp.partials = c->partials;
    bp.tape = const_cast<double *>(tape);  // read only by the contraction kernel
    bp.tape_n = b.total;
    bp.order = ordered ? c->order : nullptr;

    hipError_t e;
    if ((st = upload_batch(c, b, s)) != QS_OK) return st;
    if ((e = launch_setup(b, N, L[0].envelope, c->shot_tab, c->accum, accum_words, c->env32,
                          c->env64, s)) != hipSuccess)
        return hip_fail(c, e, "set-up kernel");
    if (ordered && (e = qs::launch_order(bp, s)) != hipSuccess)
        return hip_fail(c, e, "order kernel");
    if (tape) {
        bool obs = false;
        int max_edges = 1;
        for (int k = 0; k < n_shots; ++k) obs = obs || O[k].d_angle_hist || O[k].d_moments;
        for (int k = 0; k < n_shots; ++k)
            max_edges = std::max(max_edges, H[k].n_e + 1 + (obs ? H[k].n_th + 1 : 0));
        if ((e = qs::launch_contract(bp, obs, max_edges, s)) != hipSuccess)
            return hip_fail(c, e, "contraction kernel");
    } else if ((e = qs::launch_tangent(bp, c->env32, c->env64, b.prec, N->rr_model, N->amp_mode,
                                       false, s)) != hipSuccess) {
        return hip_fail(c, e, "adjoint kernel");
    }
    if ((e = qs::launch_grad_finalize(bp, s)) != hipSuccess)
        return hip_fail(c, e, "gradient finalize kernel");
    if (view ? view->report : want_err && !shadow) {
        // the report of the view passes, or zeros
        if ((e = qs::launch_grad_shadow(bp, view ? view->span : 0, s)) != hipSuccess)
            return hip_fail(c, e, "shadow report kernel");
    }
    if (shadow) {
        // the view of every stride-th sample, recomputed (no tape) at this
        // pass's precision and then in FP64, with the same upstream weights
        const int32_t stride = N->shadow_stride > 0 ? N->shadow_stride : 64;
        const int64_t span = (int64_t)n_shots * qs::kGradParams;
        if ((st = grow(c, &c->shadow, &c->shadow_cap, (size_t)(2 * span), "shadow outputs")) !=
            QS_OK)
            return st;
        std::vector<int64_t> nv(n_shots);
        std::vector<qs_grad_outputs> v32(O, O + n_shots), v64(O, O + n_shots);
        for (int k = 0; k < n_shots; ++k) {
            nv[k] = (n_samples[k] + stride - 1) / stride;
            v32[k].grad = c->shadow + (size_t)k * qs::kGradParams;
            v64[k].grad = v32[k].grad + span;
            v32[k].status = v64[k].status = nullptr;
            v32[k].errors = nullptr;
        }
        qs_numerics vn = *N;
        vn.flags = 0;
        const View v32v{stride, 0, false}, v64v{stride, span, true};
        if ((st = backward_impl(c, n_shots, L, B, nv.data(), &vn, H, v32.data(), nullptr, s,
                                &v32v)) != QS_OK)
            return st;
        vn.precision = QS_PREC_FP64;
        if ((st = backward_impl(c, n_shots, L, B, nv.data(), &vn, H, v64.data(), nullptr, s,
                                &v64v)) != QS_OK)
            return st;
    }
    c->last_error[0] = 0;
    return QS_OK;
}

qs_status photons_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                       const int64_t *n_samples, const qs_numerics *N, const qs_photon_bins *PB,
                       const qs_photon_outputs *PO, hipStream_t s, const View *view) {
    for (int k = 0; k < n_shots; ++k) {
        const qs_photon_bins &b = PB[k];
        if (b.n_ph < 1 || b.n_ph > 4096 || !fin(b.ph_lo) || !fin(b.ph_hi) || !(b.ph_lo >= 0.0) ||
            !(b.ph_hi > b.ph_lo))
            return set_err(c, "photon bins out of range"), QS_EINVAL;
        if (!PO[k].photon_hist || !PO[k].energy)
            return set_err(c, "null photon output pointer"), QS_EINVAL;
    }
    if (!N) return set_err(c, "null argument"), QS_EINVAL;
    for (int k = 0; k < n_shots; ++k)
        if ((double)n_samples[k] * (double)N->n_steps > 1099511627776.0)  // 2^40
            return set_err(c, "photon grids hold at most 2^40 sample-steps a shot"), QS_EINVAL;
    // the electron histograms are not used: placeholder windows
    std::vector<qs_bins> H(n_shots);
    for (qs_bins &h : H) h = qs_bins{1, 1, 1, 0, 0.0, 1.0, 0.0, 1.0};
    bool want_err = false;
    for (int k = 0; k < n_shots; ++k) want_err = want_err || PO[k].errors;
    // FP64 shadow of an FP32 pass: two view passes after this one
    const bool shadow = !view && want_err && (N->flags & QS_VALIDATE_FP64) &&
                        N->precision == QS_PREC_FP32;
    Batch b;
    qs_status st;
    if ((st = prepare_batch(c, n_shots, L, B, n_samples, N, H.data(), sizeof(qs::ShotPhot), b,
                            false, view ? view->stride : 1)) != QS_OK)
        return st;
    DeviceGuard guard(c->device);
    qs::BatchParams &bp = b.bp;
    qs::ShotPhot *sph = reinterpret_cast<qs::ShotPhot *>(b.outs);
    const double aS = 2.0 / bp.two_over_aS;
    // envelope integral of f^2 over the window (an upper bound of the
    // cos^2-weighted one), for the classical-loss bound of the energy range
    const double I2 = L[0].envelope == QS_ENV_GAUSS ? b.omega_tau * std::sqrt(kPi / (4.0 * std::log(2.0)))
                                                    : 0.75 * b.omega_tau;
    const int block = qs::phot_block(b.prec, N->rr_model == QS_RR_QUANTUM);
    int64_t pitem = 0, edges = 0;
    int max_edges = 0;
    for (int k = 0; k < n_shots; ++k) {
        qs::ShotPhot &p = sph[k];
        p = qs::ShotPhot{};
        const double g0 = B[k].gamma0, sg = B[k].sigma_gamma, a0 = L[k].a0;
        // energy range: the samples' spread above, half the classical
        // (Landau-Lifshitz, peak amplitude) bound of the loss below
        const double mu_max = g0 + 6.5 * sg;
        const double mu_lo = std::max(g0 - 6.5 * sg, 1.01);
        const double mu_min = std::max(0.5 * mu_lo / (1.0 + bp.K * mu_lo * a0 * a0 * I2), 1.0);
        // columns uniform in sqrt(mu), the energy range inside columns
        // 1 .. nv - 2 (the outer two stay empty, so the contraction's
        // deconvolution of the deposit needs no column beyond them); the
        // lowest column at no less than half the range's lowest sqrt(mu)
        p.nv = qs::kPhNV;
        const double t_min = std::sqrt(mu_min), t_max = std::sqrt(mu_max);
        p.dt = (t_max - t_min) / (p.nv - 3);
        p.t_lo = t_min - p.dt;
        if (p.t_lo < 0.5 * t_min) {
            p.t_lo = 0.5 * t_min;
            p.dt = (t_max - p.t_lo) / (p.nv - 2);
        }
        p.t_lof = (float)p.t_lo;
        p.inv_dt = (float)(1.0 / p.dt);
        // chi range: the largest chi possible above; below, stages whose
        // photons all fall in the lowest bin (y > 27 beyond 40 chi mu)
        const double width = (PB[k].ph_hi - PB[k].ph_lo) / PB[k].n_ph;
        int r_hi = 1, r_lo = 0;
        if (a0 > 0.0) {
            const double chi_max = 2.0 * mu_max * a0 / aS * 1.02;
            const double chi_floor = std::max(PB[k].ph_lo, width) / (40.0 * mu_max);
            r_hi = (int)std::ceil((std::log(chi_max) - qs::kPhU0) / qs::kPhDu) + 1;
            r_hi = std::min(std::max(r_hi, 1), qs::kPhRows - 1);
            r_lo = (int)std::floor((std::log(chi_floor) - qs::kPhU0) / qs::kPhDu);
            r_lo = std::max(r_lo, 0);
            if (r_hi - r_lo + 1 > qs::kPhNU) r_lo = r_hi - qs::kPhNU + 1;
            if (r_lo > r_hi - 1) r_lo = r_hi - 1;
        }
        p.r_lo = r_lo;
        p.nu = r_hi - r_lo + 1;
        p.n_ph = PB[k].n_ph;
        p.ph_lo = PB[k].ph_lo;
        p.ph_w = width;
        p.hist = PO[k].photon_hist;
        p.energy = PO[k].energy;
        p.status = PO[k].status;
        p.angles = PO[k].angles;
        p.errors = shadow ? nullptr : PO[k].errors;
        p.pitem0 = pitem;
        p.grid_off = (int64_t)k * qs::kPhNodes;
        p.s_off = edges;
        pitem += (n_samples[k] + block - 1) / block;
        edges += PB[k].n_ph + 2;
        max_edges = std::max(max_edges, PB[k].n_ph + 2);
    }
    bp.n_pitems = pitem;

    const size_t nenv = (size_t)2 * N->n_steps + 1;
    const size_t flag_words = ((size_t)n_shots + 1) / 2;
    const size_t accum_words = 1 + flag_words + (size_t)n_shots * qs::kPhNodes;
    if ((st = grow(c, &c->env32, &c->env32_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->env64, &c->env64_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->accum, &c->accum_cap, accum_words, "accumulators")) != QS_OK) return st;
    const size_t part_words = (size_t)pitem * qs::kPhotPartials;
    if ((st = grow(c, &c->partials, &c->part_cap, part_words + (size_t)edges,
                   "photon partials")) != QS_OK)
        return st;
    const bool ordered = b.prec == qs::PREC_F32MIX;  // FP64 steps: samples in chi order
    if (ordered && (st = grow(c, &c->order, &c->order_cap, (size_t)b.total, "chi order")) != QS_OK)
        return st;
    bp.order = ordered ? c->order : nullptr;
    if ((st = grow(c, &c->shot_tab, &c->shot_tab_cap, b.tab_bytes, "shot table")) != QS_OK)
        return st;
    bp.shots = reinterpret_cast<const qs::ShotParams *>(c->shot_tab);
    bp.phot =
        reinterpret_cast<const qs::ShotPhot *>(c->shot_tab + sizeof(qs::ShotParams) * n_shots);
    bp.rad32 = c->rad32;
    bp.rad64 = c->rad64;
    bp.phtab = c->phtab;
    bp.queue = reinterpret_cast<unsigned int *>(c->accum);
    bp.flags = reinterpret_cast<int *>(c->accum + 1);
    bp.pgrid = c->accum + 1 + flag_words;
    bp.partials = c->partials;
    bp.psum = c->partials + part_words;

    hipError_t e;
    if ((st = upload_batch(c, b, s)) != QS_OK) return st;
    if ((e = launch_setup(b, N, L[0].envelope, c->shot_tab, c->accum, accum_words, c->env32,
                          c->env64, s)) != hipSuccess)
        return hip_fail(c, e, "set-up kernel");
    if (ordered && (e = qs::launch_order(bp, s)) != hipSuccess)
        return hip_fail(c, e, "order kernel");
    if ((e = qs::launch_photon(bp, c->env32, c->env64, b.prec, N->rr_model, N->amp_mode, s)) !=
        hipSuccess)
        return hip_fail(c, e, "photon kernel");
    const double c_ph = kAlpha * aS / (2.0 * std::sqrt(3.0) * kPi);
    if ((e = qs::launch_photon_finalize(bp, max_edges, c_ph, s)) != hipSuccess)
        return hip_fail(c, e, "photon finalize kernel");
    if (view ? view->report : want_err && !shadow) {
        // the report of the view passes, or zeros
        if ((e = qs::launch_photon_shadow(bp, view ? view->span : 0, s)) != hipSuccess)
            return hip_fail(c, e, "shadow report kernel");
    }
    if (shadow) {
        // the view of every stride-th sample at this pass's precision and
        // then in FP64, on the same emission grids (they depend on the beam
        // and laser only); per shot: histogram, energies, angles
        const int32_t stride = N->shadow_stride > 0 ? N->shadow_stride : 64;
        int64_t span = 0;
        for (int k = 0; k < n_shots; ++k) span += PB[k].n_ph + 2 + 2 + 6;
        if ((st = grow(c, &c->shadow, &c->shadow_cap, (size_t)(2 * span), "shadow outputs")) !=
            QS_OK)
            return st;
        std::vector<int64_t> nv(n_shots);
        std::vector<qs_photon_outputs> v32(n_shots), v64(n_shots);
        int64_t o = 0;
        for (int k = 0; k < n_shots; ++k) {
            nv[k] = (n_samples[k] + stride - 1) / stride;
            const int64_t nh = PB[k].n_ph + 2;
            double *a = c->shadow + o, *d = a + span;
            v32[k] = qs_photon_outputs{a, a + nh, nullptr, PO[k].angles ? a + nh + 2 : nullptr,
                                       nullptr};
            v64[k] = qs_photon_outputs{d, d + nh, nullptr, PO[k].angles ? d + nh + 2 : nullptr,
                                       PO[k].errors};
            o += nh + 8;
        }
        qs_numerics vn = *N;
        vn.flags = 0;
        const View v32v{stride, 0, false}, v64v{stride, span, true};
        if ((st = photons_impl(c, n_shots, L, B, nv.data(), &vn, PB, v32.data(), s, &v32v)) !=
            QS_OK)
            return st;
        vn.precision = QS_PREC_FP64;
        if ((st = photons_impl(c, n_shots, L, B, nv.data(), &vn, PB, v64.data(), s, &v64v)) !=
            QS_OK)
            return st;
    }
    c->last_error[0] = 0;
    return QS_OK;
}

// Plane-wave reconstruction (Sec. 3.2, 3.3): node runs, interpolation,
// deposit, finalize.  The staging buffer holds the sample view of the shot
// table, the outputs, then the node view (node count and node offset in the
// sample-count and state-offset fields) that the node pass reads.
qs_status factor_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                      const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                      const qs_node_grid *G, const qs_outputs *O, hipStream_t s) {
    qs_status st;
    if (!G) return set_err(c, "null node grid"), QS_EINVAL;
    if (!B || !H) return set_err(c, "null argument"), QS_EINVAL;
    for (int k = 0; k < n_shots; ++k) {
        if ((st = validate_outputs(c, &O[k])) != QS_OK) return st;
        const qs_node_grid &g = G[k];
        if (g.n_a < 2 || g.n_a > 4096) return set_err(c, "node grid: n_a in [2, 4096]"), QS_EINVAL;
        if (B[k].sigma_gamma > 0 ? (g.n_g < 2 || g.n_g > 4096) : g.n_g != 1)
            return set_err(c, "node grid: n_g in [2, 4096] with an energy spread, else 1"),
                   QS_EINVAL;
        if ((int64_t)g.n_a * g.n_g > (1 << 20))
            return set_err(c, "node grid: at most 2^20 nodes"), QS_EINVAL;
    }
    if (N && N->amp_mode != QS_AMP_A0EFF)
        return set_err(c, "the plane-wave reconstruction needs amp_mode A0EFF"), QS_EINVAL;
    Batch b;
    if ((st = prepare_batch(c, n_shots, L, B, n_samples, N, H,
                            sizeof(qs::ShotOut) + sizeof(qs::ShotParams), b)) != QS_OK)
        return st;
    if (qs::deposit_lds_bytes(b.max_nh) > 160 * 1024)
        return set_err(c, "histograms exceed the LDS budget"), QS_EINVAL;
    DeviceGuard guard(c->device);
    qs::ShotOut *so = reinterpret_cast<qs::ShotOut *>(b.outs);
    qs::ShotParams *nv = reinterpret_cast<qs::ShotParams *>(b.outs + sizeof(qs::ShotOut) * n_shots);
    int64_t node_off = 0, node_items = 0, hoff = 0;
    int weight_words = 0;
    bool node_outputs = false;
    for (int k = 0; k < n_shots; ++k) {
        qs::ShotParams &p = b.sp[k];
        const int na = G[k].n_a, ng = G[k].n_g, nn = na * ng;
        p.n_anode = na;
        p.n_gnode = ng;
        p.node_off = node_off;
        p.g_node_lo = B[k].gamma0 - 6.0 * B[k].sigma_gamma;
        p.g_node_step = ng > 1 ? 12.0 * B[k].sigma_gamma / (ng - 1) : 0.0;
        p.hist_off = hoff;  // [energy | angle | a0,eff | node weights]
        hoff += H[k].n_e + 2 + H[k].n_th + 2 + H[k].n_a + nn;
        if (G[k].node_weights) weight_words = std::max(weight_words, nn);
        node_outputs = node_outputs || G[k].node_weights || G[k].node_states;
        nv[k] = p;
        nv[k].n_samples = nn;
        nv[k].state_off = node_off;
        nv[k].item0 = node_items;
        node_off += nn;
        node_items += (nn + qs::kPhaseBlock - 1) / qs::kPhaseBlock;
        const qs_outputs &o = O[k];
        so[k] = qs::ShotOut{};
        so[k].energy_hist = o.energy_hist;
        so[k].angle_hist = o.angle_hist;
        so[k].a0eff_hist = o.a0eff_hist;
        so[k].moments = o.moments;
        so[k].status = o.status;
        so[k].samples = o.samples;
        so[k].rec_stride = o.samples ? o.sample_stride : 1;
        so[k].rec_n = o.samples ? o.n_sample_records : 0;
        so[k].node_states = G[k].node_states;
        so[k].node_weights = G[k].node_weights;
    }
    if ((size_t)weight_words * 8 > 160 * 1024)
        return set_err(c, "node weights exceed the LDS budget (at most 20480 nodes when "
                          "node_weights is requested)"),
               QS_EINVAL;
    b.hist_words = hoff;

    // ---- device scratch: sample and node states, accumulators, partials ----
    qs::BatchParams &bp = b.bp;
    const size_t nenv = (size_t)2 * N->n_steps + 1;
    const size_t arr = ((size_t)b.total * 8 + 255) / 256 * 256;
    const size_t arrf = ((size_t)b.total * 4 + 255) / 256 * 256;
    const size_t narr = ((size_t)node_off * 8 + 255) / 256 * 256;
    const size_t narrf = ((size_t)node_off * 4 + 255) / 256 * 256;
    const size_t flag_words = ((size_t)n_shots + 1) / 2;
    const size_t accum_words = 2 + flag_words + (size_t)b.hist_words;
    if ((st = grow(c, &c->env32, &c->env32_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->env64, &c->env64_cap, nenv, "envelope table")) != QS_OK) return st;
    if ((st = grow(c, &c->accum, &c->accum_cap, accum_words, "accumulators")) != QS_OK) return st;
    if ((st = grow(c, &c->partials, &c->part_cap, (size_t)bp.n_mtiles * qs::kPartials,
                   "moment partials")) != QS_OK)
        return st;
    if ((st = grow(c, &c->states, &c->states_cap, 6 * arr + arrf + 6 * narr + narrf,
                   "sample and node states")) != QS_OK)
        return st;
    if ((st = grow(c, &c->shot_tab, &c->shot_tab_cap, b.tab_bytes, "shot table")) != QS_OK)
        return st;
    bp.shots = reinterpret_cast<const qs::ShotParams *>(c->shot_tab);
    bp.outs = reinterpret_cast<const qs::ShotOut *>(c->shot_tab + sizeof(qs::ShotParams) * n_shots);
    bp.rad32 = c->rad32;
    bp.rad64 = c->rad64;
    auto states_at = [&](unsigned char *base, size_t a8, size_t a4) {
        qs::SampleState x;
        x.mu = reinterpret_cast<double *>(base);
        x.s2 = reinterpret_cast<double *>(base + a8);
        x.S0 = reinterpret_cast<double *>(base + 2 * a8);
        x.g0 = reinterpret_cast<double *>(base + 3 * a8);
        x.thx = reinterpret_cast<double *>(base + 4 * a8);
        x.thy = reinterpret_cast<double *>(base + 5 * a8);
        x.cmx = reinterpret_cast<float *>(base + 6 * a8);
        (void)a4;
        return x;
    };
    bp.st = states_at(c->states, arr, arrf);
    bp.nst = states_at(c->states + 6 * arr + arrf, narr, narrf);
    bp.queue = reinterpret_cast<unsigned int *>(c->accum);
    bp.flags = reinterpret_cast<int *>(c->accum + 2);
    bp.hist = c->accum + 2 + flag_words;
    bp.partials = c->partials;
    qs::BatchParams bn = bp;  // the node pass: node view, writes the node states
    bn.shots = reinterpret_cast<const qs::ShotParams *>(
        c->shot_tab + (sizeof(qs::ShotParams) + sizeof(qs::ShotOut)) * n_shots);
    bn.n_items = node_items;
    bn.st = bp.nst;
    bn.draw_shots = bp.shots;
    bn.draw_st = bp.st;
    bn.n_draws = bp.n_items;

    // ---- enqueue ----
    hipError_t e;
    const bool prof = c->profiling;
    auto mark = [&](int k) {
        return prof ? hipEventRecord(c->ev[c->ev_next][k], s) : hipSuccess;
    };
    if ((st = upload_batch(c, b, s)) != QS_OK) return st;
    if ((e = mark(0)) != hipSuccess) return hip_fail(c, e, "event record");
    if ((e = launch_setup(b, N, L[0].envelope, c->shot_tab, c->accum, accum_words, c->env32,
                          c->env64, s)) != hipSuccess)
        return hip_fail(c, e, "set-up kernel");
    if ((e = mark(1)) != hipSuccess) return hip_fail(c, e, "event record");
    if ((e = mark(2)) != hipSuccess) return hip_fail(c, e, "event record");
    if ((e = qs::launch_phase_nodes(bn, c->env32, c->env64, b.prec, N->rr_model, s)) !=
        hipSuccess)
        return hip_fail(c, e, "node kernel");
    if ((e = mark(3)) != hipSuccess) return hip_fail(c, e, "event record");
    if ((e = qs::launch_node_weights(bp, weight_words, s)) != hipSuccess)
        return hip_fail(c, e, "node weight kernel");
    if ((e = mark(4)) != hipSuccess) return hip_fail(c, e, "event record");
    if ((e = qs::launch_deposit(bp, b.max_nh, true, s)) != hipSuccess)
        return hip_fail(c, e, "deposit kernel");
    if ((e = qs::launch_finalize(bp, s)) != hipSuccess) return hip_fail(c, e, "finalize kernel");
    if (node_outputs && (e = qs::launch_node_outputs(bp, s)) != hipSuccess)
        return hip_fail(c, e, "node output kernel");
    if ((e = mark(5)) != hipSuccess) return hip_fail(c, e, "event record");
    if (prof) advance_timing_ring(c);
    c->profiled_call = prof;
    c->last_error[0] = 0;
    return QS_OK;
}

// ---- launch tuning ------------------------------------------------------------
// Device identity in the cache: architecture name and compute-unit count.
std::string device_tag(int device) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return "unknown";
    std::string tag(prop.gcnArchName);
    const size_t colon = tag.find(':');
    if (colon != std::string::npos) tag.resize(colon);
    return tag + "/" + std::to_string(prop.multiProcessorCount);
}

void install_tune(qs_ctx *c, const TuneEntry &t) {
    for (TuneEntry &u : c->tunes)
        if (u.key == t.key) {
            u = t;
            return;
        }
    c->tunes.push_back(t);
}

// Cache lines: "qscatter-tune-1 <device> <key: 8 integers> <dep_tile> <phase_cap>
// <dep_cap> <phase_ms> <deposit_ms>"; the last matching line wins.
bool read_tune_cache(const char *path, const std::string &tag, const TuneKey &key, TuneEntry &t,
                     double &pms, double &dms) {
    FILE *f = std::fopen(path, "r");
    if (!f) return false;
    char line[512], dev[128];
    bool found = false;
    while (std::fgets(line, sizeof(line), f)) {
        TuneKey k;
        std::memset(&k, 0, sizeof(k));
        int tile = 0, pcap = 0, dcap = 0;
        double p = 0, d = 0;
        if (std::sscanf(line, "qscatter-tune-1 %127s %d %d %d %d %d %d %d %d %d %d %d %lf %lf", dev,
                        &k.n_steps, &k.rr, &k.amp, &k.dep, &k.prec, &k.hist_words, &k.lg_total,
                        &k.lg_shots, &tile, &pcap, &dcap, &p, &d) != 14)
            continue;
        if (tag != dev || !(k == key)) continue;
        if (tile < qs::kMomTile || tile % qs::kMomTile != 0 || tile > (1 << 20) || pcap < 0 ||
            dcap < 0)
            continue;
        t.key = key;
        t.dep_tile = tile;
        t.phase_cap = pcap;
        t.dep_cap = dcap;
        pms = p;
        dms = d;
        found = true;
    }
    std::fclose(f);
    return found;
}

// Times forward passes of one shot under each candidate launch choice (phase
// blocks per CU first, then the deposit tile and deposit blocks per CU), with
// the profiling events around the phase and deposit kernels; keeps the
// fastest, installs it for launches of the same class and appends it to the
// cache file.  Every candidate gives the same results (moment tiles are fixed).
// The tile kDepTile stands for default_dep_tile, so that the choice of an untuned
// launch is among the candidates at every size (5003 samples tuned to items of
// 1024 themselves: deposit 120 us, untuned 39).
qs_status tune_impl(qs_ctx *c, int32_t n_shots, const qs_laser *L, const qs_beam *B,
                    const int64_t *n_samples, const qs_numerics *N, const qs_bins *H,
                    const char *path, qs_tuning *out, hipStream_t s) {
    qs_status st = validate_numerics(c, N);
    if (st != QS_OK) return st;
    int max_nh = 0;
    int64_t total = 0;
    size_t nbuf = 0;
    for (int k = 0; k < n_shots; ++k) {
        if ((st = validate_shot(c, &L[k], &B[k], &H[k], n_samples[k])) != QS_OK) return st;
        const int nh = H[k].n_e + 2 + H[k].n_th + 2 + H[k].n_a;
        max_nh = std::max(max_nh, nh);
        total += n_samples[k];
        nbuf += (size_t)nh + QS_M_N;
    }
    int prec = qs::PREC_F32;
    if (N->precision == QS_PREC_FP64)
        prec = qs::PREC_F64;
    else if (N->rr_model == QS_RR_QUANTUM && N->chi_fp64 > 0)
        prec = qs::PREC_F32MIX;
    const TuneKey key = tune_key(N, prec, max_nh, total, n_shots);
    const std::string tag = device_tag(c->device);
    qs_tuning res;
    std::memset(&res, 0, sizeof(res));
    TuneEntry best;
    double pms = 0, dms = 0;
    if (path && read_tune_cache(path, tag, key, best, pms, dms)) {
        install_tune(c, best);
        res.dep_tile = best.dep_tile;
        res.phase_cap = best.phase_cap;
        res.dep_cap = best.dep_cap;
        res.from_cache = 1;
        res.phase_ms = pms;
        res.deposit_ms = dms;
        if (out) *out = res;
        return QS_OK;
    }

    // outputs of the trial passes
    double *buf = nullptr;
    int32_t *status = nullptr;
    hipError_t e = hipMalloc(&buf, nbuf * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&status, sizeof(int32_t) * n_shots);
    if (e != hipSuccess) {
        (void)hipFree(buf);
        return hip_fail(c, e, "tuning buffers");
    }
    std::vector<qs_outputs> O(n_shots);
    {
        double *p = buf;
        for (int k = 0; k < n_shots; ++k) {
            std::memset(&O[k], 0, sizeof(qs_outputs));
            O[k].energy_hist = p;
            O[k].angle_hist = p + H[k].n_e + 2;
            O[k].a0eff_hist = O[k].angle_hist + H[k].n_th + 2;
            O[k].moments = O[k].a0eff_hist + H[k].n_a;
            O[k].status = status + k;
            p = O[k].moments + QS_M_N;
        }
    }
    const bool prof = c->profiling, graphs = c->graphs;
    struct Restore {
        qs_ctx *c;
        bool prof, graphs;
        double *buf;
        int32_t *status;
        ~Restore() {
            c->tune_forced = false;
            c->graphs = graphs;
            if (!prof) (void)qs_set_profiling(c, 0);
            (void)hipDeviceSynchronize();
            (void)hipFree(buf);
            (void)hipFree(status);
        }
    } restore{c, prof, graphs, buf, status};
    if ((st = qs_set_profiling(c, 1)) != QS_OK) return st;
    c->graphs = false;

    // one warm-up launch, then the best of `reps` timed launches (two, or one
    // when a launch takes more than 100 ms)
    int reps = 2;
    auto trial = [&](const TuneEntry &t, double &phase_ms, double &dep_ms) -> qs_status {
        c->tune_forced = true;
        c->forced = t;
        phase_ms = dep_ms = 1e30;
        for (int r = 0; r <= reps; ++r) {
            qs_status q = forward_impl(c, n_shots, L, B, n_samples, N, H, O.data(), nullptr, s);
            if (q != QS_OK) return q;
            double t5[5];
            if ((q = read_timing_set(c, c->ev_last, t5)) != QS_OK) return q;
            const double tp = t5[2], td = t5[3];
            if (r > 0) {
                phase_ms = std::min(phase_ms, (double)tp);
                dep_ms = std::min(dep_ms, (double)td);
            } else if (tp + td > 100.0f) {
                reps = 1;
            }
        }
        return QS_OK;
    };
    best.key = key;
    best.dep_tile = qs::kDepTile;
    best.phase_cap = 0;
    best.dep_cap = 0;
    double best_p = 1e30, best_d = 1e30;
    for (int pcap : {0, 3, 2}) {
        TuneEntry t = best;
        t.phase_cap = pcap;
        double p, d;
        if ((st = trial(t, p, d)) != QS_OK) return st;
        if (p < best_p) {
            best_p = p;
            best.phase_cap = pcap;
        }
    }
    for (int tile : {qs::kDepTile, 2048, 4096, 8192}) {
        for (int dcap : {0, 4, 2}) {
            TuneEntry t = best;
            t.dep_tile = tile;
            t.dep_cap = dcap;
            double p, d;
            if ((st = trial(t, p, d)) != QS_OK) return st;
            if (d < best_d) {
                best_d = d;
                best.dep_tile = tile;
                best.dep_cap = dcap;
            }
        }
    }
    install_tune(c, best);
    if (path) {
        FILE *f = std::fopen(path, "a");
        if (!f) return set_err(c, "cannot append to the tuning cache"), QS_EINVAL;
        std::fprintf(f, "qscatter-tune-1 %s %d %d %d %d %d %d %d %d %d %d %d %.4f %.4f\n",
                     tag.c_str(), key.n_steps, key.rr, key.amp, key.dep, key.prec, key.hist_words,
                     key.lg_total, key.lg_shots, best.dep_tile, best.phase_cap, best.dep_cap,
                     best_p, best_d);
        std::fclose(f);
    }
    res.dep_tile = best.dep_tile;
    res.phase_cap = best.phase_cap;
    res.dep_cap = best.dep_cap;
    res.phase_ms = best_p;
    res.deposit_ms = best_d;
    if (out) *out = res;
    c->last_error[0] = 0;
    return QS_OK;
}

}  // namespace
