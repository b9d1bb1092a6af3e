// plan.cpp -- host side of the sphfilt C-ABI (include/sphfilt.h).
//
// A plan turns the filter's parameters into device tables once:
//   * one item per shell (field, radius) for the theta-pass, carrying
//     l_max = max(floor, 2 rho L) (Sec. II.A, l_max equation);
//   * one item per ring pair (j, n_theta-1-j) for the phi-pass, carrying
//     m_max = max(floor, 2 rho sin(theta_j) L) (Sec. II.A, m_max equation);
//   * twiddle tables exp(-2 pi i j / N) for both line lengths.
// Items whose mask is 1 on every mode (cutoff >= N/2 for the exponential and
// sharp filters) are sorted after the others: an in-place call launches over
// the non-identity prefix only, an out-of-place call over all items and the
// identity ones are copied.
// On grids with n_phi = 2 n_theta, shells with no identity line are run by a
// kernel that does both passes with one HBM round trip, in one launch with the
// ring pairs of the remaining shells: the fused shell kernel (through LDS) at
// n_phi = 32 and 64, the joined shell kernel (in registers) elsewhere.
#include "../../include/sphfilt.h"
#include "host_tables.h"
#include "sphfilt_internal.h"
#include "tune_cache.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace sphfilt;

namespace {

struct DeviceTables {
    ThetaItem *theta = nullptr;
    PhiItem *phi = nullptr;
    Twiddle *tw_theta = nullptr;
    Twiddle *tw_phi = nullptr;
    double *fused_c = nullptr;
    double *join_c = nullptr;
    PhiItem *phi_in = nullptr;       // phi_in, then phi_rest
    PhiItem *phi_rest = nullptr;     // in the same allocation
};

// A second stream of the plan, for ring pairs that do not depend on the theta
// pass; fork and join events tie it to the caller's stream.  Created with the
// plan when its lists allow overlap, so that no call creates a stream (a call
// may be inside a caller's graph capture); the mutex covers the
// fork-launch-join sequence, so that each call's waits refer to its own event
// records.
struct SideStream {
    std::mutex m;
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    int state = 0;          // 0: not created, 1: ready, -1: creation failed
};

}  // namespace

struct sphfilt_plan_s {
    int n_r, n_theta, n_phi, n_fields;
    int device;
    HostTables host;
    DeviceTables dev;
    int theta_cols, phi_lines;
    int fused;              // fuse shells where the grid allows it
    int theta_mfma;         // theta pass as the circulant product on the matrix cores
    int overlap;            // 0 off, 1 auto, 2 always: independent rings on the side stream
    HybridArgs hybrid;      // detector parameters; dec / replay set per call
    int compute_units;
    int n_join;             // joined plain shells: the last n_join active theta items
    int n_join_hyb;         // joined hybrid shells: theta items [0, n_join_hyb)
    SideStream side;
    uint64_t params_hash;   // grid, fields and cutoffs (the tune cache key, with the GPU arch)
    double tuned_us, default_us;
};

namespace {

void free_device(DeviceTables *d)
{
    if (d->theta) (void)hipFree(d->theta);
    if (d->phi) (void)hipFree(d->phi);
    if (d->tw_theta) (void)hipFree(d->tw_theta);
    if (d->tw_phi) (void)hipFree(d->tw_phi);
    if (d->fused_c) (void)hipFree(d->fused_c);
    if (d->join_c) (void)hipFree(d->join_c);
    if (d->phi_in) (void)hipFree(d->phi_in);
    *d = DeviceTables{};
}

enum class Pass { Theta, Phi };

struct Decisions {
    unsigned char *theta = nullptr;
    unsigned char *phi = nullptr;
    int replay = 0;
};

// Hybrid arguments of one launch: the decision buffer of its pass, and
// `present` only for a launch with hybrid items (the hybrid-capable kernel
// instance costs registers and occupancy the plain one does not).
HybridArgs pass_args(const sphfilt_plan p, unsigned char *dec, const Decisions &d, bool hybrid)
{
    HybridArgs h = p->hybrid;
    h.replay = d.replay;
    h.dec = dec;
    h.present = hybrid ? p->hybrid.present : 0;
    return h;
}

// The theta pass (or the phi pass) over items [0, n) of a list whose first
// n_hyb items are hybrid.  With hybrid items among them all go to the
// hybrid-capable kernel in one launch: it runs plain lines about as fast as the
// plain one (its workgroups of plain shells skip the detector), and a second
// launch costs more than that (a third of the fields hybrid: 5 x 37 shells of
// 48 x 128 32 us in two launches a pass, 21 in one; 20 x 148 74 / 59; 24 x 256
// of 64 x 256 266 / 257).  With the circulant variant the plain active items
// [n_hyb, n_active) go to the matrix-core kernel instead (the item lists put the
// active items first).
hipError_t theta_split(sphfilt_plan p, const double *in, double *out, const ThetaItem *items, int n,
                       int n_hyb, const Decisions &d, hipStream_t s)
{
    const int nh = n_hyb == 0 ? 0 : n_hyb < n && p->theta_mfma ? n_hyb : n;
    hipError_t e = hipSuccess;
    if (nh > 0)
        e = launch_theta(2 * p->n_theta, p->theta_cols, in, out, items, nh, p->n_theta, p->n_phi,
                         p->dev.tw_theta, pass_args(p, d.theta, d, true), s);
    int done = nh;
    if (p->theta_mfma && e == hipSuccess) {
        const int na = n < p->host.theta_active ? n : p->host.theta_active;
        if (na > nh)
            e = launch_theta_gemm(p->n_theta, p->n_phi, in, out, items + nh, na - nh,
                                  p->dev.tw_theta, s);
        done = na > nh ? na : nh;
    }
    if (e == hipSuccess && n > done)
        e = launch_theta(2 * p->n_theta, p->theta_cols, in, out, items + done, n - done, p->n_theta,
                         p->n_phi, p->dev.tw_theta, pass_args(p, d.theta, d, false), s);
    return e;
}

hipError_t phi_split(sphfilt_plan p, const double *in, double *out, const PhiItem *items, int n,
                     int n_hyb, const Decisions &d, hipStream_t s)
{
    return launch_phi(p->n_phi, p->phi_lines, in, out, items, n, p->n_theta, p->dev.tw_phi,
                      pass_args(p, d.phi, d, n_hyb > 0), s);
}

int run_pass(sphfilt_plan p, Pass which, const double *in, double *out, bool all_items,
             const Decisions &d, hipStream_t s)
{
    const HostTables &t = p->host;
    const hipError_t e =
        which == Pass::Theta
            ? theta_split(p, in, out, p->dev.theta, all_items ? (int)t.theta.size() : t.theta_active,
                          t.theta_hyb, d, s)
            : phi_split(p, in, out, p->dev.phi, all_items ? (int)t.phi.size() : t.phi_active,
                        t.phi_hyb, d, s);
    return e == hipSuccess ? SPHFILT_OK : SPHFILT_EDEVICE;
}

int check_call(sphfilt_plan p, const double *in, double *out)
{
    if (!p || !in || !out) return SPHFILT_EINVAL;
    const size_t bytes = sizeof(double) * (size_t)p->n_fields * p->n_r * p->n_theta * p->n_phi;
    const uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
    if ((a | b) & 15) return SPHFILT_EINVAL;                               // 16-byte accesses
    if (a != b && a < b + bytes && b < a + bytes) return SPHFILT_EINVAL;   // partial overlap
    if (fault("launch")) return SPHFILT_EDEVICE;
    return SPHFILT_OK;
}

// Fused shells (held in registers at n_phi = 128: 24 x 508 shells of 64 x 128
// 413 -> 325 us, the hybrid third of 24 x 128 78 -> 65) and the phi pass of
// the other shells' ring pairs, in one launch.  On a fusable grid (n_phi = 2 n_theta) a shell that the theta pass
// filters has every ring filtered too (m_max <= l_max < n_theta = n_phi / 2,
// also in floating point: rounding is monotone), so all of them are fused and
// the theta pass has nothing left: the other shells only need their rings
// (copied out of place when identity).  Returns SPHFILT_EUNSUPPORTED if some
// theta-filtered shell was not fused; the caller then runs two passes.
int apply_fused(sphfilt_plan p, bool adjoint, const double *in, double *out, const Decisions &d,
                hipStream_t s)
{
    const HostTables &t = p->host;
    if (t.theta_active != t.n_fused) return SPHFILT_EUNSUPPORTED;
    const int n_rings = in == out ? t.phi_rest_active : (int)t.phi_rest.size();
    // With hybrid shells among them, up to 128 MiB of shells go through the
    // hybrid-capable kernel in one launch with the rings (a third of the fields
    // hybrid: 5 x 37 shells of 32 x 64 17.1 us in two launches, 11.6 in one; 24 x
    // 128 24.3 / 19.0; but 24 x 1024, 400 MB, 204 / 210: its workgroups are
    // larger and hold more registers).  At n_phi = 128 both kinds are joined.
    const bool together = t.fused_hyb > 0 && p->n_phi != 128 && !p->theta_mfma &&
                          8LL * t.n_fused * p->n_theta * p->n_phi <= 128LL << 20;
    const int nh = together ? t.n_fused : t.fused_hyb, lines = p->n_theta / 2;
    const int rings_h = together ? n_rings : 0;
    hipError_t e = hipSuccess;
    // else hybrid shells with the hybrid-capable kernel; the other shells and the
    // rings of the theta-idle shells (never hybrid) with the plain one
    if (nh > 0 && p->n_phi == 128)
        e = launch_join_hybrid(adjoint, p->n_phi, in, out, p->dev.theta, p->dev.fused_c, nh, p->dev.tw_phi,
                               pass_args(p, d.theta, d, true), pass_args(p, d.phi, d, true), s);
    else if (nh > 0)
        e = launch_shell_phi(adjoint, p->n_theta, p->n_phi, in, out, p->dev.theta, p->dev.fused_c,
                             nh, p->dev.phi_rest, rings_h, p->dev.tw_phi,
                             pass_args(p, d.theta, d, true), pass_args(p, d.phi, d, true), s);
    if (e == hipSuccess && (t.n_fused > nh || n_rings > rings_h))
        e = p->n_phi == 128
                ? launch_join(adjoint, p->n_phi, in, out, p->dev.theta + nh,
                              p->dev.fused_c + (size_t)nh * lines, t.n_fused - nh, p->dev.phi_rest,
                              n_rings, 0, p->dev.tw_phi, s)
                : launch_shell_phi(adjoint, p->n_theta, p->n_phi, in, out, p->dev.theta + nh,
                                   p->dev.fused_c + (size_t)nh * lines, t.n_fused - nh,
                                   p->dev.phi_rest, n_rings, p->dev.tw_phi,
                                   pass_args(p, d.theta, d, false), pass_args(p, d.phi, d, false), s,
                                   p->theta_mfma != 0);
    return e == hipSuccess ? SPHFILT_OK : SPHFILT_EDEVICE;
}

bool side_create(SideStream &ss)
{
    if (ss.state == 0) {
        ss.state = -1;
        if (hipStreamCreateWithFlags(&ss.stream, hipStreamNonBlocking) != hipSuccess) {
            ss.stream = nullptr;
            return false;
        }
        if (hipEventCreateWithFlags(&ss.fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ss.join, hipEventDisableTiming) != hipSuccess)
            return false;
        ss.state = 1;
    }
    return ss.state == 1;
}

void side_destroy(SideStream &ss)
{
    if (ss.join) (void)hipEventDestroy(ss.join);
    if (ss.fork) (void)hipEventDestroy(ss.fork);
    if (ss.stream) (void)hipStreamDestroy(ss.stream);
    ss.stream = nullptr;
    ss.fork = ss.join = nullptr;
    ss.state = 0;
}

// Overlap needs theta work and independent ring pairs; in the automatic mode
// the independent rings must also move enough bytes to hide the fork and
// join (a few microseconds each on the device timeline).
constexpr long long kOverlapMinBytes = 128LL << 20;

bool overlap_pays(sphfilt_plan p)
{
    const HostTables &t = p->host;
    if (p->overlap == 0 || t.n_fused != 0 || t.theta_active == 0 || t.phi_rest_active == 0)
        return false;
    const long long rest_bytes = 16LL * 2 * t.phi_rest_active * p->n_phi;
    return p->overlap == 2 || rest_bytes >= kOverlapMinBytes;
}

// In place: the ring pairs of shells the theta pass leaves alone do not
// depend on it, so they run on the side stream while the caller's stream runs
// the theta pass and the rings of the theta-filtered shells (in the call's
// order); the caller's stream then waits for the side stream.  Returns
// SPHFILT_EUNSUPPORTED when the plan has no side stream (the caller then runs
// two passes).
int apply_overlap(sphfilt_plan p, bool adjoint, double *x, const Decisions &d, hipStream_t s)
{
    const HostTables &t = p->host;
    std::lock_guard<std::mutex> lock(p->side.m);
    if (p->side.state != 1) return SPHFILT_EUNSUPPORTED;
    hipStream_t side = p->side.stream;
    hipError_t e = hipEventRecord(p->side.fork, s);
    if (e == hipSuccess) e = hipStreamWaitEvent(side, p->side.fork, 0);
    auto theta = [&]() { return theta_split(p, x, x, p->dev.theta, t.theta_active, t.theta_hyb, d, s); };
    auto rings_in = [&]() {
        return phi_split(p, x, x, p->dev.phi_in, (int)t.phi_in.size(), t.phi_in_hyb, d, s);
    };
    if (e == hipSuccess) e = adjoint ? rings_in() : theta();
    // the rings of theta-idle shells: never hybrid, but by the kernel instance
    // that takes them in two passes
    if (e == hipSuccess)
        e = phi_split(p, x, x, p->dev.phi_rest, t.phi_rest_active, t.phi_hyb, d, side);
    if (e == hipSuccess) e = adjoint ? theta() : rings_in();
    if (e == hipSuccess) e = hipEventRecord(p->side.join, side);
    if (e == hipSuccess) e = hipStreamWaitEvent(s, p->side.join, 0);
    return e == hipSuccess ? SPHFILT_OK : SPHFILT_EDEVICE;
}

// Joined shells: on the 2 n_theta = n_phi grids that are not fused, active
// shells go through one kernel that holds a whole shell in registers (n_join
// of the plain ones and n_join_hyb of the hybrid ones; the rest take two
// passes), and the ring pairs of the other shells through that launch's
// ring workgroups or the phi kernel (all of them out of place, where identity
// rings are copied), so a point moves once, or twice where its shell takes two
// passes.  The sets touch different shells; with overlapped passes the last
// one runs on the side stream.  Every shell and ring takes the same kernel
// instances in place, out of place and overlapped: the results are the same bits.
int apply_joined(sphfilt_plan p, bool adjoint, const double *in, double *out, const Decisions &d,
                 hipStream_t s)
{
    const HostTables &t = p->host;
    const int nh = t.theta_hyb, nj = p->n_join_hyb, lines = p->n_theta / 2, n_join = p->n_join;
    const int first_join = t.theta_active - n_join, n_two = first_join - nj;
    const int n_rest = in == out ? t.phi_rest_active : (int)t.phi_rest.size();
    const bool along = n_join > 0;
    std::unique_lock<std::mutex> lock(p->side.m, std::defer_lock);
    hipStream_t rest = s;
    hipError_t e = hipSuccess;
    if (in == out && overlap_pays(p) && p->side.state == 1) {
        lock.lock();
        rest = p->side.stream;
        e = hipEventRecord(p->side.fork, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(rest, p->side.fork, 0);
    }
    auto theta = [&](const double *src, int first, int n, bool hybrid) {
        return launch_theta(2 * p->n_theta, p->theta_cols, src, out, p->dev.theta + first, n, p->n_theta,
                            p->n_phi, p->dev.tw_theta, pass_args(p, d.theta, d, hybrid), s);
    };
    auto phi = [&](const double *src, int first, int n, bool hybrid, hipStream_t st) {
        return launch_phi(p->n_phi, p->phi_lines, src, out, p->dev.phi_in + first, n, p->n_theta,
                          p->dev.tw_phi, pass_args(p, d.phi, d, hybrid), st);
    };
    auto join = [&](int n, int n_rings, hipStream_t st) {
        return launch_join(adjoint, p->n_phi, in, out, p->dev.theta + first_join,
                           p->dev.join_c + (size_t)first_join * lines, n, p->dev.phi_rest, n_rings,
                           p->compute_units, p->dev.tw_phi, st);
    };
    if (e == hipSuccess && nj > 0)
        e = launch_join_hybrid(adjoint, p->n_phi, in, out, p->dev.theta, p->dev.join_c, nj, p->dev.tw_phi,
                               pass_args(p, d.theta, d, true), pass_args(p, d.phi, d, true), s);
    // two passes of the shells in between, hybrid and plain ones in the same
    // launches, whose rings are phi_in's.  In place on one stream, and where no
    // plain shell is joined, the phi kernel takes the rest's rings in the same
    // launch (phi_rest follows phi_in); apart, they take the same instance.
    const bool hybrid = nh > nj;
    const bool one_phi = in == out && rest == s && !along && n_two > 0;
    if (n_two > 0) {
        const int rings = n_two * lines + (one_phi ? n_rest : 0);
        if (e == hipSuccess) e = adjoint ? phi(in, nj * lines, rings, hybrid, s) : theta(in, nj, n_two, hybrid);
        if (e == hipSuccess) e = adjoint ? theta(out, nj, n_two, hybrid) : phi(out, nj * lines, rings, hybrid, s);
    }
    if (e == hipSuccess && n_join > 0) e = join(n_join, along && rest == s ? n_rest : 0, s);
    if (e == hipSuccess && along && rest != s) e = join(0, n_rest, rest);
    if (e == hipSuccess && !along && !one_phi)
        e = phi(in, (int)t.phi_in.size(), n_rest, hybrid && n_two > 0, rest);
    if (rest != s) {
        if (e == hipSuccess) e = hipEventRecord(p->side.join, rest);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, p->side.join, 0);
    }
    return e == hipSuccess ? SPHFILT_OK : SPHFILT_EDEVICE;
}

// Out of place, forward: the rings of shells that the theta pass leaves alone
// straight from `in`, instead of a copy by the theta pass that the phi pass
// reads and writes again.  It takes a third launch, which pays from about 100 MB
// of saved traffic on (32 bytes per point of such a ring that is filtered): 144
// MB saved 471 -> 373 us (24 x 256 shells of 128 x 160 at cal-L = 3), 219 MB 132 ->
// 103, 586 MB 409 -> 308, but 55 MB 34 -> 43 and 48 MB 68 -> 72.  (The adjoint's
// first pass reads every ring once as it is.)  On grids that are joined, but have
// too few shells to join, it pays from 32 MiB on (128 x 256, 96 x 192, 80 x 160:
// 26 MiB 49.4 / 48.3 us direct / in two launches, 29 46.3 / 42.5, 32 40.4 / 45.5,
// 40 68.4 / 69.4, 50 90 / 97, 76 89.6 / 102).  Not on grids with fused shells (reached
// there with fusing off): phi_in leaves the rings of fused shells out.
constexpr long long kDirectMinBytes = 96LL << 20, kDirectMinBytesJoined = 32LL << 20;

bool rings_direct(const sphfilt_plan p)
{
    return p->host.n_fused == 0 && !p->theta_mfma &&
           32LL * p->host.phi_rest_active * p->n_phi >=
               (p->host.join_c.empty() ? kDirectMinBytes : kDirectMinBytesJoined);
}

int apply_direct(sphfilt_plan p, const double *in, double *out, const Decisions &d, hipStream_t s)
{
    const HostTables &t = p->host;
    hipError_t e = theta_split(p, in, out, p->dev.theta, t.theta_active, t.theta_hyb, d, s);
    const int n_in = (int)t.phi_in.size();
    // the same kernel instance for all rings as in place
    if (e == hipSuccess) e = phi_split(p, out, out, p->dev.phi_in, n_in, t.phi_hyb, d, s);
    if (e == hipSuccess) e = phi_split(p, in, out, p->dev.phi_rest, (int)t.phi_rest.size(), t.phi_hyb, d, s);
    return e == hipSuccess ? SPHFILT_OK : SPHFILT_EDEVICE;
}

// Two passes in the given order.  Out of place, the first pass runs over all
// items (copying identity lines) and the second works in place on `out`.
int apply_two(sphfilt_plan p, Pass first, Pass second, const double *in, double *out,
              const Decisions &d, void *stream)
{
    int rc = check_call(p, in, out);
    if (rc) return rc;
    DeviceGuard g(p->device);
    if (!g.ok) return SPHFILT_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    if (p->fused && p->host.n_fused > 0) {
        rc = apply_fused(p, first == Pass::Phi, in, out, d, s);
        if (rc != SPHFILT_EUNSUPPORTED) return rc;
    }
    // with nothing to join, two passes below (in a third launch, the rings apart: 2 x
    // 246 shells of 80 x 160 at cal-L = 0.896 out of place 31 -> 38 us)
    if (p->fused && p->n_join + p->n_join_hyb > 0) return apply_joined(p, first == Pass::Phi, in, out, d, s);
    if (overlap_pays(p) && in == out) {
        rc = apply_overlap(p, first == Pass::Phi, out, d, s);
        if (rc != SPHFILT_EUNSUPPORTED) return rc;
    }
    const bool inplace = in == out;
    if (!inplace && first == Pass::Theta && rings_direct(p)) return apply_direct(p, in, out, d, s);
    rc = run_pass(p, first, in, out, !inplace, d, s);
    if (rc) return rc;
    return run_pass(p, second, out, out, false, d, s);
}

int apply_one(sphfilt_plan p, Pass which, const double *in, double *out, void *stream)
{
    int rc = check_call(p, in, out);
    if (rc) return rc;
    DeviceGuard g(p->device);
    if (!g.ok) return SPHFILT_EDEVICE;
    return run_pass(p, which, in, out, in != out, Decisions{}, (hipStream_t)stream);
}

uint64_t hash_params(int n_r, int n_theta, int n_phi, int n_fields, const int *parity,
                     const sphfilt_cutoff *cut)
{
    uint64_t h = kFnvSeed;
    const char tag[] = "plan";
    h = fnv1a(h, tag, sizeof(tag));
    const int dims[4] = {n_r, n_theta, n_phi, n_fields};
    h = fnv1a(h, dims, sizeof(dims));
    h = fnv1a(h, parity, sizeof(int) * n_fields);
    h = fnv1a(h, cut->L, sizeof(double) * n_fields);
    const int has[2] = {cut->rho != nullptr, cut->kind != nullptr};
    h = fnv1a(h, has, sizeof(has));
    if (cut->rho) h = fnv1a(h, cut->rho, sizeof(double) * n_r);
    if (cut->kind) h = fnv1a(h, cut->kind, sizeof(int) * n_fields);
    const double d[3] = {cut->floor_modes, cut->detector_eps, cut->detector_threshold};
    return fnv1a(h, d, sizeof(d));
}

// ---- the plan's autotuner --------------------------------------------------
struct PlanSched {
    int theta_cols, phi_lines, fused, theta_mfma, overlap;
    bool operator==(const PlanSched &o) const
    {
        return theta_cols == o.theta_cols && phi_lines == o.phi_lines && fused == o.fused &&
               theta_mfma == o.theta_mfma && overlap == o.overlap;
    }
};

PlanSched plan_sched(const sphfilt_plan p)
{
    return PlanSched{p->theta_cols, p->phi_lines, p->fused, p->theta_mfma, p->overlap};
}

void set_plan_sched(sphfilt_plan p, const PlanSched &c)
{
    p->theta_cols = c.theta_cols;
    p->phi_lines = c.phi_lines;
    p->fused = c.fused;
    p->theta_mfma = c.theta_mfma;
    p->overlap = c.overlap;
}

// Rounds of back-to-back forward filters in place on x (HIP events on s
// around each round); returns the median over `reps` rounds of the time per
// filter.  Back to back, as a time-stepping loop calls the filter: timed one
// call at a time, the launch latency of each call (and of the second stream's
// fork and join) is exposed, which a caller that queues calls does not see.
constexpr int kPlanCallsPerRound = 8;

int time_plan(sphfilt_plan p, double *x, hipStream_t s, int reps, double *us)
{
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return SPHFILT_EDEVICE;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return SPHFILT_EDEVICE; }
    std::vector<float> t;
    int rc = SPHFILT_OK;
    for (int r = 0; r < reps + 2 && !rc; ++r) {
        if (hipEventRecord(e0, s) != hipSuccess) { rc = SPHFILT_EDEVICE; break; }
        for (int c = 0; c < kPlanCallsPerRound && !rc; ++c)
            rc = apply_two(p, Pass::Theta, Pass::Phi, x, x, Decisions{}, s);
        if (rc) break;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
            rc = SPHFILT_EDEVICE;
            break;
        }
        float ms = 0;
        (void)hipEventElapsedTime(&ms, e0, e1);
        if (r >= 2) t.push_back(ms / kPlanCallsPerRound);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    std::sort(t.begin(), t.end());
    *us = 1000.0 * t[t.size() / 2];
    return SPHFILT_OK;
}

// Run forward filters until the GPU has spent >= 25 ms on them.
int warm_plan(sphfilt_plan p, double *x, hipStream_t s)
{
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return SPHFILT_EDEVICE;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return SPHFILT_EDEVICE; }
    int rc = SPHFILT_OK;
    float spent = 0.0f;
    for (int k = 0; k < 256 && spent < 25.0f && !rc; ++k) {
        if (hipEventRecord(e0, s) != hipSuccess) { rc = SPHFILT_EDEVICE; break; }
        for (int i = 0; i < 8 && !rc; ++i) rc = apply_two(p, Pass::Theta, Pass::Phi, x, x, Decisions{}, s);
        if (rc) break;
        float ms = 0;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            rc = SPHFILT_EDEVICE;
            break;
        }
        spent += ms;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

// Coordinate descent from the plan's current schedule over the theta tile
// width, the ring pairs per phi workgroup, fused shells (where the grid has
// them), the theta variant (where the circulant product applies) and the
// overlap mode (where the plan has a side stream; then also every ring-pair
// count with each overlapping mode); each candidate is timed
// as a forward filter in place on zeroed scratch fields of the plan's size.
int tune_plan(sphfilt_plan p, const std::string &arch, const char *cache_path)
{
    const size_t n = (size_t)p->n_fields * p->n_r * p->n_theta * p->n_phi;
    double *x = nullptr;
    hipError_t e = hipMalloc((void **)&x, sizeof(double) * n);
    if (e != hipSuccess) return e == hipErrorOutOfMemory ? SPHFILT_ENOMEM : SPHFILT_EDEVICE;
    hipStream_t s = nullptr;
    int rc = SPHFILT_OK;
    if (hipMemset(x, 0, sizeof(double) * n) != hipSuccess ||
        hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess)
        rc = SPHFILT_EDEVICE;
    const PlanSched start = plan_sched(p);
    PlanSched best = start;
    double best_us = 1e300, default_us = -1.0;
    std::vector<PlanSched> tried;
    auto try_sched = [&](const PlanSched &c) {
        if (rc || std::find(tried.begin(), tried.end(), c) != tried.end()) return;
        tried.push_back(c);
        set_plan_sched(p, c);
        double us = 0;
        rc = time_plan(p, x, s, 9, &us);
        if (rc) return;
        if (default_us < 0) default_us = us;
        if (us < best_us) {
            best_us = us;
            best = c;
        }
    };
    // Warm the GPU up first (its clock needs ~10 ms of continuous work; timed
    // cold, the first candidates would read slow and the order of the search
    // would decide the pick).
    if (!rc) rc = warm_plan(p, x, s);
    try_sched(start);
    const int nl = 2 * p->n_theta;
    for (int w : {4, 8, 16, 32, 64})
        if (theta_shape_ok(nl, w, p->n_phi)) {
            PlanSched c = best;
            c.theta_cols = w;
            try_sched(c);
        }
    for (int l : {4, 8, 16, 32, 64})
        if (phi_shape_ok(p->n_phi, l)) {
            PlanSched c = best;
            c.phi_lines = l;
            try_sched(c);
        }
    if (p->host.n_fused > 0 || !p->host.join_c.empty())
        for (int f : {0, 1}) {
            PlanSched c = best;
            c.fused = f;
            try_sched(c);
        }
    if (theta_gemm_ok(p->n_theta, p->n_phi))
        for (int m : {0, 1}) {
            PlanSched c = best;
            c.theta_mfma = m;
            try_sched(c);
        }
    if (p->side.state == 1) {
        for (int o : {0, 1, 2}) {
            PlanSched c = best;
            c.overlap = o;
            try_sched(c);
        }
        // the phi launch shape and the overlap interact (small phi
        // workgroups on the second stream crowd the theta pass): every shape
        // with each overlapping mode
        const PlanSched base = best;
        for (int l : {4, 8, 16, 32, 64})
            for (int o : {1, 2})
                if (phi_shape_ok(p->n_phi, l)) {
                    PlanSched c = base;
                    c.phi_lines = l;
                    c.overlap = o;
                    try_sched(c);
                }
    }
    // confirm: the pick against the starting settings, three alternating
    // rounds each; keep the pick only if it is faster by more than 1 %
    if (!rc && !(best == start)) {
        std::vector<double> tb, ts;
        for (int round = 0; round < 3 && !rc; ++round) {
            double us = 0;
            set_plan_sched(p, best);
            rc = time_plan(p, x, s, 5, &us);
            tb.push_back(us);
            set_plan_sched(p, start);
            if (!rc) rc = time_plan(p, x, s, 5, &us);
            ts.push_back(us);
        }
        if (!rc) {
            std::sort(tb.begin(), tb.end());
            std::sort(ts.begin(), ts.end());
            best_us = tb[1];
            default_us = ts[1];
            if (!(tb[1] < 0.99 * ts[1])) {
                best = start;
                best_us = ts[1];
            }
        }
    }
    if (s) {
        (void)hipStreamSynchronize(s);
        (void)hipStreamDestroy(s);
    }
    (void)hipFree(x);
    set_plan_sched(p, rc ? start : best);
    if (rc) return rc;
    p->tuned_us = best_us;
    p->default_us = default_us;
    if (cache_path) {
        TuneFields f;
        f["what"] = tune_str("plan");
        f["arch"] = tune_str(arch);
        f["theta_cols"] = tune_num(best.theta_cols);
        f["phi_lines"] = tune_num(best.phi_lines);
        f["fused"] = tune_num(best.fused);
        f["theta_variant"] = tune_num(best.theta_mfma);
        f["overlap"] = tune_num(best.overlap);
        f["us"] = tune_num(best_us);
        f["default_us"] = tune_num(default_us);
        const uint64_t sig = fnv1a(p->params_hash, arch.data(), arch.size());
        if (!tune_cache_put(cache_path, hex64(sig), f)) return SPHFILT_EINVAL;
    }
    return SPHFILT_OK;
}

// A plan's default ring pairs per phi workgroup: the fastest measured for
// the phi pass alone on dense MI355X grids (smaller workgroups drain
// more evenly): 4 at n_phi = 256 (265
// against 270 us for 16), 8 at 64, 80, 96, 128, 160 and 192 (1-4 % faster
// than a full 256-lane workgroup); a full workgroup at 32 and 48, where that
// is fastest.  The batch kernels keep full workgroups.
int plan_phi_lines(int n_phi)
{
    switch (n_phi) {
    case 256: return 4;
    case 64: case 80: case 96: case 128: case 160: case 192: return 8;
    default: return default_phi_lines(n_phi);
    }
}

}  // namespace

extern "C" {

int sphfilt_workload_stats(int n_r, int n_theta, int n_phi, int n_fields, const int *parity,
                           const sphfilt_cutoff *cut, sphfilt_stats *out)
{
    if (!out) return SPHFILT_EINVAL;
    int rc = validate(n_r, n_theta, n_phi, n_fields, parity, cut);
    if (rc) return rc;
    try {
        HostTables h;
        build_items(n_r, n_theta, n_phi, n_fields, parity, cut, &h);
        fill_stats(n_r, n_theta, n_phi, n_fields, h, out);
    } catch (const std::bad_alloc &) {
        return SPHFILT_ENOMEM;
    }
    return SPHFILT_OK;
}

int sphfilt_plan_create(sphfilt_plan *out, int n_r, int n_theta, int n_phi, int n_fields,
                        const int *parity, const sphfilt_cutoff *cut)
{
    if (!out) return SPHFILT_EINVAL;
    *out = nullptr;
    int rc = validate(n_r, n_theta, n_phi, n_fields, parity, cut);
    if (rc) return rc;
    if (fault("alloc")) return SPHFILT_ENOMEM;
    sphfilt_plan p = new (std::nothrow) sphfilt_plan_s();
    if (!p) return SPHFILT_ENOMEM;
    p->n_r = n_r;
    p->n_theta = n_theta;
    p->n_phi = n_phi;
    p->n_fields = n_fields;
    p->theta_cols = default_theta_cols(2 * n_theta, n_phi);
    p->hybrid = hybrid_args(cut, n_fields);
    p->phi_lines = plan_phi_lines(n_phi);
    p->fused = 1;
    p->theta_mfma = 0;
    p->overlap = 0;
    p->params_hash = hash_params(n_r, n_theta, n_phi, n_fields, parity, cut);
    p->tuned_us = p->default_us = -1.0;
    try {
        build_items(n_r, n_theta, n_phi, n_fields, parity, cut, &p->host);
        if (hipGetDevice(&p->device) != hipSuccess) rc = SPHFILT_EDEVICE;
        if (!rc) rc = upload(&p->dev.theta, p->host.theta);
        if (!rc) rc = upload(&p->dev.phi, p->host.phi);
        if (!rc) rc = upload(&p->dev.tw_theta, twiddles(2 * n_theta));
        if (!rc) rc = upload(&p->dev.tw_phi, twiddles(n_phi));
        if (!rc) rc = upload(&p->dev.fused_c, p->host.fused_c);
        if (!rc) rc = upload(&p->dev.join_c, p->host.join_c);
        std::vector<PhiItem> rings = p->host.phi_in;
        rings.insert(rings.end(), p->host.phi_rest.begin(), p->host.phi_rest.end());
        if (!rc) rc = upload(&p->dev.phi_in, rings);
        if (!rc) p->dev.phi_rest = p->dev.phi_in + p->host.phi_in.size();
        if (!rc && !p->host.join_c.empty()) {
            const HostTables &t = p->host;
            int units = 0;
            if (hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, p->device) != hipSuccess ||
                units <= 0) {
                rc = SPHFILT_EDEVICE;
            } else {
                p->compute_units = units;
                p->n_join = join_count(n_phi, t.theta_active - t.theta_hyb, t.phi_rest_active, units);
                // hybrid shells of 256-point lines take two passes: a joined round
                // is 51 us, as long as the passes (share with 8 hybrid fields: 512
                // us either way; at 192 203 joined, 207 in two passes), with the
                // detector and the Gaussian and with 66 to 73 registers spilled
                // under the cap of 128 that 1024 lanes leave
                p->n_join_hyb = n_phi == 256 ? 0 : join_count(n_phi, t.theta_hyb, 0, units);
                // beside plain shells in two passes, hybrid ones in the same launches
                // save theirs, and joining pays only for rounds of 192 points that are
                // nearly full (one hybrid field and one plain one, joined / not: 80 x
                // 160, 150 shells each 36 / 24 us, 256 38.5 / 34.7, 400 60 / 48; 96 x
                // 192, 200 44 / 40, 256 46 / 48, 400 71 / 65, 1000 125 / 131)
                const int last = t.theta_hyb % units;
                if (p->n_join == 0 && t.theta_active > t.theta_hyb &&
                    !(n_phi == 192 && (last == 0 || 8 * last >= 7 * units)))
                    p->n_join_hyb = 0;
            }
        }
    } catch (const std::bad_alloc &) {
        rc = SPHFILT_ENOMEM;
    }
    const HostTables &t = p->host;
    if (!rc && t.n_fused == 0 && t.theta_active > 0 && t.phi_rest_active > 0 &&
        !side_create(p->side))
        rc = SPHFILT_EDEVICE;
    if (rc) {
        side_destroy(p->side);
        free_device(&p->dev);
        delete p;
        return rc;
    }
    *out = p;
    return SPHFILT_OK;
}

int sphfilt_plan_destroy(sphfilt_plan plan)
{
    if (!plan) return SPHFILT_OK;
    {
        DeviceGuard g(plan->device);
        side_destroy(plan->side);
        free_device(&plan->dev);
    }
    delete plan;
    return SPHFILT_OK;
}

int sphfilt_apply(sphfilt_plan plan, const double *in, double *out, void *stream)
{
    return apply_two(plan, Pass::Theta, Pass::Phi, in, out, Decisions{}, stream);
}

int sphfilt_apply_adjoint(sphfilt_plan plan, const double *in, double *out, void *stream)
{
    return apply_two(plan, Pass::Phi, Pass::Theta, in, out, Decisions{}, stream);
}

int sphfilt_apply_ex(sphfilt_plan plan, const double *in, double *out, int adjoint,
                     unsigned char *theta_dec, unsigned char *phi_dec, int replay, void *stream)
{
    if (replay && (!theta_dec || !phi_dec)) return SPHFILT_EINVAL;
    const Decisions d{theta_dec, phi_dec, replay ? 1 : 0};
    return adjoint ? apply_two(plan, Pass::Phi, Pass::Theta, in, out, d, stream)
                   : apply_two(plan, Pass::Theta, Pass::Phi, in, out, d, stream);
}

int sphfilt_apply_theta(sphfilt_plan plan, const double *in, double *out, void *stream)
{
    return apply_one(plan, Pass::Theta, in, out, stream);
}

int sphfilt_apply_phi(sphfilt_plan plan, const double *in, double *out, void *stream)
{
    return apply_one(plan, Pass::Phi, in, out, stream);
}

int sphfilt_plan_stats(sphfilt_plan plan, sphfilt_stats *out)
{
    if (!plan || !out) return SPHFILT_EINVAL;
    fill_stats(plan->n_r, plan->n_theta, plan->n_phi, plan->n_fields, plan->host, out);
    return SPHFILT_OK;
}

int sphfilt_plan_set_schedule(sphfilt_plan plan, int theta_cols, int phi_lines)
{
    if (!plan) return SPHFILT_EINVAL;
    const int tc = theta_cols ? theta_cols : plan->theta_cols;
    const int pl = phi_lines ? phi_lines : plan->phi_lines;
    if (!theta_shape_ok(2 * plan->n_theta, tc, plan->n_phi) || !phi_shape_ok(plan->n_phi, pl))
        return SPHFILT_EINVAL;
    plan->theta_cols = tc;
    plan->phi_lines = pl;
    return SPHFILT_OK;
}

int sphfilt_plan_get_schedule(sphfilt_plan plan, int *theta_cols, int *phi_lines)
{
    if (!plan) return SPHFILT_EINVAL;
    if (theta_cols) *theta_cols = plan->theta_cols;
    if (phi_lines) *phi_lines = plan->phi_lines;
    return SPHFILT_OK;
}

int sphfilt_plan_set_fused(sphfilt_plan plan, int enable)
{
    if (!plan || (enable != 0 && enable != 1)) return SPHFILT_EINVAL;
    plan->fused = enable;
    return SPHFILT_OK;
}

int sphfilt_plan_set_overlap(sphfilt_plan plan, int mode)
{
    if (!plan || mode < 0 || mode > 2) return SPHFILT_EINVAL;
    plan->overlap = mode;
    return SPHFILT_OK;
}

int sphfilt_plan_get_overlap(sphfilt_plan plan, int *mode)
{
    if (!plan || !mode) return SPHFILT_EINVAL;
    *mode = plan->overlap;
    return SPHFILT_OK;
}

int sphfilt_plan_tune(sphfilt_plan plan, const char *tune_cache_path)
{
    if (!plan) return SPHFILT_EINVAL;
    DeviceGuard g(plan->device);
    if (!g.ok) return SPHFILT_EDEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, plan->device) != hipSuccess) return SPHFILT_EDEVICE;
    std::string arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch.resize(colon);
    const char *cache = tune_cache_path ? tune_cache_path : tune_cache_default();
    if (cache) {
        TuneFields f;
        const uint64_t sig = fnv1a(plan->params_hash, arch.data(), arch.size());
        std::string what;
        PlanSched c{};
        if (tune_cache_get(cache, hex64(sig), &f) && tune_string(f, "what", &what) && what == "plan" &&
            tune_int(f, "theta_cols", &c.theta_cols) && tune_int(f, "phi_lines", &c.phi_lines) &&
            tune_int(f, "fused", &c.fused) && tune_int(f, "theta_variant", &c.theta_mfma) &&
            tune_int(f, "overlap", &c.overlap) &&
            theta_shape_ok(2 * plan->n_theta, c.theta_cols, plan->n_phi) &&
            phi_shape_ok(plan->n_phi, c.phi_lines) && (c.fused == 0 || c.fused == 1) &&
            (c.theta_mfma == 0 || (c.theta_mfma == 1 && theta_gemm_ok(plan->n_theta, plan->n_phi))) &&
            c.overlap >= 0 && c.overlap <= 2) {
            set_plan_sched(plan, c);
            if (!tune_double(f, "us", &plan->tuned_us)) plan->tuned_us = -1.0;
            if (!tune_double(f, "default_us", &plan->default_us)) plan->default_us = -1.0;
            return SPHFILT_OK;
        }
    }
    return tune_plan(plan, arch, cache);
}

int sphfilt_plan_tuned_times(sphfilt_plan plan, double *tuned_us, double *default_us)
{
    if (!plan) return SPHFILT_EINVAL;
    if (tuned_us) *tuned_us = plan->tuned_us;
    if (default_us) *default_us = plan->default_us;
    return SPHFILT_OK;
}

int sphfilt_plan_set_theta_variant(sphfilt_plan plan, int variant)
{
    if (!plan || (variant != SPHFILT_THETA_FFT && variant != SPHFILT_THETA_MFMA)) return SPHFILT_EINVAL;
    if (variant == SPHFILT_THETA_MFMA && !theta_gemm_ok(plan->n_theta, plan->n_phi))
        return SPHFILT_EUNSUPPORTED;
    plan->theta_mfma = variant == SPHFILT_THETA_MFMA;
    return SPHFILT_OK;
}

int sphfilt_plan_get_theta_variant(sphfilt_plan plan, int *variant)
{
    if (!plan || !variant) return SPHFILT_EINVAL;
    *variant = plan->theta_mfma ? SPHFILT_THETA_MFMA : SPHFILT_THETA_FFT;
    return SPHFILT_OK;
}

int sphfilt_plan_get_fused(sphfilt_plan plan, int *enable, int *shells_fused)
{
    if (!plan) return SPHFILT_EINVAL;
    if (enable) *enable = plan->fused;
    if (shells_fused) *shells_fused = plan->fused ? plan->host.n_fused : 0;
    return SPHFILT_OK;
}

const char *sphfilt_status_string(int status)
{
    switch (status) {
    case SPHFILT_OK: return "ok";
    case SPHFILT_EINVAL: return "invalid argument";
    case SPHFILT_ENOMEM: return "out of memory";
    case SPHFILT_EDEVICE: return "HIP device or launch error";
    case SPHFILT_EUNSUPPORTED: return "size not supported by the library";
    default: return "unknown status";
    }
}

const char *sphfilt_version(void) { return "0.1.0"; }

}  // extern "C"
