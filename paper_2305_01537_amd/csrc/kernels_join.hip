// kernels_join.hip -- kernels that run both passes of whole shells in registers
// (shell_join.h), per plan and per batch, double FFT filter
// (arXiv:2305.01537, Sec. II.A) for gfx950, FP64.
#include "batch_internal.h"
#include "shell_join.h"

namespace sphfilt {

// Waves per SIMD asked for, as many as the workgroups that fit a compute
// unit's LDS hold: the register cap is 512 / waves.
template <int N, bool HYB = false>
constexpr int join_waves()
{
    return N == 256 || (N == 128 && !HYB) ? 4 : 3;
}

// The twiddle table into LDS, before any use of it.
template <int N>
__device__ __forceinline__ void stage_table(const Twiddle *__restrict__ tw, Twiddle *table)
{
    for (int i = threadIdx.x; i < JoinShape<N>::table; i += JoinShape<N>::width) table[i] = tw[i];
    __syncthreads();
}

// One workgroup's shells, the kind picked for all of them where it can be.
template <int N, bool ADJ, bool HYB = false>
__device__ __forceinline__ void join_group(const double *in, double *out, const ThetaItem *__restrict__ shells,
                                           const double *__restrict__ ring_c, int n_valid,
                                           const Twiddle *table, double *lds,
                                           const HybridArgs &ht = HybridArgs{},
                                           const HybridArgs &hp = HybridArgs{})
{
    using S = JoinShape<N>;
    auto run = [&](auto kind) {
        join_block<N, ADJ, decltype(kind)::value>(in, out, shells, ring_c, n_valid, table, lds, ht, hp);
    };
    if constexpr (HYB) {
        run(std::integral_constant<int, 3>{});
    } else if constexpr (S::shells > 1) {
        run(std::integral_constant<int, -1>{});
    } else {
        // one shell per workgroup: one kind, and no registers held across the
        // branches between the kinds' masks
        const int kind = shells[0].flags & kKindMask;
        if (kind == 0) run(std::integral_constant<int, 0>{});
        else if (kind == 1) run(std::integral_constant<int, 1>{});
        else run(std::integral_constant<int, 2>{});
    }
}

// Shells and, in the same grid, ring pairs of other shells (as many as a
// workgroup's lanes hold).  What bounds it: at 256 points a workgroup is a
// whole compute unit, 25 us of which half is FP64 issue (1,600 instructions
// per wave and pass, 40 % of the issue slots), a quarter waits for the load and
// the store, and the LDS is busy for a third; nothing else runs on the unit
// meanwhile.  Against two passes, whose bound is HBM: 24 x 256 shells of
// 128 x 256, all filtered, 1090 -> 745 us forward (4.3 TB/s of 16 B per point),
// 1095 -> 750 adjoint; at cal-L = 3, 187 -> 150.  Shorter lines fit two to six
// workgroups per unit and come near the bandwidth: all filtered, 24 x 3600
// shells of 24 x 48 755 -> 365 us, 24 x 1300 of 40 x 80 723 -> 499, 24 x 900 of
// 48 x 96 577 -> 346, 24 x 508 of 64 x 128 412 -> 331 (in LDS before), 24 x 160 of
// 80 x 160 307 -> 232, 24 x 128 of 96 x 192 333 -> 238.  At 128 points six registers
// (eight in batches) spill under the cap of four waves.
template <int N, bool ADJ>
__global__ __launch_bounds__(JoinShape<N>::width) __attribute__((amdgpu_waves_per_eu(join_waves<N>())))
void join_kernel(const double *in, double *out, const ThetaItem *__restrict__ shells,
                 const double *__restrict__ ring_c, int n_shells, int shell_groups, int span, int total,
                 const PhiItem *__restrict__ rings, int n_rings, const Twiddle *__restrict__ tw)
{
    using S = JoinShape<N>;
    __shared__ double lds[S::lds];
    __shared__ Twiddle table[S::table];
    stage_table<N>(tw, table);
    // the shell groups are spread evenly over the first `span` items
    for (int b = blockIdx.x; b < total; b += gridDim.x) {
        const int group = b < span ? (int)((long long)b * shell_groups / span) : shell_groups;
        const bool ring = b >= span || (int)((long long)(b + 1) * shell_groups / span) == group;
        if (ring) {
            constexpr int LINES = S::width / S::N2;
            const int first = (b - group) * LINES;
            phi_block<N, LINES, false, true>(in, out, rings + first, min(LINES, n_rings - first), N / 2,
                                             tw, lds, nullptr, HybridArgs{}, join_lane());
        } else {
            const int first = group * S::shells;
            join_group<N, ADJ>(in, out, shells + first, ring_c + (size_t)first * S::lines,
                               min(S::shells, n_shells - first), table, lds);
        }
    }
}

// Hybrid shells only: the detector runs on the registers, in both layouts.  A
// third of the 24 fields hybrid, against two passes: 128 shells of 24 x 48 38.5
// -> 25 us, of 48 x 96 71 -> 44, of 64 x 128 81 -> 70 (against the form through
// LDS), of 40 x 80 63 -> 53, of 96 x 192 222 -> 195, 160 of 80 x 160 171 -> 152.
template <int N, bool ADJ>
__global__ __launch_bounds__(JoinShape<N>::width) __attribute__((amdgpu_waves_per_eu(join_waves<N, true>())))
void join_hybrid_kernel(const double *in, double *out, const ThetaItem *__restrict__ shells,
                        const double *__restrict__ ring_c, int n_shells,
                        const Twiddle *__restrict__ tw, HybridArgs ht, HybridArgs hp)
{
    using S = JoinShape<N>;
    __shared__ double lds[S::lds];
    __shared__ Twiddle table[S::table];
    stage_table<N>(tw, table);
    const int first = blockIdx.x * S::shells;
    join_group<N, ADJ, true>(in, out, shells + first, ring_c + (size_t)first * S::lines,
                             min(S::shells, n_shells - first), table, lds, ht, hp);
}

// The same for a batch, over its list of items.
template <int N, bool ADJ>
__global__ __launch_bounds__(JoinShape<N>::width) __attribute__((amdgpu_waves_per_eu(join_waves<N>())))
void batch_join_kernel(const BatchWork *__restrict__ work, int n_work, const double *const *ins, double *const *outs,
                       const ThetaItem *__restrict__ th, const PhiItem *__restrict__ ph,
                       const double *__restrict__ fc, const Twiddle *__restrict__ tw)
{
    using S = JoinShape<N>;
    __shared__ double lds[S::lds];
    __shared__ Twiddle table[S::table];
    stage_table<N>(tw, table);
    for (int k = blockIdx.x; k < n_work; k += gridDim.x) {
        const BatchWork w = work[k];
        const double *in = ins[w.patch];
        double *out = outs[w.patch];
        if (w.pass == 1)
            phi_block<N, S::width / S::N2, false, true>(in, out, ph + w.first, w.n_valid, N / 2, tw, lds,
                                                        nullptr, HybridArgs{}, join_lane());
        else
            join_group<N, ADJ>(in, out, th + w.first, fc + w.aux, w.n_valid, table, lds);
    }
}

// Workgroups of a launch over `total` items.  One per item, except where one
// workgroup fills a compute unit and every unit gets eight items or more: then
// one per unit, which takes every grid-th item.  Its waves go on to the next
// item's loads as they finish their own part of the last, which a new
// workgroup cannot do before all of them have (6144 shells of 128 x 256, all
// filtered, 787 -> 737 us forward, 831 -> 744 adjoint; 3840 of 80 x 160 261 ->
// 229; 3072 of 96 x 192 265 -> 233).  With fewer items the units end unevenly
// (1024 items: 95.6 -> 100.5 us; 1362: 154 -> 155).
template <int N>
static unsigned join_grid(int total, int compute_units)
{
    return (unsigned)(N >= 160 && compute_units > 0 && total >= 8 * compute_units ? compute_units : total);
}

template <int N>
static hipError_t join_go(bool adjoint, const double *in, double *out, const ThetaItem *shells,
                          const double *ring_c, int n_shells, const PhiItem *rings, int n_rings,
                          int compute_units, const Twiddle *tw, hipStream_t s)
{
    using S = JoinShape<N>;
    constexpr int LINES = S::width / S::N2;
    const int groups = (n_shells + S::shells - 1) / S::shells;
    const int ring_groups = (n_rings + LINES - 1) / LINES;
    const int total = groups + ring_groups;
    const dim3 grid(join_grid<N>(total, compute_units)), block(S::width);
    const int span = groups + (join_spread(N, n_rings, compute_units) ? ring_groups * 4 / 5 : 0);
    if (adjoint)
        join_kernel<N, true><<<grid, block, 0, s>>>(in, out, shells, ring_c, n_shells, groups, span, total, rings, n_rings, tw);
    else
        join_kernel<N, false><<<grid, block, 0, s>>>(in, out, shells, ring_c, n_shells, groups, span, total, rings, n_rings, tw);
    return hipGetLastError();
}

namespace {
// f(std::integral_constant<int, N>) for the line length n_line
template <typename F>
auto with_line(int n_line, F &&f)
{
    switch (n_line) {
    case 32: return f(std::integral_constant<int, 32>{});
    case 48: return f(std::integral_constant<int, 48>{});
    case 64: return f(std::integral_constant<int, 64>{});
    case 80: return f(std::integral_constant<int, 80>{});
    case 96: return f(std::integral_constant<int, 96>{});
    case 128: return f(std::integral_constant<int, 128>{});
    case 160: return f(std::integral_constant<int, 160>{});
    case 192: return f(std::integral_constant<int, 192>{});
    default: return f(std::integral_constant<int, 256>{});
    }
}
}  // namespace

bool join_supported(int n_theta, int n_phi)
{
    return n_phi == 2 * n_theta && (n_phi == 48 || n_phi == 80 || n_phi == 96 || n_phi == 160 ||
                                    n_phi == 192 || n_phi == 256);
}

// Lines of 160 points and more: one workgroup fills a compute unit, so a launch
// runs in rounds of one shell per unit, and a last round that leaves most units
// idle costs as much as a full one, where two passes spread few shells over
// all units.  Two passes against a round, us, for 96 / 128 / 192 shells: 24.8 /
// 28.4 / 37.4 against 30.0 / 30.6 / 34.0 at 256 points, 18.7 / 20.1 / 26.4
// against 21.0 / 21.2 / 22.0 at 192, 16.1 / 17.6 / 19.8 against 17.4 / 17.9 /
// 18.6 at 160: the line lies at 9/16 of the units.  Where the ring pairs of
// other shells fill the units by themselves (join_spread) no round is short.
// Shorter lines fit several workgroups per unit and are joined always (96
// points, 4 shells: 8.7 against 10.8 us).
int join_count(int n_line, int n, int n_rings, int compute_units)
{
    if (n_line < 160 || compute_units <= 0 || join_spread(n_line, n_rings, compute_units)) return n;
    const int last = n % compute_units;
    return 16 * last < 9 * compute_units ? n - last : n;
}

// Whether to spread the shells among the ring workgroups of their launch (the
// first 4/5 of them) instead of putting them first.  A unit that holds a shell
// computes for most of its time while the ring workgroups wait for memory, so
// spread shells overlap the two; but they also start later, which pays only
// where the rings run for several rounds: from two full rounds on (24 x 256
// shells of 128 x 256 at cal-L = 3, 3.4 rounds: 157 us spread, 176 shells
// first, 166 as two launches: of an earlier form, 150 now; 24 x 128 of 96 x 192 at
// cal-L = 2, 2.6 rounds:
// 88 / 93 / 102; 24 x 160 of 80 x 160 at cal-L = 4, 1.7 rounds: 43 / 40 / 42).
bool join_spread(int n_line, int n_rings, int compute_units)
{
    const int lines = n_line == 256 ? JoinShape<256>::width / JoinShape<256>::N2
                      : n_line == 192 ? JoinShape<192>::width / JoinShape<192>::N2
                      : n_line == 160 ? JoinShape<160>::width / JoinShape<160>::N2
                                      : 0;
    return lines > 0 && n_rings >= 2 * compute_units * lines;
}

hipError_t launch_join(bool adjoint, int n_line, const double *in, double *out,
                       const ThetaItem *shells, const double *ring_c, int n_shells,
                       const PhiItem *rings, int n_rings, int compute_units, const Twiddle *tw, hipStream_t s)
{
    if (n_shells < 0 || n_rings < 0) return hipErrorInvalidValue;
    if (n_shells + n_rings == 0) return hipSuccess;
    switch (n_line) {
    case 48: return join_go<48>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 80: return join_go<80>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 96: return join_go<96>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 128: return join_go<128>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 160: return join_go<160>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 192: return join_go<192>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    case 256: return join_go<256>(adjoint, in, out, shells, ring_c, n_shells, rings, n_rings, compute_units, tw, s);
    default: return hipErrorInvalidValue;
    }
}

int join_group_shells(int n_line)
{
    return with_line(n_line, [](auto n) { return JoinShape<decltype(n)::value>::shells; });
}

int join_group_rings(int n_line)
{
    return with_line(n_line, [](auto n) {
        using S = JoinShape<decltype(n)::value>;
        return S::width / S::N2;
    });
}

hipError_t launch_batch_join(int n_line, bool adjoint, const BatchWork *work, int n_work,
                             const double *const *ins, double *const *outs, const ThetaItem *th,
                             const PhiItem *ph, const double *fc, const Twiddle *tw,
                             int compute_units, hipStream_t s)
{
    if (n_work <= 0) return hipSuccess;
    return with_line(n_line, [&](auto n) {
        constexpr int N = decltype(n)::value;
        const dim3 grid(join_grid<N>(n_work, compute_units)), block(JoinShape<N>::width);
        if (adjoint)
            batch_join_kernel<N, true><<<grid, block, 0, s>>>(work, n_work, ins, outs, th, ph, fc, tw);
        else
            batch_join_kernel<N, false><<<grid, block, 0, s>>>(work, n_work, ins, outs, th, ph, fc, tw);
        return hipGetLastError();
    });
}

hipError_t launch_join_hybrid(bool adjoint, int n_line, const double *in, double *out,
                              const ThetaItem *shells, const double *ring_c, int n_shells,
                              const Twiddle *tw, const HybridArgs &ht, const HybridArgs &hp,
                              hipStream_t s)
{
    if (n_shells <= 0) return hipSuccess;
    return with_line(n_line, [&](auto n) -> hipError_t {
        constexpr int N = decltype(n)::value;
        using S = JoinShape<N>;
        if constexpr (N == 256 || N == 64 || N == 32) {   // two passes; the fused kernel through LDS
            return hipErrorInvalidValue;
        } else {
            const dim3 grid((unsigned)((n_shells + S::shells - 1) / S::shells)), block(S::width);
            if (adjoint)
                join_hybrid_kernel<N, true><<<grid, block, 0, s>>>(in, out, shells, ring_c, n_shells, tw, ht, hp);
            else
                join_hybrid_kernel<N, false><<<grid, block, 0, s>>>(in, out, shells, ring_c, n_shells, tw, ht, hp);
            return hipGetLastError();
        }
    });
}

}  // namespace sphfilt
