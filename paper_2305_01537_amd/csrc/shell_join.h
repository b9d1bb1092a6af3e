// shell_join.h -- whole shells in registers: both passes of the double FFT
// filter (arXiv:2305.01537, Sec. II.A) with one HBM round trip, on grids with
// n_phi = 2 n_theta = N (device side).
//
// A shell (field, radius) has N/4 complex theta lines (adjacent meridian pairs
// 2q and 2q + 1) and N/4 complex phi lines (ring pairs j and n_theta-1-j), all
// of length N and on one cutoff each.  A workgroup of N/4 lines of N2 lanes
// holds the whole shell in its registers (N1 complex values per lane, 256 KB
// at N = 256: half of a compute unit's register file), filters its theta
// lines, changes from the theta layout to the phi layout through LDS, filters
// the rings and stores them (the adjoint order mirrors this).  A line's lanes
// are consecutive lanes of one wave in both layouts, so the line filter
// synchronises the wave only and the waves drift apart; the exchange between
// the layouts takes two workgroup barriers per round.  The LDS holds the lines'
// transpose scratch and, in between, the exchange: the whole shell where it
// fits beside the other workgroups of the compute unit, else half of it at a
// time (Rounds): a round's lines are written by the waves that own them and
// read, in part, by every wave.
#pragma once
#include "line_filter.h"

namespace sphfilt {

template <int N> struct JoinShape {
    static constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2;
    static constexpr int lines = N / 4;                  // complex lines per shell and pass
    static constexpr int lanes = lines * N2;             // lanes per shell
    static constexpr int rounds = N == 256 || N == 128 ? 2 : N == 96 ? 3 : 1;
    // whole waves: shells per workgroup
    static constexpr int shells = lanes % 64 == 0 ? 1 : lanes % 32 == 0 ? 2 : 4;
    static constexpr int width = shells * lanes;
    // theta -> phi: all rows, the columns of a round's lines; phi -> theta: the
    // rows of a round's lines, all columns.  Row strides are 2 modulo 4 doubles,
    // so that eight lanes' 16-byte accesses to consecutive rows, and sixteen
    // lanes' accesses along a row, touch all banks once.
    static constexpr int fwd_stride = N / rounds + 2, fwd_shell = N / 2 * fwd_stride;
    static constexpr int adj_stride = N + 2, adj_shell = N / 2 / rounds * adj_stride;
    static constexpr int exchange = shells * (fwd_shell > adj_shell ? fwd_shell : adj_shell);
    static constexpr int scratch = width / N2 * line_lds<N1, N2>();
    static constexpr int lds = exchange > scratch ? exchange : scratch;
    static constexpr int table = N + N / 4;              // entries of the twiddle table
    static_assert(width % 64 == 0 && width <= 1024, "whole waves");
    static_assert(rounds == 1 || (lines / rounds * N2) % 64 == 0, "a round's lines are whole waves'");
};

// Loads in the theta layout cover 64-byte pieces of 128-byte lines where a line
// has 16 lanes (two waves share each 128-byte line: through the cache, 837
// against 933 us for 6144 shells of 128 x 256 streamed) and whole lines where
// it has 8 or 4 (streamed, 1-2 % faster).
template <int N>
constexpr bool join_theta_cached() { return Split<N>::N2 == 16; }

// The theta layout straight from / to HBM: lane t of line q moves rows N2 n1 + t
// of meridians 2q, 2q + 1 and, in the mirrored half, of those half a turn
// away, two adjacent doubles per access.
template <int N, bool LOAD>
__device__ __forceinline__ void join_theta_hbm(const double *in, double *out, cplx (&v)[Split<N>::NV],
                                               int t, int q, double s)
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2, half = N / 2;
    const int first = t * N + 2 * q, mirrored = (N2 - 1 - t) * N + half + 2 * q;
    static_for<0, N1>([&](auto nn) {
        constexpr int n1 = decltype(nn)::value;
        constexpr bool top = n1 < N1 / 2;
        constexpr int row = top ? N2 * n1 * N : (N - N2 * (n1 + 1)) * N;
        const int off = top ? first : mirrored;
        if constexpr (LOAD) {
            v[n1] = ld_pair<join_theta_cached<N>()>(in + row + off);
        } else {
            st_pair<false>(out + row + off, top ? v[n1].re : s * v[n1].re, top ? v[n1].im : s * v[n1].im);
        }
    });
    if constexpr (LOAD)
        static_for<N1 / 2, N1>([&](auto nn) {
            constexpr int n1 = decltype(nn)::value;
            v[n1] = cplx{s * v[n1].re, s * v[n1].im};
        });
}

// The phi layout: lane t of line j moves x[N2 n1 + t] of rings j and N/2-1-j.
template <int N, bool LOAD>
__device__ __forceinline__ void join_phi_hbm(const double *in, double *out, cplx (&v)[Split<N>::NV],
                                             int t, int j)
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2;
    const int a = j * N + t, b = (N / 2 - 1 - j) * N + t;
    static_for<0, N1>([&](auto nn) {
        constexpr int n1 = decltype(nn)::value;
        if constexpr (LOAD) {
            v[n1] = cplx{ld_piece<true>(in + a + N2 * n1), ld_piece<true>(in + b + N2 * n1)};
        } else {
            st_stream<ring_stores_streamed<N>()>(out + a + N2 * n1, v[n1].re);
            st_stream<ring_stores_streamed<N>()>(out + b + N2 * n1, v[n1].im);
        }
    });
}

// From the theta layout (v) to the phi layout (w): round h moves the columns
// of theta lines [h lines/rounds, (h+1) lines/rounds).  Begins and ends with a
// workgroup barrier.  sb: the shell's exchange area; line: the lane's line of
// its shell, in both layouts.
template <int N>
__device__ __forceinline__ void join_theta_to_phi(const cplx (&v)[Split<N>::NV],
                                                  cplx (&w)[Split<N>::NV], int t, int line,
                                                  double s, double *sb)
{
    using S = JoinShape<N>;
    constexpr int N1 = S::N1, N2 = S::N2, per = S::lines / S::rounds, half_cols = N / 2 / S::rounds;
    __syncthreads();
    static_for<0, S::rounds>([&](auto hh) {
        constexpr int h = decltype(hh)::value;
        if (S::rounds == 1 || line / per == h) {                     // wave-uniform
            double *col = sb + 2 * (line - h * per);
            static_for<0, N1>([&](auto nn) {
                constexpr int n1 = decltype(nn)::value;
                constexpr bool top = n1 < N1 / 2;
                double *r = top ? col + (N2 * n1 + t) * S::fwd_stride
                                : col + (N - 1 - N2 * n1 - t) * S::fwd_stride + half_cols;
                st_pair<false>(r, top ? v[n1].re : s * v[n1].re, top ? v[n1].im : s * v[n1].im);
            });
        }
        __syncthreads();
        const double *ra = sb + line * S::fwd_stride + t, *rb = sb + (N / 2 - 1 - line) * S::fwd_stride + t;
        static_for<0, N1>([&](auto nn) {
            constexpr int n1 = decltype(nn)::value;
            constexpr int m = n1 % (N1 / 2), mine = N1 / 2 / S::rounds;
            if constexpr (m / mine == h) {
                constexpr int c = n1 / (N1 / 2) * half_cols + N2 * (m - h * mine);
                w[n1] = cplx{ra[c], rb[c]};
            }
        });
        __syncthreads();
    });
}

// From the phi layout (v) to the theta layout (w): round h moves the rows of
// phi lines [h lines/rounds, (h+1) lines/rounds).
template <int N>
__device__ __forceinline__ void join_phi_to_theta(const cplx (&v)[Split<N>::NV],
                                                  cplx (&w)[Split<N>::NV], int t, int line,
                                                  double s, double *sb)
{
    using S = JoinShape<N>;
    constexpr int N1 = S::N1, N2 = S::N2, per = S::lines / S::rounds;
    __syncthreads();
    static_for<0, S::rounds>([&](auto hh) {
        constexpr int h = decltype(hh)::value;
        if (S::rounds == 1 || line / per == h) {                     // wave-uniform
            const int jl = line - h * per;
            double *ra = sb + jl * S::adj_stride + t, *rb = sb + (2 * per - 1 - jl) * S::adj_stride + t;
            static_for<0, N1>([&](auto nn) {
                constexpr int n1 = decltype(nn)::value;
                ra[N2 * n1] = v[n1].re;
                rb[N2 * n1] = v[n1].im;
            });
        }
        __syncthreads();
        const double *top_row = sb + t * S::adj_stride + 2 * line;
        const double *bot_row = sb + (N2 - 1 - t) * S::adj_stride + N / 2 + 2 * line;
        static_for<0, N1>([&](auto nn) {
            constexpr int n1 = decltype(nn)::value;
            constexpr bool top = n1 < N1 / 2;
            constexpr int b = top ? n1 : N1 - 1 - n1;                // block of N2 rows
            if constexpr (S::rounds == 1) {
                const cplx x = ld_pair<true>((top ? top_row : bot_row) + N2 * b * S::adj_stride);
                w[n1] = top ? x : cplx{s * x.re, s * x.im};
            } else {
                constexpr int jb = b < N1 / 4 ? b : N1 / 2 - 1 - b;  // of the ring pairs' blocks
                constexpr int mine = N1 / 4 / S::rounds;
                if constexpr (jb / mine == h) {
                    constexpr int lb = b < N1 / 4 ? b - h * mine : b - N1 / 2 + (h + 2) * mine;
                    const cplx x = ld_pair<true>((top ? top_row : bot_row) + N2 * lb * S::adj_stride);
                    w[n1] = top ? x : cplx{s * x.re, s * x.im};
                }
            }
        });
        __syncthreads();
    });
}

// The lane index, re-read through an opaque move: index math is redone where
// it is used instead of held across a line filter.
__device__ __forceinline__ int join_lane()
{
    unsigned v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "v"((unsigned)threadIdx.x));
    return (int)v;
}

// One workgroup: shells items[0, n_valid), n_valid <= JoinShape<N>::shells,
// with ring cutoffs ring_c[shell][j].  tw: the twiddle table in LDS.  A wave
// may start on its next item when it is done: until that item's exchange, which
// begins with a barrier, it only touches its own lines' scratch.  KIND: the kind of
// every item, or -1 for plain kinds taken from the items; ht and hp: the
// hybrid arguments of the two passes, for KIND 3.
template <int N, bool ADJ, int KIND>
__device__ __forceinline__ void join_block(const double *in, double *out,
                                           const ThetaItem *__restrict__ items,
                                           const double *__restrict__ ring_c, int n_valid,
                                           const Twiddle *tw, double *lds, const HybridArgs &ht,
                                           const HybridArgs &hp)
{
    using S = JoinShape<N>;
    constexpr int N1 = S::N1, N2 = S::N2;
    constexpr size_t shell_pts = (size_t)N * N / 2;
    constexpr int shell_exchange = ADJ ? S::adj_shell : S::fwd_shell;
    cplx v[Split<N>::NV], w[Split<N>::NV];
    // a workgroup's spare shells repeat the last one's loads and store nothing
    auto shell_of = [&](int lane) { return S::shells == 1 ? 0 : min(lane / S::lanes, n_valid - 1); };
    auto sign = [&](int u) { return (items[u].flags & kFlagOddParity) ? -1.0 : 1.0; };
    {
        const int lane = join_lane(), t = lane % N2, line = lane / N2 % S::lines, u = shell_of(lane);
        const double *src = in + (size_t)items[u].shell * shell_pts;
        if constexpr (ADJ)
            join_phi_hbm<N, true>(src, nullptr, v, t, line);
        else
            join_theta_hbm<N, true>(src, nullptr, v, t, line, sign(u));
    }
    auto filter = [&](cplx (&x)[Split<N>::NV], bool theta) {
        const int lane = join_lane(), t = lane % N2, line = lane / N2 % S::lines, u = shell_of(lane);
        const double c = theta ? items[u].c : ring_c[u * S::lines + line];
        double *L = lds + lane / N2 * line_lds<N1, N2>();
        if constexpr (KIND == 3) {
            // the decisions' bytes: meridian pairs 2q and 2q + 1, or rings j and
            // N/2 - 1 - j, of the shell
            const size_t first = (size_t)items[u].shell * (size_t)(N / 2);
            const size_t a = first + (theta ? 2 * line : line);
            const size_t b = theta ? a + 1 : first + (size_t)(N / 2 - 1 - line);
            int ka = 3, kb = 3;
            bool mixed = false;
            hybrid_kinds<N1, N2, true>(x, t, L, nullptr, 0, 0, true, 3, a, b, theta ? ht : hp, &ka, &kb,
                                       &mixed);
            filter_line<N1, N2, true, true, true>(x, t, ka & 1, kb & 1, mixed, c, L, tw);
        } else {
            filter_line<N1, N2, false, true, true>(x, t, KIND >= 0 ? KIND : items[u].flags & kKindMask,
                                                   0, false, c, L, tw);
        }
    };
    filter(v, !ADJ);
    {
        const int lane = join_lane(), t = lane % N2, line = lane / N2 % S::lines, u = shell_of(lane);
        double *sb = lds + (S::shells == 1 ? 0 : lane / S::lanes) * shell_exchange;
        if constexpr (ADJ)
            join_phi_to_theta<N>(v, w, t, line, sign(u), sb);
        else
            join_theta_to_phi<N>(v, w, t, line, sign(u), sb);
    }
    filter(w, ADJ);
    {
        const int lane = join_lane(), t = lane % N2, line = lane / N2 % S::lines, u = shell_of(lane);
        double *dst = out + (size_t)items[u].shell * shell_pts;
        if (S::shells == 1 || lane / S::lanes < n_valid) {
            if constexpr (ADJ)
                join_theta_hbm<N, false>(nullptr, dst, w, t, line, sign(u));
            else
                join_phi_hbm<N, false>(nullptr, dst, w, t, line);
        }
    }
}

}  // namespace sphfilt
