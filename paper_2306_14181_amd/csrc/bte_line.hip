// bte_line.hip -- one-dimensional geometries: the forward steady sweep of a
// whole line in one launch and the explicit step that leaves T_L behind.
//
// A line is short and a chip wide, so both kernels spread a line's cells over
// the wavefronts of a block (one cell after another in time costs a memory or
// arithmetic latency per cell): the sweep's recurrence
//   de_i = (b_i + cp de_{i-1}) / (cp + 1/tau + gamma_i)
// is solved by each thread for its few cells with no inflow, together with
// the factor by which an inflow would pass them, and the pieces are joined
// by a scan.
#include "bte_internal.h"
#include "bte_stencil.h"
#include "bte_tilelds.h"
#include "bte_col3d.h"

namespace bte {
namespace {

constexpr int kSeg = 4;          // cells of a thread
constexpr int LW = 16;           // lanes of a sweep's block
constexpr int kLineThreads = 1024;
constexpr int kFold = 4;         // groups of lanes of a folded block
constexpr int kStepThreads = 512;
constexpr int kStepCells = 64;   // most cells of an explicit step's block

// What a thread needs to know of a cell of the line, staged per block.
struct LineCell {
    int cell;        // global cell, -1 outside the line
    uint32_t code;   // its code (0 outside)
    double x;        // pending correction and periodic jump (units of C/Omega; 0 in pores)
};

__device__ inline LineCell line_cell(const Dev &d, const Film &fm, int i, const double *__restrict__ dpend)
{
    int jump;
    const int ci = wrap_pos(i, fm.n[0], fm.periodic[0], jump);
    LineCell r{-1, 0u, 0.0};
    if (ci >= 0) {
        r.cell = fm.cell0 + ci;
        r.code = d.code[r.cell];
        if (r.code & kSolidBit) r.x = (dpend ? dpend[r.cell] : 0.0) + jump * fm.pdT[0];
    }
    return r;
}

// Face-value difference of a solid cell whose upwind, second upwind and
// downwind cells are u1, u2 and dn.
template <typename T, int LIM>
__device__ inline T line_delta(const Dev &d, const Film &fm, const T *__restrict__ e, const double *__restrict__ din,
                               const LineCell &me, uint32_t code2, const LineCell &dn, int sg, const LaneT<T> &L,
                               T e2, T e1, T ec, T ed)
{
    const uint32_t ab = axis_bits(me.code, 0);
    const bool hu = side_is_cell(ab, -sg), hd = side_is_cell(ab, sg), hu2 = hu && (code2 & kSolidBit);
    if (hu && hd && hu2) return delta_fast<T, LIM>(e2, e1, ec, ed);
    return delta_wall3<T, LIM>(d, fm, e, din, me.cell, me.code, 0, sg, hu, hu2, hd, e2, e1, ec, ed, dn.cell,
                               L.C4 * (T)dn.x, L.al, L.l, L.C4, L.hh[0], L.ih[0], L.C4 * (T)me.x);
}

// n / d, 1/d at hand: the quotient of the reciprocal and one correction
__device__ inline double quot(double n, double d, double inv)
{
    const double q = n * inv;
    return fma(fma(-q, d, n), inv, q);
}
__device__ inline float quot(float n, float, float inv) { return n * inv; }
__device__ inline double recip(double d) { return 1.0 / d; }
__device__ inline float recip(float d) { return __builtin_amdgcn_rcpf(d); }

// What an inflow x adds behind cells that pass it by the factor a: nothing where
// a is zero (a pore, an end, damped below the smallest number), whatever x is.
template <typename T> __device__ inline T inflow(T a, T x) { return a * (a != (T)0 ? x : (T)0); }

// Forward sweep of a line.  Block (geometry, octant, group of 16 lanes); the
// lanes by 4 runs of kSeg cells in a wavefront, a round of (wavefronts) x 4 x
// kSeg cells at a time, the last increment of a round handed to the next.
// Bound by latency: a round is one load of its cells, kSeg steps of the
// recurrence, a scan over the block and the moment sums.  FP64, a sweep of
// one line of 200 cells x 80 lanes, of 1000 x 1280, of 256 lines of 200 x 80:
// 152, 578 and 576 us with a launch per tile of 64 cells x 64 lanes, 20, 43
// and 98 us here (38, 127 and 132 us with 64 lanes a block: a quarter of the
// wavefronts on a line).  FOLD: a block takes four groups of lanes one after
// another and adds their moments (line_fold).
template <typename T, int LIM, bool FOLD>
__global__ __launch_bounds__(kLineThreads) void k_sweep1d(Dev d, const T *__restrict__ ein, T *__restrict__ eout,
                                                          const double *__restrict__ dpend,
                                                          const double *__restrict__ TLdev,
                                                          const double *__restrict__ din, int na_oct, int nparts,
                                                          double *__restrict__ part)
{
    constexpr int NS = 64 / LW, kCells = kLineThreads / LW * kSeg;
    __shared__ LineCell tab[kCells + 3];                  // flow positions f0 - 2 .. f0 + round
    __shared__ double tl[kCells], gam[kCells], qs[kCells];
    __shared__ T totA[kLineThreads / 64][LW], totB[kLineThreads / 64][LW];
    const int film = blockIdx.x / (2 * nparts), oct = (int)(blockIdx.x / nparts) & 1, gpart = blockIdx.x % nparts;
    if (d.nfilm > 1 && d.fdone[film]) return;             // converged geometry of a batch (uniform)
    const Film &fm = d.film[film];
    const int n = fm.n[0];
    const int wave = threadIdx.x >> 6, nwave = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane / LW, kl = lane % LW;
    const int kbeg = oct * na_oct * d.nl, kend = kbeg + na_oct * d.nl;
    const int sg = octant_sign(d, oct, na_oct, 0);
    const int q0 = (wave * NS + sub) * kSeg, round = nwave * NS * kSeg;
    const T *zrow = static_cast<const T *>(d.zrow);
    const int pidx = oct * nparts + gpart;
    for (int grp = 0; grp < (FOLD ? kFold : 1); ++grp) {
        const int k0 = kbeg + (gpart * (FOLD ? kFold : 1) + grp) * LW, k = k0 + kl;
        if (FOLD && k0 >= kend) break;
        const bool active = k < kend;
        const int kk = active ? k : kbeg;
        const LaneT<T> L = lane_make<T>(d, fm, kk);
        T carry = (T)0;
        for (int f0 = 0; f0 < n; f0 += round) {
            for (int q = threadIdx.x; q < round + 3; q += blockDim.x) {
                const int f = f0 + q - 2;
                LineCell t{-1, 0u, 0.0};
                if (f <= n) t = line_cell(d, fm, sg > 0 ? f : n - 1 - f, dpend);
                tab[q] = t;
                if (q >= 2 && q < round + 2 && f < n) {
                    tl[q - 2] = TLdev[t.cell];
                    gam[q - 2] = d.gamma[t.cell];
                    qs[q - 2] = d.P ? d.P[t.cell] / fm.Ctot : 0.0;
                }
            }
            __syncthreads();
            T v[kSeg + 3], b[kSeg], g[kSeg];
    #pragma unroll
            for (int j = 0; j < kSeg + 3; ++j) {
                const int c = tab[q0 + j].cell;
                const T *row = c >= 0 ? ein + (size_t)c * d.nk : zrow;
                v[j] = row[kk];
            }
    #pragma unroll
            for (int j = 0; j < kSeg + 3; ++j) v[j] += L.C4 * (T)tab[q0 + j].x;
            // increments without inflow into the segment, and the factor of an inflow
            T de = (T)0, pass = (T)1;
    #pragma unroll
            for (int j = 0; j < kSeg; ++j) {
                const LineCell me = tab[q0 + j + 2];
                b[j] = (T)0;
                g[j] = (T)0;
                if (f0 + q0 + j < n && (me.code & kSolidBit)) {
                    const T ec = v[j + 2];
                    const uint32_t ab = axis_bits(me.code, 0);
                    const T D = L.cpl[0] * line_delta<T, LIM>(d, fm, ein, din, me, tab[q0 + j].code, tab[q0 + j + 3], sg,
                                                              L, v[j], v[j + 1], ec, v[j + 3]);
                    const T ga = (T)gam[q0 + j], itc = L.itau + ga;
                    const T rhs = -D - (ec - L.C4 * (T)tl[q0 + j]) * itc + L.C4 * (T)qs[q0 + j];
                    // a wall, a pore or a periodic face (lagged) upwind: no coupling
                    const T cp = side_is_cell(ab, -sg) && !side_wraps(ab, -sg) ? L.cpl[0] : (T)0;
                    const T den = L.cpl[0] + L.itau + ga, inv = recip(den);
                    b[j] = quot(rhs + cp * de, den, inv);
                    g[j] = quot(cp * pass, den, inv);
                }
                de = b[j];
                pass = g[j];
            }
            // join: runs of the wavefront, then wavefronts
            T A = pass, Bv = de;
    #pragma unroll
            for (int o = LW; o < 64; o *= 2) {
                const T Ap = __shfl_up(A, o, 64), Bp = __shfl_up(Bv, o, 64);
                if (lane >= o) {
                    Bv += inflow(A, Bp);
                    A *= Ap;
                }
            }
            if (sub == NS - 1) {
                totA[wave][kl] = A;
                totB[wave][kl] = Bv;
            }
            T exA = (T)1, exB = (T)0;
            const T Ap = __shfl_up(A, LW, 64), Bp = __shfl_up(Bv, LW, 64);
            if (sub > 0) exA = Ap, exB = Bp;
            __syncthreads();
            T in = carry;
            for (int w = 0; w < nwave; ++w) {
                const T next = totB[w][kl] + inflow(totA[w][kl], carry);
                if (w == wave) in = carry;
                carry = next;
            }
            in = exB + inflow(exA, in);
    #pragma unroll
            for (int j = 0; j < kSeg; ++j) {
                if (f0 + q0 + j >= n) break;
                const LineCell me = tab[q0 + j + 2];
                const bool solid = me.code & kSolidBit;
                const T en = solid ? v[j + 2] + (b[j] + inflow(g[j], in)) : v[j + 2];
                if (active) eout[(size_t)me.cell * d.nk + k] = en;
                const double x = solid && active ? (double)en : 0.0;
                const double m0 = row_sum(L.w * x), m1 = row_sum(L.witau * x), m2 = row_sum(L.wv[0] * x);
                if (kl == 0) {
                    double *o = part + ((size_t)pidx * d.nc + me.cell) * kMomN;
                    double s[3] = {m0, m1 + gam[q0 + j] * m0, m2};
                    if (FOLD && grp > 0)   // the same thread's, of the groups before
                        for (int m = 0; m < 3; ++m) s[m] += o[m];
                    for (int m = 0; m < 3; ++m) o[m] = s[m];
                    o[3] = 0.0;   // no direction of a line has components off it
                    o[4] = 0.0;
                }
            }
            __syncthreads();
        }
    }
}

// Explicit step (Sec. 4.1) of `tile` cells of a line for every lane, so that
// the block holds the whole sum for T_L of the new state and writes it (TLin
// may be TLout: a cell's T_L is read only here): no partials, no second
// launch.  A wavefront takes 64 lanes by 4 cells at a time, the lanes of
// either sign walking downwind.  Bound by latency (launch, geometry tables,
// rows, the sum).  1000 cells x 512 lanes FP32, 4 cells a block:
// 6.1 us a step (17.9 with tiles per octant and T_L in a second launch).
template <typename T, int LIM>
__global__ __launch_bounds__(kStepThreads) void k_transient1d(Dev d, const T *__restrict__ ein, T *__restrict__ eout,
                                                              const double *TLin, double *TLout,
                                                              const double *__restrict__ din,
                                                              const TileItem *__restrict__ items, int nitems, int tile,
                                                              double src, double dt)
{
    __shared__ LineCell tab[kStepCells + 8];              // positions x0 - 2 .. x0 + tile + 5
    __shared__ double tl[kStepCells], gam[kStepCells], qs[kStepCells];
    __shared__ double red[kStepThreads / 16][kStepCells];
    const int nb = gridDim.x, bb = blockIdx.x;
    const int lb = (bb & 7) * (nb >> 3) + (bb >> 3);      // neighbouring tiles on one XCD
    if (lb >= nitems) return;
    int film = 0, x0 = lb * tile;
    if (d.nfilm > 1) film = items[lb].film, x0 = items[lb].tile * tile;
    const Film &fm = d.film[film];
    const int ext = min(tile, fm.n[0] - x0);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwave = kStepThreads / 64;
    for (int q = threadIdx.x; q < ext + 8; q += kStepThreads) {
        const int i = x0 + q - 2;
        LineCell t{-1, 0u, 0.0};
        if (i <= fm.n[0] + 1) t = line_cell(d, fm, i, nullptr);
        tab[q] = t;
        if (q >= 2 && q < ext + 2) {
            tl[q - 2] = TLin[t.cell];
            gam[q - 2] = d.gamma[t.cell];
            qs[q - 2] = d.P ? d.P[t.cell] / fm.Ctot : 0.0;
        }
    }
    for (int i = threadIdx.x; i < kStepThreads / 16 * ext; i += kStepThreads) red[i / ext][i % ext] = 0.0;
    __syncthreads();
    const int ngrp = (ext + kSeg - 1) / kSeg, nch = (d.nk + 63) / 64;
    const T tdt = (T)dt, tsrc = (T)src;
    const T *zrow = static_cast<const T *>(d.zrow);
    for (int t = wave; t < ngrp * nch; t += nwave) {
        const int ch = t % nch, e0 = t / nch * kSeg;
        const int k = ch * 64 + lane;
        const bool active = k < d.nk;
        const int kk = active ? k : 0;
        const LaneT<T> L = lane_make<T>(d, fm, kk);
        const int sg = d.s[3 * L.al] > 0 ? 1 : -1;
        const int qa = sg > 0 ? e0 : e0 + kSeg + 3;       // tab entry of the flow position -2
        T v[kSeg + 3];
#pragma unroll
        for (int j = 0; j < kSeg + 3; ++j) {
            const int c = tab[qa + sg * j].cell;
            const T *row = c >= 0 ? ein + (size_t)c * d.nk : zrow;
            v[j] = row[kk];
        }
        double acc[kSeg];
#pragma unroll
        for (int j = 0; j < kSeg + 3; ++j) v[j] += L.C4 * (T)tab[qa + sg * j].x;
#pragma unroll
        for (int j = 0; j < kSeg; ++j) {
            const int q = qa + sg * (j + 2), i = q - 2;   // cell i of the tile
            acc[j] = 0.0;
            if (active && i < ext) {
                const LineCell me = tab[q];
                T en = v[j + 2];
                if (me.code & kSolidBit) {
                    const T D = L.cpl[0] * line_delta<T, LIM>(d, fm, ein, din, me, tab[q - 2 * sg].code, tab[q + sg], sg, L,
                                                              v[j], v[j + 1], en, v[j + 3]);
                    const T itc = L.itau + (T)gam[i];
                    en = en + tdt * (-D - (en - L.C4 * (T)tl[i]) * itc + L.C4 * tsrc * (T)qs[i]);
                    acc[j] = (L.witau + L.w * gam[i]) * (double)en;
                }
                eout[(size_t)me.cell * d.nk + k] = en;
            }
        }
#pragma unroll
        for (int x = 0; x < kSeg; ++x) {
            const double s = row_sum(sg > 0 ? acc[x] : acc[kSeg - 1 - x]);
            if ((lane & 15) == 0 && e0 + x < ext) red[wave * 4 + (lane >> 4)][e0 + x] += s;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < ext; i += kStepThreads) {
        double s = 0.0;
        for (int r = 0; r < kStepThreads / 16; ++r) s += red[r][i];
        const int c = tab[i + 2].cell;
        TLout[c] = (tab[i + 2].code & kSolidBit) ? s / d.S[c] : 0.0;
    }
}

int line_groups(int lanes_oct) { return (lanes_oct + LW - 1) / LW; }
int line_waves(int max_n)
{
    const int per_wave = 64 / LW * kSeg;
    return std::min(kLineThreads / 64, (max_n + per_wave - 1) / per_wave);
}

// Whether blocks are folded, which leaves a quarter of the moment partials (0.6
// bytes a value instead of 2.5): where the partials pass 256 MiB and the
// wavefronts still fill the chip's 4096 places.  20 lines of 2000 cells x 1280 lanes
// FP32: sweep 0.385 -> 0.477 ms, the sums over the partials 0.039 -> 0.021; 200 cells x
// 51 200: 0.094 -> 0.120 and 0.079 -> 0.028.
bool line_fold(int lanes_oct, int nfilm, int max_n, size_t nc)
{
    return 2.0 * nfilm * line_groups(lanes_oct) * line_waves(max_n) >= 4096.0 * kFold &&
           8 * kMomN * nc * 2 * line_groups(lanes_oct) >= size_t(256) << 20;
}

}  // namespace

// moment partials per cell of a sweep (lines of up to max_n cells)
int line_parts(int lanes_oct, int nfilm, int max_n, size_t nc)
{
    const int fold = line_fold(lanes_oct, nfilm, max_n, nc) ? kFold : 1;
    return 2 * ((line_groups(lanes_oct) + fold - 1) / fold);
}

namespace {

template <typename T, int LIM>
void sweep1d_launch(const Dev &d, const T *ein, T *eout, const double *dpend, const double *TLdev, const double *din,
                    int na_oct, int max_n, double *part, hipStream_t s)
{
    const int parts = line_parts(na_oct * d.nl, d.nfilm, max_n, d.nc) / 2;
    const dim3 grid((unsigned)d.nfilm * 2 * parts), block(64 * line_waves(max_n));
    if (line_fold(na_oct * d.nl, d.nfilm, max_n, d.nc))
        hipLaunchKernelGGL((k_sweep1d<T, LIM, true>), grid, block, 0, s, d, ein, eout, dpend, TLdev, din, na_oct, parts,
                           part);
    else
        hipLaunchKernelGGL((k_sweep1d<T, LIM, false>), grid, block, 0, s, d, ein, eout, dpend, TLdev, din, na_oct, parts,
                           part);
}

}  // namespace

template <typename T>
hipError_t launch_sweep1d(const Dev &d, const T *ein, T *eout, const double *dpend, const double *TLdev,
                          const double *din, int na_oct, int max_n, double *part, hipStream_t s)
{
#define BTE_LINE(LIM)                                                                                                \
    if (d.limiter == LIM) sweep1d_launch<T, LIM>(d, ein, eout, dpend, TLdev, din, na_oct, max_n, part, s);
    BTE_LINE(0) BTE_LINE(1) BTE_LINE(2)
#undef BTE_LINE
    return hipGetLastError();
}

// items: (geometry, octant 0, tile) of tiles of `tile` <= 64 cells
template <typename T>
hipError_t launch_transient1d(const Dev &d, const T *ein, T *eout, const double *TLin, double *TLout, const double *din,
                              const TileItem *items, int nitems, int tile, double src, double dt, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    const dim3 grid((nitems + 7) / 8 * 8);
#define BTE_LINE(LIM)                                                                                                \
    if (d.limiter == LIM)                                                                                            \
        hipLaunchKernelGGL((k_transient1d<T, LIM>), grid, dim3(kStepThreads), 0, s, d, ein, eout, TLin, TLout, din,  \
                           items, nitems, tile, src, dt);
    BTE_LINE(0) BTE_LINE(1) BTE_LINE(2)
#undef BTE_LINE
    return hipGetLastError();
}

#define BTE_INST(T)                                                                                                  \
    template hipError_t launch_sweep1d<T>(const Dev &, const T *, T *, const double *, const double *,               \
                                          const double *, int, int, double *, hipStream_t);                          \
    template hipError_t launch_transient1d<T>(const Dev &, const T *, T *, const double *, double *, const double *, \
                                              const TileItem *, int, int, double, double, hipStream_t);
BTE_INST(float)
BTE_INST(double)
#undef BTE_INST

}  // namespace bte
