// bte_cg.hip -- conjugate gradients on the diffusion operators in one launch.
//
// One solve (Chronopoulos-Gear form of Jacobi-preconditioned CG, the
// recurrences of k_cg_iter) runs in one launch of at most one block per
// compute unit.  What bounds a solve is the chain of its iterations, not
// bandwidth: every iteration ends in a reduction over all cells.  A launch per
// iteration costs 6.3 us on 8 100 cells, 11.6 us on 160 000 (about 45 FP64
// loads and seven divisions per cell), so here every vector stays in
// registers for the whole solve and an iteration moves only what crosses a
// block's edge: 3.0 and 5.0 us on the same problems, 0.9 us instead of 6.7 on
// 200 cells (one block), 5.8 instead of 10.0 us on 48^3.
//
// Split: the cells are numbered tile by tile (32 x 16 or 8 x 8 x 8 cells, so
// that few neighbours lie in other blocks) and block b owns the numbers
// [b cpb, (b + 1) cpb), cpb = 512 R, R per thread.
// u = r / diag of the block's cells and of its ghosts (cells of other blocks
// coupled to them) is in LDS, so A u reads LDS only.  A ghost's r and s follow
// the recurrences in the block itself from w = A u, which its owner sends;
// w and the block's three partial sums are sent together, so an iteration
// waits for other blocks once.  Both travel as 8-byte words holding 32 bits
// of the value and a 32-bit tag (solve epoch + iteration): a word is valid
// when its tag is, without flags or fences, and the words alternate between
// two slots (a block sends iteration k + 2 only after it has everything of
// k + 1, which every other block sends after it has read k).  Every block
// sums all partials in the same order and takes the same decisions.
//
// Blocks wait for each other, so all must be resident: the grid is at most
// one block per compute unit, and every wait is bounded in time.  A wait that
// gives up (another kernel holding the compute units, or two of these solves
// on two streams each holding half) writes the solve's epoch to the abort
// word; every block leaves and the host repeats the solve with one launch per
// iteration.
#include "bte_internal.h"
#include "bte_tilelds.h"

namespace bte {

namespace {

constexpr unsigned long long kWaitTicks = 2000000ull;   // 20 ms of the 100 MHz clock

__device__ inline void ll_store(unsigned long long *p, unsigned tag, double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned long long t = (unsigned long long)tag << 32;
    __hip_atomic_store(p, t | (b & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, t | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline double ll_value(unsigned long long lo, unsigned long long hi)
{
    return __longlong_as_double((long long)((lo & 0xffffffffull) | (hi << 32)));
}

// Read N doubles sent under `tag` (2 N words); false if the wait gave up.
template <int N>
__device__ inline bool ll_wait(const unsigned long long *p, unsigned tag, const unsigned *abortw, unsigned epoch,
                               double (&v)[N])
{
    unsigned long long t0 = 0;
    for (int n = 0;; ++n) {
        unsigned long long w[2 * N];
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 2 * N; ++i) w[i] = __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < 2 * N; ++i) ok = ok && (unsigned)(w[i] >> 32) == tag;
        if (ok) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = ll_value(w[2 * i], w[2 * i + 1]);
            return true;
        }
        if ((n & 63) == 63) {
            const unsigned long long now = __builtin_amdgcn_s_memrealtime();
            if (t0 == 0) t0 = now;
            if (now - t0 > kWaitTicks) return false;
            if (__hip_atomic_load(abortw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) return false;
        }
    }
}

// sum of the block's rows of 16 lanes, in every lane of a wave
constexpr int kRows = kCgThreads / 16;
__device__ inline void block_total(const double *srow, int lane, double (&v)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        v[i] = row_sum(srow[i * kRows + (lane & (kRows - 1))]);
        v[i] += __shfl_xor(v[i], 16, 64);
    }
}

// 1 / x by two Newton steps on the hardware's estimate
__device__ inline double reciprocal(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// The scalars of the recurrences.  They stand between two barriers of every
// iteration, so the reciprocals of the step before are formed once its own
// scalars are on their way, and one reciprocal is left in the chain.
struct CgScalars {
    double alpha = 0.0, beta = 0.0, bn2 = 0.0, gamma = 0.0, igamma = 0.0, gia = 0.0;
    // false: stop before this step
    __device__ inline bool step(int it, double ga, double de, double rr, double rtol2)
    {
        if (it == 0) bn2 = rr;
        gamma = ga;
        if (!(rr > rtol2 * bn2) || !(ga > 0.0)) return false;
        beta = it == 0 ? 0.0 : ga * igamma;
        const double den = it == 0 ? de : fma(-ga * ga, gia, de);   // de - beta ga / alpha
        alpha = ga * reciprocal(den);
        return alpha > 0.0 && isfinite(alpha) && isfinite(beta);
    }
    __device__ inline void prepare()
    {
        igamma = reciprocal(gamma);
        gia = igamma * reciprocal(alpha);
    }
};

// NF: faces with a coupling (2 per axis); R: cells per thread; MULTI: more than one block
template <int NF, int R, bool MULTI>
__global__ __launch_bounds__(kCgThreads) void k_cg_solve(Dev d, CgArgs g, CgPlan q, const double *__restrict__ b,
                                                         int maxit, unsigned epoch)
{
    extern __shared__ double lds[];
    constexpr int cpb = kCgThreads * R;
    double *u = lds;                       // [cpb + ghosts]
    double *gr = u + cpb + q.max_ghost;    // ghosts: r, s, w, 1 / diag
    double *gs = gr + q.max_ghost;
    double *gw = gs + q.max_ghost;
    double *gi = gw + q.max_ghost;
    __shared__ double srow[3 * kRows];
    __shared__ double sc[2];
    __shared__ int sflag;
    const int t = threadIdx.x, blk = blockIdx.x, nblk = gridDim.x, nthr = blockDim.x;
    const int i0 = blk * cpb;
    const int g0 = q.gptr[blk], ng = q.gptr[blk + 1] - g0;
    const int *__restrict__ gid = q.gid + g0;

    double x[R], p[R], r[R], s[R], w[R], idg[R], cf[R][NF];
    unsigned li[R][NF / 2];   // two 16-bit LDS indices each
    int cell[R];              // -1 past the end
    bool send[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = i0 + t + k * nthr;
        const bool in = i < d.nc;
        const int ii = in ? i : 0, c = q.cell[ii];
        cell[k] = in ? c : -1;
        idg[k] = 1.0 / g.dg[c];
        r[k] = in && (d.code[c] & kSolidBit) ? b[c] : 0.0;
        x[k] = p[k] = s[k] = 0.0;
        send[k] = in && (q.lidx[ii] & 0x8000u);
#pragma unroll
        for (int f = 0; f < NF; f += 2) {
            cf[k][f] = in ? g.coef[f * d.nc + c] : 0.0;
            cf[k][f + 1] = in ? g.coef[(f + 1) * d.nc + c] : 0.0;
            li[k][f / 2] = in ? (q.lidx[f * d.nc + ii] & 0x7fffu) | ((unsigned)q.lidx[(f + 1) * d.nc + ii] << 16) : 0u;
        }
        u[t + k * nthr] = r[k] * idg[k];
    }
    for (int i = t; i < ng; i += nthr) {
        const int j = gid[i];
        gr[i] = b[j];   // a coupled cell is solid
        gi[i] = 1.0 / g.dg[j];
        gs[i] = 0.0;
        u[cpb + i] = gr[i] * gi[i];
    }
    if (t == 0) sflag = 0;
    for (int i = t; i < 3 * kRows; i += nthr) srow[i] = 0.0;   // fewer threads than kCgThreads: rows of zeros
    __syncthreads();

    CgScalars st;   // of wave 0, or of every wave
    int it = 0;
    bool stopped = false;
    for (;; ++it) {
        // w = A u (diag u = r) and the partial sums of step it
        double a0 = 0, a1 = 0, a2 = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            double acc = r[k];
#pragma unroll
            for (int f = 0; f < NF; ++f) acc -= cf[k][f] * u[(f & 1) ? li[k][f / 2] >> 16 : li[k][f / 2] & 0xffffu];
            w[k] = acc;
            const double uc = r[k] * idg[k];
            a0 += r[k] * uc;
            a1 += acc * uc;
            a2 += r[k] * r[k];
        }
        if (it >= maxit) break;
        const unsigned tag = epoch + 1 + it;
        const int par = it & 1;
        unsigned long long *wsend = q.wword + 2 * (size_t)d.nc * par;
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (send[k]) ll_store(wsend + 2 * (size_t)cell[k], tag, w[k]);
        a0 = row_sum(a0);
        a1 = row_sum(a1);
        a2 = row_sum(a2);
        if ((t & 15) == 0) {
            srow[t >> 4] = a0;
            srow[kRows + (t >> 4)] = a1;
            srow[2 * kRows + (t >> 4)] = a2;
        }
        __syncthreads();
        double alpha, beta;
        if (MULTI) {
            if (t < 64) {
                double v[3];
                block_total(srow, t, v);
                unsigned long long *pw = q.pword + (size_t)6 * kCgMaxBlocks * par;
                if (t < 3) ll_store(pw + 6 * blk + 2 * t, tag, t == 0 ? v[0] : t == 1 ? v[1] : v[2]);
                bool ok = true;
                double a[3] = {0, 0, 0};
                for (int o = t; o < nblk; o += 64) {
                    double z[3];
                    ok = ll_wait<3>(pw + 6 * o, tag, q.abortw, epoch, z);
                    if (!ok) break;
#pragma unroll
                    for (int i = 0; i < 3; ++i) a[i] += z[i];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    v[i] = row_sum(a[i]);
                    v[i] += __shfl_xor(v[i], 16, 64);
                    v[i] += __shfl_xor(v[i], 32, 64);
                }
                ok = __all(ok);
                const bool stop = !st.step(it, v[0], v[1], v[2], g.rtol2);
                if (t == 0) {
                    sc[0] = st.alpha;
                    sc[1] = st.beta;
                    if (!ok) {
                        sflag = 2;
                        __hip_atomic_store(q.abortw, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    } else if (stop) {
                        sflag = 1;
                    }
                }
                st.prepare();
            }
            // the ghosts' w of this step
            const unsigned long long *wrecv = q.wword + 2 * (size_t)d.nc * par;
            for (int i = t; i < ng; i += nthr) {
                double z[1] = {0.0};
                if (!ll_wait<1>(wrecv + 2 * (size_t)gid[i], tag, q.abortw, epoch, z)) {
                    sflag = 2;
                    __hip_atomic_store(q.abortw, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                gw[i] = z[0];
            }
            __syncthreads();
            const int flag = sflag;
            if (flag == 2) return;
            if (flag == 1) {
                stopped = true;
                break;
            }
            alpha = sc[0];
            beta = sc[1];
        } else {
            // one block: every wave sums the rows itself
            double v[3];
            block_total(srow, t & 63, v);
            if (!st.step(it, v[0], v[1], v[2], g.rtol2)) {
                stopped = true;
                break;
            }
            alpha = st.alpha;
            beta = st.beta;
            st.prepare();
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            p[k] = r[k] * idg[k] + beta * p[k];
            s[k] = w[k] + beta * s[k];
            x[k] += alpha * p[k];
            r[k] -= alpha * s[k];
            u[t + k * nthr] = r[k] * idg[k];
        }
        for (int i = t; i < ng; i += nthr) {
            const double si = gw[i] + beta * gs[i];
            const double ri = gr[i] - alpha * si;
            gs[i] = si;
            gr[i] = ri;
            u[cpb + i] = ri * gi[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (cell[k] >= 0) g.x[cell[k]] = x[k];
    }
    if (blk == 0 && t == 0) {
        g.scal[5] = stopped ? 1.0 : 0.0;
        g.scal[6] = it;
        g.scal[9] += it;
        g.scal[14] = epoch;   // this solve is counted
    }
}

template <int NF> const void *cg_kernel(int R, bool multi)
{
    switch (R) {
    case 1: return multi ? (const void *)k_cg_solve<NF, 1, true> : (const void *)k_cg_solve<NF, 1, false>;
    case 2: return multi ? (const void *)k_cg_solve<NF, 2, true> : (const void *)k_cg_solve<NF, 2, false>;
    default: return multi ? (const void *)k_cg_solve<NF, 4, true> : (const void *)k_cg_solve<NF, 4, false>;
    }
}

const void *cg_kernel(int dim, int R, bool multi)
{
    return dim == 1 ? cg_kernel<2>(R, multi) : dim == 2 ? cg_kernel<4>(R, multi) : cg_kernel<6>(R, multi);
}

}  // namespace

size_t cg_solve_smem(int R, int max_ghost) { return 8 * ((size_t)kCgThreads * R + 5 * (size_t)max_ghost); }

// Whether every block of the plan can be resident at once on the current device.
hipError_t cg_solve_init(int dim, int R, int max_ghost, int nblk, bool *ok)
{
    *ok = false;
    const void *f = cg_kernel(dim, R, nblk > 1);
    const size_t smem = cg_solve_smem(R, max_ghost);
    int dev = 0, ncu = 0, per = 0;
    hipError_t e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, kCgThreads, smem)) != hipSuccess) return e;
    *ok = per >= 1 && nblk <= ncu;
    return hipSuccess;
}

hipError_t launch_cg_solve(const Dev &d, const CgArgs &g, const CgPlan &q, int nblk, int R, const double *b, int maxit,
                           unsigned epoch, hipStream_t s)
{
    Dev dd = d;
    CgArgs gg = g;
    CgPlan qq = q;
    void *args[] = {&dd, &gg, &qq, &b, &maxit, &epoch};
    // one block of one cell per thread: no more waves than cells
    const int nthr = nblk == 1 && R == 1 ? (d.nc + 63) / 64 * 64 : kCgThreads;
    return hipLaunchKernel(cg_kernel(d.dim, R, nblk > 1), dim3(nblk), dim3(nthr), args, cg_solve_smem(R, q.max_ghost),
                           s);
}

}  // namespace bte
