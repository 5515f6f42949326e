// Matrix-free element operator  w = h1 A_L(k) u + h2 B u  (NekRS paper,
// Sec. 2.3, eq. (Ae)):  A^e = [D1;D2;D3]^T (k o G^e) [D1;D2;D3].
//
// Thread layout (the 2D-thread / 1D-register structure of Sec. 3.3): a thread
// owns one (i,j) column of an element and keeps the k-line of u and of the
// t-part of the result in registers; the element's u sits in LDS and the k
// planes are swept one after another:
//   step 1: ur = D1 u, us = D2 u  (LDS plane k), ut = D3 u (registers)
//   step 2: (wr, ws, wt) = k G (ur, us, ut), G the symmetric 3x3 per point,
//           the six factors of a point contiguous ([E][np][6], 48 B, three
//           16-byte loads per lane, each wavefront reading 3 KiB contiguous
//           per plane)
//   step 3: plane k of D1^T wr + D2^T ws from two flux planes in LDS, left in
//           the plane of u that is no longer read; D3^T wt accumulated in
//           registers over the sweep
// The flux planes alternate between two buffers, so a plane costs one barrier
// (none but an ordering of LDS accesses where (N+1)^2 <= 64 and an element is
// one wavefront).  The plane loop is not unrolled: row k of Dh (the D3
// coefficients of the plane) then lives in SGPRs for one plane, where holding
// all (N+1)^2 spilled them.  The next plane's G (and B, k) is loaded while the
// current one is computed, across elements too; the grid is persistent.
// Where registers are short D^T comes from the rows of D: GLL quadrature sums the product of two degree-N
// derivatives exactly, so rho_i D[i][l] + rho_l D[l][i] is 0 but at the end
// points (-1 for i = l = 0, +1 for i = l = N), and
//   sum_l D[l][i] f_l = -rho_i sum_l D[i][l] (f_l / rho_l)  +- f_i / rho_i at the ends.
// With two register rows instead of four the FP64 kernel keeps 3 waves per
// SIMD at N = 7 and 2-3 up to N = 15 (four rows: 1-2 from N = 11 on).
// Bytes per point (FP64 Poisson): u 8 + G 48 + w 8 = 64 (+8 for B, +8 for k).
#pragma once
#include <algorithm>

#include "sem_internal.h"

// FMA contraction within single expressions only: the single-vector and the
// batched kernels below then round every point identically.
#pragma clang fp contract(on)

namespace semx {

template <int NQ>
struct AxShape {
    static constexpr int TPE = NQ * NQ;                       // threads per element
    static constexpr int EPB = TPE <= 64 ? 64 / TPE : 1;      // elements per block
    static constexpr int THREADS = EPB * TPE;
    static constexpr bool ONE_WAVE = THREADS <= 64;
    static constexpr int LD = (NQ % 2 == 0) ? NQ + 1 : NQ;    // padded LDS row
    // block of nw wavefronts with fields of their own
    static constexpr int threads(int nw) { return nw == 1 ? THREADS : 64 * nw; }
};

// Waves per SIMD asked of the compiler, FP64 (0.9 M to 2.4 M points, the two
// forms in us): N = 10 .. 12 fit three with a few spilled registers, which
// pays (N = 11 Helmholtz with k 39.5 -> 37.2, N = 12 Helmholtz 32.8 -> 27.9);
// N = 13 with k and N = 15 spill too much at three (34.7 -> 39.1, 29.6 -> 52.5).
// Below N = 10 the unforced kernel is the fastest form.
template <int NQ, typename T>
constexpr int ax_min_waves()
{
    if (sizeof(T) == 4 || NQ <= 10) return 1;
    return NQ <= 13 ? 3 : 2;
}

// Waves per SIMD the compiler may aim at.  FP64 Poisson at N = 6 fits four if
// every load waits for its use (0.45 M points 7.7 us; with three 7.2).
template <int NQ, typename T, bool HELM>
constexpr int ax_max_waves()
{
    return sizeof(T) == 8 && NQ == 7 && !HELM ? 3 : 8;
}

// Whether D^T has register rows of its own or is formed from the rows of D.  Own
// rows round least: against FP64, FP32 rms error over N = 2 .. 8 5.0e-8 .. 7.4e-8
// with them, 5.4e-8 .. 8.5e-8 without (from the rows of D N = 5 lost most, 6.5e-8
// against 8.4e-8; a sum that runs on through all three directions 8.1e-8).  FP32
// has the registers for it up to N = 7; beyond, two rows are the faster form
// (0.96 M points: N = 8 9.1 / 9.4 us, N = 10 8.5 / 10.4) at 7.6e-8 to 1.2e-7, below
// the 1.0e-7 to 1.5e-7 of the running sum.  FP64: up to N = 3 (64000 elements
// 39.7 -> 38.2 us).
template <int NQ, typename T>
constexpr bool ax_dt_rows()
{
    return NQ <= (sizeof(T) == 4 ? 8 : 4);
}

// Points up to which a single field is computed in two phases, all planes
// forward, then all planes back, instead of plane by plane: one chain of LDS
// accesses an element in place of N + 1, and every factor of it on its way at
// once, at the price of a second full plane set in LDS and registers.  us, by
// planes / in two phases: FP32 N = 2, 0.29 M points 3.6 / 3.0, 7 M 54.8 / 50.8; N = 3,
// 0.11 M 2.8 / 2.6, 0.88 M 4.6 / 4.5, 2.5 M 12.9 / 14.3; N = 5, 0.29 M 4.4 / 3.9, 0.88 M
// 6.9 / 6.4, 2.6 M 16.4 / 17.3 over and over on one mesh and 30.3 / 28.9 with QQ^T on
// three meshes in turn, 3.8 M 26.0 / 24.2, 7 M 51.7 / 53.1; N = 6, 0.45 M 4.9 / 4.6,
// 0.94 M 8.1 / 8.8; N = 7, 0.88 M 6.0 / 6.6.  FP64 N = 1 and 2: 0.09 M 3.7 / 3.2, 0.88 M
// 12.0 / 11.9, 4 M with the mass term 48.0 / 44.4; N = 3, 0.88 M 10.4 / 10.9.
template <int NQ, typename T>
constexpr int64_t ax_two_phase_points()
{
    if (NQ <= 3) return INT64_MAX;
    if (sizeof(T) == 8) return 0;
    return NQ <= 5 ? 1200000 : NQ == 6 ? 4500000 : NQ == 7 ? 600000 : 0;
}

template <bool ONE_WAVE>
__device__ inline void block_sync()
{
    if constexpr (ONE_WAVE) {
        // all threads of the block are one wavefront: order LDS accesses
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// six geometric factors of one point, stored contiguously
__device__ inline void load_g6(const double *p, double g[6])
{
    const double2 *q = reinterpret_cast<const double2 *>(p);
    const double2 a = q[0], b = q[1], c = q[2];
    g[0] = a.x; g[1] = a.y; g[2] = b.x; g[3] = b.y; g[4] = c.x; g[5] = c.y;
}
__device__ inline void load_g6(const float *p, float g[6])
{
    const float2 *q = reinterpret_cast<const float2 *>(p);
    const float2 a = q[0], b = q[1], c = q[2];
    g[0] = a.x; g[1] = a.y; g[2] = b.x; g[3] = b.y; g[4] = c.x; g[5] = c.y;
}

// Sum over the THREADS threads of a block (or of a field's wavefront) in a
// fixed order: the lanes of each wavefront by halving strides, then the
// wavefronts in order; the result is thread 0's.  sh: one slot per wavefront.
template <int THREADS>
__device__ inline double ax_block_sum(double x, int tid, double *sh)
{
    const int lane = tid & 63, n = min(64, THREADS - (tid & ~63));  // lanes of this wavefront
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) {
        const double o = __shfl_down(x, st, 64);
        if (lane + st < n) x += o;
    }
    if constexpr (THREADS > 64) {
        if (lane == 0) sh[tid >> 6] = x;
        __syncthreads();
        if (tid == 0)
#pragma unroll
            for (int q = 1; q < (THREADS + 63) / 64; ++q) x += sh[q];
    }
    return x;
}

// Decision and beta after an update (PcgDir), the same in every workgroup, from
// the sum of its records by the first N = min(64, THREADS) lanes of the block (or
// of a field's wavefront).  False: the vector's iteration has ended.  record: this
// block notes it.
template <int THREADS>
__device__ inline bool pcg_direction(const PcgDir &d, int64_t v, int tid, bool record, double *sh, double *beta)
{
    constexpr int N = THREADS < 64 ? THREADS : 64;
    KrylovScalars *sc = d.sc + v;
    // issued ahead of the records, waited for after them
    const double tol2 = sc->tol2, rz_old = sc->rz2[d.parity];
    const int maxit = sc->maxit, done = sc->done;
    double rz = 0.0, rr = 0.0;
    if (tid < N) pcg_sum_records(d.pu + v * d.pst, d.nb, tid, N, rz, rr);
    if constexpr (THREADS > 64) {
        if (tid == 0) {
            sh[0] = rz;
            sh[1] = rr;
        }
        __syncthreads();
        rz = sh[0];
        rr = sh[1];
    }
    if (ended_before(done, d.stamp)) return false;
    const bool bad = !isfinite(rz) || !isfinite(rr);
    const bool stop = bad || rr <= tol2 || d.iter >= maxit;
    *beta = rz / rz_old;
    if (record && tid == 0) {
        sc->iters = d.iter;
        sc->rr = rr;
        sc->rz = rz;
        sc->rz2[d.parity ^ 1] = rz;
        if (bad) sc->status = SEM_EBREAKDOWN;
        if (stop) sc->done = d.stamp;
    }
    return !stop;
}

// One element column's constants: its rows of D, and its rows of D^T or what
// forms them from those of D.
template <int NQ, typename T>
struct AxCol {
    static constexpr bool DT = ax_dt_rows<NQ, T>();
    T Di[NQ], Dj[NQ];
    T Ti[DT ? NQ : 1], Tj[DT ? NQ : 1];  // rows of D^T
    T rhoi, rhoj, ri, rj, bi, bj;        // weights, their inverses, end-point terms
    // D with rows of ld, the weights rho
    __device__ inline AxCol(const T *D, int ld, const T *rho, int i, int j)
    {
#pragma unroll
        for (int l = 0; l < NQ; ++l) {
            Di[l] = D[i * ld + l];
            Dj[l] = D[j * ld + l];
            if constexpr (DT) {
                Ti[l] = D[l * ld + i];
                Tj[l] = D[l * ld + j];
            }
        }
        rhoi = rho[i];
        rhoj = rho[j];
        ri = T(1) / rhoi;
        rj = T(1) / rhoj;
        bi = i == 0 ? -ri : (i == NQ - 1 ? ri : T(0));
        bj = j == 0 ? -rj : (j == NQ - 1 ? rj : T(0));
    }
    // a flux as it is left for the others, and the rows that contract it
    __device__ inline T out_r(T wr) const { return DT ? wr : wr * ri; }
    __device__ inline T out_s(T ws) const { return DT ? ws : ws * rj; }
    __device__ inline T back_r(int l) const
    {
        if constexpr (DT) return Ti[l];
        else return Di[l];
    }
    __device__ inline T back_s(int l) const
    {
        if constexpr (DT) return Tj[l];
        else return Dj[l];
    }
};

// (wr, ws, wt) = G (ur, us, ut)
template <typename T>
__device__ inline void ax_flux(const T (&g)[6], T ur, T us, T ut, T &wr, T &ws, T &wt)
{
    wr = g[0] * ur + g[1] * us + g[2] * ut;
    ws = g[1] * ur + g[3] * us + g[4] * ut;
    wt = g[2] * ur + g[4] * us + g[5] * ut;
}

// the r and s parts of a point's result (ar, as: the back rows over the fluxes
// left) with the mass term
template <int NQ, typename T, bool HELM>
__device__ inline T ax_rs_part(const AxCol<NQ, T> &C, T wr, T ws, T ar, T as, T h1, T h2, T b, T u)
{
    T acc;
    if constexpr (AxCol<NQ, T>::DT) acc = ar + as;
    else acc = (C.bi * wr - C.rhoi * ar) + (C.bj * ws - C.rhoj * as);
    acc *= h1;
    if constexpr (HELM) acc += h2 * b * u;
    return acc;
}

// A wavefront (or, for N > 7, a workgroup) computes NI fields of its element
// plane by plane, or (TWO) all planes forward, then all planes back, and a
// workgroup holds NW wavefronts with fields of their own.
// nvb: number of partial sums of u.w; record vb covers the element groups vb,
// vb + nvb, ...  With several fields fewer workgroups than nvb may run, each
// taking records in turn, so a field's records are those of a single-field call.
template <int NQ, typename T, bool HELM, bool VARK, bool DOT, int NW, int NI, bool TWO>
__global__ void __launch_bounds__((AxShape<NQ>::threads(NW)))
__attribute__((amdgpu_waves_per_eu(ax_min_waves<NQ, T>(), ax_max_waves<NQ, T, HELM>())))
ax_kernel(int64_t E, const T *__restrict__ G, const T *__restrict__ B,
          const T *__restrict__ kc, const T *__restrict__ Dg, T h1, T h2,
          const T *u, int64_t ldu, T *__restrict__ w, int64_t ldw, VSet vs,
          double *__restrict__ partial, int64_t pst, int64_t nvb, const int *__restrict__ skip,
          int skip_stride, PcgDir dir)
{
    using S = AxShape<NQ>;
    constexpr int TPE = S::TPE, EPB = S::EPB, LD = S::LD;
    constexpr int NP = NQ * NQ * NQ;
    __shared__ T su[NW][NI][EPB][NQ][NQ][LD];
    static_assert(!TWO || (S::ONE_WAVE && ax_dt_rows<NQ, T>()), "two phases: one wavefront, rows of D^T");
    // flux planes: two buffers of one each way, or of all planes the s flux (the r
    // flux takes u's place, which the wavefront has read by then)
    __shared__ T sr[NW][TWO ? 1 : 2][NI][EPB][TWO ? 1 : NQ][LD];
    __shared__ T ss[NW][TWO ? NQ : 2][NI][EPB][NQ][LD];

    // the wavefront's slot (NW > 1: 64 lanes each), lane in it
    const int fs = NW == 1 ? 0 : (int)threadIdx.x >> 6;
    const int tid = NW == 1 ? (int)threadIdx.x : (int)threadIdx.x & 63;
    if (NW > 1 && tid >= S::THREADS) return;
    bool dirn = false;
    if constexpr (DOT) dirn = dir.sc != nullptr;
    int64_t v[NI];
    bool live[NI], any = false;
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        v[q] = vs.at(fs * NI + q);
        const int done = skip == nullptr ? 0 : skip[v[q] * skip_stride];
        live[q] = dirn ? !ended_before(done, dir.stamp) : done == 0;
        any = any || live[q];
    }
    if (!any) return;  // uniform over the wavefronts of these fields
    const int el = (EPB == 1) ? 0 : tid / TPE;  // element slot within the block
    const int ij = (EPB == 1) ? tid : tid - el * TPE;
    const int i = ij % NQ;
    const int j = ij / NQ;
    const AxCol<NQ, T> C(Dg, NQ, Dg + NQ * NQ, i, j);  // the weights follow D in its buffer

    const int64_t groups = (E + EPB - 1) / EPB;
    T gn[6], bn = T(0), kn = T(0);
    if constexpr (!TWO) {
        const int64_t e0 = (int64_t)blockIdx.x * EPB + el;
        const int64_t b0 = (e0 < E ? e0 : 0) * NP + ij;
        load_g6(G + b0 * 6, gn);
        if constexpr (HELM) bn = B[b0];
        if constexpr (VARK) kn = kc[b0];
    }
    // With a direction update a column needs p, r and Dinv.  Where the registers
    // allow they are loaded ahead of their element, the first ahead of the sums
    // that give beta (512 elements, N = 7: 10.6 -> 9.5 us); else a few planes at a
    // time, since all three lines in flight would spill.
    // In two phases the FP32 column is too (N = 5, 2.6 M points 29.8 -> 28.9).
    constexpr bool AHEAD = (DOT || (TWO && sizeof(T) == 4)) && NQ <= 8 && NI == 1;
    constexpr int CH = 4;
    T rn[AHEAD ? NQ : 1];
    double rr[AHEAD ? NQ : 1], dv[AHEAD ? NQ : 1];
    auto load_column = [&](int64_t o) {
#pragma unroll
        for (int k = 0; k < (AHEAD ? NQ : 1); ++k) rn[k] = u[v[0] * ldu + o + k * TPE];
        if (dirn) {
#pragma unroll
            for (int k = 0; k < (AHEAD ? NQ : 1); ++k) {
                dv[k] = dir.Dinv[o + k * TPE];
                rr[k] = dir.r[v[0] * ldu + o + k * TPE];
            }
        }
    };
    if constexpr (AHEAD) {
        const int64_t e0 = (int64_t)blockIdx.x * EPB + el;
        load_column((e0 < E ? e0 : 0) * NP + ij);
    }
    double beta[NI];
    if constexpr (DOT) {
        if (dirn) {
            __shared__ double sh[2];
            any = false;
#pragma unroll
            for (int q = 0; q < NI; ++q) {
                if (live[q]) live[q] = pcg_direction<S::THREADS>(dir, v[q], tid, blockIdx.x == 0, sh, &beta[q]);
                any = any || live[q];
            }
            if (!any) return;
        }
    }
    for (int64_t vb = blockIdx.x; vb < nvb; vb += gridDim.x) {
        double dot[NI];
#pragma unroll
        for (int q = 0; q < NI; ++q) dot[q] = 0.0;
        for (int64_t g = vb; g < groups; g += nvb) {  // elements g*EPB .. g*EPB+EPB-1
            const int64_t e = g * EPB + el;
            const bool active = e < E;
            const int64_t base = (active ? e : 0) * NP + ij;
            const int64_t gx = NW * NI == 1 || g + nvb < groups ? g + nvb : vb + gridDim.x;
            const int64_t en = gx * EPB + el;
            const int64_t nbase = (en < E ? en : 0) * NP + ij;
            T ru[NI][NQ], rw[NI][NQ];
            if constexpr (AHEAD) {
#pragma unroll
                for (int k = 0; k < NQ; ++k) ru[0][k] = rn[k];
                if (dirn) {
#pragma unroll
                    for (int k = 0; k < NQ; ++k) ru[0][k] = dv[k] * rr[k] + beta[0] * ru[0][k];
                    if (active)
#pragma unroll
                        for (int k = 0; k < NQ; ++k) dir.p[v[0] * ldu + base + k * TPE] = ru[0][k];
                }
            } else if (DOT && dirn) {
#pragma unroll
                for (int c = 0; c < NQ; c += CH) {
                    double dk[CH];
#pragma unroll
                    for (int k = c; k < c + CH && k < NQ; ++k) dk[k - c] = dir.Dinv[base + k * TPE];
#pragma unroll
                    for (int q = 0; q < NI; ++q) {
                        const int64_t o = v[q] * ldu + base;
#pragma unroll
                        for (int k = c; k < c + CH && k < NQ; ++k)
                            ru[q][k] = dk[k - c] * dir.r[o + k * TPE] + beta[q] * dir.p[o + k * TPE];
                        if (active && live[q])
#pragma unroll
                            for (int k = c; k < c + CH && k < NQ; ++k) dir.p[o + k * TPE] = ru[q][k];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int q = 0; q < NI; ++q)
#pragma unroll
                    for (int k = 0; k < NQ; ++k) ru[q][k] = u[v[q] * ldu + base + k * TPE];
            }
#pragma unroll
            for (int q = 0; q < NI; ++q)
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    su[fs][q][el][k][j][i] = ru[q][k];
                    rw[q][k] = T(0);
                }
            // two phases: every factor of the element is on its way before the
            // lanes meet (left behind, the loads are put off to save registers)
            T ga[TWO ? NQ : 1][6], ba[TWO ? NQ : 1], ca[TWO ? NQ : 1];
            if constexpr (TWO)
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    load_g6(G + (base + k * TPE) * 6, ga[k]);
                    ba[k] = ca[k] = T(0);
                    if constexpr (HELM) ba[k] = B[base + k * TPE];
                    if constexpr (VARK) ca[k] = kc[base + k * TPE];
                }
            // wavefronts with fields of their own meet once per element, which
            // keeps the factors that one of them fetched in L1 for the others
            block_sync<S::ONE_WAVE && NW == 1>();

            if constexpr (TWO) {
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    T gg[6];
#pragma unroll
                    for (int q = 0; q < 6; ++q) gg[q] = VARK ? ga[k][q] * ca[k] : ga[k][q];
                    const T *dk = Dg + k * NQ;
#pragma unroll
                    for (int q = 0; q < NI; ++q) {
                        T ur = 0, us = 0, ut = 0, wr, ws, wt;
#pragma unroll
                        for (int l = 0; l < NQ; ++l) {
                            ur += C.Di[l] * su[fs][q][el][k][j][l];
                            us += C.Dj[l] * su[fs][q][el][k][l][i];
                            ut += dk[l] * ru[q][l];
                        }
                        ax_flux(gg, ur, us, ut, wr, ws, wt);
                        su[fs][q][el][k][j][i] = wr;  // plane k of u has been read
                        ss[fs][k][q][el][j][i] = ws;
#pragma unroll
                        for (int m = 0; m < NQ; ++m) rw[q][m] += dk[m] * wt;
                    }
                }
                block_sync<S::ONE_WAVE>();
#pragma unroll
                for (int k = 0; k < NQ; ++k)
#pragma unroll
                    for (int q = 0; q < NI; ++q) {
                        T ar = 0, as = 0;
#pragma unroll
                        for (int l = 0; l < NQ; ++l) {
                            ar += C.back_r(l) * su[fs][q][el][k][j][l];
                            as += C.back_s(l) * ss[fs][k][q][el][l][i];
                        }
                        const T out = ax_rs_part<NQ, T, HELM>(C, T(0), T(0), ar, as, h1, h2, ba[k],
                                                              ru[q][k]) + h1 * rw[q][k];
                        if (active && (NI == 1 || live[q])) w[v[q] * ldw + base + k * TPE] = out;
                        if constexpr (DOT)
                            if (active) dot[q] += (double)ru[q][k] * (double)out;
                    }
                block_sync<S::ONE_WAVE>();  // the next element's u takes their place
            } else {
#pragma unroll 1
                for (int k = 0; k < NQ; ++k) {
                    T gg[6];
                    const T bb = bn, c = kn;
#pragma unroll
                    for (int q = 0; q < 6; ++q) gg[q] = gn[q];
                    {  // the next plane's factors, loaded while this one is computed
                        const int64_t nx = k + 1 < NQ ? base + (k + 1) * TPE : nbase;
                        load_g6(G + nx * 6, gn);
                        if constexpr (HELM) bn = B[nx];
                        if constexpr (VARK) kn = kc[nx];
                    }
                    if constexpr (VARK)
#pragma unroll
                        for (int q = 0; q < 6; ++q) gg[q] *= c;
                    const T *dk = Dg + k * NQ;
                    T wr[NI], ws[NI], uk[NI];
#pragma unroll
                    for (int q = 0; q < NI; ++q) {
                        T ur = 0, us = 0, ut = 0, wt;
#pragma unroll
                        for (int l = 0; l < NQ; ++l) {
                            ur += C.Di[l] * su[fs][q][el][k][j][l];
                            us += C.Dj[l] * su[fs][q][el][k][l][i];
                            ut += dk[l] * ru[q][l];
                        }
                        ax_flux(gg, ur, us, ut, wr[q], ws[q], wt);
                        sr[fs][k & 1][q][el][j][i] = C.out_r(wr[q]);
                        ss[fs][k & 1][q][el][j][i] = C.out_s(ws[q]);
                        uk[q] = su[fs][q][el][k][j][i];
#pragma unroll
                        for (int m = 0; m < NQ; ++m) rw[q][m] += dk[m] * wt;
                    }
                    // past this barrier plane k of u has been read by every thread;
                    // the other pair of flux planes is written before the next one
                    block_sync<S::ONE_WAVE>();
#pragma unroll
                    for (int q = 0; q < NI; ++q) {
                        T ar = 0, as = 0;
#pragma unroll
                        for (int l = 0; l < NQ; ++l) {
                            ar += C.back_r(l) * sr[fs][k & 1][q][el][j][l];
                            as += C.back_s(l) * ss[fs][k & 1][q][el][l][i];
                        }
                        // read again by this thread only
                        su[fs][q][el][k][j][i] =
                            ax_rs_part<NQ, T, HELM>(C, wr[q], ws[q], ar, as, h1, h2, bb, uk[q]);
                    }
                }
#pragma unroll
                for (int q = 0; q < NI; ++q)
#pragma unroll
                    for (int k = 0; k < NQ; ++k) {
                        const T out = su[fs][q][el][k][j][i] + h1 * rw[q][k];
                        if (active && (NI == 1 || live[q])) w[v[q] * ldw + base + k * TPE] = out;
                        if constexpr (DOT)
                            if (active) dot[q] += (double)ru[q][k] * (double)out;
                    }
            }
            if constexpr (AHEAD)
                if (gx < groups) load_column(nbase);
        }
        if constexpr (DOT) {
            __shared__ double sdot[(S::THREADS + 63) / 64];
#pragma unroll
            for (int q = 0; q < NI; ++q) {
                const double s = ax_block_sum<S::THREADS>(dot[q], tid, sdot);
                if (tid == 0 && (NI == 1 || live[q])) partial[v[q] * pst + vb] = s;
            }
        }
        if constexpr (NW * NI == 1) break;  // one record per workgroup
    }
}

// The operator for few elements.  A column thread takes its N + 1 planes one
// after another, about 6 us at N = 7 however few elements there are; here an
// element's points are spread over threads that own KPT points each (one up to
// N = 9), everything is loaded at once, and the three contractions each way
// read LDS between two barriers.  Dh sits in LDS too.
template <int NQ>
struct AxSplitShape {
    static constexpr int TPE = NQ * NQ, NP = TPE * NQ;
    static constexpr int KS = NP <= 1024 ? NQ : (NQ == 11 ? 8 : 6);
    static constexpr int KPT = (NQ + KS - 1) / KS;             // points per thread
    static constexpr int EPB = NP <= 128 ? 256 / NP : 1;       // elements per block
    static constexpr int THREADS = EPB * TPE * KS;
    static constexpr int LD = (NQ % 2 == 0) ? NQ + 1 : NQ;
};

template <int NQ, typename T, bool HELM, bool VARK, bool DOT>
__global__ void __launch_bounds__(AxSplitShape<NQ>::THREADS)
ax_split_kernel(int64_t E, const T *__restrict__ G, const T *__restrict__ B,
                const T *__restrict__ kc, const T *__restrict__ Dg, T h1, T h2,
                const T *__restrict__ u, int64_t ldu, T *__restrict__ w, int64_t ldw, VSet vs,
                double *__restrict__ partial, int64_t pst, const int *__restrict__ skip,
                int skip_stride, PcgDir dir)
{
    using S = AxSplitShape<NQ>;
    constexpr int TPE = S::TPE, NP = S::NP, KS = S::KS, KPT = S::KPT, EPB = S::EPB, LD = S::LD;
    __shared__ T sD[NQ][NQ + 1];
    __shared__ T su[EPB][NQ][NQ][LD], sr[EPB][NQ][NQ][LD], ss[EPB][NQ][NQ][LD], st[EPB][NQ][NQ][LD];
    const int64_t v = vs.at(blockIdx.y);
    // with a direction update the flag is looked at after the loads below
    bool ahead = false;
    if constexpr (DOT) ahead = dir.sc != nullptr;
    if (!ahead && skip != nullptr && skip[v * skip_stride] != 0) return;
    u += v * ldu;
    w += v * ldw;
    const int tid = threadIdx.x;
    const int el = EPB == 1 ? 0 : tid / (TPE * KS);
    const int r = EPB == 1 ? tid : tid - el * (TPE * KS);
    const int kg = r / TPE, ij = r - kg * TPE;
    const int i = ij % NQ, j = ij / NQ;
    const int64_t e = (int64_t)blockIdx.x * EPB + el;
    const bool active = e < E;
    const int64_t base = (active ? e : 0) * NP + ij;
    T uu[KPT], g[KPT][6], bb[HELM ? KPT : 1], cc[VARK ? KPT : 1], wr[KPT], ws[KPT];
    double rr[DOT ? KPT : 1], dv[DOT ? KPT : 1];
    bb[0] = cc[0] = T(0);
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
        const int k = kg + p * KS;
        const int64_t q = base + (k < NQ ? k : 0) * TPE;
        if constexpr (DOT) {
            uu[p] = dir.sc != nullptr ? dir.p[v * ldu + q] : u[q];
            if (dir.sc != nullptr) {
                rr[p] = dir.r[v * ldu + q];
                dv[p] = dir.Dinv[q];
            }
        } else {
            uu[p] = u[q];
        }
        load_g6(G + q * 6, g[p]);
        if constexpr (HELM) bb[p] = B[q];
        if constexpr (VARK) cc[p] = kc[q];
    }
    for (int t = tid; t < NQ * NQ; t += S::THREADS) sD[t / NQ][t % NQ] = Dg[t];
    if constexpr (DOT) {
        if (dir.sc != nullptr) {
            __shared__ double sh[2];
            double beta;
            if (!pcg_direction<S::THREADS>(dir, v, tid, blockIdx.x == 0, sh, &beta)) return;
#pragma unroll
            for (int p = 0; p < KPT; ++p) {
                const int k = kg + p * KS;
                uu[p] = dv[p] * rr[p] + beta * uu[p];
                if (active && k < NQ) dir.p[v * ldu + base + k * TPE] = uu[p];
            }
        }
    }
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
        const int k = kg + p * KS;
        if (k < NQ) su[el][k][j][i] = uu[p];
    }
    block_sync<(S::THREADS <= 64)>();
    const AxCol<NQ, T> C(&sD[0][0], NQ + 1, Dg + NQ * NQ, i, j);
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
        const int k = kg + p * KS;
        if (k < NQ) {
            T ur = 0, us = 0, ut = 0;
#pragma unroll
            for (int l = 0; l < NQ; ++l) {
                ur += C.Di[l] * su[el][k][j][l];
                us += C.Dj[l] * su[el][k][l][i];
                ut += sD[k][l] * su[el][l][j][i];
            }
            T wt;
            if constexpr (VARK)
#pragma unroll
                for (int q = 0; q < 6; ++q) g[p][q] *= cc[p];
            ax_flux(g[p], ur, us, ut, wr[p], ws[p], wt);
            sr[el][k][j][i] = C.out_r(wr[p]);
            ss[el][k][j][i] = C.out_s(ws[p]);
            st[el][k][j][i] = wt;
        }
    }
    block_sync<(S::THREADS <= 64)>();
    double dot = 0.0;
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
        const int k = kg + p * KS;
        if (k < NQ) {
            T ar = 0, as = 0, at = 0;
#pragma unroll
            for (int l = 0; l < NQ; ++l) {
                ar += C.back_r(l) * sr[el][k][j][l];
                as += C.back_s(l) * ss[el][k][l][i];
                at += sD[l][k] * st[el][l][j][i];
            }
            const T out = ax_rs_part<NQ, T, HELM>(C, wr[p], ws[p], ar, as, h1, h2, bb[HELM ? p : 0],
                                                  uu[p]) + h1 * at;
            if (active) {
                w[base + k * TPE] = out;
                if constexpr (DOT) dot += (double)uu[p] * (double)out;
            }
        }
    }
    if constexpr (DOT) {
        __shared__ double sdot[(S::THREADS + 63) / 64];
        const double s = ax_block_sum<S::THREADS>(dot, tid, sdot);
        if (tid == 0) partial[v * pst + blockIdx.x] = s;
    }
}

// Several fields of elements of one wavefront (N <= 7): with `inside`, one
// wavefront computes all of them, the factors in registers; else
// each has a wavefront of its own and the factors come from the caches for the
// others, more wavefronts but G read once per field from L1 / L2.  Operator and
// QQ^T together, us, the per-field loop of before / inside / a wavefront each:
// three FP64 fields at N = 7, 16^3 elements 75 / 71 / 64, 32^3 574 / 564 / 572,
// N = 5, 30^3 274 / 241 / 270; FP32 16^3 43 / 40 / 39, 32^3 331 / 326 / 344.  Four
// FP64 fields inside leave one wave per SIMD (N = 7, 24^3: 327 / 353 / 311) but at
// N <= 4 (N = 4, 3 M points: inside / a wavefront each 148 / 168).  The line
// lies where the FP64 factors fill half the Infinity Cache, and at N = 1 and 2,
// whose registers hold a whole element of every field, far lower (N = 2, two
// phases, three FP64 fields: 0.09 M points 4.8 / 4.6, operator alone, 0.88 M 33.4 /
// 35.4, FP32 23.2 / 25.0).
template <int NQ, typename T>
inline bool ax_fields_inside(int64_t points, int nf)
{
    if (NQ <= 3) return NQ == 2 || points > 150000;
    return points > 2500000 && nf <= (sizeof(T) == 4 || NQ <= 5 ? 4 : 3);
}

// Workgroups per CU of the persistent grid.  One field (operator alone, N = 7,
// us; 16^3 / 32^3 elements): FP64 Poisson 4, 6, 8, 12: 23.8 / 221, 21.9 / 201,
// 21.0 / 202, 21.0 / 209; with the mass term 6, 8, 12: 22.7 / 226, 22.8 / 228,
// 22.7 / 237, and with QQ^T following 31.7 / 298, 32.1 / 302, 32.0 / 309; N = 5
// with the mass term and QQ^T, 20^3 / 40^3, 6, 8, 10, 12: 33.7 / 287, 29.8 /
// 266, 29.8 / 255, 28.9 / 257; FP32 8, 12, 16: - / 171, 167, 167 (N = 5, 23^3:
// 29.9, 27.3, 26.6); N = 2, 0.15 M elements with k 10, 16: 59.6, 56.6.  Several
// fields: a persistent grid whose last workgroups find no room (three wavefronts
// each do not pack the SIMDs evenly after a preceding kernel) runs a second
// round, 32^3 with QQ^T at 4 per CU 710 against 590 at 3; many short workgroups
// (48 per CU inside, 24 else) have no such round.  With partial sums there are
// at most as many workgroups as records.
template <int NQ, typename T>
inline int ax_blocks_per_cu(int nf, bool inside, bool dot)
{
    if (nf == 1) return sizeof(T) == 4 ? 16 : (NQ == 8 ? 6 : (NQ <= 3 ? 16 : NQ < 8 ? 10 : 8));
    if (inside) return dot ? 7 : 48;
    return 24;
}

// Persistent grid over `groups` element groups with at most `cap`
// workgroups: the fewest workgroups that keep the per-workgroup count
// ceil(groups / cap), so every workgroup sweeps the same number of groups
// (up to one) and no tail of single-group workgroups is left behind.
inline int64_t balanced_grid(int64_t groups, int64_t cap)
{
    if (groups <= cap) return groups;
    const int64_t per = (groups + cap - 1) / cap;
    return (groups + per - 1) / per;
}

// Elements per CU, over all fields, up to which the spread form is taken: what is
// resident at once, one workgroup an element from N = 5 on, more elements in one
// below.  us, column form / spread form: FP64 N = 4, 720 elements 4.5 / 3.8, 2184
// 5.2 / 5.4; N = 5, 990 5.6 / 5.2, 1716 6.8 / 7.3; N = 6, 504 5.4 / 4.7, 720 with the mass
// term 5.7 / 6.3; N = 7, 210 5.5 / 4.4, 504 6.1 / 6.1, 720 6.4 / 7.8; N = 8, 504 9.5 / 7.7,
// 720 10.5 / 11.1; N = 9, 210 9.8 / 6.9, 336 10.9 / 11.7; FP32 N = 6, 720 4.2 / 4.0; N = 8,
// 504 6.1 / 4.9; N = 10, 210 7.2 / 5.0.  Where a single field goes in two phases at the
// smallest sizes it needs none (N = 2, 3360 elements 3.2 / 3.7); several fields do
// (FP32 N = 3, three fields of 504: 3.7 / 3.1, two of 1716 3.8 / 3.4; N = 2, two of 2184
// 3.6 / 3.3, FP64 4.0 / 3.6).
template <int NQ, typename T>
constexpr int ax_spread_per_cu(int nf)
{
    if (nf == 1 && NQ <= (sizeof(T) == 4 ? 4 : 3)) return 0;
    if (NQ == 2) return 0;
    if (NQ == 3) return sizeof(T) == 4 ? 36 : 28;
    if (NQ == 4 && sizeof(T) == 4) return 16;
    return NQ <= 5 ? 8 : NQ == 6 ? 4 : NQ == 7 && sizeof(T) == 4 ? 3 : NQ <= 9 ? 2 : NQ <= 12 ? 1 : 0;
}

// The two forms give the same bits per point.  Their partial sums cover different
// points, and a batch has to have those of its single fields: with partial sums
// the line does not depend on the number of fields.  It then lies lower for some
// orders, as every workgroup adds up the records of the update for itself (a
// Jacobi-PCG iteration, us, column / spread: N = 4, 1716 elements 20.2 / 21.0; N = 5,
// 990 20.7 / 22.1; N = 7, 504 19.7 / 20.2; N = 8, 336 24.6 / 25.7; but N = 6, 336
// 16.8 / 16.3; N = 9, 210 25.1 / 21.7; N = 10, 210 27.4 / 25.9).
template <int NQ, typename T>
inline bool ax_spread(const Level &L, int nf, bool helm, bool vark, bool dot)
{
    static_assert(ax_spread_per_cu<NQ, T>(1) < kAxMaxBlocksPerCU, "the buffer of partial sums");
    // single FP64 fields in forms that spill: N = 10 with k, 120 elements 11.6 / 16.3; N = 11 with the
    // mass term 11.7 / 13.3
    if (sizeof(T) == 8 && !dot && nf == 1 && ((NQ >= 11 && vark) || (NQ >= 12 && helm))) return false;
    constexpr int half = NQ == 5 || NQ == 6 || NQ == 8 || NQ == 9 ? 2 : 1;
    const int64_t cu = L.n_cu > 0 ? L.n_cu : 256;
    if (dot) return L.E * half <= cu * ax_spread_per_cu<NQ, T>(1);
    return L.E * nf <= cu * ax_spread_per_cu<NQ, T>(nf);
}

// the compiled forms: mass term, coefficient (one field), partial sums (FP64)
#define SEM_AX_FORMS(VARK_)                                                                    \
    if constexpr (sizeof(T) == 8) {                                                            \
        if (partial != nullptr) {                                                              \
            if constexpr (VARK_) {                                                             \
                if (vark && helm) SEM_AX_LAUNCH(true, true, true);                             \
                if (vark && !helm) SEM_AX_LAUNCH(false, true, true);                           \
            }                                                                                  \
            if (!vark && helm) SEM_AX_LAUNCH(true, false, true);                               \
            if (!vark && !helm) SEM_AX_LAUNCH(false, false, true);                             \
            SEM_HIP(hipGetLastError());                                                        \
            return SEM_OK;                                                                     \
        }                                                                                      \
    }                                                                                          \
    if constexpr (VARK_) {                                                                     \
        if (vark && helm) SEM_AX_LAUNCH(true, true, false);                                    \
        if (vark && !helm) SEM_AX_LAUNCH(false, true, false);                                  \
    }                                                                                          \
    if (!vark && helm) SEM_AX_LAUNCH(true, false, false);                                      \
    if (!vark && !helm) SEM_AX_LAUNCH(false, false, false);

template <int NQ, typename T>
static int ax_split_launch(const Level &L, const T *G, const T *B, const T *D, const T *u, int64_t ldu,
                           T *w, int64_t ldw, const VSet &vs, double h1, double h2, const T *k,
                           double *partial, int64_t pst, int64_t *nblocks, hipStream_t s,
                           const int *skip, int skip_stride, const PcgDir &dir)
{
    using S = AxSplitShape<NQ>;
    const int64_t nb = (L.E + S::EPB - 1) / S::EPB;
    const bool helm = h2 != 0.0, vark = k != nullptr, dot = partial != nullptr;
    if (nblocks) *nblocks = nb;
    const dim3 grid((unsigned)nb, (unsigned)vs.n), block(S::THREADS);
#define SEM_AX_LAUNCH(H, V, P)                                                                 \
    hipLaunchKernelGGL((ax_split_kernel<NQ, T, H, V, P>), grid, block, 0, s, L.E, G, B, k, D, \
                       (T)h1, (T)h2, u, ldu, w, ldw, vs, partial, pst, skip, skip_stride, dir)
    SEM_AX_FORMS(true)
#undef SEM_AX_LAUNCH
    SEM_HIP(hipGetLastError());
    return SEM_OK;
}

// One launch for the NF vectors of vs (one, or up to kMaxRhs with nq <= 8).
// Every field's arithmetic is that of a single-field call.
template <int NQ, typename T, int NW, int NI, bool TWO>
static int ax_launch(const Level &L, const T *G, const T *B, const T *D, const T *u, int64_t ldu,
                     T *w, int64_t ldw, const VSet &vs, double h1, double h2, const T *k,
                     double *partial, int64_t pst, int64_t *nblocks, hipStream_t s, const int *skip,
                     int skip_stride, const PcgDir &dir)
{
    using S = AxShape<NQ>;
    constexpr int NF = NW * NI;
    const int64_t groups = (L.E + S::EPB - 1) / S::EPB;
    const bool helm = h2 != 0.0, vark = k != nullptr, dot = partial != nullptr;
    const int64_t cu = L.n_cu > 0 ? L.n_cu : 256;
    const int64_t nvb = balanced_grid(groups, cu * ax_blocks_per_cu<NQ, T>(1, false, dot));  // records
    const int64_t nb = NF == 1 ? nvb : balanced_grid(dot ? nvb : groups,
                                                     cu * ax_blocks_per_cu<NQ, T>(NF, NI > 1, dot));
    if (nblocks) *nblocks = nvb;
    if (nb == 0) return SEM_OK;
    const dim3 grid((unsigned)nb), block(S::threads(NW));
#define SEM_AX_LAUNCH(H, V, P)                                                                 \
    hipLaunchKernelGGL((ax_kernel<NQ, T, H, V, P, NW, NI, TWO>), grid, block, 0, s, L.E, G, B, k, \
                       D, (T)h1, (T)h2, u, ldu, w, ldw, vs, partial, pst, dot ? nvb : nb,     \
                       skip, skip_stride, dir)
    SEM_AX_FORMS(NF == 1)
#undef SEM_AX_LAUNCH
    SEM_HIP(hipGetLastError());
    return SEM_OK;
}

template <int NQ, typename T>
static int ax_dispatch(const Level &L, const T *G, const T *B, const T *D, const T *u, int64_t ldu,
                       T *w, int64_t ldw, const VSet &vs, double h1, double h2, const T *k,
                       double *partial, int64_t pst, int64_t *nblocks, hipStream_t s, const int *skip,
                       int skip_stride, const PcgDir &dir)
{
    if constexpr (ax_spread_per_cu<NQ, T>(2) > 0)
        if (ax_spread<NQ, T>(L, vs.n, h2 != 0.0, k != nullptr, partial != nullptr))
            return ax_split_launch<NQ, T>(L, G, B, D, u, ldu, w, ldw, vs, h1, h2, k, partial, pst, nblocks, s,
                                          skip, skip_stride, dir);
#define SEM_AX_NF(NW, NI, TWO)                                                                 \
    return ax_launch<NQ, T, NW, NI, TWO>(L, G, B, D, u, ldu, w, ldw, vs, h1, h2, k, partial,  \
                                         pst, nblocks, s, skip, skip_stride, dir)
    constexpr int64_t two = ax_two_phase_points<NQ, T>();
    if (vs.n == 1) {
        if constexpr (two > 0)
            if (L.nL <= two) SEM_AX_NF(1, 1, true);
        if constexpr (two < INT64_MAX) SEM_AX_NF(1, 1, false);
    }
    if constexpr (NQ <= 8) {
        if (k == nullptr) {
            if (ax_fields_inside<NQ, T>(L.nL, vs.n)) {
                // up to N = 3 in two phases (3 M points, two FP64 fields at N = 3 by
                // planes / in two phases 83.0 / 80.0, three 117 / 114)
                if (vs.n == 2) SEM_AX_NF(1, 2, NQ <= 4);
                if (vs.n == 3) SEM_AX_NF(1, 3, NQ <= 4);
                if constexpr (sizeof(T) == 4 || NQ <= 5)
                    if (vs.n == 4) SEM_AX_NF(1, 4, NQ <= 4);
            }
            if constexpr (NQ > 2) {
                if (vs.n == 2) SEM_AX_NF(2, 1, false);
                if (vs.n == 3) SEM_AX_NF(3, 1, false);
                if (vs.n == 4) SEM_AX_NF(4, 1, false);
            }
        }
    }
#undef SEM_AX_NF
    // one field at a time (several with variable coefficient, or elements wider than a wavefront)
    for (int q = 0; q < vs.n; ++q) {
        VSet one{0, 0u};
        one.push(vs.at(q));
        SEM_TRY((ax_launch<NQ, T, 1, 1, (two == INT64_MAX)>(L, G, B, D, u, ldu, w, ldw, one, h1, h2, k, partial,
                                                            pst, nblocks, s, skip, skip_stride, dir)));
    }
    return SEM_OK;
}

// lanes that sum an update's records in an operator with a direction update
template <int NQ>
static int ax_direction_lanes_nq(const Level &L, double h2, const double *k)
{
    int threads = AxShape<NQ>::THREADS;
    if constexpr (ax_spread_per_cu<NQ, double>(1) > 0)
        if (ax_spread<NQ, double>(L, 1, h2 != 0.0, k != nullptr, true)) threads = AxSplitShape<NQ>::THREADS;
    return std::min(64, threads);
}

template <typename T>
int launch_ax_multi(const Level &L, const T *G, const T *B, const T *D, const T *u, int64_t ldu, T *w,
                    int64_t ldw, const VSet &vs, double h1, double h2, const T *k, double *partial,
                    int64_t pst, int64_t *nblocks, hipStream_t s, const int *skip, int skip_stride,
                    const PcgDir &dir)
{
    if (vs.n <= 0) return SEM_OK;
    if (sizeof(T) == 4 && partial != nullptr) {
        set_error("ax: partial sums are formed in FP64 only");
        return SEM_EINVAL;
    }
#define SEM_AX_CASE(NQ)                                                                        \
    case NQ:                                                                                   \
        return ax_dispatch<NQ, T>(L, G, B, D, u, ldu, w, ldw, vs, h1, h2, k, partial, pst,    \
                                  nblocks, s, skip, skip_stride, dir);
    switch (L.nq) {
        SEM_AX_CASE(2) SEM_AX_CASE(3) SEM_AX_CASE(4) SEM_AX_CASE(5) SEM_AX_CASE(6)
        SEM_AX_CASE(7) SEM_AX_CASE(8) SEM_AX_CASE(9) SEM_AX_CASE(10) SEM_AX_CASE(11)
        SEM_AX_CASE(12) SEM_AX_CASE(13) SEM_AX_CASE(14) SEM_AX_CASE(15) SEM_AX_CASE(16)
    default: set_error("ax: unsupported order N=%d", L.N); return SEM_EINVAL;
    }
#undef SEM_AX_CASE
}

template <typename T>
int launch_ax(const Level &L, const T *G, const T *B, const T *D, const T *u, T *w, double h1,
              double h2, const T *k, double *partial, int64_t *nblocks, hipStream_t s,
              const int *skip)
{
    return launch_ax_multi<T>(L, G, B, D, u, 0, w, 0, VSet::one(), h1, h2, k, partial, 0, nblocks, s,
                              skip, 0);
}

}  // namespace semx
