// Dealiased advection operator (NekRS paper Sec. 2.1 eqs. (stdadv) and (hyp):
// the advection term of the EXT and characteristics formulations; Sec. 2.3:
// its integrand has degree 3N and needs a quadrature finer than GLL;
// Sec. 3.3: the advection kernels, whose 2D thread structure with 1D register
// arrays along the third direction is the layout used here).
//
// Per element, with the M-point Gauss rule in each direction:
//   J [M][nq]  interpolation from the GLL nodes to the Gauss points,
//   Jd = J Dh  derivative of the interpolant at the Gauss points,
//   ct [3][M^3] = rho~ |det X| dr_q/dx . (J3 c), X = dx/dr of the interpolated
//              element map (once per velocity field),
//   out = J3^T sum_q ct_q d_q(J3 w)   (every advected field).
//
// Thread layout (one workgroup per element, M^2 lanes rounded up to whole
// wavefronts): lane t = a + M b owns the Gauss column (b, a) and keeps values
// along the third index in registers.  The i-contraction runs on lanes
// t = j + nq k over GLL rows (coefficients J[a][i] are wave-uniform), the
// j-contraction on the columns with the lane's rows of J and Jd in registers,
// and the k-contractions forward and back run entirely in registers, the
// transposed interpolation along c being accumulated point by point so the
// Gauss-point integrand is never stored.
#include <algorithm>
#include <vector>

#include "sem_internal.h"

namespace semx {

namespace {

template <int NQ, int M>
struct AdvShape {
    static constexpr int NP = NQ * NQ * NQ;
    static constexpr int MM = M * M;
    static constexpr int M3 = MM * M;
    static constexpr int THREADS = ((MM + 63) / 64) * 64;
};

// The stages of a field and the last one of the field before share the
// intervals between barriers, three a field (six when every stage waited for
// the one before in two shared buffers): stage, barrier, i-contraction on the
// first wavefront beside the previous field's a -> i on the last, barrier, the
// columns, barrier, b -> j (24^3 elements, M = 11, three fields 268 -> 253 us).  A
// workgroup of one wavefront (M <= 8) ends each field before the next, which
// costs it nothing (deferred: M = 8 61 -> 64 us).
template <int NQ, int M>
__global__ void __launch_bounds__((AdvShape<NQ, M>::THREADS)) __attribute__((amdgpu_waves_per_eu(1, 8)))
    advect_kernel(int64_t E, const double *__restrict__ J, const double *__restrict__ Jd,
                  const double *__restrict__ ct, int nf, const double *__restrict__ w, int64_t ldw,
                  double *__restrict__ out, int64_t ldo)
{
    using S = AdvShape<NQ, M>;
    constexpr int NP = S::NP, MM = S::MM, M3 = S::M3, TH = S::THREADS, RM = NQ * NQ * M;
    __shared__ double sU[NP], sP[RM], sQ[RM], sG[NQ * MM], sH[RM];
    const int t = threadIdx.x;
    const bool col = t < MM;
    const int a = col ? t % M : 0, b = col ? t / M : 0;
    constexpr bool PIPE = TH >= 128;             // more than one wavefront
    const int t5 = PIPE ? t - (TH - 64) : t;  // lanes of the last contraction
    double Jb[NQ], Jdb[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        Jb[j] = J[b * NQ + j];
        Jdb[j] = Jd[b * NQ + j];
    }
    // the next field (or the next element's first field) is loaded into
    // registers while the current one is computed
    constexpr int PFN = (NP + TH - 1) / TH;
    double un[PFN];
    if (blockIdx.x < E) {
#pragma unroll
        for (int q = 0; q < PFN; ++q) {
            const int i = t + q * TH;
            un[q] = i < NP ? w[blockIdx.x * (int64_t)NP + i] : 0.0;
        }
    }
    // contraction over a -> i on GLL rows (k, j) of the field whose sH is ready
    auto finish = [&](double *o5) {
        if (t5 >= 0 && t5 < NQ * NQ) {
            double h[M];
#pragma unroll
            for (int a2 = 0; a2 < M; ++a2) h[a2] = sH[t5 * M + a2];
            double o[NQ];
#pragma unroll
            for (int i = 0; i < NQ; ++i) o[i] = 0.0;
#pragma unroll
            for (int a2 = 0; a2 < M; ++a2)
#pragma unroll
                for (int i = 0; i < NQ; ++i) o[i] += J[a2 * NQ + i] * h[a2];
#pragma unroll
            for (int i = 0; i < NQ; ++i) o5[t5 * NQ + i] = o[i];
        }
    };
    double *prev = nullptr;
    for (int64_t e = blockIdx.x; e < E; e += gridDim.x) {
        double c0[M], c1[M], c2[M];
        for (int f = 0; f < nf; ++f) {
#pragma unroll
            for (int q = 0; q < PFN; ++q) {
                const int i = t + q * TH;
                if (i < NP) sU[i] = un[q];
            }
            if (f == 0 && col) {  // issued after the staged field, consumed two stages later
                const double *cte = ct + e * 3 * M3 + t;
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    c0[c] = cte[c * MM];
                    c1[c] = cte[M3 + c * MM];
                    c2[c] = cte[2 * M3 + c * MM];
                }
            }
            {
                int64_t en = e;
                int fn = f + 1;
                if (fn == nf) {
                    fn = 0;
                    en = e + gridDim.x;
                }
                if (en < E) {
                    const double *src = w + fn * ldw + en * NP;
#pragma unroll
                    for (int q = 0; q < PFN; ++q) {
                        const int i = t + q * TH;
                        un[q] = i < NP ? src[i] : 0.0;
                    }
                }
            }
            __syncthreads();  // sU staged; the previous field's sH complete
            // contraction over i on GLL rows (k, j)
            if (t < NQ * NQ) {
                double r[NQ];
#pragma unroll
                for (int i = 0; i < NQ; ++i) r[i] = sU[t * NQ + i];
#pragma unroll
                for (int a2 = 0; a2 < M; ++a2) {
                    double p = 0.0, q = 0.0;
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        p += J[a2 * NQ + i] * r[i];
                        q += Jd[a2 * NQ + i] * r[i];
                    }
                    sP[t * M + a2] = p;
                    sQ[t * M + a2] = q;
                }
            }
            if constexpr (PIPE)
                if (prev) finish(prev);
            __syncthreads();
            if (col) {
                // contraction over j on the lane's Gauss column
                double Tr[NQ], Ts[NQ], Tt[NQ];
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    double xr = 0.0, xs = 0.0, xt = 0.0;
#pragma unroll
                    for (int j = 0; j < NQ; ++j) {
                        const double p = sP[(k * NQ + j) * M + a], q = sQ[(k * NQ + j) * M + a];
                        xr += Jb[j] * q;
                        xs += Jdb[j] * p;
                        xt += Jb[j] * p;
                    }
                    Tr[k] = xr;
                    Ts[k] = xs;
                    Tt[k] = xt;
                }
                // over k: derivatives at the Gauss points, integrand, and the
                // transposed interpolation back along k, point by point
                double G[NQ];
#pragma unroll
                for (int k = 0; k < NQ; ++k) G[k] = 0.0;
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    double dr = 0.0, ds = 0.0, dt = 0.0;
#pragma unroll
                    for (int k = 0; k < NQ; ++k) {
                        dr += J[c * NQ + k] * Tr[k];
                        ds += J[c * NQ + k] * Ts[k];
                        dt += Jd[c * NQ + k] * Tt[k];
                    }
                    const double fv = c0[c] * dr + c1[c] * ds + c2[c] * dt;
#pragma unroll
                    for (int k = 0; k < NQ; ++k) G[k] += J[c * NQ + k] * fv;
                }
#pragma unroll
                for (int k = 0; k < NQ; ++k) sG[k * MM + t] = G[k];
            }
            __syncthreads();
            // contraction over b -> j on lanes (a, k)
            for (int r = t; r < NQ * M; r += TH) {
                const int a2 = r % M, k = r / M;
                double H[NQ];
#pragma unroll
                for (int j = 0; j < NQ; ++j) H[j] = 0.0;
#pragma unroll
                for (int b2 = 0; b2 < M; ++b2) {
                    const double g = sG[(k * M + b2) * M + a2];
#pragma unroll
                    for (int j = 0; j < NQ; ++j) H[j] += J[b2 * NQ + j] * g;
                }
#pragma unroll
                for (int j = 0; j < NQ; ++j) sH[(k * NQ + j) * M + a2] = H[j];
            }
            double *o5 = out + f * ldo + e * NP;
            if constexpr (PIPE) {
                prev = o5;
            } else {
                __syncthreads();
                finish(o5);
            }
        }
    }
    if constexpr (PIPE) {
        __syncthreads();
        if (prev) finish(prev);
    }
}

// The 3D thread-block variant (Sec. 3.3: one thread per quadrature point,
// possible while the M^3 points fit one workgroup, M <= 10): thread
// t = a + M b + M^2 c owns the Gauss point (c, b, a) and keeps its three
// contravariant velocity components in registers; every contraction is a
// pass through LDS (three buffers used in rotation) with a barrier between.
template <int NQ, int M>
struct Adv3Shape {
    static constexpr int NP = NQ * NQ * NQ, MM = M * M, M3 = MM * M;
    static constexpr int THREADS = ((M3 + 63) / 64) * 64;
    static constexpr int SX = (2 * NQ * NQ * M > NQ * MM) ? 2 * NQ * NQ * M : NQ * MM;  // P, Q; then G
    static constexpr int SY = (3 * NQ * MM > NQ * NQ * M) ? 3 * NQ * MM : NQ * NQ * M;  // T; then H
    static constexpr int SZ = (NP > M3) ? NP : M3;                                     // u; then f
};

template <int NQ, int M>
__global__ void __launch_bounds__((Adv3Shape<NQ, M>::THREADS))
    advect3d_kernel(int64_t E, const double *__restrict__ J, const double *__restrict__ Jd,
                    const double *__restrict__ ct, int nf, const double *__restrict__ w, int64_t ldw,
                    double *__restrict__ out, int64_t ldo)
{
    using S = Adv3Shape<NQ, M>;
    constexpr int NP = S::NP, MM = S::MM, M3 = S::M3, TH = S::THREADS;
    static_assert(TH <= 1024, "the 3D variant needs M^3 <= 1024");
    __shared__ double sX[S::SX], sY[S::SY], sZ[S::SZ];
    __shared__ double sJ[M * NQ], sJd[M * NQ];
    const int t = threadIdx.x;
    for (int i = t; i < M * NQ; i += TH) {
        sJ[i] = J[i];
        sJd[i] = Jd[i];
    }
    const bool pt = t < M3;
    const int a = t % M, b = (t / M) % M, c = t / MM;
    for (int64_t e = blockIdx.x; e < E; e += gridDim.x) {
        double c0 = 0.0, c1 = 0.0, c2 = 0.0;
        if (pt) {
            const double *cte = ct + e * 3 * M3 + t;
            c0 = cte[0];
            c1 = cte[M3];
            c2 = cte[2 * M3];
        }
        for (int f = 0; f < nf; ++f) {
            __syncthreads();  // the previous field's last reads are done
            const double *u = w + f * ldw + e * NP;
            for (int i = t; i < NP; i += TH) sZ[i] = u[i];
            __syncthreads();
            // over i: P[k][j][a] = J u, Q[k][j][a] = Jd u
            if (t < NQ * NQ * M) {
                const int a2 = t % M, j = (t / M) % NQ, k = t / (M * NQ);
                double pp = 0.0, qq = 0.0;
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const double ui = sZ[(k * NQ + j) * NQ + i];
                    pp += sJ[a2 * NQ + i] * ui;
                    qq += sJd[a2 * NQ + i] * ui;
                }
                sX[(k * NQ + j) * M + a2] = pp;
                sX[NQ * NQ * M + (k * NQ + j) * M + a2] = qq;
            }
            __syncthreads();
            // over j: the three partial derivative fields T[d][k][b][a]
            if (t < NQ * MM) {
                const int a2 = t % M, b2 = (t / M) % M, k = t / MM;
                double xr = 0.0, xs = 0.0, xt = 0.0;
#pragma unroll
                for (int j = 0; j < NQ; ++j) {
                    const double pp = sX[(k * NQ + j) * M + a2];
                    const double qq = sX[NQ * NQ * M + (k * NQ + j) * M + a2];
                    xr += sJ[b2 * NQ + j] * qq;
                    xs += sJd[b2 * NQ + j] * pp;
                    xt += sJ[b2 * NQ + j] * pp;
                }
                sY[k * MM + b2 * M + a2] = xr;
                sY[(NQ + k) * MM + b2 * M + a2] = xs;
                sY[(2 * NQ + k) * MM + b2 * M + a2] = xt;
            }
            __syncthreads();
            // over k: reference derivatives at the thread's Gauss point, integrand
            if (pt) {
                double dr = 0.0, ds = 0.0, dt = 0.0;
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    dr += sJ[c * NQ + k] * sY[k * MM + b * M + a];
                    ds += sJ[c * NQ + k] * sY[(NQ + k) * MM + b * M + a];
                    dt += sJd[c * NQ + k] * sY[(2 * NQ + k) * MM + b * M + a];
                }
                sZ[t] = c0 * dr + c1 * ds + c2 * dt;
            }
            __syncthreads();
            // back over c: G[k][b][a]
            if (t < NQ * MM) {
                const int a2 = t % M, b2 = (t / M) % M, k = t / MM;
                double g = 0.0;
#pragma unroll
                for (int c2i = 0; c2i < M; ++c2i) g += sJ[c2i * NQ + k] * sZ[c2i * MM + b2 * M + a2];
                sX[k * MM + b2 * M + a2] = g;
            }
            __syncthreads();
            // back over b: H[k][j][a]
            if (t < NQ * NQ * M) {
                const int a2 = t % M, j = (t / M) % NQ, k = t / (M * NQ);
                double hh = 0.0;
#pragma unroll
                for (int b2 = 0; b2 < M; ++b2) hh += sJ[b2 * NQ + j] * sX[k * MM + b2 * M + a2];
                sY[(k * NQ + j) * M + a2] = hh;
            }
            __syncthreads();
            // back over a: out[k][j][i]
            if (t < NP) {
                const int i = t % NQ, j = (t / NQ) % NQ, k = t / (NQ * NQ);
                double o = 0.0;
#pragma unroll
                for (int a2 = 0; a2 < M; ++a2) o += sJ[a2 * NQ + i] * sY[(k * NQ + j) * M + a2];
                out[f * ldo + e * NP + t] = o;
            }
        }
    }
}

// ct[e][q][p] = rho~ (cofactor of dx/dr . J3 c): the contravariant velocity at
// the Gauss points from the element's coordinates and velocity alone.  The
// metric factors rho~ |det X| dr_q/dx_d are 72 M^3 bytes an element when kept
// (96 KB at M = 11, of 140 KB that the transform then moved: 0.955 ms = 4.8 TB/s
// on 32^3 elements); formed here from the 12 KB of coordinates the transform takes
// 0.68 to 0.74 ms: the LDS is busy for half of it, the FP64 units for 40%, the 57 KB
// left an element are half of it at the copy rate, and two waves a SIMD overlap
// little.
// Lane t = a + M b owns the Gauss column (b, a) as in the advection kernel.  The
// velocity components and the coordinates are contracted over i on their GLL
// rows, a row per lane straight from memory, and over j on the columns, through
// LDS; a column keeps the nine derivative lines along k in registers, its three
// velocity lines in LDS, and walks the M points: derivatives, the three cofactor
// rows as cross products, and their products with the velocity.
// From M = 9 on an element has two wavefronts or three, and two of them share the
// rows of a round: two velocity components, halves of the third, then J and Jd of
// a coordinate: five rounds of half the rows where one wavefront took six alone
// (N = 6, 343 / 4096 elements: 16.4 / 66.7 -> 14.7 / 59.2 us; at N = 7, where the
// points are most of the time, 19.2 / 83.4 -> 19.1 / 82.5).  Up to M = 5 a wavefront
// takes several elements, whose columns and rows fill its lanes (N = 1, 13824
// elements 14.8 -> 4.1; N = 2 28.8 -> 11.5; N = 3 39.5 -> 24.2).
// EW: elements of EW wavefront groups side by side.  Two workgroups of two
// wavefronts on a CU share two of its SIMDs, one workgroup of four takes all (N = 6,
// 343 elements 14.7 -> 13.7, N = 7 19.2 -> 18.2).
// CHECK: no velocity, bad |= 1 where det dx/dr <= 0.
template <int NQ, int M>
struct VelShape {
    static constexpr int MM = M * M;
    static constexpr int EPB = MM <= 32 ? 64 / MM : 1;  // elements of a workgroup
    static constexpr int COLS = EPB * MM, ROWS = EPB * NQ * NQ;
    static constexpr int THREADS = (COLS + 63) / 64 * 64;
    static constexpr bool DUO = THREADS > 64;
    static_assert(ROWS <= 64, "a row per lane of one wavefront");
};

template <int NQ, int M, bool CHECK, int EW>
__global__ void __launch_bounds__((EW * VelShape<NQ, M>::THREADS), 2)
    velocity_kernel(int64_t E, const double *__restrict__ J, const double *__restrict__ Jd,
                    const double *__restrict__ wq, const double *__restrict__ x,
                    const double *__restrict__ y, const double *__restrict__ z,
                    const double *__restrict__ cv, int64_t ldc, double *__restrict__ ct, int *bad)
{
    using S = VelShape<NQ, M>;
    constexpr int MM = S::MM, M3 = MM * M, TH = S::THREADS, EPB = S::EPB, ROWS = S::ROWS;
    // at N = 7 the rows come through LDS, since a row each of the coming round does
    // not fit beside the lines (36 registers spilled, 24^3 elements 283 -> 360 us)
    constexpr bool DUO = S::DUO, STAGE = NQ >= 8, PAIR = DUO && !STAGE && !CHECK;
    constexpr int NP = NQ * NQ * NQ, PFN = STAGE ? (NP + TH - 1) / TH : NQ;
    constexpr int ROUNDS = CHECK ? 3 : PAIR ? 5 : 6;
    __shared__ double sU_[EW][STAGE ? NP : 1];
    __shared__ double sP_[EW][ROWS * M], sQ_[EW][ROWS * M];
    __shared__ double sV_[EW][CHECK ? 1 : 3 * NQ][S::COLS];
    __shared__ double sJ[M][NQ + 1], sJd[M][NQ + 1];
    static_assert(EW == 1 || DUO, "several elements of several wavefronts");
    const int ew = EW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / TH);
    const int t = threadIdx.x - ew * TH, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    double *const sU = sU_[ew], *const sP = sP_[ew], *const sQ = sQ_[ew];
    double(*const sV)[S::COLS] = sV_[ew];
    const int el = EPB == 1 ? 0 : t / MM, tc = t - el * MM;
    const bool col = t < S::COLS;
    const int a = col ? tc % M : 0, b = col ? tc / M : 0;
    const int at0 = (col ? el : 0) * NQ * NQ * M + a;  // of the column's element in sP, sQ
    for (int i = threadIdx.x; i < M * NQ; i += EW * TH) {
        sJ[i / NQ][i % NQ] = J[i];
        sJd[i / NQ][i % NQ] = Jd[i];
    }
    const double wab = wq[a] * wq[b];
    // Workgroup g's elements lie 8 apart: each is on the XCD, whose L2 then holds its
    // ct, where the advection kernel of one element a workgroup will read it (N = 6,
    // 512 elements, both kernels: 29.7 us with neighbours, 25.6 so; N = 3, 4096: 22.9 /
    // 19.1)
    constexpr int W = EPB * EW;
    auto elem = [](int64_t g, int slot) { return (g >> 3) * (8 * W) + (g & 7) + 8 * slot; };
    const int64_t groups = E / (8 * W) * 8 + min(E % (8 * W), (int64_t)8);
    double un[PFN];  // the row of the coming round, or the lane's part of the field
    const int er = EPB == 1 ? 0 : lane / (NQ * NQ), row = lane - er * (NQ * NQ);  // element slot, row in it
    auto fetch = [&](int r, int64_t g) {
        const int f = CHECK ? 3 + r : !PAIR ? r : r == 0 ? (wv == 1 ? 1 : 0) : r + 1;
        const double *p = f < 3 ? cv + f * ldc : f == 3 ? x : f == 4 ? y : z;
        const int64_t e = elem(g, ew + er);
        const bool in = W == 1 || e < E;
        if constexpr (STAGE) {
#pragma unroll
            for (int q = 0; q < PFN; ++q) {
                const int i = t + q * TH;
                un[q] = in && i < NP ? p[e * NP + i] : 0.0;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NQ; ++i) un[i] = in && lane < ROWS ? p[e * NP + row * NQ + i] : 0.0;
        }
    };
    if (blockIdx.x < groups) fetch(0, blockIdx.x);
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        double T[3][3][NQ];  // T[d][q]: line of dx_d/dr_q before the k contraction
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const bool coord = CHECK || r >= (PAIR ? 2 : 3), pair = PAIR && r == 0;
            const int d = CHECK ? r : PAIR ? (r < 2 ? 2 * r : r - 2) : r % 3;  // component
            auto next = [&]() {
                if (r + 1 < ROUNDS)
                    fetch(r + 1, g);
                else if (g + gridDim.x < groups)
                    fetch(0, g + gridDim.x);
            };
            if constexpr (STAGE) {
#pragma unroll
                for (int q = 0; q < PFN; ++q)
                    if (t + q * TH < NP) sU[t + q * TH] = un[q];
                next();
            }
            __syncthreads();  // the columns of the round before are done with sP, sQ
            // over i on GLL rows (k, j): J u, and for a coordinate Jd u
            if (lane < ROWS && wv < 2) {
                double v[NQ];
#pragma unroll
                for (int i = 0; i < NQ; ++i) v[i] = STAGE ? sU[STAGE ? lane * NQ + i : 0] : un[STAGE ? 0 : i];
                if constexpr (DUO) {
                    const double *Jm = coord && wv == 1 ? Jd : J;
                    double *dst = (wv == 1 && (pair || coord) ? sQ : sP) + lane * M;
                    // a single component: half of the Gauss points each, all in sP
                    constexpr int H = (M + 1) / 2;
                    const int n0 = !pair && !coord && wv == 1 ? H : 0;
                    const int n1 = !pair && !coord && wv == 0 ? H : M;
// (unrolled by the 11 points of N = 7: 24^3 elements 307 us, by more 283)
#pragma unroll 16
                    for (int a2 = n0; a2 < n1; ++a2) {
                        double p = 0.0;
#pragma unroll
                        for (int i = 0; i < NQ; ++i) p += Jm[a2 * NQ + i] * v[i];
                        dst[a2] = p;
                    }
                } else {
#pragma unroll
                    for (int a2 = 0; a2 < M; ++a2) {
                        double p = 0.0, q = 0.0;
#pragma unroll
                        for (int i = 0; i < NQ; ++i) {
                            p += J[a2 * NQ + i] * v[i];
                            if (coord) q += Jd[a2 * NQ + i] * v[i];
                        }
                        sP[lane * M + a2] = p;
                        if (coord) sQ[lane * M + a2] = q;
                    }
                }
            }
            if constexpr (!STAGE) next();  // behind the rows: one row each in registers
            __syncthreads();
            if (col) {
                if (coord) {
                    double(&Tf)[3][NQ] = T[d];
#pragma unroll
                    for (int k = 0; k < NQ; ++k) Tf[0][k] = Tf[1][k] = Tf[2][k] = 0.0;
#pragma unroll
                    for (int j = 0; j < NQ; ++j) {
                        const double jb = sJ[b][j], jd = sJd[b][j];
#pragma unroll
                        for (int k = 0; k < NQ; ++k) {
                            const int at = at0 + (k * NQ + j) * M;
                            const double p = sP[at], q = sQ[at];
                            Tf[0][k] += jb * q;
                            Tf[1][k] += jd * p;
                            Tf[2][k] += jb * p;
                        }
                    }
                } else {
                    double V0[NQ], V1[NQ];
#pragma unroll
                    for (int k = 0; k < NQ; ++k) V0[k] = V1[k] = 0.0;
#pragma unroll
                    for (int j = 0; j < NQ; ++j) {
                        const double jb = sJ[b][j];
#pragma unroll
                        for (int k = 0; k < NQ; ++k) {
                            const int at = at0 + (k * NQ + j) * M;
                            V0[k] += jb * sP[at];
                            if (pair) V1[k] += jb * sQ[at];
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NQ; ++k) {
                        sV[CHECK ? 0 : d * NQ + k][t] = V0[k];
                        if (pair) sV[CHECK ? 0 : NQ + k][t] = V1[k];
                    }
                }
            }
        }
        const int64_t e = elem(g, ew + el);
        if (col && (W == 1 || e < E)) {
            double *ce = CHECK ? nullptr : ct + e * 3 * M3 + tc;
#pragma unroll 1
            for (int c = 0; c < M; ++c) {
                const double *Jc = J + c * NQ, *Jdc = Jd + c * NQ;
                double X[3][3];  // X[d][q] = dx_d/dr_q
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    X[d][0] = X[d][1] = X[d][2] = 0.0;
#pragma unroll
                    for (int k = 0; k < NQ; ++k) {
                        X[d][0] += Jc[k] * T[d][0][k];
                        X[d][1] += Jc[k] * T[d][1][k];
                        X[d][2] += Jdc[k] * T[d][2][k];
                    }
                }
                // cofactor rows: A[q] = dx/dr_{q+1} x dx/dr_{q+2}
                double A[3][3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int q1 = (q + 1) % 3, q2 = (q + 2) % 3;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const int d1 = (d + 1) % 3, d2 = (d + 2) % 3;
                        A[q][d] = X[d1][q1] * X[d2][q2] - X[d2][q1] * X[d1][q2];
                    }
                }
                if constexpr (CHECK) {
                    const double det = X[0][0] * A[0][0] + X[1][0] * A[0][1] + X[2][0] * A[0][2];
                    if (!(det > 0.0)) atomicOr(bad, 1);
                } else {
                    double v[3];
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        v[d] = 0.0;
#pragma unroll
                        for (int k = 0; k < NQ; ++k) v[d] += Jc[k] * sV[d * NQ + k][t];
                    }
                    const double rho = wab * wq[c];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        ce[q * M3 + c * MM] = rho * (A[q][0] * v[0] + A[q][1] * v[1] + A[q][2] * v[2]);
                }
            }
        }
    }
}

// The same for few elements, where one workgroup's chain of dependent steps (six
// fields, two barriers each) is the time: three lane groups of an element take a
// velocity component and a coordinate each, all six fields' rows are contracted at
// once, the lines meet in LDS (in place of the rows) and each group walks a third
// of the points.  N = 7, 27 / 216 / 512 elements: 14.6 / 16.0 / 21.9 us in turn,
// 10.5 / 11.9 / 21.7 so (N = 5: 125 / 512 elements 10.7 / 11.5 and 6.8 / 9.6).
template <int NQ, int M>
__global__ void __launch_bounds__((3 * AdvShape<NQ, M>::THREADS), 1)
    velocity_spread_kernel(int64_t E, const double *__restrict__ J, const double *__restrict__ Jd,
                           const double *__restrict__ wq, const double *__restrict__ x,
                           const double *__restrict__ y, const double *__restrict__ z,
                           const double *__restrict__ cv, int64_t ldc, double *__restrict__ ct)
{
    using S = AdvShape<NQ, M>;
    constexpr int NP = S::NP, MM = S::MM, M3 = S::M3, TH = S::THREADS, NR = NQ * NQ;
    constexpr int ROWS = 6 * NP + 9 * NR * M, LINES = 12 * NQ * MM;
    __shared__ double lds[ROWS > LINES ? ROWS : LINES];
    double *const sU = lds, *const sP = lds + 6 * NP, *const sQ = sP + 6 * NR * M;
    const int64_t e = blockIdx.x;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x / TH), t = threadIdx.x - g * TH;
    const bool col = t < MM;
    const int a = col ? t % M : 0, b = col ? t / M : 0;
    const double wab = wq[a] * wq[b];
    {
        constexpr int PF = (6 * NP + 3 * TH - 1) / (3 * TH);
        double u[PF];
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const int i = min((int)threadIdx.x + m * 3 * TH, 6 * NP - 1), f = i / NP, q = i - f * NP;
            const double *p = f < 3 ? cv + f * ldc : f == 3 ? x : f == 4 ? y : z;
            u[m] = p[e * NP + q];
        }
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const int i = threadIdx.x + m * 3 * TH;
            if (i < 6 * NP) sU[i] = u[m];
        }
    }
    __syncthreads();
    // over i on GLL rows (k, j) of every field: J u, and for a coordinate Jd u
    for (int r = threadIdx.x; r < 6 * NR; r += 3 * TH) {
        double v[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) v[i] = sU[r * NQ + i];
#pragma unroll
        for (int a2 = 0; a2 < M; ++a2) {
            double p = 0.0;
#pragma unroll
            for (int i = 0; i < NQ; ++i) p += J[a2 * NQ + i] * v[i];
            sP[r * M + a2] = p;
        }
        if (r >= 3 * NR) {
#pragma unroll
            for (int a2 = 0; a2 < M; ++a2) {
                double q = 0.0;
#pragma unroll
                for (int i = 0; i < NQ; ++i) q += Jd[a2 * NQ + i] * v[i];
                sQ[(r - 3 * NR) * M + a2] = q;
            }
        }
    }
    __syncthreads();
    // over j on the columns: this group's velocity line and derivative lines
    double Vf[NQ], Tf[3][NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) Vf[k] = Tf[0][k] = Tf[1][k] = Tf[2][k] = 0.0;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        const double jb = J[b * NQ + j], jd = Jd[b * NQ + j];
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int at = (k * NQ + j) * M + a;
            const double p = sP[(3 + g) * NR * M + at], q = sQ[g * NR * M + at];
            Vf[k] += jb * sP[g * NR * M + at];
            Tf[0][k] += jb * q;
            Tf[1][k] += jd * p;
            Tf[2][k] += jb * p;
        }
    }
    // (summed before the barrier: sunk behind it all the rows' values stay in
    // registers, 150 of them spilled)
#pragma unroll
    for (int k = 0; k < NQ; ++k) asm volatile("" : "+v"(Vf[k]), "+v"(Tf[0][k]), "+v"(Tf[1][k]), "+v"(Tf[2][k]));
    __syncthreads();  // rows consumed: the lines take their place
    double *const sV = lds, *const sT = lds + 3 * NQ * MM;
    if (col)
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            sV[(g * NQ + k) * MM + t] = Vf[k];
#pragma unroll
            for (int q = 0; q < 3; ++q) sT[((g * 3 + q) * NQ + k) * MM + t] = Tf[q][k];
        }
    __syncthreads();
    if (col) {
        double T[3][3][NQ];
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < NQ; ++k) T[d][q][k] = sT[((d * 3 + q) * NQ + k) * MM + t];
        double *ce = ct + e * 3 * M3 + t;
#pragma unroll 1
        for (int c = M * g / 3; c < M * (g + 1) / 3; ++c) {
            const double *Jc = J + c * NQ, *Jdc = Jd + c * NQ;
            double X[3][3], v[3];  // X[d][q] = dx_d/dr_q
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                X[d][0] = X[d][1] = X[d][2] = v[d] = 0.0;
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    X[d][0] += Jc[k] * T[d][0][k];
                    X[d][1] += Jc[k] * T[d][1][k];
                    X[d][2] += Jdc[k] * T[d][2][k];
                    v[d] += Jc[k] * sV[(d * NQ + k) * MM + t];
                }
            }
            const double rho = wab * wq[c];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int q1 = (q + 1) % 3, q2 = (q + 2) % 3;
                double s = 0.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int d1 = (d + 1) % 3, d2 = (d + 2) % 3;
                    s += (X[d1][q1] * X[d2][q2] - X[d2][q1] * X[d1][q2]) * v[d];
                }
                ce[q * M3 + c * MM] = rho * s;
            }
        }
    }
}

int rule_default(int N) { return (3 * N + 2) / 2; }

// automatic choice: the 3D thread block up to this M, the 2D one above.  On
// 32^3 elements, three fields, the 2D block is faster at every compiled pair
// (N, M) = (3, 5) 75 vs 126 us, (4, 7) 170 vs 488, (5, 8) 256 vs 577,
// (6, 10) 558 vs 1556, so the 3D block is never picked automatically.
constexpr int kAdv3AutoMaxM = 0;

bool rule_supported(int N, int M) { return N >= 1 && N <= 7 && (M == rule_default(N) || M == rule_default(N) + 1); }

// dispatch over the compiled (nq, M) pairs: M = ceil((3N+1)/2) and one more
#define SEM_ADV_PAIRS(X) \
    X(2, 2) X(2, 3) X(3, 4) X(3, 5) X(4, 5) X(4, 6) X(5, 7) X(5, 8) X(6, 8) X(6, 9) X(7, 10) X(7, 11) X(8, 11) X(8, 12)

// ct from the velocity c, or with bad the check of the element map
int launch_velocity(sem_handle h, int M, const double *J, const double *Jd, const double *wq, const double *c,
                    int64_t ldc, double *ct, int *bad, hipStream_t s)
{
    const Level &L = h->lv[0];
    // as many workgroups as are resident (24^3 elements, 4 / 8 / 16 per CU: M = 11
    // 292 / 313 / 313 us, two waves a SIMD; M = 8 149 / 111 / 115, M = 7 99 / 76 / 77;
    // one element a workgroup, 8 / 16 / 32 per CU at 35^3, M = 5: 138 / 129 / 123, at
    // 40^3, M = 4: 141 / 132 / 117)
    const int64_t cu = L.n_cu > 0 ? L.n_cu : 256;
    const int64_t cap = cu * (M >= 10 ? 4 : M >= 7 ? 8 : 32);
    // The spread form's three lane groups of an element pay while they are resident
    // (us, spread / in turn: N = 3, 729 elements 5.8 / 6.1, 1000 6.6 / 6.3; N = 4, 1000 8.9 /
    // 9.4, 1331 12.7 / 11.7; N = 5, 512 8.7 / 10.0, 576 12.0 / 10.6; N = 6, 216 9.4 / 11.4,
    // 294 16.1 / 13.6; N = 7, 216 10.9 / 14.6, 294 18.9 / 17.9).
    // At M = 12 its nine wavefronts an element leave too few registers (68 spilled, 27
    // elements 26.2 us, 15.4 in turn).
    const int64_t few = bad || M > 11 ? 0 : cu * (L.nq <= 4 ? 3 : L.nq == 5 ? 4 : L.nq == 6 ? 2 : 1);
    // Two elements a workgroup where one each leaves SIMDs idle: up to two elements
    // a CU (at M = 12 three wavefronts each spread by themselves, 343 elements 22.1 /
    // 24.1), and in the second round of a grid that the cap cuts (N = 6, 1331 elements
    // 30.0 / 26.4 us, N = 7 39.5 / 37.1; else the longer barriers lose: 576 22.2 / 25.8).
    const bool two = !bad && M <= 11 && ((L.E > cu && L.E <= 2 * cu) || (L.E > 5 * cu && L.E <= 6 * cu));
#define SEM_VEL_FORM(NQ_, M_, CHECK_, EW_)                                                          \
    {                                                                                               \
        using S = VelShape<NQ_, M_>;                                                                \
        constexpr int64_t W = 8 * S::EPB * (EW_);                                                   \
        const int64_t groups = L.E / W * 8 + std::min<int64_t>(L.E % W, 8);                         \
        const dim3 grid((unsigned)std::max<int64_t>(1, std::min(groups, cap / (EW_))));             \
        hipLaunchKernelGGL((velocity_kernel<NQ_, M_, CHECK_, (EW_)>), grid, dim3((EW_) * S::THREADS), 0, s, \
                           L.E, J, Jd, wq, h->cx, h->cy, h->cz, c, ldc, ct, bad);                   \
    }
#define SEM_VEL(NQ_, M_)                                                                            \
    if (L.nq == NQ_ && M == M_) {                                                                   \
        constexpr bool duo = VelShape<NQ_, M_>::DUO && M_ <= 11;                                    \
        constexpr int ms = std::min(M_, 11);                                                        \
        if (L.E <= few)                                                                             \
            hipLaunchKernelGGL((velocity_spread_kernel<NQ_, ms>), dim3((unsigned)L.E),              \
                               dim3(3 * AdvShape<NQ_, ms>::THREADS), 0, s, L.E, J, Jd, wq, h->cx, h->cy, h->cz, \
                               c, ldc, ct);                                                         \
        else if (bad)                                                                               \
            SEM_VEL_FORM(NQ_, M_, true, 1)                                                          \
        else if (duo && two)                                                                        \
            SEM_VEL_FORM(NQ_, M_, false, duo ? 2 : 1)                                               \
        else                                                                                        \
            SEM_VEL_FORM(NQ_, M_, false, 1)                                                         \
        SEM_HIP(hipGetLastError());                                                                 \
        return SEM_OK;                                                                              \
    }
    SEM_ADV_PAIRS(SEM_VEL)
#undef SEM_VEL
#undef SEM_VEL_FORM
    set_error("advection: no kernel for N = %d, M = %d", L.N, M);
    return SEM_EINVAL;
}

#define SEM_ADV3_PAIRS(X) \
    X(2, 2) X(2, 3) X(3, 4) X(3, 5) X(4, 5) X(4, 6) X(5, 7) X(5, 8) X(6, 8) X(6, 9) X(7, 10)

bool has_3d(int nq, int M)
{
#define SEM_H3(NQ_, M_) \
    if (nq == NQ_ && M == M_) return true;
    SEM_ADV3_PAIRS(SEM_H3)
#undef SEM_H3
    return false;
}

int launch_advect(const Level &L, int M, int variant, const double *J, const double *Jd, const double *ct,
                  int nf, const double *w, int64_t ldw, double *out, int64_t ldo, hipStream_t s)
{
    if (variant == SEM_ADVECT_3D) {
        const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(L.E, (int64_t)(L.n_cu > 0 ? L.n_cu : 256) * 8)));
#define SEM_ADV3(NQ_, M_)                                                                           \
    if (L.nq == NQ_ && M == M_) {                                                                   \
        hipLaunchKernelGGL((advect3d_kernel<NQ_, M_>), grid, dim3(Adv3Shape<NQ_, M_>::THREADS), 0, s, \
                           L.E, J, Jd, ct, nf, w, ldw, out, ldo);                                   \
        SEM_HIP(hipGetLastError());                                                                 \
        return SEM_OK;                                                                              \
    }
        SEM_ADV3_PAIRS(SEM_ADV3)
#undef SEM_ADV3
        set_error("advection: no 3D kernel for N = %d, M = %d", L.N, M);
        return SEM_EINVAL;
    }
    // workgroups per CU, 16 / 32 / 64 (us): M = 11 254 / 248 / 250 and M = 7
    // 63 / 55 / 56 for three fields on 24^3 elements; small rules behind the
    // velocity transform, M = 5 on 30^3 106 / 122 / 122, M = 4 on 40^3 240 / 263 / 255
    const int64_t cap = (int64_t)(L.n_cu > 0 ? L.n_cu : 256) * (M >= 7 ? 32 : 16);
    const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(L.E, cap)));
#define SEM_ADV(NQ_, M_)                                                                             \
    if (L.nq == NQ_ && M == M_) {                                                                    \
        hipLaunchKernelGGL((advect_kernel<NQ_, M_>), grid, dim3(AdvShape<NQ_, M_>::THREADS), 0, s,   \
                           L.E, J, Jd, ct, nf, w, ldw, out, ldo);                                    \
        SEM_HIP(hipGetLastError());                                                                  \
        return SEM_OK;                                                                               \
    }
    SEM_ADV_PAIRS(SEM_ADV)
#undef SEM_ADV
    set_error("advection: no kernel for N = %d, M = %d", L.N, M);
    return SEM_EINVAL;
}

int alloc_upload(double **dst, const std::vector<double> &v)
{
    SEM_HIP(hipMalloc(dst, sizeof(double) * v.size()));
    SEM_HIP(hipMemcpy(*dst, v.data(), sizeof(double) * v.size(), hipMemcpyHostToDevice));
    return SEM_OK;
}

int advect_setup(sem_handle h, int M, hipStream_t s)
{
    const Level &L = h->lv[0];
    const int N = L.N, nq = L.nq;
    std::vector<double> xi(nq), D(nq * nq), g(M), wq(M), J(M * nq), Jd(M * nq, 0.0);
    SEM_TRY(host_gll(N, xi.data(), nullptr, D.data()));
    SEM_TRY(host_gauss(M, g.data(), wq.data()));
    host_interp(nq, xi.data(), M, g.data(), J.data());
    for (int a = 0; a < M; ++a)
        for (int l = 0; l < nq; ++l) {
            double v = 0.0;
            for (int i = 0; i < nq; ++i) v += J[a * nq + i] * D[i * nq + l];
            Jd[a * nq + l] = v;
        }
    auto &A = h->adv;
    SEM_TRY(alloc_upload(&A.J, J));
    SEM_TRY(alloc_upload(&A.Jd, Jd));
    SEM_TRY(alloc_upload(&A.wq, wq));
    int *bad = nullptr;
    SEM_HIP(hipMalloc(&bad, sizeof(int)));
    int hbad = 0;
    int rc = SEM_OK;
    if (hipMemsetAsync(bad, 0, sizeof(int), s) != hipSuccess) rc = SEM_EHIP;
    if (rc == SEM_OK) rc = launch_velocity(h, M, A.J, A.Jd, A.wq, nullptr, 0, nullptr, bad, s);
    if (rc == SEM_OK && (hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
                         hipStreamSynchronize(s) != hipSuccess))
        rc = SEM_EHIP;
    (void)hipFree(bad);
    if (rc != SEM_OK) {
        set_error("advection setup: %s", hipGetErrorString(hipGetLastError()));
        return rc;
    }
    if (hbad) {
        set_error("advection setup: det(dx/dr) <= 0 at a Gauss point");
        return SEM_EMESH;
    }
    A.M = M;
    return SEM_OK;
}

}  // namespace

void free_advect(sem_handle h)
{
    auto &A = h->adv;
    void *ptrs[] = {A.J, A.Jd, A.wq};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    A = sem_handle_s::Advect{};
}

}  // namespace semx

using namespace semx;

extern "C" {

int sem_advect_setup(sem_handle h, int M, int variant, int *M_used, void *stream)
{
    if (!h || h->n_levels < 1) {
        set_error("sem_advect_setup: null handle");
        return SEM_EINVAL;
    }
    const int N = h->lv[0].N;
    if (M == 0) M = rule_default(N);
    if (M < N + 1 || M > kMaxGauss || !rule_supported(N, M)) {
        set_error("sem_advect_setup: M = %d not supported for N = %d (N <= 7, M = %d or %d)", M, N,
                  rule_default(N), rule_default(N) + 1);
        return SEM_EINVAL;
    }
    if (!h->cx) {
        set_error("sem_advect_setup: the handle holds no coordinates");
        return SEM_EINVAL;
    }
    if (variant != SEM_ADVECT_AUTO && variant != SEM_ADVECT_2D && variant != SEM_ADVECT_3D) {
        set_error("sem_advect_setup: bad variant %d", variant);
        return SEM_EINVAL;
    }
    const bool can3 = has_3d(N + 1, M);
    if (variant == SEM_ADVECT_3D && !can3) {
        set_error("sem_advect_setup: the 3D variant needs M^3 <= 1024 (M = %d, N = %d)", M, N);
        return SEM_EINVAL;
    }
    if (variant == SEM_ADVECT_AUTO) variant = (can3 && M <= kAdv3AutoMaxM) ? SEM_ADVECT_3D : SEM_ADVECT_2D;
    free_advect(h);
    const int rc = advect_setup(h, M, (hipStream_t)stream);
    if (rc != SEM_OK) {
        free_advect(h);
        return rc;
    }
    h->adv.variant = variant;
    if (M_used) *M_used = M;
    return SEM_OK;
}

int sem_advect_velocity(sem_handle h, const double *c, int64_t ldc, double *ct, void *stream)
{
    if (!h || !c || !ct) {
        set_error("sem_advect_velocity: null argument");
        return SEM_EINVAL;
    }
    const auto &A = h->adv;
    if (A.M == 0) {
        set_error("sem_advect_velocity: call sem_advect_setup first");
        return SEM_EINVAL;
    }
    const Level &L = h->lv[0];
    if (ldc < L.nL) {
        set_error("sem_advect_velocity: ldc = %lld < n_local = %lld", (long long)ldc, (long long)L.nL);
        return SEM_EINVAL;
    }
    const hipStream_t s = (hipStream_t)stream;
    return launch_velocity(h, A.M, A.J, A.Jd, A.wq, c, ldc, ct, nullptr, s);
}

int sem_advect(sem_handle h, const double *ct, int nf, const double *w, int64_t ldw, double *out, int64_t ldo,
               void *stream)
{
    if (!h) {
        set_error("sem_advect: null handle");
        return SEM_EINVAL;
    }
    const auto &A = h->adv;
    if (A.M == 0) {
        set_error("sem_advect: call sem_advect_setup first");
        return SEM_EINVAL;
    }
    if (nf < 0 || nf > kMaxRhs) {
        set_error("sem_advect: nf = %d outside [0, %d]", nf, kMaxRhs);
        return SEM_EINVAL;
    }
    if (nf == 0) return SEM_OK;
    if (!ct || !w || !out) {
        set_error("sem_advect: null argument");
        return SEM_EINVAL;
    }
    const Level &L = h->lv[0];
    if (nf > 1 && (ldw < L.nL || ldo < L.nL)) {
        set_error("sem_advect: leading dimensions must be >= n_local = %lld", (long long)L.nL);
        return SEM_EINVAL;
    }
    return launch_advect(L, A.M, A.variant, A.J, A.Jd, ct, nf, w, ldw, out, ldo, (hipStream_t)stream);
}

}  // extern "C"
