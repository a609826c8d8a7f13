// The pressure system of one IMEX stage (paper section 2: the discrete
// momentum and energy equations A U + B P = F, C U + D P = G, and the system
// D P + C A^-1 (F - B P) = G solved for the pressure).  The paper names the
// matrices without giving them; with central fluxes they are
//   (B p)_{e,i} = tau [ -int_K p d_e phi_i + int_dK p^ phi_i n_{K,e} ],
//       p^ = {p} on interior faces, the own trace on boundary faces;
//   (C u)_i     = tau [ -int_K hr u . grad Psi_i + int_dK {hr u . n_K} Psi_i ],
//       interior faces only (no flux through the boundary);
//   A = rho-weighted velocity mass (one scalar block per component),
//   D = (1/(gamma - 1)) mass (internal energy of an ideal gas),
// with hr = h rho and (k+1)-point Gauss rules on cells and faces, the rule of
// the fast block-diagonal inverse (section 3.3), so A^-1 is exact by the
// tensor-product sweeps of k_massinv.
//
// k_grad and k_div: NF threads per cell (pencil owners (a, b)), CPB cells
// per block (k_grad: one wave, so its LDS exchanges need no workgroup
// barrier; k_div: two waves, measured faster with its larger LDS), cells taken in the operator's tile traversal with one contiguous range of
// blocks per XCD, so neighbours' data are found in the same L2.  Cell terms by sum factorisation: values at the Gauss points by
// three sweeps, the pointwise metric terms W = w detJ J^-1 (times hr for C),
// and the transposed gradient (B^T / BD^T sweeps z, y, x).  Face terms: the
// traces at the face Gauss points are N x N contractions of the face layers
// (GLL nodes include the faces), the transposed contraction returns them to
// the face-layer nodes, and the pencil owners add them.  Each output is
// written by one thread: no atomics, bitwise reproducible.
#include "common.hpp"
#include "wave_sync.hpp"

namespace hx {
namespace {

// compile-time 1-D tables (generated at build time from the library's rules,
// the same values as the reference tables): in unrolled loops their entries
// become instruction operands instead of memory reads
template <int N> struct KB;
template <int N> struct KBD;
template <int N> struct KDL;
#include "optables.inc"
template <int N> struct KBI;
#include "optables_binv.inc"

template <int N>
__device__ __forceinline__ constexpr double tB(int q, int i) { return KB<N>::d[q * N + i]; }
template <int N>
__device__ __forceinline__ constexpr double tD(int q, int i) { return KBD<N>::d[q * N + i]; }
// (B^-1)_{iq}: B maps nodes to Gauss points and is square
template <int N>
__device__ __forceinline__ constexpr double tBi(int i, int q) { return KBI<N>::d[i * N + q]; }

// CPB cells of NF threads per block of at most TMAX threads (k_grad: one
// wave; k_div, with three velocity components in LDS: two waves)
template <int N, int TMAX>
struct PCfg {
    static constexpr int NF = N * N, ND = N * N * N;
    static constexpr int CPB = (TMAX / NF) > 0 ? TMAX / NF : 1;
    static constexpr int NT = ((CPB * NF + 63) / 64) * 64;
};
constexpr int GRAD_T = 64, DIV_T = 128;
template <int N> constexpr int grad_nt() { return PCfg<N, GRAD_T>::NT; }
template <int N> constexpr int div_nt() { return PCfg<N, DIV_T>::NT; }

// cell-local index of face-layer node (e1, e2) at normal coordinate m of
// direction d; e1, e2 run along the tangential directions t1 < t2
template <int N>
__device__ __forceinline__ int lay(int d, int m, int e1, int e2)
{
    const int s1 = d == 0 ? N : 1, s2 = d == 2 ? N : N * N, sd = d == 0 ? 1 : (d == 1 ? N : N * N);
    return m * sd + e1 * s1 + e2 * s2;
}

// per-lane rows and columns of B for the face contractions of lane (a, b):
// Ra[e] = B(a, e), Rb[e] = B(b, e), Ca[e] = B(e, a), Cb[e] = B(e, b)
template <int N>
struct LaneB {
    double Ra[N], Rb[N], Ca[N], Cb[N];
    __device__ __forceinline__ LaneB(const double *sB, int a, int b)
    {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            Ra[e] = sB[a * N + e];
            Rb[e] = sB[b * N + e];
            Ca[e] = sB[e * N + a];
            Cb[e] = sB[e * N + b];
        }
    }
};

// value of a face layer at the lane's face Gauss point (a, b):
// sum B(a,e1) B(b,e2) v(e1, e2), the layer at normal coordinate m of d
template <int N>
__device__ __forceinline__ double trace_at(const LaneB<N> &L, const double *v, int d, int m)
{
    double s = 0.0;
#pragma unroll
    for (int e2 = 0; e2 < N; ++e2) {
        double r = 0.0;
#pragma unroll
        for (int e1 = 0; e1 < N; ++e1) r += L.Ra[e1] * v[lay<N>(d, m, e1, e2)];
        s += L.Rb[e2] * r;
    }
    return s;
}

// the same from a face layer already gathered as v[e1 + N e2]
template <int N>
__device__ __forceinline__ double trace_at2(const LaneB<N> &L, const double *v)
{
    double s = 0.0;
#pragma unroll
    for (int e2 = 0; e2 < N; ++e2) {
        double r = 0.0;
#pragma unroll
        for (int e1 = 0; e1 < N; ++e1) r += L.Ra[e1] * v[e1 + N * e2];
        s += L.Rb[e2] * r;
    }
    return s;
}

// transposed contraction of a face field g[a' + N b'] to the lane's node
// (e1, e2) = (a, b)
template <int N>
__device__ __forceinline__ double trace_t(const LaneB<N> &L, const double *g)
{
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
        double r = 0.0;
#pragma unroll
        for (int a = 0; a < N; ++a) r += L.Ca[a] * g[a + N * b];
        s += L.Cb[b] * r;
    }
    return s;
}

// values of a cell field at the Gauss points along the lane's z pencil
// (lane (a, b) = (qx, qy)); v is the field in LDS, F a scratch field
template <int N>
__device__ __forceinline__ void to_gauss(const double *v, double *F, bool act, int a, int b,
                                         double (&out)[N])
{
    constexpr int NF = N * N;
    double r[N], w[N];
    if (act) {
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = v[i + N * a + NF * b];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) s += tB<N>(q, i) * r[i];
            w[q] = s;
        }
#pragma unroll
        for (int q = 0; q < N; ++q) F[q + N * a + NF * b] = w[q];
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = F[a + N * j + NF * b];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < N; ++j) s += tB<N>(q, j) * r[j];
            w[q] = s;
        }
    }
    __syncthreads();
    if (act)
#pragma unroll
        for (int q = 0; q < N; ++q) F[a + N * q + NF * b] = w[q];
    __syncthreads();
    if (act) {
#pragma unroll
        for (int l = 0; l < N; ++l) r[l] = F[a + N * b + NF * l];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l < N; ++l) s += tB<N>(q, l) * r[l];
            out[q] = s;
        }
    }
    __syncthreads();
}

// y = -tau sum_d G_d^T t_d, G_d the reference gradient component d at the
// Gauss points; t_d given along the lane's z pencil; F0..F2 scratch fields;
// the result is the lane's x pencil (lane (a, b) = (j, l))
template <int N>
__device__ __forceinline__ void grad_t(double *F0, double *F1, double *F2, bool act, int a, int b,
                                       const double (&t0)[N], const double (&t1)[N],
                                       const double (&t2)[N], double tau, double (&y)[N])
{
    constexpr int NF = N * N;
    if (act) {
#pragma unroll
        for (int l = 0; l < N; ++l) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                s0 += tB<N>(q, l) * t0[q];
                s1 += tB<N>(q, l) * t1[q];
                s2 += tD<N>(q, l) * t2[q];
            }
            F0[a + N * b + NF * l] = s0;
            F1[a + N * b + NF * l] = s1;
            F2[a + N * b + NF * l] = s2;
        }
    }
    __syncthreads();
    double r0[N], r12[N];
    if (act) {
        double f0[N], f1[N], f2[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            f0[q] = F0[a + N * q + NF * b];
            f1[q] = F1[a + N * q + NF * b];
            f2[q] = F2[a + N * q + NF * b];
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double s0 = 0.0, s12 = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                s0 += tB<N>(q, j) * f0[q];
                s12 += tD<N>(q, j) * f1[q] + tB<N>(q, j) * f2[q];
            }
            r0[j] = s0;
            r12[j] = s12;
        }
    }
    __syncthreads();
    if (act)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            F0[a + N * j + NF * b] = r0[j];
            F1[a + N * j + NF * b] = r12[j];
        }
    __syncthreads();
    if (act) {
        double g0[N], g1[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            g0[q] = F0[q + N * a + NF * b];
            g1[q] = F1[q + N * a + NF * b];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) s += tD<N>(q, i) * g0[q] + tB<N>(q, i) * g1[q];
            y[i] = -tau * s;
        }
    }
    __syncthreads();
}

// add face-layer contributions A[f][e1 + N e2] of the six faces to the x
// pencil (i, j=a, l=b) of the lane
// add the contribution of face f, computed on its face layer (e1, e2), to
// the pencil y of lane (a, b): x faces hold nodes (0 or N-1, a, b) with
// (e1, e2) = (j, l); y faces j = a with (e1, e2) = (i, l); z faces l = b with
// (e1, e2) = (i, j)
template <int N>
__device__ __forceinline__ void add_face(const double *A, int f, int a, int b, double (&y)[N])
{
    switch (f) {
    case 0: y[0] += A[a + N * b]; break;
    case 1: y[N - 1] += A[a + N * b]; break;
    case 2: if (a == 0) for (int i = 0; i < N; ++i) y[i] += A[i + N * b]; break;
    case 3: if (a == N - 1) for (int i = 0; i < N; ++i) y[i] += A[i + N * b]; break;
    case 4: if (b == 0) for (int i = 0; i < N; ++i) y[i] += A[i + N * a]; break;
    default: if (b == N - 1) for (int i = 0; i < N; ++i) y[i] += A[i + N * a]; break;
    }
}

// u3 = B p
template <int N>
__global__ void __launch_bounds__(grad_nt<N>())
k_grad(const double *__restrict__ p, double *__restrict__ u3, int64_t nt,
       const double *__restrict__ W, const double *__restrict__ fn, const int32_t *__restrict__ visit,
       const RefTab64 *__restrict__ T, double tau, int n_cells, int nwg)
{
    constexpr int NF = PCfg<N, GRAD_T>::NF, ND = PCfg<N, GRAD_T>::ND, CPB = PCfg<N, GRAD_T>::CPB;
    __shared__ double sB[NF];
    __shared__ double sP[CPB][ND];
    __shared__ double sF[CPB][3][ND];
    __shared__ double sG[CPB][3][NF];
    __shared__ double sA[CPB][3][NF];
    __shared__ double sL[CPB][NF];
    const int t = threadIdx.x;
    const int lc0 = t / NF;
    const bool slot = lc0 < CPB;
    const int lc = slot ? lc0 : 0;
    const int tt = t - lc0 * NF;
    const int a = tt % N, b = tt / N;
    // the operator's traversal: slot records {cell, six neighbours} in tile
    // order, one contiguous range of blocks per XCD
    const int bid = blockIdx.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    const int wg = xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
    const int64_t sl = (int64_t)wg * CPB + lc;
    const bool act = slot && sl < n_cells;
    // the 32-byte record in two 16-byte loads (slot 0's for idle threads)
    const int4 *rec4 = reinterpret_cast<const int4 *>(visit + (act ? sl : 0) * 8);
    const int4 r0 = rec4[0], r1 = rec4[1];
    const int32_t nbr6[6] = {r0.y, r0.z, r0.w, r1.x, r1.y, r1.z};
    const int64_t cid = act ? r0.x : 0;

    // one batch of loads (one memory round trip): the 1-D table, the cell's
    // values, the neighbours' face layers (one value per lane and face; a
    // missing neighbour reads the own cell and is dropped) and the first
    // face's outward ds n; they are requested before the cell part so that
    // their latency overlaps it
    static_assert(NF <= PCfg<N, GRAD_T>::NT, "one table entry per thread");
    const double fbv = t < NF ? T->B[t] : 0.0;
    double pv[N], nbv[6], fnx[3];
#pragma unroll
    for (int u = 0; u < N; ++u) pv[u] = p[cid * ND + tt + u * NF];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int32_t nb = act ? nbr6[f] : -1;
        const int64_t src = nb >= 0 ? (int64_t)nb : cid;
        const double v = p[src * ND + lay<N>(f >> 1, (f & 1) ? 0 : N - 1, a, b)];
        nbv[f] = nb >= 0 ? v : 0.0;
    }
#pragma unroll
    for (int ec = 0; ec < 3; ++ec) fnx[ec] = fn[(cid * 6 + 0) * 3 * NF + tt + ec * NF];
    __builtin_amdgcn_sched_barrier(0);
    if (t < NF) sB[t] = fbv;
    if (act) {
#pragma unroll
        for (int u = 0; u < N; ++u) sP[lc][tt + u * NF] = pv[u];
    }
    __syncthreads();
    const LaneB<N> LB(sB, a, b);
    double pq[N];
    to_gauss<N>(sP[lc], sF[lc][0], act, a, b, pq);
    double Y[3][N];
#pragma unroll
    for (int ec = 0; ec < 3; ++ec) {
        double t0[N], t1[N], t2[N];
        if (act) {
            const double *Wc = W + cid * 9 * ND + a + N * b;
            for (int q = 0; q < N; ++q) {
                t0[q] = pq[q] * Wc[(0 + ec) * ND + NF * q];
                t1[q] = pq[q] * Wc[(3 + ec) * ND + NF * q];
                t2[q] = pq[q] * Wc[(6 + ec) * ND + NF * q];
            }
        }
        grad_t<N>(sF[lc][0], sF[lc][1], sF[lc][2], act, a, b, t0, t1, t2, tau, Y[ec]);
    }
    // faces: tau ds n_e p^ at the Gauss points, back to the face-layer nodes;
    // the neighbour's face layer is gathered into LDS first (one value per lane)
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, s = f & 1;
        const int32_t nb = act ? nbr6[f] : -1;
        // this face's ds n, and the next face's requested now
        double fcur[3];
#pragma unroll
        for (int ec = 0; ec < 3; ++ec) fcur[ec] = fnx[ec];
        if (f < 5) {
#pragma unroll
            for (int ec = 0; ec < 3; ++ec) fnx[ec] = fn[(cid * 6 + f + 1) * 3 * NF + tt + ec * NF];
        }
        if (nb >= 0) sL[lc][tt] = nbv[f];
        __syncthreads();
        if (act) {
            const double po = trace_at<N>(LB, sP[lc], d, s ? N - 1 : 0);
            double ph = po;
            if (nb >= 0) ph = 0.5 * (po + trace_at2<N>(LB, sL[lc]));
            for (int ec = 0; ec < 3; ++ec) sG[lc][ec][tt] = tau * ph * fcur[ec];
        }
        __syncthreads();
        if (act)
            for (int ec = 0; ec < 3; ++ec) sA[lc][ec][tt] = trace_t<N>(LB, sG[lc][ec]);
        __syncthreads();
        if (act)
#pragma unroll
            for (int ec = 0; ec < 3; ++ec) add_face<N>(sA[lc][ec], f, a, b, Y[ec]);
    }
    if (act)
#pragma unroll
        for (int ec = 0; ec < 3; ++ec) {
            const int64_t o = ec * nt + cid * ND + N * a + NF * b;
            for (int i = 0; i < N; ++i) u3[o + i] = Y[ec][i];
        }
}

// qv = C u
template <int N>
__global__ void __launch_bounds__(div_nt<N>())
k_div(const double *__restrict__ u3, double *__restrict__ qv, int64_t nt,
      const double *__restrict__ WC, const double *__restrict__ fn, const double *__restrict__ fh,
      const int32_t *__restrict__ visit, const RefTab64 *__restrict__ T, double tau, int n_cells, int nwg)
{
    constexpr int NF = PCfg<N, DIV_T>::NF, ND = PCfg<N, DIV_T>::ND, CPB = PCfg<N, DIV_T>::CPB;
    __shared__ double sB[NF];
    __shared__ double sU[CPB][3][ND];
    __shared__ double sF[CPB][ND];
    __shared__ double sG[CPB][NF];
    __shared__ double sA[CPB][NF];
    __shared__ double sL[CPB][3][NF];
    const int t = threadIdx.x;
    const int lc0 = t / NF;
    const bool slot = lc0 < CPB;
    const int lc = slot ? lc0 : 0;
    const int tt = t - lc0 * NF;
    const int a = tt % N, b = tt / N;
    // the operator's traversal: slot records {cell, six neighbours} in tile
    // order, one contiguous range of blocks per XCD
    const int bid = blockIdx.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    const int wg = xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
    const int64_t sl = (int64_t)wg * CPB + lc;
    const bool act = slot && sl < n_cells;
    // the 32-byte record in two 16-byte loads (slot 0's for idle threads)
    const int4 *rec4 = reinterpret_cast<const int4 *>(visit + (act ? sl : 0) * 8);
    const int4 r0 = rec4[0], r1 = rec4[1];
    const int32_t nbr6[6] = {r0.y, r0.z, r0.w, r1.x, r1.y, r1.z};
    const int64_t cid = act ? r0.x : 0;

    // one batch of loads (one memory round trip): the 1-D table, the cell's
    // three velocity components, the neighbours' face layers of the three
    // (a missing neighbour reads the own cell and is dropped) and the first
    // face's ds n and h rho factors
    static_assert(NF <= PCfg<N, DIV_T>::NT, "one table entry per thread");
    const double fbv = t < NF ? T->B[t] : 0.0;
    double uv[3][N], nbu[6][3], fnx[3], fhx[2];
#pragma unroll
    for (int ec = 0; ec < 3; ++ec)
#pragma unroll
        for (int u = 0; u < N; ++u) uv[ec][u] = u3[ec * nt + cid * ND + tt + u * NF];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int32_t nb = act ? nbr6[f] : -1;
        const int64_t src = nb >= 0 ? (int64_t)nb : cid;
        const int64_t o = src * ND + lay<N>(f >> 1, (f & 1) ? 0 : N - 1, a, b);
#pragma unroll
        for (int ec = 0; ec < 3; ++ec) nbu[f][ec] = u3[ec * nt + o];
    }
    // ds n and the two h rho factors of face f (the neighbour's entry of a
    // missing neighbour reads the own cell's and is not used)
    auto face_data = [&](int f, double (&fo)[3], double (&ho)[2]) {
        const int32_t nb = act ? nbr6[f] : -1;
        const int64_t src = nb >= 0 ? (int64_t)nb : cid;
#pragma unroll
        for (int ec = 0; ec < 3; ++ec) fo[ec] = fn[(cid * 6 + f) * 3 * NF + tt + ec * NF];
        ho[0] = fh[(cid * 6 + f) * NF + tt];
        ho[1] = fh[(src * 6 + (nb >= 0 ? (f ^ 1) : f)) * NF + tt];
    };
    face_data(0, fnx, fhx);
    __builtin_amdgcn_sched_barrier(0);
    if (t < NF) sB[t] = fbv;
    if (act) {
#pragma unroll
        for (int ec = 0; ec < 3; ++ec)
#pragma unroll
            for (int u = 0; u < N; ++u) sU[lc][ec][tt + u * NF] = uv[ec][u];
    }
    __syncthreads();
    const LaneB<N> LB(sB, a, b);
    // interior faces first, while all three velocity layers are in LDS:
    // tau ds {hr u . n_K} at the Gauss points, back to the nodes; the
    // neighbour's face layers are gathered into LDS first
    double Yf[N];
#pragma unroll
    for (int i = 0; i < N; ++i) Yf[i] = 0.0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, s = f & 1;
        const int32_t nb = act ? nbr6[f] : -1;
        // this face's data, and the next face's requested now
        double fcur[3], hcur[2];
#pragma unroll
        for (int ec = 0; ec < 3; ++ec) fcur[ec] = fnx[ec];
        hcur[0] = fhx[0];
        hcur[1] = fhx[1];
        if (f < 5) face_data(f + 1, fnx, fhx);
        if (nb >= 0) {
#pragma unroll
            for (int ec = 0; ec < 3; ++ec) sL[lc][ec][tt] = nbu[f][ec];
        }
        __syncthreads();
        if (act) {
            double g = 0.0;
            if (nb >= 0) {
                double fo = 0.0, fnb = 0.0;
                for (int ec = 0; ec < 3; ++ec) {
                    const double uo = trace_at<N>(LB, sU[lc][ec], d, s ? N - 1 : 0);
                    const double un = trace_at2<N>(LB, sL[lc][ec]);
                    fo += uo * fcur[ec];
                    fnb += un * fcur[ec];
                }
                fo *= hcur[0];
                fnb *= hcur[1];
                g = tau * 0.5 * (fo + fnb);
            }
            sG[lc][tt] = g;
        }
        __syncthreads();
        if (act) sA[lc][tt] = trace_t<N>(LB, sG[lc]);
        __syncthreads();
        if (act) add_face<N>(sA[lc], f, a, b, Yf);
    }
    // cell terms: the velocity at the Gauss points, the weighted metric
    // terms, the transposed gradient; once at the Gauss points the second
    // and third velocity layers serve as its scratch
    double uq[3][N];
#pragma unroll
    for (int ec = 0; ec < 3; ++ec) to_gauss<N>(sU[lc][ec], sF[lc], act, a, b, uq[ec]);
    double t0[N], t1[N], t2[N], Y[N];
    if (act) {
        const double *Wc = WC + cid * 9 * ND + a + N * b;
        for (int q = 0; q < N; ++q) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
            for (int ec = 0; ec < 3; ++ec) {
                s0 += Wc[(0 + ec) * ND + NF * q] * uq[ec][q];
                s1 += Wc[(3 + ec) * ND + NF * q] * uq[ec][q];
                s2 += Wc[(6 + ec) * ND + NF * q] * uq[ec][q];
            }
            t0[q] = s0;
            t1[q] = s1;
            t2[q] = s2;
        }
    }
    grad_t<N>(sF[lc], sU[lc][1], sU[lc][2], act, a, b, t0, t1, t2, tau, Y);
    if (act)
#pragma unroll
        for (int i = 0; i < N; ++i) Y[i] += Yf[i];
    if (act) {
        const int64_t o = cid * ND + N * a + NF * b;
        for (int i = 0; i < N; ++i) qv[o + i] = Y[i];
    }
}

// ---------------------------------------------------------------------------
// S x = D x - C A^-1 B x in two passes, in the basis of the Gauss points.
//
// With as many Gauss points as nodes the interpolation B3 to the points is
// square, so the Lagrange basis of the points spans the same space and the
// weak forms may be tested with it; the nodal result is B3^T of that.  In
// this basis the mass matrices are diagonal (their point weights), so A^-1 is
// a division and D a product, the interpolations between B, A^-1 and C
// cancel, a derivative is one N x N matrix DG = BD B^-1 along its direction,
// and on a face the basis is already at the face's points: the trace is the
// extrapolation E along the normal line (E_s(q), rows 0 and N - 1 of B^-1)
// and the test function lifts a face value by E along that line.
//
// k_sys_cell (one wave, CPW cells): x at the points; the neighbours' traces
// from their face layers (column and row lanes as in the operator kernel);
//   g_e = tau [ -sum_d DG_d^T (x W_de) + sum_f E_f x^ (ds n_e) ],
//   v_e = g_e / mr,   own flux of face f: hr sum_e v_e ds n_e,
//   r = md x + tau sum_d DG_d^T (hr sum_e W_de v_e)
// (D x and the cell part of -C v); it writes r (point values) and the own
// fluxes.  k_sys_face: r - tau sum_f E_f (own - neighbour's flux) / 2, then
// B3^T.  Every lane (a, b) works on its x, y and z line of points in turn, and
// the geometric factors of direction d are loaded in the layout of the lines
// along d, where they are used; only sums pass through LDS.
//
// Affine cells (constant J^-1, W_de = w K_de, ds n_e = +-w_a w_b K_de): with
//   H_d = w_a w_b tau [ -DG_d^T (w x) + E_1 x^_1 - E_0 x^_0 ],
// g_e = sum_d K_de H_d, and with a_d = sum_e K_de v_e the fluxes are
// +-hr w_a w_b E a_d and the cell part of C needs hr w a_d: three scalar lines
// and ten constants per cell instead of 27 numbers per point.
//
// Bound by memory: at degree 4 a general cell moves 152 + 35 bytes per dof
// in the two passes, an affine one 51 + 35 (the former form, one pass each
// for A^-1 B and for D - C through nodal values, 133 + 24 and 142 + 16, and
// LDS-bound at 83 and 75 % of its cycles).  64x32x32 cells, degree 4: 0.713 ->
// 0.280 ms.
// ---------------------------------------------------------------------------
template <int N>
struct SysCfg {
    static constexpr int NF = N * N, ND = NF * N;
    // cells per wave as the traversal's records have them, so that a wave's
    // cells are of one kind; at N = 2 that would leave 12 of 16 lanes without
    // a line (49 us at 65,536 cells, the former form 44), so 16 cells share
    // a wave, all of them on the general data, and a lane takes three columns
    // of the faces
    static constexpr bool OWN = N == 2;
    static constexpr int LPC = OWN ? NF : op_lanes(N), CPW = 64 / LPC;
    static constexpr int COLS = (6 * N + LPC - 1) / LPC;      // face columns per lane
    // waves per SIMD asked for: at N = 3 three (145 -> 135 us at 65,536 cells);
    // above, the factors of a cell's points stay in registers instead
    static constexpr int WAVES = N == 3 ? 3 : 1;
    static constexpr int FPWV = 64 / NF;                      // cells per wave of the face pass
};

// lines of N contiguous values, two at a time where possible
typedef double dbl2 __attribute__((ext_vector_type(2), aligned(8)));
template <int N>
__device__ __forceinline__ void load_line(const double *__restrict__ p, double (&v)[N])
{
#pragma unroll
    for (int i = 0; i + 1 < N; i += 2) {
        const dbl2 t = *(const dbl2 *)(p + i);
        v[i] = t.x;
        v[i + 1] = t.y;
    }
    if (N & 1) v[N - 1] = p[N - 1];
}
template <int N>
__device__ __forceinline__ void load_line(const double *__restrict__ p, int stride, double (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i * stride];
}

// E(s, r): value at end s of the basis function of point r
template <int N>
__device__ __forceinline__ constexpr double tE(int s, int r) { return tBi<N>(s ? N - 1 : 0, r); }
// DG(q, r) = sum_i BD(q, i) B^-1(i, r): derivative at point q of the basis
// function of point r
template <int N>
struct DGTab {
    double d[N * N];
    constexpr DGTab() : d()
    {
        for (int q = 0; q < N; ++q)
            for (int r = 0; r < N; ++r) {
                double s = 0.0;
                for (int i = 0; i < N; ++i) s += KBD<N>::d[q * N + i] * KBI<N>::d[i * N + r];
                d[q * N + r] = s;
            }
    }
};

// y += sc DG^T u
template <int N>
__device__ __forceinline__ void add_dgt(const double (&u)[N], double sc, double (&y)[N])
{
    constexpr DGTab<N> G{};
#pragma unroll
    for (int r = 0; r < N; ++r) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < N; ++q) s += G.d[q * N + r] * u[q];
        y[r] += sc * s;
    }
}
// value at end s of the line u
template <int N>
__device__ __forceinline__ double at_end(int s, const double (&u)[N])
{
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) v += tE<N>(s, q) * u[q];
    return v;
}
// B u along a line
template <int N>
__device__ __forceinline__ void to_points(const double (&u)[N], double (&y)[N])
{
#pragma unroll
    for (int q = 0; q < N; ++q) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) s += tB<N>(q, i) * u[i];
        y[q] = s;
    }
}

// a field of the cell in LDS as the lane's lines along x, y and z
template <int N>
struct Lines {
    int x, y, z;   // first element
    __device__ __forceinline__ Lines(int a, int b) : x(N * a + N * N * b), y(a + N * N * b), z(a + N * b) {}
    template <int D>
    __device__ __forceinline__ int at(int i) const
    {
        return D == 0 ? x + i : (D == 1 ? y + N * i : z + N * N * i);
    }
    template <int D>
    __device__ __forceinline__ void get(const double *F, double (&v)[N]) const
    {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = F[at<D>(i)];
    }
    template <int D>
    __device__ __forceinline__ void put(double *F, const double (&v)[N]) const
    {
#pragma unroll
        for (int i = 0; i < N; ++i) F[at<D>(i)] = v[i];
    }
};

template <int N, bool AFF>
__device__ __forceinline__ void sys_cell(const double *__restrict__ x, double *__restrict__ r,
                                         double *__restrict__ flux, const double *__restrict__ W,
                                         const double *__restrict__ kc, const double *__restrict__ fn,
                                         const double *__restrict__ fh, const double *__restrict__ mr,
                                         const double *__restrict__ md, const double *__restrict__ hr,
                                         const int32_t *__restrict__ rec, const RefTab64 *__restrict__ T,
                                         double tau, bool valid, int64_t cid, int ln,
                                         double *__restrict__ F /* [3][ND] */, double *__restrict__ P /* [6][NF] */)
{
    constexpr int NF = SysCfg<N>::NF, ND = SysCfg<N>::ND;
    const bool cl = valid && ln < NF;
    const int a = ln % N, b = (ln / N) % N;
    const Lines<N> L(a, b);
    const int64_t o = cid * ND;
    // ---- loads: the nodal x line, the neighbours' face columns, and the
    // factors of the x lines
    double u[N];
    if (cl) load_line<N>(x + o + L.x, u);
    constexpr int COLS = SysCfg<N>::COLS, LPC = SysCfg<N>::LPC;
    double h[COLS][N], hq[N];
    bool fl[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        // column rr (first tangential direction) of the layer of face f's
        // neighbour
        const int col = ln + c * LPC, f = col < 6 * N ? col / N : 0, rr = col % N, fd = f >> 1, fs = f & 1;
        const int32_t nb = (valid && col < 6 * N) ? rec[1 + f] : -1;
        fl[c] = nb >= 0;
        if (!fl[c]) continue;
        const int sm = fd == 0 ? 1 : (fd == 1 ? N : NF), sp = fd == 0 ? N : 1, sr = fd == 2 ? N : NF;
        load_line<N>(x + (int64_t)nb * ND + (fs ? 0 : (N - 1) * sm) + rr * sp, sr, h[c]);
    }
    bool inner[6];
#pragma unroll
    for (int e = 0; e < 6; ++e) inner[e] = valid && rec[1 + e] >= 0;
    double K[AFF ? 10 : 1], wq[N], wab = 0.0;
    double Wx[AFF ? 1 : 3][N], Wy[AFF ? 1 : 3][N], Wz[AFF ? 1 : 3][N], n6[AFF ? 1 : 6][3], h6[6];
    if constexpr (AFF) {
#pragma unroll
        for (int q = 0; q < N; ++q) wq[q] = T->wq[q];
        wab = T->wq[a] * T->wq[b];
    }
    if (cl) {
        if constexpr (AFF) {
#pragma unroll
            for (int k = 0; k < 10; ++k) K[k] = kc[16 * cid + k];
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                load_line<N>(W + (cid * 9 + e) * ND + L.x, Wx[e]);
                load_line<N>(W + (cid * 9 + 3 + e) * ND + L.y, N, Wy[e]);
                load_line<N>(W + (cid * 9 + 6 + e) * ND + L.z, NF, Wz[e]);
            }
#pragma unroll
            for (int g = 0; g < 6; ++g)
#pragma unroll
                for (int e = 0; e < 3; ++e) n6[g][e] = fn[((cid * 6 + g) * 3 + e) * NF + ln];
        }
#pragma unroll
        for (int g = 0; g < 6; ++g) h6[g] = fh[(cid * 6 + g) * NF + ln];
    }
    // ---- the neighbours' traces at the face points: second tangential
    // direction by the column lanes, then the first by the row lanes, in place
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        if (!fl[c]) continue;
        const int col = ln + c * LPC;
        double *Pf = P + col / N * NF;
        to_points<N>(h[c], hq);
#pragma unroll
        for (int q = 0; q < N; ++q) Pf[q * N + col % N] = hq[q];
    }
    // ---- x at the points: pz (z line), px, py
    double px[N], py[N], pz[N], t[N];
    if (cl) {
        to_points<N>(u, t);
        L.template put<0>(F, t);
    }
    lds_wave_sync();
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        if (!fl[c]) continue;
        double *Pr = P + (ln + c * LPC) * N;
#pragma unroll
        for (int i = 0; i < N; ++i) h[c][i] = Pr[i];
        to_points<N>(h[c], hq);
#pragma unroll
        for (int q = 0; q < N; ++q) Pr[q] = hq[q];
    }
    if (cl) {
        L.template get<1>(F, u);
        to_points<N>(u, t);
        L.template put<1>(F, t);
    }
    lds_wave_sync();
    if (cl) {
        L.template get<2>(F, u);
        to_points<N>(u, pz);
        L.template put<2>(F, pz);
    }
    lds_wave_sync();
    // ---- face means x^ at the lane's point of each face (a: first, b: second
    // tangential direction), times tau
    double ph[6];
    if (cl) {
        L.template get<0>(F, px);
        L.template get<1>(F, py);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            ph[s] = at_end<N>(s, px);
            ph[2 + s] = at_end<N>(s, py);
            ph[4 + s] = at_end<N>(s, pz);
        }
#pragma unroll
        for (int g = 0; g < 6; ++g) ph[g] = tau * (inner[g] ? 0.5 * (ph[g] + P[g * NF + ln]) : ph[g]);
    }
    lds_wave_sync();
    double rz[N], fx[6];
    if constexpr (AFF) {
        // H_d along the lines of d; H_x and H_y pass to the z lines in F0, F1
        double H[N], mi[N], hz[N], wl[N];
        auto line = [&](const double (&p)[N], double e0, double e1, double (&out)[N]) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                wl[q] = wq[q] * p[q];
                out[q] = wab * (tE<N>(1, q) * e1 - tE<N>(0, q) * e0);
            }
            add_dgt<N>(wl, -tau * wab, out);
        };
        if (cl) {
            line(px, ph[0], ph[1], H);
            L.template put<0>(F, H);
            line(py, ph[2], ph[3], H);
            L.template put<1>(F + ND, H);
            line(pz, ph[4], ph[5], hz);
            load_line<N>(mr + o + L.z, NF, mi);
        }
        lds_wave_sync();
        // v_e = sum_d K_de H_d / mr and a_d = sum_e K_de v_e
        if (cl) {
            double hx[N], hy[N];
            L.template get<2>(F, hx);
            L.template get<2>(F + ND, hy);
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const double im = 1.0 / mi[q];
                double v[3];
#pragma unroll
                for (int e = 0; e < 3; ++e) v[e] = im * (K[e] * hx[q] + K[3 + e] * hy[q] + K[6 + e] * hz[q]);
                hx[q] = K[0] * v[0] + K[1] * v[1] + K[2] * v[2];
                hy[q] = K[3] * v[0] + K[4] * v[1] + K[5] * v[2];
                hz[q] = K[6] * v[0] + K[7] * v[1] + K[8] * v[2];
            }
            L.template put<2>(F, hx);
            L.template put<2>(F + ND, hy);
        }
        lds_wave_sync();
        auto cline = [&](const double (&ad)[N], const double (&hl)[N], double &f0, double &f1, double (&out)[N]) {
            f0 = -wab * at_end<N>(0, ad);
            f1 = wab * at_end<N>(1, ad);
#pragma unroll
            for (int q = 0; q < N; ++q) wl[q] = wq[q] * hl[q] * ad[q];
            add_dgt<N>(wl, tau * wab, out);
        };
        double hl[N], ad[N], c0[N], c1[N];
#pragma unroll
        for (int q = 0; q < N; ++q) c0[q] = c1[q] = rz[q] = 0.0;
        if (cl) {
            L.template get<0>(F, ad);
            load_line<N>(hr + o + L.x, hl);
            cline(ad, hl, fx[0], fx[1], c0);
            L.template get<1>(F + ND, ad);
            load_line<N>(hr + o + L.y, N, hl);
            cline(ad, hl, fx[2], fx[3], c1);
            load_line<N>(hr + o + L.z, NF, hl);
            cline(hz, hl, fx[4], fx[5], rz);
#pragma unroll
            for (int q = 0; q < N; ++q) rz[q] += K[9] * wab * wq[q] * pz[q];
        }
        lds_wave_sync();
        if (cl) {
            L.template put<0>(F, c0);
            L.template put<1>(F + ND, c1);
        }
        lds_wave_sync();
        if (cl) {
            L.template get<2>(F, c0);
            L.template get<2>(F + ND, c1);
#pragma unroll
            for (int q = 0; q < N; ++q) rz[q] += c0[q] + c1[q];
        }
    } else {
        // g_e: the x lines' part to F_e, the y lines add theirs, the z lines
        // collect
        auto gline = [&](const double (&p)[N], const double (&w)[N], double e0, double e1, double (&out)[N]) {
            double tw[N];
#pragma unroll
            for (int q = 0; q < N; ++q) {
                tw[q] = p[q] * w[q];
                out[q] += tE<N>(0, q) * e0 + tE<N>(1, q) * e1;
            }
            add_dgt<N>(tw, -tau, out);
        };
        double v[3][N];
        if (cl)
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                double g[N] = {};
                gline(px, Wx[e], ph[0] * n6[0][e], ph[1] * n6[1][e], g);
                L.template put<0>(F + e * ND, g);
            }
        lds_wave_sync();
        if (cl)
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                double g[N];
                L.template get<1>(F + e * ND, g);
                gline(py, Wy[e], ph[2] * n6[2][e], ph[3] * n6[3][e], g);
                L.template put<1>(F + e * ND, g);
            }
        lds_wave_sync();
        if (cl) {
            double mi[N];
            load_line<N>(mr + o + L.z, NF, mi);
#pragma unroll
            for (int q = 0; q < N; ++q) mi[q] = 1.0 / mi[q];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                L.template get<2>(F + e * ND, v[e]);
                gline(pz, Wz[e], ph[4] * n6[4][e], ph[5] * n6[5][e], v[e]);
#pragma unroll
                for (int q = 0; q < N; ++q) v[e][q] *= mi[q];
                L.template put<2>(F + e * ND, v[e]);
            }
        }
        lds_wave_sync();
        // own fluxes and hr sum_e W_de v_e on the lines of d, its DG^T
        auto cline = [&](const double (&ve)[3][N], const double (&w)[3][N], const double (&hl)[N], int f0,
                         double (&out)[N]) {
            double tw[N];
#pragma unroll
            for (int q = 0; q < N; ++q)
                tw[q] = hl[q] * (w[0][q] * ve[0][q] + w[1][q] * ve[1][q] + w[2][q] * ve[2][q]);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                double sum = 0.0;
#pragma unroll
                for (int e = 0; e < 3; ++e) sum += at_end<N>(s, ve[e]) * n6[f0 + s][e];
                fx[f0 + s] = sum;
            }
            add_dgt<N>(tw, tau, out);
        };
        double hl[N], c0[N], c1[N];
#pragma unroll
        for (int q = 0; q < N; ++q) c0[q] = c1[q] = rz[q] = 0.0;
        if (cl) {
            load_line<N>(hr + o + L.z, NF, hl);
            cline(v, Wz, hl, 4, rz);
            double mq[N];
            load_line<N>(md + o + L.z, NF, mq);
#pragma unroll
            for (int q = 0; q < N; ++q) rz[q] += mq[q] * pz[q];
#pragma unroll
            for (int e = 0; e < 3; ++e) L.template get<0>(F + e * ND, v[e]);
            load_line<N>(hr + o + L.x, hl);
            cline(v, Wx, hl, 0, c0);
#pragma unroll
            for (int e = 0; e < 3; ++e) L.template get<1>(F + e * ND, v[e]);
            load_line<N>(hr + o + L.y, N, hl);
            cline(v, Wy, hl, 2, c1);
        }
        lds_wave_sync();
        if (cl) {
            L.template put<0>(F, c0);
            L.template put<1>(F + ND, c1);
        }
        lds_wave_sync();
        if (cl) {
            L.template get<2>(F, c0);
            L.template get<2>(F + ND, c1);
#pragma unroll
            for (int q = 0; q < N; ++q) rz[q] += c0[q] + c1[q];
        }
    }
    if (cl) {
#pragma unroll
        for (int q = 0; q < N; ++q) r[o + L.z + NF * q] = rz[q];
#pragma unroll
        for (int g = 0; g < 6; ++g) flux[(cid * 6 + g) * NF + ln] = h6[g] * fx[g];
    }
}

// MODE: the waves' cells are general (0), affine (1) or of either kind, the
// first record of a wave telling which (2), as in the operator kernel.  One
// launch of both kinds gives the affine waves the registers of the general ones
// (236 instead of 110 at N = 5), but a launch for each kind is slower: terrain
// 64x32x32, both passes, degree 2 131 / 146 us, 4 281 / 302, 7 1130 / 1186 (5 780
// / 760), and 8x4x3 cells, degree 4, 11.6 / 17.1.
template <int N, int MODE>
__global__ void __launch_bounds__(64, SysCfg<N>::WAVES)
k_sys_cell(const double *__restrict__ x, double *__restrict__ r, double *__restrict__ flux,
           const double *__restrict__ W, const double *__restrict__ kc, const double *__restrict__ fn,
           const double *__restrict__ fh, const double *__restrict__ mr, const double *__restrict__ md,
           const double *__restrict__ hr, const int32_t *__restrict__ visit, const RefTab64 *__restrict__ T,
           double tau, int n_slots, int nwg)
{
    constexpr int LPC = SysCfg<N>::LPC, CPW = SysCfg<N>::CPW;
    __shared__ double sF[CPW][3 * SysCfg<N>::ND], sP[CPW][6 * SysCfg<N>::NF];
    const int bid = blockIdx.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    const int wg = xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
    const int cs = threadIdx.x / LPC, ln = threadIdx.x % LPC;
    const int slot = wg * CPW + cs;
    const int32_t *rec = visit + (int64_t)(slot < n_slots ? slot : 0) * 8;
    const int32_t rc = rec[0];
    const bool valid = slot < n_slots && rc >= 0;
    const int64_t cid = valid ? rc : 0;
    const bool waff = MODE == 2 ? visit[(int64_t)wg * CPW * 8 + 7] & 1 : MODE == 1;
    if (MODE == 1 || (MODE == 2 && waff))
        sys_cell<N, true>(x, r, flux, W, kc, fn, fh, mr, md, hr, rec, T, tau, valid, cid, ln, sF[cs], sP[cs]);
    else if (MODE != 1)
        sys_cell<N, false>(x, r, flux, W, kc, fn, fh, mr, md, hr, rec, T, tau, valid, cid, ln, sF[cs], sP[cs]);
}

// y (or b - y) = B3^T (r - tau sum_f E_f (own - neighbour's flux) / 2); 64 / NF
// cells per wave, lane (a, b) of a cell
template <int N>
__global__ void __launch_bounds__(64)
k_sys_face(const double *__restrict__ r, const double *__restrict__ flux, const int32_t *__restrict__ visit,
           double tau, const double *__restrict__ bv, double *__restrict__ y, int n_cells, int nwg)
{
    constexpr int NF = SysCfg<N>::NF, ND = SysCfg<N>::ND, CPW = SysCfg<N>::FPWV;
    __shared__ double sF[CPW][ND], sP[CPW][4 * NF];
    const int bid = blockIdx.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    const int wg = xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
    const int cs = threadIdx.x / NF, ln = threadIdx.x % NF;
    const int slot = wg * CPW + cs;
    const bool cl = cs < CPW && slot < n_cells;
    const int32_t *rec = visit + (int64_t)(cl ? slot : 0) * 8;
    const int64_t cid = rec[0];
    const int a = ln % N, b = ln / N;
    const Lines<N> L(a, b);
    double *F = sF[cs < CPW ? cs : 0], *P = sP[cs < CPW ? cs : 0];
    double u[N], t[N], g[6];
    if (cl) {
        load_line<N>(r + cid * ND + L.z, NF, u);
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int32_t nb = rec[1 + f];
            const double own = flux[(cid * 6 + f) * NF + ln];
            const double nbr = flux[((nb >= 0 ? (int64_t)nb : cid) * 6 + (f ^ 1)) * NF + ln];
            g[f] = nb >= 0 ? -0.5 * tau * (own - nbr) : 0.0;
        }
        // the x and y faces' values where the z lines read them
#pragma unroll
        for (int f = 0; f < 4; ++f) P[f * NF + ln] = g[f];
    }
    lds_wave_sync();
    if (cl) {
        double ex[2] = {0.0, 0.0}, ey[2] = {0.0, 0.0};   // E at the lane's x and y index
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int m = 0; m < N; ++m) {
                if (m == a) ex[s] = tE<N>(s, m);
                if (m == b) ey[s] = tE<N>(s, m);
            }
        // lane (qx = a, qy = b): x faces' points (qy, qz), y faces' (qx, qz)
#pragma unroll
        for (int q = 0; q < N; ++q)
            u[q] += tE<N>(0, q) * g[4] + tE<N>(1, q) * g[5] + ex[0] * P[b + N * q] + ex[1] * P[NF + b + N * q] +
                    ey[0] * P[2 * NF + a + N * q] + ey[1] * P[3 * NF + a + N * q];
    }
    auto back = [&](const double (&w)[N], double (&z)[N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) s += tB<N>(q, i) * w[q];
            z[i] = s;
        }
    };
    if (cl) {
        back(u, t);
        L.template put<2>(F, t);
    }
    lds_wave_sync();
    if (cl) {
        L.template get<1>(F, u);
        back(u, t);
        L.template put<1>(F, t);
    }
    lds_wave_sync();
    if (cl) {
        L.template get<0>(F, u);
        back(u, t);
        double *yo = y + cid * ND + L.x;
        if (bv) {
            load_line<N>(bv + cid * ND + L.x, u);
#pragma unroll
            for (int i = 0; i < N; ++i) t[i] = u[i] - t[i];
        }
#pragma unroll
        for (int i = 0; i + 1 < N; i += 2) *(dbl2 *)(yo + i) = dbl2{t[i], t[i + 1]};
        if (N & 1) yo[N - 1] = t[N - 1];
    }
}

template <int N>
hipError_t grad_n(hx_ctx *c, const double *p, double *u3)
{
    const int cpb = PCfg<N, GRAD_T>::CPB;
    const int nb = (int)((c->n_cells + cpb - 1) / cpb);
    hipLaunchKernelGGL(k_grad<N>, dim3(nb), dim3(PCfg<N, GRAD_T>::NT), 0, c->stream, p, u3, c->n_dofs,
                       c->psW, c->psFn, c->visitp, c->ref, c->ps_tau, (int)c->n_cells, nb);
    return hipGetLastError();
}

template <int N>
hipError_t div_n(hx_ctx *c, const double *u3, double *q)
{
    const int cpb = PCfg<N, DIV_T>::CPB;
    const int nb = (int)((c->n_cells + cpb - 1) / cpb);
    hipLaunchKernelGGL(k_div<N>, dim3(nb), dim3(PCfg<N, DIV_T>::NT), 0, c->stream, u3, q, c->n_dofs,
                       c->psWC, c->psFn, c->psFh, c->visitp, c->ref, c->ps_tau, (int)c->n_cells, nb);
    return hipGetLastError();
}

// y = S x, or b - S x when b is given
template <int N>
hipError_t sys_n(hx_ctx *c, const double *x, double *y, const double *b)
{
    const int cpw = SysCfg<N>::CPW;
    const bool own = SysCfg<N>::OWN;
    const int32_t *visit = own ? c->visitp : c->visit;
    const int64_t slots = own ? c->n_cells : c->n_vis_op;
    const int mode = own ? 0 : c->vis_mode;
    const int nw = (int)((slots + cpw - 1) / cpw);
    double *r = c->psWork + 3 * c->n_dofs, *flux = r + c->n_dofs;
#define HX_SYS(MODE)                                                                              \
    hipLaunchKernelGGL((k_sys_cell<N, MODE>), dim3(nw), dim3(64), 0, c->stream, x, r, flux, c->psW, \
                       c->psK, c->psFn, c->psFh, c->psMr, c->psMd, c->psHr, visit, c->ref,          \
                       c->ps_tau, (int)slots, nw)
    if constexpr (!SysCfg<N>::OWN) {
        if (mode == 2) HX_SYS(2);
        else if (mode == 1) HX_SYS(1);
        else HX_SYS(0);
    } else {
        HX_SYS(0);
    }
#undef HX_SYS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nf = (int)((c->n_cells + SysCfg<N>::FPWV - 1) / SysCfg<N>::FPWV);
    hipLaunchKernelGGL(k_sys_face<N>, dim3(nf), dim3(64), 0, c->stream, r, flux, c->visitp, c->ps_tau, b, y,
                       (int)c->n_cells, nf);
    return hipGetLastError();
}

#define HX_BY_DEGREE(F, ...)                      \
    switch (c->n) {                               \
    case 2: return F<2>(__VA_ARGS__);             \
    case 3: return F<3>(__VA_ARGS__);             \
    case 4: return F<4>(__VA_ARGS__);             \
    case 5: return F<5>(__VA_ARGS__);             \
    case 6: return F<6>(__VA_ARGS__);             \
    case 7: return F<7>(__VA_ARGS__);             \
    case 8: return F<8>(__VA_ARGS__);             \
    default: return hipErrorInvalidValue;         \
    }

// h = gamma p / ((gamma - 1) rho): specific enthalpy of an ideal gas
__global__ void k_enthalpy(int64_t n, const double *__restrict__ p, const double *__restrict__ rho,
                           double f, double *h)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) h[i] = f * p[i] / rho[i];
}

}  // namespace

hipError_t launch_enthalpy(hx_ctx *c, const double *p, const double *rho, double gamma, double *h)
{
    const int64_t n = c->n_dofs;
    hipLaunchKernelGGL(k_enthalpy, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, n, p,
                       rho, gamma / (gamma - 1.0), h);
    return hipGetLastError();
}

hipError_t launch_grad(hx_ctx *c, const double *p, double *u3) { HX_BY_DEGREE(grad_n, c, p, u3) }

hipError_t launch_div(hx_ctx *c, const double *u3, double *q) { HX_BY_DEGREE(div_n, c, u3, q) }

hipError_t press_apply64(hx_ctx *c, const double *x, double *y, const double *b)
{
    HX_BY_DEGREE(sys_n, c, x, y, b)
}

}  // namespace hx
