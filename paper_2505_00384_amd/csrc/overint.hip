// The operator with consistent integration (paper section 3.3: a Gauss rule
// of 2r+1 points per direction, which integrates the products of three
// polynomials of the variable-coefficient terms without aliasing, against
// the r+1 points of the fast evaluation).  Same form as k_apply; the 1-D
// interpolation B (nq x n) and its derivative BD are rectangular now, so the
// sweeps change pencil lengths (n nodes <-> nq points).
//
// A workgroup serves one cell: wave 0 (two waves for N = 8) the cell integrals,
// one further wave (two for N > 5) the face terms, at the same time; they meet
// at one barrier, after which wave 0 adds the faces and writes its output
// pencils.  Inside a wave only the order of its LDS accesses matters, so there
// are no other barriers, except with two cell waves.
//  * cell: x sweep by lanes (j, l), y sweep by items (qx, l), z sweep,
//    quadrature-point operation and transposed z sweep by items (qx, qy), two
//    rounds of lanes for N = 5, then back; fields in LDS between the sweeps;
//    the point data of the next plane always in flight.
//  * faces: column lanes (f, p) hold a face's layer values and normal
//    derivatives, interpolate them along the second tangential direction
//    (step 1); row lanes (f, q2) along the first one, where they form the flux
//    terms point by point and sweep back (steps 2, 3); the column lanes finish
//    (step 4).  The neighbour's side goes first and leaves its flux and value
//    in registers.
// The 1-D tables are compile-time scalars.  What bounds it: the quadrature
// data stream (452 bytes per dof at degree 4, 140 on affine cells, which read
// two values per point and their constants) and the LDS traffic between the
// sweeps, and with them how many waves the registers leave room for.  The
// former form (two waves per cell in lock step, 23 barriers, face contractions
// with both operands and the tables from LDS) was bound by LDS: 0.500 ms at
// 64x16x32 cells, degree 4, and no faster with the compressed data of the
// affine cells (0.508); this one 0.365 ms.
//
// The lanes of a face wave hold faces of both kinds.  A branch on the kind at
// every point made the compiler carry the four interpolated values of all 2N-1
// points of a row past it (8 N doubles: 206 registers at N = 6, two waves per
// SIMD where there is room for three, and spills at N = 4), so a compressed
// face takes the same loads, from the one place it has, and the factors of
// the other kind are ones.  From N = 6 on the neighbour's side keeps two points
// in flight instead of the whole row.  64x16x32 cells, branch / without:
// degree 2 125 / 107 us, 3 230 / 195, 4 378 / 365, 5 1083 / 723 (the former form
// 862); at degree 1 the branch is the better one (49.5 / 52.0).  N = 7 and 8
// read the own values where they are needed instead of keeping them in LDS, so
// that at N = 8 two workgroups share a CU's 160 KB, and its cell integrals
// take two waves: degree 6 1830 / 1696 us, 7 4794 / 2587; 96 cells, degree 7,
// 36.4 / 26.4 (the former form 29.5).  N = 6 is slower without the LDS copy
// (923 us), and two cell waves lose at N = 5 (521), 6 (1032) and 7 (1783).  The
// bound on the waves per SIMD matters at N = 6 only, which has room for three
// with its 159 registers (737 us when three are asked for); N = 4 and 5 take the
// same times with one less.
#include "common.hpp"
#include "wave_sync.hpp"

namespace hx {
namespace {

// compile-time B and BD at the 2N-1 Gauss points (generated at build time
// from the library's rules, the same values as the set-up tables)
template <int N> struct KBQ;
template <int N> struct KBDQ;
#include "optables_q.inc"
// and the (k+1)-point tables, of which the end derivatives KDL are used
template <int N> struct KB;
template <int N> struct KBD;
template <int N> struct KDL;
#include "optables.inc"

template <int N>
__device__ __forceinline__ constexpr double tq(int q, int i) { return KBQ<N>::d[q * N + i]; }
template <int N>
__device__ __forceinline__ constexpr double tdq(int q, int i) { return KBDQ<N>::d[q * N + i]; }

template <int N>
struct QCfg {
    static constexpr int Q = 2 * N - 1, ND = N * N * N, NF = N * N, Q2 = Q * Q, Q3 = Q * Q * Q;
    static constexpr int QN = Q * N, QNN = Q * N * N, QQN = Q * Q * N;
    static constexpr int FW = 6 * Q <= 64 ? 1 : 2;   // face waves
    static constexpr int FPW = 6 / FW;               // faces per face wave
    static constexpr int CW = N <= 7 ? 1 : 2;        // cell waves
    static constexpr bool OWN_LDS = N <= 6;          // own values by way of LDS (face waves)
    static constexpr bool BRANCH = N == 2;           // a branch on the kind of a face at every point
    static constexpr int AHEAD = N <= 5 ? Q : 2;     // points of the neighbour's side in flight
    static constexpr int NT = 64 * (CW + FW);
    static_assert(NF <= 64 && FPW * Q <= 64, "one row lane per face row");
};

// between the sweeps: the waves of a role wait for each other, if there are two
// by the workgroup's barrier, which the other role then meets as often
template <int N>
__device__ __forceinline__ void q_sync()
{
    if constexpr (QCfg<N>::CW > 1) __syncthreads();
    else lds_wave_sync();
}

// y = B u (W = 0) or BD u (W = 1), n -> nq
template <int N, int W>
__device__ __forceinline__ void up(const double (&u)[N], double (&y)[2 * N - 1])
{
#pragma unroll
    for (int q = 0; q < 2 * N - 1; ++q) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) s += (W ? tdq<N>(q, i) : tq<N>(q, i)) * u[i];
        y[q] = s;
    }
}

// Cell integrals by CW waves (lane: 0 .. 64 CW - 1); U0, U1 (Q N^2 each) and
// V0, V1, V2 (Q^2 N each) in LDS; the output pencil of lane (j, l) in Y.
template <int N, bool AFF>
__device__ __forceinline__ void q_cell(const double *__restrict__ x, const double *__restrict__ cell,
                                       const double *__restrict__ kk, int64_t cid, int lane,
                                       double *__restrict__ U, double *__restrict__ V, double (&Y)[N])
{
    using C = QCfg<N>;
    constexpr int Q = C::Q, ND = C::ND, NF = C::NF, Q2 = C::Q2, Q3 = C::Q3, QN = C::QN, QNN = C::QNN,
                  QQN = C::QQN, NC = AFF ? 2 : 7;
    const double *cp = cell + cid * 7 * Q3;
    double *U1 = U + QNN, *V1 = V + QQN, *V2 = V1 + QQN;
    double kc[6];
    if constexpr (AFF)
#pragma unroll
        for (int k = 0; k < 6; ++k) kc[k] = kk[8 * cid + k];
    // the first plane's point data, in flight during the x and y sweeps
    double nx[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) nx[k] = cp[(lane < Q2 ? lane : 0) + k * Q3];
    // x sweep: lane (j, l): u and du/dxi at (qx, j, l), layout qx + Q (j + N l)
    if (lane < NF) {
        double v[N], s0[Q], s1[Q];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = x[cid * ND + N * lane + i];
        up<N, 0>(v, s0);
        up<N, 1>(v, s1);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            U[q + Q * lane] = s0[q];
            U1[q + Q * lane] = s1[q];
        }
    }
    q_sync<N>();
    // y sweep: item (qx, l): u, d/deta (from u) and d/dxi (from U1) at
    // (qx, qy, l), layout qx + Q (qy + Q l)
    for (int it = lane; it < QN; it += 64 * C::CW) {
        const int qx = it % Q, l = it / Q;
        double v0[N], v1[N], s0[Q], s1[Q], s2[Q];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            v0[j] = U[qx + Q * (j + N * l)];
            v1[j] = U1[qx + Q * (j + N * l)];
        }
        up<N, 0>(v0, s0);
        up<N, 1>(v0, s1);
        up<N, 0>(v1, s2);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            V[qx + Q * (q + Q * l)] = s0[q];
            V1[qx + Q * (q + Q * l)] = s1[q];
            V2[qx + Q * (q + Q * l)] = s2[q];
        }
    }
    q_sync<N>();
    // z sweep, quadrature-point operation, transposed z sweep: item (qx, qy),
    // in place (an item reads and writes its own columns only)
    for (int it = lane; it < Q2; it += 64 * C::CW) {
        double a0[N], a1[N], a2[N], w0[N], w1[N], w2[N];
#pragma unroll
        for (int l = 0; l < N; ++l) {
            a0[l] = V[it + Q2 * l];
            a1[l] = V1[it + Q2 * l];
            a2[l] = V2[it + Q2 * l];
            w0[l] = w1[l] = w2[l] = 0.0;
        }
        // (the last plane requests the next round's first one)
        const int nit = it + 64 * C::CW < Q2 ? it + 64 * C::CW : it;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            double cd[7];
#pragma unroll
            for (int k = 0; k < NC; ++k) cd[k] = nx[k];
#pragma unroll
            for (int k = 0; k < NC; ++k) nx[k] = cp[(q + 1 < Q ? it + Q2 * (q + 1) : nit) + k * Q3];
            if constexpr (AFF) {
                const double bw = cd[1];
#pragma unroll
                for (int k = 0; k < 6; ++k) cd[1 + k] = bw * kc[k];
            }
            double u = 0.0, dz = 0.0, dy = 0.0, dx = 0.0;
#pragma unroll
            for (int l = 0; l < N; ++l) {
                u += tq<N>(q, l) * a0[l];
                dz += tdq<N>(q, l) * a0[l];
                dy += tq<N>(q, l) * a1[l];
                dx += tq<N>(q, l) * a2[l];
            }
            const double m = cd[0], gxx = cd[1], gxy = cd[2], gxz = cd[3], gyy = cd[4], gyz = cd[5],
                         gzz = cd[6];
            const double v = m * u;
            const double fx = gxx * dx + gxy * dy + gxz * dz;
            const double fy = gxy * dx + gyy * dy + gyz * dz;
            const double fz = gxz * dx + gyz * dy + gzz * dz;
#pragma unroll
            for (int l = 0; l < N; ++l) {
                w0[l] += tq<N>(q, l) * v + tdq<N>(q, l) * fz;
                w1[l] += tq<N>(q, l) * fy;
                w2[l] += tq<N>(q, l) * fx;
            }
        }
#pragma unroll
        for (int l = 0; l < N; ++l) {
            V[it + Q2 * l] = w0[l];
            V1[it + Q2 * l] = w1[l];
            V2[it + Q2 * l] = w2[l];
        }
    }
    q_sync<N>();
    // transposed y sweep: item (qx, l) -> (qx, j, l): s0 = B^T w0 + BD^T w1,
    // s1 = B^T w2
    for (int it = lane; it < QN; it += 64 * C::CW) {
        const int qx = it % Q, l = it / Q;
        double s0[N], s1[N];
#pragma unroll
        for (int j = 0; j < N; ++j) s0[j] = s1[j] = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double a0 = V[qx + Q * (q + Q * l)], a1 = V1[qx + Q * (q + Q * l)],
                         a2 = V2[qx + Q * (q + Q * l)];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                s0[j] += tq<N>(q, j) * a0 + tdq<N>(q, j) * a1;
                s1[j] += tq<N>(q, j) * a2;
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            U[qx + Q * (j + N * l)] = s0[j];
            U1[qx + Q * (j + N * l)] = s1[j];
        }
    }
    q_sync<N>();
    // transposed x sweep: lane (j, l) keeps its output pencil
#pragma unroll
    for (int i = 0; i < N; ++i) Y[i] = 0.0;
    if (lane < NF)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double a0 = U[q + Q * lane], a1 = U1[q + Q * lane];
#pragma unroll
            for (int i = 0; i < N; ++i) Y[i] += tq<N>(q, i) * a0 + tdq<N>(q, i) * a1;
        }
}

// Face terms of faces f0 .. f0 + FPW - 1 by one wave.  S: own values (N^3, OWN_LDS);
// F: three fields of Q x N per face, [field][q2][p], layer weights and
// normal-derivative weights in fields 0 and 1, [r][p], on return.
template <int N>
__device__ __forceinline__ void q_faces(const double *__restrict__ x, const double *__restrict__ face,
                                        const int32_t *__restrict__ nbr, const uint8_t *__restrict__ ctype,
                                        bool aff, int64_t cid, int lane, int f0, double *__restrict__ S,
                                        double *__restrict__ F)
{
    using C = QCfg<N>;
    constexpr int Q = C::Q, ND = C::ND, NF = C::NF, Q2 = C::Q2, QN = C::QN, FPW = C::FPW;
    // column lane (f, p) and row lane (f, q2); the face data belong to the row
    const bool cl0 = lane < FPW * N, rl0 = lane < FPW * Q;
    const int fc = f0 + (cl0 ? lane / N : 0), p = lane % N;
    const int fr = f0 + (rl0 ? lane / Q : 0), q2 = lane % Q;
    const int32_t nbc = cl0 ? nbr[6 * cid + fc] : -1, nbr_ = rl0 ? nbr[6 * cid + fr] : -1;
    const bool cl = nbc >= 0, rl = nbr_ >= 0;
    const int dc = fc >> 1, sc = fc & 1, dr = fr >> 1, sr_ = fr & 1;
    // strides of the normal, column and row index in a cell's numbering
    const int sm = dc == 0 ? 1 : (dc == 1 ? N : NF), sp = dc == 0 ? N : 1, sr = dc == 2 ? N : NF;
    double *gc = F + (cl0 ? lane / N : 0) * 3 * QN, *gr = F + (rl0 ? lane / Q : 0) * 3 * QN + q2 * N;
    // own values to LDS, the neighbour's normal lines to registers: layer
    // values and normal derivatives, walked from the shared face inwards (so
    // both sides use the derivative weights of the lower end, mirrored and
    // negated at the upper one)
    double L[N], D[N];
    if (cl) {
        const int m0 = sc ? 0 : (N - 1) * sm, dm = sc ? sm : -sm;
        const double sgn = sc ? 1.0 : -1.0;
        const double *xn = x + (int64_t)nbc * ND + p * sp + m0;
#pragma unroll
        for (int r = 0; r < N; ++r) {
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < N; ++m) s += KDL<N>::d[m] * xn[r * sr + m * dm];
            D[r] = sgn * s;
            L[r] = xn[r * sr];
        }
    }
    if constexpr (C::OWN_LDS) {
#pragma unroll
        for (int k = 0; k < (ND + 63) / 64; ++k)
            if (lane + 64 * k < ND) S[lane + 64 * k] = x[cid * ND + lane + 64 * k];
    }
    // face data of the row: g of the neighbour's side (the plus side's if the
    // own cell is the minus cell), g of the own side, penalty factor; on a
    // face between two affine cells beta w of both sides and constants
    const bool cmp = aff && rl && ctype[nbr_];
    const int64_t fid = sr_ ? cid : (int64_t)nbr_;
    const double *fd = face + ((rl ? fid : 0) * 3 + dr) * 7 * Q2 + q2;
    const double *kf = fd - q2 + 2 * Q2;
    const int gn = sr_ ? 3 : 0, go = sr_ ? 0 : 3;
    const double *fn = fd + (cmp ? (sr_ ? 1 : 0) : gn) * Q2, *fo = fd + (cmp ? (sr_ ? 0 : 1) : go) * Q2;
    // the second and third component of a point; a compressed face reads the
    // first one again (st = 0)
    const int st = cmp ? 0 : Q2;
    constexpr int AH = C::AHEAD;
    double gv[AH][3];
    auto request_nb = [&](int q, double (&g)[3]) {
        g[0] = fn[Q * q];
        if (AH < Q || !cmp) {
            g[1] = fn[Q * q + st];
            g[2] = fn[Q * q + 2 * st];
        }
    };
    if (rl)
#pragma unroll
        for (int q = 0; q < AH; ++q) request_nb(q, gv[q]);
    auto step1 = [&](const double (&l)[N], const double (&d)[N]) {
        double g[Q];
        up<N, 0>(l, g);
#pragma unroll
        for (int q = 0; q < Q; ++q) gc[q * N + p] = g[q];
        up<N, 1>(l, g);
#pragma unroll
        for (int q = 0; q < Q; ++q) gc[QN + q * N + p] = g[q];
        up<N, 0>(d, g);
#pragma unroll
        for (int q = 0; q < Q; ++q) gc[2 * QN + q * N + p] = g[q];
    };
    if (cl) step1(L, D);
    q_sync<N>();
    // step 2, neighbour's side: flux and value at (q1, q2)
    double fnb[Q], vnb[Q];
    if (rl) {
        double h0[N], h1[N], h2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            h0[i] = gr[i];
            h1[i] = gr[QN + i];
            h2[i] = gr[2 * QN + i];
        }
        double v0 = 1.0, v1 = 1.0, v2 = 1.0;
        if (cmp) {
            v0 = kf[gn];
            v1 = kf[gn + 1];
            v2 = kf[gn + 2];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            double v = 0.0, t1 = 0.0, t2 = 0.0, dn = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v += tq<N>(q, i) * h0[i];
                t1 += tdq<N>(q, i) * h0[i];
                t2 += tq<N>(q, i) * h1[i];
                dn += tq<N>(q, i) * h2[i];
            }
            vnb[q] = v;
            const double g0 = gv[q % AH][0], g1 = gv[q % AH][1], g2 = gv[q % AH][2];
            if (q + AH < Q) request_nb(q + AH, gv[q % AH]);
            if constexpr (AH < Q) {
                fnb[q] = g0 * v0 * dn + g1 * v1 * t1 + g2 * v2 * t2;
            } else {
                if (cmp) fnb[q] = g0 * (v0 * dn + v1 * t1 + v2 * t2);
                else fnb[q] = g0 * dn + g1 * t1 + g2 * t2;
            }
        }
    }
    q_sync<N>();
    // step 1, own side
    if (cl) {
        const int m0 = sc ? (N - 1) * sm : 0, dm = sc ? -sm : sm;
        const double sgn = sc ? -1.0 : 1.0;
        const double *uo = (C::OWN_LDS ? S : x + cid * ND) + p * sp + m0;
#pragma unroll
        for (int r = 0; r < N; ++r) {
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < N; ++m) s += KDL<N>::d[m] * uo[r * sr + m * dm];
            D[r] = sgn * s;
            L[r] = uo[r * sr];
        }
        step1(L, D);
    }
    q_sync<N>();
    // steps 2 and 3, own side: flux terms point by point and the transposed
    // sweep along the first direction, written over the row read; the next
    // point's data always in flight
    if (rl) {
        double h0[N], h1[N], h2[N], A0[N], A1[N], A2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            h0[i] = gr[i];
            h1[i] = gr[QN + i];
            h2[i] = gr[2 * QN + i];
            A0[i] = A1[i] = A2[i] = 0.0;
        }
        double w0 = 1.0, w1 = 1.0, w2 = 1.0, sd = 1.0;
        if (cmp) {
            w0 = kf[go];
            w1 = kf[go + 1];
            w2 = kf[go + 2];
            sd = kf[6];
        }
        const double sg = sr_ ? 1.0 : -1.0;
        // the last value: penalty factor, or beta w of the neighbour's side
        const double *fp = cmp ? fn : fd + 6 * Q2;
        double nx[4];
        auto request = [&](int q) {
            nx[0] = fo[Q * q];
            if (!C::BRANCH || !cmp) {
                nx[1] = fo[Q * q + st];
                nx[2] = fo[Q * q + 2 * st];
                nx[3] = fp[Q * q];
            }
        };
        request(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            double g0 = nx[0], g1 = nx[1], g2 = nx[2], pen = nx[3];
            if (!C::BRANCH || cmp) {
                const double bo = nx[0], bn = C::BRANCH ? gv[q % AH][0] : nx[3];
                g0 = bo * w0;
                g1 = (C::BRANCH ? bo : nx[1]) * w1;
                g2 = (C::BRANCH ? bo : nx[2]) * w2;
                if (cmp) pen = sd * (bo + bn);
            }
            if (q + 1 < Q) request(q + 1);
            double v = 0.0, t1 = 0.0, t2 = 0.0, dn = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v += tq<N>(q, i) * h0[i];
                t1 += tdq<N>(q, i) * h0[i];
                t2 += tq<N>(q, i) * h1[i];
                dn += tq<N>(q, i) * h2[i];
            }
            const double flux = g0 * dn + g1 * t1 + g2 * t2 + fnb[q];
            const double jump = sr_ ? (v - vnb[q]) : (vnb[q] - v);
            const double cv = sg * (-0.5 * flux + pen * jump), hj = -0.5 * jump;
            const double ct1 = hj * g1, ct2 = hj * g2, cn = hj * g0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                A0[i] += tq<N>(q, i) * cv + tdq<N>(q, i) * ct1;
                A1[i] += tq<N>(q, i) * ct2;
                A2[i] += tq<N>(q, i) * cn;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            gr[i] = A0[i];
            gr[QN + i] = A1[i];
            gr[2 * QN + i] = A2[i];
        }
    }
    q_sync<N>();
    // step 4, column lanes: transposed sweep along the second direction, in
    // place (a column lane reads and writes its own column only)
    if (cl0) {
        double o0[N], o1[N];
#pragma unroll
        for (int r = 0; r < N; ++r) o0[r] = o1[r] = 0.0;
        if (cl)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const double b0 = gc[q * N + p], b1 = gc[QN + q * N + p], b2 = gc[2 * QN + q * N + p];
#pragma unroll
                for (int r = 0; r < N; ++r) {
                    o0[r] += tq<N>(q, r) * b0 + tdq<N>(q, r) * b1;
                    o1[r] += tq<N>(q, r) * b2;
                }
            }
#pragma unroll
        for (int r = 0; r < N; ++r) {
            gc[r * N + p] = o0[r];
            gc[QN + r * N + p] = o1[r];
        }
    }
}

template <int N>
__global__ void __launch_bounds__(QCfg<N>::NT, N <= 4 ? 4 : (N <= 5 ? 3 : 2))
k_apply_q(const double *__restrict__ x, double *__restrict__ y, const double *__restrict__ cell,
          const double *__restrict__ face, const int32_t *__restrict__ nbr,
          const uint8_t *__restrict__ ctype, const double *__restrict__ kk, int nwg)
{
    using C = QCfg<N>;
    constexpr int ND = C::ND, NF = C::NF, QN = C::QN, QNN = C::QNN, QQN = C::QQN, FPW = C::FPW;
    __shared__ double sU[2 * QNN], sV[3 * QQN], sX[C::OWN_LDS ? C::FW : 1][C::OWN_LDS ? ND : 1], sF[6 * 3 * QN];
    // contiguous ranges of the cells per XCD
    const int bid = blockIdx.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    const int64_t cid = xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = wave < C::CW ? threadIdx.x : threadIdx.x & 63;
    // affine cell with compressed data (no ctype: every cell has the general
    // ones): the same for the whole workgroup, so branches on it are uniform
    const bool aff = ctype && __builtin_amdgcn_readfirstlane(ctype[cid]);
    if (wave >= C::CW) {
        const int fw = wave - C::CW;
        q_faces<N>(x, face, nbr, ctype, aff, cid, lane, fw * FPW, sX[C::OWN_LDS ? fw : 0], sF + fw * FPW * 3 * QN);
        __syncthreads();
        return;
    }
    double Y[N];
    if (aff) q_cell<N, true>(x, cell, kk, cid, lane, sU, sV, Y);
    else q_cell<N, false>(x, cell, kk, cid, lane, sU, sV, Y);
    __syncthreads();
    // pencil owners (j, l) add the six faces
    if (lane >= NF) return;
    const int j = lane % N, l = lane / N;
    auto dl = [&](int s, int k) {   // derivative weight of a lane-dependent node
        double v = 0.0;
#pragma unroll
        for (int m = 0; m < N; ++m)
            if (m == k) v = KDL<N>::d[s * N + m];
        return v;
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int layer = s ? N - 1 : 0;
        const double *F = sF + s * 3 * QN;
        // x faces: normal coordinate i, (p, r) = (j, l)
        {
            const double f0 = F[j + N * l], f1 = F[QN + j + N * l];
#pragma unroll
            for (int i = 0; i < N; ++i) Y[i] += KDL<N>::d[s * N + i] * f1 + (i == layer ? f0 : 0.0);
        }
        // y faces: normal coordinate j, (p, r) = (i, l)
        const double ey = dl(s, j), ez = dl(s, l);
        const double *Fy = F + 6 * QN + N * l, *Fz = F + 12 * QN + N * j;
#pragma unroll
        for (int i = 0; i < N; ++i) Y[i] += ey * Fy[QN + i] + (j == layer ? Fy[i] : 0.0);
        // z faces: normal coordinate l, (p, r) = (i, j)
#pragma unroll
        for (int i = 0; i < N; ++i) Y[i] += ez * Fz[QN + i] + (l == layer ? Fz[i] : 0.0);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) y[cid * ND + N * lane + i] = Y[i];
}

template <int N>
hipError_t apply_q_n(hx_ctx *c, const double *x, double *y)
{
    hipLaunchKernelGGL(k_apply_q<N>, dim3((unsigned)c->n_cells), dim3(QCfg<N>::NT), 0, c->stream, x, y,
                       c->qcell, c->qface, c->nbr, c->q_lean ? c->ctype : nullptr, c->kk64, (int)c->n_cells);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_apply_q(hx_ctx *c, const double *x, double *y)
{
    if (c->nq != 2 * c->n - 1) return hipErrorInvalidValue;
    switch (c->n) {
    case 2: return apply_q_n<2>(c, x, y);
    case 3: return apply_q_n<3>(c, x, y);
    case 4: return apply_q_n<4>(c, x, y);
    case 5: return apply_q_n<5>(c, x, y);
    case 6: return apply_q_n<6>(c, x, y);
    case 7: return apply_q_n<7>(c, x, y);
    case 8: return apply_q_n<8>(c, x, y);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hx
