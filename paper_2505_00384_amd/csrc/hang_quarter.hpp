// The terms of one 2:1 quarter face, computed by one wave: shared by the
// operator kernel, which serves the quarters with workgroups of its own
// launch, and the launch for the face part alone.
#pragma once

#include "common.hpp"

namespace hx {

// The whole operator computes the quarters in its own launch.  From n = 7 its
// registers leave two waves per SIMD, too few for the quarters' latencies:
// there a launch of their own is faster on meshes that fill the chip.  32x8x16
// cells refined over the ridge, FP64, own launch / operator's: degree 1 14.4 /
// 11.6 us, 4 43.5 / 40.8, 5 92.3 / 88.1, 6 116.2 / 125.9, 7 168.7 / 179.7 (FP32
// 65.5 / 60.4, 79.5 / 86.9; 16x4x8 cells, FP64, 31.8 / 28.5, 43.1 / 40.0).
constexpr bool hang_in_operator(int n) { return n < 7; }

// contributions of one quarter to the test functions of both cells (one
// wave per quarter): contrib[h][side][nd], side 0 coarse, 1 fine.  Both
// sides' traces are sum-factorised on the face: items (side, i1, i2) take the
// face layer and the normal-derivative column (GLL nodes lie on the face, so
// the normal direction needs the end node and the derivative weights only),
// items (side, a, i2) contract along the first tangential direction with the
// side's 1-D tables at the quarter's points (the coarse side's at
// ((s + xi)/2)), items (a, b) along the second and form the flux terms of
// both sides, and the same steps run backwards to the face layer and the
// normal lines, which each item (side, i1, i2) writes whole.  A quarter is a
// chain of latencies, so everything it reads is requested at its start, and
// the coarse side's tables come from the set-up (each quarter used to evaluate
// the basis at its points).
template <int N, typename T>
struct HangLds {
    static constexpr int NF = N * N;
    T tb[2][2][2][NF];          // [side][tangential axis][value, derivative][a * N + i]
    T sDL[2][N];                // l_m'(0), l_m'(1)
    T Lv[2][NF], Ld[2][NF];     // face layer and normal derivative, [side][i1 + N i2]
    T T0[2][NF], T1[2][NF], T2[2][NF];   // along t1, [side][a + N i2]
    T Wv[2][NF], Wa[2][NF], Wb[2][NF], Wn[2][NF];   // weights per point a + N b
    T Gv[2][NF], Gb[2][NF], Gn[2][NF];   // back along t1, [side][i1 + N b]
};

template <int N, typename T>
__device__ __forceinline__ void
hang_quarter(int64_t h, const int32_t *__restrict__ hang, const RefTab64 *__restrict__ TB,
             const T *__restrict__ hd, const T *__restrict__ x, T *__restrict__ contrib,
             HangLds<N, T> &sh)
{
    constexpr int NF = N * N, ND = NF * N;
    auto &tb = sh.tb;
    auto &sDL = sh.sDL;
    auto &Lv = sh.Lv, &Ld = sh.Ld, &T0 = sh.T0, &T1 = sh.T1, &T2 = sh.T2;
    auto &Wv = sh.Wv, &Wa = sh.Wa, &Wb = sh.Wb, &Wn = sh.Wn, &Gv = sh.Gv, &Gb = sh.Gb, &Gn = sh.Gn;
    const int32_t *rec = hang + 4 * h;
    const int fc = rec[1], d = fc >> 1, sq = rec[3];
    const int t1 = d == 0 ? 1 : 0, t2 = d == 2 ? 1 : 2;
    const int s1 = d == 0 ? N : 1, s2 = d == 2 ? N : NF, sn = d == 0 ? 1 : (d == 1 ? N : NF);
    // end node along the normal: the coarse cell's face fc, the fine cell's fc ^ 1
    const int ec = fc & 1;
    const int minus = (fc & 1) ? 0 : 1;
    const int tid = threadIdx.x;
    constexpr int IPL = (2 * NF + 63) / 64;   // items (side, i1, i2) per lane
    T xv[IPL][N], gq[7];
#pragma unroll
    for (int w = 0; w < IPL; ++w) {
        const int it = tid + 64 * w < 2 * NF ? tid + 64 * w : 0;
        const int side = it / NF, k = it % NF;
        const T *xp = x + (int64_t)(side ? rec[2] : rec[0]) * ND + (k % N) * s1 + (k / N) * s2;
#pragma unroll
        for (int m = 0; m < N; ++m) xv[w][m] = xp[m * sn];
    }
    // data of point tid: coarse side and fine side along (t1, t2, normal), s
    {
        const T *g = hd + h * 7 * NF + (tid < NF ? tid : 0);
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            gq[3 * sd] = g[(3 * sd + t1) * NF];
            gq[3 * sd + 1] = g[(3 * sd + t2) * NF];
            gq[3 * sd + 2] = g[(3 * sd + d) * NF];
        }
        gq[6] = g[6 * NF];
    }
    // 1-D tables: fine side from the set-up tables, coarse side at the
    // quarter's points
    for (int e = tid; e < 2 * NF; e += 64) {
        const int ax = e / NF, k = e % NF;
        const int half = ax == 0 ? (sq & 1) : (sq >> 1);
        tb[0][ax][0][k] = (T)TB->Bh[half][0][k];
        tb[0][ax][1][k] = (T)TB->Bh[half][1][k];
        tb[1][ax][0][k] = (T)TB->B[k];
        tb[1][ax][1][k] = (T)TB->BD[k];
    }
    if (tid < 2 * N) sDL[tid / N][tid % N] = (T)TB->DL[tid / N][tid % N];
    __syncthreads();
    // face layer and normal derivative: item (side, i1, i2)
#pragma unroll
    for (int w = 0; w < IPL; ++w) {
        const int it = tid + 64 * w;
        if (it >= 2 * NF) break;
        const int side = it / NF, k = it % NF, e = side ? 1 - ec : ec;
        T dn = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) dn += sDL[e][m] * xv[w][m];
        Lv[side][k] = e ? xv[w][N - 1] : xv[w][0];
        Ld[side][k] = dn;
    }
    __syncthreads();
    // along t1: item (side, a, i2)
    for (int it = tid; it < 2 * NF; it += 64) {
        const int side = it / NF, k = it % NF;
        const int a = k % N, i2 = k / N;
        const T *B1 = tb[side][0][0] + a * N, *D1 = tb[side][0][1] + a * N;
        T c0 = 0, c1 = 0, c2 = 0;
#pragma unroll
        for (int i1 = 0; i1 < N; ++i1) {
            c0 += B1[i1] * Lv[side][i1 + N * i2];
            c1 += D1[i1] * Lv[side][i1 + N * i2];
            c2 += B1[i1] * Ld[side][i1 + N * i2];
        }
        T0[side][k] = c0;
        T1[side][k] = c1;
        T2[side][k] = c2;
    }
    __syncthreads();
    // along t2 and the flux terms at point (a, b): both sides in one item
    static_assert(NF <= 64, "a lane per point");
    if (tid < NF) {
        const int pt = tid, a = pt % N, b = pt / N;
        T u[2], ga[2], gb[2], gn[2];
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            const T *B2 = tb[sd][1][0] + b * N, *D2 = tb[sd][1][1] + b * N;
            u[sd] = ga[sd] = gb[sd] = gn[sd] = 0;
#pragma unroll
            for (int i2 = 0; i2 < N; ++i2) {
                u[sd] += B2[i2] * T0[sd][a + N * i2];
                ga[sd] += B2[i2] * T1[sd][a + N * i2];
                gb[sd] += D2[i2] * T0[sd][a + N * i2];
                gn[sd] += B2[i2] * T2[sd][a + N * i2];
            }
        }
        T flux = 0;
#pragma unroll
        for (int sd = 0; sd < 2; ++sd)
            flux += gq[3 * sd] * ga[sd] + gq[3 * sd + 1] * gb[sd] + gq[3 * sd + 2] * gn[sd];
        const T jump = minus ? u[1] - u[0] : u[0] - u[1];
        const T pen = gq[6];
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            const T z = sd == minus ? T(1) : T(-1);
            const T hj = T(-0.5) * jump;
            Wv[sd][pt] = z * (T(-0.5) * flux + pen * jump);
            Wa[sd][pt] = hj * gq[3 * sd];
            Wb[sd][pt] = hj * gq[3 * sd + 1];
            Wn[sd][pt] = hj * gq[3 * sd + 2];
        }
    }
    __syncthreads();
    // back along t1: item (side, i1, b)
    for (int it = tid; it < 2 * NF; it += 64) {
        const int side = it / NF, k = it % NF;
        const int i1 = k % N, b = k / N;
        const T *B1 = tb[side][0][0], *D1 = tb[side][0][1];
        T gv = 0, gb = 0, gn = 0;
#pragma unroll
        for (int a = 0; a < N; ++a) {
            const int pt = a + N * b;
            gv += B1[a * N + i1] * Wv[side][pt] + D1[a * N + i1] * Wa[side][pt];
            gb += B1[a * N + i1] * Wb[side][pt];
            gn += B1[a * N + i1] * Wn[side][pt];
        }
        Gv[side][k] = gv;
        Gb[side][k] = gb;
        Gn[side][k] = gn;
    }
    __syncthreads();
    // back along t2 and out: item (side, i1, i2) writes its normal line
    for (int it = tid; it < 2 * NF; it += 64) {
        const int side = it / NF, k = it % NF;
        const int i1 = k % N, i2 = k / N;
        const T *B2 = tb[side][1][0], *D2 = tb[side][1][1];
        T f0 = 0, f1 = 0;
#pragma unroll
        for (int b = 0; b < N; ++b) {
            f0 += B2[b * N + i2] * Gv[side][i1 + N * b] + D2[b * N + i2] * Gb[side][i1 + N * b];
            f1 += B2[b * N + i2] * Gn[side][i1 + N * b];
        }
        const int e = side ? 1 - ec : ec;
        T *out = contrib + (h * 2 + side) * ND + i1 * s1 + i2 * s2;
#pragma unroll
        for (int m = 0; m < N; ++m) out[m * sn] = sDL[e][m] * f1 + (m == (e ? N - 1 : 0) ? f0 : T(0));
    }
}

}  // namespace hx
