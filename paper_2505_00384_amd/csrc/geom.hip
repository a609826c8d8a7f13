// Geometry and coefficient set-up (FP64): cell metric terms, face normals,
// surface elements and penalties, merged per-quadrature-point operator data,
// the separable block-Jacobi eigen-tables and dof coordinates.
//
// The geometry kernels run once per mesh (setup_mesh) and favour clarity over
// speed; the coefficient kernels (k_set_cell, k_set_face) run at every
// fixed-point iteration of the paper's pressure solve (section 3.1).
#include "common.hpp"

#include <cmath>

namespace hx {
namespace {

// compile-time copies of the 1-D tables (generated at build time from the
// library's rules)
template <int N> struct KB;
template <int N> struct KBD;
template <int N> struct KDL;
#include "optables.inc"

// Lagrange basis through the equispaced nodes a/g, a = 0..g (the geometry
// nodes of the mesh format): values and derivatives at t.
__device__ inline void lag_equi(int ng, double t, double *v, double *d)
{
    const double g = ng - 1;
    for (int i = 0; i < ng; ++i) {
        const double xi = i / g;
        double val = 1.0, der = 0.0;
        for (int m = 0; m < ng; ++m) {
            if (m == i) continue;
            const double xm = m / g;
            const double f = (t - xm) / (xi - xm);
            der = der * f + val / (xi - xm);
            val *= f;
        }
        v[i] = val;
        d[i] = der;
    }
}

// x(xi) and J = dx/dxi of one cell from its geometry nodes X[(g+1)^3][3].
__device__ inline void cell_map(const double *__restrict__ X, int ng, const double xi[3],
                                double x[3], double J[3][3])
{
    double v[3][MAXG + 1], d[3][MAXG + 1];
    for (int c = 0; c < 3; ++c) lag_equi(ng, xi[c], v[c], d[c]);
    for (int r = 0; r < 3; ++r) x[r] = J[r][0] = J[r][1] = J[r][2] = 0.0;
    for (int cz = 0; cz < ng; ++cz)
        for (int cy = 0; cy < ng; ++cy) {
            const double vyz = v[1][cy] * v[2][cz], dyz = d[1][cy] * v[2][cz], yzd = v[1][cy] * d[2][cz];
            for (int cx = 0; cx < ng; ++cx) {
                const double *P = X + 3 * (cx + ng * (cy + ng * cz));
                const double s = v[0][cx] * vyz, s0 = d[0][cx] * vyz, s1 = v[0][cx] * dyz,
                             s2 = v[0][cx] * yzd;
                for (int r = 0; r < 3; ++r) {
                    const double p = P[r];
                    x[r] += s * p;
                    J[r][0] += s0 * p;
                    J[r][1] += s1 * p;
                    J[r][2] += s2 * p;
                }
            }
        }
}

__device__ inline double det3(const double J[3][3])
{
    return J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
           J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
           J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
}

// Ji = J^{-1}
__device__ inline void inv3(const double J[3][3], double det, double Ji[3][3])
{
    const double id = 1.0 / det;
    Ji[0][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) * id;
    Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
    Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
    Ji[1][0] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) * id;
    Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
    Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
    Ji[2][0] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) * id;
    Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
    Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
}

__device__ inline int lidx(int n, int i, int j, int l) { return i + n * (j + n * l); }

// local index of the point with coordinate m along d and tangential (p, r),
// t1 < t2 the other two directions
__device__ inline int layer_idx(int n, int d, int m, int p, int r)
{
    int c[3];
    const int t1 = d == 0 ? 1 : 0, t2 = d == 2 ? 1 : 2;
    c[d] = m;
    c[t1] = p;
    c[t2] = r;
    return lidx(n, c[0], c[1], c[2]);
}

__device__ inline void face_xi(const RefTab64 *T, int d, int plus, int a, int b, double xi[3])
{
    const int t1 = d == 0 ? 1 : 0, t2 = d == 2 ? 1 : 2;
    xi[d] = plus ? 1.0 : 0.0;
    xi[t1] = T->xq[a];
    xi[t2] = T->xq[b];
}

// -------------------------------------------------------------------------
// per cell: volume, mean column lengths l_d, minimum detJ (thread per cell)
// -------------------------------------------------------------------------
__global__ void k_cell_geometry(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                                const RefTab64 *__restrict__ T, double *vol, double *ell,
                                double *mindet)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= n_cells) return;
    const double *X = nodes + c * (int64_t)ng * ng * ng * 3;
    double v = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0, md = 1e300;
    for (int l = 0; l < n; ++l)
        for (int j = 0; j < n; ++j)
            for (int i = 0; i < n; ++i) {
                double xi[3] = {T->xq[i], T->xq[j], T->xq[l]}, x[3], J[3][3];
                cell_map(X, ng, xi, x, J);
                const double det = det3(J);
                md = fmin(md, det);
                v += T->wq[i] * T->wq[j] * T->wq[l] * det;
                e0 += sqrt(J[0][0] * J[0][0] + J[1][0] * J[1][0] + J[2][0] * J[2][0]);
                e1 += sqrt(J[0][1] * J[0][1] + J[1][1] * J[1][1] + J[2][1] * J[2][1]);
                e2 += sqrt(J[0][2] * J[0][2] + J[1][2] * J[1][2] + J[2][2] * J[2][2]);
            }
    const double inv = 1.0 / (n * n * n);
    vol[c] = v;
    ell[3 * c + 0] = e0 * inv;
    ell[3 * c + 1] = e1 * inv;
    ell[3 * c + 2] = e2 * inv;
    mindet[c] = md;
}

// -------------------------------------------------------------------------
// penalty of the +d face of each cell (thread per (cell, d))
// -------------------------------------------------------------------------
__global__ void k_face_sigma(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                             const int32_t *__restrict__ nbr, const RefTab64 *__restrict__ T,
                             const double *__restrict__ vol, double P, double *sigma)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= 3 * n_cells) return;
    const int64_t c = t / 3;
    const int d = (int)(t % 3);
    const int32_t nb = nbr[6 * c + 2 * d + 1];
    if (nb < 0) {
        sigma[t] = -1.0;
        return;
    }
    const double *X = nodes + c * (int64_t)ng * ng * ng * 3;
    double area = 0.0;
    for (int b = 0; b < n; ++b)
        for (int a = 0; a < n; ++a) {
            double xi[3], x[3], J[3][3], Ji[3][3];
            face_xi(T, d, 1, a, b, xi);
            cell_map(X, ng, xi, x, J);
            const double det = det3(J);
            inv3(J, det, Ji);
            // |J^{-T} e_d| = norm of row d of J^{-1}
            const double len = sqrt(Ji[d][0] * Ji[d][0] + Ji[d][1] * Ji[d][1] + Ji[d][2] * Ji[d][2]);
            area += T->wq[a] * T->wq[b] * det * len;
        }
    const double r = fmax(area / vol[c], area / vol[nb]);
    sigma[t] = P * (double)(n * n) * r;
}

// -------------------------------------------------------------------------
// generalised eigenproblems of the separable block (thread per (cell, d)):
// L_d s = lambda M s with L_d the 1-D SIP block of the cell in direction d.
// -------------------------------------------------------------------------
template <int N>
__device__ void jacobi_eig(double (&A)[N][N], double (&V)[N][N])
{
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) V[i][j] = (i == j) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int i = 0; i < N; ++i)
            for (int j = 0; j < N; ++j) {
                tot += A[i][j] * A[i][j];
                if (i != j) off += A[i][j] * A[i][j];
            }
        if (off <= 1e-34 * tot) break;
        for (int p = 0; p < N - 1; ++p)
            for (int q = p + 1; q < N; ++q) {
                const double apq = A[p][q];
                if (apq == 0.0) continue;
                const double theta = (A[q][q] - A[p][p]) / (2.0 * apq);
                const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
                for (int k = 0; k < N; ++k) {
                    const double akp = A[k][p], akq = A[k][q];
                    A[k][p] = cs * akp - sn * akq;
                    A[k][q] = sn * akp + cs * akq;
                }
                for (int k = 0; k < N; ++k) {
                    const double apk = A[p][k], aqk = A[q][k];
                    A[p][k] = cs * apk - sn * aqk;
                    A[q][k] = sn * apk + cs * aqk;
                }
                for (int k = 0; k < N; ++k) {
                    const double vkp = V[k][p], vkq = V[k][q];
                    V[k][p] = cs * vkp - sn * vkq;
                    V[k][q] = sn * vkp + cs * vkq;
                }
            }
    }
}

template <int N>
__global__ void k_bj_eigen(int64_t n_cells, const int32_t *__restrict__ nbr,
                           const RefTab64 *__restrict__ T, const double *__restrict__ ell,
                           const double *__restrict__ sigma, const double *__restrict__ endsig,
                           double *S64, float *S32, double *L64, float *L32)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= 3 * n_cells) return;
    const int64_t c = t / 3;
    const int d = (int)(t % 3);
    const double l = ell[3 * c + d];
    const int32_t lo = nbr[6 * c + 2 * d], hi = nbr[6 * c + 2 * d + 1];
    // a non-conforming end (neighbour -2) takes its penalty from endsig
    const double sig_lo = lo >= 0 ? sigma[3 * (int64_t)lo + d] : (lo == -2 ? endsig[6 * c + 2 * d] : -1.0);
    const double sig_hi = hi >= 0 ? sigma[3 * c + d] : (hi == -2 ? endsig[6 * c + 2 * d + 1] : -1.0);
    double L[N][N];
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) L[i][j] = T->L0[i * N + j];
    // end terms; the GLL basis is 1 at its own end node and 0 at the others
    if (sig_lo >= 0.0) {   // end 0, outward reference normal -1
        for (int i = 0; i < N; ++i) {
            L[i][0] += 0.5 * T->DL[0][i];
            L[0][i] += 0.5 * T->DL[0][i];
        }
        L[0][0] += sig_lo * l;
    }
    if (sig_hi >= 0.0) {   // end 1, outward reference normal +1
        for (int i = 0; i < N; ++i) {
            L[i][N - 1] -= 0.5 * T->DL[1][i];
            L[N - 1][i] -= 0.5 * T->DL[1][i];
        }
        L[N - 1][N - 1] += sig_hi * l;
    }
    // C = Cinv L Cinv^T
    double A[N][N], tmp[N][N], V[N][N];
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            double s = 0.0;
            for (int r = 0; r < N; ++r) s += T->Cinv[i * N + r] * L[r][j];
            tmp[i][j] = s;
        }
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            double s = 0.0;
            for (int r = 0; r < N; ++r) s += tmp[i][r] * T->Cinv[j * N + r];
            A[i][j] = s;
        }
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < i; ++j) A[i][j] = A[j][i] = 0.5 * (A[i][j] + A[j][i]);
    jacobi_eig<N>(A, V);
    // S = Cinv^T V, stored row-major S[i][m]
    double *S = S64 + t * N * N;
    float *Sf = S32 + t * N * N;
    for (int i = 0; i < N; ++i)
        for (int m = 0; m < N; ++m) {
            double s = 0.0;
            for (int r = 0; r < N; ++r) s += T->Cinv[r * N + i] * V[r][m];
            S[i * N + m] = s;
            Sf[i * N + m] = (float)s;
        }
    for (int m = 0; m < N; ++m) {
        L64[t * N + m] = A[m][m];
        L32[t * N + m] = (float)A[m][m];
    }
}

// -------------------------------------------------------------------------
// Geometric factors, once per mesh (block per cell / thread per face point).
// Cell quadrature point q:   cg[0] = w detJ,
//                            cg[1..6] = w detJ (J^-1 J^-T)_{xx,xy,xz,yy,yz,zz}.
// Point (a, b) of the +d face of a cell (a, b along the first and second
// tangential direction, stored at b + n a):
//                            fg[0..2] = ds J-^{-1} n,  fg[3..5] = ds J+^{-1} n
// (components in the face's own order: normal direction d, first, second
// tangential), fg[6] = ds / 2, with n and ds from the minus cell; zero on
// boundary faces.  Coefficients multiply these in k_set_cell / k_set_face.
// -------------------------------------------------------------------------
__global__ void k_cell_geofac(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                              const RefTab64 *__restrict__ T, double *cellgeo)
{
    const int nd = n * n * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n_cells * nd) return;
    const int64_t c = t / nd;
    const int q = (int)(t % nd);
    const int i = q % n, j = (q / n) % n, l = q / (n * n);
    double xi[3] = {T->xq[i], T->xq[j], T->xq[l]}, x[3], J[3][3], Ji[3][3];
    cell_map(nodes + c * (int64_t)ng * ng * ng * 3, ng, xi, x, J);
    const double det = det3(J);
    inv3(J, det, Ji);
    const double w = T->wq[i] * T->wq[j] * T->wq[l] * det;
    double *dst = cellgeo + c * 7 * nd + q;
    dst[0] = w;
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
    for (int s = 0; s < 6; ++s) {
        const int A = pa[s], Bq = pb[s];
        dst[(1 + s) * nd] = w * (Ji[A][0] * Ji[Bq][0] + Ji[A][1] * Ji[Bq][1] + Ji[A][2] * Ji[Bq][2]);
    }
}

__global__ void k_face_geofac(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                              const int32_t *__restrict__ nbr, const RefTab64 *__restrict__ T,
                              double *facegeo)
{
    const int nf = n * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= 3 * n_cells * nf) return;
    const int pt = (int)(t % nf);
    const int64_t cd = t / nf;
    const int64_t c = cd / 3;
    const int d = (int)(cd % 3);
    const int b = pt % n, a = pt / n;
    double *dst = facegeo + cd * 7 * nf + pt;
    const int32_t nb = nbr[6 * c + 2 * d + 1];
    if (nb < 0) {
        for (int s = 0; s < 7; ++s) dst[s * nf] = 0.0;
        return;
    }
    double xim[3], xip[3], x[3], Jm[3][3], Jp[3][3], Jmi[3][3], Jpi[3][3];
    face_xi(T, d, 1, a, b, xim);
    face_xi(T, d, 0, a, b, xip);
    const int64_t gsz = (int64_t)ng * ng * ng * 3;
    cell_map(nodes + c * gsz, ng, xim, x, Jm);
    cell_map(nodes + (int64_t)nb * gsz, ng, xip, x, Jp);
    const double detm = det3(Jm), detp = det3(Jp);
    inv3(Jm, detm, Jmi);
    inv3(Jp, detp, Jpi);
    // J^{-T} e_d is row d of J^{-1}
    double nv[3] = {Jmi[d][0], Jmi[d][1], Jmi[d][2]};
    const double len = sqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    for (int r = 0; r < 3; ++r) nv[r] /= len;
    const double ds = T->wq[a] * T->wq[b] * detm * len;
    const int dir[3] = {d, d == 0 ? 1 : 0, d == 2 ? 1 : 2};
    for (int k = 0; k < 3; ++k) {
        const int r = dir[k];
        dst[k * nf] = ds * (Jmi[r][0] * nv[0] + Jmi[r][1] * nv[1] + Jmi[r][2] * nv[2]);
        dst[(3 + k) * nf] = ds * (Jpi[r][0] * nv[0] + Jpi[r][1] * nv[1] + Jpi[r][2] * nv[2]);
    }
    dst[6 * nf] = 0.5 * ds;
}

// -------------------------------------------------------------------------
// Affine cells (thread per cell): the geometry nodes are the image of the
// reference nodes under x0 + A xi, A from the three edges at the first corner,
// to 1e-14 of the longest edge.  Their Jacobian is constant, so the operator
// may read one J^-1 J^-T per cell and the coefficients at the points instead
// of the seven merged values per point.  The per-cell constants are taken
// from the general geometric factors of the first Gauss point:
// kk = (w detJ J^-1 J^-T) / (w detJ), and detJ.
// -------------------------------------------------------------------------
__global__ void k_affine_detect(const double *__restrict__ nodes, int ng, int nd, int64_t n_cells,
                                const RefTab64 *__restrict__ T, const double *__restrict__ cellgeo,
                                uint8_t *ctype, double *kk64, float *kk32)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= n_cells) return;
    const double *X = nodes + c * (int64_t)ng * ng * ng * 3;
    const int g = ng - 1;
    const int corner[3] = {g, g * ng, g * ng * ng};
    double A[3][3], diam = 0.0;
    for (int d = 0; d < 3; ++d) {
        double s = 0.0;
        for (int r = 0; r < 3; ++r) {
            A[r][d] = X[3 * corner[d] + r] - X[r];
            s += A[r][d] * A[r][d];
        }
        diam = fmax(diam, sqrt(s));
    }
    double dev = 0.0;
    for (int az = 0; az < ng; ++az)
        for (int ay = 0; ay < ng; ++ay)
            for (int ax = 0; ax < ng; ++ax) {
                const double xi[3] = {(double)ax / g, (double)ay / g, (double)az / g};
                const double *P = X + 3 * (ax + ng * (ay + ng * az));
                for (int r = 0; r < 3; ++r) {
                    const double pr = X[r] + A[r][0] * xi[0] + A[r][1] * xi[1] + A[r][2] * xi[2];
                    dev = fmax(dev, fabs(P[r] - pr));
                }
            }
    ctype[c] = dev <= 1e-14 * diam ? 1 : 0;
    const double *geo = cellgeo + c * 7 * nd;
    const double w0 = geo[0];
    for (int s = 0; s < 6; ++s) {
        const double v = geo[(1 + s) * nd] / w0;
        kk64[8 * c + s] = v;
        kk32[8 * c + s] = (float)v;
    }
    const double det = w0 / (T->wq[0] * T->wq[0] * T->wq[0]);
    kk64[8 * c + 6] = det;
    kk32[8 * c + 6] = (float)det;
    kk64[8 * c + 7] = 0.0;
    kk32[8 * c + 7] = 0.0f;
}

// -------------------------------------------------------------------------
// Coefficient update, cell part: from nodal alpha, beta of a cell
//   m = alpha_q w detJ,  G = beta_q w detJ J^-1 J^-T  (alpha_q, beta_q: the
// nodal fields at the Gauss point), on affine cells alpha w detJ and beta w
// detJ in their place, the cell means of the separable block (volume-weighted
// alpha, beta), the network's coefficient feature, and the inverse volume
// diagonals
//   d_i = sum_q [ m_q phi_i(q)^2 + grad phi_i(q)^T G_q grad phi_i(q) ],
// phi_i(q) = B(qx,a) B(qy,b) B(qz,l), reference gradient from BD: dg[0] of
// mass plus stiffness (the paper's Helmholtz preconditioner, section 3.1),
// dg[1] of the mass alone (its internal-energy variant).
//
// One wave serves CPW cells with LPC lanes each (N = 5: 2 x 32), lane (a, b)
// owning a pencil as in the operator kernel.  alpha and beta go to the Gauss
// points by three sweeps; the z-pencil lanes form the merged values plane by
// plane, store them and contract them along z on the fly with the products
// of the 1-D tables P0 = B B, P1 = B BD, P2 = BD BD (every term of the
// diagonal is a tensor contraction of one quadrature field with such
// products, e.g. the Gxy term is 2 sum_q Gxy P1(qx,a) P1(qy,b) P0(qz,l); terms
// that share their remaining tables are merged); y and x follow through LDS.
// The bound is memory: at degree 4 a general cell reads 72 and writes 108
// bytes per dof, an affine one, whose six G components nothing reads while
// the compressed data are in use, 24 and 60 (FULL writes them all the same).
// The former kernels (N^6 interpolation with one point per lane, a second
// kernel that read the merged data back for the diagonals) took 1.17 ms at
// 64x32x32 cells, degree 4; this one 0.28 ms, with the two waves per SIMD
// that its registers allow (three or four waves, by spilling or with the
// geometric factors loaded plane by plane, 0.32 to 0.44: more concurrent
// streams only scatter the writes).
// -------------------------------------------------------------------------
template <int N>
struct SCfg {
    static constexpr int NF = N * N, ND = NF * N, LPC = pow2_at_least(NF), CPW = 64 / LPC;
    // face kernel: 6 N columns per cell
    static constexpr int FLPC = pow2_at_least(6 * N), FCPW = 64 / FLPC;
    static_assert(NF <= 64 && 6 * N <= 64, "one wave per cell at most");
};

// this workgroup's place when every XCD takes one contiguous range (they are
// dealt round-robin to the XCDs): the cache lines that two neighbouring
// cells share are then written through one L2 (both kernels together at
// 64x32x32 cells, degree 4: 0.48 -> 0.42 ms)
__device__ __forceinline__ int64_t xcd_range()
{
    const int bid = blockIdx.x, nwg = gridDim.x;
    const int q8 = nwg / NXCD, r8 = nwg % NXCD, xcd = bid % NXCD;
    return xcd * q8 + (xcd < r8 ? xcd : r8) + bid / NXCD;
}

// products of the 1-D tables: kind 0 B B, 1 B BD, 2 BD BD
template <int N, int KIND>
__device__ __forceinline__ constexpr double ptab(int q, int a)
{
    const double bv = KB<N>::d[q * N + a], dv = KBD<N>::d[q * N + a];
    return KIND == 0 ? bv * bv : (KIND == 1 ? bv * dv : dv * dv);
}

// y += P^T u along a pencil (table index q, output index a)
template <int N, int KIND>
__device__ __forceinline__ void padd(const double (&u)[N], double (&y)[N])
{
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
        for (int q = 0; q < N; ++q) y[a] += ptab<N, KIND>(q, a) * u[q];
}

template <int N, bool FULL>
__global__ void __launch_bounds__(64)
k_set_cell(int64_t n_cells, const double *__restrict__ alpha, const double *__restrict__ beta,
           const double *__restrict__ ell, const double *__restrict__ cellgeo,
           const uint8_t *__restrict__ ctype, const double *__restrict__ kk, double *__restrict__ cell64,
           float *__restrict__ cell32, double *__restrict__ acell64, float *__restrict__ acell32,
           double *__restrict__ bjC64, float *__restrict__ bjC32, double *__restrict__ coef_feat,
           double *__restrict__ dg64, float *__restrict__ dg32)
{
    constexpr int NF = SCfg<N>::NF, ND = SCfg<N>::ND, LPC = SCfg<N>::LPC, CPW = SCfg<N>::CPW;
    __shared__ double sm[CPW][4 * ND];
    const int cs = threadIdx.x / LPC, ln = threadIdx.x % LPC;
    const int64_t cid = xcd_range() * CPW + cs;
    const bool valid = cid < n_cells, on = valid && ln < NF;
    const int a = ln % N, b = ln / N;
    double *S = sm[cs];
    const bool aff = on && ctype[cid];
    // alpha, beta to the Gauss points: x, y, z sweeps, lane (a, b) the pencil's
    // two fixed indices
    double u[N], v[N], p[N], q_[N];
    if (on) {
        const int64_t o = cid * ND + N * a + NF * b;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            u[i] = alpha[o + i];
            v[i] = beta[o + i];
        }
    }
    // the quadrature points' geometric factors, requested before the sweeps
    // (degrees up to 4; above, plane by plane in the loop below)
    constexpr bool PRE = N <= 5;
    const double *g = cellgeo + (on ? cid : 0) * 7 * ND + a + N * b;
    double gq[PRE ? N : 1][7];
    if constexpr (PRE) {
        if (on) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                gq[q][0] = __builtin_nontemporal_load(g + NF * q);
                if (FULL || !aff)
#pragma unroll
                    for (int s = 1; s < 7; ++s) gq[q][s] = __builtin_nontemporal_load(g + NF * q + s * ND);
            }
        }
    }
    auto interp = [&](const double (&w)[N], double (&y)[N]) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) s += KB<N>::d[q * N + i] * w[i];
            y[q] = s;
        }
    };
    if (on) {
        interp(u, p);
        interp(v, q_);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            S[q + N * a + NF * b] = p[q];
            S[ND + q + N * a + NF * b] = q_[q];
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            u[j] = S[a + N * j + NF * b];
            v[j] = S[ND + a + N * j + NF * b];
        }
        interp(u, p);
        interp(v, q_);
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            S[a + N * q + NF * b] = p[q];
            S[ND + a + N * q + NF * b] = q_[q];
        }
    }
    __syncthreads();
    // z sweep, merged values and the diagonals' z contraction: lane (qx, qy)
    double sw = 0.0, sa = 0.0, sb = 0.0;
    // contracted fields: m, Gxx, Gxy, Gxz, Gyy, Gyz, Gzz (tables P0, P0, P0,
    // P1, P0, P1, P2)
    double t[7][N];
#pragma unroll
    for (int s = 0; s < 7; ++s)
#pragma unroll
        for (int l = 0; l < N; ++l) t[s][l] = 0.0;
    if (on) {
#pragma unroll
        for (int l = 0; l < N; ++l) {
            u[l] = S[a + N * b + NF * l];
            v[l] = S[ND + a + N * b + NF * l];
        }
        interp(u, p);
        interp(v, q_);
        double kc[6];
        if (aff)
#pragma unroll
            for (int s = 0; s < 6; ++s) kc[s] = kk[8 * cid + s];
        double *dst = cell64 + cid * 7 * ND + a + N * b;
        float *dstf = cell32 + cid * 7 * ND + a + N * b;
        double *ad = acell64 + cid * 2 * ND + a + N * b;
        float *af = acell32 + cid * 2 * ND + a + N * b;
        auto pz = [&](int kind, int q, int l) {
            return kind == 0 ? ptab<N, 0>(q, l) : (kind == 1 ? ptab<N, 1>(q, l) : ptab<N, 2>(q, l));
        };
        constexpr int zk[7] = {0, 0, 0, 1, 0, 1, 2};
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const double w = PRE ? gq[PRE ? q : 0][0] : g[NF * q];
            const double am = p[q] * w, bm = q_[q] * w;
            sw += w;
            sa += am;
            sb += bm;
            dst[NF * q] = am;
            dstf[NF * q] = (float)am;
            if (FULL || !aff) {
                double G[7];
#pragma unroll
                for (int s = 1; s < 7; ++s) {
                    G[s] = q_[q] * (PRE ? gq[PRE ? q : 0][s] : g[NF * q + s * ND]);
                    dst[NF * q + s * ND] = G[s];
                    dstf[NF * q + s * ND] = (float)G[s];
                }
                G[0] = am;
#pragma unroll
                for (int s = 0; s < 7; ++s)
#pragma unroll
                    for (int l = 0; l < N; ++l) t[s][l] += pz(zk[s], q, l) * G[s];
            } else {
                // G = bm J^-1 J^-T: contract bm once with each table
#pragma unroll
                for (int l = 0; l < N; ++l) {
                    t[0][l] += ptab<N, 0>(q, l) * am;
                    t[1][l] += ptab<N, 0>(q, l) * bm;
                    t[3][l] += ptab<N, 1>(q, l) * bm;
                    t[6][l] += ptab<N, 2>(q, l) * bm;
                }
            }
            if (aff) {
                ad[NF * q] = am;
                ad[ND + NF * q] = bm;
                af[NF * q] = (float)am;
                af[ND + NF * q] = (float)bm;
            }
        }
        if (!FULL && aff) {
#pragma unroll
            for (int l = 0; l < N; ++l) {
                const double b0 = t[1][l], b1 = t[3][l];
                t[1][l] = kc[0] * b0;
                t[2][l] = kc[1] * b0;
                t[3][l] = kc[2] * b1;
                t[4][l] = kc[3] * b0;
                t[5][l] = kc[4] * b1;
                t[6][l] *= kc[5];
            }
        }
    }
    // cell means (fixed order: pencils, then lanes folded by halves)
#pragma unroll
    for (int o = LPC / 2; o > 0; o >>= 1) {
        sw += __shfl_xor(sw, o, 64);
        sa += __shfl_xor(sa, o, 64);
        sb += __shfl_xor(sb, o, 64);
    }
    if (valid && ln == 0) {
        const double ab = sa / sw, bb = sb / sw;
        const double lx = ell[3 * cid], ly = ell[3 * cid + 1], lz = ell[3 * cid + 2];
        const double cc[4] = {ab * lx * ly * lz, bb * ly * lz / lx, bb * lx * lz / ly, bb * lx * ly / lz};
        for (int r = 0; r < 4; ++r) {
            bjC64[4 * cid + r] = cc[r];
            bjC32[4 * cid + r] = (float)cc[r];
        }
        const double l2 = cbrt(lx * ly * lz);
        coef_feat[cid] = log(bb / (ab * l2 * l2));
    }
    // y contraction, lane (qx, l), in two rounds of LDS: the terms whose x
    // table is P0 (mass; m + Gzz, Gyy, 2 Gyz), then P2 (Gxx) and P1 (2 Gxy,
    // 2 Gxz)
    auto put = [&](int f, const double (&w)[N], double sc) {
#pragma unroll
        for (int l = 0; l < N; ++l) S[f * ND + a + N * b + NF * l] = sc * w[l];
    };
    auto get = [&](int f, double (&w)[N]) {
#pragma unroll
        for (int q = 0; q < N; ++q) w[q] = S[f * ND + a + N * q + NF * b];
    };
    __syncthreads();
    if (on) {
#pragma unroll
        for (int l = 0; l < N; ++l) t[6][l] += t[0][l];
        put(0, t[0], 1.0);
        put(1, t[6], 1.0);
        put(2, t[4], 1.0);
        put(3, t[5], 2.0);
    }
    __syncthreads();
    double cm[N], c0[N], c1[N], c2[N], w[N];
#pragma unroll
    for (int i = 0; i < N; ++i) cm[i] = c0[i] = c1[i] = c2[i] = 0.0;
    if (on) {
        get(0, w);
        padd<N, 0>(w, cm);
        get(1, w);
        padd<N, 0>(w, c0);
        get(2, w);
        padd<N, 2>(w, c0);
        get(3, w);
        padd<N, 1>(w, c0);
    }
    __syncthreads();
    if (on) {
        put(0, t[1], 1.0);
        put(1, t[2], 2.0);
        put(2, t[3], 2.0);
    }
    __syncthreads();
    if (on) {
        get(0, w);
        padd<N, 0>(w, c2);
        get(1, w);
        padd<N, 1>(w, c1);
        get(2, w);
        padd<N, 0>(w, c1);
    }
    __syncthreads();
    // x contraction: lane (j, l)
    if (on) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int e = a + N * j + NF * b;
            S[e] = cm[j];
            S[ND + e] = c0[j];
            S[2 * ND + e] = c2[j];
            S[3 * ND + e] = c1[j];
        }
    }
    __syncthreads();
    if (!on) return;
    double dm[N], dt[N];
#pragma unroll
    for (int i = 0; i < N; ++i) dm[i] = dt[i] = 0.0;
    auto row = [&](int f) {
#pragma unroll
        for (int q = 0; q < N; ++q) w[q] = S[f * ND + q + N * a + NF * b];
    };
    row(0);
    padd<N, 0>(w, dm);
    row(1);
    padd<N, 0>(w, dt);
    row(2);
    padd<N, 2>(w, dt);
    row(3);
    padd<N, 1>(w, dt);
    const int64_t o = cid * ND + N * a + NF * b, nt = n_cells * ND;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double ih = 1.0 / dt[i], im = 1.0 / dm[i];
        dg64[o + i] = ih;
        dg64[nt + o + i] = im;
        dg32[o + i] = (float)ih;
        dg32[nt + o + i] = (float)im;
    }
}

// -------------------------------------------------------------------------
// Coefficient update, face part: merged data of the +d face of every cell,
// [cell][d][component][a][b] with a, b the first and second tangential index:
//   g- = beta- ds J-^{-1} n,  g+ = beta+ ds J+^{-1} n,  s = sigma 1/2 (b- + b+) ds
// with n and ds from the minus cell; the three components of g are stored in
// the order (d, first tangential, second tangential) so that the operator
// pairs them with its reference derivatives without a per-lane selection.
// A face between two affine cells takes beta- w, beta+ w with w the face
// weight instead (g- = (beta- w) v-, g+ = (beta+ w) v+, s = sd ((beta- w) +
// (beta+ w)), constants in k_face_const); its general values are written only
// with FULL.
//
// One wave serves FCPW cells with FLPC lanes each (N = 5: 2 x 32), in the
// operator's traversal (one record gives neighbours and kind, so that all
// loads leave in one round trip after it).  Lane (d, side, p) takes column p of the face layer of beta, own or neighbour's,
// to the Gauss points of the second tangential direction, one LDS transpose,
// then the first; with the traces in LDS all lanes of the cell write its
// 21 N^2 values in memory order.  Memory bound (read 34, write 50 bytes per
// dof at degree 4 on general faces, 2 and 10 on compressed ones); the former
// kernel interpolated with N^2 work per point and lane: 0.355 ms at 64x32x32
// cells, degree 4, this one 0.14 ms.
// -------------------------------------------------------------------------
template <int N, bool FULL>
__global__ void __launch_bounds__(64)
k_set_face(int64_t n_cells, const int32_t *__restrict__ visit, const RefTab64 *__restrict__ T,
           const double *__restrict__ beta, const double *__restrict__ sigma,
           const double *__restrict__ facegeo, const uint8_t *__restrict__ ctype,
           double *__restrict__ face64, float *__restrict__ face32, double *__restrict__ aface64,
           float *__restrict__ aface32)
{
    constexpr int NF = SCfg<N>::NF, ND = SCfg<N>::ND, LPC = SCfg<N>::FLPC, CPW = SCfg<N>::FCPW;
    constexpr bool PT = face32_by_point(N);
    __shared__ double sT[CPW][6][NF], sV[CPW][6][NF];
    __shared__ float sF[CPW][3][7 * NF];   // FP32 data, put into their own order
    const int cs = threadIdx.x / LPC, ln = threadIdx.x % LPC;
    const int64_t slot = xcd_range() * CPW + cs;
    // the traversal record {cell, neighbours, mask}; bit 2 + 2 e of the mask:
    // the +e face lies between two affine cells
    const int32_t *rec = visit + (slot < n_cells ? slot : 0) * 8;
    const int32_t rc = rec[0];
    const bool valid = slot < n_cells && rc >= 0;
    const int64_t cid = valid ? rc : 0;
    const bool on = valid && ln < 6 * N;
    const int f = on ? ln / N : 0, p = ln % N, d = f >> 1, plus = f & 1;
    int32_t nb[3];
    bool cmp[3];
    const int32_t mask = rec[7];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        nb[e] = valid ? rec[2 + 2 * e] : -1;
        cmp[e] = valid && (mask >> (2 + 2 * e)) & 1;
    }
    if constexpr (FULL) {
        // (the records hold no masks while the compression is off)
#pragma unroll
        for (int e = 0; e < 3; ++e) cmp[e] = valid && ctype[cid] && nb[e] >= 0 && ctype[nb[e]];
    }
    const int32_t nbd = d == 0 ? nb[0] : (d == 1 ? nb[1] : nb[2]);
    const bool fl = on && nbd >= 0;
    // every load up front: the column of beta, then the geometric factors
    double h[N], y[N], sg[3];
    if (fl) {
        const int sd = d == 0 ? 1 : (d == 1 ? N : NF), sp = d == 0 ? N : 1, sr = d == 2 ? N : NF;
        const double *src = beta + (int64_t)(plus ? nbd : cid) * ND + (plus ? 0 : (N - 1) * sd) + p * sp;
#pragma unroll
        for (int r = 0; r < N; ++r) h[r] = src[r * sr];
    }
    constexpr int GPL = (7 * NF + LPC - 1) / LPC;
    double g[3][GPL];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        sg[e] = valid ? sigma[3 * cid + e] : 0.0;
        if (nb[e] >= 0 && (FULL || !cmp[e]))
#pragma unroll
            for (int k = 0; k < GPL; ++k)
                g[e][k] = __builtin_nontemporal_load(facegeo + (3 * cid + e) * 7 * NF +
                                                     (ln + k * LPC < 7 * NF ? ln + k * LPC : 0));
        else
#pragma unroll
            for (int k = 0; k < GPL; ++k) g[e][k] = 0.0;
    }
    auto interp = [&](const double (&w)[N], double (&z)[N]) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) s += KB<N>::d[q * N + i] * w[i];
            z[q] = s;
        }
    };
    if (fl) {
        interp(h, y);
#pragma unroll
        for (int q = 0; q < N; ++q) sT[cs][f][q * N + p] = y[q];
    }
    __syncthreads();
    if (on) {
        // lane (f, q2 = p): along the first tangential direction; point (a, b)
        // at b + N a (a boundary face's traces are zero)
#pragma unroll
        for (int i = 0; i < N; ++i) h[i] = fl ? sT[cs][f][p * N + i] : 0.0;
        interp(h, y);
#pragma unroll
        for (int q = 0; q < N; ++q) sV[cs][f][q * N + p] = y[q];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int64_t cd = 3 * cid + e;
        if (valid && (FULL || !cmp[e])) {
            double *dst = face64 + cd * 7 * NF;
#pragma unroll
            for (int u = 0; u < GPL; ++u) {
                const int k = ln + u * LPC;
                if (k >= 7 * NF) break;
                const int s = k / NF, pt = k - s * NF;
                const double bm = sV[cs][2 * e][pt], bp = sV[cs][2 * e + 1][pt];
                const double out = (s < 3 ? bm : (s < 6 ? bp : sg[e] * (bm + bp))) * g[e][u];
                dst[k] = out;
                sF[cs][e][PT ? 7 * pt + s : k] = (float)out;
            }
        }
        if (cmp[e]) {
            double *dst = aface64 + cd * 2 * NF;
            float *dstf = aface32 + cd * 2 * NF;
#pragma unroll
            for (int u = 0; u < (2 * NF + LPC - 1) / LPC; ++u) {
                const int k = ln + u * LPC;
                if (k >= 2 * NF) break;
                const int s = k / NF, pt = k - s * NF;
                dst[k] = sV[cs][2 * e + s][pt] * (T->wq[pt / N] * T->wq[pt % N]);
                const int pf = PT ? k >> 1 : pt, sf = PT ? k & 1 : s;
                dstf[k] = (float)(sV[cs][2 * e + sf][pf] * (T->wq[pf / N] * T->wq[pf % N]));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        if (!valid || (!FULL && cmp[e])) continue;
        float *dstf = face32 + (3 * cid + e) * 7 * NF;
#pragma unroll
        for (int u = 0; u < GPL; ++u) {
            const int k = ln + u * LPC;
            if (k < 7 * NF) dstf[k] = sF[cs][e][k];
        }
    }
}

// Constants of the +d face between two affine cells (thread per (cell, d)):
// v- = ds0 J-^-1 n, v+ = ds0 J+^-1 n and sd = sigma ds0 / 2 (ds = w ds0, w the
// face weight), from the general factors of the first face point.  They
// follow the mesh and the penalty, not the coefficients.
__global__ void k_face_const(int n, int64_t n_cells, const int32_t *__restrict__ nbr,
                             const RefTab64 *__restrict__ T, const double *__restrict__ sigma,
                             const double *__restrict__ facegeo, const uint8_t *__restrict__ ctype,
                             double *fc64, float *fc32)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= 3 * n_cells) return;
    const int64_t c = t / 3;
    const int32_t nb = nbr[6 * c + 2 * (int)(t % 3) + 1];
    if (nb < 0 || !ctype[c] || !ctype[nb]) return;
    const int nf = n * n;
    const double *g = facegeo + t * 7 * nf;
    const double w0 = T->wq[0] * T->wq[0];
    for (int k = 0; k < 8; ++k) {
        const double v = k < 6 ? g[k * nf] / w0 : (k == 6 ? sigma[t] * g[6 * nf] / w0 : 0.0);
        fc64[t * 8 + k] = v;
        fc32[t * 8 + k] = (float)v;
    }
}

// General values of the affine cells and of the faces between two of them,
// rebuilt from the compressed ones (m is always there): for a caller that
// turns the compression off or exports them.
__global__ void k_expand_cell(int64_t total, int nd, const uint8_t *__restrict__ ctype,
                              const double *__restrict__ acell, const double *__restrict__ kk,
                              double *cell64, float *cell32)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int64_t c = t / nd;
    const int q = (int)(t % nd);
    if (!ctype[c]) return;
    const double bw = acell[c * 2 * nd + nd + q];
    for (int s = 0; s < 6; ++s) {
        const double v = bw * kk[8 * c + s];
        cell64[(c * 7 + 1 + s) * nd + q] = v;
        cell32[(c * 7 + 1 + s) * nd + q] = (float)v;
    }
}

__global__ void k_expand_face(int64_t total, int nf, const int32_t *__restrict__ nbr,
                              const uint8_t *__restrict__ ctype, const double *__restrict__ aface,
                              const double *__restrict__ fc, bool by_point, double *face64,
                              float *face32)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int64_t cd = t / nf, c = cd / 3;
    const int pt = (int)(t % nf);
    const int32_t nb = nbr[6 * c + 2 * (int)(cd % 3) + 1];
    if (nb < 0 || !ctype[c] || !ctype[nb]) return;
    const double bm = aface[cd * 2 * nf + pt], bp = aface[cd * 2 * nf + nf + pt];
    for (int s = 0; s < 7; ++s) {
        const double v = s < 6 ? (s < 3 ? bm : bp) * fc[cd * 8 + s] : fc[cd * 8 + 6] * (bm + bp);
        face64[(cd * 7 + s) * nf + pt] = v;
        face32[by_point ? t * 7 + s : (cd * 7 + s) * nf + pt] = (float)v;
    }
}

// -------------------------------------------------------------------------
// dof coordinates (thread per dof)
// -------------------------------------------------------------------------
__global__ void k_dof_coords(const double *__restrict__ nodes, int ng, int n, int64_t n_dofs,
                             const RefTab64 *__restrict__ T, double *xyz)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n_dofs) return;
    const int nd = n * n * n;
    const int64_t c = t / nd;
    const int q = (int)(t % nd);
    double xi[3] = {T->xl[q % n], T->xl[(q / n) % n], T->xl[q / (n * n)]}, x[3], J[3][3];
    cell_map(nodes + c * (int64_t)ng * ng * ng * 3, ng, xi, x, J);
    xyz[t] = x[0];
    xyz[n_dofs + t] = x[1];
    xyz[2 * n_dofs + t] = x[2];
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_cell_geometry(hx_ctx *c)
{
    hipLaunchKernelGGL(k_cell_geometry, dim3(nblk(c->n_cells, 64)), dim3(64), 0, c->stream,
                       c->nodes, c->g + 1, c->n, c->n_cells, c->ref, c->vol, c->ell, c->mindet);
    return hipGetLastError();
}

hipError_t launch_face_sigma(hx_ctx *c)
{
    hipLaunchKernelGGL(k_face_sigma, dim3(nblk(3 * c->n_cells, 64)), dim3(64), 0, c->stream,
                       c->nodes, c->g + 1, c->n, c->n_cells, c->nbr, c->ref, c->vol, c->P,
                       c->sigma);
    return hipGetLastError();
}

template <int N>
static hipError_t bj_eigen_n(hx_ctx *c)
{
    hipLaunchKernelGGL(k_bj_eigen<N>, dim3(nblk(3 * c->n_cells, 64)), dim3(64), 0, c->stream,
                       c->n_cells, c->nbr, c->ref, c->ell, c->sigma, c->endsig, c->bjS64, c->bjS32,
                       c->bjL64, c->bjL32);
    return hipGetLastError();
}

hipError_t launch_bj_eigen(hx_ctx *c)
{
    switch (c->n) {
    case 2: return bj_eigen_n<2>(c);
    case 3: return bj_eigen_n<3>(c);
    case 4: return bj_eigen_n<4>(c);
    case 5: return bj_eigen_n<5>(c);
    case 6: return bj_eigen_n<6>(c);
    case 7: return bj_eigen_n<7>(c);
    case 8: return bj_eigen_n<8>(c);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_geofac(hx_ctx *c)
{
    hipLaunchKernelGGL(k_cell_geofac, dim3(nblk(c->n_cells * c->nd, 128)), dim3(128), 0, c->stream,
                       c->nodes, c->g + 1, c->n, c->n_cells, c->ref, c->cellgeo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nt = 3 * c->n_cells * c->nf;
    hipLaunchKernelGGL(k_face_geofac, dim3(nblk(nt, 128)), dim3(128), 0, c->stream, c->nodes,
                       c->g + 1, c->n, c->n_cells, c->nbr, c->ref, c->facegeo);
    return hipGetLastError();
}

hipError_t launch_affine_detect(hx_ctx *c)
{
    hipLaunchKernelGGL(k_affine_detect, dim3(nblk(c->n_cells, 128)), dim3(128), 0, c->stream, c->nodes,
                       c->g + 1, c->nd, c->n_cells, c->ref, c->cellgeo, c->ctype, c->kk64, c->kk32);
    return hipGetLastError();
}

hipError_t launch_face_const(hx_ctx *c)
{
    hipLaunchKernelGGL(k_face_const, dim3(nblk(3 * c->n_cells, 256)), dim3(256), 0, c->stream, c->n,
                       c->n_cells, c->nbr, c->ref, c->sigma, c->facegeo, c->ctype, c->fc64, c->fc32);
    return hipGetLastError();
}

hipError_t launch_expand_general(hx_ctx *c)
{
    const int64_t nt = c->n_dofs, nf = 3 * c->n_cells * c->nf;
    hipLaunchKernelGGL(k_expand_cell, dim3(nblk(nt, 256)), dim3(256), 0, c->stream, nt, c->nd, c->ctype,
                       c->acell64, c->kk64, c->cell64, c->cell32);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_expand_face, dim3(nblk(nf, 256)), dim3(256), 0, c->stream, nf, c->nf, c->nbr,
                       c->ctype, c->aface64, c->fc64, face32_by_point(c->n), c->face64, c->face32);
    return hipGetLastError();
}

template <int N, bool FULL>
static hipError_t set_coefficients_n(hx_ctx *c, const double *alpha, const double *beta)
{
    hipLaunchKernelGGL((k_set_cell<N, FULL>), dim3(nblk(c->n_cells, SCfg<N>::CPW)), dim3(64), 0, c->stream,
                       c->n_cells, alpha, beta, c->ell, c->cellgeo, c->ctype, c->kk64, c->cell64, c->cell32,
                       c->acell64, c->acell32, c->bjC64, c->bjC32, c->coef_feat, c->dg64, c->dg32);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_set_face<N, FULL>), dim3(nblk(c->n_vis_op, SCfg<N>::FCPW)), dim3(64), 0, c->stream,
                       c->n_vis_op, c->visit, c->ref, beta, c->sigma, c->facegeo, c->ctype, c->face64,
                       c->face32, c->aface64, c->aface32);
    return hipGetLastError();
}

template <bool FULL>
static hipError_t set_coefficients_all(hx_ctx *c, const double *alpha, const double *beta)
{
    switch (c->n) {
    case 2: return set_coefficients_n<2, FULL>(c, alpha, beta);
    case 3: return set_coefficients_n<3, FULL>(c, alpha, beta);
    case 4: return set_coefficients_n<4, FULL>(c, alpha, beta);
    case 5: return set_coefficients_n<5, FULL>(c, alpha, beta);
    case 6: return set_coefficients_n<6, FULL>(c, alpha, beta);
    case 7: return set_coefficients_n<7, FULL>(c, alpha, beta);
    case 8: return set_coefficients_n<8, FULL>(c, alpha, beta);
    default: return hipErrorInvalidValue;
    }
}

// with the compressed data in use the general values of affine cells and
// faces are not written (c->lean); hx_set_cell_compression(c, 0) and the
// export rebuild them when they are asked for
hipError_t launch_set_coefficients(hx_ctx *c, const double *alpha, const double *beta)
{
    c->lean = c->compress != 0;
    const hipError_t e = c->lean ? set_coefficients_all<false>(c, alpha, beta)
                                 : set_coefficients_all<true>(c, alpha, beta);
    if (e != hipSuccess || c->n_hang == 0) return e;
    return launch_hang_coefficients(c, beta);
}

hipError_t launch_dof_coords(hx_ctx *c, double *xyz)
{
    hipLaunchKernelGGL(k_dof_coords, dim3(nblk(c->n_dofs, 128)), dim3(128), 0, c->stream,
                       c->nodes, c->g + 1, c->n, c->n_dofs, c->ref, xyz);
    return hipGetLastError();
}

}  // namespace hx

namespace hx {
namespace {

// -------------------------------------------------------------------------
// Data of the pressure system of one IMEX stage (section 2: A U + B P = F,
// C U + D P = G).  At cell Gauss point q of cell c:
//   W[c][3d+e][q]  = w detJ (J^-1)_{de}   (so that (grad phi)_e = sum_d W ... / (w detJ))
//   WC[c][3d+e][q] = hr_q W[c][3d+e][q]   (hr = h rho formed at the nodes, interpolated)
//   mr[c][q] = rho_q w detJ,  md[c][q] = w detJ / (gamma - 1),  hr[c][q] = hr_q;
//   kc[c][3d+e] = detJ (J^-1)_{de}, kc[c][9] = detJ / (gamma - 1) at the first
//   point (the cell's constants when it is affine; rows of 16);
// at Gauss point (a, b) of the cell's own face f = 2d + s:
//   fn[c][f][e][a + N b] = ds n_e (outward),  fh[c][f][a + N b] = hr.
// -------------------------------------------------------------------------
__global__ void k_press_cell(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                             const RefTab64 *__restrict__ T, const double *__restrict__ rho,
                             const double *__restrict__ h, double inv_gm1, double *W, double *WC,
                             double *mr, double *md, double *hr, double *kc)
{
    const int nd = n * n * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n_cells * nd) return;
    const int64_t c = t / nd;
    const int q = (int)(t % nd);
    const int i = q % n, j = (q / n) % n, l = q / (n * n);
    double xi[3] = {T->xq[i], T->xq[j], T->xq[l]}, x[3], J[3][3], Ji[3][3];
    cell_map(nodes + c * (int64_t)ng * ng * ng * 3, ng, xi, x, J);
    const double det = det3(J);
    inv3(J, det, Ji);
    const double w = T->wq[i] * T->wq[j] * T->wq[l] * det;
    double rq = 0.0, hq = 0.0;
    const double *rc = rho + c * nd, *hc = h + c * nd;
    for (int l2 = 0; l2 < n; ++l2)
        for (int j2 = 0; j2 < n; ++j2) {
            const double byz = T->B[j * n + j2] * T->B[l * n + l2];
            for (int i2 = 0; i2 < n; ++i2) {
                const double wgt = T->B[i * n + i2] * byz;
                const int e = lidx(n, i2, j2, l2);
                rq += wgt * rc[e];
                hq += wgt * (hc[e] * rc[e]);
            }
        }
    for (int d = 0; d < 3; ++d)
        for (int e = 0; e < 3; ++e) {
            const double v = w * Ji[d][e];
            W[(c * 9 + 3 * d + e) * nd + q] = v;
            WC[(c * 9 + 3 * d + e) * nd + q] = hq * v;
        }
    mr[c * nd + q] = rq * w;
    md[c * nd + q] = w * inv_gm1;
    hr[c * nd + q] = hq;
    if (q == 0) {
        for (int d = 0; d < 3; ++d)
            for (int e = 0; e < 3; ++e) kc[c * 16 + 3 * d + e] = det * Ji[d][e];
        kc[c * 16 + 9] = det * inv_gm1;
    }
}

__global__ void k_press_face(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                             const RefTab64 *__restrict__ T, const double *__restrict__ rho,
                             const double *__restrict__ h, double *fn, double *fh)
{
    const int nf = n * n, nd = nf * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n_cells * 6 * nf) return;
    const int pt = (int)(t % nf);
    const int64_t cf = t / nf;
    const int64_t c = cf / 6;
    const int f = (int)(cf % 6), d = f >> 1, s = f & 1;
    const int a = pt % n, b = pt / n;
    double xi[3], x[3], J[3][3], Ji[3][3];
    face_xi(T, d, s, a, b, xi);
    cell_map(nodes + c * (int64_t)ng * ng * ng * 3, ng, xi, x, J);
    const double det = det3(J);
    inv3(J, det, Ji);
    // ds n = +-w_a w_b detJ J^-T e_d (row d of J^-1), outward
    const double sw = (s ? 1.0 : -1.0) * T->wq[a] * T->wq[b] * det;
    for (int e = 0; e < 3; ++e) fn[(cf * 3 + e) * nf + pt] = sw * Ji[d][e];
    // trace of hr: the face layer of GLL nodes interpolated to the point
    const int m = s ? n - 1 : 0;
    double hv = 0.0;
    for (int e2 = 0; e2 < n; ++e2)
        for (int e1 = 0; e1 < n; ++e1) {
            const int64_t e = c * nd + layer_idx(n, d, m, e1, e2);
            hv += T->B[a * n + e1] * T->B[b * n + e2] * (h[e] * rho[e]);
        }
    fh[cf * nf + pt] = hv;
}

}  // namespace

hipError_t launch_press_setup(hx_ctx *c, const double *rho, const double *h, double gamma)
{
    const int64_t nt = c->n_cells * c->nd;
    hipLaunchKernelGGL(k_press_cell, dim3(nblk(nt, 128)), dim3(128), 0, c->stream, c->nodes, c->g + 1,
                       c->n, c->n_cells, c->ref, rho, h, 1.0 / (gamma - 1.0), c->psW, c->psWC,
                       c->psMr, c->psMd, c->psHr, c->psK);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nf = c->n_cells * 6 * c->nf;
    hipLaunchKernelGGL(k_press_face, dim3(nblk(nf, 128)), dim3(128), 0, c->stream, c->nodes, c->g + 1,
                       c->n, c->n_cells, c->ref, rho, h, c->psFn, c->psFh);
    return hipGetLastError();
}

}  // namespace hx

namespace hx {
namespace {

// -------------------------------------------------------------------------
// Consistent integration (section 3.3: 2r+1 Gauss points per direction):
// the merged cell and face data of the operator at the nq-point rule, the
// same quantities as k_cell_geofac / k_set_cell and k_face_geofac /
// k_set_face, with alpha and beta interpolated from the nodes to the points.
// Cell point index qx + nq (qy + nq qz); face point b + nq a (a along t1).
// With the compression on (ctype given) an affine cell takes alpha w detJ and
// beta w detJ in the first two of its seven fields, and a face between two
// affine cells beta- w, beta+ w in its first two and the constants v- (3), v+
// (3), sigma ds0 / 2 (ds = w ds0, v = ds0 J^-1 n) at the start of the third.
// -------------------------------------------------------------------------
__global__ void k_q_cell(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                         const RefTabQ *__restrict__ Q, const double *__restrict__ alpha,
                         const double *__restrict__ beta, const uint8_t *__restrict__ ctype,
                         double *qcell)
{
    const int nq = Q->nq, nq3 = nq * nq * nq, nd = n * n * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n_cells * nq3) return;
    const int64_t c = t / nq3;
    const int q = (int)(t % nq3);
    const int i = q % nq, j = (q / nq) % nq, l = q / (nq * nq);
    double xi[3] = {Q->xq[i], Q->xq[j], Q->xq[l]}, x[3], J[3][3], Ji[3][3];
    cell_map(nodes + c * (int64_t)ng * ng * ng * 3, ng, xi, x, J);
    const double det = det3(J);
    inv3(J, det, Ji);
    const double w = Q->wq[i] * Q->wq[j] * Q->wq[l] * det;
    double aq = 0.0, bq = 0.0;
    const double *ac = alpha + c * nd, *bc = beta + c * nd;
    for (int l2 = 0; l2 < n; ++l2)
        for (int j2 = 0; j2 < n; ++j2) {
            const double byz = Q->B[j * n + j2] * Q->B[l * n + l2];
            for (int i2 = 0; i2 < n; ++i2) {
                const double wgt = Q->B[i * n + i2] * byz;
                const int e = lidx(n, i2, j2, l2);
                aq += wgt * ac[e];
                bq += wgt * bc[e];
            }
        }
    double *dst = qcell + c * 7 * nq3 + q;
    dst[0] = aq * w;
    if (ctype && ctype[c]) {
        dst[nq3] = bq * w;
        return;
    }
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
    for (int s = 0; s < 6; ++s) {
        const int A = pa[s], Bq = pb[s];
        dst[(1 + s) * nq3] =
            bq * w * (Ji[A][0] * Ji[Bq][0] + Ji[A][1] * Ji[Bq][1] + Ji[A][2] * Ji[Bq][2]);
    }
}

__global__ void k_q_face(const double *__restrict__ nodes, int ng, int n, int64_t n_cells,
                         const int32_t *__restrict__ nbr, const RefTabQ *__restrict__ Q,
                         const double *__restrict__ beta, const double *__restrict__ sigma,
                         const uint8_t *__restrict__ ctype, double *qface)
{
    const int nq = Q->nq, nq2 = nq * nq, nd = n * n * n;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= 3 * n_cells * nq2) return;
    const int pt = (int)(t % nq2);
    const int64_t cd = t / nq2;
    const int64_t c = cd / 3;
    const int d = (int)(cd % 3);
    const int a = pt / nq, b = pt % nq;
    double *dst = qface + cd * 7 * nq2 + pt;
    const int32_t nb = nbr[6 * c + 2 * d + 1];
    if (nb < 0) {
        for (int s = 0; s < 7; ++s) dst[s * nq2] = 0.0;
        return;
    }
    const int t1 = d == 0 ? 1 : 0, t2 = d == 2 ? 1 : 2;
    double xim[3], xip[3], x[3], Jm[3][3], Jp[3][3], Jmi[3][3], Jpi[3][3];
    xim[d] = 1.0;
    xip[d] = 0.0;
    xim[t1] = xip[t1] = Q->xq[a];
    xim[t2] = xip[t2] = Q->xq[b];
    const int64_t gsz = (int64_t)ng * ng * ng * 3;
    cell_map(nodes + c * gsz, ng, xim, x, Jm);
    cell_map(nodes + (int64_t)nb * gsz, ng, xip, x, Jp);
    const double detm = det3(Jm), detp = det3(Jp);
    inv3(Jm, detm, Jmi);
    inv3(Jp, detp, Jpi);
    double nv[3] = {Jmi[d][0], Jmi[d][1], Jmi[d][2]};
    const double len = sqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    for (int r = 0; r < 3; ++r) nv[r] /= len;
    const double ds = Q->wq[a] * Q->wq[b] * detm * len;
    // beta on both sides: the face layers interpolated to the point
    double bm = 0.0, bp = 0.0;
    for (int e2 = 0; e2 < n; ++e2)
        for (int e1 = 0; e1 < n; ++e1) {
            const double wgt = Q->B[a * n + e1] * Q->B[b * n + e2];
            bm += wgt * beta[c * nd + layer_idx(n, d, n - 1, e1, e2)];
            bp += wgt * beta[(int64_t)nb * nd + layer_idx(n, d, 0, e1, e2)];
        }
    const int dir[3] = {d, t1, t2};
    if (ctype && ctype[c] && ctype[nb]) {
        const double wab = Q->wq[a] * Q->wq[b];
        dst[0] = bm * wab;
        dst[nq2] = bp * wab;
        if (pt == 0) {
            double *fc = dst + 2 * nq2;
            const double ds0 = ds / wab;
            for (int k = 0; k < 3; ++k) {
                const int r = dir[k];
                fc[k] = ds0 * (Jmi[r][0] * nv[0] + Jmi[r][1] * nv[1] + Jmi[r][2] * nv[2]);
                fc[3 + k] = ds0 * (Jpi[r][0] * nv[0] + Jpi[r][1] * nv[1] + Jpi[r][2] * nv[2]);
            }
            fc[6] = sigma[3 * c + d] * 0.5 * ds0;
        }
        return;
    }
    for (int k = 0; k < 3; ++k) {
        const int r = dir[k];
        dst[k * nq2] = bm * ds * (Jmi[r][0] * nv[0] + Jmi[r][1] * nv[1] + Jmi[r][2] * nv[2]);
        dst[(3 + k) * nq2] = bp * ds * (Jpi[r][0] * nv[0] + Jpi[r][1] * nv[1] + Jpi[r][2] * nv[2]);
    }
    dst[6 * nq2] = sigma[3 * c + d] * 0.5 * (bm + bp) * ds;
}

}  // namespace

hipError_t launch_q_setup(hx_ctx *c, const double *alpha, const double *beta)
{
    const int nq = c->nq;
    c->q_lean = c->compress != 0;
    const uint8_t *ctype = c->q_lean ? c->ctype : nullptr;
    const int64_t nt = c->n_cells * nq * nq * nq;
    hipLaunchKernelGGL(k_q_cell, dim3(nblk(nt, 128)), dim3(128), 0, c->stream, c->nodes, c->g + 1, c->n,
                       c->n_cells, c->refq, alpha, beta, ctype, c->qcell);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nf = 3 * c->n_cells * nq * nq;
    hipLaunchKernelGGL(k_q_face, dim3(nblk(nf, 128)), dim3(128), 0, c->stream, c->nodes, c->g + 1, c->n,
                       c->n_cells, c->nbr, c->refq, beta, c->sigma, ctype, c->qface);
    return hipGetLastError();
}

}  // namespace hx
