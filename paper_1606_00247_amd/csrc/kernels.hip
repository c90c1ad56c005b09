// HIP kernels of the tetrahedral FMM for CDNA4 (gfx950), FP64.
//
//   p2m   multipole coefficients of a leaf (eq. expCoeffs) from the tets'
//         geometric moments (exact quadrature, once per plan) and affine M
//   m2m   binomial shift of child multipoles to the parent centre
//   m2l   multipole -> local translation of the Cartesian Taylor expansion on
//         the matrix cores, translations packed by key or target cells in tiles
//   l2l   binomial shift of a local expansion to the child centres
//   l2p   evaluation of the local expansion at the targets (adds into u)
//   p2p   exact near-field tet-to-target potential (Sec. 2.1), source-major:
//         one wavefront per 64 targets and block of up to 64 tets of a source
//         leaf, taken chunk by chunk, the tets' (one field: their shared nodes',
//         edges' and faces') data read through the scalar unit, atomically
//         accumulated into u
//
// Multi-indices |n| <= p are stored in graded order: degree ascending, within
// a degree n_x descending, then n_y descending.  idx(n) = d(d+1)(d+2)/6 +
// r(r+1)/2 + n_z with d = |n| and r = n_y + n_z.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <type_traits>
#include <vector>

#include "../../include/tetfmm.h"
#include "device.h"
#include "pair.h"

namespace tfmm {

// ---------------------------------------------------------------------------
// constant tables
// ---------------------------------------------------------------------------
constexpr int kPmax = TFMM_PMAX;
constexpr int kNcoefMax = (kPmax + 1) * (kPmax + 2) * (kPmax + 3) / 6;

struct MiTable {
    int8_t v[kNcoefMax][4];  // nx, ny, nz, |n|
};
constexpr MiTable make_mi()
{
    MiTable t{};
    int k = 0;
    for (int d = 0; d <= kPmax; ++d)
        for (int nx = d; nx >= 0; --nx)
            for (int ny = d - nx; ny >= 0; --ny) {
                t.v[k][0] = (int8_t)nx;
                t.v[k][1] = (int8_t)ny;
                t.v[k][2] = (int8_t)(d - nx - ny);
                t.v[k][3] = (int8_t)d;
                ++k;
            }
    return t;
}
struct BinomTable {
    double c[2 * kPmax + 1][2 * kPmax + 1];
    double invfact[2 * kPmax + 1];
};
constexpr BinomTable make_binom()
{
    BinomTable t{};
    for (int n = 0; n <= 2 * kPmax; ++n)
        for (int r = 0; r <= 2 * kPmax; ++r) t.c[n][r] = 0.0;
    for (int n = 0; n <= 2 * kPmax; ++n) {
        t.c[n][0] = 1.0;
        for (int r = 1; r <= n; ++r) t.c[n][r] = t.c[n - 1][r - 1] + (r <= n - 1 ? t.c[n - 1][r] : 0.0);
    }
    double f = 1.0;
    for (int n = 0; n <= 2 * kPmax; ++n) {
        if (n > 0) f *= n;
        t.invfact[n] = 1.0 / f;
    }
    return t;
}
__constant__ MiTable c_mi = make_mi();
// compile-time view of the same table (loops unrolled over a template order)
constexpr MiTable kMi = make_mi();
__host__ __device__ constexpr int mi_x(int m) { return kMi.v[m][0]; }
__host__ __device__ constexpr int mi_y(int m) { return kMi.v[m][1]; }
__host__ __device__ constexpr int mi_z(int m) { return kMi.v[m][2]; }

__host__ __device__ constexpr int mi_index(int nx, int ny, int nz)
{
    int d = nx + ny + nz, r = ny + nz;
    return d * (d + 1) * (d + 2) / 6 + r * (r + 1) / 2 + nz;
}
__host__ __device__ constexpr int ncoef_of(int p) { return (p + 1) * (p + 2) * (p + 3) / 6; }


// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  A grid of 8 * ceil(n/8) workgroups in x is remapped so that XCD x
// runs items [x * per, (x + 1) * per): neighbouring items (Morton order) share
// an L2.  Returns -1 for the padding workgroups.
constexpr int kXcds = 8;
__host__ __device__ constexpr unsigned xcd_grid(int n) { return (unsigned)(kXcds * ((n + kXcds - 1) / kXcds)); }
__device__ __forceinline__ int xcd_item(int n)
{
    const int w = blockIdx.x, per = (n + kXcds - 1) / kXcds;
    const int item = (w % kXcds) * per + w / kXcds;
    return item < n ? item : -1;
}

// Memory that no thread writes during the launch: uniform reads of it go to
// the scalar unit whatever the compiler can prove about aliasing.
template <typename T>
using ScalarMem = T __attribute__((address_space(4)));
template <typename T>
__device__ __forceinline__ const ScalarMem<T> *scalar_mem(const T *p)
{
    return (const ScalarMem<T> *)p;
}

// cell int fields
enum { CI_TBEG = 0, CI_TEND, CI_XBEG, CI_XEND, CI_CBEG, CI_NCHILD, CI_PARENT, CI_LEVEL, CI_N };

// ---------------------------------------------------------------------------
// fill
// ---------------------------------------------------------------------------
__global__ void k_fill(double *__restrict__ a, int64_t n, double v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) a[i] = v;
}

// ---------------------------------------------------------------------------
// P2M (eq. expCoeffs).  M is affine on a tet, M_k(y) = M_k(c) + sum_d G_kd
// (y_d - c_d) with G = dM/dy, so with the geometric moments of the tet about
// its leaf centre c,  S_m = int_T (y - c)^m dy  (|m| <= p),
//   Q_n = sum_k n_k int_T M_k(y) (y - c)^{n - e_k} dy
//       = sum_k n_k [ M_k(c) S_{n-e_k} + sum_d G_kd S_{n-e_k+e_d} ].
// S depends on the mesh only: k_tet_moments computes it once per plan with
// an exact collapsed Gauss-Jacobi rule (degree p); k_p2m streams it.
// ---------------------------------------------------------------------------
constexpr int kMomThreads = 256;
constexpr int kMomChunk = 256;

// One workgroup per leaf holding tets: S of each of its tets, [T][ncoef].
__global__ __launch_bounds__(kMomThreads) void k_tet_moments(const int32_t *__restrict__ cells,
                                                             const int32_t *__restrict__ cell_i,
                                                             const double *__restrict__ cell_c, int64_t C,
                                                             const double *__restrict__ tet_xyz, int64_t T,
                                                             const double *__restrict__ quad, int nq, int p,
                                                             int points, double *__restrict__ mom)
{
    __shared__ double s_pw[kMomChunk][3][kPmax + 1];  // powers 0..p of (y - c)
    __shared__ double s_w[kMomChunk];
    const int cell = cells[blockIdx.x];
    const int tbeg = cell_i[CI_N * cell + CI_TBEG], tend = cell_i[CI_N * cell + CI_TEND];
    const double cc[3] = {cell_c[cell], cell_c[C + cell], cell_c[2 * C + cell]};
    const int ncoef = ncoef_of(p);
    const int tid = threadIdx.x;
    if (points) {  // point sources: S_m = (y - c)^m at the point
        for (int i = tid; i < (tend - tbeg) * ncoef; i += kMomThreads) {
            const int t = tbeg + i / ncoef, m = i % ncoef;
            double r = 1.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double y = tet_xyz[(int64_t)k * T + t] - cc[k];
                for (int j = 0; j < c_mi.v[m][k]; ++j) r *= y;
            }
            mom[(int64_t)t * ncoef + m] = r;
        }
        return;
    }
    for (int t = tbeg; t < tend; ++t) {
        double v[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 3; ++k) v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + t];
        double e[3][3];
#pragma unroll
        for (int c = 1; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 3; ++k) e[c - 1][k] = v[c][k] - v[0][k];
        const double vol6 = fabs(e[0][0] * (e[1][1] * e[2][2] - e[1][2] * e[2][1]) -
                                 e[0][1] * (e[1][0] * e[2][2] - e[1][2] * e[2][0]) +
                                 e[0][2] * (e[1][0] * e[2][1] - e[1][1] * e[2][0]));
        double acc[2] = {0.0, 0.0};
        for (int base = 0; base < nq; base += kMomChunk) {
            __syncthreads();
            const int q = base + tid;
            if (q < nq) {
                const double l1 = quad[4 * q], l2 = quad[4 * q + 1], l3 = quad[4 * q + 2];
                const double l0 = 1.0 - (l1 + l2 + l3);
                s_w[tid] = quad[4 * q + 3] * vol6;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double y = ((l0 * (v[0][k] - cc[k]) + l1 * (v[1][k] - cc[k])) + l2 * (v[2][k] - cc[k])) +
                                     l3 * (v[3][k] - cc[k]);
                    double pw = 1.0;
                    for (int j = 0; j <= p; ++j) {
                        s_pw[tid][k][j] = pw;
                        pw *= y;
                    }
                }
            }
            __syncthreads();
            const int n = min(kMomChunk, nq - base);
            for (int r = 0; r < 2; ++r) {
                const int m = tid + r * kMomThreads;
                if (m >= ncoef) break;
                const int a = c_mi.v[m][0], b = c_mi.v[m][1], c = c_mi.v[m][2];
                double s = 0.0;
                for (int i = 0; i < n; ++i) s += s_w[i] * (s_pw[i][0][a] * s_pw[i][1][b] * s_pw[i][2][c]);
                acc[r] += s;
            }
        }
        for (int r = 0; r < 2; ++r) {
            const int m = tid + r * kMomThreads;
            if (m < ncoef) mom[(int64_t)t * ncoef + m] = acc[r];
        }
    }
}

// ---------------------------------------------------------------------------
// P2M.  One workgroup per leaf holding tets and FC fields (XCD-contiguous, the
// field chunks of a leaf next to each other).  With the per-tet moments
// S_m = int_T (y - c)^m (exact, once per plan) and, per field, the affine
// magnetisation M(y) = M(c) + G (y - c) of the tet,
//   Q_n = sum_T sum_k n_k [M_k(c) S_{n-e_k} + sum_d G_kd S_{n-e_k+e_d}]
//       = sum_k n_k [U_k,{n-e_k} + sum_d U_kd,{n-e_k+e_d}],
//   U_j,m = sum_T W_jT S_m,T   (j the 12 field values of a tet),
// a contraction over the leaf's tets on the FP64 matrix cores: A = W (rows
// field x 12 values), B = the moments, straight from memory in their operand
// layout (four rows of 128 consecutive bytes), columns dealt to the four
// wavefronts.  The shifts by e_k and e_d are taken once per leaf, on U in LDS.
// Bound: the moments' bytes (507 MB on the 40^3 cube, one field: 105 us at the
// rate of a large copy).  One field there 416 -> 239 us, on a film of 387k tets
// (17 a leaf) 1.23 -> 0.44 ms, 16 fields on a 26^3 cube 0.60 -> 0.29 ms, against
// one coefficient a thread with its 12 gathers a tet from LDS; the rest is the
// field values of a leaf, formed before its contraction can start.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int field_chunk(int F) { return F >= 3 ? 4 : 1; }
constexpr int kP2MThreads = 256;
constexpr int kP2MStage = 16;
// column tiles (16 coefficients) of each of the four wavefronts
__host__ __device__ constexpr int p2m_tiles(int p) { return ((ncoef_of(p) + 15) / 16 + 3) / 4; }

// M(c) [3] and G [3][3] of tet t for one field (nodal values Mf).
__device__ inline void tet_affine_field(const double *__restrict__ tet_xyz, const int32_t *__restrict__ tet_node,
                                        int64_t T, int64_t t, const double *__restrict__ Mf, const double c[3],
                                        double *__restrict__ out)
{
    double v[4][3], mm[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int nd = tet_node[(int64_t)q * T + t];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v[q][k] = tet_xyz[(int64_t)(3 * q + k) * T + t];
            mm[q][k] = Mf[3 * (int64_t)nd + k];
        }
    }
    double e1[3], e2[3], e3[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e1[k] = v[1][k] - v[0][k];
        e2[k] = v[2][k] - v[0][k];
        e3[k] = v[3][k] - v[0][k];
    }
    // gradients of the barycentric coordinates
    double g[4][3];
    g[1][0] = e2[1] * e3[2] - e2[2] * e3[1];
    g[1][1] = e2[2] * e3[0] - e2[0] * e3[2];
    g[1][2] = e2[0] * e3[1] - e2[1] * e3[0];
    g[2][0] = e3[1] * e1[2] - e3[2] * e1[1];
    g[2][1] = e3[2] * e1[0] - e3[0] * e1[2];
    g[2][2] = e3[0] * e1[1] - e3[1] * e1[0];
    g[3][0] = e1[1] * e2[2] - e1[2] * e2[1];
    g[3][1] = e1[2] * e2[0] - e1[0] * e2[2];
    g[3][2] = e1[0] * e2[1] - e1[1] * e2[0];
    const double idet = 1.0 / (e1[0] * g[1][0] + e1[1] * g[1][1] + e1[2] * g[1][2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        g[1][k] *= idet;
        g[2][k] *= idet;
        g[3][k] *= idet;
        g[0][k] = -(g[1][k] + g[2][k] + g[3][k]);
    }
    const double dc[3] = {c[0] - v[0][0], c[1] - v[0][1], c[2] - v[0][2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double G[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) G[b] = mm[0][a] * g[0][b] + mm[1][a] * g[1][b] + mm[2][a] * g[2][b] + mm[3][a] * g[3][b];
        out[a] = mm[0][a] + (G[0] * dc[0] + G[1] * dc[1] + G[2] * dc[2]);  // M_a(c)
        out[3 + 3 * a] = G[0];
        out[4 + 3 * a] = G[1];
        out[5 + 3 * a] = G[2];
    }
}

// Dynamic LDS: U [12][64 NT] doubles.
template <int FC, int NT>
__global__ __launch_bounds__(kP2MThreads, FC == 1 ? 4 : (NT <= 3 ? 3 : 2)) void k_p2m(const int32_t *__restrict__ cells, const int32_t *__restrict__ cell_i,
                                                     const double *__restrict__ cell_c, int64_t C,
                                                     const double *__restrict__ tet_xyz, const int32_t *__restrict__ tet_node,
                                                     int64_t T, const double *__restrict__ mom,
                                                     const double *__restrict__ M, int64_t n_nodes, int F, int p,
                                                     int ncells, int points, LevelOrders lo, double *__restrict__ Q)
{
    using v4 = double __attribute__((ext_vector_type(4)));
    constexpr int NROW = FC == 1 ? 16 : 12 * FC, NRT = NROW / 16;  // rows, row tiles
    extern __shared__ double s_U[];
    __shared__ double s_W[kP2MStage][NROW];
    const int ncoef = ncoef_of(p), nch = (F + FC - 1) / FC;
    const int item = xcd_item(ncells * nch);
    if (item < 0) return;
    const int cell = cells[item / nch], f0 = item % nch * FC;
    const int tbeg = cell_i[CI_N * cell + CI_TBEG], tend = cell_i[CI_N * cell + CI_TEND];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const double cc[3] = {cell_c[cell], cell_c[C + cell], cell_c[2 * C + cell]};
    v4 acc[NRT][NT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[rt][j] = v4{0, 0, 0, 0};
    for (int i = tid; i < kP2MStage * NROW; i += kP2MThreads) (&s_W[0][0])[i] = 0.0;
    for (int sb = tbeg; sb < tend; sb += kP2MStage) {
        const int nt = min(kP2MStage, tend - sb), nk = (nt + 3) >> 2;
        __syncthreads();
        for (int i = tid; i < 4 * nk * FC; i += kP2MThreads) {
            const int t = i / FC, j = i - t * FC;
            double *w = &s_W[t][12 * j];
            if (t >= nt || f0 + j >= F)
                for (int q = 0; q < 12; ++q) w[q] = 0.0;
            else if (points) {  // a dipole: M(c) = its moment, no gradient
                const double *m = M + ((int64_t)(f0 + j) * n_nodes + tet_node[sb + t]) * 3;
                for (int q = 0; q < 12; ++q) w[q] = q < 3 ? m[q] : 0.0;
            } else
                tet_affine_field(tet_xyz, tet_node, T, sb + t, M + (int64_t)(f0 + j) * n_nodes * 3, cc, w);
        }
        // moments of the first four tets, on their way during the field values
        auto moments = [&](double (&b)[NT], int ks) {
            const double *S = mom + (int64_t)(sb + min(4 * ks + kq, nt - 1)) * ncoef;
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = S[min(16 * (wave + 4 * j) + col, ncoef - 1)];
        };
        double b[2][NT];
        moments(b[0], 0);
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kP2MStage / 4; ++ks) {
            if (ks >= nk) break;
            if (ks + 1 < kP2MStage / 4) moments(b[(ks + 1) & 1], ks + 1);
            double a[NRT];
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) a[rt] = s_W[4 * ks + kq][16 * rt + col];
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int rt = 0; rt < NRT; ++rt)
                    acc[rt][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rt], b[ks & 1][j], acc[rt][j], 0, 0, 0);
        }
    }
    // kept to the order of the leaf's level (the rest stays zero)
    const int nkeep = ncoef_of(lo.q[cell_i[CI_N * cell + CI_LEVEL]]);
    // the terms of coefficient n: weights and places in U, found once for all fields
    double nv[3];
    int at[3][4];
    auto terms = [&](int n) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int b[3] = {c_mi.v[n][0], c_mi.v[n][1], c_mi.v[n][2]};
            const bool on = b[k] > 0 && n < nkeep;
            nv[k] = on ? (double)b[k] : 0.0;
            if (on) --b[k];
            const int row = 64 * NT;
            at[k][0] = k * row + (on ? mi_index(b[0], b[1], b[2]) : 0);
            at[k][1] = (3 + 3 * k) * row + (on ? mi_index(b[0] + 1, b[1], b[2]) : 0);
            at[k][2] = (4 + 3 * k) * row + (on ? mi_index(b[0], b[1] + 1, b[2]) : 0);
            at[k][3] = (5 + 3 * k) * row + (on ? mi_index(b[0], b[1], b[2] + 1) : 0);
        }
    };
    terms(min(tid, ncoef - 1));
#pragma unroll
    for (int f = 0; f < FC; ++f) {
        if (f0 + f >= F) break;
        __syncthreads();
#pragma unroll
        for (int g = 3 * f; g < 3 * f + 3; ++g)  // rows 4 g + kq: the field's values 4 (g - 3 f) + kq
#pragma unroll
            for (int j = 0; j < NT; ++j)
                s_U[(4 * (g - 3 * f) + kq) * 64 * NT + 16 * (wave + 4 * j) + col] = acc[g >> 2][j][g & 3];
        __syncthreads();
        for (int n = tid; n < ncoef; n += kP2MThreads) {
            if (n != tid) terms(n);  // only above order 9
            double q = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (nv[k] != 0.0) q += nv[k] * (s_U[at[k][0]] + s_U[at[k][1]] + s_U[at[k][2]] + s_U[at[k][3]]);
            Q[((int64_t)(f0 + f) * C + cell) * ncoef + n] = q;
        }
        if (ncoef > kP2MThreads) terms(tid);
    }
}

// ---------------------------------------------------------------------------
// M2M and L2L as three one-dimensional binomial shifts.  The shift by t of a
// multipole (k <= n) or local (k >= m, |k| <= p) expansion factorises over the
// axes, C(n, k) t^(n-k) = prod_i C(n_i, k_i) t_i^(n_i - k_i), so it is applied
// axis by axis.  A workgroup holds kShiftItems items (children), one field
// (blockIdx.y), the coefficients of an item in LDS as a (P+1)^3 cube; a thread
// takes one line of an item along the axis into registers (at most P + 1
// values) and shifts it by repeated multiply-adds with t alone, no table of
// coefficients.  Bound on large levels: the expansions' bytes; on the few
// cells of the upper levels the launch and the chain of three passes.
// 40^3 cube, p = 8, all levels, one field: M2M 195 -> 98 us, L2L 165 -> 104 us
// against one coefficient a lane with table look-ups and index arithmetic.
// ---------------------------------------------------------------------------
constexpr int kShiftItems = 8;
__host__ __device__ constexpr int shift_lines(int P) { return (P + 1) * (P + 2) / 2; }
__host__ __device__ constexpr int shift_threads(int P) { return (kShiftItems * shift_lines(P) + 63) / 64 * 64; }
// line (i, j), i + j <= P: i-major
struct LineTable {
    int8_t v[(kPmax + 1) * (kPmax + 2) / 2][2];
};
template <int P>
constexpr LineTable make_lines()
{
    LineTable t{};
    int k = 0;
    for (int i = 0; i <= P; ++i)
        for (int j = 0; i + j <= P; ++j) {
            t.v[k][0] = (int8_t)i;
            t.v[k][1] = (int8_t)j;
            ++k;
        }
    return t;
}
template <int P>
__constant__ LineTable c_line = make_lines<P>();

// place of coefficient n in an item's cube
template <int P>
__device__ __forceinline__ int cube_at(int n)
{
    return (c_mi.v[n][0] * (P + 1) + c_mi.v[n][1]) * (P + 1) + c_mi.v[n][2];
}

// shifts one line (values at s[i * step], i <= len) by t
template <int P, bool Up>
__device__ __forceinline__ void shift_line(double *s, int step, int len, double t)
{
    double c[P + 1];
#pragma unroll
    for (int i = 0; i <= P; ++i) c[i] = i <= len ? s[i * step] : 0.0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (Up) {  // out_a = sum_{k <= a} C(a, k) t^(a-k) in_k
#pragma unroll
            for (int j = P; j > i; --j) c[j] = fma(t, c[j - 1], c[j]);
        } else {  // out_m = sum_{k >= m} C(k, m) t^(k-m) in_k
#pragma unroll
            for (int j = P - 1; j >= i; --j) c[j] = fma(t, c[j + 1], c[j]);
        }
    }
#pragma unroll
    for (int i = 0; i <= P; ++i)
        if (i <= len) s[i * step] = c[i];
}
// the three axes of the workgroup's items (t: shift of each item)
template <int P, bool Up>
__device__ __forceinline__ void shift_items(double *s_c, const double (*t)[3], uint32_t live)
{
    constexpr int D = P + 1, D3 = D * D * D, NL = shift_lines(P);
    const int g = (int)threadIdx.x / NL, l = (int)threadIdx.x % NL;
    const bool on = g < kShiftItems && (live >> g & 1);
    const int a = c_line<P>.v[l][0], b = c_line<P>.v[l][1];
    double *s = s_c + (on ? g : 0) * D3;
    if (on) shift_line<P, Up>(s + a * D + b, D * D, P - a - b, t[g][0]);
    __syncthreads();
    if (on) shift_line<P, Up>(s + a * D * D + b, D, P - a - b, t[g][1]);
    __syncthreads();
    if (on) shift_line<P, Up>(s + a * D * D + b * D, 1, P - a - b, t[g][2]);
    __syncthreads();
}

// M2M: one workgroup per parent of a level; child g of the parent is item g.
//   Q_n(P) = sum_children sum_{k <= n} C(n,k) (c_C - c_P)^{n-k} Q_k(C)
template <int P>
__global__ __launch_bounds__(shift_threads(P)) void k_m2m(const int32_t *__restrict__ cells,
                                                          const int32_t *__restrict__ cell_i,
                                                          const double *__restrict__ cell_c, int64_t C, int pout,
                                                          double *__restrict__ Q)
{
    constexpr int NC = ncoef_of(P), D3 = (P + 1) * (P + 1) * (P + 1);
    __shared__ double s_c[kShiftItems * D3], s_t[kShiftItems][3];
    const int cell = cells[blockIdx.x], f = blockIdx.y;
    const int cbeg = cell_i[CI_N * cell + CI_CBEG], nch = min(cell_i[CI_N * cell + CI_NCHILD], kShiftItems);
    uint32_t live = 0;  // children holding tets
    for (int g = 0; g < nch; ++g)
        if (cell_i[CI_N * (cbeg + g) + CI_TEND] > cell_i[CI_N * (cbeg + g) + CI_TBEG]) live |= 1u << g;
    if ((int)threadIdx.x < 3 * nch) {
        const int g = threadIdx.x / 3, k = threadIdx.x % 3;
        s_t[g][k] = cell_c[k * C + cbeg + g] - cell_c[k * C + cell];
    }
    for (int i = threadIdx.x; i < nch * NC; i += blockDim.x) {
        const int g = i / NC, n = i - g * NC;
        if (live >> g & 1) s_c[g * D3 + cube_at<P>(n)] = Q[((int64_t)f * C + cbeg + g) * NC + n];
    }
    __syncthreads();
    shift_items<P, true>(s_c, s_t, live);
    const int nkeep = ncoef_of(pout);  // kept to the parent level's order
    for (int n = threadIdx.x; n < NC; n += blockDim.x) {
        const int at = cube_at<P>(n);
        double q = 0.0;
        for (int g = 0; g < nch; ++g)
            if (live >> g & 1) q += s_c[g * D3 + at];
        Q[((int64_t)f * C + cell) * NC + n] = n < nkeep ? q : 0.0;
    }
}

// L2L: items are kShiftItems consecutive child cells of a level (each with
// its own parent).
//   l_m(C) += sum_{k >= m, |k| <= p} C(k,m) (c_C - c_P)^{k-m} l_k(P)
template <int P>
__global__ __launch_bounds__(shift_threads(P)) void k_l2l(const int32_t *__restrict__ cells, int ncells,
                                                          const int32_t *__restrict__ cell_i,
                                                          const double *__restrict__ cell_c, int64_t C, int pout,
                                                          double *__restrict__ L)
{
    constexpr int NC = ncoef_of(P), D3 = (P + 1) * (P + 1) * (P + 1);
    __shared__ double s_c[kShiftItems * D3], s_t[kShiftItems][3];
    const int f = blockIdx.y, it = blockIdx.x * kShiftItems, n_it = min(ncells - it, kShiftItems);
    if ((int)threadIdx.x < 3 * n_it) {
        const int g = threadIdx.x / 3, k = threadIdx.x % 3, cell = cells[it + g];
        s_t[g][k] = cell_c[k * C + cell] - cell_c[k * C + cell_i[CI_N * cell + CI_PARENT]];
    }
    for (int i = threadIdx.x; i < n_it * NC; i += blockDim.x) {
        const int g = i / NC, n = i - g * NC;
        s_c[g * D3 + cube_at<P>(n)] = L[((int64_t)f * C + cell_i[CI_N * cells[it + g] + CI_PARENT]) * NC + n];
    }
    __syncthreads();
    shift_items<P, false>(s_c, s_t, (1u << n_it) - 1u);
    const int nkeep = ncoef_of(pout);
    for (int i = threadIdx.x; i < n_it * NC; i += blockDim.x) {
        const int g = i / NC, n = i - g * NC;
        if (n < nkeep) L[((int64_t)f * C + cells[it + g]) * NC + n] += s_c[g * D3 + cube_at<P>(n)];
    }
}

constexpr int kM2LWaves = 4;


// The two matrix-core shapes used by M2L: 16x16x4 with FP64 or FP32 operands.
// A (16 x 4): lane l holds row l%16, column l/16; B (4 x 16): lane l holds
// row l/16, column l%16.  The 16x16 result: lane l, register r holds
// column l%16 and row (l/16) + 4r (FP64) or 4(l/16) + r (FP32).
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    using v4 = double __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(double a, double b, v4 c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct Mfma<float> {
    using v4 = float __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(float a, float b, v4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// ---------------------------------------------------------------------------
// Harmonic reduction of the translation.  D_k = d^k (1/|R|) is harmonic, so
// D_{k + 2e_z} = -D_{k + 2e_x} - D_{k + 2e_y}: every term of the contraction
// sum_n D_{n+m} Qt_n with n_z >= 2 folds, degree by degree, onto the n_z <= 1
// terms (Qr = reduced multipoles), and every output with m_z >= 2 follows from
// the m_z <= 1 outputs of the same degree.  Both keep |n| and |m|, so the
// truncation |n| + |m| <= p is unchanged and the result is the same
// contraction up to rounding, with (p+1)^2 instead of ncoef(p) indices per
// side (81 vs 165 at p = 8).
//
// Reduced indices (z <= 1), degree d block at d^2:
//   ridx(x, y, 0) = d^2 + y,   ridx(x, y, 1) = d^2 + d + 1 + y.
// Derivative table per key, entries with k_z <= 2 only, degree d block at
//   sd(d) = 0 (d = 0), 1 + 3 d (d - 1) / 2:  didx = sd(d) + {0, d + 1, 2d + 1}[k_z] + k_y.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int nr_of(int p) { return (p + 1) * (p + 1); }
__host__ __device__ constexpr int nd_of(int p) { return 1 + 3 * p * (p + 1) / 2; }
__host__ __device__ constexpr int rdeg(int j)
{
    int d = 0;
    while ((d + 1) * (d + 1) <= j) ++d;
    return d;
}
__host__ __device__ constexpr int ridx(int x, int y, int z)
{
    const int d = x + y + z;
    return d * d + z * (d + 1) + y;
}
__host__ __device__ constexpr int didx_of(int x, int y, int z)
{
    const int d = x + y + z;
    return (d == 0 ? 0 : 1 + 3 * d * (d - 1) / 2) + (z == 0 ? 0 : (z == 1 ? d + 1 : 2 * d + 1)) + y;
}
constexpr int kNrMax = (kPmax + 1) * (kPmax + 1);
constexpr int kNdMax = 1 + 3 * kPmax * (kPmax + 1) / 2;
struct RedTable {
    int8_t r[kNrMax][4];  // reduced index -> x, y, z, d
    int8_t d[kNdMax][4];  // table index -> x, y, z, d
};
constexpr RedTable make_red()
{
    RedTable t{};
    for (int d = 0; d <= kPmax; ++d)
        for (int z = 0; z <= 2; ++z)
            for (int y = 0; y + z <= d; ++y) {
                const int x = d - y - z;
                if (z <= 1) {
                    const int j = ridx(x, y, z);
                    t.r[j][0] = (int8_t)x, t.r[j][1] = (int8_t)y, t.r[j][2] = (int8_t)z, t.r[j][3] = (int8_t)d;
                }
                const int k = didx_of(x, y, z);
                t.d[k][0] = (int8_t)x, t.d[k][1] = (int8_t)y, t.d[k][2] = (int8_t)z, t.d[k][3] = (int8_t)d;
            }
    return t;
}
__constant__ RedTable c_red = make_red();

// MFMA tiling of the reduced contraction: rows m = reduced indices of degree
// <= p - 1 (degree p rows only meet n = 0, and Q_0 = 0), in tiles of 16;
// columns n = 1 .. nr(p) - 1 in steps of 4; row tile rt only needs columns
// of degree <= p - |m_min(rt)|.
__host__ __device__ constexpr int m2l_nrows(int P) { return P * P; }
__host__ __device__ constexpr int m2l_nrt(int P) { return (m2l_nrows(P) + 15) / 16; }
__host__ __device__ constexpr int m2l_ks(int P, int rt)
{
    const int d = rdeg(16 * rt);
    if (d >= P) return 0;
    return (nr_of(P - d) - 1 + 3) / 4;
}
// Rows of the tile form's multipoles: row length at order p, and the place of
// column n >= 1 (step ks = (n - 1) / 4, quarter (n - 1) % 4), grouped by the
// wavefront that takes the step and the quarter of it that loads the column.
__host__ __device__ constexpr int m2l_tile_row(int p) { return 16 * ((m2l_ks(p, 0) + kM2LWaves - 1) / kM2LWaves); }
__host__ __device__ constexpr int m2l_tile_col(int i, int row)  // column at place i
{
    const int g = i / (row / 16), j = i % (row / 16);
    return 1 + 4 * (g / 4 + kM2LWaves * j) + g % 4;
}
// Column steps of wave W: ks = W, W + kM2LWaves, ... of every row tile.
__host__ __device__ constexpr int m2l_wave_steps(int P, int W)
{
    int s = 0;
    for (int rt = 0; rt < m2l_nrt(P); ++rt) {
        const int KS = m2l_ks(P, rt);
        if (KS > W) s += (KS - W + kM2LWaves - 1) / kM2LWaves;
    }
    return s;
}
template <int P, int W>
using M2LIdx = int[m2l_wave_steps(P, W) > 0 ? m2l_wave_steps(P, W) : 1];

// Derivative tables: one thread per key, 2^(dl (|k| + 1)) D_k(rho) for
// |k| <= p, k_z <= 2, with D_k by
//   |k| r^2 D_k = -(2|k| - 1) sum_i k_i rho_i D_{k-e_i} - (|k| - 1) sum_i k_i (k_i - 1) D_{k-2e_i}
// (every term on the right has k_z no larger than k's).
__global__ void k_m2l_table(const int32_t *__restrict__ keys, int nkeys, int p, double *__restrict__ D)
{
    const int key = blockIdx.x * blockDim.x + threadIdx.x;
    if (key >= nkeys) return;
    const int nd = nd_of(p);
    const int dl = keys[4 * key];
    const double unit = dl >= 0 ? 0.5 : ldexp(0.5, dl);  // rho = k * unit
    const double Rx = keys[4 * key + 1] * unit, Ry = keys[4 * key + 2] * unit, Rz = keys[4 * key + 3] * unit;
    const double r2 = (Rx * Rx + Ry * Ry) + Rz * Rz;
    double *row = D + (int64_t)key * nd;
    row[0] = 1.0 / sqrt(r2);
    for (int k = 1; k < nd; ++k) {
        const int kx = c_red.d[k][0], ky = c_red.d[k][1], kz = c_red.d[k][2], d = c_red.d[k][3];
        double s1 = 0.0, s2 = 0.0;
        if (kx > 0) s1 += kx * Rx * row[didx_of(kx - 1, ky, kz)];
        if (ky > 0) s1 += ky * Ry * row[didx_of(kx, ky - 1, kz)];
        if (kz > 0) s1 += kz * Rz * row[didx_of(kx, ky, kz - 1)];
        if (kx > 1) s2 += kx * (kx - 1) * row[didx_of(kx - 2, ky, kz)];
        if (ky > 1) s2 += ky * (ky - 1) * row[didx_of(kx, ky - 2, kz)];
        if (kz > 1) s2 += kz * (kz - 1) * row[didx_of(kx, ky, kz - 2)];
        row[k] = -((2.0 * d - 1.0) * s1 + (d - 1.0) * s2) / (d * r2);
    }
    // level-difference factor 2^(dl (|k| + 1)) (exact)
    for (int k = 0; k < nd; ++k) row[k] = ldexp(row[k], dl * (c_red.d[k][3] + 1));
}

__global__ void k_to_float(const double *__restrict__ a, int64_t n, float *__restrict__ b)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) b[i] = (float)a[i];
}

// Reduced scaled multipoles of the cells holding tets, for reduced indices
// n = (a, b, c), c <= 1:
//   Qr_n = (-1)^|n| s_B^-|n| sum_{j >= 0} (-1)^j sum_{i <= j} C(j, i) Q_n'/n'!,
//   n' = (a - 2i, b - 2(j - i), c + 2j),
// and back: Lt_m of the reduced locals (see k_m2l_mfma) times 1 / (4 pi m!).
// Both as lists of terms (coefficient, weight) per output, made at compile time.
constexpr int kReduceTerms = 1024, kExpandTerms = 704;
struct ReduceTable {
    int16_t start[kNrMax + 1], at[kReduceTerms];
    double w[kReduceTerms];
};
constexpr ReduceTable make_reduce()
{
    constexpr BinomTable bin = make_binom();
    constexpr RedTable red = make_red();
    ReduceTable t{};
    int k = 0;
    for (int n = 0; n < kNrMax; ++n) {
        const int a = red.r[n][0], b = red.r[n][1], c = red.r[n][2], d = red.r[n][3];
        t.start[n] = (int16_t)k;
        for (int j = 0; c + 2 * j <= d; ++j)
            for (int i = 0; i <= j; ++i) {
                const int x = a - 2 * i, y = b - 2 * (j - i), z = c + 2 * j;
                if (x < 0 || y < 0) continue;
                t.at[k] = (int16_t)mi_index(x, y, z);
                t.w[k++] = (j & 1 ? -1.0 : 1.0) * bin.c[j][i] * bin.invfact[x] * bin.invfact[y] * bin.invfact[z];
            }
    }
    t.start[kNrMax] = (int16_t)k;
    return t;
}
constexpr int kNcMax = ncoef_of(kPmax);
struct ExpandTable {
    int16_t start[kNcMax + 1], at[kExpandTerms];
    double w[kExpandTerms];
};
constexpr ExpandTable make_expand()
{
    constexpr BinomTable bin = make_binom();
    ExpandTable t{};
    int k = 0;
    for (int m = 0; m < kNcMax; ++m) {
        const int x = kMi.v[m][0], y = kMi.v[m][1], z = kMi.v[m][2], j = z / 2;
        t.start[m] = (int16_t)k;
        for (int i = 0; i <= j; ++i) {
            t.at[k] = (int16_t)ridx(x + 2 * i, y + 2 * (j - i), z % 2);
            t.w[k++] = (j & 1 ? -1.0 : 1.0) * bin.c[j][i] * kInv4Pi * bin.invfact[x] * bin.invfact[y] * bin.invfact[z];
        }
    }
    t.start[kNcMax] = (int16_t)k;
    return t;
}
__constant__ ReduceTable c_reduce = make_reduce();
__constant__ ExpandTable c_expand = make_expand();

// A workgroup takes up to kRowCells consecutive cells of a field (fewer on small
// meshes, for 1024 workgroups): their coefficients and the terms go to LDS in whole
// lines.  Bound by its bytes (37,449 cells, order
// 8, in us: 95 with a thread per output walking the multi-indices in global
// memory, now 30; the locals 57, now 24).
constexpr int kRowCells = 16;
__host__ __device__ constexpr size_t row_lds(int nin, int nterm, int nout)
{
    return sizeof(double) * (size_t)(kRowCells * (nin + kPmax + 1) + nterm) + sizeof(int16_t) * (size_t)(nterm + nout + 1);
}
inline int row_cells(int64_t C, int32_t F)
{
    return (int)std::min<int64_t>(kRowCells, std::max<int64_t>(1, C * F / 1024));
}
struct RowLds {
    double *in, *scale, *w;
    int16_t *at, *start;
    __device__ RowLds(double *s, int nin, int nterm)
        : in(s), scale(in + kRowCells * nin), w(scale + kRowCells * (kPmax + 1)), at((int16_t *)(w + nterm)),
          start(at + nterm)
    {
    }
    // sum of output n of cell c
    __device__ double sum(int c, int nin, int n) const
    {
        double v = 0.0;
        for (int k = start[n]; k < start[n + 1]; ++k) v = fma(w[k], in[c * nin + at[k]], v);
        return v;
    }
};

__device__ __forceinline__ void bf16_split3(float x, __bf16 &x0, __bf16 &x1, __bf16 &x2)
{
    x0 = (__bf16)x;
    const float r1 = x - (float)x0;
    x1 = (__bf16)r1;
    x2 = (__bf16)(r1 - (float)x1);
}

// Row forms of the reduced multipoles, each the operand order of one form of M2L:
// by n, len a cell and field (packed form); by wavefront of the tile form, field
// of a group of fpt and place (m2l_tile_col), len = m2l_tile_row; and split in np
// BF16 parts by column step, part, field of a group and n, len = 32 steps.
enum { ROW_PLAIN, ROW_TILE, ROW_BF16 };

// (Lr: the accumulators of M2L, lrs a cell, cleared here)
template <int kForm, typename T>
__global__ __launch_bounds__(256) void k_qreduce(const double *__restrict__ Q, const int32_t *__restrict__ cell_i,
                                                 int64_t C, double side, int p, int len, int fpt, int np,
                                                 T *__restrict__ Qr, double *__restrict__ Lr, int lrs, int cells)
{
    extern __shared__ double s_row[];
    const int ncoef = ncoef_of(p), nr = nr_of(p), nterm = c_reduce.start[nr], tid = threadIdx.x, f = blockIdx.y;
    const RowLds S(s_row, ncoef, nterm);
    const int64_t c0 = (int64_t)blockIdx.x * cells;
    const int n_c = (int)min<int64_t>(cells, C - c0);
    const double *q = Q + ((int64_t)f * C + c0) * ncoef;
    for (int i = tid; i < n_c * ncoef; i += 256) S.in[i] = q[i];
    for (int i = tid; i < nterm; i += 256) {
        S.w[i] = c_reduce.w[i];
        S.at[i] = c_reduce.at[i];
    }
    for (int i = tid; i <= nr; i += 256) S.start[i] = c_reduce.start[i];
    if (tid < n_c) {  // (-1 / s)^d, zero for a cell without tets
        const int32_t *ci = cell_i + CI_N * (c0 + tid);
        const double is = -1.0 / ldexp(side, -ci[CI_LEVEL]);
        double sp = ci[CI_TEND] > ci[CI_TBEG] ? 1.0 : 0.0;
        for (int d = 0; d <= p; ++d, sp *= is) S.scale[tid * (kPmax + 1) + d] = sp;
    }
    __syncthreads();
    const int64_t cell = (int64_t)(f / fpt) * C + c0;  // first cell, in the rows of f's group
    for (int i = tid; i < n_c * len; i += 256) {
        const int c = i / len, at = i - c * len;
        const int n = kForm == ROW_TILE ? m2l_tile_col(at, len) : (kForm == ROW_BF16 ? at + 1 : at);
        double v = 0.0;
        if (n < nr) {
            const double sp = S.scale[c * (kPmax + 1) + (int)sqrtf((float)n)];  // degree: exact, d starts at d^2
            if (sp != 0.0) v = sp * S.sum(c, ncoef, n);
        }
        if constexpr (kForm == ROW_PLAIN) {
            Qr[((int64_t)f * C + c0) * len + i] = (T)v;
        } else if constexpr (kForm == ROW_TILE) {
            const int part = len / kM2LWaves;
            Qr[(((cell + c) * kM2LWaves + at / part) * fpt + f % fpt) * part + at % part] = (T)v;
        } else {
            T x[3];
            bf16_split3((float)v, x[0], x[1], x[2]);
            T *o = Qr + (((cell + c) * (len / 32) + at / 32) * np * fpt + f % fpt) * 32 + at % 32;
            for (int k = 0; k < np; ++k) o[(int64_t)k * fpt * 32] = x[k];
        }
    }
    for (int i = tid; i < n_c * lrs; i += 256) Lr[((int64_t)f * C + c0) * lrs + i] = 0.0;
}

// Steps of wave W in issue order: column step ks = W, W + 4, ... (outer),
// row tiles rt with ks < KS(rt) (inner), so consecutive MFMAs of a wave feed
// different accumulators; row tile 0 (the longest) rotates over 2 of its own.
// m2l_wave_index gives this lane's D-table index of the A-operand element of
// every step (the zero slot ND outside |n| + |m| <= P).
template <int P, int W>
__device__ __forceinline__ void m2l_wave_index(int lane, M2LIdx<P, W> &didx)
{
    constexpr int NR = nr_of(P), NROW = m2l_nrows(P), ND = nd_of(P), NRT = m2l_nrt(P), KS0 = m2l_ks(P, 0);
    int s = 0;
#pragma unroll
    for (int ks = W; ks < KS0; ks += kM2LWaves) {
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
            if (ks < m2l_ks(P, rt)) {
                const int m = 16 * rt + (lane & 15), n = 1 + 4 * ks + (lane >> 4);
                int di = ND;  // the zero slot of the staged D row
                if (m < NROW && n < NR && c_red.r[m][3] + c_red.r[n][3] <= P)
                    di = didx_of(c_red.r[m][0] + c_red.r[n][0], c_red.r[m][1] + c_red.r[n][1],
                                 c_red.r[m][2] + c_red.r[n][2]);
                didx[s++] = di;
            }
        }
    }
}

// Geometry of a tile: TPT target cells x FPT fields = 16 MFMA columns,
// column c = t * FPT + g (target slot t, field f0 + g).
struct M2LCols {
    int tpt, fpt, f0, F;
    int dstr;  // row stride of the derivative tables (the plan's order; P may be lower)
};

// Column steps of wavefront W (see k_m2l_mfma): KJ of them, ks = W + kM2LWaves j,
// whose multipoles lie together in a row of Qr (m2l_tile_col).  The wavefronts
// share nothing until their sums meet: each gathers its A operands from its own
// copy of the key's derivative row in LDS and loads its B operands in place, two
// entries ahead, in one of two register sets.  (With operands staged for all four
// by all four, a barrier per entry, the matrix cores were busy 38% of the time;
// F = 16, order 8, 1.4 million translations: 1.53 ms of M2L, now 1.06
// with rows in whole lines.)
template <typename T, int P, int W>
__device__ __forceinline__ void m2l_tile(const int32_t *__restrict__ tile_rng, const int32_t *__restrict__ ent_key,
                                         const int32_t *__restrict__ ent_src, const int32_t *__restrict__ keys,
                                         const T *__restrict__ Dtab, const T *__restrict__ Qr, int qrow, int64_t C,
                                         M2LCols cols, int tile, T *D, typename Mfma<T>::v4 (&acc)[m2l_nrt(P)])
{
    using v4 = typename Mfma<T>::v4;
    constexpr int ND = nd_of(P), NRT = m2l_nrt(P), KS0 = m2l_ks(P, 0);
    constexpr int KJ = (KS0 - W + kM2LWaves - 1) / kM2LWaves, DREG = (ND + 63) / 64;
    if constexpr (KJ > 0) {
        const int lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4;
        const int tslot = col / cols.fpt, field = cols.f0 + col % cols.fpt;
        M2LIdx<P, W> didx;
        m2l_wave_index<P, W>(lane, didx);
        constexpr int NS = m2l_wave_steps(P, W);
        v4 acc0[2] = {v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
        const int e0 = tile_rng[2 * tile], e1 = tile_rng[2 * tile + 1];
        if (e0 >= e1) return;
        const bool active = field < cols.F;
        const int part = qrow / kM2LWaves;
        const T *qf = Qr + (((int64_t)(cols.f0 / cols.fpt) * C * kM2LWaves + W) * cols.fpt + col % cols.fpt) * part +
                      kq * (part / 4);
        const int64_t stride = (int64_t)qrow * cols.fpt;  // a cell and field group
        auto source = [&](int e) { return ent_src[(int64_t)min(e, e1 - 1) * cols.tpt + tslot]; };
        auto key_of = [&](int e) { return ent_key[min(e, e1 - 1)]; };
        // Loads go to in-bounds addresses unconditionally and are masked when used.
        struct Ops {
            T q[KJ], d[DREG];
            int dl;
            bool ok;
        };
        auto load = [&](Ops &o, int src, int key) {
            o.ok = active && src >= 0;
            const T *q = qf + max(src, 0) * stride;
#pragma unroll
            for (int j = 0; j < KJ; ++j) o.q[j] = q[j];
#pragma unroll
            for (int j = 0; j < DREG; ++j) o.d[j] = Dtab[(int64_t)key * cols.dstr + min(lane + 64 * j, ND - 1)];
            o.dl = keys[4 * key];
        };
        auto stage = [&](const Ops &o) {  // a wavefront's LDS operations keep their order
#pragma unroll
            for (int j = 0; j < DREG; ++j)
                if (lane + 64 * j < ND) D[lane + 64 * j] = o.d[j];
        };
        Ops oa, ob;
        load(oa, source(e0), key_of(e0));
        load(ob, source(e0 + 1), key_of(e0 + 1));
        int src2 = source(e0 + 2), src3 = source(e0 + 3), key2 = key_of(e0 + 2), key3 = key_of(e0 + 3);
        stage(oa);
        auto step = [&](Ops &cur, const Ops &nxt, int e) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            T a[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) a[s] = D[didx[s]];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (e + 1 < e1) stage(nxt);
            if (cur.dl != 0) {  // uniform over the wavefront; 2^(-dl |n|), exact
#pragma unroll
                for (int j = 0; j < KJ; ++j) {
                    const int deg = (int)sqrtf((float)(1 + 4 * (W + kM2LWaves * j) + kq));  // exact: degree d starts at d^2
                    cur.q[j] = ldexp(cur.q[j], -cur.dl * deg);
                }
            }
            int s = 0;
#pragma unroll
            for (int j = 0; j < KJ; ++j) {
                const int ks = W + kM2LWaves * j;
                const T b = cur.ok ? cur.q[j] : (T)0;
#pragma unroll
                for (int rt = 0; rt < NRT; ++rt)
                    if (ks < m2l_ks(P, rt)) {
                        if (rt == 0)
                            acc0[j & 1] = Mfma<T>::mma(a[s++], b, acc0[j & 1]);
                        else
                            acc[rt] = Mfma<T>::mma(a[s++], b, acc[rt]);
                    }
            }
            load(cur, src2, key2);
            src2 = src3;
            key2 = key3;
            src3 = source(e + 4);
            key3 = key_of(e + 4);
        };
        for (int e = e0; e < e1; e += 2) {
            step(oa, ob, e);
            if (e + 1 < e1) step(ob, oa, e + 1);
        }
        acc[0] += acc0[0] + acc0[1];
    }
}

// ---------------------------------------------------------------------------
// M2L on matrix cores.
//
// With cell sides s and the scaled multipoles
//   Qt_n(B) = (-1)^|n| Q_n(B) / (n! s_B^|n|),
// and rho = (c_A - c_B) / s_B, dl = level(B) - level(A), the translation is
//   l_m(A) = 1 / (4 pi m! s_A^(|m|+1)) * Lt_m(A),
//   Lt_m(A) = sum_B 2^(dl (|m|+1)) sum_{|n|>=1, |n|+|m|<=p} D_{n+m}(rho) Qt_n(B),
// D_k = d^k (1/|rho|) depending only on the key (dl, rho): one table row per
// distinct key serves every level, and all magnitudes are O(1) (the FP32 form
// needs no other scaling).  The level factor splits exactly as
// 2^(dl (|n|+|m|+1)) * 2^(-dl |n|): the first is in the key's table, the
// second is applied to the multipoles as they are used.  The contraction runs on the harmonic reduction
// (reduced multipoles Qr, outputs Lr with m_z <= 1); the epilogue expands Lr
// to all m by
//   Lt_(x, y, c + 2j) = (-1)^j sum_{i <= j} C(j, i) Lr_(x + 2i, y + 2(j - i), c).
// A tile (16 MFMA columns: TPT target cells of one level x FPT fields) runs
// through the keys its cells use; per key the source multipoles form the B
// operand (columns without that key are zero), the Hankel matrix
// H[m][n] = D_{n+m} the A operand, and the 16x16x4 MFMA accumulates Lr for
// all columns in registers.  Four wavefronts split the column steps; their
// partial sums meet in LDS.
// ---------------------------------------------------------------------------
template <typename T, int P>
__global__ __launch_bounds__(64 * kM2LWaves, sizeof(T) == 4 ? 4 : 2) void k_m2l_mfma(
    const int32_t *__restrict__ tile_tgt, const int32_t *__restrict__ tile_rng, const int32_t *__restrict__ ent_key,
    const int32_t *__restrict__ ent_src, const int32_t *__restrict__ keys, const T *__restrict__ Dtab,
    const T *__restrict__ Qr, int qrow, int64_t C, int tpt, int fpt, int F, int ntiles, int dstr,
    double *__restrict__ Lr, int lrs)
{
    using v4 = typename Mfma<T>::v4;
    constexpr int NROW = m2l_nrows(P), ND = nd_of(P), NRT = m2l_nrt(P), RSTR = NROW | 1;
    static_assert(kM2LWaves == 4, "wave specialisation below");
    __shared__ T s_D[kM2LWaves][ND + 1];
    __shared__ double red[16 * RSTR];  // the waves' sums: red[c][m], c = column
    const int tile = blockIdx.x;
    if (tile >= ntiles) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const M2LCols cols{tpt, fpt, (int)blockIdx.y * fpt, F, dstr};
    for (int i = tid; i < 16 * RSTR; i += blockDim.x) red[i] = 0.0;
    T *D = s_D[wave];
    if ((tid & 63) == 0) D[ND] = (T)0;  // the zero slot
    v4 acc[NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) acc[rt] = v4{0, 0, 0, 0};
    switch (wave) {
    case 0: m2l_tile<T, P, 0>(tile_rng, ent_key, ent_src, keys, Dtab, Qr, qrow, C, cols, tile, D, acc); break;
    case 1: m2l_tile<T, P, 1>(tile_rng, ent_key, ent_src, keys, Dtab, Qr, qrow, C, cols, tile, D, acc); break;
    case 2: m2l_tile<T, P, 2>(tile_rng, ent_key, ent_src, keys, Dtab, Qr, qrow, C, cols, tile, D, acc); break;
    default: m2l_tile<T, P, 3>(tile_rng, ent_key, ent_src, keys, Dtab, Qr, qrow, C, cols, tile, D, acc); break;
    }
    // sum the waves' partial accumulators in LDS (FP64)
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * rt + Mfma<T>::row(lane, r);
            if (m < NROW) atomicAdd(&red[(lane & 15) * RSTR + m], (double)acc[rt][r]);
        }
    __syncthreads();
    for (int i = tid; i < 16 * NROW; i += blockDim.x) {
        const int c = i / NROW, m = i - c * NROW, field = cols.f0 + c % fpt;
        const int A = tile_tgt[tile * tpt + c / fpt];
        if (A >= 0 && field < F) atomicAdd(&Lr[((int64_t)field * C + A) * lrs + m], red[c * RSTR + m]);
    }
}

// ---------------------------------------------------------------------------
// M2L packed by key (FP64, fewer than 16 fields).
//
// The contraction is that of k_m2l_mfma (scaled, harmonically reduced
// multipoles; Hankel operand H[m][n] = D_{n+m} of the key; outputs Lr with
// m_z <= 1), but the 16 matrix-core columns of a step are 16 / fpt
// translations of one key x fpt fields, taken from a block of up to
// nb = slots / fpt target cells: every column carries a translation except
// in the last group of each key.  The reduced locals of the block's
// (cell, field) slots are summed in LDS (FP64) and added to Lr once per
// work item; k_lr_expand then expands Lr to all m and adds it to L.
//
// Each wavefront takes a contiguous run of the item's groups (consecutive
// groups mostly share the key).  The key's derivative row is staged in the
// wavefront's own LDS row when the key changes.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int m2l_all_steps(int P)
{
    int s = 0;
    for (int rt = 0; rt < m2l_nrt(P); ++rt) s += m2l_ks(P, rt);
    return s;
}
// One workgroup a CU, with a block of m2l_pack_slots(P) accumulator slots (target
// cell x field) in its LDS: the larger block fills the matrix-core columns better
// (40^3 cube: 0.91 with 256 slots, 0.85 with 128).  Two wavefronts a SIMD keep a
// whole group's multipoles in registers; three spill (2.34 against 2.16 ms).
constexpr int kM2LPWaves = 8;

// Column steps of the packed form.  A step contracts four columns n, one for
// each quarter kq of the wavefront; row tile rt takes the first m2l_ks(P, rt)
// steps, so within a run of steps that the same row tiles take (a segment) the
// columns may be dealt freely: quarter kq takes consecutive ones, and a lane
// loads its column's multipoles two at a time (a load of a wavefront touches the
// lines of 16 sources, whatever its width: 2.50 ms with one at a time, 2.34 with
// two; 40^3 cube, three wavefronts a SIMD).
__host__ __device__ constexpr int m2lp_seg_end(int P, int ks)  // end of the segment of step ks
{
    int e = m2l_ks(P, 0);
    for (int rt = 1; rt < m2l_nrt(P); ++rt)
        if (m2l_ks(P, rt) > ks && m2l_ks(P, rt) < e) e = m2l_ks(P, rt);
    return e;
}
__host__ __device__ constexpr int m2lp_seg_begin(int P, int ks)
{
    int b = 0;
    for (int rt = 0; rt < m2l_nrt(P); ++rt)
        if (m2l_ks(P, rt) <= ks && m2l_ks(P, rt) > b) b = m2l_ks(P, rt);
    return b;
}
// n = m2lp_col0 + m2lp_len * kq
__host__ __device__ constexpr int m2lp_len(int P, int ks) { return m2lp_seg_end(P, ks) - m2lp_seg_begin(P, ks); }
__host__ __device__ constexpr int m2lp_col0(int P, int ks) { return 1 + 3 * m2lp_seg_begin(P, ks) + ks; }
// whether step ks is loaded together with the step before it
__host__ __device__ constexpr bool m2lp_second(int P, int ks) { return (ks - m2lp_seg_begin(P, ks)) % 2 == 1; }
// whether step ks + 1 is loaded together with step ks
__host__ __device__ constexpr bool m2lp_first(int P, int ks) { return !m2lp_second(P, ks) && ks + 1 < m2lp_seg_end(P, ks); }

template <int P>
__global__ __launch_bounds__(64 * kM2LPWaves, 2) void k_m2l_pack(
    const int32_t *__restrict__ item, int nitems, const int32_t *__restrict__ blk_cells, int nb, int tpg,
    const int32_t *__restrict__ grp_key, const int32_t *__restrict__ grp_src, const uint8_t *__restrict__ grp_slot,
    const int32_t *__restrict__ keys, const double *__restrict__ Dtab, int dstr, const double *__restrict__ Qr, int qpad,
    int64_t C, int fpt, int F, double *__restrict__ Lr, int lrs)
{
    using v4 = Mfma<double>::v4;
    constexpr int NW = kM2LPWaves;
    constexpr int NR = nr_of(P), ND = nd_of(P), NROW = m2l_nrows(P), NRT = m2l_nrt(P), KS0 = m2l_ks(P, 0);
    constexpr int NS = m2l_all_steps(P), NSLOT = m2l_pack_slots(P), DSTR = ND + 1;
    constexpr bool kKeep = NS <= 32;
    // odd row stride of the accumulators: the 16 columns of an output
    // register (the same row of 16 slots) fall in 16 different bank pairs
    // when their slots differ mod 16, as the packer arranges
    constexpr int LSTR = NROW | 1;
    __shared__ double s_L[NSLOT * LSTR];
    __shared__ double s_D[NW][DSTR];
    const int it = blockIdx.x;
    if (it >= nitems) return;
    // the wavefront index made visibly uniform: the group bounds, keys and
    // the key-change branch then live in scalar registers
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4, pair = col / fpt, fsub = col % fpt, field = (int)blockIdx.y * fpt + fsub;
    const bool fok = field < F;
    for (int i = tid; i < NSLOT * LSTR; i += blockDim.x) s_L[i] = 0.0;
    double *D = s_D[w];
    if (lane == 0) D[ND] = 0.0;  // the zero slot
    // this lane's place in the derivative row of the A operand of every step
    // (ks-major, row tiles inner; the zero slot outside |n| + |m| <= P)
    const double *ap[NS];
    {
        int s = 0;
#pragma unroll
        for (int ks = 0; ks < KS0; ++ks) {
            const int n = m2lp_col0(P, ks) + m2lp_len(P, ks) * kq;
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
                if (ks < m2l_ks(P, rt)) {
                    const int m = 16 * rt + col;
                    int di = ND;
                    if (m < NROW && n < NR && c_red.r[m][3] + c_red.r[n][3] <= P)
                        di = didx_of(c_red.r[m][0] + c_red.r[n][0], c_red.r[m][1] + c_red.r[n][1],
                                     c_red.r[m][2] + c_red.r[n][2]);
                    ap[s++] = D + di;
                }
        }
    }
    __syncthreads();
    const int blk = item[3 * it], g0 = item[3 * it + 1], g1 = item[3 * it + 2];
    const int wg0 = g0 + (int)((int64_t)(g1 - g0) * w / NW), wg1 = g0 + (int)((int64_t)(g1 - g0) * (w + 1) / NW);
    const double *qf = Qr + (int64_t)(fok ? field : 0) * C * qpad;
    constexpr int DREG = (ND + 63) / 64;
    // Software pipeline, in one register set: the sources of group g + 2 are
    // on their way while group g runs, and the multipoles of group g + 1 are
    // loaded into the registers of group g as its matrix steps are issued.
    // Loads go to in-bounds addresses unconditionally (a row of Qr holds
    // qpad > 4 KS0 entries) and are masked when used.
    if (wg0 < wg1) {
        auto source = [&](int g) { return grp_src[(int64_t)min(g, wg1 - 1) * tpg + pair]; };
        auto place = [&](int g) { return (int)grp_slot[(int64_t)min(g, wg1 - 1) * tpg + pair]; };
        // multipoles of step ks, or of steps ks - 1 and ks once both are used
        auto load = [&](double (&b)[KS0], const double *q, int ks) {
            using two = double __attribute__((ext_vector_type(2), aligned(8)));
            if (m2lp_first(P, ks)) return;
            if (m2lp_second(P, ks)) {
                const two v = *reinterpret_cast<const two *>(q + m2lp_col0(P, ks - 1) + m2lp_len(P, ks) * kq);
                b[ks - 1] = v.x;
                b[ks] = v.y;
            } else {
                b[ks] = q[m2lp_col0(P, ks) + m2lp_len(P, ks) * kq];
            }
        };
        double b[KS0], d[DREG];
        int src = source(wg0), slot = place(wg0), src1 = source(wg0 + 1), slot1 = place(wg0 + 1);
        {
            const double *q = qf + (int64_t)(fok && src >= 0 ? src : 0) * qpad;
#pragma unroll
            for (int ks = 0; ks < KS0; ++ks) load(b, q, ks);
        }
        int key = grp_key[wg0], dl = keys[4 * key];
        auto row = [&](int k) {
#pragma unroll
            for (int j = 0; j < DREG; ++j) d[j] = Dtab[(int64_t)k * dstr + min(lane + 64 * j, ND - 1)];
        };
        auto stage = [&]() {  // a wavefront's LDS operations keep their order
#pragma unroll
            for (int j = 0; j < DREG; ++j)
                if (lane + 64 * j < ND) D[lane + 64 * j] = d[j];
        };
        row(key);
        stage();
        // A operand, gathered at each change of key where it fits in registers
        // (to order 8; with a gather per group the LDS bounds: 40^3 cube, items of 256 groups, 2.09 and 1.99 ms)
        double a[kKeep ? NS : 1];
        auto gather = [&]() {
            if constexpr (kKeep) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int s = 0; s < NS; ++s) a[s] = *ap[s];
            }
        };
        gather();
        for (int g = wg0; g < wg1; ++g) {
            const bool ok = fok && src >= 0;
            const int src2 = source(g + 2), slot2 = place(g + 2);
            const int next = grp_key[min(g + 1, wg1 - 1)];
            if (next != key) row(next);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // B operand: the multipoles times 2^(-dl |n|) (exact).  Columns of
            // empty slots and rows n >= NR hold finite values that meet zero A
            // entries or are never added out, so they need no masking.
            if (dl != 0) {  // uniform over the wavefront
#pragma unroll
                for (int ks = 0; ks < KS0; ++ks) {
                    const int n = m2lp_col0(P, ks) + m2lp_len(P, ks) * kq;
                    const int deg = (int)sqrtf((float)n);  // exact: degree d starts at d^2
                    b[ks] = ldexp(b[ks], -dl * deg);
                }
            }
            const double *q = qf + (int64_t)(fok && src1 >= 0 ? src1 : 0) * qpad;
            v4 acc[NRT], acc0[2] = {v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) acc[rt] = v4{0, 0, 0, 0};
            int s = 0;
#pragma unroll
            for (int ks = 0; ks < KS0; ++ks) {
#pragma unroll
                for (int rt = 0; rt < NRT; ++rt)
                    if (ks < m2l_ks(P, rt)) {
                        double as;
                        if constexpr (kKeep)
                            as = a[s];
                        else
                            as = *ap[s];
                        ++s;
                        if (rt == 0)
                            acc0[ks & 1] = Mfma<double>::mma(as, b[ks], acc0[ks & 1]);
                        else
                            acc[rt] = Mfma<double>::mma(as, b[ks], acc[rt]);
                    }
                load(b, q, ks);
            }
            acc[0] = acc0[0] + acc0[1];
            if (next != key) {
                key = next;
                dl = keys[4 * key];
                stage();
                gather();
            }
            if (ok) {
                double *Ls = s_L + (slot * fpt + fsub) * LSTR;
#pragma unroll
                for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int m = 16 * rt + Mfma<double>::row(lane, r);
                        if (m < NROW) atomicAdd(&Ls[m], acc[rt][r]);
                    }
            }
            src = src1;
            slot = slot1;
            src1 = src2;
            slot1 = slot2;
        }
    }
    __syncthreads();
    // add the block's reduced locals to Lr
    for (int i = tid; i < NSLOT * NROW; i += blockDim.x) {
        const int c = i / NROW, m = i - c * NROW;
        const double v = s_L[c * LSTR + m];
        if (v == 0.0) continue;
        const int fld = (int)blockIdx.y * fpt + c % fpt, cell = c / fpt < nb ? blk_cells[(int64_t)blk * nb + c / fpt] : -1;
        if (cell >= 0 && fld < F) atomicAdd(&Lr[((int64_t)fld * C + cell) * lrs + m], v);
    }
}

// L_m(A) = Lt_m(A) / (4 pi m! s_A^(|m|+1)), Lt expanded from the reduced
// locals Lr (see k_m2l_mfma), for |m| < the order of A's level, 0 above.
__global__ __launch_bounds__(256) void k_lr_expand(const double *__restrict__ Lr, int lrs,
                                                   const int32_t *__restrict__ cell_i, double side, int64_t C, int p,
                                                   LevelOrders lo, int cells, double *__restrict__ L)
{
    extern __shared__ double s_row[];
    // outputs below order p only: their reduced locals are the lrs = p^2 of a row
    const int ncoef = ncoef_of(p), nm = ncoef_of(p - 1), nterm = c_expand.start[nm], tid = threadIdx.x, f = blockIdx.y;
    const RowLds S(s_row, lrs, nterm);
    const int64_t c0 = (int64_t)blockIdx.x * cells;
    const int n_c = (int)min<int64_t>(cells, C - c0);
    const double *r = Lr + ((int64_t)f * C + c0) * lrs;
    for (int i = tid; i < n_c * lrs; i += 256) S.in[i] = r[i];
    for (int i = tid; i < nterm; i += 256) {
        S.w[i] = c_expand.w[i];
        S.at[i] = c_expand.at[i];
    }
    for (int i = tid; i <= nm; i += 256) S.start[i] = c_expand.start[i];
    if (tid < n_c) {
        const int lev = cell_i[CI_N * (c0 + tid) + CI_LEVEL];
        const double is = 1.0 / ldexp(side, -lev);
        double sp = is;
        for (int d = 0; d <= p; ++d, sp *= is) S.scale[tid * (kPmax + 1) + d] = d < lo.q[lev] ? sp : 0.0;
    }
    __syncthreads();
    double *out = L + ((int64_t)f * C + c0) * ncoef;
    for (int i = tid; i < n_c * ncoef; i += 256) {
        const int c = i / ncoef, m = i - c * ncoef;
        double v = 0.0;
        if (m < nm) {
            const double sp = S.scale[c * (kPmax + 1) + c_mi.v[m][3]];
            if (sp != 0.0) v = sp * S.sum(c, lrs, m);
        }
        out[i] = v;
    }
}

// ---------------------------------------------------------------------------
// M2L with split BF16 operands on matrix cores (v_mfma_f32_16x16x32_bf16).
//
// The FP32 operands of the FP32 form (derivative rows and reduced multipoles,
// all O(1) by the level scaling) are split,
// x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)
// (each difference exact in FP32), and the product is formed from the part
// products of total order < NP: NP = 2 takes a0 b0 + a0 b1 + a1 b0 (BF16x3),
// NP = 3 adds a1 b1 + a0 b2 + a2 b0 (BF16x6), accumulated in FP32.
// Operand layout: A (16 x 32): lane l holds row l%16, columns 8(l/16) + i;
// B (32 x 16): lane l holds rows 8(l/16) + i, column l%16; result as the
// FP32 16x16x4 form (row 4(l/16) + r, column l%16).
// Column steps are 32 wide (n = 1 + 32 ks + ...).  The sums of a row tile are kept
// in two accumulators, of the even and of the odd (step, row tile) pairs, which
// meet in FP64.
//
// One wavefront per tile of 16 columns: the derivative parts of a key are gathered
// from the wavefront's copy in LDS, the multipoles come split and in operand order
// from k_qreduce, straight into the registers of the entry before as its matrix
// steps consume them.  (With two
// wavefronts splitting and staging both operands for one group, the LDS was busy
// 64% of the time and the matrix cores 10%: 64 fields, order 8, 1.1 million
// translations, BF16x3: 6.3 ms of M2L, now 2.41.)  Bound by the multipoles: 42% of
// the lines read, 12.6 GB, come from beyond the L2, at 6.4 TB/s; the matrix cores are
// busy 0.26 of the time, the vector unit 0.53.  Two field groups a wavefront, with
// half the gathers, keep twice as many multipoles in use at a time and take 2.64 ms.
// ---------------------------------------------------------------------------
using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));

__host__ __device__ constexpr int m2lb_ks(int P, int rt)
{
    const int d = rdeg(16 * rt);
    if (d >= P) return 0;
    return (nr_of(P - d) - 1 + 31) / 32;
}
__host__ __device__ constexpr int m2lb_steps(int P)
{
    int s = 0;
    for (int rt = 0; rt < m2l_nrt(P); ++rt) s += m2lb_ks(P, rt);
    return s;
}

template <int P, int NP>
__global__ __launch_bounds__(64, P <= 8 ? 3 : 2) void k_m2l_bf16(
    const int32_t *__restrict__ tile_tgt, const int32_t *__restrict__ tile_rng, const int32_t *__restrict__ ent_key,
    const int32_t *__restrict__ ent_src, const int32_t *__restrict__ keys, const float *__restrict__ Dtab, int dstr,
    const __bf16 *__restrict__ Qb, int ksp, int64_t C, int tpt, int fpt, int F, int ntiles,
    double *__restrict__ Lr, int lrs)
{
    using v4 = Mfma<float>::v4;
    using u4 = uint32_t __attribute__((ext_vector_type(4)));
    constexpr int NR = nr_of(P), NROW = m2l_nrows(P), ND = nd_of(P), NRT = m2l_nrt(P), KS = m2lb_ks(P, 0);
    constexpr int NS = m2lb_steps(P), DW = NP == 3 ? 2 : 1, RSTR = NROW | 1, DREG = (ND + 63) / 64;
    __shared__ uint32_t s_D[(ND + 1) * DW];  // parts 0 and 1 of an entry in a word, part 2 in the next
    __shared__ double red[16 * RSTR];
    const int tile = blockIdx.x;
    if (tile >= ntiles) return;
    const int lane = threadIdx.x, col = lane & 15, kq = lane >> 4, tslot = col / fpt, fsub = col % fpt;
    const int e0 = tile_rng[2 * tile], e1 = tile_rng[2 * tile + 1];
    if (e0 >= e1) return;
    const int fg = (int)blockIdx.y;            // field group
    if (lane < DW) s_D[ND * DW + lane] = 0;    // the zero slot
    // byte offsets in s_D of this lane's A operand elements, two to a register (the zero slot outside |n| + |m| <= P)
    uint32_t at[NS][4];
    {
        int s = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
                if (ks < m2lb_ks(P, rt)) {
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        uint32_t o = 0;
#pragma unroll
                        for (int i = 2 * h; i < 2 * h + 2; ++i) {
                            const int m = 16 * rt + col, n = 1 + 32 * ks + 8 * kq + i;
                            int di = ND;
                            if (m < NROW && n < NR && c_red.r[m][3] + c_red.r[n][3] <= P)
                                di = didx_of(c_red.r[m][0] + c_red.r[n][0], c_red.r[m][1] + c_red.r[n][1],
                                             c_red.r[m][2] + c_red.r[n][2]);
                            o |= (uint32_t)(di * DW * 4) << (16 * (i & 1));
                        }
                        at[s][h] = o;
                    }
                    ++s;
                }
    }
    const int64_t row = (int64_t)ksp * NP * fpt * 32;  // a cell and field group
    const __bf16 *qb = Qb + (int64_t)fg * C * row + fsub * 32 + kq * 8;
    auto source = [&](int e) { return ent_src[(int64_t)min(e, e1 - 1) * tpt + tslot]; };
    auto key_of = [&](int e) { return ent_key[min(e, e1 - 1)]; };
    bf16x8 b[KS][NP];
    auto load = [&](int src, int ks) {  // in-bounds unconditionally, masked when used
        const __bf16 *q = qb + (int64_t)max(src, 0) * row + ks * NP * fpt * 32;
#pragma unroll
        for (int k = 0; k < NP; ++k) b[ks][k] = *reinterpret_cast<const bf16x8 *>(q + k * fpt * 32);
    };
    float d[DREG];
    auto fetch_row = [&](int key) {
#pragma unroll
        for (int j = 0; j < DREG; ++j) d[j] = Dtab[(int64_t)key * dstr + min(lane + 64 * j, ND - 1)];
    };
    auto stage = [&]() {  // a wavefront's LDS operations keep their order
#pragma unroll
        for (int j = 0; j < DREG; ++j) {
            __bf16 x[3];
            bf16_split3(d[j], x[0], x[1], x[2]);
            const uint32_t lo = __builtin_bit_cast(uint16_t, x[0]) | (uint32_t)__builtin_bit_cast(uint16_t, x[1]) << 16;
            if (lane + 64 * j < ND) {
                s_D[(lane + 64 * j) * DW] = lo;
                if constexpr (NP == 3) s_D[(lane + 64 * j) * DW + 1] = __builtin_bit_cast(uint16_t, x[2]);
            }
        }
    };
    v4 acc[2][NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) acc[0][rt] = acc[1][rt] = v4{0, 0, 0, 0};
    int src = source(e0), src1 = source(e0 + 1), key = key_of(e0), key1 = key_of(e0 + 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) load(src, ks);
    fetch_row(key);
    stage();
    for (int e = e0; e < e1; ++e) {
        const int src2 = source(e + 2), key2 = key_of(e + 2), dl = keys[4 * key];
        fetch_row(key1);
        if (tpt > 1) {  // columns without a source
            const uint32_t keep = src >= 0 ? 0xffffffffu : 0u;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int k = 0; k < NP; ++k) b[ks][k] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u4, b[ks][k]) & keep);
        }
        if (dl != 0) {  // uniform; 2^(-dl |n|), exact
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int deg = (int)sqrtf((float)(1 + 32 * ks + 8 * kq + i));  // exact: degree d starts at d^2
#pragma unroll
                    for (int k = 0; k < NP; ++k) b[ks][k][i] = (__bf16)ldexpf((float)b[ks][k][i], -dl * deg);
                }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int s = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
                if (ks < m2lb_ks(P, rt)) {
                    uint32_t w[8], w2[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t *p = (const uint32_t *)((const char *)s_D + (i & 1 ? at[s][i / 2] >> 16 : at[s][i / 2] & 0xffffu));
                        w[i] = p[0];
                        if constexpr (NP == 3) w2[i] = p[1];
                    }
                    bf16x8 a[NP];
                    u4 q0, q1, q2;
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        q0[h] = __builtin_amdgcn_perm(w[2 * h + 1], w[2 * h], 0x05040100u);
                        q1[h] = __builtin_amdgcn_perm(w[2 * h + 1], w[2 * h], 0x07060302u);
                        if constexpr (NP == 3) q2[h] = w2[2 * h] | w2[2 * h + 1] << 16;
                    }
                    a[0] = __builtin_bit_cast(bf16x8, q0);
                    a[1] = __builtin_bit_cast(bf16x8, q1);
                    if constexpr (NP == 3) a[2] = __builtin_bit_cast(bf16x8, q2);
                    auto mma = [&](int i, int k) {
                        acc[s & 1][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[ks][k], acc[s & 1][rt], 0, 0, 0);
                    };
                    // smallest terms first
                    if constexpr (NP == 3) {
                        mma(2, 0);
                        mma(0, 2);
                        mma(1, 1);
                    }
                    mma(1, 0);
                    mma(0, 1);
                    mma(0, 0);
                    ++s;
                }
            load(src1, ks);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        stage();
        src = src1;
        src1 = src2;
        key = key1;
        key1 = key2;
    }
    // the sums, through LDS in whole rows, to Lr
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * rt + Mfma<float>::row(lane, r);
            if (m < NROW) red[col * RSTR + m] = (double)acc[0][rt][r] + (double)acc[1][rt][r];
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < 16 * NROW; i += 64) {
        const int c = i / NROW, m = i - c * NROW, field = fg * fpt + c % fpt;
        const int A = tile_tgt[tile * tpt + c / fpt];
        if (A >= 0 && field < F) atomicAdd(&Lr[((int64_t)field * C + A) * lrs + m], red[c * RSTR + m]);
    }
}

// Place in u of target i of the octree's order; perm null: u is kept in that order.
__device__ __forceinline__ int64_t place(const int32_t *perm, int64_t i) { return perm ? perm[i] : i; }

// u[f][perm[i]] = v[f][i], one thread per target, fields in blockIdx.y.
__global__ __launch_bounds__(256) void k_scatter(const double *__restrict__ v, const int32_t *__restrict__ perm, int64_t N,
                                                 double *__restrict__ u)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, f = blockIdx.y;
    if (i < N) u[f * N + perm[i]] = v[f * N + i];
}

// ---------------------------------------------------------------------------
// L2P.  One thread per target (octree order) and field (blockIdx.y); adds
// into u[f][perm[i]].
//   u(x) = sum_m l_m (x - c)^m
// The order is a template parameter, so the loop over m unrolls and every
// monomial is a product of three powers held in registers.
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_l2p(const double *__restrict__ tgt_xyz, const int32_t *__restrict__ tgt_perm,
                                             const int32_t *__restrict__ tgt_leaf, int64_t N,
                                             const double *__restrict__ cell_c, int64_t C,
                                             const double *__restrict__ L, double *__restrict__ u)
{
    constexpr int NC = ncoef_of(P);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    if (i >= N) return;
    const int leaf = tgt_leaf[i];
    const double y[3] = {tgt_xyz[i] - cell_c[leaf], tgt_xyz[N + i] - cell_c[C + leaf],
                         tgt_xyz[2 * N + i] - cell_c[2 * C + leaf]};
    double pw[3][P + 1];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pw[k][0] = 1.0;
#pragma unroll
        for (int j = 1; j <= P; ++j) pw[k][j] = pw[k][j - 1] * y[k];
    }
    const double *Ll = L + ((int64_t)f * C + leaf) * NC;
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < NC; ++m) s = fma(Ll[m], pw[0][mi_x(m)] * pw[1][mi_y(m)] * pw[2][mi_z(m)], s);
    atomicAdd(&u[(int64_t)f * N + place(tgt_perm, i)], s);  // the near field is added concurrently
}

// One workgroup per P2P block (<= 64 tets of a source leaf and the targets of
// its near target leaves): one wavefront for one or two fields, four for more
// (they share the staged field coefficients).  Tets are staged in LDS BT at a
// time, thread l preparing field l % FCH of tet l / FCH (geometry 240 B + 208
// B per field per tet; 8 tets for 32 fields); every thread then takes targets
// ib + l, ib + l + NT, ... over the staged tets and adds its potentials
// atomically.  With band_skip the pairs of the surrogate's distance band
// (in_band) are left out: they are evaluated from the band pair list.
// WIDE: four wavefronts also for one or two fields (a plan's tuning choice).
__host__ __device__ constexpr int p2p_threads(int FCH, bool wide) { return FCH <= 2 && !wide ? 64 : 256; }
__host__ __device__ constexpr int p2p_stage(int FCH, bool wide)
{
    return FCH <= 2 ? (wide ? 64 / FCH : 16) : (FCH >= 32 ? 8 : (FCH >= 16 ? 16 : (FCH >= 8 ? 32 : 64)));
}

template <int FCH, bool WIDE>
__global__ __launch_bounds__(p2p_threads(FCH, WIDE), 2) void k_p2p(const int32_t *__restrict__ blk, int nblk, int band_skip, int64_t T,
                                                     const double *__restrict__ tet_xyz, const int32_t *__restrict__ tet_node,
                                                     const int32_t *__restrict__ idx, const double *__restrict__ tgt_xyz,
                                                     const int32_t *__restrict__ tgt_perm, int64_t N,
                                                     const double *__restrict__ M, int64_t n_nodes, int f0,
                                                     double *__restrict__ u)
{
    constexpr int BT = p2p_stage(FCH, WIDE), NT = p2p_threads(FCH, WIDE);
    static_assert(BT * FCH <= NT, "one thread per staged tet and field");
    __shared__ TetGeom s_g[BT];
    __shared__ TetField s_f[BT][FCH];
    __shared__ double s_bc[BT][4];  // band test: centroid, 1 / diam^2
    const int b = xcd_item(nblk);
    if (b < 0) return;
    const int tb = blk[4 * b], te = blk[4 * b + 1], ib = blk[4 * b + 2], ie = blk[4 * b + 3];
    const int lane = threadIdx.x;
    for (int sb = tb; sb < te; sb += BT) {
        const int nt = min(BT, te - sb);
        __syncthreads();
        {
            const int t = lane / FCH, f = lane % FCH;
            if (t < nt) {
                tet_prepare(tet_xyz, tet_node, T, sb + t, M + (int64_t)(f0 + f) * n_nodes * 3, f == 0 ? &s_g[t] : nullptr,
                            s_f[t][f]);
                if (band_skip && f == 0) {
                    double v[4][3];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int k = 0; k < 3; ++k) v[q][k] = tet_xyz[(int64_t)(3 * q + k) * T + sb + t];
                    band_geom(v, s_bc[t], s_bc[t][3]);
                }
            }
        }
        __syncthreads();
        for (int i = ib + lane; i < ie; i += NT) {
            const int s = idx[i];
            const double x[3] = {tgt_xyz[s], tgt_xyz[N + s], tgt_xyz[2 * N + s]};
            double acc[FCH];
#pragma unroll
            for (int f = 0; f < FCH; ++f) acc[f] = 0.0;
#pragma unroll 1
            for (int t = 0; t < nt; ++t) {
                if (band_skip && in_band(x, s_bc[t], s_bc[t][3])) continue;
                pair_accumulate<FCH>(x, s_g[t], s_f[t], acc);
            }
            const int64_t o = tgt_perm[s];
#pragma unroll
            for (int f = 0; f < FCH; ++f) atomicAdd(&u[(int64_t)(f0 + f) * N + o], acc[f] * kInv4Pi);
        }
    }
}

// ---------------------------------------------------------------------------
// Direct sum: every target against every tet.  Far from a tet the closed form
// of pair_accumulate adds terms much larger than their sum and loses about
// (d/diam)^4 eps (d = |x - centroid|, diam = the longest edge).  From 3
// diameters on the pair is instead integrated by a collapsed Gauss-Jacobi
// rule of the integrand of eq. approx1,
//   4 pi u_T(x) = 6|V| sum_q w_q M(y_q) . (x - y_q) / |x - y_q|^3.
// With y = v_0 + sum_i lambda_i e_i, M = M_0 + sum_i lambda_i (M_i - M_0) this is
//   6|V| (M_0 . S + sum_i (M_i - M_0) . K_i),
//   S = x' A_0 - sum_j A_j e_j,  K_i = x' A_i - sum_j A_ij e_j,  x' = x - v_0,
// of the ten moments A_0, A_i, A_ij of |x - y_q|^-3 with w_q (1, lambda_i,
// lambda_i lambda_j): independent of the field and summed loop by loop of the
// collapsed rule (far_moments), three multiply-adds a point and nothing read
// but one-dimensional tables in scalar registers.
//
// Bound by FP64 issue: 15 slots a point (2 for the squared distance, 4 for the
// hardware estimate of its root's reciprocal, 6 to refine and cube it, 3 for the
// moments) and 20 for each row of points.  10,368 tets, 2,197 targets, 2 fields:
// 15.8 ms with a rule per lane and 40 slots a point, now 3.5; 5 fields: 31.8 in
// two passes, now 4.0.
//
// A workgroup stages 16 consecutive tets in LDS (four times 4 with 16 fields, whose
// coefficients take the room) and takes 256 targets at a time:
// the pairs are sorted by class (rule, or closed form) and its wavefronts take 64
// pairs of one class after another, the most points first, so that no lane waits
// for another's larger rule (5,900 slots a pair with the wavefront's largest, 4,400
// sorted) and the loops stay uniform.  The sums are kept in LDS and added to u once
// a target and workgroup.
// ---------------------------------------------------------------------------
struct DirectTet {
    double c[3];     // centroid
    double id2;      // 1 / diam^2
    double e[3][3];  // v_1 - v_0, v_2 - v_0, v_3 - v_0
    double vol6;     // 6 |V|
};
constexpr int kDirectFieldsMax = 16;
__host__ __device__ constexpr int direct_stage(int FCH) { return FCH >= 16 ? 4 : 16; }
// Tets of a workgroup: the fewer, the more sums are added to u one by one, each with
// a rounding of u (24,576 tets: 2.9e-15 of the result with 4, 1.4e-15 with 16).
constexpr int kDirectTets = 16;

// Moments m = (A_0, A_1, A_2, A_3, A_11, A_12, A_13, A_22, A_23, A_33) of one
// tet (edge vectors e[i] = v_(i+1) - v_0) at x = target - v_0 by the rule of N^3
// points lambda = (a, (1-a) b, (1-a)(1-b) c).
template <int N>
__device__ __forceinline__ void far_moments(const double (&x)[3], const double (&e)[3][3], const double *table,
                                            double (&m)[10])
{
    const ScalarMem<FarC> *C = (const ScalarMem<FarC> *)scalar_mem(table);
    const ScalarMem<FarB> *Bt = (const ScalarMem<FarB> *)(scalar_mem(table) + 4 * N);
    const ScalarMem<FarA> *At = (const ScalarMem<FarA> *)(scalar_mem(table) + 12 * N);
    const double e33 = e[2][0] * e[2][0] + e[2][1] * e[2][1] + e[2][2] * e[2][2];
    const double k0 = scalar_const<dbits(1.5)>(), k1 = vector_const<dbits(1.875)>();
#pragma unroll
    for (int i = 0; i < 10; ++i) m[i] = 0.0;
#pragma unroll 1
    for (int ia = 0; ia < N; ++ia) {
        const ScalarMem<FarA> &a = At[ia];
        const double xa[3] = {fma(-a.a, e[0][0], x[0]), fma(-a.a, e[0][1], x[1]), fma(-a.a, e[0][2], x[2])};
        const double t = a.t, e2[3] = {t * e[1][0], t * e[1][1], t * e[1][2]};
        double b0 = 0.0, b1 = 0.0, b2 = 0.0, c0 = 0.0, c1 = 0.0, d0 = 0.0;
#pragma unroll 1
        for (int ib = 0; ib < N; ++ib) {
            const ScalarMem<FarB> &b = Bt[ib];
            const double xb[3] = {fma(-b.b, e2[0], xa[0]), fma(-b.b, e2[1], xa[1]), fma(-b.b, e2[2], xa[2])};
            // |xb - s c e_3|^2 = alpha + c (beta + c gamma)
            const double s = t * b.u;
            const double alpha = fma(xb[0], xb[0], fma(xb[1], xb[1], xb[2] * xb[2]));
            const double beta = -2.0 * s * fma(xb[0], e[2][0], fma(xb[1], e[2][1], xb[2] * e[2][2]));
            const double gamma = s * s * e33;
            double g0 = 0.0, g1 = 0.0, g2 = 0.0;
#pragma unroll
            for (int ic = 0; ic < N; ++ic) {
                const ScalarMem<FarC> &c = C[ic];
                const double r2 = fma(c.c, fma(c.c, gamma, beta), alpha);
                // r^-3 = y^3 (1 - h)^(-3/2), y^2 = (1 - h) / r^2, |h| < 2^-20
                const double y = __builtin_amdgcn_rsq(r2), y2 = y * y, y3 = y2 * y;
                const double h = fma(-r2, y2, 1.0);
                const double g = fma(y3, h * fma_sv(h, k1, k0), y3);
                g0 = fma(g, c.w, g0);
                g1 = fma(g, c.wc, g1);
                g2 = fma(g, c.wcc, g2);
            }
            b0 = fma(g0, b.w, b0);
            b1 = fma(g0, b.wb, b1);
            b2 = fma(g0, b.wbb, b2);
            c0 = fma(g1, b.wu, c0);
            c1 = fma(g1, b.wbu, c1);
            d0 = fma(g2, b.wuu, d0);
        }
        m[0] = fma(b0, a.w, m[0]);
        m[1] = fma(b0, a.wa, m[1]);
        m[2] = fma(b1, a.wt, m[2]);
        m[3] = fma(c0, a.wt, m[3]);
        m[4] = fma(b0, a.waa, m[4]);
        m[5] = fma(b1, a.wat, m[5]);
        m[6] = fma(c0, a.wat, m[6]);
        m[7] = fma(b2, a.wtt, m[7]);
        m[8] = fma(c1, a.wtt, m[8]);
        m[9] = fma(d0, a.wtt, m[9]);
    }
}

template <int FCH>
__global__ __launch_bounds__(256, FCH <= 4 ? 3 : 2) void k_direct(int nblk, int64_t T, const double *__restrict__ tet_xyz,
                                                const int32_t *__restrict__ tet_node,
                                                const double *__restrict__ tgt_xyz,
                                                const int32_t *__restrict__ tgt_perm, int64_t N,
                                                const double *__restrict__ M, int64_t n_nodes, int f0, int F,
                                                const double *__restrict__ rules, double *__restrict__ u)
{
    constexpr int DT = direct_stage(FCH);
    static_assert(DT * FCH <= 256, "one thread per staged tet and field");
    __shared__ TetGeom s_g[DT];
    __shared__ TetField s_f[DT][FCH];
    __shared__ DirectTet s_t[DT];
    __shared__ double s_m[DT][FCH][12];  // M_0 and M_i - M_0
    constexpr int NC = kFarRules + 1;    // classes: the far rules, then the closed form
    __shared__ double s_x[3][256], s_u[FCH][256];
    __shared__ uint16_t s_pair[DT * 256];
    __shared__ int s_cnt[NC], s_next;
    const int b = xcd_item(nblk);
    if (b < 0) return;
    constexpr int NST = kDirectTets / DT;  // stages
    const int lane = threadIdx.x;
    auto stage = [&](int64_t tb, int nt) {
        const int t = lane / FCH, f = lane % FCH;
        if (t < nt) {
            const int64_t tt = tb + t;
            const double *Mf = M + (int64_t)min(f0 + f, F - 1) * n_nodes * 3;
            tet_prepare(tet_xyz, tet_node, T, tt, Mf, f == 0 ? &s_g[t] : nullptr, s_f[t][f]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t nd = tet_node[(int64_t)c * T + tt];
#pragma unroll
                for (int k = 0; k < 3; ++k) s_m[t][f][3 * c + k] = Mf[3 * nd + k] - (c ? s_m[t][f][k] : 0.0);
            }
            if (f == 0) {
                double v[4][3];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int k = 0; k < 3; ++k) v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + tt];
                DirectTet &D = s_t[t];
                double l2 = 0.0;
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int q = a + 1; q < 4; ++q) {
                        const double dx = v[q][0] - v[a][0], dy = v[q][1] - v[a][1], dz = v[q][2] - v[a][2];
                        l2 = fmax(l2, dx * dx + dy * dy + dz * dz);
                    }
                D.id2 = 1.0 / l2;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    D.c[k] = 0.25 * ((v[0][k] + v[1][k]) + (v[2][k] + v[3][k]));
                    D.e[0][k] = v[1][k] - v[0][k];
                    D.e[1][k] = v[2][k] - v[0][k];
                    D.e[2][k] = v[3][k] - v[0][k];
                }
                const double det = D.e[0][0] * (D.e[1][1] * D.e[2][2] - D.e[1][2] * D.e[2][1]) -
                                   D.e[0][1] * (D.e[1][0] * D.e[2][2] - D.e[1][2] * D.e[2][0]) +
                                   D.e[0][2] * (D.e[1][0] * D.e[2][1] - D.e[1][1] * D.e[2][0]);
                D.vol6 = fabs(det);
            }
        }
    };
    const int64_t tb0 = (int64_t)b * kDirectTets;
    if constexpr (NST == 1) stage(tb0, (int)min<int64_t>(DT, T - tb0));
    __syncthreads();
    const int wl = lane & 63;
    for (int64_t i0 = (int64_t)blockIdx.y * 256; i0 < N; i0 += 256 * (int64_t)gridDim.y) {
        const bool ok = i0 + lane < N;
        const int64_t i = ok ? i0 + lane : N - 1;
        const double x[3] = {tgt_xyz[i], tgt_xyz[N + i], tgt_xyz[2 * N + i]};
#pragma unroll
        for (int k = 0; k < 3; ++k) s_x[k][lane] = x[k];
#pragma unroll
        for (int f = 0; f < FCH; ++f) s_u[f][lane] = 0.0;
#pragma unroll 1
        for (int st = 0; st < NST; ++st) {
            const int64_t tb = tb0 + st * DT;
            const int nt = (int)min<int64_t>(DT, T - tb);
            if (nt <= 0) break;
            if constexpr (NST > 1) stage(tb, nt);
            if (lane < NC) s_cnt[lane] = 0;
            if (lane == NC) s_next = 0;
            __syncthreads();
            // sort the pairs (tet, target) by class: count, then place
            uint64_t cls = 0;  // this target's class per tet, 4 bits each
            int at[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) at[k] = 0;
#pragma unroll 1
            for (int t = 0; t < nt; ++t) {
                const DirectTet &D = s_t[t];
                const double dc0 = x[0] - D.c[0], dc1 = x[1] - D.c[1], dc2 = x[2] - D.c[2];
                const double rat2 = (dc0 * dc0 + dc1 * dc1 + dc2 * dc2) * D.id2;
                int c = 0;
#pragma unroll
                for (int k = 1; k < kFarRules; ++k) c += !(rat2 < kFarRatio[k] * kFarRatio[k]);
                if (rat2 < kFarRatio[0] * kFarRatio[0]) c = kFarRules;
                if (!ok) c = 15;
                cls |= (uint64_t)c << (4 * t);
#pragma unroll
                for (int k = 0; k < NC; ++k) at[k] += __popcll(__ballot(c == k));
            }
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                int base = 0;
                if (wl == 0) base = atomicAdd(&s_cnt[k], at[k]);
                at[k] = __builtin_amdgcn_readfirstlane(base);
            }
            __syncthreads();
            int cnt[NC], start[NC + 1];
            start[0] = 0;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                cnt[k] = __builtin_amdgcn_readfirstlane(s_cnt[k]);
                start[k + 1] = start[k] + cnt[k];
                at[k] += start[k];
            }
#pragma unroll 1
            for (int t = 0; t < nt; ++t) {
                const int c = (int)(cls >> (4 * t)) & 15;
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    const uint64_t mask = __ballot(c == k);
                    if (c == k) s_pair[at[k] + __popcll(mask & ((1ull << wl) - 1))] = (uint16_t)(t * 256 + lane);
                    at[k] += __popcll(mask);
                }
            }
            __syncthreads();
            for (;;) {
                int chunk = 0;
                if (wl == 0) chunk = atomicAdd(&s_next, 1);
                chunk = __builtin_amdgcn_readfirstlane(chunk);
                int c = 0, p0 = 0, p1 = 0;
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    const int nch = (cnt[k] + 63) / 64;
                    if (chunk >= 0 && chunk < nch) {
                        c = k;
                        p0 = start[k] + 64 * chunk;
                        p1 = start[k + 1];
                    }
                    chunk -= nch;
                }
                if (chunk >= 0) break;
                const bool on = p0 + wl < p1;
                const int pr = s_pair[on ? p0 + wl : p1 - 1], t = pr >> 8, j = pr & 255;
                const double y[3] = {s_x[0][j], s_x[1][j], s_x[2][j]};
                double acc[FCH];
                if (c == kFarRules) {
#pragma unroll
                    for (int f = 0; f < FCH; ++f) acc[f] = 0.0;
                    pair_accumulate<FCH>(y, s_g[t], s_f[t], acc);
                } else {
                    const DirectTet &D = s_t[t];
                    const double xv[3] = {y[0] - s_g[t].v[0][0], y[1] - s_g[t].v[0][1], y[2] - s_g[t].v[0][2]};
                    double e[3][3], m[10];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int k = 0; k < 3; ++k) e[q][k] = D.e[q][k];
                    switch (c) {
                    case 0: far_moments<kFarPts[0]>(xv, e, rules + far_offset(0), m); break;
                    case 1: far_moments<kFarPts[1]>(xv, e, rules + far_offset(1), m); break;
                    case 2: far_moments<kFarPts[2]>(xv, e, rules + far_offset(2), m); break;
                    default: far_moments<kFarPts[3]>(xv, e, rules + far_offset(3), m); break;
                    }
                    double K[4][3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        K[0][k] = D.vol6 * fma(m[0], xv[k], -fma(m[1], e[0][k], fma(m[2], e[1][k], m[3] * e[2][k])));
                        K[1][k] = D.vol6 * fma(m[1], xv[k], -fma(m[4], e[0][k], fma(m[5], e[1][k], m[6] * e[2][k])));
                        K[2][k] = D.vol6 * fma(m[2], xv[k], -fma(m[5], e[0][k], fma(m[7], e[1][k], m[8] * e[2][k])));
                        K[3][k] = D.vol6 * fma(m[3], xv[k], -fma(m[6], e[0][k], fma(m[8], e[1][k], m[9] * e[2][k])));
                    }
#pragma unroll
                    for (int f = 0; f < FCH; ++f) {
                        const double *M4 = s_m[t][f];
                        double v = 0.0;
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int k = 0; k < 3; ++k) v = fma(M4[3 * q + k], K[q][k], v);
                        acc[f] = v;
                    }
                }
                if (on)
#pragma unroll
                    for (int f = 0; f < FCH; ++f) atomicAdd(&s_u[f][j], acc[f]);
            }
            __syncthreads();
        }
        if (ok) {
            const int64_t o = tgt_perm[i];
#pragma unroll
            for (int f = 0; f < FCH; ++f)
                if (f0 + f < F) atomicAdd(&u[(int64_t)(f0 + f) * N + o], s_u[f][lane] * kInv4Pi);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Point dipoles (the second source kind): u(x) = 1/(4 pi) sum_i m_i . (x - y_i)
// / |x - y_i|^3 over the sources of the near leaves (or all, direct sum); a
// target at a source's own position takes nothing from it.  Blocks as in
// k_p2p; the positions and the FCH moments of kPtStage sources are staged in
// LDS, every thread takes targets ib + l, ib + l + 256, ...
// ---------------------------------------------------------------------------
constexpr int kPtStage = 128, kPtThreads = 256;
constexpr int kP2PTets = 64;  // sources per block of the dipole direct sum

template <int FCH>
__global__ __launch_bounds__(kPtThreads) void k_p2p_points(const int32_t *__restrict__ blk, int nblk, int direct_src,
                                                           int64_t T, const double *__restrict__ src_xyz,
                                                           const int32_t *__restrict__ src_node,
                                                           const int32_t *__restrict__ idx,
                                                           const double *__restrict__ tgt_xyz,
                                                           const int32_t *__restrict__ tgt_perm, int64_t N,
                                                           const double *__restrict__ M, int64_t n_nodes, int f0,
                                                           double *__restrict__ u)
{
    __shared__ double s_y[kPtStage][3];
    __shared__ double s_m[kPtStage][FCH][3];
    const int b = xcd_item(nblk);
    if (b < 0) return;
    int tb, te, ib, ie;
    if (direct_src) {
        tb = b * kP2PTets;
        te = min<int64_t>(T, tb + kP2PTets);
        ib = 0;
        ie = (int)N;
    } else {
        tb = blk[4 * b];
        te = blk[4 * b + 1];
        ib = blk[4 * b + 2];
        ie = blk[4 * b + 3];
    }
    const int lane = threadIdx.x;
    for (int sb = tb; sb < te; sb += kPtStage) {
        const int ns = min(kPtStage, te - sb);
        __syncthreads();
        for (int i = lane; i < ns; i += kPtThreads) {
#pragma unroll
            for (int k = 0; k < 3; ++k) s_y[i][k] = src_xyz[(int64_t)k * T + sb + i];
            const int64_t nd = src_node[sb + i];
#pragma unroll
            for (int f = 0; f < FCH; ++f)
#pragma unroll
                for (int k = 0; k < 3; ++k) s_m[i][f][k] = M[((int64_t)(f0 + f) * n_nodes + nd) * 3 + k];
        }
        __syncthreads();
        for (int i = ib + lane; i < ie; i += kPtThreads) {
            const int s = direct_src ? i : idx[i];
            const double x[3] = {tgt_xyz[s], tgt_xyz[N + s], tgt_xyz[2 * N + s]};
            double acc[FCH];
#pragma unroll
            for (int f = 0; f < FCH; ++f) acc[f] = 0.0;
            for (int j = 0; j < ns; ++j) {
                const double d0 = x[0] - s_y[j][0], d1 = x[1] - s_y[j][1], d2 = x[2] - s_y[j][2];
                const double r2 = (d0 * d0 + d1 * d1) + d2 * d2;
                const double w = r2 > 0.0 ? 1.0 / (r2 * sqrt(r2)) : 0.0;
#pragma unroll
                for (int f = 0; f < FCH; ++f)
                    acc[f] = fma(w, (s_m[j][f][0] * d0 + s_m[j][f][1] * d1) + s_m[j][f][2] * d2, acc[f]);
            }
            const int64_t o = tgt_perm[s];
#pragma unroll
            for (int f = 0; f < FCH; ++f) atomicAdd(&u[(int64_t)(f0 + f) * N + o], acc[f] * kInv4Pi);
        }
    }
}

// ---------------------------------------------------------------------------
// Single-field near field over the shared mesh entities of a source chunk.
//
// Summed over the tets T of a chunk, the pair formula regroups by entity:
//   4 pi u(x) = sum_edges [ f_e il_e B_e(y) + Gamma_e g_e ] - sum_faces A_F(y) h_F Omega_F
// with y = x - c (c the chunk's node centroid), f_e the edge log (the line
// integral of 1/R, independent of the edge direction), g_e = R0^2 f +
// l_b R_b - l_a R_a (also direction independent), h_F Omega_F the face's
// height times solid angle in any fixed orientation (the product does not
// change with it), and the field weights
//   A_F(y)   = sum_{T, k: face k of T is F} alpha_{T,k}(y)                     (affine)
//   B_e(y)   = sum_{T, k, e in face k} s_{k,e} alpha_{T,k}(y) n_k.(d_a x d_b)  (quadratic)
//   Gamma_e  = sum_{T: e in T} gamma_{T,e}
// (alpha affine in y, d = v - x).  k_topo_static fills the geometry of every
// entity record once per plan, k_topo_coef the field weights once per
// evaluation; k_p2p_topo then evaluates one square root per node, one log per
// edge and one solid angle per face of the chunk for every target.
// ---------------------------------------------------------------------------
// One wavefront takes kTopoChunksPerWave chunks, 16 lanes (one per tet) each.
constexpr int kTopoChunksPerWave = 4;
static_assert(kTopoTets <= 64 / kTopoChunksPerWave, "one lane per tet of a chunk");
static_assert(kTopoEdges <= 64 && kTopoFaces <= 64, "one bit per entity, and its lines within one load a lane");
static_assert(kTopoEdges % 2 == 0 && kTopoFaces % 2 == 0, "pairs");

// Geometry of the entity records; one wavefront per chunk.
__global__ __launch_bounds__(64) void k_topo_static(const int32_t *__restrict__ ch_i, int nch,
                                                    const double *__restrict__ w, const int32_t *__restrict__ ab,
                                                    const int32_t *__restrict__ pqr, TopoEdge *__restrict__ edge,
                                                    TopoFace *__restrict__ face)
{
    const int ch = blockIdx.x;
    if (ch >= nch) return;
    const int noff = ch_i[8 * ch + 2], eoff = ch_i[8 * ch + 4], ne = ch_i[8 * ch + 5], foff = ch_i[8 * ch + 6],
              nf = ch_i[8 * ch + 7];
    const double *wn = w + 4 * (int64_t)noff;
    auto dist2 = [&](int a, int b) {
        const double d0 = wn[4 * b] - wn[4 * a], d1 = wn[4 * b + 1] - wn[4 * a + 1], d2 = wn[4 * b + 2] - wn[4 * a + 2];
        return (d0 * d0 + d1 * d1) + d2 * d2;
    };
    for (int i = threadIdx.x; i < ne; i += 64) {
        const int64_t e = (int64_t)eoff + i;
        const int a = ab[2 * e], b = ab[2 * e + 1];
        TopoEdge &E = edge[e];
        const int64_t en = e + (i + 2 < ne ? 2 : 0);
        E.l2 = dist2(a, b);
        E.L = sqrt(E.l2);
        E.il = 1.0 / E.L;
        E.own = (uint32_t)(a | b << 8);
        E.next = (uint32_t)(ab[2 * en] | ab[2 * en + 1] << 8);
    }
    for (int i = threadIdx.x; i < nf; i += 64) {
        const int64_t f = (int64_t)foff + i;
        const int p = pqr[3 * f], q = pqr[3 * f + 1], r = pqr[3 * f + 2];
        double u[3], v[3];
        for (int k = 0; k < 3; ++k) {
            u[k] = wn[4 * q + k] - wn[4 * p + k];
            v[k] = wn[4 * r + k] - wn[4 * p + k];
        }
        const double n[3] = {u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]};
        const double a2 = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]), ia = 1.0 / a2;
        TopoFace &F = face[f];
        for (int k = 0; k < 3; ++k) F.n[k] = n[k] * ia;
        F.h0 = F.n[0] * wn[4 * p] + F.n[1] * wn[4 * p + 1] + F.n[2] * wn[4 * p + 2];
        F.a4 = 2.0 * a2;
        F.l2pq = dist2(p, q);
        F.l2pr = dist2(p, r);
        F.l2qr = dist2(q, r);
        F.own = (uint32_t)(p | q << 8 | r << 16);
        const int64_t fnx = f + (i + 2 < nf ? 2 : 0);
        F.next = (uint32_t)(pqr[3 * fnx] | pqr[3 * fnx + 1] << 8 | pqr[3 * fnx + 2] << 16);
    }
}

__global__ __launch_bounds__(64) void k_topo_coef(const int32_t *__restrict__ ch_i, const double *__restrict__ ch_c,
                                                  int nch, const int32_t *__restrict__ inc,
                                                  const double *__restrict__ tet_xyz,
                                                  const int32_t *__restrict__ tet_node, int64_t T,
                                                  const double *__restrict__ M, const TopoEdge *__restrict__ edge,
                                                  TopoEdgeW *__restrict__ edge_w, TopoFaceW *__restrict__ face_w)
{
    constexpr int LPC = 64 / kTopoChunksPerWave;  // lanes per chunk
    __shared__ double s_Aw[kTopoChunksPerWave][kTopoFaces][4];
    __shared__ double s_Bw[kTopoChunksPerWave][kTopoEdges][11];
    const int sub = (int)threadIdx.x / LPC, tl = (int)threadIdx.x % LPC;
    const int ch = (int)blockIdx.x * kTopoChunksPerWave + sub;
    const bool live = ch < nch;
    const int chl = live ? ch : nch - 1;  // clamped: reads stay in bounds, nothing is written
    const int tb = ch_i[8 * chl], nt = live ? ch_i[8 * chl + 1] : 0, eoff = ch_i[8 * chl + 4],
              ne = ch_i[8 * chl + 5], foff = ch_i[8 * chl + 6], nf = ch_i[8 * chl + 7];
    const double c[3] = {ch_c[3 * chl], ch_c[3 * chl + 1], ch_c[3 * chl + 2]};
    double (*s_A)[4] = s_Aw[sub];
    double (*s_B)[11] = s_Bw[sub];
    for (int i = threadIdx.x; i < kTopoChunksPerWave * kTopoFaces * 4; i += blockDim.x) (&s_Aw[0][0][0])[i] = 0.0;
    for (int i = threadIdx.x; i < kTopoChunksPerWave * kTopoEdges * 11; i += blockDim.x) (&s_Bw[0][0][0])[i] = 0.0;
    __syncthreads();
    if (tl < nt) {
        const int64_t t = tb + tl;
        TetGeom G;
        TetField Fd;
        tet_prepare(tet_xyz, tet_node, T, t, M, &G, Fd);
        double w[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < 3; ++k) w[q][k] = G.v[q][k] - c[k];
        const int32_t *ti = inc + 10 * t;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double *n = G.n[k];
            const int a = kFv[k][0];
            // alpha_k(y) = a0 + a1 . y
            const double a1[3] = {Fd.b[k][0] - Fd.c[k] * n[0], Fd.b[k][1] - Fd.c[k] * n[1], Fd.b[k][2] - Fd.c[k] * n[2]};
            const double a0 = Fd.a[k] - (w[0][0] * Fd.b[k][0] + w[0][1] * Fd.b[k][1] + w[0][2] * Fd.b[k][2]) +
                              Fd.c[k] * (n[0] * w[a][0] + n[1] * w[a][1] + n[2] * w[a][2]);
            double *Af = s_A[ti[6 + k]];
            atomicAdd(&Af[0], a0);
            atomicAdd(&Af[1], a1[0]);
            atomicAdd(&Af[2], a1[1]);
            atomicAdd(&Af[3], a1[2]);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int e = kFe[k][j];
                const double sg = kFs[k][j];
                const int ea = kEa[e], eb = kEb[e];
                // n . ((w_a - y) x (w_b - y)) = t0 + t1 . y
                const double cx[3] = {w[ea][1] * w[eb][2] - w[ea][2] * w[eb][1], w[ea][2] * w[eb][0] - w[ea][0] * w[eb][2],
                                      w[ea][0] * w[eb][1] - w[ea][1] * w[eb][0]};
                const double t0 = n[0] * cx[0] + n[1] * cx[1] + n[2] * cx[2];
                const double u[3] = {w[ea][0] - w[eb][0], w[ea][1] - w[eb][1], w[ea][2] - w[eb][2]};
                const double t1[3] = {u[1] * n[2] - u[2] * n[1], u[2] * n[0] - u[0] * n[2], u[0] * n[1] - u[1] * n[0]};
                double *Be = s_B[ti[e]];
                atomicAdd(&Be[0], sg * a0 * t0);
                atomicAdd(&Be[1], sg * (a0 * t1[0] + t0 * a1[0]));
                atomicAdd(&Be[2], sg * (a0 * t1[1] + t0 * a1[1]));
                atomicAdd(&Be[3], sg * (a0 * t1[2] + t0 * a1[2]));
                atomicAdd(&Be[4], sg * a1[0] * t1[0]);
                atomicAdd(&Be[5], sg * (a1[0] * t1[1] + a1[1] * t1[0]));
                atomicAdd(&Be[6], sg * (a1[0] * t1[2] + a1[2] * t1[0]));
                atomicAdd(&Be[7], sg * a1[1] * t1[1]);
                atomicAdd(&Be[8], sg * (a1[1] * t1[2] + a1[2] * t1[1]));
                atomicAdd(&Be[9], sg * a1[2] * t1[2]);
            }
        }
#pragma unroll
        for (int e = 0; e < 6; ++e) atomicAdd(&s_B[ti[e]][10], Fd.g[e]);
    }
    __syncthreads();
    if (!live) return;
    // the records hold -2 A (the solid angle enters as its half), 2 il B and
    // Gamma / 2 (f and g enter as f/2 and 2 g)
    for (int i = tl; i < nf * 4; i += LPC) face_w[(int64_t)foff + (i >> 2)].A[i & 3] = -2.0 * (&s_A[0][0])[i];
    for (int i = tl; i < ne * 12; i += LPC) {
        const int e = i / 12, q = i - 12 * e;
        const double w = q < 10 ? 2.0 * edge[(int64_t)eoff + e].il : 0.5;
        (&edge_w[(int64_t)eoff + e].B[0])[q] = q < 11 ? s_B[e][q] * w : 0.0;
    }
}

// Work item: up to 64 targets of one source block, one wavefront, one target
// per lane, all chunks of the block.  Splitting a block's targets over
// wavefronts, not one wavefront a block, fills the chip on small meshes (806
// blocks of a 17^3 cube: 4.7 -> 0.45 ms).  The chunk's entities are the same for
// every lane, so they are read on the scalar path, and only the corner
// distances R, each lane its own column, live in LDS; no barrier is needed.
// Corner distances and per-entity constants are all that the terms need (see
// AtanhFar); the few targets close to an edge or face take a vote of the
// wavefront into the shifted forms or, closer still, put the pair off to a
// second loop.  The block's target list is ordered by distance, so that few
// wavefronts hold such targets.
// Bound: FP64 issue, about 45 slots a (target, edge) and 43 a (target, face);
// the vector unit is busy 0.86 of the time on the 40^3 cube, 0.91 on the sphere
// below.  40^3 cube (160M pairs, 11.7 tets a
// block): 4.05 -> 2.1 ms against the form with difference vectors, cross
// products and branch-free selects; 14.2 -> 11.0 ms on 853M pairs of a sphere
// with 45 tets a block.  4 wavefronts a SIMD without spills beat 5 with 13
// spilled registers (2.30 against 2.45 ms, field weights included); 2 and 4
// wavefronts a workgroup were slower (+9%, +33%: their slots free up together).
__global__ __launch_bounds__(64, 4) void k_p2p_topo(const int32_t *__restrict__ item, int nitems,
                                                    const int32_t *__restrict__ ch_i, const double *__restrict__ ch_c,
                                                    const double *__restrict__ nw, const TopoEdge *__restrict__ edge,
                                                    const TopoFace *__restrict__ face,
                                                    const TopoEdgeW *__restrict__ edge_w,
                                                    const TopoFaceW *__restrict__ face_w,
                                                    const int32_t *__restrict__ idx,
                                                    const double *__restrict__ tgt_xyz,
                                                    const int32_t *__restrict__ tgt_perm, int64_t N,
                                                    double *__restrict__ u)
{
    __shared__ double s_R[kTopoNodes][64];
    const int lane = (int)threadIdx.x;
    const int it = xcd_item(nitems);
    if (it < 0) return;
    const int cb = item[4 * it], ce = item[4 * it + 1], ib = item[4 * it + 2], ie = item[4 * it + 3];
    const int s = idx[min(ib + lane, ie - 1)];  // the lanes past the end repeat the last target
    const double x[3] = {tgt_xyz[s], tgt_xyz[N + s], tgt_xyz[2 * N + s]};
    double *R = &s_R[0][lane];
    double acc = 0.0;
    // The scalar loads below each wait for their line; from HBM that would be
    // most of the time.  So the lines of a chunk are all brought into L2 at
    // once, by one vector load a lane, while the chunk before it is worked on.
    auto line = [&](const auto *p, int n) {  // one of the 128-byte lines of p[0 .. n)
        const uint32_t at = 128u * (uint32_t)lane;
        return at < (uint32_t)(n * sizeof(*p)) ? *(const int32_t *)((const char *)p + at) : 0;
    };
    auto touch = [&](int ch) {
        const int64_t eo = ch_i[8 * ch + 4], fo = ch_i[8 * ch + 6];
        const int ne = ch_i[8 * ch + 5], nf = ch_i[8 * ch + 7];
        return line(edge + eo, ne) + line(edge_w + eo, ne) + line(face + fo, nf) + line(face_w + fo, nf);
    };
    int seen = touch(cb);
    for (int ch = cb; ch < ce; ++ch) {
        asm volatile("" ::"v"(seen));
        seen = touch(min(ch + 1, ce - 1));
        const int noff = ch_i[8 * ch + 2], nn = ch_i[8 * ch + 3], eoff = ch_i[8 * ch + 4], ne = ch_i[8 * ch + 5],
                  foff = ch_i[8 * ch + 6], nf = ch_i[8 * ch + 7];
        const double y[3] = {x[0] - ch_c[3 * ch], x[1] - ch_c[3 * ch + 1], x[2] - ch_c[3 * ch + 2]};
        const ScalarMem<double> *w = scalar_mem(nw + 4 * (int64_t)noff);
#pragma unroll 2
        for (int j = 0; j < nn; ++j) {
            const double d0 = w[4 * j] - y[0], d1 = w[4 * j + 1] - y[1], d2 = w[4 * j + 2] - y[2];
            R[64 * j] = sqrt_nr((d0 * d0 + d1 * d1) + d2 * d2);
        }
        const double m[9] = {y[0],        y[1],        y[2],        y[0] * y[0], y[0] * y[1],
                             y[0] * y[2], y[1] * y[1], y[1] * y[2], y[2] * y[2]};
        // Entities are taken in pairs, which share one reciprocal.  Software
        // pipeline: at the top of a pair its field weights, the next pair's
        // geometry and (record e names the corners of e + 2) its corner
        // distances are asked for, and waited for once, before the weights
        // are used.  Two register sets, alternating without copies.
        if (ne > 0) {
            const AtanhFar atanh_far;
            const ScalarMem<TopoEdge> *E0 = scalar_mem(edge + eoff);
            const ScalarMem<TopoEdgeW> *W0 = scalar_mem(edge_w + eoff);
            uint64_t near = 0;  // edges with a target of this wavefront too close, taken after the others
            struct Ops {
                uint32_t next;
                double L, il, l2, Ra, Rb;
            };
            auto load = [&](Ops (&o)[2], int e, uint32_t c0, uint32_t c1) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const ScalarMem<TopoEdge> &E = E0[e + k];
                    o[k].next = E.next;
                    o[k].L = E.L;
                    o[k].il = E.il;
                    o[k].l2 = E.l2;
                    o[k].Ra = R[64 * ((k ? c1 : c0) & 255)];
                    o[k].Rb = R[64 * ((k ? c1 : c0) >> 8)];
                }
            };
            auto step = [&](const Ops (&o)[2], Ops (&next)[2], int e) {
                double Bq[2][11];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int q = 0; q < 11; ++q) Bq[k][q] = W0[e + k].B[q];
                load(next, e + 2 < ne ? e + 2 : e, o[0].next, o[1].next);
                const double S[2] = {o[0].Ra + o[0].Rb, o[1].Ra + o[1].Rb};
                const double ri = rcp_nr(S[0] * S[1]);
                double sv[2] = {o[0].L * (ri * S[1]), o[1].L * (ri * S[0])};
                double lin[2] = {sv[0], sv[1]};
                if (__any(fmax(sv[0], sv[1]) > kEdgeFar)) {
                    // At a corner of the edge f does not count (its weight is
                    // zero to rounding) and any finite value serves; a target
                    // past kEdgeMid puts the pair off; between the two
                    // atanh(s) = atanh(c) + atanh((s - c)/(1 - c s)).
                    double c[2], den[2];
                    bool put_off = false;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const bool close = sv[k] > kEdgeFar && fmin(o[k].Ra, o[k].Rb) > 0.0;
                        put_off = put_off || (close && sv[k] > kEdgeMid);
                        c[k] = close ? kEdgeShift : 0.0;
                        den[k] = fma(-c[k], o[k].L, S[k]);
                    }
                    if (__any(put_off)) {
                        near |= 3ull << e;
                        return;
                    }
                    const double r2 = rcp_nr(den[0] * den[1]);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        sv[k] = fma(-c[k], S[k], o[k].L) * (r2 * den[1 - k]);
                        lin[k] = fma(c[k], kEdgeShiftAtanh / kEdgeShift, sv[k]);
                    }
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const double t = (o[k].Rb - o[k].Ra) * o[k].il, t2 = t * t, SL = S[k] * o[k].L;
                    const double F = atanh_far(sv[k], lin[k]);  // f / 2 and 2 g
                    const double g = fma(fma(S[k], S[k], -o[k].l2) * (1.0 - t2), F, fma(t2, SL, SL));
                    double bq = Bq[k][1] * m[0];
#pragma unroll
                    for (int q = 1; q < 9; ++q) bq = fma(Bq[k][q + 1], m[q], bq);
                    bq += Bq[k][0];
                    acc = fma(F, bq, fma(Bq[k][10], g, acc));
                }
            };
            Ops oa[2], ob[2];
            load(oa, 0, E0[0].own, E0[1].own);
#pragma unroll 1
            for (int e = 0; e < ne; e += 4) {
                step(oa, ob, e);
                if (e + 2 >= ne) break;
                step(ob, oa, e + 2);
            }
            while (near) {
                const int e = __builtin_ctzll(near);
                near &= near - 1;
                const ScalarMem<TopoEdge> &E = E0[e];
                const int a = E.own & 255, b = E.own >> 8;
                const double Ra = R[64 * a], Rb = R[64 * b], S = Ra + Rb;
                const double sv = E.L * rcp_nr(S);
                const bool off = Ra > 0.0 && Rb > 0.0;  // at a corner f does not count
                double F, g;
                if (!__any(off && sv > kEdgeMid)) {
                    const double t = (Rb - Ra) * E.il, t2 = t * t, SL = S * E.L;
                    F = 0.5 * log_ratio<true>(S + E.L, S - E.L);
                    F = off ? F : 0.0;
                    g = fma(fma(S, S, -E.l2) * (1.0 - t2), F, fma(t2, SL, SL));
                } else {
                    const ScalarMem<double> *wa = w + 4 * a, *wb = w + 4 * b;
                    const double da[3] = {wa[0] - y[0], wa[1] - y[1], wa[2] - y[2]};
                    const double db[3] = {wb[0] - y[0], wb[1] - y[1], wb[2] - y[2]};
                    const double Dab = da[0] * db[0] + da[1] * db[1] + da[2] * db[2];
                    const double la = fma(-Ra, Ra, Dab) * E.il;  // (v_a - x) . e_hat
                    const double lb = fma(Rb, Rb, -Dab) * E.il;  // (v_b - x) . e_hat
                    const double cx0 = da[1] * db[2] - da[2] * db[1], cx1 = da[2] * db[0] - da[0] * db[2],
                                 cx2 = da[0] * db[1] - da[1] * db[0];
                    const double r0sq = (cx0 * cx0 + cx1 * cx1 + cx2 * cx2) * (E.il * E.il);
                    const bool far = kEdgeMid * S >= E.L;
                    const double f = edge_log_mixed(far, S, E.L, Ra, Rb, la, lb, r0sq);
                    const double t = (Rb - Ra) * E.il, t2 = t * t, SL = S * E.L;
                    F = 0.5 * f;
                    g = far ? fma(fma(S, S, -E.l2) * (1.0 - t2), F, fma(t2, SL, SL))
                            : 2.0 * (r0sq * f + lb * Rb - la * Ra);
                }
                const ScalarMem<TopoEdgeW> &W = W0[e];
                double bq = W.B[1] * m[0];
#pragma unroll
                for (int q = 1; q < 9; ++q) bq = fma(W.B[q + 1], m[q], bq);
                bq += W.B[0];
                acc = fma(F, bq, fma(W.B[10], g, acc));
            }
        }
        if (nf > 0) {
            const AtanFar atan_far;
            const ScalarMem<TopoFace> *F0 = scalar_mem(face + foff);
            const ScalarMem<TopoFaceW> *W0 = scalar_mem(face_w + foff);
            uint64_t near = 0;
            struct Ops {
                uint32_t next;
                double l2pq, l2pr, l2qr, Rp, Rq, Rr;
            };
            auto load = [&](Ops (&o)[2], int f, uint32_t c0, uint32_t c1) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const ScalarMem<TopoFace> &K = F0[f + k];
                    const uint32_t c = k ? c1 : c0;
                    o[k].next = K.next;
                    o[k].l2pq = K.l2pq;
                    o[k].l2pr = K.l2pr;
                    o[k].l2qr = K.l2qr;
                    o[k].Rp = R[64 * (c & 255)];
                    o[k].Rq = R[64 * (c >> 8 & 255)];
                    o[k].Rr = R[64 * (c >> 16)];
                }
            };
            auto step = [&](const Ops (&o)[2], Ops (&next)[2], int f) {
                double n[2][3], h0[2], a4[2], A[2][4];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const ScalarMem<TopoFace> &K = F0[f + k];
#pragma unroll
                    for (int q = 0; q < 3; ++q) n[k][q] = K.n[q];
                    h0[k] = K.h0;
                    a4[k] = K.a4;
#pragma unroll
                    for (int q = 0; q < 4; ++q) A[k][q] = W0[f + k].A[q];
                }
                load(next, f + 2 < nf ? f + 2 : f, o[0].next, o[1].next);
                double P[2], den[2], h[2], num[2], tn[2];  // den: twice the denominator; h: height; tn: tan(Omega/2)
                bool bad = false;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    P[k] = (o[k].Rp + o[k].Rq) * (o[k].Rq + o[k].Rr) * (o[k].Rr + o[k].Rp);
                    den[k] = P[k] - fma(o[k].l2pq, o[k].Rr, fma(o[k].l2pr, o[k].Rq, o[k].l2qr * o[k].Rp));
                    bad = bad || !(den[k] >= kFaceCond * P[k]);
                }
                const double ri = rcp_nr(den[0] * den[1]);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    h[k] = h0[k] - (n[k][0] * y[0] + n[k][1] * y[1] + n[k][2] * y[2]);
                    num[k] = h[k] * a4[k];
                    tn[k] = num[k] * (ri * den[1 - k]);
                }
                bad = bad || !(fmax(fabs(tn[0]), fabs(tn[1])) <= kFaceTan);
                double lin[2] = {tn[0], tn[1]};
                if (__any(bad)) {
                    // At a corner of the face h is zero (to rounding) and any
                    // denominator serves; a denominator small against P puts
                    // the pair off, as does t > 1 / kFaceTan; between the two
                    // atan(t) = pi/4 + atan((t - 1)/(t + 1)).
                    double top[2], dn[2], off[2];
                    bool put_off = false;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const bool corner = !(fmin(fmin(o[k].Rp, o[k].Rq), o[k].Rr) > 0.0);
                        const double d = corner ? 1.0 : den[k], an = fabs(num[k]);
                        const bool wide = an > kFaceTan * d;
                        put_off = put_off || (!corner && (!(d >= kFaceCond * P[k]) || kFaceTan * an > d));
                        top[k] = copysign(wide ? an - d : an, num[k]);
                        top[k] = wide && an < d ? -top[k] : top[k];
                        dn[k] = wide ? an + d : d;
                        off[k] = wide ? copysign(0.78539816339744827900, num[k]) : 0.0;
                    }
                    if (__any(put_off)) {
                        near |= 3ull << f;
                        return;
                    }
                    const double r2 = rcp_nr(dn[0] * dn[1]);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        tn[k] = top[k] * (r2 * dn[1 - k]);
                        lin[k] = tn[k] + off[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const double af = A[k][0] + (A[k][1] * y[0] + A[k][2] * y[1] + A[k][3] * y[2]);
                    acc = fma(af * h[k], atan_far(tn[k], lin[k]), acc);
                }
            };
            Ops oa[2], ob[2];
            load(oa, 0, F0[0].own, F0[1].own);
#pragma unroll 1
            for (int f = 0; f < nf; f += 4) {
                step(oa, ob, f);
                if (f + 2 >= nf) break;
                step(ob, oa, f + 2);
            }
            while (near) {
                const int f = __builtin_ctzll(near);
                near &= near - 1;
                const ScalarMem<TopoFace> &K = F0[f];
                const int p = K.own & 255, q = K.own >> 8 & 255, r = K.own >> 16;
                const double Rp = R[64 * p], Rq = R[64 * q], Rr = R[64 * r];
                const double P = (Rp + Rq) * (Rq + Rr) * (Rr + Rp);
                const double den = P - fma(K.l2pq, Rr, fma(K.l2pr, Rq, K.l2qr * Rp));
                const double h = K.h0 - (K.n[0] * y[0] + K.n[1] * y[1] + K.n[2] * y[2]);
                const bool off = Rp > 0.0 && Rq > 0.0 && Rr > 0.0;  // at a corner h = 0
                double num = h * K.a4, dn = off ? den : 1.0;
                if (__any(off && !(den >= kFaceCond * P))) {
                    const ScalarMem<double> *wp = w + 4 * p, *wq = w + 4 * q, *wr = w + 4 * r;
                    const double dp[3] = {wp[0] - y[0], wp[1] - y[1], wp[2] - y[2]};
                    const double dq[3] = {wq[0] - y[0], wq[1] - y[1], wq[2] - y[2]};
                    const double dr[3] = {wr[0] - y[0], wr[1] - y[1], wr[2] - y[2]};
                    const double Dpq = dp[0] * dq[0] + dp[1] * dq[1] + dp[2] * dq[2];
                    const double Dpr = dp[0] * dr[0] + dp[1] * dr[1] + dp[2] * dr[2];
                    const double Dqr = dq[0] * dr[0] + dq[1] * dr[1] + dq[2] * dr[2];
                    // [d_p, d_q, d_r] = d_p . ((q - p) x (r - p)) = h |(q - p) x (r - p)|
                    num *= 0.5;
                    dn = Rp * Rq * Rr + Dpq * Rr + Dpr * Rq + Dqr * Rp;
                }
                const ScalarMem<TopoFaceW> &W = W0[f];
                const double af = W.A[0] + (W.A[1] * y[0] + W.A[2] * y[1] + W.A[3] * y[2]);
                acc = fma(af * h, atan2_nr<true>(num, dn), acc);
            }
        }
    }
    asm volatile("" ::"v"(seen));
    if (ib + lane < ie) atomicAdd(&u[place(tgt_perm, s)], acc * kInv4Pi);
}

// ---------------------------------------------------------------------------
// Near field of several fields.
//
// The nodal M is continuous over the mesh, so in
//   4 pi u(x) = sum_faces int_F M.n / R  -  sum_T div M_T int_T 1/R
// the surface charges of a face between two tets of a chunk cancel, and a
// field enters a (target, tet) pair only with its divergence and, on the
// chunk's boundary faces, with three corner charges: 1 + 3 x 1.7 numbers a tet
// where the coefficients of the whole pair formula are 26.  With the
// barycentric coordinates lambda of the target in the tet, F' = f / (2 L) of an
// edge (see AtanhFar) and a_k the half solid angle of face k,
//   lambda_i^(k) = lambda_i - 6V (grad lambda_i . grad lambda_k) mu_k,
//                  mu_k = lambda_k 6V / (2 A_k)^2     (of the foot on face k),
//   I_k = int_Fk 1/R / (4 A_k) = sum_{i != k} lambda_i^(k) F'_{edge opposite i in k} - mu_k a_k,
//   int_T 1/R = 6V sum_k lambda_k I_k,
//   int_Fk lambda_i/R / (4 A_k) = lambda_i^(k) I_k + sum_e C_{k,i,e} g'_e,
//   g' = 2 g / L = (S^2 - L^2)(1 - t^2) F' + S (1 + t^2),  tan a_k = 12V lambda_k / den_k.
// ---------------------------------------------------------------------------
// edge joining corners a and b
constexpr int kEdgeOf[4][4] = {{-1, 0, 1, 2}, {0, -1, 3, 4}, {1, 3, -1, 5}, {2, 4, 5, -1}};
constexpr int kNearFieldsMax = 16;  // fields of one pass

// One lane per tet of a chunk.
__global__ __launch_bounds__(64) void k_tet_static(const int32_t *__restrict__ ch_i, const double *__restrict__ ch_c,
                                                   int nch, const double *__restrict__ tet_xyz, int64_t T,
                                                   const uint8_t *__restrict__ skin, const int64_t *__restrict__ row,
                                                   const uint32_t *__restrict__ corner, NearTet *__restrict__ out,
                                                   uint32_t *__restrict__ ch_flat, int32_t *__restrict__ n_flat)
{
    const int ch = blockIdx.x;
    if (ch >= nch || (int)threadIdx.x >= ch_i[8 * ch + 1]) return;
    const int64_t t = ch_i[8 * ch] + (int64_t)threadIdx.x;
    NearTet &K = out[t];
    K.corner = corner[t];
    K.skin = skin[t];
    K.row = row[t];
    double v[4][3];
    for (int c = 0; c < 4; ++c)
        for (int k = 0; k < 3; ++k) v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + t] - ch_c[3 * ch + k];
    double N[4][3];  // |.| = 2 A_k, outward: -6V grad lambda_k
    for (int f = 0; f < 4; ++f) {
        const int a = kFv[f][0], b = kFv[f][1], c = kFv[f][2];
        const double p[3] = {v[b][0] - v[a][0], v[b][1] - v[a][1], v[b][2] - v[a][2]};
        const double q[3] = {v[c][0] - v[a][0], v[c][1] - v[a][1], v[c][2] - v[a][2]};
        N[f][0] = p[1] * q[2] - p[2] * q[1];
        N[f][1] = p[2] * q[0] - p[0] * q[2];
        N[f][2] = p[0] * q[1] - p[1] * q[0];
    }
    const double e[3] = {v[1][0] - v[0][0], v[1][1] - v[0][1], v[1][2] - v[0][2]};
    const double v6 = -(e[0] * N[1][0] + e[1] * N[1][1] + e[2] * N[1][2]), iv = 1.0 / v6;
    K.v12 = 2.0 * v6;
    for (int i = 1; i < 4; ++i) {
        for (int k = 0; k < 3; ++k) K.lam[i - 1][k] = -N[i][k] * iv;
    }
    for (int k = 0; k < 3; ++k) K.c[k] = 0.25 * ((v[0][k] + v[1][k]) + (v[2][k] + v[3][k]));
    for (int k = 0; k < 4; ++k) K.kap[k] = v6 / (N[k][0] * N[k][0] + N[k][1] * N[k][1] + N[k][2] * N[k][2]);
    for (int i = 0; i < 6; ++i) {
        const int a = kEa[i], b = kEb[i];
        double d2 = 0.0, g = 0.0;
        for (int k = 0; k < 3; ++k) {
            d2 += (v[b][k] - v[a][k]) * (v[b][k] - v[a][k]);
            g += N[a][k] * N[b][k];
        }
        K.l2[i] = d2;
        K.il2[i] = 1.0 / d2;
        K.L[i] = sqrt(d2);
        K.G[i] = g * iv;
    }
    // sine of the angle between faces a and b: 6V L / (2 A_a 2 A_b), L the other two corners' edge
    bool flat = false;
    for (int i = 0; i < 6; ++i) {
        const double *p = N[kEa[i]], *q = N[kEb[i]];
        flat = flat || v6 * K.L[5 - i] < kFlatSine * sqrt((p[0] * p[0] + p[1] * p[1] + p[2] * p[2]) *
                                                          (q[0] * q[0] + q[1] * q[1] + q[2] * q[2]));
    }
    K.flat = flat ? atomicAdd(n_flat, 1) : -1;
    const uint64_t all = __ballot(flat);
    if (threadIdx.x == 0) ch_flat[ch] = (uint32_t)all;
    for (int f = 0; f < 4; ++f) {
        const int *c = kFv[f];
        const double a2 = N[f][0] * N[f][0] + N[f][1] * N[f][1] + N[f][2] * N[f][2];
        for (int i = 1; i < 3; ++i)
            for (int j = 0; j < 3; ++j) {  // E_i . E_j of the edges opposite corners i and j, in cyclic direction
                const double *p = v[c[(i + 1) % 3]], *q = v[c[(i + 2) % 3]], *r = v[c[(j + 1) % 3]], *s = v[c[(j + 2) % 3]];
                double d = 0.0;
                for (int k = 0; k < 3; ++k) d += (q[k] - p[k]) * (s[k] - r[k]);
                K.C[f][i - 1][j] = -d / (8.0 * a2);
            }
    }
}

// The flat tets' records, one lane per tet of a chunk (as k_tet_static).
__global__ __launch_bounds__(64) void k_flat_static(const int32_t *__restrict__ ch_i, const double *__restrict__ ch_c,
                                                    int nch, const double *__restrict__ tet_xyz, int64_t T,
                                                    const NearTet *__restrict__ tet, NearFlat *__restrict__ out)
{
    const int ch = blockIdx.x;
    if (ch >= nch || (int)threadIdx.x >= ch_i[8 * ch + 1]) return;
    const int64_t t = ch_i[8 * ch] + (int64_t)threadIdx.x;
    if (tet[t].flat < 0) return;
    NearFlat &K = out[tet[t].flat];
    double v[4][3], cen[3];
    for (int c = 0; c < 4; ++c)
        for (int k = 0; k < 3; ++k) v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + t] - ch_c[3 * ch + k];
    for (int k = 0; k < 3; ++k) cen[k] = 0.25 * ((v[0][k] + v[1][k]) + (v[2][k] + v[3][k]));  // as in k_tet_static
    for (int f = 0; f < 4; ++f) {
        const double *v0 = v[kFv[f][0]];
        double e[2][3], n[3];  // corners 1 and 2 from corner 0, and the normal
        for (int j = 0; j < 2; ++j)
            for (int k = 0; k < 3; ++k) e[j][k] = v[kFv[f][j + 1]][k] - v0[k];
        for (int k = 0; k < 3; ++k) n[k] = e[0][(k + 1) % 3] * e[1][(k + 2) % 3] - e[0][(k + 2) % 3] * e[1][(k + 1) % 3];
        const double i2 = 1.0 / (n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
        for (int j = 0; j < 2; ++j) {  // gradients e_2 x n / n^2 and n x e_1 / n^2
            const double *p = j ? n : e[1], *q = j ? e[0] : n;
            double at = 0.0;
            for (int k = 0; k < 3; ++k) {
                const double g = (p[(k + 1) % 3] * q[(k + 2) % 3] - p[(k + 2) % 3] * q[(k + 1) % 3]) * i2;
                K.f[f][j][1 + k] = g;
                at += g * (cen[k] - v0[k]);
            }
            K.f[f][j][0] = at;
        }
    }
}

// Field weights of one pass, [rows][FC]: per tet -6V div M, then per boundary
// face w_0, w_1 - w_0, w_2 - w_0 with w_i = 4 A_k n_k . M at its corner i (zero
// past the last field).  Thread (tet, field), fields consecutive.
template <int FC>
__global__ __launch_bounds__(256) void k_near_weights(const NearTet *__restrict__ tet, int64_t T,
                                                      const double *__restrict__ tet_xyz,
                                                      const int32_t *__restrict__ tet_node,
                                                      const double *__restrict__ M, int64_t n_nodes, int f0, int F,
                                                      double *__restrict__ W)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, t = i / FC;
    const int f = (int)(i % FC);
    if (t >= T || tet[t].row < 0) return;
    double v[4][3], m[4][3];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int64_t nd = tet_node[(int64_t)c * T + t];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + t];
            m[c][k] = f0 + f < F ? M[((int64_t)(f0 + f) * n_nodes + nd) * 3 + k] : 0.0;
        }
    }
    double N[4][3], div = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int a = kFv[q][0], b = kFv[q][1], c = kFv[q][2];
        const double p[3] = {v[b][0] - v[a][0], v[b][1] - v[a][1], v[b][2] - v[a][2]};
        const double r[3] = {v[c][0] - v[a][0], v[c][1] - v[a][1], v[c][2] - v[a][2]};
        N[q][0] = p[1] * r[2] - p[2] * r[1];
        N[q][1] = p[2] * r[0] - p[0] * r[2];
        N[q][2] = p[0] * r[1] - p[1] * r[0];
        div += N[q][0] * m[q][0] + N[q][1] * m[q][1] + N[q][2] * m[q][2];  // -6V grad lambda_q . M_q
    }
    double *w = W + tet[t].row * FC + f;
    w[0] = div;
    const uint32_t skin = tet[t].skin;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (!(skin >> q & 1)) continue;
        double s[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double *mm = m[kFv[q][j]];
            s[j] = 2.0 * (N[q][0] * mm[0] + N[q][1] * mm[1] + N[q][2] * mm[2]);
        }
        w[FC] = s[0];
        w[2 * FC] = s[1] - s[0];
        w[3 * FC] = s[2] - s[0];
        w += 3 * FC;
    }
}

// q <- q z + c of N values, c a scalar constant (see scalar_const).
template <int N, unsigned long long kBits>
__device__ __forceinline__ void horner(double (&q)[N], const double (&z)[N])
{
    const double c = scalar_const<kBits>();
    static_assert(N == 4 || N == 6, "faces or edges of a tet");
    if constexpr (N == 4)
        asm("v_fma_f64 %0, %0, %4, %8\n\tv_fma_f64 %1, %1, %5, %8\n\t"
            "v_fma_f64 %2, %2, %6, %8\n\tv_fma_f64 %3, %3, %7, %8"
            : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3])
            : "v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]), "s"(c));
    else
        asm("v_fma_f64 %0, %0, %6, %12\n\tv_fma_f64 %1, %1, %7, %12\n\tv_fma_f64 %2, %2, %8, %12\n\t"
            "v_fma_f64 %3, %3, %9, %12\n\tv_fma_f64 %4, %4, %10, %12\n\tv_fma_f64 %5, %5, %11, %12"
            : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5])
            : "v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]), "v"(z[4]), "v"(z[5]), "s"(c));
}
template <int N, unsigned long long... kBits>
__device__ __forceinline__ void horner_all(double (&q)[N], const double (&z)[N])
{
    (horner<N, kBits>(q, z), ...);
}
// AtanhFar's and AtanFar's polynomials of z, of all edges or faces of a tet
__device__ __forceinline__ void atanh_poly(double (&q)[6], const double (&z)[6])
{
#pragma unroll
    for (int e = 0; e < 6; ++e) q[e] = 1.97454264785334926424e-01;
    horner_all<6, dbits(-1.09516507426128548164e-01), dbits(1.14547545108890203025e-01),
               dbits(2.69135450515010227202e-02), dbits(5.65994173773324837917e-02),
               dbits(5.83095311569123558870e-02), dbits(6.67117797972938270101e-02),
               dbits(7.69204426675997310348e-02), dbits(9.09091891139124363974e-02),
               dbits(1.11111108941550865148e-01), dbits(1.42857142881957860370e-01),
               dbits(1.99999999999888822266e-01), dbits(3.33333333333333425852e-01)>(q, z);
}
__device__ __forceinline__ void atan_poly(double (&q)[4], const double (&z)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = -1.91768871190622589893e-2;
    horner_all<4, dbits(3.923165829558719130283e-2), dbits(-5.085449737940259861323e-2),
               dbits(5.858148912802209881646e-2), dbits(-6.664511447381948000098e-2),
               dbits(7.692183190826086563693e-2), dbits(-9.090904578123901890479e-2),
               dbits(1.111111101525636172749e-1), dbits(-1.428571428466654292249e-1),
               dbits(1.999999999999552067782e-1), dbits(-3.333333333333333015966e-1)>(q, z);
}

// Work items, chunks, corner distances and closer forms as in k_p2p_topo; the
// tets of a chunk are taken one at a time, all edges and faces of a tet side
// by side, those with a close target in a second loop.  Bound: FP64 issue, about
// 390 slots a (target, tet) pair and 6 more a field (the whole pair formula in
// every lane took 935 and 27); the vector unit is busy 0.70 of the time (16
// fields on a 26^3 cube; 0.55 on an 18^3 cube, where the last wavefronts leave
// the chip half empty), the rest is waiting for the scalar reads of geometry and
// weights.  16 fields on a 26^3 cube (81M pairs): 4.8 -> 2.0 ms; 5 fields on a 21^3 cube: 1.77 ->
// 0.57; 64 on an 18^3 cube: 9.9 -> 4.6.  32 fields a pass leave two wavefronts
// a SIMD and a quarter of the rate.  Four wavefronts a workgroup: the kernel
// alone takes the same, but the expansion kernels beside it find room sooner
// (whole evaluation 4.71 -> 4.43 ms at 16 fields).  kFlat: for meshes that hold
// flat tets (see NearFlat); all of it in one form is 0.5 to 0.8% slower on others.
constexpr int kFieldWaves = 4;

template <int FC, bool kFlat>
__global__ __launch_bounds__(64 * kFieldWaves, 3) void k_p2p_fields(
    const int32_t *__restrict__ item, int nitems, const int32_t *__restrict__ ch_i, const double *__restrict__ ch_c,
    const double *__restrict__ nw, const NearTet *__restrict__ tet, const NearFlat *__restrict__ flat,
    const uint32_t *__restrict__ ch_flat, const double *__restrict__ W, const int32_t *__restrict__ idx, const double *__restrict__ tgt_xyz, const int32_t *__restrict__ tgt_perm,
    int64_t N, int f0, int F, double *__restrict__ u)
{
    __shared__ double s_R[kFieldWaves][kTopoNodes][64];
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wg = xcd_item((nitems + kFieldWaves - 1) / kFieldWaves), it = wg * kFieldWaves + wave;
    if (wg < 0 || it >= nitems) return;
    const int cb = item[4 * it], ce = item[4 * it + 1], ib = item[4 * it + 2], ie = item[4 * it + 3];
    const int s = idx[min(ib + lane, ie - 1)];
    const double x[3] = {tgt_xyz[s], tgt_xyz[N + s], tgt_xyz[2 * N + s]};
    double *R = &s_R[wave][0][lane];
    double acc[FC];
#pragma unroll
    for (int f = 0; f < FC; ++f) acc[f] = 0.0;
    // brings the lines of a chunk's records and weights into L2 while the chunk
    // before it is worked on (see k_p2p_topo)
    auto touch = [&](int ch) {
        const int t0 = ch_i[8 * ch], n = ch_i[8 * ch + 1];
        const ScalarMem<NearTet> *K = scalar_mem(tet + t0);
        const int64_t r0 = K[0].row, rows = K[n - 1].row + 1 + 3 * __builtin_popcount(K[n - 1].skin) - r0;
        const uint32_t nk = (uint32_t)(n * sizeof(NearTet)), nw = (uint32_t)(rows * FC * sizeof(double));
        const char *pk = (const char *)(tet + t0), *pw = (const char *)(W + r0 * FC);
        int v = 0;
        const uint32_t at = 128u * (uint32_t)lane;
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j)
            if (at + 8192u * j < nk) v ^= *(const int32_t *)(pk + at + 8192u * j);
#pragma unroll
        for (uint32_t j = 0; j < (FC >= 16 ? 2 : 1); ++j)
            if (at + 8192u * j < nw) v ^= *(const int32_t *)(pw + at + 8192u * j);
        return v;
    };
    int seen = touch(cb);
    for (int ch = cb; ch < ce; ++ch) {
        asm volatile("" ::"v"(seen));
        seen = touch(min(ch + 1, ce - 1));
        const int tb = ch_i[8 * ch], nt = ch_i[8 * ch + 1], noff = ch_i[8 * ch + 2], nn = ch_i[8 * ch + 3];
        const double y[3] = {x[0] - ch_c[3 * ch], x[1] - ch_c[3 * ch + 1], x[2] - ch_c[3 * ch + 2]};
        const ScalarMem<double> *w = scalar_mem(nw + 4 * (int64_t)noff);
#pragma unroll 2
        for (int j = 0; j < nn; ++j) {
            const double d0 = w[4 * j] - y[0], d1 = w[4 * j + 1] - y[1], d2 = w[4 * j + 2] - y[2];
            R[64 * j] = sqrt_nr((d0 * d0 + d1 * d1) + d2 * d2);
        }
        // barycentric coordinates of the target in tet K
        auto coords = [&](const ScalarMem<NearTet> &K, double (&lam)[4]) {
            const double yc[3] = {y[0] - K.c[0], y[1] - K.c[1], y[2] - K.c[2]};
            double off = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double g = K.lam[i][0] * yc[0] + K.lam[i][1] * yc[1] + K.lam[i][2] * yc[2];
                lam[i + 1] = 0.25 + g;
                off += g;
            }
            lam[0] = 0.25 - off;
        };
        // Barycentric coordinates on face k of its foot, mu as above.
        auto foot_of = [&](const ScalarMem<NearTet> &K, const double (&lam)[4], int k, double mu, double (&foot)[3]) {
#pragma unroll
            for (int j = 0; j < 3; ++j) foot[j] = fma(-K.G[kEdgeOf[kFv[k][j]][k]], mu, lam[kFv[k][j]]);
        };
        // Adds tet K to the sums of all fields: F' of its edges, half solid
        // angles of its faces, the feet of its faces and g' of an edge on demand.
        auto add = [&](const ScalarMem<NearTet> &K, const double (&lam)[4], const double (&Fe)[6],
                       const double (&at)[4], auto &&foot_at, auto &&edge_g) {
            const ScalarMem<double> *wr = scalar_mem(W) + K.row * FC, *w0 = wr;
            const uint32_t skin = K.skin;
            double vol = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int *c = kFv[k];
                const double mu = K.kap[k] * lam[k];
                double foot[3], I = -mu * at[k];
                foot_at(k, mu, foot);
#pragma unroll
                for (int j = 0; j < 3; ++j) I = fma(foot[j], Fe[kEdgeOf[c[(j + 1) % 3]][c[(j + 2) % 3]]], I);
                vol = fma(lam[k], I, vol);
                if (!(skin >> k & 1)) continue;
                wr += 3 * FC;
                double s1 = foot[1] * I, s2 = foot[2] * I;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const double g = edge_g(kEdgeOf[c[(m + 1) % 3]][c[(m + 2) % 3]]);
                    s1 = fma(K.C[k][0][m], g, s1);
                    s2 = fma(K.C[k][1][m], g, s2);
                }
#pragma unroll
                for (int f = 0; f < FC; ++f)
                    acc[f] = fma(wr[f], s2, fma(wr[f - FC], s1, fma(wr[f - 2 * FC], I, acc[f])));
            }
#pragma unroll
            for (int f = 0; f < FC; ++f) acc[f] = fma(w0[f], vol, acc[f]);
        };
        // F' = a + a z Q(z) (shifted by as - a) and the half angles t + t^3 Q(t^2)
        // (shifted by ts - t).
        auto series = [&](const double (&z)[6], const double (&a)[6], const double (&as)[6], const double (&t)[4],
                          const double (&ts)[4], double (&Fe)[6], double (&at)[4]) {
            double q[6], r[4], zf[4];
            atanh_poly(q, z);
#pragma unroll
            for (int e = 0; e < 6; ++e) Fe[e] = fma(a[e] * z[e], q[e], as[e]);
#pragma unroll
            for (int k = 0; k < 4; ++k) zf[k] = t[k] * t[k];
            atan_poly(r, zf);
#pragma unroll
            for (int k = 0; k < 4; ++k) at[k] = fma(t[k] * zf[k], r[k], ts[k]);
        };
        auto far_g = [&](const ScalarMem<NearTet> &K, const double (&Rc)[4], const double (&Fe)[6], int e) {
            const double D = Rc[kEb[e]] - Rc[kEa[e]], S = Rc[kEa[e]] + Rc[kEb[e]], t2 = D * (D * K.il2[e]);
            return fma(fma(S, S, -K.l2[e]) * (1.0 - t2), Fe[e], fma(t2, S, S));
        };
        // flat tets, and those with a target of this wavefront too close, are taken after the others
        const uint32_t flats = kFlat ? ch_flat[ch] : 0;
        uint32_t near = flats;
#pragma unroll 1
        for (int j = 0; j < nt; ++j) {
            if (kFlat && flats >> j & 1) continue;
            const ScalarMem<NearTet> &K = *scalar_mem(tet + tb + j);
            const uint32_t cn = K.corner;
            double Rc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) Rc[c] = R[64 * (cn >> (8 * c) & 255)];
            double S[6], z[6], iv[6], top = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e) S[e] = Rc[kEa[e]] + Rc[kEb[e]];
#pragma unroll
            for (int e = 0; e < 6; e += 2) {
                const double ri = rcp_nr(S[e] * S[e + 1]);
                iv[e] = ri * S[e + 1];
                iv[e + 1] = ri * S[e];
            }
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                z[e] = K.l2[e] * (iv[e] * iv[e]);
                top = fmax(top, z[e]);
            }
            double lam[4], den[4], tn[4];
            coords(K, lam);
            bool bad = !(top <= kEdgeFar * kEdgeFar);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int a = kFv[k][0], b = kFv[k][1], c = kFv[k][2];
                const int ea = kEdgeOf[b][c], eb = kEdgeOf[a][c], ec = kEdgeOf[a][b];
                const double P = S[ec] * S[ea] * S[eb];
                den[k] = P - fma(K.l2[ec], Rc[c], fma(K.l2[eb], Rc[b], K.l2[ea] * Rc[a]));
                bad = bad || !(den[k] >= kFaceCond * P);
            }
#pragma unroll
            for (int k = 0; k < 4; k += 2) {
                const double ri = rcp_nr(den[k] * den[k + 1]) * K.v12;
                tn[k] = lam[k] * (ri * den[k + 1]);
                tn[k + 1] = lam[k + 1] * (ri * den[k]);
            }
            bad = bad || !(fmax(fmax(fabs(tn[0]), fabs(tn[1])), fmax(fabs(tn[2]), fabs(tn[3]))) <= kFaceTan);
            if (__any(bad)) {
                near |= 1u << j;
                continue;
            }
            double Fe[6], at[4];
            series(z, iv, iv, tn, tn, Fe, at);
            add(K, lam, Fe, at, [&](int k, double mu, double (&foot)[3]) { foot_of(K, lam, k, mu, foot); },
                [&](int e) { return far_g(K, Rc, Fe, e); });
        }
        // the shifted forms (see k_p2p_topo), or closer still the branch-free
        // forms of the pair formula
        while (near) {
            const int j = __builtin_ctz(near);
            near &= near - 1;
            const ScalarMem<NearTet> &K = *scalar_mem(tet + tb + j);
            const uint32_t cn = K.corner;
            double Rc[4], lam[4], Fe[6], gp[6], at[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) Rc[c] = R[64 * (cn >> (8 * c) & 255)];
            coords(K, lam);
            bool close = false;
            double c[6], nm[4], df[4], of[4];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const double Ra = Rc[kEa[e]], Rb = Rc[kEb[e]], Sm = Ra + Rb;
                const bool in = kEdgeFar * Sm < K.L[e] && fmin(Ra, Rb) > 0.0;
                close = close || (in && kEdgeMid * Sm < K.L[e]);
                c[e] = in ? kEdgeShift : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double Ra = Rc[kFv[k][0]], Rb = Rc[kFv[k][1]], Rd = Rc[kFv[k][2]];
                const double Pk = (Ra + Rb) * (Rb + Rd) * (Rd + Ra);
                const double dk = Pk - fma(K.l2[kEdgeOf[kFv[k][0]][kFv[k][1]]], Rd,
                                           fma(K.l2[kEdgeOf[kFv[k][0]][kFv[k][2]]], Rb,
                                               K.l2[kEdgeOf[kFv[k][1]][kFv[k][2]]] * Ra));
                const bool corner = !(fmin(fmin(Ra, Rb), Rd) > 0.0);
                const double nk = K.v12 * lam[k], an = fabs(nk), d = corner ? 1.0 : dk;
                const bool wide = an > kFaceTan * d;
                close = close || (!corner && (!(d >= kFaceCond * Pk) || kFaceTan * an > d));
                const double p = copysign(wide ? an - d : an, nk);
                nm[k] = wide && an < d ? -p : p;
                df[k] = wide ? an + d : d;
                of[k] = wide ? copysign(0.78539816339744827900, nk) : 0.0;
            }
            if (!__any(close)) {
                double zs[6], as[6], a1[6], ts[4], t1[4];
#pragma unroll
                for (int e = 0; e < 6; e += 2) {
                    const double S0 = Rc[kEa[e]] + Rc[kEb[e]], S1 = Rc[kEa[e + 1]] + Rc[kEb[e + 1]];
                    const double d0 = fma(-c[e], K.L[e], S0), d1 = fma(-c[e + 1], K.L[e + 1], S1);
                    const double ri = rcp_nr(d0 * d1);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const double sv = fma(-c[e + j], j ? S1 : S0, K.L[e + j]) * (ri * (j ? d0 : d1));
                        const double il = K.L[e + j] * K.il2[e + j];
                        zs[e + j] = sv * sv;
                        a1[e + j] = sv * il;
                        as[e + j] = fma(c[e + j], kEdgeShiftAtanh / kEdgeShift, sv) * il;
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; k += 2) {
                    const double ri = rcp_nr(df[k] * df[k + 1]);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        t1[k + j] = nm[k + j] * (ri * df[k + 1 - j]);
                        ts[k + j] = t1[k + j] + of[k + j];
                    }
                }
                series(zs, a1, as, t1, ts, Fe, at);
#pragma unroll
                for (int e = 0; e < 6; ++e) gp[e] = far_g(K, Rc, Fe, e);
            } else {
                double d[4][3];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const ScalarMem<double> *v = w + 4 * (cn >> (8 * q) & 255);
#pragma unroll
                    for (int k = 0; k < 3; ++k) d[q][k] = v[k] - y[k];
                }
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    const int p = kEa[e], q = kEb[e];
                    const double il2 = K.il2[e], il = K.L[e] * il2;
                    const double dab = d[p][0] * d[q][0] + d[p][1] * d[q][1] + d[p][2] * d[q][2];
                    const double la = fma(-Rc[p], Rc[p], dab) * il, lb = fma(Rc[q], Rc[q], -dab) * il;
                    const double c0 = d[p][1] * d[q][2] - d[p][2] * d[q][1],
                                 c1 = d[p][2] * d[q][0] - d[p][0] * d[q][2],
                                 c2 = d[p][0] * d[q][1] - d[p][1] * d[q][0];
                    const double r0sq = (c0 * c0 + c1 * c1 + c2 * c2) * il2;
                    const double S = Rc[p] + Rc[q];
                    const bool far = kEdgeMid * S >= K.L[e];
                    const double f = edge_log_mixed(far, S, K.L[e], Rc[p], Rc[q], la, lb, r0sq);
                    Fe[e] = 0.5 * f * il;
                    gp[e] = far ? far_g(K, Rc, Fe, e) : 2.0 * il * (r0sq * f + lb * Rc[q] - la * Rc[p]);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i0 = kFv[k][0], i1 = kFv[k][1], i2 = kFv[k][2];
                    auto dt = [&](int p, int q) { return d[p][0] * d[q][0] + d[p][1] * d[q][1] + d[p][2] * d[q][2]; };
                    at[k] = atan2_nr<true>(0.5 * (K.v12 * lam[k]), Rc[i0] * Rc[i1] * Rc[i2] + dt(i0, i1) * Rc[i2] +
                                                                       dt(i0, i2) * Rc[i1] + dt(i1, i2) * Rc[i0]);
                }
            }
            const int32_t fl = kFlat ? K.flat : -1;
            add(K, lam, Fe, at,
                [&](int k, double mu, double (&foot)[3]) {
                    if (fl < 0) {
                        foot_of(K, lam, k, mu, foot);
                        return;
                    }
                    const ScalarMem<NearFlat> &P = *scalar_mem(flat + fl);
                    foot[0] = 1.0;
#pragma unroll
                    for (int j = 1; j < 3; ++j) {
                        foot[j] = P.f[k][j - 1][0];
#pragma unroll
                        for (int q = 0; q < 3; ++q) foot[j] = fma(P.f[k][j - 1][1 + q], y[q] - K.c[q], foot[j]);
                        foot[0] -= foot[j];
                    }
                },
                [&](int e) { return gp[e]; });
        }
    }
    asm volatile("" ::"v"(seen));
    if (ib + lane < ie) {
        const int64_t o = place(tgt_perm, s);
#pragma unroll
        for (int f = 0; f < FC; ++f)
            if (f0 + f < F) atomicAdd(&u[(int64_t)(f0 + f) * N + o], acc[f] * kInv4Pi);
    }
}

// ---------------------------------------------------------------------------
// Stored near-field operator (Sec. 2.1: the direct part is linear in the
// nodal magnetisation, so its node-to-node coefficients can be kept for a
// fixed mesh).  u_T(x) = sum_{corners c, axes j} C_{T,c,j}(x) M_{node(T,c), j}
// where C_{T,c,j}(x) is the potential of the field that is the unit vector e_j
// at corner c and zero at the other corners.  k_near_assemble evaluates the
// pair formula for these 12 unit fields (staged in LDS like the fields of
// k_p2p) for every near (target, tet) pair and adds the coefficients into the
// target's row of its leaf block [nt][3][ncols]; the column of a node is found
// by binary search in the leaf's sorted column list.
// ---------------------------------------------------------------------------
constexpr int kNearAsmTets = 16, kNearAsmThreads = 256;

__global__ __launch_bounds__(kNearAsmThreads) void k_near_assemble(
    const int32_t *__restrict__ blk, int nblk, int64_t T, const double *__restrict__ tet_xyz,
    const int32_t *__restrict__ tet_node, const int32_t *__restrict__ idx, const double *__restrict__ tgt_xyz,
    int64_t N, const int32_t *__restrict__ tgt_leaf, const int32_t *__restrict__ cell_i,
    const int64_t *__restrict__ near_off, const int32_t *__restrict__ near_nc, const int32_t *__restrict__ near_cols,
    double *__restrict__ val)
{
    __shared__ TetGeom s_g[kNearAsmTets];
    __shared__ TetField s_f[kNearAsmTets][12];
    __shared__ int32_t s_n[kNearAsmTets][4];
    const int b = xcd_item(nblk);
    if (b < 0) return;
    const int tb = blk[4 * b], te = blk[4 * b + 1], ib = blk[4 * b + 2], ie = blk[4 * b + 3];
    const int lane = threadIdx.x;
    for (int sb = tb; sb < te; sb += kNearAsmTets) {
        const int nt = min(kNearAsmTets, te - sb);
        __syncthreads();
        {
            const int t = lane / 12, f = lane % 12;
            if (t < nt) {
                TetGeom G;
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int k = 0; k < 3; ++k) G.v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + sb + t];
                double gl[4][3], eh[6][3];
                tet_geometry(G, gl, eh);
                double m[4][3];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int k = 0; k < 3; ++k) m[c][k] = (3 * c + k == f) ? 1.0 : 0.0;
                tet_field(G, gl, eh, m, s_f[t][f]);
                if (f == 0) {
                    s_g[t] = G;
#pragma unroll
                    for (int c = 0; c < 4; ++c) s_n[t][c] = tet_node[(int64_t)c * T + sb + t];
                }
            }
        }
        __syncthreads();
        for (int i = ib + lane; i < ie; i += kNearAsmThreads) {
            const int s = idx[i];
            const double x[3] = {tgt_xyz[s], tgt_xyz[N + s], tgt_xyz[2 * N + s]};
            const int32_t a = tgt_leaf[s];
            const int64_t voff = near_off[2 * a + 1];
            if (voff < 0) continue;
            const int nc = near_nc[a];
            const int32_t *cl = near_cols + near_off[2 * a];
            double *row = val + voff + (int64_t)(s - cell_i[8 * a + 2]) * 3 * nc;
#pragma unroll 1
            for (int t = 0; t < nt; ++t) {
                PairGeo P;
                pair_geometry(x, s_g[t], P);
#pragma unroll 1
                for (int c = 0; c < 4; ++c) {
                    const int32_t node = s_n[t][c];
                    int lo = 0, hi = nc;  // first column >= node
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (cl[mid] < node) lo = mid + 1; else hi = mid;
                    }
                    if (lo >= nc || cl[lo] != node) continue;
#pragma unroll
                    for (int j = 0; j < 3; ++j)
                        atomicAdd(&row[(int64_t)j * nc + lo], pair_contract(P, s_f[t][3 * c + j]) * kInv4Pi);
                }
            }
        }
    }
}

// Applies the stored operator.  Work item = up to kNearRows consecutive target
// rows of one leaf (they share the leaf's column list): one wavefront per
// item, lanes striding the columns; per column the node's M is gathered once
// for FC fields and applied to every row of the item (three coalesced
// coefficient streams per row).  Row sums are reduced across the wavefront
// and added into u (L2P adds concurrently).
constexpr int kNearRows = 4, kNearItemsPerBlock = 4;

template <int FC>
__global__ __launch_bounds__(64 * kNearItemsPerBlock) void k_near_apply(
    int nitems, const int32_t *__restrict__ items, const int32_t *__restrict__ cell_i,
    const int64_t *__restrict__ near_off, const int32_t *__restrict__ near_nc, const int32_t *__restrict__ near_cols,
    const double *__restrict__ val, const int32_t *__restrict__ tgt_perm, int64_t N, const double *__restrict__ M,
    int64_t n_nodes, int F, double *__restrict__ u)
{
    const int blk = xcd_item((nitems + kNearItemsPerBlock - 1) / kNearItemsPerBlock);
    if (blk < 0) return;
    const int lane = threadIdx.x & 63;
    // one item per wavefront, its index made visibly uniform (the item's
    // bounds, column list and rows are then read on the scalar path)
    const int it = blk * kNearItemsPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (it >= nitems) return;
    const int32_t a = items[2 * it], r0 = items[2 * it + 1];
    const int xb = cell_i[8 * a + 2];
    const int nr = min(kNearRows, cell_i[8 * a + 3] - xb - r0);
    const int64_t voff = near_off[2 * a + 1];
    const int nc = near_nc[a];
    const int32_t *cl = near_cols + near_off[2 * a];
    const double *row = val + voff + (int64_t)r0 * 3 * nc;
    const int f0 = blockIdx.y * FC;
    double acc[kNearRows][FC];
#pragma unroll
    for (int r = 0; r < kNearRows; ++r)
#pragma unroll
        for (int f = 0; f < FC; ++f) acc[r][f] = 0.0;
    for (int c = lane; c < nc; c += 64) {
        const int64_t n = cl[c];
        double w[kNearRows][3];
#pragma unroll
        for (int r = 0; r < kNearRows; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) w[r][k] = r < nr ? row[((int64_t)r * 3 + k) * nc + c] : 0.0;
#pragma unroll
        for (int f = 0; f < FC; ++f) {
            if (f0 + f < F) {
                const double *m = M + ((int64_t)(f0 + f) * n_nodes + n) * 3;
                const double m0 = m[0], m1 = m[1], m2 = m[2];
#pragma unroll
                for (int r = 0; r < kNearRows; ++r)
                    acc[r][f] = fma(w[r][0], m0, fma(w[r][1], m1, fma(w[r][2], m2, acc[r][f])));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kNearRows; ++r)
#pragma unroll
        for (int f = 0; f < FC; ++f) {
            double v = acc[r][f];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane == 0 && r < nr && f0 + f < F) atomicAdd(&u[(int64_t)(f0 + f) * N + tgt_perm[xb + r0 + r]], v);
        }
}

// ---------------------------------------------------------------------------
// Demagnetising field and energy from nodal potentials (P1 interpolation):
// per tet H_T = -grad u = -sum_i u_i grad lambda_i, and
//   E / mu0 = 1/2 sum_T int_T M . grad u = 1/2 sum_T V_T (mean_i M_i) . grad u_T
// (M affine on the tet).  One thread per tet (octree order); the block sums
// are added in a fixed order by k_sum_blocks.
// ---------------------------------------------------------------------------
constexpr int kEnergyThreads = 256;

// grad u of the P1 interpolant on tet t (octree order) of the nodal values u,
// with its corner node ids, 6|V| and the mean nodal M (when M is not null).
__device__ inline void p1_gradient(const double *__restrict__ tet_xyz, const int32_t *__restrict__ tet_node, int64_t T,
                                   int64_t t, const double *__restrict__ u, const double *__restrict__ M,
                                   double gu[3], int64_t nd[4], double &vol6, double mbar[3])
{
    double v[4][3], uc[4];
#pragma unroll
    for (int k = 0; k < 3; ++k) mbar[k] = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        nd[c] = tet_node[(int64_t)c * T + t];
        uc[c] = u[nd[c]];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v[c][k] = tet_xyz[(int64_t)(3 * c + k) * T + t];
            if (M) mbar[k] += 0.25 * M[3 * nd[c] + k];
        }
    }
    double e1[3], e2[3], e3[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e1[k] = v[1][k] - v[0][k];
        e2[k] = v[2][k] - v[0][k];
        e3[k] = v[3][k] - v[0][k];
    }
    // grad u = (u1-u0) g1 + (u2-u0) g2 + (u3-u0) g3, g_i = rows of the inverse Jacobian
    double g1[3], g2[3], g3[3];
    g1[0] = e2[1] * e3[2] - e2[2] * e3[1];
    g1[1] = e2[2] * e3[0] - e2[0] * e3[2];
    g1[2] = e2[0] * e3[1] - e2[1] * e3[0];
    g2[0] = e3[1] * e1[2] - e3[2] * e1[1];
    g2[1] = e3[2] * e1[0] - e3[0] * e1[2];
    g2[2] = e3[0] * e1[1] - e3[1] * e1[0];
    g3[0] = e1[1] * e2[2] - e1[2] * e2[1];
    g3[1] = e1[2] * e2[0] - e1[0] * e2[2];
    g3[2] = e1[0] * e2[1] - e1[1] * e2[0];
    const double det = e1[0] * g1[0] + e1[1] * g1[1] + e1[2] * g1[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) gu[k] = ((uc[1] - uc[0]) * g1[k] + (uc[2] - uc[0]) * g2[k] + (uc[3] - uc[0]) * g3[k]) / det;
    vol6 = fabs(det);
}

__global__ __launch_bounds__(kEnergyThreads) void k_demag(const double *__restrict__ tet_xyz,
                                                          const int32_t *__restrict__ tet_node,
                                                          const int32_t *__restrict__ tet_perm, int64_t T,
                                                          const double *__restrict__ M, const double *__restrict__ u,
                                                          double *__restrict__ H, double *__restrict__ part)
{
    __shared__ double s_e[kEnergyThreads];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double e = 0.0;
    if (t < T) {
        double gu[3], vol6, mbar[3];
        int64_t nd[4];
        p1_gradient(tet_xyz, tet_node, T, t, u, M, gu, nd, vol6, mbar);
        e = 0.5 * (vol6 / 6.0) * (mbar[0] * gu[0] + mbar[1] * gu[1] + mbar[2] * gu[2]);
        if (H) {
            const int64_t o = tet_perm[t];
#pragma unroll
            for (int k = 0; k < 3; ++k) H[3 * o + k] = -gu[k];
        }
    }
    s_e[threadIdx.x] = e;
    __syncthreads();
    for (int w = kEnergyThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) s_e[threadIdx.x] += s_e[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s_e[0];
}

// Mass-lumped nodal field (the lumped L2 projection of the P1 field onto the
// nodes): H_j = sum_{T ni j} (V_T / 4) H_T / w_j, w_j = sum_{T ni j} V_T / 4.
// k_demag_scatter adds (V_T / 4) H_T of every tet to its corners (and, when w
// is not null, V_T / 4 to the weights); k_lump_divide divides by w.
__global__ __launch_bounds__(kEnergyThreads) void k_demag_scatter(const double *__restrict__ tet_xyz,
                                                                  const int32_t *__restrict__ tet_node, int64_t T,
                                                                  const double *__restrict__ u, double *__restrict__ Hn,
                                                                  double *__restrict__ w)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    double gu[3], vol6, mbar[3];
    int64_t nd[4];
    p1_gradient(tet_xyz, tet_node, T, t, u, nullptr, gu, nd, vol6, mbar);
    const double q = vol6 / 24.0;  // V_T / 4
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int k = 0; k < 3; ++k) atomicAdd(&Hn[3 * nd[c] + k], -q * gu[k]);
        if (w) atomicAdd(&w[nd[c]], q);
    }
}

__global__ void k_lump_divide(double *__restrict__ Hn, const double *__restrict__ w, int64_t n)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const double wj = w[j];
    const double r = wj > 0.0 ? 1.0 / wj : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) Hn[3 * j + k] *= r;
}

__global__ __launch_bounds__(kEnergyThreads) void k_sum_blocks(const double *__restrict__ part, int n,
                                                               double *__restrict__ out)
{
    __shared__ double s_e[kEnergyThreads];
    double e = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) e += part[i];
    s_e[threadIdx.x] = e;
    __syncthreads();
    for (int w = kEnergyThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) s_e[threadIdx.x] += s_e[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s_e[0];
}

// ---------------------------------------------------------------------------
// The near field's own elementary functions, one call per element (for
// checking them against an independent implementation).
// ---------------------------------------------------------------------------
__global__ void k_elementary(int fn, const double *__restrict__ a, const double *__restrict__ b, int64_t n,
                             double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = a[i], y = b[i];
    double r;
    switch (fn) {
    case 0: r = log_ratio(x, y); break;
    case 1: r = atan2_nr(x, y); break;
    case 2: r = div_nr(x, y); break;
    default: r = rsqrt_nr(x); break;
    }
    out[i] = r;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
std::vector<int32_t> xcd_dispatch_items(int n)
{
    std::vector<int32_t> out;
    out.reserve(n > 0 ? n : 0);
    const int per = (n + kXcds - 1) / kXcds;
    for (int w = 0; w < kXcds * per; ++w) {
        const int item = (w % kXcds) * per + w / kXcds;
        if (item < n) out.push_back(item);
    }
    return out;
}

void hip_check(hipError_t e, const char *what)
{
    if (e != hipSuccess) throw DeviceError{std::string(what) + ": " + hipGetErrorString(e)};
}

namespace {

// Calls fn with std::integral_constant<int, p> for 1 <= p <= kPmax.
template <class Fn>
void with_order(int p, Fn &&fn)
{
    switch (p) {
    case 1: fn(std::integral_constant<int, 1>{}); break;
    case 2: fn(std::integral_constant<int, 2>{}); break;
    case 3: fn(std::integral_constant<int, 3>{}); break;
    case 4: fn(std::integral_constant<int, 4>{}); break;
    case 5: fn(std::integral_constant<int, 5>{}); break;
    case 6: fn(std::integral_constant<int, 6>{}); break;
    case 7: fn(std::integral_constant<int, 7>{}); break;
    case 8: fn(std::integral_constant<int, 8>{}); break;
    case 9: fn(std::integral_constant<int, 9>{}); break;
    default: fn(std::integral_constant<int, 10>{}); break;
    }
}

// Calls fn with the field chunk and the column tiles of P2M.
template <class Fn>
void with_p2m(int F, int p, Fn &&fn)
{
    auto tiles = [&](auto fc) {
        switch (p2m_tiles(p)) {
        case 1: fn(fc, std::integral_constant<int, 1>{}); break;
        case 2: fn(fc, std::integral_constant<int, 2>{}); break;
        case 3: fn(fc, std::integral_constant<int, 3>{}); break;
        case 4: fn(fc, std::integral_constant<int, 4>{}); break;
        default: fn(fc, std::integral_constant<int, 5>{}); break;
        }
    };
    if (field_chunk(F) == 1)
        tiles(std::integral_constant<int, 1>{});
    else
        tiles(std::integral_constant<int, 4>{});
}
static_assert(p2m_tiles(kPmax) <= 5, "column tiles of P2M");

hipEvent_t pool_event(DevicePlan &dp)
{
    if (dp.events_used == dp.event_pool.size()) {
        hipEvent_t e;
        hip_check(hipEventCreate(&e), "hipEventCreate");
        dp.event_pool.push_back(e);
    }
    return dp.event_pool[dp.events_used++];
}

// Records an event pair around one phase on the evaluation stream; nothing is
// synchronised here.
struct KTimer {
    DevicePlan &dp;
    int slot;
    hipStream_t st;
    hipEvent_t a = nullptr;
    KTimer(DevicePlan &d, int s, hipStream_t stream) : dp(d), slot(s), st(stream)
    {
        if (!dp.timing) return;
        if (dp.spans.size() >= 4096) collect_timing(dp);
        a = pool_event(dp);
        hip_check(hipEventRecord(a, st), "hipEventRecord");
    }
    ~KTimer() noexcept(false)
    {
        if (!dp.timing) return;
        hipEvent_t b = pool_event(dp);
        hip_check(hipEventRecord(b, st), "hipEventRecord");
        dp.spans.push_back({slot, a, b});
    }
};

// Ragged batches evaluated as one merged plan: mesh i's nodal M (device
// [n_i][3]) times scale[i] into rows off[i] .. off[i+1] of the merged M, and
// the merged u back into each mesh's u (device [n_i]).
__device__ __forceinline__ int batch_mesh(const int64_t *__restrict__ off, int n, int64_t j)
{
    int lo = 0, hi = n;  // last i with off[i] <= j
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= j) lo = mid; else hi = mid;
    }
    return lo;
}
__global__ void k_batch_gather(const double *const *__restrict__ M, const int64_t *__restrict__ off,
                               const double *__restrict__ scale, int n, double *__restrict__ out)
{
    const int64_t N = off[n];
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < N; j += (int64_t)gridDim.x * blockDim.x) {
        const int i = batch_mesh(off, n, j);
        const double *m = M[i] + 3 * (j - off[i]);
        const double s = scale[i];
        out[3 * j] = s * m[0];
        out[3 * j + 1] = s * m[1];
        out[3 * j + 2] = s * m[2];
    }
}
__global__ void k_batch_scatter(const double *__restrict__ u, const int64_t *__restrict__ off, int n,
                                double *const *__restrict__ U)
{
    const int64_t N = off[n];
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < N; j += (int64_t)gridDim.x * blockDim.x) {
        const int i = batch_mesh(off, n, j);
        U[i][j - off[i]] = u[j];
    }
}
void fill(double *a, int64_t n, double v, hipStream_t st)
{
    if (n <= 0) return;
    int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
    k_fill<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(a, n, v);
    hip_check(hipGetLastError(), "k_fill launch");
}

template <int FCH, bool WIDE>
void launch_p2p_w(DevicePlan &dp, bool band_skip, int f0, const double *M, double *u, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const unsigned nblk = (unsigned)dp.n_p2p_blk;
    if (nblk == 0) return;
    k_p2p<FCH, WIDE><<<dim3(xcd_grid((int)nblk)), dim3(p2p_threads(FCH, WIDE)), 0, st>>>(
        dp.p2p_blk, (int)nblk, band_skip ? 1 : 0, hp.n_tets, dp.tet_xyz, dp.tet_node, dp.p2p_idx, dp.tgt_xyz,
        dp.tgt_perm, hp.n_targets, M, hp.n_nodes, f0, u);
    hip_check(hipGetLastError(), "k_p2p launch");
}

template <int FCH>
void launch_p2p(DevicePlan &dp, bool band_skip, int f0, const double *M, double *u, hipStream_t st)
{
    if constexpr (FCH <= 2) {
        if (dp.p2p_wide) {
            launch_p2p_w<FCH, true>(dp, band_skip, f0, M, u, st);
            return;
        }
    }
    launch_p2p_w<FCH, false>(dp, band_skip, f0, M, u, st);
}

void run_p2p_points(DevicePlan &dp, bool direct, const double *M, int32_t F, double *u, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const unsigned nblk = direct ? (unsigned)((hp.n_tets + kP2PTets - 1) / kP2PTets) : (unsigned)dp.n_p2p_blk;
    if (nblk == 0) return;
    for (int f = 0; f < F;) {
        const int left = F - f;
#define TFMM_P2P_POINTS(FCV)                                                                                       \
    k_p2p_points<FCV><<<dim3(xcd_grid((int)nblk)), dim3(kPtThreads), 0, st>>>(                                      \
        dp.p2p_blk, (int)nblk, direct ? 1 : 0, hp.n_tets, dp.tet_xyz, dp.tet_node, dp.p2p_idx, dp.tgt_xyz,            \
        dp.tgt_perm, hp.n_targets, M, hp.n_nodes, f, u)
        if (left >= 8) {
            TFMM_P2P_POINTS(8);
            f += 8;
        } else if (left >= 4) {
            TFMM_P2P_POINTS(4);
            f += 4;
        } else if (left >= 2) {
            TFMM_P2P_POINTS(2);
            f += 2;
        } else {
            TFMM_P2P_POINTS(1);
            f += 1;
        }
#undef TFMM_P2P_POINTS
        hip_check(hipGetLastError(), "k_p2p_points launch");
    }
}

// One field over the shared mesh entities.
void run_p2p_topo(DevicePlan &dp, const double *M, double *u, const int32_t *perm, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    if (dp.n_topo_items == 0) return;
    k_topo_coef<<<dim3((unsigned)((dp.n_topo_ch + kTopoChunksPerWave - 1) / kTopoChunksPerWave)), dim3(64), 0, st>>>(
        dp.topo_ch_i, dp.topo_ch_c, dp.n_topo_ch, dp.topo_inc, dp.tet_xyz, dp.tet_node, hp.n_tets, M, dp.topo_edge,
        dp.topo_edge_w, dp.topo_face_w);
    hip_check(hipGetLastError(), "k_topo_coef launch");
    k_p2p_topo<<<dim3(xcd_grid(dp.n_topo_items)), dim3(64), 0, st>>>(
        dp.topo_item, dp.n_topo_items, dp.topo_ch_i, dp.topo_ch_c, dp.topo_w, dp.topo_edge, dp.topo_face,
        dp.topo_edge_w, dp.topo_face_w, dp.p2p_idx, dp.tgt_xyz, perm, hp.n_targets, u);
    hip_check(hipGetLastError(), "k_p2p_topo launch");
}

// Fields of the pass that starts with `left` fields to go: the geometry of a
// pair (about 390 issue slots) costs as much as the fields' part of 65 fields
// (6 slots each), so the next power of two covers what is left, padded, rather
// than two passes; one field alone takes the shared entities.
int near_pass(int left)
{
    int fc = 1;
    while (fc < left && fc < kNearFieldsMax) fc *= 2;
    return fc;
}

// Calls fn with the pass width as an integral constant (2, 4, ..., kNearFieldsMax).
template <class Fn>
void with_near_pass(int fc, Fn &&fn)
{
    switch (fc) {
    case 16: fn(std::integral_constant<int, 16>{}); break;
    case 8: fn(std::integral_constant<int, 8>{}); break;
    case 4: fn(std::integral_constant<int, 4>{}); break;
    default: fn(std::integral_constant<int, 2>{}); break;
    }
}

// Several fields, in passes.
void run_p2p_fields(DevicePlan &dp, const double *M, int32_t F, double *u, const int32_t *perm, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    if (dp.n_topo_items == 0) return;
    for (int f = 0; f < F;) {
        const int fc = near_pass(F - f);
        if (fc == 1) {
            run_p2p_topo(dp, M + (int64_t)f * hp.n_nodes * 3, u + (int64_t)f * hp.n_targets, perm, st);
        } else {
            if (dp.near_w_cap < dp.near_rows * fc) throw DeviceError{"near-field weights not prepared"};
            with_near_pass(fc, [&](auto c) {
                constexpr int FC = decltype(c)::value;
                k_near_weights<FC><<<dim3((unsigned)((hp.n_tets * FC + 255) / 256)), dim3(256), 0, st>>>(
                    dp.near_tet, hp.n_tets, dp.tet_xyz, dp.tet_node, M, hp.n_nodes, f, F, dp.near_w);
                const auto kernel = dp.near_flat ? k_p2p_fields<FC, true> : k_p2p_fields<FC, false>;
                kernel<<<dim3(xcd_grid((dp.n_topo_items + kFieldWaves - 1) / kFieldWaves)), dim3(64 * kFieldWaves), 0, st>>>(
                    dp.topo_item, dp.n_topo_items, dp.topo_ch_i, dp.topo_ch_c, dp.topo_w, dp.near_tet, dp.near_flat,
                    dp.ch_flat, dp.near_w, dp.p2p_idx, dp.tgt_xyz, perm, hp.n_targets, f, F, u);
            });
            hip_check(hipGetLastError(), "k_p2p_fields launch");
        }
        f += fc;
    }
}

// Whether an evaluation keeps its sums in the octree's order (dp.u_tree) and puts
// them in the caller's order at the end: the near field of several fields, whose
// adds (a field and target of every work item) then fall in shared lines.  Whole
// evaluations, caller's order and tree's, us: a 12^3 cube with 5 fields 346 and 349,
// 7 381 and 378, 8 412 and 404, 16 530 and 492; a 21^3 cube with 6 fields 1,693 and
// 1,701, 8 2,006 and 1,999, 16 3,127 and 3,057; with fewer fields the adds are too
// few to pay for the last step.
constexpr int kInOrderFields = 8;
bool near_in_order(const DevicePlan &dp, int32_t F)
{
    return F >= kInOrderFields && !dp.near_stored && !dp.hp.points && dp.sur_mode == TFMM_SUR_OFF && dp.p2p_topo && dp.n_topo_ch > 0;
}

// Near field by the pair integrals: point dipoles (or, direct, the dipole
// sum); one field of tets over the shared mesh entities; otherwise the
// per-tet kernel, without the band's pairs when band_skip.
void run_p2p(DevicePlan &dp, bool direct, const double *M, int32_t F, double *u, hipStream_t st, bool band_skip = false)
{
    if (dp.hp.points) {
        run_p2p_points(dp, direct, M, F, u, st);
        return;
    }
    if (direct) throw DeviceError{"the tet direct sum runs in k_direct"};
    if (!band_skip && dp.p2p_topo && dp.n_topo_ch > 0) {
        if (F == 1)
            run_p2p_topo(dp, M, u, dp.tgt_perm, st);
        else
            run_p2p_fields(dp, M, F, u, near_in_order(dp, F) ? nullptr : dp.tgt_perm, st);
        return;
    }
    int f = 0;
    while (f < F) {
        const int left = F - f;
        if (left >= 32) {
            launch_p2p<32>(dp, band_skip, f, M, u, st);
            f += 32;
        } else if (left >= 16) {
            launch_p2p<16>(dp, band_skip, f, M, u, st);
            f += 16;
        } else if (left >= 8) {
            launch_p2p<8>(dp, band_skip, f, M, u, st);
            f += 8;
        } else if (left >= 4) {
            launch_p2p<4>(dp, band_skip, f, M, u, st);
            f += 4;
        } else if (left >= 2) {
            launch_p2p<2>(dp, band_skip, f, M, u, st);
            f += 2;
        } else {
            launch_p2p<1>(dp, band_skip, f, M, u, st);
            f += 1;
        }
    }
}

// Near field from the stored operator (F fields, FC per pass).
void run_near_stored(DevicePlan &dp, const double *M, int32_t F, double *u, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const int64_t N = hp.n_targets;
    if (N == 0 || dp.near_nvals == 0) return;
    const int ni = dp.near_nitems;
    if (ni == 0) return;
    const int nblk = (ni + kNearItemsPerBlock - 1) / kNearItemsPerBlock;
    const int fc = F >= 8 ? 8 : (F >= 4 ? 4 : (F >= 2 ? 2 : 1));
    const dim3 grid(xcd_grid(nblk), (unsigned)((F + fc - 1) / fc));
    const dim3 thr(64 * kNearItemsPerBlock);
#define TFMM_NEAR_APPLY(FCV)                                                                                       \
    k_near_apply<FCV><<<grid, thr, 0, st>>>(ni, dp.near_items, dp.cell_i, dp.near_off, dp.near_nc, dp.near_cols,    \
                                            dp.near_val, dp.tgt_perm, N, M, hp.n_nodes, F, u)
    switch (fc) {
    case 8: TFMM_NEAR_APPLY(8); break;
    case 4: TFMM_NEAR_APPLY(4); break;
    case 2: TFMM_NEAR_APPLY(2); break;
    default: TFMM_NEAR_APPLY(1); break;
    }
#undef TFMM_NEAR_APPLY
    hip_check(hipGetLastError(), "k_near_apply launch");
}

// Near field of an evaluation: the stored operator when the plan holds one;
// with the surrogate switched on, the exact integrals outside the band and
// the band's pairs by the network (or a control); else the pair integrals.
void run_near(DevicePlan &dp, const double *M, int32_t F, double *u, hipStream_t st)
{
    if (dp.near_stored) {
        run_near_stored(dp, M, F, u, st);
    } else if (dp.sur_mode != TFMM_SUR_OFF && !dp.hp.points) {
        run_p2p(dp, false, M, F, u, st, true);
        run_band_pairs(dp, dp.sur_mode, M, F, u, st);
    } else {
        run_p2p(dp, false, M, F, u, st);
    }
}

template <typename T, int P>
void launch_m2l_p(DevicePlan &dp, const DevicePlan::Tiles &tl, const T *D, const T *Qt, int fpt, int32_t F,
                  hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const unsigned groups = (unsigned)((F + fpt - 1) / fpt);
    k_m2l_mfma<T, P><<<dim3(tl.ntiles, groups), dim3(64 * kM2LWaves), 0, st>>>(
        tl.tile_tgt, tl.tile_rng, tl.ent_key, tl.ent_src, dp.m2l_keys, D, Qt, m2l_tile_row(hp.p),
        (int64_t)hp.cells.size(), tl.tpt, fpt, F, tl.ntiles, m2l_table_width(hp.p), dp.Lr, m2l_nrows(hp.p));
    hip_check(hipGetLastError(), "k_m2l_mfma launch");
}

template <int NP>
void launch_m2lb(DevicePlan &dp, const DevicePlan::Tiles &tl, int fpt, int32_t F, hipStream_t st, int p)
{
    const HostPlan &hp = dp.hp;
    with_order(p, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_m2l_bf16<P, NP><<<dim3(tl.ntiles, (unsigned)((F + fpt - 1) / fpt)), dim3(64), 0, st>>>(
            tl.tile_tgt, tl.tile_rng, tl.ent_key, tl.ent_src, dp.m2l_keys, dp.m2l_Df, m2l_table_width(hp.p),
            reinterpret_cast<const __bf16 *>(dp.Qtf), m2lb_ks(hp.p, 0), (int64_t)hp.cells.size(), tl.tpt, fpt, F, tl.ntiles,
            dp.Lr, m2l_nrows(hp.p));
    });
    hip_check(hipGetLastError(), "k_m2l_bf16 launch");
}

template <typename T>
void launch_m2l_t(DevicePlan &dp, const DevicePlan::Tiles &tl, const T *D, const T *Qt, int fpt, int32_t F,
                  hipStream_t st, int p)
{
    switch (p) {
    case 1: launch_m2l_p<T, 1>(dp, tl, D, Qt, fpt, F, st); break;
    case 2: launch_m2l_p<T, 2>(dp, tl, D, Qt, fpt, F, st); break;
    case 3: launch_m2l_p<T, 3>(dp, tl, D, Qt, fpt, F, st); break;
    case 4: launch_m2l_p<T, 4>(dp, tl, D, Qt, fpt, F, st); break;
    case 5: launch_m2l_p<T, 5>(dp, tl, D, Qt, fpt, F, st); break;
    case 6: launch_m2l_p<T, 6>(dp, tl, D, Qt, fpt, F, st); break;
    case 7: launch_m2l_p<T, 7>(dp, tl, D, Qt, fpt, F, st); break;
    case 8: launch_m2l_p<T, 8>(dp, tl, D, Qt, fpt, F, st); break;
    case 9: launch_m2l_p<T, 9>(dp, tl, D, Qt, fpt, F, st); break;
    case 10: launch_m2l_p<T, 10>(dp, tl, D, Qt, fpt, F, st); break;
    default: throw DeviceError{"unsupported expansion order"};
    }
}

int pack_cut(const DevicePlan &dp, const DevicePlan::Packs &k, int32_t F)
{
    return m2l_pack_cut(k.npairs, 16 / k.tpg, F, dp.m2l_max_grp);
}

// The work items of list k for F fields, null if they were not made.
const DevicePlan::Packs::Items *pack_items(const DevicePlan &dp, const DevicePlan::Packs &k, int32_t F)
{
    const int cut = pack_cut(dp, k, F);
    for (const auto &it : k.items)
        if (it.cut == cut) return &it;
    return nullptr;
}

// The translations of one pack list at order p (the plan's or a level's).
void launch_m2l_pack(DevicePlan &dp, const DevicePlan::Packs &k, int fpt, int32_t F, hipStream_t st, int p)
{
    const HostPlan &hp = dp.hp;
    const DevicePlan::Packs::Items *it = pack_items(dp, k, F);
    if (!it) throw DeviceError{"M2L work items not prepared"};
    if (it->n == 0) return;
    if (k.nb * fpt != m2l_pack_slots(p) || k.tpg * fpt != 16 || k.p != p)
        throw DeviceError{"M2L packs do not match the translation order"};
    const unsigned groups = (unsigned)((F + fpt - 1) / fpt);
    with_order(p, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_m2l_pack<P><<<dim3((unsigned)it->n, groups), dim3(64 * kM2LPWaves), 0, st>>>(
            it->item, it->n, k.blk_cells, k.nb, k.tpg, k.grp_key, k.grp_src, k.grp_slot, dp.m2l_keys, dp.m2l_D,
            m2l_table_width(hp.p), dp.Qt, dp.qpad, (int64_t)hp.cells.size(), fpt, F, dp.Lr, m2l_nrows(hp.p));
    });
    hip_check(hipGetLastError(), "k_m2l_pack launch");
}

// Scaled multipoles, then the translations, in the plan's M2L precision.
// Field tile width of M2L for F fields: FPT fields x 16/FPT target cells.
int m2l_fpt(int32_t F)
{
    int fpt = 1;
    while (fpt * 2 <= std::min<int32_t>(F, 16)) fpt *= 2;
    return fpt;
}

// Field width of the packed form for F fields: the width whose passes carry the
// fewest padded fields, the widest among equals.  Whole evaluations, this width and
// the largest power of two below F, us: a 12^3 cube with 3 fields 294 and 311, 7 380
// and 402, 9 433 and 495, 13 492 and 526; a 21^3 cube with 3 fields 1,169 and 1,298,
// 7 1,975 and 1,943, 9 2,408 and 2,966, 13 2,951 and 3,118.
int m2l_pack_fpt(int32_t F)
{
    int best = 1;
    for (int fpt = 2; fpt <= 8; fpt *= 2)
        if ((F + fpt - 1) / fpt * fpt <= (F + best - 1) / best * best) best = fpt;
    return best;
}

// Whether M2L runs in the packed form: FP64 translations of fewer than 16
// fields (the tiles of 16 or more fields carry one target cell x 16 fields,
// every column used; the FP32 and split-BF16 tiles are faster than their
// packed forms, whose few matrix-core cycles per group leave the LDS
// accumulation as the bound).
bool m2l_packed(const DevicePlan &dp, int32_t F)
{
    return dp.m2l_pack && m2l_fpt(F) < 16 && dp.m2l_precision == TFMM_M2L_FP64;
}

// Row form of the reduced multipoles of an evaluation of F fields (see k_qreduce).
struct QRows {
    int form, len, fpt, np;
    int64_t count;  // numbers of all fields and cells (np parts of BF16 each)
};
static QRows q_rows(const DevicePlan &dp, int32_t F)
{
    const int64_t C = (int64_t)dp.hp.cells.size();
    if (m2l_packed(dp, F)) return {ROW_PLAIN, dp.qpad, 1, 1, F * C * dp.qpad};
    const int fpt = m2l_fpt(F);
    const int64_t cells = (int64_t)((F + fpt - 1) / fpt) * fpt * C;
    if (dp.m2l_precision <= TFMM_M2L_FP32) return {ROW_TILE, m2l_tile_row(dp.hp.p), fpt, 1, cells * m2l_tile_row(dp.hp.p)};
    const int len = 32 * m2lb_ks(dp.hp.p, 0);
    return {ROW_BF16, len, fpt, dp.m2l_precision == TFMM_M2L_BF16X3 ? 2 : 3, cells * len};
}
// elements of the buffer they take: doubles of Qt or floats of Qtf
static int64_t q_elems(const QRows &q) { return q.form == ROW_BF16 ? (q.count * q.np + 1) / 2 : q.count; }
// elements that any form of up to F fields takes in Qt (fp64) or Qtf
static int64_t q_room(const DevicePlan &dp, int32_t F, bool fp64)
{
    const int fpt = m2l_fpt(F);
    const int64_t C = (int64_t)dp.hp.cells.size(), cells = (int64_t)((F + fpt - 1) / fpt) * fpt * C;
    const int64_t tile = cells * m2l_tile_row(dp.hp.p);
    return std::max<int64_t>(tile, fp64 ? F * C * dp.qpad : (cells * 32 * m2lb_ks(dp.hp.p, 0) * 3 + 1) / 2);
}
int m2l_pack_slot(int fpt)
{
    int s = 0;
    while ((1 << s) < fpt) ++s;
    return s;
}

// The translations of one tile list at order p in the plan's M2L precision.
void launch_m2l_tiles(DevicePlan &dp, const DevicePlan::Tiles &tl, int fpt, int32_t F, hipStream_t st, int p)
{
    if (tl.ntiles == 0) return;
    if (dp.m2l_precision == TFMM_M2L_BF16X3)
        launch_m2lb<2>(dp, tl, fpt, F, st, p);
    else if (dp.m2l_precision == TFMM_M2L_BF16X6)
        launch_m2lb<3>(dp, tl, fpt, F, st, p);
    else if (dp.m2l_precision == TFMM_M2L_FP32)
        launch_m2l_t<float>(dp, tl, dp.m2l_Df, dp.Qtf, fpt, F, st, p);
    else
        launch_m2l_t<double>(dp, tl, dp.m2l_D, dp.Qt, fpt, F, st, p);
}

void run_m2l(DevicePlan &dp, int32_t F, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const int64_t C = (int64_t)hp.cells.size();
    if (hp.m2l_src.empty()) {
        fill(dp.L, (int64_t)F * C * dp.ncoef, 0.0, st);
        return;
    }
    const bool fp64 = dp.m2l_precision == TFMM_M2L_FP64;
    const QRows q = q_rows(dp, F);
    if (dp.lr_cap < F || (fp64 ? dp.qt_cap : dp.qtf_cap) < q_elems(q) || (!fp64 && !dp.m2l_Df))
        throw DeviceError{"M2L buffers not prepared"};
    const int cells = row_cells(C, F), lrs = m2l_nrows(hp.p);
    const dim3 rgrid((unsigned)((C + cells - 1) / cells), F);
    constexpr ReduceTable rt = make_reduce();
    const size_t rlds = row_lds(dp.ncoef, rt.start[nr_of(hp.p)], nr_of(hp.p));
    auto reduce = [&](auto form, auto *rows) {
        k_qreduce<decltype(form)::value><<<rgrid, dim3(256), rlds, st>>>(dp.Q, dp.cell_i, C, hp.side, hp.p, q.len, q.fpt, q.np,
                                                                         rows, dp.Lr, lrs, cells);
    };
    if (q.form == ROW_PLAIN)
        reduce(std::integral_constant<int, ROW_PLAIN>{}, dp.Qt);
    else if (q.form == ROW_BF16)
        reduce(std::integral_constant<int, ROW_BF16>{}, reinterpret_cast<__bf16 *>(dp.Qtf));
    else if (fp64)
        reduce(std::integral_constant<int, ROW_TILE>{}, dp.Qt);
    else
        reduce(std::integral_constant<int, ROW_TILE>{}, dp.Qtf);
    hip_check(hipGetLastError(), "k_qreduce launch");
    // with per-level orders, one launch per target level at that level's order
    // (the source multipoles already hold no terms above their own level's)
    if (q.form == ROW_PLAIN) {
        const int fpt = m2l_pack_fpt(F);
        auto go = [&](const DevicePlan::Packs &k, int p) { launch_m2l_pack(dp, k, fpt, F, st, p); };
        if (!dp.level_orders) {
            go(dp.m2l_packs[m2l_pack_slot(fpt)], hp.p);
        } else {
            for (size_t lv = 0; lv < dp.lvl_packs.size(); ++lv) go(dp.lvl_packs[lv], dp.lo.q[lv]);
        }
    } else if (!dp.level_orders) {
        launch_m2l_tiles(dp, ensure_m2l_tiles(dp, 16 / q.fpt), q.fpt, F, st, hp.p);
    } else {
        const std::vector<DevicePlan::Tiles> &lt = ensure_m2l_level_tiles(dp, 16 / q.fpt);
        for (size_t lv = 0; lv < lt.size(); ++lv) launch_m2l_tiles(dp, lt[lv], q.fpt, F, st, dp.lo.q[lv]);
    }
    constexpr ExpandTable et = make_expand();
    const int nm = ncoef_of(hp.p - 1);
    k_lr_expand<<<rgrid, dim3(256), row_lds(lrs, et.start[nm], nm), st>>>(dp.Lr, lrs, dp.cell_i, hp.side, C, hp.p, dp.lo,
                                                                          cells, dp.L);
    hip_check(hipGetLastError(), "k_lr_expand launch");
}

}  // namespace

void batch_gather(const double *const *M, const int64_t *off, const double *scale, int n, int64_t N, double *out,
                  hipStream_t st)
{
    if (N <= 0) return;
    k_batch_gather<<<dim3((unsigned)std::min<int64_t>((N + 255) / 256, 65536)), dim3(256), 0, st>>>(M, off, scale, n,
                                                                                                   out);
    hip_check(hipGetLastError(), "k_batch_gather launch");
}
void batch_scatter(const double *u, const int64_t *off, int n, int64_t N, double *const *U, hipStream_t st)
{
    if (N <= 0) return;
    k_batch_scatter<<<dim3((unsigned)std::min<int64_t>((N + 255) / 256, 65536)), dim3(256), 0, st>>>(u, off, n, U);
    hip_check(hipGetLastError(), "k_batch_scatter launch");
}


void store_near(DevicePlan &dp, hipStream_t st)
{
    if (dp.near_stored) return;
    const HostPlan &hp = dp.hp;
    NearOpLayout lay;
    build_near_operator_layout(hp, lay);
    const size_t C = hp.cells.size();
    const size_t b_off = sizeof(int64_t) * 2 * std::max<size_t>(C, 1), b_nc = sizeof(int32_t) * std::max<size_t>(C, 1),
                 b_cols = sizeof(int32_t) * std::max<size_t>(lay.cols.size(), 1),
                 b_val = sizeof(double) * (size_t)std::max<int64_t>(lay.nvals, 1);
    // apply work items: (leaf, first row) per kNearRows rows of a leaf block
    std::vector<int32_t> items;
    for (size_t a = 0; a < C; ++a) {
        if (lay.leaf_off[2 * a + 1] < 0) continue;
        const Cell &K = hp.cells[a];
        for (int32_t r = 0; r < K.xend - K.xbeg; r += kNearRows) {
            items.push_back((int32_t)a);
            items.push_back(r);
        }
    }
    const size_t b_items = sizeof(int32_t) * std::max<size_t>(items.size(), 1);
    void *p[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
    const size_t sz[5] = {b_off, b_nc, b_cols, b_val, b_items};
    for (int i = 0; i < 5; ++i) {
        const hipError_t e = hipMalloc(&p[i], sz[i]);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            for (int j = 0; j < i; ++j) (void)hipFree(p[j]);
            if (e == hipErrorOutOfMemory)
                throw PlanError{TFMM_ENOMEM, "stored near-field operator: device memory exhausted (" +
                                                 std::to_string(b_val >> 20) + " MiB of coefficients)"};
            hip_check(e, "hipMalloc near operator");
        }
    }
    dp.near_off = (int64_t *)p[0];
    dp.near_nc = (int32_t *)p[1];
    dp.near_cols = (int32_t *)p[2];
    dp.near_val = (double *)p[3];
    dp.near_items = (int32_t *)p[4];
    dp.near_nitems = (int32_t)(items.size() / 2);
    dp.near_nvals = lay.nvals;
    dp.near_ncols = (int64_t)lay.cols.size();
    dp.near_nnz = lay.nnz;
    dp.near_bytes = (int64_t)(b_off + b_nc + b_cols + b_val + b_items);
    dp.device_bytes += dp.near_bytes;
    try {
        if (!items.empty())
            hip_check(hipMemcpy(dp.near_items, items.data(), sizeof(int32_t) * items.size(), hipMemcpyHostToDevice),
                      "hipMemcpy near items");
        hip_check(hipMemcpy(dp.near_off, lay.leaf_off.data(), sizeof(int64_t) * lay.leaf_off.size(), hipMemcpyHostToDevice),
                  "hipMemcpy near offsets");
        hip_check(hipMemcpy(dp.near_nc, lay.leaf_nc.data(), sizeof(int32_t) * lay.leaf_nc.size(), hipMemcpyHostToDevice),
                  "hipMemcpy near counts");
        if (!lay.cols.empty())
            hip_check(hipMemcpy(dp.near_cols, lay.cols.data(), sizeof(int32_t) * lay.cols.size(), hipMemcpyHostToDevice),
                      "hipMemcpy near columns");
        fill(dp.near_val, lay.nvals, 0.0, st);
        if (dp.n_p2p_blk > 0) {
            k_near_assemble<<<dim3(xcd_grid(dp.n_p2p_blk)), dim3(kNearAsmThreads), 0, st>>>(
                dp.p2p_blk, dp.n_p2p_blk, hp.n_tets, dp.tet_xyz, dp.tet_node, dp.p2p_idx, dp.tgt_xyz, hp.n_targets,
                dp.tgt_leaf, dp.cell_i, dp.near_off, dp.near_nc, dp.near_cols, dp.near_val);
            hip_check(hipGetLastError(), "k_near_assemble launch");
        }
        hip_check(hipStreamSynchronize(st), "hipStreamSynchronize (near operator)");
    } catch (...) {
        drop_near(dp);  // a failed assembly leaves no operator behind
        throw;
    }
    dp.near_stored = true;
    ++dp.schedule_gen;
}

void drop_near(DevicePlan &dp)
{
    if (!dp.near_off) return;
    (void)hipDeviceSynchronize();  // also called on a failure path: freeing must not throw
    void *p[5] = {dp.near_off, dp.near_nc, dp.near_cols, dp.near_val, dp.near_items};
    for (void *q : p)
        if (q) (void)hipFree(q);
    dp.near_items = nullptr;
    dp.near_nitems = 0;
    dp.near_off = nullptr;
    dp.near_nc = nullptr;
    dp.near_cols = nullptr;
    dp.near_val = nullptr;
    dp.device_bytes -= dp.near_bytes;
    dp.near_bytes = dp.near_nvals = dp.near_ncols = dp.near_nnz = 0;
    dp.near_stored = false;
    ++dp.schedule_gen;
}

void build_tet_moments(DevicePlan &dp)
{
    if (dp.n_p2m_cells == 0) return;
    k_tet_moments<<<dim3(dp.n_p2m_cells), dim3(kMomThreads)>>>(dp.p2m_cells, dp.cell_i, dp.cell_c,
                                                               (int64_t)dp.hp.cells.size(), dp.tet_xyz, dp.hp.n_tets,
                                                               dp.quad, dp.nq, dp.hp.p, dp.hp.points ? 1 : 0,
                                                               dp.tet_mom);
    hip_check(hipGetLastError(), "k_tet_moments launch");
    hip_check(hipDeviceSynchronize(), "k_tet_moments");
}

void build_topo_records(DevicePlan &dp, const int32_t *ab, const int32_t *pqr)
{
    if (dp.n_topo_ch == 0) return;
    k_topo_static<<<dim3((unsigned)dp.n_topo_ch), dim3(64)>>>(dp.topo_ch_i, dp.n_topo_ch, dp.topo_w, ab, pqr,
                                                              dp.topo_edge, dp.topo_face);
    hip_check(hipGetLastError(), "k_topo_static launch");
    hip_check(hipDeviceSynchronize(), "k_topo_static");
}

int32_t build_near_tets(const DevicePlan &dp, const uint32_t *corner, const uint8_t *skin, const int64_t *row, NearTet *tet,
                        uint32_t *ch_flat)
{
    if (dp.n_topo_ch == 0) return 0;
    // tets outside every block (leaves without near targets) keep row -1
    hip_check(hipMemset(tet, 0xff, sizeof(NearTet) * (size_t)dp.hp.n_tets), "hipMemset near-field tets");
    int32_t *count = nullptr, n = 0;
    hip_check(hipMalloc(&count, sizeof(n)), "hipMalloc flat tets");
    hipError_t e = hipMemcpy(count, &n, sizeof(n), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        k_tet_static<<<dim3((unsigned)dp.n_topo_ch), dim3(64)>>>(dp.topo_ch_i, dp.topo_ch_c, dp.n_topo_ch, dp.tet_xyz,
                                                                 dp.hp.n_tets, skin, row, corner, tet, ch_flat, count);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(&n, count, sizeof(n), hipMemcpyDeviceToHost);
    (void)hipFree(count);
    hip_check(e, "k_tet_static");
    return n;
}

void build_near_flat(const DevicePlan &dp, const NearTet *tet, NearFlat *flat)
{
    k_flat_static<<<dim3((unsigned)dp.n_topo_ch), dim3(64)>>>(dp.topo_ch_i, dp.topo_ch_c, dp.n_topo_ch, dp.tet_xyz,
                                                              dp.hp.n_tets, tet, flat);
    hip_check(hipGetLastError(), "k_flat_static launch");
    hip_check(hipDeviceSynchronize(), "k_flat_static");
}

void build_m2l_table(DevicePlan &dp)
{
    if (dp.n_m2l_keys == 0) return;
    k_m2l_table<<<dim3((dp.n_m2l_keys + 63) / 64), dim3(64)>>>(dp.m2l_keys, dp.n_m2l_keys, dp.hp.p, dp.m2l_D);
    hip_check(hipGetLastError(), "k_m2l_table launch");
    hip_check(hipDeviceSynchronize(), "k_m2l_table");
}

static void free_tiles(DevicePlan &dp, DevicePlan::Tiles &t)
{
    for (int32_t *q : {t.tile_tgt, t.tile_rng, t.ent_key, t.ent_src})
        if (q) (void)hipFree(q);
    dp.device_bytes -= t.bytes;
    t = DevicePlan::Tiles{};
}

static void upload_tiles(DevicePlan &dp, const M2LTiles &h, int tpt, DevicePlan::Tiles &t)
{
    auto up = [&](const std::vector<int32_t> &v, int32_t *&d) {
        const size_t b = sizeof(int32_t) * std::max<size_t>(v.size(), 1);
        hip_check(hipMalloc(&d, b), "hipMalloc M2L tiles");
        t.bytes += (int64_t)b;
        dp.device_bytes += (int64_t)b;
        if (!v.empty())
            hip_check(hipMemcpy(d, v.data(), sizeof(int32_t) * v.size(), hipMemcpyHostToDevice), "hipMemcpy M2L tiles");
    };
    up(h.tile_tgt, t.tile_tgt);
    up(h.tile_rng, t.tile_rng);
    up(h.ent_key, t.ent_key);
    up(h.ent_src, t.ent_src);
    t.ntiles = (int32_t)(h.tile_rng.size() / 2);
    t.nent = (int64_t)h.ent_key.size();
    t.tpt = tpt;
    t.max_ent = dp.m2l_max_ent;
}

DevicePlan::Tiles &ensure_m2l_tiles(DevicePlan &dp, int tpt)
{
    int slot = 0;
    while ((16 >> slot) != tpt && slot < 4) ++slot;
    if ((16 >> slot) != tpt) throw DeviceError{"bad M2L tile width"};
    DevicePlan::Tiles &t = dp.m2l_tiles[slot];
    if (t.tpt == tpt && t.max_ent == dp.m2l_max_ent) return t;
    // a captured graph may hold the old tile pointers
    ++dp.schedule_gen;
    free_tiles(dp, t);
    M2LTiles h;
    build_m2l_tiles(dp.hp, tpt, dp.m2l_max_ent, h);
    upload_tiles(dp, h, tpt, t);
    return t;
}

void drop_m2l_level_tiles(DevicePlan &dp)
{
    if (!dp.lvl_tiles.empty()) ++dp.schedule_gen;  // a captured graph may hold them
    for (auto &t : dp.lvl_tiles) free_tiles(dp, t);
    dp.lvl_tiles.clear();
}

const std::vector<DevicePlan::Tiles> &ensure_m2l_level_tiles(DevicePlan &dp, int tpt)
{
    if (!dp.lvl_tiles.empty() && dp.lvl_tiles[0].tpt == tpt && dp.lvl_tiles[0].max_ent == dp.m2l_max_ent)
        return dp.lvl_tiles;
    drop_m2l_level_tiles(dp);
    ++dp.schedule_gen;
    dp.lvl_tiles.resize((size_t)dp.hp.depth + 1);
    for (int lv = 0; lv <= dp.hp.depth; ++lv) {
        M2LTiles h;
        build_m2l_tiles(dp.hp, tpt, dp.m2l_max_ent, h, lv);
        upload_tiles(dp, h, tpt, dp.lvl_tiles[lv]);
    }
    return dp.lvl_tiles;
}

static void free_pack_items(DevicePlan &dp, DevicePlan::Packs &k)
{
    for (auto &it : k.items) {
        if (it.item) (void)hipFree(it.item);
        const int64_t b = (int64_t)(3 * sizeof(int32_t)) * it.n;
        k.bytes -= b;
        dp.device_bytes -= b;
    }
    k.items.clear();
}

static void free_packs(DevicePlan &dp, DevicePlan::Packs &k)
{
    free_pack_items(dp, k);
    void *q[] = {k.blk_cells, k.grp_key, k.grp_src, k.grp_slot};
    for (void *x : q)
        if (x) (void)hipFree(x);
    dp.device_bytes -= k.bytes;
    k = DevicePlan::Packs{};
}

void free_m2l_packs(DevicePlan &dp)
{
    bool any = !dp.lvl_packs.empty();
    for (auto &k : dp.m2l_packs) {
        any = any || k.nb != 0;
        free_packs(dp, k);
    }
    for (auto &k : dp.lvl_packs) free_packs(dp, k);
    dp.lvl_packs.clear();
    if (any) ++dp.schedule_gen;  // a captured graph may hold them
}

template <typename E>
static void upload_pack_list(DevicePlan &dp, DevicePlan::Packs &k, const std::vector<E> &v, E *&d)
{
    const size_t b = sizeof(E) * std::max<size_t>(v.size(), 1);
    hip_check(hipMalloc(&d, b), "hipMalloc M2L packs");
    k.bytes += (int64_t)b;
    dp.device_bytes += (int64_t)b;
    if (!v.empty()) hip_check(hipMemcpy(d, v.data(), sizeof(E) * v.size(), hipMemcpyHostToDevice), "hipMemcpy M2L packs");
}

// Packs of fpt fields for translations of order p (all levels, or one).
static void build_packs(DevicePlan &dp, int fpt, int p, int only_level, DevicePlan::Packs &k)
{
    M2LPacks h;
    build_m2l_packs(dp.hp, m2l_pack_slots(p) / fpt, 16 / fpt, h, only_level);
    upload_pack_list(dp, k, h.blk_cells, k.blk_cells);
    upload_pack_list(dp, k, h.grp_key, k.grp_key);
    upload_pack_list(dp, k, h.grp_src, k.grp_src);
    upload_pack_list(dp, k, h.grp_slot, k.grp_slot);
    k.blk_grp.swap(h.blk_grp);
    k.nb = h.nb;
    k.tpg = h.tpg;
    k.p = p;
    k.ngrp = (int64_t)h.grp_key.size();
    k.npairs = h.npairs;
}

// The work items of list k for F fields; those of another schedule's cap are freed.
static void ensure_pack_items(DevicePlan &dp, DevicePlan::Packs &k, int32_t F)
{
    if (k.max_grp != dp.m2l_max_grp) {
        if (!k.items.empty()) ++dp.schedule_gen;  // a captured graph may hold them
        free_pack_items(dp, k);
        k.max_grp = dp.m2l_max_grp;
    }
    if (pack_items(dp, k, F)) return;
    const int cut = pack_cut(dp, k, F);
    const std::vector<int32_t> h = m2l_pack_items(k.blk_grp, cut);
    k.items.push_back({0, nullptr, 0});
    DevicePlan::Packs::Items &it = k.items.back();
    if (!h.empty()) {
        hip_check(hipMalloc(&it.item, sizeof(int32_t) * h.size()), "hipMalloc M2L work items");
        it.n = (int32_t)(h.size() / 3);
        k.bytes += (int64_t)(sizeof(int32_t) * h.size());
        dp.device_bytes += (int64_t)(sizeof(int32_t) * h.size());
        hip_check(hipMemcpy(it.item, h.data(), sizeof(int32_t) * h.size(), hipMemcpyHostToDevice), "hipMemcpy M2L work items");
    }
    it.cut = cut;  // last: found only when complete
}

static void ensure_m2l_packs(DevicePlan &dp, int32_t F)
{
    if (!m2l_packed(dp, F)) return;
    const HostPlan &hp = dp.hp;
    const int fpt = m2l_pack_fpt(F);
    if (!dp.level_orders) {
        DevicePlan::Packs &k = dp.m2l_packs[m2l_pack_slot(fpt)];
        if (k.nb == 0 || k.p != hp.p) {
            ++dp.schedule_gen;
            free_packs(dp, k);
            build_packs(dp, fpt, hp.p, -1, k);
        }
        ensure_pack_items(dp, k, F);
    } else {
        bool ok = dp.lvl_packs.size() == (size_t)hp.depth + 1;
        for (size_t lv = 0; ok && lv < dp.lvl_packs.size(); ++lv) {
            const DevicePlan::Packs &k = dp.lvl_packs[lv];
            ok = k.tpg * fpt == 16 && k.p == dp.lo.q[lv];
        }
        if (!ok) {
            ++dp.schedule_gen;
            for (auto &k : dp.lvl_packs) free_packs(dp, k);
            dp.lvl_packs.assign((size_t)hp.depth + 1, DevicePlan::Packs{});
            for (int lv = 0; lv <= hp.depth; ++lv) build_packs(dp, fpt, dp.lo.q[lv], lv, dp.lvl_packs[lv]);
        }
        for (auto &k : dp.lvl_packs) ensure_pack_items(dp, k, F);
    }
}

void collect_timing(DevicePlan &dp)
{
    for (const auto &sp : dp.spans) {
        hip_check(hipEventSynchronize(sp.b), "hipEventSynchronize");
        float ms = 0.f;
        hip_check(hipEventElapsedTime(&ms, sp.a, sp.b), "hipEventElapsedTime");
        dp.kt_ms[sp.slot] += ms;
        dp.kt_n[sp.slot] += 1;
    }
    dp.spans.clear();
    dp.events_used = 0;
}

void reset_timing(DevicePlan &dp)
{
    dp.spans.clear();
    dp.events_used = 0;
    for (int i = 0; i < KT_COUNT; ++i) {
        dp.kt_ms[i] = 0.0;
        dp.kt_n[i] = 0;
    }
}

void ensure_expansions(DevicePlan &dp, int32_t F)
{
    if (F <= dp.Fcap) return;
    ++dp.schedule_gen;  // a captured graph may hold the old Q and L
    if (dp.Q) (void)hipFree(dp.Q);
    if (dp.L) (void)hipFree(dp.L);
    dp.Q = dp.L = nullptr;
    dp.Fcap = 0;
    const size_t bytes = sizeof(double) * (size_t)F * dp.hp.cells.size() * dp.ncoef;
    hip_check(hipMalloc(&dp.Q, bytes), "hipMalloc Q");
    hip_check(hipMalloc(&dp.L, bytes), "hipMalloc L");
    // an evaluation writes the multipoles of every cell that holds sources; the others' stay 0
    fill(dp.Q, (int64_t)(bytes / sizeof(double)), 0.0, nullptr);
    hip_check(hipStreamSynchronize(nullptr), "clear Q");
    dp.Fcap = F;
}

int64_t evaluation_bytes(const DevicePlan &dp)
{
    const int64_t C = (int64_t)dp.hp.cells.size(), nd = (int64_t)dp.n_m2l_keys * nd_of(dp.hp.p);
    const int64_t doubles = 2 * dp.Fcap * C * dp.ncoef                 // Q, L
                            + dp.lr_cap * C * m2l_nrows(dp.hp.p)       // Lr
                            + (dp.Qt ? dp.qt_cap + 2 : 0)              // Qt
                            + dp.near_w_cap + dp.u_cap * dp.hp.n_targets;
    return (int64_t)sizeof(double) * doubles + (int64_t)sizeof(float) * (dp.qtf_cap + (dp.m2l_Df ? nd : 0));
}

void prepare_evaluate(DevicePlan &dp, int32_t F)
{
    const int64_t C = (int64_t)dp.hp.cells.size();
    if (dp.sur_mode != TFMM_SUR_OFF && !dp.hp.points && !dp.near_stored) {
        if (dp.sur_mode == TFMM_SUR_MLP && !dp.sur_wb)
            throw PlanError{TFMM_EINVAL, "the surrogate is switched on but no network is attached"};
        build_band_list(dp, nullptr);
    }
    if (!dp.side) {
        hip_check(hipStreamCreateWithFlags(&dp.side, hipStreamNonBlocking), "hipStreamCreate");
        hip_check(hipEventCreateWithFlags(&dp.ev_fork, hipEventDisableTiming), "hipEventCreate");
        hip_check(hipEventCreateWithFlags(&dp.ev_join, hipEventDisableTiming), "hipEventCreate");
    }
    ensure_expansions(dp, F);
    // Every buffer is made for the most fields yet and for every form of them, so that
    // one in use is only ever replaced where the expansions are, on more fields: a
    // graph that a caller captured stays good through other settings of the plan.
    const int32_t most = dp.Fcap;
    const bool several = F > 1 && !dp.near_stored && dp.sur_mode == TFMM_SUR_OFF && dp.p2p_topo;
    if (several) ensure_near_tets(dp);
    if (several && dp.near_w_cap < dp.near_rows * near_pass(most)) {
        ++dp.schedule_gen;  // a captured graph may hold the old weights
        if (dp.near_w) (void)hipFree(dp.near_w);
        dp.near_w = nullptr;
        dp.near_w_cap = 0;
        hip_check(hipMalloc(&dp.near_w, sizeof(double) * (size_t)(dp.near_rows * near_pass(most))), "hipMalloc near weights");
        dp.near_w_cap = dp.near_rows * near_pass(most);
    }
    if (near_in_order(dp, F) && dp.u_cap < most) {
        ++dp.schedule_gen;  // a captured graph may hold the old potentials
        if (dp.u_tree) (void)hipFree(dp.u_tree);
        dp.u_tree = nullptr;
        dp.u_cap = 0;
        hip_check(hipMalloc(&dp.u_tree, sizeof(double) * (size_t)most * std::max<int64_t>(1, dp.hp.n_targets)),
                  "hipMalloc potentials");
        dp.u_cap = most;
    }
    if (m2l_packed(dp, F)) {
        ensure_m2l_packs(dp, F);
    } else {
        ensure_m2l_tiles(dp, 16 / m2l_fpt(F));
        if (dp.level_orders) ensure_m2l_level_tiles(dp, 16 / m2l_fpt(F));
    }
    if (dp.lr_cap < most) {
        ++dp.schedule_gen;
        if (dp.Lr) (void)hipFree(dp.Lr);
        dp.Lr = nullptr;
        dp.lr_cap = 0;
        hip_check(hipMalloc(&dp.Lr, sizeof(double) * (size_t)most * C * m2l_nrows(dp.hp.p)), "hipMalloc Lr");
        dp.lr_cap = most;
    }
    const bool fp64 = dp.m2l_precision == TFMM_M2L_FP64;
    const int64_t room = q_room(dp, most, fp64);
    if (!fp64) {
        if (!dp.m2l_Df) {
            ++dp.schedule_gen;
            const int64_t n = (int64_t)dp.n_m2l_keys * nd_of(dp.hp.p);
            hip_check(hipMalloc(&dp.m2l_Df, sizeof(float) * std::max<int64_t>(n, 1)), "hipMalloc M2L table f32");
            k_to_float<<<dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 65536))), dim3(256)>>>(
                dp.m2l_D, n, dp.m2l_Df);
            hip_check(hipGetLastError(), "k_to_float launch");
            hip_check(hipDeviceSynchronize(), "k_to_float");
        }
        if (dp.qtf_cap < room) {
            ++dp.schedule_gen;
            if (dp.Qtf) (void)hipFree(dp.Qtf);
            dp.Qtf = nullptr;
            dp.qtf_cap = 0;
            hip_check(hipMalloc(&dp.Qtf, sizeof(float) * (size_t)room), "hipMalloc Qt f32");
            dp.qtf_cap = room;
        }
    } else if (dp.qt_cap < room) {
        ++dp.schedule_gen;
        if (dp.Qt) (void)hipFree(dp.Qt - 1);
        dp.Qt = nullptr;
        dp.qt_cap = 0;
        hip_check(hipMalloc(&dp.Qt, sizeof(double) * (size_t)(room + 2)), "hipMalloc Qt");
        dp.Qt += 1;  // entry 1 of every plain row (the first that counts) on a 16-byte boundary
        dp.qt_cap = room;
    }
}

// Times one configuration: the median of three evaluations (after one warm
// evaluation) with events on st.
static float time_config(DevicePlan &dp, const double *M, double *u, hipStream_t st)
{
    prepare_evaluate(dp, 1);
    run_evaluate(dp, M, 1, u, st);
    hipEvent_t a, b;
    hip_check(hipEventCreate(&a), "hipEventCreate");
    hip_check(hipEventCreate(&b), "hipEventCreate");
    float ms[3];
    for (float &m : ms) {
        hip_check(hipEventRecord(a, st), "hipEventRecord");
        run_evaluate(dp, M, 1, u, st);
        hip_check(hipEventRecord(b, st), "hipEventRecord");
        hip_check(hipEventSynchronize(b), "hipEventSynchronize");
        hip_check(hipEventElapsedTime(&m, a, b), "hipEventElapsedTime");
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    std::sort(ms, ms + 3);
    return ms[1];
}

void autotune(DevicePlan &dp, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    double *M = nullptr, *u = nullptr;
    hip_check(hipMalloc(&M, sizeof(double) * 3 * std::max<int64_t>(hp.n_nodes, 1)), "hipMalloc tuning M");
    if (hipMalloc(&u, sizeof(double) * std::max<int64_t>(hp.n_targets, 1)) != hipSuccess) {
        (void)hipFree(M);
        throw DeviceError{"hipMalloc tuning u failed"};
    }
    const bool timing = dp.timing;
    dp.timing = false;
    try {
        fill(M, 3 * hp.n_nodes, 1.0, st);
        // M2L form and work item size, then the P2P workgroup shape; every
        // candidate computes the same contraction, only the schedule differs
        int best_ent = dp.m2l_max_ent, best_grp = dp.m2l_max_grp;
        bool best_pack = false;
        float best = -1.f;
        dp.m2l_pack = false;
        for (int ent : {128, 256, 512, 1024}) {
            dp.m2l_max_ent = ent;
            const float t = time_config(dp, M, u, st);
            if (best < 0.f || t < best) best = t, best_ent = ent;
        }
        dp.m2l_max_ent = best_ent;
        dp.m2l_pack = true;
        if (m2l_packed(dp, 1)) {
            // caps with the same cuts are one schedule, known by the plan's own cap or the
            // largest; timed in turn, twice, so that a clock still rising favours none
            std::vector<std::vector<int>> tried;
            std::vector<int> caps;
            for (int grp : {best_grp, 1024, 512}) {
                dp.m2l_max_grp = grp;
                prepare_evaluate(dp, 1);
                std::vector<int> cuts;
                if (dp.level_orders)
                    for (const auto &k : dp.lvl_packs) cuts.push_back(pack_cut(dp, k, 1));
                else
                    cuts.push_back(pack_cut(dp, dp.m2l_packs[0], 1));
                if (std::find(tried.begin(), tried.end(), cuts) != tried.end()) continue;
                tried.push_back(cuts);
                caps.push_back(grp);
            }
            std::vector<float> ms(caps.size(), FLT_MAX);
            for (int turn = 0; turn < 2; ++turn)
                for (size_t c = 0; c < caps.size(); ++c) {
                    dp.m2l_max_grp = caps[c];
                    ms[c] = std::min(ms[c], time_config(dp, M, u, st));
                }
            for (size_t c = 0; c < caps.size(); ++c)
                if (ms[c] < best) best = ms[c], best_grp = caps[c], best_pack = true;
        }
        dp.m2l_pack = best_pack;
        dp.m2l_max_grp = best_grp;
        // the work lists of the form not taken are rebuilt if it is set later
        if (best_pack)
            free_tiles(dp, dp.m2l_tiles[0]);
        else
            free_m2l_packs(dp);
        // the per-tet near field's workgroup shape, where one field runs it
        if (dp.sur_mode != TFMM_SUR_OFF && !dp.near_stored && !hp.points) {
            bool best_wide = false;
            for (bool wide : {false, true}) {
                dp.p2p_wide = wide;
                const float t = time_config(dp, M, u, st);
                if (!wide || t < best) best = t, best_wide = wide;
            }
            dp.p2p_wide = best_wide;
        }
        ++dp.schedule_gen;
        prepare_evaluate(dp, 1);
        hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");
    } catch (...) {
        dp.timing = timing;
        (void)hipFree(M);
        (void)hipFree(u);
        throw;
    }
    dp.timing = timing;
    (void)hipFree(M);
    (void)hipFree(u);
}

void run_evaluate(DevicePlan &dp, const double *M, int32_t F, double *u, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    const int64_t C = (int64_t)hp.cells.size();
    const int p = hp.p;
    prepare_evaluate(dp, F);
    dp.last_F = F;
    // u = 0, then the near field (P2P, needs only M) runs on the plan's side
    // stream while the expansions are formed; both add into u atomically.
    // Under stream capture (batch graphs) the near field stays on st, after
    // the far field.
    const bool in_order = near_in_order(dp, F);
    const int32_t *perm = in_order ? nullptr : dp.tgt_perm;
    double *const out = u;
    if (in_order) {
        if (dp.u_cap < F) throw DeviceError{"potentials not prepared"};
        u = dp.u_tree;
    }
    fill(u, (int64_t)F * hp.n_targets, 0.0, st);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hip_check(hipStreamIsCapturing(st, &cap), "hipStreamIsCapturing");
    // with per-phase timing on, the phases run one after another (isolated times)
    const bool fork = cap == hipStreamCaptureStatusNone && !dp.timing;
    auto fork_p2p = [&]() {
        hip_check(hipEventRecord(dp.ev_fork, st), "hipEventRecord");
        hip_check(hipStreamWaitEvent(dp.side, dp.ev_fork, 0), "hipStreamWaitEvent");
        {
            KTimer kt(dp, KT_P2P, dp.side);
            run_near(dp, M, F, u, dp.side);
        }
        hip_check(hipEventRecord(dp.ev_join, dp.side), "hipEventRecord");
    };
    if (fork) fork_p2p();
    {
        KTimer kt(dp, KT_P2M, st);
        if (dp.n_p2m_cells > 0) with_p2m(F, p, [&](auto fc, auto nt) {
            constexpr int FC = decltype(fc)::value, NT = decltype(nt)::value;
            // a grid holds fewer than 2^32 threads: many fields in several launches
            constexpr int64_t kItems = (1ll << 32) / kP2MThreads / 2;
            const int32_t per = (int32_t)std::min<int64_t>(std::max<int64_t>(1, kItems / dp.n_p2m_cells) * FC, F);
            for (int32_t f = 0; f < F; f += per) {
                const int32_t n = std::min(per, F - f);
                k_p2m<FC, NT><<<dim3(xcd_grid(dp.n_p2m_cells * ((n + FC - 1) / FC))), dim3(kP2MThreads),
                                sizeof(double) * 12 * 64 * NT, st>>>(
                    dp.p2m_cells, dp.cell_i, dp.cell_c, C, dp.tet_xyz, dp.tet_node, hp.n_tets, dp.tet_mom,
                    M + (int64_t)f * hp.n_nodes * 3, hp.n_nodes, n, p, dp.n_p2m_cells, hp.points ? 1 : 0, dp.lo,
                    dp.Q + (int64_t)f * C * dp.ncoef);
                hip_check(hipGetLastError(), "k_p2m launch");
            }
        });
    }
    {
        KTimer kt(dp, KT_M2M, st);
        for (int Lv = hp.depth - 1; Lv >= 0; --Lv) {
            int b = dp.m2m_level_ptr[Lv], e = dp.m2m_level_ptr[Lv + 1];
            if (e > b) {
                with_order(p, [&](auto pc) {
                    constexpr int PP = decltype(pc)::value;
                    k_m2m<PP><<<dim3(e - b, F), dim3(shift_threads(PP)), 0, st>>>(
                        dp.m2m_cells + b, dp.cell_i, dp.cell_c, C, dp.lo.q[Lv], dp.Q);
                });
                hip_check(hipGetLastError(), "k_m2m launch");
            }
        }
    }
    {
        KTimer kt(dp, KT_M2L, st);
        run_m2l(dp, F, st);
    }
    {
        KTimer kt(dp, KT_L2L, st);
        for (int Lv = 1; Lv <= hp.depth; ++Lv) {
            int b = dp.l2l_level_ptr[Lv], e = dp.l2l_level_ptr[Lv + 1];
            if (e > b) {
                with_order(p, [&](auto pc) {
                    constexpr int PP = decltype(pc)::value;
                    k_l2l<PP><<<dim3((e - b + kShiftItems - 1) / kShiftItems, F), dim3(shift_threads(PP)), 0, st>>>(
                        dp.l2l_cells + b, e - b, dp.cell_i, dp.cell_c, C, dp.lo.q[Lv], dp.L);
                });
                hip_check(hipGetLastError(), "k_l2l launch");
            }
        }
    }
    {
        KTimer kt(dp, KT_L2P, st);
        const unsigned nb = (unsigned)((hp.n_targets + 255) / 256);
        with_order(p, [&](auto pc) {
            constexpr int PP = decltype(pc)::value;
            k_l2p<PP><<<dim3(nb, F), dim3(256), 0, st>>>(dp.tgt_xyz, perm, dp.tgt_leaf, hp.n_targets, dp.cell_c,
                                                         C, dp.L, u);
        });
        hip_check(hipGetLastError(), "k_l2p launch");
    }
    if (fork) {
        hip_check(hipStreamWaitEvent(st, dp.ev_join, 0), "hipStreamWaitEvent");
    } else {
        KTimer kt(dp, KT_P2P, st);
        run_near(dp, M, F, u, st);
    }
    if (in_order) {
        k_scatter<<<dim3((unsigned)((hp.n_targets + 255) / 256), (unsigned)F), dim3(256), 0, st>>>(u, dp.tgt_perm,
                                                                                                  hp.n_targets, out);
        hip_check(hipGetLastError(), "k_scatter launch");
    }
}

double run_demag(DevicePlan &dp, const double *M, const double *u, double *H, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    if (!hp.targets_are_nodes) throw DeviceError{"the plan's targets are not its nodes"};
    const int64_t T = hp.n_tets;
    const int nb = (int)((T + kEnergyThreads - 1) / kEnergyThreads);
    double *part = nullptr;
    hip_check(hipMalloc(&part, sizeof(double) * (size_t)(nb + 1)), "hipMalloc energy");
    double E = 0.0;
    hipError_t err = hipSuccess;
    if (T > 0) {
        k_demag<<<nb, kEnergyThreads, 0, st>>>(dp.tet_xyz, dp.tet_node, dp.tet_perm, T, M, u, H, part);
        k_sum_blocks<<<1, kEnergyThreads, 0, st>>>(part, nb, part + nb);
        err = hipGetLastError();
        if (err == hipSuccess) err = hipMemcpyAsync(&E, part + nb, sizeof(double), hipMemcpyDeviceToHost, st);
        if (err == hipSuccess) err = hipStreamSynchronize(st);
    }
    (void)hipFree(part);
    hip_check(err, "demag energy");
    return E;
}

void run_elementary(int fn, const double *a, const double *b, int64_t n, double *out)
{
    double *d = nullptr;
    hip_check(hipMalloc(&d, sizeof(double) * 3 * (size_t)n), "hipMalloc elementary");
    hipError_t e = hipMemcpy(d, a, sizeof(double) * n, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d + n, b, sizeof(double) * n, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        k_elementary<<<(unsigned)((n + 255) / 256), 256>>>(fn, d, d + n, n, d + 2 * n);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(out, d + 2 * n, sizeof(double) * n, hipMemcpyDeviceToHost);
    (void)hipFree(d);
    hip_check(e, "elementary functions");
}

// ---------------------------------------------------------------------------
// Scratch of the allocation-free entry point: one file-scope device array of
// kNoAllocScratchDoubles doubles; every device the library runs on holds its
// own copy until the process ends.  In host code the array's name is only a
// stand-in (not a device address), so host code reaches it through the
// address hipGetSymbolAddress returns on each device, taken once per device
// with that device current and kept.  Every call on a device shares that
// device's array (it keeps the last call's contents): calls that overlap on
// one device race.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

static double *scratch_address(int device)
{
    static std::mutex mu;
    static std::vector<double *> addr;
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0) throw DeviceError{"no device"};
    if ((int)addr.size() <= device) addr.resize((size_t)device + 1, nullptr);
    if (!addr[device]) {
        int cur = -1;
        hip_check(hipGetDevice(&cur), "hipGetDevice");
        if (cur != device) throw DeviceError{"scratch address requested for a device that is not current"};
        void *p = nullptr;
        hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
        addr[device] = static_cast<double *>(p);
    }
    return addr[device];
}

void run_demag_noalloc(DevicePlan &dp, const double *M, const double *u, double *H, double *energy_dev,
                       hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    if (!hp.targets_are_nodes) throw DeviceError{"the plan's targets are not its nodes"};
    const int64_t T = hp.n_tets;
    const int64_t nb = (T + kEnergyThreads - 1) / kEnergyThreads;
    if (nb + 1 > kNoAllocScratchDoubles)
        throw PlanError{TFMM_EINVAL, "tfmm_demag_energy_noalloc: " + std::to_string(T) + " tets exceed the limit of " +
                                         std::to_string((int64_t)TFMM_NOALLOC_MAX_TETS)};
    double *part = scratch_address(dp.device);
    // every slot read below is written first in this call (block partials,
    // then their sum): nothing has to start at zero
    if (T > 0) {
        k_demag<<<(unsigned)nb, kEnergyThreads, 0, st>>>(dp.tet_xyz, dp.tet_node, dp.tet_perm, T, M, u, H, part);
        k_sum_blocks<<<1, kEnergyThreads, 0, st>>>(part, (int)nb, energy_dev);
    } else {
        k_sum_blocks<<<1, kEnergyThreads, 0, st>>>(part, 0, energy_dev);
    }
    hip_check(hipGetLastError(), "demag energy (no allocation) launch");
}

void run_demag_nodes(DevicePlan &dp, const double *u, double *Hn, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    if (!hp.targets_are_nodes) throw DeviceError{"the plan's targets are not its nodes"};
    const int64_t T = hp.n_tets, N = hp.n_nodes;
    const unsigned nb = (unsigned)((T + kEnergyThreads - 1) / kEnergyThreads);
    fill(Hn, 3 * N, 0.0, st);
    if (!dp.node_lump) {  // lumped volumes, once per plan
        hip_check(hipMalloc(&dp.node_lump, sizeof(double) * (size_t)std::max<int64_t>(N, 1)), "hipMalloc lumped volumes");
        dp.device_bytes += (int64_t)(sizeof(double) * (size_t)std::max<int64_t>(N, 1));
        fill(dp.node_lump, N, 0.0, st);
        if (T > 0)
            k_demag_scatter<<<nb, kEnergyThreads, 0, st>>>(dp.tet_xyz, dp.tet_node, T, u, Hn, dp.node_lump);
    } else if (T > 0) {
        k_demag_scatter<<<nb, kEnergyThreads, 0, st>>>(dp.tet_xyz, dp.tet_node, T, u, Hn, nullptr);
    }
    if (N > 0) k_lump_divide<<<(unsigned)((N + 255) / 256), 256, 0, st>>>(Hn, dp.node_lump, N);
    hip_check(hipGetLastError(), "lumped field launch");
}

void run_direct(DevicePlan &dp, const double *M, int32_t F, double *u, hipStream_t st)
{
    const HostPlan &hp = dp.hp;
    fill(u, (int64_t)F * hp.n_targets, 0.0, st);
    if (hp.points) {
        run_p2p(dp, true, M, F, u, st);
        return;
    }
    if (hp.n_tets == 0 || hp.n_targets == 0) return;
    for (int f = 0; f < F;) {
        // one pass for up to 16 fields: the integrals cost more than padded fields
        const int left = F - f;
        auto go = [&](auto fc) {
            constexpr int FC = decltype(fc)::value;
            const int nblk = (int)((hp.n_tets + kDirectTets - 1) / kDirectTets);
            // enough workgroups for five rounds of three a CU; more would only stage the tets again
            const int64_t shares = std::min<int64_t>((hp.n_targets + 255) / 256, std::max(1, (4096 + nblk - 1) / nblk));
            k_direct<FC><<<dim3(xcd_grid(nblk), (unsigned)shares), dim3(256), 0, st>>>(
                nblk, hp.n_tets, dp.tet_xyz, dp.tet_node, dp.tgt_xyz, dp.tgt_perm, hp.n_targets, M, hp.n_nodes, f, F,
                dp.far_rule, u);
            f += FC;
        };
        if (left > 8)
            go(std::integral_constant<int, kDirectFieldsMax>{});
        else if (left > 4)
            go(std::integral_constant<int, 8>{});
        else if (left > 2)
            go(std::integral_constant<int, 4>{});
        else if (left > 1)
            go(std::integral_constant<int, 2>{});
        else
            go(std::integral_constant<int, 1>{});
        hip_check(hipGetLastError(), "k_direct launch");
    }
}

// ---------------------------------------------------------------------------
// quadrature: Gauss-Jacobi nodes on [0, 1] for the weight (1 - t)^alpha by
// bracketing the sign changes of the Jacobi polynomial and bisection, weights
// from the classical closed form; collapsed onto the simplex.
// ---------------------------------------------------------------------------
namespace {

void jacobi_eval(int n, double a, double x, double &P, double &dP)
{
    // P_n^{(a,0)}(x) by the three-term recurrence, derivative by the standard identity
    double p0 = 1.0, p1 = 0.5 * (a + 2.0) * x + 0.5 * a;
    if (n == 0) {
        P = 1.0;
        dP = 0.0;
        return;
    }
    const double b = 0.0;
    for (int k = 2; k <= n; ++k) {
        const double c = 2.0 * k + a + b;
        const double a1 = 2.0 * k * (k + a + b) * (c - 2.0);
        const double a2 = (c - 1.0) * (a * a - b * b);
        const double a3 = (c - 2.0) * (c - 1.0) * c;
        const double a4 = 2.0 * (k + a - 1.0) * (k + b - 1.0) * c;
        const double p2 = ((a2 + a3 * x) * p1 - a4 * p0) / a1;
        p0 = p1;
        p1 = p2;
    }
    P = p1;
    const double c = 2.0 * n + a + b;
    dP = (n * (a - b - c * x) * p1 + 2.0 * (n + a) * (n + b) * p0) / (c * (1.0 - x * x));
}

void gauss_jacobi01(int n, double a, std::vector<double> &t, std::vector<double> &w)
{
    t.clear();
    w.clear();
    const int grid = 20000;
    double xl = -1.0 + 1e-14, Pl, dPl;
    jacobi_eval(n, a, xl, Pl, dPl);
    for (int i = 1; i <= grid && (int)t.size() < n; ++i) {
        double xr = -1.0 + 2.0 * i / grid - (i == grid ? 1e-14 : 0.0), Pr, dPr;
        jacobi_eval(n, a, xr, Pr, dPr);
        if ((Pl < 0.0) != (Pr < 0.0)) {
            double lo = xl, hi = xr, flo = Pl;
            for (int it = 0; it < 200; ++it) {
                double mid = 0.5 * (lo + hi), fm, dm;
                jacobi_eval(n, a, mid, fm, dm);
                if ((fm < 0.0) == (flo < 0.0)) {
                    lo = mid;
                    flo = fm;
                } else {
                    hi = mid;
                }
            }
            double x = 0.5 * (lo + hi), P, dP;
            jacobi_eval(n, a, x, P, dP);
            // classical weight for weight (1-x)^a on [-1,1], b = 0
            const double lw = std::lgamma(n + a + 1.0) + std::lgamma(n + 1.0) - std::lgamma(n + a + 1.0) -
                              std::lgamma(n + 1.0) + (a + 1.0) * std::log(2.0);
            const double wx = std::exp(lw) / ((1.0 - x * x) * dP * dP);
            t.push_back(0.5 * (x + 1.0));
            w.push_back(wx * std::pow(2.0, -a - 1.0));
        }
        xl = xr;
        Pl = Pr;
    }
}

}  // namespace

std::vector<double> far_tables()
{
    std::vector<double> out;
    for (int n : kFarPts) {
        std::vector<double> t[3], w[3];
        for (int k = 0; k < 3; ++k) {
            gauss_jacobi01(n, (double)k, t[k], w[k]);
            double sum = 0.0;
            for (double x : w[k]) sum += x;
            for (double &x : w[k]) x /= sum * (k + 1);  // the weights sum to 1 / (k + 1)
        }
        for (int i = 0; i < n; ++i) {
            const double c = t[0][i], wc = w[0][i];
            out.insert(out.end(), {c, wc, wc * c, wc * c * c});
        }
        for (int i = 0; i < n; ++i) {
            const double b = t[1][i], u = 1.0 - b, wb = w[1][i];
            out.insert(out.end(), {b, u, wb, wb * b, wb * b * b, wb * u, wb * b * u, wb * u * u});
        }
        for (int i = 0; i < n; ++i) {
            const double a = t[2][i], q = 1.0 - a, wa = w[2][i];
            out.insert(out.end(), {a, q, wa, wa * a, wa * a * a, wa * q, wa * a * q, wa * q * q});
        }
    }
    return out;
}

std::vector<double> simplex_rule(int deg, int *npts)
{
    const int q = (deg + 2) / 2;  // 2q - 1 >= deg
    std::vector<double> ta, wa, tb, wb, tc, wc;
    gauss_jacobi01(q, 2.0, ta, wa);
    gauss_jacobi01(q, 1.0, tb, wb);
    gauss_jacobi01(q, 0.0, tc, wc);
    std::vector<double> out;
    for (int i = 0; i < q; ++i)
        for (int j = 0; j < q; ++j)
            for (int k = 0; k < q; ++k) {
                const double a = ta[i], b = tb[j], c = tc[k];
                out.push_back(a);
                out.push_back((1.0 - a) * b);
                out.push_back((1.0 - a) * (1.0 - b) * c);
                out.push_back(wa[i] * wb[j] * wc[k]);
            }
    *npts = q * q * q;
    return out;
}

}  // namespace tfmm
