// St Venant-Kirchhoff hyperelasticity: energy, residual and Jacobian, and the
// reverse pass of the energy.
//
// Per quadrature point (the paper's section 2 kernel structure, with the
// coefficient evaluated at the point as in Listing 2): the displacement
// gradient grad u = U K (U[i][a] = sum_r u_{r,i} dphi_r/dX_a in reference
// coordinates), F = I + grad u, E = (F^T F - I)/2, S = lambda tr(E) I + 2 mu E,
// P = F S, psi = lambda/2 tr(E)^2 + mu E:E. Then
//   energy   Pi_e = sum_q w_q |det J| psi
//   residual b_(c,a) = sum_q w_q |det J| sum_j P_cj dphi_a/dx_j
//   Jacobian A_(c,a),(c',b) = sum_q w_q |det J| sum_jl dphi_a/dx_j C_cjc'l dphi_b/dx_l,
// with the tangent C_cjc'l = delta_cc' S_lj + lambda F_cj F_c'l + mu F_cl F_c'j
// + mu delta_lj (F F^T)_cc' (the derivative of P along e_c' (x) e_l). In
// reference coordinates the Jacobian block is sum_q sum_ab dphi_a/dX_a H_ab
// dphi_b/dX_b with H = w |det J| K C K^T, accumulated as two rank-structured
// updates per point and reference direction.
//
// Work layout: energy, residual and the energy's reverse pass one thread per
// cell (the reverse pass also scatters the residual into the displacement
// gradient, and combines its scatter-adds per wave in LDS). Jacobian: a wave
// takes a few consecutive cells; F and K S K^T at each (cell, point) are formed
// once into LDS, then each lane accumulates a slice of rows of one block
// c <= c' (the mirrored block comes from the same values: the Jacobian is
// symmetric), and the cells' tensors are staged in LDS and written as
// contiguous 16-byte stores. Reference gradients and weights are read at
// wave-uniform addresses through the scalar path (staged in LDS where the
// Jacobian's lanes read different rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "library.h"
#include "linear.hpp"
#include "tables.h"

namespace coffee {
namespace dev {

struct SvkArgs {
    const double* coords;
    const int32_t* c2v;
    int64_t ncells;
    FieldArg u;          // displacement, ncomp = D
    double mu, lambda;
    const double* tab;   // W[nq], dphi[D][nq][NS], then N[nq][NV]: the nodal basis of degree P - 1
    void* out;
    // reverse passes (energy; residual against lam)
    double seed;
    double* grad_coords;
    double* grad_u;
    double* cell_value;
    const double* lam;   // residual reverse pass: [E][D * NS] component-blocked
    // deterministic mode: per-cell contributions written here instead of
    // scatter-added (scatter.hip sums them in a fixed order); NULL otherwise
    double* det_x;       // [E][D+1][D]
    double* det_u;       // [E][NS][D]
};

// F = I + U K at point q from the reference displacement gradient.
template <int D, int NS>
__device__ inline void svk_F(const double (&uv)[NS * D], const double (&K)[D][D], const double* dphi_q, int nq,
                             double (&F)[D][D]) {
    double U[D][D];  // U[i][a] = sum_r u_{r,i} dphi_r/dX_a
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int a = 0; a < D; ++a) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < NS; ++r) s += uv[r * D + i] * dphi_q[(size_t)a * nq * NS + r];
            U[i][a] = s;
        }
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double g = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a) g += U[i][a] * K[a][j];
            F[i][j] = (i == j ? 1.0 : 0.0) + g;
        }
}

// S = lambda tr(E) I + 2 mu E with E = (F^T F - I) / 2.
template <int D>
__device__ inline void svk_S(const double (&F)[D][D], double mu, double lm, double (&S)[D][D]) {
    double E[D][D], trE = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) t += F[k][i] * F[k][j];
            E[i][j] = 0.5 * (t - (i == j ? 1.0 : 0.0));
        }
#pragma unroll
    for (int i = 0; i < D; ++i) trE += E[i][i];
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) S[i][j] = (i == j ? lm * trE : 0.0) + 2.0 * mu * E[i][j];
}

// psi and P = F S at a point with displacement gradient H = grad u, in the
// arithmetic type T (FP64, or FP32 for the FP32 energy and residual). E is
// formed as (H + H^T + H^T H)/2, which equals (F^T F - I)/2 without the
// cancellation of F^T F against I.
template <int D, typename T>
__device__ inline void svk_point(const T (&H)[D][D], T mu, T lm, T* psi, T (&Pout)[D][D]) {
    T E[D][D], trE = T(0);
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = i; j < D; ++j) {
            T t = H[i][j] + H[j][i];
#pragma unroll
            for (int k = 0; k < D; ++k) t += H[k][i] * H[k][j];
            E[i][j] = E[j][i] = T(0.5) * t;
        }
#pragma unroll
    for (int i = 0; i < D; ++i) trE += E[i][i];
    T EE = T(0);
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) EE += E[i][j] * E[i][j];
    *psi = T(0.5) * lm * trE * trE + mu * EE;
    T S[D][D];
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) S[i][j] = (i == j ? lm * trE : T(0)) + T(2) * mu * E[i][j];
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) {
            T t = S[i][j];
#pragma unroll
            for (int k = 0; k < D; ++k) t += H[i][k] * S[k][j];
            Pout[i][j] = t;
        }
}

template <int D, int NS>
struct SvkCell {
    int vid[D + 1], uid[NS];
    double x[D + 1][D], u[NS * D];
};

template <int D, int NS>
__device__ inline void svk_load_ids(const SvkArgs& A, int64_t cell, SvkCell<D, NS>& c) {
#pragma unroll
    for (int v = 0; v <= D; ++v) c.vid[v] = A.c2v[cell * (D + 1) + v];
    if (A.u.map) {
#pragma unroll
        for (int r = 0; r < NS; ++r) c.uid[r] = A.u.map[cell * NS + r];
    }
}

// The components of a point share a line of the L1, which holds the lines of
// four loads of 64 scattered points: they are loaded together. Left free, the
// compiler put the first two components of all ten dofs before the third ones,
// and cells in random order fetched their lines twice. 600,011 P2 tetrahedra in
// random order, us: energy FP64 126 -> 100, FP32 140 -> 97, residual 184 -> 145
// and 166 -> 125; 199,997 in mesh order 18.3 -> 18.6, 15.8 -> 15.5, 39.7 ->
// 39.0 and 31.6 -> 30.4.
template <int D, int NS>
__device__ inline void svk_load_values(const SvkArgs& A, int64_t cell, SvkCell<D, NS>& c) {
#pragma unroll
    for (int v = 0; v <= D; ++v) {
#pragma unroll
        for (int i = 0; i < D; ++i) c.x[v][i] = A.coords[(int64_t)c.vid[v] * D + i];
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const int64_t base = A.u.map ? (int64_t)c.uid[r] * D : (cell * NS + r) * D;
#pragma unroll
        for (int i = 0; i < D; ++i) c.u[r * D + i] = A.u.values[base + i];
        asm volatile("" ::: "memory");
    }
}

template <int D, int NS>
__device__ inline void svk_load(const SvkArgs& A, int64_t cell, Geom<D>& g, double (&uv)[NS * D],
                                int (&vid)[D + 1], int (&uid)[NS]) {
    SvkCell<D, NS> c;
    svk_load_ids<D, NS>(A, cell, c);
    svk_load_values<D, NS>(A, cell, c);
    geometry_from_coords<D>(c.x, g);
#pragma unroll
    for (int v = 0; v <= D; ++v) vid[v] = c.vid[v];
#pragma unroll
    for (int r = 0; r < NS; ++r) uid[r] = c.uid[r];
#pragma unroll
    for (int r = 0; r < NS * D; ++r) uv[r] = c.u[r];
}

typedef unsigned int svk_u32x4 __attribute__((ext_vector_type(4)));

// The per-cell results of a reverse pass: the vertex-coordinate gradients vx
// (seed already applied) and, if U, the displacement-dof gradients
// f * g[c * NS + r] (component-blocked). Deterministic mode writes them to
// the cell's slots of the workspace; otherwise they are scatter-added through
// the wave's combining tables.
template <int D, int NS, int TS, int TU, bool U, typename GT>
__device__ inline void svk_scatter_cell(const SvkArgs& A, bool det, int64_t cell, const int (&vid)[D + 1],
                                        const int (&uid)[NS], const double (&vx)[D + 1][D], const GT* g, double f,
                                        unsigned long long* ckeys, double* cvals, unsigned long long* ukeys,
                                        double* uvals) {
    if (det) {
#pragma unroll
        for (int v = 0; v <= D; ++v)
#pragma unroll
            for (int i = 0; i < D; ++i) A.det_x[(cell * (D + 1) + v) * D + i] = vx[v][i];
        if constexpr (U) {
#pragma unroll
            for (int r = 0; r < NS; ++r)
#pragma unroll
                for (int c = 0; c < D; ++c) A.det_u[(cell * NS + r) * D + c] = f * (double)g[c * NS + r];
        }
        return;
    }
    if (A.grad_coords) {
        unsigned long long key[D + 1];
#pragma unroll
        for (int v = 0; v <= D; ++v) key[v] = (unsigned long long)vid[v];
        combine_add<D, TS>(ckeys, cvals, key, vx, A.grad_coords);
    }
    if constexpr (U) {
        // NULL: the caller skips this gradient (a full table adds to it directly)
        if (!A.grad_u) return;
        unsigned long long key[NS];
        double v[NS][D];
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            key[r] = A.u.map ? (unsigned long long)uid[r] : (unsigned long long)(cell * NS + r);
#pragma unroll
            for (int c = 0; c < D; ++c) v[r][c] = f * (double)g[c * NS + r];
        }
        combine_add<D, TU>(ukeys, uvals, key, v, A.grad_u);
    }
}

// Vertex-coordinate gradients of a cell from Kbar = dS/dK (already scaled by
// |det J|) and S (every term is linear in |det J|):
//   Jbar = -K^T Kbar K^T + S K^T,  xbar_{j+1} = Jbar[:, j],  xbar_0 = -sum_j Jbar[:, j].
template <int D>
__device__ inline void svk_coord_bars(const double (&K)[D][D], const double (&Kbar)[D][D], double S, double sd,
                                      double (&vx)[D + 1][D]) {
    double Jbar[D][D];
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double s = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a)
#pragma unroll
                for (int b = 0; b < D; ++b) s += K[a][i] * Kbar[a][b] * K[j][b];
            Jbar[i][j] = -s + S * K[j][i];
        }
#pragma unroll
    for (int i = 0; i < D; ++i) {
        double x0 = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            vx[j + 1][i] = sd * Jbar[i][j];
            x0 -= Jbar[i][j];
        }
        vx[0][i] = sd * x0;
    }
}

// MODE 0: energy, 1: residual, 2: reverse pass of the energy (coordinates),
// 3: the reverse pass with the displacement gradient (the residual) too.
//
// One thread per cell. The displacement gradient has degree P - 1: it is
// formed at its NV nodes once (H_k), a point takes H = sum_k N_k H_k and gives
// back the moments Pm_k += w N_k P, so that the residual (Pm_k K^T against the
// basis gradients at node k) and the coordinate bars (T = sum_k H_k^T Pm_k) are
// formed once per cell: about 150 multiply-adds per point for P2 tetrahedra,
// where going through the ten dofs at every point took 400 (energy and both
// gradients through autograd, 2,058,000 cells: 1,282 -> 656 us together with
// the group-hashed combining table; residual, 196,608 cells: 49 -> 36 us).
template <int D, int P, int NQ, int MODE, typename OT>
__global__ __launch_bounds__(256) void k_svk_vec(SvkArgs A) {
    constexpr int NS = nsc(D, P), NV = grad_nv(D, P);
    // arithmetic type of the point loop: the output type for the forward
    // energy and residual (FP32 mode computes them in FP32 from the FP64
    // geometry and node gradients), FP64 for the reverse pass
    using T = std::conditional_t<(MODE <= 1), OT, double>;
    // every table read below has the same address in all lanes: scalar path
    const double* W = A.tab;
    const double* Nk = A.tab + NQ + D * NQ * NS;
    // reverse pass: the scatter-adds (vertex coordinates; MODE 3 also the
    // displacement dofs) are combined per wave
    constexpr bool REV = MODE >= 2;                 // reverse pass
    constexpr bool RES = MODE == 1 || MODE == 3;    // residual (MODE 3: scattered into grad_u)
    // 48 KB of tables with both gradients: three workgroups per CU
    constexpr int TS = REV ? 128 : 1;
    constexpr int TU = MODE == 3 ? 256 : 1;
    __shared__ unsigned long long ckeys[4][TS], ukeys[4][TU];
    __shared__ double cvals[4][TS * D], uvals[4][TU * D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // reverse pass: the next cell's dofs and values, loaded during the current
    // one's combining and complete before its flush
    SvkCell<D, NS> nx;
    auto cell_at = [&](int64_t b) { return b + lane < A.ncells ? b + lane : A.ncells - 1; };
    if constexpr (REV) {
        const int64_t b = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane;
        if (b >= A.ncells) return;  // wave-uniform; no workgroup barrier follows
        svk_load_ids<D, NS>(A, cell_at(b), nx);
        svk_load_values<D, NS>(A, cell_at(b), nx);
    }
    // wave-uniform loop (every lane takes part in the table's clear and flush)
    for (int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane; base < A.ncells;
         base += (int64_t)gridDim.x * blockDim.x) {
        const bool valid = base + lane < A.ncells;
        const int64_t cell = valid ? base + lane : A.ncells - 1;
        const bool det = A.det_x != nullptr;  // same in every lane
        if (REV && !det) {
            combine_clear<D, TS>(ckeys[wave], cvals[wave], lane);
            if constexpr (MODE == 3) combine_clear<D, TU>(ukeys[wave], uvals[wave], lane);
            wave_sync();
        }
        Geom<D> g;
        T H[NV][D][D];  // displacement gradient at the nodes
        int vid[D + 1], uid[NS];
        {
            if constexpr (!REV) {
                svk_load_ids<D, NS>(A, cell, nx);
                svk_load_values<D, NS>(A, cell, nx);
            }
            geometry_from_coords<D>(nx.x, g);
            const double(&uvd)[NS * D] = nx.u;
#pragma unroll
            for (int v = 0; v <= D; ++v) vid[v] = nx.vid[v];
#pragma unroll
            for (int r = 0; r < NS; ++r) uid[r] = nx.uid[r];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                double v[NS], gr[NV][D];
#pragma unroll
                for (int r = 0; r < NS; ++r) v[r] = uvd[r * D + c];
                grad_nodes<D, P>(v, gr);
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        double x = 0.0;
#pragma unroll
                        for (int a = 0; a < D; ++a) x += gr[k][a] * g.K[a][j];
                        H[k][c][j] = (T)x;
                    }
            }
        }
        T energy = T(0);
        T Pm[MODE > 0 ? NV : 1][D][D];
#pragma unroll
        for (int k = 0; k < (MODE > 0 ? NV : 1); ++k)
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) Pm[k][i][j] = T(0);
#pragma unroll 1
        for (int q = 0; q < NQ; ++q) {
            T n[NV], Hq[D][D], psi, Pq[D][D];
#pragma unroll
            for (int k = 0; k < NV; ++k) n[k] = (T)cload(Nk + q * NV + k);
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    T x = n[0] * H[0][i][j];
#pragma unroll
                    for (int k = 1; k < NV; ++k) x += n[k] * H[k][i][j];
                    Hq[i][j] = x;
                }
            svk_point<D, T>(Hq, (T)A.mu, (T)A.lambda, &psi, Pq);
            const T wq = (T)cload(W + q);
            energy += wq * psi;
            if constexpr (MODE > 0) {
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const T wn = wq * n[k];
#pragma unroll
                    for (int i = 0; i < D; ++i)
#pragma unroll
                        for (int j = 0; j < D; ++j) Pm[k][i][j] += wn * Pq[i][j];
                }
            }
        }
        const double ad = g.adet;
        T res[RES ? D * NS : 1];
        if constexpr (RES) {
            // b_(c,a) = sum_k (Pm_k K^T)_c . grad phi_a at node k
#pragma unroll
            for (int c = 0; c < D; ++c) {
                T Q[NV][D];
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int al = 0; al < D; ++al) {
                        T t = T(0);
#pragma unroll
                        for (int j = 0; j < D; ++j) t += Pm[k][c][j] * (T)g.K[al][j];
                        Q[k][al] = t;
                    }
                grad_nodes_t<D, P, T>(Q, res + c * NS);
            }
        }
        if constexpr (MODE == 0) {
            if (valid) reinterpret_cast<OT*>(A.out)[cell] = (OT)((T)ad * energy);
        } else if constexpr (MODE == 1) {
            OT* o = reinterpret_cast<OT*>(A.out) + cell * (D * NS);
            if (valid) {
#pragma unroll
                for (int i = 0; i < D * NS; ++i) o[i] = (OT)((T)ad * res[i]);
            }
        } else {
            const double Pi = ad * energy;
            if (A.cell_value && valid) A.cell_value[cell] = Pi;
            // every term is linear in |det J| and H = (reference gradient) K:
            // Jbar = (Pi I - |det J| sum_k H_k^T Pm_k) K^T, xbar_{j+1} = Jbar[:, j]
            const double sd = A.seed;
            double vx[D + 1][D], R[D][D];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int k = 0; k < NV; ++k)
#pragma unroll
                        for (int c = 0; c < D; ++c) t += H[k][c][i] * Pm[k][c][j];
                    R[i][j] = (i == j ? Pi : 0.0) - ad * t;
                }
#pragma unroll
            for (int i = 0; i < D; ++i) {
                double x0 = 0.0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) t += R[i][a] * g.K[j][a];
                    vx[j + 1][i] = sd * t;
                    x0 -= t;
                }
                vx[0][i] = sd * x0;
            }
            const int64_t next = base + (int64_t)gridDim.x * blockDim.x;
            const bool more = next < A.ncells;  // wave-uniform
            // (no next cell: zeros, so that the registers hold no old values)
            if (more) svk_load_ids<D, NS>(A, cell_at(next), nx);
            else nx = SvkCell<D, NS>{};
            if (valid) {
                svk_scatter_cell<D, NS, TS, TU, MODE == 3>(A, det, cell, vid, uid, vx, res, sd * ad, ckeys[wave],
                                                           cvals[wave], ukeys[wave], uvals[wave]);
            }
            // (one in-order counter: a load behind the atomics would wait for them)
            if (more) {
                svk_load_values<D, NS>(A, cell_at(next), nx);
#pragma unroll
                for (int v = 0; v <= D; ++v)
#pragma unroll
                    for (int i = 0; i < D; ++i) asm volatile("" ::"v"(nx.x[v][i]));
#pragma unroll
                for (int r = 0; r < NS * D; ++r) asm volatile("" ::"v"(nx.u[r]));
            } else {
                nx = SvkCell<D, NS>{};
            }
            if (!det) {
                wave_sync();
                if (A.grad_coords) combine_flush<D, TS>(ckeys[wave], cvals[wave], A.grad_coords, lane);
                if constexpr (MODE == 3) combine_flush<D, TU>(ukeys[wave], uvals[wave], A.grad_u, lane);
                wave_sync();
            }
        }
    }
}

// Reverse pass of the residual: S_e = lam_e^T b_e with b_(c,a) = sum_q w |det J|
// P(F) : grad phi_a e_c, i.e. S_e = sum_q w |det J| P : L with L = Lam K the
// physical gradient of the field lam_e (Lam[c][al] = sum_a lam_(c,a) dphi_a/dX_al).
// Per point, with Pbar = w L and Lbar = w P (|det J| applied at the end):
//   P = F S(F):  Fbar = Pbar S + F sym(Z),  M = F^T Pbar,  Z = lambda tr(M) I + 2 mu M
//                (S symmetric; dS = lambda tr(dE) I + 2 mu dE, dE = (dF^T F + F^T dF)/2)
//   F = I + U K: Ubar = Fbar K^T -> u-dof bars Ubar dphi_r;  Kbar += U^T Fbar
//   L = Lam K:   Kbar += Lam^T Lbar
// so the displacement gradient is (db/du)^T lam = A_e lam_e (the Jacobian is
// symmetric). One thread per cell, FP64.
template <int D, int P, int NQ>
__global__ __launch_bounds__(256) void k_svk_res_adj(SvkArgs A) {
    constexpr int NS = nsc(D, P), N = D * NS;
    const double* W = A.tab;
    const double* dphi = A.tab + NQ;
    constexpr int TS = 256;
    __shared__ unsigned long long ckeys[4][TS], ukeys[4][TS];
    __shared__ double cvals[4][TS * D], uvals[4][TS * D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double mu = A.mu, lm = A.lambda;
    for (int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane; base < A.ncells;
         base += (int64_t)gridDim.x * blockDim.x) {
        const bool valid = base + lane < A.ncells;
        const int64_t cell = valid ? base + lane : A.ncells - 1;
        const bool det = A.det_x != nullptr;
        if (!det) {
            combine_clear<D, TS>(ckeys[wave], cvals[wave], lane);
            combine_clear<D, TS>(ukeys[wave], uvals[wave], lane);
            wave_sync();
        }
        Geom<D> g;
        double uv[NS * D];
        int vid[D + 1], uid[NS];
        svk_load<D, NS>(A, cell, g, uv, vid, uid);
        const auto& K = g.K;
        const double* lam = A.lam + cell * N;
        double val = 0.0, Kbar[D][D], gu[N];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int j = 0; j < D; ++j) Kbar[i][j] = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) gu[i] = 0.0;
#pragma unroll 1
        for (int q = 0; q < NQ; ++q) {
            const double* dq = dphi + q * NS;
            double U[D][D], Lm[D][D];  // reference gradients of u and of lam
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int al = 0; al < D; ++al) {
                    double s = 0.0, t = 0.0;
#pragma unroll
                    for (int r = 0; r < NS; ++r) {
                        const double dp = cload(dq + (size_t)al * NQ * NS + r);
                        s += uv[r * D + i] * dp;
                        t += lam[i * NS + r] * dp;
                    }
                    U[i][al] = s;
                    Lm[i][al] = t;
                }
            double H[D][D], F[D][D], L[D][D];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double h = 0.0, l = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) {
                        h += U[i][a] * K[a][j];
                        l += Lm[i][a] * K[a][j];
                    }
                    H[i][j] = h;
                    F[i][j] = (i == j ? 1.0 : 0.0) + h;
                    L[i][j] = l;
                }
            double E[D][D], trE = 0.0;
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = H[i][j] + H[j][i];
#pragma unroll
                    for (int k = 0; k < D; ++k) t += H[k][i] * H[k][j];
                    E[i][j] = 0.5 * t;
                }
#pragma unroll
            for (int i = 0; i < D; ++i) trE += E[i][i];
            double S[D][D], Pm[D][D];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) S[i][j] = (i == j ? lm * trE : 0.0) + 2.0 * mu * E[i][j];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int k = 0; k < D; ++k) t += F[i][k] * S[k][j];
                    Pm[i][j] = t;
                }
            const double wq = cload(W + q);
            double pl = 0.0;
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) pl += Pm[i][j] * L[i][j];
            val += wq * pl;
            // M = F^T Pbar with Pbar = w L; Z = lambda tr(M) I + 2 mu M
            double M[D][D], trM = 0.0;
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int k = 0; k < D; ++k) t += F[k][i] * L[k][j];
                    M[i][j] = wq * t;
                }
#pragma unroll
            for (int i = 0; i < D; ++i) trM += M[i][i];
            // Fbar = Pbar S + F sym(Z), sym(Z) = lambda tr(M) I + mu (M + M^T)
            double Fb[D][D];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0, z = 0.0;
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        t += L[i][k] * S[k][j];
                        z += F[i][k] * ((k == j ? lm * trM : 0.0) + mu * (M[k][j] + M[j][k]));
                    }
                    Fb[i][j] = wq * t + z;
                }
            // Kbar += U^T Fbar + Lam^T (w P); Ubar = Fbar K^T -> u-dof bars
#pragma unroll
            for (int al = 0; al < D; ++al)
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int i = 0; i < D; ++i) t += U[i][al] * Fb[i][j] + Lm[i][al] * wq * Pm[i][j];
                    Kbar[al][j] += t;
                }
            double Ub[D][D];
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int al = 0; al < D; ++al) {
                    double t = 0.0;
#pragma unroll
                    for (int j = 0; j < D; ++j) t += Fb[i][j] * K[al][j];
                    Ub[i][al] = t;
                }
#pragma unroll
            for (int r = 0; r < NS; ++r) {
                double dp[D];
#pragma unroll
                for (int al = 0; al < D; ++al) dp[al] = cload(dq + (size_t)al * NQ * NS + r);
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    double t = 0.0;
#pragma unroll
                    for (int al = 0; al < D; ++al) t += Ub[i][al] * dp[al];
                    gu[i * NS + r] += t;
                }
            }
        }
        const double ad = g.adet;
        const double Se = ad * val;
        if (A.cell_value && valid) A.cell_value[cell] = Se;
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int j = 0; j < D; ++j) Kbar[i][j] *= ad;
        const double sd = A.seed;
        if (valid) {
            double vx[D + 1][D];
            svk_coord_bars<D>(K, Kbar, Se, sd, vx);
            svk_scatter_cell<D, NS, TS, TS, true>(A, det, cell, vid, uid, vx, gu, sd * ad, ckeys[wave], cvals[wave],
                                                  ukeys[wave], uvals[wave]);
        }
        if (!det) {
            wave_sync();
            if (A.grad_coords) combine_flush<D, TS>(ckeys[wave], cvals[wave], A.grad_coords, lane);
            if (A.grad_u) combine_flush<D, TS>(ukeys[wave], uvals[wave], A.grad_u, lane);
            wave_sync();
        }
    }
}

// Jacobian, shared-point layout: CPW cells per wave, lane (cell, block
// c1 <= c2, row slice h) accumulating rows h*NA .. h*NA + NA - 1 of that block.
// At every (cell, point), F and S^ = K S K^T are formed once, by the cell's
// lanes in turn, into LDS. Each lane forms its block's H = w K C K^T for the
// tangent above, with k_c = K F_c (row c of F mapped by K), as
//   H = w (delta_c1c2 S^ + lambda k_c1 k_c2^T + mu k_c2 k_c1^T + mu (F_c1 . F_c2) K K^T)
// and accumulates its rows as A[a][b] += sum_be (sum_al dphi_al,a H[al][be])
// dphi_be,b.
template <int D, int P, int NQ, typename AT, int AH>
__global__ __launch_bounds__(256, 2) void k_svk_jac(SvkArgs A) {
    constexpr int NS = nsc(D, P);
    constexpr int N = D * NS;
    constexpr int NB = D * (D + 1) / 2;
    constexpr int LPC = NB * AH;  // lanes per cell
    constexpr int CPW = 64 / LPC;  // cells per wave
    constexpr int NA = (NS + AH - 1) / AH;
    constexpr int TE = NQ + D * NQ * NS;
    // per wave: F and S (upper) at the group's points, later one cell's
    // staged tensor
    constexpr int PEQ = D * D + NB;
    constexpr int FE = CPW * NQ * PEQ;
    constexpr int SE = (N * N * (int)sizeof(AT) + 7) / 8;  // one staged cell, in doubles
    // cells staged per round: as many as the point data's area holds, or as
    // fit in 6 KiB
    constexpr int CR0 = FE / SE > 6144 / (SE * 8) ? FE / SE : 6144 / (SE * 8);
    constexpr int CR = CR0 < 1 ? 1 : (CR0 > CPW ? CPW : CR0);
    __shared__ double tab[TE];
    constexpr int WE = ((FE > CR * SE ? FE : CR * SE) + 1) / 2 * 2;  // 16-byte multiple
    __shared__ __attribute__((aligned(16))) double fbuf[4][WE];
    for (int i = threadIdx.x; i < TE; i += blockDim.x) tab[i] = A.tab[i];
    __syncthreads();
    const double* W = tab;
    const double* dphi = tab + NQ;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k = lane % LPC, cl = lane / LPC;
    const int blk = k % NB, h = k / NB;
    int c1 = 0, c2 = 0;
    {
        int t = blk;
        while (t >= D - c1) { t -= D - c1; ++c1; }
        c2 = c1 + t;
    }
    const int a0 = h * NA;
    const double diag = c1 == c2 ? 1.0 : 0.0;
    double* Fw = fbuf[wave];
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t w0 = (int64_t)blockIdx.x * 4 + wave; w0 * CPW < A.ncells; w0 += nwaves) {
        const int64_t cell = w0 * CPW + cl;
        const bool active = cl < CPW && cell < A.ncells;
        // lanes without a cell work on the group's last one and store nothing
        const int64_t lcell = active ? cell : (w0 * CPW + CPW - 1 < A.ncells ? w0 * CPW + CPW - 1 : A.ncells - 1);
        Geom<D> g;
        double uv[NS * D];
        int vid[D + 1], uid[NS];
        svk_load<D, NS>(A, lcell, g, uv, vid, uid);
        double M[D][D];  // K K^T
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int b = 0; b < D; ++b) {
                double x = 0.0;
#pragma unroll
                for (int i = 0; i < D; ++i) x += g.K[a][i] * g.K[b][i];
                M[a][b] = x;
            }
        double* Fc = Fw + (cl < CPW ? cl : CPW - 1) * NQ * PEQ;
        // F at the cell's points, LPC points at a time
#pragma unroll 1
        for (int q = k; q < NQ; q += LPC) {
            if (!active) break;
            double F[D][D], S[D][D], KS[D][D];
            svk_F<D, NS>(uv, g.K, dphi + q * NS, NQ, F);
            svk_S<D>(F, A.mu, A.lambda, S);
            double* pq = Fc + q * PEQ;
#pragma unroll
            for (int c = 0; c < D; ++c)
#pragma unroll
                for (int a = 0; a < D; ++a) pq[c * D + a] = F[c][a];
            // S^ = K S K^T (upper)
#pragma unroll
            for (int a = 0; a < D; ++a)
#pragma unroll
                for (int l = 0; l < D; ++l) {
                    double x = 0.0;
#pragma unroll
                    for (int j = 0; j < D; ++j) x += g.K[a][j] * S[j][l];
                    KS[a][l] = x;
                }
            int t = 0;
#pragma unroll
            for (int a = 0; a < D; ++a)
#pragma unroll
                for (int b = a; b < D; ++b, ++t) {
                    double x = 0.0;
#pragma unroll
                    for (int l = 0; l < D; ++l) x += KS[a][l] * g.K[b][l];
                    pq[D * D + t] = x;
                }

        }
        wave_sync();
        AT acc[NA][NS];
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NS; ++b) acc[a][b] = (AT)0;
#pragma unroll 1
        for (int q = 0; q < NQ; ++q) {
            const double* Fq = Fc + q * PEQ;
            // rows c1, c2 of F; k_c = K F_c
            double F1[D], F2[D], k1[D], k2[D], Sh[D][D];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                F1[j] = Fq[c1 * D + j];
                F2[j] = Fq[c2 * D + j];
            }
#pragma unroll
            for (int a = 0; a < D; ++a) {
                double x = 0.0, y = 0.0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    x += g.K[a][j] * F1[j];
                    y += g.K[a][j] * F2[j];
                }
                k1[a] = x;
                k2[a] = y;
            }
            // S^ enters the diagonal blocks only
            {
                int t = 0;
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int b = a; b < D; ++b, ++t) {
                        Sh[a][b] = diag * Fq[D * D + t];
                        Sh[b][a] = Sh[a][b];
                    }
            }
            double FF = 0.0;
#pragma unroll
            for (int j = 0; j < D; ++j) FF += F1[j] * F2[j];
            // H = w K C K^T = w (delta S^ + lambda k1 k2^T + mu k2 k1^T + mu FF K K^T)
            double H[D][D];
            const double wq = W[q];
#pragma unroll
            for (int a = 0; a < D; ++a)
#pragma unroll
                for (int b = 0; b < D; ++b)
                    H[a][b] = wq * (Sh[a][b] + A.lambda * k1[a] * k2[b] + A.mu * k2[a] * k1[b] + A.mu * FF * M[a][b]);
            // this lane's rows: wv[i][be] = sum_al dphi_al,a H[al][be], then
            // A[a][b] += sum_be wv[i][be] dphi_be,b
            AT wv[NA][D];
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int a = a0 + i < NS ? a0 + i : NS - 1;
#pragma unroll
                for (int be = 0; be < D; ++be) {
                    double s = 0.0;
#pragma unroll
                    for (int al = 0; al < D; ++al) s += dphi[(size_t)al * NQ * NS + q * NS + a] * H[al][be];
                    wv[i][be] = (AT)s;
                }
            }
#pragma unroll
            for (int be = 0; be < D; ++be)
#pragma unroll
                for (int b = 0; b < NS; ++b) {
                    // wave-uniform: through the scalar path, not an LDS broadcast
                    const AT db = (AT)cload(A.tab + NQ + (size_t)be * NQ * NS + q * NS + b);
#pragma unroll
                    for (int i = 0; i < NA; ++i) acc[i][b] += wv[i][be] * db;
                }
        }
        wave_sync();  // the next cell's F overwrites this one's
        const AT ad = (AT)g.adet;
        // the wave's cells are consecutive: stage CR cells' tensors at a time in
        // LDS (over the point data, no longer needed) and write them as
        // contiguous 16-byte stores
        AT* stg = reinterpret_cast<AT*>(Fw);
        AT* out = reinterpret_cast<AT*>(A.out);
        wave_sync();
#pragma unroll 1
        for (int r0 = 0; r0 < CPW; r0 += CR) {
            const int64_t rc = w0 * CPW + r0;
            if (rc >= A.ncells) break;  // wave-uniform
            // cells of this round: CR, fewer in the group's last round and at
            // the end of the mesh
            const int nc = CPW - r0 < CR ? CPW - r0 : CR;
            const int nr = (int)(A.ncells - rc < nc ? A.ncells - rc : nc);
            if (active && cl >= r0 && cl < r0 + CR) {
                AT* sc = stg + (cl - r0) * N * N;
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const int a = a0 + i;
                    if (a >= NS) continue;
#pragma unroll
                    for (int b = 0; b < NS; ++b) {
                        const AT x = ad * acc[i][b];
                        sc[(c1 * NS + a) * N + c2 * NS + b] = x;
                        if (c1 != c2) sc[(c2 * NS + b) * N + c1 * NS + a] = x;
                    }
                }
            }
            wave_sync();
            AT* o = out + rc * (int64_t)N * N;
            if constexpr ((N * N * sizeof(AT)) % 16 == 0) {
                constexpr int NV = (int)(N * N * sizeof(AT) / 16);
                const int nv = nr * NV;
                const svk_u32x4* s4 = reinterpret_cast<const svk_u32x4*>(stg);
                svk_u32x4* o4 = reinterpret_cast<svk_u32x4*>(o);
#pragma unroll
                for (int e0 = 0; e0 < CR * NV; e0 += 64)
                    if (e0 + lane < nv) __builtin_nontemporal_store(s4[e0 + lane], &o4[e0 + lane]);
            } else {
                const int ne = nr * N * N;
#pragma unroll
                for (int e0 = 0; e0 < CR * N * N; e0 += 64)
                    if (e0 + lane < ne) o[e0 + lane] = stg[e0 + lane];
            }
            wave_sync();
        }
    }
}

// ---------------------------------------------------------------- Jacobian, degree 2
// At degree 2 the tangent in reference coordinates,
//     H_cc' = lambda k_c k_c'^T + mu k_c' k_c^T + mu (F_c . F_c') K K^T + delta_cc' K S K^T,   k_c = K F_c,
// is a quadratic function on the cell (F is linear), and the gradient of a
// basis function is linear: phi_v gives (4 lambda_v - 1) grad lambda_v, the
// function of edge (i, n) gives 4 lambda_n grad lambda_i + 4 lambda_i grad lambda_n.
// With H_ij = grad lambda_i . H grad lambda_j = sum_vw lambda_v lambda_w h^vw (h
// symmetric in v, w), a block's entries are sums of the moments
//     int (4 lambda_n - d_ni) (4 lambda_q - d_qj) H_ij,
// one for each pair of (i, n) (the vertex i if n = i, else the edge (i, n))
// and (j, q). The moments of barycentric monomials, int prod lambda_v^m_v =
// prod m_v! / (d + sum m_v)! on the reference cell, give with C = sum_vw h^vw +
// sum_v h^vv and r_n = 2 sum_w h^nw + 2 h^nn, in units of 1 / (d + 4)!,
//     int lambda_n lambda_q H = (1 + d_nq) (C + r_n + r_q + 2 h^nq),
//     int lambda_n H = (d + 4) (C + r_n),   int H = (d + 3) (d + 4) C.
// The integrand has degree 4, so this equals the sum over every rule of that
// degree (the only ones the entry point takes for this form). A lane runs
// about 2,300 FP64 operations for half a block of a P2 tetrahedron, where the
// sum over the 14 points took 3,600 (196,608 cells: FP64 572 -> 480 us, FP32
// 456 -> 433). It is bound by its instructions: of the 25,000 cycles a group
// of five cells takes, 9,800 go to the block, 7,600 to the geometry and the
// shared coefficients, 6,700 to staging and stores. Two waves per SIMD (the
// k_c read from LDS where used, two cells staged at a time) ran 548 us: 64
// registers spilled, and the instructions are the same. Triangles, whose
// blocks have 36 entries, stay with the point kernel (62 us against 97).
//
// Work layout: a wave takes CPW consecutive cells; lane (cell, block c <= c',
// half). A block's columns are split in halves {v0, v1, e01, e02, e13} and its
// image under the vertex permutation 0 -> 2, 1 -> 3, 2 -> 1, 3 -> 0, so that
// both halves run the same code on permuted data (50 accumulators each). The
// cell's lanes load its dofs, form m_c = K K^T (reference gradient of u_c) and
// k_c = K e_c + m_c at the vertices, F_c . F_c' and the K S K^T coefficients
// together in LDS; the whole tensors are staged over that and leave as one
// contiguous range of 16-byte stores. The next group's gathers are in flight
// meanwhile.
struct SvkJ2 {
    static constexpr int D = 3, V = D + 1, NS = nsc(D, 2), N = D * NS, NB = D * (D + 1) / 2;
    static constexpr int LPC = 2 * NB, CPW = 64 / LPC;
    static constexpr int NP = V * (V + 1) / 2;       // pairs n <= l, also i <= j
    static constexpr int NCOL = NS / 2;              // columns per lane
    static constexpr int RL = (NS + LPC - 1) / LPC;  // dofs a lane loads
    // LDS of one cell, in doubles
    static constexpr int X = 0, U = X + V * D, MM = U + NS * D, GG = MM + D * V * V, HH = GG + D * V * D,
                         KB = HH + D * V * D, MB = KB + V * D, SB = MB + NP, KF = SB + NP * NP, PH = KF + D * V * V,
                         CELL = (PH + NB * NP) | 1;
    // column of the lane's half for (j, q), -1 if it is not one of them
    static constexpr int col(int j, int q) {
        const int lo = j < q ? j : q, hi = j < q ? q : j;
        if (lo == hi) return lo < 2 ? lo : -1;
        return lo == 0 && hi == 1 ? 2 : (lo == 0 && hi == 2 ? 3 : (lo == 1 && hi == 3 ? 4 : -1));
    }
    static constexpr int row(int i, int n) { return i == n ? i : edge_dof<D>(i, n); }
    static constexpr int pair(int a, int b) {
        const int lo = a < b ? a : b, hi = a < b ? b : a;
        return lo * V - lo * (lo - 1) / 2 + hi - lo;
    }
    template <typename OT>
    static constexpr int wave_bytes() {
        const int a = CPW * CELL * 8, b = CPW * N * N * (int)sizeof(OT);
        return ((a > b ? a : b) + 15) / 16 * 16;
    }
};

// f(0), ..., f(N - 1) with compile-time arguments (a loop whose unrolling
// would exceed the compiler's limit would leave the accumulators in memory).
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<N, I + 1>(f);
    }
}

template <int V>
__device__ inline int pair_rt(int a, int b) {
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return lo * V - lo * (lo - 1) / 2 + hi - lo;
}

template <typename OT>
__global__ __launch_bounds__(256, 1) void k_svk_jac2(SvkArgs A) {
    using C = SvkJ2;
    constexpr int D = C::D, V = C::V, NS = C::NS, N = C::N, NB = C::NB, LPC = C::LPC, CPW = C::CPW, NP = C::NP, RL = C::RL;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double* wl = reinterpret_cast<double*>(lds + wave * C::wave_bytes<OT>());
    const int cl = lane / LPC < CPW ? lane / LPC : CPW - 1, k = lane % LPC;
    const bool owner = lane < CPW * LPC;
    double* cc = wl + cl * C::CELL;
    const double mu = A.mu, lm = A.lambda;
    // dofs of the permuted pairs (i, n), four bits each; and the pairs' own numbers
    uint64_t dofs4 = 0, pairs4 = 0;
    {
        const int half = k / NB;
        int pi[V];
#pragma unroll
        for (int v = 0; v < V; ++v) pi[v] = half == 0 ? v : (v < 2 ? v + 2 : 3 - v);
#pragma unroll
        for (int i = 0; i < V; ++i)
#pragma unroll
            for (int n = i; n < V; ++n) {
                const int d = i == n ? pi[i] : edge_dof_rt<D>(pi[i], pi[n]);
                dofs4 |= (uint64_t)d << (4 * C::pair(i, n));
                pairs4 |= (uint64_t)pair_rt<V>(pi[i], pi[n]) << (4 * C::pair(i, n));
            }
    }
    // gathers of a group: lane k of a cell takes vertex k and the dofs k, k + LPC, ...
    const int64_t ngroups = (A.ncells + CPW - 1) / CPW;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    int vid = 0, uid[RL];
    double xr[D], ur[RL][D];
    auto cell_of = [&](int64_t g) -> int64_t {
        const int64_t c = g * CPW + cl;
        return c < A.ncells ? c : A.ncells - 1;
    };
    auto load_ids = [&](int64_t g) {
        const int64_t c = cell_of(g);
        vid = A.c2v[c * V + (k < V ? k : 0)];
        if (A.u.map) {
#pragma unroll
            for (int t = 0; t < RL; ++t) uid[t] = A.u.map[c * NS + (k + t * LPC < NS ? k + t * LPC : 0)];
        }
    };
    auto load_vals = [&](int64_t g) {
        const int64_t c = cell_of(g);
#pragma unroll
        for (int i = 0; i < D; ++i) xr[i] = A.coords[(int64_t)vid * D + i];
#pragma unroll
        for (int t = 0; t < RL; ++t) {
            const int r = k + t * LPC < NS ? k + t * LPC : 0;
            const int64_t at = A.u.map ? (int64_t)uid[t] * D : (c * NS + r) * D;
#pragma unroll
            for (int i = 0; i < D; ++i) ur[t][i] = A.u.values[at + i];
        }
    };
    int64_t grp = (int64_t)blockIdx.x * 4 + wave;
    if (grp >= ngroups) return;  // wave-uniform; no workgroup barrier follows
    load_ids(grp);
    load_vals(grp);
    load_ids(grp + nwaves < ngroups ? grp + nwaves : grp);
    for (; grp < ngroups; grp += nwaves) {
        // the lane's place in its cell, read again opaquely for every group:
        // the LDS offsets that follow from it are formed where they are used
        // instead of being kept across the loop (hundreds of registers)
        int kk = lane % LPC;
        asm volatile("" : "+v"(kk));
        const int blk = kk % NB, half = kk / NB;
        int c1 = 0, c2 = 0;
        {
            int t = blk;
            while (t >= D - c1) { t -= D - c1; ++c1; }
            c2 = c1 + t;
        }
        const double dg = c1 == c2 ? 1.0 : 0.0, dg2 = 2.0 * dg;
        // vertex permutation of the half, pairs of permuted vertices
        int pi[V], pr[NP];
#pragma unroll
        for (int v = 0; v < V; ++v) pi[v] = half == 0 ? v : (v < 2 ? v + 2 : 3 - v);
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int w = v; w < V; ++w) pr[C::pair(v, w)] = (int)((pairs4 >> (4 * C::pair(v, w))) & 15);
        // the cell's vertices and dofs to LDS; the next group's gathers
        if (owner) {
            if (k < V) {
#pragma unroll
                for (int i = 0; i < D; ++i) cc[C::X + k * D + i] = xr[i];
            }
#pragma unroll
            for (int t = 0; t < RL; ++t)
                if (k + t * LPC < NS) {
#pragma unroll
                    for (int i = 0; i < D; ++i) cc[C::U + (k + t * LPC) * D + i] = ur[t][i];
                }
        }
        const int64_t n1 = grp + nwaves < ngroups ? grp + nwaves : grp;
        const int64_t n2 = grp + 2 * nwaves < ngroups ? grp + 2 * nwaves : n1;
        load_vals(n1);
        load_ids(n2);
        wave_sync();
        Geom<D> g;
        {
            double x[V][D];
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int i = 0; i < D; ++i) x[v][i] = cc[C::X + v * D + i];
            geometry_from_coords<D>(x, g);
        }
        const double scale = g.adet * (16.0 / 5040.0);  // 16 |det J| / (D + 4)!
        if (owner && k < D) {
            // component k: reference gradient (GG), physical gradient (HH) and
            // m = K K^T (reference gradient) in barycentric components (MM) at the vertices
            double v[NS], gr[V][D], kc[D];  // kc: column k of K
#pragma unroll
            for (int a = 0; a < D; ++a) {
                kc[a] = g.K[a][0];
#pragma unroll
                for (int e = 1; e < D; ++e) kc[a] = k == e ? g.K[a][e] : kc[a];
            }
#pragma unroll
            for (int r = 0; r < NS; ++r) v[r] = cc[C::U + r * D + k];
            grad_nodes<D, 2>(v, gr);
#pragma unroll
            for (int n = 0; n < V; ++n) {
                double h[D], y0 = 0.0, z0 = 0.0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) t += gr[n][a] * g.K[a][j];
                    h[j] = t;
                    cc[C::HH + (k * V + n) * D + j] = t;
                    cc[C::GG + (k * V + n) * D + j] = gr[n][j];
                }
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    double t = 0.0;
#pragma unroll
                    for (int j = 0; j < D; ++j) t += g.K[a][j] * h[j];
                    cc[C::MM + (k * V + n) * V + a + 1] = t;
                    cc[C::KF + (k * V + n) * V + a + 1] = kc[a] + t;
                    y0 -= t;
                    z0 -= kc[a] + t;
                }
                cc[C::MM + (k * V + n) * V] = y0;
                cc[C::KF + (k * V + n) * V] = z0;
            }
        }
        if (owner && k == LPC - 1) {
            // barycentric rows of K and their products
            double kb[V][D];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                double t = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    kb[a + 1][j] = g.K[a][j];
                    t -= g.K[a][j];
                }
                kb[0][j] = t;
            }
#pragma unroll
            for (int i = 0; i < V; ++i) {
#pragma unroll
                for (int j = 0; j < D; ++j) cc[C::KB + i * D + j] = kb[i][j];
#pragma unroll
                for (int j = i; j < V; ++j) {
                    double t = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) t += kb[i][a] * kb[j][a];
                    cc[C::MB + C::pair(i, j)] = t;
                }
            }
        }
        wave_sync();
        // for the pair (v, w): the coefficient of tr E = sum_e H_ee + |H_e|^2 / 2, then those of
        // (K S K^T)_ij = lambda tr E (K K^T)_ij + mu sum_e (K_ie m_e,j + m_e,i K_je + m_e,i m_e,j)
#pragma unroll 1
        for (int p = kk; owner && p < NP; p += LPC) {
            int v = 0, w = p;
            while (w >= V - v) { w -= V - v; ++v; }
            w += v;
            double mv[D][V], mw[D][V], tau = 0.0;
#pragma unroll
            for (int e = 0; e < D; ++e) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    mv[e][i] = cc[C::MM + (e * V + v) * V + i];
                    mw[e][i] = cc[C::MM + (e * V + w) * V + i];
                }
                double x = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a)
                    x += cc[C::GG + (e * V + v) * D + a] * mw[e][a + 1] + cc[C::GG + (e * V + w) * D + a] * mv[e][a + 1];
                tau += 0.5 * (cc[C::HH + (e * V + v) * D + e] + cc[C::HH + (e * V + w) * D + e]) + 0.25 * x;
            }
            // mu F_c . F_c' (twice the coefficient for v < w, as e_nl below)
            {
                double gv[D][D], gw[D][D], hh[D][D];
#pragma unroll
                for (int e = 0; e < D; ++e)
#pragma unroll
                    for (int a = 0; a < D; ++a) {
                        gv[e][a] = cc[C::GG + (e * V + v) * D + a];
                        gw[e][a] = cc[C::GG + (e * V + w) * D + a];
                        hh[e][a] = cc[C::HH + (e * V + v) * D + a] + cc[C::HH + (e * V + w) * D + a];
                    }
                const double f2 = v == w ? 0.5 * mu : mu;
                int blk2 = 0;
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int b = a; b < D; ++b, ++blk2) {
                        double x = hh[a][b] + hh[b][a];
#pragma unroll
                        for (int t = 0; t < D; ++t) x += gv[a][t] * mw[b][t + 1] + gw[a][t] * mv[b][t + 1];
                        cc[C::PH + blk2 * NP + p] = f2 * ((a == b ? 2.0 : 0.0) + x);
                    }
            }
#pragma unroll
            for (int i = 0; i < V; ++i)
#pragma unroll
                for (int j = i; j < V; ++j) {
                    double x = 0.0;
#pragma unroll
                    for (int e = 0; e < D; ++e)
                        x += cc[C::KB + i * D + e] * (mv[e][j] + mw[e][j]) + cc[C::KB + j * D + e] * (mv[e][i] + mw[e][i]) +
                             mv[e][i] * mw[e][j] + mw[e][i] * mv[e][j];
                    cc[C::SB + C::pair(i, j) * NP + p] = lm * tau * cc[C::MB + C::pair(i, j)] + 0.5 * mu * x;
                }
        }
        wave_sync();
        // this lane's k_c1, k_c2 at the (permuted) vertices, mu (F_c1 . F_c2)
        double f[V][V], q2[V][V], ph[NP];
#pragma unroll
        for (int n = 0; n < V; ++n) {
            const double *fn = cc + C::KF + (c1 * V + pi[n]) * V, *qn = cc + C::KF + (c2 * V + pi[n]) * V;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                f[n][i] = fn[pi[i]];
                q2[n][i] = qn[pi[i]];
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) ph[p] = cc[C::PH + blk * NP + pr[p]];
        double acc[NS][C::NCOL];
#pragma unroll
        for (int a = 0; a < NS; ++a)
#pragma unroll
            for (int b = 0; b < C::NCOL; ++b) acc[a][b] = 0.0;
        static_for<V>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            double lf[V], mg[V];
#pragma unroll
            for (int n = 0; n < V; ++n) {
                lf[n] = lm * f[n][i];
                mg[n] = mu * q2[n][i];
            }
            // the gradients of the barycentric coordinates sum to zero: j = 0
            // is minus the sum of the others, formed last
            double hs[V], es[V][V], rs[V], cs = 0.0;
#pragma unroll
            for (int n = 0; n < V; ++n) {
                hs[n] = rs[n] = 0.0;
#pragma unroll
                for (int l = 0; l < V; ++l) es[n][l] = 0.0;
            }
            static_for<V>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = (decltype(jc)::value + 1) % V;
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                // e_nl = 2 h^nl (n < l), hd_n = h^nn
                double hd[V], e[V][V], rn[V], Cs = 0.0;
                if constexpr (j != 0) {
                    const int ij = pr[C::pair(i, j)];
                    const double* sbij = cc + C::SB + ij * NP;
                    const double mij = cc[C::MB + ij];
#pragma unroll
                    for (int n = 0; n < V; ++n) {
                        hd[n] = lf[n] * q2[n][j] + mg[n] * f[n][j] + ph[C::pair(n, n)] * mij + dg * sbij[pr[C::pair(n, n)]];
                        rn[n] = 4.0 * hd[n];
                        Cs += 2.0 * hd[n];
                        hs[n] -= hd[n];
                    }
#pragma unroll
                    for (int n = 0; n < V; ++n)
#pragma unroll
                        for (int l = n + 1; l < V; ++l) {
                            const double x = lf[n] * q2[l][j] + mg[n] * f[l][j] + lf[l] * q2[n][j] + mg[l] * f[n][j] +
                                             ph[C::pair(n, l)] * mij + dg2 * sbij[pr[C::pair(n, l)]];
                            e[n][l] = e[l][n] = x;
                            rn[n] += x;
                            rn[l] += x;
                            Cs += x;
                            es[n][l] -= x;
                            es[l][n] = es[n][l];
                        }
#pragma unroll
                    for (int n = 0; n < V; ++n) rs[n] -= rn[n];
                    cs -= Cs;
                } else {
                    Cs = cs;
#pragma unroll
                    for (int n = 0; n < V; ++n) {
                        hd[n] = hs[n];
                        rn[n] = rs[n];
#pragma unroll
                        for (int l = 0; l < V; ++l) e[n][l] = es[n][l];
                    }
                }
                static_for<V * V>([&](auto nq) __attribute__((always_inline)) {
                    constexpr int n = decltype(nq)::value / V, q = decltype(nq)::value % V;
                    if constexpr (C::col(j, q) >= 0) {
                        double w = n == q ? 2.0 * (Cs + 2.0 * rn[n] + 2.0 * hd[n]) : Cs + rn[n] + rn[q] + e[n][q];
                        if (n == i) w -= 0.25 * (D + 4) * (Cs + rn[q]);
                        if (q == j) w -= 0.25 * (D + 4) * (Cs + rn[n]);
                        if (n == i && q == j) w += 0.0625 * (D + 3) * (D + 4) * Cs;
                        acc[C::row(i, n)][C::col(j, q)] += w;
                        // in order: left free, the sums of all (i, j) are kept apart until the end
                        asm volatile("" : "+v"(acc[C::row(i, n)][C::col(j, q)]));
                    }
                });
            });
        });
        wave_sync();
        // stage the group's tensors and write them
        if (owner) {
            asm volatile("" : "+v"(dofs4));
            // element offsets: upper block at (rd, cd), its transpose at (cd, rd)
            OT* up = reinterpret_cast<OT*>(wl) + cl * N * N + c1 * NS * N + c2 * NS;
            OT* lo = reinterpret_cast<OT*>(wl) + cl * N * N + c2 * NS * N + c1 * NS;
            int cd[C::NCOL];
            static_for<V * V>([&](auto jq) __attribute__((always_inline)) {
                constexpr int j = decltype(jq)::value / V, q = decltype(jq)::value % V;
                if constexpr (j <= q && C::col(j, q) >= 0) cd[C::col(j, q)] = (int)((dofs4 >> (4 * C::pair(j, q))) & 15);
            });
            static_for<V * V>([&](auto in) __attribute__((always_inline)) {
                constexpr int i = decltype(in)::value / V, n = decltype(in)::value % V;
                if constexpr (i <= n) {
                    const int rd = (int)((dofs4 >> (4 * C::pair(i, n))) & 15);
                    OT *ur = up + rd * N, *lr = lo + rd;
#pragma unroll
                    for (int b = 0; b < C::NCOL; ++b) acc[C::row(i, n)][b] *= scale;
#pragma unroll
                    for (int b = 0; b < C::NCOL; ++b) ur[cd[b]] = (OT)acc[C::row(i, n)][b];
                    if (c1 != c2) {
#pragma unroll
                        for (int b = 0; b < C::NCOL; ++b) lr[cd[b] * N] = (OT)acc[C::row(i, n)][b];
                    }
                }
            });
        }
        wave_sync();
        const int64_t c0 = grp * CPW;
        const int nc = A.ncells - c0 < CPW ? (int)(A.ncells - c0) : CPW;
        constexpr int CPC = N * N * (int)sizeof(OT) / 16;  // 16-byte chunks per cell
        static_assert(N * N * sizeof(OT) % 16 == 0, "whole cells in 16-byte stores");
        const svk_u32x4* s4 = reinterpret_cast<const svk_u32x4*>(wl);
        svk_u32x4* o4 = reinterpret_cast<svk_u32x4*>(A.out) + c0 * CPC;
        const int nv = nc * CPC;
#pragma unroll
        for (int e0 = 0; e0 < CPW * CPC; e0 += 64)
            if (e0 + lane < nv) gstore_nt(&o4[e0 + lane], s4[e0 + lane]);
        wave_sync();
    }
}

}  // namespace dev

// ---------------------------------------------------------------- host side

// workgroups of the degree-2 Jacobian per CU
constexpr int kJac2Grid = 4;

static std::mutex g_svk_mu;
static std::map<std::tuple<int, int, int, int>, void*> g_svk_tabs;  // (dev, dim, p, q)

static coffee_status svk_table(int dev, int dim, int p, int q, const double** out) {
    std::lock_guard<std::mutex> lk(g_svk_mu);
    auto key = std::make_tuple(dev, dim, p, q);
    auto it = g_svk_tabs.find(key);
    if (it != g_svk_tabs.end()) {
        *out = (const double*)it->second;
        return COFFEE_OK;
    }
    // The SVK integrands at q = 2p are polynomials of degree exactly 2p on an
    // affine cell (F is of degree p - 1), so every rule exact to degree q
    // gives the same integral up to rounding: P2 uses the fully symmetric
    // rule (6 points on triangles, 14 on tetrahedra, against 9 and 27 for the
    // collapsed Gauss-Jacobi rule of that degree).
    Tables t;
    if (!t.init(dim, p, p == 2 ? COFFEE_QUAD(q & 15, COFFEE_RULE_SYMMETRIC) : q)) return COFFEE_E_INVALID_ARG;
    std::vector<double> h;
    if (p == 1) {
        // P1 on an affine cell: the displacement gradient, hence the whole
        // integrand, is the same at every point, so the point loop is
        // invariant (section 3.2's loop-invariant code motion applied to the
        // whole loop): one point carrying the summed weight.
        long double w = 0.0L;
        for (int k = 0; k < t.nq; ++k) w += t.W[k];
        h.push_back((double)w);
        for (int al = 0; al < dim; ++al)
            for (int a = 0; a < t.n; ++a) h.push_back((double)t.dphi[((size_t)al * t.nq + 0) * t.n + a]);
    } else {
        for (int k = 0; k < t.nq; ++k) h.push_back((double)t.W[k]);
        for (size_t i = 0; i < t.dphi.size(); ++i) h.push_back((double)t.dphi[i]);
    }
    // the basis of degree p - 1 at the points (P1: the one value 1)
    Tables nd;
    if (!nd.init(dim, p - 1, t.q)) return COFFEE_E_INVALID_ARG;
    for (int k = 0; k < (p == 1 ? 1 : nd.nq); ++k)
        for (int i = 0; i < nd.n; ++i) h.push_back((double)nd.phi[(size_t)k * nd.n + i]);
    void* d = nullptr;
    if (hipMalloc(&d, h.size() * sizeof(double)) != hipSuccess) return COFFEE_E_NOMEM;
    if (hipMemcpy(d, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(d);
        return COFFEE_E_HIP;
    }
    g_svk_tabs[key] = d;
    *out = (const double*)d;
    return COFFEE_OK;
}

void free_svk_tables() {
    std::lock_guard<std::mutex> lk(g_svk_mu);
    for (auto& kv : g_svk_tabs) {
        (void)hipSetDevice(std::get<0>(kv.first));
        (void)hipFree(kv.second);
    }
    g_svk_tabs.clear();
}

namespace {

constexpr int svk_jac_slices(int, int p) { return p == 2 ? 2 : 1; }

template <typename OT>
hipError_t launch_jac2(const dev::SvkArgs& a, hipStream_t s, int ncu) {
    using C = dev::SvkJ2;
    constexpr int lds = 4 * C::wave_bytes<OT>();
    static_assert(lds <= 160 * 1024, "LDS");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&dev::k_svk_jac2<OT>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    const int64_t groups = (a.ncells + C::CPW - 1) / C::CPW;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((groups + 3) / 4, (int64_t)ncu * kJac2Grid));
    hipLaunchKernelGGL((dev::k_svk_jac2<OT>), dim3(grid), dim3(256), lds, s, a);
    return hipGetLastError();
}

// compiled set: triangles and tetrahedra, P1 (q = 2, evaluated at one point
// with the summed weight) and P2 (q = 4)
template <int D, int P, int NQ>
hipError_t launch_svk(int form, int precision, const dev::SvkArgs& a, hipStream_t s, int ncu, bool reverse) {
    const int64_t blocks = (a.ncells + 255) / 256;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(blocks, (int64_t)ncu * 8));
    // reverse pass: the workgroups that fit, by registers and LDS (both
    // gradients, us: P2 tetrahedra, 196,608 / 2,058,000 cells: one per CU 54 and
    // 495, two 58 and 494, eight 63 and 519; P1 tetrahedra, 196,608 /
    // 1,296,000: two 18 and 93, three 19 and 108, eight 20 and 96; P1
    // triangles, 720,000: one 37, two 29, three 25, eight 27; the coordinates
    // alone, against eight per CU and no loads ahead, P2 tetrahedra, 200,003, 45 ->
    // 35, P1 tetrahedra, 600,011, 61 -> 31; the deterministic mode, whose sort
    // outweighs the kernel, 486 -> 459 and 564 -> 563). Loading each
    // cell's values behind the previous one's atomics, eight per CU: P2
    // tetrahedra 59 and 557, P1 22 and 95, P1 triangles 29, P2 triangles,
    // 180,000, 21 -> 18.
    auto rgrid = [&](int mode) {
        const int fit = D == 2 ? 3 : (P == 2 && mode == 3 ? 1 : 2);
        return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, (int64_t)ncu * fit));
    };
    if (reverse) {
        if (form == COFFEE_SVK_RESIDUAL)
            hipLaunchKernelGGL((dev::k_svk_res_adj<D, P, NQ>), dim3(grid), dim3(256), 0, s, a);
        else if (!a.grad_u && !a.grad_coords && !a.det_x) {
            // the values alone: the energy's own kernel, without tables, and at
            // the occupancy that a gather wants (600,011 cells, mesh / random
            // order, us, the coordinates' kernel -> this: P1 tetrahedra 19 / 40 ->
            // 14 / 40, P2 71 / 113 -> 40 / 100, P2 triangles 21 / 57 -> 15 / 56)
            dev::SvkArgs v = a;
            v.out = a.cell_value;
            if (v.out) hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 0, double>), dim3(grid), dim3(256), 0, s, v);
        } else if (a.grad_u || a.det_u)
            hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 3, double>), dim3(rgrid(3)), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 2, double>), dim3(rgrid(2)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    const bool f64 = precision == COFFEE_FP64;
    if (form == COFFEE_SVK_ENERGY) {
        if (f64) hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 0, double>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 0, float>), dim3(grid), dim3(256), 0, s, a);
    } else if (form == COFFEE_SVK_RESIDUAL) {
        if (f64) hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 1, double>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((dev::k_svk_vec<D, P, NQ, 1, float>), dim3(grid), dim3(256), 0, s, a);
    } else {
        if constexpr (P == 2 && D == 3)
            return f64 ? launch_jac2<double>(a, s, ncu) : launch_jac2<float>(a, s, ncu);
        constexpr int AH = svk_jac_slices(D, P);
        constexpr int CPW = 64 / (D * (D + 1) / 2 * AH);
        const int64_t waves = (a.ncells + CPW - 1) / CPW;
        const int g2 = (int)std::max<int64_t>(1, std::min<int64_t>((waves + 3) / 4, (int64_t)ncu * 16));
        if constexpr (P == 1 || D == 2) {
            if (f64) hipLaunchKernelGGL((dev::k_svk_jac<D, P, NQ, double, AH>), dim3(g2), dim3(256), 0, s, a);
            else hipLaunchKernelGGL((dev::k_svk_jac<D, P, NQ, float, AH>), dim3(g2), dim3(256), 0, s, a);
        }
    }
    return hipGetLastError();
}

hipError_t dispatch_svk(int form, int dim, int p, int q, int precision, const dev::SvkArgs& a, hipStream_t s,
                        int ncu, bool reverse, bool* found) {
    *found = true;
    q &= 15;  // either rule family: the integrands are integrated exactly (svk_table)
    if (dim == 2 && p == 1 && q == 2) return launch_svk<2, 1, 1>(form, precision, a, s, ncu, reverse);
    if (dim == 2 && p == 2 && q == 4) return launch_svk<2, 2, 6>(form, precision, a, s, ncu, reverse);
    if (dim == 3 && p == 1 && q == 2) return launch_svk<3, 1, 1>(form, precision, a, s, ncu, reverse);
    if (dim == 3 && p == 2 && q == 4) return launch_svk<3, 2, 14>(form, precision, a, s, ncu, reverse);
    *found = false;
    return hipSuccess;
}

coffee_status svk_common(int cell, int degree, int q, const double* coords, const int32_t* c2v, int64_t ncells,
                         const coffee_field* coeffs, const double* constants, int nconst, dev::SvkArgs& a,
                         const double** tab, int* dev_out) {
    if (coeffs[0].degree != degree) return COFFEE_E_UNSUPPORTED;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return COFFEE_E_HIP;
    coffee_status st = svk_table(dev, cell, degree, q, tab);
    if (st != COFFEE_OK) return st;
    std::memset(&a, 0, sizeof a);
    a.coords = coords;
    a.c2v = c2v;
    a.ncells = ncells;
    a.u = dev::FieldArg{coeffs[0].values, coeffs[0].cell_to_dof};
    a.mu = nconst > 0 ? constants[0] : 1.0;
    a.lambda = nconst > 1 ? constants[1] : 1.0;
    a.tab = *tab;
    *dev_out = dev;
    return COFFEE_OK;
}

}  // namespace

coffee_status assemble_svk(int form, int cell, int degree, int q, int precision, const double* coords, int64_t nvert,
                           const int32_t* c2v, int64_t ncells, const coffee_field* coeffs, const double* constants,
                           int nconst, void* out, void* hip_stream) {
    (void)nvert;
    if (precision == COFFEE_BF16X3)
        return assemble_svk_bf16(form, cell, degree, q, coords, c2v, ncells, coeffs, constants, nconst, out,
                                 hip_stream);
    if (ncells == 0) return COFFEE_OK;
    dev::SvkArgs a;
    const double* tab = nullptr;
    int dev = 0;
    coffee_status st = svk_common(cell, degree, q, coords, c2v, ncells, coeffs, constants, nconst, a, &tab, &dev);
    if (st != COFFEE_OK) return st;
    a.out = out;
    bool found = false;
    hipError_t e = dispatch_svk(form, cell, degree, q, precision, a, (hipStream_t)hip_stream, num_cu(dev), false, &found);
    if (!found) return COFFEE_E_UNSUPPORTED;
    return e == hipSuccess ? COFFEE_OK : COFFEE_E_HIP;
}

coffee_status adjoint_svk(int form, int cell, int degree, int q, const double* coords, const int32_t* c2v,
                          int64_t ncells, const coffee_field* coeffs, const double* constants, int nconst,
                          const double* lam, double seed, double* grad_coords, double* const* grad_coeff_values,
                          double* cell_value, const DetTarget* det, void* hip_stream) {
    if (form == COFFEE_SVK_RESIDUAL && ncells > 0 && !lam) return COFFEE_E_INVALID_ARG;
    if (ncells == 0) return COFFEE_OK;
    dev::SvkArgs a;
    const double* tab = nullptr;
    int dev = 0;
    coffee_status st = svk_common(cell, degree, q, coords, c2v, ncells, coeffs, constants, nconst, a, &tab, &dev);
    if (st != COFFEE_OK) return st;
    a.seed = seed;
    a.grad_coords = grad_coords;
    a.grad_u = grad_coeff_values ? grad_coeff_values[0] : nullptr;
    a.cell_value = cell_value;
    a.lam = lam;
    if (det) {
        a.det_x = det[0].local;
        a.det_u = det[1].local;
    }
    bool found = false;
    hipError_t e = dispatch_svk(form, cell, degree, q, COFFEE_FP64, a, (hipStream_t)hip_stream, num_cu(dev), true,
                                &found);
    if (!found) return COFFEE_E_UNSUPPORTED;
    return e == hipSuccess ? COFFEE_OK : COFFEE_E_HIP;
}

// The gradient arrays of a reverse pass as deterministic-scatter targets:
// vertex coordinates (entries: cells x vertices, keys cell_to_vertex), then
// each coefficient field (entries: cells x local dofs, keys its dof map, or
// one entry per value for a cell-major field).
int adjoint_det_targets(int cell, int64_t nvert, const int32_t* c2v, int64_t ncells, const coffee_field* coeffs,
                        int ncoeff, double* grad_coords, double* const* grad_coeff_values, DetTarget* t) {
    const int d = cell;
    t[0] = DetTarget{c2v, 1, ncells * (d + 1), d, nvert, nullptr, grad_coords};
    for (int i = 0; i < ncoeff; ++i) {
        const int64_t n = ncells * n_scalar(d, coeffs[i].degree);
        const int32_t* keys = coeffs[i].cell_to_dof;
        // the field's dof count is not passed: its keys are sorted over 31 bits
        t[1 + i] = DetTarget{keys, keys ? 1 : 0, n, coeffs[i].ncomp, keys ? ((int64_t)1 << 31) : n, nullptr,
                             grad_coeff_values ? grad_coeff_values[i] : nullptr};
    }
    return 1 + ncoeff;
}

}  // namespace coffee

extern "C" coffee_status coffee_assemble_adjoint(int form, int cell, int degree, int quad_degree,
                                                 const double* coords, int64_t nvert, const int32_t* c2v,
                                                 int64_t ncells, const coffee_field* coeffs, int ncoeff,
                                                 const double* constants, int nconst, const double* lam,
                                                 const double* u, double seed, double* grad_coords,
                                                 double* const* grad_coeff_values, double* cell_value,
                                                 int deterministic, void* workspace, int64_t workspace_bytes,
                                                 void* hip_stream) {
    using namespace coffee;
    int q = 0, fd = 0;
    coffee_status st = validate_common(form, cell, degree, quad_degree, coords, nvert, c2v, ncells, coeffs, ncoeff,
                                       constants, nconst, &q, &fd);
    if (st != COFFEE_OK) return st;
    if (deterministic != 0 && deterministic != 1) return COFFEE_E_INVALID_ARG;
    if (form == COFFEE_SVK_JACOBIAN || cell == COFFEE_PRISM) return COFFEE_E_UNSUPPORTED;
    if (!is_svk_form(form) && ncells > 0 && (!lam || !u)) return COFFEE_E_INVALID_ARG;
    for (int i = 0; i < ncoeff; ++i)
        if (coeffs[i].ncomp > 3) return COFFEE_E_UNSUPPORTED;
    DetTarget det[3];
    int ndet = 0;
    if (deterministic) {
        ndet = adjoint_det_targets(cell, nvert, c2v, ncells, coeffs, ncoeff, grad_coords, grad_coeff_values, det);
        st = det_carve(workspace, workspace_bytes, det, ndet);
        if (st != COFFEE_OK) return st;
    }
    if (is_svk_form(form))
        st = adjoint_svk(form, cell, degree, q, coords, c2v, ncells, coeffs, constants, nconst, lam, seed,
                         grad_coords, grad_coeff_values, cell_value, deterministic ? det : nullptr, hip_stream);
    else
        st = adjoint_linear(form, cell, degree, q, fd, coords, nvert, c2v, ncells, coeffs, ncoeff, constants, nconst,
                            lam, u, seed, grad_coords, grad_coeff_values, cell_value, deterministic ? det : nullptr,
                            hip_stream);
    if (st != COFFEE_OK || !deterministic || ncells == 0) return st;
    return det_scatter(det, ndet, workspace, (hipStream_t)hip_stream);
}

extern "C" int64_t coffee_adjoint_workspace_size(int form, int cell, int degree, int64_t nvert, int64_t ncells,
                                                 const coffee_field* coeffs, int ncoeff) {
    using namespace coffee;
    if (form < COFFEE_MASS || form > COFFEE_DIFFUSION || form == COFFEE_SVK_JACOBIAN) return -1;
    if ((cell != COFFEE_TRIANGLE && cell != COFFEE_TETRAHEDRON) || degree < 1 || degree > kMaxP) return -1;
    if (nvert < 0 || ncells < 0 || ncoeff < 0 || ncoeff > 2 || (ncoeff > 0 && !coeffs)) return -1;
    for (int i = 0; i < ncoeff; ++i)
        if (coeffs[i].degree < 1 || coeffs[i].degree > kMaxP || coeffs[i].ncomp < 1 || coeffs[i].ncomp > 3) return -1;
    DetTarget det[3];
    const int ndet = adjoint_det_targets(cell, nvert, nullptr, ncells, coeffs, ncoeff, nullptr, nullptr, det);
    return det_workspace_bytes(det, ndet);
}
