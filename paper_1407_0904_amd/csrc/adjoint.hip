// Reverse mode of the linear-form assembly.
//
// For a bilinear form the per-cell functional S_e = lam_e^T A_e u_e equals
// sum_blk sum_k G^blk_k T^blk_k with T^blk_k = lam_{c1}^T R_k u_{c2}: the
// reference tensors are contracted with the test and trial vectors once, and
// the geometry tensor G carries every dependence on the cell. The transpose of
// the G builder (reverse_G, beside build_G in linear.hpp) maps Gbar = T to
// Kbar = dS/dK and to the bars of the local coefficient dofs; every term of G
// is linear in |det J|, so dS/d|det J| = S / |det J|. The chain to the vertex
// coordinates is analytic:
//     dK = -K dJ K  ->  Jbar = -K^T Kbar K^T,
//     d|det J| = |det J| tr(K dJ)  ->  Jbar += Sbar_adet |det J| K^T,
//     J = [x1 - x0, ..., xd - x0]  ->  xbar_{j+1} = Jbar[:, j], xbar_0 = -sum_j Jbar[:, j].
// One thread per cell; gradients are scatter-added with FP64 atomics.
#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "library.h"
#include "linear.hpp"
#include "tables.h"

namespace coffee {
namespace dev {

struct AdjArgs {
    LinArgs L;               // mesh, fields, constants (rfrag/out unused)
    const double* R;         // reference tensors [KR][NS * NS]
    const double* lam;       // [E][N]
    const double* u;         // [E][N]
    double seed;
    double* grad_coords;     // [V][D]
    double* grad_f0;         // shaped like f0 values, or NULL
    double* grad_f1;
    double* cell_value;      // [E] or NULL
    // deterministic mode: per-cell contributions written here instead of
    // scatter-added (scatter.hip sums them in a fixed order); NULL otherwise
    double* det_x;           // [E][D+1][D]
    double* det_f0;          // [E][nloc][ncomp of field 0]
    double* det_f1;          // [E][nloc]
};

template <int FORM, int D, int FD>
struct AdjDirs {
    static constexpr int NF = nfield(D, FD);
    static constexpr int WC = (FORM == F_BURG) ? D : 1;
    static constexpr int N0 = FD > 0 ? NF * WC : 0;                      // field 0 dofs
};

// Accumulate the contribution of block B: value, Kbar and coefficient bars.
template <int FORM, int D, int P, int FD, int B>
__device__ inline void adjoint_block(const AdjArgs& A, const double* Rs, const CellData<FORM, D, FD, double>& cd,
                                     const double* lam_e,
                                     const double* u_e, double& S, double (&Kbar)[D][D], double* f0bar) {
    constexpr int NS = nsc(D, P), NN = NS * NS;
    constexpr int NC = ncomp_space(FORM, D);
    constexpr int C1 = B / NC, C2 = B % NC;
    // the block's rows of lam_e and u_e (re-read per block from the L1 cache)
    double lam[NS], u[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        lam[i] = lam_e[C1 * NS + i];
        u[i] = u_e[C2 * NS + i];
    }
    // gbar(k) = T_k = lam_c1^T R_k u_c2 (R_k read with wave-uniform addresses)
    auto gbar = [&](int k) -> double {
        // keeps the compiler from hoisting every R_k load of the block into
        // registers at once
        asm volatile("" ::: "memory");
        const double* Rk = Rs + (size_t)k * NN;
        double t = 0.0;
#pragma unroll 1
        for (int a = 0; a < NS; ++a) {
            double r = 0.0;
#pragma unroll
            for (int b = 0; b < NS; ++b) r += Rk[a * NS + b] * u[b];
            t += lam[a] * r;
        }
        return t;
    };
    reverse_G<FORM, D, FD, C1, C2>(cd, A.L, gbar, S, Kbar, f0bar);
}

// One block per iteration of a runtime loop, so that the compiler keeps one
// block's temporaries live at a time.
template <int FORM, int D, int P, int FD, int B, int NB>
__device__ inline void adjoint_block_switch(int b, const AdjArgs& A, const double* Rs,
                                            const CellData<FORM, D, FD, double>& cd, const double* lam,
                                            const double* u, double& S, double (&Kbar)[D][D], double* f0bar) {
    if constexpr (B < NB) {
        if (b == B) adjoint_block<FORM, D, P, FD, B>(A, Rs, cd, lam, u, S, Kbar, f0bar);
        else adjoint_block_switch<FORM, D, P, FD, B + 1, NB>(b, A, Rs, cd, lam, u, S, Kbar, f0bar);
    }
}

template <int FORM, int D, int P, int FD, int NB>
__device__ inline void adjoint_blocks(const AdjArgs& A, const double* Rs, const CellData<FORM, D, FD, double>& cd,
                                      const double* lam, const double* u, double& S, double (&Kbar)[D][D],
                                      double* f0bar) {
#pragma unroll 1
    for (int b = 0; b < NB; ++b)
        adjoint_block_switch<FORM, D, P, FD, 0, NB>(b, A, Rs, cd, lam, u, S, Kbar, f0bar);
}

// Reference tensors of the adjoint kernels live in LDS when they fit.
template <int FORM, int D, int P, int FD>
constexpr int adj_r_elems() { return kref(FORM, D, FD) * nsc(D, P) * nsc(D, P); }
template <int FORM, int D, int P, int FD>
constexpr bool adj_r_in_lds() { return adj_r_elems<FORM, D, P, FD>() * 8 <= 56 * 1024; }

template <int FORM, int D, int P, int FD>
__global__ __launch_bounds__(256) void k_adjoint_linear(AdjArgs A) {
    constexpr int NS = nsc(D, P);
    constexpr int NC = ncomp_space(FORM, D);
    constexpr int N = NC * NS;
    using Dirs = AdjDirs<FORM, D, FD>;
    constexpr bool LDSR = adj_r_in_lds<FORM, D, P, FD>();
    constexpr int RE = adj_r_elems<FORM, D, P, FD>();
    __shared__ double sR[LDSR ? RE : 1];
    const double* Rs = A.R;
    if constexpr (LDSR) {
        for (int i = threadIdx.x; i < RE; i += blockDim.x) sR[i] = A.R[i];
        __syncthreads();
        Rs = sR;
    }
    // per-wave combining of the gradient scatter-adds (vertex coordinates and
    // the field's dofs)
    constexpr int TS = 128;
    constexpr int W0 = Dirs::N0 > 0 ? Dirs::WC : 1;
    __shared__ unsigned long long ckx[4][TS], ck0[4][TS];
    __shared__ double cvx[4][TS * D], cv0[4][TS * W0];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // wave-uniform loop: every lane takes part in the tables' clear and flush
    for (int64_t wbase = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane; wbase < A.L.ncells;
         wbase += (int64_t)gridDim.x * blockDim.x) {
        const bool valid = wbase + lane < A.L.ncells;
        const int64_t cell = valid ? wbase + lane : A.L.ncells - 1;
        const bool det = A.det_x != nullptr;  // same in every lane
        if (!det) {
            combine_clear<D, TS>(ckx[wave], cvx[wave], lane);
            if constexpr (Dirs::N0 > 0) combine_clear<W0, TS>(ck0[wave], cv0[wave], lane);
            wave_sync();
        }
        CellIdx<FORM, D, FD> ix;
        CellRaw<FORM, D, FD> raw;
        load_idx<FORM, D, FD>(A.L, cell, ix);
        load_raw<FORM, D, FD>(A.L, cell, ix, raw);
        CellData<FORM, D, FD, double> cd;
        cell_from_raw<FORM, D, FD>(raw, cd);
        const double* lam = A.lam + cell * N;
        const double* u = A.u + cell * N;
        double S = 0.0, Kbar[D][D];
        double f0bar[Dirs::N0 > 0 ? Dirs::N0 : 1];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int j = 0; j < D; ++j) Kbar[i][j] = 0.0;
#pragma unroll
        for (int r = 0; r < (Dirs::N0 > 0 ? Dirs::N0 : 1); ++r) f0bar[r] = 0.0;
        adjoint_blocks<FORM, D, P, FD, NC * NC>(A, Rs, cd, lam, u, S, Kbar, f0bar);
        if (A.cell_value && valid) A.cell_value[cell] = S;

        // chain to the coordinates
        const auto& K = cd.g.K;
        const double adbar_ad = S;  // d S / d|det J| * |det J|
        double Jbar[D][D];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int j = 0; j < D; ++j) {
                // -(K^T Kbar K^T)_ij = -sum_ab K[a][i] Kbar[a][b] K[j][b]
                double s = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int b = 0; b < D; ++b) s += K[a][i] * Kbar[a][b] * K[j][b];
                Jbar[i][j] = -s + adbar_ad * K[j][i];
            }
        const double sd = A.seed;
        if (valid) {
            double vx[D + 1][D];
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
            if (det) {
#pragma unroll
                for (int v = 0; v <= D; ++v)
#pragma unroll
                    for (int i = 0; i < D; ++i) A.det_x[(cell * (D + 1) + v) * D + i] = vx[v][i];
                if constexpr (Dirs::N0 > 0) {
#pragma unroll
                    for (int r = 0; r < Dirs::N0; ++r) A.det_f0[cell * Dirs::N0 + r] = sd * f0bar[r];
                }
            } else {
                if (A.grad_coords) {
#pragma unroll
                    for (int v = 0; v <= D; ++v)
                        combine_add<D, TS>(ckx[wave], cvx[wave], (unsigned long long)ix.v[v], vx[v], A.grad_coords);
                }
                if constexpr (Dirs::N0 > 0) {
                    if (A.grad_f0) {
                        constexpr int NF = Dirs::NF;
#pragma unroll
                        for (int r = 0; r < NF; ++r) {
                            const int64_t key = A.L.f0.map ? (int64_t)ix.f0[r] : cell * NF + r;
                            double v[W0];
#pragma unroll
                            for (int c = 0; c < W0; ++c) v[c] = sd * f0bar[r * W0 + c];
                            combine_add<W0, TS>(ck0[wave], cv0[wave], (unsigned long long)key, v, A.grad_f0);
                        }
                    }
                }
            }
        }
        if (!det) {
            wave_sync();
            if (A.grad_coords) combine_flush<D, TS>(ckx[wave], cvx[wave], A.grad_coords, lane);
            if constexpr (Dirs::N0 > 0) {
                if (A.grad_f0) combine_flush<W0, TS>(ck0[wave], cv0[wave], A.grad_f0, lane);
            }
            wave_sync();
        }
    }
}

// Elasticity, degrees 1 and 2. The gradients of lam and u on a cell are
// polynomials of degree P - 1, fixed by their values H_k at the NV nodes of
// that degree (one node, or the vertices), and with
//     c_rkl = sum_q W_q psi_r N_k N_l   (psi_r: coefficient basis, N_k: degree P - 1 basis)
// the quadrature sum is exactly
//     S = |det J| sum_kl (sum_r c_rkl mu_r) 2 eps(Hlam_k):eps(Hu_l) + (sum_r c_rkl lambda_r) tr Hlam_k tr Hu_l.
// Each H_k takes a few differences of dofs (grad_nodes), so a cell costs about
// 1,000 multiply-adds for P2 tetrahedra, gradients included, where
// contracting lam and u with the reference tensors of all pairs of basis
// functions took 14,000 (663,552 cells: 665 us for that kernel, 190 for this).
// With Wu_k = sum_l (mu_kl (Hu_l + Hu_l^T) + lambda_kl tr Hu_l I), symmetric,
// and Wlam_k likewise: S = |det J| sum_k Hlam_k : Wu_k, and since every H is
// (reference gradient) K, the derivative in J is (S I - T) K^T,
//     T = |det J| sum_k (Hlam_k^T Wu_k + Hu_k^T Wlam_k).
// What is left is the read of lam and u, 480 bytes per cell: component by
// component through LDS (coalesced 8-byte reads) into rows of odd length per
// cell; and the scatter-adds. Of the 37,000 cycles a wave took for 64 P2
// tetrahedra the arithmetic was 3,000, the loads 10,000 to 14,000 (behind the
// previous cells' atomics), the combining 9,000, its flush 9,000. A persistent
// grid (one workgroup per CU and residency) now has all loads of the next
// cells in flight over the combining, complete before the flush issues its
// atomics: 170 -> 128 us (eight workgroups per CU 153); P2 triangles 49 -> 34.
// Values alone and the deterministic mode take the same grid: 600,011 P2
// tetrahedra, against the contraction with R at eight workgroups per CU, 586 ->
// 99 us and, with the sort, 1,379 -> 886.

// The H of P2 tetrahedra (144 registers) and what is formed from them need one
// wave per SIMD: at two, 255 registers spilled (352 us against 190).
template <int D, int P, int FD>
__global__ __launch_bounds__(256, (D == 3 && P == 2) ? 1 : 2) void k_adjoint_elast(AdjArgs A) {
    constexpr int NS = nsc(D, P), N = D * NS, NV = P == 1 ? 1 : D + 1, NF = nfield(D, FD), ROW = NS | 1;
    static_assert(FD == 1, "P1 coefficients");
    // per-wave combining of the gradient scatter-adds (vertex coordinates and
    // the two fields' dofs); the dof staging shares the memory of the values
    constexpr int TS = 256;
    static_assert(64 * ROW <= TS * D, "staging");
    __shared__ unsigned long long ckx[4][TS], ckf[4][2][TS];
    __shared__ double cvx[4][TS * D], cvf[4][2][TS];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double* stage = cvx[wave];
    const bool det = A.det_x != nullptr;  // same in every lane, as the next
    const bool shared_keys = A.L.f0.map == A.L.c2v && A.L.f1.map == A.L.c2v;  // the fields' dofs are the vertices
    // wave-uniform loop: every lane takes part in the staging, clear and flush
    int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane;
    if (base >= A.L.ncells) return;  // wave-uniform; no workgroup barrier follows
    CellIdx<F_ELAST, D, FD> ix, nx;  // of this unit and the next
    CellRaw<F_ELAST, D, FD> raw;
    double pre[2][D][NS];  // component c of lam, u of the wave's cells: flat entry 64 i + lane
    auto cell_at = [&](int64_t b) { return b + lane < A.L.ncells ? b + lane : A.L.ncells - 1; };
    // all of them are in flight at once; `more` false (no next unit): those of
    // one cell, so that the registers have one definition and little is read
    auto fetch = [&](int64_t b, bool more) {
        load_idx<F_ELAST, D, FD>(A.L, cell_at(b), nx);
        const int last = !more ? 0 : (A.L.ncells - b < 64 ? (int)(A.L.ncells - b) - 1 : 63);
        int ln = lane;  // opaque: the offsets are formed here, not kept across the loop
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int c = 0; c < D; ++c)
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const int t = 64 * i + ln, e = t / NS, a = t - e * NS;
                    pre[f][c][i] = gload((f == 0 ? A.lam : A.u) + b * N + (e < last ? e : last) * N + c * NS + a);
                }
    };
    fetch(base, true);
    load_raw<F_ELAST, D, FD>(A.L, cell_at(base), nx, raw);
    for (; base < A.L.ncells; base += (int64_t)gridDim.x * blockDim.x) {
        const bool valid = base + lane < A.L.ncells;
        const int64_t cell = cell_at(base), next = base + (int64_t)gridDim.x * blockDim.x;
        ix = nx;
        CellData<F_ELAST, D, FD, double> cd;
        cell_from_raw<F_ELAST, D, FD>(raw, cd);
        const auto& K = cd.g.K;
        const double ad = cd.g.adet;
        double H[2][NV][D][D];  // physical gradients of lam, u at the nodes
        wave_sync();
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int c = 0; c < D; ++c) {
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const int t = 64 * i + lane, e = t / NS;
                    stage[e * ROW + t - e * NS] = pre[f][c][i];
                }
                wave_sync();
                double v[NS], g[NV][D];
#pragma unroll
                for (int i = 0; i < NS; ++i) v[i] = stage[lane * ROW + i];
                wave_sync();
                grad_nodes<D, P>(v, g);
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        double x = 0.0;
#pragma unroll
                        for (int a = 0; a < D; ++a) x += g[k][a] * K[a][j];
                        H[f][k][c][j] = x;
                    }
            }
        if (!det) {
            combine_clear<D, TS>(ckx[wave], cvx[wave], lane);
            combine_clear<1, TS>(ckf[wave][0], cvf[wave][0], lane);
            combine_clear<1, TS>(ckf[wave][1], cvf[wave][1], lane);
            wave_sync();
        }
        double tr[2][NV];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                tr[f][k] = 0.0;
#pragma unroll
                for (int i = 0; i < D; ++i) tr[f][k] += H[f][k][i][i];
            }
        // coefficient weights of the node pairs and, with the pair products
        // eps:eps and tr tr, the bars of the coefficient dofs
        double mw[NV][NV], lw[NV][NV], mub[NF], lmb[NF];
#pragma unroll
        for (int r = 0; r < NF; ++r) mub[r] = lmb[r] = 0.0;
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int l = k; l < NV; ++l) {
                double pm = 0.0, pl = tr[0][k] * tr[1][l];
#pragma unroll
                for (int i = 0; i < D; ++i)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        pm += H[0][k][i][j] * (H[1][l][i][j] + H[1][l][j][i]);
                        if (l != k) pm += H[0][l][i][j] * (H[1][k][i][j] + H[1][k][j][i]);
                    }
                if (l != k) pl += tr[0][l] * tr[1][k];
                double m = 0.0, q = 0.0;
#pragma unroll
                for (int r = 0; r < NF; ++r) {
                    const double c = cload(A.R + (r * NV + k) * NV + l);
                    m += c * cd.f0[r];
                    q += c * cd.f1[r];
                    mub[r] += c * pm;
                    lmb[r] += c * pl;
                }
                mw[k][l] = mw[l][k] = m;
                lw[k][l] = lw[l][k] = q;
            }
        // S and T
        double S = 0.0, T[D][D];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int j = 0; j < D; ++j) T[i][j] = 0.0;
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                // W of the other field at node k
                double Wk[D][D], dil = 0.0;
#pragma unroll
                for (int l = 0; l < NV; ++l) dil += lw[k][l] * tr[1 - f][l];
#pragma unroll
                for (int i = 0; i < D; ++i)
#pragma unroll
                    for (int j = i; j < D; ++j) {
                        double x = i == j ? dil : 0.0;
#pragma unroll
                        for (int l = 0; l < NV; ++l) x += mw[k][l] * (H[1 - f][l][i][j] + H[1 - f][l][j][i]);
                        Wk[i][j] = Wk[j][i] = x;
                    }
#pragma unroll
                for (int c = 0; c < D; ++c)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        if (f == 0) S += H[0][k][c][j] * Wk[c][j];
#pragma unroll
                        for (int i = 0; i < D; ++i) T[i][j] += H[f][k][c][i] * Wk[c][j];
                    }
            }
        S *= ad;
        if (A.cell_value && valid) A.cell_value[cell] = S;
        // chain to the coordinates: Jbar = (S I - T) K^T, xbar_{j+1} = Jbar[:, j]
        const double sd = A.seed;
        double vx[D + 1][D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            double x0 = 0.0;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                double t = S * K[j][i];
#pragma unroll
                for (int a = 0; a < D; ++a) t -= ad * T[i][a] * K[j][a];
                vx[j + 1][i] = sd * t;
                x0 -= t;
            }
            vx[0][i] = sd * x0;
        }
        // the next unit's loads, complete before this one's atomics are issued
        // (one in-order counter: a load behind them would wait for them)
        const int64_t ahead = next < A.L.ncells ? next : base;
        fetch(ahead, next < A.L.ncells);
        __builtin_amdgcn_sched_barrier(0);
        if (valid && det) {
#pragma unroll
            for (int v = 0; v <= D; ++v)
#pragma unroll
                for (int i = 0; i < D; ++i) A.det_x[(cell * (D + 1) + v) * D + i] = vx[v][i];
#pragma unroll
            for (int r = 0; r < NF; ++r) {
                A.det_f0[cell * NF + r] = sd * ad * mub[r];
                A.det_f1[cell * NF + r] = sd * ad * lmb[r];
            }
        } else if (valid && !det) {
            static_assert(NF == D + 1, "a coefficient dof per vertex");
            unsigned long long kv[D + 1];
#pragma unroll
            for (int r = 0; r <= D; ++r) kv[r] = (unsigned long long)ix.v[r];
            if (shared_keys) {
                // vertex r: coordinates and both coefficients in one slot
                int h[D + 1];
                combine_slots<TS>(ckx[wave], kv, h);
#pragma unroll
                for (int r = 0; r <= D; ++r) {
                    const double m = sd * ad * mub[r], q = sd * ad * lmb[r];
                    if (h[r] >= 0) {
#pragma unroll
                        for (int i = 0; i < D; ++i) atomicAdd(&cvx[wave][h[r] * D + i], vx[r][i]);
                        atomicAdd(&cvf[wave][0][h[r]], m);
                        atomicAdd(&cvf[wave][1][h[r]], q);
                    } else {
#pragma unroll
                        for (int i = 0; i < D; ++i)
                            if (A.grad_coords) atomicAdd(A.grad_coords + (int64_t)ix.v[r] * D + i, vx[r][i]);
                        if (A.grad_f0) atomicAdd(A.grad_f0 + ix.v[r], m);
                        if (A.grad_f1) atomicAdd(A.grad_f1 + ix.v[r], q);
                    }
                }
            } else {
                unsigned long long k0[NF], k1[NF];
                double m[NF][1], q[NF][1];
#pragma unroll
                for (int r = 0; r < NF; ++r) {
                    k0[r] = (unsigned long long)(A.L.f0.map ? (int64_t)ix.f0[r] : cell * NF + r);
                    k1[r] = (unsigned long long)(A.L.f1.map ? (int64_t)ix.f1[r] : cell * NF + r);
                    m[r][0] = sd * ad * mub[r];
                    q[r][0] = sd * ad * lmb[r];
                }
                if (A.grad_coords) combine_add<D, TS>(ckx[wave], cvx[wave], kv, vx, A.grad_coords);
                if (A.grad_f0) combine_add<1, TS>(ckf[wave][0], cvf[wave][0], k0, m, A.grad_f0);
                if (A.grad_f1) combine_add<1, TS>(ckf[wave][1], cvf[wave][1], k1, q, A.grad_f1);
            }
        }
        load_raw<F_ELAST, D, FD>(A.L, cell_at(ahead), nx, raw);
#pragma unroll
        for (int v = 0; v <= D; ++v)
#pragma unroll
            for (int i = 0; i < D; ++i) asm volatile("" ::"v"(raw.x[v][i]));
#pragma unroll
        for (int r = 0; r < NF; ++r) asm volatile("" ::"v"(raw.f0[r]), "v"(raw.f1[r]));
        if (!det) {
            wave_sync();
            const unsigned long long* k0 = shared_keys ? ckx[wave] : ckf[wave][0];
            const unsigned long long* k1 = shared_keys ? ckx[wave] : ckf[wave][1];
            if (A.grad_coords) combine_flush<D, TS>(ckx[wave], cvx[wave], A.grad_coords, lane);
            if (A.grad_f0) combine_flush<1, TS>(k0, cvf[wave][0], A.grad_f0, lane);
            if (A.grad_f1) combine_flush<1, TS>(k1, cvf[wave][1], A.grad_f1, lane);
            wave_sync();
        }
    }
}

}  // namespace dev

typedef hipError_t (*AdjLaunch)(const dev::AdjArgs&, hipStream_t, int64_t blocks, int ncu);
struct AdjEntry {
    int form, dim, p, fd;
    AdjLaunch launch;
};

// Elasticity at the registered degrees (1 and 2, P1 coefficients) uses the
// node kernel, whose table AdjArgs::R is c_rkl (node_weights).
template <int FORM, int D, int P, int FD>
hipError_t launch_adjoint(const dev::AdjArgs& a, hipStream_t s, int64_t blocks, int ncu) {
    if constexpr (FORM == dev::F_ELAST) {
        const int grid = (int)std::min<int64_t>(blocks, (int64_t)ncu * (D == 3 && P == 2 ? 1 : 2));
        hipLaunchKernelGGL((dev::k_adjoint_elast<D, P, FD>), dim3(grid), dim3(256), 0, s, a);
    } else {
        const int grid = (int)std::min<int64_t>(blocks, (int64_t)ncu * 8);
        hipLaunchKernelGGL((dev::k_adjoint_linear<FORM, D, P, FD>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

static const std::vector<AdjEntry>& adj_registry() {
    using namespace dev;
    static const std::vector<AdjEntry> reg = {
        {F_MASS, 2, 1, 1, &launch_adjoint<F_MASS, 2, 1, 1>},
        {F_MASS, 3, 1, 1, &launch_adjoint<F_MASS, 3, 1, 1>},
        {F_MASS, 3, 2, 2, &launch_adjoint<F_MASS, 3, 2, 2>},
        {F_HELM, 2, 1, 1, &launch_adjoint<F_HELM, 2, 1, 1>},
        {F_HELM, 2, 2, 1, &launch_adjoint<F_HELM, 2, 2, 1>},
        {F_HELM, 3, 1, 1, &launch_adjoint<F_HELM, 3, 1, 1>},
        {F_HELM, 3, 2, 2, &launch_adjoint<F_HELM, 3, 2, 2>},
        {F_ELAST, 2, 1, 1, &launch_adjoint<F_ELAST, 2, 1, 1>},
        {F_ELAST, 2, 2, 1, &launch_adjoint<F_ELAST, 2, 2, 1>},
        {F_ELAST, 3, 1, 1, &launch_adjoint<F_ELAST, 3, 1, 1>},
        {F_ELAST, 3, 2, 1, &launch_adjoint<F_ELAST, 3, 2, 1>},
        {F_BURG, 2, 1, 1, &launch_adjoint<F_BURG, 2, 1, 1>},
        {F_BURG, 3, 1, 1, &launch_adjoint<F_BURG, 3, 1, 1>},
        {F_BURG, 3, 2, 2, &launch_adjoint<F_BURG, 3, 2, 2>},
        {F_DIFF, 2, 1, 0, &launch_adjoint<F_DIFF, 2, 1, 0>},
        {F_DIFF, 2, 2, 0, &launch_adjoint<F_DIFF, 2, 2, 0>},
        {F_DIFF, 3, 1, 0, &launch_adjoint<F_DIFF, 3, 1, 0>},
        {F_DIFF, 3, 2, 0, &launch_adjoint<F_DIFF, 3, 2, 0>},
    };
    return reg;
}

static std::mutex g_adj_mu;
static std::map<std::tuple<int, int, int, int, int, int>, void*> g_adj_tables;  // (dev, form, dim, p, q, fd)

// FP64 reference tensors [KR][NS * NS] (unpacked), host values.
bool r64_table(int form, int dim, int p, int q, int fd, std::vector<double>& h) {
    RefTensor R;
    if (!build_reference(form, dim, p, q, fd, R)) return false;
    h.resize(R.R.size());
    for (size_t i = 0; i < h.size(); ++i) h[i] = (double)R.R[i];
    return true;
}

// c_rkl = sum_q W_q psi_r N_k N_l [NF][NV][NV]: coefficient basis of degree
// fd, nodal basis of degree p - 1.
static bool node_weights(int dim, int p, int q, int fd, std::vector<double>& h) {
    Tables nd, fl;
    if (!nd.init(dim, p - 1, q) || !fl.init(dim, fd, q)) return false;
    h.assign((size_t)fl.n * nd.n * nd.n, 0.0);
    for (int r = 0; r < fl.n; ++r)
        for (int k = 0; k < nd.n; ++k)
            for (int l = 0; l < nd.n; ++l) {
                long double s = 0.0L;
                for (int t = 0; t < nd.nq; ++t)
                    s += nd.W[t] * fl.phi[(size_t)t * fl.n + r] * nd.phi[(size_t)t * nd.n + k] *
                         nd.phi[(size_t)t * nd.n + l];
                h[((size_t)r * nd.n + k) * nd.n + l] = (double)s;
            }
    return true;
}

constexpr int kNodeWeights = 0x100;  // added to the form in the table key

// A device table of g_adj_tables, built by `build` and uploaded on first use.
template <typename B>
static coffee_status device_table(const std::tuple<int, int, int, int, int, int>& key, B&& build, const double** out) {
    std::lock_guard<std::mutex> lk(g_adj_mu);
    auto it = g_adj_tables.find(key);
    if (it != g_adj_tables.end()) {
        *out = (const double*)it->second;
        return COFFEE_OK;
    }
    std::vector<double> h;
    if (!build(h)) return COFFEE_E_INVALID_ARG;
    void* d = nullptr;
    if (hipMalloc(&d, h.size() * sizeof(double)) != hipSuccess) return COFFEE_E_NOMEM;
    if (hipMemcpy(d, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(d);
        return COFFEE_E_HIP;
    }
    g_adj_tables[key] = d;
    *out = (const double*)d;
    return COFFEE_OK;
}

// FP64 reference tensors [KR][NS * NS] (unpacked), built and uploaded on first
// use; shared by the adjoint kernels and the degree-1 FMA kernels.
coffee_status reference_table_f64(int dev, int form, int dim, int p, int q, int fd, const double** out) {
    return device_table(std::make_tuple(dev, form, dim, p, q, fd),
                        [&](std::vector<double>& h) { return r64_table(form, dim, p, q, fd, h); }, out);
}

void free_adjoint_tables() {
    std::lock_guard<std::mutex> lk(g_adj_mu);
    for (auto& kv : g_adj_tables) {
        (void)hipSetDevice(std::get<0>(kv.first));
        (void)hipFree(kv.second);
    }
    g_adj_tables.clear();
}

coffee_status adjoint_linear(int form, int cell, int degree, int q, int fd, const double* coords, int64_t nvert,
                             const int32_t* c2v, int64_t ncells, const coffee_field* coeffs, int ncoeff,
                             const double* constants, int nconst, const double* lam, const double* u,
                             double seed, double* grad_coords, double* const* grad_coeff_values,
                             double* cell_value, const DetTarget* det, void* hip_stream) {
    const AdjEntry* e = nullptr;
    for (const AdjEntry& x : adj_registry())
        if (x.form == form && x.dim == cell && x.p == degree && x.fd == fd) e = &x;
    if (!e) return COFFEE_E_UNSUPPORTED;
    if (ncells > 0 && (!lam || !u)) return COFFEE_E_INVALID_ARG;
    if (ncells == 0) return COFFEE_OK;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return COFFEE_E_HIP;
    const double* R = nullptr;
    coffee_status st =
        form == COFFEE_ELASTICITY
            ? device_table(std::make_tuple(dev, form + kNodeWeights, cell, degree, q, fd),
                           [&](std::vector<double>& h) { return node_weights(cell, degree, q, fd, h); }, &R)
            : reference_table_f64(dev, form, cell, degree, q, fd, &R);
    if (st != COFFEE_OK) return st;
    dev::AdjArgs a;
    std::memset(&a, 0, sizeof a);
    a.L.coords = coords;
    a.L.c2v = c2v;
    a.L.ncells = ncells;
    if (ncoeff >= 1) a.L.f0 = dev::FieldArg{coeffs[0].values, coeffs[0].cell_to_dof};
    if (ncoeff >= 2) a.L.f1 = dev::FieldArg{coeffs[1].values, coeffs[1].cell_to_dof};
    if (form == COFFEE_BURGERS) {
        a.L.c0 = nconst > 0 ? constants[0] : 1.0;
        a.L.c1 = nconst > 1 ? constants[1] : 1.0;
    } else if (form == COFFEE_ELASTICITY && ncoeff == 0) {
        a.L.c0 = constants[0];
        a.L.c1 = constants[1];
    } else if (form == COFFEE_DIFFUSION) {
        a.L.c0 = (nconst > 0 ? constants[0] : 1.0) * (nconst > 1 ? constants[1] : 1.0);  // kappa dt
    }
    a.R = R;
    a.lam = lam;
    a.u = u;
    a.seed = seed;
    a.grad_coords = grad_coords;
    a.grad_f0 = (grad_coeff_values && ncoeff >= 1) ? grad_coeff_values[0] : nullptr;
    a.grad_f1 = (grad_coeff_values && ncoeff >= 2) ? grad_coeff_values[1] : nullptr;
    a.cell_value = cell_value;
    if (det) {
        a.det_x = det[0].local;
        a.det_f0 = ncoeff >= 1 ? det[1].local : nullptr;
        a.det_f1 = ncoeff >= 2 ? det[2].local : nullptr;
    }
    const int64_t blocks = (ncells + 255) / 256;
    if (e->launch(a, (hipStream_t)hip_stream, blocks, num_cu(dev)) != hipSuccess) return COFFEE_E_HIP;
    return COFFEE_OK;
}

}  // namespace coffee
