// Prism cells (triangle x interval): mass, Helmholtz and diffusion.
//
// The paper's benchmarks run on prisms as well as on simplices (section 5.2;
// at p = 1 a prism's j and k loops have 6 iterations). A prism is the image
// of the reference prism under the map spanned by its six degree-1 basis
// functions; that map is not affine, so J, det J and K = J^-1 change from
// quadrature point to point and the quadrature sum cannot be folded into
// point-free reference tensors as on simplices (the point loop carries the
// geometry). It stays the contraction of section 3.3's outer-product form,
// with the point index inside K:
//     A[e][a][b] = sum_{q, j} G[e][q, j] R[q, j][a][b]
//     G[e][q, j] = W_q |det J_q| (K_q K_q^T)_{al be}   (j over al <= be; kappa dt for diffusion)
//                  W_q |det J_q| f(X_q)                 (mass term; f = 1 without a field)
//     R[q, j][a][b] = d_al phi_a d_be phi_b (+ d_be phi_a d_al phi_b for al != be), phi_a phi_b at X_q
// so K = nq x (6 + 1) for Helmholtz, nq x 6 for diffusion, nq for mass. Over
// 16 cells this is a 16 x K by K x 16 product per 16 unique entries (a <= b;
// the matrices are symmetric), on the same MFMA instructions as the simplex
// engines (linear.hpp).
//
// Degree 1 (k_prism), per wave: one tile of 16 cells at a time. The 64
// lanes are 16 cells x 4 groups of quadrature points: each lane gathers its
// cell (all four lanes of a cell read the same lines), forms J, K and |det J|
// in FP64 at its points and writes those G entries to the tile's LDS rows.
// The MFMA loop then runs over all n-tiles at once, and the 16 element
// matrices leave through LDS as contiguous 16-byte stores (the staging area
// reuses the G rows). Degrees 2 and 3 (k_prism_fac): the contraction is
// factored over the triangle and the interval, the waves of a workgroup share
// 16 cells (degree 2) or 32 (degree 3), each taking pairs of interval dofs.
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

typedef unsigned int u32x4p __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

constexpr int prism_ns(int p) { return (p + 1) * (p + 2) / 2 * (p + 1); }
// G entries per point: the six pairs al <= be, then the mass term
constexpr int prism_jq(int form) { return form == F_MASS ? 1 : (form == F_HELM ? 7 : 6); }

template <int FORM, int P, int FD, int PREC, int NQ>
struct PrismCfg {
    using g_t = typename PrecT<PREC>::gtype;
    using frag_t = typename PrecT<PREC>::frag;
    using acc_t = typename PrecT<PREC>::acc;
    using out_t = typename PrecT<PREC>::otype;
    static constexpr int NS = prism_ns(P);
    static constexpr int NN = NS * NS;
    static constexpr int NU = NS * (NS + 1) / 2;
    static constexpr int NT = (NU + 15) / 16;
    static constexpr int JQ = prism_jq(FORM);
    static constexpr int KR = NQ * JQ;
    static constexpr int KE = PREC == PREC_BF16X3 ? 3 * KR : KR;
    static constexpr int KS = (KE + kstep(PREC) - 1) / kstep(PREC);
    // odd FP64/FP32 rows spread a fragment's 16 rows over the banks; BF16
    // rows stay 16-byte aligned
    static constexpr int ROW = PREC == PREC_BF16X3 ? KS * 32 + 8 : KS * 4 + 1;
    static constexpr int GT_BYTES = 16 * ROW * (int)sizeof(g_t);
    static constexpr int ST_BYTES = 8 * NN * (int)sizeof(out_t);
    static constexpr int WAVE_BYTES = ((GT_BYTES > ST_BYTES ? GT_BYTES : ST_BYTES) + 15) / 16 * 16;
    // two waves per workgroup when four would take more than half the LDS
    static constexpr int WAVES = 4 * WAVE_BYTES <= 80 * 1024 ? 4 : 2;
    static constexpr int LDS_BYTES = WAVES * WAVE_BYTES;
    // the reference fragments are held in registers
    static_assert(NT * KS * (PREC == PREC_F64 ? 2 : (PREC == PREC_F32 ? 1 : 4)) <= 64, "registers");
};

// Word 3 of a raw buffer resource on gfx9-family chips: 32-bit data format
// (a zero format would make untyped buffer accesses read zeros).
constexpr int kBufferWord3 = 0x00020000;

// One MFMA fragment (8, 4 or 16 bytes) from a raw buffer.
template <typename F>
__device__ inline F buffer_frag(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    if constexpr (sizeof(F) == 4) {
        return __builtin_bit_cast(F, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    } else if constexpr (sizeof(F) == 8) {
        return __builtin_bit_cast(F, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    } else {
        static_assert(sizeof(F) == 16, "fragment of 4, 8 or 16 bytes");
        return __builtin_bit_cast(F, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    }
}

struct PrismArgs {
    const double* coords;  // [nvert][3]
    const int32_t* c2v;    // [ncells][6]
    int64_t ncells;
    FieldArg f;            // degree-1 prism field (6 dofs per cell); values NULL: none
    double kdt;            // kappa dt (diffusion)
    const double* qtab;    // [NQ][4]: X, Y, Z, W; degrees 2, 3: then the interval weights
    const void* rfrag;     // packed reference fragments
    void* out;
    int64_t ntiles;        // ceil(ncells / 16)
};

// K = J^-1 (K[a][i] = d X_a / d x_i, J[i][a] = d x_i / d X_a) and |det J|.
__device__ inline void prism_inverse(const double (&J)[3][3], double (&K)[3][3], double& adet) {
    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    const double c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    const double c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    const double det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
    const double r = 1.0 / det;
    K[0][0] = c00 * r;
    K[1][0] = c01 * r;
    K[2][0] = c02 * r;
    K[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * r;
    K[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * r;
    K[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * r;
    K[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * r;
    K[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * r;
    K[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * r;
    adet = fabs(det);
}

// One G value into LDS column k (with the hi/lo split for BF16X3: columns k,
// KR + k hold the high part, 2 KR + k the low part, against R's (hi, lo, hi)).
template <int PREC, int KR>
__device__ inline void put_g(typename PrecT<PREC>::gtype* row, int k, double g) {
    if constexpr (PREC == PREC_F64) {
        row[k] = g;
    } else if constexpr (PREC == PREC_F32) {
        row[k] = (float)g;
    } else {
        const float x = (float)g;
        const u16 hi = bf16_bits_rne(x);
        row[k] = hi;
        row[KR + k] = hi;
        row[2 * KR + k] = bf16_bits_rne(x - bf16_to_float(hi));
    }
}

// The gathers of one cell in two dependent stages (indices, then values), so
// that the tile loop can issue them ahead of use.
struct PrismIdx {
    int v[6];
    int fm[6];
};
template <int FD>
struct PrismRaw {
    double x[6][3];
    double f[FD > 0 ? 6 : 1];
};

template <int FD>
__device__ inline void prism_idx(const PrismArgs& A, int64_t cell, PrismIdx& ix) {
#pragma unroll
    for (int v = 0; v < 6; ++v) ix.v[v] = gload_nt(A.c2v + cell * 6 + v);
    if constexpr (FD > 0) {
        if (A.f.map) {
#pragma unroll
            for (int v = 0; v < 6; ++v) ix.fm[v] = gload_nt(A.f.map + cell * 6 + v);
        }
    }
}

template <int FD>
__device__ inline void prism_raw(const PrismArgs& A, int64_t cell, const PrismIdx& ix, PrismRaw<FD>& r) {
#pragma unroll
    for (int v = 0; v < 6; ++v)
#pragma unroll
        for (int i = 0; i < 3; ++i) r.x[v][i] = gload(A.coords + (int64_t)ix.v[v] * 3 + i);
    if constexpr (FD > 0) {
#pragma unroll
        for (int v = 0; v < 6; ++v) r.f[v] = gload(A.f.values + (A.f.map ? (int64_t)ix.fm[v] : cell * 6 + v));
    }
}

template <int FORM, int P, int FD, int PREC, int NQ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_prism(PrismArgs A) {
    using C = PrismCfg<FORM, P, FD, PREC, NQ>;
    using g_t = typename C::g_t;
    using frag_t = typename C::frag_t;
    using acc_t = typename C::acc_t;
    using out_t = typename C::out_t;
    constexpr int NS = C::NS, NN = C::NN, NU = C::NU, NT = C::NT, KS = C::KS, ROW = C::ROW, JQ = C::JQ,
                  KR = C::KR;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int col = lane & 15, grp = lane >> 4;
    g_t* gt = reinterpret_cast<g_t*>(lds + wave * C::WAVE_BYTES);
    out_t* st = reinterpret_cast<out_t*>(lds + wave * C::WAVE_BYTES);
    const frag_t* rf = reinterpret_cast<const frag_t*>(A.rfrag);
    out_t* out = reinterpret_cast<out_t*>(A.out);

    // (a, b) of the unique entry u = 16 t + col, a <= b, row-major over the upper triangle
    int ua[NT], ub[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int u = t * 16 + col, a = 0;
        while (a < NS - 1 && u >= NS - a) { u -= NS - a; ++a; }
        ua[t] = a;
        ub[t] = a + u;
    }
    frag_t rreg[NT][KS];  // the reference fragments
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) rreg[t][s] = gload(rf + (t * KS + s) * 64 + lane);

    // the rule's points and weights, once per workgroup
    __shared__ double sq[NQ * 4];
    for (int i = threadIdx.x; i < NQ * 4; i += blockDim.x) sq[i] = gload(A.qtab + i);
    __syncthreads();

    // Persistent loop over 16-cell tiles, software-pipelined:
    // while tile i is contracted and stored, the vertices and field values of
    // tile i + 1 and the indices of tile i + 2 are in flight (issued before
    // this tile's stores, which share the in-order memory counter with them).
    const int64_t stride = (int64_t)gridDim.x * C::WAVES;
    int64_t tile = (int64_t)blockIdx.x * C::WAVES + wave;
    if (tile >= A.ntiles) return;  // wave-uniform; no workgroup barrier follows
    auto clamp = [&](int64_t t) -> int64_t {
        const int64_t c = (t < A.ntiles ? t : tile) * 16 + col;
        return c < A.ncells ? c : A.ncells - 1;
    };
    PrismIdx ix;
    PrismRaw<FD> raw;
    {
        prism_idx<FD>(A, clamp(tile), ix);
        prism_raw<FD>(A, clamp(tile), ix, raw);
        prism_idx<FD>(A, clamp(tile + stride), ix);
        // Complete the prologue's loads here (no store is outstanding yet):
        // the loop's first wait then merges with an empty queue, and the
        // waits inside the loop can leave this tile's stores in flight.
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            asm volatile("" ::"v"(ix.v[v]));
            if constexpr (FD > 0) asm volatile("" ::"v"(ix.fm[v]), "v"(raw.f[v]));
#pragma unroll
            for (int i = 0; i < 3; ++i) asm volatile("" ::"v"(raw.x[v][i]));
        }
    }
    // One tile. FULL: all 16 cells exist, so the stores have compile-time counts
    // and the next tile's waits need not drain them.
    auto tile_body = [&](auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t base = tile * 16;
        const bool valid = FULL || base + col < A.ncells;

        // per-cell edge vectors of the map (bottom and top triangle edges from
        // vertex t0, vertical edges)
        double e[7][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            e[0][i] = raw.x[2][i] - raw.x[0][i];
            e[1][i] = raw.x[3][i] - raw.x[1][i];
            e[2][i] = raw.x[4][i] - raw.x[0][i];
            e[3][i] = raw.x[5][i] - raw.x[1][i];
            e[4][i] = raw.x[1][i] - raw.x[0][i];
            e[5][i] = raw.x[3][i] - raw.x[2][i];
            e[6][i] = raw.x[5][i] - raw.x[4][i];
        }
        double f[6];
#pragma unroll
        for (int v = 0; v < 6; ++v) f[v] = FD > 0 ? raw.f[v] : 0.0;
        // next tile's values (indices loaded one tile ago), then the indices two ahead
        prism_raw<FD>(A, clamp(tile + stride), ix, raw);
        prism_idx<FD>(A, clamp(tile + 2 * stride), ix);

        // G entries of this lane's points q = grp, grp + 4, ...
        g_t* row = gt + col * ROW;
#pragma unroll
        for (int it = 0; it < (NQ + 3) / 4; ++it) {
            const int q = grp + 4 * it;
            if (q >= NQ) break;
            const double X = sq[4 * q], Y = sq[4 * q + 1], Z = sq[4 * q + 2], W = sq[4 * q + 3];
            const double zb = 1.0 - Z, l0 = 1.0 - X - Y;
            double J[3][3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                J[i][0] = zb * e[0][i] + Z * e[1][i];
                J[i][1] = zb * e[2][i] + Z * e[3][i];
                J[i][2] = l0 * e[4][i] + X * e[5][i] + Y * e[6][i];
            }
            double K[3][3], adet;
            prism_inverse(J, K, adet);
            const double w = valid ? W * adet : 0.0;
            int j = q * JQ;
            if constexpr (FORM != F_MASS) {
                const double sc = FORM == F_DIFF ? w * A.kdt : w;
#pragma unroll
                for (int al = 0; al < 3; ++al)
#pragma unroll
                    for (int be = al; be < 3; ++be) {
                        const double s = K[al][0] * K[be][0] + K[al][1] * K[be][1] + K[al][2] * K[be][2];
                        put_g<PREC, KR>(row, j++, sc * s);
                    }
            }
            if constexpr (FORM != F_DIFF) {
                double fq = 1.0;
                if constexpr (FD > 0) {
                    // degree-1 prism basis lambda_t(X, Y) l_s(Z) at the point
                    fq = (l0 * f[0] + X * f[2] + Y * f[4]) * zb + (l0 * f[1] + X * f[3] + Y * f[5]) * Z;
                }
                put_g<PREC, KR>(row, j, w * fq);
            }
        }
        // zero K padding up to a whole number of k-steps
        constexpr int KFILL = PREC == PREC_BF16X3 ? 3 * KR : KR;
#pragma unroll 1
        for (int k = KFILL + grp; k < KS * kstep(PREC); k += 4) row[k] = g_t(0);
        wave_sync();

        acc_t acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = acc_t{0, 0, 0, 0};
        // straight-line code; every G fragment is read from LDS before the
        // first product, so the reads overlap one another instead of each MFMA
        // pair waiting for its own read
        frag_t afr[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) afr[s] = load_afrag<PREC>(gt, ROW, lane, s);
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(afr[s]));  // one wait for all reads
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = mfma<PREC>(afr[s], rreg[t][s], acc[t]);
        wave_sync();  // every G read is done: the staging area reuses the rows

        // two halves of 8 cells, each written to LDS in full (both triangles)
        // and copied out as contiguous 16-byte stores
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t c0 = base + 8 * h;
            if (!FULL && c0 >= A.ncells) break;  // wave-uniform
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (t * 16 + col >= NU) continue;
                const int oab = ua[t] * NS + ub[t], oba = ub[t] * NS + ua[t];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = acc_row<PREC>(lane, v);
                    if ((r >> 3) != h) continue;
                    const out_t xv = (out_t)acc[t][v];
                    st[(r & 7) * NN + oab] = xv;
                    st[(r & 7) * NN + oba] = xv;
                }
            }
            wave_sync();
            constexpr int PER16 = 16 / (int)sizeof(out_t);
            const u32x4p* s4 = reinterpret_cast<const u32x4p*>(st);
            out_t* dst = out + c0 * NN;
            u32x4p* d4 = reinterpret_cast<u32x4p*>(dst);
            if constexpr (FULL) {
                // 8 NN is a multiple of PER16; groups of four LDS reads, then
                // their four nontemporal stores. Every lane stores (lanes past
                // the end repeat the last vector, same address and value), so
                // no branch hides the store count from the wait counters.
                constexpr int NV = 8 * NN / PER16;
                constexpr int PL = (NV + 63) / 64;
#pragma unroll
                for (int i0 = 0; i0 < PL; i0 += 4) {
                    u32x4p tmp[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int k = (i0 + i) * 64 + lane < NV ? (i0 + i) * 64 + lane : NV - 1;
                        if (i0 + i < PL) tmp[i] = s4[k];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int k = (i0 + i) * 64 + lane < NV ? (i0 + i) * 64 + lane : NV - 1;
                        if (i0 + i < PL) gstore_nt(&d4[k], tmp[i]);
                    }
                }
            } else {
                const int nc = A.ncells - c0 < 8 ? (int)(A.ncells - c0) : 8;
                const int nelem = nc * NN;
                const int nvec = nelem / PER16;
                for (int i = lane; i < nvec; i += 64) gstore_nt(&d4[i], s4[i]);
                for (int i = nvec * PER16 + lane; i < nelem; i += 64) gstore(&dst[i], st[i]);
            }
            wave_sync();
        }
    };
    const int64_t nfull = A.ncells / 16;  // tiles whose 16 cells all exist
    for (; tile < nfull; tile += stride) tile_body(std::integral_constant<bool, true>());
    if (tile < A.ntiles) tile_body(std::integral_constant<bool, false>());
}

// ---------------------------------------------------------------- degrees 2, 3
// The basis, the rule and so the point products are tensor products of a
// triangle and an interval factor. For interval dofs b, b' the block of the
// element matrix over the triangle dofs is
//     A[(a,b)][(a',b')] = sum_i sum_types (sum_j G_type(i, j) w_type,bb'(j)) R_type(i)[a][a'],
// i the triangle points, j the interval points: the interval sum is taken
// first (p + 1 multiply-adds per coefficient), and what is left is a
// contraction over (i, type) with products of triangle functions alone. Types,
// with the interval weight w: the pairs (0,0), (0,1), (1,1) of the triangle
// directions (l_b l_b'), d_al phi_a phi_a' (l_b l'_b') and phi_a d_al phi_a'
// (l'_b l_b') for al = 0, 1 (one type where b = b'), phi_a phi_a' (l'_b l'_b',
// and l_b l_b' for the mass term). Only b <= b' is formed (the matrix is
// symmetric) and, for b = b', a <= a'. Degree 2: 246 matrix products of 4 k's
// per 16 cells, against 451 for the products over (point, term) with all
// dof pairs; degree 3: 1,728 against 4,992.
//
// A workgroup takes one 16-cell tile at degree 2, two at degree 3. Its threads,
// one per cell and triangle point, form G at the points in LDS (FP64). Each
// wave then owns pairs (b, b'): three waves with one pair b < b' and one pair
// b = b' each at degree 2, eight at degree 3 (six with a pair b < b', two with
// two pairs b = b'), which balances their products. Lane (cell, g) of a wave
// forms the coefficients of its cell at the triangle points i = 4 ib + g, which
// are its k's of the steps (ib, type): the G operand of a product never passes
// through LDS. A ninth point (degree 2) is spread over the four lane groups
// type by type. The R fragments, shared by every pair of a kind, are raw
// buffer loads, one step ahead (BF16X3: a block's at its start). Then, in passes of as many cells as the LDS
// holds, the waves write their accumulators (both mirrored entries) into a
// staging area over the G values, and the workgroup copies whole cells out as
// 16-byte stores (a matrix written a few entries at a time leaves partial
// lines that the L2 evicts).
//
// Degree 2 is bound by its instructions and the phases of a workgroup, so the
// small tile (25 KB of LDS, many workgroups per CU) matters: two tiles per
// workgroup ran 613 us in FP64 with three waves, 640 to 780 with six. Its
// gathers go through LDS, each value read by one thread: read by all threads
// of a cell they took 25 to 60 us of the mass form's time (below, "all
// gather"). 524,288 P2 prisms, us:
//                          points and terms   all gather   as it is
//   mass            FP64         290              313          262
//   mass, field     FP64         315              346          289
//   mass            BF16X3       189              250          189
//   mass, field     BF16X3       194              261          195
//   diffusion       FP64         667              497          490
//   diffusion       FP32         376              301          299
//   diffusion       BF16X3       258              269          254
// (the BF16X3 mass form also packs its products: kMassParts). 65,536 P3
// prisms: diffusion FP64 765 -> 367, FP32 415 -> 217, BF16X3 222 -> 157; mass
// BF16X3 109 -> 128 with one product per slot, 101 packed.

// Workgroup barrier that orders LDS accesses only. Nothing passes between the
// threads through global memory, and __syncthreads would also wait until
// every outstanding store has reached memory and every prefetch has arrived
// (two microseconds or more per staging pass).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Mass form in BF16X3: coefficient and table value are split in three bf16
// parts (0 hi, 1 lo, 2 third), and the six products that matter fill six of
// the 8 KS slots of a lane for each of its points: {part of the coefficient,
// part of the table}. The leftover point's are spread over three lane groups,
// two slots each: kMassRest[lane group][slot].
constexpr int kMassParts[6][2] = {{0, 0}, {1, 0}, {0, 1}, {2, 0}, {0, 2}, {1, 1}};
constexpr int kMassRest[3][2] = {{0, 1}, {2, 3}, {4, 5}};  // indices into kMassParts

template <int FORM, int P, int FD, int PREC>
struct PrismFacCfg {
    using frag_t = typename PrecT<PREC>::frag;
    using acc_t = typename PrecT<PREC>::acc;
    using out_t = typename PrecT<PREC>::otype;
    static constexpr bool BF = PREC == PREC_BF16X3;
    static constexpr int M1 = P + 1;               // interval points, and dofs
    static constexpr int NI = M1 * M1;             // triangle points
    static constexpr int NQ = NI * M1;
    static constexpr int NTRI = (P + 1) * (P + 2) / 2;
    static constexpr int NS = NTRI * M1, NN = NS * NS;
    static constexpr int JQ = prism_jq(FORM);      // G values per point
    static constexpr int CELLG = (NQ * JQ) | 1;    // doubles of one cell
    static constexpr int CT = P == 2 ? 1 : 2, CELLS = 16 * CT;  // tiles and cells of a workgroup
    static constexpr int NOFF = M1 * (M1 - 1) / 2;
    // kind 0: b < b', kind 1: b = b'
    static constexpr int types(int kind) { return FORM == F_MASS ? 1 : (kind == 0 ? 8 : 6); }
    static constexpr int entries(int kind) { return kind == 0 ? NTRI * NTRI : NTRI * (NTRI + 1) / 2; }
    static constexpr int tiles(int kind) { return (entries(kind) + 15) / 16; }
    static constexpr int FULLB = NI / 4, REM = NI % 4;
    static_assert(REM <= 1, "one leftover point");
    // k-steps (BF16X3: blocks of four points, eight type slots each, with a hi
    // and a lo fragment; the mass form, with one type, packs the products of
    // its splits over the slots instead: kMassParts)
    static constexpr int steps(int kind) {
        if (BF && types(kind) == 1) return (6 * FULLB + 2 * REM + 7) / 8;
        return BF ? 2 * ((NI + 3) / 4) : FULLB * types(kind) + (REM ? (types(kind) + 3) / 4 : 0);
    }
    static constexpr int frags(int kind) { return steps(kind) * tiles(kind) * 64; }
    static constexpr int WAVES = P == 2 ? 3 : 8;
    // degree 2: the workgroups of a CU hide each other's gathers; degree 3 has
    // one per CU and prefetches
    static constexpr bool PIPE = P == 3;
    // (BF16X3 mass with three: 190.8 us against 189.3, FP32 mass with four 195
    // against 189.5; diffusion takes what it needs)
    static constexpr int WPE = P == 2 ? (FORM == F_MASS && BF ? 4 : 3) : 2;
    // accumulator slots of a wave: degree 2 the tiles of its two pairs, degree
    // 3 those of one pair b < b' or of two pairs b = b'
    static constexpr int TW = P == 2 ? tiles(0) + tiles(1) : 2 * tiles(1);
    static_assert(P == 2 || tiles(0) <= TW, "slots");
    static constexpr int G_BYTES = CELLS * CELLG * 8;
    static constexpr int CB = NN * (int)sizeof(out_t);
    // accumulator elements (rows of a tile) and cells per staging pass
    static constexpr int VP = (P == 2 ? 2 : 1) * (PREC == PREC_F64 ? 1 : 2), PC = 4 * CT * VP;
    // staging rows and cells: degree 3 rows of 40 values would put the 16
    // lanes of a mirrored column on two banks and the four cells of a lane
    // group on the same ones (17 conflicting accesses per write on average;
    // with 16 bytes more per row and per cell 3 to 5)
    static constexpr int PADV = P == 3 ? 16 / (int)sizeof(out_t) : 0;
    static constexpr int RS = NS + PADV, CS = NS * RS + PADV;
    static constexpr int ST_BYTES = PC * CS * (int)sizeof(out_t);
    // degree 2: vertices and field values of a cell, in LDS (doubles; odd)
    static constexpr int XS = 25;
    static constexpr int LDS_BYTES = ((G_BYTES > ST_BYTES ? G_BYTES : ST_BYTES) + 15) / 16 * 16;
    static_assert(LDS_BYTES + NQ * 32 <= 160 * 1024 && CB % 16 == 0, "LDS");
};

// Coefficients c[type] of a pair at triangle point i from the cell's G values.
// w: the pair's interval weights [4][M1]: l l, l l', l' l, l' l'.
template <int FORM, int P, int KIND>
__device__ __forceinline__ void prism_coefs(const double* g, const double (&w)[4][P + 1], double* c) {
    constexpr int M1 = P + 1, JQ = prism_jq(FORM), T = FORM == F_MASS ? 1 : (KIND == 0 ? 8 : 6);
#pragma unroll
    for (int t = 0; t < T; ++t) c[t] = 0.0;
#pragma unroll
    for (int j = 0; j < M1; ++j) {
        const double* gj = g + j * JQ;
        if constexpr (FORM == F_MASS) {
            c[0] += w[0][j] * gj[0];
        } else {
            const double g02 = gj[2], g12 = gj[4];
            c[0] += w[0][j] * gj[0];
            c[1] += w[0][j] * gj[1];
            c[2] += w[0][j] * gj[3];
            c[3] += w[1][j] * g02;
            c[4] += w[1][j] * g12;
            if constexpr (KIND == 0) {
                c[5] += w[2][j] * g02;
                c[6] += w[2][j] * g12;
            }
            c[T - 1] += w[3][j] * gj[5];
            if constexpr (FORM == F_HELM) c[T - 1] += w[0][j] * gj[6];
        }
    }
}

// Contraction of one pair (weights wt) of the given kind for the wave's tiles
// (gt: their G values) into acc[c][S0 ...]. rf0: first fragment of the kind.
template <int FORM, int P, int FD, int PREC, int KIND, int S0>
__device__ __forceinline__ void prism_contract(const double* gt, const double* wt, __amdgpu_buffer_rsrc_t rsrc,
                                               unsigned rf0, int lane,
                                               typename PrecT<PREC>::acc (&acc)[PrismFacCfg<FORM, P, FD, PREC>::CT]
                                                                              [PrismFacCfg<FORM, P, FD, PREC>::TW]) {
    using C = PrismFacCfg<FORM, P, FD, PREC>;
    using frag_t = typename C::frag_t;
    constexpr int T = C::types(KIND), NT = C::tiles(KIND), M1 = C::M1, JQ = C::JQ, NC = C::CT;
    constexpr unsigned FB = sizeof(frag_t);
    const int g = lane >> 4;
    const double* row[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) row[c] = gt + (16 * c + (lane & 15)) * C::CELLG;
    double w[4][M1];  // wave-uniform
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int j = 0; j < M1; ++j) w[k][j] = cload(wt + k * M1 + j);
    auto load_b = [&](frag_t* b, int s) {
        const unsigned vo = (rf0 + (unsigned)(s * NT * 64) + lane) * FB;
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = buffer_frag<frag_t>(rsrc, vo, (unsigned)(t * 64) * FB);
    };
    if constexpr (C::BF && T == 1) {
        constexpr int KS = C::steps(KIND), NP = C::FULLB + C::REM;
        frag_t b[2][NT], a[NC][KS];
        load_b(b[0], 0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            __bf16 x[NP][3];  // the parts of the coefficients at the points 4 m + g, then the leftover one
#pragma unroll
            for (int m = 0; m < NP; ++m) {
                double cf[1];
                prism_coefs<FORM, P, KIND>(row[c] + (m < C::FULLB ? 4 * m + g : C::NI - 1) * (M1 * JQ), w, cf);
                const float v = (float)cf[0];
                x[m][0] = (__bf16)v;
                x[m][1] = (__bf16)(v - (float)x[m][0]);
                x[m][2] = (__bf16)(v - (float)x[m][0] - (float)x[m][1]);
            }
#pragma unroll
            for (int f = 0; f < 8 * KS; ++f) {
                __bf16 v = (__bf16)0.0f;
                if (f < 6 * C::FULLB) {
                    v = x[f / 6][kMassParts[f % 6][0]];
                } else if (f < 6 * C::FULLB + 2 * C::REM) {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        v = g == k ? x[NP - 1][kMassParts[kMassRest[k][f - 6 * C::FULLB]][0]] : v;
                }
                a[c][f / 8][f % 8] = v;
            }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s + 1 < KS) load_b(b[(s + 1) & 1], s + 1);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c][S0 + t] = mfma<PREC>(a[c][s], b[s & 1][t], acc[c][S0 + t]);
        }
    } else if constexpr (C::BF) {
        frag_t bh[NT], bl[NT];
#pragma unroll 1
        for (int ib = 0; ib < (C::NI + 3) / 4; ++ib) {
            frag_t ah[NC], al[NC];
            // in flight while the coefficients are formed (a block ahead, held
            // over the products: diffusion P2 268 us against 264)
            load_b(bh, 2 * ib);
            load_b(bl, 2 * ib + 1);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                // points that do not exist take another's coefficients, against zeros in the table
                const int i = 4 * ib + g;
                double cf[T];
                prism_coefs<FORM, P, KIND>(row[c] + (i < C::NI ? i : 0) * (M1 * JQ), w, cf);
#pragma unroll
                for (int t = 0; t < 8; t += 2) {
                    // two at a time: one conversion instruction
                    const f2v x = {t < T ? (float)cf[t < T ? t : 0] : 0.0f, t + 1 < T ? (float)cf[t + 1 < T ? t + 1 : 0] : 0.0f};
                    const bf2v hi = __builtin_convertvector(x, bf2v);
                    const bf2v lo = __builtin_convertvector(x - __builtin_convertvector(hi, f2v), bf2v);
                    ah[c][t] = hi[0];
                    ah[c][t + 1] = hi[1];
                    al[c][t] = lo[0];
                    al[c][t + 1] = lo[1];
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    acc[c][S0 + t] = mfma<PREC>(ah[c], bh[t], acc[c][S0 + t]);
                    acc[c][S0 + t] = mfma<PREC>(al[c], bh[t], acc[c][S0 + t]);
                    acc[c][S0 + t] = mfma<PREC>(ah[c], bl[t], acc[c][S0 + t]);
                    // the fourth product of the splits too: without it the
                    // error against FP64 was 3.0e-6 (diffusion P3, norm), with
                    // it 2.3e-6; over points and terms, without it, 2.6e-6
                    acc[c][S0 + t] = mfma<PREC>(al[c], bl[t], acc[c][S0 + t]);
                }
        }
    } else {
        constexpr int KS = C::steps(KIND);
        frag_t b[2][NT];
        load_b(b[0], 0);
#pragma unroll 1
        for (int ib = 0; ib < C::FULLB; ++ib) {
            double cf[NC][T];
#pragma unroll
            for (int c = 0; c < NC; ++c) prism_coefs<FORM, P, KIND>(row[c] + (4 * ib + g) * (M1 * JQ), w, cf[c]);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int s = ib * T + t;
                load_b(b[(t + 1) & 1], s + 1 < KS ? s + 1 : s);
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        acc[c][S0 + n] = mfma<PREC>((frag_t)cf[c][t], b[t & 1][n], acc[c][S0 + n]);
            }
            if constexpr (T % 2 == 1) {
#pragma unroll
                for (int n = 0; n < NT; ++n) b[0][n] = b[1][n];
            }
        }
        if constexpr (C::REM > 0) {
            // the leftover point: lane group g takes the types 4 t + g
            double cf[NC][T];
#pragma unroll
            for (int c = 0; c < NC; ++c) prism_coefs<FORM, P, KIND>(row[c] + (C::NI - 1) * (M1 * JQ), w, cf[c]);
#pragma unroll
            for (int t = 0; t < (T + 3) / 4; ++t) {
                const int s = C::FULLB * T + t;
                load_b(b[(t + 1) & 1], s + 1 < KS ? s + 1 : s);
                frag_t x[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    double v = cf[c][4 * t];
#pragma unroll
                    for (int k = 1; k < 4; ++k) {
                        const double y = 4 * t + k < T ? cf[c][4 * t + k < T ? 4 * t + k : 0] : 0.0;
                        v = g == k ? y : v;
                    }
                    x[c] = (frag_t)v;
                }
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc[c][S0 + n] = mfma<PREC>(x[c], b[t & 1][n], acc[c][S0 + n]);
            }
        }
    }
}

template <int FORM, int P, int FD, int PREC>
__global__ __launch_bounds__((PrismFacCfg<FORM, P, FD, PREC>::WAVES * 64))
__attribute__((amdgpu_waves_per_eu(PrismFacCfg<FORM, P, FD, PREC>::WPE))) void k_prism_fac(PrismArgs A) {
    using C = PrismFacCfg<FORM, P, FD, PREC>;
    using frag_t = typename C::frag_t;
    using acc_t = typename C::acc_t;
    using out_t = typename C::out_t;
    constexpr int M1 = C::M1, NN = C::NN, NS = C::NS, NTRI = C::NTRI, NQ = C::NQ, JQ = C::JQ, TW = C::TW,
                  CELLS = C::CELLS, NOFF = C::NOFF;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ double sq[NQ * 4];
    __shared__ double sx[C::PIPE ? 1 : CELLS * C::XS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double* gt = reinterpret_cast<double*>(lds);
    out_t* st = reinterpret_cast<out_t*>(lds);
    out_t* out = reinterpret_cast<out_t*>(A.out);

    // staging offsets of this lane's entry in each accumulator slot: (row, col)
    // in the low half, its mirror in the high half; all ones: no entry
    static_assert(C::CS < 65535, "offsets in 16 bits");
    unsigned off[TW];
#pragma unroll
    for (int s = 0; s < TW; ++s) {
        // slot -> pair (b, b2) and n-tile
        int kind, pair, t;
        if (P == 2) {
            kind = s < C::tiles(0) ? 0 : 1;
            pair = wave;
            t = kind == 0 ? s : s - C::tiles(0);
        } else {
            kind = wave < NOFF ? 0 : 1;
            pair = kind == 0 ? wave : 2 * (wave - NOFF) + s / C::tiles(1);
            t = kind == 0 ? s : s % C::tiles(1);
        }
        int b = pair, b2 = pair, a, a2, u = 16 * t + (lane & 15);
        const bool ok = u < C::entries(kind);
        if (kind == 0) {
            b = 0;
            int r = pair;
            while (r >= M1 - 1 - b) {
                r -= M1 - 1 - b;
                ++b;
            }
            b2 = b + 1 + r;
            a = u / NTRI;
            a2 = u - a * NTRI;
        } else {
            a = 0;
            while (a < NTRI - 1 && u >= NTRI - a) {
                u -= NTRI - a;
                ++a;
            }
            a2 = a + u;
        }
        const int rr = a * M1 + b, cc = a2 * M1 + b2;
        off[s] = ok ? (unsigned)(rr * C::RS + cc) | (unsigned)(cc * C::RS + rr) << 16 : ~0u;
    }
    for (int i = tid; i < NQ * 4; i += blockDim.x) sq[i] = gload(A.qtab + i);
    // the interval weights follow the rule: [pairs b < b', then b = b'][4][M1]
    const double* wtab = A.qtab + NQ * 4;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<frag_t*>(reinterpret_cast<const frag_t*>(A.rfrag)), (short)0,
        (C::frags(0) + C::frags(1)) * (int)sizeof(frag_t), kBufferWord3);

    const int64_t ngroups = (A.ncells + CELLS - 1) / CELLS;
    const int r = tid % CELLS, pg = tid / CELLS;
    static_assert(64 * C::WAVES / CELLS >= C::NI, "a thread per cell and triangle point");
    auto cell_of = [&](int64_t grp) -> int64_t {
        const int64_t c = grp * CELLS + r;
        return c < A.ncells ? c : A.ncells - 1;
    };
    int64_t grp = blockIdx.x;
    if (grp >= ngroups) return;  // the whole workgroup
    // the next group's vertices and field values are in flight during the
    // contraction, the indices of the one after it too
    const int64_t GS = gridDim.x;
    PrismIdx ix;
    PrismRaw<FD> raw;
    if constexpr (C::PIPE) {
        prism_idx<FD>(A, cell_of(grp), ix);
        prism_raw<FD>(A, cell_of(grp), ix, raw);
        prism_idx<FD>(A, cell_of(grp + GS < ngroups ? grp + GS : grp), ix);
    }
    for (; grp < ngroups; grp += GS) {
        const int64_t base = grp * CELLS;
        if constexpr (!C::PIPE) {
            // each vertex and each field value is read by one thread
            static_assert(64 * C::WAVES / CELLS >= 12, "a thread per cell and value");
            const int64_t cell = cell_of(grp);
            double* x = sx + r * C::XS;
            if (pg < (FD > 0 ? 12 : 6)) {
                // vertex pg, or field value pg - 6: one code path, so that a
                // wave with both does not wait for two chains of loads
                const bool vert = FD == 0 || pg < 6;
                int64_t at = cell * 6 + (vert ? pg : pg - 6);
                const int32_t* map = vert ? A.c2v : A.f.map;
                if (map) at = gload_nt(map + at);
                const double* src = vert ? A.coords + at * 3 : A.f.values + at;
                double v[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) v[i] = gload(src + (vert ? i : 0));
                if (vert) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) x[pg * 3 + i] = v[i];
                } else {
                    x[12 + pg] = v[0];
                }
            }
        }
        // the previous group's staging reads are done, sx (and sq) is written
        lds_barrier();
        if constexpr (!C::PIPE) {
            const double* x = sx + r * C::XS;
#pragma unroll
            for (int v = 0; v < 6; ++v) {
#pragma unroll
                for (int i = 0; i < 3; ++i) raw.x[v][i] = x[v * 3 + i];
                if constexpr (FD > 0) raw.f[v] = x[18 + v];
            }
        }
        // G: thread (cell r, triangle point pg) forms the points of that vertical line
        {
            const bool valid = base + r < A.ncells;
            double e[7][3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                e[0][i] = raw.x[2][i] - raw.x[0][i];
                e[1][i] = raw.x[3][i] - raw.x[1][i];
                e[2][i] = raw.x[4][i] - raw.x[0][i];
                e[3][i] = raw.x[5][i] - raw.x[1][i];
                e[4][i] = raw.x[1][i] - raw.x[0][i];
                e[5][i] = raw.x[3][i] - raw.x[2][i];
                e[6][i] = raw.x[5][i] - raw.x[4][i];
            }
            if (pg < C::NI) {
                double* row = gt + r * C::CELLG + pg * (M1 * JQ);
                const double X = sq[4 * pg * M1], Y = sq[4 * pg * M1 + 1], l0 = 1.0 - X - Y;
                double J2[3];  // the vertical column does not depend on Z
#pragma unroll
                for (int i = 0; i < 3; ++i) J2[i] = l0 * e[4][i] + X * e[5][i] + Y * e[6][i];
#pragma unroll
                for (int jz = 0; jz < M1; ++jz) {
                    const double Z = sq[4 * (pg * M1 + jz) + 2], W = sq[4 * (pg * M1 + jz) + 3], zb = 1.0 - Z;
                    double J[3][2];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        J[i][0] = zb * e[0][i] + Z * e[1][i];
                        J[i][1] = zb * e[2][i] + Z * e[3][i];
                    }
                    // rows of det J K (cofactors)
                    const double c[3][3] = {{J[1][1] * J2[2] - J2[1] * J[2][1], J2[0] * J[2][1] - J[0][1] * J2[2],
                                             J[0][1] * J2[1] - J2[0] * J[1][1]},
                                            {J2[1] * J[2][0] - J[1][0] * J2[2], J[0][0] * J2[2] - J2[0] * J[2][0],
                                             J2[0] * J[1][0] - J[0][0] * J2[1]},
                                            {J[1][0] * J[2][1] - J[1][1] * J[2][0], J[0][1] * J[2][0] - J[0][0] * J[2][1],
                                             J[0][0] * J[1][1] - J[0][1] * J[1][0]}};
                    const double det = J[0][0] * c[0][0] + J[1][0] * c[0][1] + J[2][0] * c[0][2], adet = fabs(det);
                    double* pq = row + jz * JQ;
                    int t = 0;
                    if constexpr (FORM != F_MASS) {
                        // W |det J| K K^T = (W / |det J|) c c^T
                        const double w = valid ? (FORM == F_DIFF ? W * A.kdt : W) / adet : 0.0;
#pragma unroll
                        for (int al = 0; al < 3; ++al)
#pragma unroll
                            for (int be = al; be < 3; ++be)
                                pq[t++] = w * (c[al][0] * c[be][0] + c[al][1] * c[be][1] + c[al][2] * c[be][2]);
                    }
                    if constexpr (FORM != F_DIFF) {
                        double fq = valid ? W * adet : 0.0;
                        if constexpr (FD > 0)
                            fq *= (l0 * raw.f[0] + X * raw.f[2] + Y * raw.f[4]) * zb +
                                  (l0 * raw.f[1] + X * raw.f[3] + Y * raw.f[5]) * Z;
                        pq[t] = fq;
                    }
                }
            }
        }
        if constexpr (C::PIPE) {
            const int64_t n1 = grp + GS < ngroups ? grp + GS : grp;
            prism_raw<FD>(A, cell_of(n1), ix, raw);
            prism_idx<FD>(A, cell_of(n1 + GS < ngroups ? n1 + GS : n1), ix);
        }
        lds_barrier();

        acc_t acc[C::CT][TW];
#pragma unroll
        for (int c = 0; c < C::CT; ++c)
#pragma unroll
            for (int i = 0; i < TW; ++i) acc[c][i] = acc_t{0, 0, 0, 0};
        const double* wd = wtab + NOFF * 4 * M1;  // weights of the pairs b = b'
        if constexpr (P == 2) {
            prism_contract<FORM, P, FD, PREC, 0, 0>(gt, wtab + wave * 4 * M1, rsrc, 0, lane, acc);
            prism_contract<FORM, P, FD, PREC, 1, C::tiles(0)>(gt, wd + wave * 4 * M1, rsrc, C::frags(0), lane, acc);
        } else if (wave < NOFF) {
            prism_contract<FORM, P, FD, PREC, 0, 0>(gt, wtab + wave * 4 * M1, rsrc, 0, lane, acc);
        } else {
            const double* w2 = wd + 2 * (wave - NOFF) * 4 * M1;
            prism_contract<FORM, P, FD, PREC, 1, 0>(gt, w2, rsrc, C::frags(0), lane, acc);
            prism_contract<FORM, P, FD, PREC, 1, TW - C::tiles(1)>(gt, w2 + 4 * M1, rsrc, C::frags(0), lane, acc);
        }

        // 4 / VP passes: pass p holds the accumulator elements v = p VP + vv of
        // every tile c, the cells acc_row(16 g, v) of lane groups g, in slots
        // of increasing cell
        constexpr int VP = C::VP;
        constexpr int NV1 = NN * (int)sizeof(out_t) / 16;  // 16-byte vectors per cell
        const u32x4p* s4 = reinterpret_cast<const u32x4p*>(st);
#pragma unroll
        for (int p = 0; p < 4 / VP; ++p) {
            lds_barrier();  // G reads (first pass) or the previous pass's copies are done
#pragma unroll
            for (int i = 0; i < TW; ++i) {
                if (off[i] == ~0u) continue;
#pragma unroll
                for (int c = 0; c < C::CT; ++c)
#pragma unroll
                    for (int vv = 0; vv < VP; ++vv) {
                        const out_t x = (out_t)acc[c][i][p * VP + vv];
                        out_t* sl = st + (c * 4 * VP + (PREC == PREC_F64 ? vv * 4 + (lane >> 4) : (lane >> 4) * VP + vv)) * C::CS;
                        sl[off[i] & 0xffff] = x;
                        sl[off[i] >> 16] = x;
                    }
            }
            lds_barrier();
            // copy out the pass's cells in memory order (consecutive ones share
            // lines), four vectors a thread at a time so that their LDS reads
            // overlap
            constexpr int NVEC = C::PC * NV1, TH = 64 * C::WAVES;
            if constexpr (C::PADV == 0 && C::CT == 1) {
                // one range in LDS and in memory
                static_assert(PREC == PREC_F64 || VP == 4, "consecutive cells");
                const int64_t c0 = base + 4 * VP * p;
                const int nv = A.ncells - c0 < 4 * VP ? (int)(A.ncells - c0) * NV1 : NVEC;
                u32x4p* o4 = reinterpret_cast<u32x4p*>(out + c0 * NN);
#pragma unroll
                for (int k0 = 0; k0 < NVEC; k0 += 4 * TH) {
                    u32x4p x[4];
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        if (k0 + n * TH < NVEC) x[n] = s4[k0 + n * TH + tid < NVEC ? k0 + n * TH + tid : tid];
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        if (k0 + n * TH < NVEC && k0 + n * TH + tid < nv) gstore_nt(&o4[k0 + n * TH + tid], x[n]);
                }
            } else {
#pragma unroll 1
                for (int k0 = tid; k0 < NVEC; k0 += 4 * TH) {
                    u32x4p x[4];
                    int64_t cl[4];
                    int at[4];
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        const int k = k0 + n * TH < NVEC ? k0 + n * TH : k0;
                        const int slot = k / NV1, in = k - slot * NV1;  // cell of the pass, vector of its matrix
                        const int c = slot / (4 * VP), m = slot % (4 * VP);
                        const int g = PREC == PREC_F64 ? m % 4 : m / VP, vv = PREC == PREC_F64 ? m / 4 : m % VP;
                        cl[n] = k0 + n * TH < NVEC ? base + 16 * c + acc_row<PREC>(16 * g, p * VP + vv) : A.ncells;
                        at[n] = in;
                        constexpr int RV = NS * (int)sizeof(out_t) / 16, PV = C::PADV > 0 ? 1 : 0;  // vectors of a row
                        const int row = in / RV;
                        x[n] = s4[slot * (C::CS * (int)sizeof(out_t) / 16) + row * (RV + PV) + (in - row * RV)];
                    }
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        if (cl[n] < A.ncells) gstore_nt(reinterpret_cast<u32x4p*>(out + cl[n] * NN) + at[n], x[n]);
                }
            }
        }
    }
}

}  // namespace dev

namespace {

using ld = long double;

uint16_t bf16_bits_host(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
float bf16_float_host(uint16_t h) {
    const uint32_t u = ((uint32_t)h) << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// Reference products per point (no weights; the weights are in G), in the
// device's column order k = q JQ + j.
bool prism_reference(int form, int p, int quad, RefTensor& R, std::vector<double>& qtab) {
    PrismTables t;
    if (!t.init(p, quad)) return false;
    const int n = t.n, nq = t.nq, NN = n * n;
    const int JQ = dev::prism_jq(form == COFFEE_MASS ? dev::F_MASS : (form == COFFEE_HELMHOLTZ ? dev::F_HELM
                                                                                                : dev::F_DIFF));
    R.NS = n;
    R.KR = nq * JQ;
    R.R.assign((size_t)R.KR * NN, 0.0L);
    auto ph = [&](int k, int a) -> ld { return t.phi[(size_t)k * n + a]; };
    auto dph = [&](int al, int k, int a) -> ld { return t.dphi[((size_t)al * nq + k) * n + a]; };
    for (int k = 0; k < nq; ++k) {
        int j = k * JQ;
        if (form != COFFEE_MASS) {
            for (int al = 0; al < 3; ++al)
                for (int be = al; be < 3; ++be, ++j)
                    for (int a = 0; a < n; ++a)
                        for (int b = 0; b < n; ++b) {
                            ld v = dph(al, k, a) * dph(be, k, b);
                            if (al != be) v += dph(be, k, a) * dph(al, k, b);
                            R.R[(size_t)j * NN + a * n + b] = v;
                        }
        }
        if (form != COFFEE_DIFFUSION)
            for (int a = 0; a < n; ++a)
                for (int b = 0; b < n; ++b) R.R[(size_t)j * NN + a * n + b] = ph(k, a) * ph(k, b);
    }
    qtab.resize(4 * (size_t)nq);
    for (int k = 0; k < nq; ++k) {
        for (int i = 0; i < 3; ++i) qtab[4 * k + i] = (double)t.X[3 * k + i];
        qtab[4 * k + 3] = (double)t.W[k];
    }
    return true;
}

// Degrees 2 and 3: fragments of the triangle products of both kinds of pairs
// in the k order of k_prism_fac, and the rule followed by the interval weights.
template <typename C>
void prism_fac_pack(const std::vector<ld> (&R)[2], int prec, std::vector<char>& frag) {
    // R[kind]: [type][triangle point][entry]
    for (int kind = 0; kind < 2; ++kind) {
        const int T = C::types(kind), NE = C::entries(kind), NT = C::tiles(kind);
        auto val = [&](int type, int i, int u) -> double {
            return type < T && i < C::NI && u < NE ? (double)R[kind][((size_t)type * C::NI + i) * NE + u] : 0.0;
        };
        auto put = [&](const void* p, size_t n) { frag.insert(frag.end(), (const char*)p, (const char*)p + n); };
        for (int s = 0; s < C::steps(kind); ++s)
            for (int t = 0; t < NT; ++t)
                for (int l = 0; l < 64; ++l) {
                    const int g = l / 16, u = 16 * t + l % 16;
                    if (C::BF) {
                        // parts of the value: hi, lo, third
                        auto part = [&](int type, int i, int k) -> uint16_t {
                            const float x = (float)val(type, i, u);
                            const uint16_t hi = bf16_bits_host(x), lo = bf16_bits_host(x - bf16_float_host(hi));
                            return k == 0 ? hi : (k == 1 ? lo : bf16_bits_host(x - bf16_float_host(hi) - bf16_float_host(lo)));
                        };
                        for (int k = 0; k < 8; ++k) {
                            uint16_t h = 0;
                            if (T == 1) {
                                const int f = 8 * s + k, r = f - 6 * C::FULLB;
                                if (r < 0) h = part(0, 4 * (f / 6) + g, dev::kMassParts[f % 6][1]);
                                else if (r < 2 * C::REM && g < 3)
                                    h = part(0, C::NI - 1, dev::kMassParts[dev::kMassRest[g][r]][1]);
                            } else {
                                // block s / 2 of four points, slot = type; hi, then lo
                                h = part(k, 4 * (s / 2) + g, s % 2);
                            }
                            put(&h, 2);
                        }
                    } else {
                        const bool full = s < C::FULLB * T;
                        const int type = full ? s % T : 4 * (s - C::FULLB * T) + g;
                        const int i = full ? 4 * (s / T) + g : C::NI - 1;
                        const double x = val(type, i, u);
                        const float f = (float)x;
                        if (prec == COFFEE_FP64) put(&x, 8);
                        else put(&f, 4);
                    }
                }
    }
}

template <int FORM, int P, int PREC>
void prism_fac_pack_prec(const std::vector<ld> (&R)[2], std::vector<char>& frag) {
    prism_fac_pack<dev::PrismFacCfg<FORM, P, 0, PREC>>(R, PREC, frag);
}

template <int FORM, int P>
bool prism_fac_tables(int quad, int prec, std::vector<char>& frag, std::vector<double>& qtab) {
    Tables tri;
    std::vector<ld> l, dl;
    constexpr int M1 = P + 1;
    PrismTables pt;
    if (!tri.init(2, P, quad) || tri.nq != M1 * M1 || !interval_tables(P, M1, l, dl) || !pt.init(P, quad)) return false;
    const int n = tri.n, ni = tri.nq;
    std::vector<ld> R[2];
    for (int kind = 0; kind < 2; ++kind) {
        const int T = FORM == dev::F_MASS ? 1 : (kind == 0 ? 8 : 6);
        for (int type = 0; type < T; ++type)
            for (int i = 0; i < ni; ++i)
                for (int a = 0; a < n; ++a)
                    for (int b = kind == 0 ? 0 : a; b < n; ++b) {
                        auto ph = [&](int x) { return tri.phi[(size_t)i * n + x]; };
                        auto d = [&](int al, int x) { return tri.dphi[((size_t)al * ni + i) * n + x]; };
                        ld v;
                        if (FORM == dev::F_MASS || type == T - 1) v = ph(a) * ph(b);
                        else if (type == 0) v = d(0, a) * d(0, b);
                        else if (type == 1) v = d(0, a) * d(1, b) + d(1, a) * d(0, b);
                        else if (type == 2) v = d(1, a) * d(1, b);
                        else if (kind == 1) v = d(type - 3, a) * ph(b) + ph(a) * d(type - 3, b);
                        else if (type <= 4) v = d(type - 3, a) * ph(b);
                        else v = ph(a) * d(type - 5, b);
                        R[kind].push_back(v);
                    }
    }
    frag.clear();
    if (prec == COFFEE_FP64) prism_fac_pack_prec<FORM, P, dev::PREC_F64>(R, frag);
    else if (prec == COFFEE_FP32) prism_fac_pack_prec<FORM, P, dev::PREC_F32>(R, frag);
    else prism_fac_pack_prec<FORM, P, dev::PREC_BF16X3>(R, frag);
    qtab.clear();
    for (int k = 0; k < pt.nq; ++k) {
        for (int i = 0; i < 3; ++i) qtab.push_back((double)pt.X[3 * k + i]);
        qtab.push_back((double)pt.W[k]);
    }
    auto weights = [&](int b, int b2) {
        for (int k = 0; k < 4; ++k)
            for (int j = 0; j < M1; ++j)
                qtab.push_back((double)((k & 2 ? dl : l)[j * M1 + b] * (k & 1 ? dl : l)[j * M1 + b2]));
    };
    for (int b = 0; b < M1; ++b)
        for (int b2 = b + 1; b2 < M1; ++b2) weights(b, b2);
    for (int b = 0; b < M1; ++b) weights(b, b);
    return true;
}

template <int P>
bool prism_fac_tables_form(int form, int quad, int prec, std::vector<char>& frag, std::vector<double>& qtab) {
    if (form == COFFEE_MASS) return prism_fac_tables<dev::F_MASS, P>(quad, prec, frag, qtab);
    if (form == COFFEE_HELMHOLTZ) return prism_fac_tables<dev::F_HELM, P>(quad, prec, frag, qtab);
    return prism_fac_tables<dev::F_DIFF, P>(quad, prec, frag, qtab);
}

struct PrismTable {
    void* frag = nullptr;
    double* qtab = nullptr;
};

std::mutex g_prism_mu;
std::map<std::tuple<int, int, int, int, int>, PrismTable> g_prism_tabs;  // (dev, form, p, quad, prec)

coffee_status prism_table(int dev, int form, int p, int quad, int prec, PrismTable* out) {
    std::lock_guard<std::mutex> lk(g_prism_mu);
    auto key = std::make_tuple(dev, form, p, quad, prec);
    auto it = g_prism_tabs.find(key);
    if (it != g_prism_tabs.end()) {
        *out = it->second;
        return COFFEE_OK;
    }
    std::vector<double> qtab;
    std::vector<char> frag;
    if (p == 1) {
        RefTensor R;
        if (!prism_reference(form, p, quad, R, qtab)) return COFFEE_E_INVALID_ARG;
        frag = pack_fragments(R, prec, true, 0);
    } else if (!(p == 2 ? prism_fac_tables_form<2>(form, quad, prec, frag, qtab)
                        : prism_fac_tables_form<3>(form, quad, prec, frag, qtab))) {
        return COFFEE_E_INVALID_ARG;
    }
    PrismTable t;
    if (hipMalloc(&t.frag, frag.size()) != hipSuccess) return COFFEE_E_NOMEM;
    if (hipMalloc((void**)&t.qtab, qtab.size() * sizeof(double)) != hipSuccess) {
        (void)hipFree(t.frag);
        return COFFEE_E_NOMEM;
    }
    if (hipMemcpy(t.frag, frag.data(), frag.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(t.qtab, qtab.data(), qtab.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(t.frag);
        (void)hipFree(t.qtab);
        return COFFEE_E_HIP;
    }
    g_prism_tabs[key] = t;
    *out = t;
    return COFFEE_OK;
}

template <int FORM, int P, int FD, int PREC, int NQ>
hipError_t launch_prism(const dev::PrismArgs& a, hipStream_t s, int dev_id) {
    using C = dev::PrismCfg<FORM, P, FD, PREC, NQ>;
    const void* kern = reinterpret_cast<const void*>(&dev::k_prism<FORM, P, FD, PREC, NQ>);
    static const hipError_t attr =
        hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const int64_t wgs_needed = (a.ntiles + C::WAVES - 1) / C::WAVES;
    // grid multiplier from the tuning cache (prism keys: cell COFFEE_PRISM)
    int tuned_variant = 0;
    const int tuned = tuned_linear(FORM, COFFEE_PRISM, P, FD, PREC, &tuned_variant);
    const int grid = grid_for(dev_id, kern, C::WAVES * 64, C::LDS_BYTES, wgs_needed, tuned > 0 ? tuned : 1);
    hipLaunchKernelGGL((dev::k_prism<FORM, P, FD, PREC, NQ>), dim3(grid), dim3(C::WAVES * 64), C::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <int FORM, int P, int FD, int PREC>
hipError_t launch_prism_fac(const dev::PrismArgs& a, hipStream_t s, int dev_id) {
    using C = dev::PrismFacCfg<FORM, P, FD, PREC>;
    const void* kern = reinterpret_cast<const void*>(&dev::k_prism_fac<FORM, P, FD, PREC>);
    static const hipError_t attr =
        hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const int64_t wgs_needed = (a.ncells + C::CELLS - 1) / C::CELLS;  // one cell group per workgroup at a time
    int tuned_variant = 0;
    const int tuned = tuned_linear(FORM, COFFEE_PRISM, P, FD, PREC, &tuned_variant);
    // degree 2: short-lived workgroups (16 grids of the resident set) ran 494
    // us against 522 for one persistent set (FP64 diffusion, 524,288 cells);
    // degree 3, which prefetches: 385 against 367 (65,536 cells)
    const int grid = grid_for(dev_id, kern, C::WAVES * 64, C::LDS_BYTES, wgs_needed,
                              tuned > 0 ? tuned : (P == 2 ? 16 : 1));
    hipLaunchKernelGGL((dev::k_prism_fac<FORM, P, FD, PREC>), dim3(grid), dim3(C::WAVES * 64), C::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <int FORM, int P, int FD, int NQ>
hipError_t launch_prism_prec(int prec, const dev::PrismArgs& a, hipStream_t s, int dev_id) {
    if constexpr (P >= 2) {
        if (prec == COFFEE_FP64) return launch_prism_fac<FORM, P, FD, dev::PREC_F64>(a, s, dev_id);
        if (prec == COFFEE_FP32) return launch_prism_fac<FORM, P, FD, dev::PREC_F32>(a, s, dev_id);
        return launch_prism_fac<FORM, P, FD, dev::PREC_BF16X3>(a, s, dev_id);
    } else {
        if (prec == COFFEE_FP64) return launch_prism<FORM, P, FD, dev::PREC_F64, NQ>(a, s, dev_id);
        if (prec == COFFEE_FP32) return launch_prism<FORM, P, FD, dev::PREC_F32, NQ>(a, s, dev_id);
        return launch_prism<FORM, P, FD, dev::PREC_BF16X3, NQ>(a, s, dev_id);
    }
}

template <int P, int NQ>
hipError_t launch_prism_form(int form, int fd, int prec, const dev::PrismArgs& a, hipStream_t s, int dev_id) {
    using namespace dev;
    if (form == COFFEE_DIFFUSION) return launch_prism_prec<F_DIFF, P, 0, NQ>(prec, a, s, dev_id);
    if (form == COFFEE_MASS)
        return fd ? launch_prism_prec<F_MASS, P, 1, NQ>(prec, a, s, dev_id)
                  : launch_prism_prec<F_MASS, P, 0, NQ>(prec, a, s, dev_id);
    return fd ? launch_prism_prec<F_HELM, P, 1, NQ>(prec, a, s, dev_id)
              : launch_prism_prec<F_HELM, P, 0, NQ>(prec, a, s, dev_id);
}

}  // namespace

// Prism entry of coffee_assemble: arguments already validated (form mass,
// Helmholtz or diffusion; field none or degree 1 scalar).
coffee_status assemble_prism(int form, int degree, int quad, int precision, const double* coords,
                             const int32_t* c2v, int64_t ncells, const coffee_field* coeffs, int ncoeff,
                             const double* constants, int nconst, void* out, void* hip_stream) {
    // compiled: the default rule (q = 2p) at degree 1 (8 points), 2 (27 points) and 3 (64 points)
    if (degree < 1 || degree > 3 || quad != 2 * degree) return COFFEE_E_UNSUPPORTED;
    if (ncells == 0) return COFFEE_OK;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return COFFEE_E_HIP;
    PrismTable t;
    coffee_status st = prism_table(dev, form, degree, quad, precision, &t);
    if (st != COFFEE_OK) return st;
    dev::PrismArgs a;
    std::memset(&a, 0, sizeof a);
    a.coords = coords;
    a.c2v = c2v;
    a.ncells = ncells;
    if (ncoeff >= 1) a.f = dev::FieldArg{coeffs[0].values, coeffs[0].cell_to_dof};
    a.kdt = (nconst > 0 ? constants[0] : 1.0) * (nconst > 1 ? constants[1] : 1.0);
    a.qtab = t.qtab;
    a.rfrag = t.frag;
    a.out = out;
    a.ntiles = (ncells + 15) / 16;
    const int fd = ncoeff >= 1 ? 1 : 0;
    hipStream_t s = (hipStream_t)hip_stream;
    const hipError_t e = degree == 1   ? launch_prism_form<1, 8>(form, fd, precision, a, s, dev)
                         : degree == 2 ? launch_prism_form<2, 27>(form, fd, precision, a, s, dev)
                                       : launch_prism_form<3, 64>(form, fd, precision, a, s, dev);
    return e == hipSuccess ? COFFEE_OK : COFFEE_E_HIP;
}

void free_prism_tables() {
    std::lock_guard<std::mutex> lk(g_prism_mu);
    for (auto& kv : g_prism_tabs) {
        (void)hipSetDevice(std::get<0>(kv.first));
        (void)hipFree(kv.second.frag);
        (void)hipFree(kv.second.qtab);
    }
    g_prism_tabs.clear();
}

}  // namespace coffee
