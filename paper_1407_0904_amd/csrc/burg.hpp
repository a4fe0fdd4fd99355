// Device engine for the Burgers Jacobian at degrees 1 and 2 (cell-row engine).
//
// Block (c, c') of the Jacobian at state w is
//     A_cc' = delta_cc' D + E_cc'
//     D     = (1/dt) mass + nu stiffness + convection by w      (one matrix per cell)
//     E_cc'[a][b] = int phi_a phi_b d w_c / d x_c'
// so D is contracted once per cell, with K0 = 1 + d(d+1)/2 + n d terms, not
// once per diagonal block. The gradient of w has degree P - 1: its values at
// the NV nodes of that degree fix it, and E_cc' = sum_k |det J| (d w_c / d x_c')(X_k) T_k,
// T_k = sum_q W_q N_k phi_a phi_b, takes NV terms (4 for P2 tetrahedra) where
// the expansion over the state's dofs takes n d (30). For P2 tetrahedra the
// matrix cores run 133 products per 16 cells, against 763 when every block's
// row holds all 67 terms.
//
// Work unit as in elast.hpp: a wave takes 16 cells. D of the 16 cells is one
// 16-row product, kept in LDS. The rows of the E products are (cell, block)
// pairs in cell-major order, 16 at a time; their accumulators start from the
// cell's D in the diagonal blocks and from zero in the others, so a tile's
// results are final. They go to a ring of whole-cell slots in LDS, and the
// cells a tile completes leave as one contiguous range of 16-byte stores
// (whole cells in order: row pieces of many cells at a time reached only 60%
// of that write rate).
//
// Degree 1: four waves a workgroup, so that a small mesh reaches more CUs, and
// a larger ring (bg_sizes). P1 tetrahedra, 383,997 cells, FP64 / FP32 / BF16X3:
// 98 / 67 / 75 us (all terms in every block 105 / 67 / 82; eight waves and the
// ring of degree 2 101 / 75 / 89); 1,293 cells 6.7 / 6.3 / 7.4 (11.0 / 7.5 /
// 9.1; 9.5 / 8.8 / 10.1). P1 triangles, 524,285: 51 / 37 / 44 (51 / 42 / 44; 53 /
// 39 / 45).
// 663,552 P2 tetrahedra: 980 us in FP64, 555 in FP32, 565 in BF16X3, against
// 1,694, 814 and 846 for all terms in every block; what is left is the write
// of the tensors (4.78 GB in FP64).
#pragma once
#include "vector.hpp"

namespace coffee {
namespace dev {

struct BgSizes {
    int ns, nn, n, cellv, nb, nv, kr0, ks0, row0, nt, ring, erow;
    int e_bytes, d_bytes, ring_bytes, wave_bytes, waves, lds_bytes;
    bool rreg;
};

__host__ __device__ constexpr BgSizes bg_sizes(int d, int p, int prec) {
    BgSizes s{};
    s.ns = nsc(d, p);
    s.nn = s.ns * s.ns;
    s.n = d * s.ns;
    s.cellv = s.n * s.n;
    s.nb = d * d;
    s.nv = grad_nv(d, p);
    s.kr0 = 1 + npair(d) + s.ns * d;
    s.ks0 = prec == PREC_BF16X3 ? (4 * s.kr0 + 31) / 32 : (s.kr0 + 3) / 4;
    s.row0 = prec == PREC_BF16X3 ? s.ks0 * 32 + 8 : s.ks0 * 4 + 1;
    s.nt = (s.nn + 15) / 16;
    const int gsz = prec == PREC_F64 ? 8 : (prec == PREC_F32 ? 4 : 2);
    const int osz = prec == PREC_F64 ? 8 : 4;
    const int fsz = prec == PREC_F64 ? 8 : (prec == PREC_F32 ? 4 : 16);
    // E rows: one k-step of four entries (BF16X3: four slots an entry; the
    // upper half of its 32 is zero and not stored)
    s.erow = prec == PREC_BF16X3 ? 16 : 4;
    s.e_bytes = 16 * s.nb * s.erow * gsz;
    s.d_bytes = (16 * s.nn * osz + 15) / 16 * 16;
    // the ring; before the first tile its memory holds the D rows and the state
    const int g0 = (16 * s.row0 * gsz + 15) / 16 * 16, w = 16 * (s.n | 1) * 8;
    constexpr int L = 160 * 1024;
    const int most = p == 1 ? 4 : 8;  // waves
    // Cells: degree 2 those that a 16-row tile touches (four whole ones of 4
    // blocks, at most three of 9). Cells of degree 1 are small (576 bytes in
    // FP32 on tetrahedra): one or two at a time fill neither the lanes nor the
    // lines of a store, so the ring takes all 16 of the unit where three
    // workgroups still fit a CU, else nine, which leave as eight and eight.
    for (int cells : {16, 9, s.nb == 4 ? 4 : 3}) {
        s.ring = cells;
        s.ring_bytes = (cmax(cells * s.cellv * osz, g0 + w) + 15) / 16 * 16;
        s.wave_bytes = s.e_bytes + s.d_bytes + s.ring_bytes;
        if (p == 1 && (cells == 9 || 3 * most * s.wave_bytes <= L)) break;
    }
    const int fit = L / s.wave_bytes;
    s.waves = fit < most ? fit : most;
    // D's reference fragments in registers: 160 of them at one wave per SIMD,
    // 80 at two, else through the caches
    const int rregs = s.nt * s.ks0 * (fsz / 4);
    s.rreg = rregs <= (s.waves <= 4 ? 160 : 80);
    s.lds_bytes = s.waves * s.wave_bytes;
    return s;
}

template <int D, int P, int PREC>
struct BgCfg {
    using g_t = typename PrecT<PREC>::gtype;
    using frag_t = typename PrecT<PREC>::frag;
    using acc_t = typename PrecT<PREC>::acc;
    using out_t = typename PrecT<PREC>::otype;
    static constexpr BgSizes S = bg_sizes(D, P, PREC);
    static constexpr int NS = S.ns, NN = S.nn, N = S.n, CELLV = S.cellv, NB = S.nb, NV = S.nv;
    static constexpr int KR0 = S.kr0, KS0 = S.ks0, ROW0 = S.row0, NT = S.nt, RING = S.ring, EROW = S.erow;
    static constexpr int WAVES = S.waves;
    static constexpr int WROW = N | 1;                           // state of one cell in LDS
    static constexpr int G0B = (16 * ROW0 * (int)sizeof(g_t) + 15) / 16 * 16;
    static constexpr int CPC = CELLV * (int)sizeof(out_t) / 16;  // 16-byte chunks per cell
    static constexpr int RPL = VLane<F_BURG, D, P>::RPL;
    static_assert(WAVES >= 4 && CELLV * (int)sizeof(out_t) % 16 == 0 && NV <= 4, "sizes");
};

template <int D, int P, int PREC>
struct BgWave {
    using C = BgCfg<D, P, PREC>;
    typename C::g_t* ebuf;    // 16 NB rows of E coefficients
    typename C::out_t* dbuf;  // D of the 16 cells
    typename C::out_t* ring;  // RING cell slots
    typename C::g_t* g0;      // D rows and the state, in the ring's memory
    double* wbuf;
    const typename C::frag_t* rd;  // D's fragments (global)
    typename C::frag_t rreg[C::S.rreg ? C::NT : 1][C::S.rreg ? C::KS0 : 1];
    typename C::frag_t et[C::NT];  // T's fragments
    int lane;
};

// D of the unit's cells into dbuf and the E rows into ebuf. Lane (cell, g)
// holds the state at the dofs g, g + 4, ... and forms the D entries of those
// dofs, then the gradient of the state at node g.
template <int D, int P, int PREC>
__device__ __forceinline__ void bg_prepare(const LinArgs& A, BgWave<D, P, PREC>& W, const VCell<F_BURG, D, P>& cd,
                                           bool valid) {
    using C = BgCfg<D, P, PREC>;
    using acc_t = typename C::acc_t;
    using frag_t = typename C::frag_t;
    using out_t = typename C::out_t;
    constexpr int NS = C::NS, NN = C::NN, KR0 = C::KR0, KS0 = C::KS0, NT = C::NT;
    const int lane = W.lane, cell = lane & 15, g = lane >> 4;
    const double ad = valid ? cd.ad : 0.0;
    typename C::g_t* row = W.g0 + cell * C::ROW0;
    double* wc = W.wbuf + cell * C::WROW;
    if (g == 0) {
        put_g<PREC, KR0>(row, 0, ad * A.c1);
        int t = 1;
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int b = a; b < D; ++b) put_g<PREC, KR0>(row, t++, ad * A.c0 * cd.M[a][b]);
        if constexpr (PREC == PREC_BF16X3) {
#pragma unroll
            for (int k = 4 * KR0; k < KS0 * 32; ++k) row[k] = 0;
        } else {
#pragma unroll
            for (int k = KR0; k < KS0 * 4; ++k) row[k] = 0;
        }
    }
#pragma unroll
    for (int j = 0; j < C::RPL; ++j) {
        const int r = g + 4 * j;
        if (r < NS) {
            const double* w = cd.f[0][j];
#pragma unroll
            for (int a = 0; a < D; ++a) {
                double t = 0.0;
#pragma unroll
                for (int i = 0; i < D; ++i) t += w[i] * cd.K[a][i];
                put_g<PREC, KR0>(row, 1 + npair(D) + r * D + a, ad * t);
                wc[r * D + a] = w[a];
            }
        }
    }
    wave_sync();
    {
        acc_t acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS0; ++s) {
            const frag_t a = load_afrag<PREC>(W.g0, C::ROW0, lane, s);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                frag_t b;
                if constexpr (C::S.rreg) b = W.rreg[t][s];
                else b = W.rd[(t * KS0 + s) * 64 + lane];
                acc[t] = mfma<PREC>(a, b, acc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int el = 16 * t + (lane & 15);
            if (16 * t + 16 <= NN || el < NN) {
#pragma unroll
                for (int v = 0; v < 4; ++v) W.dbuf[acc_row<PREC>(lane, v) * NN + el] = (out_t)acc[t][v];
            }
        }
    }
    if (g < C::NV) {
        double gw[D][D];  // physical gradient of the state at node g, times |det J|
#pragma unroll
        for (int c = 0; c < D; ++c) {
            double y[D + 1];  // derivatives in the barycentric coordinates
#pragma unroll
            for (int i = 0; i <= D; ++i) {
                if constexpr (P == 1) y[i] = wc[i * D + c];
                else {
                    const double at = wc[i * D + c], ed = wc[(i == g ? 0 : edge_dof_rt<D>(g, i)) * D + c];
                    y[i] = i == g ? 3.0 * at : 4.0 * ed - at;
                }
            }
#pragma unroll
            for (int j = 0; j < D; ++j) {
                double t = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a) t += (y[a + 1] - y[0]) * cd.K[a][j];
                gw[c][j] = ad * t;
            }
        }
#pragma unroll
        for (int c = 0; c < D; ++c)
#pragma unroll
            for (int j = 0; j < D; ++j) put_g<PREC, 4>(W.ebuf + (cell * C::NB + c * D + j) * C::EROW, g, gw[c][j]);
    }
    wave_sync();
}

// The first cell that has not left the ring before row tile m: cells leave
// when the next tile's would not fit beside them (and after the last tile).
constexpr int bg_left(int nb, int ring, int m) {
    int left = 0;
    for (int t = 0; t < m; ++t)
        if (t + 1 == nb || (16 * (t + 2) + nb - 1) / nb - left > ring) left = 16 * (t + 1) / nb;
    return left;
}

// Row tile m: E products on top of D, into the cell ring; then, when the ring
// has no room for the next tile's cells, the complete ones leave as one
// contiguous store range.
template <int D, int P, int PREC, bool FULL, int m>
__device__ __forceinline__ void bg_rowtile(const LinArgs& A, const BgWave<D, P, PREC>& W, int64_t unit_base) {
    using C = BgCfg<D, P, PREC>;
    using acc_t = typename C::acc_t;
    using frag_t = typename C::frag_t;
    using out_t = typename C::out_t;
    constexpr int NB = C::NB, NS = C::NS, N = C::N, NN = C::NN, NT = C::NT;
    __builtin_amdgcn_sched_barrier(0);
    // the lane index re-read opaquely: the staging offsets below are formed
    // per tile instead of being hoisted out of the unit loop
    int lane = W.lane;
    asm volatile("" : "+v"(lane));
    frag_t a;
    if constexpr (PREC == PREC_BF16X3) {
        // slots 16 .. 31 of the k-step (lanes 32 .. 63) are zero
        const bf8 x = *reinterpret_cast<const bf8*>(W.ebuf + (16 * m + (lane & 15)) * C::EROW + 8 * ((lane >> 4) & 1));
        const bf8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        a = lane < 32 ? x : zero;
    } else {
        a = W.ebuf[(16 * m + (lane & 15)) * C::EROW + (lane >> 4)];
    }
    int base[4], dsrc[4];  // ring origin of row v's block, its cell's D
    bool diag[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * m + acc_row<PREC>(lane, v);
        const int ci = row / NB, bk = row - (row / NB) * NB, c = bk / D, c2 = bk - (bk / D) * D;
        base[v] = (ci % C::RING) * C::CELLV + c * NS * N + c2 * NS;
        dsrc[v] = ci * NN;
        diag[v] = c == c2;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        // this lane's column of n-tile t is entry (ea, eb) of the block
        const int el = 16 * t + (lane & 15);
        const bool ok = 16 * t + 16 <= NN || el < NN;
        const int ea = el / NS, eb = el - (el / NS) * NS;
        acc_t acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const out_t x = W.dbuf[dsrc[v] + (ok ? el : 0)];
            acc[v] = diag[v] ? x : out_t(0);
        }
        acc = mfma<PREC>(a, W.et[t], acc);
        if (ok) {
#pragma unroll
            for (int v = 0; v < 4; ++v) W.ring[base[v] + ea * N + eb] = (out_t)acc[v];
        }
    }
    // cells [cd0, cd1) of the unit leave; their slots are consecutive except
    // where the ring wraps (at chunk WQ of the range)
    constexpr int cd0 = bg_left(NB, C::RING, m), cd1 = bg_left(NB, C::RING, m + 1);
    constexpr int CPC = C::CPC, NQ = (cd1 - cd0) * CPC;
    constexpr int s0 = cd0 % C::RING, WQ = (C::RING - s0) * CPC, WRAP = C::RING * CPC;
    static_assert(cd1 - cd0 <= C::RING, "ring");
    if constexpr (NQ > 0) {
        wave_sync();
        const vu32x4* rb = reinterpret_cast<const vu32x4*>(W.ring) + s0 * CPC;
        // a wave-uniform base and 32-bit byte offsets: scalar base addressing
        char* dst = reinterpret_cast<char*>(uniform_ptr(reinterpret_cast<vu32x4*>(A.out) +
                                                        (unit_base + cd0) * (int64_t)CPC));
#pragma unroll
        for (int q0 = 0; q0 < NQ; q0 += 64) {
            const int q = q0 + lane;
            int li = q;
            if constexpr (WQ < NQ) {
                if (q0 >= WQ) li = q - WRAP;
                else if (q0 + 64 > WQ) li = q >= WQ ? q - WRAP : q;
            }
            bool ok = q0 + 64 <= NQ || q < NQ;
            if constexpr (!FULL) ok = ok && unit_base + cd0 + q / CPC < A.ncells;
            if (ok) gstore_nt(reinterpret_cast<vu32x4*>(dst + (uint32_t)(q * 16)), rb[li]);
        }
        wave_sync();
    }
}

template <int D, int P, int PREC, bool FULL, int m>
__device__ __forceinline__ void bg_rowtiles(const LinArgs& A, const BgWave<D, P, PREC>& W, int64_t unit_base) {
    bg_rowtile<D, P, PREC, FULL, m>(A, W, unit_base);
    if constexpr (m + 1 < BgCfg<D, P, PREC>::NB) bg_rowtiles<D, P, PREC, FULL, m + 1>(A, W, unit_base);
}

// Persistent kernel: units of 16 cells, WAVES units per chunk, XCD-aware chunk
// order and two-deep gather prefetch as in the other engines.
// LinArgs::nchunks = ceil(ncells / (16 WAVES)); LinArgs::rfrag holds the
// fragments of D's tensors, then those of T.
template <int D, int P, int PREC>
__global__ __launch_bounds__((BgCfg<D, P, PREC>::WAVES * 64)) void k_burgers(LinArgs A) {
    using C = BgCfg<D, P, PREC>;
    using frag_t = typename C::frag_t;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    BgWave<D, P, PREC> W;
    W.lane = threadIdx.x & 63;
    const int g = W.lane >> 4;
    unsigned char* mine = lds + wave * C::S.wave_bytes;
    W.ebuf = reinterpret_cast<typename C::g_t*>(mine);
    W.dbuf = reinterpret_cast<typename C::out_t*>(mine + C::S.e_bytes);
    W.ring = reinterpret_cast<typename C::out_t*>(mine + C::S.e_bytes + C::S.d_bytes);
    W.g0 = reinterpret_cast<typename C::g_t*>(W.ring);
    W.wbuf = reinterpret_cast<double*>(mine + C::S.e_bytes + C::S.d_bytes + C::G0B);
    W.rd = reinterpret_cast<const frag_t*>(A.rfrag);
    if constexpr (C::S.rreg) {
#pragma unroll
        for (int t = 0; t < C::NT; ++t)
#pragma unroll
            for (int s = 0; s < C::KS0; ++s) W.rreg[t][s] = W.rd[(t * C::KS0 + s) * 64 + W.lane];
    }
#pragma unroll
    for (int t = 0; t < C::NT; ++t) W.et[t] = W.rd[(C::NT * C::KS0 + t) * 64 + W.lane];
    // E entries of nodes that do not exist stay zero
    for (int i = W.lane; i < 16 * C::NB * C::EROW; i += 64) W.ebuf[i] = 0;
    wave_sync();
    const int64_t GS = gridDim.x;
    const int64_t b = blockIdx.x;
    int64_t chunk = (GS % 8 == 0) ? (b % 8) * (GS / 8) + b / 8 : b;
    const int64_t nfull = A.ncells / 16;  // units whose 16 cells all exist
    auto unit_of = [&](int64_t ch) -> int64_t { return ch * C::WAVES + wave; };
    auto cell_of = [&](int64_t unit) -> int64_t { return unit * 16 + (W.lane & 15); };
    int64_t unit = unit_of(chunk);
    VIdx<F_BURG, D, P> ix;
    VRaw<F_BURG, D, P> raw;
    VCell<F_BURG, D, P> cd;
    if (unit < nfull) {
        vload_idx<F_BURG, D, P>(A, cell_of(unit), g, ix);
        vload_raw<F_BURG, D, P>(A, cell_of(unit), g, ix, raw);
        vcell_from_raw<F_BURG, D, P>(raw, cd);
        const int64_t u1 = unit_of(chunk + GS) < nfull ? unit_of(chunk + GS) : unit;
        vload_idx<F_BURG, D, P>(A, cell_of(u1), g, ix);
#pragma unroll
        for (int v = 0; v <= D; ++v) asm volatile("" ::"v"(ix.v[v]));
        asm volatile("" ::"v"(cd.ad));
    }
    while (unit < nfull) {
        const int64_t next = unit_of(chunk + GS);
        const int64_t n1 = next < nfull ? next : unit;
        const int64_t n2 = unit_of(chunk + 2 * GS) < nfull ? unit_of(chunk + 2 * GS) : unit;
        bg_prepare<D, P, PREC>(A, W, cd, true);
        vload_raw<F_BURG, D, P>(A, cell_of(n1), g, ix, raw);
        vload_idx<F_BURG, D, P>(A, cell_of(n2), g, ix);
        bg_rowtiles<D, P, PREC, true, 0>(A, W, unit * 16);
        vcell_from_raw<F_BURG, D, P>(raw, cd);
        chunk += GS;
        unit = next;
    }
    if (unit * 16 < A.ncells) {
        // the one partial unit: clamped loads, bounds-checked stores
        const int64_t last = A.ncells - 1;
        const int64_t c = cell_of(unit) < last ? cell_of(unit) : last;
        VIdx<F_BURG, D, P> ix2;
        VRaw<F_BURG, D, P> raw2;
        vload_idx<F_BURG, D, P>(A, c, g, ix2);
        vload_raw<F_BURG, D, P>(A, c, g, ix2, raw2);
        vcell_from_raw<F_BURG, D, P>(raw2, cd);
        bg_prepare<D, P, PREC>(A, W, cd, cell_of(unit) < A.ncells);
        bg_rowtiles<D, P, PREC, false, 0>(A, W, unit * 16);
    }
}

}  // namespace dev
}  // namespace coffee
