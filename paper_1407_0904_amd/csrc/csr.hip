// Global assembly: the element tensors summed into the sparse matrix of the
// linear system (paper, section 2: the per-cell contributions are added to
// the global system; local assembly is the step before this one).
//
// Pattern (symbolic phase, once per mesh and space): every pair of dofs
// that share a cell is a nonzero. The pairs (dof_i, dof_j) of all cells,
// as 64-bit keys dof_i * ndofs + dof_j, are radix-sorted and deduplicated;
// the sorted unique keys are the scalar pattern in CSR order, the row
// pointers come from a histogram of their rows and a prefix sum. For a
// vector space with ncomp components (global index dof * ncomp + c) every
// scalar nonzero becomes an ncomp x ncomp block.
//
// Numeric phase: the cells are assembled in chunks into a workspace by the
// local-assembly engines (coffee_assemble), then the tensors of runs of
// consecutive cells are summed in LDS and added to the matrix rows with
// atomic adds (FP64 or FP32 by precision; k_scatter_csr).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "library.h"
#include "tables.h"

namespace coffee {
namespace dev {

__global__ __launch_bounds__(256) void k_pair_keys(const int32_t* __restrict__ c2d, int64_t ncells, int nloc,
                                                  uint64_t ndofs, uint64_t* __restrict__ keys) {
    const int64_t total = ncells * nloc * nloc;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = t / (nloc * nloc);
        const int ij = (int)(t - e * nloc * nloc), i = ij / nloc, j = ij - (ij / nloc) * nloc;
        keys[t] = (uint64_t)(uint32_t)c2d[e * nloc + i] * ndofs + (uint32_t)c2d[e * nloc + j];
    }
}

// flag[k] = 1 if sorted key k differs from key k-1 (first of its run)
__global__ __launch_bounds__(256) void k_run_heads(const uint64_t* __restrict__ sk, int64_t n,
                                                  int32_t* __restrict__ flag) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        flag[k] = (k == 0 || sk[k] != sk[k - 1]) ? 1 : 0;
}

// unique key u = pos[k] for run heads: scalar column and per-row count
__global__ __launch_bounds__(256) void k_compact(const uint64_t* __restrict__ sk, const int32_t* __restrict__ flag,
                                                const int64_t* __restrict__ pos, int64_t n, uint64_t ndofs,
                                                int32_t* __restrict__ scol, int64_t* __restrict__ rowcnt) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        if (!flag[k]) continue;
        const uint64_t key = sk[k];
        scol[pos[k]] = (int32_t)(key % ndofs);
        atomicAdd(reinterpret_cast<unsigned long long*>(&rowcnt[key / ndofs]), 1ull);
    }
}

// block expansion of the scalar pattern into the ncomp-component pattern
__global__ __launch_bounds__(256) void k_expand(const int64_t* __restrict__ srow, const int32_t* __restrict__ scol,
                                               int64_t ndofs, int nc, int64_t* __restrict__ row_ptr,
                                               int32_t* __restrict__ col_idx) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < ndofs; r += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = srow[r], len = srow[r + 1] - b;
        for (int c1 = 0; c1 < nc; ++c1) {
            const int64_t R = r * nc + c1, start = (int64_t)nc * nc * b + (int64_t)c1 * nc * len;
            row_ptr[R] = start;
            for (int64_t m = 0; m < len; ++m)
                for (int c2 = 0; c2 < nc; ++c2) col_idx[start + m * nc + c2] = scol[b + m] * nc + c2;
        }
        if (r == ndofs - 1) row_ptr[ndofs * nc] = (int64_t)nc * nc * srow[ndofs];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_zero(T* p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = T(0);
}

// Numeric scatter. A workgroup takes a run of consecutive cells and sums
// their tensors before it touches the matrix: the run's distinct dofs are
// numbered by an LDS hash, every tensor entry is added to a dense matrix over
// them in LDS, and each of its rows is then added to the matrix row by 16
// lanes, which read the row's columns, look them up in the hash and add the
// nonzero sums on consecutive addresses.
// Why: the matrix is bound by its atomic adds. Cells of a run share rows, so
// it sees about half as many, and lanes on consecutive addresses share a
// request; one thread per tensor row, each searching its own matrix row and
// adding on its own, made one request per entry and waited for every search
// step. A column costs one hash probe, no search but in long rows. (Summing
// into copies of the matrix rows in LDS, with a binary search per entry, was
// bound by the LDS reads of the search: 443 us in all for the case below.)
// Helmholtz P2 tetrahedra, FP64, 384,000 cells (assembly of the tensors
// included): 1,597 -> 474 us, of which the adds themselves take 185.
// Two workgroups of 16 waves fill a CU (71 KB of LDS each in FP64, 64 registers;
// with 68 of them, one workgroup, elasticity on 82,941 P1 tetrahedra took 303
// us instead of 258): the steps of a run are short and wait for one another.
// Measured for the case above and for elasticity P2 (41,154 cells): 512 threads
// and 81 rows 535 and 491 us, 1,024 threads and 90 rows 474 and 448 us, 96 rows
// (one workgroup per CU) 475 and 450 us.
constexpr int kCsrThreads = 1024;
constexpr int kCsrDense = 90;   // rows of the LDS matrix
constexpr int kCsrHash = 1024;  // more slots than a run has local dofs
constexpr int kCsrAhead = 5;    // columns in flight per lane and row
// A row with more columns is searched for the run's columns (at most 90)
// instead of being read by every run that touches it: a fan of 100,000 P1
// triangles around one vertex, whose row has a column for each, 3,460 us when
// it is read, 63 when it is searched (10,000 triangles 129 and 20).
constexpr int kCsrLong = 1024;

// Cells that fit the LDS matrix in any order, at most the cells of a run.
constexpr int csr_safe(int nl, int nc, int cells) {
    return kCsrDense / nc / nl < cells ? kCsrDense / nc / nl : cells;
}

// The element tensor is component-blocked ((c, a) -> c * n + a); the global
// index of local dof (c, a) is dof(a) * NC + c. CELLS: cells per run, such
// that a run of a mesh in spatial order has at most kCsrDense / NC dofs; a run
// that has more is taken in parts of SAFE cells, which cannot. (CELLS as an
// argument of the kernel: elasticity on P1 and P2 triangles 3% slower.)
template <typename T, int NL, int NC, int CELLS>
__global__ __launch_bounds__(kCsrThreads, 8) void k_scatter_csr(const T* __restrict__ A, const int32_t* __restrict__ c2d,
                                                            int64_t ncells, const int64_t* __restrict__ row_ptr,
                                                            const int32_t* __restrict__ col_idx,
                                                            T* __restrict__ values) {
    constexpr int N = NL * NC, UMAX = kCsrDense / NC, SAFE = csr_safe(NL, NC, CELLS);
    static_assert(SAFE >= 1 && CELLS * NL <= kCsrThreads && 2 * CELLS * NL <= kCsrHash, "run too long");
    constexpr int PL = (CELLS * N * NL + kCsrThreads - 1) / kCsrThreads;        // entry groups of a thread
    constexpr int GROUPS = kCsrThreads / 16, RL = (kCsrDense + GROUPS - 1) / GROUPS;  // rows of a lane group
    __shared__ T dense[kCsrDense * kCsrDense];
    __shared__ int32_t hkey[kCsrHash];    // dof, or -1
    __shared__ uint8_t hnum[kCsrHash];    // its number
    __shared__ int32_t udof[UMAX];        // dofs by number
    __shared__ int64_t ustart[UMAX * NC]; // their matrix rows
    __shared__ int32_t ulen[UMAX * NC];
    __shared__ uint8_t lnum[CELLS * NL];  // local dof -> number
    __shared__ int nuniq;
    const int tid = threadIdx.x, lane = tid & 15;
    // consecutive runs on one XCD: the rows they share stay in its L2
    const int64_t G = gridDim.x, b = blockIdx.x;
    const int64_t run = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
    const int64_t e1 = (run + 1) * CELLS < ncells ? (run + 1) * CELLS : ncells;
    int step = CELLS;
    for (int64_t e0 = run * CELLS; e0 < e1;) {
        const int m = e1 - e0 < step ? (int)(e1 - e0) : step;
        const int nd = m * NL, np = m * N * NL;
        // local dofs and tensor entries: all loads at once
        const int32_t mydof = c2d[e0 * NL + (tid < nd ? tid : 0)];
        const T* Ar = A + e0 * (N * N);
        T v[PL][NC];
#pragma unroll
        for (int k = 0; k < PL; ++k) {
            const int q = tid + k * kCsrThreads, p = q < np ? q : 0, r = p / NL, aj = p - r * NL;
#pragma unroll
            for (int cj = 0; cj < NC; ++cj) v[k][cj] = Ar[r * N + cj * NL + aj];
        }
        for (int i = tid; i < kCsrHash; i += kCsrThreads) hkey[i] = -1;
        if (tid == 0) nuniq = 0;
        int64_t rp[NC + 1];  // the matrix rows of this thread's dof
#pragma unroll
        for (int c = 0; c <= NC; ++c) rp[c] = row_ptr[(int64_t)mydof * NC + c];
        __syncthreads();
        int h = (int)(((uint32_t)mydof * 2654435761u) >> 22);
        if (tid < nd) {
            int old;
            for (;;) {  // ends: fewer dofs than slots
                old = atomicCAS(&hkey[h], -1, mydof);
                if (old == -1 || old == mydof) break;
                h = (h + 1) & (kCsrHash - 1);
            }
            if (old == -1) {
                const int u = atomicAdd(&nuniq, 1);
                if (u < UMAX) {
                    hnum[h] = (uint8_t)u;
                    udof[u] = mydof;
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const int64_t n1 = rp[c + 1] - rp[c];  // a row outside the pattern has none
                        ustart[u * NC + c] = rp[c];
                        ulen[u * NC + c] = n1 < INT32_MAX ? (int)n1 : INT32_MAX;
                    }
                }
            }
        }
        __syncthreads();
        const int nu = nuniq;
        if (nu > UMAX) {  // uniform; cannot happen with m <= SAFE
            step = SAFE;
            __syncthreads();
            continue;
        }
        const int W = nu * NC;  // rows and columns of the dense matrix
        if (tid < nd) lnum[tid] = hnum[h];
        for (int i = tid; i < W * W; i += kCsrThreads) dense[i] = T(0);
        // first columns of this lane group's matrix rows (long rows: later)
        int64_t b0[RL];
        int len[RL];
        bool more = false;
        int32_t x[RL][kCsrAhead];
#pragma unroll
        for (int k = 0; k < RL; ++k) {
            const int r = (tid >> 4) + k * GROUPS;
            b0[k] = r < W ? ustart[r] : 0;
            len[k] = r < W ? ulen[r] : 0;
            if (len[k] > kCsrLong) {
                len[k] = 0;
                more = true;
            }
        }
#pragma unroll
        for (int k = 0; k < RL; ++k)
#pragma unroll
            for (int j = 0; j < kCsrAhead; ++j) {
                x[k][j] = -1;
                if (lane + 16 * j < len[k]) x[k][j] = col_idx[b0[k] + lane + 16 * j];
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PL; ++k) {
            const int p = tid + k * kCsrThreads;
            if (p < np) {
                const int r = p / NL, aj = p - r * NL, c = r / N, i = r - c * N, ci = i / NL, ai = i - ci * NL;
                T* at = dense + (lnum[c * NL + ai] * NC + ci) * W + lnum[c * NL + aj] * NC;
#pragma unroll
                for (int cj = 0; cj < NC; ++cj) atomicAdd(at + cj, v[k][cj]);
            }
        }
        __syncthreads();
        auto add = [&](int r, int64_t at, int32_t col) {
            const int32_t dof = col / NC;
            int g = (int)(((uint32_t)dof * 2654435761u) >> 22);
            int32_t key = hkey[g];
            while (key != dof && key != -1) {  // ends: the hash has free slots
                g = (g + 1) & (kCsrHash - 1);
                key = hkey[g];
            }
            if (key != dof) return;  // no cell of the run has this column
            const T s = dense[r * W + hnum[g] * NC + col % NC];
            if (s != T(0)) atomicAdd(&values[at], s);  // also true for NaN
        };
#pragma unroll
        for (int k = 0; k < RL; ++k) {
            const int r = (tid >> 4) + k * GROUPS;
#pragma unroll
            for (int j = 0; j < kCsrAhead; ++j)
                if (lane + 16 * j < len[k]) add(r, b0[k] + lane + 16 * j, x[k][j]);
            for (int i = lane + 16 * kCsrAhead; i < len[k]; i += 16) add(r, b0[k] + i, col_idx[b0[k] + i]);
        }
        if (more) {
#pragma unroll 1
            for (int r = tid >> 4; r < W; r += GROUPS) {
                const int n = ulen[r];
                const int64_t at = ustart[r];
                if (n <= kCsrLong) continue;
                // the run's columns, searched in the row
                for (int j = lane; j < W; j += 16) {
                    const T s = dense[r * W + j];
                    if (s == T(0)) continue;
                    const int32_t col = udof[j / NC] * NC + j % NC;
                    int lo = 0, hi = n - 1;
                    while (lo < hi) {  // first index with col_idx >= col
                        const int mid = lo + (hi - lo) / 2;
                        if (col_idx[at + mid] < col) lo = mid + 1;
                        else hi = mid;
                    }
                    if (col_idx[at + lo] == col) atomicAdd(&values[at + lo], s);
                }
            }
        }
        __syncthreads();
        e0 += m;
    }
}

}  // namespace dev

namespace {

constexpr int64_t kAlign = 256;
int64_t al(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

unsigned pair_bits(int64_t ndofs) {
    const unsigned __int128 m = (unsigned __int128)ndofs * (unsigned __int128)ndofs;
    unsigned b = 1;
    while (b < 64 && ((unsigned __int128)1 << b) < m) ++b;
    return b;
}

bool pattern_temp(int64_t npairs, int64_t ndofs, size_t* sort_bytes, size_t* scan_bytes) {
    *sort_bytes = *scan_bytes = 0;
    if (npairs == 0) return true;
    if (rocprim::radix_sort_keys(nullptr, *sort_bytes, (const uint64_t*)nullptr, (uint64_t*)nullptr, (size_t)npairs,
                                 0u, pair_bits(ndofs), (hipStream_t)0) != hipSuccess)
        return false;
    size_t a = 0, b = 0;
    if (rocprim::exclusive_scan(nullptr, a, (const int32_t*)nullptr, (int64_t*)nullptr, (int64_t)0, (size_t)npairs,
                                rocprim::plus<int64_t>(), (hipStream_t)0) != hipSuccess)
        return false;
    if (rocprim::exclusive_scan(nullptr, b, (const int64_t*)nullptr, (int64_t*)nullptr, (int64_t)0,
                                (size_t)(ndofs + 1), rocprim::plus<int64_t>(), (hipStream_t)0) != hipSuccess)
        return false;
    *scan_bytes = std::max(a, b);
    return true;
}

struct PatternWs {
    uint64_t *keys, *skeys;
    int32_t *flag, *scol;
    int64_t *pos, *rowcnt, *srow;
    void* temp;
    int64_t bytes;
};

bool pattern_layout(int64_t ncells, int nloc, int64_t ndofs, char* base, PatternWs* w) {
    const int64_t np = ncells * nloc * nloc;
    size_t sb = 0, scb = 0;
    if (!pattern_temp(np, ndofs, &sb, &scb)) return false;
    int64_t o = 0;
    auto take = [&](int64_t n) { char* p = base ? base + o : nullptr; o += al(n); return p; };
    w->keys = (uint64_t*)take(np * 8);
    w->skeys = (uint64_t*)take(np * 8);
    w->flag = (int32_t*)take(np * 4);
    w->pos = (int64_t*)take(np * 8);
    w->scol = (int32_t*)take(np * 4);
    w->rowcnt = (int64_t*)take((ndofs + 1) * 8);
    w->srow = (int64_t*)take((ndofs + 1) * 8);
    w->temp = take((int64_t)std::max(sb, scb));
    w->bytes = o;
    return true;
}

int grid_of(int64_t work) { return (int)std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, 16384)); }

}  // namespace

}  // namespace coffee

using namespace coffee;

extern "C" int64_t coffee_csr_pattern_workspace_size(int64_t ncells, int nloc, int64_t ndofs) {
    if (ncells < 0 || nloc < 1 || nloc > kMaxN || ndofs < 1 || ndofs > INT32_MAX) return -1;
    PatternWs w;
    if (!pattern_layout(ncells, nloc, ndofs, nullptr, &w)) return -1;
    return w.bytes;
}

extern "C" coffee_status coffee_csr_pattern(const int32_t* cell_to_dof, int64_t ncells, int nloc, int64_t ndofs,
                                            int ncomp, int64_t* row_ptr, int32_t* col_idx, int64_t col_capacity,
                                            int64_t* nnz, void* workspace, int64_t workspace_bytes,
                                            void* hip_stream) {
    if (!nnz || ncells < 0 || nloc < 1 || nloc > kMaxN || ndofs < 1 || ndofs > INT32_MAX || ncomp < 1 || ncomp > 3)
        return COFFEE_E_INVALID_ARG;
    if ((int64_t)ndofs * ncomp > INT32_MAX) return COFFEE_E_UNSUPPORTED;
    if (!row_ptr || (ncells > 0 && (!cell_to_dof || !workspace))) return COFFEE_E_INVALID_ARG;
    if (((uintptr_t)workspace & 255) != 0) return COFFEE_E_INVALID_ARG;
    PatternWs w;
    if (!pattern_layout(ncells, nloc, ndofs, (char*)workspace, &w)) return COFFEE_E_HIP;
    if (ncells > 0 && workspace_bytes < w.bytes) return COFFEE_E_BUFFER_TOO_SMALL;
    hipStream_t s = (hipStream_t)hip_stream;
    const int64_t np = ncells * nloc * nloc;
    int64_t nscal = 0;
    if (np > 0) {
        hipLaunchKernelGGL(dev::k_pair_keys, dim3(grid_of(np)), dim3(256), 0, s, cell_to_dof, ncells, nloc,
                           (uint64_t)ndofs, w.keys);
        size_t sb = 0, scb = 0;
        pattern_temp(np, ndofs, &sb, &scb);
        if (rocprim::radix_sort_keys(w.temp, sb, w.keys, w.skeys, (size_t)np, 0u, pair_bits(ndofs), s) != hipSuccess)
            return COFFEE_E_HIP;
        hipLaunchKernelGGL(dev::k_run_heads, dim3(grid_of(np)), dim3(256), 0, s, w.skeys, np, w.flag);
        if (rocprim::exclusive_scan(w.temp, scb, w.flag, w.pos, (int64_t)0, (size_t)np, rocprim::plus<int64_t>(), s) !=
            hipSuccess)
            return COFFEE_E_HIP;
        hipLaunchKernelGGL(dev::k_zero<int64_t>, dim3(grid_of(ndofs + 1)), dim3(256), 0, s, w.rowcnt, ndofs + 1);
        hipLaunchKernelGGL(dev::k_compact, dim3(grid_of(np)), dim3(256), 0, s, w.skeys, w.flag, w.pos, np,
                           (uint64_t)ndofs, w.scol, w.rowcnt);
        if (rocprim::exclusive_scan(w.temp, scb, w.rowcnt, w.srow, (int64_t)0, (size_t)(ndofs + 1),
                                    rocprim::plus<int64_t>(), s) != hipSuccess)
            return COFFEE_E_HIP;
        if (hipMemcpyAsync(&nscal, w.srow + ndofs, sizeof(int64_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return COFFEE_E_HIP;
    }
    const int64_t total = nscal * ncomp * ncomp;
    *nnz = total;
    if (!col_idx || col_capacity < total) return COFFEE_E_BUFFER_TOO_SMALL;
    if (np == 0) {
        hipLaunchKernelGGL(dev::k_zero<int64_t>, dim3(grid_of(ndofs * ncomp + 1)), dim3(256), 0, s, row_ptr,
                           ndofs * ncomp + 1);
    } else {
        hipLaunchKernelGGL(dev::k_expand, dim3(grid_of(ndofs)), dim3(256), 0, s, w.srow, w.scol, ndofs, ncomp, row_ptr,
                           col_idx);
    }
    return hipGetLastError() == hipSuccess ? COFFEE_OK : COFFEE_E_HIP;
}

namespace {

// chunk of cells assembled into the workspace at a time
constexpr int64_t kCsrChunk = 1 << 17;

template <typename T, int NL, int NC, int CELLS>
void scatter_runs(const T* A, const int32_t* map, int64_t ncells, const int64_t* row_ptr, const int32_t* col_idx,
                  T* values, hipStream_t s) {
    const int64_t runs = (ncells + CELLS - 1) / CELLS;
    hipLaunchKernelGGL((dev::k_scatter_csr<T, NL, NC, CELLS>), dim3((unsigned)((runs + 7) / 8 * 8)),
                       dim3(dev::kCsrThreads), 0, s, A, map, ncells, row_ptr, col_idx, values);
}

// The shortest runs that are all resident at once (two workgroups per CU), of
// SAFE cells, which fit the LDS matrix in any order of the cells, of half the
// long runs' cells, and else of CELLS: a small mesh has too few long runs for
// the CUs, and a long run of scattered cells is taken in parts, one after the
// other. Mass matrices FP64, the whole call in a graph, us, runs of SAFE / half
// / CELLS (one thread per tensor row): P1 tetrahedra in mesh order, 12,001
// cells, 13.3 / 11.9 / 12.4 (17.1), 20,007 15.0 / 13.0 / 13.6 (22.8); in random
// order 17.7 / 19.4 / 26.8 (20.8) and 21.0 / 22.0 / 28.8 (28.0); Helmholtz,
// 1,293 cells, SAFE / CELLS 9.0 / 10.0 and 10.1 / 21.6 (13.0); P1 triangles,
// 20,007, 13.0 / 11.6 / 12.0 (14.1) and 16.4 / 16.5 / 19.0 (17.6). Beyond, P1
// triangles in random order are near one thread per tensor row: 24,003 cells
// 20.9 (19.9), 50,003 31.5 (30.2).
template <typename T, int NL, int NC, int CELLS>
bool scatter_launch(const T* A, const int32_t* map, int64_t ncells, const int64_t* row_ptr, const int32_t* col_idx,
                    T* values, hipStream_t s) {
    constexpr int SAFE = dev::csr_safe(NL, NC, CELLS);
    constexpr int MID = CELLS / 2 > SAFE ? CELLS / 2 : SAFE;
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return false;
    const int64_t resident = 2 * num_cu(device);  // workgroups
    if (ncells <= SAFE * resident)
        scatter_runs<T, NL, NC, SAFE>(A, map, ncells, row_ptr, col_idx, values, s);
    else if (MID > SAFE && ncells <= MID * resident)
        scatter_runs<T, NL, NC, MID>(A, map, ncells, row_ptr, col_idx, values, s);
    else
        scatter_runs<T, NL, NC, CELLS>(A, map, ncells, row_ptr, col_idx, values, s);
    return true;
}

// Cells per run: as many as have at most 90 / nc dofs on a mesh in spatial
// order (s squares of two triangles, cubes of six tetrahedra or stacked prisms
// in a row have (p s + 1)(p + 1), (p s + 1)(p + 1)^2 and (p s + 1) n_tri dofs).
template <typename T>
bool scatter_csr(int cell, int n, int nc, const T* A, const int32_t* map, int64_t ncells, const int64_t* row_ptr,
                 const int32_t* col_idx, T* values, hipStream_t s) {
#define COFFEE_SCATTER(NL, NC, CELLS) \
    if (n == NL && nc == NC) return scatter_launch<T, NL, NC, CELLS>(A, map, ncells, row_ptr, col_idx, values, s)
    if (cell == COFFEE_TRIANGLE) {
        COFFEE_SCATTER(3, 1, 86);
        COFFEE_SCATTER(6, 1, 28);
        COFFEE_SCATTER(10, 1, 14);
        COFFEE_SCATTER(15, 1, 6);
        COFFEE_SCATTER(3, 2, 42);
        COFFEE_SCATTER(6, 2, 14);
        COFFEE_SCATTER(10, 2, 6);
    } else if (cell == COFFEE_TETRAHEDRON) {
        COFFEE_SCATTER(4, 1, 114);
        COFFEE_SCATTER(10, 1, 20);
        COFFEE_SCATTER(20, 1, 6);
        COFFEE_SCATTER(35, 1, 2);
        COFFEE_SCATTER(4, 3, 30);
        COFFEE_SCATTER(10, 3, 6);
        COFFEE_SCATTER(20, 3, 1);
    } else {
        COFFEE_SCATTER(6, 1, 28);
        COFFEE_SCATTER(18, 1, 7);
        COFFEE_SCATTER(40, 1, 2);
    }
#undef COFFEE_SCATTER
    return false;  // no engine assembles another space
}

}  // namespace

extern "C" int64_t coffee_assemble_csr_workspace_size(int form, int cell, int degree, int precision, int64_t ncells) {
    const int N = coffee_tensor_dim(form, cell, degree);
    if (N <= 0 || ncells < 0 || precision < COFFEE_FP64 || precision > COFFEE_BF16X3) return -1;
    const int64_t chunk = std::min<int64_t>(ncells, kCsrChunk);
    return al(chunk * N * N * (precision == COFFEE_FP64 ? 8 : 4));
}

extern "C" coffee_status coffee_assemble_csr(int form, int cell, int degree, int quad_degree, int precision,
                                             const double* coords, int64_t nvert, const int32_t* c2v,
                                             int64_t ncells, const coffee_field* coeffs, int ncoeff,
                                             const double* constants, int nconst, const int32_t* cell_to_dof,
                                             int64_t ndofs, const int64_t* row_ptr, const int32_t* col_idx,
                                             int64_t nnz, void* values, void* workspace, int64_t workspace_bytes,
                                             void* hip_stream) {
    if (form == COFFEE_SVK_ENERGY || form == COFFEE_SVK_RESIDUAL) return COFFEE_E_UNSUPPORTED;
    const int N = coffee_tensor_dim(form, cell, degree);
    if (N <= 0) return COFFEE_E_INVALID_ARG;
    const int n = cell_nscalar(cell, degree), nc = N / n;
    if (degree > 1 && !cell_to_dof) return COFFEE_E_INVALID_ARG;  // P1: the vertices are the dofs
    const int32_t* map = cell_to_dof ? cell_to_dof : c2v;
    if (ndofs < 1 || nnz < 0 || (nnz > 0 && (!row_ptr || !col_idx || !values))) return COFFEE_E_INVALID_ARG;
    const int64_t need = coffee_assemble_csr_workspace_size(form, cell, degree, precision, ncells);
    if (need < 0) return COFFEE_E_INVALID_ARG;
    if (ncells > 0 && (!workspace || workspace_bytes < need)) return workspace ? COFFEE_E_BUFFER_TOO_SMALL
                                                                               : COFFEE_E_INVALID_ARG;
    if (((uintptr_t)workspace & 15) != 0) return COFFEE_E_INVALID_ARG;
    if (ncoeff < 0 || ncoeff > 2 || (ncoeff > 0 && !coeffs)) return COFFEE_E_INVALID_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    const bool f64 = precision == COFFEE_FP64;
    if (nnz > 0) {
        if (f64) hipLaunchKernelGGL(dev::k_zero<double>, dim3(grid_of(nnz)), dim3(256), 0, s, (double*)values, nnz);
        else hipLaunchKernelGGL(dev::k_zero<float>, dim3(grid_of(nnz)), dim3(256), 0, s, (float*)values, nnz);
    }
    coffee_field fl[2];
    for (int64_t e0 = 0; e0 < ncells; e0 += kCsrChunk) {
        const int64_t m = std::min<int64_t>(kCsrChunk, ncells - e0);
        for (int i = 0; i < ncoeff; ++i) {
            // the chunk's cells: offset the dof map, or the cell-major values
            fl[i] = coeffs[i];
            const int64_t nl = cell_nscalar(cell, coeffs[i].degree);
            if (coeffs[i].cell_to_dof) fl[i].cell_to_dof = coeffs[i].cell_to_dof + e0 * nl;
            else if (coeffs[i].values) fl[i].values = coeffs[i].values + e0 * nl * coeffs[i].ncomp;
        }
        coffee_status st = coffee_assemble(form, cell, degree, quad_degree, precision, coords, nvert,
                                           c2v + e0 * cell_nverts(cell), m, fl, ncoeff, constants, nconst, workspace,
                                           hip_stream);
        if (st != COFFEE_OK) return st;
        const bool ok = f64 ? scatter_csr<double>(cell, n, nc, (const double*)workspace, map + e0 * n, m, row_ptr, col_idx,
                                                  (double*)values, s)
                            : scatter_csr<float>(cell, n, nc, (const float*)workspace, map + e0 * n, m, row_ptr, col_idx,
                                                 (float*)values, s);
        if (!ok || hipGetLastError() != hipSuccess) return COFFEE_E_HIP;
    }
    return COFFEE_OK;
}
