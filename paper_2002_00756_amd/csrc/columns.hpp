// Data layout and the column solve shared by the device kernels of the
// Helmholtz multigrid path (gfx950, wave64).
//
// Data layout in HBM, per multigrid level with ncol columns and nz levels.
// Columns are grouped into tiles of kTile = 32 consecutive columns, and every
// per-level array stores one tile after the other, each tile holding its nz
// levels as rows of 32 values:
//     element (k, c) sits at tile_base(c) + 32 k,
//     tile_base(c) = (c / 32) * 32 nz + c % 32.
// For storage ncol is rounded up to ncolp, a multiple of 32. nvp = nz * ncolp.
// The padding columns of the coefficients, of the Krylov vectors (r, p, q, z and
// BiCGStab's) and of the finest level's right-hand side and solution hold zeros:
// the workspace is cleared at set-up and no kernel writes them, so reductions over
// these may run over the padded length. The Jacobi partner t of every level and
// the right-hand side and solution of the coarser ones may hold anything there: the
// legs on patches store them column by column in the same memory (patch.hpp).
//   vectors        [batch][nvp]        tiled as above
//   kh             [2][nvp]            E-face plane, then N-face plane
//   kv             [nvp]               face k|k+1; row nz-1 is zero (no flux
//                                      through the top), so loads need no guard
//   dl (delta)     [nvp]
//   kv2            [nvp]               9-cell stencil only: coupling of levels
//                                      k and k+2; rows nz-2, nz-1 are zero
//   s              [nvp]               weighted operator only: row weight of
//                                      H = delta + S L (below)
//   cc, mm         [nvp]               factors of the column operator (below)
//   nbr            [4][ncol]           E, W, N, S neighbour column
//   fface          [2][ncol]           offset in kh of the W and S face at
//                                      level 0 (plane * nvp + tile_base(owner));
//                                      the E and N faces are at tile_base(c)
//                                      and nvp + tile_base(c)
//   pofs           [3][ncol]           tiled offsets on the next coarser level
//                                      of the parent of the column and of the
//                                      parents of its outward E/W and N/S
//                                      neighbours (prolongation)
// A workgroup that owns a tile reads one contiguous block of every array and
// a wave reads two adjacent rows of one tile. Vectors passed through the C ABI
// keep the natural [batch][nz][ncol] layout; the kernels that take them in or
// hand them out convert on the fly.
//
// Column factorisation. The smoother solves with the column operator Hz (the
// couplings between neighbouring levels of a column plus the full diagonal of
// H; Section 3.5, Eq. jacobi; with the 9-cell stencil the couplings two
// levels apart are dropped from it but stay in its diagonal, Section 3.6) by
// an LU factorisation computed once per operator (the paper stores the same
// factors; Section 3.8). Pivots are computed in a form free of cancellation:
// with s_k = delta_k + sum of the 4 horizontal couplings (+ kv2_k + kv2_{k-2}),
// the top-down pivot excess is e_0 = s_0, e_k = s_k + kv_{k-1} e_{k-1} /
// (e_{k-1} + kv_{k-1}), pivot p_k = e_k + kv_k. Stored: mm_k = 1/p_k and
// cc_k = kv_k / p_k, so that forward elimination is t_k = r_k + cc_{k-1} t_{k-1}
// and back substitution is z_k = mm_k t_k + cc_k z_{k+1}.
// Weighted operator H = delta + S L (S = diag(s), L the flux terms): its column
// matrix is S Hz' with Hz' = delta/s + (the column part of L) symmetric, so the
// factors are those of Hz' (delta/s in place of delta) and the sweeps scale
// by 1/s: forward, Hz^-1 (b + S sum K x_n) = Hz'^-1 (b/s + sum K x_n); for
// H^T = delta + L S, Hz^-T (b + sum K s_n x_n) = S^-1 Hz'^-1 (b + sum K s_n x_n).
// The smoother uses a "twisted" split at row mid = nz / 2: rows above mid
// are factored top-down as above, rows below mid bottom-up (f_{nz-1} =
// s_{nz-1}, f_k = s_k + kv_k f_{k+1} / (f_{k+1} + kv_k), q_k = f_k + kv_{k-1},
// mm_k = 1/q_k, cc_k = kv_{k-1}/q_k) and row mid with both neighbours
// eliminated, so two lanes per column share the sequential work.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace hh {

constexpr int kBlock = 256;

// Workgroups of one launch are handed to the 8 XCDs round-robin (bid -> XCD
// bid % 8). Renumber them so that each XCD works through one contiguous range
// of logical blocks: neighbouring tiles (the N/S neighbour rows, the batch
// members sharing coefficients) then meet in the same L2. rev: each XCD walks
// its range backwards. Consecutive kernels on a level alternate the direction,
// so that each starts on the data the previous one touched last, which the
// last-level cache still holds when a level's streams exceed it.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks, int rev = 0) {
    const int xcd = bid & 7, slot = bid >> 3;
    const int q = nblocks >> 3, r = nblocks & 7;
    const int cnt = q + (xcd < r ? 1 : 0);
    return xcd * q + (xcd < r ? xcd : r) + (rev ? cnt - 1 - slot : slot);
}

// Logical block of a launch without the XCD renumbering, walked backwards
// when rev is set.
__device__ __forceinline__ int logical_block(int rev) {
    return rev ? int(gridDim.x) - 1 - int(blockIdx.x) : int(blockIdx.x);
}

constexpr int kTile = 32;
constexpr int kNzMax = 120;  // deepest column the library takes

// Offset of element (0, c) of a tiled array; element (k, c) is 32 k further.
__device__ __forceinline__ int tile_base(int c, int nz) {
    return (c >> 5) * (kTile * nz) + (c & (kTile - 1));
}

template <typename T>
struct LevelView {
    int ncol, nz, nvp;
    int N;  // columns per panel edge (c = p N^2 + j N + i)
    const int32_t* __restrict__ nbr;
    const uint32_t* __restrict__ fface;
    // [3][ncol] on every level but the coarsest: tiled offsets on the next
    // coarser level of the column's parent and of the parents of its outward
    // E/W and N/S neighbours (the other two neighbours share its parent)
    const int32_t* __restrict__ pofs;
    const T* __restrict__ kh;
    const T* __restrict__ kv;
    const T* __restrict__ dl;
    const T* __restrict__ cc;
    const T* __restrict__ mm;
    const T* __restrict__ kv2;  // null for the 7-point stencil
    const T* __restrict__ s;    // row weight; null for the symmetric operator
};

// Loads and stores of a stream that the cache need not keep (NT: non-temporal).
template <bool NT, typename T>
__device__ __forceinline__ T stream_load(const T* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void stream_store(T* p, T v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) {
    return __builtin_fma(a, b, c);
}

// Operator form a kernel is built for: symmetric, row-weighted H = delta + S L,
// or its transpose H^T = delta + L S.
enum { kSym = 0, kRowW = 1, kRowWT = 2 };

// Phases 2-4 of the column solve z = Hz^-1 r for ncol columns held in LDS
// with row stride S: on entry R[k*S + col] holds r and Cf[k*S + col] the
// factor cc; the calling thread owns column lc (if lc < ncol) at levels
// kg + j KG, whose pivot reciprocals it holds in mo[j]. On exit R holds z.
// Two lanes per column (tid < ncol: rows above mid, top-down; BOT <= tid <
// BOT + ncol: rows below mid, bottom-up) walk the column, SEQ levels per LDS
// round trip; row mid combines both eliminations. E1, E2 hold ncol values.
//
// Each walk is a run of rows k = first + dir * i, i < count, with a
// first-order recurrence along it. Full batches of SEQ rows carry no range
// tests, so their SEQ reads issue together and the recurrence is a plain
// chain of fused multiply-adds; the last, partial batch reads row indices
// clamped into the run and tests only the arithmetic and the stores.
template <typename T, int SEQ, bool ELIM>
__device__ __forceinline__ T walk(T* R, const T* Cf, int S, int lane, int first, int dir,
                                  int count, T v, T& carry) {
    // ELIM: t_k = r_k + carry * t_prev, carry <- cf_k   (elimination; v = t)
    // else: z_k = r_k + cf_k * z_prev                     (substitution; v = z)
    int i0 = 0;
    for (; i0 + SEQ <= count; i0 += SEQ) {
        T rr[SEQ], cf[SEQ];
#pragma unroll
        for (int i = 0; i < SEQ; ++i) {
            const int k = first + dir * (i0 + i);
            rr[i] = R[k * S + lane];
            cf[i] = Cf[k * S + lane];
        }
#pragma unroll
        for (int i = 0; i < SEQ; ++i) {
            if (ELIM) {
                v = rr[i] + carry * v;
                carry = cf[i];
            } else {
                v = rr[i] + cf[i] * v;
            }
            rr[i] = v;
        }
#pragma unroll
        for (int i = 0; i < SEQ; ++i) R[(first + dir * (i0 + i)) * S + lane] = rr[i];
    }
    if (i0 < count) {
        const int last = count - 1;
        T rr[SEQ], cf[SEQ];
#pragma unroll
        for (int i = 0; i < SEQ; ++i) {
            const int k = first + dir * min(i0 + i, last);
            rr[i] = R[k * S + lane];
            cf[i] = Cf[k * S + lane];
        }
#pragma unroll
        for (int i = 0; i < SEQ; ++i) {
            if (i0 + i < count) {
                if (ELIM) {
                    v = rr[i] + carry * v;
                    carry = cf[i];
                } else {
                    v = rr[i] + cf[i] * v;
                }
                rr[i] = v;
            }
        }
#pragma unroll
        for (int i = 0; i < SEQ; ++i)
            if (i0 + i < count) R[(first + dir * (i0 + i)) * S + lane] = rr[i];
    }
    return v;
}

template <typename T, int JMAX>
__device__ __forceinline__ void column_solve(T* R, T* Cf, T* E1, T* E2, const T (&mo)[JMAX],
                                             int tid, int lc, int kg, int KG, int BOT, int mid,
                                             int nz, int S, int ncol) {
    constexpr int SEQ = 8;
    // ---- phase 2: eliminate towards row mid -------------------------------
    if (tid < ncol) {
        T cp = T(0);
        const T t = walk<T, SEQ, true>(R, Cf, S, tid, 0, 1, mid, T(0), cp);
        E1[tid] = cp * t;
    } else if (tid >= BOT && tid < BOT + ncol) {
        const int l2 = tid - BOT;
        T cn = T(0);
        const T t = walk<T, SEQ, true>(R, Cf, S, l2, nz - 1, -1, nz - 1 - mid, T(0), cn);
        E2[l2] = cn * t;
    }
    __syncthreads();

    // ---- phase 3: pivot reciprocals (row mid takes both eliminations) ------
    if (lc < ncol) {
#pragma unroll
        for (int j = 0; j < JMAX; ++j) {
            const int k = kg + j * KG;
            if (k < nz) {
                T v = R[k * S + lc];
                if (k == mid) v += E1[lc] + E2[lc];
                R[k * S + lc] = mo[j] * v;
            }
        }
    }
    __syncthreads();

    // ---- phase 4: back substitution outwards from row mid ----------------
    T unused = T(0);
    if (tid < ncol) {
        walk<T, SEQ, false>(R, Cf, S, tid, mid - 1, -1, mid, R[mid * S + tid], unused);
    } else if (tid >= BOT && tid < BOT + ncol) {
        const int l2 = tid - BOT;
        walk<T, SEQ, false>(R, Cf, S, l2, mid + 1, 1, nz - 1 - mid, R[mid * S + l2], unused);
    }
    __syncthreads();
}

}  // namespace hh
