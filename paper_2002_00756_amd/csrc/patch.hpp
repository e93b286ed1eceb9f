// One leg of the V-cycle on a small level in one launch (gfx950, wave64).
//
// A level of a few thousand columns cannot fill the GPU: each of its sweeps
// and its residual restriction is bound by launch and memory latency (4 to
// 8 us for less than 1 us of traffic), and they depend on each other only
// through neighbouring columns. Here a workgroup owns a small block of columns
// ("patch") and runs a whole leg on it:
//   kDown    sweep from zero, plain sweep, residual and restriction;
//   kUp      prolongation, two plain sweeps;
//   kCoarse  all sweeps of the coarsest level, from zero.
// What a sweep needs from other patches it computes itself: the first sweep of
// a leg also runs on the rings of columns around the patch (ring r: the
// columns r steps away), each later one on one ring less. Columns are listed
// per patch, the patch's own first, then ring by ring, so a sweep runs on a
// prefix of the list; the lists come from the neighbour table and hold panel
// edges and cube corners without special cases. The iterate stays in LDS.
//
// These levels hold a second copy of their coefficients, column by column (the
// W and S faces as planes of their own), and their vectors between two such
// levels are stored column by column as well (element (k, c) at c nz + k): a
// patch with its rings is a scattered set of columns, and of a 128-byte line of
// a tile row it would use a quarter or less (with tiles a down leg on C24 x 70
// moved about 700 KB per workgroup into L1 for 100 KB of values, 19.9 us).
// In LDS a column's rows stand in the order of the column solve ("places": the
// rows above mid downwards, mid, the rows below it upwards, see ColumnPlaces),
// each half padded to HMAX rows with r = 0, cc = 1, which pass the recurrences
// on unchanged. Both halves are then walked by the same straight-line code with
// all reads issued ahead (with a loop and tests of the row count a walk took 60
// cycles a row). The coefficients stand in the same order in memory, pads
// included. A thread owns pairs of places of one column, 16 places apart, so
// its addresses are one base plus constants and a wave reads 64- (float32) or
// 128-byte runs (dealing single elements to threads cost 100 instructions of
// index arithmetic per element and sweep; single places 8 apart fetched each
// line up to four times).
//
// Measured (V-cycle entry point, kernel by kernel with conversion passes against
// patches, us): C12 x 10 float64 64 / 30, C24 x 30 float32 90 / 45, C64 x 30 124 /
// 70, C192 x 70 (C24, C12 and C6 on patches) 738 / 667. A leg takes 5 to 12 us, of
// which 2 are the launch, 1 to 2 the first loads and 0.8 to 1.5 each sweep.
//
// Every value is formed by the operations of k_sweep and k_resid_restrict in
// their order (fused multiply-adds written out as the compiler forms them
// there), so the results are the same bits, infinities and NaN among them.
#pragma once
#include "columns.hpp"

namespace hh {

enum PatchLeg { kDown = 0, kUp = 1, kCoarse = 2 };
enum PatchLayout { kTiled = 0, kByColumn = 1, kAbi = 2 };

constexpr int kPatchCounts = 8;  // per patch: columns through ring 0, 1, 2, 3; own width

// Planes of the column-by-column coefficients.
enum { kColE = 0, kColW, kColN, kColS, kColM, kColC, kColD, kColV, kColX, kColPlanes };
// (kColM mm, kColC cc, kColD delta, kColV kv, kColX kv2 or s)

template <typename T>
struct PatchView {
    const int32_t* __restrict__ col;     // [npatch][ncp] columns, own first, then by ring
    const uint32_t* __restrict__ lnb;    // [npatch][ncp] E, W, N, S neighbours' places, a byte each
    const int32_t* __restrict__ par;     // [npatch][ncp] parents of col (not on the coarsest)
    const int32_t* __restrict__ cnt;     // [npatch][kPatchCounts]
    const T* __restrict__ co;            // [kColPlanes][ncol][8 JMAX] coefficients by place
    int npatch;
};

constexpr int kPatchLanes = 8;  // threads of one column

// Compiled patch sizes: own columns, rings, columns with all rings.
struct PatchShape {
    int pw, ph, depth, ncp;
    constexpr int threads() const { return (ncp * kPatchLanes + 63) / 64 * 64; }
};
constexpr PatchShape kPatchShapes[] = {
    {2, 2, 2, 24}, {4, 4, 2, 52}, {2, 2, 3, 40}, {4, 4, 3, 76}, {8, 4, 2, 84}};
constexpr int kPatchKinds = int(sizeof(kPatchShapes) / sizeof(kPatchShapes[0]));

// Levels per thread that are compiled for: every thread works on JMAX places
// without range tests (a test per place splits the loop into blocks that each
// wait for LDS).
constexpr int patch_levels(int nz, bool seven_point) {
    const int jn = (nz + kPatchLanes - 1) / kPatchLanes;
    const int sizes[] = {2, 4, 6, 8, 10, 16};
    for (int j : sizes)
        if (jn <= j && (seven_point || (j != 2 && j != 8))) return j;
    return 0;
}

// Deepest column that a patch size is taken for: beyond it a thread's values
// spill, and the legs lose to single kernels even where every workgroup has a CU
// (V-cycles take, times as long on patches: coarsest level C14 x 100 float32 1.34,
// C14 x 64 9-cell float64 3.1; C28 x 60 9-cell float32 1.19, float64 1.03).
template <typename T>
constexpr int patch_deepest(int kind, bool nine) {
    constexpr bool f32 = sizeof(T) == 4;
    switch (kind) {
        case 0:
        case 2: return nine ? (f32 ? 80 : 48) : kNzMax;
        case 1: return nine ? (f32 ? 80 : 48) : (f32 ? kNzMax : 80);
        case 3: return nine ? 32 : (f32 ? 64 : 48);
        default: return nine ? (f32 ? 48 : 32) : (f32 ? 80 : 48);
    }
}

// The next smaller size compiled, 0 for the smallest.
constexpr int patch_below(int jmax, bool seven_point) {
    int below = 0;
    for (int nz = kPatchLanes; nz < kPatchLanes * jmax; nz += kPatchLanes)
        if (patch_levels(nz, seven_point) < jmax) below = patch_levels(nz, seven_point);
    return below;
}

// LDS stride of a column: an odd number of values, so that lanes on
// neighbouring columns read different banks.
constexpr int patch_stride(int jmax) { return kPatchLanes * jmax + 1; }

// A thread's j-th place, from its first one (twice its lane in the column) on.
constexpr int patch_place(int j) { return 2 * kPatchLanes * (j >> 1) + (j & 1); }

// Rows of a column of nz levels, split at row mid, in 8 JMAX places.
struct ColumnPlaces {
    int nz, mid;
    int HMAX;  // rows of a half, mid's place
    // place of level k
    __host__ __device__ int of(int k) const {
        return k < mid ? k : (k == mid ? HMAX : HMAX + nz - k);
    }
    // level at a place, -1 for a pad
    __host__ __device__ int level(int p) const {
        const int k = p <= HMAX ? p : HMAX + nz - p;
        return p == HMAX ? mid : ((p < HMAX ? k < mid : k > mid) ? k : -1);
    }
};

constexpr size_t kLdsBytes = size_t(160) << 10;  // LDS that one workgroup may take

// LDS of one workgroup: right-hand side, factor and iterate per place, two
// values and a table entry per column.
template <typename T>
constexpr size_t patch_lds_bytes(int ncp, int jmax) {
    return (3 * size_t(patch_stride(jmax)) * ncp + 2 * ncp) * sizeof(T) +
           size_t(ncp) * sizeof(int32_t);
}

// Whether a patch size is compiled for jmax levels per thread: some column that
// it is taken for needs that many, and its workgroup fits the LDS.
template <typename T>
constexpr bool patch_compiled(int kind, int jmax, bool nine, bool seven_point) {
    return patch_levels(patch_deepest<T>(kind, nine), seven_point) >= jmax &&
           patch_lds_bytes<T>(kPatchShapes[kind].ncp, jmax) <= kLdsBytes;
}

// Whether the couplings stay in registers from one sweep of a leg to the next
// (as far as that leaves the column solve its registers), or are read again;
// and whether the residual's values are read after the last column solve
// instead of before it.
template <typename T, int JMAX, bool K2>
constexpr bool kPatchHold = JMAX * (K2 ? 6 : 4) * int(sizeof(T) / 4) <= 64;
template <typename T, int JMAX>
constexpr bool kPatchLate = JMAX * int(sizeof(T) / 4) >= 16;

template <typename T>
struct PatchArgs {
    PatchView<T> P;
    int ncol, nz, nvp;
    const T* b;
    const T* x;   // kUp: the iterate after the down leg (column by column)
    const T* xc;  // kUp: the coarse correction
    T* y;         // the iterate after the leg (kDown: column by column)
    T* bc;        // kDown: the coarse right-hand side
    int nvp_c;
    int layout;  // of b (and y of kUp, kCoarse): PatchLayout
    int ccol;    // whether the coarse vectors are column by column
    const void* ext_b;  // kAbi: b and the result (float64 values if ext_wide)
    void* ext_y;
    int ext_wide;
    T omega;
    int batch;
    const int* active;
    int mid, nsweep;  // nsweep: sweeps of the coarsest level
    int om_first;     // kUp: see the first sweep's relaxation
    int rev;
};

// One lane's walk over half a column (the recurrences of walk in columns.hpp):
// HMAX rows from r and c on, upwards (ELIM: t_i = r_i + c_{i-1} t_{i-1}; returns
// c_last t_last, what row mid takes) or downwards (z_i = r_i + c_i z_{i+1}, with
// v in place of z_HMAX). The lower half (!top) has one row less: its last row
// is taken as a pad.
template <typename T, int HMAX, bool ELIM>
__device__ __forceinline__ T run_walk(T* r, const T* c, bool top, T v) {
    constexpr int CW = sizeof(T) == 4 ? 40 : 10;  // rows read ahead at once
    constexpr int NB = (HMAX + CW - 1) / CW;
    T rr[2][CW], cc[2][CW], carry = T(0);
    auto place = [](int i) { return ELIM ? i : HMAX - 1 - i; };  // of the i-th step
    auto read = [&](int n) {
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int i = place(n * CW + j);
            if (n * CW + j < HMAX) {
                rr[n & 1][j] = r[i];
                cc[n & 1][j] = c[i];
                if (i == HMAX - 1) {
                    rr[n & 1][j] = top ? rr[n & 1][j] : T(0);
                    cc[n & 1][j] = top ? cc[n & 1][j] : T(1);
                }
            }
        }
    };
    read(0);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        if (n + 1 < NB) read(n + 1);
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            if (n * CW + j < HMAX) {
                v = fused(ELIM ? carry : cc[n & 1][j], v, rr[n & 1][j]);
                carry = cc[n & 1][j];
                rr[n & 1][j] = v;
            }
        }
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int i = place(n * CW + j);
            if (n * CW + j < HMAX && i != HMAX - 1) r[i] = rr[n & 1][j];
            if (n * CW + j < HMAX && i == HMAX - 1 && top) r[i] = rr[n & 1][j];
        }
    }
    return carry * v;
}

template <typename T, int KIND, int JMAX, int LEG, bool K2, int SC>
__global__ void __launch_bounds__(kPatchShapes[KIND].threads()) k_patch(PatchArgs<T> A) {
    static_assert(!(K2 && SC != kSym), "the weighted operator has the 7-point stencil");
    static_assert(SC != kRowWT, "H^T forms s x inside its fluxes: kernel by kernel");
    constexpr int NCP = kPatchShapes[KIND].ncp, NT = kPatchShapes[KIND].threads();
    constexpr int OWN = kPatchShapes[KIND].pw * kPatchShapes[KIND].ph, KL = kPatchLanes;
    constexpr int BOT = (NCP + 63) / 64 * 64;
    static_assert(BOT + NCP <= NT, "two elimination lane groups must fit the workgroup");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int S = patch_stride(JMAX), P = KL * JMAX, HMAX = P / 2;
    const int nz = A.nz;
    const ColumnPlaces at{nz, A.mid, HMAX};
    T* R = reinterpret_cast<T*>(smem_raw);  // [NCP][S]: rhs, then t, u, z
    T* Cf = R + NCP * S;                    // [NCP][S]: cc
    T* X = Cf + NCP * S;                    // [NCP][S]: iterate
    T* E1 = X + NCP * S;                    // [NCP], [NCP]: what mid's row takes from each half
    T* E2 = E1 + NCP;
    int32_t* cols = reinterpret_cast<int32_t*>(E2 + NCP);  // [NCP] columns

    const int lb = xcd_remap(blockIdx.x, gridDim.x, A.rev);
    const int rhs = lb % A.batch, p = lb / A.batch;
    if (A.active && !A.active[rhs]) return;
    const int64_t nv = A.nvp;
    const int32_t* cn = A.P.cnt + p * kPatchCounts;
    // sweep i (0, 1, ...) of a leg runs on the columns through ring `last - i`
    const int nsweep = LEG == kCoarse ? A.nsweep : 2;
    const int last = LEG == kDown ? 2 : (LEG == kUp ? 1 : nsweep - 1);
    const int nAll = cn[LEG == kUp ? 2 : last];  // columns loaded
    // columns whose neighbours are read
    const int nNb = LEG == kUp ? cn[1] : (last > 0 ? cn[last - 1] : 0);
    const int tid = threadIdx.x;
    const int lq = tid / KL, pl = 2 * (tid % KL);  // column, first place
    const int c = lq < NCP ? A.P.col[p * NCP + lq] : 0;
    const uint32_t nb = lq < NCP ? A.P.lnb[p * NCP + lq] : 0;  // the neighbours' places
    const int par = LEG == kUp && lq < NCP ? A.P.par[p * NCP + lq] : 0;
    const T* b = A.b + rhs * nv;
    T* y = A.y + rhs * nv;
    // element e of an array, as a 32-bit byte offset from a base that is the
    // same for the whole workgroup
    auto load = [](const T* base, uint32_t e) -> T {
        return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                           e * uint32_t(sizeof(T)));
    };
    const size_t plane = size_t(A.ncol) * P;
    const uint32_t oc0 = uint32_t(c * P + pl);
    auto co = [&](int w, uint32_t e) -> T { return load(A.P.co + w * plane, e); };
    // the thread's places 2 i and 2 i + 1 of a plane
    auto pair = [&](int w, int i, T& v0, T& v1) {
        typedef T V2 __attribute__((ext_vector_type(2)));
        const V2 v = *reinterpret_cast<const V2*>(
            reinterpret_cast<const char*>(A.P.co + w * plane) +
            (oc0 + uint32_t(2 * KL * i)) * uint32_t(sizeof(T)));
        v0 = v.x;
        v1 = v.y;
    };
    // the level at the thread's place j (-1: a pad), and one to load from
    auto level = [&](int j) { return at.level(pl + patch_place(j)); };
    auto from = [&](int j) { return uint32_t(max(level(j), 0)); };
    // pads hold zero where a column solve starts and where it scales by the
    // pivots, whatever their neighbours hold (zero times an infinity is not).
    // Each half has more rows than half the next smaller size has places, which
    // leaves most places without a test; a mask of the thread's pads, held, took
    // 704-thread workgroups over the registers of two on a CU (down leg C48 x 30
    // float32 12.4 -> 16.2 us).
    constexpr int ROWS = KL * patch_below(JMAX, !K2 && SC == kSym) / 2;
    const int end = HMAX + nz - A.mid;  // first place below the last row
    auto row = [&](int j, T v) {
        const int q = patch_place(j);
        const bool top = q < HMAX && q + 2 * KL - 2 >= ROWS;  // may hold pads of that half
        const bool bottom = q + 2 * KL - 2 > HMAX + ROWS;
        bool pad = false;
        if (top) pad = q + 2 * KL - 2 < HMAX ? pl >= A.mid - q
                                              : uint32_t(pl - (A.mid - q)) < uint32_t(HMAX - A.mid);
        if (bottom) pad = pad || pl >= end - q;
        return pad ? T(0) : v;
    };
    const uint32_t o = uint32_t(c * nz);
    if (pl == 0 && lq < NCP) cols[lq] = c;
    T* Rq = R + lq * S + pl;
    T* Cq = Cf + lq * S + pl;
    T* Xq = X + lq * S + pl;
    const T* const XE = X + int(nb & 255u) * S + pl;
    const T* const XW = X + int((nb >> 8) & 255u) * S + pl;
    const T* const XN = X + int((nb >> 16) & 255u) * S + pl;
    const T* const XS = X + int(nb >> 24) * S + pl;

    // ---- what the leg reads per element -------------------------------------
    T vb[JMAX], mo[JMAX], vk[JMAX][4];
    T so[SC != kSym ? JMAX : 1];               // own row weight
    T k2u[K2 ? JMAX : 1], k2d[K2 ? JMAX : 1];  // kv2 at k and k - 2
    constexpr bool HOLD = kPatchHold<T, JMAX, K2>;
    auto load_b = [&]() {
        if (A.layout == kAbi && A.ext_wide) {
            const double* e = static_cast<const double*>(A.ext_b) +
                              rhs * (int64_t(nz) * A.ncol) + c;
#pragma unroll
            for (int j = 0; j < JMAX; ++j) vb[j] = T(e[from(j) * uint32_t(A.ncol)]);
            return;
        }
        const T* e = A.layout == kAbi
                         ? static_cast<const T*>(A.ext_b) + rhs * (int64_t(nz) * A.ncol) : b;
        const uint32_t ob = A.layout == kByColumn ? o
                            : (A.layout == kAbi ? uint32_t(c) : uint32_t(tile_base(c, nz)));
        const uint32_t sb = A.layout == kByColumn ? 1 : (A.layout == kAbi ? A.ncol : kTile);
#pragma unroll
        for (int j = 0; j < JMAX; ++j) vb[j] = load(e, ob + sb * from(j));
    };
    auto couplings = [&](int i) {  // of places 2 i and 2 i + 1
        pair(kColE, i, vk[2 * i][0], vk[2 * i + 1][0]);
        pair(kColW, i, vk[2 * i][1], vk[2 * i + 1][1]);
        pair(kColN, i, vk[2 * i][2], vk[2 * i + 1][2]);
        pair(kColS, i, vk[2 * i][3], vk[2 * i + 1][3]);
        if constexpr (K2) {
            pair(kColX, i, k2u[2 * i], k2u[2 * i + 1]);
#pragma unroll
            for (int j = 2 * i; j < 2 * i + 2; ++j)
                k2d[j] = co(kColX, uint32_t(c * P + at.of(max(level(j) - 2, 0))));
        }
    };
    auto load_couplings = [&](int n) {
        if (lq >= n) return;
#pragma unroll
        for (int i = 0; i < JMAX / 2; ++i) couplings(i);
    };
    if (lq < nAll) {
        T vc[JMAX];
        load_b();
        if constexpr (LEG == kUp) {
            const uint32_t oc = A.ccol ? par * nz : tile_base(par, nz), sc = A.ccol ? 1 : kTile;
            const T* x = A.x + rhs * nv;
            const T* xc = A.xc + rhs * int64_t(A.nvp_c);
            T vx[JMAX], vp[JMAX];
#pragma unroll
            for (int j = 0; j < JMAX; ++j) {
                vx[j] = load(x, o + from(j));
                vp[j] = load(xc, oc + sc * from(j));
            }
#pragma unroll
            for (int j = 0; j < JMAX; ++j) Xq[patch_place(j)] = vx[j] + vp[j];
        }
#pragma unroll
        for (int j = 0; j < JMAX; ++j) {
            if (j & 1) continue;
            pair(kColC, j >> 1, vc[j], vc[j + 1]);
            pair(kColM, j >> 1, mo[j], mo[j + 1]);
            if constexpr (SC != kSym) pair(kColX, j >> 1, so[j], so[j + 1]);
        }
        if constexpr (HOLD && LEG == kUp) load_couplings(nNb);
#pragma unroll
        for (int j = 0; j < JMAX; ++j) {
            Cq[patch_place(j)] = vc[j];
            vb[j] = row(j, vb[j]);
            if constexpr (SC == kRowW) vb[j] = vb[j] / so[j];
        }
    }

    // kDown: the residual; KR threads take the levels of one coarse cell
    constexpr int KR = NT / (OWN / 4), RMAX = LEG == kDown ? (P + KR - 1) / KR : 1;
    T rd[RMAX][4], rkv[RMAX][4], rkvd[RMAX][4], rkh[RMAX][8];
    T rx[RMAX][4], rxd[RMAX][4], ri4[RMAX][4];  // kv2 at k, k - 2, or s; sibling faces (H)
    const int rc = tid / KR, rk = tid % KR;
    const bool res = LEG == kDown && rc < (cn[0] >> 2);
    int cl[4] = {0, 0, 0, 0};  // the cell's children
    if (res) {
        const int w = cn[4], I = rc % (w >> 1), J = rc / (w >> 1);
        cl[0] = 2 * J * w + 2 * I;
        cl[1] = cl[0] + 1;
        cl[2] = cl[0] + w;
        cl[3] = cl[2] + 1;
    }
    auto load_residual = [&]() {
        if (!res) return;
        uint32_t oq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) oq[q] = uint32_t(cols[cl[q]] * P);
#pragma unroll
        for (int i = 0; i < RMAX; ++i) {
            // threads past the last level read it again
            const int kk = min(rk + i * KR, nz - 1);
            const uint32_t k = uint32_t(at.of(kk)), kd = uint32_t(at.of(max(kk - 1, 0))),
                           kd2 = uint32_t(at.of(max(kk - 2, 0)));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                rd[i][q] = co(kColD, oq[q] + k);
                rkv[i][q] = co(kColV, oq[q] + k);
                rkvd[i][q] = co(kColV, oq[q] + kd);
                if constexpr (K2 || SC == kRowW) rx[i][q] = co(kColX, oq[q] + k);
                if constexpr (K2) rxd[i][q] = co(kColX, oq[q] + kd2);
            }
            // outer faces, two per child: (W, S), (E, S), (W, N), (E, N)
            rkh[i][0] = co(kColW, oq[0] + k);
            rkh[i][1] = co(kColS, oq[0] + k);
            rkh[i][2] = co(kColE, oq[1] + k);
            rkh[i][3] = co(kColS, oq[1] + k);
            rkh[i][4] = co(kColW, oq[2] + k);
            rkh[i][5] = co(kColN, oq[2] + k);
            rkh[i][6] = co(kColE, oq[3] + k);
            rkh[i][7] = co(kColN, oq[3] + k);
            if constexpr (SC == kRowW) {
                ri4[i][0] = co(kColE, oq[0] + k);
                ri4[i][1] = co(kColE, oq[2] + k);
                ri4[i][2] = co(kColN, oq[0] + k);
                ri4[i][3] = co(kColN, oq[1] + k);
            }
        }
    };

    const T om = A.omega, om1 = T(1) - A.omega;
    // ---- sweeps ---------------------------------------------------------------
    for (int it = 0; it < nsweep; ++it) {
        const bool zero = LEG != kUp && it == 0;
        const int n = cn[last - it];
        if (!zero) __syncthreads();  // the iterate is complete
        if (lq < n) {
            T r[JMAX];
            if (zero) {
#pragma unroll
                for (int j = 0; j < JMAX; ++j) r[j] = vb[j];
            } else {
#pragma unroll
                for (int j = 0; j < JMAX; ++j) {
                    if constexpr (!HOLD) {
                        if (!(j & 1)) couplings(j >> 1);
                    }
                    T a = vk[j][1] * XW[patch_place(j)];
                    a = fused(vk[j][0], XE[patch_place(j)], a);
                    a = fused(vk[j][2], XN[patch_place(j)], a);
                    a = fused(vk[j][3], XS[patch_place(j)], a);
                    r[j] = vb[j] + a;
                    if constexpr (K2) {
                        const int k = level(j);
                        const T xu = X[lq * S + at.of(min(k + 2, nz - 1))];
                        const T xd = X[lq * S + at.of(max(k - 2, 0))];
                        T v2 = k + 2 < nz ? k2u[j] * xu : T(0);
                        v2 = k >= 2 ? fused(k2d[j], xd, v2) : v2;
                        r[j] += v2;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < JMAX; ++j) Rq[patch_place(j)] = zero ? r[j] : row(j, r[j]);
        }
        // what the next phases read from memory arrives during the solve
        if constexpr (HOLD && LEG != kUp) {
            if (zero) load_couplings(nNb);
        }
        if constexpr (LEG == kDown && !kPatchLate<T, JMAX>) {
            if (!zero) load_residual();
        }
        __syncthreads();
        // column solve (column_solve): eliminate towards row mid
        const bool top = tid < BOT;
        const int wq = top ? tid : tid - BOT;  // the column a walking lane takes
        const int wb = wq * S + (top ? 0 : HMAX + 1);
        if (wq < n) {
            const T e = run_walk<T, HMAX, true>(R + wb, Cf + wb, top, T(0));
            (top ? E1 : E2)[wq] = e;
        }
        __syncthreads();
        if (lq < n) {
            const T e = E1[lq] + E2[lq];
            T v[JMAX];
#pragma unroll
            for (int j = 0; j < JMAX; ++j) {
                v[j] = Rq[patch_place(j)];
                v[j] = row(j, mo[j] * (pl + patch_place(j) == HMAX ? v[j] + e : v[j]));
            }
#pragma unroll
            for (int j = 0; j < JMAX; ++j) Rq[patch_place(j)] = v[j];
        }
        __syncthreads();
        if (wq < n) run_walk<T, HMAX, false>(R + wb, Cf + wb, top, R[wq * S + HMAX]);
        __syncthreads();
        if (lq < n) {
            const bool store = it == nsweep - 1 && (LEG == kDown || A.layout == kByColumn) && lq < cn[0];
            T v[JMAX];
#pragma unroll
            for (int j = 0; j < JMAX; ++j) v[j] = Rq[patch_place(j)];
            if (zero) {
#pragma unroll
                for (int j = 0; j < JMAX; ++j) v[j] = om * v[j];
            } else if (LEG == kUp && it == 0 && A.om_first) {
                // k_sweep's float32 sweep with prolongation over deep columns
                // is compiled to round the other product of the two
#pragma unroll
                for (int j = 0; j < JMAX; ++j) v[j] = fused(om, v[j], om1 * Xq[patch_place(j)]);
            } else {
#pragma unroll
                for (int j = 0; j < JMAX; ++j) v[j] = fused(om1, Xq[patch_place(j)], om * v[j]);
            }
#pragma unroll
            for (int j = 0; j < JMAX; ++j) Xq[patch_place(j)] = v[j];
            if (store) {
#pragma unroll
                for (int j = 0; j < JMAX; ++j)
                    if (level(j) >= 0) y[o + from(j)] = v[j];
            }
        }
    }
    if constexpr (LEG != kDown) {
        if (A.layout == kByColumn) return;
        __syncthreads();
        T* const xt = static_cast<T*>(A.ext_y) + rhs * (int64_t(nz) * A.ncol);
        double* const xw = static_cast<double*>(A.ext_y) + rhs * (int64_t(nz) * A.ncol);
        for (int e = tid; e < OWN * nz; e += NT) {
            const int q = e % OWN, k = e / OWN;
            if (q >= cn[0]) continue;
            const T v = X[q * S + at.of(k)];
            if (A.layout == kTiled) y[tile_base(cols[q], nz) + kTile * k] = v;
            else if (A.ext_wide) xw[k * A.ncol + cols[q]] = double(v);
            else xt[k * A.ncol + cols[q]] = v;
        }
        return;
    }

    // ---- residual and restriction (k_resid_restrict) -----------------------
    // b of the own columns goes back into R (H holds b / s and reads b again)
    if (lq < cn[0]) {
        if constexpr (SC == kRowW) load_b();
#pragma unroll
        for (int j = 0; j < JMAX; ++j) Rq[patch_place(j)] = vb[j];
    }
    if constexpr (kPatchLate<T, JMAX>) load_residual();
    __syncthreads();
    if (!res) return;
    int out[8];  // the outer neighbours, as rkh
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t w = A.P.lnb[p * NCP + cl[q]];
        const uint32_t ew = (q & 1) ? w : w >> 8, ns = (q & 2) ? w >> 16 : w >> 24;
        out[2 * q] = int(ew & 255u) * S;
        out[2 * q + 1] = int(ns & 255u) * S;
    }
    const int C = A.P.par[p * NCP + cl[0]];
    T* const bc = A.bc + rhs * int64_t(A.nvp_c);
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
        const int k = rk + i * KR;
        if (k >= nz) break;
        const int p0 = at.of(k);
        auto val = [&](int kk, int q) -> T {
            const T v = X[cl[q] * S + at.of(min(max(kk, 0), nz - 1))];
            return kk >= 0 && kk < nz ? v : T(0);
        };
        if (k == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) rkvd[i][q] = T(0);
        }
        if constexpr (K2) {
            if (k < 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) rxd[i][q] = T(0);
            }
        }
        T xo[4], xup[4], xdn[4], vxo[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            xo[q] = val(k, q);
            xup[q] = val(k + 1, q);
            xdn[q] = val(k - 1, q);
        }
#pragma unroll
        for (int f = 0; f < 8; ++f) vxo[f] = X[out[f] + p0];
        T acc = ((R[cl[0] * S + p0] + R[cl[1] * S + p0]) + R[cl[2] * S + p0]) + R[cl[3] * S + p0];
        if constexpr (SC == kRowW) {
            T Lr[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                Lr[q] = fused(rkv[i][q], xo[q] - xup[q], rkvd[i][q] * (xo[q] - xdn[q]));
#pragma unroll
            for (int f = 0; f < 8; ++f)
                Lr[f >> 1] = fused(rkh[i][f], xo[f >> 1] - vxo[f], Lr[f >> 1]);
            Lr[0] += fused(ri4[i][0], xo[0] - xo[1], ri4[i][2] * (xo[0] - xo[2]));
            Lr[1] += fused(ri4[i][0], xo[1] - xo[0], ri4[i][3] * (xo[1] - xo[3]));
            Lr[2] += fused(ri4[i][1], xo[2] - xo[3], ri4[i][2] * (xo[2] - xo[0]));
            Lr[3] += fused(ri4[i][1], xo[3] - xo[2], ri4[i][3] * (xo[3] - xo[1]));
#pragma unroll
            for (int q = 0; q < 4; ++q) acc -= fused(rd[i][q], xo[q], rx[i][q] * Lr[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc = fused(-rd[i][q], xo[q], acc);
                acc -= fused(rkv[i][q], xo[q] - xup[q], rkvd[i][q] * (xo[q] - xdn[q]));
            }
#pragma unroll
            for (int f = 0; f < 8; ++f) acc = fused(-rkh[i][f], xo[f >> 1] - vxo[f], acc);
        }
        if constexpr (K2) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc -= fused(rx[i][q], xo[q] - val(k + 2, q),
                             rxd[i][q] * (xo[q] - val(k - 2, q)));
        }
        bc[A.ccol ? C * nz + k : tile_base(C, nz) + kTile * k] = acc;
    }
}

// Launch one leg with the compiled patch size `kind` (an index of
// kPatchShapes). Defined per precision in patch_f32.hip and patch_f64.hip.
template <typename T>
void launch_patch(int kind, int leg, bool nine, bool weighted, const PatchArgs<T>& A, hipStream_t s);

template <typename T, int KIND, int JMAX, int LEG, bool K2, int SC>
void launch_patch_one(const PatchArgs<T>& A, hipStream_t s) {
    constexpr PatchShape S = kPatchShapes[KIND];
    // (no other size is selected: patch_runs)
    if constexpr (patch_compiled<T>(KIND, JMAX, K2, !K2 && SC == kSym))
        hipLaunchKernelGGL((k_patch<T, KIND, JMAX, LEG, K2, SC>), dim3(A.P.npatch * A.batch),
                           dim3(S.threads()), patch_lds_bytes<T>(S.ncp, JMAX), s, A);
}

template <typename T, int KIND, int LEG, bool K2, int SC>
void launch_patch_j(const PatchArgs<T>& A, hipStream_t s) {
    constexpr bool seven_point = !K2 && SC == kSym;
    const int j = patch_levels(A.nz, seven_point);
    if constexpr (seven_point) {
        if (j == 2) return launch_patch_one<T, KIND, 2, LEG, K2, SC>(A, s);
        if (j == 8) return launch_patch_one<T, KIND, 8, LEG, K2, SC>(A, s);
    }
    if (j == 4) return launch_patch_one<T, KIND, 4, LEG, K2, SC>(A, s);
    if (j == 6) return launch_patch_one<T, KIND, 6, LEG, K2, SC>(A, s);
    if (j == 10) return launch_patch_one<T, KIND, 10, LEG, K2, SC>(A, s);
    launch_patch_one<T, KIND, 16, LEG, K2, SC>(A, s);
}

template <typename T, int KIND, int LEG>
void launch_patch_form(bool nine, bool weighted, const PatchArgs<T>& A, hipStream_t s) {
    if (nine) return launch_patch_j<T, KIND, LEG, true, kSym>(A, s);
    if (weighted) return launch_patch_j<T, KIND, LEG, false, kRowW>(A, s);
    launch_patch_j<T, KIND, LEG, false, kSym>(A, s);
}

template <typename T>
void launch_patch_impl(int kind, int leg, bool nine, bool weighted, const PatchArgs<T>& A,
                       hipStream_t s) {
#define HH_PATCH(K)                                                   \
    case K:                                                           \
        if constexpr (kPatchShapes[K].depth == 3)                     \
            return launch_patch_form<T, K, kCoarse>(nine, weighted, A, s);  \
        else if (leg == kDown)                                        \
            return launch_patch_form<T, K, kDown>(nine, weighted, A, s);    \
        else                                                          \
            return launch_patch_form<T, K, kUp>(nine, weighted, A, s);
    switch (kind) {
        HH_PATCH(0)
        HH_PATCH(1)
        HH_PATCH(2)
        HH_PATCH(3)
        HH_PATCH(4)
    }
#undef HH_PATCH
}

}  // namespace hh
