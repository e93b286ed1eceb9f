// Set-up after the coarse coefficients: column factors, float32 copies and the
// small levels' column-by-column coefficients, for all levels of a hierarchy at
// once (gfx950, wave64).
#pragma once
#include "columns.hpp"
#include "patch.hpp"

namespace hh {

constexpr int kSetupLevels = 20;  // deepest hierarchy a configuration may ask for

// One level's arrays. cc, mm may be null (no float64 V-cycle), kv2 and s are
// for the 9-cell and the weighted operator, co64 and co32 for levels on patches.
struct SetupLevel {
    int ncol, nvp;
    int tile0;  // first workgroup of the level
    const uint32_t* fface;
    const double *kh, *kv, *dl, *kv2, *s;
    double *cc, *mm;
    float *kh32, *kv32, *dl32, *cc32, *mm32, *kv2_32, *s32;
    double* co64;
    float* co32;
};
struct SetupLevels {
    SetupLevel lev[kSetupLevels];
    int count;
    __device__ __forceinline__ int of(int block) const {
        int l = 0;
        while (l + 1 < count && block >= lev[l + 1].tile0) ++l;
        return l;
    }
};

// Column factors (columns.hpp) and float32 copies: one workgroup per tile of 32
// columns, the levels' tiles one after the other in one launch (the levels do
// not depend on each other here, and the small ones are all latency). The
// coefficients are read once, coalesced; only the pivot recurrence runs in two
// lanes per column, from LDS, and the divisions for the pivots themselves are
// spread over the workgroup. One thread per column reading its own levels and
// one launch per level, with a conversion pass per array, took 530 us for
// C144 x 50 with 5 levels.
__global__ void __launch_bounds__(kBlock)
k_factor_levels(const SetupLevels A, int nz, int mid) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* E = reinterpret_cast<double*>(smem_raw);  // [nz][32]: s, then the pivot excess
    double* V = E + nz * kTile;                       // [nz][32]: kv
    const SetupLevel& L = A.lev[A.of(blockIdx.x)];
    const int ncol = L.ncol;
    const int tid = threadIdx.x, lc = tid % kTile, g = tid / kTile;
    constexpr int KG = kBlock / kTile;
    const int c = (int(blockIdx.x) - L.tile0) * kTile + lc;
    const bool valid = c < ncol;
    const int ob = tile_base(c, nz);
    if (valid) {
        const uint32_t fW = L.fface[c], fS = L.fface[ncol + c];
        const double* khN = L.kh + L.nvp;
#pragma unroll 2
        for (int k = g; k < nz; k += KG) {
            const int r = kTile * k, o = ob + r;
            const double e = L.kh[o], w = L.kh[fW + uint32_t(r)], n = khN[o],
                         s = L.kh[fS + uint32_t(r)], d = L.dl[o], a = L.kv[o];
            // weighted operator: the factors are those of Hz' (delta / s)
            double v = (L.s ? d / L.s[o] : d) + e + w + n + s;
            // 9-cell: the dropped couplings two levels apart stay in the diagonal
            if (L.kv2) v += L.kv2[o] + (k >= 2 ? L.kv2[o - 2 * kTile] : 0.0);
            E[k * kTile + lc] = v;
            V[k * kTile + lc] = a;
            L.kh32[o] = float(e);
            L.kh32[L.nvp + o] = float(n);
            L.kv32[o] = float(a);
            L.dl32[o] = float(d);
            if (L.kv2) L.kv2_32[o] = float(L.kv2[o]);
            if (L.s) L.s32[o] = float(L.s[o]);
        }
    }
    __syncthreads();
    if (tid < kTile) {  // rows above mid, top-down
        double e = mid > 0 ? E[tid] : 0.0;
        for (int k = 1; k < mid; ++k) {
            const double a = V[(k - 1) * kTile + tid];
            e = E[k * kTile + tid] + a * e / (e + a);
            E[k * kTile + tid] = e;
        }
    } else if (tid >= 64 && tid < 64 + kTile) {  // rows below mid, bottom-up
        const int q = tid - 64;
        double f = E[(nz - 1) * kTile + q];
        for (int k = nz - 2; k > mid; --k) {
            const double a = V[k * kTile + q];
            f = E[k * kTile + q] + a * f / (f + a);
            E[k * kTile + q] = f;
        }
    }
    __syncthreads();
    if (!valid) return;
    for (int k = g; k < nz; k += KG) {
        double t = E[k * kTile + lc], m, cv;
        if (k == mid) {
            if (mid > 0) {
                const double a = V[(mid - 1) * kTile + lc], e = E[(mid - 1) * kTile + lc];
                t += a * e / (e + a);
            }
            if (mid < nz - 1) {
                const double a = V[mid * kTile + lc], f = E[(mid + 1) * kTile + lc];
                t += a * f / (f + a);
            }
            m = 1.0 / t;
            cv = 0.0;
        } else {
            const double a = V[(k < mid ? k : k - 1) * kTile + lc];
            m = 1.0 / (t + a);
            cv = a * m;
        }
        const int o = ob + kTile * k;
        if (L.mm) {
            L.mm[o] = m;
            L.cc[o] = cv;
        }
        L.mm32[o] = float(m);
        L.cc32[o] = float(cv);
    }
}

// Coefficients of the levels on patches, column by column (PatchView::co), P
// places a column, mid's at P / 2; the pads are zero, in cc (and s) one. One
// workgroup per tile of 32 columns and plane: the columns are one contiguous
// block of the plane, and rows turn into columns through LDS.
__global__ void __launch_bounds__(kBlock)
k_patch_coefficients(const SetupLevels A, int nz, int mid, int P) {
    __shared__ double buf[kTile][kNzMax + 1];
    const SetupLevel& L = A.lev[A.of(blockIdx.x)];
    const ColumnPlaces at{nz, mid, P / 2};
    const int ncol = L.ncol, plane = blockIdx.y;
    const int c0 = (int(blockIdx.x) - L.tile0) * kTile;
    const int lc = threadIdx.x % kTile, g = threadIdx.x / kTile, nc = min(kTile, ncol - c0);
    const int ob = tile_base(c0, nz) + lc;
    const double* src = nullptr;
    const float* src32 = nullptr;  // the factors of a handle without float64 ones
    if (lc < nc) {
        switch (plane) {
            case kColE: src = L.kh + ob; break;
            case kColW: src = L.kh + L.fface[c0 + lc]; break;
            case kColN: src = L.kh + L.nvp + ob; break;
            case kColS: src = L.kh + L.fface[ncol + c0 + lc]; break;
            case kColM: src32 = L.mm32 + ob; if (L.mm) src = L.mm + ob; break;
            case kColC: src32 = L.cc32 + ob; if (L.cc) src = L.cc + ob; break;
            case kColD: src = L.dl + ob; break;
            case kColV: src = L.kv + ob; break;
            default: src = L.kv2 ? L.kv2 + ob : (L.s ? L.s + ob : nullptr); break;
        }
        if (src || src32)
            for (int k = g; k < nz; k += kBlock / kTile)
                buf[lc][k] = src ? src[kTile * k] : double(src32[kTile * k]);
    }
    __syncthreads();
    const double pad = plane == kColC || (plane == kColX && L.s) ? 1.0 : 0.0;
    const int64_t dst = (int64_t(plane) * ncol + c0) * P;
    for (int e = threadIdx.x; e < nc * P; e += kBlock) {
        const int k = at.level(e % P);
        const double v = k < 0 ? pad : buf[e / P][k];
        if (L.co64) L.co64[dst + e] = v;
        if (L.co32) L.co32[dst + e] = float(v);
    }
}

}  // namespace hh
