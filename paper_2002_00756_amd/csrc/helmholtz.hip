// Host side of the C ABI declared in include/helmholtz.h: workspace layout,
// operator set-up, the V-cycle of Algorithm 1 and the conjugate-gradient
// loop, all as stream-ordered launches of the kernels in kernels.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "helmholtz.h"
#include "kernels.hpp"
#include "mesh.hpp"
#include "patch.hpp"
#include "setup.hpp"

using namespace hh;

namespace {

constexpr int kRedBlocks = 2048;  // partial sums per right-hand side for vector reductions
constexpr int kMaxLevels = kSetupLevels;
constexpr int kApplyChunk = 4;   // vertical levels per thread in apply / residual kernels
constexpr int kSmallSweepCols = 5000;  // levels below this use narrow sweep tiles

// Per-level arrays use the column-tile layout of the kernels (element (k, c)
// at tile_base(c) + 32 k, columns padded to ncolp, nvp = nz * ncolp).
template <typename T>
struct LevelData {
    T* kh = nullptr;  // [2][nvp]  E faces, N faces
    T* kv = nullptr;  // [nvp]
    T* dl = nullptr;  // [nvp]
    T* cc = nullptr;  // [nvp]
    T* mm = nullptr;  // [nvp]
    T* kv2 = nullptr; // [nvp]     9-cell stencil only
    T* s = nullptr;   // [nvp]     weighted operator only: row weight
    T* co = nullptr;  // [kColPlanes][ncol][places] column by column, small levels only
    T* b = nullptr;   // [B][nvp]   level >= 1 (and level 0 for float32)
    T* x = nullptr;   // [B][nvp]   level >= 1 (and level 0 for float32)
    T* t = nullptr;   // [B][nvp]   ping-pong partner of x
};

// The vectors one V-cycle works in, per level: right-hand side b, iterate x
// and its Jacobi ping-pong partner t. They come from the handle's workspace
// or, for the allocation-free entry point, from the static scratch array.
template <typename T>
struct VBufs {
    T* b[kMaxLevels] = {};
    T* x[kMaxLevels] = {};
    T* t[kMaxLevels] = {};
};

struct Level {
    int N = 0;
    int ncol = 0;
    int ncolp = 0;              // ncol rounded up to whole tiles
    int nvp = 0;                // nz * ncolp
    int32_t* nbr = nullptr;     // [4][ncol]
    uint32_t* fface = nullptr;  // [2][ncol] offsets of the W and S faces in kh
    int32_t* parent = nullptr;  // [ncol] into level + 1 (not on the coarsest)
    int32_t* pofs = nullptr;    // [3][ncol] prolongation offsets (not on the coarsest)
    int32_t* child = nullptr;   // [4][ncol] into level - 1 (not on the finest)
    // levels whose legs run on patches in float64 or float32 V-cycles: patch size
    // (index of kPatchShapes, -1: neither) and its tables
    bool patch64 = false, patch32 = false;
    int patch = -1, npatch = 0;
    int32_t* pcol = nullptr;
    int32_t* ppar = nullptr;
    int32_t* pcnt = nullptr;
    uint32_t* plnb = nullptr;
    LevelData<double> d;
    LevelData<float> f;
};

// Bump allocator over the caller's workspace; run with base 0 to size it.
struct Carver {
    uintptr_t base;
    size_t off = 0;
    template <typename T>
    T* take(size_t count) {
        off = (off + HELMHOLTZ_WORKSPACE_ALIGN - 1) / HELMHOLTZ_WORKSPACE_ALIGN *
              HELMHOLTZ_WORKSPACE_ALIGN;
        T* p = reinterpret_cast<T*>(base + off);
        off += count * sizeof(T);
        return p;
    }
};

bool config_ok(const helmholtz_config* c) {
    if (!c) return false;
    if (c->N < 1 || c->nz < 1 || c->nz > HELMHOLTZ_NZ_MAX || c->nlevels < 1 ||
        c->nlevels > kMaxLevels)
        return false;
    if (c->n_pre < 0 || c->n_post < 0 || c->n_coarse < 1) return false;
    if (!(c->omega > 0.0 && c->omega <= 1.5)) return false;
    if (c->mg_precision != HELMHOLTZ_FP64 && c->mg_precision != HELMHOLTZ_FP32) return false;
    if (c->cg_variant != HELMHOLTZ_CG_STANDARD && c->cg_variant != HELMHOLTZ_CG_FLEXIBLE &&
        c->cg_variant != HELMHOLTZ_BICGSTAB)
        return false;
    if (c->max_batch < 1) return false;
    if (c->stencil != 0 && c->stencil != 7 && c->stencil != 9) return false;
    if (c->weighted != 0 && c->weighted != 1) return false;
    // the weighted operator is not symmetric: BiCGStab, 7-point stencil
    if (c->weighted && (c->cg_variant != HELMHOLTZ_BICGSTAB || c->stencil == 9)) return false;
    return true;
}

int shape_error(const helmholtz_config* c) {
    if (c->N % (1 << (c->nlevels - 1)) != 0) return HELMHOLTZ_ESHAPE;
    const int64_t ncol = 6 * int64_t(c->N) * c->N;
    const int64_t ncolp = (ncol + kTile - 1) / kTile * kTile;
    // tables and offsets inside one vector are 32-bit (face offsets into the
    // two kh planes unsigned); batch offsets are 64-bit
    if (2 * ncol >= (int64_t(1) << 31)) return HELMHOLTZ_ESHAPE;
    if (int64_t(c->nz) * ncolp >= (int64_t(1) << 31)) return HELMHOLTZ_ESHAPE;
    return HELMHOLTZ_OK;
}

}  // namespace

// ---- allocation-free V-cycle: static scratch -------------------------------
// helmholtz_vcycle_noalloc keeps its level vectors in this file-scope device
// array instead of the workspace. Each GPU holds its own copy until the
// process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the device that is current (the array's
// name is a host-side stand-in, not a device address).
constexpr size_t kScratchBytes = HELMHOLTZ_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Address of the scratch array on the current device, looked up once per
// device; `dev` receives the device index.
int scratch_of_current_device(unsigned char** out, int* dev) {
    *out = nullptr;
    if (hipGetDevice(dev) != hipSuccess) return HELMHOLTZ_EHIP;
    if (*dev < 0 || *dev >= kMaxDevices) return HELMHOLTZ_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[*dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
            return HELMHOLTZ_EHIP;
        g_scratch_ptr[*dev] = static_cast<unsigned char*>(p);
    }
    *out = g_scratch_ptr[*dev];
    return HELMHOLTZ_OK;
}

}  // namespace

struct helmholtz_s {
    helmholtz_config cfg{};
    int L = 0, nz = 0, B = 0;
    bool nine = false;  // 9-cell stencil (next-to-nearest vertical couplings)
    bool weighted = false;  // row-weighted operator H = delta + S L
    bool adj = false;       // the current call works with H^T (weighted handles)
    int64_t n = 0;    // unknowns per right-hand side on the finest level
    int64_t nvp = 0;  // tiled length of a finest-level vector (n plus padding)
    std::vector<Level> lev;
    // Krylov vectors [B][n]
    double* r = nullptr;
    double* p = nullptr;
    double* q = nullptr;
    double* z = nullptr;  // float64 preconditioned residual (float64 V-cycle)
    // BiCGStab only: shadow residual r0, s, t, s_hat (p_hat is z, v is q)
    double* r0 = nullptr;
    double* s = nullptr;
    double* t = nullptr;
    double* sh = nullptr;
    // r, p, q, z are tiled [B][nvp]; x and b of the ABI are [B][n]
    double* partial = nullptr;
    double* partial2 = nullptr;
    double* partial3 = nullptr;
    double* partial4 = nullptr;
    int pstride = 0;
    double* sc = nullptr;     // [B][8] scalars
    int* active = nullptr;    // [B]
    int* upd = nullptr;       // [B] CG: the last residual update included the rhs
    int* flags = nullptr;     // set-up validation bits
    // pinned, host-coherent mirror written by the device: scalars, flags,
    // per-RHS sequence numbers; plus the set-up flags
    double* hsc = nullptr;
    int* hact = nullptr;
    int* hseq = nullptr;
    int* hflags = nullptr;
    size_t ws_bytes = 0, table_bytes = 0;
    // kernel timing hook: event pairs recorded around profiled launches
    struct Prof {
        double ms = 0.0, bytes = 0.0;
        int64_t launches = 0;
        std::vector<hipEvent_t> start, stop;
        std::vector<double> pend_bytes;
    };
    bool prof_on = false;
    mutable Prof prof[HELMHOLTZ_PROF_COUNT];
    // V-cycle vectors in the workspace (float64: level 0 comes from the caller)
    VBufs<double> vb64;
    VBufs<float> vb32;
    // this device's copy of the static scratch array (allocation-free entry
    // point) and the device the handle was created on
    unsigned char* scratch = nullptr;
    int device = -1;
    // traversal direction of the next kernel on each level (alternates, see
    // xcd_remap)
    mutable int dir[kMaxLevels] = {};
    int flip(int l) const {
        const int d = dir[l];
        dir[l] ^= 1;
        return d;
    }
};

namespace {

// Patch size of a level (index of kPatchShapes), -1 if its legs run kernel by
// kernel (k_patch). By the columns of all right-hand sides: the smallest
// levels take the smallest patches, so that a workgroup has least to do; larger
// ones larger patches, whose rings repeat less work. V-cycle with one patched
// level, one right-hand side, against kernel by kernel (us, float32): C12 x 30
// 40 / 49 (2 x 2 columns; 42 with 4 x 4), C24 x 30 42 / 53 (4 x 4; 45 with
// 2 x 2 or 8 x 4), C32 x 70 72 / 88 (8 x 4; 87 with 4 x 4). Coarsest level,
// four sweeps: C12 x 70 23 / 30 (2 x 2), C24 x 30 16 / 25 (4 x 4), C48 x 30
// 35 / 33.
int patch_kind(const helmholtz_config* c, int N, bool coarsest) {
    const int64_t cols = 6 * int64_t(N) * N * c->max_batch;
    if (coarsest) {
        if (c->n_coarse > 4) return -1;
        return cols <= 1000 ? 2 : (cols <= 6200 ? 3 : -1);
    }
    if (c->n_pre != 2 || c->n_post != 2) return -1;
    return cols <= 1000 ? 0 : (cols <= 4096 ? 1 : (cols <= 40000 ? 4 : -1));
}

// Whether the legs pay on patches, on columns of nz levels in `places` rows (fill
// rows included: 16 at least, 32 with the 9-cell and the weighted operators).
// A CU holds one workgroup of a leg on deep columns (two on those of up to 32
// float32 rows), so a leg's time goes with the generations of 256 workgroups that
// it takes, whole ones, while kernel by kernel it goes with the values. V-cycles,
// this level on patches / kernel by kernel (us, two levels, the coarsest on patches
// both ways, float32 unless noted):
// * 8 x 4 patches, one generation: gain at all depths that the registers hold
//   (patch_deepest): C32 x 32 26 / 44, C32 x 80 58 / 86, C32 x 48 float64 50 / 68;
// * two: up to 64 rows (C40 x 64 63 / 68, C40 x 70 85 / 83; 9-cell C40 x 47 70 /
//   79), in float64 up to 32 (C40 x 30 48 / 52, C40 x 47 76 / 69), and not for the
//   few levels whose columns are mostly fill (9-cell C36 x 1 31 / 30; float64 C40
//   x 1 30 / 25, 9-cell 48 / 34, x 20 53 / 58);
// * three: float32, up to 32 rows (C54 x 6 30 / 36, C54 x 30 45 / 53, C54 x 40 74 /
//   71; 9-cell C54 x 6 53 / 48; float64 C54 x 6 46 / 42); four: 16 rows (C72 x 10
//   44 / 49, C72 x 40 105 / 92); five no more (C80 x 8 50 / 47);
// * levels below kSmallSweepCols columns in a batch, which kernel by kernel run
//   with the narrow tiles, take one generation more beyond the second (C24 x 30
//   float64, six right-hand sides 73 / 83).
// 4 x 4 patches need less of a CU: in float32 only the deep columns lose to a second
// generation (C24 x 100 50 / 70, C26 x 100 81 / 80; 9-cell C26 x 48 46 / 59, x 64
// 70 / 67). In float64 all deeper ones do (coarsest level C20 x 48 19 / 31, C26 x 48
// 36 / 33), and, below a level that leaves nothing of theirs in the L2, those of
// the larger stencils (times as long on patches: C26 in C104, 4 to 47 levels, 9-cell
// 0.99 to 1.08, weighted with few levels 1.02; coarsest C25 to C32 in C50 to C64,
// 9-cell 1.05, weighted with few levels 1.02, with 20 to 30 0.98).
template <typename T>
bool patch_pays(int kind, int nz, int places, int ncol, int64_t workgroups, bool nine,
                bool weighted) {
    constexpr bool f32 = sizeof(T) == 4;
    constexpr int kWave = 256;  // workgroups of one generation
    if (nz > patch_deepest<T>(kind, nine)) return false;
    const int64_t gen = (workgroups + kWave - 1) / kWave;
    if (gen == 1 || kind == 0 || kind == 2) return true;
    const int fill = places - nz;
    if (kind != 4) {
        if (f32) return places <= (kind == 3 ? 64 : (nine || weighted ? 48 : 80));
        return gen == 2 && !nine && fill <= 13 && places <= (kind == 1 && !weighted ? 48 : 32);
    }
    switch (gen > 2 && ncol < kSmallSweepCols && !nine ? gen - 1 : gen) {
        case 2: return f32 ? places <= 64 && fill <= 28 : places <= 32 && fill <= 13;
        case 3: return f32 && places <= 32 && fill <= (nine ? 4 : 12);
        case 4: return f32 && places <= 16 && fill <= 12;
        default: return false;
    }
}

// Whether V-cycles of precision T run the legs of a level of ncol columns on
// patches of this size, in one launch each (k_patch).
template <typename T>
bool patch_runs(const helmholtz_s* h, int kind, int ncol, int npatch) {
    const bool seven_point = !h->nine && !h->weighted;
    const int jmax = patch_levels(h->nz, seven_point);
    return patch_compiled<T>(kind, jmax, h->nine, seven_point) &&
           patch_pays<T>(kind, h->nz, kPatchLanes * jmax, ncol, int64_t(h->B) * npatch, h->nine,
                         h->weighted);
}

template <typename T>
bool patch_level(const helmholtz_s* h, int l) {
    return sizeof(T) == 8 ? h->lev[l].patch64 : h->lev[l].patch32;
}

void layout(helmholtz_s* h, Carver& cv) {
    const int nz = h->nz, B = h->B;
    // the tables of all levels come first: one copy fills them (create)
    for (int l = 0; l < h->L; ++l) {
        Level& v = h->lev[l];
        const size_t nc = size_t(v.ncol);
        v.nbr = cv.take<int32_t>(4 * nc);
        v.fface = cv.take<uint32_t>(2 * nc);
        v.parent = (l + 1 < h->L) ? cv.take<int32_t>(nc) : nullptr;
        v.pofs = (l + 1 < h->L) ? cv.take<int32_t>(3 * nc) : nullptr;
        v.child = (l > 0) ? cv.take<int32_t>(4 * nc) : nullptr;
        if (v.patch >= 0) {
            const size_t np = size_t(v.npatch), ncp = size_t(kPatchShapes[v.patch].ncp);
            v.pcol = cv.take<int32_t>(np * ncp);
            v.ppar = cv.take<int32_t>(np * ncp);
            v.pcnt = cv.take<int32_t>(np * kPatchCounts);
            v.plnb = cv.take<uint32_t>(np * ncp);
        }
    }
    h->table_bytes = cv.off;
    for (int l = 0; l < h->L; ++l) {
        Level& v = h->lev[l];
        const size_t nc = size_t(v.ncol);
        const size_t nv = size_t(v.nvp);
        const size_t places = size_t(kPatchLanes) * patch_levels(nz, !h->nine && !h->weighted);
        if (patch_level<double>(h, l)) v.d.co = cv.take<double>(size_t(kColPlanes) * places * nc);
        if (patch_level<float>(h, l)) v.f.co = cv.take<float>(size_t(kColPlanes) * places * nc);
        v.d.kh = cv.take<double>(2 * nv);
        v.d.kv = cv.take<double>(nv);
        v.d.dl = cv.take<double>(nv);
        v.d.cc = cv.take<double>(nv);
        v.d.mm = cv.take<double>(nv);
        // float32 copies
        v.f.kh = cv.take<float>(6 * nv);
        v.f.kv = v.f.kh + 2 * nv;
        v.f.dl = v.f.kh + 3 * nv;
        v.f.cc = v.f.kh + 4 * nv;
        v.f.mm = v.f.kh + 5 * nv;
        if (h->nine) {
            v.d.kv2 = cv.take<double>(nv);
            v.f.kv2 = cv.take<float>(nv);
        }
        if (h->weighted) {
            v.d.s = cv.take<double>(nv);
            v.f.s = cv.take<float>(nv);
        }
        if (l > 0) {
            v.d.b = cv.take<double>(size_t(B) * nv);
            v.d.x = cv.take<double>(size_t(B) * nv);
        }
        v.d.t = cv.take<double>(size_t(B) * nv);
        v.f.b = cv.take<float>(size_t(B) * nv);
        v.f.x = cv.take<float>(size_t(B) * nv);
        v.f.t = cv.take<float>(size_t(B) * nv);
        h->vb64.b[l] = v.d.b;
        h->vb64.x[l] = v.d.x;
        h->vb64.t[l] = v.d.t;
        h->vb32.b[l] = v.f.b;
        h->vb32.x[l] = v.f.x;
        h->vb32.t[l] = v.f.t;
    }
    const size_t nb = size_t(B) * size_t(h->nvp);
    h->r = cv.take<double>(nb);
    h->p = cv.take<double>(nb);
    h->q = cv.take<double>(nb);
    h->z = cv.take<double>(nb);
    if (h->cfg.cg_variant == HELMHOLTZ_BICGSTAB) {
        h->r0 = cv.take<double>(nb);
        h->s = cv.take<double>(nb);
        h->t = cv.take<double>(nb);
        h->sh = cv.take<double>(nb);
    }
    const int ntile0 = (h->lev[0].ncol + kBlock - 1) / kBlock;
    const int nkc0 = (nz + kApplyChunk - 1) / kApplyChunk;
    const int ntile32 = h->lev[0].ncolp / kTile;
    h->pstride = std::max(std::max(kRedBlocks, ntile0 * nkc0), ntile32);
    h->partial = cv.take<double>(size_t(B) * h->pstride);
    h->partial2 = cv.take<double>(size_t(B) * h->pstride);
    h->partial3 = cv.take<double>(size_t(B) * h->pstride);
    h->partial4 = cv.take<double>(size_t(B) * h->pstride);
    h->sc = cv.take<double>(size_t(B) * kScal);
    h->active = cv.take<int>(size_t(B));
    h->upd = cv.take<int>(size_t(B));
    h->flags = cv.take<int>(4);
}

void init_shape(helmholtz_s* h, const helmholtz_config* cfg) {
    h->cfg = *cfg;
    h->L = cfg->nlevels;
    h->nz = cfg->nz;
    h->B = cfg->max_batch;
    h->nine = cfg->stencil == 9;
    h->weighted = cfg->weighted == 1;
    h->lev.assign(h->L, Level{});
    for (int l = 0; l < h->L; ++l) {
        Level& v = h->lev[l];
        v.N = cfg->N >> l;
        v.ncol = 6 * v.N * v.N;
        v.ncolp = (v.ncol + kTile - 1) / kTile * kTile;
        v.nvp = cfg->nz * v.ncolp;
        const int kind = patch_kind(cfg, v.N, l == h->L - 1);
        if (kind < 0) continue;
        const int np = patch_count(v.N, kPatchShapes[kind].pw, kPatchShapes[kind].ph);
        // a float32 handle never runs a float64 V-cycle
        v.patch64 = cfg->mg_precision == HELMHOLTZ_FP64 &&
                    patch_runs<double>(h, kind, v.ncol, np);
        v.patch32 = patch_runs<float>(h, kind, v.ncol, np);
        if (!v.patch64 && !v.patch32) continue;
        v.patch = kind;
        v.npatch = np;
    }
    h->n = int64_t(cfg->nz) * h->lev[0].ncol;
    h->nvp = h->lev[0].nvp;
}

inline int grid_for(int64_t n) {
    return int(std::min<int64_t>((n + kBlock - 1) / kBlock, 65536));
}

#define HH_CHECK(expr)                                   \
    do {                                                 \
        if ((expr) != hipSuccess) return HELMHOLTZ_EHIP; \
    } while (0)

inline int last_error() { return hipGetLastError() == hipSuccess ? HELMHOLTZ_OK : HELMHOLTZ_EHIP; }

// Fold the finished event pairs of one profiled kernel into its totals.
int prof_flush(const helmholtz_s* h, int kernel) {
    helmholtz_s::Prof& P = h->prof[kernel];
    for (size_t i = 0; i < P.start.size(); ++i) {
        float ms = 0.f;
        if (hipEventSynchronize(P.stop[i]) != hipSuccess) return HELMHOLTZ_EHIP;
        if (hipEventElapsedTime(&ms, P.start[i], P.stop[i]) != hipSuccess) return HELMHOLTZ_EHIP;
        P.ms += ms;
        P.bytes += P.pend_bytes[i];
        P.launches += 1;
        (void)hipEventDestroy(P.start[i]);
        (void)hipEventDestroy(P.stop[i]);
    }
    P.start.clear();
    P.stop.clear();
    P.pend_bytes.clear();
    return HELMHOLTZ_OK;
}

// Record an event before a profiled launch; returns false when profiling is off.
bool prof_begin(const helmholtz_s* h, int kernel, hipStream_t s) {
    if (!h->prof_on) return false;
    helmholtz_s::Prof& P = h->prof[kernel];
    if (P.start.size() >= 256 && prof_flush(h, kernel) != HELMHOLTZ_OK) return false;
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return false;
    if (hipEventCreate(&b) != hipSuccess) {
        (void)hipEventDestroy(a);
        return false;
    }
    P.start.push_back(a);
    P.stop.push_back(b);
    P.pend_bytes.push_back(0.0);
    (void)hipEventRecord(a, s);
    return true;
}

void prof_end(const helmholtz_s* h, int kernel, double bytes, hipStream_t s) {
    helmholtz_s::Prof& P = h->prof[kernel];
    P.pend_bytes.back() = bytes;
    (void)hipEventRecord(P.stop.back(), s);
}

CgState cg_state(const helmholtz_s* h) {
    return CgState{h->partial, h->partial2, h->partial3, h->partial4, h->pstride, h->sc,
                   h->active,  h->upd,      h->hsc,      h->hact,     h->hseq};
}

template <typename T>
LevelView<T> view(const helmholtz_s* h, int l) {
    const Level& v = h->lev[l];
    const LevelData<T>& d = [&]() -> const LevelData<T>& {
        if constexpr (std::is_same<T, double>::value) return v.d;
        else return v.f;
    }();
    return LevelView<T>{v.ncol, h->nz, v.nvp, v.N,  v.nbr, v.fface, v.pofs,
                        d.kh,   d.kv,  d.dl,  d.cc, d.mm,  d.kv2,  d.s};
}

// ---- sweep launch: compile-time bound on levels per thread ---------------
inline int sweep_mid(int nz) { return nz / 2; }

// Whether one sweep over level l streams far more data than the last-level
// cache (256 MiB Infinity Cache) holds: then its read-once streams bypass the
// cache (k_sweep with NTS). On smaller levels the next kernel finds the
// previous one's output there, and plain accesses are faster.
bool streams_past_cache(const helmholtz_s* h, int l, int batch, size_t word) {
    constexpr int64_t kLastLevelCache = int64_t(256) << 20;
    // kh[2], cc, mm and the neighbour couplings; b, x, x_new per right-hand side
    return int64_t(h->lev[l].nvp) * int64_t(word) * (5 + 3 * int64_t(batch)) > kLastLevelCache;
}

// The sweep and the residual restriction stream past the cache only for one
// right-hand side: the members of a batch share each tile's coefficients
// through L2, so there the coefficients stay cached (float32 V-cycle at
// C384 x 70 with four right-hand sides: 7.19 -> 7.09 ms).
bool sweep_streams_past_cache(const helmholtz_s* h, int l, int batch, size_t word) {
    return batch == 1 && streams_past_cache(h, l, batch, word);
}

template <typename T, int JMAX, int MODE, int TC, bool VARIANTS>
void launch_sweep_b(const helmholtz_s* h, int l, const T* b, const T* x, const T* xc, T* y,
                    int batch, const int* active, hipStream_t s) {
    const Level& v = h->lev[l];
    using Tile = SweepTile<T, TC, kBlock>;
    const int ntile = (v.ncol + TC - 1) / TC;
    const int nvp_c = (l + 1 < h->L) ? h->lev[l + 1].nvp : 0;
    const bool prof = (l == 0 && MODE == kPlain) && prof_begin(h, HELMHOLTZ_PROF_SWEEP_FINE, s);
    const int rev = h->flip(l);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(ntile * batch), dim3(kBlock), Tile::lds_bytes(h->nz), s,
                           view<T>(h, l), b, x, xc, nvp_c, y, T(h->cfg.omega), batch, active,
                           sweep_mid(h->nz), rev, static_cast<T*>(nullptr),
                           static_cast<double*>(nullptr), 0);
    };
    // only the large levels use 32-column tiles and can stream past the cache
    constexpr bool kCanStream = TC == kTile;
    const bool nts = kCanStream && sweep_streams_past_cache(h, l, batch, sizeof(T));
    auto pick = [&](auto plain, auto streamed) {
        if constexpr (kCanStream) {
            if (nts) {
                go(streamed);
                return;
            }
        }
        go(plain);
    };
    if constexpr (VARIANTS) {
        if (h->weighted && h->adj)
            pick(k_sweep<T, JMAX, MODE, TC, kBlock, 0, false, kRowWT>,
                 k_sweep<T, JMAX, MODE, TC, kBlock, 0, false, kRowWT, kCanStream>);
        else if (h->weighted)
            pick(k_sweep<T, JMAX, MODE, TC, kBlock, 0, false, kRowW>,
                 k_sweep<T, JMAX, MODE, TC, kBlock, 0, false, kRowW, kCanStream>);
        else
            pick(k_sweep<T, JMAX, MODE, TC, kBlock, 0, true>,
                 k_sweep<T, JMAX, MODE, TC, kBlock, 0, true, kSym, kCanStream>);
    } else {
        pick(k_sweep<T, JMAX, MODE, TC, kBlock, 0, false>,
             k_sweep<T, JMAX, MODE, TC, kBlock, 0, false, kSym, kCanStream>);
    }
    if (prof)  // b, x, kh[2], cc, mm (, kv2) read; x_new written
        prof_end(h, HELMHOLTZ_PROF_SWEEP_FINE,
                 (h->nine ? 8.0 : 7.0) * sizeof(T) * double(batch) * h->nz * v.ncol, s);
}

// Large levels: 32-column tiles (8 level groups, several workgroups per CU).
// Small levels cannot fill the GPU and are bound by the latency of a few
// dependent steps per thread: 8-column tiles with 32 level groups let each
// thread load its few levels in one batch.
template <typename T, int MODE, int TC>
void launch_sweep_tc(const helmholtz_s* h, int l, const T* b, const T* x, const T* xc, T* y,
                     int batch, const int* active, hipStream_t s) {
    constexpr int KG = kBlock / TC;
    const int jn = (h->nz + KG - 1) / KG;
#define HH_SWEEP_BUCKET(J, V)                                                    \
    if (jn <= J) {                                                               \
        launch_sweep_b<T, J, MODE, TC, V>(h, l, b, x, xc, y, batch, active, s);  \
        return;                                                                  \
    }
    if (h->nine || h->weighted) {
        // the 9-cell and weighted operators: fewer compiled bucket sizes
        HH_SWEEP_BUCKET(4, true)
        if (TC == 32) {
            HH_SWEEP_BUCKET(9, true)
            HH_SWEEP_BUCKET(15, true)
        }
        return;
    }
    HH_SWEEP_BUCKET(1, false)
    HH_SWEEP_BUCKET(2, false)
    HH_SWEEP_BUCKET(4, false)
    if (TC == 32) {
        HH_SWEEP_BUCKET(9, false)
        HH_SWEEP_BUCKET(15, false)
    }
#undef HH_SWEEP_BUCKET
}

template <typename T, int MODE>
void launch_sweep_m(const helmholtz_s* h, int l, const T* b, const T* x, const T* xc, T* y,
                    int batch, const int* active, hipStream_t s) {
    if (h->lev[l].ncol < kSmallSweepCols)
        launch_sweep_tc<T, MODE, 8>(h, l, b, x, xc, y, batch, active, s);
    else
        launch_sweep_tc<T, MODE, 32>(h, l, b, x, xc, y, batch, active, s);
}

// The first (kIoIn, from zero) or the last (kIoOut, plain) sweep of the finest
// level with b or the result in the ABI layout, S values, or the last one with
// r . z (kIoDot): 7-point operator, 32-column tiles.
template <typename T, typename S, int JMAX, int MODE, int IO>
void launch_sweep_io_j(const helmholtz_s* h, const T* b, const T* x, T* y, S* ext, int batch,
                       const int* active, hipStream_t s) {
    const Level& v = h->lev[0];
    using Tile = SweepTile<T>;
    const bool prof = MODE == kPlain && prof_begin(h, HELMHOLTZ_PROF_SWEEP_FINE, s);
    const int rev = h->flip(0);
    auto go = [&](auto kern) {
        const T* xc = nullptr;
        hipLaunchKernelGGL(kern, dim3(v.ncolp / kTile * batch), dim3(kBlock),
                           Tile::lds_bytes(h->nz), s, view<T>(h, 0), b, x, xc, 0, y,
                           T(h->cfg.omega), batch, active, sweep_mid(h->nz), rev, ext,
                           h->partial, h->pstride);
    };
    if (sweep_streams_past_cache(h, 0, batch, sizeof(T)))
        go(k_sweep<T, JMAX, MODE, kTile, kBlock, 0, false, kSym, true, S, IO>);
    else
        go(k_sweep<T, JMAX, MODE, kTile, kBlock, 0, false, kSym, false, S, IO>);
    if (prof)
        prof_end(h, HELMHOLTZ_PROF_SWEEP_FINE,
                 7.0 * sizeof(T) * double(batch) * h->nz * v.ncol, s);
}

template <typename T, typename S, int MODE, int IO>
void launch_sweep_io(const helmholtz_s* h, const T* b, const T* x, T* y, S* ext, int batch,
                     const int* active, hipStream_t s) {
    const int jn = (h->nz + 7) / 8;
    if (jn <= 4) launch_sweep_io_j<T, S, 4, MODE, IO>(h, b, x, y, ext, batch, active, s);
    else if (jn <= 9) launch_sweep_io_j<T, S, 9, MODE, IO>(h, b, x, y, ext, batch, active, s);
    else launch_sweep_io_j<T, S, 15, MODE, IO>(h, b, x, y, ext, batch, active, s);
}

// Levels too small to fill the GPU are bound by the latency of a few dependent
// steps per thread; their kernels give each thread less work.
inline bool small_level(const helmholtz_s* h, int l) { return h->lev[l].ncol < 4096; }

template <typename T>
void launch_sweep(const helmholtz_s* h, int l, int mode, const T* b, const T* x, const T* xc,
                  T* y, int batch, const int* active, hipStream_t s) {
    switch (mode) {
        case kZero: launch_sweep_m<T, kZero>(h, l, b, x, xc, y, batch, active, s); break;
        case kPlain: launch_sweep_m<T, kPlain>(h, l, b, x, xc, y, batch, active, s); break;
        case kProlong: launch_sweep_m<T, kProlong>(h, l, b, x, xc, y, batch, active, s); break;
        default: launch_sweep_m<T, kProlongZero>(h, l, b, x, xc, y, batch, active, s); break;
    }
}

template <typename T>
void launch_resid_restrict(const helmholtz_s* h, int l, const T* b, const T* x, T* bc, int batch,
                           const int* active, hipStream_t s) {
    const Level& c = h->lev[l + 1];
    const int ntile = (c.ncol + kBlock - 1) / kBlock;
    // one level per thread on small levels (one dependent step), four otherwise
    const int kchunk = small_level(h, l) ? 1 : kApplyChunk;
    const int nkc = (h->nz + kchunk - 1) / kchunk;
    const dim3 grid(ntile * nkc * batch);
    // child pairs load as one vector when b and x are aligned to two elements
    // (the level's own arrays always are: tiles hold an even number of values)
    const uintptr_t al = 2 * sizeof(T);
    const bool pair = reinterpret_cast<uintptr_t>(b) % al == 0 &&
                      reinterpret_cast<uintptr_t>(x) % al == 0;
    const int rev = h->flip(l);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, s, view<T>(h, l), c.child, c.ncol, c.nvp,
                           b, x, bc, batch, kchunk, nkc, active, rev);
    };
    // paired loads (the library's own buffers): streamed past the cache on
    // levels far larger than it
    const bool nts = sweep_streams_past_cache(h, l, batch, sizeof(T));
    auto pick = [&](auto plain, auto streamed) {
        if (nts) go(streamed);
        else go(plain);
    };
    // each operator form: where the coarse panels tile into patches (32 x 8,
    // else 16 x 16 coarse cells), the children's values go through LDS
    // (k_resid_restrict_lds); otherwise the gathering kernel
    auto form = [&](auto k2, auto sc) {
        constexpr bool K2 = decltype(k2)::value;
        constexpr int SC = decltype(sc)::value;
        if (pair && c.N % 32 == 0)
            pick(k_resid_restrict_lds<T, false, 32, K2, SC>,
                 k_resid_restrict_lds<T, true, 32, K2, SC>);
        else if (pair && c.N % 16 == 0)
            pick(k_resid_restrict_lds<T, false, 16, K2, SC>,
                 k_resid_restrict_lds<T, true, 16, K2, SC>);
        else if (pair)
            pick(k_resid_restrict<T, false, true, K2, SC>,
                 k_resid_restrict<T, false, true, K2, SC, true>);
        else
            go(k_resid_restrict<T, false, false, K2, SC>);
    };
    using Sym = std::integral_constant<int, kSym>;
    if (!x) {
        if (pair)
            pick(k_resid_restrict<T, true, true>,
                 k_resid_restrict<T, true, true, false, kSym, true>);
        else go(k_resid_restrict<T, true, false>);
    } else if (h->nine) {
        form(std::true_type{}, Sym{});
    } else if (h->weighted && h->adj) {
        form(std::false_type{}, std::integral_constant<int, kRowWT>{});
    } else if (h->weighted) {
        form(std::false_type{}, std::integral_constant<int, kRowW>{});
    } else {
        form(std::false_type{}, Sym{});
    }
}

template <typename T, typename X = T>
void launch_apply(const helmholtz_s* h, int l, const X* x, T* y, int batch, int dot,
                  const int* active, hipStream_t s, const T* w = nullptr) {
    const Level& v = h->lev[l];
    const int ntile = (v.ncol + kBlock - 1) / kBlock;
    const int nkc = (h->nz + kApplyChunk - 1) / kApplyChunk;
    const dim3 grid(ntile * nkc * batch);
    const bool prof = (l == 0 && sizeof(T) == 8) && prof_begin(h, HELMHOLTZ_PROF_APPLY_FINE, s);
    const int rev = h->flip(l);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, s, view<T>(h, l), x, y, w, batch, nkc,
                           cg_state(h), active, rev);
    };
    if (v.N % kTile == 0 && !h->weighted) {
        // the panels tile into patches of 64 x 4 (else 32 x 8) columns:
        // neighbours' values through LDS (7-point and 9-cell stencils; with
        // the row-weighted operator it was no faster: each thread's weights
        // must arrive before it publishes s x, H 227 -> 229, H^T 263 -> 278 us)
        auto patch = [&](auto nts, auto px, auto k2) {
            constexpr bool NT = decltype(nts)::value;
            constexpr int PX = decltype(px)::value;
            constexpr bool K2 = decltype(k2)::value;
            switch (dot) {
                case kDotXY: go(k_apply_lds<T, kDotXY, kApplyChunk, NT, PX, K2, false, X>); break;
                case kDotWY: go(k_apply_lds<T, kDotWY, kApplyChunk, NT, PX, K2, false, X>); break;
                default: go(k_apply_lds<T, kDotWYYY, kApplyChunk, NT, PX, K2, false, X>); break;
            }
        };
        auto by_width = [&](auto nts, auto k2) {
            if (v.N % 64 == 0) patch(nts, std::integral_constant<int, 64>{}, k2);
            else patch(nts, std::integral_constant<int, 32>{}, k2);
        };
        if (streams_past_cache(h, l, batch, sizeof(T)))
            h->nine ? by_width(std::true_type{}, std::true_type{})
                    : by_width(std::true_type{}, std::false_type{});
        else
            h->nine ? by_width(std::false_type{}, std::true_type{})
                    : by_width(std::false_type{}, std::false_type{});
    } else if (h->weighted) {
        if (h->adj) {
            switch (dot) {
                case kDotXY: go(k_apply<T, kDotXY, kApplyChunk, false, kRowWT, false, false, X>); break;
                case kDotWY: go(k_apply<T, kDotWY, kApplyChunk, false, kRowWT, false, false, X>); break;
                default: go(k_apply<T, kDotWYYY, kApplyChunk, false, kRowWT, false, false, X>); break;
            }
        } else {
            switch (dot) {
                case kDotXY: go(k_apply<T, kDotXY, kApplyChunk, false, kRowW, false, false, X>); break;
                case kDotWY: go(k_apply<T, kDotWY, kApplyChunk, false, kRowW, false, false, X>); break;
                default: go(k_apply<T, kDotWYYY, kApplyChunk, false, kRowW, false, false, X>); break;
            }
        }
    } else if (h->nine) {
        switch (dot) {
            case kDotXY: go(k_apply<T, kDotXY, kApplyChunk, true, kSym, false, false, X>); break;
            case kDotWY: go(k_apply<T, kDotWY, kApplyChunk, true, kSym, false, false, X>); break;
            default: go(k_apply<T, kDotWYYY, kApplyChunk, true, kSym, false, false, X>); break;
        }
    } else if (streams_past_cache(h, l, batch, sizeof(T))) {
        switch (dot) {
            case kDotXY: go(k_apply<T, kDotXY, kApplyChunk, false, kSym, true, false, X>); break;
            case kDotWY: go(k_apply<T, kDotWY, kApplyChunk, false, kSym, true, false, X>); break;
            default: go(k_apply<T, kDotWYYY, kApplyChunk, false, kSym, true, false, X>); break;
        }
    } else {
        switch (dot) {
            case kDotXY: go(k_apply<T, kDotXY, kApplyChunk, false, kSym, false, false, X>); break;
            case kDotWY: go(k_apply<T, kDotWY, kApplyChunk, false, kSym, false, false, X>); break;
            default: go(k_apply<T, kDotWYYY, kApplyChunk, false, kSym, false, false, X>); break;
        }
    }
    if (prof)  // x, kh[2], kv, delta (, kv2) read; y written
        prof_end(h, HELMHOLTZ_PROF_APPLY_FINE,
                 (h->nine ? 7.0 : 6.0) * sizeof(T) * double(batch) * h->nz * v.ncol, s);
}

// y = H x on the finest level with x and y in the ABI layout.
void launch_apply_natural(const helmholtz_s* h, const double* x, double* y, int batch,
                          hipStream_t s) {
    const Level& v = h->lev[0];
    const int ntile = (v.ncol + kBlock - 1) / kBlock;
    const int nkc = (h->nz + kApplyChunk - 1) / kApplyChunk;
    const bool prof = prof_begin(h, HELMHOLTZ_PROF_APPLY_FINE, s);
    const int rev = h->flip(0);
    auto go = [&](auto kern) {
        const double* none = nullptr;
        hipLaunchKernelGGL(kern, dim3(ntile * nkc * batch), dim3(kBlock), 0, s,
                           view<double>(h, 0), x, y, none, batch, nkc, cg_state(h),
                           static_cast<const int*>(nullptr), rev);
    };
    // the same choice of kernel as for tiled vectors (launch_apply)
    constexpr int KC = kApplyChunk;
    const bool nts = streams_past_cache(h, 0, batch, sizeof(double));
    if (v.N % kTile == 0 && !h->weighted) {
        auto by_width = [&](auto nt, auto k2) {
            constexpr bool NT = decltype(nt)::value, K2 = decltype(k2)::value;
            if (v.N % 64 == 0) go(k_apply_lds<double, kDotNone, KC, NT, 64, K2, true>);
            else go(k_apply_lds<double, kDotNone, KC, NT, 32, K2, true>);
        };
        if (nts) h->nine ? by_width(std::true_type{}, std::true_type{})
                         : by_width(std::true_type{}, std::false_type{});
        else h->nine ? by_width(std::false_type{}, std::true_type{})
                     : by_width(std::false_type{}, std::false_type{});
    } else if (h->weighted && h->adj) {
        go(k_apply<double, kDotNone, KC, false, kRowWT, false, true>);
    } else if (h->weighted) {
        go(k_apply<double, kDotNone, KC, false, kRowW, false, true>);
    } else if (h->nine) {
        go(k_apply<double, kDotNone, KC, true, kSym, false, true>);
    } else if (nts) {
        go(k_apply<double, kDotNone, KC, false, kSym, true, true>);
    } else {
        go(k_apply<double, kDotNone, KC, false, kSym, false, true>);
    }
    if (prof)
        prof_end(h, HELMHOLTZ_PROF_APPLY_FINE,
                 (h->nine ? 7.0 : 6.0) * sizeof(double) * double(batch) * h->nz * v.ncol, s);
}

// ---- V-cycle (Algorithm 1) ------------------------------------------------
// Number of x writes on level l and the buffer that write j goes to: the
// writes alternate between out_l and tmp_l, assigned from the last one
// backwards so that the last lands in out_l.
inline int level_writes(const helmholtz_s* h, int l) {
    const helmholtz_config& cfg = h->cfg;
    return l == h->L - 1 ? cfg.n_coarse : cfg.n_pre + std::max(cfg.n_post, 1);
}

template <typename T>
T* write_dst(const helmholtz_s* h, int l, int j, T* out, T* tmp) {
    return ((level_writes(h, l) - 1 - j) % 2 == 0) ? out : tmp;
}

// Whether they do in the present call: not with H^T; and with the timing hook
// on, the finest level runs kernel by kernel, so that the hook finds the sweeps
// it times.
template <typename T>
bool on_patches(const helmholtz_s* h, int l) {
    return patch_level<T>(h, l) && !(h->weighted && h->adj) && !(l == 0 && h->prof_on);
}

// b and x of a V-cycle entry point in the ABI layout; wide: float64 ones of a
// float32 V-cycle. Or only r: the last sweep takes b from it and leaves the
// partial sums of r . z, one per tile.
struct AbiVectors {
    const void* b;
    void* x;
    bool wide;
    const double* r = nullptr;
};

// Vectors between two levels on patches are stored column by column: those
// of level l (b and the solution) if l and l - 1 are such levels.
template <typename T>
bool vectors_by_column(const helmholtz_s* h, int l) {
    return l > 0 && l < h->L && on_patches<T>(h, l) && on_patches<T>(h, l - 1);
}

template <typename T>
void patch_leg(const helmholtz_s* h, int l, int leg, const T* b, const T* x, const T* xc, T* y,
               T* bc, int batch, const int* active, hipStream_t s, const AbiVectors* io) {
    const Level& v = h->lev[l];
    PatchArgs<T> A;
    if constexpr (std::is_same<T, double>::value) A.P.co = v.d.co;
    else A.P.co = v.f.co;
    A.P.col = v.pcol;
    A.P.lnb = v.plnb;
    A.P.cnt = v.pcnt;
    A.P.par = v.ppar;
    A.P.npatch = v.npatch;
    A.ncol = v.ncol;
    A.nz = h->nz;
    A.nvp = v.nvp;
    A.b = b;
    A.x = x;
    A.xc = xc;
    A.y = y;
    A.bc = bc;
    A.nvp_c = l + 1 < h->L ? h->lev[l + 1].nvp : 0;
    A.layout = vectors_by_column<T>(h, l) ? kByColumn : (io ? kAbi : kTiled);
    A.ext_b = io ? io->b : nullptr;
    A.ext_y = io ? io->x : nullptr;
    A.ext_wide = io && io->wide;
    A.ccol = vectors_by_column<T>(h, l + 1);
    A.omega = T(h->cfg.omega);
    A.batch = batch;
    A.active = active;
    A.mid = sweep_mid(h->nz);
    A.nsweep = h->cfg.n_coarse;
    // where the kernel-by-kernel path would run k_sweep<float, 9, kProlong, 32>
    A.om_first = sizeof(T) == 4 && !h->nine && !h->weighted && v.ncol >= kSmallSweepCols &&
                 h->nz > 32 && h->nz <= 72;
    A.rev = h->flip(l);
    launch_patch<T>(v.patch, leg, h->nine, h->weighted, A, s);
}

// Level l smooths b_l into out_l (Algorithm 1), using V.t[l] as the Jacobi
// ping-pong partner and V.b, V.x of the coarser levels. io (level 0 only): the
// first kernel reads b, and the last one writes the result, in the ABI layout;
// b and out are then this level's own buffers.
template <typename T>
void vcycle_level(helmholtz_s* h, const VBufs<T>& V, int l, const T* b, T* out, int batch,
                  const int* active, hipStream_t s, const AbiVectors* io = nullptr) {
    const helmholtz_config& cfg = h->cfg;
    T* tmp = V.t[l];
    const int W = level_writes(h, l);
    if (on_patches<T>(h, l)) {
        const T* none = nullptr;
        if (l == h->L - 1) {
            patch_leg<T>(h, l, kCoarse, b, none, none, out, nullptr, batch, active, s, io);
            return;
        }
        patch_leg<T>(h, l, kDown, b, none, none, tmp, V.b[l + 1], batch, active, s, io);
        vcycle_level<T>(h, V, l + 1, V.b[l + 1], V.x[l + 1], batch, active, s);
        patch_leg<T>(h, l, kUp, b, tmp, V.x[l + 1], out, nullptr, batch, active, s, io);
        return;
    }
    // the first sweep from zero and the last plain one, with b and the result in
    // the ABI layout where io is given
    auto sweep_first = [&](T* dst) {
        if (io && io->b && io->wide)
            launch_sweep_io<T, double, kZero, kIoIn>(
                h, b, nullptr, dst, static_cast<double*>(const_cast<void*>(io->b)), batch, active,
                s);
        else if (io && io->b)
            launch_sweep_io<T, T, kZero, kIoIn>(
                h, b, nullptr, dst, static_cast<T*>(const_cast<void*>(io->b)), batch, active, s);
        else
            launch_sweep<T>(h, l, kZero, b, nullptr, nullptr, dst, batch, active, s);
    };
    auto sweep_last = [&](const T* prev, T* dst) {
        if (io && io->r)
            launch_sweep_io<T, double, kPlain, kIoDot>(h, b, prev, dst,
                                                       const_cast<double*>(io->r), batch, active,
                                                       s);
        else if (io && io->wide)
            launch_sweep_io<T, double, kPlain, kIoOut>(
                h, b, prev, dst, static_cast<double*>(io->x), batch, active, s);
        else if (io)
            launch_sweep_io<T, T, kPlain, kIoOut>(h, b, prev, dst, static_cast<T*>(io->x), batch,
                                                  active, s);
        else
            launch_sweep<T>(h, l, kPlain, b, prev, nullptr, dst, batch, active, s);
    };
    if (l == h->L - 1) {
        const T* prev = nullptr;
        for (int j = 0; j < W; ++j) {
            T* dst = write_dst<T>(h, l, j, out, tmp);
            if (j == 0) sweep_first(dst);
            else if (j == W - 1) sweep_last(prev, dst);
            else launch_sweep<T>(h, l, kPlain, b, prev, nullptr, dst, batch, active, s);
            prev = dst;
        }
        return;
    }
    int j = 0;
    const T* prev = nullptr;
    for (int i = 0; i < cfg.n_pre; ++i, ++j) {
        T* dst = write_dst<T>(h, l, j, out, tmp);
        if (j == 0) sweep_first(dst);
        else launch_sweep<T>(h, l, kPlain, b, prev, nullptr, dst, batch, active, s);
        prev = dst;
    }
    T* cb = V.b[l + 1];
    T* cx = V.x[l + 1];
    launch_resid_restrict<T>(h, l, b, prev, cb, batch, active, s);
    vcycle_level<T>(h, V, l + 1, cb, cx, batch, active, s);
    if (cfg.n_post == 0) {
        T* dst = write_dst<T>(h, l, j, out, tmp);
        const Level& v = h->lev[l];
        const int64_t total = int64_t(batch) * h->nz * v.ncol;
        hipLaunchKernelGGL((k_prolong<T>), dim3(grid_for(total)), dim3(kBlock), 0, s, v.ncol,
                           h->nz, v.nvp, h->lev[l + 1].nvp, v.parent, prev, cx, dst, total);
        return;
    }
    for (int i = 0; i < cfg.n_post; ++i, ++j) {
        T* dst = write_dst<T>(h, l, j, out, tmp);
        int mode = kPlain;
        if (i == 0) mode = prev ? kProlong : kProlongZero;
        if (i > 0 && i == cfg.n_post - 1) sweep_last(prev, dst);
        else launch_sweep<T>(h, l, mode, b, prev, cx, dst, batch, active, s);
        prev = dst;
    }
}

// Whether a V-cycle of precision T can take b and hand out x in the ABI layout
// within its own kernels, without conversion passes: the finest level runs on
// patches, or begins with a sweep from zero and ends with a plain one on 32-
// column tiles (7-point operator; the others keep the passes: two more
// compiled forms of every sweep).
bool ends_in_plain_sweeps(const helmholtz_s* h) {
    const helmholtz_config& c = h->cfg;
    if (h->nine || h->weighted || h->lev[0].ncol < kSmallSweepCols) return false;
    return h->L == 1 ? c.n_coarse >= 2 : c.n_pre >= 1 && c.n_post >= 2;
}

template <typename T>
bool abi_within(const helmholtz_s* h) {
    return on_patches<T>(h, 0) || ends_in_plain_sweeps(h);
}

// Whether the last sweep of a CG preconditioner also forms r . z (kIoDot): as
// above, where the finest level never runs on patches (with the timing hook on
// it would run kernel by kernel, and the sums have one order), and the standard
// beta (the flexible one needs z . q too, of vectors that are in no cache).
bool dot_within(const helmholtz_s* h) {
    const bool mixed = h->cfg.mg_precision == HELMHOLTZ_FP32;
    return h->cfg.cg_variant == HELMHOLTZ_CG_STANDARD && ends_in_plain_sweeps(h) &&
           !(mixed ? patch_level<float>(h, 0) : patch_level<double>(h, 0));
}

int check_batch(const helmholtz_s* h, int32_t batch) {
    if (!h) return HELMHOLTZ_EINVAL;
    if (batch < 1 || batch > h->B) return HELMHOLTZ_ESHAPE;
    return HELMHOLTZ_OK;
}

// Finest-level vector between the ABI layout and the tiled layout, with a cast.
template <typename S, typename D, bool TO_TILED>
void retile(const helmholtz_s* h, const S* src, D* dst, int batch, hipStream_t s) {
    const Level& v = h->lev[0];
    hipLaunchKernelGGL((k_retile<S, D, TO_TILED>), dim3(v.ncolp / kTile * batch), dim3(kBlock), 0,
                       s, src, dst, v.ncol, h->nz, v.nvp);
}

// Algorithmic bytes of one V-cycle with these kernels (the words each kernel
// must move per unknown of its level, times the unknowns and the batch):
// first sweep from zero 4 words (b, two factors, x_new), further sweeps 7
// (b, x, two face couplings, two factors, x_new), residual + restriction 6.25
// (b, x, kh[2], kv, delta; a quarter-size coarse b), sweep with prolongation
// 7.25 (the coarse x), a lone prolongation 2.25; the 9-cell and the weighted
// operators add one word (kv2 or s) to every sweep and residual.
double vcycle_bytes(const helmholtz_s* h, int batch, size_t word) {
    const helmholtz_config& c = h->cfg;
    const double extra = (h->nine || h->weighted) ? 1.0 : 0.0;
    const double sw = 7.0 + extra;
    auto smooth = [&](int n) { return n > 0 ? 4.0 + sw * (n - 1) : 0.0; };
    double total = 0.0;
    for (int l = 0; l < h->L; ++l) {
        double w;
        if (l == h->L - 1) {
            w = smooth(c.n_coarse);
        } else {
            w = smooth(c.n_pre) + (c.n_pre > 0 ? 6.25 + extra : 1.25);
            w += c.n_post > 0 ? sw + 0.25 + sw * (c.n_post - 1) : 2.25;
        }
        total += w * double(h->nz) * h->lev[l].ncol;
    }
    return total * double(batch) * double(word);
}

// z = M r on the finest level in the handle's precision (tiled vectors). The
// float32 V-cycle reads r32 (the level-0 float32 right-hand side, which the
// Krylov kernels keep equal to float(r)) and leaves z32 in the level-0 float32
// solution buffer; r and z are then not touched. `prof`: time the V-cycle
// with the kernel timing hook (the solves). `dot`: leave the partial sums of
// r . z (dot_within).
int precondition(helmholtz_s* h, const double* r, double* z, int batch, const int* active,
                 hipStream_t s, bool prof, bool dot) {
    const bool mixed = h->cfg.mg_precision == HELMHOLTZ_FP32;
    prof = prof && prof_begin(h, HELMHOLTZ_PROF_VCYCLE, s);
    const AbiVectors with_r{nullptr, nullptr, false, r};
    const AbiVectors* io = dot ? &with_r : nullptr;
    if (!mixed) {
        vcycle_level<double>(h, h->vb64, 0, r, z, batch, active, s, io);
    } else {
        vcycle_level<float>(h, h->vb32, 0, h->vb32.b[0], h->vb32.x[0], batch, active, s, io);
    }
    if (prof) prof_end(h, HELMHOLTZ_PROF_VCYCLE, vcycle_bytes(h, batch, mixed ? 4 : 8), s);
    return last_error();
}

// Wait until the device has published sequence number `seq` for every
// right-hand side with need[i] != 0 (written by the last block of a norm
// reduction into host-coherent memory). Polls the flags; falls back on the
// stream state so that a failed launch cannot leave the host spinning.
int wait_published(helmholtz_s* h, hipStream_t s, const std::vector<int>& need, int seq) {
    using clock = std::chrono::steady_clock;
    const auto t0 = clock::now();
    for (unsigned spin = 1;; ++spin) {
        bool done = true;
        for (size_t i = 0; i < need.size(); ++i)
            if (need[i] && __atomic_load_n(&h->hseq[i], __ATOMIC_ACQUIRE) != seq) {
                done = false;
                break;
            }
        if (done) return HELMHOLTZ_OK;
        if (spin % 256 == 0) {
            const hipError_t q = hipStreamQuery(s);
            if (q == hipSuccess) {
                // the stream is idle: the values must be there now
                for (size_t i = 0; i < need.size(); ++i)
                    if (need[i] && __atomic_load_n(&h->hseq[i], __ATOMIC_ACQUIRE) != seq)
                        return HELMHOLTZ_EHIP;
                return HELMHOLTZ_OK;
            }
            if (q != hipErrorNotReady) return HELMHOLTZ_EHIP;
            if (clock::now() - t0 > std::chrono::seconds(120)) return HELMHOLTZ_EHIP;
        }
    }
}

// out = M u for tiled vectors of the V-cycle's precision.
template <typename T>
int precondition_into(helmholtz_s* h, const VBufs<T>& V, const T* u, T* out, int batch,
                      const int* active, hipStream_t s) {
    const bool prof = prof_begin(h, HELMHOLTZ_PROF_VCYCLE, s);
    vcycle_level<T>(h, V, 0, u, out, batch, active, s);
    if (prof) prof_end(h, HELMHOLTZ_PROF_VCYCLE, vcycle_bytes(h, batch, sizeof(T)), s);
    return last_error();
}

// Whether the Krylov scalars are formed by the kernels that use them instead of
// in launches of their own (kMergeMax): few partial sums, and few workgroups
// that add them up (for C192 x 70 an apply leaves 15552).
bool scalars_merged(const helmholtz_s* h) {
    const Level& v = h->lev[0];
    const int ntile0 = (v.ncol + kBlock - 1) / kBlock;
    const int nkc0 = (h->nz + kApplyChunk - 1) / kApplyChunk;
    return ntile0 * nkc0 <= kMergeMax && v.ncolp / kTile <= kMergeMax;
}

// Workgroups of a vector reduction over the finest level: a few elements per
// thread, at most kRedBlocks.
int reduction_blocks(const helmholtz_s* h) {
    return int(std::min<int64_t>(kRedBlocks, (h->nvp + 4 * kBlock - 1) / (4 * kBlock)));
}

// Right-preconditioned BiCGStab (Section 4.1) after the shared start
// (x = 0, r = r0 = b, rho = ||b||^2 published). Per iteration two products
// with H and two V-cycles; the inner products (r0, v), (t, s) with (t, t),
// and (r0, r) with ||r||^2 are the four global sums of Section 3.7. it/rel
// are updated for every right-hand side that was active in an iteration.
template <typename Z>
int bicgstab_loop(helmholtz_s* h, const VBufs<Z>& V, double* x, int batch, double rtol, int maxiter,
                  const std::vector<double>& bnorm2, std::vector<int32_t>& it,
                  std::vector<double>& rel, hipStream_t s) {
    const Level& v0 = h->lev[0];
    const int64_t n = h->nvp;
    const int ntile32 = v0.ncolp / kTile;
    const int ntile0 = (v0.ncol + kBlock - 1) / kBlock;
    const int nkc0 = (h->nz + kApplyChunk - 1) / kApplyChunk;
    const int nred = reduction_blocks(h);
    const dim3 red(nred * batch), blk(kBlock), fin(kFinBlock), tgrid(ntile32 * batch);
    const CgState st = cg_state(h);
    const int ndot = ntile0 * nkc0;
    const int merged = scalars_merged(h) ? ndot : 0;  // partial sums to add where they are used
    // a float32 V-cycle takes p and s rounded and leaves p_hat and s_hat in
    // float32 (in the memory of the float64 ones)
    constexpr bool mixed = sizeof(Z) == 4;
    float* const u32 = mixed ? h->vb32.b[0] : nullptr;
    Z* const ph = reinterpret_cast<Z*>(h->z);
    Z* const shat = reinterpret_cast<Z*>(h->sh);
    auto precondition_from = [&](const double* u, Z* out) -> int {
        if constexpr (mixed) return precondition_into<Z>(h, V, u32, out, batch, h->active, s);
        else return precondition_into<Z>(h, V, u, out, batch, h->active, s);
    };
    std::vector<int> was_active(batch);
    bool broke = false;
    // Everything of an iteration up to its x and r update skips the
    // right-hand sides whose device flag the last norm cleared, so, as in CG,
    // it is queued before the host reads that norm when the norm is predicted
    // to stay above 4x the tolerance (the update and the published norm are
    // queued after the read: the host mirror holds one iteration's values).
    const bool ahead = !h->prof_on;
    auto first_half = [&](int iter) -> int {
        // p = r + beta (p - omega v); p_hat = M p; v = H p_hat; alpha = rho / (r0, v)
        hipLaunchKernelGGL(k_bicg_p, red, blk, 0, s, h->r, h->q, h->p, u32, n, nred, h->sc,
                           h->active, iter == 1 ? 1 : 0);
        if (int e = precondition_from(h->p, ph)) return e;
        launch_apply<double, Z>(h, 0, ph, h->q, batch, kDotWY, h->active, s, h->r0);
        if (!merged)
            hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinBiAlpha), ndot, 0,
                               0.0);
        // s = r - alpha v; s_hat = M s; t = H s_hat; omega = (t, s) / (t, t)
        hipLaunchKernelGGL(k_bicg_s, red, blk, 0, s, h->r, h->q, h->s, u32, n, nred, st, merged);
        if (int e = precondition_from(h->s, shat)) return e;
        launch_apply<double, Z>(h, 0, shat, h->t, batch, kDotWYYY, h->active, s, h->s);
        if (!merged)
            hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinBiOmega), ndot, 0,
                               0.0);
        return last_error();
    };
    std::vector<double> fac(batch, 0.05), rel_prev(batch, 1.0);
    auto expect_more = [&]() {
        for (int i = 0; i < batch; ++i)
            if (h->hact[i] && rel_prev[i] * fac[i] > 4.0 * rtol) return true;
        return false;
    };
    if (int e = first_half(1)) return e;
    for (int iter = 1;; ++iter) {
        for (int i = 0; i < batch; ++i) was_active[i] = h->hact[i];
        // x += alpha p_hat + omega s_hat; r = s - omega t; (r0, r), ||r||^2, published
        hipLaunchKernelGGL((k_bicg_xr<Z>), tgrid, blk, 0, s, x, h->r, ph, shat, h->s, h->t, h->r0,
                           v0.ncol, h->nz, v0.nvp, st, merged);
        hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinBiRR), ntile32, iter,
                           0.0);
        const bool queued = ahead && iter < maxiter && expect_more();
        if (queued)
            if (int e = first_half(iter + 1)) return e;
        if (last_error() != HELMHOLTZ_OK) return HELMHOLTZ_EHIP;
        if (int e = wait_published(h, s, was_active, iter)) return e;
        bool still = false;
        for (int i = 0; i < batch; ++i) {
            if (!was_active[i]) continue;
            it[i] = iter;
            const double rr = h->hsc[i * kScal + kRR];
            if (!std::isfinite(rr)) {
                HH_CHECK(hipStreamSynchronize(s));
                return HELMHOLTZ_ENONFINITE;
            }
            rel[i] = std::sqrt(rr / bnorm2[i]);
            fac[i] = rel[i] / rel_prev[i];
            rel_prev[i] = rel[i];
            broke = broke || h->hsc[i * kScal + kBreak] != 0.0;
            still = still || h->hact[i];
        }
        if (!still) break;
        if (iter >= maxiter) {
            broke = true;
            break;
        }
        if (!queued)
            if (int e = first_half(iter + 1)) return e;
    }
    // the caller may read x as soon as this returns on the host
    HH_CHECK(hipStreamSynchronize(s));
    return broke ? HELMHOLTZ_NOT_CONVERGED : HELMHOLTZ_OK;
}

int create_impl(const helmholtz_config* cfg, const double* kh, const double* kv,
                const double* kv2, const double* delta, const double* sw, void* workspace,
                size_t workspace_bytes, helmholtz_stream_t stream_, helmholtz_t* out);
int set_coefficients(helmholtz_s* h, const double* kh, const double* kv, const double* kv2,
                     const double* delta, const double* sw, hipStream_t s);

// Level vectors b, x, t of every level for `batch` right-hand sides, carved
// from `base`; returns the bytes they take.
template <typename T>
size_t carve_levels(const helmholtz_s* h, uintptr_t base, int batch, VBufs<T>& V) {
    Carver cv{base};
    for (int l = 0; l < h->L; ++l) {
        const size_t nv = size_t(batch) * size_t(h->lev[l].nvp);
        V.b[l] = cv.take<T>(nv);
        V.x[l] = cv.take<T>(nv);
        V.t[l] = cv.take<T>(nv);
    }
    return cv.off;
}

// Whether the caller's vectors a and b ([batch][nz][ncol]) share memory.
template <typename S>
bool overlap(const helmholtz_s* h, const S* a, const S* b, int batch) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return (p < q ? q - p : p - q) < uintptr_t(batch) * uintptr_t(h->n) * sizeof(S);
}

// One V-cycle from the ABI layout to the ABI layout, in V; bt and xt are the
// tiled vectors of the finest level. On patches the last leg reads b of the
// columns around a patch while other workgroups store x, so where the two
// overlap the conversion passes run: all of b is then read before any of x is
// written, as it is by the first and the last of the single sweeps.
template <typename T, typename S>
int vcycle_abi(helmholtz_s* h, const VBufs<T>& V, T* bt, T* xt, const S* b, S* x, int batch,
               hipStream_t s) {
    if (abi_within<T>(h) && !(on_patches<T>(h, 0) && overlap(h, b, x, batch))) {
        const AbiVectors io{b, x, sizeof(S) != sizeof(T)};
        vcycle_level<T>(h, V, 0, bt, xt, batch, nullptr, s, &io);
    } else {
        retile<S, T, true>(h, b, bt, batch, s);
        vcycle_level<T>(h, V, 0, bt, xt, batch, nullptr, s);
        retile<T, S, false>(h, xt, x, batch, s);
    }
    return last_error();
}

// One V-cycle from the ABI layout to the ABI layout with the level vectors in
// the static scratch array (helmholtz_vcycle_noalloc).
template <typename T>
int vcycle_in_scratch(helmholtz_s* h, const double* b, double* x, int batch, hipStream_t s) {
    VBufs<T> V;
    if (carve_levels<T>(h, reinterpret_cast<uintptr_t>(h->scratch), batch, V) > kScratchBytes)
        return HELMHOLTZ_ESCRATCH;
    return vcycle_abi<T, double>(h, V, V.b[0], V.x[0], b, x, batch, s);
}

// Weighted handles run the calls that take H^T with the transposed kernels.
struct AdjointScope {
    helmholtz_s* h;
    bool old;
    explicit AdjointScope(helmholtz_s* h_) : h(h_), old(h_->adj) { h->adj = h->weighted; }
    ~AdjointScope() { h->adj = old; }
};

}  // namespace

// ===========================================================================
extern "C" {

size_t helmholtz_workspace_bytes(const helmholtz_config* cfg) {
    if (!config_ok(cfg) || shape_error(cfg) != HELMHOLTZ_OK) return 0;
    helmholtz_s tmp;
    init_shape(&tmp, cfg);
    Carver cv{0};
    layout(&tmp, cv);
    return cv.off;
}

const char* helmholtz_strerror(int code) {
    switch (code) {
        case HELMHOLTZ_OK: return "ok";
        case HELMHOLTZ_NOT_CONVERGED: return "solve reached maxiter before rtol";
        case HELMHOLTZ_EINVAL: return "invalid argument, configuration or coefficient";
        case HELMHOLTZ_ESHAPE: return "invalid shape (N, nz, levels or batch)";
        case HELMHOLTZ_EWORKSPACE: return "workspace missing, too small or misaligned";
        case HELMHOLTZ_ENONFINITE: return "non-finite value (NaN or Inf)";
        case HELMHOLTZ_EHIP: return "HIP runtime error";
        case HELMHOLTZ_ESCRATCH:
            return "level vectors exceed the static scratch of the allocation-free entry point";
        default: return "unknown error code";
    }
}

int helmholtz_mesh_tables(int32_t N, int32_t* nbr, int32_t* ftab, int32_t* parent) {
    if (N < 1 || !nbr || !ftab) return HELMHOLTZ_EINVAL;
    if (2 * 6 * int64_t(N) * N >= (int64_t(1) << 31)) return HELMHOLTZ_ESHAPE;
    build_neighbours(N, nbr);
    build_face_table(N, nbr, ftab);
    if (parent && N % 2 == 0) build_parent(N, parent);
    return HELMHOLTZ_OK;
}

int helmholtz_create(const helmholtz_config* cfg, const double* kh, const double* kv,
                     const double* delta, void* workspace, size_t workspace_bytes,
                     helmholtz_stream_t stream_, helmholtz_t* out) {
    if (!out) return HELMHOLTZ_EINVAL;
    *out = nullptr;
    if (config_ok(cfg) && (cfg->stencil == 9 || cfg->weighted)) return HELMHOLTZ_EINVAL;
    return create_impl(cfg, kh, kv, nullptr, delta, nullptr, workspace, workspace_bytes, stream_,
                       out);
}

int helmholtz_create9(const helmholtz_config* cfg, const double* kh, const double* kv,
                      const double* kv2, const double* delta, void* workspace,
                      size_t workspace_bytes, helmholtz_stream_t stream_, helmholtz_t* out) {
    if (!out) return HELMHOLTZ_EINVAL;
    *out = nullptr;
    if (config_ok(cfg) && cfg->weighted) return HELMHOLTZ_EINVAL;
    return create_impl(cfg, kh, kv, kv2, delta, nullptr, workspace, workspace_bytes, stream_, out);
}

int helmholtz_create_weighted(const helmholtz_config* cfg, const double* kh, const double* kv,
                              const double* delta, const double* s, void* workspace,
                              size_t workspace_bytes, helmholtz_stream_t stream_,
                              helmholtz_t* out) {
    if (!out) return HELMHOLTZ_EINVAL;
    *out = nullptr;
    if (config_ok(cfg) && (!cfg->weighted || !s)) return HELMHOLTZ_EINVAL;
    return create_impl(cfg, kh, kv, nullptr, delta, s, workspace, workspace_bytes, stream_, out);
}

}  // extern "C"

namespace {

int create_impl(const helmholtz_config* cfg, const double* kh, const double* kv,
                const double* kv2, const double* delta, const double* sw, void* workspace,
                size_t workspace_bytes, helmholtz_stream_t stream_, helmholtz_t* out) {
    if (!out) return HELMHOLTZ_EINVAL;
    *out = nullptr;
    if (!config_ok(cfg)) return HELMHOLTZ_EINVAL;
    if (int e = shape_error(cfg)) return e;
    if (!kh || !delta || (cfg->nz > 1 && !kv)) return HELMHOLTZ_EINVAL;
    const bool nine = cfg->stencil == 9;
    if (nine != (kv2 != nullptr) && !(nine && cfg->nz <= 2)) return HELMHOLTZ_EINVAL;
    if ((cfg->weighted == 1) != (sw != nullptr)) return HELMHOLTZ_EINVAL;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % HELMHOLTZ_WORKSPACE_ALIGN))
        return HELMHOLTZ_EWORKSPACE;
    const size_t need = helmholtz_workspace_bytes(cfg);
    if (workspace_bytes < need) return HELMHOLTZ_EWORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
    // padding columns of the tiled arrays must read as zero
    if (hipMemsetAsync(workspace, 0, need, s) != hipSuccess) return HELMHOLTZ_EHIP;

    helmholtz_s* h = new (std::nothrow) helmholtz_s;
    if (!h) return HELMHOLTZ_EINVAL;
    init_shape(h, cfg);
    Carver cv{reinterpret_cast<uintptr_t>(workspace)};
    layout(h, cv);
    h->ws_bytes = need;
    auto fail = [&](int code) {
        helmholtz_destroy(h);
        return code;
    };
    if (int e = scratch_of_current_device(&h->scratch, &h->device)) return fail(e);
    // host-coherent pinned memory: the device publishes the CG scalars here
    if (hipHostMalloc(reinterpret_cast<void**>(&h->hsc),
                      size_t(h->B) * kScal * sizeof(double) + size_t(h->B) * 2 * sizeof(int) + 16,
                      hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess) {
        h->hsc = nullptr;
        return fail(HELMHOLTZ_EHIP);
    }
    h->hact = reinterpret_cast<int*>(h->hsc + size_t(h->B) * kScal);
    h->hseq = h->hact + h->B;
    h->hflags = h->hseq + h->B;
    for (int i = 0; i < h->B; ++i) h->hseq[i] = -1;

    // mesh tables of every level, built on the host and copied at once
    const int nz = h->nz;
    // (not cleared: every table is written whole)
    std::unique_ptr<unsigned char[]> tables(new (std::nothrow) unsigned char[h->table_bytes]);
    if (!tables) return fail(HELMHOLTZ_EINVAL);
    auto host = [&](auto* device) {  // where a table's host image stands
        return reinterpret_cast<decltype(device)>(
            tables.get() + (reinterpret_cast<uintptr_t>(device) -
                             reinterpret_cast<uintptr_t>(workspace)));
    };
    std::vector<int32_t> ft;
    for (int l = 0; l < h->L; ++l) {
        Level& v = h->lev[l];
        const size_t nc = size_t(v.ncol);
        int32_t* const nbr = host(v.nbr);
        build_neighbours(v.N, nbr);
        ft.resize(4 * nc);
        build_face_table(v.N, nbr, ft.data());
        // W and S faces: stored face slot * ncol + owner -> offset in the tiled kh
        uint32_t* const ff = host(v.fface);
        for (size_t c = 0; c < nc; ++c) {
            for (int w = 0; w < 2; ++w) {
                const int32_t f = ft[(w == 0 ? 1 : 3) * nc + c];
                const int slot = f >= v.ncol ? 1 : 0, owner = f - slot * v.ncol;
                ff[w * nc + c] = uint32_t(slot) * uint32_t(v.nvp) +
                                 uint32_t((owner / kTile) * kTile * nz + owner % kTile);
            }
        }
        if (v.parent) {
            int32_t* const par = host(v.parent);
            build_parent(v.N, par);
            // prolongation offsets: the parent and the parents of the outward
            // E/W (W for even i, E for odd i) and N/S (S for even j, N for
            // odd j) neighbours, as tiled offsets on the coarse level
            auto tb = [&](int32_t cc) { return (cc >> 5) * (kTile * nz) + (cc & (kTile - 1)); };
            int32_t* const po = host(v.pofs);
            for (size_t c = 0, i = 0, j = 0; c < nc; ++c) {
                const int32_t ew = nbr[((i & 1) ? 0 : 1) * nc + c];
                const int32_t ns = nbr[((j & 1) ? 2 : 3) * nc + c];
                po[c] = tb(par[c]);
                po[nc + c] = tb(par[ew]);
                po[2 * nc + c] = tb(par[ns]);
                if (++i == size_t(v.N)) {
                    i = 0;
                    if (++j == size_t(v.N)) j = 0;
                }
            }
        }
        if (v.child) build_children(v.N, host(v.child));
        if (v.patch >= 0) {
            const PatchShape& S = kPatchShapes[v.patch];
            int32_t* const col = host(v.pcol);
            build_patches(v.N, nbr, S.pw, S.ph, S.depth, S.ncp, col, host(v.plnb), host(v.pcnt));
            const int32_t* par = v.parent ? host(v.parent) : nullptr;
            int32_t* const ppar = host(v.ppar);
            for (size_t i = 0; i < size_t(v.npatch) * S.ncp; ++i) ppar[i] = par ? par[col[i]] : 0;
        }
    }
    // the host image must stay alive until the copy has run
    if (hipMemcpyAsync(workspace, tables.get(), h->table_bytes, hipMemcpyHostToDevice, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return fail(HELMHOLTZ_EHIP);

    if (int e = set_coefficients(h, kh, kv, kv2, delta, sw, s)) return fail(e);
    *out = h;
    return HELMHOLTZ_OK;
}

// Coefficients of every level: finest from the caller (validated), coarser by
// re-discretisation, then the column factors and the float32 copies.
// Synchronises `s` once.
int set_coefficients(helmholtz_s* h, const double* kh, const double* kv, const double* kv2,
                     const double* delta, const double* sw, hipStream_t s) {
    const int nz = h->nz;
    if (hipMemsetAsync(h->flags, 0, 4 * sizeof(int), s) != hipSuccess) return HELMHOLTZ_EHIP;
    {
        Level& v = h->lev[0];
        const int64_t nv = int64_t(nz) * v.ncol;
        hipLaunchKernelGGL(k_setup_fine, dim3(grid_for(nv)), dim3(kBlock), 0, s, v.ncol, nz,
                           v.nvp, kh, kv, delta, kv2, sw, v.d.kh, v.d.kv, v.d.dl,
                           kv2 ? v.d.kv2 : nullptr, sw ? v.d.s : nullptr, h->flags);
    }
    for (int l = 1; l < h->L; ++l) {
        Level& f = h->lev[l - 1];
        Level& c = h->lev[l];
        const int64_t nv = int64_t(nz) * c.ncol;
        hipLaunchKernelGGL(k_coarsen, dim3(grid_for(nv)), dim3(kBlock), 0, s, c.ncol, nz, f.nvp,
                           c.nvp, c.child, f.d.kh, f.d.kv, f.d.dl, f.d.kv2, f.d.s, c.d.kh,
                           c.d.kv, c.d.dl, c.d.kv2, c.d.s);
    }
    // factors and float32 copies of every level, then the coefficients of the
    // levels on patches
    const bool f64 = h->cfg.mg_precision == HELMHOLTZ_FP64;
    SetupLevels all{}, patched{};
    int tiles = 0, ptiles = 0;
    for (int l = 0; l < h->L; ++l) {
        const Level& v = h->lev[l];
        SetupLevel S{v.ncol, v.nvp, tiles, v.fface, v.d.kh, v.d.kv, v.d.dl, v.d.kv2, v.d.s,
                     f64 ? v.d.cc : nullptr, f64 ? v.d.mm : nullptr, v.f.kh, v.f.kv, v.f.dl,
                     v.f.cc, v.f.mm, v.f.kv2, v.f.s, v.d.co, v.f.co};
        all.lev[all.count++] = S;
        tiles += v.ncolp / kTile;
        if (!v.d.co && !v.f.co) continue;
        S.tile0 = ptiles;
        patched.lev[patched.count++] = S;
        ptiles += v.ncolp / kTile;
    }
    hipLaunchKernelGGL(k_factor_levels, dim3(tiles), dim3(kBlock),
                       2 * size_t(nz) * kTile * sizeof(double), s, all, nz, sweep_mid(nz));
    if (ptiles)
        hipLaunchKernelGGL(k_patch_coefficients, dim3(ptiles, kColPlanes), dim3(kBlock), 0, s,
                           patched, nz, sweep_mid(nz),
                           kPatchLanes * patch_levels(nz, !h->nine && !h->weighted));
    if (last_error() != HELMHOLTZ_OK) return HELMHOLTZ_EHIP;
    if (hipMemcpyAsync(h->hflags, h->flags, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess)
        return HELMHOLTZ_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return HELMHOLTZ_EHIP;
    if (h->hflags[0] & 1) return HELMHOLTZ_ENONFINITE;
    if (h->hflags[0] & 2) return HELMHOLTZ_EINVAL;
    return HELMHOLTZ_OK;
}

}  // namespace

extern "C" {

int helmholtz_update(helmholtz_t h, const double* kh, const double* kv, const double* kv2,
                     const double* delta, const double* s, helmholtz_stream_t stream) {
    if (!h || !kh || !delta || (h->nz > 1 && !kv)) return HELMHOLTZ_EINVAL;
    if ((kv2 != nullptr) != (h->nine && h->nz > 2)) return HELMHOLTZ_EINVAL;
    if ((s != nullptr) != h->weighted) return HELMHOLTZ_EINVAL;
    return set_coefficients(h, kh, kv, kv2, delta, s, reinterpret_cast<hipStream_t>(stream));
}

int helmholtz_profile_enable(helmholtz_t h, int enable) {
    if (!h) return HELMHOLTZ_EINVAL;
    for (int k = 0; k < HELMHOLTZ_PROF_COUNT; ++k) {
        if (int e = prof_flush(h, k)) return e;
        h->prof[k].ms = h->prof[k].bytes = 0.0;
        h->prof[k].launches = 0;
    }
    h->prof_on = enable != 0;
    return HELMHOLTZ_OK;
}

int helmholtz_profile_read(helmholtz_t h, int32_t kernel, double* ms, int64_t* launches,
                           double* bytes) {
    if (!h || kernel < 0 || kernel >= HELMHOLTZ_PROF_COUNT) return HELMHOLTZ_EINVAL;
    if (int e = prof_flush(h, kernel)) return e;
    if (ms) *ms = h->prof[kernel].ms;
    if (launches) *launches = h->prof[kernel].launches;
    if (bytes) *bytes = h->prof[kernel].bytes;
    return HELMHOLTZ_OK;
}

int helmholtz_destroy(helmholtz_t h) {
    if (!h) return HELMHOLTZ_EINVAL;
    for (int k = 0; k < HELMHOLTZ_PROF_COUNT; ++k) (void)prof_flush(h, k);
    if (h->hsc) (void)hipHostFree(h->hsc);
    delete h;
    return HELMHOLTZ_OK;
}

int helmholtz_apply(helmholtz_t h, const double* x, double* y, int32_t batch,
                    helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!x || !y) return HELMHOLTZ_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (overlap(h, x, y, batch)) {
        // y would overwrite x that other workgroups have yet to read
        retile<double, double, true>(h, x, h->p, batch, s);
        launch_apply<double>(h, 0, h->p, h->q, batch, kDotXY, nullptr, s);
        retile<double, double, false>(h, h->q, y, batch, s);
    } else {
        launch_apply_natural(h, x, y, batch, s);
    }
    return last_error();
}

int helmholtz_vcycle(helmholtz_t h, const double* b, double* x, int32_t batch,
                     helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!b || !x) return HELMHOLTZ_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (h->cfg.mg_precision == HELMHOLTZ_FP64)
        return vcycle_abi<double, double>(h, h->vb64, h->r, h->z, b, x, batch, s);
    return vcycle_abi<float, double>(h, h->vb32, h->vb32.b[0], h->vb32.x[0], b, x, batch, s);
}

int helmholtz_vcycle_noalloc(helmholtz_t h, const double* b, double* x, int32_t batch,
                             helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!b || !x) return HELMHOLTZ_EINVAL;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return HELMHOLTZ_EHIP;
    if (dev != h->device || !h->scratch) return HELMHOLTZ_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (h->cfg.mg_precision == HELMHOLTZ_FP64) return vcycle_in_scratch<double>(h, b, x, batch, s);
    return vcycle_in_scratch<float>(h, b, x, batch, s);
}

int helmholtz_vcycle_f32(helmholtz_t h, const float* b, float* x, int32_t batch,
                         helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!b || !x) return HELMHOLTZ_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    return vcycle_abi<float, float>(h, h->vb32, h->vb32.b[0], h->vb32.x[0], b, x, batch, s);
}

int helmholtz_solve(helmholtz_t h, const double* b, double* x, int32_t batch, double rtol,
                    int32_t maxiter, int32_t* iters, double* relres, helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!b || !x || maxiter < 1 || !(rtol >= 0.0)) return HELMHOLTZ_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t n = h->nvp;  // tiled vector length (elementwise kernels)
    const Level& v0 = h->lev[0];
    const int ntile32 = v0.ncolp / kTile;
    const dim3 tgrid(ntile32 * batch);
    const bool mixed = h->cfg.mg_precision == HELMHOLTZ_FP32;
    const bool flex = h->cfg.cg_variant == HELMHOLTZ_CG_FLEXIBLE;
    const bool bicg = h->cfg.cg_variant == HELMHOLTZ_BICGSTAB;
    float* r32 = mixed && !bicg ? h->vb32.b[0] : nullptr;
    float* z32 = mixed ? h->vb32.x[0] : nullptr;
    const bool dotted = dot_within(h);
    const int nred = dotted ? ntile32 : reduction_blocks(h);  // partial sums of r . z
    const dim3 red(nred * batch), blk(kBlock), fin(kFinBlock);
    const CgState st = cg_state(h);
    const int ndot = ((v0.ncol + kBlock - 1) / kBlock) *
                     ((h->nz + kApplyChunk - 1) / kApplyChunk);  // partial sums of an apply
    const bool merged = scalars_merged(h);
    int rho = kRho;  // where rho stands (alternates if merged)

    for (int i = 0; i < batch; ++i) __atomic_store_n(&h->hseq[i], -1, __ATOMIC_RELEASE);
    // x = 0, r = b, ||b||^2
    // (CG writes x in its first update; the right-hand sides that do not
    // start are zeroed after the norms)
    hipLaunchKernelGGL(k_cg_init, tgrid, blk, 0, s, b, bicg ? x : nullptr, h->r, r32,
                       bicg ? h->r0 : nullptr, v0.ncol, h->nz, v0.nvp, st);
    hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinBB), ntile32, 0,
                       rtol * rtol);
    if (last_error() != HELMHOLTZ_OK) return HELMHOLTZ_EHIP;

    // vectors far larger than the last-level cache: the streams that are not
    // read again soon bypass it (see the kernels)
    const bool vnt = streams_past_cache(h, 0, batch, sizeof(double));
    auto dot_rz = [&](const double* q) {
        if (dotted) {
            if (!h->prof_on) return;  // the preconditioner's last sweep has left them
            if (mixed)
                hipLaunchKernelGGL(k_dot_tiles<float>, tgrid, blk, 0, s, h->r, z32, v0.ncol,
                                   h->nz, v0.nvp, st);
            else
                hipLaunchKernelGGL(k_dot_tiles<double>, tgrid, blk, 0, s, h->r, h->z, v0.ncol,
                                   h->nz, v0.nvp, st);
            return;
        }
        const int rev = h->flip(0);
        auto go = [&](auto kern, auto z) {
            hipLaunchKernelGGL(kern, red, blk, 0, s, h->r, z, q, n, nred, st, rev);
        };
        if (mixed) vnt ? go(k_dot_rz<float, true>, z32) : go(k_dot_rz<float, false>, z32);
        else vnt ? go(k_dot_rz<double, true>, h->z) : go(k_dot_rz<double, false>, h->z);
    };
    // p = z + beta p, with the x update owed from the last iteration (xmode)
    auto p_update = [&](int init, int xmode) {
        const int rev = h->flip(0);
        auto go = [&](auto kern, auto z) {
            hipLaunchKernelGGL(kern, tgrid, blk, 0, s, z, h->p, x, v0.ncol, h->nz, v0.nvp, st,
                               init, xmode, merged ? nred : 0, rho, int(flex), rev);
            if (merged) rho = rho == kRho ? int(kRho2) : int(kRho);
        };
        if (mixed) vnt ? go(k_p_update<float, true>, z32) : go(k_p_update<float, false>, z32);
        else vnt ? go(k_p_update<double, true>, h->z) : go(k_p_update<double, false>, h->z);
    };
    // the owed x update where the iteration stops, for the right-hand sides
    // that `sel` names (see k_cg_x)
    auto x_update = [&](int xmode, int sel) {
        const int rev = h->flip(0);
        if (vnt)
            hipLaunchKernelGGL(k_cg_x<true>, tgrid, blk, 0, s, x, h->p, v0.ncol, h->nz, v0.nvp,
                               st, xmode, sel, rev);
        else
            hipLaunchKernelGGL(k_cg_x<false>, tgrid, blk, 0, s, x, h->p, v0.ncol, h->nz, v0.nvp,
                               st, xmode, sel, rev);
    };
    // z = M r, rho = r.z, p = z
    auto cg_start = [&]() -> int {
        if (int e = precondition(h, h->r, h->z, batch, h->active, s, true, dotted && !h->prof_on)) return e;
        dot_rz(nullptr);
        if (!merged)
            hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinRho), nred, 0, 0.0);
        p_update(1, kXNone);
        return last_error();
    };
    // z = M r and beta of the next iteration
    auto cg_next_m = [&]() -> int {
        if (int e = precondition(h, h->r, h->z, batch, h->active, s, true, dotted && !h->prof_on)) return e;
        dot_rz(flex ? h->q : nullptr);
        if (!merged)
            hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st,
                               int(flex ? kFinBetaFlex : kFinBeta), nred, 0, 0.0);
        return last_error();
    };

    // Work queued ahead of the host's decisions. The host reads each published
    // norm before it decides how to go on, and the GPU would sit idle through
    // that round trip and the next launch (~25 us; about 2.5 % of a float32
    // solve at C192 x 70). Every kernel of M r, r.z and beta skips the
    // right-hand sides whose device flag the norm reduction cleared, so the
    // host may queue them before it knows the norm: the results are the same
    // either way, and a wrong guess costs only launches that return at once.
    // Off while the timing hooks are on, so that each timed V-cycle is a whole
    // one.
    const bool ahead = !bicg && !h->prof_on;
    if (ahead)
        if (int e = cg_start()) return e;  // b = 0 or not finite: flag cleared

    std::vector<int> need(batch, 1);
    if (int e = wait_published(h, s, need, 0)) return e;
    std::vector<double> bnorm2(batch);
    std::vector<int32_t> it(batch, 0);
    std::vector<double> rel(batch, 0.0);
    bool any = false, finite = true;
    for (int i = 0; i < batch; ++i) {
        bnorm2[i] = h->hsc[i * kScal + kBB];
        finite = finite && std::isfinite(bnorm2[i]);
        any = any || h->hact[i];
        rel[i] = h->hact[i] ? 1.0 : 0.0;
    }
    auto finish = [&](int status) {
        for (int i = 0; i < batch; ++i) {
            if (iters) iters[i] = it[i];
            if (relres) relres[i] = rel[i];
        }
        return status;
    };
    // x of the right-hand sides that do not start (b = 0 or not finite)
    bool idle = false;
    for (int i = 0; i < batch; ++i) idle = idle || !h->hact[i];
    if (idle && !bicg)
        hipLaunchKernelGGL(k_cg_zero_idle, tgrid, blk, 0, s, x, v0.ncol, h->nz, st);
    if (!finite || !any) HH_CHECK(hipStreamSynchronize(s));
    if (!finite) return HELMHOLTZ_ENONFINITE;
    if (!any) return finish(HELMHOLTZ_OK);
    if (bicg)
        return finish(mixed ? bicgstab_loop<float>(h, h->vb32, x, batch, rtol, maxiter, bnorm2, it,
                                                   rel, s)
                            : bicgstab_loop<double>(h, h->vb64, x, batch, rtol, maxiter, bnorm2,
                                                    it, rel, s));
    if (!ahead)
        if (int e = cg_start()) return e;

    // The next norm predicted from the last one and the last contraction
    // (1/20 before there is one): if some right-hand side is expected to stay
    // above 4x the tolerance, M r of the next iteration is queued ahead;
    // otherwise the x update of those that stop is.
    std::vector<double> fac(batch, 0.05), rel_prev(batch, 1.0);
    auto expect_more = [&]() {
        for (int i = 0; i < batch; ++i)
            if (h->hact[i] && rel_prev[i] * fac[i] > 4.0 * rtol) return true;
        return false;
    };

    std::vector<int> was_active(batch);
    int status = HELMHOLTZ_OK;
    for (int iter = 1;; ++iter) {
        for (int i = 0; i < batch; ++i) was_active[i] = h->hact[i];
        const bool more = ahead && iter < maxiter && expect_more();
        // q = H p, alpha = rho / p.q
        launch_apply<double>(h, 0, h->p, h->q, batch, kDotXY, h->active, s);
        if (!merged)
            hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinAlpha), ndot, 0,
                               0.0);
        // r -= alpha q, ||r||^2 and the convergence flags, published; the
        // matching x += alpha p is owed (applied with the next p update, or
        // by x_update where the iteration stops)
        const int rev = h->flip(0);
        if (vnt)
            hipLaunchKernelGGL(k_cg_update<true>, tgrid, blk, 0, s, h->r, r32, h->q, v0.ncol,
                               h->nz, v0.nvp, st, merged ? ndot : 0, rho, rev);
        else
            hipLaunchKernelGGL(k_cg_update<false>, tgrid, blk, 0, s, h->r, r32, h->q, v0.ncol,
                               h->nz, v0.nvp, st, merged ? ndot : 0, rho, rev);
        hipLaunchKernelGGL(k_finalize, dim3(batch), fin, 0, s, st, int(kFinRR), ntile32, iter,
                           0.0);
        const int xmode = iter == 1 ? kXSet : kXAdd;  // x is first written here
        // queued ahead of the norm: M r of the next iteration, or the x update
        // of the right-hand sides that stop here (no-op for the others)
        const bool queued_m = more, queued_x = ahead && !more;
        if (queued_m)
            if (int e = cg_next_m()) return e;
        if (queued_x) x_update(xmode, kXDone);
        if (last_error() != HELMHOLTZ_OK) return HELMHOLTZ_EHIP;
        if (int e = wait_published(h, s, was_active, iter)) return e;
        bool still = false, some_done = false;
        for (int i = 0; i < batch; ++i) {
            if (!was_active[i]) continue;
            it[i] = iter;
            const double rr = h->hsc[i * kScal + kRR];
            if (!std::isfinite(rr)) {
                HH_CHECK(hipStreamSynchronize(s));
                return finish(HELMHOLTZ_ENONFINITE);
            }
            rel[i] = std::sqrt(rr / bnorm2[i]);
            fac[i] = rel[i] / rel_prev[i];
            rel_prev[i] = rel[i];
            still = still || h->hact[i];
            some_done = some_done || !h->hact[i];
        }
        if (!still || iter >= maxiter) {
            if (!queued_x) x_update(xmode, kXAll);
            else if (still) x_update(xmode, kXLive);
            if (still) status = HELMHOLTZ_NOT_CONVERGED;
            break;
        }
        if (some_done && !queued_x) x_update(xmode, kXDone);
        // z = M r, beta (unless queued ahead), p = z + beta p (with the owed
        // x update)
        if (!queued_m)
            if (int e = cg_next_m()) return e;
        p_update(0, xmode);
    }
    // the caller may read x as soon as this returns on the host
    HH_CHECK(hipStreamSynchronize(s));
    return finish(status);
}

int helmholtz_bandwidth_kernel(int32_t kind, const float* a, const float* b, float* c, int64_t n,
                               float sv, helmholtz_stream_t stream) {
    if (n <= 0 || n % 4 != 0) return HELMHOLTZ_EINVAL;
    const int64_t nblk = (n + kStreamPerBlock - 1) / kStreamPerBlock;
    if (nblk >= (int64_t(1) << 31)) return HELMHOLTZ_ESHAPE;
    auto aligned = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const float4* a4 = reinterpret_cast<const float4*>(a);
    const float4* b4 = reinterpret_cast<const float4*>(b);
    float4* c4 = reinterpret_cast<float4*>(c);
    const int64_t n4 = n / 4;
    const dim3 grid(static_cast<unsigned>(nblk)), blk(kBlock);
    switch (kind) {
        case HELMHOLTZ_BW_READ:
            if (!a || !c || !aligned(a)) return HELMHOLTZ_EINVAL;
            hipLaunchKernelGGL(k_stream<kStreamRead>, grid, blk, 0, s, a4, b4, c4, n4, sv, c);
            break;
        case HELMHOLTZ_BW_WRITE:
            if (!c || !aligned(c)) return HELMHOLTZ_EINVAL;
            hipLaunchKernelGGL(k_stream<kStreamWrite>, grid, blk, 0, s, a4, b4, c4, n4, sv, c);
            break;
        case HELMHOLTZ_BW_COPY:
            if (!a || !c || !aligned(a) || !aligned(c)) return HELMHOLTZ_EINVAL;
            hipLaunchKernelGGL(k_stream<kStreamCopy>, grid, blk, 0, s, a4, b4, c4, n4, sv, c);
            break;
        case HELMHOLTZ_BW_TRIAD:
            if (!a || !b || !c || !aligned(a) || !aligned(b) || !aligned(c)) return HELMHOLTZ_EINVAL;
            hipLaunchKernelGGL(k_stream<kStreamTriad>, grid, blk, 0, s, a4, b4, c4, n4, sv, c);
            break;
        default:
            return HELMHOLTZ_EINVAL;
    }
    return last_error();
}

int helmholtz_face_grad(helmholtz_t h, const double* lam, const double* x, int32_t batch,
                        double* g_kh, double* g_kv, double* g_delta, helmholtz_stream_t stream) {
    return helmholtz_face_grad9(h, lam, x, batch, g_kh, g_kv, nullptr, g_delta, stream);
}

int helmholtz_face_grad9(helmholtz_t h, const double* lam, const double* x, int32_t batch,
                         double* g_kh, double* g_kv, double* g_kv2, double* g_delta,
                         helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!lam || !x || !g_kh || !g_delta || (h->nz > 1 && !g_kv)) return HELMHOLTZ_EINVAL;
    if (g_kv2 && !h->nine) return HELMHOLTZ_EINVAL;
    if (h->weighted) return HELMHOLTZ_EINVAL;  // helmholtz_face_grad_weighted
    const Level& v = h->lev[0];
    const int64_t total = int64_t(h->nz) * v.ncol;
    const int grid = int((total + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_face_grad, dim3(grid), dim3(kBlock), 0,
                       reinterpret_cast<hipStream_t>(stream), v.ncol, h->nz, v.nbr, lam, x, batch,
                       g_kh, g_kv, g_delta, h->nz > 2 ? g_kv2 : nullptr);
    return last_error();
}

int helmholtz_apply_adjoint(helmholtz_t h, const double* x, double* y, int32_t batch,
                            helmholtz_stream_t stream) {
    if (!h) return HELMHOLTZ_EINVAL;
    AdjointScope scope(h);
    return helmholtz_apply(h, x, y, batch, stream);
}

int helmholtz_vcycle_adjoint(helmholtz_t h, const double* b, double* x, int32_t batch,
                             helmholtz_stream_t stream) {
    if (!h) return HELMHOLTZ_EINVAL;
    AdjointScope scope(h);
    return helmholtz_vcycle(h, b, x, batch, stream);
}

int helmholtz_solve_adjoint(helmholtz_t h, const double* g, double* lam, int32_t batch,
                            double rtol, int32_t maxiter, int32_t* iters, double* relres,
                            helmholtz_stream_t stream) {
    if (!h) return HELMHOLTZ_EINVAL;
    AdjointScope scope(h);
    return helmholtz_solve(h, g, lam, batch, rtol, maxiter, iters, relres, stream);
}

int helmholtz_face_grad_weighted(helmholtz_t h, const double* lam, const double* x,
                                 int32_t batch, double* g_kh, double* g_kv, double* g_delta,
                                 double* g_s, helmholtz_stream_t stream) {
    if (int e = check_batch(h, batch)) return e;
    if (!h->weighted) return HELMHOLTZ_EINVAL;
    if (!lam || !x || !g_kh || !g_delta || !g_s || (h->nz > 1 && !g_kv)) return HELMHOLTZ_EINVAL;
    const Level& v = h->lev[0];
    const int64_t total = int64_t(h->nz) * v.ncol;
    const int grid = int((total + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_face_grad_w, dim3(grid), dim3(kBlock), 0,
                       reinterpret_cast<hipStream_t>(stream), view<double>(h, 0), lam, x, batch,
                       g_kh, g_kv, g_delta, g_s);
    return last_error();
}

}  // extern "C"
