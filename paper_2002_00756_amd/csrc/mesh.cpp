// Cubed-sphere column mesh and its horizontal 2x2 hierarchy (host side).
//
// The paper coarsens the mesh horizontally only, each coarse cell being the
// union of 2x2 fine cells (Section 3.6), and runs on cubed-sphere meshes of
// 6 x N x N columns (Section 5.1). The topology is built here from integer
// geometry on the cube [0, 2N]^3: panel p has outward normal n, origin O and
// in-panel axes a (E, index i) and b (N, index j); cell (p,i,j) is centred at
// O + (2i+1)a + (2j+1)b. A step off the panel goes to the edge and one unit
// down the adjacent face, the one whose normal is the step direction.
#include "mesh.hpp"

#include <algorithm>
#include <array>
#include <cstdint>
#include <vector>

namespace hh {
namespace {

struct Vec3 {
    int64_t x, y, z;
};
inline Vec3 operator+(Vec3 u, Vec3 v) { return {u.x + v.x, u.y + v.y, u.z + v.z}; }
inline Vec3 operator-(Vec3 u, Vec3 v) { return {u.x - v.x, u.y - v.y, u.z - v.z}; }
inline Vec3 operator*(int64_t s, Vec3 v) { return {s * v.x, s * v.y, s * v.z}; }
inline Vec3 operator-(Vec3 v) { return {-v.x, -v.y, -v.z}; }
inline int64_t dot(Vec3 u, Vec3 v) { return u.x * v.x + u.y * v.y + u.z * v.z; }
inline bool same(Vec3 u, Vec3 v) { return u.x == v.x && u.y == v.y && u.z == v.z; }

struct Panel {
    Vec3 normal, origin_unit, east, north;  // origin in units of 2N
};

// p0 +x, p1 +y, p2 -x, p3 -y, p4 +z, p5 -z
const std::array<Panel, 6> kPanels = {{
    {{1, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}},
    {{0, 1, 0}, {1, 1, 0}, {-1, 0, 0}, {0, 0, 1}},
    {{-1, 0, 0}, {0, 1, 1}, {0, 0, -1}, {0, -1, 0}},
    {{0, -1, 0}, {0, 0, 1}, {0, 0, -1}, {1, 0, 0}},
    {{0, 0, 1}, {1, 1, 1}, {-1, 0, 0}, {0, -1, 0}},
    {{0, 0, -1}, {0, 0, 0}, {0, 1, 0}, {1, 0, 0}},
}};

int panel_with_normal(Vec3 n) {
    for (int q = 0; q < 6; ++q)
        if (same(kPanels[q].normal, n)) return q;
    return -1;
}

}  // namespace

void build_neighbours(int N, int32_t* nbr) {
    const int64_t M = 2 * int64_t(N);
    const int64_t ncol = 6 * int64_t(N) * N;
    for (int p = 0; p < 6; ++p) {
        const Panel& P = kPanels[p];
        const Vec3 O = M * P.origin_unit;
        const Vec3 steps[4] = {P.east, -P.east, P.north, -P.north};
        const int di[4] = {1, -1, 0, 0}, dj[4] = {0, 0, 1, -1};
        int target[4];
        for (int d = 0; d < 4; ++d) target[d] = panel_with_normal(steps[d]);
        for (int j = 0; j < N; ++j) {
            for (int i = 0; i < N; ++i) {
                const int64_t c = int64_t(p) * N * N + int64_t(j) * N + i;
                if (i > 0 && i + 1 < N && j > 0 && j + 1 < N) {
                    nbr[c] = int32_t(c + 1);
                    nbr[ncol + c] = int32_t(c - 1);
                    nbr[2 * ncol + c] = int32_t(c + N);
                    nbr[3 * ncol + c] = int32_t(c - N);
                    continue;
                }
                const Vec3 centre = O + (2 * i + 1) * P.east + (2 * j + 1) * P.north;
                for (int d = 0; d < 4; ++d) {
                    const int i2 = i + di[d], j2 = j + dj[d];
                    int64_t n;
                    if (i2 >= 0 && i2 < N && j2 >= 0 && j2 < N) {
                        n = int64_t(p) * N * N + int64_t(j2) * N + i2;
                    } else {
                        const Panel& Q = kPanels[target[d]];
                        const Vec3 rel = centre + steps[d] - P.normal - M * Q.origin_unit;
                        const int64_t ia = (dot(rel, Q.east) - 1) / 2;
                        const int64_t jb = (dot(rel, Q.north) - 1) / 2;
                        n = int64_t(target[d]) * N * N + jb * N + ia;
                    }
                    nbr[d * ncol + c] = int32_t(n);
                }
            }
        }
    }
}

void build_face_table(int N, const int32_t* nbr, int32_t* ftab) {
    const int64_t ncol = 6 * int64_t(N) * N;
    for (int64_t c = 0; c < ncol; ++c) {
        ftab[0 * ncol + c] = int32_t(c);          // E: own face, slot 0
        ftab[2 * ncol + c] = int32_t(ncol + c);   // N: own face, slot 1
        for (int d : {1, 3}) {                    // W, S: the neighbour's face
            const int64_t o = nbr[d * ncol + c];
            const bool east_of_owner = nbr[0 * ncol + o] == c;
            ftab[d * ncol + c] = int32_t(east_of_owner ? o : ncol + o);
        }
    }
}

void build_parent(int N, int32_t* parent) {
    const int64_t Nc = N / 2;
    for (int p = 0; p < 6; ++p)
        for (int j = 0; j < N; ++j)
            for (int i = 0; i < N; ++i)
                parent[int64_t(p) * N * N + int64_t(j) * N + i] =
                    int32_t(p * Nc * Nc + (j / 2) * Nc + (i / 2));
}

void build_children(int Nc, int32_t* child) {
    const int64_t Nf = 2 * int64_t(Nc);
    const int64_t ncc = 6 * int64_t(Nc) * Nc;
    for (int p = 0; p < 6; ++p)
        for (int J = 0; J < Nc; ++J)
            for (int I = 0; I < Nc; ++I) {
                const int64_t C = int64_t(p) * Nc * Nc + int64_t(J) * Nc + I;
                for (int s = 0; s < 4; ++s) {
                    const int64_t di = s & 1, dj = s >> 1;  // (0,0),(1,0),(0,1),(1,1)
                    child[s * ncc + C] =
                        int32_t(p * Nf * Nf + (2 * J + dj) * Nf + (2 * I + di));
                }
            }
}

void build_patches(int N, const int32_t* nbr, int pw, int ph, int depth, int ncp, int32_t* cols,
                   uint32_t* lnbs, int32_t* cnts) {
    const size_t ncol = 6 * size_t(N) * N;
    std::vector<int32_t> place(ncol, -1);  // column -> place in the current list
    const size_t row = size_t((N + pw - 1) / pw);  // patches of one row of a panel
    // whether a patch from x on keeps its rings within its panel along one axis,
    // and so does the one before it
    auto clear = [&](int x, int size) { return x >= size + depth && x + size + depth <= N; };
    size_t p = 0;
    for (int pan = 0; pan < 6; ++pan)
        for (int j0 = 0; j0 < N; j0 += ph)
            for (int i0 = 0; i0 < N; i0 += pw, ++p) {
                const int w = std::min(pw, N - i0), h = std::min(ph, N - j0);
                const int32_t first = int32_t((int64_t(pan) * N + j0) * N + i0);
                int32_t* col = cols + p * ncp;
                int32_t* cnt = cnts + p * 8;
                uint32_t* lnb = lnbs + p * ncp;
                // Along an axis on which its rings stay inside the panel, a patch is
                // the one before it, shifted: its panel's columns by one patch, those
                // across the panel edge (one edge at most) by that on the other panel.
                const bool right = clear(i0, pw) && h == ph, up = clear(j0, ph) && w == pw;
                if (right || up) {
                    const size_t like = right ? p - 1 : p - row;
                    const int32_t by = right ? pw : ph * N;
                    // the edge that the other axis reaches, if any: a column on it
                    int d, at;
                    if (right) {
                        d = j0 < depth ? 3 : 2;
                        at = (pan * N + (d == 3 ? 0 : N - 1)) * N + i0;
                    } else {
                        d = i0 < depth ? 1 : 0;
                        at = (pan * N + j0) * N + (d == 1 ? 0 : N - 1);
                    }
                    const int32_t* nd = nbr + d * ncol;
                    const int32_t across = nd[at] - nd[at - by];
                    const int32_t base = pan * N * N;
                    const int32_t* from = cols + like * ncp;
                    for (int q = 0; q < ncp; ++q)
                        col[q] = from[q] +
                                 (uint32_t(from[q] - base) < uint32_t(N * N) ? by : across);
                    std::copy_n(cnts + like * 8, 8, cnt);
                    std::copy_n(lnbs + like * ncp, ncp, lnb);
                    continue;
                }
                std::fill_n(cnt, 8, 0);
                std::fill_n(lnb, ncp, 0u);
                int n = 0;
                auto add = [&](int32_t c) {
                    if (place[c] < 0) {
                        place[c] = n;
                        col[n++] = c;
                    }
                };
                for (int j = 0; j < h; ++j)
                    for (int i = 0; i < w; ++i) add(first + j * N + i);
                cnt[4] = w;
                cnt[0] = n;
                for (int r = 1; r <= depth; ++r) {
                    const int from = r == 1 ? 0 : cnt[r - 2], to = cnt[r - 1];
                    for (int q = from; q < to; ++q)
                        for (int d = 0; d < 4; ++d) add(nbr[d * ncol + col[q]]);
                    cnt[r] = n;
                }
                for (int q = 0; q < cnt[depth - 1]; ++q)
                    for (int d = 0; d < 4; ++d)
                        lnb[q] |= uint32_t(place[nbr[d * ncol + col[q]]]) << (8 * d);
                for (int q = 0; q < n; ++q) place[col[q]] = -1;
                for (int q = n; q < ncp; ++q) col[q] = col[0];
            }
}

}  // namespace hh
