// Host-side cubed-sphere mesh tables (see mesh.cpp).
#pragma once
#include <cstdint>
#include <vector>

namespace hh {

// nbr[4][6N^2]: neighbour column in directions E, W, N, S.
void build_neighbours(int N, int32_t* nbr);
// ftab[4][6N^2]: stored face (slot*ncol + owner) behind each direction.
void build_face_table(int N, const int32_t* nbr, int32_t* ftab);
// parent[6N^2]: column of C<N/2> containing each column of C<N> (N even).
void build_parent(int N, int32_t* parent);
// child[4][6Nc^2]: children (0,0),(1,0),(0,1),(1,1) of each column of C<Nc> in C<2Nc>.
void build_children(int Nc, int32_t* child);

// Patches of pw x ph columns of one panel (smaller at its far edges) and the
// rings of columns around them (ring r: r steps away), for the kernels that
// run several sweeps on a patch. Per patch: col[ncp] lists its own columns row
// by row, then ring by ring up to `depth`; lnb[ncp] the places in that list of
// each column's E, W, N, S neighbours, a byte each (columns of the last ring:
// 0); cnt[8] the columns through ring 0, 1, 2, 3 and the own block's width.
// Unused places repeat the first column.
inline int patch_count(int N, int pw, int ph) {
    return 6 * ((N + pw - 1) / pw) * ((N + ph - 1) / ph);
}
void build_patches(int N, const int32_t* nbr, int pw, int ph, int depth, int ncp, int32_t* col,
                   uint32_t* lnb, int32_t* cnt);

}  // namespace hh
