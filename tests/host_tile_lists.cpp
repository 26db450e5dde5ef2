// Host harness of tests/test_host_tile_lists.py: the gather lists of the tiled
// edge pass for a mesh, built as sse_mesh_create and sse_state_set_edge_variant
// build them.  Returns the number of entries out of range, or of operands whose
// list entry is not the mesh's; -1 without lists (a tile of more than 255 columns).
#include "sse_internal.h"

using namespace sse;

extern "C" long check_tile_lists(const sse_mesh_desc *d0, int T, int canonical) {
    MeshOrder ord;
    locality_order(d0, 64, ord);
    PermutedDesc pd;
    permute_desc(d0, ord, pd);
    std::vector<int32_t> chain;
    if (canonical && !canonical_stencils(pd, chain)) return -2;
    const sse_mesh_desc &d = pd.d;
    HostTiles t;
    if (!build_tiles(&d, T, t)) return -1;
    long bad = 0;
    for (int x : t.ue) bad += x < 0 || x >= d.n_edges;
    for (int x : t.uv) bad += x < 0 || x >= d.n_vertices;
    for (int x : t.uc) bad += x < 0 || x >= d.n_cells;
    if (bad) return bad;
    for (int e = 0; e < d.n_edges; ++e) {
        const int tile = e / T;
        const uint8_t *L = &t.loc[(size_t)e * kLocPerEdge];
        auto E = [&](int i) { return t.ue[t.ue_off[tile] + L[i]]; };
        auto V = [&](int i) { return t.uv[t.uv_off[tile] + L[i]]; };
        bad += E(0) != e;
        for (int j = 0; j < kMaxEdges2; ++j) {
            const int want = j < d.n_edges_on_edge[e] ? d.edges_on_edge[(size_t)e * d.max_edges2 + j] : -1;
            const int got = E(5 + j);
            bad += want >= 0 ? got != want : got != e;
            bad += V(15 + 2 * j) != d.vertices_on_edge[2 * (size_t)got] || V(16 + 2 * j) != d.vertices_on_edge[2 * (size_t)got + 1];
        }
    }
    return bad;
}
