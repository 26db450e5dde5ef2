// Internal declarations shared by the host orchestration and the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ssprkse.h"

namespace sse {

constexpr int kMaxEdges = 6;    // edges per cell (hexagons / pentagons)
constexpr int kMaxEdges2 = 10;  // edges in the tangential-reconstruction stencil
constexpr int kEdgeRec = 32;    // int32 words of one per-edge record (128 bytes)
constexpr int kWave = 64;       // CDNA wavefront
constexpr int kColsPerBlock = 4;
constexpr int kXcd = 8;           // accelerator complex dies of an MI355X
constexpr int kBlock = kWave * kColsPerBlock;
constexpr size_t kAlign = 256;

// Device-resident mesh tables.  Per-entity neighbour lists used by the
// column kernels are stored entity-major ([entity][slot]); the 2D barotropic
// kernels, with one thread per entity, read the slot-major copies
// ([slot][entity]) so that every load instruction is coalesced.
struct DevMesh {
    int C = 0, E = 0, V = 0;
    // cells
    const int32_t *cell_edges = nullptr;    // [C][6], padded with a valid index and zero coefficients
    const int32_t *cell_nbrs = nullptr;     // [C][6]
    const int32_t *cell_nedges = nullptr;   // [C]
    const double *cell_div = nullptr;       // [C][6]  s_{i,e} l_e / A_i
    const double *cell_ke = nullptr;        // [C][6]  l_e d_e / (4 A_i)
    const int32_t *cell_edges_t = nullptr;  // [6][C]
    const int32_t *cell_nbrs_t = nullptr;   // [6][C]
    const double *cell_div_t = nullptr;     // [6][C]
    const double *H = nullptr;              // [C]
    const uint8_t *cmask = nullptr;         // [C]
    // edges
    const int32_t *edge_cells = nullptr;    // [E][2]
    const int32_t *edge_verts = nullptr;    // [E][2]
    const int32_t *eoe = nullptr;           // [10][E]
    const int32_t *neoe = nullptr;          // [E]
    const int32_t *erec = nullptr;          // [E][32] per-edge record for the column kernels:
                                            //   stencil edges [10], cells [2] at 30/31, and either
                                            //   the stencil edges' vertices [10][2] (generic) or the
                                            //   vertex chains of the two cells (chain == 1)
    int chain = 0;                          // 1: stencils in canonical two-cell order (see sse_mesh.cpp)
    const double *w = nullptr;              // [10][E]  W_{e,j}
    const double *wf = nullptr;             // [10][E]  W_{e,j} (f_e + f_j) / 2
    const double *wpair = nullptr;          // [E][10][2] (W_{e,j} / 4, W_{e,j} (f_e + f_j) / 2), entity-major
    const double *dc = nullptr;             // [E]
    const double *dv = nullptr;             // [E]
    const double *inv_dc = nullptr;         // [E] 1 / d_e
    const double *inv_dv = nullptr;         // [E] 1 / l_e
    const uint8_t *emask = nullptr;         // [E]
    // vertices
    const int32_t *vert_edges = nullptr;    // [V][3]
    const double *vert_curl = nullptr;      // [V][3]  r_{v,e} d_e / A_v
    // FP32 copies of the tables the barotropic loop reads in mixed precision
    const float *wf_f = nullptr;            // [10][E]
    const float *inv_dc_f = nullptr;        // [E]
    const float *cell_div_t_f = nullptr;    // [6][C]
    const float *H_f = nullptr;             // [C]
    const float *wpair_f = nullptr;         // [E][10][2] wpair rounded to FP32 (the edge pass in mixed precision)
    // 16-bit index tables of the barotropic evaluation (delta16 == 1 when every
    // offset fits): stencil edges as e + eoe16[j][e]; the cells of edge e as
    // bc(e) + low / high half of ecells16[e]; the edges and neighbours of cell
    // i as be(i) + cedges16[j][i] and i + cnbrs16[j][i], with the fixed-point
    // bases bc(e) = (e ratio_ce) >> 16 and be(i) = (i ratio_ec) >> 16.
    int delta16 = 0;
    uint32_t ratio_ce = 0, ratio_ec = 0;
    const int16_t *eoe16 = nullptr;         // [10][E]
    const int32_t *ecells16 = nullptr;      // [E]
    const int16_t *cedges16 = nullptr;      // [6][C]
    const int16_t *cnbrs16 = nullptr;       // [6][C]
    // the caller's numbering: internal cell i / edge e is caller cell
    // cell_old[i] / edge edge_old[e]
    const int32_t *cell_old = nullptr;      // [C]
    const int32_t *edge_old = nullptr;      // [E]
};

// Per-cell record of the split forward-Euler pass (meshes with factored
// weights, see DevFact): what one wavefront needs for its cell's column, read
// with scalar loads from one place.  Slots past the cell's last edge repeat its
// first edge with zero coefficients.
template <typename R>
struct alignas(64) CellRec {
    R lhs[6];       // s_b l_b / 2
    R fh[6];        // f_b / 2
    R S[6];         // 2 S_1 .. 2 S_5, 2 S_n
    R curl[18];     // a quarter of the curl weights at vertex m (between edges m and m + 1): edge m,
                    // edge m + 1, and the edge that leaves the cell there
    R ke[6];        // l d / (4 A)
    R rk[6];        // 2 d / l
    R ia;           // 1 / A
    R pad;
    int32_t own[6], out[6], nbr[6];   // its edges, the outgoing edges at its vertices, its neighbours
    int32_t n;
    uint32_t side;  // bit b: the cell is the second cell of edge b
};

// Fixed-point base of the 16-bit offsets (see DevMesh).
__host__ __device__ inline int delta_base(int x, uint32_t ratio) {
    return (int)(((unsigned long long)x * ratio) >> 16);
}

// Gather lists of the LDS-staged baroclinic edge pass.  The edges are cut
// into tiles of T consecutive edges; for every tile the unique edge columns
// (the tiles' edges and their reconstruction stencils), vertex columns and
// cell columns it reads are listed once, and every edge stores the 8-bit
// positions of its operands in those lists.
constexpr int kTileVariants = 3;
constexpr int kTileSizes[kTileVariants] = {8, 16, 32};
constexpr int kLocPerEdge = 36;  // self, c1, c2, v1, v2, stencil[10], stencil vertices[10][2], pad
struct DevTiles {
    int T = 0, nT = 0;
    int max_ue = 0, max_uv = 0, max_uc = 0;  // largest list sizes over the tiles
    const int32_t *ue_off = nullptr, *uv_off = nullptr, *uc_off = nullptr;  // [nT + 1]
    const int32_t *ue = nullptr, *uv = nullptr, *uc = nullptr;              // global ids
    const uint8_t *loc = nullptr;                                           // [E][kLocPerEdge]
};

}  // namespace sse

namespace sse {
// Tiled barotropic substeps.  The cells are cut into compact patches; a patch
// with its halo rings is everything one SSPRK3 substep (three evaluations)
// of its own cells and edges reads, so one workgroup advances its patch a
// whole substep with the state in LDS and the stencil tables in registers,
// and the launches per barotropic loop drop from 3M to M.
//
// Region of a patch, by level k = 0..3: cells R_k (R_0 the patch, R_{k+1} =
// R_k and its neighbours) and edges E_k (E_0 the owned edges, those whose
// first cell is in the patch; E_k = all edges of R_k for k >= 1), listed
// level by level, so a level-k set is a prefix of the region lists.  The
// evaluation that produces level k reads level k + 1.
constexpr int kBtThreads = 512;    // threads per workgroup
constexpr int kFactSmall = 256;    // the same, factored weights, where every region fits them
// Workgroups of a CU at once (4 waves per SIMD, 128 VGPRs): two, so one
// workgroup's table loads overlap the other's evaluations.
constexpr int kBtWavesPerSimd = 4;
// Target cells per patch.  Measured, C1 FP64 / mixed ms/step and C2 FP64 /
// mixed ms/step: 1024 threads and 352 cells (one workgroup per CU, no
// overlap): 7.98 / 6.23, 5.69 / 4.46; 512 threads and 176 cells: 7.85 /
// 6.08, 5.77 / 4.49; 160 cells: 7.87 / 6.12, 5.85 / 4.52.  From 192 cells
// the level-2 edges of many patches exceed 2 x 512, and the split halves
// cost more (8.45 ms C1).  256 threads with 72 or 88 cells (four workgroups
// per CU, a deeper halo per cell): the barotropic class alone takes 4.75 /
// 5.68 ms per C1 step in FP64 against 2.92.
constexpr int kBtPatch = 176;
constexpr int kBtEdgeSlots = 2;    // edges of level 2 per thread (at most)
constexpr int kBtPatchMin = 64;
// Cells per patch of a mesh of C cells run on its own: what spreads it evenly
// over the 256 CUs (up to kBtPatch per patch; a few percent more than the
// even share, since the breadth-first cut leaves some patches short), down to
// kBtPatchMin, below which the halo outweighs what a smaller patch saves.  A
// mesh whose edges fit one workgroup is one patch and needs no exchange.
// Resident loop, ms per step of 60 or 90 substeps in FP64, 176 cells per patch
// against this rule: 64 x 64 0.44 / 0.33, 128 x 128 0.44 / 0.37, 256 x 256 0.54
// / 0.48, level-5 sphere 0.63 / 0.48.
constexpr int kCus = 256;
inline int bt_patch_cells(int C) {
    if (3 * C <= kBtEdgeSlots * kBtThreads) return C;
    const int per_cu = (C + kCus * kBtPatch - 1) / (kCus * kBtPatch);
    const int even = (int)(1.06 * C / (kCus * per_cu)) + 1;
    return even < kBtPatchMin ? kBtPatchMin : even < kBtPatch ? even : kBtPatch;
}
constexpr int kBtRec = 16;         // ints per patch record

// Factored TRiSK weights.  Around one cell with edges 0 .. n-1 in
// counter-clockwise order, the reconstruction weights are differences of one
// prefix sum S of the cell's kite fractions (Thuburn et al. 2009):
//   W_{a,b} = s_a s_b (l_b / d_a) (1/2 - (S_b - S_a)),  b > a,
//   W_{a,b} = s_a s_b (l_b / d_a) (1/2 - (S_n - S_a + S_b)),  b < a.
// With x_b = s_b l_b u_b, the sum over a cell's edges is then, for every one
// of them, a combination of X = sum x, Y = sum S x and the running sum
// P_a = sum_{b<a} x_b: six numbers per cell (S_1 .. S_5, S_n) in the place of
// ten weights per edge.  A mesh takes this form when its weights reproduce it
// to a few units in the last place (sse_mesh.cpp); any other mesh keeps the
// weight tables.
constexpr int kFactEdges = 3;      // region edges per thread, level 3
constexpr int kFactNbrs = 64;      // neighbour patches one wavefront polls
struct DevFact {
    const double *lh = nullptr, *fh = nullptr;      // [E] l_e / 2, f_e / 2
    const double *S = nullptr, *ia = nullptr;       // [6][C] 2 S_1 .. 2 S_5, 2 S_n; [C] 1 / A
    const float *lh_f = nullptr, *fh_f = nullptr, *S_f = nullptr, *ia_f = nullptr;
};
struct DevBtTiles {
    int nP = 0;                    // patches (0: tiling not available)
    int ks = 0;                    // edge slots per thread needed (1 or 2)
    int dry = 0;                   // 1: the mesh has land cells or coast edges
    size_t lds_d = 0, lds_f = 0;   // dynamic LDS bytes for R = double / float
    // per patch: e0, es0, c0, cs0, ne[4], nc[4] (offsets into the region
    // lists / the stencil tables, prefix counts per level)
    const int32_t *patch = nullptr;
    const int32_t *eid = nullptr;     // [sum ne3] global edge of each region edge
    const int32_t *cid = nullptr;     // [sum nc3] global cell of each region cell
    const double *cH = nullptr;       // [sum nc3] H of region cells
    const float *cH_f = nullptr;
    // stencil tables of the edges of levels 0..2 (es0 + le), per patch slot-major
    // with stride ne2: entry (j, le) at es0 * J + j * ne2 + le
    const uint32_t *ec = nullptr;     // [sum ne2] local c1 | c2 << 15 | wet << 30
    const uint32_t *enb = nullptr;    // [5][..] local stencil edges, two 16-bit indices per word
    const double *ew = nullptr;       // [10][..] W (f_e + f_j) / 2
    const float *ew_f = nullptr;
    const double *eidc = nullptr;     // [..] 1 / d_e
    const float *eidc_f = nullptr;
    // cell tables of the cells of levels 0..2 (cs0 + lc), stride nc2
    const uint32_t *cen = nullptr;    // [6][..] local edge | local neighbour << 16
    const double *ccd = nullptr;      // [6][..] s l / A
    const float *ccd_f = nullptr;
    const uint8_t *cwet = nullptr;    // [..]
    // Factored form (fact == 1): these in the place of enb, ew, cen, ccd and
    // cwet.  Edges at e0 + le over all region edges; cells at c0 + lc over all
    // region cells; the slot-major cell tables at J c0 + j nc3 + lc.
    int fact = 0;
    int nt = 0;                       // threads per workgroup
    int nA = 0;                       // patches with an ocean cell (listed first in order)
    int resident = 0;                 // 1: every patch has at most kFactNbrs neighbours
    // patch record words 12..14: offset and count of its neighbours, ocean flag
    const int32_t *order = nullptr;   // [nP] patches with ocean cells, then the others
    const int32_t *nbr = nullptr;     // patches whose values a patch reads or that read its values
    const uint32_t *fec = nullptr;    // [sum ne3] local c1 | c2 << 15 | wet << 30 | read by another patch << 31
    const double *elh = nullptr, *efh = nullptr;    // [sum ne3] l_e / 2, f_e / 2
    const float *elh_f = nullptr, *efh_f = nullptr;
    const double *fidc = nullptr;     // [sum ne3] 1 / d_e
    const float *fidc_f = nullptr;
    const uint32_t *fcen = nullptr;   // [3][..] local edges, 16 bits each: index | (edge points inwards) << 15
    const double *cS = nullptr, *cia = nullptr;     // [6][..], [..]
    const float *cS_f = nullptr, *cia_f = nullptr;
    const uint8_t *cflag = nullptr;   // [sum nc3] wet | read by another patch << 1
    DevFact g;                        // the same numbers per mesh entity (one launch per evaluation)
};
}  // namespace sse

namespace sse {
struct PermutedDesc;
}

struct sse_mesh {
    sse::DevMesh d;
    int C = 0, E = 0, V = 0;
    int n_ocean_cells = 0;
    // Internal (locality) numbering: entity i of the device arrays is entity
    // cell_old[i] / edge_old[i] of the caller's numbering.
    std::vector<int32_t> cell_old, edge_old;
    bool identity = false;                  // both are the identity
    std::vector<int32_t> cells_on_edge;     // host copy (for debug helpers)
    // Gather lists of the LDS-staged edge pass (T = 8, 16, 32 edges per
    // tile), built and uploaded into their reserved part of the mesh buffer
    // the first time a state selects the variant (ensure_tiles).
    sse::DevTiles tiles[sse::kTileVariants];
    size_t tile_off[sse::kTileVariants] = {};
    int tile_state[sse::kTileVariants] = {};  // 0 not built, 1 built, -1 not possible
    // Records of the split forward-Euler pass, in the lists' reserved part
    // (null: the weights do not factor; the lists are then built on demand).
    const sse::CellRec<double> *cell_rec = nullptr;
    const sse::CellRec<float> *cell_rec_f = nullptr;
    std::mutex tile_mu;
    std::unique_ptr<sse::PermutedDesc> host_desc;  // internal numbering, for building the lists
    sse::DevBtTiles bt;                       // patches of the tiled barotropic substeps
    sse::DevBtTiles bt_batch;                 // patches for batch members (kBtPatch cells, kBtThreads threads)
    void *dev_buf = nullptr;
    size_t dev_bytes = 0;
};

namespace sse {

// Sizes of the device mesh image (bytes) and the offsets of its tables, in
// the order in which mesh_create uploads them.
constexpr int kMeshTables = 35;
void mesh_table_sizes(int C, int E, int V, size_t (&sizes)[kMeshTables]);
struct MeshLayout {
    size_t off[kMeshTables] = {};
    size_t total = 0;
};
MeshLayout mesh_layout(int C, int E, int V);

// Host-side table building (sse_mesh.cpp).
int validate_desc(const sse_mesh_desc *d, std::string &err);

struct HostMeshTables {
    std::vector<int32_t> cell_edges, cell_nbrs, cell_nedges, cell_edges_t, cell_nbrs_t;
    std::vector<double> cell_div, cell_ke, cell_div_t, H;
    std::vector<uint8_t> cmask;
    std::vector<int32_t> edge_cells, edge_verts, eoe, neoe, erec;
    std::vector<double> w, wf, dc, dv, inv_dc, inv_dv, wpair;
    std::vector<uint8_t> emask;
    std::vector<int32_t> vert_edges;
    std::vector<double> vert_curl;
    std::vector<float> wf_f, inv_dc_f, cell_div_t_f, H_f, wpair_f;
    std::vector<int16_t> eoe16, cedges16, cnbrs16;
    std::vector<int32_t> ecells16;
    int delta16 = 0;
    uint32_t ratio_ce = 0, ratio_ec = 0;
    int n_ocean_cells = 0;
    // [E][kChainWords] vertex chains of canonical stencils (empty: generic)
    std::vector<int32_t> chain;
    // factored weights (see DevFact; empty: the weights are not of that form)
    std::vector<double> fS, fia, flh, ffh;
};
// Fills t.fS .. t.ffh if every weight of d (canonical stencils) is within
// kFactTol of the factored form.
constexpr double kFactTol = 4.0e-15;
void factor_weights(const sse_mesh_desc *d, HostMeshTables &t);
// The cell records of a mesh with factored weights; false if some vertex has
// no third edge.
bool build_cell_recs(const sse_mesh_desc *d, const HostMeshTables &t, std::vector<CellRec<double>> &v);
void build_tables(const sse_mesh_desc *d, HostMeshTables &t);

struct HostTiles {
    int T = 0, nT = 0, max_ue = 0, max_uv = 0, max_uc = 0;
    std::vector<int32_t> ue_off, uv_off, uc_off, ue, uv, uc;
    std::vector<uint8_t> loc;
};
// Returns false if a tile needs more than 255 entries in one list.
bool build_tiles(const sse_mesh_desc *d, int T, HostTiles &t);
size_t tiles_bytes(const sse_mesh_desc *d, int T);
// Bytes of the FP32 weight pairs (DevMesh::wpair_f), placed after the tile
// tables so that the other tables keep their offsets in the mesh image.
size_t wpair_f_bytes(const sse_mesh_desc *d);

// Locality order of a mesh (new -> old and old -> new numbering): cells in
// compact breadth-first patches of `patch` cells, edges following the first
// cell that lists them, vertices following the first edge that lists them.
struct MeshOrder {
    std::vector<int32_t> cell_old, edge_old, vert_old;
    std::vector<int32_t> cell_new, edge_new, vert_new;
};
void locality_order(const sse_mesh_desc *d, int patch, MeshOrder &o);

// A copy of a mesh description renumbered by `o` (same conventions; the
// stencil order inside every row is kept, so results do not change).
struct PermutedDesc {
    sse_mesh_desc d{};
    std::vector<int32_t> coe, eoc, neoc, voe, eov, eoe, neoe;
    std::vector<double> w, dc, dv, f, area, H, tri;
    std::vector<uint8_t> mask;
};
void permute_desc(const sse_mesh_desc *d, const MeshOrder &o, PermutedDesc &p);

// Rewrites every reconstruction stencil of p in the canonical two-cell order
// and returns the vertex chains ([E][kChainWords]), or returns false and
// leaves p unchanged when some stencil is not "the other edges of the two
// cells of e" (then the generic tables are used).
constexpr int kChainWords = 11;  // A0..A5, B0..B3, flag (A0 is vertex 0 of the edge)
bool canonical_stencils(PermutedDesc &p, std::vector<int32_t> &chain);

// Patches of the tiled barotropic substeps, computed in the numbering of d:
// breadth-first patches of about kBtPatch cells, split in two (in their
// breadth-first order) until every patch's level-2 region fits the
// workgroup (kBtEdgeSlots edges and one cell per thread).  With `mask` (may be
// NULL) no patch holds cells of both kinds.  pid[c] = patch of cell c.
// Returns false if no such partition exists.
bool bt_partition(const sse_mesh_desc *d, int target, const uint8_t *mask, std::vector<int32_t> &pid, int &nP);

struct HostBtTiles {
    int nP = 0, ks = 0;
    size_t lds_d = 0, lds_f = 0;
    std::vector<int32_t> patch, eid, cid;
    std::vector<double> cH, ew, eidc, ccd;
    std::vector<float> cH_f, ew_f, eidc_f, ccd_f;
    std::vector<uint32_t> ec, enb, cen;
    std::vector<uint8_t> cwet;
    // factored form
    bool fact = false;
    int nt = 0, nA = 0, resident = 0;
    std::vector<int32_t> order, nbr;
    std::vector<uint32_t> fec, fcen;
    std::vector<double> elh, efh, fidc, cS, cia;
    std::vector<uint8_t> cflag;
};
// A partition of a mesh with the device bytes of its tables.
struct BtPartition {
    bool ok = false;
    int nP = 0;
    std::vector<int32_t> pid;
    size_t bytes = 0;
};
// Device bytes of the factored tables over TE region edges and TC region cells
// in nP patches (global tables of E edges and C cells included).
size_t fact_tiles_bytes(size_t nP, size_t TE, size_t TC, size_t E, size_t C);
// Region lists and tables of the partition pid (numbering of d, the same
// numbering as the tables t).  With t == nullptr only the sizes are filled
// (patch records, list lengths), which is what the device-bytes query needs.
bool build_bt_tiles(const sse_mesh_desc *d, const std::vector<int32_t> &pid, int nP, const HostMeshTables *t,
                    HostBtTiles &bt);
// The same partition in the factored form; false if a region does not fit it.
// min_nt: kFactSmall or kBtThreads, the fewest threads to take.
bool build_fact_tiles(const sse_mesh_desc *d, const std::vector<int32_t> &pid, int nP, const HostMeshTables &t,
                      int min_nt, HostBtTiles &bt);
// Device bytes of the tiled barotropic tables of d (0 if d cannot be tiled),
// and its partitions; both come from a cache keyed by the topology.  The first
// has patches of kBtPatch cells (its tables in either form fit its bytes), the
// second, where it differs, bt_patch_cells (factored form only).
size_t bt_tiles_bytes(const sse_mesh_desc *d);
void bt_cached_partitions(const sse_mesh_desc *d, BtPartition &coarse, BtPartition &fine);
// The same two cut along the coast, for the factored form: ocean patches sized
// by the ocean cells, and land patches, which take no work.  Not ok where the
// mesh has no land, or where the cut leaves more than twice the ocean patches
// that full ones would be (an ocean of scattered cells).
void bt_coast_partitions(const sse_mesh_desc *d, BtPartition &coarse, BtPartition &fine);
// Range checks of the topology tables the size queries read.
int check_topology(const sse_mesh_desc *d, std::string &err);

void set_error(const std::string &msg);

}  // namespace sse
