// plan.h -- host-side mesh preprocessing for the block-LDS assembly.
//
// Section 4.3 of the paper groups elements by geometric type, renumbers them
// and packs them so that a SIMD/SIMT unit processes a pack at once.  The gfx950
// form of that idea built here:
//   * elements are reordered along a Morton curve of their centroids and nodes
//     renumbered by first touch, so that a block of consecutive elements is
//     spatially compact and touches few CSR rows;
//   * a block is at most one wavefront (64) of elements, cut early when the
//     LDS image of the rows it touches would exceed the budget, and at the
//     fixed element chunks the planner builds blocks in (kPlanElemChunk);
//   * blocks are coloured so that no two blocks of one colour share a node:
//     one launch per colour runs without write conflicts (no atomics);
//   * inside a block, elements are split into phases so that no two lanes of
//     one phase hold the same node at the same local position, which makes
//     every LDS accumulation instruction conflict-free and the summation
//     order fixed;
//   * for each touched row the first block (in launch order) that touches it
//     overwrites it, later blocks read-modify-write it.
#pragma once

#include <cstdint>
#include <functional>
#include <memory>
#include <new>
#include <utility>
#include <string>
#include <vector>

namespace feasm {

// LDS budget of one assembly work-group (bytes).  The momentum kernel stages
// 8 fields per touched node, 3 RHS images, one int descriptor and the row image.
constexpr int kBlockElems = 64;
constexpr int kLdsBudget = 40 * 1024;
constexpr int kNodeFields = 8;
constexpr int kMaxRhs = 3;
constexpr int kMaxRow = 255;   // in-row offsets are stored as uint8
// The planner's parallel stages work on fixed chunks (elements for the
// assembly blocks, rows for the SpMV row blocks), so a plan does not depend
// on the number of host threads that built it.
constexpr int64_t kPlanElemChunk = 1 << 16;   // a multiple of kBlockElems
constexpr int64_t kPlanRowChunk = 1 << 15;
// Touched-row descriptor: image offset (bits 0-15) | row length (16-23) |
// first-writer flag (bit 31).
constexpr uint32_t kFirstBit = 0x80000000u;

// One assembly launch: blocks color_blk[first, first + count) of one colour
// and one element type (nen nodes per element).
struct AsmSeg {
    int nen, first, count;
};

// Position of an element type (by node count) in the order a mixed mesh
// groups them: HEX08, PEN06, PYR05, TET04.
inline int type_rank(int nen) { return nen == 8 ? 0 : nen == 6 ? 1 : nen == 5 ? 2 : 3; }

// Images of a single-type mesh's blocks, in matrices, up to which the mesh
// assembles by blocks with a gather, and beyond which, elements or nodes being
// in an order of poor locality, by owner groups (which compute an element once
// for each group that owns one of its rows).  FP64 momentum / mixed Poisson, us
// by blocks against owner groups, elements and nodes shuffled within windows
// of a Morton order: TET04 40^3 cubes, 3.5 matrices 64 / 53 against 81 / 58,
// 5.3 72 / 59 against 87 / 61, 7.8 83 / 70 against 92 / 64, 22.7 (random order)
// 225 / 179 against 115 / 83; PEN06 36^3 6.2 85 / 74 against 104 / 81, 11.3 144 /
// 123 against 133 / 91; PYR05 30^3 4.5 78 / 72 against 104 / 73, 6.8 98 / 91
// against 121 / 83.  Meshes of few blocks wait for the gather's chain instead:
// TET04 16^3 3.2 28 / 26 against 28 / 26, 4.9 30 / 28 against 30 / 27, 20.5 45 /
// 42 against 30 / 28; PYR05 10^3 3.9 36 / 36 against 35 / 34.  Renumbered meshes
// hold 1.2 to 4.
constexpr int64_t kFewBlocks = 512;
constexpr double max_images(int64_t blocks) { return blocks < kFewBlocks ? 4.1 : 6.5; }

struct Plan {
    int nen = 0;          // connectivity stride: nodes of the largest element type
    int off_stride = 0;   // bytes of elem_off per element (nen * nen rounded up to 4)
    int64_t N = 0, E = 0, nnz = 0;
    std::vector<int32_t> node_perm;   // mesh index -> user node id
    std::vector<int32_t> node_iperm;  // user node id -> mesh index
    std::vector<int32_t> elem_perm;   // mesh element -> user element id
    std::vector<double> X;            // [3][N] coordinates, mesh numbering
    std::vector<int32_t> conn;        // [E][nen] mesh numbering, mesh order (short types padded)
    std::vector<uint8_t> etype;       // [E] nodes of each element (mesh order); empty: all nen
    std::vector<int32_t> rowptr, colidx, diagpos;
    int max_row = 0;

    // element blocks
    std::vector<int32_t> blk_elem_ptr;   // [nblk+1]
    std::vector<int32_t> blk_node_ptr;   // [nblk+1]
    std::vector<int32_t> blk_nodes;      // touched rows, ascending mesh ids
    std::vector<int32_t> blk_img;        // [nblk] entries of the touched rows (the block's row image)
    std::vector<int32_t> blk_rdesc;      // packed descriptor of each touched row (see kFirstBit)
    std::vector<int32_t> blk_rowstart;   // CSR start of each touched row
    std::vector<int32_t> blk_color;      // [nblk]
    std::vector<uint8_t> blk_nphase;     // [nblk]
    std::vector<uint16_t> elem_lnode;    // [nen][E] local row index of node a
    std::vector<uint8_t> elem_off;       // [E][off_stride]: offset of col b in row a at a * n_e + b
    std::vector<uint8_t> blk_nen;        // [nblk] element type of each block
    std::vector<uint8_t> elem_phase;     // [E]
    std::vector<int32_t> color_ptr;      // [ncolor+1]
    std::vector<int32_t> color_blk;      // blocks ordered by colour, then type (type_rank)
    std::vector<AsmSeg> segs;            // launch order: colour-major, one per type present
    // the element-vector passes' gather (want_gather): per node its places in
    // blk_nodes, ascending, at node_slot[node_slot_ptr[i] ..]
    bool want_gather = false;
    std::vector<int32_t> node_slot_ptr, node_slot;
    // the matrix gather (want_images): the blocks' row images one after the
    // other, block b's at blk_img_ptr[b]; node_img parallel to node_slot, the
    // row's place in all images.  Left empty when they exceed 2^31 entries, or
    // max_images times the matrix (0: any number).
    bool want_images = false, bounded_images = false;
    std::vector<int32_t> blk_img_ptr, node_img;
    int n_colors = 0, max_T = 0, max_L = 0, max_phase = 0;

    int64_t n_blocks() const { return (int64_t)blk_elem_ptr.size() - 1; }
    // Empties the plan but keeps its arrays' capacity, so that a plan object
    // reused for the next mesh (the serving runtime's planners) does not
    // fault its pages in again.
    void clear();
};

// conn [n_elems][stride]; types [n_elems] gives each element's node count
// (4, 5, 6 or 8, at most stride; the remaining slots are ignored) or is NULL
// for a mesh of one type with stride nodes.  Returns 0 on success, else an
// fe_status code with a message in err.
int build_plan(int stride, const uint8_t *types, int64_t n_nodes, const double *coords, int64_t n_elems,
               const int32_t *conn, bool renumber, Plan &P, std::string &err);

// Host memory of the planner's temporaries (per calling thread, kept between
// calls up to kPlanScratchKeep bytes so that a thread planning mesh after
// mesh reuses it; larger ones are released after the call).
constexpr size_t kPlanScratchKeep = (size_t)256 << 20;

// Runs f(c) for every c in [0, n) on up to host_threads() threads (chunks
// handed out in increasing order; f must only write chunk c's results).
void parallel_chunks(int64_t n, const std::function<void(int64_t)> &f);
// The same with the worker's index w in [0, parallel_workers(n)) passed as
// f(c, w), for per-worker scratch arrays.
int parallel_workers(int64_t n);
void parallel_chunks_w(int64_t n, const std::function<void(int64_t, int)> &f);

// Row-owner plan of the 3x3-block momentum operator (rowplan.cpp): tasks =
// (element, row) pairs ordered by row, then element; whole rows packed into
// groups of at most `lanes` lanes and kRowImage(lanes) block values.  A group's
// distinct elements and nodes are listed once.  A task adds its element's
// nodes in the order of its slots: in one (round, slot) the tasks of a row hold
// distinct columns, and lie in one wavefront (lanes between are idle).
constexpr int kRowElemsMax = 64;   // elements at a node
constexpr int kRowTasks = 256, kRowTasksSmall = 64;   // lanes
// Meshes of fewer tasks, which 256-lane groups would leave CUs without one, take
// the small groups: HEX08 10^3 (8 k tasks) 42 us against 48, TET04 10^3 34 against
// 43; just below and above the line HEX08 20^3 (64 k) 49, 21^3 (74 k) 56 against 69
// with one wave per 64 tasks as before.
constexpr int64_t kRowSmallMesh = 1 << 16;
constexpr int row_image(int lanes) { return lanes == kRowTasks ? 8192 : 3072; }
struct RowWave {
    int32_t first_task, n_tasks, first_row, n_rows;
};
// The other form, each task alone: a wavefront of whole rows, of at most 64
// tasks, every lane computing its element's points itself.  It runs where it
// is the faster (us by shared groups / alone):
//   * small HEX08 meshes, whose shared groups of 64 lanes wait for a barrier
//     per point: 10^3 39 / 34 plain, 42 / 37 with full stress; 20^3 44 / 44;
//   * orders of poor locality, where a group's tasks share few elements (more
//     than kRowPoor of them distinct; Morton order HEX08 0.31, TET04 0.69):
//     HEX08 40^3 in random order 314 / 252 plain, 366 / 323 with full stress,
//     TET04 15^3 58 / 43 and 62 / 51, hybrid 32^3 331 / 200 and 427 / 322; on
//     small meshes as fast, but sooner planned: TET04 8^3 0.77 / 0.44 ms; not
//     small meshes of PYR05, 10^3 38 / 41, or of several types, 10^3 45 / 52;
//   * hybrid meshes of kRowPlainHybrid tasks without the full-stress term: 32^3
//     200 / 175 (with it 239 / 278), 24^3 (260 k) 103 / 97, 16^3 48 / 55.
enum RowForm { kRowAuto = -1, kRowShared = 0, kRowAlone = 1 };
constexpr double kRowPoor = 0.85;
constexpr int64_t kRowPlainHybrid = 1 << 18;
struct RowLists {
    int32_t first_elem, n_elems, first_node, n_nodes;
};
constexpr uint32_t kRowNoTask = 0x7fffffffu, kRowFirstTask = 0x80000000u;   // task_meta: idle lane; a row's first
// Gauss points whose element data a group of ne elements holds at a time.  A
// wave's lanes take one point; at most 200 (element, point) pairs, while that is
// a point at least, so that two groups of 256 lanes share a CU's LDS.
constexpr int row_points(int ne, int lanes)
{
    if (ne < 1) return 1;
    const int by_waves = lanes / 64 / ((ne + 63) / 64), by_lds = 200 / ne;
    return by_lds < 1 || by_waves < 1 ? 1 : by_lds < by_waves ? by_lds : by_waves;
}
// Left unset by resize, so that the threads that fill a large array also fault its pages in.
template <class T> struct UnsetAllocator : std::allocator<T> {
    template <class U> struct rebind {
        using other = UnsetAllocator<U>;
    };
    template <class U> void construct(U *) {}
    template <class U, class... A> void construct(U *p, A &&...a) { ::new ((void *)p) U(std::forward<A>(a)...); }
};
template <class T> using UnsetVector = std::vector<T, UnsetAllocator<T>>;

struct RowPlan {
    int64_t n_tasks = 0, n_elems = 0, n_nodes = 0;   // entries of the arrays below
    int64_t max_img = 0, max_items = 0, max_nodes = 0;
    int lanes = 0;                     // of a group
    int nen = 0;                       // nodes per element, 0 for several types: then the groups of several,
    int32_t class_end[4] = {};         // HEX08, PYR05 and PEN06 alone, each to its end, before TET04's
    std::vector<RowWave> wdesc;        // [groups]; between their tasks entries may be unused
    std::vector<RowLists> wlists;      // [groups] places in the listed elements and nodes
    bool alone = false;                // each task alone: wdesc's groups are wavefronts, tasks as below
    // The large arrays in two pieces, as they go to the device.
    UnsetVector<char> tasks;
    // alone: [8] position of the element's node b in the row; element; local row (bits 0-3) | place among the row's tasks
    const uint8_t *alone_cols() const { return (const uint8_t *)tasks.data(); }
    const int32_t *alone_elem() const { return (const int32_t *)(alone_cols() + 8 * n_tasks); }
    const uint16_t *alone_meta() const { return (const uint16_t *)(alone_elem() + n_tasks); }
    static size_t alone_bytes(int64_t n) { return 14 * (size_t)n; }
    const uint32_t *task_meta() const   // group's element (bits 0-7) | local row a (8-10) | group's row (11-18) | round (19-30)
    {
        return (const uint32_t *)tasks.data();
    }
    const uint32_t *task_perm() const { return task_meta() + n_tasks; }   // slot s adds node (perm >> 4 s) & 15, 8 = none
    const uint8_t *task_cols() const { return (const uint8_t *)(task_perm() + n_tasks); }   // [8] slot s: its node's position in the row
    static size_t task_bytes(int64_t n) { return 16 * (size_t)n; }
    UnsetVector<char> lists;
    const uint16_t *wave_ln() const { return (const uint16_t *)lists.data(); }   // [8] the group's node of each element node
    const int32_t *wave_elem() const { return (const int32_t *)(wave_ln() + 8 * n_elems); }
    const int32_t *wave_node() const { return wave_elem() + n_elems; }
    static size_t list_bytes(int64_t elems, int64_t nodes) { return 20 * (size_t)elems + 4 * (size_t)nodes; }
};
// conn [E][stride] and rowptr/colidx in mesh numbering; etype [E] node
// counts or NULL (every element has stride nodes).  0 or an fe_status code
// with a message in err (FE_EBADMESH: a node in more than kRowElemsMax
// elements).  fetch: fills rowptr and colidx, on the calling thread while
// others plan what needs neither.  form: the form planned; kRowAuto: the one
// that suits the mesh's size and order (R.alone says which).
int build_row_plan(int stride, const uint8_t *etype, int64_t N, int64_t E, const int32_t *conn,
                   const int32_t *rowptr, const int32_t *colidx, RowPlan &R, std::string &err,
                   const std::function<void()> &fetch = nullptr, RowForm form = kRowShared);

// Owner plan of the matrix assembly (rowplan.cpp): the CSR rows are cut
// into groups of consecutive rows (mesh numbering, so spatially compact);
// one work-group owns a group, computes every element contribution to its
// rows and writes each row once.  A task is one lane's share: an element's
// rows that the group owns, at most 4 of them for HEX08 (the element is
// presented in a rotated node order that puts them on its first face; an
// element with owned nodes on no single face gives two tasks), every row of
// the element for the other types (rows the group does not own are
// dropped).  Tasks of one phase hold distinct owned rows (of the group, or,
// for wave-private accumulation, of the wave).
constexpr int kOwnTasks = 256;            // lanes of an owner work-group
constexpr int kOwnNodes = 1024;           // touched nodes of a group (uint16 local ids)
using OwnLn = uint16_t;                   // a task's group-local node index
constexpr int kOwnLdsBytes = 64 * 1024;   // LDS of a group for the momentum operator
struct OwnGroup {
    int32_t first_task, n_tasks, first_row, n_rows;
};
struct OwnerPlan {
    int ra = 0;                          // rows per task (4 for HEX08, else nodes per element)
    bool wave_private = false;           // each wave accumulates into its own copy of the group's rows
                                         // (phases per wave, no barriers; the copies are summed in wave
                                         // order); else one copy, phases over the group with barriers
    int ln_stride = 0, off_stride = 0;   // entries per task of tk_ln, bytes per task of tk_off
    int max_nodes = 0, max_img = 0, max_rows = 0, max_phase = 0;
    std::vector<OwnGroup> groups;
    std::vector<int32_t> node_ptr, nodes;   // per group: owned rows first, then the halo ascending
    std::vector<uint8_t> nphase;            // [groups]
    std::vector<int32_t> tk_elem;           // [T] mesh element
    std::vector<OwnLn> tk_ln;               // [T][ln_stride] local node of each (rotated) element node
    std::vector<uint8_t> tk_off;            // [T][off_stride] position of column b in row r (owned rows)
    std::vector<uint8_t> tk_phase;          // [T]
};
// Single-type meshes only (P.etype empty).  0 or an fe_status code with a
// message in err.
int build_owner_plan(const Plan &P, OwnerPlan &O, std::string &err);
// Rearranges a HEX08 owner plan for the kernel: each group's tasks dealt to
// its wavefronts of 64 (all but the last full) so that tasks of one wavefront
// hold a row at different local places where possible.  tk_phase becomes the
// task's step within its wavefront (tasks of one step hold any row at most
// once per local place) and nphase the steps of the group's longest wavefront:
// the kernel adds wavefront after wavefront, local row after local row.
void arrange_waves(OwnerPlan &O);
// The node order of a HEX08 element seen from face f (0..5: -z, +z, -y, +y,
// -x, +x): kHexFaceRot[f][b] is the element's local node at the rotated
// element's node b; nodes 0-3 of the rotated element are face f.
extern const int kHexFaceRot[6][8];

// Row blocks of the symmetric PCG SpMV (Section 5.2's matrix-vector product
// on an SPD matrix).  A block is a run of consecutive rows r0..r1-1, built
// like the general SpMV's blocks.  Of each pair of entries (i, j), (j, i)
// with both rows in the block, only the upper one (j > i) is stored; the
// lower one is a mirror entry that reads the stored value.  Per block:
//   * <= kSymRows rows, <= kSymStored stored entries, <= kSymMirrors mirror
//     entries, <= kSymCols columns in its column set;
//   * the column set lists the block's own rows first (slot r - r0), then
//     its other columns in first-touch order;
//   * desc[4 b .. 4 b + 3] = {first row, first stored entry in the packed
//     value array, first mirror word, first column of the set}; b = nrb is
//     the end sentinel;
//   * roff[first row + b + i] (i = 0..rows) = offset of row i's stored
//     entries from the block's first | offset of its mirrors from the
//     block's first mirror << 16;
//   * lidx: one set slot per packed entry (parallel to the packed values);
//   * mir: two 16-bit mirror entries per word, each the window position of
//     the stored value (first stored entry's position modulo 4 plus its
//     index in the block; 10 bits) | the mirrored row minus the first row
//     << 10 (6 bits); a block's mirrors start at an even index;
//   * mstart[i]: the position in row i of its first mirror.  Rows are
//     sorted, so a row's mirrors (columns r0 .. i-1) are one run of its
//     entries; the packed position of entry k of row i is the block's first
//     stored entry + row i's stored offset + k, less the run's length when
//     k is past the run.
// Packed positions of stored entries follow CSR order with the mirrors left
// out; each row chunk (kPlanRowChunk rows) starts at a multiple of 4.
constexpr int kSymRows = 64, kSymStored = 1021, kSymMirrors = 512, kSymCols = 256;
struct SymMap {
    int64_t nrb = 0, n_packed = 0, n_mirror_words = 0;
    std::vector<int32_t> desc;    // [nrb + 1][4]
    std::vector<uint32_t> roff;   // [N + nrb]
    std::vector<uint8_t> lidx;    // [n_packed + 4]
    std::vector<uint32_t> mir;    // [n_mirror_words + 1]
    std::vector<int32_t> cols;
    std::vector<uint8_t> mstart;  // [N]
};
// 0, or FE_EBADMESH when the pattern is not structurally symmetric, a row is
// not sorted or does not fit a block (err says which).
int build_sym_map(int64_t N, const int32_t *rowptr, const int32_t *colidx, SymMap &S, std::string &err);

// Number of worker threads used by the host preprocessing.
int host_threads();
// Caps host_threads() for the calling thread (0: no cap); planner threads
// of the serving runtime plan one mesh each on a single thread.
void set_thread_budget(int n);

}  // namespace feasm
