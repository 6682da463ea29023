// rowplan.cpp -- host planning of the row-owner assembly (3x3-block momentum
// operator).
//
// The block operator's values are nine times the scalar operator's, so it is
// assembled with every CSR row written exactly once and never read back:
//   * a task is one (element, row) pair: element e's contribution to the
//     block row of one of its nodes;
//   * tasks are ordered by row (mesh numbering), and within a row by element;
//   * consecutive rows are packed into groups: whole rows only, at most
//     256 lanes (small meshes: 64) and row_image block values, so each group owns
//     its rows outright (no other adds to them) and holds their image in LDS;
//     its distinct elements (~90 to 256 tasks of HEX08; 35 to 64) and nodes
//     are listed, so that their data is computed and staged once;
//   * a row's tasks add in rounds of up to 8, all at once: the order in which
//     each adds its element's nodes is an edge colouring of the bipartite
//     graph (tasks, columns), so no two add to one column in one step.
#include <algorithm>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "../../include/feasm.h"
#include "plan.h"

namespace feasm {

namespace {

// The slots and rounds of one row's tasks.  Tasks are taken in order, up to D
// to a round while no column occurs more than D times in it; D colours (slots)
// then suffice (Koenig's theorem), found edge by edge, exchanging two colours
// along a path where an edge's ends share no free one.
class RowSlots {
  public:
    // D: the most nodes of the row's elements; cols_of [nt][8]: the columns (positions in the row) of each task's nen nodes
    void row(int D, int nt, const uint8_t *cols_of, const uint8_t *nen, uint32_t *perm, uint8_t *cols, uint8_t *round)
    {
        D_ = D;
        int t0 = 0, r = 0;
        while (t0 < nt) {
            int m = 0;
            for (; t0 + m < nt && m < D_; ++m) {
                const uint8_t *c = cols_of + 8 * (t0 + m);
                int b = 0;
                for (; b < nen[t0 + m]; ++b)
                    if (++mult_[c[b]] > D_) break;
                if (b < nen[t0 + m]) {
                    for (; b >= 0; --b) --mult_[c[b]];
                    break;
                }
            }
            colour(m, cols_of + 8 * t0, nen + t0);
            for (int i = 0; i < m; ++i) {
                const uint8_t *c = cols_of + 8 * (t0 + i);
                perm[t0 + i] = 0;
                for (int q = 0; q < 8; ++q) {
                    const int b = q < D_ ? at_task_[i][q] : -1;
                    perm[t0 + i] |= (uint32_t)(b < 0 ? 8 : b) << (4 * q);
                    cols[8 * (t0 + i) + q] = b < 0 ? 0 : c[b];
                }
                round[t0 + i] = (uint8_t)r;
                for (int b = 0; b < nen[t0 + i]; ++b) mult_[c[b]] = used_[c[b]] = 0;
            }
            t0 += m;
            ++r;
        }
    }

  private:
    void colour(int m, const uint8_t *cols_of, const uint8_t *nen)
    {
        const unsigned all = (1u << D_) - 1;
        for (int i = 0; i < m; ++i) {
            unsigned free_t = all;
            for (int q = 0; q < 8; ++q) at_task_[i][q] = -1;
            for (int b = 0; b < nen[i]; ++b) {
                const int x = cols_of[8 * i + b];
                const unsigned both = free_t & ~used_[x];
                int q;
                if (both) {
                    q = __builtin_ctz(both);
                } else {
                    q = __builtin_ctz(free_t);
                    exchange(x, q, __builtin_ctz(all & ~used_[x]), cols_of);
                }
                free_t &= ~(1u << q);
                used_[x] |= (uint8_t)(1u << q);
                at_task_[i][q] = (int8_t)b;
                at_col_[x][q] = (int8_t)i;
            }
        }
    }
    // Exchanges colours al and be along the path from column x along al (be is
    // free at x; the path does not reach the task that al is free at).
    void exchange(int x, int al, int be, const uint8_t *cols_of)
    {
        struct Edge {
            int task, node, col, q;
        } path[16];
        int n = 0;
        for (int y = x; used_[y] >> al & 1;) {
            const int j = at_col_[y][al];
            path[n++] = {j, at_task_[j][al], y, al};
            const int nb = at_task_[j][be];
            if (nb < 0) break;
            y = cols_of[8 * j + nb];
            path[n++] = {j, nb, y, be};
        }
        for (int k = 0; k < n; ++k) {
            at_task_[path[k].task][path[k].q] = -1;
            used_[path[k].col] &= (uint8_t)~(1u << path[k].q);
        }
        for (int k = 0; k < n; ++k) {
            const int q = path[k].q == al ? be : al;
            at_task_[path[k].task][q] = (int8_t)path[k].node;
            at_col_[path[k].col][q] = (int8_t)path[k].task;
            used_[path[k].col] |= (uint8_t)(1u << q);
        }
    }
    int D_ = 8;
    int8_t at_task_[8][8], at_col_[256][8];   // a task's node, a column's task in each slot
    uint8_t used_[256] = {};                  // a column's slots (which at_col_ holds)
    uint8_t mult_[256] = {};
};

}  // namespace

int build_row_plan(int stride, const uint8_t *etype, int64_t N, int64_t E, const int32_t *conn,
                   const int32_t *rowptr, const int32_t *colidx, RowPlan &R, std::string &err)
{
    R = RowPlan();
    auto nen_of = [&](int64_t e) { return etype ? (int)etype[e] : stride; };
    // node -> element incidence, elements ascending
    std::vector<int32_t> inc_ptr(N + 1, 0);
    for (int64_t e = 0; e < E; ++e)
        for (int a = 0; a < nen_of(e); ++a) ++inc_ptr[conn[e * stride + a] + 1];
    for (int64_t i = 0; i < N; ++i) {
        if (inc_ptr[i + 1] > kRowElemsMax) {
            err = "node " + std::to_string(i) + " (mesh numbering) lies in " + std::to_string(inc_ptr[i + 1]) +
                  " elements; the block operator's row-owner assembly takes at most " +
                  std::to_string(kRowElemsMax);
            return FE_EBADMESH;
        }
        inc_ptr[i + 1] += inc_ptr[i];
    }
    const int64_t T = inc_ptr[N];
    R.lanes = T < kRowSmallMesh ? kRowTasksSmall : kRowTasks;
    UnsetVector<int32_t> task_elem(T);
    UnsetVector<uint8_t> task_row(T);   // local row a
    {
        std::vector<int32_t> fill(inc_ptr.begin(), inc_ptr.end() - 1);
        for (int64_t e = 0; e < E; ++e)
            for (int a = 0; a < nen_of(e); ++a) {
                const int32_t t = fill[conn[e * stride + a]]++;
                task_elem[t] = (int32_t)e;
                task_row[t] = (uint8_t)a;
            }
    }
    // the rows' slots, in tasks order
    UnsetVector<uint32_t> perm(T);
    UnsetVector<uint8_t> cols((size_t)T * 8), round(T);
    constexpr int64_t kRows = 512;   // per chunk
    const int64_t CR = (N + kRows - 1) / kRows;
    std::vector<uint8_t> missing(CR, 0);
    std::vector<std::vector<int32_t>> place(parallel_workers(CR));   // per worker, [N]: a column's position
    parallel_chunks_w(CR, [&](int64_t c, int wk) {
        RowSlots slots;
        uint8_t of[kRowElemsMax * 8], nen[kRowElemsMax];
        std::vector<int32_t> &at = place[wk];
        at.resize(N);
        for (int64_t row = c * kRows; row < std::min(N, (c + 1) * kRows); ++row) {
            const int32_t *c0 = colidx + rowptr[row];
            const int32_t len = std::min(rowptr[row + 1] - rowptr[row], 256);
            for (int32_t p = 0; p < len; ++p) at[c0[p]] = p;
            const int32_t t0 = inc_ptr[row];
            const int nt = inc_ptr[row + 1] - t0;
            int D = 1;
            for (int t = 0; t < nt; ++t) {
                const int64_t e = task_elem[t0 + t];
                nen[t] = (uint8_t)nen_of(e);
                D = std::max<int>(D, nen[t]);
                for (int b = 0; b < nen[t]; ++b) {
                    const int32_t j = conn[e * stride + b], p = at[j];
                    if (p < 0 || p >= len || c0[p] != j) missing[c] = 1;
                    of[8 * t + b] = (uint8_t)p;
                }
            }
            if (nt > 0 && !missing[c]) slots.row(D, nt, of, nen, &perm[t0], &cols[(size_t)t0 * 8], &round[t0]);
        }
    });
    for (int64_t c = 0; c < CR; ++c)
        if (missing[c]) {
            err = "the CSR pattern lacks an element's node pair";
            return FE_EBADMESH;
        }
    // Lane of each of a row's tasks in its group, from lane p on (at [0] of its
    // tasks' lanes if given); the next free lane.  A round's tasks lie in one
    // wavefront, so that they add in step.
    const auto lanes_of = [&](int64_t row, int p, int *lane) {
        for (int32_t t = inc_ptr[row]; t < inc_ptr[row + 1];) {
            int m = 1;
            while (t + m < inc_ptr[row + 1] && round[t + m] == round[t]) ++m;
            if (p % 64 + m > 64) p = (p + 63) / 64 * 64;
            for (int q = 0; q < m; ++q, ++p)
                if (lane) *lane++ = p;
            t += m;
        }
        return p;
    };
    // whole rows into groups
    int64_t r = 0;
    int32_t tasks = 0;
    while (r < N) {
        const int64_t r0 = r;
        int p = 0;
        while (r < N) {
            const int next = lanes_of(r, p, nullptr);
            const int64_t img = 9 * (int64_t)(rowptr[r + 1] - rowptr[r0]);
            if (r > r0 && (next > R.lanes || img > row_image(R.lanes) || r - r0 >= R.lanes)) break;
            p = next;
            ++r;
        }
        R.wdesc.push_back({tasks, p, (int32_t)r0, (int32_t)(r - r0)});
        tasks += p;
        R.max_img = std::max<int64_t>(R.max_img, 9 * (int64_t)(rowptr[r] - rowptr[r0]));
    }
    R.n_tasks = tasks;
    R.nen = !etype ? stride : std::all_of(etype, etype + E, [&](uint8_t n) { return n == etype[0]; }) ? etype[0] : 0;
    if (R.nen == 0) {
        std::vector<uint8_t> cls(R.wdesc.size());
        for (size_t w = 0; w < R.wdesc.size(); ++w) {
            const RowWave &q = R.wdesc[w];
            const int32_t t0 = inc_ptr[q.first_row], t1 = inc_ptr[q.first_row + q.n_rows];
            cls[w] = t0 < t1 ? etype[task_elem[t0]] : 0;
            for (int32_t t = t0; t < t1; ++t)
                if (etype[task_elem[t]] != cls[w]) cls[w] = 0;
        }
        std::vector<RowWave> by_row = std::move(R.wdesc);
        R.wdesc.clear();
        const int order[5] = {0, 8, 5, 6, 4};
        for (int c = 0; c < 5; ++c) {
            for (size_t w = 0; w < by_row.size(); ++w)
                if (cls[w] == order[c]) R.wdesc.push_back(by_row[w]);
            if (c < 4) R.class_end[c] = (int32_t)R.wdesc.size();
        }
    }
    // each group's elements and nodes, in the order of their first use by its
    // tasks: counted, then listed
    const int64_t W = (int64_t)R.wdesc.size();
    R.task_meta.resize(tasks);
    R.task_perm.resize(tasks);
    R.task_cols.resize((size_t)tasks * 8);
    R.wlists.resize(W);
    constexpr int64_t kGroups = 32;   // per chunk
    const int64_t C = (W + kGroups - 1) / kGroups;
    // per worker: an element's and a node's place in its group's list, which
    // counts if the list holds it there; the lists
    struct Lists {
        std::vector<int32_t> elem_at, node_at, elems, nodes;
        std::vector<uint16_t> ln;
    };
    std::vector<Lists> work(parallel_workers(C));
    const auto listed = [](std::vector<int32_t> &list, std::vector<int32_t> &at, int32_t x) {
        const size_t p = (size_t)(uint32_t)at[x];
        if (p < list.size() && list[p] == x) return (int32_t)p;
        list.push_back(x);
        return at[x] = (int32_t)list.size() - 1;
    };
    const auto make = [&](const RowWave &q, Lists &l) {
        l.elem_at.resize(E);
        l.node_at.resize(N);
        l.elems.clear();
        l.nodes.clear();
        l.ln.clear();
        for (int32_t t = inc_ptr[q.first_row]; t < inc_ptr[q.first_row + q.n_rows]; ++t)
            (void)listed(l.elems, l.elem_at, task_elem[t]);
        for (const int32_t e : l.elems) {
            const int32_t *ce = conn + (int64_t)e * stride;
            const int n = nen_of(e);
            for (int b = 0; b < 8; ++b) l.ln.push_back(b < n ? (uint16_t)listed(l.nodes, l.node_at, ce[b]) : (uint16_t)0);
        }
    };
    parallel_chunks_w(C, [&](int64_t c, int wk) {
        for (int64_t w = c * kGroups; w < std::min(W, (c + 1) * kGroups); ++w) {
            make(R.wdesc[w], work[wk]);
            R.wlists[w] = {0, (int32_t)work[wk].elems.size(), 0, (int32_t)work[wk].nodes.size()};
        }
    });
    int32_t ne = 0, nn = 0;
    for (RowLists &l : R.wlists) {
        l.first_elem = ne;
        l.first_node = nn;
        ne += l.n_elems;
        nn += l.n_nodes;
        R.max_items = std::max<int64_t>(R.max_items, (int64_t)l.n_elems * row_points(l.n_elems, R.lanes));
        R.max_nodes = std::max<int64_t>(R.max_nodes, l.n_nodes);
    }
    R.wave_elem.resize(ne);
    R.wave_node.resize(nn);
    R.wave_ln.resize((size_t)ne * 8);
    parallel_chunks_w(C, [&](int64_t c, int wk) {
        Lists &l = work[wk];
        int lane[kRowElemsMax];
        for (int64_t w = c * kGroups; w < std::min(W, (c + 1) * kGroups); ++w) {
            const RowWave &q = R.wdesc[w];
            make(q, l);
            std::copy(l.elems.begin(), l.elems.end(), R.wave_elem.begin() + R.wlists[w].first_elem);
            std::copy(l.nodes.begin(), l.nodes.end(), R.wave_node.begin() + R.wlists[w].first_node);
            std::copy(l.ln.begin(), l.ln.end(), R.wave_ln.begin() + (size_t)R.wlists[w].first_elem * 8);
            const size_t t0 = (size_t)q.first_task;
            std::fill_n(R.task_meta.begin() + t0, q.n_tasks, kRowNoTask);
            std::fill_n(R.task_perm.begin() + t0, q.n_tasks, 0x88888888u);
            std::fill_n(R.task_cols.begin() + t0 * 8, (size_t)q.n_tasks * 8, (uint8_t)0);
            int p = 0;
            for (int i = 0; i < q.n_rows; ++i) {
                const int64_t row = q.first_row + i;
                p = lanes_of(row, p, lane);
                for (int32_t t = inc_ptr[row]; t < inc_ptr[row + 1]; ++t) {
                    const int k = t - inc_ptr[row];
                    const size_t d = t0 + lane[k];
                    R.task_meta[d] = (uint32_t)l.elem_at[task_elem[t]] | (uint32_t)task_row[t] << 8 | (uint32_t)i << 11 |
                                     (uint32_t)round[t] << 19 | (k == 0 ? kRowFirstTask : 0u);
                    R.task_perm[d] = perm[t];
                    memcpy(&R.task_cols[d * 8], &cols[(size_t)t * 8], 8);
                }
            }
        }
    });
    return FE_OK;
}

}  // namespace feasm

namespace feasm {

// Proper rotations of the reference cube taking each face to the first one
// (z = -1): rotated node b is the original node kHexFaceRot[f][b].
const int kHexFaceRot[6][8] = {
    {0, 1, 2, 3, 4, 5, 6, 7},   // -z: identity
    {7, 6, 5, 4, 3, 2, 1, 0},   // +z: half turn about the x axis
    {4, 5, 1, 0, 7, 6, 2, 3},   // -y: quarter turn about x
    {3, 2, 6, 7, 0, 1, 5, 4},   // +y: quarter turn about x, the other way
    {4, 0, 3, 7, 5, 1, 2, 6},   // -x: quarter turn about y
    {1, 5, 6, 2, 0, 4, 7, 3},   // +x: quarter turn about y, the other way
};

namespace {

// Bit masks of the six faces' nodes.
uint8_t face_mask(int f)
{
    uint8_t m = 0;
    for (int b = 0; b < 4; ++b) m |= (uint8_t)(1u << kHexFaceRot[f][b]);
    return m;
}

}  // namespace

int build_owner_plan(const Plan &P, OwnerPlan &O, std::string &err)
{
    O = OwnerPlan();
    if (!P.etype.empty()) {
        err = "owner plan: one element type per mesh";
        return FE_EINVAL;
    }
    const int nen = P.nen;
    const int64_t N = P.N, E = P.E;
    const bool hex = nen == 8;
    O.ra = hex ? 4 : nen;
    // the other types' nodes lie in many elements (24 for a Kuhn
    // tetrahedron's), which would make as many barrier-separated phases:
    // their waves accumulate privately instead
    O.wave_private = !hex;
    const int copies = O.wave_private ? kOwnTasks / 64 : 1;
    O.ln_stride = nen;
    O.off_stride = (O.ra * nen + 3) & ~3;
    const int32_t *conn = P.conn.data();
    const int32_t *rowptr = P.rowptr.data(), *colidx = P.colidx.data();

    // tasks needed to cover a set of owned element nodes
    uint8_t fmask[6];
    for (int f = 0; f < 6; ++f) fmask[f] = face_mask(f);
    uint8_t cover[256];
    for (int m = 0; m < 256; ++m) {
        if (m == 0) cover[m] = 0;
        else if (!hex) cover[m] = 1;
        else {
            cover[m] = 2;
            for (int f = 0; f < 6; ++f)
                if ((m & ~fmask[f]) == 0) cover[m] = 1;
        }
    }
    // node -> (element, local index) incidence, elements ascending
    std::vector<int32_t> inc_ptr(N + 1, 0);
    for (int64_t e = 0; e < E; ++e)
        for (int a = 0; a < nen; ++a) ++inc_ptr[conn[e * nen + a] + 1];
    for (int64_t i = 0; i < N; ++i) inc_ptr[i + 1] += inc_ptr[i];
    std::vector<int32_t> inc(inc_ptr[N]);
    {
        std::vector<int32_t> fill(inc_ptr.begin(), inc_ptr.end() - 1);
        for (int64_t e = 0; e < E; ++e)
            for (int a = 0; a < nen; ++a) inc[fill[conn[e * nen + a]]++] = (int32_t)(e * 8 + a);
    }
    auto lds_bytes = [&](int64_t tn, int64_t img, int64_t nr) {
        return (kNodeFields * tn + copies * (img + kMaxRhs * nr)) * 8;
    };

    // 1. groups of consecutive rows: row r joins the open group unless the
    //    group's tasks, touched nodes or LDS would then exceed their limits
    std::vector<int32_t> estamp(E, -1), nstamp(N, -1);
    std::vector<int64_t> nmark(N, -1);
    std::vector<uint8_t> emask(E, 0);
    std::vector<int32_t> gstart(1, 0);   // first row of each group
    int32_t gid = 0;
    int64_t mark = 0;
    auto cost = [&](int64_t r, int64_t &dt, int64_t &dn) {
        dt = dn = 0;
        ++mark;
        for (int32_t q = inc_ptr[r]; q < inc_ptr[r + 1]; ++q) {
            const int32_t e = inc[q] >> 3, a = inc[q] & 7;
            const uint8_t old = estamp[e] == gid ? emask[e] : 0;
            dt += cover[old | (1u << a)] - cover[old];
            if (estamp[e] == gid) continue;
            for (int b = 0; b < nen; ++b) {
                const int32_t v = conn[(int64_t)e * nen + b];
                if (nstamp[v] != gid && nmark[v] != mark) {
                    nmark[v] = mark;
                    ++dn;
                }
            }
        }
    };
    auto commit = [&](int64_t r) {
        for (int32_t q = inc_ptr[r]; q < inc_ptr[r + 1]; ++q) {
            const int32_t e = inc[q] >> 3, a = inc[q] & 7;
            if (estamp[e] != gid) {
                estamp[e] = gid;
                emask[e] = 0;
                for (int b = 0; b < nen; ++b) nstamp[conn[(int64_t)e * nen + b]] = gid;
            }
            emask[e] |= (uint8_t)(1u << a);
        }
    };
    int64_t tasks = 0, tn = 0, img = 0, r0 = 0;
    for (int64_t r = 0; r < N; ++r) {
        int64_t dt, dn;
        cost(r, dt, dn);
        const int64_t len = rowptr[r + 1] - rowptr[r];
        auto over = [&](int64_t t_, int64_t n_, int64_t img_, int64_t nr_) {
            return t_ > kOwnTasks || n_ > kOwnNodes || nr_ > kOwnNodes || lds_bytes(n_, img_, nr_) > kOwnLdsBytes;
        };
        if (r > r0 && over(tasks + dt, tn + dn, img + len, r - r0 + 1)) {
            ++gid;
            gstart.push_back((int32_t)r);
            r0 = r;
            tasks = tn = img = 0;
            cost(r, dt, dn);
        }
        if (over(tasks + dt, tn + dn, img + len, r - r0 + 1)) {
            err = "node " + std::to_string(r) + " (mesh numbering): its elements exceed one owner group";
            return FE_EBADMESH;
        }
        commit(r);
        tasks += dt;
        tn += dn;
        img += len;
    }
    gstart.push_back((int32_t)N);
    const int64_t G = (int64_t)gstart.size() - 1;

    // 2. per group: node list, tasks, in-row offsets, phases.  Groups are
    //    independent; a first pass counts each group's nodes and tasks, a
    //    second writes them at their final places.
    std::vector<int32_t> gnodes(G), gtasks(G);
    std::vector<uint8_t> gbad(G, 0);
    const int nt = std::max(1, std::min<int>(host_threads(), (int)((G + 63) / 64)));
    auto run = [&](auto &&body) {
        std::vector<std::thread> th;
        for (int t = 0; t < nt; ++t) th.emplace_back([&, t] { body(t); });
        for (auto &x : th) x.join();
    };
    // the elements of group g, ascending (est: per-thread stamps, [E])
    auto group_elems = [&](int64_t g, std::vector<int32_t> &elems, std::vector<int32_t> &est) {
        elems.clear();
        for (int32_t r = gstart[g]; r < gstart[g + 1]; ++r)
            for (int32_t q = inc_ptr[r]; q < inc_ptr[r + 1]; ++q) {
                const int32_t e = inc[q] >> 3;
                if (est[e] != (int32_t)g) {
                    est[e] = (int32_t)g;
                    elems.push_back(e);
                }
            }
        std::sort(elems.begin(), elems.end());
    };
    auto owned_mask = [&](int32_t e, int32_t a0, int32_t a1) {
        uint8_t m = 0;
        for (int b = 0; b < nen; ++b) {
            const int32_t v = conn[(int64_t)e * nen + b];
            if (v >= a0 && v < a1) m |= (uint8_t)(1u << b);
        }
        return m;
    };
    run([&](int t) {
        std::vector<int32_t> elems, est(E, -1), nst(N, -1);
        for (int64_t g = t; g < G; g += nt) {
            const int32_t a0 = gstart[g], a1 = gstart[g + 1];
            group_elems(g, elems, est);
            int32_t tasks_g = 0, nh = 0;
            for (int32_t e : elems) {
                tasks_g += cover[owned_mask(e, a0, a1)];
                for (int b = 0; b < nen; ++b) {
                    const int32_t v = conn[(int64_t)e * nen + b];
                    if ((v < a0 || v >= a1) && nst[v] != (int32_t)g) {
                        nst[v] = (int32_t)g;
                        ++nh;
                    }
                }
            }
            gnodes[g] = (a1 - a0) + nh;
            gtasks[g] = tasks_g;
        }
    });
    O.node_ptr.assign(G + 1, 0);
    O.groups.resize(G);
    int64_t T = 0;
    for (int64_t g = 0; g < G; ++g) {
        O.node_ptr[g + 1] = O.node_ptr[g] + gnodes[g];
        O.groups[g] = {(int32_t)T, gtasks[g], gstart[g], gstart[g + 1] - gstart[g]};
        T += gtasks[g];
    }
    O.nodes.resize(O.node_ptr[G]);
    O.nphase.assign(G, 0);
    O.tk_elem.resize(T);
    O.tk_ln.assign((size_t)T * O.ln_stride, 0);
    O.tk_off.assign((size_t)T * O.off_stride, 0);
    O.tk_phase.resize(T);
    std::vector<int32_t> gimg(G);
    run([&](int t) {
        std::vector<int32_t> lidx(N, -1);   // node -> local index in the current group
        std::vector<int32_t> elems, est(E, -1);
        std::vector<uint8_t> pos;             // [owned row][local node]: position in the row
        std::vector<uint64_t> used;
        struct Tk {
            int32_t e;
            uint8_t ph, off[36];
            OwnLn ln[8];
        };
        std::vector<Tk> tk;
        std::vector<int32_t> cnt, wcnt, wfill, wof;
        for (int64_t g = t; g < G; g += nt) {
            const int32_t a0 = gstart[g], a1 = gstart[g + 1], nr = a1 - a0;
            int32_t *gn = O.nodes.data() + O.node_ptr[g];
            const int32_t T_g = gnodes[g];
            group_elems(g, elems, est);
            for (int32_t r = a0; r < a1; ++r) gn[r - a0] = r;
            int32_t nh = nr;
            for (int32_t e : elems)
                for (int b = 0; b < nen; ++b) {
                    const int32_t v = conn[(int64_t)e * nen + b];
                    if ((v < a0 || v >= a1) && lidx[v] != -2) {
                        lidx[v] = -2;   // mark: collected once
                        gn[nh++] = v;
                    }
                }
            std::sort(gn + nr, gn + nh);
            if (nh != T_g || T_g > kOwnNodes) gbad[g] = 1;
            for (int32_t k = 0; k < nh; ++k) lidx[gn[k]] = k;
            // in-row position of every touched node for each owned row
            pos.assign((size_t)nr * T_g, 0xff);
            for (int32_t r = a0; r < a1; ++r)
                for (int32_t q = rowptr[r]; q < rowptr[r + 1]; ++q) {
                    const int32_t lc = lidx[colidx[q]];
                    if (lc < 0 || lc >= T_g) {
                        gbad[g] = 1;
                        continue;
                    }
                    pos[(size_t)(r - a0) * T_g + lc] = (uint8_t)(q - rowptr[r]);
                }
            gimg[g] = rowptr[a1] - rowptr[a0];
            used.assign(4 * (size_t)nr, 0);
            tk.clear();
            int nph = 0;
            auto add_task = [&](int32_t e, const int *rot) {
                Tk x{};
                x.e = e;
                for (int b = 0; b < nen; ++b) x.ln[b] = (OwnLn)lidx[conn[(int64_t)e * nen + (rot ? rot[b] : b)]];
                for (int r = 0; r < O.ra; ++r) {
                    if (x.ln[r] >= nr) continue;   // a row another group owns
                    const uint8_t *pr = pos.data() + (size_t)x.ln[r] * T_g;
                    for (int b = 0; b < nen; ++b) {
                        const uint8_t o = pr[x.ln[b]];
                        if (o == 0xff) gbad[g] = 1;
                        x.off[r * nen + b] = o;
                    }
                }
                tk.push_back(x);
            };
            // greedy phase: the smallest one none of the task's owned rows has
            // taken (among the tasks sharing its accumulation copy)
            auto take_phase = [&](Tk &x) {
                uint64_t m[4] = {0, 0, 0, 0};
                for (int r = 0; r < O.ra; ++r)
                    if (x.ln[r] < nr)
                        for (int w = 0; w < 4; ++w) m[w] |= used[4 * (size_t)x.ln[r] + w];
                int ph = 0;
                while (ph < 256 && ((m[ph >> 6] >> (ph & 63)) & 1)) ++ph;
                if (ph >= 256) {   // cannot happen: a group holds at most 256 tasks
                    gbad[g] = 1;
                    ph = 255;
                }
                for (int r = 0; r < O.ra; ++r)
                    if (x.ln[r] < nr) used[4 * (size_t)x.ln[r] + (ph >> 6)] |= 1ull << (ph & 63);
                x.ph = (uint8_t)ph;
                nph = std::max(nph, ph + 1);
            };
            for (int32_t e : elems) {
                const uint8_t m = owned_mask(e, a0, a1);
                if (!hex) {
                    add_task(e, nullptr);
                } else if (cover[m] == 1) {
                    int f = 0;
                    while ((m & ~fmask[f]) != 0) ++f;
                    add_task(e, kHexFaceRot[f]);
                } else {
                    add_task(e, kHexFaceRot[0]);
                    add_task(e, kHexFaceRot[1]);
                }
            }
            if ((int32_t)tk.size() != gtasks[g] || (int)tk.size() > kOwnTasks) gbad[g] = 1;
            if (O.wave_private) {
                // spread each row's tasks over the waves: a task goes to the
                // wave (with room) where its owned rows have the fewest tasks
                // yet, which bounds the phases each wave steps through
                const int nw = (int)((tk.size() + 63) / 64);
                wcnt.assign((size_t)nw * nr, 0);
                wfill.assign(nw, 0);
                wof.resize(tk.size());
                // every wave but the last holds exactly 64 tasks (a task's
                // wave is its lane / 64 in the kernel)
                auto cap = [&](int w) { return w < nw - 1 ? 64 : (int)tk.size() - 64 * (nw - 1); };
                for (size_t q = 0; q < tk.size(); ++q) {
                    int best = -1, bcost = 1 << 30;
                    for (int w = 0; w < nw; ++w) {
                        if (wfill[w] >= cap(w)) continue;
                        int c = 0;
                        for (int r = 0; r < O.ra; ++r)
                            if (tk[q].ln[r] < nr) c = std::max(c, wcnt[(size_t)w * nr + tk[q].ln[r]]);
                        if (c < bcost) {
                            bcost = c;
                            best = w;
                        }
                    }
                    wof[q] = best;
                    ++wfill[best];
                    for (int r = 0; r < O.ra; ++r)
                        if (tk[q].ln[r] < nr) ++wcnt[(size_t)best * nr + tk[q].ln[r]];
                }
                std::vector<Tk> by;   // tasks wave by wave, each wave in generation order
                for (int w = 0; w < nw; ++w) {
                    used.assign(4 * (size_t)nr, 0);
                    for (size_t q = 0; q < tk.size(); ++q)
                        if (wof[q] == w) {
                            take_phase(tk[q]);
                            by.push_back(tk[q]);
                        }
                }
                tk.swap(by);
            } else {
                for (Tk &x : tk) take_phase(x);
            }
            // tasks by phase, stably (a counting sort), over the group or,
            // wave-private, within each wave's 64: a wave then spans few
            // phases and skips the others' LDS additions
            const int64_t t0 = O.groups[g].first_task;
            const size_t span = O.wave_private ? 64 : tk.size() + 1;
            for (size_t w0 = 0; w0 < tk.size(); w0 += span) {
                const size_t w1 = std::min(tk.size(), w0 + span);
                cnt.assign(nph + 1, 0);
                for (size_t q = w0; q < w1; ++q) ++cnt[tk[q].ph + 1];
                for (int p = 0; p < nph; ++p) cnt[p + 1] += cnt[p];
                for (size_t q = w0; q < w1; ++q) {
                    const Tk &x = tk[q];
                    const int64_t d = t0 + (int64_t)w0 + cnt[x.ph]++;
                    if (d >= t0 + gtasks[g]) {
                        gbad[g] = 1;
                        continue;
                    }
                    O.tk_elem[d] = x.e;
                    O.tk_phase[d] = x.ph;
                    memcpy(&O.tk_ln[(size_t)d * O.ln_stride], x.ln, O.ln_stride * sizeof(OwnLn));
                    memcpy(&O.tk_off[(size_t)d * O.off_stride], x.off, O.off_stride);
                }
            }
            if (nph > 255) gbad[g] = 1;   // phase counts are stored in a byte
            O.nphase[g] = (uint8_t)nph;
            for (int32_t k = 0; k < nh; ++k) lidx[gn[k]] = -1;
        }
    });
    for (int64_t g = 0; g < G; ++g) {
        if (gbad[g]) {
            err = "owner plan: group " + std::to_string(g) + " exceeds its limits";
            return FE_EBADMESH;
        }
        O.max_nodes = std::max<int>(O.max_nodes, gnodes[g]);
        O.max_img = std::max(O.max_img, gimg[g]);
        O.max_rows = std::max<int>(O.max_rows, gstart[g + 1] - gstart[g]);
        O.max_phase = std::max<int>(O.max_phase, O.nphase[g]);
    }
    return FE_OK;
}

void arrange_waves(OwnerPlan &O)
{
    const int64_t G = (int64_t)O.groups.size();
    const int ra = O.ra, ls = O.ln_stride, os = O.off_stride;
    parallel_chunks((G + 255) / 256, [&](int64_t c) {
        std::vector<uint8_t> cnt;   // [wave][owned row][local place]: tasks that hold it
        std::vector<int32_t> of, elem;
        std::vector<uint8_t> step, off;
        std::vector<OwnLn> ln;
        for (int64_t g = c * 256; g < std::min<int64_t>(G, (c + 1) * 256); ++g) {
            const OwnGroup &q = O.groups[g];
            const int n = q.n_tasks, nr = q.n_rows, nw = (n + 63) / 64;
            cnt.assign((size_t)nw * nr * ra, 0);
            int fill[kOwnTasks / 64] = {};
            of.resize(n);
            step.resize(n);
            int steps = 1;
            for (int t = 0; t < n; ++t) {
                const OwnLn *l = &O.tk_ln[(size_t)(q.first_task + t) * ls];
                int best = -1, bc = 256;
                for (int w = 0; w < nw; ++w) {
                    if (fill[w] >= (w < nw - 1 ? 64 : n - 64 * (nw - 1))) continue;
                    int m = 0;
                    for (int r = 0; r < ra; ++r)
                        if (l[r] < nr) m = std::max<int>(m, cnt[((size_t)w * nr + l[r]) * ra + r]);
                    if (m < bc) {
                        bc = m;
                        best = w;
                    }
                }
                of[t] = best;
                step[t] = (uint8_t)bc;
                ++fill[best];
                for (int r = 0; r < ra; ++r)
                    if (l[r] < nr) cnt[((size_t)best * nr + l[r]) * ra + r] = (uint8_t)(bc + 1);
                steps = std::max(steps, bc + 1);
            }
            const size_t t0 = (size_t)q.first_task;
            elem.assign(O.tk_elem.begin() + t0, O.tk_elem.begin() + t0 + n);
            ln.assign(O.tk_ln.begin() + t0 * ls, O.tk_ln.begin() + (t0 + n) * ls);
            off.assign(O.tk_off.begin() + t0 * os, O.tk_off.begin() + (t0 + n) * os);
            size_t d = t0;
            for (int w = 0; w < nw; ++w)
                for (int t = 0; t < n; ++t)
                    if (of[t] == w) {
                        O.tk_elem[d] = elem[t];
                        O.tk_phase[d] = step[t];
                        memcpy(&O.tk_ln[d * ls], &ln[(size_t)t * ls], ls * sizeof(OwnLn));
                        memcpy(&O.tk_off[d * os], &off[(size_t)t * os], os);
                        ++d;
                    }
            O.nphase[g] = (uint8_t)steps;
        }
    });
}

}  // namespace feasm
