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
//     (or, see RowForm, consecutive rows into wavefronts of single tasks);
//   * a row's tasks add in rounds of up to 8, all at once: the order in which
//     each adds its element's nodes is an edge colouring of the bipartite
//     graph (tasks, columns), so no two add to one column in one step.
#include <algorithm>
#include <array>
#include <atomic>
#include <climits>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <string>
#include <thread>
#include <vector>

#include "../../include/feasm.h"
#include "plan.h"

namespace feasm {

namespace {

// The slots and rounds of one row's tasks.  Tasks are taken in order, up to D
// to a round while no column occurs more than D times in it; D colours (slots)
// then suffice (Koenig's theorem).  Where every task may take its nodes in
// their own order (a row of HEX08 elements of one orientation) it does; else
// the slots are found edge by edge, exchanging two colours along a path where
// an edge's ends share no free one, and kept for the next round whose tasks
// share columns in the same way (a mesh repeats few such patterns).
class RowSlots {
  public:
    // D: the most nodes of the row's elements; cols_of [nt][8]: the columns (positions in the row) of each task's nen nodes
    void row(int D, int nt, const uint8_t *cols_of, const uint8_t *nen, uint32_t *perm, uint8_t *round)
    {
        int t0 = 0, r = 0;
        while (t0 < nt) {
            int m = std::min(nt - t0, D);
            if (!in_order(m, cols_of + 8 * t0, nen + t0, perm + t0)) {
                m = pattern(D, m, cols_of + 8 * t0, nen + t0);
                const Known &k = known(D, m, nen + t0);
                std::copy(k.perm, k.perm + m, perm + t0);
            }
            std::fill_n(round + t0, m, (uint8_t)r);
            t0 += m;
            ++r;
        }
    }

  private:
    // Slot b takes node b, if that gives no column twice in one slot.
    bool in_order(int m, const uint8_t *cols_of, const uint8_t *nen, uint32_t *perm)
    {
        const uint32_t gen = next_gen();
        for (int i = 0; i < m; ++i)
            for (int b = 0; b < nen[i]; ++b) {
                uint32_t &s = seen_[cols_of[8 * i + b]];
                if (s >> 8 != gen) s = gen << 8;
                if (s >> b & 1) return false;
                s |= 1u << b;
            }
        for (int i = 0; i < m; ++i) perm[i] = nen[i] == 8 ? 0x76543210u : 0x76543210u | 0x88888888u << (4 * nen[i]);
        return true;
    }
    // The first tasks of the m in which no column occurs more than D times
    // (their number is returned), their columns by first appearance in key_.
    int pattern(int D, int m, const uint8_t *cols_of, const uint8_t *nen)
    {
        const uint32_t gen = next_gen();
        int labels = 0;
        for (int i = 0; i < m; ++i) {
            uint8_t *k = reinterpret_cast<uint8_t *>(key_) + 8 * i;
            key_[i] = ~(uint64_t)0;
            for (int b = 0; b < nen[i]; ++b) {
                uint32_t &s = seen_[cols_of[8 * i + b]];
                if (s >> 8 != gen) {
                    s = gen << 8 | (uint32_t)labels;
                    times_[labels++] = 0;
                }
                k[b] = (uint8_t)s;
                if (++times_[k[b]] > D) return i;
            }
        }
        return m;
    }
    uint32_t next_gen()
    {
        if (++gen_ == 1u << 24) {
            std::fill(seen_, seen_ + 256, 0u);
            gen_ = 1;
        }
        return gen_;
    }
    struct Known {
        uint64_t key[8];
        uint32_t perm[8];
        int m = 0, D = 0;
    };
    const Known &known(int D, int m, const uint8_t *nen)
    {
        uint64_t h = (uint64_t)(8 * D + m);
        for (int i = 0; i < m; ++i) h = (h ^ key_[i]) * 0x9e3779b97f4a7c15ull, h ^= h >> 29;
        Known &k = known_[h >> 56];
        if (k.m == m && k.D == D && memcmp(k.key, key_, m * sizeof(uint64_t)) == 0) return k;
        D_ = D;
        const uint8_t *cols = reinterpret_cast<const uint8_t *>(key_);
        memset(used_, 0, sizeof used_);
        colour(m, cols, nen);
        for (int i = 0; i < m; ++i) {
            k.key[i] = key_[i];
            k.perm[i] = 0;
            for (int q = 0; q < 8; ++q) {
                const int b = q < D ? at_task_[i][q] : -1;
                k.perm[i] |= (uint32_t)(b < 0 ? 8 : b) << (4 * q);
            }
        }
        k.m = m;
        k.D = D;
        return k;
    }
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
    int8_t at_task_[8][8], at_col_[64][8];   // a task's node, a column's task in each slot
    uint8_t used_[64];                       // a column's slots (which at_col_ holds)
    uint8_t times_[64];
    uint64_t key_[8];
    uint32_t seen_[256] = {}, gen_ = 0;      // per column: the round that saw it, then its slots or label
    Known known_[256];
};

// nt threads that run f(w, team) together; barrier() waits for all of them.
class Team {
  public:
    explicit Team(int n) : n_(n) {}
    int size() const { return n_; }
    void barrier()
    {
        const unsigned now = turn_.load(std::memory_order_acquire);
        if (here_.fetch_add(1, std::memory_order_acq_rel) + 1 == n_) {
            here_.store(0, std::memory_order_relaxed);
            turn_.store(now + 1, std::memory_order_release);
        } else {
            while (turn_.load(std::memory_order_acquire) == now) std::this_thread::yield();
        }
    }
    template <class F> static void run(int n, F f)
    {
        Team team(n);
        start(0, n, team, f);
    }

  private:
    // Threads [lo, hi): each starts the upper half of what is left to it, since
    // starting one takes 10 us.
    template <class F> static void start(int lo, int hi, Team &team, F &f)
    {
        std::vector<std::thread> th;
        while (hi - lo > 1) {
            const int mid = (lo + hi + 1) / 2;
            th.emplace_back([mid, hi, &team, &f] { start(mid, hi, team, f); });
            hi = mid;
        }
        f(lo, team);
        for (auto &t : th) t.join();
    }
    const int n_;
    std::atomic<int> here_{0};
    std::atomic<unsigned> turn_{0};
};

// An element's or node's place in the lists of group `group` (counted from 1).
struct Placed {
    uint32_t group, place;
};
// n zeros, of which the pages that are never touched cost nothing.
template <class T> class Zeros {
  public:
    explicit Zeros(size_t n) : p_((T *)std::calloc(std::max<size_t>(n, 1), sizeof(T)))
    {
        if (!p_) throw std::bad_alloc();
    }
    Zeros(const Zeros &) = delete;
    ~Zeros() { std::free(p_); }
    T &operator[](size_t i) { return p_[i]; }

  private:
    T *p_;
};

// What one thread plans: the groups of its rows, the places in their lists
// counted from 0.  (The tasks go straight to the plan's arrays.)
struct alignas(64) RowPart {
    std::vector<RowWave> wdesc;
    std::vector<RowLists> wlists;
    std::vector<uint8_t> cls;   // a group's element type, 0 for several
    UnsetVector<int32_t> elem, node;              // of which n_elems and n_nodes are used
    UnsetVector<std::array<uint16_t, 8>> ln;
    int64_t n_elems = 0, n_nodes = 0;
    int64_t max_img = 0, max_items = 0, max_nodes = 0, too_many = -1;
    bool failed = false;
};

// The tasks of rows [r0, r1) in order of row and element, and wavefronts of
// whole rows of them (the form of each task alone).
struct RowTasks {
    int stride;
    const uint8_t *etype;
    const int32_t *conn, *rowptr, *colidx, *inc_ptr;
    const uint32_t *inc;
    uint8_t *cols;   // the plan's arrays
    int32_t *elem;
    uint16_t *meta;

    void run(int64_t N, int64_t r0, int64_t r1, RowPart &P) const
    {
        Zeros<int32_t> at(N);   // a column's position in its row
        RowWave g{inc_ptr[r0], 0, (int32_t)r0, 0};
        const auto close = [&](int64_t row) {
            g.n_rows = (int32_t)(row - g.first_row);
            g.n_tasks = inc_ptr[row] - g.first_task;
            if (g.n_rows > 0) P.wdesc.push_back(g);
            P.max_img = std::max<int64_t>(P.max_img, 9 * (int64_t)(rowptr[row] - rowptr[g.first_row]));
            g = {inc_ptr[row], 0, (int32_t)row, 0};
        };
        for (int64_t row = r0; row < r1; ++row) {
            const int64_t img = 9 * (int64_t)(rowptr[row + 1] - rowptr[g.first_row]);
            if (row > g.first_row && (inc_ptr[row + 1] - g.first_task > kRowTasksSmall ||
                                      img > row_image(kRowTasksSmall) || row - g.first_row >= kRowTasksSmall))
                close(row);
            const int32_t *c0 = colidx + rowptr[row];
            const int32_t len = std::min(rowptr[row + 1] - rowptr[row], 256);
            for (int32_t q = 0; q < len; ++q) at[c0[q]] = q;
            for (int32_t t = inc_ptr[row]; t < inc_ptr[row + 1]; ++t) {
                const int64_t e = inc[t] >> 3;
                const int n = etype ? (int)etype[e] : stride;
                uint8_t c[8] = {};
                for (int b = 0; b < n; ++b) {
                    const int32_t j = conn[e * stride + b], q = at[j];
                    if (q < 0 || q >= len || c0[q] != j) {
                        P.failed = true;
                        return;
                    }
                    c[b] = (uint8_t)q;
                }
                memcpy(cols + 8 * (size_t)t, c, 8);
                elem[t] = (int32_t)e;
                meta[t] = (uint16_t)((inc[t] & 7) | (t - inc_ptr[row]) << 4);
            }
        }
        close(r1);
    }
};

// Tasks of rows [r0, r1), of a few groups' worth (seen), and the distinct
// elements that those hold.
std::pair<int64_t, int64_t> row_sharing(const int32_t *inc_ptr, const uint32_t *inc, int64_t r0, int64_t r1)
{
    constexpr int kWindows = 4;
    std::pair<int64_t, int64_t> s{0, 0};
    std::vector<uint32_t> e;
    for (int k = 0; k < kWindows; ++k) {
        const int64_t row = r0 + (r1 - r0) * k / kWindows;
        int64_t end = row;
        while (end < r1 && inc_ptr[end + 1] - inc_ptr[row] <= kRowTasks) ++end;
        e.assign(inc + inc_ptr[row], inc + inc_ptr[end]);
        for (uint32_t &x : e) x >>= 3;
        std::sort(e.begin(), e.end());
        s.first += (int64_t)e.size();
        s.second += std::unique(e.begin(), e.end()) - e.begin();
    }
    return s;
}

// The groups of rows [r0, r1): their lanes, elements and nodes.
struct RowGrouping {
    int stride, lanes;
    const uint8_t *etype;
    const int32_t *conn, *rowptr, *colidx, *inc_ptr;
    const uint32_t *inc;   // 8 element + local row, by row
    uint32_t *meta, *perm;   // the plan's arrays
    uint64_t *cols;
    int nen_of(int64_t e) const { return etype ? (int)etype[e] : stride; }

    // Lanes that the tasks of rows [r0, r1) take at most: a round of m <= 8 may
    // leave m - 1 lanes of a wavefront idle.
    int64_t most_lanes(int64_t r0, int64_t r1) const
    {
        const int64_t n = inc_ptr[r1] - inc_ptr[r0];
        return n + 7 * (n / 57 + 1);
    }

    // first: where this range's tasks start
    // (What a thread fills step by step it allocates itself: page faults of
    // several threads in one mapping hold each other up.)
    void run(int64_t N, int64_t E, int64_t r0, int64_t r1, int64_t first, RowPart &P) const
    {
        const auto slots = std::make_unique<RowSlots>();
        Zeros<Placed> elems(E), nodes(N);
        Zeros<int32_t> at(N);   // a column's position in its row
        const size_t tasks = (size_t)(inc_ptr[r1] - inc_ptr[r0]);
        P.elem.resize(tasks + 8);   // at most one to a task; pages that stay unused are never touched
        P.ln.resize(tasks + 8);
        P.node.resize(tasks + 8);
        uint32_t gid = 1;       // the open group
        const int64_t last = first + most_lanes(r0, r1);
        uint8_t of[kRowElemsMax * 8], nen[kRowElemsMax], round[kRowElemsMax];
        uint32_t slots_of[kRowElemsMax];
        int lane[kRowElemsMax];
        RowWave g{(int32_t)first, 0, (int32_t)r0, 0};
        RowLists l{0, 0, 0, 0};
        int p = 0, type = -1;   // the open group's next lane; its elements' type
        const auto close = [&](int64_t row) {
            if (row == g.first_row) return;
            g.n_rows = (int32_t)(row - g.first_row);
            g.n_tasks = p;
            P.wdesc.push_back(g);
            P.wlists.push_back(l);
            P.cls.push_back((uint8_t)std::max(type, 0));
            P.max_img = std::max<int64_t>(P.max_img, 9 * (int64_t)(rowptr[row] - rowptr[g.first_row]));
            P.max_items = std::max<int64_t>(P.max_items, (int64_t)l.n_elems * row_points(l.n_elems, lanes));
            P.max_nodes = std::max<int64_t>(P.max_nodes, l.n_nodes);
            ++gid;
            g = {g.first_task + p, 0, (int32_t)row, 0};
            l = {(int32_t)P.n_elems, 0, (int32_t)P.n_nodes, 0};
            p = 0;
            type = -1;
        };
        for (int64_t row = r0; row < r1; ++row) {
            const int32_t *c0 = colidx + rowptr[row];
            const int32_t len = std::min(rowptr[row + 1] - rowptr[row], 256);
            for (int32_t q = 0; q < len; ++q) at[c0[q]] = q;
            const uint32_t *t0 = inc + inc_ptr[row];
            const int nt = inc_ptr[row + 1] - inc_ptr[row];
            int D = 1;
            for (int t = 0; t < nt; ++t) {
                const int64_t e = t0[t] >> 3;
                const int32_t *ce = conn + e * stride;
                const int n = nen_of(e);
                nen[t] = (uint8_t)n;
                D = std::max(D, n);
                for (int b = 0; b < n; ++b) {
                    const int32_t j = ce[b], q = at[j];
                    if (q < 0 || q >= len || c0[q] != j) {
                        P.failed = true;
                        return;
                    }
                    of[8 * t + b] = (uint8_t)q;
                }
            }
            if (nt > 0) slots->row(D, nt, of, nen, slots_of, round);
            // Lanes of the row's tasks from lane q on: a round's tasks lie in one
            // wavefront, so that they add in step.
            const auto lanes_from = [&](int q) {
                for (int t = 0; t < nt;) {
                    int m = 1;
                    while (t + m < nt && round[t + m] == round[t]) ++m;
                    if (q % 64 + m > 64) q = (q + 63) / 64 * 64;
                    for (int i = 0; i < m; ++i) lane[t + i] = q++;
                    t += m;
                }
                return q;
            };
            int next = lanes_from(p);
            const int64_t img = 9 * (int64_t)(rowptr[row + 1] - rowptr[g.first_row]);
            if (row > g.first_row && (next > lanes || img > row_image(lanes) || row - g.first_row >= lanes)) {
                close(row);
                next = lanes_from(0);
            }
            if (g.first_task + next > last) {   // cannot happen
                P.failed = true;
                return;
            }
            for (int q = p, t = 0; q < next; ++q) {   // idle lanes between the rounds
                if (t < nt && lane[t] == q) {
                    ++t;
                    continue;
                }
                meta[g.first_task + q] = kRowNoTask;
                perm[g.first_task + q] = 0x88888888u;
                cols[g.first_task + q] = 0;
            }
            const uint32_t row_bits = (uint32_t)(row - g.first_row) << 11;
            for (int t = 0; t < nt; ++t) {
                const int64_t e = t0[t] >> 3;
                Placed &pe = elems[e];
                if (pe.group != gid) {
                    pe = {gid, (uint32_t)l.n_elems++};
                    if ((size_t)P.n_nodes + 8 > P.node.size()) P.node.resize(2 * P.node.size());
                    const int32_t *ce = conn + e * stride;
                    int32_t *const list = P.node.data() + P.n_nodes;
                    std::array<uint16_t, 8> &ln = P.ln[P.n_elems];
                    int n = 0;
                    for (int b = 0; b < nen[t]; ++b) {   // (whether a node is new is unpredictable: no branch)
                        Placed &pn = nodes[ce[b]];
                        const bool is_new = pn.group != gid;
                        list[n] = ce[b];
                        pn = {gid, is_new ? (uint32_t)(l.n_nodes + n) : pn.place};
                        ln[b] = (uint16_t)pn.place;
                        n += is_new;
                    }
                    for (int b = nen[t]; b < 8; ++b) ln[b] = 0;
                    P.elem[P.n_elems++] = (int32_t)e;
                    P.n_nodes += n;
                    l.n_nodes += n;
                    type = type < 0 ? nen[t] : type == nen[t] ? type : 0;
                }
                uint64_t c;
                if (slots_of[t] == 0x76543210u) {
                    memcpy(&c, of + 8 * t, 8);
                } else {
                    c = 0;
                    for (int q = 0; q < D; ++q) {
                        const uint32_t b = slots_of[t] >> (4 * q) & 15;
                        c |= (uint64_t)(b < 8 ? of[8 * t + b] : 0) << (8 * q);
                    }
                }
                const size_t d = (size_t)g.first_task + lane[t];
                meta[d] = pe.place | (t0[t] & 7) << 8 | row_bits | (uint32_t)round[t] << 19 |
                                (t == 0 ? kRowFirstTask : 0u);
                perm[d] = slots_of[t];
                cols[d] = c;
            }
            p = next;
        }
        close(r1);
    }
};

}  // namespace

int build_row_plan(int stride, const uint8_t *etype, int64_t N, int64_t E, const int32_t *conn,
                   const int32_t *rowptr, const int32_t *colidx, RowPlan &R, std::string &err,
                   const std::function<void()> &fetch, RowForm form)
{
    R = RowPlan();
    auto nen_of = [&](int64_t e) { return etype ? (int)etype[e] : stride; };
    int64_t T = E * stride;
    if (etype) {
        T = 0;
        for (int64_t e = 0; e < E; ++e) T += etype[e];
    }
    if (T > INT32_MAX) {
        err = "the block operator's plan holds at most 2^31 element nodes";
        return FE_EBADMESH;
    }
    R.lanes = T < kRowSmallMesh ? kRowTasksSmall : kRowTasks;
    R.nen = !etype ? stride : std::all_of(etype, etype + E, [&](uint8_t n) { return n == etype[0]; }) ? etype[0] : 0;
    // One team of threads for all stages (starting one takes up to 0.1 ms);
    // each plans a range of rows on its own.  First calls with 8192 / 12288
    // tasks to a thread at least, ms: HEX08 16^3 0.55 / 0.82, 24^3 0.95 / 1.06,
    // TET04 13^3 cubes 0.64 / 0.74, 24^3 2.5 / 2.8.
    constexpr int64_t kTasksPerThread = 8192, kScan = 64;
    const int nt = (int)std::max<int64_t>(1, std::min<int64_t>(host_threads(), T / kTasksPerThread));
    const int64_t scans = (E + kScan - 1) / kScan;
    UnsetVector<int32_t> inc_ptr(N + 1), lo(scans), hi(scans);
    UnsetVector<uint32_t> inc(T);
    std::vector<RowPart> part(nt);
    std::vector<int64_t> total(nt, 0);
    struct Offsets {
        int64_t group, elem, node;
    };
    std::vector<Offsets> off(nt + 1, Offsets{0, 0, 0});
    std::vector<int64_t> first(nt + 1, 0);   // each thread's tasks in the plan
    std::vector<std::pair<int64_t, int64_t>> sharing(nt, {0, 0});
    const bool small = T < kRowSmallMesh;
    if (form == kRowAuto && small && R.nen != 4 && R.nen != 6) form = R.nen == 8 ? kRowAlone : kRowShared;
    R.alone = form == kRowAlone;
    int status = FE_OK;   // set by thread 0 alone
    Team::run(nt, [&](int w, Team &team) {
        const auto begin = [&](int64_t n) { return n * w / nt; };
        const auto end = [&](int64_t n) { return n * (w + 1) / nt; };
        if (w == 0 && fetch) fetch();
        // the nodes of every kScan elements lie in [lo, hi]
        for (int64_t s = begin(scans); s < end(scans); ++s) {
            int32_t a = INT32_MAX, b = -1;
            for (int64_t e = s * kScan; e < std::min(E, (s + 1) * kScan); ++e)
                for (int q = 0; q < nen_of(e); ++q) {
                    a = std::min(a, conn[e * stride + q]);
                    b = std::max(b, conn[e * stride + q]);
                }
            lo[s] = a;
            hi[s] = b;
        }
        team.barrier();
        // node -> (element, local row), ascending: this thread's rows, counted, then filled
        const int64_t r0 = begin(N), r1 = end(N);
        const uint32_t rows = (uint32_t)(r1 - r0);
        const auto each = [&](auto f) {
            for (int64_t s = 0; s < scans; ++s) {
                if (hi[s] < r0 || lo[s] >= r1) continue;
                for (int64_t e = s * kScan; e < std::min(E, (s + 1) * kScan); ++e) {
                    const int n = nen_of(e);
                    for (int q = 0; q < n; ++q) {
                        const uint32_t i = (uint32_t)(conn[e * stride + q] - (int32_t)r0);
                        if (i < rows) f(i, (uint32_t)(8 * e + q));
                    }
                }
            }
        };
        std::vector<int32_t> fill(rows, 0);
        each([&](uint32_t i, uint32_t) { ++fill[i]; });
        for (uint32_t i = 0; i < rows; ++i) {
            if (fill[i] > kRowElemsMax && part[w].too_many < 0) part[w].too_many = r0 + i;
            total[w] += fill[i];
        }
        team.barrier();
        int64_t at = 0;
        bool ok = true;
        for (int v = 0; v < nt; ++v) {
            if (v < w) at += total[v];
            ok = ok && part[v].too_many < 0;
        }
        if (!ok) return;   // (every thread alike)
        if (w == 0) inc_ptr[0] = 0;
        for (uint32_t i = 0; i < rows; ++i) {
            const int32_t n = fill[i];
            fill[i] = (int32_t)at;
            inc_ptr[r0 + i + 1] = (int32_t)(at += n);
        }
        each([&](uint32_t i, uint32_t x) { inc[fill[i]++] = x; });
        team.barrier();
        RowPart &P = part[w];
        if (form == kRowAuto) {
            sharing[w] = row_sharing(inc_ptr.data(), inc.data(), r0, r1);
            team.barrier();
            if (w == 0) {
                int64_t seen = 0, distinct = 0;
                for (const auto &q : sharing) {
                    seen += q.first;
                    distinct += q.second;
                }
                R.alone = (double)distinct > kRowPoor * (double)seen;
            }
            team.barrier();
        }
        if (R.alone) {
            if (w == 0) {
                R.lanes = kRowTasksSmall;
                R.n_tasks = T;
                R.tasks.resize(RowPlan::alone_bytes(T));
            }
            team.barrier();
            RowTasks{stride, etype, conn, rowptr, colidx, inc_ptr.data(), inc.data(), const_cast<uint8_t *>(R.alone_cols()),
                     const_cast<int32_t *>(R.alone_elem()), const_cast<uint16_t *>(R.alone_meta())}
                .run(N, r0, r1, P);
            return;
        }
        RowGrouping G{stride, R.lanes, etype, conn, rowptr, colidx, inc_ptr.data(), inc.data(), nullptr, nullptr, nullptr};
        if (w == 0) {
            for (int v = 0; v < nt; ++v) first[v + 1] = first[v] + G.most_lanes(N * v / nt, N * (v + 1) / nt);
            R.n_tasks = first[nt];
            if (R.n_tasks <= INT32_MAX) R.tasks.resize(RowPlan::task_bytes(R.n_tasks));
            else status = FE_EBADMESH;
        }
        team.barrier();
        if (status != FE_OK) return;
        G.meta = const_cast<uint32_t *>(R.task_meta());
        G.perm = const_cast<uint32_t *>(R.task_perm());
        G.cols = (uint64_t *)const_cast<uint8_t *>(R.task_cols());
        G.run(N, E, r0, r1, first[w], P);
        team.barrier();
        if (w == 0) {
            for (int v = 0; v < nt; ++v) {
                const RowPart &Q = part[v];
                if (Q.failed) status = FE_EBADMESH;
                off[v + 1] = {off[v].group + (int64_t)Q.wdesc.size(), off[v].elem + Q.n_elems,
                              off[v].node + Q.n_nodes};
                R.max_img = std::max(R.max_img, Q.max_img);
                R.max_items = std::max(R.max_items, Q.max_items);
                R.max_nodes = std::max(R.max_nodes, Q.max_nodes);
            }
            R.n_elems = off[nt].elem;
            R.n_nodes = off[nt].node;
            R.lists.resize(RowPlan::list_bytes(R.n_elems, R.n_nodes));
            R.wdesc.resize(off[nt].group);
            R.wlists.resize(off[nt].group);
        }
        team.barrier();
        if (status != FE_OK) return;
        const Offsets &o = off[w];
        std::copy_n(P.elem.begin(), P.n_elems, const_cast<int32_t *>(R.wave_elem()) + o.elem);
        std::copy_n(P.node.begin(), P.n_nodes, const_cast<int32_t *>(R.wave_node()) + o.node);
        if (P.n_elems) memcpy(const_cast<uint16_t *>(R.wave_ln()) + 8 * o.elem, P.ln.data(), P.n_elems * sizeof P.ln[0]);
        for (size_t g = 0; g < P.wdesc.size(); ++g) {
            P.wlists[g].first_elem += (int32_t)o.elem;
            P.wlists[g].first_node += (int32_t)o.node;
            R.wdesc[o.group + g] = P.wdesc[g];
            R.wlists[o.group + g] = P.wlists[g];
        }
    });
    for (const RowPart &Q : part)
        if (Q.too_many >= 0) {
            int64_t n = 0;
            for (int64_t e = 0; e < E; ++e)
                for (int q = 0; q < nen_of(e); ++q) n += conn[e * stride + q] == Q.too_many;
            err = "node " + std::to_string(Q.too_many) + " (mesh numbering) lies in " + std::to_string(n) +
                  " elements; the block operator's row-owner assembly takes at most " + std::to_string(kRowElemsMax);
            return FE_EBADMESH;
        }
    if (R.alone)
        for (const RowPart &Q : part) {
            if (Q.failed) status = FE_EBADMESH;
            R.max_img = std::max(R.max_img, Q.max_img);
            R.wdesc.insert(R.wdesc.end(), Q.wdesc.begin(), Q.wdesc.end());
        }
    if (status != FE_OK) {
        err = "the CSR pattern lacks an element's node pair";
        return status;
    }
    if (R.nen == 0 && !R.alone) {   // of several types: each type's groups together
        std::vector<uint8_t> cls;
        for (const RowPart &Q : part) cls.insert(cls.end(), Q.cls.begin(), Q.cls.end());
        const std::vector<RowWave> wdesc = std::move(R.wdesc);
        const std::vector<RowLists> wlists = std::move(R.wlists);
        R.wdesc.clear();
        R.wlists.clear();
        const int order[5] = {0, 8, 5, 6, 4};
        for (int c = 0; c < 5; ++c) {
            for (size_t g = 0; g < wdesc.size(); ++g)
                if (cls[g] == order[c]) {
                    R.wdesc.push_back(wdesc[g]);
                    R.wlists.push_back(wlists[g]);
                }
            if (c < 4) R.class_end[c] = (int32_t)R.wdesc.size();
        }
    }
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
