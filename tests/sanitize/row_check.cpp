// row_check.cpp -- what the kernels take for granted of the row plan of the
// 3x3-block operator (csrc/rowplan.cpp, build_row_plan) and of the owner plan
// as the HEX08 kernel runs it (arrange_waves).  Test infrastructure: built and
// run by tests/test_row_plan_cpu.py.
#include <algorithm>
#include <cstdio>
#include <map>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "../../paper_2107_11541_amd/csrc/plan.h"
#include "meshes.h"

using namespace feasm;

static int fails = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            if (++fails < 20) fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
        }                                                           \
    } while (0)

// Per (element, local row): the round and the order of its nodes.
using Order = std::map<std::pair<int64_t, int>, std::pair<int, uint32_t>>;

static Order check_rows(const Plan &P, const RowPlan &R)
{
    const uint8_t *et = P.etype.empty() ? nullptr : P.etype.data();
    auto nen_of = [&](int64_t e) { return et ? (int)et[e] : P.nen; };
    Order order;
    std::vector<char> row_seen((size_t)P.N, 0);
    CHECK(R.lanes == kRowTasks || R.lanes == kRowTasksSmall);
    int64_t max_img = 0, max_items = 0, max_nodes = 0;
    std::set<int64_t> used;   // task entries
    for (size_t w = 0; w < R.wdesc.size(); ++w) {
        const RowWave &g = R.wdesc[w];
        const RowLists &l = R.wlists[w];
        CHECK(g.n_rows >= 1 && g.n_tasks >= 1 && g.n_tasks <= R.lanes && g.n_rows <= R.lanes);
        CHECK(g.first_task >= 0 && g.first_task + g.n_tasks <= R.n_tasks);
        CHECK(l.n_elems >= 1 && l.n_elems <= 256 && l.first_elem >= 0 && l.first_elem + l.n_elems <= R.n_elems);
        CHECK(l.first_node >= 0 && l.first_node + l.n_nodes <= R.n_nodes);
        const int64_t img = 9 * (int64_t)(P.rowptr[g.first_row + g.n_rows] - P.rowptr[g.first_row]);
        CHECK(img <= row_image(R.lanes));
        max_img = std::max(max_img, img);
        max_items = std::max<int64_t>(max_items, (int64_t)l.n_elems * row_points(l.n_elems, R.lanes));
        max_nodes = std::max<int64_t>(max_nodes, l.n_nodes);
        std::set<int32_t> elems, nodes;
        for (int k = 0; k < l.n_elems; ++k) {
            const int32_t e = R.wave_elem()[l.first_elem + k];
            CHECK(elems.insert(e).second);
            for (int b = 0; b < nen_of(e); ++b) {
                const int n = R.wave_ln()[8 * (size_t)(l.first_elem + k) + b];
                CHECK(n < l.n_nodes && R.wave_node()[l.first_node + n] == P.conn[(size_t)e * P.nen + b]);
            }
        }
        for (int k = 0; k < l.n_nodes; ++k) CHECK(nodes.insert(R.wave_node()[l.first_node + k]).second);
        for (int i = 0; i < g.n_rows; ++i) {
            CHECK(!row_seen[(size_t)(g.first_row + i)]);
            row_seen[(size_t)(g.first_row + i)] = 1;
        }
        std::set<std::tuple<int, int, int, int>> met;   // row, round, slot, column
        std::map<std::pair<int, int>, int> wave_of;     // row, round
        std::vector<int> first(g.n_rows, -1), last(g.n_rows, -1);
        for (int lane = 0; lane < g.n_tasks; ++lane) {
            const size_t d = (size_t)g.first_task + lane;
            CHECK(used.insert((int64_t)d).second);
            const uint32_t meta = R.task_meta()[d], perm = R.task_perm()[d];
            if (meta == kRowNoTask) continue;
            const int le = meta & 255, a = meta >> 8 & 7, rl = meta >> 11 & 255, round = meta >> 19 & 0xfff;
            CHECK(le < l.n_elems && rl < g.n_rows);
            if (le >= l.n_elems || rl >= g.n_rows) continue;
            const int32_t e = R.wave_elem()[l.first_elem + le];
            const int32_t row = g.first_row + rl;
            CHECK(a < nen_of(e) && P.conn[(size_t)e * P.nen + a] == row);
            CHECK(order.insert({{e, a}, {round, perm}}).second);
            CHECK(((meta & kRowFirstTask) != 0) == (first[rl] < 0));
            if (first[rl] < 0) first[rl] = lane;
            CHECK(last[rl] < 0 || wave_of.empty() || last[rl] < lane);
            last[rl] = lane;
            const auto at = wave_of.insert({{rl, round}, lane / 64}).first;
            CHECK(at->second == lane / 64);
            unsigned nodes_seen = 0;
            for (int s = 0; s < 8; ++s) {
                const int b = perm >> (4 * s) & 15;
                if (b >= 8) continue;
                CHECK(b < nen_of(e) && !(nodes_seen >> b & 1));
                nodes_seen |= 1u << b;
                const int col = R.task_cols()[8 * d + s];
                CHECK(P.rowptr[row] + col < P.rowptr[row + 1] &&
                      P.colidx[P.rowptr[row] + col] == P.conn[(size_t)e * P.nen + b]);
                // a task may hold a column twice (a repeated node), in different slots
                CHECK(met.insert(std::make_tuple(rl, round, s, col)).second);
            }
            CHECK(nodes_seen == (1u << nen_of(e)) - 1);
        }
        for (int i = 0; i < g.n_rows; ++i) {   // between a row's first and last lane: its tasks or idle lanes
            CHECK(first[i] >= 0);
            for (int lane = first[i]; lane >= 0 && lane <= last[i]; ++lane) {
                const uint32_t meta = R.task_meta()[(size_t)g.first_task + lane];
                CHECK(meta == kRowNoTask || (int)(meta >> 11 & 255) == i);
            }
        }
    }
    CHECK(max_img <= R.max_img && max_items <= R.max_items && max_nodes <= R.max_nodes);
    CHECK(std::count(row_seen.begin(), row_seen.end(), 1) == (int64_t)P.N);
    int64_t tasks = 0;
    for (int64_t e = 0; e < P.E; ++e) tasks += nen_of(e);
    CHECK((int64_t)order.size() == tasks);
    if (R.nen == 0) {   // the groups' types, class after class
        const int type[5] = {0, 8, 5, 6, 4};
        size_t w = 0;
        for (int c = 0; c < 5; ++c)
            for (; w < (c < 4 ? (size_t)R.class_end[c] : R.wdesc.size()); ++w) {
                std::set<int> types;
                for (int k = 0; k < R.wlists[w].n_elems; ++k)
                    types.insert(nen_of(R.wave_elem()[R.wlists[w].first_elem + k]));
                CHECK(c == 0 ? types.size() > 1 : types.size() == 1 && *types.begin() == type[c]);
            }
    }
    return order;
}

// The plan of each task alone: every (element, local row) once, by row and
// element, whole rows to wavefronts of at most 64.
static void check_alone(const Plan &P, const RowPlan &R)
{
    const uint8_t *et = P.etype.empty() ? nullptr : P.etype.data();
    auto nen_of = [&](int64_t e) { return et ? (int)et[e] : P.nen; };
    int64_t tasks = 0, next_row = 0, next_task = 0, max_img = 0;
    for (int64_t e = 0; e < P.E; ++e) tasks += nen_of(e);
    CHECK(R.alone && R.n_tasks == tasks);
    std::set<std::pair<int64_t, int>> seen;
    for (const RowWave &w : R.wdesc) {
        CHECK(w.first_row == next_row && w.first_task == next_task && w.n_rows >= 1 && w.n_rows <= 64);
        CHECK(w.n_tasks >= 1 && w.n_tasks <= 64);
        const int64_t img = 9 * (int64_t)(P.rowptr[w.first_row + w.n_rows] - P.rowptr[w.first_row]);
        CHECK(img <= row_image(kRowTasksSmall));
        max_img = std::max(max_img, img);
        int32_t row = -1, last = -1;
        int place = 0;
        for (int64_t t = w.first_task; t < w.first_task + w.n_tasks; ++t) {
            const int32_t e = R.alone_elem()[t];
            const int a = R.alone_meta()[t] & 15;
            CHECK(a < nen_of(e) && seen.insert({e, a}).second);
            const int32_t i = P.conn[(size_t)e * P.nen + a];
            CHECK(i >= w.first_row && i < w.first_row + w.n_rows && i >= row);
            place = i == row ? place + 1 : 0;
            CHECK(R.alone_meta()[t] >> 4 == place && (i != row || e >= last));
            row = i;
            last = e;
            for (int b = 0; b < nen_of(e); ++b) {
                const int col = R.alone_cols()[8 * (size_t)t + b];
                CHECK(P.rowptr[i] + col < P.rowptr[i + 1] &&
                      P.colidx[P.rowptr[i] + col] == P.conn[(size_t)e * P.nen + b]);
            }
        }
        next_row += w.n_rows;
        next_task += w.n_tasks;
    }
    CHECK(next_row == P.N && next_task == tasks && max_img <= R.max_img && (int64_t)seen.size() == tasks);
}

// The HEX08 owner plan dealt to wavefronts: the same tasks, and in one step of
// a wavefront each owned row at most once per local place.
static void check_waves(const Plan &P)
{
    OwnerPlan A, B;
    std::string err;
    CHECK(build_owner_plan(P, A, err) == 0);
    B = A;
    arrange_waves(B);
    CHECK(A.groups.size() == B.groups.size() && A.nodes == B.nodes && A.node_ptr == B.node_ptr);
    for (size_t g = 0; g < A.groups.size(); ++g) {
        const OwnGroup &q = A.groups[g];
        auto task = [&](const OwnerPlan &O, int t) {
            std::vector<int> v{O.tk_elem[t]};
            for (int b = 0; b < O.ln_stride; ++b) v.push_back(O.tk_ln[(size_t)t * O.ln_stride + b]);
            for (int b = 0; b < O.off_stride; ++b) v.push_back(O.tk_off[(size_t)t * O.off_stride + b]);
            return v;
        };
        std::multiset<std::vector<int>> a, b;
        std::set<std::tuple<int, int, int, int>> met;   // wavefront, step, local place, owned row
        for (int t = q.first_task; t < q.first_task + q.n_tasks; ++t) {
            a.insert(task(A, t));
            b.insert(task(B, t));
            CHECK(B.tk_phase[t] < B.nphase[g]);
            for (int r = 0; r < B.ra; ++r) {
                const int row = B.tk_ln[(size_t)t * B.ln_stride + r];
                if (row < q.n_rows)
                    CHECK(met.insert(std::make_tuple((t - q.first_task) / 64, (int)B.tk_phase[t], r, row)).second);
            }
        }
        CHECK(a == b);
    }
}

// collapse: some elements repeat a node (as a hexahedron collapsed to a wedge does)
static void check(int kind, int n, bool renumber, bool collapse)
{
    SanMesh m = san_cube(n, kind);
    if (collapse)
        for (int64_t e = 0; e < m.n_elems; e += 3) {
            int32_t *c = m.conn + e * m.stride;
            c[1] = c[0];
            if (e % 2 == 0 && m.stride == 8 && !m.types) c[5] = c[4];
        }
    Plan P;
    std::string err;
    const int st = build_plan(m.stride, m.types, m.n_nodes, m.coords, m.n_elems, m.conn, renumber, P, err);
    if (st != 0) {   // (a collapse may leave a node without an element)
        CHECK(collapse);
        san_free(&m);
        return;
    }
    Order first;
    for (int threads : {1, 5}) {
        RowPlan R;
        set_thread_budget(threads);
        CHECK(build_row_plan(P.nen, P.etype.empty() ? nullptr : P.etype.data(), P.N, P.E, P.conn.data(),
                             P.rowptr.data(), P.colidx.data(), R, err) == 0);
        set_thread_budget(0);
        const Order o = check_rows(P, R);
        RowPlan S, A;
        set_thread_budget(threads);
        for (RowPlan *Q : {&S, &A})
            CHECK(build_row_plan(P.nen, P.etype.empty() ? nullptr : P.etype.data(), P.N, P.E, P.conn.data(),
                                 P.rowptr.data(), P.colidx.data(), *Q, err, nullptr, Q == &S ? kRowAlone : kRowAuto) == 0);
        set_thread_budget(0);
        check_alone(P, S);
        // the form for the mesh: small ones by type, the others by their order
        int64_t tasks = 0;
        for (int64_t e = 0; e < P.E; ++e) tasks += P.etype.empty() ? P.nen : P.etype[e];
        if (tasks >= kRowSmallMesh) CHECK(A.alone == !renumber);
        else if (!P.etype.empty() || P.nen == 8 || P.nen == 5) CHECK(A.alone == (P.etype.empty() && P.nen == 8));
        else CHECK(!A.alone || !renumber);
        // the order of every sum is the same for any number of threads
        if (threads == 1) first = o;
        CHECK(o == first);
    }
    if (P.etype.empty() && P.nen == 8) check_waves(P);
    san_free(&m);
}

int main()
{
    for (int kind = 0; kind < 3; ++kind)
        for (bool renumber : {false, true})
            for (bool collapse : {false, true})
                for (int n : {1, 2, 3, 6}) check(kind, n, renumber, collapse);
    // several threads; groups of 256 lanes (from 2^16 element nodes on), and of 64
    check(0, 21, true, true);
    check(0, 14, false, false);
    check(1, 15, true, false);
    check(2, 16, false, false);
    // a node in more than kRowElemsMax elements is refused, with its number of elements
    {
        const int k = kRowElemsMax + 1;
        std::vector<double> x(3 * (3 * k + 1));
        std::vector<int32_t> c;
        for (size_t i = 0; i < x.size(); ++i) x[i] = 1e-3 * (double)((i * 7919) % 1009);
        for (int e = 0; e < k; ++e)
            for (int v : {0, 3 * e + 1, 3 * e + 2, 3 * e + 3}) c.push_back(v);
        Plan P;
        RowPlan R;
        std::string err;
        CHECK(build_plan(4, nullptr, 3 * k + 1, x.data(), k, c.data(), false, P, err) == 0);
        CHECK(build_row_plan(4, nullptr, P.N, P.E, P.conn.data(), P.rowptr.data(), P.colidx.data(), R, err) != 0);
        CHECK(err.find("lies in 65 elements") != std::string::npos);
        // ... and a pattern without an element's pair
        std::vector<int32_t> ci = P.colidx;
        ci[1] = ci[0];
        CHECK(build_row_plan(4, nullptr, P.N, P.E - 1, P.conn.data(), P.rowptr.data(), ci.data(), R, err) != 0);
    }
    printf("%d failed checks\n", fails);
    return fails != 0;
}
