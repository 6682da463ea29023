// resident.hip -- a whole Jacobi-PCG solve in one launch, the matrix held in
// registers.
//
// The solver of Section 5.2 is bound by memory and, on meshes of up to a few
// hundred thousand nodes, by launches: three dependent kernels per iteration
// that each read the matrix or the vectors again.  A CU has 512 KB of vector
// registers and 160 KB of LDS; 256 of them hold the rows of such a matrix for
// the length of a solve.  Work-group g keeps a contiguous range of rows: each
// thread up to S rows of up to W entries (values and 16-bit window places in
// registers), r in registers, x and D^-1 in LDS, and in LDS the window of p
// that its rows touch (the columns of other groups, the halo, then its own).
//
// Per iteration the groups meet twice, each time in a reduction whose partial
// sums are also the barrier: a group publishes its partial, then reads every
// group's, so all hold bitwise the same alpha, beta and stop decision.  The
// second meeting carries z = D^-1 r with it: z is stored before the partial
// of r.z is published, and each group then forms p = z + beta p itself on its
// own rows and on its halo, so p never travels.  Results do not depend on
// timing: entries, lanes, waves and groups are summed in fixed orders.
//
// Measured per iteration on one MI355X against three recorded launches (FP64,
// HEX08 / TET04 Poisson matrices): 10^3 4.0 us (12.3), 32^3 5.9 (13.5), 48^3
// 7.8 (19.9), 64^3 10.2 (30.9), 71^3 12.1 (36.5); 6 x 80^3 TET04 11.7 (35.7).
// At 64^3 the products take 2.0 us (LDS gathers), the two meetings 2.9 and
// 4.2 (the second waits for the stores of z) and the halo 0.9.  Reading the
// matrix once into the registers takes 9 us (10^3) to 50 us (71^3) per solve.
//
// Every wait is bounded.  A group that waits longer than the limit (other
// work holds the CUs that the remaining groups need) marks the solve as
// abandoned and leaves; the others see the mark while they wait, or when they
// start (those that had no CU until then, which would else wait out the limit
// one CU's load after the other).  The caller then runs the solve in the
// general form.
#include "internal.h"

namespace feasm {
namespace {

constexpr int kRB = kResidentThreads;          // threads of a group, one group per CU
constexpr int kWaves = kRB / 64;
constexpr int kHaloCap = kResidentHalo;        // halo columns of a group
constexpr int kHash = 2 * kHaloCap;            // slots of the planning kernel's table
template <int W> constexpr int kBatch = W == 27 ? 7 : 8;   // window reads of one row in flight together
// (4, 7, 9 and 14 of 27, and 4, 6 and 8 of 16, are within 0.3 us per iteration of
// each other at 10^3 to 80^3; 16 of 16 spills, TET04 80^3 cubes 12.6 -> 14.3 us)
constexpr unsigned long long kEmpty = 0xfff8dead00000001ull;   // no arithmetic result (bits() below)
constexpr unsigned long long kNaN = 0x7ff8000000000000ull;
constexpr int kMaxProbe = 64, kLine = 8;
// A column's place in the planning table: a bucket per run of kLine columns,
// the column's place in the run within it.
__device__ inline unsigned home(int c)
{
    return (((unsigned)c / kLine * 2654435761u) / (0x100000000ull / (kHash / kLine))) * kLine + (unsigned)c % kLine;
}
constexpr size_t kMeetBuffer = (size_t)kResidentCopies * 2 * kResidentMaxGroups;

__device__ inline unsigned long long bits(double v)
{
    // an arithmetic NaN never carries the mark
    return v != v ? kNaN : (unsigned long long)__double_as_longlong(v);
}

template <class U> __device__ inline U agent_load(const U *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class U> __device__ inline void agent_store(U *p, U v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the wave's 64 lanes, in lane 63: shifts within rows of 16, then
// row broadcasts (data-parallel moves: a fixed order, no LDS round trips).
template <int CTRL, int ROWS> __device__ inline double dpp_add(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ inline double wave_sum63(double v)
{
    v = dpp_add<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add<0x112, 0xf>(v);   // row_shr:2
    v = dpp_add<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
}

// The groups' meeting point.  slots[buffer][copy][value][group]: a group
// publishes its partials in every copy and reads one (all groups polling the
// same lines queue at their memory channel), in three buffers in turn: a group clears its entry of meeting m - 1 when it has completed
// meeting m (every group has then read it), and completes that store before
// it publishes at meeting m + 1, two meetings before the buffer's next use.
struct Meet {
    unsigned long long *slots;
    ResidentOut *out;
    uint32_t *stop;              // nonzero: the solve is abandoned
    unsigned long long limit;    // 100 MHz ticks
    int G, g, phase;
    double (*sa)[kWaves];        // LDS: wave partials of the group, of the collected values
    double (*sb)[kWaves];
    int *failed;                 // LDS
};

// v[q] summed over all threads of all groups, in a fixed order; false: the
// solve is abandoned.  Agent-scope stores made before the call are visible
// to every group's agent-scope loads after it.
template <int NV>
__device__ inline bool meet_sum(Meet &M, double (&v)[NV])
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const double s = wave_sum63(v[q]);
        if (lane == 63) M.sa[q][w] = s;
    }
    // this wave's stores have reached the coherent level
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    double own[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double s = M.sa[q][0];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) s += M.sa[q][k];
        own[q] = s;
    }
    if (M.G == 1) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = own[q];
        return true;
    }
    unsigned long long *buf = M.slots + (size_t)(M.phase % 3) * kMeetBuffer;
    if (tid < kResidentCopies) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
            agent_store(buf + (tid * 2 + q) * kResidentMaxGroups + M.g, bits(own[q]));
    }
    buf += (size_t)(M.g % kResidentCopies) * 2 * kResidentMaxGroups;
    double got[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) got[q] = 0.0;
    if (tid < M.G) {
        unsigned long long u[NV];
        const unsigned long long t0 = wall_clock64();
        for (unsigned polls = 1;; ++polls) {
            bool all = true;
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                u[q] = agent_load(buf + q * kResidentMaxGroups + tid);
                all = all && u[q] != kEmpty;
            }
            if (!all && (wall_clock64() - t0 > M.limit || (polls % 32 == 0 && agent_load(M.stop) != 0))) {
                *M.failed = 1;
                break;
            }
            if (all) break;
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) got[q] = __longlong_as_double((long long)u[q]);
    }
    if (w < kResidentMaxGroups / 64) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double s = wave_sum63(got[q]);
            if (lane == 63) M.sb[q][w] = s;
        }
    }
    __syncthreads();
    if (*M.failed) {
        if (tid == 0) {
            agent_store(M.stop, 1u);
            agent_store(&M.out->abandoned, 1);
        }
        return false;
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double s = M.sb[q][0];
#pragma unroll
        for (int k = 1; k < kResidentMaxGroups / 64; ++k) s += M.sb[q][k];
        v[q] = s;
    }
    if (tid < 2 * kResidentCopies && M.phase > 0)
        agent_store(M.slots + (size_t)((M.phase + 2) % 3) * kMeetBuffer + tid * kResidentMaxGroups + M.g, kEmpty);
    ++M.phase;
    return true;
}

// Plans the groups of a pattern: per group its halo (every column outside its
// rows, once) and per entry the column's place in the group's window (the halo
// first, the own rows from kHaloCap on), two 16-bit places per word, the
// words of a row in off[group][row / kRB][word][row % kRB].  Padding up to W
// entries points at the row itself.
__global__ void __launch_bounds__(kRB) k_resident_plan(ResidentPlan P, int N, int R, int W,
                                                       const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ colidx, int32_t *bad)
{
    __shared__ int32_t key[kHash];
    __shared__ uint16_t slot[kHash];
    __shared__ int failed, nhalo, taken;
    const int tid = threadIdx.x, g = blockIdx.x;
    const int r0 = g * R, nr = min(R, N - r0), Sp = (R + kRB - 1) / kRB, W2 = (W + 1) / 2;
    for (int q = tid; q < kHash; q += kRB) key[q] = -1;
    if (tid == 0) {
        failed = 0;
        nhalo = 0;
        taken = 0;
    }
    __syncthreads();
    // a pattern in random order is given up as soon as the halo does not fit
    // (filling the table to the end took 0.5 ms of a 48^3 HEX08 mesh's first solve)
    for (int i = tid; i < nr; i += kRB) {
        if (__hip_atomic_load(&failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
        int added = 0;
        for (int p = rowptr[r0 + i]; p < rowptr[r0 + i + 1]; ++p) {
            const int c = colidx[p];
            if ((unsigned)(c - r0) < (unsigned)nr) continue;
            unsigned h = home(c);
            int probe = 0;
            for (; probe < kMaxProbe; ++probe, h = (h + kLine) & (kHash - 1)) {
                const int was = atomicCAS(&key[h], -1, c);
                added += was == -1;
                if (was == -1 || was == c) break;
            }
            if (probe == kMaxProbe) failed = 1;
        }
        if (added && atomicAdd(&taken, added) + added > kHaloCap) failed = 1;
    }
    __syncthreads();
    // halo slots in table order within each thread's part of the table, so
    // that columns of one cache line are gathered by neighbouring lanes
    constexpr int kPart = kHash / kRB;
    int n = 0;
    for (int q = 0; q < kPart; ++q) n += key[tid * kPart + q] != -1;
    int k = n ? atomicAdd(&nhalo, n) : 0;
    for (int q = 0; q < kPart; ++q)
        if (key[tid * kPart + q] != -1) {
            if (k < kHaloCap) {
                slot[tid * kPart + q] = (uint16_t)k;
                P.hcol[(size_t)g * kHaloCap + k] = key[tid * kPart + q];
            }
            ++k;
        }
    __syncthreads();
    if (failed || nhalo > kHaloCap) {   // uniform over the group
        if (tid == 0) *bad = 1;
        return;
    }
    if (tid == 0) P.nh[g] = nhalo;
    for (int s = 0; s < Sp; ++s) {
        const int i = tid + s * kRB;
        const int p0 = i < nr ? rowptr[r0 + i] : 0, len = i < nr ? rowptr[r0 + i + 1] - p0 : 0;
        for (int w2 = 0; w2 < W2; ++w2) {
            uint32_t word = 0;
            for (int b = 0; b < 2; ++b) {
                uint32_t o = (uint32_t)(kHaloCap + i);
                if (2 * w2 + b < len) {
                    const int c = colidx[p0 + 2 * w2 + b];
                    o = (uint32_t)(kHaloCap + c - r0);
                    if ((unsigned)(c - r0) >= (unsigned)nr) {
                        unsigned h = home(c);
                        while (key[h] != c) h = (h + kLine) & (kHash - 1);   // it was inserted above
                        o = slot[h];
                    }
                }
                word |= o << (16 * b);
            }
            P.off[(((size_t)g * Sp + s) * W2 + w2) * kRB + tid] = word;
        }
    }
}

// S rows per thread, the last L of them (0 or 1) with their values and
// places in LDS: the registers hold five rows of 27 FP64 entries per thread,
// LDS a sixth.
template <class T, int W, int S, int L>
__global__ void __launch_bounds__(kRB, 1) k_resident(ResidentArgs A)
{
    constexpr int kOwn = S * kRB, W2 = (W + 1) / 2, SR = S - L;
    static_assert((kOwn + kHaloCap) * sizeof(T) <= 65536, "window places are 16-bit byte offsets");
    __shared__ T win[kHaloCap + kOwn];       // p: the halo, then the own rows
    __shared__ int32_t hcol[kHaloCap];       // the halo's columns
    __shared__ T x[kOwn], dinv[kOwn];        // (each entry its thread's alone)
    __shared__ T lv[L ? W : 1][kRB];
    __shared__ uint32_t lo[L ? W2 : 1][kRB];
    __shared__ double sa[2][kWaves], sb[2][kWaves];
    __shared__ int failed;

    const int tid = threadIdx.x, g = blockIdx.x;
    const uint32_t stopped = agent_load(A.stop);
    if (A.bad && agent_load(A.bad) != 0) return;   // the caller takes the general form (every group alike)
    if (stopped) {                                 // abandoned before this group had a CU
        if (tid == 0) agent_store(&A.out->abandoned, 1);
        return;
    }
    const int r0 = g * A.R, nr = min(A.R, A.N - r0), Sp = (A.R + kRB - 1) / kRB;
    if (tid == 0) failed = 0;
    Meet M{A.slots, A.out, A.stop, A.limit, (int)gridDim.x, g, 0, sa, sb, &failed};

    // 1. the rows: values and window offsets (bytes) of each thread's rows
    const int nh = A.plan.nh[g];
    T *const own = win + kHaloCap;
    T v[SR][W];
    uint32_t off[SR][W2];
    T r[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int i = tid + s * kRB;
        const bool live = i < nr;
        const int p0 = live ? A.rowptr[r0 + i] : 0, len = live ? A.rowptr[r0 + i + 1] - p0 : 0;
        // rows past the plan's (s >= Sp) have no entries: any places will do
        const uint32_t *__restrict__ po = A.plan.off + ((size_t)g * Sp + (s < Sp ? s : 0)) * W2 * kRB + tid;
#pragma unroll
        for (int w2 = 0; w2 < W2; ++w2) {
            const uint32_t o = po[w2 * kRB] * (uint32_t)sizeof(T);   // both halves stay below 65536
            if (s < SR) off[s < SR ? s : 0][w2] = o;
            else lo[w2][tid] = o;
        }
        double raw[W];
#pragma unroll
        for (int w = 0; w < W; ++w) raw[w] = A.vals[p0 + (w < len ? w : 0)];
        __builtin_amdgcn_sched_barrier(0);   // the row's loads in flight together
#pragma unroll
        for (int w = 0; w < W; ++w) {
            T a = w < len ? T(raw[w]) : T(0);
            asm volatile("" : "+v"(a));   // masked here, not after the last row
            if (s < SR) v[s < SR ? s : 0][w] = a;
            else lv[w][tid] = a;
        }
        const double dg = live ? A.vals[A.diagpos[r0 + i]] : 1.0;
        const T x0 = live && !A.x_zero ? ((const T *)A.x)[r0 + i] : T(0);
        dinv[i] = live ? T(1) / T(dg) : T(0);
        x[i] = x0;
        own[i] = x0;
        if (live && !A.x_zero) ((T *)A.x0)[r0 + i] = x0;   // for a caller that has to start again
        __builtin_amdgcn_sched_barrier(0);                 // one row's temporaries at a time
    }
    for (int h = tid; h < nh; h += kRB) {
        const int c = A.plan.hcol[(size_t)g * kHaloCap + h];
        hcol[h] = c;
        win[h] = A.x_zero ? T(0) : ((const T *)A.x)[c];
    }
    __syncthreads();

    // row sums of A times the window: even and odd entries, then their sum.
    // The window is read in batches of F entries, one batch ahead of the
    // products (LDS is the bound: ~9 cycles per 64-lane gather).  Waves without
    // a last row leave it out.
    constexpr int F = kBatch<W>, NB = (W + F - 1) / F;
    auto place = [&](int s, int w) -> uint32_t {
        const uint32_t pk = s < SR ? off[s < SR ? s : 0][w / 2] : lo[w / 2][tid];
        uint32_t o;
        // (written out, or the compiler keeps the unpacked offsets of every
        // iteration in registers and moves a row's gathers to its top)
        if (w & 1) asm volatile("v_lshrrev_b32 %0, 16, %1" : "=v"(o) : "v"(pk));
        else asm volatile("v_and_b32 %0, 0xffff, %1" : "=v"(o) : "v"(pk));
        return o;
    };
    auto issue = [&](int s, int b, T (&t)[F]) {
#pragma unroll
        for (int k = 0; k < F; ++k)
            if (b * F + k < W) t[k] = *(const T *)((const char *)win + place(s, b * F + k));
    };
    auto consume = [&](int s, int b, const T (&t)[F], T &y0, T &y1) {
#pragma unroll
        for (int k = 0; k < F; ++k) {
            const int w = b * F + k;
            if (w >= W) continue;
            T a;
            if (s < SR) a = v[s < SR ? s : 0][w];
            else a = lv[w][tid];
            if (w & 1) y1 += a * t[k];
            else y0 += a * t[k];
        }
        // the products belong here, not after the last gather
        asm volatile("" : "+v"(y0), "+v"(y1));
    };
    const bool last = (S - 1) * kRB + (tid & ~63) < nr;
    auto multiply = [&](T (&y)[S]) {
        T t[2][F];
        if (S > 1 || last) issue(0, 0, t[0]);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            y[s] = T(0);
            if (s == S - 1 && !last) continue;
            T y0 = T(0), y1 = T(0);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int e = s * NB + b;
                if (b + 1 < NB) issue(s, b + 1, t[(e + 1) & 1]);
                else if (s + 1 < S) {
                    if (s + 1 < S - 1 || last) issue(s + 1, 0, t[(e + 1) & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                consume(s, b, t[e & 1], y0, y1);
                __builtin_amdgcn_sched_barrier(0);
            }
            y[s] = y0 + y1;
        }
    };
    // put(h, value): z of the halo, from every group's store before the last meeting
    auto halo = [&](auto put) {
        for (int h0 = 0; h0 < nh; h0 += 4 * kRB) {
            T t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int h = h0 + u * kRB + tid;
                t[u] = agent_load((const T *)A.z + hcol[h < nh ? h : 0]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int h = h0 + u * kRB + tid;
                if (h < nh) put(h, t[u]);
            }
        }
    };
    auto store_z = [&](int s, T z) {
        if (tid + s * kRB < nr) agent_store((T *)A.z + r0 + tid + s * kRB, z);
    };

    // 2. r = b - A x, z = D^-1 r, p = z
    double m3[3] = {0.0, 0.0, 0.0};
    T q[S];
#pragma unroll
    for (int s = 0; s < S; ++s) q[s] = T(0);
    if (!A.x_zero) multiply(q);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int i = tid + s * kRB;
        const T b = i < nr ? ((const T *)A.b)[r0 + i] : T(0);
        r[s] = b - q[s];
        const T z = dinv[i] * r[s];
        store_z(s, z);
        m3[0] += (double)r[s] * (double)z;
        m3[1] += (double)r[s] * (double)r[s];
        m3[2] += (double)b * (double)b;
    }
    // (two meetings: a meeting carries two values)
    double m2[2] = {m3[0], m3[1]}, m1[1] = {m3[2]};
    if (!meet_sum(M, m2) || !meet_sum(M, m1)) return;
    double rz = m2[0], rr = m2[1];
    const double bb = m1[0], thr2 = A.rtol > 0.0 ? A.rtol * A.rtol * bb : -1.0;
    int it = 0, status = FE_OK, done = rr <= thr2 ? 1 : 0;
#pragma unroll
    for (int s = 0; s < S; ++s) own[tid + s * kRB] = dinv[tid + s * kRB] * r[s];
    halo([&](int h, T t) { win[h] = t; });
    __syncthreads();

    // 3. iterations
    while (!done && it < A.max_iter) {
        multiply(q);
        double pq[1] = {0.0};
#pragma unroll
        for (int s = 0; s < S; ++s) pq[0] += (double)own[tid + s * kRB] * (double)q[s];
        if (!meet_sum(M, pq)) return;
        if (!(pq[0] > 0.0) || !isfinite(pq[0])) {
            status = FE_EBREAKDOWN;
            done = 1;
            break;
        }
        const double alpha = rz / pq[0];
        const T a = T(alpha);
        m2[0] = m2[1] = 0.0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int i = tid + s * kRB;
            r[s] -= a * q[s];
            const T z = dinv[i] * r[s];
            store_z(s, z);
            x[i] += a * own[i];
            m2[0] += (double)r[s] * (double)z;
            m2[1] += (double)r[s] * (double)r[s];
        }
        if (!meet_sum(M, m2)) return;
        const T beta = T(m2[0] / rz);
        rz = m2[0];
        rr = m2[1];
        ++it;
        if (rr <= thr2) {
            done = 1;
            break;
        }
        if (it == A.max_iter) break;
#pragma unroll
        for (int s = 0; s < S; ++s) own[tid + s * kRB] = dinv[tid + s * kRB] * r[s] + beta * own[tid + s * kRB];
        halo([&](int h, T t) { win[h] = t + beta * win[h]; });
        __syncthreads();
    }

    // 4. FP64: the true residual ||b - A x||^2, x exchanged like z
    double tr = 0.0;
    if constexpr (sizeof(T) == 8) {
        double none[1] = {0.0};
#pragma unroll
        for (int s = 0; s < S; ++s) store_z(s, x[tid + s * kRB]);
        if (!meet_sum(M, none)) return;
#pragma unroll
        for (int s = 0; s < S; ++s) own[tid + s * kRB] = x[tid + s * kRB];
        halo([&](int h, T t) { win[h] = t; });
        __syncthreads();
        multiply(q);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int i = tid + s * kRB;
            const T d = (i < nr ? ((const T *)A.b)[r0 + i] : T(0)) - q[s];
            none[0] += (double)d * (double)d;
        }
        M.limit = A.last_limit;
        if (!meet_sum(M, none)) return;
        tr = none[0];
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (tid + s * kRB < nr) ((T *)A.x)[r0 + tid + s * kRB] = x[tid + s * kRB];
    if (tid == 0) {
        agent_store(&A.out->wrote_x, 1);
        if (g == 0) {
            A.out->done = done;
            A.out->status = status;
            A.out->iterations = it;
            A.out->rr = rr;
            A.out->bb = bb;
            A.out->true_rr = tr;
            A.out->ran = 1;
        }
    }
}

__global__ void __launch_bounds__(256) k_resident_init(unsigned long long *slots, uint32_t *stop, uint32_t stopped,
                                                       ResidentOut *out, int32_t *bad)
{
    for (int q = threadIdx.x; q < (int)(3 * kMeetBuffer); q += 256) slots[q] = kEmpty;
    if (threadIdx.x == 0) {
        *out = ResidentOut{};
        *stop = stopped;
        if (bad) *bad = 0;
    }
}

template <class T, int W, int S, int L = 0>
hipError_t launch_ws(const ResidentArgs &A, int G, hipStream_t s)
{
    hipLaunchKernelGGL((k_resident<T, W, S, L>), dim3(G), dim3(kRB), 0, s, A);
    return hipGetLastError();
}

template <class T, int W>
hipError_t launch_w(const ResidentArgs &A, int G, int S, hipStream_t s)
{
    if (S <= 1) return launch_ws<T, W, 1>(A, G, s);
    if (S == 2) return launch_ws<T, W, 2>(A, G, s);
    if (S <= 4) return launch_ws<T, W, 4>(A, G, s);
    if constexpr (sizeof(T) == 8 && W == 27) {
        if (S == 5) return launch_ws<T, W, 5>(A, G, s);
        if (S == 6) return launch_ws<T, W, 6, 1>(A, G, s);
    } else {
        if (S <= 6) return launch_ws<T, W, 6>(A, G, s);
        if (S <= resident_rows(sizeof(T), W)) return launch_ws<T, W, resident_rows(sizeof(T), W)>(A, G, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool resident_shape(int elem_bytes, int64_t N, int max_row, int cus, int &G, int &R)
{
    const int W = resident_width(max_row);
    if (W == 0 || N < 1 || cus < 1) return false;
    const int64_t cap = (int64_t)resident_rows(elem_bytes, W) * kRB;
    const int64_t most = cus < kResidentMaxGroups ? cus : kResidentMaxGroups;
    // Rows per thread: a row costs ~0.3 us per iteration, a meeting of G groups
    // 1.1 us at 6, 1.9 at 62, 2.7 at 141 and 3.2 at 256.  So 1, 2 or 4 rows, the
    // least that needs no more than 48 groups, else 4 on as many as it takes
    // and then more on all of them (35937 rows of 27: 6.7 us per iteration with
    // 1 row, 141 groups).
    int64_t s = 1;
    while (s < 4 && N > 48 * kRB * s) s *= 2;
    int64_t g = (N + kRB * s - 1) / (kRB * s);
    if (g > most) g = most;
    const int64_t r = (N + g - 1) / g;
    if (r > cap) return false;
    R = (int)r;
    G = (int)((N + r - 1) / r);   // no group without rows
    return true;
}

size_t resident_off_words(int G, int R, int max_row)
{
    return (size_t)G * ((R + kRB - 1) / kRB) * ((resident_width(max_row) + 1) / 2) * kRB;
}

hipError_t launch_resident_plan(const DevMesh &m, const ResidentPlan &P, int G, int R, int32_t *bad, hipStream_t s)
{
    hipLaunchKernelGGL(k_resident_plan, dim3(G), dim3(kRB), 0, s, P, (int)m.N, R, resident_width(m.max_row), m.rowptr,
                       m.colidx, bad);
    return hipGetLastError();
}

hipError_t launch_resident_init(unsigned long long *slots, uint32_t *stop, bool stopped, ResidentOut *out, int32_t *bad,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_resident_init, dim3(1), dim3(256), 0, s, slots, stop, stopped ? 1u : 0u, out, bad);
    return hipGetLastError();
}

template <class T>
hipError_t launch_resident(const ResidentArgs &A, int max_row, int G, hipStream_t s)
{
    const int S = (A.R + kRB - 1) / kRB;
    if (G < 1 || G > kResidentMaxGroups || (int64_t)G * A.R < A.N || (int64_t)(G - 1) * A.R >= A.N ||
        S > resident_rows(sizeof(T), resident_width(max_row)))
        return hipErrorInvalidValue;
    switch (resident_width(max_row)) {
    case 16: return launch_w<T, 16>(A, G, S, s);
    case 27: return launch_w<T, 27>(A, G, S, s);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_resident<double>(const ResidentArgs &, int, int, hipStream_t);
template hipError_t launch_resident<float>(const ResidentArgs &, int, int, hipStream_t);

}  // namespace feasm
