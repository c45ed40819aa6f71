// The PCG solve of one step in a single launch, with the matrix on chip.
//
// A solve reads the same matrix once per iteration.  On a mesh whose matrix
// fits the register files (512 KB a CU, 128 MB in all) and the LDS, the
// streaming kernels (mdx_solver.hip, mdx_mixed.hip) spend an iteration on
// re-reading it and on four to five launches of 2-5 us each.  Here the rows
// are cut into one compact block per CU (recursive coordinate bisection,
// build_onchip in mdx_layout.hip); a 512-thread workgroup loads its block's
// values into registers and their 16-bit local columns into LDS once per solve
// and keeps r, p, q, x (or the FP32 form's correction) in registers until the
// end.  z of the block and of its halo (the neighbouring blocks' rows that its
// columns name) lies in LDS, so a row's gathers are LDS reads; per iteration
// only the halo and one or two FP64 sums per exchange cross workgroups.  15
// entries of 8 to 10 rows a thread do not fit: see AWAY below.
//
// What bounds it: the two exchanges.  An iteration's parts by the clock, us,
// (products, exchange, update, exchange, halo): 9,261-node FP64 cube, 19
// workgroups of a row a thread, 0.3 + 1.3 + 0.1 + 1.7 + 0.5; 442,401-node slab,
// 256 of 4 rows, 1.0 + 2.9 + 0.2 + 3.2 + 0.7; FP32, 871,221 nodes, 7 rows, 2.0 +
// 3.4 + 0.4 + 3.6 + 0.6; 1,255,450-node shell, 10 rows, 5.1 + 7.0 + 3.0 + 5.2 +
// 3.4.  Wavefronts wait 64-81% of their cycles.  An exchange alone measured 1.3
// us at 16 workgroups, 1.8 at 256, there 3.0 with one copy of the slots and 2.1-2.3
// over two levels.  Time steps, streaming kernels -> this (solve): cube 283 -> 82
// us (65-67), 58,176-node slab 406 -> 133 (108-111), 442,401-node slab 696 ->
// 258 (171-178), FP32 iteration on 871,221 nodes 464 -> 263 (106-115), learned
// 1,255,450-node shell 727 -> 569 (300-315).
// Gathering z through the caches instead of LDS took 4.3 us of the FP64 slab's
// iteration and 14 of the shell's.
//
// Iteration k (Algorithm 1, A being linear as in the two-kernel schemes):
//   q = A z_k + beta_k q, p = z_k + beta_k p; exchange p.q; alpha_k;
//   x += alpha p, r -= alpha q, z = D^-1 r (to LDS and written through);
//   exchange r.z and z.z; stopping test, beta_{k+1}; halo of z.
// The FP32 form's residual replacement (mdx_mixed.hip) happens in the same
// launch: the correction takes z's place in the window, r64 -= A delta in
// FP64, x64 += delta, an exchange, the test on the true residual.
//
// Exchange: every workgroup writes its partial sums to its slots and polls all
// workgroups' slots until none holds the empty word, then sums them in slot
// order: all workgroups form the same bits and take the same branch, no
// counter is contended, and a value and its arrival are one 8-byte access.
// Slots are kept once per XCD (fewer pollers per line) and in three turns: on
// leaving exchange e a workgroup empties its slots of exchange e - 1 (every
// workgroup has left that one: it has written e), and they are empty before it
// writes e + 1, so before any workgroup looks for e + 2 in them.  What crosses
// workgroups is stored and loaded with agent scope (write-through past the XCD's
// L2, read past it) and complete (vmcnt) before the slot is written, so no cache
// is flushed or invalidated.
//
// The wait needs every workgroup resident: a launch has at most one per CU, and
// launches are in flight together only as far as the CUs reach (OnchipCus).
// Polls are bounded: where other work keeps a workgroup off the chip for long,
// the launch gives up and changes nothing but scratch and x; the host then forms
// the step's right-hand side again and solves it with the streaming kernels.
//
// A launch has one outcome: a workgroup whose polls are used up enters "gave
// up", the first workgroup "finished" where it has seen the last exchange, and
// the first of these entries holds (settle()).  A workgroup that comes too late
// to give up keeps looking: its exchange is the last one, which the first
// workgroup has seen whole, so the sums it lacks have been stored and arrive.
// One that has finished where the launch gave up has only written rows of x.  So
// what the first workgroup publishes, and what kernels behind the launch read in
// the scalars, holds for all workgroups.
#include "mdx_device.h"
#include "mdx_internal.h"

#include <algorithm>

namespace mdx {

namespace {

constexpr int OB = kOnchipThreads;  // threads of a workgroup
constexpr int OW = OB / SLICE;      // its wavefronts
constexpr int HT = kOnchipHaloPass, HR = kOnchipHalo / HT;   // halo entries of a pass, passes

typedef unsigned long long u64;
constexpr u64 kEmpty = ~0ull;       // slot without a value (a NaN no arithmetic gives)

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp0(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}
// sum over the wavefront by data-parallel moves; the total is in lane 63
__device__ __forceinline__ double wave_total63(double v)
{
    v += dpp0<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8: lane 15 of each row of 16
    v += dpp0<0x112, 0xf>(v);
    v += dpp0<0x114, 0xf>(v);
    v += dpp0<0x118, 0xf>(v);
    v += dpp0<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp0<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

template <class T>
__device__ __forceinline__ T ld_agent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_agent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// this wavefront's stores have reached the agent's point of coherence
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One try to enter the launch's outcome, 2 * launch + (1: gave up), over an
// earlier launch's: what it found, `was` if the entry now stands.
__device__ __forceinline__ uint32_t try_settle(uint32_t *word, uint32_t was, uint32_t outcome)
{
    __hip_atomic_compare_exchange_strong(word, &was, outcome, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return was;
}
// The launch's outcome if it has one, else this one.
__device__ __forceinline__ bool settle(uint32_t *word, unsigned launch, bool gave_up)
{
    uint32_t now = ld_agent(word);
    while (now >> 1 != launch)   // at most one other entry gets in between
        if (__hip_atomic_compare_exchange_strong(word, &now, launch << 1 | (gave_up ? 1u : 0u),
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return gave_up;
    return now & 1;
}

struct ExchangeLds {
    double part[3][OW];
    double tot[2];
    int ok;
};

// The workgroups that exchange: those of one system, g0 .. g0 + G - 1.
struct Team {
    u64 *words;
    int polls, g, g0, G;
};
// a workgroup's part in a launch with one outcome
struct SolveTeam : Team {
    const OnchipSolve &a;
    // exchange at which this workgroup takes its looks for used up (-1: none)
    int stops_at;
    __device__ __forceinline__ SolveTeam(const OnchipSolve &a, int g, int G)
        : Team{a.words, a.polls, g, 0, G}, a(a),
          stops_at(a.give_up.group == g ? a.give_up.exchange - 1 : -1)
    {
    }
    __device__ __forceinline__ bool stops(int at) const { return at == stops_at; }
    // no more looking: true if the launch gives up
    __device__ __forceinline__ bool gives_up() const
    {
        uint32_t *const word = &a.sc->onchip_verdict;
        if (stops_at >= 0 && a.give_up.wait)
            for (int n = 0; n < polls && ld_agent(word) >> 1 != a.launch;) ++n;
        const int r = (threadIdx.x & 63) == 0 && settle(word, a.launch, true);
        return __builtin_amdgcn_readfirstlane(r) != 0;
    }
};
// the batched form: a kernel behind it looks at every instance's outcome
struct BatchTeam : Team {
    __device__ __forceinline__ bool stops(int) const { return false; }
    __device__ __forceinline__ bool gives_up() const { return true; }
};
// exchanges of iteration `it` (kind 0 p.q, 1 r.z; 2, 3, 4 of a replacement after
// it), as OnchipGiveUp counts them from 1 on
__device__ __forceinline__ int exchange_of(int it, int kind) { return 8 * it + kind; }

// Sum v over all threads of the team; false when the wait gave up.
// turn: 0, 1, 2, 0, ... in successive exchanges; at: which one this is.
// during() runs once the workgroup's sums are on their way: loads issued there
// are hidden by the wait (issued before it they would hold up the sums: the store
// count that orders them counts loads too).
template <int NV, class T, class F>
__device__ __forceinline__ bool exchange(double (&v)[NV], ExchangeLds &l, const T &team,
                                         int &turn, int at, F &&during)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr size_t TURN = NXCD * 2 * kOnchipGroups;   // slots of a turn: [XCD][value][workgroup]
    u64 *const words = team.words;
    const int g = team.g, G = team.G;
    u64 *buf = words + turn * TURN;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const double s = wave_total63(v[k]);
        if (lane == 63) l.part[k][w] = s;
    }
    stores_done();
    __syncthreads();
    if (w == 0) {
        double s[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            s[k] = l.part[k][0];
#pragma unroll
            for (int i = 1; i < OW; ++i) s[k] += l.part[k][i];
        }
        if (lane < NXCD * NV) {
            const double x = lane < NXCD ? s[0] : s[NV - 1];
            u64 b = (u64)__double_as_longlong(x);
            if (b == kEmpty) b = 0x7ff8000000000000ull;
            st_agent(buf + (lane % NXCD * 2 + lane / NXCD) * kOnchipGroups + g, b);
        }
    }
    during();
    if (w == 0) {
        buf += blockIdx.x % NXCD * (2 * kOnchipGroups) + team.g0;
        constexpr int C = kOnchipGroups / SLICE;
        double acc[NV];
        bool all = false;
        // (the outer loop's second pass: the sums that lack are on their way)
        for (bool look = !team.stops(at);; look = true) {
            int n = 0;
            if (look)
                do {
                    u64 s[C][NV];
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (c * SLICE < G) {
                            const int slot = c * SLICE + lane;
#pragma unroll
                            for (int k = 0; k < NV; ++k)
                                s[c][k] = slot < G ? ld_agent(buf + k * kOnchipGroups + slot) : 0ull;
                        }
                    all = true;
#pragma unroll
                    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (c * SLICE < G)
#pragma unroll
                            for (int k = 0; k < NV; ++k) {
                                all = all && s[c][k] != kEmpty;
                                acc[k] += __longlong_as_double((long long)s[c][k]);
                            }
                    all = __all(all);
                } while (!all && ++n < team.polls);
            if (all || team.gives_up()) break;
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double t = wave_total63(acc[k]);
            if (lane == 63) l.tot[k] = t;
        }
        if (lane == 0) l.ok = all ? 1 : 0;
        // empty the slots of the previous exchange, which every workgroup has
        // left (it has written this one's): the next but one uses them again
        const int prev = turn == 0 ? 2 : turn - 1;
        if (lane < 2 * NXCD) st_agent(words + prev * TURN + lane * kOnchipGroups + g, kEmpty);
    }
    turn = turn == 2 ? 0 : turn + 1;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = l.tot[k];
    return l.ok != 0;
}
__device__ __forceinline__ void nothing() {}

// the solve's start: either the right-hand-side pass's partials summed here
// (every workgroup, in one fixed order) or the scalars a finalize kernel wrote
struct Start {
    double rho, z0, ref, floor_;
    bool finite, done;
};
// (at most 4 partials a thread, loaded before the matrix so that their sum
// does not wait for it)
struct Partials {
    double v[3];
    __device__ __forceinline__ void load(const OnchipSolve &a)
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = 0.0;
        double t[4][3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = j * OB + (int)threadIdx.x;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                t[j][k] = i < a.part_groups ? a.part[k * a.part_groups + i] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k] += t[j][k];
    }
};
// sums over the workgroup, in every thread
__device__ __forceinline__ void block_totals(double (&v)[3], ExchangeLds &l)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double t = wave_total63(v[k]);
        if (lane == 63) l.part[k][w] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[k] = l.part[k][0];
#pragma unroll
        for (int i = 1; i < OW; ++i) v[k] += l.part[k][i];
    }
    __syncthreads();
}
__device__ __forceinline__ Start start_of(const OnchipSolve &a, Partials &q, ExchangeLds &l)
{
    Start s;
    const Scalars *sc = a.sc;
    if (a.part_groups == 0) {
        s.rho = sc->rho[0];
        s.z0 = sc->z0;
        s.ref = sc->ref;
        s.floor_ = sc->floor_;
        s.finite = sc->nonfinite == 0;
        s.done = sc->done != 0;
        return s;
    }
    double (&v)[3] = q.v;
    block_totals(v, l);
    s.rho = v[0];
    s.z0 = sqrt(v[1]);
    const double db = sqrt(v[2]);
    s.ref = a.rel_mode == 1 ? db : s.z0;
    s.floor_ = 1e-15 * db;
    s.finite = isfinite(s.z0) && isfinite(db) && isfinite(v[0]);
    s.done = !s.finite || s.z0 <= s.floor_ || s.z0 < sc->atol;
    return s;
}

// The outcome into the scalars and to the host (first workgroup).
struct Outcome {
    double rho, znorm;
    int it, done, nonfinite, aborted;
};
// The first workgroup enters "finished", over the last launch's outcome as a
// rule: before the stores of x and of the scalars and the copy, which hide the
// way there and back.  (Without an exchange nobody has given up.)
__device__ __forceinline__ uint32_t enter_finished(const OnchipSolve &a, const Outcome &o)
{
    uint32_t found = (a.launch - 1) << 1;
    if (blockIdx.x == 0 && threadIdx.x == 0 && !o.aborted && o.it > 0)
        found = try_settle(&a.sc->onchip_verdict, found, a.launch << 1);
    return found;
}
__device__ void report(const OnchipSolve &a, const Start &s, const Outcome &o, int turn, uint32_t found)
{
    if (blockIdx.x != 0 || threadIdx.x >= SLICE) return;
    Scalars *sc = a.sc;
    if (threadIdx.x == 0) {
        st_agent(&sc->rho[o.it & 1], o.rho);
        st_agent(&sc->ref, s.ref);
        st_agent(&sc->floor_, s.floor_);
        st_agent(&sc->z0, s.z0);
        st_agent(&sc->znorm, o.znorm);
        st_agent(&sc->nonfinite, o.nonfinite);
        st_agent(&sc->iters, o.done ? o.it : 0);
        st_agent(&sc->replace, 0);
        st_agent(&sc->beta, 0.0);
        st_agent(&sc->it_next, o.it);
        st_agent(&sc->onchip_turn, turn);
        st_agent(&sc->onchip_gave_up, o.aborted);
        st_agent(&sc->done, o.aborted ? 0 : o.done);
    }
    stores_done();
    copy_scalars(sc, a.pub);
    // looked at now: the host and kernels behind this one look after it
    if (found != (a.launch - 1) << 1 && settle(&sc->onchip_verdict, a.launch, false)) {
        stores_done();   // the copy, by other lanes
        st_agent(&sc->onchip_gave_up, 1);
        st_agent(&sc->done, 0);
        a.pub->s.onchip_gave_up = 1;
        a.pub->s.done = 0;
    }
    __threadfence_system();
    if (threadIdx.x == 0) a.pub->seq = a.seq;
}

// This thread's rows: pass i holds row i * OB + thread of the block, if the
// block has that many.  Local columns, four 16-bit window positions to an
// 8-byte LDS word; the quads past LQ stay in registers.
template <int W, int R, int LQ>
struct Rows {
    static constexpr int Q = (W + 3) / 4, NR = Q - LQ;
    uint2 reg[NR > 0 ? R : 1][NR > 0 ? NR : 1];
    __device__ __forceinline__ void load(const uint2 *col, int g, uint2 (*lds)[OB])
    {
        const uint2 *c = col + (size_t)g * R * Q * OB + threadIdx.x;
#pragma unroll
        for (int i = 0; i < R; ++i) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const uint2 v = c[(i * Q + q) * OB];
                    if (q < LQ)
                        lds[i * LQ + q][threadIdx.x] = v;
                    else if constexpr (NR > 0)
                        reg[i][q - LQ] = v;
                }
            }
    }
    __device__ __forceinline__ uint2 get(const uint2 (*lds)[OB], int i, int q, int t) const
    {
        if (q < LQ) return lds[i * LQ + q][t];
        uint2 c = reg[NR > 0 ? i : 0][NR > 0 ? q - LQ : 0];
        asm volatile("" : "+v"(c.x), "+v"(c.y));   // unpacked here, not once before the loop
        return c;
    }
    // sum_j val_j x[col_j] in column order, accumulated in ACC; x in LDS
    template <class ACC, class T>
    __device__ __forceinline__ ACC product(const T (&val)[R][W], const uint2 (*lds)[OB], int i, int t,
                                           const T *x) const
    {
        T xx[W];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint2 c = get(lds, i, q, t);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * q + j < W) {
                    const unsigned h = j < 2 ? c.x : c.y;
                    xx[4 * q + j] = x[j & 1 ? h >> 16 : h & 0xffffu];
                }
        }
        ACC s = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            T v = val[i][j];
            // converted here: kept converted across the iterations the values
            // would take twice their registers
            if constexpr (sizeof(ACC) != sizeof(T)) asm volatile("" : "+v"(v));
            s += (ACC)v * (ACC)xx[j];
        }
        return s;
    }
    // sum_j val_j x[col_j] over the wavefront's first nq quads (even; all for
    // even rows), as L lanes of the streaming product add them: entry j to the
    // (j mod L)-th of L sums in FP32, then the sums by a butterfly
    template <int L, bool UNEVEN>
    __device__ __forceinline__ float product_l(const float (&val)[R][W], const uint2 (*lds)[OB], int i,
                                               int t, const float *x, int nq) const
    {
        constexpr int STEP = UNEVEN ? 2 : Q;   // quads whose gathers go out together
        float s[L];
#pragma unroll
        for (int u = 0; u < L; ++u) s[u] = 0.0f;
#pragma unroll
        for (int q0 = 0; q0 < Q; q0 += STEP)
            if (!UNEVEN || q0 < nq) {
                float xx[4 * STEP];
#pragma unroll
                for (int q = q0; q < q0 + STEP && q < Q; ++q) {
                    const uint2 c = get(lds, i, q, t);
                    xx[4 * (q - q0)] = x[c.x & 0xffffu];
                    xx[4 * (q - q0) + 1] = x[c.x >> 16];
                    xx[4 * (q - q0) + 2] = x[c.y & 0xffffu];
                    if (4 * q + 3 < W) xx[4 * (q - q0) + 3] = x[c.y >> 16];
                }
#pragma unroll
                for (int j = 4 * q0; j < 4 * (q0 + STEP) && j < W; ++j)
                    s[j % L] = __builtin_fmaf(val[i][j], xx[j - 4 * q0], s[j % L]);
            }
#pragma unroll
        for (int off = L / 2; off > 0; off /= 2)
#pragma unroll
            for (int u = 0; u < off; ++u) s[u] += s[u + off];
        return s[0];
    }
    template <bool UNEVEN>
    __device__ __forceinline__ float product_as(int lanes, const float (&val)[R][W],
                                                const uint2 (*lds)[OB], int i, int t, const float *x,
                                                int nq) const
    {
        switch (lanes) {
        case 2: return product_l<2, UNEVEN>(val, lds, i, t, x, nq);
        case 4: return product_l<4, UNEVEN>(val, lds, i, t, x, nq);
        case 8: return product_l<8, UNEVEN>(val, lds, i, t, x, nq);
        case 16: return product_l<16, UNEVEN>(val, lds, i, t, x, nq);
        default: return product_l<1, UNEVEN>(val, lds, i, t, x, nq);
        }
    }
    // FP64 sum with the FP32 values read here again (A: the thread's first)
    __device__ __forceinline__ double reread(const float4 *A, const uint2 (*lds)[OB], int i, int t,
                                             const float *x) const
    {
        float4 v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = A[(i * Q + q) * OB];
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint2 c = get(lds, i, q, t);
            const float a[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * q + j < W) {
                    const unsigned h = j < 2 ? c.x : c.y;
                    s += (double)a[j] * (double)x[j & 1 ? h >> 16 : h & 0xffffu];
                }
        }
        return s;
    }
    // the same with FP64 values read here, in pairs (A: the thread's first)
    __device__ __forceinline__ double streamed(const double2 *A, const uint2 (*lds)[OB], int i, int t,
                                               const float *x, int nq) const
    {
        constexpr int P = (W + 1) / 2;
        double2 v[P];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q < nq) {
                v[2 * q] = A[(i * P + 2 * q) * OB];
                v[2 * q + 1] = A[(i * P + 2 * q + 1) * OB];
            }
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q < nq) {
                const uint2 c = get(lds, i, q, t);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * q + j < W) {
                        const unsigned h = j < 2 ? c.x : c.y;
                        const double a = j & 1 ? v[2 * q + j / 2].y : v[2 * q + j / 2].x;
                        s += a * (double)x[j & 1 ? h >> 16 : h & 0xffffu];
                    }
            }
        return s;
    }
};

// Has row i's product formed here: the compiler would put the sums off and
// hold every row's gathered values until then.
__device__ __forceinline__ void formed(double &q) { asm volatile("" : "+v"(q)); }
__device__ __forceinline__ void formed(float &q) { asm volatile("" : "+v"(q)); }

// the values of the thread's rows, 16 bytes a load
template <int W, int R>
__device__ __forceinline__ void load_values(const double *__restrict__ A, double (&val)[R][W])
{
    constexpr int P = (W + 1) / 2;
    const double2 *p = reinterpret_cast<const double2 *>(A) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const double2 v = p[(i * P + j) * OB];
            val[i][2 * j] = v.x;
            if (2 * j + 1 < W) val[i][2 * j + 1] = v.y;
        }
}
template <int W, int R>
__device__ __forceinline__ void load_values(const float *__restrict__ A, float (&val)[R][W])
{
    constexpr int P = (W + 3) / 4;
    const float4 *p = reinterpret_cast<const float4 *>(A) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const float4 v = p[(i * P + j) * OB];
            val[i][4 * j] = v.x;
            if (4 * j + 1 < W) val[i][4 * j + 1] = v.y;
            if (4 * j + 2 < W) val[i][4 * j + 2] = v.z;
            if (4 * j + 3 < W) val[i][4 * j + 3] = v.w;
        }
}

// the first nq quads of pass i of the thread's rows
template <int W, int R>
__device__ __forceinline__ void load_values_n(const float *__restrict__ A, float (&val)[R][W], int i,
                                              int nq)
{
    constexpr int P = (W + 3) / 4;
    const float4 *p = reinterpret_cast<const float4 *>(A) + threadIdx.x;
#pragma unroll
    for (int j = 0; j < P; ++j)
        if (j < nq) {
            const float4 v = p[(i * P + j) * OB];
            val[i][4 * j] = v.x;
            val[i][4 * j + 1] = v.y;
            val[i][4 * j + 2] = v.z;
            if (4 * j + 3 < W) val[i][4 * j + 3] = v.w;
        }
}

// Halo of the window, filled by all wavefronts but the first (which polls):
// fetch() reads the entries' places (during an exchange, whose wait hides it),
// fill() the entries themselves after it.  Lists are padded to whole passes.
struct Halo {
    unsigned at[HR];   // byte offsets (one register each beside the uniform base)
    template <class T>
    __device__ __forceinline__ void fetch(const unsigned *idx, int passes)
    {
        if (threadIdx.x < SLICE) return;
        const unsigned h = threadIdx.x - SLICE;
#pragma unroll
        for (int k = 0; k < HR; ++k)
            if (k < passes) at[k] = (idx + k * HT)[h] * (unsigned)sizeof(T);
    }
    template <class T>
    __device__ __forceinline__ void fill(const T *zb, T *win, int passes) const
    {
        combine(zb, win, passes, [](T z, T, int) { return z; });
        __syncthreads();
    }
    // win = f(entry, win, pass), without the barrier
    template <class T, class F>
    __device__ __forceinline__ void combine(const T *zb, T *win, int passes, F &&f) const
    {
        if (threadIdx.x < SLICE) return;
        const unsigned h = threadIdx.x - SLICE;
        T v[HR];
#pragma unroll
        for (int k = 0; k < HR; ++k)
            if (k < passes)
                v[k] = ld_agent(reinterpret_cast<const T *>(reinterpret_cast<const char *>(zb) + at[k]));
#pragma unroll
        for (int k = 0; k < HR; ++k)
            if (k < passes) win[k * HT + h] = f(v[k], win[k * HT + h], k);
    }
};

// The FP64 values that a residual replacement reads and writes of the thread's
// rows (rows: the thread's first place).
template <int R>
struct Ahead {
    int at[R];   // -1 past the block's last row
    double r[R], x[R], d[R];
    __device__ __forceinline__ void places(const int32_t *rows)
    {
#pragma unroll
        for (int i = 0; i < R; ++i) at[i] = rows[i * OB];
    }
    __device__ __forceinline__ void read(const double *r64, const double *x64, const double *dinv, int i)
    {
        const int k = max(at[i], 0);
        r[i] = r64[k];
        x[i] = x64[k];
        d[i] = dinv[k];
    }
};

// The small shapes need few registers more than the 128 with which a CU holds two
// workgroups, and so two such launches find room where one would (no spills).
constexpr int waves_per_simd(int W, int R) { return W * R <= 15 ? 4 : 2; }

// ---- plain FP64 ------------------------------------------------------------
template <int W, int R>
__global__ __launch_bounds__(OB, waves_per_simd(W, R)) void k_onchip(OnchipSolve a)
{
    constexpr int LQ = (W + 3) / 4, own = R * OB;
    __shared__ ExchangeLds xl;
    __shared__ uint2 lcol[R * LQ][OB];
    __shared__ double win[own + kOnchipHalo];
    __shared__ double ldv[R][OB];
    const int G = gridDim.x, g = logical_group(G);
    const SolveTeam team(a, g, G);
    int t = threadIdx.x;
    unsigned at0 = (unsigned)g * own + t;   // block position of pass i: at0 + i * OB
    double *zb = static_cast<double *>(a.zb);
    Partials parts;
    parts.load(a);
    const int h0 = a.map.halo_ptr[g], nh = (a.map.halo_ptr[g + 1] - h0) / HT;   // its passes
    double val[R][W], r[R], p[R], q[R], x[R];
    Rows<W, R, LQ> rows;
    rows.load(a.map.col, g, lcol);
    asm volatile("" ::: "memory");   // the columns' registers are free again
    load_values<W, R>(a.map.val64 + (size_t)g * own * (W + 1), val);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = a.map.row[at0 + i * OB], at = max(row, 0);
        const double ri = a.r[at], xi = a.x[at], zi = a.z[at];
        r[i] = row < 0 ? 0.0 : ri;
        x[i] = row < 0 ? 0.0 : xi;
        p[i] = q[i] = 0.0;
        win[i * OB + t] = row < 0 ? 0.0 : zi;
        ldv[i][t] = a.map.dinv64[at0 + i * OB];
    }
    for (int h = t; h < nh * HT; h += OB) win[own + h] = a.z[a.map.halo_row[h0 + h]];
    const Start st = start_of(a, parts, xl);
    Outcome o{st.rho, st.z0, 0, 1, st.finite ? 0 : 2, 0};
    int turn = a.sc->onchip_turn;   // the first workgroup writes it after every exchange
    if (st.done) {
        report(a, st, o, turn, (a.launch - 1) << 1);
        return;
    }
    __syncthreads();
    const StopTest test = {a.sc->atol, a.sc->rtol, st.ref, st.floor_};
    double rho = st.rho, beta = 0.0;
    int it = 0;
    o.done = 0;
    for (;;) {
        // addresses and columns are formed anew in each iteration: kept across
        // iterations they would take more registers than the vectors
        asm volatile("" : "+v"(at0), "+v"(t));
        double pq[1] = {0.0};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            q[i] = rows.template product<double>(val, lcol, i, t, win) + beta * q[i];
            formed(q[i]);
            p[i] = win[i * OB + t] + beta * p[i];
            pq[0] += p[i] * q[i];
        }
        if (!exchange<1>(pq, xl, team, turn, exchange_of(it, 0), nothing)) {
            o.aborted = 1;
            break;
        }
        const double alpha = rho / pq[0];
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            x[i] += alpha * p[i];
            r[i] -= alpha * q[i];
            const double z = ldv[i][t] * r[i];
            win[i * OB + t] = z;
            st_agent(zb + at0 + i * OB, z);
            v[0] += r[i] * z;
            v[1] += z * z;
        }
        Halo halo;
        if (!exchange<2>(v, xl, team, turn, exchange_of(it, 1), [&] { halo.fetch<double>(a.map.halo_at + h0, nh); })) {
            o.aborted = 1;
            break;
        }
        ++it;
        const double zn = sqrt(v[1]);
        o.znorm = zn;
        if (!isfinite(zn)) {
            o.nonfinite = 2;
            o.done = 1;
            break;
        }
        if (passes(test, zn)) {
            o.done = 1;
            break;
        }
        if (it >= a.max_iter) break;   // cap: the host reports no convergence
        beta = v[0] / rho;
        rho = v[0];
        halo.fill(zb, win + own, nh);
    }
    o.it = it;
    o.rho = rho;
    const uint32_t found = enter_finished(a, o);
    if (!o.aborted)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int row = a.map.row[at0 + i * OB];
            if (row >= 0) a.x[row] = x[i];
        }
    report(a, st, o, turn, found);
}

// ---- FP32 iteration with FP64 residual replacement ---------------------------
// LQ: quads of columns in LDS (fewer than all where R rows' would not fit).
// AWAY: r, the correction and D^-1, which the product does not need, are kept in
// memory by block position and come back for the update: with them the largest
// blocks do not fit.  Nor do they quite without: 10 rows of 15 entries spill 672
// bytes a lane (8 rows 408), and by counters a solve of the 1,255,450-node shell
// moves 717 MB in and 355 MB out beyond the L2s where its matrix and vectors are
// some 180 MB.
template <int W, int R, int LQ, bool AWAY>
__global__ __launch_bounds__(OB) void k_onchip32(OnchipSolve a)
{
    constexpr int own = R * OB;
    __shared__ ExchangeLds xl;
    __shared__ uint2 lcol[R * LQ][OB];
    __shared__ float win[own + kOnchipHalo];
    __shared__ float ldv[AWAY ? 1 : R][OB];
    const int G = gridDim.x, g = logical_group(G);
    const SolveTeam team(a, g, G);
    int t = threadIdx.x;
    unsigned at0 = (unsigned)g * own + t;
    float *zb = static_cast<float *>(a.zb);
    Partials parts;
    parts.load(a);
    Start st;
    if constexpr (AWAY) st = start_of(a, parts, xl);   // no registers to wait with
    const int h0 = a.map.halo_ptr[g], nh = (a.map.halo_ptr[g + 1] - h0) / HT;   // its passes
    float val[R][W], p[R], q[R], r[R], d[R];
    Rows<W, R, LQ> rows;
    rows.load(a.map.col, g, lcol);
    asm volatile("" ::: "memory");   // the columns' registers are free again
    if constexpr (!AWAY) load_values<W, R>(a.map.val32 + (size_t)g * own * (W + 1), val);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = a.map.row[at0 + i * OB], at = max(row, 0);
        const float ri = a.r32[at], zi = a.z32[at];
        r[i] = row < 0 ? 0.0f : ri;
        p[i] = q[i] = d[i] = 0.0f;
        win[i * OB + t] = row < 0 ? 0.0f : zi;
        if constexpr (AWAY) {
            a.map.r_away[at0 + i * OB] = r[i];
            a.map.d_away[at0 + i * OB] = 0.0f;
        } else {
            ldv[i][t] = a.map.dinv32[at0 + i * OB];
        }
    }
    for (int h = t; h < nh * HT; h += OB) win[own + h] = a.z32[a.map.halo_row[h0 + h]];
    if constexpr (!AWAY) st = start_of(a, parts, xl);
    Outcome o{st.rho, st.z0, 0, 1, st.finite ? 0 : 2, 0};
    int turn = a.sc->onchip_turn;   // the first workgroup writes it after every exchange
    if (st.done) {
        report(a, st, o, turn, (a.launch - 1) << 1);
        return;
    }
    __syncthreads();
    const StopTest test = {a.sc->atol, a.sc->rtol, st.ref, st.floor_};
    double rho = st.rho, beta = 0.0;
    int it = 0;
    o.done = 0;
    for (;;) {
        // AWAY: the values are read for each run of iterations and again, row
        // by row, for its replacement: held through it they would be spilled
        if constexpr (AWAY) {
            asm volatile("" ::: "memory");
            load_values<W, R>(a.map.val32 + (size_t)g * own * (W + 1), val);
        }
        Halo halo;
        double v[2], zn;
        bool pass, out = false;
        for (;;) {
            asm volatile("" : "+v"(at0), "+v"(t));   // as in k_onchip
            const float bf = (float)beta;
            double pq[1] = {0.0};
            float dv[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                q[i] = rows.template product<float>(val, lcol, i, t, win) + bf * q[i];
                formed(q[i]);
                p[i] = win[i * OB + t] + bf * p[i];
                pq[0] += (double)p[i] * (double)q[i];
            }
            if (!exchange<1>(pq, xl, team, turn, exchange_of(it, 0), nothing)) {
                o.aborted = 1;
                out = true;
                break;
            }
            const float alpha = (float)(rho / pq[0]);
            v[0] = v[1] = 0.0;
#pragma unroll
            for (int i = 0; i < R; ++i)
                if constexpr (AWAY) {
                    dv[i] = a.map.dinv32[at0 + i * OB];
                    r[i] = a.map.r_away[at0 + i * OB];
                    d[i] = a.map.d_away[at0 + i * OB];
                }
#pragma unroll
            for (int i = 0; i < R; ++i) {
                d[i] += alpha * p[i];
                r[i] -= alpha * q[i];
                if constexpr (AWAY) {
                    a.map.d_away[at0 + i * OB] = d[i];
                    a.map.r_away[at0 + i * OB] = r[i];
                }
                const float z = (AWAY ? dv[i] : ldv[AWAY ? 0 : i][t]) * r[i];
                win[i * OB + t] = z;
                st_agent(zb + at0 + i * OB, z);
                v[0] += (double)r[i] * (double)z;
                v[1] += (double)z * (double)z;
            }
            if (!exchange<2>(v, xl, team, turn, exchange_of(it, 1), [&] { halo.fetch<float>(a.map.halo_at + h0, nh); })) {
                o.aborted = 1;
                out = true;
                break;
            }
            ++it;
            zn = sqrt(v[1]);
            o.znorm = zn;
            if (!isfinite(zn)) {
                o.nonfinite = 2;
                o.done = 1;
                out = true;
                break;
            }
            pass = passes(test, zn);
            if (pass || (a.rr > 0 && it % a.rr == 0) || it >= a.max_iter) break;
            beta = v[0] / rho;
            rho = v[0];
            halo.fill(zb, win + own, nh);
        }
        if (out) break;
        // ---- replacement: r64 -= A delta, x64 += delta, the test on r64 ----
        // (zb is overwritten: no workgroup reads z from it at this exchange)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float di = AWAY ? a.map.d_away[at0 + i * OB] : d[i];
            win[i * OB + t] = di;
            st_agent(zb + at0 + i * OB, di);
        }
        // the rows' FP64 residual, solution and D^-1 are read ahead: all of
        // them where the values are gone, else a row ahead of its product
        Ahead<R> row;
        double none[1] = {0.0};
        const bool there = exchange<1>(none, xl, team, turn, exchange_of(it, 2), [&] {
            row.places(a.map.row + at0);
            if constexpr (AWAY)
#pragma unroll
                for (int i = 0; i < R; ++i) row.read(a.r, a.x, a.dinv, i);
            else
                row.read(a.r, a.x, a.dinv, 0);
        });
        if (!there) {
            o.aborted = 1;
            break;
        }
        halo.fill(zb, win + own, nh);
        v[0] = v[1] = 0.0;
        const float4 *A = reinterpret_cast<const float4 *>(a.map.val32) + (size_t)g * (own * (W + 1) / 4) + t;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            double ad;
            if constexpr (AWAY) {
                ad = rows.reread(A, lcol, i, t, win);
            } else {
                if (i + 1 < R) row.read(a.r, a.x, a.dinv, i + 1);
                ad = rows.template product<double>(val, lcol, i, t, win);
            }
            formed(ad);
            float ri = 0.0f;
            if (row.at[i] >= 0) {
                const double r64 = row.r[i] - ad;
                a.r[row.at[i]] = r64;
                a.x[row.at[i]] = row.x[i] + (double)win[i * OB + t];
                ri = (float)r64;
                const double zi = row.d[i] * r64;
                v[1] += zi * zi;
            }
            v[0] += (double)ri * (double)(a.map.dinv32[at0 + i * OB] * ri);
            if constexpr (AWAY) {
                a.map.r_away[at0 + i * OB] = ri;
                a.map.d_away[at0 + i * OB] = 0.0f;
            } else {
                r[i] = ri;
                d[i] = 0.0f;
            }
        }
        if (!exchange<2>(v, xl, team, turn, exchange_of(it, 3), nothing)) {
            o.aborted = 1;
            break;
        }
        zn = sqrt(v[1]);
        o.znorm = zn;
        if (!isfinite(zn)) {
            o.nonfinite = 2;
            o.done = 1;
            break;
        }
        if (passes(test, zn)) {
            o.done = 1;
            break;
        }
        if (it >= a.max_iter) break;
        // restart (p = z) where the recursive residual had passed, the
        // recurrence kept after a periodic replacement
        beta = pass ? 0.0 : v[0] / rho;
        rho = v[0];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float ri = AWAY ? a.map.r_away[at0 + i * OB] : r[i];
            const float z = a.map.dinv32[at0 + i * OB] * ri;
            win[i * OB + t] = z;
            st_agent(zb + at0 + i * OB, z);
        }
        if (!exchange<1>(none, xl, team, turn, exchange_of(it, 4), nothing)) {
            o.aborted = 1;
            break;
        }
        halo.fill(zb, win + own, nh);
    }
    o.it = it;
    o.rho = rho;
    const uint32_t found = enter_finished(a, o);
    report(a, st, o, turn, found);
}

// ---- batched: independent systems, FP32 iteration, FP64 replacement ----------
// The recurrences of mdx_batch.hip, every instance by a team of workgroups of
// its own that leaves when the instance is done.  The window holds the search
// direction: a workgroup forms its own rows' p = D^-1 r + beta p and, from the r
// that their owners wrote, its halo's, with the same operations and so the
// same bits, and q = A p needs no recurrence.  A row's FP32 sum is added up as
// the installed streaming layout does (lanes per row), so iterates and counts
// are the streaming kernels' but for the order of the FP64 sums (an instance
// alone and in a batch agree to that order too, bitwise where both take the
// same rows a thread).  The replacement updates the FP64 residual by the
// correction (r64 -= A delta, FP64 values of A streamed by block), which is
// b - A (x + delta) up to the rounding of x.
//
// Solve of a step, streaming kernels -> this (and the whole step, with the
// ionic update's fused passes): 12 unstructured shells of 232,472 nodes in
// all, 4.0 iterations, 130 -> 49 us (187 -> 96); 8 surfaces of 1,310,736, 1.8
// iterations, 165 -> 69 (280 -> 171).
// Bound by one read of the values and columns (23 and 45 MB), the replacement's
// read of the FP64 values and some 3 us per exchange.
//
// UNEVEN: unstructured meshes, whose rows' lengths spread (12 to 33 entries,
// 16 on average): a block's rows are sorted by length and a wavefront forms
// the quads that its longest row has.
template <int W, int R, bool UNEVEN>
__global__ __launch_bounds__(OB) void k_onchip_batch(OnchipBatch a)
{
    constexpr int LQ = (W + 3) / 4, own = R * OB;
    __shared__ ExchangeLds xl;
    __shared__ uint2 lcol[R * LQ][OB];
    __shared__ float win[own + kOnchipHalo];
    __shared__ float ldv[R][OB];
    const int g = logical_group(gridDim.x);
    const int4 gr = a.grp[g];
    const BatchTeam team = {{a.words, g == a.once ? 1 : a.polls, g, gr.y, gr.z}};
    int t = threadIdx.x;
    unsigned at0 = (unsigned)g * own + t;
    // the instance's partials, summed by each of its workgroups in one order
    Start st;
    {
        double v[3] = {0.0, 0.0, 0.0};
        const int i1 = a.inst_grp[gr.x + 1];
        for (int i = a.inst_grp[gr.x] + t; i < i1; i += OB)
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k] += a.part[k * a.part_groups + i];
        block_totals(v, xl);
        st.rho = v[0];
        st.z0 = sqrt(v[1]);
        const double db = sqrt(v[2]);
        st.ref = a.bp.rel_mode == 1 ? db : st.z0;
        st.floor_ = 1e-15 * db;
        st.finite = isfinite(st.z0) && isfinite(db) && isfinite(v[0]);
        st.done = !st.finite || st.z0 <= st.floor_ || st.z0 < a.bp.atol;
    }
    BScalars &s = a.sc[gr.x];
    const bool lead = g == gr.y && t == 0;
    if (lead) {
        s.alpha = s.beta = 0.0;
        s.ref = st.ref;
        s.floor_ = st.floor_;
        s.z0 = st.z0;
        s.replace = s.redirect = 0;
    }
    if (st.done) {
        if (lead) {
            s.rho = st.rho;
            s.znorm = st.z0;
            s.it = s.iters = s.failed = 0;
            s.nonfinite = st.finite ? 0 : 1;
            s.done = 1;
        }
        return;
    }
    const int h0 = a.map.halo_ptr[g], nh = (a.map.halo_ptr[g + 1] - h0) / HT;   // its passes
    float val[R][W], q[R], r[R], d[R];
    Rows<W, R, LQ> rows;
    rows.load(a.map.col, g, lcol);
    asm volatile("" ::: "memory");   // the columns' registers are free again
    int nq[R];   // quads of the wavefront's rows
#pragma unroll
    for (int i = 0; i < R; ++i)
        nq[i] = UNEVEN ? __builtin_amdgcn_readfirstlane(a.map.quads[(g * R + i) * OW + (t >> 6)]) : LQ;
    if constexpr (UNEVEN) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            load_values_n<W, R>(a.map.val32 + (size_t)g * own * (W + 1), val, i, nq[i]);
    } else {
        load_values<W, R>(a.map.val32 + (size_t)g * own * (W + 1), val);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = a.map.row[at0 + i * OB];
        const float ri = a.r32[max(row, 0)], dv = a.map.dinv32[at0 + i * OB];   // 0 past the last row
        r[i] = row < 0 ? 0.0f : ri;
        d[i] = 0.0f;
        ldv[i][t] = dv;
        win[i * OB + t] = dv * r[i];
    }
    float hdv[HR];   // D^-1 of the thread's halo entries
    if (t >= SLICE)
#pragma unroll
        for (int k = 0; k < HR; ++k)
            if (k < nh) {
                const int h = k * HT + t - SLICE, row = a.map.halo_row[h0 + h];
                hdv[k] = a.dinv32[row];
                win[own + h] = hdv[k] * a.r32[row];
            }
    int turn = a.turn[gr.x];
    __syncthreads();
    const StopTest test = {a.bp.atol, a.bp.rtol, st.ref, st.floor_};
    double rho = st.rho, znorm = st.z0;
    int it = 0;
    bool gave_up = false, nonfinite = false, failed = false;
    for (;;) {
        asm volatile("" : "+v"(at0), "+v"(t));   // as in k_onchip
        double pq[1] = {0.0};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            q[i] = rows.template product_as<UNEVEN>(a.lanes, val, lcol, i, t, win, nq[i]);
            formed(q[i]);
            pq[0] += (double)win[i * OB + t] * (double)q[i];
        }
        gave_up = !exchange<1>(pq, xl, team, turn, 0, nothing);
        if (gave_up) break;
        const float alpha = (float)(rho / pq[0]);
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            d[i] += alpha * win[i * OB + t];
            r[i] -= alpha * q[i];
            const float z = ldv[i][t] * r[i];
            st_agent(a.zb + at0 + i * OB, r[i]);
            v[0] += (double)r[i] * (double)z;
            v[1] += (double)z * (double)z;
        }
        Halo halo;
        gave_up = !exchange<2>(v, xl, team, turn, 0, [&] { halo.fetch<float>(a.map.halo_at + h0, nh); });
        if (gave_up) break;
        ++it;
        znorm = sqrt(v[1]);
        nonfinite = !isfinite(znorm) || !isfinite(v[0]);
        if (nonfinite) break;
        const bool pass = passes(test, znorm);
        if (!pass && !(a.bp.rr > 0 && it % a.bp.rr == 0) && it < a.bp.max_iter) {
            const float bf = (float)(v[0] / rho);
            rho = v[0];
#pragma unroll
            for (int i = 0; i < R; ++i)
                win[i * OB + t] = __builtin_fmaf(ldv[i][t], r[i], bf * win[i * OB + t]);
            halo.combine(a.zb, win + own, nh, [&](float rh, float p, int k) {
                return __builtin_fmaf(hdv[k], rh, bf * p);
            });
            __syncthreads();
            continue;
        }
        // ---- replacement: r64 -= A delta, x64 += delta, the test on r64 ----
        float p[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            p[i] = win[i * OB + t];
            win[i * OB + t] = d[i];
            st_agent(a.zb + at0 + i * OB, d[i]);
        }
        Ahead<R> row;
        double none[1] = {0.0};
        gave_up = !exchange<1>(none, xl, team, turn, 0, [&] {
            row.places(a.map.row + at0);
            row.read(a.r, a.x, a.dinv, 0);
        });
        if (gave_up) break;
        halo.fill(a.zb, win + own, nh);
        v[0] = v[1] = 0.0;
        const double2 *A = reinterpret_cast<const double2 *>(a.map.val64) + (size_t)g * (own * (W + 1) / 2) + t;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i + 1 < R) row.read(a.r, a.x, a.dinv, i + 1);
            double ad = rows.streamed(A, lcol, i, t, win, nq[i]);
            formed(ad);
            float ri = 0.0f;
            if (row.at[i] >= 0) {
                const double r64 = row.r[i] - ad;
                a.r[row.at[i]] = r64;
                a.x[row.at[i]] = row.x[i] + (double)d[i];
                ri = (float)r64;
                const double zi = row.d[i] * r64;
                v[1] += zi * zi;
            }
            r[i] = ri;
            d[i] = 0.0f;
            v[0] += (double)ri * (double)(ldv[i][t] * ri);
        }
        gave_up = !exchange<2>(v, xl, team, turn, 0, nothing);
        if (gave_up) break;
        znorm = sqrt(v[1]);
        nonfinite = !isfinite(znorm) || !isfinite(v[0]);
        if (nonfinite || passes(test, znorm)) break;
        if (it >= a.bp.max_iter) {
            failed = true;
            break;
        }
        // restart (p = z) where the recursive residual had passed, the
        // recurrence kept after a periodic replacement
        const float bf = (float)(pass ? 0.0 : v[0] / rho);
        rho = v[0];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float pi = __builtin_fmaf(ldv[i][t], r[i], bf * p[i]);
            win[i * OB + t] = pi;
            st_agent(a.zb + at0 + i * OB, pi);
        }
        gave_up = !exchange<1>(none, xl, team, turn, 0, nothing);
        if (gave_up) break;
        halo.fill(a.zb, win + own, nh);
    }
    if (gave_up) {
        if (t == 0) st_agent(&s.gave_up, 1);
        return;
    }
    if (lead) {
        s.rho = rho;
        s.znorm = znorm;
        s.it = s.iters = it;
        s.nonfinite = nonfinite ? 1 : 0;
        s.failed = failed ? 1 : 0;
        s.done = 1;
        a.turn[gr.x] = turn;
    }
}

// values and diagonals of the blocks' rows from the sliced layout
template <class T, class V>
__global__ __launch_bounds__(256) void k_onchip_values(int64_t n, int rows, int width, OnchipMap m,
                                                       const int64_t *__restrict__ slice_ptr,
                                                       const V *__restrict__ A,
                                                       const V *__restrict__ dinv,
                                                       T *__restrict__ val, T *__restrict__ dv)
{
    const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // block position
    if (at >= n) return;
    const int64_t pass = at / OB;   // g * rows + i
    const int t = (int)(at % OB);
    constexpr int L = 16 / sizeof(T);   // entries of a 16-byte load
    const int row = m.row[at];
    int w = 0;
    int64_t b0 = 0;
    if (row >= 0) {
        const int64_t sl = row / SLICE;
        b0 = slice_ptr[sl] + row % SLICE;
        w = (int)((slice_ptr[sl + 1] - slice_ptr[sl]) / SLICE);
    }
    for (int j = 0; j <= width; ++j)
        val[(pass * ((width + 1) / L) + j / L) * (OB * L) + t * L + j % L] =
            j < w ? (T)A[b0 + (int64_t)j * SLICE] : T(0);
    dv[at] = row >= 0 ? (T)dinv[row] : T(0);
}

struct OnchipShape {
    int width, rows;   // entries of a row, rows per thread
    void (*k)(OnchipSolve);
};
struct OnchipBatchShape {
    int width, rows;
    void (*k)(OnchipBatch);
};
// Every count of rows a thread from 1 on: a block's time goes with its count, and
// a mesh that needs 5 loses a sixth with 6.  The last count of each row length is
// the last whose block fits the LDS, with spills of at most 152 bytes a lane or,
// for 15 entries, r and the correction kept away (8 to 10 rows).  In FP64 the
// lists end earlier: 7 rows of 7 entries would fit (249 registers); 8 of 7, 5 of
// 15 and 3 of 31 would spill 44, 124 and 256 bytes.  None of these was timed.
// Above the last count the streaming kernels run, as for single meshes whose
// longest row has more than 31 entries and for batches beyond 39 (quads of
// columns and values in registers grow with the longest row of all; the batch's
// 39 pays for itself by forming only the quads that a wavefront's rows have).
#define MDX_OC(w, r) {w, r, k_onchip<w, r>}
const OnchipShape kShapes64[] = {
    MDX_OC(7, 1),  MDX_OC(7, 2),  MDX_OC(7, 3),  MDX_OC(7, 4),  MDX_OC(7, 5),  MDX_OC(7, 6),
    MDX_OC(15, 1), MDX_OC(15, 2), MDX_OC(15, 3), MDX_OC(15, 4), MDX_OC(31, 1), MDX_OC(31, 2),
};
#undef MDX_OC
#define MDX_OC(w, r) {w, r, k_onchip32<w, r, (w + 3) / 4, false>}
#define MDX_OC_AWAY(w, r) {w, r, k_onchip32<w, r, 3, true>}
const OnchipShape kShapes32[] = {
    MDX_OC(7, 1),       MDX_OC(7, 2),       MDX_OC(7, 3),        MDX_OC(7, 4),  MDX_OC(7, 5),
    MDX_OC(7, 6),       MDX_OC(7, 7),       MDX_OC(7, 8),        MDX_OC(7, 9),  MDX_OC(7, 10),
    MDX_OC(7, 11),      MDX_OC(7, 12),      MDX_OC(15, 1),       MDX_OC(15, 2), MDX_OC(15, 3),
    MDX_OC(15, 4),      MDX_OC(15, 5),      MDX_OC(15, 6),       MDX_OC(15, 7), MDX_OC_AWAY(15, 8),
    MDX_OC_AWAY(15, 9), MDX_OC_AWAY(15, 10), MDX_OC(31, 1),      MDX_OC(31, 2), MDX_OC(31, 3),
    MDX_OC(31, 4),
};
#undef MDX_OC_AWAY
#undef MDX_OC
#define MDX_OCB(w, r) {w, r, k_onchip_batch<w, r, (w > 15)>}
const OnchipBatchShape kShapesB[] = {
    MDX_OCB(7, 1),  MDX_OCB(7, 2),  MDX_OCB(7, 3),  MDX_OCB(7, 4),  MDX_OCB(7, 5),  MDX_OCB(7, 6),
    MDX_OCB(7, 7),  MDX_OCB(7, 8),  MDX_OCB(7, 9),  MDX_OCB(7, 10), MDX_OCB(7, 11), MDX_OCB(7, 12),
    MDX_OCB(15, 1), MDX_OCB(15, 2), MDX_OCB(15, 3), MDX_OCB(15, 4), MDX_OCB(15, 5), MDX_OCB(15, 6),
    MDX_OCB(15, 7), MDX_OCB(39, 1), MDX_OCB(39, 2), MDX_OCB(39, 3),
};
#undef MDX_OCB
constexpr int kMostRows = 12;

template <class S, int N>
const S *pick(const S (&s)[N], int width, int rows)
{
    for (const S &c : s)
        if (width == c.width && rows == c.rows) return &c;
    return nullptr;
}

}  // namespace

OnchipPlan onchip_plan(int device, int64_t n, int width)
{
    OnchipPlan p;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return p;
    p.xcd_cus = std::max(1, cus / NXCD);
    const int64_t cap = std::min(cus, kOnchipGroups);
    if (cap < 1 || n < 1) return p;
    p.width = width <= 7 ? 7 : width <= 15 ? 15 : 31;
    if (width > 31) return p;
    const int64_t need = (n + cap * OB - 1) / (cap * OB);
    if (need > kMostRows) return p;
    p.rows = (int)need;
    const OnchipShape *s[2] = {pick(kShapes64, p.width, p.rows), pick(kShapes32, p.width, p.rows)};
    for (int i = 0; i < 2; ++i) {
        int resident = 0;
        if (s[i] && hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, s[i]->k, OB, 0) == hipSuccess &&
            resident >= 1) {
            p.shape[i] = s[i];
            p.per_cu[i] = resident;
        }
    }
    if (p.shape[0] || p.shape[1]) p.groups = (int)std::min(cap, (n + OB - 1) / OB);
    p.first = {0, p.groups};
    return p;
}

OnchipPlan onchip_plan_batch(int device, const std::vector<int64_t> &n, int width)
{
    OnchipPlan p;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return p;
    p.xcd_cus = std::max(1, cus / NXCD);
    const int64_t cap = std::min(cus, kOnchipGroups);
    p.width = width <= 7 ? 7 : width <= 15 ? 15 : 39;
    if (width > 39 || (int64_t)n.size() > cap) return p;
    p.uneven = p.width == 39;
    // the fewest rows a thread with which every instance has workgroups enough
    for (int r = 1; r <= kMostRows; ++r) {
        int64_t need = 0;
        for (int64_t k : n) need += (k + r * OB - 1) / (r * OB);
        if (need > cap) continue;
        const OnchipBatchShape *s = pick(kShapesB, p.width, r);
        int resident = 0;
        if (!s || hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, s->k, OB, 0) != hipSuccess ||
            resident < 1)
            return p;
        p.rows = r;
        p.shape[2] = s;
        p.per_cu[2] = resident;
        for (int64_t k : n) {
            p.first.push_back(p.groups);
            p.groups += (int)((k + r * OB - 1) / (r * OB));
        }
        p.first.push_back(p.groups);
        return p;
    }
    return p;
}

void launch_onchip_values(hipStream_t s, const OnchipPlan &p, const OnchipMap &m,
                          const int64_t *slice_ptr, const double *A, const double *dinv,
                          const float *A32, const float *dinv32)
{
    const int64_t n = (int64_t)p.groups * p.rows * OB;
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (p.shape[0] || p.shape[2])
        hipLaunchKernelGGL((k_onchip_values<double, double>), grid, block, 0, s, n, p.rows, p.width, m,
                           slice_ptr, A, dinv, m.val64, m.dinv64);
    if (p.shape[1] || p.shape[2])
        hipLaunchKernelGGL((k_onchip_values<float, float>), grid, block, 0, s, n, p.rows, p.width, m,
                           slice_ptr, A32, dinv32, m.val32, m.dinv32);
}

void launch_onchip(hipStream_t s, const OnchipPlan &p, bool fp32, const OnchipSolve &a)
{
    const OnchipShape *sh = static_cast<const OnchipShape *>(p.shape[fp32 ? 1 : 0]);
    hipLaunchKernelGGL(sh->k, dim3(p.groups), dim3(OB), 0, s, a);
}

void launch_onchip_batch(hipStream_t s, const OnchipPlan &p, const OnchipBatch &a)
{
    const OnchipBatchShape *sh = static_cast<const OnchipBatchShape *>(p.shape[2]);
    hipLaunchKernelGGL(sh->k, dim3(p.groups), dim3(OB), 0, s, a);
}

}  // namespace mdx
