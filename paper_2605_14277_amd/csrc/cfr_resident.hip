// The resident loop: whole iterations of small and medium games inside one
// launch (layout and ownership: cfr_resident.h).
//
// What bounds it: a launch per step costs 2.3 to 7 us whatever it computes
// (dispatch, the cold first loads after a kernel boundary), eight to ten
// times an iteration.  Here a step between workgroups costs a barrier (0.8 us
// among 8 to 32 workgroups of one XCD, 2.3 us among 256), and an iteration
// has one or two of them per player; everything else is LDS and the payoff
// streams, which a workgroup reads from its own XCD's L2 or the last-level
// cache.  What is left is latency: about 0.6 us for each treeplex level on the
// way up (a chain of LDS accesses and a division), 1 to 2 us a product of a
// small game.  One iteration, launch per step against resident: 144 nonzeros
// 25.7 against 7.6 us; 4.9e4 (double) 42 / 18; 1.7e5 38 / 23; 1.3e6 with 9
// or 10 actions (double) 106 / 33; 3.4e6 (double) 73 / 54; 3.7e6 (float) 90 /
// 30; 9.7e6 (quads) 110 / 50.  The products of the larger ones run at 4 TB/s
// (16 waves a compute unit; 8: 28 instead of 20 us for both of the 3.4e6 game)
// and wait for their gathers, which fetch as many bytes again as the streams:
// vector instructions issue in 6 % of the waves' cycles.
#include "cfr_resident.h"

#include "cfr.h"

namespace cfr {

namespace {

template <int P>
struct Types;
template <>
struct Types<CFR_FP64> {
    using V = double;
    using R = double;
    using C = double;
};
template <>
struct Types<CFR_FP32> {
    using V = float;
    using R = float;
    using C = float;
};
template <>
struct Types<CFR_FP32_ACC64> {
    using V = float;
    using R = double;
    using C = double;
};

// Pointers into LDS that the compiler knows as such (a plain pointer that
// went through a structure becomes a flat access)
template <typename T>
using Lds = __attribute__((address_space(3))) T *;
// ... and into device memory, for those that come out of a structure there.
template <typename T>
using Gbl = __attribute__((address_space(1))) T *;
// ... and to what no launch changes: read with scalar loads where uniform.
template <typename T>
using Cst = __attribute__((address_space(4))) const T *;

// Exchanged values are read and written with relaxed agent-scope accesses:
// they go past the first-level cache and are coherent over the XCDs, so no
// cache is invalidated and the payoff streams stay where they are.
__device__ __forceinline__ float ag_load(const float *p)
{
    return __uint_as_float(__hip_atomic_load((Gbl<const uint32_t>)p, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ double ag_load(const double *p)
{
    return __longlong_as_double((long long)__hip_atomic_load((Gbl<const uint64_t>)p, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void ag_store(float *p, float v)
{
    __hip_atomic_store((Gbl<uint32_t>)p, __float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ag_store(double *p, double v)
{
    __hip_atomic_store((Gbl<uint64_t>)p, (uint64_t)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
// Four consecutive entries at a multiple of four.
__device__ __forceinline__ void ag_load4(const float *p, float (&o)[4])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint64_t t = __hip_atomic_load((Gbl<const uint64_t>)p + k, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        o[2 * k] = __uint_as_float((uint32_t)t);
        o[2 * k + 1] = __uint_as_float((uint32_t)(t >> 32));
    }
}
__device__ __forceinline__ void ag_load4(const double *p, double (&o)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = ag_load(p + k);
}
__device__ __forceinline__ uint32_t ag_load(const uint32_t *p)
{
    return __hip_atomic_load((Gbl<const uint32_t>)p, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until *p reaches target (as a wrapping counter).  Every wait ends:
// after kSpins polls (some ten seconds) it marks the team as failed, and a
// workgroup that finds the mark gives up too.
constexpr int kSpins = 1 << 24;
__device__ __forceinline__ bool bar_wait(const uint32_t *p, uint32_t target, uint32_t *failed)
{
    for (int i = 0; i < kSpins; ++i) {
        if ((int32_t)(ag_load(p) - target) >= 0) return true;
        if ((i & 1023) == 1023 && ag_load(failed)) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    __hip_atomic_store((Gbl<uint32_t>)failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// Counters of a team: [0] arrivals (of workgroups, or of groups), [16] the
// failure mark, [32] the barriers passed by earlier launches, [64 (g + 1)]
// arrivals of group g.  The counters only grow.
// One counter up to 64 workgroups, else one per group of every eighth (the
// group of an XCD) and one over the groups: 256 arrivals on one counter
// measured 3.9 us, in groups 2.3 us.
struct TeamBar {
    uint32_t *c;
    uint32_t n, rank, epoch;
    Lds<int> ok;
    int32_t *mark;  // the game's scalars: tells the host that the team failed

    // Every earlier store of every thread is complete before the workgroup
    // counts as arrived.
    __device__ __forceinline__ void arrive()
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ++epoch;
        if (n > 1 && threadIdx.x == 0) {
            if (n <= 64) {
                __hip_atomic_fetch_add((Gbl<uint32_t>)c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const uint32_t g = rank % kResXcds;
                const uint32_t m = (n - g + kResXcds - 1) / kResXcds;
                const uint32_t old = __hip_atomic_fetch_add((Gbl<uint32_t>)(c + 64 * (g + 1)), 1u, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                if (old + 1 == m * epoch)
                    __hip_atomic_fetch_add((Gbl<uint32_t>)c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    // Returns false when the team has failed.
    __device__ __forceinline__ bool wait()
    {
        if (n > 1 && threadIdx.x == 0) {
            *ok = bar_wait(c, (n <= 64 ? n : (uint32_t)kResXcds) * epoch, c + 16) ? 1 : 0;
            if (!*ok) *mark = 1;
        }
        __syncthreads();
        return *ok != 0;
    }
    __device__ __forceinline__ bool pass()
    {
        arrive();
        return wait();
    }
};

struct LdsScalars {
    double t, w, W, dpos, dneg;
    int ok;
};
static_assert(sizeof(LdsScalars) <= kResLdsHead, "fits the head of LDS");

// One player's LDS arrays (res_layout).
template <int P>
struct Part {
    Lds<typename Types<P>::R> r, s;
    Lds<typename Types<P>::C> v;
    Lds<typename Types<P>::V> g, b, x;
    Lds<int32_t> pub;
    Lds<uint16_t> kn, in, cp, pq;
    __device__ __forceinline__ Part(Lds<char> lds, const ResOff &o)
        : r((Lds<typename Types<P>::R>)(lds + o.r)), s((Lds<typename Types<P>::R>)(lds + o.s)),
          v((Lds<typename Types<P>::C>)(lds + o.v)), g((Lds<typename Types<P>::V>)(lds + o.g)),
          b((Lds<typename Types<P>::V>)(lds + o.b)), x((Lds<typename Types<P>::V>)(lds + o.x)),
          pub((Lds<int32_t>)(lds + o.pub)), kn((Lds<uint16_t>)(lds + o.kn)),
          in((Lds<uint16_t>)(lds + o.in)), cp((Lds<uint16_t>)(lds + o.cp)),
          pq((Lds<uint16_t>)(lds + o.pq))
    {
    }
};

// The regret minimiser's update, uniform over a workgroup.
template <int P>
struct Rule {
    typename Types<P>::C usign, dpos, dneg;
    bool floor, dcfr, pred;
    __device__ __forceinline__ typename Types<P>::C post(typename Types<P>::C r) const
    {
        if (floor) return r > 0 ? r : 0;
        if (dcfr) {
            if (r > 0) return r * dpos;
            if (r < 0) return r * dneg;
        }
        return r;
    }
};

// The decision points of one group, a lane per sequence: counterfactual
// values, regret update and regret matching from LDS.  A decision point's
// sums are taken by each of its lanes from the wave's staging (which the LDS
// serves in order), in the order of its actions, so the operations and their
// order are those of the launch-per-level kernels (up_infoset) and every
// result is the same bit for bit.  A thread per decision point, with its
// actions one after another, took 640 instructions a level, 0.9 us of a
// lone wave; this takes about 170.  Returns the decision point's value.  m: the
// player's predictions (of the last iteration: nothing reads them in
// between), kept at its sequences gs, or null.
template <int P>
__device__ __forceinline__ typename Types<P>::C res_up(const Part<P> &t, int a, int lane, int k,
                                                       int n, const Rule<P> &ru,
                                                       Lds<typename Types<P>::C> st,
                                                       typename Types<P>::R *m, Cst<int32_t> gs)
{
    using V = typename Types<P>::V;
    using R = typename Types<P>::R;
    using C = typename Types<P>::C;
    constexpr int N = 4;
    const int first = lane - k;
    // a decision point's terms in order; lanes past n take the first
    auto sum = [&]() __attribute__((always_inline)) {
        C acc = 0;
        for (int i = 0; i < n; i += N) {
            C w[N];
#pragma unroll
            for (int j = 0; j < N; ++j) w[j] = st[first + (i + j < n ? i + j : 0)];
#pragma unroll
            for (int j = 0; j < N; ++j) acc = i + j < n ? acc + w[j] : acc;
        }
        return acc;
    };
    const C bv = (C)t.b[a], rv = (C)t.r[a];
    C q = ru.usign * (C)t.g[a];
    const int c1 = t.cp[a + 1];
    for (int c = t.cp[a]; c < c1; c += N) {
        C kv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) kv[i] = t.v[c + i < c1 ? c + i : c];
#pragma unroll
        for (int i = 0; i < N; ++i) q = c + i < c1 ? q + kv[i] : q;
    }
    st[lane] = bv * q;
    __builtin_amdgcn_wave_barrier();
    const C V_ = sum();
    const C inst = q - V_;
    const C rr = ru.post(rv + inst);
    t.r[a] = (R)rr;
    C zz = (C)(R)rr;
    if (ru.pred) {
        if (m) m[gs[a]] = (R)inst;
        zz = zz + (C)(R)inst;
    }
    zz = zz > 0 ? zz : 0;
    __builtin_amdgcn_wave_barrier();
    st[lane] = zz;
    __builtin_amdgcn_wave_barrier();
    const C Z = sum();
    const C num = Z > 0 ? zz : (C)1, den = Z > 0 ? Z : (C)n;
    t.b[a] = (V)(num / den);
    __builtin_amdgcn_wave_barrier();
    return V_;
}

__device__ __forceinline__ float fetch(const float *p) { return ag_load(p); }
__device__ __forceinline__ double fetch(const double *p) { return ag_load(p); }
__device__ __forceinline__ float fetch(Lds<float> p) { return *p; }
__device__ __forceinline__ double fetch(Lds<double> p) { return *p; }

// A lane's U elements of a chunk, 64 apart (lanes past the end take the
// first one).  Products are rounded to the value type, as k_spmv stages them.
template <int P, typename X, int U>
struct Elements {
    using V = typename Types<P>::V;
    using C = typename Types<P>::C;
    uint32_t ci[U];
    V vi[U], xv[U];
    __device__ __forceinline__ void load(Gbl<const char> idx, Gbl<const char> val, int off, int n,
                                         int lane)
    {
        const Gbl<const char> ip = idx + 4 * (int64_t)off, vp = val + sizeof(V) * (int64_t)off;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t k = 64 * j + lane < n ? 64 * j + lane : 0;
            ci[j] = *(Gbl<const uint32_t>)(ip + 4 * k);
            vi[j] = *(Gbl<const V>)(vp + (uint32_t)sizeof(V) * k);
        }
    }
    __device__ __forceinline__ void gather(X x)
    {
#pragma unroll
        for (int j = 0; j < U; ++j) xv[j] = fetch(x + ci[j]);
    }
    __device__ __forceinline__ V product(int j) const { return (V)((C)vi[j] * (C)xv[j]); }
};

// The same with quads: the present positions of a quad added in order.
template <int P, int U>
struct Quads {
    using V = typename Types<P>::V;
    using C = typename Types<P>::C;
    typedef V V4 __attribute__((ext_vector_type(4)));
    uint32_t ci[U];
    V4 vi[U];
    V xv[U][4];
    __device__ __forceinline__ void load(Gbl<const char> idx, Gbl<const char> val, int off, int n,
                                         int lane)
    {
        const Gbl<const char> ip = idx + 4 * (int64_t)off, vp = val + 4 * sizeof(V) * (int64_t)off;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t k = 64 * j + lane < n ? 64 * j + lane : 0;
            ci[j] = *(Gbl<const uint32_t>)(ip + 4 * k);
            vi[j] = *(Gbl<const V4>)(vp + (uint32_t)(4 * sizeof(V)) * k);
        }
    }
    __device__ __forceinline__ void gather(const V *x)
    {
#pragma unroll
        for (int j = 0; j < U; ++j) ag_load4(x + 4 * (ci[j] & kQuadIndexMask), xv[j]);
    }
    __device__ __forceinline__ V product(int j) const
    {
        C qs = (C)(-0.0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((ci[j] >> (kQuadMaskShift + e)) & 1u) qs = qs + (C)vi[j][e] * (C)xv[j][e];
        return (V)qs;
    }
};

// The payoff rows of one workgroup's sequences: a wave takes every
// NW-th chunk, stages its products in its own part of LDS (which
// serves one wave's accesses in order, so no barrier is needed) and sums the
// rows from there in the order of k_spmv: 1 << lr lanes a row, each its
// products in order, then across the lanes.  Consecutive lanes take
// consecutive elements of a row, whose columns lie close together.
template <int P, int NT, int U, typename E, typename X>
__device__ __forceinline__ void res_product(Cst<ResTeam> T, int w, Cst<ResPart> q, X x,
                                            Lds<typename Types<P>::V> g,
                                            Lds<typename Types<P>::V> st)
{
    using V = typename Types<P>::V;
    using C = typename Types<P>::C;
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Cst<ResChunk> chunks = (Cst<ResChunk>)T->chunk + q->c0;
    const Gbl<const char> idx = (Gbl<const char>)T->idx[w], val = (Gbl<const char>)T->val[w];
    const Gbl<const uint32_t> row_of = (Gbl<const uint32_t>)T->row;
    V *const gx = (V *)T->gx[w];
    const int nc = q->nc, nq = q->nq;
    if (wave >= nc) return;
    // the next piece's streams and the next chunk's rows are in flight while
    // a piece is summed
    E e;
    e.load(idx, val, chunks[wave].off, chunks[wave].n, lane);
    int off = chunks[wave].off, n = chunks[wave].n, rows_lr = chunks[wave].rows_lr;
    uint32_t meta = (uint32_t)chunks[wave].meta, m0 = 0, m1 = 0;
    auto rows_of = [&](int row, int rows) __attribute__((always_inline)) {
        const uint32_t at = meta + (uint32_t)(row < rows ? row : rows - 1);
        m0 = row_of[at];
        m1 = row_of[at + 1];
    };
    rows_of(lane >> (rows_lr >> 16), rows_lr & 0xffff);
    for (int c = wave; c < nc; c += NW) {
        const int rows = rows_lr & 0xffff, lr = rows_lr >> 16;
        const int sub = lane & ((1 << lr) - 1), per = 64 >> lr;
        C acc = 0;
        // one piece, unless the chunk is one row longer than a piece
        for (int done = 0;; done += 64 * U) {
            const int left = n - done;
            int row = lane >> lr;
            e.gather(x);
#pragma unroll
            for (int j = 0; j < U; ++j) st[64 * j + lane] = e.product(j);
            const int cn = c + NW;
            if (left > 64 * U) e.load(idx, val, off + done + 64 * U, left - 64 * U, lane);
            else if (cn < nc) e.load(idx, val, chunks[cn].off, chunks[cn].n, lane);
            __builtin_amdgcn_wave_barrier();
            for (int r0 = 0;;) {
                if (row < rows) {
                    int i = (rows == 1 ? 0 : (int)(m0 >> 16)) + sub;
                    const int z = rows == 1 ? (left < 64 * U ? left : 64 * U) : (int)(m1 >> 16);
                    constexpr int N = 8;
                    const int s = 1 << lr;
                    for (; i + (N - 1) * s < z; i += N * s) {
                        V pr[N];
#pragma unroll
                        for (int j = 0; j < N; ++j) pr[j] = st[i + j * s];
#pragma unroll
                        for (int j = 0; j < N; ++j) acc = acc + (C)pr[j];
                    }
                    if (i < z) {
                        V pr[N - 1];
#pragma unroll
                        for (int j = 0; j < N - 1; ++j) pr[j] = st[i + j * s < z ? i + j * s : i];
#pragma unroll
                        for (int j = 0; j < N - 1; ++j) acc = i + j * s < z ? acc + (C)pr[j] : acc;
                    }
                }
                if (left > 64 * U) break;
                for (int o = (1 << lr) >> 1; o > 0; o >>= 1) acc = acc + __shfl_xor(acc, o, 1 << lr);
                if (sub == 0 && row < rows) {
                    const int dest = (int)(m0 & 0xffffu);
                    if (dest < nq) g[dest] = (V)acc;
                    else ag_store(gx + (dest - nq), (V)acc);
                }
                r0 += per;
                if (r0 >= rows) break;
                row += per;
                acc = 0;
                rows_of(row, rows);
            }
            __builtin_amdgcn_wave_barrier();
            if (left <= 64 * U) {
                if (cn < nc) {
                    off = chunks[cn].off;
                    n = chunks[cn].n;
                    rows_lr = chunks[cn].rows_lr;
                    meta = (uint32_t)chunks[cn].meta;
                    rows_of(lane >> (rows_lr >> 16), rows_lr & 0xffff);
                }
                break;
            }
        }
    }
}

// The iteration's scalars (begin_iteration of cfr_kernels.hip).  Out of line:
// its pow calls are as long as the rest of an iteration's code.
__device__ __noinline__ void res_begin(Lds<LdsScalars> ls, const Scalars *gs, int kind, bool factors)
{
    const double t = ls->t + 1.0;
    ls->t = t;
    double w = 1.0;
    if (kind == CFR_AVG_LINEAR) w = t;
    else if (kind == CFR_AVG_QUADRATIC) w = t * t;
    else if (kind == CFR_AVG_POW_GAMMA) w = pow(t, gs->gamma);
    ls->w = w;
    ls->W = ls->W + w;
    if (factors) {
        const double ta = pow(t, gs->alpha), tb = pow(t, gs->beta);
        ls->dpos = ta / (ta + 1.0);
        ls->dneg = tb / (tb + 1.0);
    }
}

// Code that runs once an iteration is fetched once an iteration: it is kept
// small (one copy for both players) to stay in the instruction cache.
template <int P, int NT>
__global__ __launch_bounds__(NT) void k_resident(const ResTeam *__restrict__ teams,
                                                          const int32_t *__restrict__ map, int n,
                                                          int mode, Scalars *sc, DevPlayer d0,
                                                          DevPlayer d1)
{
    using V = typename Types<P>::V;
    using R = typename Types<P>::R;
    using C = typename Types<P>::C;
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) char lds[];
    const int32_t who = ((Cst<int32_t>)map)[blockIdx.x];
    if (who < 0) return;
    const Cst<ResTeam> T = (Cst<ResTeam>)teams + (who & 0xffff);
    const int rank = who >> 16;
    const Cst<int32_t> i32 = (Cst<int32_t>)T->i32;
    const Cst<uint16_t> u16 = (Cst<uint16_t>)T->u16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Cst<ResPart> pt = (Cst<ResPart>)T->part + 2 * (int64_t)rank;
    ResOff o0, o1;
    const uint32_t end = res_layout((Cst<ResShallow>)T->sh, pt, sizeof(V), sizeof(R), sizeof(C),
                                    T->lean, o0, o1);
    const Lds<char> base = (Lds<char>)lds;
    const Lds<char> stage = base + (end + kResStage * (threadIdx.x >> 6));  // the wave's
    const Lds<LdsScalars> ls = (Lds<LdsScalars>)base;
    Scalars *gs = sc + T->slot;
    TeamBar bar{T->bar, (uint32_t)T->blocks, (uint32_t)rank, T->bar[32], (Lds<int>)&ls->ok, gs->pad};
    const bool lean = T->lean != 0;
    // a player's arrays (p is uniform: the offsets are selected as scalars)
    auto part = [&](int p) __attribute__((always_inline)) {
        ResOff o;
        o.r = p ? o1.r : o0.r;
        o.s = p ? o1.s : o0.s;
        o.v = p ? o1.v : o0.v;
        o.g = p ? o1.g : o0.g;
        o.b = p ? o1.b : o0.b;
        o.x = p ? o1.x : o0.x;
        o.pub = p ? o1.pub : o0.pub;
        o.kn = p ? o1.kn : o0.kn;
        o.in = p ? o1.in : o0.in;
        o.cp = p ? o1.cp : o0.cp;
        o.pq = p ? o1.pq : o0.pq;
        return Part<P>(base, o);
    };
    // global sequence of a local one (own, then shallow)
    auto global = [&](int p, int k) __attribute__((always_inline)) {
        const int nq = pt[p].nq;
        return (int64_t)(k < nq ? i32[pt[p].gs + k] : i32[T->sh[p].gs + k - nq]);
    };

    // structure and state into LDS
    for (int p = 0; p < 2; ++p) {
        const R *dr = (const R *)(p ? d1.r : d0.r), *ds = (const R *)(p ? d1.s : d0.s);
        const V *db = (const V *)(p ? d1.b : d0.b), *dx = (const V *)(p ? d1.x : d0.x);
        const int32_t *pos = p ? d1.pos : d0.pos;
        const Cst<ResPart> q = pt + p;
        const Cst<ResShallow> h = (Cst<ResShallow>)T->sh + p;
        const Part<P> t = part(p);
        const int nq = q->nq, ni = q->ni, all = nq + h->nq;
        for (int i = tid; i <= nq; i += NT) t.cp[i] = u16[q->cp + i];
        for (int i = tid; i < nq; i += NT) {
            t.kn[i] = u16[q->kn + i];
            t.in[i] = u16[q->in + i];
            t.pq[i] = (uint16_t)(u16[q->pq + i] + (h->c > 0 && i > 0 && i < q->first_q ? nq : 0));
        }
        if (h->c > 0) {
            for (int i = 1 + tid; i <= h->nq; i += NT)
                t.cp[nq + i] = (uint16_t)(u16[h->cp + i] + ni);
            for (int i = tid; i < h->nq; i += NT) {
                t.kn[nq + i] = u16[h->kn + i];
                t.in[nq + i] = (uint16_t)(u16[h->in + i] + ni);
                t.pq[nq + i] = (uint16_t)(u16[h->pq + i] + nq);
            }
        }
        for (int k = tid; k < all; k += NT) {
            const int64_t a = global(p, k);
            const bool empty = k == 0 || k == nq;
            t.r[k] = dr[a];
            if (!lean) {
                t.s[k] = ds[a];
                t.x[k] = empty ? (V)1 : ag_load(dx + a);
            }
            t.b[k] = empty ? (V)1 : db[a];
            t.g[k] = 0;
            t.pub[k] = T->pub[p] == 2 ? pos[a] : (int32_t)a;
        }
    }
    const int variant = gs->variant;
    int kind = gs->avg_kind;
    if (kind == CFR_AVG_DEFAULT)
        kind = variant == CFR_PLUS        ? CFR_AVG_LINEAR
               : variant == CFR_DCFR      ? CFR_AVG_POW_GAMMA
               : variant == CFR_PCFR_PLUS ? CFR_AVG_QUADRATIC
                                          : CFR_AVG_UNIFORM;
    if (tid == 0) {
        ls->t = gs->t;
        ls->W = gs->W;
        ls->ok = 1;
    }
    __syncthreads();

    // Where the gatherers of a player's strategy read it.
    auto target = [&](int p) __attribute__((always_inline)) {
        V *const x = (V *)(p ? d1.x : d0.x), *const xp = (V *)(p ? d1.xp : d0.xp);
        return T->pub[p] == 2 ? xp : x;
    };
    if (T->pub[0] == 2 || T->pub[1] == 2) {
        // the permuted copy is not kept current between launches
        for (int p = 0; p < 2; ++p) {
            if (T->pub[p] != 2) continue;
            const Part<P> t = part(p);
            const int nq = pt[p].nq, all = nq + (rank == 0 ? T->sh[p].nq : 0);
            for (int k = tid; k < all; k += NT)
                if (k > 0 || rank == 0) {
                    const V *dx = (const V *)(p ? d1.x : d0.x);
                    ag_store(target(p) + t.pub[k], ag_load(dx + global(p, k)));
                }
        }
        if (!bar.pass()) return;
    }

    // A team that has failed stays so: its counters hold what was left of the
    // launch that did, and no later wait on them means anything.  (Nothing of
    // the state is written before this; earlier in the kernel, or read through
    // LDS, the same test cost 0.7 % of every iteration by its code's place.)
    if (bar.n > 1 && ((Cst<uint32_t>)bar.c)[16]) {
        if (tid == 0) *bar.mark = 1;
        return;
    }
    Rule<P> ru;
    ru.floor = variant == CFR_PLUS || variant == CFR_PCFR_PLUS;
    ru.dcfr = variant == CFR_DCFR;
    ru.pred = variant == CFR_PCFR || variant == CFR_PCFR_PLUS;
    ru.dpos = ru.dneg = (C)1;

    // ObserveUtility on the levels of a player's own part, or of its shallow
    // part, deepest first, a wave to a group (q0: the part's first sequence).
    // The cut level's values go to the other workgroups.
    auto up = [&](int p, const Part<P> &t, int levels, int lev, int grp, int q0, bool own, R *m,
                  Cst<int32_t> seq) __attribute__((always_inline)) {
        ru.usign = p == 0 ? (C)1 : (C)-1;
        if (ru.dcfr) {
            ru.dpos = (C)ls->dpos;
            ru.dneg = (C)ls->dneg;
        }
        C *const cut = own && T->sh[p].c > 0 ? (C *)T->cutv[p] : nullptr;
        const int cut_at = pt[p].cut;
        int hi = i32[lev + levels];
        for (int L = levels - 1; L >= 0; --L) {
            const int lo = i32[lev + L];
            for (int g = lo + wave; g < hi; g += NW) {
                const int a = i32[grp + g] + q0 + lane;
                if (a < i32[grp + g + 1] + q0) {
                    const int kn = t.kn[a], k = kn & 255;
                    const C v = res_up<P>(t, a, lane, k, kn >> 8, ru, (Lds<C>)stage, m, seq);
                    if (k == 0) {
                        const int i = t.in[a];
                        if (L > 0 || !own) t.v[i] = v;
                        else if (cut) ag_store(cut + i32[cut_at + i], v);
                    }
                }
            }
            hi = lo;
            __syncthreads();
        }
    };

    const bool both = mode == CFR_SIMULTANEOUS;
    for (int it = 0; it < n; ++it) {
        const bool last = it == n - 1;
        // by a thread of the last wave (which has the fewest chunks), while
        // the products run
        if (tid == NT - 1) res_begin(ls, gs, kind, ru.dcfr || last);
        // alternating: player 1's turn, then player 2's; simultaneous: one
        // turn of both
        for (int turn = 0; turn < (both ? 1 : 2); ++turn) {
            const int p0 = both ? 0 : turn, p1 = both ? 2 : turn + 1;
            for (int p = p0; p < p1; ++p) {
                const Lds<V> g = part(p).g, st = (Lds<V>)stage;
                const V *const x = target(1 - p) + T->seq0[1 - p];
                constexpr int U = res_rounds(sizeof(V), false), UQ = res_rounds(sizeof(V), true);
                if (T->quads[p])
                    res_product<P, NT, UQ, Quads<P, UQ>>(T, p, pt + p, x, g, st);
                else if (T->pub[1 - p] == 0)
                    res_product<P, NT, U, Elements<P, Lds<V>, U>>(T, p, pt + p, part(1 - p).x, g, st);
                else
                    res_product<P, NT, U, Elements<P, const V *, U>>(T, p, pt + p, x, g, st);
            }
            __syncthreads();
            bool exchange = both;
            for (int p = p0; p < p1; ++p) {
                R *const m = last && ru.pred ? (R *)(p ? d1.m : d0.m) : nullptr;
                up(p, part(p), pt[p].nlev, pt[p].lev, pt[p].grp, 0, true, m, i32 + pt[p].gs);
                exchange = exchange || T->sh[p].c > 0;
            }
            // simultaneous: the strategies are overwritten only once every
            // workgroup has read them
            if (exchange) bar.arrive();
            // the average of the strategy that is overwritten next, which
            // needs nothing from the others; rank 0 does the shallow part's
            for (int p = p0; p < p1; ++p) {
                const Part<P> t = part(p);
                const R w = (R)ls->w;
                R *const ds = (R *)(p ? d1.s : d0.s);
                const int nq = pt[p].nq, all = nq + (rank == 0 ? T->sh[p].nq : 0);
                const V *const out = target(p);
                if (!lean) {
                    for (int k = 1 + tid; k < all; k += NT)
                        if (k != nq) t.s[k] = t.s[k] + w * (R)t.x[k];
                    continue;
                }
                // (past the end: the workgroup's own empty sequence, skipped)
                constexpr int N = 4;
                for (int k0 = 1 + tid; k0 < all; k0 += N * NT) {
                    int64_t a[N];
                    R s[N];
                    V xo[N];
#pragma unroll
                    for (int j = 0; j < N; ++j) a[j] = global(p, k0 + j * NT < all ? k0 + j * NT : 0);
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        s[j] = ds[a[j]];
                        xo[j] = ag_load(out + t.pub[k0 + j * NT < all ? k0 + j * NT : 0]);
                    }
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        const int k = k0 + j * NT;
                        if (k < all && k != nq) ds[a[j]] = s[j] + w * (R)xo[j];
                    }
                }
            }
            if (!exchange) __syncthreads();
            else if (!bar.wait()) return;
            // the shallow levels, computed alike by every workgroup
            for (int p = p0; p < p1; ++p) {
                const Cst<ResShallow> h = (Cst<ResShallow>)T->sh + p;
                if (h->c == 0) continue;
                const Part<P> t = part(p);
                const int nq = pt[p].nq, ni = pt[p].ni;
                const C *const cut = (const C *)T->cutv[p];
                const V *const gx = (const V *)T->gx[p];
                for (int i = tid; i < h->ncut; i += NT)
                    t.v[ni + h->ni + i] = ag_load(cut + i);
                for (int i = tid; i < h->nq; i += NT) t.g[nq + i] = ag_load(gx + i);
                __syncthreads();
                R *const m = last && ru.pred && rank == 0 ? (R *)(p ? d1.m : d0.m) : nullptr;
                up(p, t, h->c, h->lev, h->grp, nq, false, m, i32 + (h->gs - nq));
            }
            // NextStrategy's top-down pass: each sequence multiplies its chain
            // of behavioural strategies from the root down, as k_down_all
            // does; the shallow ones' strategies are rank 0's to write
            for (int p = p0; p < p1; ++p) {
                const Part<P> t = part(p);
                const Cst<ResShallow> h = (Cst<ResShallow>)T->sh + p;
                const int nq = pt[p].nq, all = nq + (rank == 0 ? h->nq : 0);
                const int depth = h->c + pt[p].nlev;
                const bool publish = T->pub[p] != 0;
                V *const out = target(p);
                for (int k = 1 + tid; k < all; k += NT) {
                    if (k == nq) continue;
                    // past the top the chain stays at the empty sequence,
                    // whose factor is exactly 1
                    V chain[kDownAllMaxDepth];
                    int u = k;
#pragma unroll
                    for (int i = 0; i < kDownAllMaxDepth; ++i) {
                        if (i >= depth) break;
                        chain[i] = t.b[u];
                        u = t.pq[u];
                    }
                    V xv = (V)1;
#pragma unroll
                    for (int i = kDownAllMaxDepth - 1; i >= 0; --i)
                        if (i < depth) xv = xv * chain[i];
                    if (!lean) t.x[k] = xv;
                    if (publish) ag_store(out + t.pub[k], xv);
                }
            }
            if (!bar.pass()) return;
        }
    }

    // state back to device memory
    for (int p = 0; p < 2; ++p) {
        R *dr = (R *)(p ? d1.r : d0.r), *ds = (R *)(p ? d1.s : d0.s);
        V *db = (V *)(p ? d1.b : d0.b), *dx = (V *)(p ? d1.x : d0.x);
        const Part<P> t = part(p);
        const int nq = pt[p].nq, all = nq + (rank == 0 ? T->sh[p].nq : 0);
        for (int k = 1 + tid; k < all; k += NT) {
            if (k == nq) continue;
            const int64_t a = global(p, k);
            dr[a] = t.r[k];
            if (!lean) ds[a] = t.s[k];
            db[a] = t.b[k];
            dx[a] = lean ? ag_load(target(p) + t.pub[k]) : t.x[k];
        }
    }
    if (rank == 0 && tid == 0) {
        gs->t = ls->t;
        gs->w = ls->w;
        gs->W = ls->W;
        gs->dpos = ls->dpos;
        gs->dneg = ls->dneg;
        T->bar[32] = bar.epoch;
    }
}

// Fills one product's streams: one wave per chunk.  Columns lose the gathered
// player's first sequence, col0 (a multiple of four).  A team of one workgroup
// gathers elements from LDS, by local (not null): the local sequence of the
// game's column, after unperm (or null: the gathered player's sequence of each
// permuted column).
template <int P, bool QUADS>
__global__ __launch_bounds__(256) void k_res_fill(int nc, const ResChunk *__restrict__ chunk,
                                                  const uint32_t *__restrict__ row,
                                                  const int32_t *__restrict__ src,
                                                  const int32_t *__restrict__ idx,
                                                  const typename Types<P>::V *__restrict__ val,
                                                  int64_t base, const int32_t *__restrict__ unperm,
                                                  const int32_t *__restrict__ local, int32_t col0,
                                                  int32_t *__restrict__ out_idx,
                                                  typename Types<P>::V *__restrict__ out_val)
{
    const int c = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (c >= nc) return;
    const int lane = threadIdx.x & 63;
    const ResChunk ch = chunk[c];
    const int rows = ch.rows_lr & 0xffff;
    for (int r = 0; r < rows; ++r) {
        const int s0 = (int)(row[ch.meta + r] >> 16);
        const int s1 = r + 1 < rows ? (int)(row[ch.meta + r + 1] >> 16) : ch.n;
        const int64_t e0 = base + src[ch.meta + r];
        for (int k = lane; k < s1 - s0; k += 64) {
            const int64_t o = (int64_t)ch.off + s0 + k, e = e0 + k;
            int32_t col = idx[e];
            if (QUADS) {
                for (int j = 0; j < 4; ++j) out_val[4 * o + j] = val[4 * e + j];
                col -= col0 / 4;
            } else {
                col = local ? local[(unperm ? unperm[col] : col) - col0] : col - col0;
                out_val[o] = val[e];
            }
            out_idx[o] = col;
        }
    }
}

template <int P>
hipError_t res_fill_t(bool quads, int nc, const ResChunk *chunk, const uint32_t *row,
                      const int32_t *src, const int32_t *idx, const void *val, int64_t base,
                      const int32_t *unperm, const int32_t *local, int32_t col0, int32_t *out_idx,
                      void *out_val, hipStream_t st)
{
    using V = typename Types<P>::V;
    if (nc == 0) return hipSuccess;
    const dim3 grid((unsigned)((nc + 3) / 4));
    if (quads)
        hipLaunchKernelGGL((k_res_fill<P, true>), grid, dim3(256), 0, st, nc, chunk, row, src, idx,
                           (const V *)val, base, unperm, local, col0, out_idx, (V *)out_val);
    else
        hipLaunchKernelGGL((k_res_fill<P, false>), grid, dim3(256), 0, st, nc, chunk, row, src, idx,
                           (const V *)val, base, unperm, local, col0, out_idx, (V *)out_val);
    return hipGetLastError();
}

template <int P, int NT>
hipError_t resident_t(const ResTeam *teams, const int32_t *map, int grid, uint32_t lds,
                      bool cooperative, int n, int mode, Scalars *sc, const DevPlayer &p0,
                      const DevPlayer &p1, hipStream_t st)
{
    hipError_t e = hipFuncSetAttribute((const void *)k_resident<P, NT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
    if (e != hipSuccess) return e;
    if (!cooperative) {
        hipLaunchKernelGGL((k_resident<P, NT>), dim3((unsigned)grid), dim3(NT), lds, st, teams, map,
                           n, mode, sc, p0, p1);
        return hipGetLastError();
    }
    DevPlayer a = p0, b = p1;
    void *args[] = {&teams, &map, &n, &mode, &sc, &a, &b};
    return hipLaunchCooperativeKernel((const void *)k_resident<P, NT>, dim3((unsigned)grid),
                                      dim3(NT), args, lds, st);
}

}  // namespace

#define CFR_RES_DISPATCH(prec, call)                               \
    switch (prec) {                                                \
    case CFR_FP64: { constexpr int P = CFR_FP64; return call; }    \
    case CFR_FP32: { constexpr int P = CFR_FP32; return call; }    \
    case CFR_FP32_ACC64: { constexpr int P = CFR_FP32_ACC64; return call; } \
    default: return hipErrorInvalidValue;                          \
    }

hipError_t launch_res_fill(int prec, bool quads, int n_chunk, const ResChunk *chunk,
                           const uint32_t *row, const int32_t *src, const int32_t *idx,
                           const void *val, int64_t base, const int32_t *unperm,
                           const int32_t *local, int32_t col0, int32_t *out_idx, void *out_val,
                           hipStream_t st)
{
    CFR_RES_DISPATCH(prec, res_fill_t<P>(quads, n_chunk, chunk, row, src, idx, val, base, unperm,
                                         local, col0, out_idx, out_val, st));
}

hipError_t launch_resident(int prec, const ResTeam *teams, const int32_t *map, int grid,
                           uint32_t lds, int threads, bool cooperative, int n, int mode,
                           Scalars *sc, const DevPlayer &p0, const DevPlayer &p1, hipStream_t st)
{
    lds += (uint32_t)threads / 64 * kResStage;
    if (threads == 256 && !cooperative)
        CFR_RES_DISPATCH(prec, (resident_t<P, 256>(teams, map, grid, lds, false, n, mode, sc, p0,
                                                   p1, st)));
    if (threads == kResThreadsMax)
        CFR_RES_DISPATCH(prec, (resident_t<P, kResThreadsMax>(teams, map, grid, lds, cooperative, n,
                                                              mode, sc, p0, p1, st)));
    return hipErrorInvalidValue;
}

}  // namespace cfr
