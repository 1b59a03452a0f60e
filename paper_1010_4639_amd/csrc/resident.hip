// A whole conjugate-gradient solve of a small system in one kernel: the
// matrix stays in registers, the search direction in LDS, x and r in
// registers, and the workgroups -- all resident at once -- exchange only the
// two scalar products of an iteration and the residual entries that their
// neighbours need.
//
// The arithmetic is the two-kernel iteration's (kernels.hip, IterCtx::fused)
// operation by operation and in the same order of every sum, so a solve gives
// the same bits either way, and a solve that cannot be resident (another one
// holds the compute units, a wait ran out) takes the launches instead.
//
// The launches' reductions are over "product workgroups" (four slices: a sum
// of p'q each) and "vector workgroups" (`chunk` rows: a sum of r'r each).
// Workgroup b of G here stands for a contiguous run of product workgroups --
// S slices per wavefront, a row per lane -- and for one vector workgroup per
// 256 of its T threads: T = 256, S = 1 up to 65 536 rows, T = 512 and S = 1 or
// 2 up to 262 144.  Its product rows and its vector rows differ at their ends,
// and the product sums in the difference are exchanged.  `gcol` lists every
// column that the product rows touch (the rows themselves among them); pl[]
// in LDS holds p at those columns, and each workgroup advances its own copy,
// p = r + beta p.
//
// Exchange: everything another workgroup needs -- a workgroup's share of a
// sum, a residual entry, a product sum -- is one 8-byte word, written once
// with an agent-scope store and polled until it leaves the "empty" pattern, so
// no word has to be ordered after another.  The first wavefront (or two)
// publishes and polls the sums while the others poll the residual entries of
// their columns.  The words rotate over kRing rounds: writing
// round k a workgroup empties its word of round k + 2 (= k - 2: whoever read
// that has published a later sum, which this workgroup has seen), and waits
// for these stores before it publishes anything of the next round, which
// every reader of round k + 2 has seen by then.
//
// Latency bounds it: two exchanges of about 1.7 us (a store to memory and a
// poll from it) and the steps between them, and at the largest sizes the words
// of the residual (about 2800 columns a workgroup).  Iteration, launches /
// here: 4096 rows 8.1 / 3.9 us, 30 720 8.5 / 4.9, 62 400 8.7 / 5.8, 125 000
// 10.2 / 6.6, 205 143 13.4 / 9.7, 262 144 16.2 / 9.3.  With the residual
// entries behind the sums (stores completed, then the sum published, then the
// entries loaded) 30 720 rows took 6.5 and 62 400 9.0; with agent-scope fences
// around each sum (an L2 write-back and invalidation per wavefront) the sums
// alone take 18 us on 256 workgroups.
//
// Every wait ends: a poll gives up after `wait` ticks or when another
// workgroup did, and the host then repeats the solve with launches.
#include "kernels.h"
#include "devutil.h"

#include <hip/hip_runtime.h>

namespace cgmi {

namespace {

using namespace dev;

typedef unsigned long long u64;
constexpr u64 kEmpty = ~0ull;
constexpr int kRing = kResidentRing;
__device__ __forceinline__ u64 agent_load(const u64 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void agent_store(u64 *p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Place of word `i` of round `round` in the ring at `ring` (32-bit places in
// one array of words: a scalar base and a 32-bit offset per access).
__device__ __forceinline__ uint32_t word(uint32_t ring, int round, int n, int i)
{
    return ring + (uint32_t)(round % kRing) * (uint32_t)n + (uint32_t)i;
}

__device__ __forceinline__ void publish(u64 *words, uint32_t ring, int round, int n, int i, double v)
{
    const u64 bits = (u64)__double_as_longlong(v);
    // (a NaN with the empty pattern: another NaN)
    agent_store(words + word(ring, round, n, i), bits == kEmpty ? 0x7ff8000000000000ull : bits);
    agent_store(words + word(ring, round + 2, n, i), kEmpty);
}

// Every store of this wavefront has completed: visible to the device.
__device__ __forceinline__ void stores_done()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// LDS of the exchange: the sums of slices or wavefronts; per sum of an
// iteration the four wavefronts' parts of block_sum over the partials; a wait
// that ran out.
struct Exchange {
    double red[32], part[2][kWaves];
    int bad;
};

// How long a poll goes on.
struct Patience {
    DevState *st;
    int64_t wait, t0 = 0;
    int n = 0;
    __device__ Patience(DevState *s, int64_t w) : st(s), wait(w) {}
    __device__ __forceinline__ bool over()
    {
        if (wait < 0) // (tests: the first wait gives up)
            return true;
        if ((++n & 63) != 0)
            return false;
        const int64_t now = wall_clock64();
        if (t0 == 0)
            t0 = now;
        return now - t0 > wait || __hip_atomic_load(&st->aborted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
};

// The N words at places at[] (kNone: absent, 0.0) once all of a wavefront's are
// there.
constexpr uint32_t kNone = ~0u;
template <int N>
__device__ __forceinline__ void await_words(const u64 *words, const uint32_t (&at)[N], double (&v)[N], Patience p,
                                            Exchange &ex)
{
    u64 got[N];
    for (;;) {
        bool all = true;
#pragma unroll
        for (int u = 0; u < N; ++u)
            got[u] = agent_load(words + (at[u] != kNone ? at[u] : 0u));
#pragma unroll
        for (int u = 0; u < N; ++u)
            all = all && (got[u] != kEmpty || at[u] == kNone);
        if (__all(all))
            break;
        if (p.over()) {
            ex.bad = 1;
            break;
        }
        // many words a lane: leave the memory to the stores for a while
        // (205 143 rows 9.8 -> 9.65 us an iteration; fewer words lose by it)
        if constexpr (N > 8)
            __builtin_amdgcn_s_sleep(10);
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
        v[u] = at[u] != kNone ? __longlong_as_double((long long)got[u]) : 0.0;
}

// The sum over m <= J * 256 published partials as the launches form it: thread
// t of 256 adds partials t, t + 256, ... in turn, then block_sum.  Wavefront w
// of W does the part of kWaves / W of those wavefronts and leaves each one's
// sum in `part`.
template <int W, int J>
__device__ __forceinline__ void sum_words(const u64 *words, uint32_t ring, int m, int w, double (&part)[kWaves],
                                          const Patience &pt, Exchange &ex)
{
    constexpr int N = kWaves / W;
    const int lane = threadIdx.x & 63;
    uint32_t at[J * N];
    double q[J * N];
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = 64 * (w * N + u) + lane + j * kBlock;
            at[J * u + j] = i < m ? ring + i : kNone;
        }
    await_words<J * N>(words, at, q, pt, ex);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        double s = q[J * u];
#pragma unroll
        for (int j = 1; j < J; ++j)
            s = at[J * u + j] != kNone ? s + q[J * u + j] : s;
        s = group_sum<64>(s);
        if (lane == 0)
            part[w * N + u] = s;
    }
}

__device__ __forceinline__ double total(const double (&part)[kWaves])
{
    double s = part[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w)
        s += part[w];
    return s;
}

// T threads, S slices per wavefront and vector rows per thread, E entries per
// line at most (slice widths), C columns per polling thread at most.
template <int T, int S, int E, int C>
__global__ __launch_bounds__(T) void k_resident_cg(ResidentArgs A)
{
#pragma clang fp contract(off)
    constexpr int NW = T / 64, NG = T / kBlock; // wavefronts; vector workgroups
    constexpr int PW = NG;                      // wavefronts that poll the sums
    constexpr int kFetch = T - 64 * PW;         // threads that poll residual entries
    constexpr int J = T == kBlock ? 1 : 4;      // partials of a sum: at most J * 256
    extern __shared__ double pl[];              // p at the workgroup's columns
    __shared__ double rl[S * T], ql[S * T];     // r and q of the vector rows
    __shared__ Exchange ex;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, tf = t - 64 * PW;
    const int G = gridDim.x, b = xcd_remap(blockIdx.x, G), n = A.n;
    DevState *st = A.st;
    if (st->status != kRun)
        return;
    u64 *words = A.words;
    const uint32_t sx = 0, hx = kRing * A.nsig, rx = hx + kRing * A.nvec, qx = rx + kRing * n;
    // product workgroups, their slices and rows; vector workgroups and rows
    const int g0 = (int)((int64_t)b * A.nsig / G), g1 = (int)((int64_t)(b + 1) * A.nsig / G);
    const int s0 = (int)((int64_t)g0 * A.ns / A.nsig), s1 = (int)((int64_t)g1 * A.ns / A.nsig);
    const int q0 = s0 * kSliceRows, q1 = min(n, s1 * kSliceRows);
    const int v0 = b * NG * A.chunk, v1 = min(n, v0 + NG * A.chunk);
    const int vg = b * NG + t / kBlock; // this thread's vector workgroup (may be past the last)
    const int i0 = vg * A.chunk + t % kBlock, i1 = min(n, (vg + 1) * A.chunk);
    // vector rows whose product sums another workgroup makes: `head` from v0
    // on, then `tail` from tail0 on
    const int head = max(0, min(v1, q0) - v0), tail0 = max(v0, q1), tail = max(0, v1 - tail0);
    const int j0 = A.gptr[b], np = A.gptr[b + 1] - j0;
    // the matrix: value and LDS place of the column of each entry of the lines
    double v[S][E], x[S], r[S];
    uint32_t li[S][E / 2];
    int l[S], own[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int sl = s0 + wv + u * NW;
        int e0 = 0, w = 0;
        if (sl < s1) {
            e0 = A.off[sl];
            w = (A.off[sl + 1] - e0) / kSliceRows;
        }
        l[u] = sl < s1 ? sl * kSliceRows + lane : n;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int e = k < (w & ~1) ? e0 + (k >> 1) * (2 * kSliceRows) + 2 * lane + (k & 1) : e0 + k * kSliceRows + lane;
            v[u][k] = k < w ? A.val[e] : 0.0;
            const uint32_t c = k < w ? A.lcol[e0 + k * kSliceRows + lane] : 0xffffu;
            li[u][k >> 1] = (k & 1) ? li[u][k >> 1] | c << 16 : c;
        }
        const bool row = l[u] < n;
        own[u] = row ? A.lown[l[u]] : 0;
        x[u] = row ? A.x[l[u]] : 0.0;
        const int i = i0 + u * kBlock;
        r[u] = i < i1 ? A.r[i] : 0.0;
        if (i < i1)
            rl[i - v0] = r[u];
    }
    // the fetching threads' columns and the residual there
    int col[C];
    double rc[C];
#pragma unroll
    for (int u = 0; u < C; ++u) {
        const int j = tf + u * kFetch;
        col[u] = -1;
        rc[u] = 0.0;
        if (tf >= 0 && j < np) {
            col[u] = A.gcol[j0 + j];
            pl[j] = A.p[col[u]];
            rc[u] = A.r[col[u]];
        }
    }
    double rho_old = st->rho, rho = st->rho_next;
    const double tol_nb = st->tol_nb;
    const int maxit = st->maxit;
    int k = st->k, status = kRun, it = 0;
    const Patience pt(st, A.wait);
    if (t == 0)
        ex.bad = 0;
    __syncthreads();
    for (;; ++it, ++k) {
        if (sqrt(rho) <= tol_nb) {
            status = kConverged;
            break;
        }
        if (k >= maxit) {
            status = kMaxit;
            break;
        }
        if (it == A.iters)
            break;
        // p = r + beta p at every column of the product rows
        const double beta = rho / rho_old;
#pragma unroll
        for (int u = 0; u < C; ++u)
            if (col[u] >= 0)
                pl[tf + u * kFetch] = fma(beta, pl[tf + u * kFetch], rc[u]);
        __syncthreads();
        // q = A p, p'q (padding reads the first place and is not added)
        const char *plb = reinterpret_cast<const char *>(pl);
        double p[S];
#pragma unroll
        for (int u = 0; u < S; ++u) {
            double xv[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t c = (li[u][e >> 1] >> (16 * (e & 1))) & 0xffffu;
                xv[e] = *reinterpret_cast<const double *>(plb + (c != 0xffffu ? c : 0u));
            }
            double a = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const double s = a + v[u][e] * xv[e];
                a = ((li[u][e >> 1] >> (16 * (e & 1))) & 0xffffu) != 0xffffu ? s : a;
            }
            p[u] = pl[own[u]];
            const bool row = l[u] < n;
            if (row) {
                if (l[u] >= v0 && l[u] < v1)
                    ql[l[u] - v0] = a;
                else
                    publish(words, qx, it, n, l[u], a);
            }
            const double s = group_sum<64>(row ? fma(p[u], a, 0.0) : 0.0);
            if (lane == 0)
                ex.red[wv + u * NW] = s;
        }
        __syncthreads();
        if (t < 64 * PW) {
            if (t < g1 - g0) { // the sum of one product workgroup: its (at most four) slices in turn
                const int a = (int)((int64_t)(g0 + t) * A.ns / A.nsig) - s0;
                const int z = (int)((int64_t)(g0 + t + 1) * A.ns / A.nsig) - s0;
                double s = ex.red[a];
#pragma unroll
                for (int w = 1; w < kWaves; ++w)
                    s += a + w < z ? ex.red[a + w] : 0.0;
                publish(words, sx, it, A.nsig, g0 + t, s);
            }
            sum_words<PW, J>(words, word(sx, it, A.nsig, 0), A.nsig, wv, ex.part[0], pt, ex);
        } else {
            for (int m = tf; m < head + tail; m += kFetch) {
                const int o = m < head ? v0 + m : tail0 + (m - head);
                const uint32_t at[1] = {word(qx, it, n, o)};
                double q[1];
                await_words<1>(words, at, q, pt, ex);
                ql[o - v0] = q[0];
            }
        }
        __syncthreads();
        const double sigma = total(ex.part[0]);
        if (ex.bad)
            break;
        if (!(sigma > 0.0) || !isfinite(sigma)) {
            status = kBreakdown;
            break;
        }
        const double alpha = rho / sigma;
        // r -= alpha q, r'r; x += alpha p
        double rr = 0.0;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int i = i0 + u * kBlock;
            if (i < i1) {
                r[u] = fma(-alpha, ql[i - v0], r[u]);
                rl[i - v0] = r[u];
                publish(words, rx, it, n, i, r[u]);
                rr = fma(r[u], r[u], rr);
            }
        }
        rho_old = rho;
        rr = group_sum<64>(rr);
        if (lane == 0)
            ex.red[wv] = rr;
#pragma unroll
        for (int u = 0; u < S; ++u)
            x[u] = fma(alpha, p[u], x[u]);
        __syncthreads();
        if (t < 64 * PW) {
            if (t < NG && b * NG + t < A.nvec) { // the sum of one vector workgroup: its four wavefronts in turn
                double s = ex.red[kWaves * t];
#pragma unroll
                for (int w = 1; w < kWaves; ++w)
                    s += ex.red[kWaves * t + w];
                publish(words, hx, it, A.nvec, b * NG + t, s);
            }
            sum_words<PW, J>(words, word(hx, it, A.nvec, 0), A.nvec, wv, ex.part[1], pt, ex);
        } else {
            uint32_t at[C];
#pragma unroll
            for (int u = 0; u < C; ++u)
                at[u] = col[u] >= 0 && (col[u] < v0 || col[u] >= v1) ? word(rx, it, n, col[u]) : kNone;
            await_words<C>(words, at, rc, pt, ex);
#pragma unroll
            for (int u = 0; u < C; ++u)
                if (col[u] >= v0 && col[u] < v1)
                    rc[u] = rl[col[u] - v0];
        }
        stores_done(); // this round's words and the emptied ones
        __syncthreads();
        rho = total(ex.part[1]);
        if (ex.bad)
            break;
    }
    if (ex.bad) {
        if (t == 0)
            __hip_atomic_store(&st->aborted, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
        if (l[u] < n) {
            A.x[l[u]] = x[u];
            A.p[l[u]] = pl[own[u]];
        }
        if (i0 + u * kBlock < i1)
            A.r[i0 + u * kBlock] = r[u];
    }
    if (b == 0 && t == 0) {
        st->k = k;
        st->rho_next = rho;
        if (status == kRun) {
            st->rho = rho_old; // to be continued
        } else {
            st->rho = rho;
            st->iters = k;
            st->status = status;
        }
    }
}

// Before a launch: all words empty; before the first one of a solve also p = 0
// (the first step forms p_0 = r_0 + beta 0).
__global__ __launch_bounds__(kBlock) void k_resident_begin(u64 *w, int64_t nw, double *p, int n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < nw)
        w[i] = kEmpty;
    if (i < n)
        p[i] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_copy_out(int n, const DevState *st, const double *__restrict__ xw,
                                                     const int32_t *__restrict__ inv, double *__restrict__ x)
{
    const int status = st->status;
    const bool iterate = (status == kConverged || status == kMaxit || status == kBreakdown) && st->aborted == 0;
    if (!iterate && status != kZeroRhs)
        return;
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n)
        x[i] = iterate ? xw[inv != nullptr ? inv[i] : i] : 0.0;
}

template <int T, int S, int E, int C>
void resident_launch(const DevMatrix &m, const ResidentArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((k_resident_cg<T, S, E, C>), dim3(m.rs_wgs), dim3(T), (size_t)m.rs_cols * sizeof(double), s, a);
}

} // namespace

// The kernel of a planned resident solve: the smallest registers that hold its
// lines and column lists (plan_resident keeps to the largest).
void launch_resident(const DevMatrix &m, const ResidentArgs &a, bool first, hipStream_t s)
{
    const int64_t nw = resident_words(a.nsig, a.nvec, m.n);
    hipLaunchKernelGGL(k_resident_begin, dim3((unsigned)((nw + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a.words, nw,
                       a.p, first ? m.n : 0); // (nw > n)
    const int cols = m.rs_cols, w = m.rs_width;
    if (m.rs_threads == kBlock) {
        if (cols <= 6 * 192 && w <= 8)
            resident_launch<256, 1, 8, 6>(m, a, s);
        else if (cols <= 6 * 192 && w <= 16)
            resident_launch<256, 1, 16, 6>(m, a, s);
        else
            resident_launch<256, 1, 32, 16>(m, a, s);
    } else if (m.rs_slices == 1) {
        resident_launch<512, 1, 16, 6>(m, a, s);
    } else {
        resident_launch<512, 2, 16, 10>(m, a, s);
    }
}

void launch_copy_out(const DevMatrix &m, const DevState *st, const double *xw, double *x, hipStream_t s)
{
    if (m.n > 0)
        hipLaunchKernelGGL(k_copy_out, dim3((m.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, m.n, st, xw, m.vinv, x);
}

} // namespace cgmi
