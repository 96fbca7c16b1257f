// The V-cycle on its small levels (App. A multigrid).
//
// Below 128^3 a level's fields fit a few caches and a pass over them costs a
// kernel's launch and drain (3-6 us), not its bytes, so a V-cycle made of one
// kernel per sweep, residual and transfer spends its time between kernels.
// Here a level takes two launches, and everything from 16^3 down takes one:
//   k_pre_tile:  the two pre-smoothing sweeps (from u = 0), the residual and
//                its full weighting, per 3-D tile with the halo recomputed;
//   k_post_tile: the coarse correction and the two post-smoothing sweeps;
//   k_tail:      the whole rest of the cycle in one workgroup's LDS, with the
//                coarsest level's relaxation as a product with its matrix
//                (k_coarse_matrix, once per coefficient).
// The sweeps, residual and transfers are formed node by node in the order of
// the kernels of the larger levels (faces +i, -i, +j, -j, +k, -k), so they
// give the same values bit for bit.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace recon {

namespace {

constexpr int kTailThreads = 1024;

// Workgroup barrier that orders LDS only: every exchange here is through LDS,
// and loads from memory stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum of one value per thread over a workgroup of kTailThreads threads (every
// thread gets it), by halving: the sums of a 1024-word tree, in its order.
// red: kTailThreads words, free again afterwards.
__device__ __forceinline__ double tail_sum(double v, double *red)
{
    const int t = threadIdx.x;
    red[t] = v;
    lds_barrier();
    if (t < 64) {
        double x[kTailThreads / 64];
#pragma unroll
        for (int m = 0; m < kTailThreads / 64; ++m) x[m] = red[t + 64 * m];
#pragma unroll
        for (int w = kTailThreads / 128; w > 0; w >>= 1)
#pragma unroll
            for (int m = 0; m < w; ++m) x[m] += x[m + w];
        for (int off = 32; off > 0; off >>= 1) x[0] += __shfl_down(x[0], off, 64);
        if (t == 0) red[0] = x[0];
    }
    lds_barrier();
    const double s = red[0];
    lds_barrier();
    return s;
}

// x / d rounded as the division is, from y = 1 / d: two residual corrections
// of x y (Markstein), a third of the division's latency.
template <typename T>
__device__ __forceinline__ T divide_by(T x, T d, T y)
{
    T q = x * y;
    q = fma(fma(-d, q, x), y, q);
    return fma(fma(-d, q, x), y, q);
}

// LDS position of node (i, j, k) of an n^3 level: the even and odd k of a row
// sit in separate halves, so the nodes of one colour and each of their
// neighbours are contiguous across a wavefront.
__device__ __forceinline__ int spos(int i, int j, int k, int n)
{
    return (i * n + j) * n + (k & 1) * (n >> 1) + (k >> 1);
}

// Node m of colour `col` (i + j + k = col mod 2) in the order of rows: its
// position and its six neighbours' (+i, -i, +j, -j, +k, -k).
__device__ __forceinline__ void colour_node(int m, int col, int n, int &self, int (&q)[6])
{
    const int h = n >> 1, row = m / h, i = row / n, j = row - i * n;
    const int k = 2 * (m - row * h) + ((i + j + col) & 1);
    self = spos(i, j, k, n);
    q[0] = spos(wrapc(i + 1, n), j, k, n);
    q[1] = spos(wrapc(i - 1, n), j, k, n);
    q[2] = spos(i, wrapc(j + 1, n), k, n);
    q[3] = spos(i, wrapc(j - 1, n), k, n);
    q[4] = spos(i, j, wrapc(k + 1, n), n);
    q[5] = spos(i, j, wrapc(k - 1, n), n);
}

// ------------------------------------------------------------ coarsest level
//
// The coarsest level relaxes u from zero by (red, black)^pairs red, 2 pairs + 1
// dependent passes of a workgroup (38-42 us per V-cycle at 8^3, more than all
// other small levels together).  In exact arithmetic the black nodes end at
//   u_b = -Hs w,  w = beta_b + C D_r^-1 beta_r,  beta = b / scale,
//   Hs = (sum_{k < pairs} T^k) D_b^-1,  T = D_b^-1 C D_r^-1 C,
// with D the sums of face coefficients and C the couplings between colours, and
// the last red pass gives u_r = D_r^-1 (C u_b - beta_r).  Hs depends on the
// coefficient alone, so it is formed once per hierarchy (column c by the
// recurrence itself, one workgroup each, in FP64) and every V-cycle makes one
// product with it.  Hs is symmetric and has (n^3/2)^2 entries: 256 KB in FP32
// and 512 KB in FP64 at 8^3, which one workgroup reads from L2 in 2-4 us.
template <typename T>
__global__ void __launch_bounds__(512) k_coarse_matrix(const T *__restrict__ ag, T *__restrict__ H, int n, T a_min,
                                                       int pairs)
{
    __shared__ double sa[1000], su[1000];
    const int t = threadIdx.x, n3 = n * n * n, nb = n3 >> 1, c = blockIdx.x;
    for (int p = t; p < n3; p += 512) {
        const int i = p / (n * n), j = p / n % n, k = p % n;
        sa[spos(i, j, k, n)] = (double)ag[p];
        su[p] = 0.0;
    }
    __syncthreads();
    // thread t: red node t and black node t
    int q[2][6], self[2];
    double cf[2][6], id[2];
#pragma unroll
    for (int col = 0; col < 2; ++col) {
        colour_node(t < nb ? t : 0, col, n, self[col], q[col]);
        double d = 0.0;
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            cf[col][f] = (double)facec((T)sa[self[col]], (T)sa[q[col][f]], a_min);
            d += cf[col][f];
        }
        id[col] = 1.0 / d;
    }
    const bool on = t < nb;
    const double g = t == c ? id[1] : 0.0;
    double u = pairs > 0 ? g : 0.0;
    if (on) su[self[1]] = u;
    __syncthreads();
    for (int p = 1; p < pairs; ++p) {
        double s = 0.0;
#pragma unroll
        for (int f = 0; f < 6; ++f) s += cf[0][f] * su[q[0][f]];
        if (on) su[self[0]] = s * id[0];
        __syncthreads();
        s = 0.0;
#pragma unroll
        for (int f = 0; f < 6; ++f) s += cf[1][f] * su[q[1][f]];
        u = s * id[1] + g;
        if (on) su[self[1]] = u;
        __syncthreads();
    }
    if (on) H[(size_t)c * nb + t] = (T)u;
}

// ----------------------------------------------------------------- the tail
//
// One workgroup runs a V-cycle from a level of at most 16^3 down to the
// coarsest one with every field in LDS (a, u, b of each level, and the
// residual: 145 KB in FP64 from 16^3).  Nothing else is worth more than one
// CU here: a 16^3 half-sweep is two nodes per thread, and a barrier across
// workgroups costs more than its arithmetic.  At 16 waves per CU every
// instruction of a thread takes 16 cycles, so what counts is their number:
// the edges are template parameters (every index is a shift or a constant),
// and a thread keeps the face coefficients, neighbours and right-hand side of
// its nodes (up to two of each colour) in registers over a level's sweeps.
template <typename T>
struct TailArgs {
    T scale[kTailLevels];
    const T *a[kTailLevels];
    const T *b;  // right-hand side of the tail's finest level
    T *u;        // its solution
    const T *H;  // coarsest level's matrix, or null: relax it
    T a_min;
    int n_pre, n_post, pairs;
};

// This thread's nodes of an N^3 level: S slots of each colour, slot s of
// colour c the node tid + s * kTailThreads of that colour.
template <typename T, int N>
struct TailNodes {
    static constexpr int HALF = N * N * N / 2, S = (HALF + kTailThreads - 1) / kTailThreads;
    int self[2][S], q[2][S][6];
    T cf[2][S][6], den[2][S], bv[2][S];

    static __device__ __forceinline__ bool on(int s) { return (int)threadIdx.x + s * kTailThreads < HALF; }

    // (the thread's number is made opaque, or the compiler keeps one level's
    // coefficients alive across the levels below it, in scratch)
    __device__ __forceinline__ void setup(const T *a, const T *b, T inv_scale, T a_min)
    {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                colour_node(on(s) ? t + s * kTailThreads : 0, c, N, self[c][s], q[c][s]);
                const T h = a[self[c][s]];
                T d = 0;
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    cf[c][s][f] = fmax(h + a[q[c][s][f]], a_min);
                    d += cf[c][s][f];
                }
                den[c][s] = d;
                bv[c][s] = b[self[c][s]] * inv_scale;
            }
    }
    // the weighted sum of a node's neighbours
    __device__ __forceinline__ T sum(const T *u, int c, int s) const
    {
        T num = 0;
#pragma unroll
        for (int f = 0; f < 6; ++f) num += cf[c][s][f] * u[q[c][s][f]];
        return num;
    }
    // relax the nodes of colour c
    __device__ __forceinline__ void relax(T *u, int c) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (on(s)) u[self[c][s]] = qdiv(sum(u, c, s) - bv[c][s], den[c][s]);
        lds_barrier();
    }
};

template <typename T, int N>
__device__ __forceinline__ void tail_coarsest(const TailArgs<T> &g, T scale, const T *a, T *u, T *b, T *R)
{
    constexpr int NT = kTailThreads, N3 = N * N * N, HALF = N3 / 2;
    const int t = threadIdx.x;
    const T inv = (T)1 / scale;
    double *red = reinterpret_cast<double *>(R);
    // H: rows over the lanes, columns split over groups of whole waves; the
    // first of a thread's columns are loaded now, ahead of their use
    constexpr int ROWS = (HALF + 63) & ~63, GROUPS = ROWS <= NT ? NT / ROWS : 1, COLS = (HALF + GROUPS - 1) / GROUPS;
    constexpr int MOST = sizeof(T) == 4 ? 64 : 32, PRE = COLS < MOST ? COLS : MOST;
    const int grp = t / ROWS, row = t - grp * ROWS;
    T *w = R, *part = R + 512;
    T hp[PRE];
    const T *h = g.H + (row < HALF ? row : 0);
    auto column = [&](int c) {
        const int x = grp + c * GROUPS;
        return x < HALF ? x : HALF - 1;
    };
    if (N <= 10 && g.H) {
#pragma unroll
        for (int c = 0; c < PRE; ++c) hp[c] = h[(size_t)column(c) * HALF];
    }
    double sum = 0.0;
    for (int p = t; p < N3; p += NT) sum += (double)b[spos(0, p / N, p % N, N)];
    const T mb = (T)(tail_sum(sum, red) / N3);
    for (int p = t; p < N3; p += NT) b[p] -= mb;
    lds_barrier();
    TailNodes<T, N> nd;
    nd.setup(a, b, inv, g.a_min);
    if (N <= 10 && g.H) {
        // half <= 500: one node of each colour per thread
        if (nd.on(0)) u[nd.self[0][0]] = qdiv(nd.bv[0][0], nd.den[0][0]);
        lds_barrier();
        if (t < ROWS) w[t] = nd.on(0) ? nd.bv[1][0] + nd.sum(u, 1, 0) : (T)0;
        lds_barrier();
        T acc = 0;
#pragma unroll
        for (int c = 0; c < PRE; ++c) acc += hp[c] * (grp + c * GROUPS < HALF ? w[column(c)] : (T)0);
#pragma unroll 16
        for (int c = PRE; c < COLS; ++c)
            acc += h[(size_t)column(c) * HALF] * (grp + c * GROUPS < HALF ? w[column(c)] : (T)0);
        part[t] = acc;
        lds_barrier();
        if (nd.on(0)) {
            T s = 0;
#pragma unroll
            for (int x = 0; x < GROUPS; ++x) s += part[x * ROWS + t];
            u[nd.self[1][0]] = -s;
        }
        lds_barrier();
        nd.relax(u, 0);
    } else {
        T y[2][TailNodes<T, N>::S];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int s = 0; s < TailNodes<T, N>::S; ++s) y[c][s] = (T)1 / nd.den[c][s];
        auto pass = [&](auto cc) {
            constexpr int c = decltype(cc)::value;
#pragma unroll
            for (int s = 0; s < TailNodes<T, N>::S; ++s)
                if (nd.on(s))
                    u[nd.self[c][s]] = divide_by(nd.sum(u, c, s) - nd.bv[c][s], nd.den[c][s], y[c][s]);
            lds_barrier();
        };
        for (int p = 0; p < g.pairs; ++p) {
            pass(std::integral_constant<int, 0>{});
            pass(std::integral_constant<int, 1>{});
        }
        pass(std::integral_constant<int, 0>{});
    }
    sum = 0.0;
    for (int p = t; p < N3; p += NT) sum += (double)u[spos(0, p / N, p % N, N)];
    const T mu = (T)(tail_sum(sum, red) / N3);
    for (int p = t; p < N3; p += NT) u[p] -= mu;
    lds_barrier();
}

// The cycle on an N^3 level and the LV - 1 levels below it; mem: its a, u and
// b, then the next level's.
template <typename T, int N, int LV>
__device__ __forceinline__ void tail_level(const TailArgs<T> &g, int l, T *mem, T *R)
{
    constexpr int NT = kTailThreads, N3 = N * N * N;
    const int t = threadIdx.x;
    T *a = mem, *u = mem + N3, *b = mem + 2 * N3;
    if constexpr (LV == 1) {
        tail_coarsest<T, N>(g, g.scale[l], a, u, b, R);
    } else {
        constexpr int NC = N / 2, NC3 = NC * NC * NC;
        const T inv = (T)1 / g.scale[l];
        T *ec = mem + 3 * N3 + NC3, *bc = ec + NC3;
        TailNodes<T, N> nd;
        nd.setup(a, b, inv, g.a_min);
        for (int s = 0; s < g.n_pre; ++s) {
            nd.relax(u, 0);
            nd.relax(u, 1);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int s = 0; s < TailNodes<T, N>::S; ++s)
                if (nd.on(s)) {
                    const T un = u[nd.self[c][s]];
                    T acc = 0;
#pragma unroll
                    for (int f = 0; f < 6; ++f) acc += nd.cf[c][s][f] * (u[nd.q[c][s][f]] - un);
                    const T Au = g.scale[l] * acc;
                    R[nd.self[c][s]] = b[nd.self[c][s]] - Au;
                }
        lds_barrier();
        // full weighting
        for (int p = t; p < NC3; p += NT) {
            const int I = p / (NC * NC), J = p / NC % NC, K = p % NC;
            const T w[3] = {(T)0.25, (T)0.5, (T)0.25};
            const int km = K == 0 ? NC - 1 : K - 1;  // position of 2K - 1 among the odd nodes
            T acc = 0;
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const int ii = x == 0 && I == 0 ? N - 1 : 2 * I + x - 1;
                T pa = 0;
#pragma unroll
                for (int y = 0; y < 3; ++y) {
                    const int jj = y == 0 && J == 0 ? N - 1 : 2 * J + y - 1;
                    const T *r = R + (ii * N + jj) * N;
                    pa += w[y] * (w[0] * r[NC + km] + w[1] * r[K] + w[2] * r[NC + K]);
                }
                acc += w[x] * pa;
            }
            bc[spos(I, J, K, NC)] = acc;
        }
        lds_barrier();
        tail_level<T, NC, LV - 1>(g, l + 1, mem + 3 * N3, R);
        // u += P e (trilinear): weights 1/2 along k, then j, then i
#pragma unroll
        for (int r = 0; r < (N3 + NT - 1) / NT; ++r) {
            const int p = t + r * NT;
            if (N3 % NT && p >= N3) break;
            const int i = p / (N * N), j = p / N % N, k = p % N;
            const int i0 = i >> 1, j0 = j >> 1, k0 = k >> 1;
            const int i1 = i0 + 1 == NC ? 0 : i0 + 1, j1 = j0 + 1 == NC ? 0 : j0 + 1;
            const int k1 = (k & 1) ? (k0 + 1 == NC ? 0 : k0 + 1) : k0;
            const int p0 = spos(0, 0, k0, NC), p1 = spos(0, 0, k1, NC);
            auto inplane = [&](int ic) {
                const T *e0 = ec + (ic * NC + j0) * NC;
                const T r0 = (k & 1) ? (T)0.5 * (e0[p0] + e0[p1]) : e0[p0];
                if (!(j & 1)) return r0;
                const T *e1 = ec + (ic * NC + j1) * NC;
                const T r1 = (k & 1) ? (T)0.5 * (e1[p0] + e1[p1]) : e1[p0];
                return (T)0.5 * (r0 + r1);
            };
            T acc = inplane(i0);
            if (i & 1) acc = (T)0.5 * (acc + inplane(i1));
            u[spos(i, j, k, N)] += acc;
        }
        nd.setup(a, b, inv, g.a_min);
        lds_barrier();
        for (int s = 0; s < g.n_post; ++s) {
            nd.relax(u, 1);
            nd.relax(u, 0);
        }
    }
}

// words of a, u and b of the LV levels from edge n down
constexpr int tail_words(int n, int levels) { return levels ? 3 * n * n * n + tail_words(n / 2, levels - 1) : 0; }

template <typename T, int N, int LV>
__global__ void __launch_bounds__(kTailThreads) k_tail(const TailArgs<T> g)
{
    constexpr int NT = kTailThreads, N3 = N * N * N, W = tail_words(N, LV);
    // the residual of the level in work; the coarsest level's vectors and sums
    constexpr int RW = LV > 1 && N3 > 2048 ? N3 : 2048;
    __shared__ __align__(16) T mem[(W + 3) / 4 * 4 + RW];
    const int t = threadIdx.x;
    // coefficients of every level (halved: the face coefficient is
    // max(a_min, h + h')), the finest right-hand side, u = 0
    T *w = mem;
#pragma unroll
    for (int l = 0; l < LV; ++l) {
        const int n = N >> l, n3 = n * n * n;
        const T *ag = g.a[l];
#pragma unroll
        for (int r = 0; r < (n3 + NT - 1) / NT; ++r) {
            const int p = t + r * NT;
            if (n3 % NT && p >= n3) break;
            const int q = spos(0, p / n, p % n, n);
            w[q] = (T)0.5 * ag[p];
            w[n3 + q] = 0;
            if (l == 0) w[2 * n3 + q] = g.b[p];
        }
        w += 3 * n3;
    }
    lds_barrier();
    tail_level<T, N, LV>(g, 0, mem, mem + (W + 3) / 4 * 4);
#pragma unroll
    for (int r = 0; r < (N3 + NT - 1) / NT; ++r) {
        const int p = t + r * NT;
        if (N3 % NT && p >= N3) break;
        g.u[p] = mem[N3 + spos(0, p / N, p % N, N)];
    }
}

}  // namespace

bool tail_supported(int n) { return n <= 16; }

// The product with the matrix replaces the coarsest level's relaxation where
// its bytes are few enough for one workgroup: up to 10^3 nodes (at 12^3 it is
// 6 MB in FP64, which takes as long to read as the passes take).
bool coarse_matrix_supported(int n) { return n <= 10; }

template <typename T>
hipError_t launch_coarse_matrix(const T *a, T *H, int n, T a_min, int pairs, hipStream_t s)
{
    if (!coarse_matrix_supported(n) || (n & 1)) return hipErrorInvalidValue;
    k_coarse_matrix<T><<<n * n * n / 2, 512, 0, s>>>(a, H, n, a_min, pairs);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tail(const T *const *a, const int *n, const T *scale, int levels, const T *b, T *u, const T *H,
                       T a_min, int n_pre, int n_post, int pairs, hipStream_t s)
{
    if (levels < 1 || levels > kTailLevels || !tail_supported(n[0]) ||
        (H && !coarse_matrix_supported(n[levels - 1])))
        return hipErrorInvalidValue;
    TailArgs<T> g;
    for (int l = 0; l < kTailLevels; ++l) {
        g.scale[l] = l < levels ? scale[l] : (T)1;
        g.a[l] = l < levels ? a[l] : nullptr;
    }
    g.b = b;
    g.u = u;
    g.H = H;
    g.a_min = a_min;
    g.n_pre = n_pre;
    g.n_post = n_post;
    g.pairs = pairs;
    // every chain of edges coarse_n * 2^k <= 16 with an even coarse_n
    switch (n[0] * 8 + levels) {
#define RECON_TAIL(N, LV)                                 \
    case N * 8 + LV:                                      \
        k_tail<T, N, LV><<<1, kTailThreads, 0, s>>>(g);   \
        break;
        RECON_TAIL(16, 1)
        RECON_TAIL(16, 2)
        RECON_TAIL(16, 3)
        RECON_TAIL(16, 4)
        RECON_TAIL(14, 1)
        RECON_TAIL(12, 1)
        RECON_TAIL(12, 2)
        RECON_TAIL(10, 1)
        RECON_TAIL(8, 1)
        RECON_TAIL(8, 2)
        RECON_TAIL(8, 3)
        RECON_TAIL(6, 1)
        RECON_TAIL(4, 1)
        RECON_TAIL(4, 2)
        RECON_TAIL(2, 1)
#undef RECON_TAIL
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define RECON_INSTANTIATE(T)                                                                                  \
    template hipError_t launch_coarse_matrix<T>(const T *, T *, int, T, int, hipStream_t);                    \
    template hipError_t launch_tail<T>(const T *const *, const int *, const T *, int, const T *, T *, const T *, T, \
                                       int, int, int, hipStream_t);

RECON_INSTANTIATE(double)
RECON_INSTANTIATE(float)

}  // namespace recon
