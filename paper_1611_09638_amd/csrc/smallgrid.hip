// The V-cycle on its small levels (App. A multigrid).
//
// Below 128^3 a level's fields fit a few caches and a pass over them costs a
// kernel's launch and drain (3-6 us), not its bytes, so a V-cycle made of one
// kernel per sweep, residual and transfer spends its time between kernels.
// Here a level takes two launches, and everything from 16^3 down takes one:
//   k_pre_tile:  the two pre-smoothing sweeps (from u = 0), the residual and
//                its full weighting, per 3-D tile with the halo recomputed;
//   k_post_tile: the coarse correction and the two post-smoothing sweeps;
//   k_tail:      the whole rest of the cycle in one workgroup's LDS.
// The sweeps, residual and transfers are formed node by node in the order of
// the kernels of the larger levels (faces +i, -i, +j, -j, +k, -k), so they
// give the same values bit for bit.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace recon {

namespace {

constexpr int kTailThreads = 1024;
// Up to this edge the tiles are 8 x 4 x 4, so that they number one per CU at
// 32^3 (5.5 us per launch in FP32, 6.7 in FP64, against 6.4 and 8.0 with 8^3);
// above, 8^3: half the recomputation per node (64^3: 10.4 and 16.5 us, 8 x 8 x 4
// 17-19 and 26, 8 x 4 x 4 29 and 42).
constexpr int kTileSmall = 32;

// Workgroup barrier that orders LDS only: every exchange here is through LDS,
// and loads from memory stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
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

// ----------------------------------------------------------------- the tail
//
// One workgroup runs a V-cycle from a level of at most 16^3 down to the
// coarsest one with every field in LDS.  Nothing here is worth more than one
// CU: a 16^3 half-sweep is two nodes per thread, and a barrier across
// workgroups costs more than its arithmetic.  At 16 waves per CU every
// instruction of a thread takes 16 cycles and the coarsest level's passes (129
// of them, each dependent on the last) are LDS latency, so what counts is the
// number of instructions and of LDS reads:
//   - the edges are template parameters;
//   - a colour's nodes form an array of their own, [i][j][k / 2], in which five
//     of a node's six neighbours sit at the same k / 2 of the other colour's
//     array, so positions are a few registers and immediates;
//   - a thread owns the pair (k even, k + 1) of one or two consecutive planes:
//     one node of each colour per plane, whose values, coefficients and
//     right-hand side stay in registers, and which are each other's neighbours.
// From 16^3 with coarsest level 8^3 a cycle takes 24.5 us in FP32 and 28.6 in
// FP64, of which the coarsest passes are 17 (0.13 us each: the LDS write, the
// barrier, the reads and the chain of one relaxation); 8.2 and 11.4 us are the
// rest.  The launches it replaces took 74 and 78 us (coarsest level 38 and 42).
template <typename T>
struct TailArgs {
    T scale[kTailLevels];
    const T *a[kTailLevels];
    const T *b;  // right-hand side of the tail's finest level
    T *u;        // its solution
    T a_min;
    int n_pre, n_post, pairs;
};

// A thread's nodes of an N^3 level: plane p < PPT of the thread, colour c.
template <typename T, int N>
struct TailNodes {
    static constexpr int H = N / 2, HALF = N * N * H, PPT = HALF > kTailThreads ? 2 : 1, OWN = HALF / PPT;
    static constexpr int P = N * H;  // words of a plane of one colour
    bool on, s;       // owns nodes; the pair's even node on the first plane is black
    int self, nat;    // position of the pair in a colour's array (first plane); of its even node in natural order
    int ip, im, jp, jm, ka[2];  // neighbours: planes after and before, rows, the pair before or after (by parity)
    T cf[2][PPT][6], den[2][PPT], rd[2][PPT], bv[2][PPT], u[2][PPT];

    __device__ __forceinline__ void place()
    {
        // (made opaque, or the compiler keeps one level's coefficients alive
        // across the levels below it, in scratch)
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        on = OWN == kTailThreads || t < OWN;
        if (!on) t = 0;
        const int row = t / H, kk = t - row * H, g = row / N, j = row - g * N, i = g * PPT;
        s = (i + j) & 1;
        self = (i * N + j) * H + kk;
        nat = (i * N + j) * N + 2 * kk;
        ip = self + (i + PPT == N ? -i : PPT) * P;
        im = self + (i == 0 ? N - 1 : -1) * P;
        jp = self + (j + 1 == N ? 1 - N : 1) * H;
        jm = self + (j == 0 ? N - 1 : -1) * H;
        const int before = self + (kk == 0 ? H - 1 : -1), after = self + (kk + 1 == H ? 1 - H : 1);
        ka[0] = s ? after : before;  // of a node that is odd in its pair: the pair after
        ka[1] = s ? before : after;
    }
    // the neighbours (+i, -i, +j, -j, +k, -k) of node (c, p) in the colour
    // arrays x, of which the thread's own values are o
    __device__ __forceinline__ void faces(const T *x, const T (&o)[2][PPT], int c, int p, T (&v)[6]) const
    {
        const T *y = x + (1 - c) * HALF;
        v[0] = p + 1 < PPT ? o[1 - c][PPT - 1] : y[ip];
        v[1] = p > 0 ? o[1 - c][0] : y[im];
        v[2] = y[jp + p * P];
        v[3] = y[jm + p * P];
        const T far = y[ka[(p + c) & 1] + p * P], near = o[1 - c][p];
        const bool odd = ((p + c) & 1) ? !s : s;
        v[4] = odd ? far : near;
        v[5] = odd ? near : far;
    }
    // coefficients from a (halved: the face coefficient is max(a_min, h + h'))
    __device__ __forceinline__ void setup(const T *a, T a_min)
    {
        T h[2][PPT];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int p = 0; p < PPT; ++p) h[c][p] = a[c * HALF + self + p * P];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                T v[6], d = 0;
                faces(a, h, c, p, v);
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    cf[c][p][f] = fmax(h[c][p] + v[f], a_min);
                    d += cf[c][p][f];
                }
                den[c][p] = d;
            }
    }
    __device__ __forceinline__ void reciprocals()
    {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int p = 0; p < PPT; ++p) rd[c][p] = qrecip(den[c][p]);
    }
    // a pair's values (even node x, odd node y) on plane p, by colour
    __device__ __forceinline__ void split(T x, T y, int p, T &red, T &black) const
    {
        const bool swap = (p & 1) ? !s : s;
        red = swap ? y : x;
        black = swap ? x : y;
    }
    __device__ __forceinline__ void put(T *x, int c) const
    {
        if (on)
#pragma unroll
            for (int p = 0; p < PPT; ++p) x[c * HALF + self + p * P] = u[c][p];
    }
    // sum over the faces of coefficient times (neighbour - u0)
    __device__ __forceinline__ T sum(const T *x, int c, int p, T u0) const
    {
        T v[6], num = 0;
        faces(x, u, c, p, v);
#pragma unroll
        for (int f = 0; f < 6; ++f) num += cf[c][p][f] * (v[f] - u0);
        return num;
    }
    // relax colour c; zero: from u = 0, of which nothing is read
    __device__ __forceinline__ void relax(const T *x, int c, bool zero)
    {
#pragma unroll
        for (int p = 0; p < PPT; ++p)
            u[c][p] = qdiv((zero ? (T)0 : sum(x, c, p, (T)0)) - bv[c][p], den[c][p], rd[c][p]);
    }
};

// Mean of the N^3 values of x (natural order), by halving: thread t of 1024
// takes x[t], x[t + 1024], ..., and a tree folds the threads (lanes 0-15 of the
// first wave read the 1024 words and keep the tree's order).  red: 1024
// words where N^3 is larger, else one.
template <typename T, int N>
__device__ __forceinline__ T tail_mean(const T *x, double *red)
{
    constexpr int N3 = N * N * N;
    const int t = threadIdx.x;
    if constexpr (N3 > kTailThreads) {
        double v = 0.0;
        for (int p = t; p < N3; p += kTailThreads) v += (double)x[p];
        red[t] = v;
        lds_barrier();
    }
    if (t < 64) {
        double q[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            double m[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int at = (t & 15) + 16 * w + 64 * k;
                if constexpr (N3 > kTailThreads) m[k] = red[at];
                else m[k] = 64 * k + 16 * w < N3 && at < N3 ? (double)x[at < N3 ? at : 0] : 0.0;
            }
#pragma unroll
            for (int h = 8; h > 0; h >>= 1)
#pragma unroll
                for (int k = 0; k < h; ++k) m[k] += m[k + h];
            q[w] = m[0];
        }
        double v = (q[0] + q[2]) + (q[1] + q[3]);
        v += lane_down<8>(v);
        v += lane_down<4>(v);
        v += lane_down<2>(v);
        v += lane_down<1>(v);
        if (t == 0) red[0] = v;
    }
    lds_barrier();
    return (T)(red[0] / N3);
}

// The coarsest level: x holds the right-hand side and receives the solution
// (natural order); a, u: colour arrays.
template <typename T, int N>
__device__ __forceinline__ void tail_coarsest(const TailArgs<T> &g, T scale, const T *a, T *u, T *x, double *red)
{
    using Nodes = TailNodes<T, N>;
    constexpr int PPT = Nodes::PPT;
    const T inv = (T)1 / scale;
    const T mb = tail_mean<T, N>(x, red);
    Nodes nd;
    nd.place();
    nd.setup(a, g.a_min);
    T y[2][PPT];
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        nd.split(x[nd.nat + p * N * N] - mb, x[nd.nat + p * N * N + 1] - mb, p, nd.bv[0][p], nd.bv[1][p]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            nd.bv[c][p] *= inv;
            y[c][p] = (T)1 / nd.den[c][p];
            nd.u[c][p] = 0;
        }
    }
    auto pass = [&](auto cc, auto zero) {
        constexpr int c = decltype(cc)::value;
        if (nd.on) {
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                const T num = decltype(zero)::value ? (T)0 : nd.sum(u, c, p, (T)0);
                nd.u[c][p] = divide_by(num - nd.bv[c][p], nd.den[c][p], y[c][p]);
                u[c * Nodes::HALF + nd.self + p * Nodes::P] = nd.u[c][p];
            }
        }
        lds_barrier();
    };
    constexpr std::integral_constant<int, 0> red_{};
    constexpr std::integral_constant<int, 1> black_{};
    pass(red_, std::true_type{});
    for (int q = 0; q < g.pairs; ++q) {
        pass(black_, std::false_type{});
        pass(red_, std::false_type{});
    }
    // natural order again, mean removed
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        T e, o;
        nd.split(nd.u[0][p], nd.u[1][p], p, e, o);
        if (nd.on) {
            x[nd.nat + p * N * N] = e;
            x[nd.nat + p * N * N + 1] = o;
        }
    }
    lds_barrier();
    const T mu = tail_mean<T, N>(x, red);
#pragma unroll
    for (int p = 0; p < PPT; ++p)
        if (nd.on) {
            T e, o;
            nd.split(nd.u[0][p], nd.u[1][p], p, e, o);
            x[nd.nat + p * N * N] = e - mu;
            x[nd.nat + p * N * N + 1] = o - mu;
        }
    lds_barrier();
}

// The cycle on an N^3 level and the LV - 1 levels below it.  mem: its a and u
// (by colour) and a third field: the right-hand side on entry (natural order,
// not on the finest level, which reads memory), then the residual (by
// colour), then the solution (natural order); the next level's follow.
template <typename T, int N, int LV, bool TOP>
__device__ __forceinline__ void tail_level(const TailArgs<T> &g, int l, T *mem, double *red)
{
    constexpr int N3 = N * N * N;
    const int t = threadIdx.x;
    T *a = mem, *u = mem + N3, *x = mem + 2 * N3;
    if constexpr (LV == 1) {
        tail_coarsest<T, N>(g, g.scale[l], a, u, x, red);
    } else {
        using Nodes = TailNodes<T, N>;
        constexpr int PPT = Nodes::PPT, P = Nodes::P, HALF = Nodes::HALF, NC = N / 2, NC3 = NC * NC * NC;
        const T inv = (T)1 / g.scale[l];
        T *ec = mem + 3 * N3 + 2 * NC3;
        Nodes nd;
        nd.place();
        nd.setup(a, g.a_min);
        nd.reciprocals();
#pragma unroll
        for (int p = 0; p < PPT; ++p) {
            const T *b = (TOP ? g.b : x) + nd.nat + p * N * N;
            nd.split(b[0] * inv, b[1] * inv, p, nd.bv[0][p], nd.bv[1][p]);
            nd.u[0][p] = nd.u[1][p] = 0;
        }
        if (g.n_pre == 0) {
            nd.put(u, 0);
            nd.put(u, 1);
        }
        for (int q = 0; q < g.n_pre; ++q) {
            nd.relax(u, 0, q == 0);
            nd.put(u, 0);
            lds_barrier();
            nd.relax(u, 1, false);
            nd.put(u, 1);
            lds_barrier();
        }
        if (!TOP || g.n_pre == 0) lds_barrier();  // (every right-hand side has been read)
        // residual b - scale A u (the scale is a power of two)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                const T r = g.scale[l] * (nd.bv[c][p] - nd.sum(u, c, p, nd.u[c][p]));
                if (nd.on) x[c * HALF + nd.self + p * P] = r;
            }
        lds_barrier();
        // full weighting
        if (t < NC3) {
            const int I = t / (NC * NC), J = t / NC % NC, K = t % NC;
            const int before = K == 0 ? NC - 1 : -1;  // of the odd node before the even one
            const T w[3] = {(T)0.25, (T)0.5, (T)0.25};
            T acc = 0;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int ii = dx == 0 && I == 0 ? N - 1 : 2 * I + dx - 1;
                T pa = 0;
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int jj = dy == 0 && J == 0 ? N - 1 : 2 * J + dy - 1;
                    // the even nodes of row (ii, jj) have colour dx + dy, the odd ones the other
                    const T *e = x + ((dx + dy) & 1) * HALF + (ii * N + jj) * NC + K;
                    const T *o = x + ((dx + dy + 1) & 1) * HALF + (ii * N + jj) * NC + K;
                    pa += w[dy] * (w[0] * o[before] + w[1] * e[0] + w[2] * o[0]);
                }
                acc += w[dx] * pa;
            }
            ec[t] = acc;
        }
        lds_barrier();
        tail_level<T, NC, LV - 1, false>(g, l + 1, mem + 3 * N3, red);
        // u += P e (trilinear): weights 1/2 along k, then j, then i; an even
        // index takes its node twice, and half of x + x is x
        nd.place();
        {
            const int row = nd.self / NC, kk = nd.self - row * NC, i = row / N, j = row - i * N;
            const int j0 = j >> 1, k1 = kk + 1 == NC ? 0 : kk + 1;
            const int j1 = (j & 1) ? (j0 + 1 == NC ? 0 : j0 + 1) : j0;
            auto inplane = [&](int ic, T &even, T &odd) {
                const T *e0 = ec + (ic * NC + j0) * NC, *e1 = ec + (ic * NC + j1) * NC;
                const T x0 = e0[kk], x1 = e1[kk], y0 = e0[k1], y1 = e1[k1];
                even = (T)0.5 * (x0 + x1);
                odd = (T)0.5 * ((T)0.5 * (x0 + y0) + (T)0.5 * (x1 + y1));
            };
            const int i0 = i >> 1, i1 = i0 + 1 == NC ? 0 : i0 + 1;
            T e0, o0, e1, o1;
            inplane(i0, e0, o0);
            inplane(PPT == 2 || (i & 1) ? i1 : i0, e1, o1);
            T r, b;
            if constexpr (PPT == 2) {  // planes 2 i0 and 2 i0 + 1
                nd.split(e0, o0, 0, r, b);
                nd.u[0][0] += r;
                nd.u[1][0] += b;
                nd.split((T)0.5 * (e0 + e1), (T)0.5 * (o0 + o1), 1, r, b);
                nd.u[0][PPT - 1] += r;
                nd.u[1][PPT - 1] += b;
            } else {
                nd.split((T)0.5 * (e0 + e1), (T)0.5 * (o0 + o1), 0, r, b);
                nd.u[0][0] += r;
                nd.u[1][0] += b;
            }
        }
        nd.put(u, 0);
        nd.setup(a, g.a_min);
        nd.reciprocals();
        lds_barrier();
        for (int q = 0; q < g.n_post; ++q) {
            nd.relax(u, 1, false);
            nd.put(u, 1);
            lds_barrier();
            nd.relax(u, 0, false);
            nd.put(u, 0);
            lds_barrier();
        }
#pragma unroll
        for (int p = 0; p < PPT; ++p) {
            T e, o;
            nd.split(nd.u[0][p], nd.u[1][p], p, e, o);
            T *out = (TOP ? g.u : x) + nd.nat + p * N * N;
            if (nd.on) {
                out[0] = e;
                out[1] = o;
            }
        }
        if (!TOP) lds_barrier();
    }
}

// words of a level's three fields and of those below it
constexpr int tail_words(int n, int levels) { return levels ? 3 * n * n * n + tail_words(n / 2, levels - 1) : 0; }

template <typename T, int N, int LV>
__global__ void __launch_bounds__(kTailThreads) k_tail(const TailArgs<T> g)
{
    constexpr int NT = kTailThreads, NL = N >> (LV - 1);
    __shared__ T mem[tail_words(N, LV)];
    __shared__ double red[NL * NL * NL > NT ? NT : 1];
    const int t = threadIdx.x;
    // coefficients of every level, by colour
    T *w = mem;
#pragma unroll
    for (int l = 0; l < LV; ++l) {
        const int n = N >> l, n3 = n * n * n, h = n / 2;
        const T *ag = g.a[l];
#pragma unroll
        for (int r = 0; r < (n3 / 2 + NT - 1) / NT; ++r) {
            const int m = t + r * NT;
            if (n3 / 2 % NT && m >= n3 / 2) break;
            const int row = m / h, s = (row / n + row % n) & 1;
            const T e = (T)0.5 * ag[2 * m], o = (T)0.5 * ag[2 * m + 1];
            w[s * (n3 / 2) + m] = e;
            w[(1 - s) * (n3 / 2) + m] = o;
        }
        w += 3 * n3;
    }
    if constexpr (LV == 1)
        for (int p = t; p < N * N * N; p += NT) mem[2 * N * N * N + p] = g.b[p];
    lds_barrier();
    tail_level<T, N, LV, true>(g, 0, mem, red);
    if constexpr (LV == 1)
        for (int p = t; p < N * N * N; p += NT) g.u[p] = mem[2 * N * N * N + p];
}

// ---------------------------------------------------------------- the tiles
//
// A workgroup owns a CI x CJ x CK block of nodes and recomputes what it needs
// of its neighbours' (two sweeps reach four nodes, the residual and its full
// weighting two more on the low side), so a level's whole downward or upward
// half is one launch without exchange between workgroups.  An 8^3 block does
// 5.8 times the relaxations of its own nodes before the coarse level (half of
// 17^3, 15^3, 13^3 and 11^3 nodes) and 2.9 times after it (14^3, 12^3, 10^3
// and 8^3): cheaper than the launches it saves while a level is a few rounds of
// workgroups.
//
// Positions are counted in the local frame of a block's corner, which sits on
// even nodes, so local and global colours agree.  A field in LDS covers the
// box from -L to C + H (exclusive) of the frame; its rows along k keep the
// even and the odd nodes in separate halves (no bank conflict among the nodes
// of one colour).
template <int CI, int CJ, int CK, int L, int H>
struct Box {
    static constexpr int NI = CI + L + H, NJ = CJ + L + H, NK = CK + L + H;
    static constexpr int E = (L + 1) / 2 * 2;            // even shift of k
    static constexpr int HW = (E + CK + H + 1) / 2, WK = 2 * HW;
    static constexpr int NODES = NI * NJ * NK, WORDS = NI * NJ * WK, PLANE = NJ * WK;
    static __device__ __forceinline__ int at(int i, int j, int k)
    {
        const int x = k + E;
        return ((i + L) * NJ + j + L) * WK + (x & 1) * HW + (x >> 1);
    }
};

// Threads over a box: `cols` columns (one in-plane place each) times G groups
// of threads, group g taking planes g, g + G, ...; thread t is column
// t % cols, group t / cols.  With G even a column's plane parity, and so the
// place of a colour's node in it, is the same in every plane of a thread, and
// every LDS position is the first plus an immediate.  Threads beyond G * cols
// repeat the last group's work on no nodes.
constexpr int even_groups(int cols, int nt) { return nt / cols / 2 * 2; }

// A field over a box in pairs (k even, k + 1), held in registers between the
// load and the LDS store.
template <typename T, typename B, int L, int NT>
struct PairLoad {
    static constexpr int NP = B::HW, COLS = B::NJ * NP, G = even_groups(COLS, NT), S = (B::NI + G - 1) / G;
    static_assert(G >= 2, "two planes of pairs per pass of the workgroup");
    typedef T Pair __attribute__((ext_vector_type(2)));
    Pair v[S];
    int i, j, kp, word;  // first plane, row and pair; LDS word of its even node (the odd node: HW words on)

    __device__ __forceinline__ bool on(int s) const { return i + s * G < B::NI; }
    __device__ __forceinline__ void load(const T *__restrict__ f, int i0, int j0, int k0, int n)
    {
        const int t = threadIdx.x;
        i = t / COLS;
        const int col = t - i * COLS;
        if (i >= G) i = B::NI;  // no planes
        j = col / NP;
        kp = col - j * NP;
        word = i * B::PLANE + j * B::WK + kp;
        const T *p = f + (unsigned)(wrapc(j0 - L + j, n) * n + wrapc(k0 - B::E + 2 * kp, n));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int x = min(i + s * G, B::NI - 1);
            v[s] = *reinterpret_cast<const Pair *>(p + (unsigned)(wrapc(i0 - L + x, n) * n * n));
        }
    }
};

// This thread's nodes of colour COL in the box from -LO to C + HI, with
// everything that does not change between passes in registers: LDS positions,
// face coefficients, their sum and its reciprocal, b / scale.
template <typename T, int CI, int CJ, int CK, typename BU, int NT, int LO, int HI, int COL>
struct TileNodes {
    static constexpr int NI = CI + LO + HI, NJ = CJ + LO + HI, NK = (CK + LO + HI + 1) / 2, COLS = NJ * NK;
    static constexpr int G = even_groups(COLS, NT), S = (NI + G - 1) / G, W = BU::WK, P = BU::PLANE;
    static_assert(G >= 2, "two planes per pass of the workgroup");
    int c, kp;            // position of the first node and of its +k neighbour (the -k one is the word before that)
    int i, depth;         // first plane; how deep inside the box the column lies in j and k
    T cf[S][6], den[S], rd[S], bv[S];

    __device__ __forceinline__ void locate(const T *__restrict__ b, int i0, int j0, int k0, int n, T inv_scale)
    {
        const int t = threadIdx.x;
        int g = t / COLS;
        const int col = t - g * COLS, row = col / NK, j = row - LO;
        const bool none = g >= G;
        if (none) g = 0;
        i = g - LO;
        int k = 2 * (col - row * NK) - LO + ((i + j + LO + COL) & 1);
        const bool out = k >= CK + HI;
        if (out) k -= 2;
        depth = none || out ? 0 : 1 + min(min(j, k) + LO, HI - 1 - max(j - CJ, k - CK));
        c = BU::at(i, j, k);
        kp = BU::at(i, j, k + 1);
        const T *p = b + (unsigned)(wrapc(j0 + j, n) * n + wrapc(k0 + k, n));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int x = min(i + s * G, CI + HI - 1);
            bv[s] = p[(unsigned)(wrapc(i0 + x, n) * n * n)] * inv_scale;
        }
    }
    // the node of slot s lies d deep in the box or more (1: is one of its nodes)
    __device__ __forceinline__ bool inside(int s, int d) const
    {
        return depth >= d && i + s * G >= d - 1 - LO && i + s * G < CI + HI + 1 - d;
    }
    __device__ __forceinline__ void coefficients(const T *a, T a_min)
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const T *x = a + c + s * G * P, *y = a + kp + s * G * P;
            const T h = x[0];
            cf[s][0] = fmax(h + x[P], a_min);
            cf[s][1] = fmax(h + x[-P], a_min);
            cf[s][2] = fmax(h + x[W], a_min);
            cf[s][3] = fmax(h + x[-W], a_min);
            cf[s][4] = fmax(h + y[0], a_min);
            cf[s][5] = fmax(h + y[-1], a_min);
            T d = 0;
#pragma unroll
            for (int f = 0; f < 6; ++f) d += cf[s][f];
            den[s] = d;
            rd[s] = qrecip(d);
        }
    }
    // sum over the faces of coefficient times (neighbour - u0)
    __device__ __forceinline__ T sum(const T *u, int s, T u0) const
    {
        const T *x = u + c + s * G * P, *y = u + kp + s * G * P;
        T num = 0;
        num += cf[s][0] * (x[P] - u0);
        num += cf[s][1] * (x[-P] - u0);
        num += cf[s][2] * (x[W] - u0);
        num += cf[s][3] * (x[-W] - u0);
        num += cf[s][4] * (y[0] - u0);
        num += cf[s][5] * (y[-1] - u0);
        return num;
    }
    // relax the nodes at depth d or more
    __device__ __forceinline__ void relax(T *u, int d) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const T x = qdiv(sum(u, s, (T)0) - bv[s], den[s], rd[s]);
            if (inside(s, d)) u[c + s * G * P] = x;
        }
    }
    // relax from u = 0, of which nothing is read
    __device__ __forceinline__ void relax_zero(T *u) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const T num = 0;
            if (inside(s, 1)) u[c + s * G * P] = qdiv(num - bv[s], den[s], rd[s]);
        }
    }
};

// Words of a box and of the planes past it that the slots without a node read.
template <typename BU, typename N1, typename N2>
constexpr int padded_words()
{
    const int p1 = N1::G * N1::S - N1::NI, p2 = N2::G * N2::S - N2::NI, p = p1 > p2 ? p1 : p2;
    return BU::WORDS + p * BU::PLANE;
}

// the block's corner: consecutive blocks of one XCD (block b runs on XCD
// b mod 8) take a contiguous range, whose halos share that XCD's L2
template <int CI, int CJ, int CK>
__device__ __forceinline__ void tile_corner(int n, int &i0, int &j0, int &k0)
{
    const int tk = n / CK, tj = n / CJ, nblk = gridDim.x;
    int t = blockIdx.x;
    if ((nblk & 7) == 0) t = (t & 7) * (nblk >> 3) + (t >> 3);
    k0 = t % tk * CK;
    j0 = t / tk % tj * CJ;
    i0 = t / (tk * tj) * CI;
}

// u = two sweeps (red, black) of A u = b from u = 0; c = R (b - scale A u).
template <typename T, int CI, int CJ, int CK, int NT>
__global__ void __launch_bounds__(NT) k_pre_tile(const T *__restrict__ ag, const T *__restrict__ bg,
                                                 T *__restrict__ ug, T *__restrict__ cg, int n, T scale, T inv_scale,
                                                 T a_min)
{
    using BU = Box<CI, CJ, CK, 6, 5>;  // a, then u
    using Red = TileNodes<T, CI, CJ, CK, BU, NT, 5, 4, 0>;
    using Black = TileNodes<T, CI, CJ, CK, BU, NT, 4, 3, 1>;
    // the residual's planes start at -1
    __shared__ T f[padded_words<BU, Red, Black>()], res[(CI + 1) * BU::PLANE];
    int i0, j0, k0;
    tile_corner<CI, CJ, CK>(n, i0, j0, k0);
    Red red;
    Black black;
    {
        PairLoad<T, BU, 6, NT> la;
        la.load(ag, i0, j0, k0, n);
        red.locate(bg, i0, j0, k0, n, inv_scale);
        black.locate(bg, i0, j0, k0, n, inv_scale);
#pragma unroll
        for (int s = 0; s < la.S; ++s)
            if (la.on(s)) {
                T *w = f + la.word + s * la.G * BU::PLANE;
                w[0] = (T)0.5 * la.v[s].x;
                w[BU::HW] = (T)0.5 * la.v[s].y;
            }
    }
    lds_barrier();
    red.coefficients(f, a_min);
    black.coefficients(f, a_min);
    lds_barrier();
    // f is u from here: every value read below is written first
    red.relax_zero(f);
    lds_barrier();
    black.relax(f, 1);
    lds_barrier();
    red.relax(f, 3);
    lds_barrier();
    black.relax(f, 3);
    lds_barrier();
    for (int m = threadIdx.x; m < CI * CJ * CK; m += NT) {
        const int i = m / (CJ * CK), j = m / CK % CJ, k = m % CK;
        ug[lin(i0 + i, j0 + j, k0 + k, n)] = f[BU::at(i, j, k)];
    }
    // residual over -1 .. C - 1
    auto residual = [&](const auto &nd, int depth) {
#pragma unroll
        for (int s = 0; s < nd.S; ++s) {
            const int c = nd.c + s * nd.G * BU::PLANE;
            const T acc = nd.sum(f, s, f[c]);
            // b - scale A u (the scale is a power of two)
            if (nd.inside(s, depth)) res[c - 5 * BU::PLANE] = scale * (nd.bv[s] - acc);
        }
    };
    residual(red, 5);
    residual(black, 4);
    lds_barrier();
    const int nc = n >> 1;
    for (int m = threadIdx.x; m < CI * CJ * CK / 8; m += NT) {
        const int I = m / (CJ * CK / 4), J = m / (CK / 2) % (CJ / 2), K = m % (CK / 2);
        const T w[3] = {(T)0.25, (T)0.5, (T)0.25};
        T acc = 0;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            T pa = 0;
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                const T *r = res + BU::at(2 * I + x - 1, 2 * J + y - 1, 2 * K) - 5 * BU::PLANE;
                // the odd nodes sit HW words after the even ones
                pa += w[y] * (w[0] * r[BU::HW - 1] + w[1] * r[0] + w[2] * r[BU::HW]);
            }
            acc += w[x] * pa;
        }
        cg[lin((i0 >> 1) + I, (j0 >> 1) + J, (k0 >> 1) + K, nc)] = acc;
    }
}

// uo = two sweeps (black, red) of A u = b from ui + P e, P the trilinear
// prolongation of e (edge n/2).  The first pass overwrites the black nodes
// without reading them.
template <typename T, int CI, int CJ, int CK, int NT>
__global__ void __launch_bounds__(NT) k_post_tile(const T *__restrict__ ag, const T *__restrict__ bg,
                                                  const T *__restrict__ ui, const T *__restrict__ eg,
                                                  T *__restrict__ uo, int n, T inv_scale, T a_min)
{
    using BU = Box<CI, CJ, CK, 4, 4>;              // a, then u
    using BE = Box<CI / 2, CJ / 2, CK / 2, 2, 3>;  // e
    using Black = TileNodes<T, CI, CJ, CK, BU, NT, 3, 3, 1>;
    using Red = TileNodes<T, CI, CJ, CK, BU, NT, 2, 2, 0>;
    __shared__ T f[padded_words<BU, Red, Black>()], e[BE::NODES];
    int i0, j0, k0;
    tile_corner<CI, CJ, CK>(n, i0, j0, k0);
    Black black;
    Red red;
    PairLoad<T, BU, 4, NT> lu;
    {
        PairLoad<T, BU, 4, NT> la;
        constexpr int ER = (BE::NODES + NT - 1) / NT;
        T ev[ER];
        const int nc = n >> 1;
#pragma unroll
        for (int r = 0; r < ER; ++r) {
            const int m = min((int)threadIdx.x + r * NT, BE::NODES - 1);
            const int I = m / (BE::NJ * BE::NK) - 2, J = m / BE::NK % BE::NJ - 2, K = m % BE::NK - 2;
            ev[r] = eg[lin(wrapc((i0 >> 1) + I, nc), wrapc((j0 >> 1) + J, nc), wrapc((k0 >> 1) + K, nc), nc)];
        }
        la.load(ag, i0, j0, k0, n);
        lu.load(ui, i0, j0, k0, n);
        black.locate(bg, i0, j0, k0, n, inv_scale);
        red.locate(bg, i0, j0, k0, n, inv_scale);
#pragma unroll
        for (int r = 0; r < ER; ++r) e[min((int)threadIdx.x + r * NT, BE::NODES - 1)] = ev[r];
#pragma unroll
        for (int s = 0; s < la.S; ++s)
            if (la.on(s)) {
                T *w = f + la.word + s * la.G * BU::PLANE;
                w[0] = (T)0.5 * la.v[s].x;
                w[BU::HW] = (T)0.5 * la.v[s].y;
            }
    }
    lds_barrier();
    black.coefficients(f, a_min);
    red.coefficients(f, a_min);
    lds_barrier();
    {
        // weights 1/2 along k, then j, then i; an even index takes its node
        // twice, and half of x + x is x (a thread's planes have one parity)
        const int p = ((lu.i >> 1) * BE::NJ + (lu.j >> 1)) * BE::NK + lu.kp;
        const int dj = (lu.j & 1) * BE::NK, di = (lu.i & 1) * BE::NJ * BE::NK;
        auto inplane = [&](const T *q, T &even, T &odd) {
            const T x0 = q[0], x1 = q[dj], y0 = q[1], y1 = q[dj + 1];
            even = (T)0.5 * (x0 + x1);
            odd = (T)0.5 * ((T)0.5 * (x0 + y0) + (T)0.5 * (x1 + y1));
        };
#pragma unroll
        for (int s = 0; s < lu.S; ++s) {
            if (!lu.on(s)) continue;
            const T *q = e + p + s * (lu.G / 2) * BE::NJ * BE::NK;
            T e0, o0, e1, o1;
            inplane(q, e0, o0);
            inplane(q + di, e1, o1);
            T *w = f + lu.word + s * lu.G * BU::PLANE;
            w[0] = lu.v[s].x + (T)0.5 * (e0 + e1);
            w[BU::HW] = lu.v[s].y + (T)0.5 * (o0 + o1);
        }
    }
    lds_barrier();
    black.relax(f, 1);
    lds_barrier();
    red.relax(f, 1);
    lds_barrier();
    black.relax(f, 3);
    lds_barrier();
    red.relax(f, 3);
    lds_barrier();
    for (int m = threadIdx.x; m < CI * CJ * CK; m += NT) {
        const int i = m / (CJ * CK), j = m / CK % CJ, k = m % CK;
        uo[lin(i0 + i, j0 + j, k0 + k, n)] = f[BU::at(i, j, k)];
    }
}

}  // namespace

bool tail_supported(int n) { return n <= 16; }

template <typename T>
hipError_t launch_tail(const T *const *a, const int *n, const T *scale, int levels, const T *b, T *u, T a_min,
                       int n_pre, int n_post, int pairs, hipStream_t s)
{
    if (levels < 1 || levels > kTailLevels || !tail_supported(n[0])) return hipErrorInvalidValue;
    TailArgs<T> g;
    for (int l = 0; l < kTailLevels; ++l) {
        g.scale[l] = l < levels ? scale[l] : (T)1;
        g.a[l] = l < levels ? a[l] : nullptr;
    }
    g.b = b;
    g.u = u;
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

// Tiles of 8 x 4 x 4 nodes up to kTileSmall and of 8^3 above where 8 divides the
// edge, else of 4^3 (every level's edge above 16 is a multiple of 4).
bool tile_supported(int n)
{
    return n > 16 && n % 4 == 0;
}

// the pair loads need fields on 16-byte boundaries
static bool paired(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

template <typename T, int CI, int CJ, int CK, int NT>
hipError_t pre_shape(const T *a, const T *b, T *u, T *c, int n, T scale, T a_min, hipStream_t s)
{
    const int blocks = (n / CI) * (n / CJ) * (n / CK);
    k_pre_tile<T, CI, CJ, CK, NT><<<blocks, NT, 0, s>>>(a, b, u, c, n, scale, (T)1 / scale, a_min);
    return hipGetLastError();
}

template <typename T, int CI, int CJ, int CK, int NT>
hipError_t post_shape(const T *a, const T *b, const T *u_in, const T *e, T *u_out, int n, T scale, T a_min,
                      hipStream_t s)
{
    const int blocks = (n / CI) * (n / CJ) * (n / CK);
    k_post_tile<T, CI, CJ, CK, NT><<<blocks, NT, 0, s>>>(a, b, u_in, e, u_out, n, (T)1 / scale, a_min);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pre_tile(const T *a, const T *b, T *u, T *c, int n, T scale, T a_min, hipStream_t s)
{
    if (!tile_supported(n) || !paired(a)) return hipErrorInvalidValue;
    if (n % 8) return pre_shape<T, 4, 4, 4, 512>(a, b, u, c, n, scale, a_min, s);
    if (n <= kTileSmall) return pre_shape<T, 8, 4, 4, 576>(a, b, u, c, n, scale, a_min, s);
    return pre_shape<T, 8, 8, 8, 1024>(a, b, u, c, n, scale, a_min, s);
}

template <typename T>
hipError_t launch_post_tile(const T *a, const T *b, const T *u_in, const T *e, T *u_out, int n, T scale, T a_min,
                            hipStream_t s)
{
    if (!tile_supported(n) || u_in == u_out || !paired(a) || !paired(u_in)) return hipErrorInvalidValue;
    if (n % 8) return post_shape<T, 4, 4, 4, 512>(a, b, u_in, e, u_out, n, scale, a_min, s);
    if (n <= kTileSmall) return post_shape<T, 8, 4, 4, 576>(a, b, u_in, e, u_out, n, scale, a_min, s);
    return post_shape<T, 8, 8, 8, 1024>(a, b, u_in, e, u_out, n, scale, a_min, s);
}

#define RECON_INSTANTIATE(T)                                                                                  \
    template hipError_t launch_tail<T>(const T *const *, const int *, const T *, int, const T *, T *, T, int, int, int, \
                                        hipStream_t);                                          \
    template hipError_t launch_pre_tile<T>(const T *, const T *, T *, T *, int, T, T, hipStream_t);           \
    template hipError_t launch_post_tile<T>(const T *, const T *, const T *, const T *, T *, int, T, T, hipStream_t);

RECON_INSTANTIATE(double)
RECON_INSTANTIATE(float)

}  // namespace recon
