// dense.hip -- the minimum spanning tree of few points from the matrix of
// their exact distances.
//
// A call with a few hundred or thousand points is launches, copies and host
// waits: the tile-pair screen's rounds take some 130 launches and a dozen waits
// (n = 150, d = 5: 0.75 ms; n = 2048, d = 16: 1.08 ms), while all n^2 / 2 exact
// distances are a few million operations.  So up to DENSE_MAX_N points every
// pair's D^2 is formed once, in the recheck's own arithmetic, into an n x n
// matrix that stays in the last-level cache; each Boruvka round is one launch
// over its rows, whose last workgroup joins the components, and one workgroup
// roots the tree.  The edge order is that of the rechecked screen, (D^2, smaller
// id, larger id), and so is the tree.  No host wait before the end.  0.12 and
// 0.16 ms on those two, half of it the launches.
#include <cmath>

#include "common.hpp"
#include "dense.hpp"

namespace iso {

namespace {

constexpr int DT = 64;            // tile of the distance matrix
constexpr int DB = 1024;          // threads of a round's workgroup: a wave per row
constexpr float DENSE_BIG = 1e36f;  // larger D^2 (or NaN): left to the screened rounds and their checks

template <class T>
__device__ __forceinline__ bool too_big(T v) {
    return !(v <= (T)DENSE_BIG);
}

// Writes a 64 x 64 tile and, off the diagonal, its transpose (through LDS, so
// that both are whole rows); thread (lane, w) holds rows 16 w + r, column lane.
// The columns n .. nd - 1 that pad a row to whole 16 bytes are +inf.
template <class T>
__device__ __forceinline__ void put_tile(T (&t)[DT][DT + 1], const T (&v)[16], int64_t n, int64_t nd, int64_t I0, int64_t J0,
                                         T *__restrict__ D) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const T inf = (T)__builtin_huge_val();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t i = I0 + 16 * w + r, j = J0 + lane;
        const T d2 = i == j ? inf : v[r];
        if (i < n && j < nd) D[i * nd + j] = j < n ? d2 : inf;
        t[16 * w + r][lane] = d2;
    }
    if (I0 == J0) return;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t j = J0 + 16 * w + r, i = I0 + lane;
        if (i < n && j < n) D[j * nd + i] = t[lane][16 * w + r];
    }
}

// Rows I0 .. I0 + 63 of X, coordinates c .. c + W - 1 (0 past the end), as
// xi[row][coordinate] or transposed: lane = coordinate, a wave takes every
// fourth row (64 / W of them at once), and every load is issued before the first
// is used.
template <int W, class Put>
__device__ __forceinline__ void load_rows(const float *__restrict__ X, int64_t n, int64_t d, int64_t ld, int64_t I0,
                                          int64_t c, Put put) {
    constexpr int PER = 64 / W, STEPS = DT / (4 * PER);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = lane & (W - 1), sub = lane / W;
    float v[STEPS];
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
        const int64_t r = I0 + (q * 4 + w) * PER + sub;
        v[q] = X[min(r, n - 1) * ld + min(c + t, d - 1)];
    }
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
        const int r = (q * 4 + w) * PER + sub;
        put(r, t, I0 + r < n && c + t < d ? v[q] : 0.0f);
    }
}

// FP32 distances, d <= W <= 64: one thread per pair holds the partial sums that
// the lanes of a wave hold in the recheck (one square each here) and adds them
// in its butterfly's order; the sums of the lanes past W, all 0, are left out.
// Bound by those additions; a wave per pair would spend six cross-lane steps on
// each.  n = 2000, d = 16: 16 us (35
// with all 64 sums and the rows loaded one by one).
template <int W>
__global__ __launch_bounds__(256) void k_dense_f32_low(const float *__restrict__ X, int64_t n, int64_t d, int64_t ld,
                                                       int64_t nd, float *__restrict__ D, DenseState *__restrict__ st) {
    if (blockIdx.y < blockIdx.x) return;
    __shared__ __attribute__((aligned(16))) float xi[DT][W];
    __shared__ float xj[W][DT + 1];  // [coordinate][column]
    __shared__ float tile[DT][DT + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t I0 = (int64_t)blockIdx.x * DT, J0 = (int64_t)blockIdx.y * DT;
    load_rows<W>(X, n, d, ld, I0, 0, [&](int r, int t, float v) { xi[r][t] = v; });
    load_rows<W>(X, n, d, ld, J0, 0, [&](int r, int t, float v) { xj[t][r] = v; });
    __syncthreads();
    float y[W];
#pragma unroll
    for (int t = 0; t < W; ++t) y[t] = xj[t][lane];
    bool big = false;
#pragma unroll 1
    for (int r = 0; r < 16; ++r) {
        float p[W];
#pragma unroll
        for (int t = 0; t < W; ++t) {
            const float df = xi[16 * w + r][t] - y[t];
            p[t] = fmaf(df, df, 0.0f);
        }
#pragma unroll
        for (int o = W / 2; o >= 1; o >>= 1)
#pragma unroll
            for (int t = 0; t < o; ++t) p[t] = p[t] + p[t + o];
        // (r is not a constant: the value goes to the thread's own tile slot)
        tile[16 * w + r][lane] = p[0];
        big |= too_big(p[0]);
    }
    float v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = tile[16 * w + r][lane];
    if (big) st->bad = 1;
    put_tile(tile, v, n, nd, I0, J0, D);
}

// Sums over the 64 lanes of 16 values, each in the order of an xor butterfly
// (distances 32, 16, 8, 4, 2, 1): the first four steps also halve the values
// that a lane carries on with, so that lanes 4 q .. 4 q + 3 end with value q.
__device__ __forceinline__ float sum_scatter16(const float (&v)[16], int lane) {
    float a[8], b[4], c[2];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[q]), __float_as_uint(v[q + 8]), false, false);
        a[q] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[q]), __float_as_uint(a[q + 4]), false, false);
        b[q] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const bool up = lane & 8;
        c[q] = (up ? b[q + 2] : b[q]) + __shfl_xor(up ? b[q] : b[q + 2], 8, 64);
    }
    const bool up = lane & 4;
    float t = (up ? c[1] : c[0]) + __shfl_xor(up ? c[0] : c[1], 4, 64);
    t = t + __shfl_xor(t, 2, 64);
    return t + __shfl_xor(t, 1, 64);
}

// FP32 distances, d > 64: a wave holds 4 x 4 pairs, lane l its partial sums over
// coordinates l, l + 64, ..., and the butterfly follows, as in the recheck.
// Eight loads feed sixteen pairs.  The tree of n = 4096, d = 128: 0.81 ms with a
// whole butterfly for each pair, 0.41 with the halving one.
__global__ __launch_bounds__(256) void k_dense_f32(const float *__restrict__ X, int64_t n, int64_t d, int64_t ld,
                                                   int64_t nd, float *__restrict__ D, DenseState *__restrict__ st) {
    constexpr int B = 4;
    if (blockIdx.y < blockIdx.x) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t I0 = (int64_t)blockIdx.x * 4 * B, J0 = (int64_t)blockIdx.y * 4 * B + B * w;
    const float inf = (float)__builtin_huge_val();
    bool big = false;
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
        const float *xi[B], *xj[B];
#pragma unroll
        for (int a = 0; a < B; ++a) {
            xi[a] = X + min(I0 + B * s + a, n - 1) * ld;
            xj[a] = X + min(J0 + a, n - 1) * ld;
        }
        float acc[B][B];
#pragma unroll
        for (int a = 0; a < B; ++a)
#pragma unroll
            for (int b = 0; b < B; ++b) acc[a][b] = 0.0f;
#pragma unroll 2
        for (int64_t t = lane; t < d; t += 64) {
            float p[B], q[B];
#pragma unroll
            for (int a = 0; a < B; ++a) {
                p[a] = xi[a][t];
                q[a] = xj[a][t];
            }
#pragma unroll
            for (int a = 0; a < B; ++a)
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const float df = p[a] - q[b];
                    acc[a][b] = fmaf(df, df, acc[a][b]);
                }
        }
        float v[B * B];
#pragma unroll
        for (int q = 0; q < B * B; ++q) v[q] = acc[q / B][q % B];
        const float mine = sum_scatter16(v, lane);
        big |= too_big(mine);
        // lanes 4 q .. 4 q + 3 hold pair q = (a, b): the first writes it, the second its mirror
        const int q = lane >> 2;
        const int64_t i = I0 + B * s + q / B, j = J0 + q % B;
        if ((lane & 3) == 0 && i < n && j < nd) D[i * nd + j] = i == j || j >= n ? inf : mine;
        if ((lane & 3) == 1 && i < n && j < n) D[j * nd + i] = i == j ? inf : mine;
    }
    if (big) st->bad = 1;
}

// FP64 distances: left to right over the coordinates, one thread per pair.
__global__ __launch_bounds__(256) void k_dense_f64(const float *__restrict__ X, int64_t n, int64_t d, int64_t ld,
                                                   int64_t nd, double *__restrict__ D, DenseState *__restrict__ st) {
    constexpr int C = 32;  // coordinates per chunk
    if (blockIdx.y < blockIdx.x) return;
    __shared__ double tile[DT][DT + 1];
    __shared__ float xi[DT][C], xj[C][DT + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t I0 = (int64_t)blockIdx.x * DT, J0 = (int64_t)blockIdx.y * DT;
    double v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = 0.0;
    for (int64_t c = 0; c < d; c += C) {
        const int m = (int)min((int64_t)C, d - c);
        __syncthreads();
        load_rows<C>(X, n, d, ld, I0, c, [&](int r, int t, float x) { xi[r][t] = x; });
        load_rows<C>(X, n, d, ld, J0, c, [&](int r, int t, float x) { xj[t][r] = x; });
        __syncthreads();
#pragma unroll 2
        for (int t = 0; t < m; ++t) {
            const double y = (double)xj[t][lane];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const double df = (double)xi[16 * w + r][t] - y;
                const double sq = df * df;
                v[r] = v[r] + sq;
            }
        }
    }
    bool big = false;
#pragma unroll
    for (int r = 0; r < 16; ++r) big |= too_big(v[r]);
    if (big) st->bad = 1;
    put_tile(tile, v, n, nd, I0, J0, D);
}

// Every point its own component; no edges yet (0, 0: valid ids for what reads
// them before the host knows whether the tree is whole).
__global__ void k_dense_init(int64_t n, int32_t *__restrict__ comp, int32_t *__restrict__ eu, int32_t *__restrict__ ev,
                             DenseState *__restrict__ st) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *st = DenseState{(int32_t)n, 0, 0, 0, 0, 0};
    if (i >= n) return;
    comp[i] = (int32_t)i;
    eu[i] = ev[i] = 0;
}

struct RoundLDS {
    unsigned long long k1[DENSE_MAX_N];  // a component's least D^2
    uint32_t k2[DENSE_MAX_N];            // then its edge, smaller id in the high half
    uint16_t comp[DENSE_MAX_N + 4];
    uint16_t par[DENSE_MAX_N];
    uint16_t id[DENSE_MAX_N];
    int32_t last, edges, ncomp, bad;
};

// One Boruvka round.  A wave per row finds its lightest edge to another
// component, (D^2, j): of a row's equal distances the smallest j has the
// smallest (smaller id, larger id).  The last workgroup to finish joins the
// components: the lightest edge of each by two minima (D^2, then the ids), the
// roots of the pairs that chose the same edge, pointer jumping and new labels.
// D^2 is nonnegative, so its bits order like the values.
template <class T>
__global__ __launch_bounds__(DB) void k_dense_round(int64_t n, int64_t nd, const T *__restrict__ D, int32_t *__restrict__ comp,
                                                    unsigned long long *__restrict__ rowv, int32_t *__restrict__ rowj,
                                                    int32_t *__restrict__ eu, int32_t *__restrict__ ev,
                                                    DenseState *__restrict__ st) {
    using U = typename std::conditional<sizeof(T) == 4, uint32_t, unsigned long long>::type;
    __shared__ RoundLDS S;
    if (st->ncomp <= 1 || st->bad) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nn = (int)n;
    const int i = (int)blockIdx.x * (DB / 64) + (tid >> 6);
    constexpr int V = 16 / sizeof(T);  // values per load
    typedef U Vec __attribute__((ext_vector_type(V)));
    // the labels of all columns, V of them next to each other as the loads are
    for (int q = tid; q < (int)nd; q += DB) S.comp[q] = q < nn ? (uint16_t)comp[q] : (uint16_t)0;
    __syncthreads();
    if (i < nn) {
        const int ci = S.comp[i];
        const Vec *row = reinterpret_cast<const Vec *>(D + (int64_t)i * nd);
        const int nv = (int)(nd / V);
        U bv = ~U(0);
        int bj = -1;
        // (every load of a batch is in flight before the first is looked at; the
        // padding's +inf is the row's own label's or above every distance)
        constexpr int AHEAD = 8;
        for (int q0 = 0; q0 < nv; q0 += 64 * AHEAD) {
            Vec v[AHEAD];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) v[a] = row[min(q0 + 64 * a + lane, nv - 1)];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                const int q = q0 + 64 * a + lane;
                if (q >= nv) continue;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    if (S.comp[q * V + e] != ci && v[a][e] < bv) {
                        bv = v[a][e];
                        bj = q * V + e;
                    }
                }
            }
        }
        if (bj >= nn) bj = -1;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const U ov = (U)__shfl_xor((unsigned long long)bv, o, 64);
            const int oj = __shfl_xor(bj, o, 64);
            if (ov < bv || (ov == bv && (uint32_t)oj < (uint32_t)bj)) {
                bv = ov;
                bj = oj;
            }
        }
        if (lane == 0) {
            rowv[i] = (unsigned long long)bv;
            rowj[i] = bj;
        }
    }
    // This workgroup's rows before its arrival, the others' before the reads.
    // (One fence per workgroup, between barriers, orders all its waves once their
    // stores have drained; each writes back the L2: with one per wave a round of n = 2000 took 46 us, 15 so.)
    drain_stores();
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        S.last = atomicAdd(&st->arrived, 1) == (int)gridDim.x - 1;
        __threadfence();
    }
    __syncthreads();
    if (!S.last) return;
    const int nc = st->ncomp;
    for (int c = tid; c < nc; c += DB) {
        S.k1[c] = ~0ull;
        S.k2[c] = ~0u;
    }
    if (tid == 0) {
        S.edges = st->edges;
        S.ncomp = 0;
        S.bad = 0;
    }
    __syncthreads();
    constexpr int PER = DENSE_MAX_N / DB;
    unsigned long long v[PER];
    int j[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int q = tid + e * DB;
        v[e] = ~0ull;
        j[e] = -1;
        if (q < nn) {
            v[e] = __hip_atomic_load(&rowv[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            j[e] = __hip_atomic_load(&rowj[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (j[e] >= 0) atomicMin(&S.k1[S.comp[q]], v[e]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int q = tid + e * DB;
        if (j[e] >= 0 && v[e] == S.k1[S.comp[q]])
            atomicMin(&S.k2[S.comp[q]], (uint32_t)min(q, j[e]) << 16 | (uint32_t)max(q, j[e]));
    }
    __syncthreads();
    // the other end's component
    for (int c = tid; c < nc; c += DB) {
        const uint32_t k = S.k2[c];
        if (k == ~0u) {
            S.bad = 1;
            S.par[c] = (uint16_t)c;
            continue;
        }
        const int ca = S.comp[k >> 16], cb = S.comp[k & 0xFFFFu];
        S.par[c] = (uint16_t)(ca == c ? cb : ca);
    }
    __syncthreads();
    int root[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int c = tid + e * DB;
        root[e] = 0;
        if (c < nc) {
            const int o = S.par[c];
            root[e] = o == c || (S.par[o] == c && S.k2[o] == S.k2[c] && c < o);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int c = tid + e * DB;
        if (c >= nc) continue;
        if (root[e]) {
            S.par[c] = (uint16_t)c;
            S.id[c] = (uint16_t)atomicAdd(&S.ncomp, 1);
        } else {
            const int at = atomicAdd(&S.edges, 1);
            if (at < nn - 1) {
                eu[at] = (int32_t)(S.k2[c] >> 16);
                ev[at] = (int32_t)(S.k2[c] & 0xFFFFu);
            }
        }
    }
    __syncthreads();
    // (in place: a pointer only ever moves to an ancestor, twice as far each time)
    for (int span = 1; span < nc; span *= 2) {
        bool moved = false;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int c = tid + e * DB;
            if (c >= nc) continue;
            const int p = S.par[c], g = S.par[p];
            if (g != p) {
                S.par[c] = (uint16_t)g;
                moved = true;
            }
        }
        if (!__syncthreads_or(moved)) break;
    }
    for (int q = tid; q < nn; q += DB) comp[q] = S.id[S.par[S.comp[q]]];
    if (tid == 0) {
        st->ncomp = S.ncomp;
        st->edges = S.edges;
        st->joined = nc;
        st->rounds = st->rounds + 1;
        st->arrived = 0;
        if (S.bad) st->bad = 1;
    }
}

struct RootLDS {
    uint32_t hop[2][2 * DENSE_MAX_N];  // an arc's successor (high half) and distance to the end of the tour
    uint16_t slot[2 * DENSE_MAX_N];    // an arc's place among those that leave its vertex
    uint16_t arc[2 * DENSE_MAX_N];     // the arc at a place
    uint16_t head[DENSE_MAX_N + 1];    // a vertex's first place
    int32_t cnt[DENSE_MAX_N];
    int32_t wsum[DB / 64];
};

// The tree rooted at vertex 0, in one workgroup: arcs 2 e = (u, v) and
// 2 e + 1 = (v, u), the Euler tour's successors (the arc after the twin around
// the vertex that the arc enters), pointer jumping in LDS, and the earlier of an
// edge's two arcs enters the child.
__global__ __launch_bounds__(DB) void k_dense_root(int64_t n, const int32_t *__restrict__ eu,
                                                   const int32_t *__restrict__ ev, const double *__restrict__ elen,
                                                   int32_t *__restrict__ parent, double *__restrict__ length,
                                                   DenseState *__restrict__ st) {
    __shared__ RootLDS S;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int nn = (int)n, m = nn - 1, arcs = 2 * m;
    if (st->bad || st->ncomp != 1 || st->edges != m) {
        __syncthreads();
        if (tid == 0) st->bad = 1;
        return;
    }
    constexpr int PER = DENSE_MAX_N / DB;
    for (int v = tid; v < nn; v += DB) S.cnt[v] = 0;
    __syncthreads();
    for (int a = tid; a < arcs; a += DB) {
        const int from = a & 1 ? ev[a >> 1] : eu[a >> 1];
        S.slot[a] = (uint16_t)atomicAdd(&S.cnt[from], 1);
    }
    __syncthreads();
    // exclusive scan of the degrees, PER consecutive vertices per thread
    int my[PER], sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int v = tid * PER + e;
        my[e] = sum;
        sum += v < nn ? S.cnt[v] : 0;
    }
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) S.wsum[w] = inc;
    __syncthreads();
    int base = inc - sum;
    for (int q = 0; q < w; ++q) base += S.wsum[q];
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (tid * PER + e < nn) S.head[tid * PER + e] = (uint16_t)(base + my[e]);
    if (tid == 0) S.head[nn] = (uint16_t)arcs;
    __syncthreads();
    for (int a = tid; a < arcs; a += DB) {
        const int from = a & 1 ? ev[a >> 1] : eu[a >> 1];
        const int p = S.head[from] + S.slot[a];
        S.slot[a] = (uint16_t)p;
        S.arc[p] = (uint16_t)a;
    }
    __syncthreads();
    const int first = S.arc[S.head[0]];
    for (int a = tid; a < arcs; a += DB) {
        const int to = a & 1 ? eu[a >> 1] : ev[a >> 1];
        int p = S.slot[a ^ 1] + 1;
        if (p == S.head[to + 1]) p = S.head[to];
        const int nx = S.arc[p];
        S.hop[0][a] = nx == first ? (uint32_t)a << 16 : (uint32_t)nx << 16 | 1u;
    }
    __syncthreads();
    int cur = 0;
    for (int span = 1; span < arcs; span *= 2) {
        for (int a = tid; a < arcs; a += DB) {
            const uint32_t h = S.hop[cur][a], g = S.hop[cur][h >> 16];
            S.hop[cur ^ 1][a] = (g & 0xFFFF0000u) | ((h & 0xFFFFu) + (g & 0xFFFFu));
        }
        cur ^= 1;
        __syncthreads();
    }
    for (int e = tid; e < m; e += DB) {
        const bool down = (S.hop[cur][2 * e] & 0xFFFFu) > (S.hop[cur][2 * e + 1] & 0xFFFFu);
        const int child = down ? ev[e] : eu[e];
        parent[child] = down ? eu[e] : ev[e];
        length[child] = elen[e];
    }
    if (tid == 0) {
        parent[0] = -1;
        length[0] = 0.0;
        // the tour covers every arc exactly when the edges form one tree
        if ((int)(S.hop[cur][first] & 0xFFFFu) != arcs - 1) st->bad = 1;
    }
}

}  // namespace

// Columns of a row of the matrix: whole 16-byte loads.
static int64_t row_stride(int64_t n) { return (n + 3) / 4 * 4; }

size_t dense_bytes(int64_t n, bool f64) {
    return align_up((size_t)(n * row_stride(n)) * (f64 ? 8 : 4), 256) + align_up((size_t)n * 8, 256) + align_up((size_t)n * 4, 256);
}

void launch_dense_tree(const DenseArgs &A, hipStream_t s) {
    const int64_t n = A.n;
    ISO_REQUIRE(n >= 2 && n <= DENSE_MAX_N && A.d >= 1 && A.ld >= A.d, ISO_ERR_INTERNAL, "dense tree of %lld points",
                (long long)n);
    char *p = static_cast<char *>(A.buf);
    float *const Df = reinterpret_cast<float *>(p);
    double *const Dd = reinterpret_cast<double *>(p);
    const int64_t nd = row_stride(n);
    p += align_up((size_t)(n * nd) * (A.f64 ? 8 : 4), 256);
    unsigned long long *const rowv = reinterpret_cast<unsigned long long *>(p);
    p += align_up((size_t)n * 8, 256);
    int32_t *const rowj = reinterpret_cast<int32_t *>(p);
    hipLaunchKernelGGL(k_dense_init, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, A.comp, A.eu, A.ev, A.st);
    LAUNCH_CHECK();
    const unsigned t64 = (unsigned)((n + DT - 1) / DT), t16 = (unsigned)((n + 15) / 16);
    if (A.f64) {
        hipLaunchKernelGGL(k_dense_f64, dim3(t64, t64), dim3(256), 0, s, A.X, n, A.d, A.ld, nd, Dd, A.st);
    } else if (A.d <= 64) {
        auto kern = A.d <= 8    ? k_dense_f32_low<8>
                    : A.d <= 16 ? k_dense_f32_low<16>
                    : A.d <= 32 ? k_dense_f32_low<32>
                                : k_dense_f32_low<64>;
        hipLaunchKernelGGL(kern, dim3(t64, t64), dim3(256), 0, s, A.X, n, A.d, A.ld, nd, Df, A.st);
    } else {
        hipLaunchKernelGGL(k_dense_f32, dim3(t16, t16), dim3(256), 0, s, A.X, n, A.d, A.ld, nd, Df, A.st);
    }
    LAUNCH_CHECK();
    const dim3 g((unsigned)((n + DB / 64 - 1) / (DB / 64)));
    for (int64_t c = 1; c < n; c *= 2) {  // a round at least halves the components
        if (A.f64)
            hipLaunchKernelGGL(k_dense_round<double>, g, dim3(DB), 0, s, n, nd, Dd, A.comp, rowv, rowj, A.eu, A.ev, A.st);
        else
            hipLaunchKernelGGL(k_dense_round<float>, g, dim3(DB), 0, s, n, nd, Df, A.comp, rowv, rowj, A.eu, A.ev, A.st);
        LAUNCH_CHECK();
    }
}

void launch_dense_root(const DenseArgs &A, const double *elen, int32_t *parent, double *length, hipStream_t s) {
    hipLaunchKernelGGL(k_dense_root, dim3(1), dim3(DB), 0, s, A.n, A.eu, A.ev, elen, parent, length, A.st);
    LAUNCH_CHECK();
}

}  // namespace iso
