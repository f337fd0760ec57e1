// tree.hip -- optimal k-subpartition of a weighted tree on gfx950
// (Sec. 2.2 Algorithms 1-2; labels as in Algorithm 4).
//
// Algorithm 1 visits the vertices in x-order (depth descending, id ascending)
// and either cuts a vertex from its parent, joins it to its parent, or
// discards it.  A vertex's decision depends only on its subtree, and the
// parent folds its children's contributions in ascending id, so any order in
// which children come before their parent and siblings ascend gives the
// sequential algorithm's FP64 arithmetic bit for bit.  Here that order is the
// depth-first postorder with the children ascending, which turns Algorithm 1
// into a stack machine over a stream of records (k_walk0, k_walk): one wave walks a
// piece of the tree, its 64 lanes hold 64 thresholds, and the open vertices'
// (p, omega) stay in registers and LDS.
//
// Pieces: the vertices are split into tiers by subtree size (at most 32, 1024,
// 16384 vertices, larger); a piece is a connected set of vertices of one tier.
// The pieces of a tier are independent (one launch, many waves).  On trees
// whose depth is small against n (MSTs of clustered data: depth 127 at
// n = 200,000) the lowest tier holds 98 % of the vertices and the top one a few
// hundred, so a pass over the whole tree is four short launches instead of one
// per level.  An upper tier's piece has few vertices but thousands of children
// in lower tiers (hubs): their contributions, its feeds, are brought to LDS by
// the workgroup's other waves, and the walking wave only adds them in order.
//
// Bisection (Algorithm 2) is speculative: one pass evaluates 64 thresholds, and
// the walk over the answers repeats the sequential bisection's arithmetic, so
// the sequence of brackets is exactly the sequential one.  Besides the number
// of cuts a lane reports the largest threshold at which one of its cut vertices
// still is cut (num / den, corrected to the last bit): when a bracket's upper
// end has exactly k cuts that value predicts the final threshold, and the next
// pass evaluates the midpoints along the path the bisection then takes, down
// to the last bit.  The image-like, mixture and blobs trees need one pass along
// the all-YES path from the wide power-of-two bracket and one along the
// predicted path (10 passes of six bisection steps each before).  A wrong
// prediction costs passes, never the result.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <utility>
#include <vector>

#include "common.hpp"

namespace iso {

namespace {

constexpr int M = 64;           // thresholds (lanes) per pass and search
constexpr int HI_LANE = M - 1;  // always evaluates the bracket's upper end
constexpr int NMID = M - 1;     // midpoints per pass
constexpr int TREE_LEVELS = 6;  // bisection levels whose midpoints fill the other lanes
// Candidate layouts of a pass: MODE_TREE the midpoints of the next six levels
// in heap order; MODE_DOWN / MODE_UP the midpoints along the path on which every
// answer is YES (NO), while the bracket's lower (upper) end has never moved;
// MODE_PATH those along the path towards a predicted threshold; MODE_RECORD
// every lane at the final threshold, to record the decisions.
constexpr int MODE_TREE = 0, MODE_DOWN = 1, MODE_UP = 2, MODE_PATH = 3, MODE_RECORD = 4;

constexpr int MAXG = 32;        // searches (values of k) that run together
constexpr int CUT_CAP = 4096;   // cut vertices recorded per search; more take the sorting path

constexpr int NT = 4;  // tiers
// Largest subtree of tier 0, 1, 2.  32 bounds the stack of a tier-0 piece (16
// open vertices: 16 KB of LDS, ten waves per CU).
constexpr int64_t TIER_SIZE[NT - 1] = {32, 1024, 16384};
constexpr int STACK = 16;       // open accumulators a wave keeps in LDS
constexpr int FEEDERS = 7;      // waves of an upper-tier workgroup that bring the feeds (two waves per SIMD in all)
constexpr int FEED_PER = 6;     // feeds each of them holds per chunk
constexpr int CHUNK = FEEDERS * FEED_PER;
constexpr int WIN = 8;          // feeds the walking wave reads from LDS ahead

// One search: the bisection for one k.
struct Search {
    double alpha, beta;
    double hi_t;      // largest threshold of a cut vertex at beta
    double i_k;
    int32_t hi_cnt;   // cuts at beta (-1: not evaluated yet)
    int32_t k, iters, max_iters, passes;
    int32_t done;     // the bracket is final
    int32_t final;    // and the last pass recorded the decisions at beta
    int32_t mode, rec;  // this pass's candidate layout and recorded lane (-1: none)
    int32_t slow;     // the last predicted path was left early
    int32_t jstar, pad;
};

struct TreeState {
    double alpha0_raw, beta0_raw, alpha0, beta0;
    double phi_sum, phi_min, om_sum, om_min, p_sum, p_min;
    double sigma;
    int32_t bad, maxdepth;
    int32_t nops[NT], npiece[NT], nfeed[NT];  // per tier: records, pieces, feeds (tier 0 has none: all tiers' contributions)
};

template <class T>
__global__ void k_fill_t(T *p, T v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

template <class T>
void fill_t(T *p, T v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    unsigned g = grid_for(n, 256);
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_t<T>, dim3(g), dim3(256), 0, s, p, v, n);
    LAUNCH_CHECK();
}

// ------------------------------------------------------------------ validation, child lists, depth-first order

__global__ void k_init(TreeState *__restrict__ st, Search *__restrict__ S, int32_t ns, int32_t k0, int32_t max_iters,
                       double sigma, int32_t *__restrict__ cnt, unsigned long long *__restrict__ thr,
                       int32_t *__restrict__ ncut) {
    for (int i = threadIdx.x; i < 2 * MAXG * M; i += blockDim.x) {
        cnt[i] = 0;
        thr[i] = 0;
    }
    if (threadIdx.x == 0) {
        TreeState t{};
        t.sigma = sigma;
        *st = t;
    }
    if ((int)threadIdx.x < ns) {
        Search x{};
        x.k = k0 + (int)threadIdx.x;
        x.max_iters = max_iters;
        x.hi_cnt = -1;
        x.rec = -1;
        S[threadIdx.x] = x;
        ncut[threadIdx.x] = 0;
    }
}

// Flags malformed entries; child-list sort keys (parent + 1, 0 for the root and
// for malformed vertices, so that what follows stays in bounds).
__global__ void k_check_tree(const int32_t *__restrict__ parent, const double *__restrict__ length, int64_t n,
                             int32_t root, uint32_t *__restrict__ ckey, uint32_t *__restrict__ cval,
                             TreeState *__restrict__ st) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int32_t p = parent[v];
    bool bad;
    if (v == root) {
        bad = p != -1;
        ckey[v] = 0;
    } else {
        const double L = length[v];
        const bool out = p < 0 || p >= n || p == v;
        bad = out || !(L >= 0.0) || !isfinite(L);
        ckey[v] = out ? 0u : (uint32_t)(p + 1);
    }
    cval[v] = (uint32_t)v;
    if (bad) atomicOr(&st->bad, 1);
}

// koff[u] = position of u's first child in the sorted child lists (cval + 1):
// the number of keys <= u, less the root's.
__global__ void k_child_off(const uint32_t *__restrict__ ckey, int64_t n, int32_t *__restrict__ koff) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u > n) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ckey[mid] <= (uint32_t)u)
            lo = mid + 1;
        else
            hi = mid;
    }
    koff[u] = (int32_t)(lo - 1);
}

// The depth-first tour as a linked list of 2n arcs: arc v enters v (from its
// parent; arc root starts the tour), arc n + v leaves it.  Entering v is
// followed by entering its first child, or by leaving v; leaving v by entering
// its next sibling, or by leaving its parent; leaving the root ends the tour.
// Thread i takes the vertex at place i of the sorted child lists.
__global__ void k_tour_links(const uint32_t *__restrict__ ckey, const uint32_t *__restrict__ cval,
                             const int32_t *__restrict__ koff, int64_t n, int32_t *__restrict__ nxt,
                             int32_t *__restrict__ own, int32_t *__restrict__ place) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = (int32_t)cval[i];
    const uint32_t key = ckey[i];
    const int32_t a0 = koff[v], a1 = koff[v + 1];
    nxt[v] = a0 < a1 ? (int32_t)cval[a0 + 1] : (int32_t)(n + v);
    int32_t up = -1;
    if (key > 0) up = (i + 1 < n && ckey[i + 1] == key) ? (int32_t)cval[i + 1] : (int32_t)(n + key - 1);
    nxt[n + v] = up;
    own[v] = -1;
    own[n + v] = -1;
    place[v] = (int32_t)i;
}

// List ranking.  One element of every group of eight is a splitter (a hashed
// one, so that no order of the list can keep them apart; the head in its own
// group); each splitter walks to the next one, and the splitters form a list
// an eighth as long, with the walked lengths as weights, ranked the same way;
// a list of at most RANK_LDS elements is ranked in one workgroup by pointer
// jumping.  Two weights per element: the arcs and the entering arcs from it to
// the tour's end.  (Jumping over all 2n arcs takes log2(2n) rounds over memory.)
// The links are injective also for a malformed parent array, so every walk
// ends at a splitter or at the list's end.
constexpr int RANK_LDS = 8192;
__device__ inline int32_t splitter_of(int32_t j, int32_t m, int32_t head) {
    if (j == (head >> 3)) return head;
    uint32_t h = (uint32_t)j * 0x9E3779B1u;
    h ^= h >> 15;
    const int32_t x = 8 * j + (int32_t)(h & 7u);
    return x < m ? x : 8 * j;
}

struct RankLevel {
    const int32_t *nxt, *len, *ent;  // links and weights (level 0: weight 1, entering arcs are the first half)
    int32_t *own, *olen, *oent;      // splitter of every element, distance from it
    int32_t *rlen, *rent;            // ranks
    int32_t m, head, half;           // elements, the list's head, level 0: n (else 0)
};

__global__ void k_rank_walk(RankLevel L, int32_t m1, int32_t *__restrict__ nxt1, int32_t *__restrict__ len1,
                            int32_t *__restrict__ ent1, int32_t *__restrict__ own1) {
    const int32_t j = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (j >= m1) return;
    int32_t x = splitter_of(j, L.m, L.head);
    int32_t len = 0, ent = 0;
    while (true) {
        L.own[x] = j;
        L.olen[x] = len;
        L.oent[x] = ent;
        len += L.half ? 1 : L.len[x];
        ent += L.half ? (x < L.half ? 1 : 0) : L.ent[x];
        x = L.nxt[x];
        if (x < 0 || splitter_of(x >> 3, L.m, L.head) == x) break;
    }
    nxt1[j] = x < 0 ? -1 : x >> 3;
    len1[j] = len;
    ent1[j] = ent;
    own1[j] = -1;
}

__global__ __launch_bounds__(1024) void k_rank_lds(RankLevel L) {
    __shared__ int32_t nx[RANK_LDS], ln[RANK_LDS], en[RANK_LDS];
    constexpr int PER = RANK_LDS / 1024;
    for (int x = threadIdx.x; x < L.m; x += 1024) {
        nx[x] = L.nxt[x];
        ln[x] = L.half ? 1 : L.len[x];
        en[x] = L.half ? (x < L.half ? 1 : 0) : L.ent[x];
    }
    __syncthreads();
    for (int32_t span = 1; span < L.m; span *= 2) {
        int32_t a[PER], b[PER], c[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int x = threadIdx.x + 1024 * u;
            a[u] = -1;
            b[u] = c[u] = 0;
            if (x < L.m) {
                const int32_t y = nx[x];
                if (y >= 0) {
                    a[u] = nx[y];
                    b[u] = ln[y];
                    c[u] = en[y];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int x = threadIdx.x + 1024 * u;
            if (x < L.m) {
                nx[x] = a[u];
                ln[x] += b[u];
                en[x] += c[u];
            }
        }
        __syncthreads();
    }
    for (int x = threadIdx.x; x < L.m; x += 1024) {
        L.rlen[x] = ln[x];
        L.rent[x] = en[x];
    }
}

__global__ void k_rank_back(RankLevel L, const int32_t *__restrict__ rlen1, const int32_t *__restrict__ rent1) {
    const int32_t x = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (x >= L.m) return;
    const int32_t j = L.own[x];
    L.rlen[x] = j < 0 ? 0 : rlen1[j] - L.olen[x];
    L.rent[x] = j < 0 ? 0 : rent1[j] - L.oent[x];
}

// Depth, subtree size and postorder place of every vertex from its two arcs'
// ranks; the tour from the root has 2n arcs exactly when the edges form a tree.
__global__ __launch_bounds__(256) void k_place(const int32_t *__restrict__ rlen, const int32_t *__restrict__ rent,
                                               int64_t n, int32_t root, int32_t *__restrict__ depth,
                                               int32_t *__restrict__ size, int32_t *__restrict__ pv,
                                               TreeState *__restrict__ st) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t dep = 0;
    if (v < n) {
        const int32_t rd = rlen[v], ed = rent[v], ru = rlen[n + v], eu = rent[n + v];
        if (v == root && rd != (int32_t)(2 * n)) atomicOr(&st->bad, 2);
        dep = rd - 2 * ed;
        depth[v] = dep;
        size[v] = ed - eu;
        const int64_t post = n - (int64_t)(ru - eu);
        if (post >= 0 && post < n) pv[post] = (int32_t)v;
    }
    for (int off = 32; off >= 1; off >>= 1) dep = max(dep, __shfl_xor(dep, off, 64));
    // (most waves find a larger depth there already: one atomic per wave to one address took 37 us at n = 200,000)
    if ((threadIdx.x & 63) == 0 &&
        dep > __hip_atomic_load(&st->maxdepth, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&st->maxdepth, dep);
}

// ------------------------------------------------------------------ weights (eqs. 2.1-2.2)

__device__ inline double flow_of(double dist, double sigma, int phi_kind) {
    return (phi_kind == ISO_PHI_GAUSS_SQ) ? exp(-(dist * dist) / (2.0 * sigma * sigma)) : exp(-dist / sigma);
}

__global__ void k_phi(const int32_t *__restrict__ parent, const double *__restrict__ length, int64_t n,
                      const TreeState *__restrict__ st, int phi_kind, double *__restrict__ phi,
                      double *__restrict__ p0) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    phi[v] = parent[v] >= 0 ? flow_of(length[v], st->sigma, phi_kind) : 0.0;
    p0[v] = 0.0;
}

// omega0(v): sum over tree neighbours w of v in ascending w of phi(vw),
// starting from +0.0 (children come sorted by id; the parent is merged in).
// A vertex with more than OMEGA_OWN children is summed by its whole wave: the
// lanes load 64 children at a time and every lane adds them in order (a hub's
// own thread would wait for a round trip per batch: 720 children took 85 us).
constexpr int OMEGA_OWN = 16;
__global__ __launch_bounds__(256) void k_omega_tree(const int32_t *__restrict__ parent, const double *__restrict__ phi,
                                                    const uint32_t *__restrict__ kids, const int32_t *__restrict__ koff,
                                                    int64_t n, double *__restrict__ om0) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    int32_t p = -1, a0 = 0, a1 = 0;
    double fv = 0.0;
    if (v < n) {
        p = parent[v];
        fv = phi[v];
        a0 = koff[v];
        a1 = koff[v + 1];
    }
    if (v < n && a1 - a0 <= OMEGA_OWN) {
        double s = 0.0;
        bool parent_done = p < 0;
        int32_t c[OMEGA_OWN];
        double f[OMEGA_OWN];
#pragma unroll
        for (int u = 0; u < OMEGA_OWN; ++u) c[u] = a0 + u < a1 ? (int32_t)kids[a0 + u] : (int32_t)v;
#pragma unroll
        for (int u = 0; u < OMEGA_OWN; ++u) f[u] = phi[c[u]];
#pragma unroll
        for (int u = 0; u < OMEGA_OWN; ++u) {
            if (a0 + u < a1) {
                if (!parent_done && p < c[u]) {
                    s = s + fv;
                    parent_done = true;
                }
                s = s + f[u];
            }
        }
        if (!parent_done) s = s + fv;
        om0[v] = s;
    }
    uint64_t hubs = __ballot(v < n && a1 - a0 > OMEGA_OWN);
    while (hubs) {
        const int l = __ffsll((unsigned long long)hubs) - 1;
        hubs &= hubs - 1;
        const int32_t hp = __shfl(p, l, 64), h0 = __shfl(a0, l, 64), h1 = __shfl(a1, l, 64);
        const double hf = __shfl(fv, l, 64);
        double s = 0.0;
        bool parent_done = hp < 0;
        for (int32_t b = h0; b < h1; b += 64) {
            const int32_t c = (int32_t)kids[min(b + lane, h1 - 1)];
            const double f = phi[c];
            const int nb = min(64, h1 - b);
            for (int u = 0; u < nb; ++u) {
                if (!parent_done && hp < __shfl(c, u, 64)) {
                    s = s + hf;
                    parent_done = true;
                }
                s = s + __shfl(f, u, 64);
            }
        }
        if (!parent_done) s = s + hf;
        if (lane == l) om0[v] = s;
    }
}

// Sums and minima of phi (tree edges), omega0 and p0; bracket of Algorithm 2.
// k_stats_part: STATS_BLOCKS workgroups, each over a contiguous range of the
// vertices, write partial sums and minima; k_stats (one workgroup) combines
// them in a fixed order and sets the bracket.
constexpr int STATS_BLOCKS = 256;

__global__ __launch_bounds__(256) void k_stats_part(const int32_t *__restrict__ parent, const double *__restrict__ phi,
                                                    const double *__restrict__ om0, const double *__restrict__ p0,
                                                    int64_t n, double *__restrict__ part) {
    __shared__ double s_sum[3][256];
    __shared__ double s_min[3][256];
    const int64_t per = (n + STATS_BLOCKS - 1) / STATS_BLOCKS;
    const int64_t lo = (int64_t)blockIdx.x * per, hi = min(n, lo + per);
    double ps = 0.0, os = 0.0, qs = 0.0;
    double pm = __builtin_huge_val(), om = __builtin_huge_val(), qm = __builtin_huge_val();
    for (int64_t v = lo + threadIdx.x; v < hi; v += 256) {
        const double f = phi[v], o = om0[v], q = p0[v];
        if (parent[v] >= 0) {
            ps = ps + f;
            pm = fmin(pm, f);
        }
        os = os + o;
        om = fmin(om, o);
        qs = qs + q;
        qm = fmin(qm, q);
    }
    s_sum[0][threadIdx.x] = ps;
    s_sum[1][threadIdx.x] = os;
    s_sum[2][threadIdx.x] = qs;
    s_min[0][threadIdx.x] = pm;
    s_min[1][threadIdx.x] = om;
    s_min[2][threadIdx.x] = qm;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int q = 0; q < 3; ++q) {
                s_sum[q][threadIdx.x] = s_sum[q][threadIdx.x] + s_sum[q][threadIdx.x + w];
                s_min[q][threadIdx.x] = fmin(s_min[q][threadIdx.x], s_min[q][threadIdx.x + w]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 3) {
        part[blockIdx.x * 6 + threadIdx.x] = s_sum[threadIdx.x][0];
        part[blockIdx.x * 6 + 3 + threadIdx.x] = s_min[threadIdx.x][0];
    }
}

__global__ __launch_bounds__(256) void k_stats(const double *__restrict__ part, int bracket,
                                               TreeState *__restrict__ st) {
    static_assert(STATS_BLOCKS == 256, "one partial per thread");
    __shared__ double s_sum[3][256];
    __shared__ double s_min[3][256];
    for (int q = 0; q < 3; ++q) {
        s_sum[q][threadIdx.x] = part[threadIdx.x * 6 + q];
        s_min[q][threadIdx.x] = part[threadIdx.x * 6 + 3 + q];
    }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int q = 0; q < 3; ++q) {
                s_sum[q][threadIdx.x] = s_sum[q][threadIdx.x] + s_sum[q][threadIdx.x + w];
                s_min[q][threadIdx.x] = fmin(s_min[q][threadIdx.x], s_min[q][threadIdx.x + w]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        st->phi_sum = s_sum[0][0];
        st->om_sum = s_sum[1][0];
        st->p_sum = s_sum[2][0];
        st->phi_min = s_min[0][0];
        st->om_min = s_min[1][0];
        st->p_min = s_min[2][0];
        const double a0 = (st->phi_min + st->p_min) / st->om_sum;
        const double b0 = (st->phi_sum + st->p_sum) / st->om_min;
        st->alpha0_raw = a0;
        st->beta0_raw = b0;
        double a, b;
        if (bracket == ISO_BRACKET_PAPER) {
            a = a0;
            b = nextafter(b0, __builtin_huge_val());
        } else {
            int e;
            if (a0 > 0.0) {
                frexp(a0, &e);
                a = ldexp(1.0, e - 1);
            } else {
                a = 0.0;
            }
            frexp(b0, &e);
            b = ldexp(1.0, e);
        }
        st->alpha0 = a;
        st->beta0 = b;
        if (!(b0 > 0.0) || !isfinite(b0)) st->bad |= 4;
    }
}

// ------------------------------------------------------------------ record streams

// One step of the stack machine: a vertex (its decision, then the fold of its
// contribution into its parent's accumulators), or a run of feeds of one vertex
// to fold (consecutive children in lower tiers).
struct __attribute__((aligned(16))) Op {
    double fe;       // phi of the parent edge (0 at the root)
    double om0, p0;  // tier-0 leaf: its weight and potential; upper tiers: om0's low word = feeds before this record
    double iw, ip;   // OP_FIRST: the parent's weight and potential, which its first child's fold starts from;
                     // OP_ROOT: iw's low word = slot of its contribution
    int32_t v;       // vertex; OP_FEED: slot of the run's first feed
    int32_t flags;
};
static_assert(sizeof(Op) == 48, "a record is three 16-byte pieces");
constexpr int OP_LEAF = 1;   // a vertex without children
constexpr int OP_FEED = 2;   // a run of feeds
constexpr int OP_FIRST = 4;  // the (run's first) child is the first of its parent
constexpr int OP_ROOT = 8;   // the piece's last vertex
constexpr int OP_TREE = 16;  // the tree's root

// A child in a lower tier: a leaf, evaluated by the wave that brings it, or
// (v < 0) the root of a piece, whose contribution is in the buffer at `slot`.
// (A run's leaf has a slot too when the walk may spill to it.)
struct __attribute__((aligned(16))) Feed {
    double fe, om0, p0;
    int32_t v, slot;
};

__device__ inline int tier_of(int32_t size) {
    return size <= TIER_SIZE[0] ? 0 : size <= TIER_SIZE[1] ? 1 : size <= TIER_SIZE[2] ? 2 : 3;
}

// Counters of the streams' layout, in postorder: records, pieces and feeds per
// tier (no feeds in tier 0: that counter numbers the contribution slots).
constexpr int NCTR = 3 * NT;
struct OpPlace {
    int t, tp;            // the vertex's tier and its parent's (NT at the root)
    bool vertex;          // it has a record of its own (leaves fed to an upper tier have none)
    bool feed, run;       // a feed of its parent; the first one of a run
    bool slot;            // it has a contribution slot
};
__device__ inline OpPlace op_place(int32_t v, int32_t root, const int32_t *size, const int32_t *parent,
                                   const uint32_t *cval, const int32_t *place, const int32_t *koff) {
    OpPlace q;
    const int32_t s = size[v];
    const int32_t u = v == root ? -1 : parent[v];
    q.t = tier_of(s);
    q.tp = u < 0 ? NT : tier_of(size[u]);
    q.feed = u >= 0 && q.tp != q.t;
    q.vertex = !(q.feed && s == 1);
    q.run = q.slot = false;
    if (q.feed) {
        const int32_t at = place[v];
        const bool first = at == koff[u] + 1;
        q.run = first || tier_of(size[cval[at - 1]]) == q.tp;  // first child, or after a sibling with a record
        q.slot = s > 1 || first;
    }
    return q;
}

constexpr int OPB = 1024;  // postorder places per workgroup
constexpr int RUN0 = 32;   // records a wave of tier 0 takes, to the next piece's end
static_assert(RUN0 >= TIER_SIZE[0], "a piece covers at most one multiple of RUN0");
// COUNT: per-workgroup totals of the counters.  Otherwise the records: every
// thread's places in the streams from the scanned totals and the block's scan.
template <bool COUNT>
__global__ __launch_bounds__(OPB) void k_ops(const int32_t *__restrict__ pv, const int32_t *__restrict__ size,
                                             const int32_t *__restrict__ parent, const uint32_t *__restrict__ cval,
                                             const int32_t *__restrict__ place, const int32_t *__restrict__ koff,
                                             const double *__restrict__ phi, const double *__restrict__ om0,
                                             const double *__restrict__ p0, int64_t n, int32_t root, int64_t nb,
                                             int32_t *__restrict__ ctr, const TreeState *__restrict__ st,
                                             Op *__restrict__ ops, Feed *__restrict__ feeds, int32_t *__restrict__ pend,
                                             int32_t *__restrict__ pfeed, int32_t *__restrict__ start0) {
    if (st->bad) return;
    __shared__ int32_t wsum[OPB / 64][NCTR];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t i = (int64_t)blockIdx.x * OPB + tid;
    const bool live = i < n;
    const int32_t v = live ? pv[i] : root;
    const OpPlace q = op_place(v, root, size, parent, cval, place, koff);
    int32_t pre[NCTR];
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int c = 0; c < NCTR; ++c) {
        const int t = c % NT;
        bool f;
        if (c < NT)
            f = (q.vertex && q.t == t) || (q.run && q.tp == t);
        else if (c < 2 * NT)
            f = q.vertex && q.t == t && q.tp != q.t;
        else
            f = t == 0 ? q.slot : q.feed && q.tp == t;
        const uint64_t b = __ballot(live && f);
        pre[c] = __popcll(b & lt);
        if (lane == 0) wsum[w][c] = __popcll(b);
    }
    __syncthreads();
    if (COUNT) {
        if (tid < NCTR) {
            int32_t s = 0;
            for (int k = 0; k < OPB / 64; ++k) s += wsum[k][tid];
            ctr[(int64_t)tid * nb + blockIdx.x] = s;
        }
        return;
    }
    if (!live) return;
#pragma unroll
    for (int c = 0; c < NCTR; ++c) {
        pre[c] += ctr[(int64_t)c * nb + blockIdx.x];
        for (int k = 0; k < w; ++k) pre[c] += wsum[k][c];
    }
    // the streams, pieces and feeds of the tiers follow each other
    const int t = q.t, tp = q.tp;
    int32_t ob_t = 0, pb_t = 0, fb_t = 0, ob_p = 0, fb_p = 0;    // bases of t's and tp's streams, pieces, feeds
    int32_t op_t = 0, pi_t = 0, fd_t = 0, op_p = 0, fd_p = 0;    // this thread's places in them
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        const int32_t no = st->nops[c], npc = st->npiece[c], nf = c ? st->nfeed[c] : 0;
        ob_t += c < t ? no : 0;
        pb_t += c < t ? npc : 0;
        fb_t += c < t ? nf : 0;
        ob_p += c < tp ? no : 0;
        fb_p += c < tp ? nf : 0;
        op_t = c == t ? pre[c] : op_t;
        pi_t = c == t ? pre[NT + c] : pi_t;
        fd_t = c && c == t ? pre[2 * NT + c] : fd_t;
        op_p = c == tp ? pre[c] : op_p;
        fd_p = c == tp ? pre[2 * NT + c] : fd_p;
    }
    const int32_t u = v == root ? -1 : parent[v];
    const bool leaf = size[v] == 1;
    const double fe = v == root ? 0.0 : phi[v];
    const int first = (u >= 0 && place[v] == koff[u] + 1) ? OP_FIRST : 0;
    Op op{};
    op.iw = u >= 0 ? om0[u] : 0.0;
    op.ip = u >= 0 ? p0[u] : 0.0;
    const int32_t feed = fb_p + fd_p, slot = q.slot ? pre[2 * NT] : 0;
    if (q.feed) {
        feeds[feed] = Feed{fe, om0[v], p0[v], leaf ? v : -1, slot};
        if (q.run) {
            op.om0 = __hiloint2double(0, feed);
            op.v = slot;
            op.flags = OP_FEED | first;
            ops[(int64_t)ob_p + op_p] = op;
        }
    }
    if (q.vertex) {
        op.fe = fe;
        op.om0 = t == 0 ? om0[v] : __hiloint2double(0, fb_t + fd_t);
        op.p0 = p0[v];
        op.v = v;
        op.flags = (leaf ? OP_LEAF : 0) | first | (tp != t ? OP_ROOT : 0) | (v == root ? OP_TREE : 0);
        if (tp != t) {
            // the piece ends here: its records, and its tier's feeds, up to here
            op.iw = __hiloint2double(0, slot);
            pend[pb_t + pi_t] = op_t + 1;
            pfeed[pb_t + pi_t] = fd_t;
        }
        ops[(int64_t)ob_t + op_t] = op;
        if (t == 0 && tp != t) {
            // where a wave of tier 0 may begin: the first piece's end at or after every multiple of RUN0 records
            // (a piece is at most that long, so it covers at most one)
            const int32_t end = op_t + 1, begin = end - size[v];
            if (end / RUN0 != begin / RUN0) start0[end / RUN0] = end;
        }
    }
}

// Exclusive scans of the NCTR counters over the workgroups, and their totals.
__global__ __launch_bounds__(1024) void k_ops_scan(int32_t *__restrict__ ctr, int64_t nb, TreeState *__restrict__ st) {
    if (st->bad) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w >= NCTR) return;  // one wave per counter
    int32_t run = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += 64) {
        const int64_t b = b0 + lane;
        const int32_t x = b < nb ? ctr[(int64_t)w * nb + b] : 0;
        int32_t inc = x;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (b < nb) ctr[(int64_t)w * nb + b] = run + inc - x;
        run += __shfl(inc, 63, 64);
    }
    if (lane == 0) {
        const int t = w % NT;
        if (w < NT)
            st->nops[t] = run;
        else if (w < 2 * NT)
            st->npiece[t] = run;
        else
            st->nfeed[t] = run;
    }
}

// ------------------------------------------------------------------ the bisection's bookkeeping

// Largest double N with the vertex cut, i.e. the smallest N with num <= fl(N den).
__device__ inline double cut_threshold(double num, double den) {
    double t = num / den;
    if (t * den < num) t = nextafter(t, __builtin_huge_val());
    const double d = nextafter(t, 0.0);
    if (d * den >= num) t = d;
    return t;
}

// Walks the answers of the pass just run (YES: at least k cuts => beta = mid,
// else alpha = mid), then chooses the next pass's thresholds.  One wave.  Every
// threshold repeats the midpoint arithmetic the sequential bisection performs
// on its way to it.  `recorded`: the pass wrote this search's own decisions (a
// shared pass gives every search the counts, but walks search 0 alone).
__device__ __forceinline__ void search_step(Search *__restrict__ gS, TreeState *__restrict__ st, double *__restrict__ Nvals,
                            const int32_t *__restrict__ cnt, const unsigned long long *__restrict__ thr,
                            int32_t *__restrict__ cnt_next, unsigned long long *__restrict__ thr_next,
                            int32_t *__restrict__ ncut, bool first, bool recorded) {
    const int lane = threadIdx.x & 63;
    Search S = *gS;
    cnt_next[lane] = 0;
    thr_next[lane] = 0;
    if (S.final) return;
    const double N = Nvals[lane];
    const int32_t c = first ? 0 : __hip_atomic_load(&cnt[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double t = first ? 0.0
                           : __longlong_as_double((long long)__hip_atomic_load(&thr[lane], __ATOMIC_RELAXED,
                                                                               __HIP_MEMORY_SCOPE_AGENT));
    int bad = 0;
    if (first) {
        S.alpha = st->alpha0;
        S.beta = st->beta0;
        const double mid = (S.alpha + S.beta) / 2.0;
        if (mid <= S.alpha || mid >= S.beta || S.iters >= S.max_iters || !(S.beta > S.alpha)) S.done = 1;
        if (S.alpha != S.alpha) bad |= 8;  // (weights that are no numbers: no midpoint to compare with)
    } else {
        S.passes += 1;
        const int32_t ch = __shfl(c, HI_LANE, 64);
        if (S.mode == MODE_RECORD) {
            // (a bracket that is closed from the start: the shared pass records
            // search 0, the others record in the next one)
            S.final = recorded ? 1 : 0;
            S.hi_cnt = ch;
        } else {
            if ((S.mode == MODE_TREE || S.mode == MODE_PATH) && ch < S.k) bad |= 16;  // beta must stay YES
            S.hi_cnt = ch;
            const double goal = S.hi_t;
            S.hi_t = __shfl(t, HI_LANE, 64);
            int q = 0, steps = 0, at_beta = HI_LANE;
            const int most = S.mode == MODE_TREE ? TREE_LEVELS : NMID;
            while (steps < most) {
                const double a = S.alpha, b = S.beta;
                const double mid = (a + b) / 2.0;
                if (mid <= a || mid >= b || S.iters >= S.max_iters) break;
                if (mid != __shfl(N, q, 64)) {  // (a predicted path ends where the bracket does; cannot happen otherwise)
                    bad |= 8;
                    break;
                }
                const int32_t cq = __shfl(c, q, 64);
                const bool yes = cq >= S.k;
                S.iters += 1;
                ++steps;
                if (yes) {
                    S.beta = mid;
                    S.hi_cnt = cq;
                    S.hi_t = __shfl(t, q, 64);
                    at_beta = q;
                } else {
                    S.alpha = mid;
                }
                if (S.mode == MODE_TREE) {
                    q = yes ? 2 * q + 1 : 2 * q + 2;
                } else {
                    const bool expected = S.mode == MODE_DOWN || (S.mode == MODE_PATH && mid >= goal);
                    if (yes != expected) break;  // the walk left the path
                    ++q;
                }
            }
            S.slow = S.mode == MODE_PATH && steps < TREE_LEVELS;
            const double mid = (S.alpha + S.beta) / 2.0;
            if (mid <= S.alpha || mid >= S.beta || S.iters >= S.max_iters) {
                S.done = 1;
                if (at_beta == S.rec) S.final = 1;
            }
            if (steps == 0 && !S.done) bad |= 8;
        }
    }
    // the next pass
    double a = S.alpha, b = S.beta, cand = b;
    S.rec = -1;
    if (S.done) {
        S.mode = MODE_RECORD;
        S.rec = HI_LANE;
    } else if (S.hi_cnt == S.k && S.hi_t > a && S.hi_t <= b && !S.slow) {
        S.mode = MODE_PATH;
        const double goal = S.hi_t;
        bool on = lane < NMID;
        for (int l = 0; l <= lane && on; ++l) {
            const double mid = (a + b) / 2.0;
            on = mid > a && mid < b;
            if (!on) break;
            cand = mid;
            if (mid >= goal)
                b = mid;
            else
                a = mid;
        }
        if (!on) cand = S.beta;
        // the predicted final upper end
        const uint64_t yes = __ballot(on && cand >= goal);
        S.rec = yes ? 63 - __clzll((long long)yes) : HI_LANE;
    } else if (S.alpha == st->alpha0 || S.beta == st->beta0) {
        S.mode = S.alpha == st->alpha0 ? MODE_DOWN : MODE_UP;
        if (lane < NMID) {
            for (int l = 0; l < lane; ++l) (S.mode == MODE_DOWN ? b : a) = (a + b) / 2.0;
            cand = (a + b) / 2.0;
        }
    } else {
        S.mode = MODE_TREE;
        if (lane < NMID) {
            const int node = lane + 1;
            const int lvl = 31 - __clz(node);  // depth of the node below the root
            for (int l = lvl - 1; l >= 0; --l) {
                const double mid = (a + b) / 2.0;
                if ((node >> l) & 1)
                    a = mid;
                else
                    b = mid;
            }
            cand = (a + b) / 2.0;
        }
    }
    Nvals[lane] = cand;
    if (lane == 0) {
        *gS = S;
        if (!S.final) *ncut = 0;
        if (bad) atomicOr(&st->bad, bad);
    }
}

// ------------------------------------------------------------------ one pass of Algorithm 1

struct Cut {
    unsigned long long key;  // (~depth, vertex): ascending is the x-order
    double num, den;
};

struct WalkArgs {
    const Op *ops;
    const Feed *feeds;
    const int32_t *start0;        // tier 0: first piece's end at or after every multiple of RUN0 records
    const int32_t *pend, *pfeed;  // per piece: end of its records in its tier's stream, of its feeds in its tier's feeds
    double2 *cw;                  // [search][slot][M] contributions (p, omega)
    int64_t cw_stride;            // slots per search
    int32_t *spill_prev;          // [search][slot] next older spilled accumulator
    const double *Nvals;          // [search][M]
    int32_t *cnt;                 // [search][M] cuts
    unsigned long long *thr;      // [search][M] bits of the largest threshold of a cut vertex
    const Search *S;
    TreeState *st;
    int32_t *ncut;                // [search] recorded cuts (may exceed CUT_CAP)
    uint8_t *dec;                 // [search][n] recorded decisions: 0 discard, 1 join, 2 cut
    Cut *cuts;                    // [search][CUT_CAP] recorded cut vertices
    double *num, *den;            // [n] (one search, NULL otherwise): the same by vertex
    const int32_t *depth;
    int64_t n;
};

// What a wave keeps over the vertices it decides: cuts, and the pair (num, den)
// of the largest ratio among them, per lane.
struct Tally {
    int32_t cuts = 0;
    double num = 0.0, den = 1.0;
};

// A recorded cut: the list of the search's cut vertices, and the arrays by vertex.
__device__ __forceinline__ void record_cut(const WalkArgs &A, int g, int32_t v, double num, double den) {
    const int32_t e = atomicAdd(&A.ncut[g], 1);
    if (e < CUT_CAP) {
        Cut *const to = A.cuts + (int64_t)g * CUT_CAP + e;
        to->key = ((unsigned long long)(0x7FFFFFFFu - (uint32_t)A.depth[v]) << 32) | (uint32_t)v;
        to->num = num;
        to->den = den;
    }
    if (A.num) {
        A.num[v] = num;
        A.den[v] = den;
    }
}

// Algorithm 1 at a vertex with accumulators (w, p), threshold N: the
// contribution to the parent, (p, w) if joined, (fe, 0) if cut or discarded;
// cut_m / join_m: the lanes that cut / join.  No branches: a taken branch costs
// a wave its instruction buffer, and with ten of them per record the walk
// waited 700 cycles a record for instructions.
__device__ __forceinline__ double2 decide(double N, double fe, double w, double p, bool tree_root, Tally &T,
                                          uint64_t &cut_m, uint64_t &join_m, double &lhs_out) {
    const double lhs = fe + p;
    const double rhs = N * w;
    const bool cut = lhs <= rhs;
    const bool join = !cut & !tree_root & ((p - fe) < rhs);
    const bool more = cut & (lhs * T.den > T.num * w);
    T.cuts += cut ? 1 : 0;
    T.num = more ? lhs : T.num;
    T.den = more ? w : T.den;
    cut_m = __ballot(cut);
    join_m = __ballot(join);
    lhs_out = lhs;
    return make_double2(join ? p : fe, join ? w : 0.0);
}

// The recorded decision of vertex v (rec >= 0), by lane rec.
__device__ __forceinline__ void record(const WalkArgs &A, int g, int rec, int m, int32_t v, uint64_t cut_m,
                                       uint64_t join_m, double num, double den) {
    if (m == rec) {
        const bool cut = (cut_m >> rec) & 1;
        A.dec[(int64_t)g * A.n + v] = cut ? 2 : (uint8_t)((join_m >> rec) & 1);
        if (cut) record_cut(A, g, v, num, den);
    }
}

__device__ __forceinline__ void add_tally(const WalkArgs &A, int g, int m, const Tally &T) {
    if (T.cuts) {
        atomicAdd(&A.cnt[g * M + m], T.cuts);
        if (T.den > 0.0)
            atomicMax(&A.thr[g * M + m], (unsigned long long)__double_as_longlong(cut_threshold(T.num, T.den)));
    }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The records of a run of a stream, staged through LDS a block at a time by one
// wave.  AHEAD: the next block's loads are in flight while a block is worked on
// (upper tiers, few stores); without it a block is loaded when it is reached
// (tier 0: blocks of 128 records cover most waves' whole run, and a wait for
// loads in flight also waits for every store issued since, at 16 records a
// block 700 cycles a record).
template <int BLOCK, bool AHEAD>
struct Records {
    static constexpr int PIECES = 3 * BLOCK, LOADS = (PIECES + 63) / 64, NBUF = AHEAD ? 2 : 1;
    const u32x4 *src;
    u32x4 *buf;    // [NBUF][LOADS * 64]
    int64_t last;  // index of the run's last 16-byte piece
    int m;
    u32x4 ahead[LOADS];
    __device__ __forceinline__ void load(int64_t block) {
#pragma unroll
        for (int u = 0; u < LOADS; ++u) ahead[u] = src[min(block * PIECES + 64 * u + m, last)];
    }
    __device__ __forceinline__ void store(int64_t block) {
        // (every lane's reads of the block's last contents are done: they are waited for before their values are used)
#pragma unroll
        for (int u = 0; u < LOADS; ++u) buf[(block % NBUF) * (LOADS * 64) + 64 * u + m] = ahead[u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ void start(const Op *ops, int32_t count, int lane, u32x4 *b) {
        src = reinterpret_cast<const u32x4 *>(ops);
        buf = b;
        last = (int64_t)count * 3 - 1;
        m = lane;
        load(0);
        if (AHEAD) {
            store(0);
            load(1);
        }
    }
    // before record i is worked on (i in order), record i itself having been read if AHEAD
    __device__ __forceinline__ void advance(int32_t i) {
        if (i % BLOCK == 0) {
            if (AHEAD) {
                store(i / BLOCK + 1);
                load(i / BLOCK + 2);
            } else {
                if (i) load(i / BLOCK);
                store(i / BLOCK);
            }
        }
    }
    __device__ __forceinline__ void at(int32_t i, u32x4 &a, u32x4 &b, u32x4 &c) {
        const u32x4 *r = buf + (i / BLOCK % NBUF) * (LOADS * 64) + 3 * (i % BLOCK);
        a = r[0];
        b = r[1];
        c = r[2];
    }
};
using Records0 = Records<128, false>;
using RecordsUp = Records<16, true>;
__device__ inline double lo64(u32x4 q) { return __hiloint2double((int)q.y, (int)q.x); }
__device__ inline double hi64(u32x4 q) { return __hiloint2double((int)q.w, (int)q.z); }

// Threshold of this lane.  The empty asm makes the load complete here: a value
// first used inside the walking loop is waited for there, in every iteration,
// and with it every store issued before.
__device__ __forceinline__ double own_threshold(const WalkArgs &A, int g, int m) {
    double N = A.Nvals[g * M + m];
    asm volatile("" : "+v"(N));
    return N;
}

// Tier 0: a contiguous run of whole pieces per wave, about as many records for
// each (by start0), one wave per workgroup; lane m
// holds threshold m.  (cp, cw) are the accumulators of the innermost open vertex
// with a finished child; the first child of a vertex below another open one
// pushes them, a later child with children of its own pops them.  A piece has
// at most 32 records, so at most 15 are pushed.
//
// Bound by the issue of about 30 instructions per record and wave (6 of them
// FP64) and their latency; stack and records (22 KB) allow seven waves per CU.
__device__ __forceinline__ void walk_tier0(const WalkArgs &A, int g, int wave, int nwaves, double2 (*__restrict__ stack)[M],
                           u32x4 *rbuf) {
    const int m = threadIdx.x & 63;
    const int32_t total = A.st->nops[0];
    const int32_t nrun = (total + RUN0 - 1) / RUN0;
    const int32_t r_lo = (int32_t)((int64_t)nrun * wave / nwaves), r_hi = (int32_t)((int64_t)nrun * (wave + 1) / nwaves);
    if (r_lo >= r_hi) return;
    const int32_t o = __builtin_amdgcn_readfirstlane(r_lo ? A.start0[r_lo] : 0);
    const int32_t count = __builtin_amdgcn_readfirstlane(r_hi < nrun ? A.start0[r_hi] : total) - o;
    if (count <= 0) return;
    const double N = own_threshold(A, g, m);
    const int rec = A.S[g].rec;
    double2 *const cw_g = A.cw + (int64_t)g * A.cw_stride * M;
    uint8_t *const dec_g = A.dec + (int64_t)g * A.n;
    Tally T;
    double cp = 0.0, cw = 0.0;
    int sp = 0;
    bool open = false;     // (cp, cw) belong to an open vertex of this piece
    int vdec = 0, vat = 0;  // recorded decisions and vertices of the last 64 records, one per lane
    Records0 R;
    R.start(A.ops + o, count, m, rbuf);
    R.advance(0);
    u32x4 a, b, c;
    R.at(0, a, b, c);
    for (int32_t i = 0; i < count; ++i) {
        // the next record's reads run under this one's arithmetic, except into a new block
        u32x4 na, nb, nc;
        R.at(i + 1, na, nb, nc);  // (into the next block or past the end: stale LDS, not used)
        const int flags = __builtin_amdgcn_readfirstlane((int)c.w);
        const bool leaf = (flags & OP_LEAF) != 0, first = (flags & OP_FIRST) != 0;
        const double w = leaf ? hi64(a) : cw, p = leaf ? lo64(b) : cp;
        uint64_t cut_m, join_m;
        double lhs;
        const double2 x = decide(N, lo64(a), w, p, (flags & OP_TREE) != 0, T, cut_m, join_m, lhs);
        if (rec >= 0) {
            const int d = (int)((cut_m >> rec) & 1) * 2 + (int)((join_m >> rec) & 1);
            const int v = __builtin_amdgcn_readfirstlane((int)c.z);
            const bool here = m == (i & 63);
            vdec = here ? d : vdec;
            vat = here ? v : vat;
            if (__builtin_expect(d & 2, 0)) {
                if (m == rec) record_cut(A, g, v, lhs, w);
            }
            if (__builtin_expect((i & 63) == 63 || i + 1 == count, 0)) {
                if (m <= (i & 63)) dec_g[vat] = (uint8_t)vdec;
            }
        }
        if (__builtin_expect(flags & OP_ROOT, 0)) {
            if (!(flags & OP_TREE)) cw_g[(int64_t)(int32_t)b.z * M + m] = x;
        }
        if (__builtin_expect(leaf && first && open, 0)) {
            stack[sp][m] = make_double2(cp, cw);
            ++sp;
        }
        cp = first ? lo64(c) : cp;
        cw = first ? hi64(b) : cw;
        if (__builtin_expect((flags & (OP_LEAF | OP_FIRST | OP_ROOT)) == 0, 0)) {
            --sp;
            const double2 y = stack[sp][m];
            cp = y.x;
            cw = y.y;
        }
        cp = cp + x.x;
        cw = cw + x.y;
        open = !(flags & OP_ROOT);
        if (__builtin_expect((i + 1) % 128 == 0, 0)) {
            if (i + 1 < count) {
                R.advance(i + 1);
                R.at(i + 1, na, nb, nc);
            }
        }
        a = na;
        b = nb;
        c = nc;
    }
    add_tally(A, g, m, T);
}

// Upper tiers: one piece per workgroup at a time.  Waves 1 .. FEEDERS bring the
// piece's feeds to LDS in order, a chunk at a time into one of two buffers, with
// the loads of the two chunks after it in flight; wave 0 walks the records and
// adds the feeds.  One barrier per chunk: wave 0 arrives at barrier k when it
// needs chunk k, having finished chunk k - 1, the others when chunk k is
// written.  Open accumulators beyond the LDS stack are spilled to the slot of
// the feed that pushes them (already brought).
//
// A hub's folds are a chain of additions; at n = 200,000 the image-like tree's
// top piece has 146 vertices and 6,308 feeds.  One wave doing everything by
// itself took 283 ns per feed (1.83 ms for that piece).
struct UpperLds {
    double2 ring[2][CHUNK + WIN][M];  // (the walking wave reads up to WIN places past a chunk and ignores them)
    double2 stack[STACK][M];
    u32x4 rec[RecordsUp::NBUF * RecordsUp::LOADS * 64];
};

// Wave w brings feeds w, w + FEEDERS, ...: FEED_PER of them per chunk.  Their
// Feed records are loaded 60 at a time, one per lane (ten chunks), a group
// ahead, and read across lanes, so that a contribution's load waits for no
// other load.
constexpr int GROUP_CHUNKS = 10;
static_assert(GROUP_CHUNKS * FEED_PER <= 64 && GROUP_CHUNKS % 2 == 0, "a group's records are one per lane");
struct FeedGroup {
    double fe, om0, p0;
    int32_t v, slot;
};
__device__ __forceinline__ double lane_f64(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

__device__ __forceinline__ void feed_piece(const WalkArgs &A, int g, int rec, double N, int64_t f0, int64_t f1,
                                           UpperLds &L, Tally &T) {
    const int m = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) - 1);
    const double2 *const cw_m = A.cw + (int64_t)g * A.cw_stride * M + m;
    const int total = __builtin_amdgcn_readfirstlane((int)(f1 - f0));
    const int nch = __builtin_amdgcn_readfirstlane((int)((f1 - f0 + CHUNK - 1) / CHUNK));
    if (nch == 0) return;
    auto group = [&](int j) {
        const Feed *f = A.feeds + min(f0 + ((int64_t)j * (GROUP_CHUNKS * FEED_PER) + m) * FEEDERS + w, f1 - 1);
        FeedGroup q;
        q.fe = f->fe;
        q.om0 = f->om0;
        q.p0 = f->p0;
        q.v = f->v;
        q.slot = f->slot;
        return q;
    };
    FeedGroup P = group(0), Q = group(1);
    int pg = 0;  // group P holds, Q the next one
    double2 F[FEED_PER], G[FEED_PER];
    auto fetch = [&](int k, double2(&X)[FEED_PER]) {
        const bool in_p = k / GROUP_CHUNKS == pg;
        const int32_t v = in_p ? P.v : Q.v, slot = in_p ? P.slot : Q.slot;
#pragma unroll
        for (int u = 0; u < FEED_PER; ++u) {
            // (a leaf loads slot 0, unused: with the loads conditional, the wait for a chunk's loads became a wait for
            // every load in flight)
            const int l = k % GROUP_CHUNKS * FEED_PER + u;
            const int from = __builtin_amdgcn_readlane(v, l) < 0 ? __builtin_amdgcn_readlane(slot, l) : 0;
            X[u] = cw_m[(int64_t)from * M];
        }
    };
    auto put = [&](int k, const double2(&X)[FEED_PER]) {
#pragma unroll
        for (int u = 0; u < FEED_PER; ++u) {
            const int e = u * FEEDERS + w, l = k % GROUP_CHUNKS * FEED_PER + u;
            if (k * CHUNK + e < total) {
                double2 y = X[u];
                const int32_t v = __builtin_amdgcn_readlane(P.v, l);
                if (v >= 0) {
                    uint64_t cut_m, join_m;
                    double lhs;
                    const double w = lane_f64(P.om0, l);
                    y = decide(N, lane_f64(P.fe, l), w, lane_f64(P.p0, l), false, T, cut_m, join_m, lhs);
                    if (rec >= 0) record(A, g, rec, m, v, cut_m, join_m, lhs, w);
                }
                L.ring[k & 1][e][m] = y;
            }
        }
    };
    fetch(0, F);
    fetch(1, G);
    for (int k = 0; k < nch; k += 2) {
        put(k, F);
        fetch(k + 2, F);
        lds_barrier();
        if (k + 1 < nch) {
            put(k + 1, G);
            if ((k + 2) % GROUP_CHUNKS == 0) {
                P = Q;
                Q = group(++pg + 1);
            }
            fetch(k + 3, G);
            lds_barrier();
        }
    }
}

__device__ __forceinline__ void walk_piece(const WalkArgs &A, int g, int rec, double N, int64_t o, int32_t count, int64_t f0,
                           UpperLds &L, Tally &T) {
    const int m = threadIdx.x & 63;
    double2 *const cw_g = A.cw + (int64_t)g * A.cw_stride * M;
    int32_t *const prev_g = A.spill_prev + (int64_t)g * A.cw_stride;
    double cp = 0.0, cw = 0.0;
    int sp = 0, chunk = -1, used = CHUNK;  // feeds taken from the current chunk
    int32_t spill_top = -1;
    bool open = false;
    // win: the next WIN feeds of the chunk (win_at on), read from LDS ahead of
    // their use.  Fixed offsets from one address keep a feed at three
    // instructions: one wave issues an instruction about every five cycles, and
    // that is what bounds the walk (57 ns a feed with the places computed).
    double2 win[WIN];
    const double2 *win_at = &L.ring[0][0][m];
    auto look = [&]() {
#pragma unroll
        for (int u = 0; u < WIN; ++u) win[u] = win_at[u * M];
    };
    auto next_chunk = [&]() {
        lds_barrier();
        ++chunk;
        used = 0;
        win_at = &L.ring[chunk & 1][0][m];
        look();
    };
    RecordsUp R;
    R.start(A.ops + o, count, m, L.rec);
    u32x4 a, b, c;
    R.at(0, a, b, c);
    for (int32_t i = 0; i < count; ++i) {
        R.advance(i);
        u32x4 na, nb, nc;
        R.at(i + 1, na, nb, nc);
        const int flags = __builtin_amdgcn_readfirstlane((int)c.w);
        const int32_t feed = __builtin_amdgcn_readfirstlane((int)a.z);
        const int32_t slot = __builtin_amdgcn_readfirstlane((int)c.z);  // of a run's first feed (else the vertex)
        if (flags & OP_FEED) {
            if (flags & OP_FIRST) {
                if (open) {
                    const double2 y = make_double2(cp, cw);
                    // (the feed has to be brought before its place is reused)
                    if (used == CHUNK) next_chunk();
                    if (sp < STACK) {
                        L.stack[sp][m] = y;
                    } else {
                        cw_g[(int64_t)slot * M + m] = y;
                        prev_g[slot] = spill_top;  // (by every lane, so that each reads back its own store)
                        spill_top = slot;
                    }
                    ++sp;
                }
                cp = lo64(c);
                cw = hi64(b);
            }
            int32_t left = __builtin_amdgcn_readfirstlane((int)na.z) - feed;
            while (left > 0) {
                if (used == CHUNK) next_chunk();
                const int take = min(left, CHUNK - used);
                used += take;
                left -= take;
                int rest = take;
                for (; rest >= WIN; rest -= WIN) {
#pragma unroll
                    for (int u = 0; u < WIN; ++u) {
                        cp = cp + win[u].x;
                        cw = cw + win[u].y;
                        win[u] = win_at[(WIN + u) * M];
                    }
                    win_at += WIN * M;
                }
                if (rest) {
#pragma unroll
                    for (int u = 0; u < WIN - 1; ++u) {
                        if (u == rest) break;
                        cp = cp + win[u].x;
                        cw = cw + win[u].y;
                    }
                    win_at += rest * M;
                    look();
                }
            }
            open = true;
        } else {
            uint64_t cut_m, join_m;
            double lhs;
            const double2 x = decide(N, lo64(a), cw, cp, (flags & OP_TREE) != 0, T, cut_m, join_m, lhs);
            if (rec >= 0) record(A, g, rec, m, slot, cut_m, join_m, lhs, cw);
            if (flags & OP_ROOT) {
                if (!(flags & OP_TREE)) cw_g[(int64_t)(int32_t)b.z * M + m] = x;
                open = false;
            } else {
                if (flags & OP_FIRST) {
                    cp = lo64(c);
                    cw = hi64(b);
                } else {
                    --sp;
                    double2 y;
                    if (sp < STACK) {
                        y = L.stack[sp][m];
                    } else {
                        y = cw_g[(int64_t)spill_top * M + m];
                        spill_top = __builtin_amdgcn_readfirstlane(prev_g[spill_top]);
                    }
                    cp = y.x;
                    cw = y.y;
                }
                cp = cp + x.x;
                cw = cw + x.y;
                open = true;
            }
        }
        a = na;
        b = nb;
        c = nc;
    }
}

constexpr int UPPER_THREADS = 64 * (1 + FEEDERS);

__device__ __forceinline__ void walk_upper(const WalkArgs &A, int tier, int g, int first_piece, int stride, UpperLds &L) {
    const int m = threadIdx.x & 63;
    int32_t ob = 0, pb = 0, fb = 0;
    for (int t = 0; t < tier; ++t) {
        ob += A.st->nops[t];
        pb += A.st->npiece[t];
        fb += t ? A.st->nfeed[t] : 0;  // (entry 0 counts the contributions)
    }
    const int32_t np = A.st->npiece[tier];
    const double N = own_threshold(A, g, m);
    const int rec = A.S[g].rec;
    if (threadIdx.x < 64) __builtin_amdgcn_s_setprio(3);  // the walking wave is the critical path
    Tally T;
    for (int32_t p = first_piece; p < np; p += stride) {
        const int32_t o0 = p ? A.pend[pb + p - 1] : 0, o1 = A.pend[pb + p];
        const int64_t f0 = fb + (p ? A.pfeed[pb + p - 1] : 0), f1 = fb + A.pfeed[pb + p];
        if (threadIdx.x >= 64)
            feed_piece(A, g, rec, N, f0, f1, L, T);
        else
            walk_piece(A, g, rec, N, (int64_t)ob + __builtin_amdgcn_readfirstlane(o0),
                       __builtin_amdgcn_readfirstlane(o1 - o0), f0, L, T);
        __syncthreads();
    }
    add_tally(A, g, m, T);
}

__global__ __launch_bounds__(64) void k_walk0(WalkArgs A) {
    __shared__ double2 stack[STACK][M];
    __shared__ u32x4 rec[Records0::NBUF * Records0::LOADS * 64];
    const int g = blockIdx.y;
    if (A.st->bad || A.S[g].final) return;
    walk_tier0(A, g, blockIdx.x, gridDim.x, stack, rec);
}

__global__ __launch_bounds__(UPPER_THREADS) void k_walk(WalkArgs A, int tier) {
    __shared__ UpperLds L;
    const int g = blockIdx.y;
    if (A.st->bad || A.S[g].final) return;
    walk_upper(A, tier, g, blockIdx.x, gridDim.x, L);
}

// The topmost tier (one piece, the root's) and the step to the next pass.
__global__ __launch_bounds__(64) void k_walk0_top(WalkArgs A, Search *S, double *Nvals, int32_t *cnt_next,
                                                  unsigned long long *thr_next) {
    __shared__ double2 stack[STACK][M];
    __shared__ u32x4 rec[Records0::NBUF * Records0::LOADS * 64];
    if (!A.st->bad && !A.S[0].final) walk_tier0(A, 0, 0, 1, stack, rec);
    __threadfence();  // this wave's atomics before the reads below
    search_step(S, A.st, Nvals, A.cnt, A.thr, cnt_next, thr_next, A.ncut, false, true);
}

__global__ __launch_bounds__(UPPER_THREADS) void k_walk_top(WalkArgs A, int tier, Search *S, double *Nvals,
                                                            int32_t *cnt_next, unsigned long long *thr_next) {
    __shared__ UpperLds L;
    if (!A.st->bad && !A.S[0].final) walk_upper(A, tier, 0, 0, 1, L);
    drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) __threadfence();  // the waves' atomics before the reads below
    __syncthreads();
    if (threadIdx.x < 64) search_step(S, A.st, Nvals, A.cnt, A.thr, cnt_next, thr_next, A.ncut, false, true);
}

// The step alone, for the first pass and for several searches: search g reads
// the pass's results from row g, or from row 0 when `shared`.
__global__ __launch_bounds__(64) void k_step(Search *S, TreeState *st, double *Nvals, const int32_t *cnt,
                                             const unsigned long long *thr, int32_t *cnt_next,
                                             unsigned long long *thr_next, int32_t *ncut, int first, int shared) {
    const int g = blockIdx.x, row = shared ? 0 : g;
    search_step(S + g, st, Nvals + g * M, cnt + row * M, thr + row * M, cnt_next + g * M, thr_next + g * M, ncut + g,
                first != 0, !shared || g == 0);
}

// ------------------------------------------------------------------ labels (Algorithm 4)

// The first k recorded cuts in x-order: sorted keys, the clusters' costs, i_k =
// max_j num_j / den_j and the smallest j attaining it.  One workgroup per
// search; more than CUT_CAP cuts (or clusters) are left to the sorting path.
__global__ __launch_bounds__(1024) void k_pick_cuts(Search *__restrict__ S, const TreeState *__restrict__ st,
                                                    const Cut *__restrict__ cuts,
                                                    const int32_t *__restrict__ ncut,
                                                    unsigned long long *__restrict__ ckeys, double *__restrict__ cl_num,
                                                    double *__restrict__ cl_den, int32_t *__restrict__ cl_size) {
    __shared__ unsigned long long key[CUT_CAP];
    __shared__ int32_t idx[CUT_CAP];
    __shared__ double s_best[16];
    __shared__ int32_t s_j[16];
    const int g = blockIdx.x, tid = threadIdx.x;
    const int C = ncut[g], k = S[g].k;
    if (st->bad || !S[g].final || C > CUT_CAP || C < k) return;
    const Cut *const in = cuts + (int64_t)g * CUT_CAP;
    int P2 = 1;
    while (P2 < C) P2 *= 2;
    for (int i = tid; i < P2; i += 1024) {
        key[i] = i < C ? in[i].key : ~0ull;
        idx[i] = i;
    }
    __syncthreads();
    for (int w = 2; w <= P2; w *= 2)
        for (int h = w / 2; h >= 1; h /= 2) {
            for (int i = tid; i < P2; i += 1024) {
                const int j = i ^ h;
                if (j > i && (key[i] > key[j]) == ((i & w) == 0)) {
                    const unsigned long long a = key[i];
                    key[i] = key[j];
                    key[j] = a;
                    const int32_t b = idx[i];
                    idx[i] = idx[j];
                    idx[j] = b;
                }
            }
            __syncthreads();
        }
    double best = -1.0;
    int32_t bj = 0;
    for (int j = tid; j < k; j += 1024) {
        const Cut c = in[idx[j]];
        ckeys[(int64_t)g * CUT_CAP + j] = key[j];
        if (cl_num) {
            cl_num[j] = c.num;
            cl_den[j] = c.den;
            cl_size[j] = 0;
        }
        const double cost = c.num / c.den;
        if (cost > best) {
            best = cost;
            bj = j;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const double ob = __shfl_xor(best, off, 64);
        const int32_t oj = __shfl_xor(bj, off, 64);
        if (ob > best || (ob == best && oj < bj)) {
            best = ob;
            bj = oj;
        }
    }
    if ((tid & 63) == 0) {
        s_best[tid >> 6] = best;
        s_j[tid >> 6] = bj;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 16; ++w)
            if (s_best[w] > best || (s_best[w] == best && s_j[w] < bj)) {
                best = s_best[w];
                bj = s_j[w];
            }
        S[g].i_k = best;
        S[g].jstar = bj;
    }
}

constexpr int HOPS = 64;  // joined edges a launch follows at most
// rep[v] = the vertex reached from v over joined edges: the first launch (init)
// follows the parents, the next ones the pointers found so far (a pointer read
// while another thread moves it on is an ancestor on the same path either way).
__global__ __launch_bounds__(256) void k_rep_hop(const Search *__restrict__ S, const TreeState *__restrict__ st,
                                                 const uint8_t *__restrict__ dec, const int32_t *__restrict__ parent,
                                                 int64_t n, int init, int32_t *rep_base) {
    const int g = blockIdx.y;
    if (st->bad || !S[g].final) return;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const uint8_t *const d = dec + (int64_t)g * n;
    int32_t *const rep = rep_base + (int64_t)g * n;
    int32_t x = init ? (int32_t)v : rep[v];
    for (int h = 0; h < HOPS && d[x] == 1; ++h) x = init ? parent[x] : rep[x];
    rep[v] = x;
}

// Label of v: the index of its representative among the first k cuts, or -1
// (rep may be the label array itself: each thread reads only its own entry);
// cluster sizes when cl_size is given.
__global__ __launch_bounds__(256) void k_label(const Search *__restrict__ S, const TreeState *__restrict__ st,
                                               const uint8_t *__restrict__ dec, const int32_t *__restrict__ depth,
                                               const unsigned long long *__restrict__ ckeys,
                                               const int32_t *__restrict__ ncut, int64_t n, int32_t *rep_base, int32_t *__restrict__ cl_size) {
    __shared__ int32_t h[CUT_CAP];
    const int g = blockIdx.y;
    const int k = S[g].k, C = ncut[g];
    if (st->bad || !S[g].final || C > CUT_CAP || C < k) return;
    if (cl_size) {
        for (int j = threadIdx.x; j < k; j += 256) h[j] = 0;
        __syncthreads();
    }
    int32_t *const rep = rep_base + (int64_t)g * n;
    const uint8_t *const d = dec + (int64_t)g * n;
    const unsigned long long *const ck = ckeys + (int64_t)g * CUT_CAP;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (int64_t)gridDim.x * 256) {
        const int32_t x = rep[v];
        int32_t lab = -1;
        if (d[x] == 2) {
            const unsigned long long key =
                ((unsigned long long)(0x7FFFFFFFu - (uint32_t)depth[x]) << 32) | (uint32_t)x;
            int lo = 0, hi = k;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (ck[mid] < key)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            if (lo < k && ck[lo] == key) lab = lo;
        }
        rep[v] = lab;
        if (cl_size && lab >= 0) atomicAdd(&h[lab], 1);
    }
    if (cl_size) {
        __syncthreads();
        for (int j = threadIdx.x; j < k; j += 256)
            if (h[j]) atomicAdd(&cl_size[j], h[j]);
    }
}

// ---- the sorting path (more than CUT_CAP cuts): cut flags in x-order, their
// exclusive scan, labels through the representatives

__global__ void k_order_keys(const int32_t *__restrict__ depth, int64_t n, int32_t maxdepth, uint32_t *__restrict__ key,
                             uint32_t *__restrict__ val) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    key[v] = (uint32_t)(maxdepth - depth[v]);
    val[v] = (uint32_t)v;
}

__global__ void k_cut_in_xorder(const uint32_t *__restrict__ order, const uint8_t *__restrict__ dec, int64_t n,
                                int32_t *__restrict__ cf) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    cf[i] = dec[order[i]] == 2 ? 1 : 0;
}

// Cluster index of each of the first k cuts (exclusive scan of the cut flags), -1 for every other vertex.
__global__ void k_cluster_index(const uint32_t *__restrict__ order, const uint8_t *__restrict__ dec,
                                const int32_t *__restrict__ rank, int64_t n, int32_t k, int32_t *__restrict__ cidx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = (int32_t)order[i];
    cidx[v] = (dec[v] == 2 && rank[i] < k) ? rank[i] : -1;
}

__global__ void k_labels_sorted(int32_t *rep, const int32_t *__restrict__ cidx, const double *__restrict__ num,
                                const double *__restrict__ den, int64_t n, double *__restrict__ cl_num,
                                double *__restrict__ cl_den) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    rep[v] = cidx[rep[v]];
    const int32_t j = cidx[v];
    if (j >= 0) {
        cl_num[j] = num[v];
        cl_den[j] = den[v];
    }
}

__global__ __launch_bounds__(64) void k_final_cost(const double *__restrict__ cl_num, const double *__restrict__ cl_den,
                                                   int32_t k, Search *__restrict__ S) {
    double best = -1.0;
    int32_t js = 0x7FFFFFFF;
    for (int32_t j = threadIdx.x; j < k; j += 64) {
        const double c = cl_num[j] / cl_den[j];
        if (c > best) {
            best = c;
            js = j;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const double ob = __shfl_xor(best, off, 64);
        const int32_t oj = __shfl_xor(js, off, 64);
        if (ob > best || (ob == best && oj < js)) {
            best = ob;
            js = oj;
        }
    }
    if (threadIdx.x == 0) {
        S->i_k = best;
        S->jstar = js == 0x7FFFFFFF ? 0 : js;  // (no cost above -1: the first, as where the cuts fit their list)
    }
}

__global__ void k_force_record(Search *S, double *Nvals, int32_t *ncut) {
    Nvals[threadIdx.x] = S->beta;
    if (threadIdx.x == 0) {
        S->final = 0;
        S->mode = MODE_RECORD;
        S->rec = HI_LANE;
        *ncut = 0;
    }
}

// ------------------------------------------------------------------ plan

constexpr int RANK_LEVELS = 12;

struct SubPlan {
    int64_t n;
    int32_t k;
    int32_t ng;  // searches that may run together
    uint32_t *ckey, *cval, *tk, *tv;
    int32_t *koff, *depth, *size, *pv, *place, *ctr, *pend, *pfeed, *start0, *spill, *cf, *rank, *cidx, *lab_tmp, *scan_scratch, *cl_size_tmp;
    int32_t *nxt[RANK_LEVELS], *len[RANK_LEVELS], *ent[RANK_LEVELS], *own[RANK_LEVELS], *olen[RANK_LEVELS],
        *oent[RANK_LEVELS], *rlen[RANK_LEVELS], *rent[RANK_LEVELS];
    int32_t m[RANK_LEVELS];
    int levels;
    double2 *cw;
    Op *ops;
    Feed *feeds;
    double *phi, *om0, *p0, *Nvals, *num, *den, *cl_num_tmp, *cl_den_tmp, *stats_part;
    int32_t *cnt, *ncut;
    unsigned long long *thr, *ckeys;
    Cut *cuts;
    uint8_t *dec;
    Search *S;
    TreeState *st;
    void *sort_scratch, *sel_scratch;

    int64_t op_blocks() const { return (n + OPB - 1) / OPB; }

    void carve(Arena &a) {
        ng = std::max<int32_t>(1, std::min<int32_t>(k - 1, MAXG));
        ckey = a.take<uint32_t>(n);
        cval = a.take<uint32_t>(n);
        tk = a.take<uint32_t>(n);
        tv = a.take<uint32_t>(n);
        koff = a.take<int32_t>(n + 1);
        depth = a.take<int32_t>(n);
        size = a.take<int32_t>(n);
        pv = a.take<int32_t>(n);
        place = a.take<int32_t>(n);
        ctr = a.take<int32_t>((size_t)op_blocks() * NCTR);
        pend = a.take<int32_t>(n);
        pfeed = a.take<int32_t>(n);
        start0 = a.take<int32_t>(n / RUN0 + 2);
        spill = a.take<int32_t>(n);
        cf = a.take<int32_t>(n);
        rank = a.take<int32_t>(n);
        cidx = a.take<int32_t>(n);
        lab_tmp = a.take<int32_t>(n);
        scan_scratch = a.take<int32_t>(scan_scratch_bytes(n + 1) / sizeof(int32_t));
        cl_size_tmp = a.take<int32_t>(k);
        levels = 0;
        for (int64_t mm = 2 * n;; mm = (mm + 7) / 8) {
            m[levels] = (int32_t)mm;
            nxt[levels] = a.take<int32_t>(mm);
            len[levels] = levels ? a.take<int32_t>(mm) : nullptr;
            ent[levels] = levels ? a.take<int32_t>(mm) : nullptr;
            own[levels] = a.take<int32_t>(mm);
            olen[levels] = a.take<int32_t>(mm);
            oent[levels] = a.take<int32_t>(mm);
            rlen[levels] = a.take<int32_t>(mm);
            rent[levels] = a.take<int32_t>(mm);
            ++levels;
            if (mm <= RANK_LDS) break;
        }
        ops = a.take<Op>((size_t)n * 2);
        feeds = a.take<Feed>(n);
        cw = a.take<double2>((size_t)n * M);
        phi = a.take<double>(n);
        om0 = a.take<double>(n);
        p0 = a.take<double>(n);
        num = a.take<double>(n);
        den = a.take<double>(n);
        Nvals = a.take<double>(MAXG * M);
        cl_num_tmp = a.take<double>(k);
        cl_den_tmp = a.take<double>(k);
        stats_part = a.take<double>(STATS_BLOCKS * 6);
        cnt = a.take<int32_t>(2 * MAXG * M);
        ncut = a.take<int32_t>(MAXG);
        thr = a.take<unsigned long long>(2 * MAXG * M);
        ckeys = a.take<unsigned long long>((size_t)ng * CUT_CAP);
        cuts = a.take<Cut>((size_t)ng * CUT_CAP);
        dec = a.take<uint8_t>((size_t)ng * n);
        S = a.take<Search>(MAXG);
        st = a.take<TreeState>(1);
        sort_scratch = a.take<char>(radix_sort_scratch_bytes(n));
        sel_scratch = a.take<char>(radix_select_scratch_bytes());
    }
};

size_t sub_plan_bytes(int64_t n, int32_t k) {
    SubPlan p{};
    p.n = n;
    p.k = k;
    Arena a;
    p.carve(a);
    return a.used;
}

int bits_for(int64_t maxval) {
    int b = 0;
    while (b < 32 && (int64_t(1) << b) <= maxval) ++b;
    return b < 1 ? 1 : b;
}

// Passes queued before the host looks at the state.
constexpr int PASSES_AHEAD = 3;

// Single k (kmax == 0), or every k = 2 .. kmax (kmax >= 2): each k's search is
// the single-k bisection; up to MAXG of them (as many as the contribution
// buffer holds) run side by side in each pass's launches and share the first
// pass, whose thresholds are the same.  i_k_all[k - 2] and the label rows
// labels_all[(k - 2) n ..] receive the results.
void run_sub(SubPlan &P, const int32_t *parent, const double *length, int32_t root, double sigma,
             const iso_sub_opts &o, int32_t *labels, double *i_k, double *cl_num, double *cl_den, int32_t *cl_size,
             iso_sub_info *info, hipStream_t s, int32_t kmax = 0, double *i_k_all = nullptr,
             int32_t *labels_all = nullptr, int32_t *passes_out = nullptr) {
    const int64_t n = P.n;
    const unsigned gn = grid_for(n, 256);
    const bool timed = timing().enabled != 0;
    const int32_t max_iters = o.max_iters > 0 ? o.max_iters : 2000;
    EventPair whole(timed);
    whole.start(s);
    const int32_t k_first = kmax ? 2 : P.k, nk = kmax ? kmax - 1 : 1;
    auto init_searches = [&](int32_t k0, int32_t ns, double sg) {
        hipLaunchKernelGGL(k_init, dim3(1), dim3(1024), 0, s, P.st, P.S, ns, k0, max_iters, sg, P.cnt, P.thr,
                           P.ncut);
        LAUNCH_CHECK();
    };
    init_searches(k_first, std::min<int32_t>(nk, P.ng), sigma);

    // child lists: the vertices sorted by parent (stable, so ascending within one)
    hipLaunchKernelGGL(k_check_tree, dim3(gn), dim3(256), 0, s, parent, length, n, root, P.ckey, P.cval, P.st);
    LAUNCH_CHECK();
    radix_sort_pairs_u32(P.ckey, P.cval, P.tk, P.tv, n, bits_for(n), P.sort_scratch, s);
    hipLaunchKernelGGL(k_child_off, dim3(grid_for(n + 1, 256)), dim3(256), 0, s, P.ckey, n, P.koff);
    LAUNCH_CHECK();
    const uint32_t *kids = P.cval + 1;  // the root (key 0) sorts first; vertex v is at cval[place[v]]

    // depth-first order
    hipLaunchKernelGGL(k_tour_links, dim3(gn), dim3(256), 0, s, P.ckey, P.cval, P.koff, n, P.nxt[0], P.own[0],
                       P.place);
    LAUNCH_CHECK();
    RankLevel R[RANK_LEVELS];
    for (int l = 0; l < P.levels; ++l)
        R[l] = RankLevel{P.nxt[l], P.len[l], P.ent[l], P.own[l], P.olen[l], P.oent[l], P.rlen[l], P.rent[l],
                         P.m[l],   l ? R[l - 1].head >> 3 : root, l ? 0 : (int32_t)n};
    for (int l = 0; l + 1 < P.levels; ++l) {
        hipLaunchKernelGGL(k_rank_walk, dim3(grid_for(P.m[l + 1], 64)), dim3(64), 0, s, R[l], P.m[l + 1], P.nxt[l + 1],
                           P.len[l + 1], P.ent[l + 1], P.own[l + 1]);
        LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_rank_lds, dim3(1), dim3(1024), 0, s, R[P.levels - 1]);
    LAUNCH_CHECK();
    for (int l = P.levels - 2; l >= 0; --l) {
        hipLaunchKernelGGL(k_rank_back, dim3(grid_for(P.m[l], 256)), dim3(256), 0, s, R[l], P.rlen[l + 1],
                           P.rent[l + 1]);
        LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_place, dim3(gn), dim3(256), 0, s, P.rlen[0], P.rent[0], n, root, P.depth, P.size, P.pv, P.st);
    LAUNCH_CHECK();

    // sigma, phi, omega0, stats, bracket
    if (sigma == 0.0) {
        radix_select_f64(length, parent, n, (n - 2) / 2, &P.st->sigma, P.sel_scratch, s);
    }
    hipLaunchKernelGGL(k_phi, dim3(gn), dim3(256), 0, s, parent, length, n, P.st, o.phi, P.phi, P.p0);
    LAUNCH_CHECK();
    // vertex weights: the tree degree, or the caller's full-graph weights;
    // potential p: zero, or the caller's (eq. 2.3)
    const double *om0 = P.om0, *p0 = o.p0 ? o.p0 : P.p0;
    if (o.omega == ISO_OMEGA_FULL) {
        om0 = o.omega0;
    } else {
        hipLaunchKernelGGL(k_omega_tree, dim3(gn), dim3(256), 0, s, parent, P.phi, kids, P.koff, n, P.om0);
        LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_stats_part, dim3(STATS_BLOCKS), dim3(256), 0, s, parent, P.phi, om0, p0, n, P.stats_part);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(k_stats, dim3(1), dim3(256), 0, s, P.stats_part, o.bracket, P.st);
    LAUNCH_CHECK();

    // the record streams
    const int64_t nb = P.op_blocks();
    hipLaunchKernelGGL(k_ops<true>, dim3((unsigned)nb), dim3(OPB), 0, s, P.pv, P.size, parent, P.cval, P.place, P.koff,
                       P.phi, om0, p0, n, root, nb, P.ctr, P.st, P.ops, P.feeds, P.pend, P.pfeed,
                       P.start0);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(k_ops_scan, dim3(1), dim3(1024), 0, s, P.ctr, nb, P.st);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(k_ops<false>, dim3((unsigned)nb), dim3(OPB), 0, s, P.pv, P.size, parent, P.cval, P.place, P.koff,
                       P.phi, om0, p0, n, root, nb, P.ctr, P.st, P.ops, P.feeds, P.pend, P.pfeed,
                       P.start0);
    LAUNCH_CHECK();

    int top = 0;  // the root's tier
    while (top < NT - 1 && n > TIER_SIZE[top]) ++top;
    const int par_stride = MAXG * M;
    int parity = 0;  // half of cnt / thr the next pass adds to (the other one is clear)
    WalkArgs A{};
    A.ops = P.ops;
    A.pend = P.pend;
    A.pfeed = P.pfeed;
    A.start0 = P.start0;
    A.feeds = P.feeds;
    A.cw = P.cw;
    A.cw_stride = n;
    A.spill_prev = P.spill;
    A.Nvals = P.Nvals;
    A.S = P.S;
    A.ncut = P.ncut;
    A.st = P.st;
    A.dec = P.dec;
    A.cuts = P.cuts;
    A.depth = P.depth;
    A.n = n;
    // tier 0: at least RUN0 records per wave, at most the waves the LDS stacks let the
    // chip hold at once; upper tiers: a workgroup per piece, as far as the
    // subtree sizes allow pieces
    auto walk = [&](int t, unsigned g) {
        const int64_t cus = device_cus();
        if (t == 0)
            hipLaunchKernelGGL(k_walk0, dim3((unsigned)std::min<int64_t>(n / RUN0 + 1, 7 * cus), g), dim3(64), 0, s, A);
        else
            hipLaunchKernelGGL(k_walk, dim3((unsigned)std::min<int64_t>(n / TIER_SIZE[t - 1] + 1, cus), g),
                               dim3(UPPER_THREADS), 0, s, A, t);
        LAUNCH_CHECK();
    };
    // one pass of `g` searches and the step of `gs`
    auto pass = [&](unsigned g, unsigned gs, bool shared) {
        A.cnt = P.cnt + parity * par_stride;
        A.thr = P.thr + parity * par_stride;
        int32_t *const cn = P.cnt + (parity ^ 1) * par_stride;
        unsigned long long *const tn = P.thr + (parity ^ 1) * par_stride;
        for (int t = 0; t < top; ++t) walk(t, g);
        if (gs == 1) {
            if (top == 0)
                hipLaunchKernelGGL(k_walk0_top, dim3(1), dim3(64), 0, s, A, P.S, P.Nvals, cn, tn);
            else
                hipLaunchKernelGGL(k_walk_top, dim3(1), dim3(UPPER_THREADS), 0, s, A, top, P.S, P.Nvals, cn, tn);
            LAUNCH_CHECK();
        } else {
            walk(top, g);
            hipLaunchKernelGGL(k_step, dim3(gs), dim3(64), 0, s, P.S, P.st, P.Nvals, A.cnt, A.thr, cn, tn,
                               P.ncut, 0, shared ? 1 : 0);
            LAUNCH_CHECK();
        }
        parity ^= 1;
    };
    auto first_step = [&](unsigned gs) {
        hipLaunchKernelGGL(k_step, dim3(gs), dim3(64), 0, s, P.S, P.st, P.Nvals, P.cnt + parity * par_stride,
                           P.thr + parity * par_stride, P.cnt + (parity ^ 1) * par_stride,
                           P.thr + (parity ^ 1) * par_stride, P.ncut, 1, 0);
        LAUNCH_CHECK();
        parity ^= 1;
    };
    // representatives of `g` searches into rep ([g][n]), then their labels
    auto reps = [&](unsigned g, int32_t *rep) {
        int64_t reach = HOPS;
        for (bool init = true;; init = false) {
            hipLaunchKernelGGL(k_rep_hop, dim3(gn, g), dim3(256), 0, s, P.S, P.st, P.dec, parent, n, init ? 1 : 0, rep);
            LAUNCH_CHECK();
            if (reach >= n) break;
            reach *= HOPS;
        }
    };
    auto finish = [&](unsigned g, int32_t *lab, double *cn, double *cd, int32_t *cs) {
        hipLaunchKernelGGL(k_pick_cuts, dim3(g), dim3(1024), 0, s, P.S, P.st, P.cuts, P.ncut, P.ckeys, cn, cd,
                           cs);
        LAUNCH_CHECK();
        if (!lab) return;
        reps(g, lab);
        hipLaunchKernelGGL(k_label, dim3(std::min<unsigned>(gn, 4u * (unsigned)device_cus()), g), dim3(256), 0, s, P.S,
                           P.st, P.dec, P.depth, P.ckeys, P.ncut, n, lab, cs);
        LAUNCH_CHECK();
    };
    TreeState h{};
    std::vector<Search> hs(MAXG);
    std::vector<int32_t> hcut(MAXG);
    auto read_state = [&](int32_t ns) {
        HIP_CHECK(hipMemcpyAsync(&h, P.st, sizeof(h), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipMemcpyAsync(hs.data(), P.S, sizeof(Search) * (size_t)ns, hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipMemcpyAsync(hcut.data(), P.ncut, sizeof(int32_t) * (size_t)ns, hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        ISO_REQUIRE(!(h.bad & 1), ISO_ERR_INVALID_ARG,
                    "parent/length malformed: parent[root] must be -1, other parents in [0,n) and not self, lengths "
                    "finite and >= 0");
        ISO_REQUIRE(!(h.bad & 2), ISO_ERR_INVALID_ARG, "parent array has a cycle (not a tree rooted at %d)", root);
        ISO_REQUIRE(h.sigma > 0.0 && std::isfinite(h.sigma), ISO_ERR_INVALID_ARG,
                    "sigma must be positive (the median edge length is %g)", h.sigma);
        ISO_REQUIRE(!(h.bad & 4), ISO_ERR_INVALID_ARG, "degenerate weights: the bracket of the bisection is not finite");
        ISO_REQUIRE(!(h.bad & 8), ISO_ERR_INTERNAL, "bisection candidates out of step");
        ISO_REQUIRE(!(h.bad & 16), ISO_ERR_INTERNAL, "decision at beta turned NO during bisection");
        for (int32_t j = 0; j < ns; ++j)
            ISO_REQUIRE(!hs[j].final || hs[j].hi_cnt >= hs[j].k, ISO_ERR_INTERNAL, "decision at beta found %d < k = %d cuts",
                        hs[j].hi_cnt, hs[j].k);
    };
    // search j (its bracket is final) by the sorting path: decisions, numerators
    // and denominators of every vertex from one more pass
    auto finish_sorted = [&](int32_t j, int32_t *lab, double *cn, double *cd, int32_t *cs) {
        if (j) HIP_CHECK(hipMemcpyAsync(P.S, P.S + j, sizeof(Search), hipMemcpyDeviceToDevice, s));
        hipLaunchKernelGGL(k_force_record, dim3(1), dim3(M), 0, s, P.S, P.Nvals, P.ncut);
        LAUNCH_CHECK();
        A.num = P.num;
        A.den = P.den;
        pass(1, 1, false);
        A.num = A.den = nullptr;
        hipLaunchKernelGGL(k_order_keys, dim3(gn), dim3(256), 0, s, P.depth, n, h.maxdepth, P.ckey, P.tk);
        LAUNCH_CHECK();
        // (the child lists are no longer needed once the records are built, except cval: sort into spare arrays)
        uint32_t *key = P.ckey, *val = reinterpret_cast<uint32_t *>(P.rlen[0]);
        HIP_CHECK(hipMemcpyAsync(val, P.tk, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToDevice, s));
        radix_sort_pairs_u32(key, val, P.tk, P.tv, n, bits_for(h.maxdepth), P.sort_scratch, s);
        hipLaunchKernelGGL(k_cut_in_xorder, dim3(gn), dim3(256), 0, s, val, P.dec, n, P.cf);
        LAUNCH_CHECK();
        exclusive_scan_i32(P.cf, P.rank, n, nullptr, P.scan_scratch, s);
        hipLaunchKernelGGL(k_cluster_index, dim3(gn), dim3(256), 0, s, val, P.dec, P.rank, n, hs[j].k, P.cidx);
        LAUNCH_CHECK();
        reps(1, lab);
        hipLaunchKernelGGL(k_labels_sorted, dim3(gn), dim3(256), 0, s, lab, P.cidx, P.num, P.den, n, cn, cd);
        LAUNCH_CHECK();
        fill_t<int32_t>(cs, 0, hs[j].k, s);
        histogram_i32(lab, n, hs[j].k, cs, s);
        hipLaunchKernelGGL(k_final_cost, dim3(1), dim3(64), 0, s, cn, cd, hs[j].k, P.S);
        LAUNCH_CHECK();
        Search r{};
        HIP_CHECK(hipMemcpyAsync(&r, P.S, sizeof(r), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        hs[j].i_k = r.i_k;
        hs[j].jstar = r.jstar;
    };

    int32_t passes = 0;
    if (kmax >= 2) {
        // ---- all k, in batches of as many searches as fit the contribution buffer
        read_state(std::min<int32_t>(nk, P.ng));
        const int64_t slots = std::max<int64_t>(1, h.nfeed[0]);
        const int32_t batch = (int32_t)std::max<int64_t>(1, std::min<int64_t>(P.ng, n / slots));
        A.cw_stride = slots;
        for (int32_t k0 = 2; k0 <= kmax; k0 += batch) {
            const int32_t ns = std::min<int32_t>(batch, kmax - k0 + 1);
            if (k0 > 2 || ns != std::min<int32_t>(nk, P.ng)) {
                // fresh searches (the tree's own state is kept)
                std::vector<Search> fresh(ns);
                for (int32_t j = 0; j < ns; ++j) {
                    fresh[j] = Search{};
                    fresh[j].k = k0 + j;
                    fresh[j].max_iters = max_iters;
                    fresh[j].hi_cnt = -1;
                    fresh[j].rec = -1;
                }
                HIP_CHECK(hipMemcpyAsync(P.S, fresh.data(), sizeof(Search) * (size_t)ns, hipMemcpyHostToDevice, s));
                HIP_CHECK(hipStreamSynchronize(s));
                fill_t<int32_t>(P.cnt, 0, 2 * MAXG * M, s);
                fill_t<int32_t>(P.ncut, 0, MAXG, s);
                fill_t<unsigned long long>(P.thr, 0ull, 2 * MAXG * M, s);
            }
            int32_t *const lab = labels_all ? labels_all + (int64_t)(k0 - 2) * n : nullptr;
            first_step((unsigned)ns);
            for (int32_t round = 0;; ++round) {
                ISO_REQUIRE(round <= max_iters + 8, ISO_ERR_INTERNAL, "bisection did not terminate");
                for (int q = 0; q < PASSES_AHEAD; ++q) {
                    const bool shared = round == 0 && q == 0;  // every search's first thresholds are the same
                    pass(shared ? 1u : (unsigned)ns, (unsigned)ns, shared);
                }
                finish((unsigned)ns, lab, nullptr, nullptr, nullptr);
                read_state(ns);
                bool all = true;
                for (int32_t j = 0; j < ns; ++j) all = all && hs[j].final;
                if (all) break;
            }
            int32_t most = 0;
            for (int32_t j = 0; j < ns; ++j) most = std::max(most, hs[j].passes);
            passes += most;
            for (int32_t j = 0; j < ns; ++j) {
                if (hcut[j] > CUT_CAP)
                    finish_sorted(j, lab ? lab + (int64_t)j * n : P.lab_tmp, P.cl_num_tmp, P.cl_den_tmp, P.cl_size_tmp);
                i_k_all[k0 + j - 2] = hs[j].i_k;
            }
        }
        if (passes_out) *passes_out = passes;
    } else {
        double *cn = cl_num ? cl_num : P.cl_num_tmp;
        double *cd = cl_den ? cl_den : P.cl_den_tmp;
        int32_t *cs = cl_size ? cl_size : P.cl_size_tmp;
        first_step(1);
        for (int32_t round = 0;; ++round) {
            ISO_REQUIRE(round <= max_iters + 8, ISO_ERR_INTERNAL, "bisection did not terminate");
            for (int q = 0; q < PASSES_AHEAD; ++q) pass(1, 1, false);
            finish(1, labels, cn, cd, cs);
            read_state(1);
            if (hs[0].final) break;
        }
        passes = hs[0].passes;
        if (hcut[0] > CUT_CAP) finish_sorted(0, labels, cn, cd, cs);
        *i_k = hs[0].i_k;
    }
    whole.stop(s);
    if (timed) {
        timing().sub_calls += 1;
        timing().sub_ms += whole.elapsed_ms();
        timing().sub_passes += passes;
    }
    if (info) {
        const Search &x = hs[0];
        info->sigma = h.sigma;
        info->alpha0_raw = h.alpha0_raw;
        info->beta0_raw = h.beta0_raw;
        info->alpha0 = h.alpha0;
        info->beta0 = h.beta0;
        info->alpha = x.alpha;
        info->beta = x.beta;
        info->i_k = x.i_k;
        const double tt = std::log2(2.0 * h.om_sum * h.om_sum * (h.beta0_raw - h.alpha0_raw)) -
                          std::log2(h.phi_min + h.p_min);
        info->t_paper = std::isfinite(tt) ? (int32_t)std::ceil(tt) : -1;
        info->iters = x.iters;
        info->passes = x.passes;
        info->max_depth = h.maxdepth;
        info->jstar = x.jstar;
        info->reserved0 = 0;
    }
}

}  // namespace

// ------------------------------------------------------------------ allocation-free workspace

// Workspace of iso_subpartition_noalloc: one fixed array per device, reserved
// for the life of the process.  In host code `scratch` names only the host-side
// shadow of the symbol; kernels receive the device address that
// hipGetSymbolAddress reports for the current device.
static __device__ __align__(256) char scratch[ISO_SUB_NOALLOC_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device, looked up on the first
// call made with that device current.
char *noalloc_scratch() {
    int dev = -1;
    HIP_CHECK(hipGetDevice(&dev));
    ISO_REQUIRE(dev >= 0 && dev < MAX_DEVICES, ISO_ERR_NO_DEVICE, "device ordinal %d outside [0, %d)", dev,
                MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        ISO_REQUIRE(ptr != nullptr, ISO_ERR_HIP, "hipGetSymbolAddress returned no address for the scratch array");
        g_scratch_ptr[dev] = static_cast<char *>(ptr);
    }
    return g_scratch_ptr[dev];
}

}  // namespace

}  // namespace iso

using namespace iso;

extern "C" iso_status iso_sub_workspace_size(int64_t n, int32_t k, size_t *bytes) {
    return guarded([&] {
        ISO_REQUIRE(bytes != nullptr, ISO_ERR_INVALID_ARG, "bytes is NULL");
        ISO_REQUIRE(n >= 2 && n < (int64_t(1) << 31) - 2, ISO_ERR_INVALID_ARG, "n = %lld outside [2, 2^31)", (long long)n);
        ISO_REQUIRE(k >= 2 && k <= n, ISO_ERR_INVALID_ARG, "k = %d outside [2, n]", k);
        *bytes = sub_plan_bytes(n, k);
    });
}

extern "C" iso_status iso_subpartition_all_k(const int32_t *parent, const double *length, int64_t n, int32_t root,
                                             int32_t kmax, double sigma, const iso_sub_opts *opts, double *i_k,
                                             int32_t *labels, int32_t *passes, void *ws, size_t ws_bytes,
                                             void *stream) {
    return guarded([&] {
        ISO_REQUIRE(parent && length && i_k, ISO_ERR_INVALID_ARG, "parent, length and i_k must be non-NULL");
        ISO_REQUIRE(n >= 2 && n < (int64_t(1) << 31) - 2, ISO_ERR_INVALID_ARG, "n = %lld outside [2, 2^31)", (long long)n);
        ISO_REQUIRE(kmax >= 2 && kmax <= n, ISO_ERR_INVALID_ARG, "kmax = %d outside [2, n]", kmax);
        ISO_REQUIRE(root >= 0 && root < n, ISO_ERR_INVALID_ARG, "root = %d outside [0, n)", root);
        ISO_REQUIRE(sigma >= 0.0 && std::isfinite(sigma), ISO_ERR_INVALID_ARG, "sigma = %g must be finite and >= 0",
                    sigma);
        iso_sub_opts o{ISO_OMEGA_TREE, ISO_PHI_EXP_DIST, ISO_BRACKET_POW2, 2000, nullptr, nullptr};
        if (opts) o = *opts;
        ISO_REQUIRE(o.omega == ISO_OMEGA_TREE || o.omega == ISO_OMEGA_FULL, ISO_ERR_INVALID_ARG,
                    "unsupported omega reading %d", o.omega);
        ISO_REQUIRE(o.omega != ISO_OMEGA_FULL || o.omega0 != nullptr, ISO_ERR_INVALID_ARG,
                    "ISO_OMEGA_FULL needs the vertex weights in opts->omega0");
        ISO_REQUIRE(o.phi == ISO_PHI_EXP_DIST || o.phi == ISO_PHI_GAUSS_SQ, ISO_ERR_INVALID_ARG, "unknown phi %d", o.phi);
        ISO_REQUIRE(o.bracket == ISO_BRACKET_POW2 || o.bracket == ISO_BRACKET_PAPER, ISO_ERR_INVALID_ARG,
                    "unknown bracket %d", o.bracket);
        require_device();
        hipStream_t s = static_cast<hipStream_t>(stream);
        SubPlan P{};
        P.n = n;
        P.k = kmax;
        const size_t need = sub_plan_bytes(n, kmax);
        ScopedWorkspace owned;
        if (ws == nullptr) {
            owned.stream = s;
            HIP_CHECK(hipMallocAsync(&owned.ptr, need, s));
            ws = owned.ptr;
            ws_bytes = need;
        }
        ISO_REQUIRE(ws_bytes >= need, ISO_ERR_WORKSPACE, "workspace %zu bytes < required %zu", ws_bytes, need);
        Arena a{static_cast<char *>(ws), 0, ws_bytes};
        P.carve(a);
        double ik_dummy = 0.0;
        run_sub(P, parent, length, root, sigma, o, P.lab_tmp, &ik_dummy, nullptr, nullptr, nullptr, nullptr, s, kmax,
                i_k, labels, passes);
    });
}

extern "C" iso_status iso_subpartition(const int32_t *parent, const double *length, int64_t n, int32_t root, int32_t k,
                                       double sigma, const iso_sub_opts *opts, int32_t *labels, double *i_k,
                                       double *cluster_num, double *cluster_den, int32_t *cluster_size,
                                       iso_sub_info *info, void *ws, size_t ws_bytes, void *stream) {
    return guarded([&] {
        ISO_REQUIRE(parent && length && labels && i_k, ISO_ERR_INVALID_ARG,
                    "parent, length, labels and i_k must be non-NULL");
        ISO_REQUIRE(n >= 2 && n < (int64_t(1) << 31) - 2, ISO_ERR_INVALID_ARG, "n = %lld outside [2, 2^31)", (long long)n);
        ISO_REQUIRE(k >= 2 && k <= n, ISO_ERR_INVALID_ARG, "k = %d outside [2, n]", k);
        ISO_REQUIRE(root >= 0 && root < n, ISO_ERR_INVALID_ARG, "root = %d outside [0, n)", root);
        ISO_REQUIRE(sigma >= 0.0 && std::isfinite(sigma), ISO_ERR_INVALID_ARG, "sigma = %g must be finite and >= 0",
                    sigma);
        iso_sub_opts o{ISO_OMEGA_TREE, ISO_PHI_EXP_DIST, ISO_BRACKET_POW2, 2000, nullptr, nullptr};
        if (opts) o = *opts;
        ISO_REQUIRE(o.omega == ISO_OMEGA_TREE || o.omega == ISO_OMEGA_FULL, ISO_ERR_INVALID_ARG,
                    "unsupported omega reading %d", o.omega);
        ISO_REQUIRE(o.omega != ISO_OMEGA_FULL || o.omega0 != nullptr, ISO_ERR_INVALID_ARG,
                    "ISO_OMEGA_FULL needs the vertex weights in opts->omega0");
        ISO_REQUIRE(o.phi == ISO_PHI_EXP_DIST || o.phi == ISO_PHI_GAUSS_SQ, ISO_ERR_INVALID_ARG, "unknown phi %d", o.phi);
        ISO_REQUIRE(o.bracket == ISO_BRACKET_POW2 || o.bracket == ISO_BRACKET_PAPER, ISO_ERR_INVALID_ARG,
                    "unknown bracket %d", o.bracket);
        require_device();
        hipStream_t s = static_cast<hipStream_t>(stream);
        SubPlan P{};
        P.n = n;
        P.k = k;
        const size_t need = sub_plan_bytes(n, k);
        ScopedWorkspace owned;
        if (ws == nullptr) {
            owned.stream = s;
            HIP_CHECK(hipMallocAsync(&owned.ptr, need, s));
            ws = owned.ptr;
            ws_bytes = need;
        }
        ISO_REQUIRE(ws_bytes >= need, ISO_ERR_WORKSPACE, "workspace %zu bytes < required %zu", ws_bytes, need);
        Arena a{static_cast<char *>(ws), 0, ws_bytes};
        P.carve(a);
        run_sub(P, parent, length, root, sigma, o, labels, i_k, cluster_num, cluster_den, cluster_size, info, s);
    });
}

extern "C" iso_status iso_subpartition_noalloc(const int32_t *parent, const double *length, int64_t n, int32_t root,
                                               int32_t k, double sigma, const iso_sub_opts *opts, int32_t *labels,
                                               double *i_k, double *cluster_num, double *cluster_den,
                                               int32_t *cluster_size, iso_sub_info *info, void *stream) {
    return guarded([&] {
        ISO_REQUIRE(parent && length && labels && i_k, ISO_ERR_INVALID_ARG,
                    "parent, length, labels and i_k must be non-NULL");
        ISO_REQUIRE(n >= 2 && n <= ISO_SUB_NOALLOC_MAX_N, ISO_ERR_INVALID_ARG,
                    "n = %lld outside [2, %d] (the allocation-free entry point's maximum)", (long long)n,
                    ISO_SUB_NOALLOC_MAX_N);
        ISO_REQUIRE(k >= 2 && k <= n, ISO_ERR_INVALID_ARG, "k = %d outside [2, n]", k);
        ISO_REQUIRE(root >= 0 && root < n, ISO_ERR_INVALID_ARG, "root = %d outside [0, n)", root);
        ISO_REQUIRE(sigma >= 0.0 && std::isfinite(sigma), ISO_ERR_INVALID_ARG, "sigma = %g must be finite and >= 0",
                    sigma);
        iso_sub_opts o{ISO_OMEGA_TREE, ISO_PHI_EXP_DIST, ISO_BRACKET_POW2, 2000, nullptr, nullptr};
        if (opts) o = *opts;
        ISO_REQUIRE(o.omega == ISO_OMEGA_TREE || o.omega == ISO_OMEGA_FULL, ISO_ERR_INVALID_ARG,
                    "unsupported omega reading %d", o.omega);
        ISO_REQUIRE(o.omega != ISO_OMEGA_FULL || o.omega0 != nullptr, ISO_ERR_INVALID_ARG,
                    "ISO_OMEGA_FULL needs the vertex weights in opts->omega0");
        ISO_REQUIRE(o.phi == ISO_PHI_EXP_DIST || o.phi == ISO_PHI_GAUSS_SQ, ISO_ERR_INVALID_ARG, "unknown phi %d", o.phi);
        ISO_REQUIRE(o.bracket == ISO_BRACKET_POW2 || o.bracket == ISO_BRACKET_PAPER, ISO_ERR_INVALID_ARG,
                    "unknown bracket %d", o.bracket);
        const size_t need = sub_plan_bytes(n, k);
        ISO_REQUIRE(need <= ISO_SUB_NOALLOC_BYTES, ISO_ERR_INTERNAL, "workspace %zu bytes exceeds the fixed %zu", need,
                    (size_t)ISO_SUB_NOALLOC_BYTES);
        require_device();
        char *ws = noalloc_scratch();
        hipStream_t s = static_cast<hipStream_t>(stream);
        SubPlan P{};
        P.n = n;
        P.k = k;
        Arena a{ws, 0, (size_t)ISO_SUB_NOALLOC_BYTES};
        P.carve(a);
        run_sub(P, parent, length, root, sigma, o, labels, i_k, cluster_num, cluster_den, cluster_size, info, s);
    });
}
