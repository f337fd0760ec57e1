// graph.hip -- full-graph vertex weights of eqs. 2.2 and 2.3 on gfx950, and the
// "median MST edge" sigma.
//
//   omega0[v] = sum over j != v, ascending j, of phi(D(v, j))          (eq. 2.2)
//   p0[v]     = alpha * sum over j != v, ascending j, of D(v, j)       (eq. 2.3)
//
// D(v, j) is the square root of the FP64 left-to-right sum over coordinates of
// the squared differences (each difference and square rounded separately, as
// everywhere on the exact path), so every distance is the same double the
// FP64 definition gives.  That arithmetic is symmetric in v and j bit for bit,
// so each unordered pair's distance is formed once and used for both rows,
// while each row's sums still follow the definition's order:
//
// The points are cut into G blocks of W consecutive points.  For every pair of
// blocks (A, B), A <= B -- B ascending, A ascending within B -- k_gw_dist forms
// the W x W distances in parallel into one buffer, then k_gw_sum adds them to
// the running sums of A's rows (columns B) and of B's rows (columns A).  In
// this order a row of block R meets the column blocks 0, 1, .., G - 1 in turn
// (the pairs (0, R) .. (R, R), then (R, R + 1) .. (R, G - 1)).
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace iso {

namespace {

constexpr int GW_K = 16;           // coordinates per LDS stage
constexpr int GW_R = 4;            // elements per thread and direction of a distance tile
constexpr int GW_T = 16 * GW_R;    // rows and columns of a distance tile; W is a multiple of it
// W is at most 4096 points: the buffer (W^2 doubles, 134 MB) then stays in the
// 256 MB last-level cache between the two kernels.  At n = 50,000, d = 64 the
// sums take 6.1 ms with it, against 10.7 ms with W = 6272 (315 MB); with W = 2048
// the 256 workgroups of a pair's sums leave the CUs waiting on the exponentials'
// latency (10.6 ms).  And W is at most 2048 or W^2 at most n * GW_BUF: fewer, larger
// blocks win up to 2048 points (fewer launches) and lose above, where the sums read
// a buffer several times the L2s' 32 MB (d = 64, ms: n = 2,048 one block 0.14, two
// 0.17; n = 3,000 two of 1,536 0.21, one 0.42; n = 6,500 three of 2,176 0.54, two of
// 3,264 0.66; n = 8,000 three of 2,688 0.64, two of 4,032 0.79; but n = 5,000 0.38
// and 0.34, and at d = 784 1.75 and 1.52; no difference from n = 12,000 on).
constexpr int64_t GW_BUF = 1024, GW_WMAX = 4096;

// Dt[jj * W + ii] = D(a0 + ii, b0 + jj) for ii < wa, jj < wb: the square root of
// the sum over t (left to right) of (x_it - x_jt)^2, each difference and square
// rounded separately.  A workgroup forms a T x T tile, R x R elements per
// thread (rows 2 ti + {0, 1} + 32 a, likewise columns, so a thread's operands
// are 16-byte LDS reads of consecutive points and its stores 16 bytes wide).
// With a0 == b0 only the tiles on and above the diagonal are formed and each
// is stored twice.
//
// Bound by the FP64 vector rate: 3 instructions per pair and coordinate (no
// fused multiply-add, the definition rounds the square), of which it reaches
// 75 % (W = 3968, d = 64: 102 us a pair of blocks).  R = 8 reached 69-73 % (its
// two workgroups per CU leave a last, half empty wave of tiles).  All ordered
// pairs of n = 50,000, d = 64 took 18.3 ms; the unordered ones take 9.2 ms.
__global__ __launch_bounds__(256) void k_gw_dist(const float *__restrict__ X, int64_t d, int64_t ld, int64_t a0,
                                                 int64_t wa, int64_t b0, int64_t wb, int64_t W,
                                                 double *__restrict__ Dt) {
    constexpr int R = GW_R, T = GW_T;
    constexpr int LP = T + 2;                   // padded row of the LDS stages
    constexpr int LN = T * GW_K / 256;          // elements a thread stages per operand
    __shared__ double xr[GW_K][LP], xc[GW_K][LP];
    const bool diag = a0 == b0;
    if (diag && blockIdx.x > blockIdx.y) return;
    const int tid = threadIdx.x;
    const int ti = tid & 15, tj = tid >> 4;
    const int64_t i0 = (int64_t)blockIdx.x * T, c0 = (int64_t)blockIdx.y * T;
    double acc[R][R];
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < R; ++b) acc[a][b] = 0.0;
    // element q of a stage: coordinate q % GW_K of point q / GW_K
    float pr[LN], pc[LN];
    auto fetch = [&](int64_t t0) {
#pragma unroll
        for (int u = 0; u < LN; ++u) {
            const int q = tid + 256 * u;
            const int64_t r = q / GW_K, t = t0 + q % GW_K;
            pr[u] = (i0 + r < wa && t < d) ? X[(a0 + i0 + r) * ld + t] : 0.0f;
            pc[u] = (c0 + r < wb && t < d) ? X[(b0 + c0 + r) * ld + t] : 0.0f;
        }
    };
    fetch(0);
    for (int64_t t0 = 0; t0 < d; t0 += GW_K) {
#pragma unroll
        for (int u = 0; u < LN; ++u) {
            const int q = tid + 256 * u;
            xr[q % GW_K][q / GW_K] = (double)pr[u];
            xc[q % GW_K][q / GW_K] = (double)pc[u];
        }
        __syncthreads();
        if (t0 + GW_K < d) fetch(t0 + GW_K);  // the next stage's loads run under this stage's arithmetic
        const int tn = d - t0 < GW_K ? (int)(d - t0) : GW_K;
        for (int c = 0; c < tn; ++c) {
            double xa[R], xb[R];
#pragma unroll
            for (int a = 0; a < R; a += 2) {
                const double2 v = *reinterpret_cast<const double2 *>(&xr[c][2 * ti + 16 * a]);
                xa[a] = v.x;
                xa[a + 1] = v.y;
                const double2 w = *reinterpret_cast<const double2 *>(&xc[c][2 * tj + 16 * a]);
                xb[a] = w.x;
                xb[a + 1] = w.y;
            }
#pragma unroll
            for (int a = 0; a < R; ++a)
#pragma unroll
                for (int b = 0; b < R; ++b) {
                    const double df = xa[a] - xb[b];
                    const double sq = df * df;
                    acc[a][b] = acc[a][b] + sq;
                }
        }
        __syncthreads();
    }
    // (element a of a thread is row 16 (a & ~1) + 2 ti + (a & 1) of the tile; W
    // is even and at least wa, so the second of a pair may be padding but lies
    // in the buffer)
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < R; ++b) acc[a][b] = sqrt(acc[a][b]);
#pragma unroll
    for (int b = 0; b < R; ++b) {
        const int64_t jj = c0 + 16 * (b & ~1) + 2 * tj + (b & 1);
        if (jj >= wb) continue;
#pragma unroll
        for (int a = 0; a < R; a += 2) {
            const int64_t ii = i0 + 16 * a + 2 * ti;
            if (ii < wa) *reinterpret_cast<double2 *>(Dt + jj * W + ii) = make_double2(acc[a][b], acc[a + 1][b]);
        }
    }
    if (diag && blockIdx.x != blockIdx.y) {
#pragma unroll
        for (int a = 0; a < R; ++a) {
            const int64_t ii = i0 + 16 * (a & ~1) + 2 * ti + (a & 1);
            if (ii >= wa) continue;
#pragma unroll
            for (int b = 0; b < R; b += 2) {
                const int64_t jj = c0 + 16 * b + 2 * tj;
                if (jj < wb) *reinterpret_cast<double2 *>(Dt + ii * W + jj) = make_double2(acc[a][b], acc[a][b + 1]);
            }
        }
    }
}

// Adds the buffer's distances (and phi of them) to the rows' sums, ascending
// column, the row's own column skipped.  Workgroups 0 .. ra-1 take GW_SR rows of
// block A each (columns: block B), the following ones GW_SR rows of block B
// (columns: block A; none when the blocks are the same).  Eight waves load and
// map GW_SC columns at a time into one of two LDS buffers while the ninth, one
// lane per row and sum, adds the other buffer's columns in order; the loads run
// GW_AHEAD steps ahead (the barrier orders LDS only, so they stay in flight).
// The row's own column and the padding columns hold +0, which leaves the
// (nonnegative) sums as they are, so the chain of additions has no branches.
// Bound by the latency of the exponentials (about 35 dependent FP64
// instructions): two elements per thread and 18 waves per workgroup pair on a
// CU hide it better than four (7.0 ms at n = 50,000) or a branch and an LDS
// round trip per column in the adding wave (11.5 ms).
// `first` marks the pair in which the rows' sums start (bit 0: A's rows, bit 1:
// B's), `last` the one that completes them: the potential is then scaled.
constexpr int GW_SR = 16, GW_SC = 64, GW_PT = 512, GW_SQ = GW_SR * GW_SC / GW_PT, GW_SB = 16, GW_AHEAD = 2;
template <int PHI, bool WO, bool WP>
__global__ __launch_bounds__(64 + GW_PT) void k_gw_sum(const double *__restrict__ Dt, int64_t a0, int64_t wa, int64_t b0,
                                                int64_t wb, int64_t W, double sigma, double alpha, int first, int last,
                                                unsigned ra, double *__restrict__ so, double *__restrict__ sp) {
    constexpr int NQ = (WO ? 1 : 0) + (WP ? 1 : 0);  // sums per row: omega, then the potential
    __shared__ __attribute__((aligned(16))) double buf[2][NQ][GW_SR][GW_SC + 2];
    const int tid = threadIdx.x;
    const bool role_b = blockIdx.x >= ra;
    const int bit = role_b ? 2 : 1;
    const int64_t r0 = (int64_t)(role_b ? blockIdx.x - ra : blockIdx.x) * GW_SR;
    const int64_t rows = role_b ? wb : wa, cols = role_b ? wa : wb;
    const int64_t row_base = role_b ? b0 : a0, col_base = role_b ? a0 : b0;
    const int steps = (int)((cols + GW_SC - 1) / GW_SC);
    const bool producer = tid >= 64;
    const int p = tid - 64;
    double v[GW_AHEAD][GW_SQ];  // the elements of the next GW_AHEAD steps
    // element q of this producer in a step: column cl0 + dcl q, row rl0 + drl q
    const int cl0 = role_b ? p % GW_SC : p / GW_SR, dcl = role_b ? 0 : GW_PT / GW_SR;
    const int rl0 = role_b ? p / GW_SC : p % GW_SR, drl = role_b ? GW_PT / GW_SC : 0;
    auto fetch = [&](int step, double(&x)[GW_SQ]) {
#pragma unroll
        for (int q = 0; q < GW_SQ; ++q) {
            const int64_t c = (int64_t)step * GW_SC + cl0 + dcl * q, rr = r0 + rl0 + drl * q;
            x[q] = (c < cols && rr < rows) ? Dt[role_b ? rr * W + c : c * W + rr] : 0.0;
        }
    };
    // lane tid < NQ * GW_SR adds sum tid / GW_SR of row tid % GW_SR
    const int sq = tid / GW_SR, sr = tid % GW_SR;
    const int64_t r = r0 + sr;
    const bool adds = tid < NQ * GW_SR && r < rows;
    const bool pot = WP && (!WO || sq == 1);
    double *const sum = pot ? sp : so;
    double a = 0.0;
    if (producer) {
#pragma unroll
        for (int u = 0; u < GW_AHEAD; ++u) fetch(u, v[u]);
    } else if (adds && !(first & bit)) {
        a = sum[row_base + r];
    }
    auto one_step = [&](int step, double(&x)[GW_SQ]) {
        const int hb = step & 1;
        if (producer) {
#pragma unroll
            for (int q = 0; q < GW_SQ; ++q) {
                const int cl = cl0 + dcl * q, rl = rl0 + drl * q;
                const double dist = x[q];
                const int64_t c = (int64_t)step * GW_SC + cl;
                const bool in = c < cols && col_base + c != row_base + r0 + rl;
                if (WP) buf[hb][NQ - 1][rl][cl] = in ? dist : 0.0;
                if (WO) {
                    const double f =
                        PHI == ISO_PHI_GAUSS_SQ ? exp(-(dist * dist) / (2.0 * sigma * sigma)) : exp(-dist / sigma);
                    buf[hb][0][rl][cl] = in ? f : 0.0;
                }
            }
            fetch(step + GW_AHEAD, x);
        }
        lds_barrier();  // (the adding wave is done with this buffer's last contents: it added them before this barrier)
        if (tid < NQ * GW_SR) {
#pragma unroll
            for (int c0 = 0; c0 < GW_SC; c0 += GW_SB) {
                double2 f[GW_SB / 2];
#pragma unroll
                for (int c = 0; c < GW_SB / 2; ++c)
                    f[c] = *reinterpret_cast<const double2 *>(&buf[hb][sq][sr][c0 + 2 * c]);
#pragma unroll
                for (int c = 0; c < GW_SB / 2; ++c) {
                    a = a + f[c].x;
                    a = a + f[c].y;
                }
            }
        }
    };
    for (int step = 0; step < steps; step += GW_AHEAD) {
#pragma unroll
        for (int u = 0; u < GW_AHEAD; ++u)
            if (step + u < steps) one_step(step + u, v[u]);
    }
    if (adds) sum[row_base + r] = (pot && (last & bit)) ? alpha * a : a;
}

__global__ void k_gw_zero(double *__restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

}  // namespace

}  // namespace iso

using namespace iso;

extern "C" iso_status iso_graph_weights(const float *X, int64_t n, int64_t d, int64_t ld, double sigma,
                                        int32_t phi_kind, double alpha, double *omega0, double *p0, void *stream) {
    return guarded([&] {
        ISO_REQUIRE(X != nullptr, ISO_ERR_INVALID_ARG, "X must be non-NULL");
        ISO_REQUIRE(n >= 2 && n < (int64_t(1) << 31), ISO_ERR_INVALID_ARG, "n = %lld outside [2, 2^31)", (long long)n);
        ISO_REQUIRE(d >= 1, ISO_ERR_INVALID_ARG, "d = %lld < 1", (long long)d);
        ISO_REQUIRE(ld >= d, ISO_ERR_INVALID_ARG, "ld = %lld < d = %lld", (long long)ld, (long long)d);
        ISO_REQUIRE(sigma > 0.0 && std::isfinite(sigma), ISO_ERR_INVALID_ARG, "sigma = %g must be finite and > 0", sigma);
        ISO_REQUIRE(alpha >= 0.0 && std::isfinite(alpha), ISO_ERR_INVALID_ARG, "alpha = %g must be finite and >= 0",
                    alpha);
        ISO_REQUIRE(phi_kind == ISO_PHI_EXP_DIST || phi_kind == ISO_PHI_GAUSS_SQ, ISO_ERR_INVALID_ARG, "unknown phi %d",
                    phi_kind);
        require_device();
        if (omega0 == nullptr && p0 == nullptr) return;
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (p0 != nullptr && alpha == 0.0) {
            hipLaunchKernelGGL(k_gw_zero, dim3(grid_for(n, 256)), dim3(256), 0, s, p0, n);
            LAUNCH_CHECK();
            p0 = nullptr;
            if (omega0 == nullptr) return;
        }
        // G blocks of W points (see GW_WMAX)
        auto width = [&](int64_t g) { return (n + g * GW_T - 1) / (g * GW_T) * GW_T; };
        int64_t G = 1;
        while (width(G) > GW_WMAX || (width(G) > 2048 && width(G) * width(G) > n * GW_BUF)) ++G;
        int64_t W = width(G);
        // the buffer: allocated and released in stream order (no synchronisation)
        struct StreamBuffer {
            void *p = nullptr;
            hipStream_t s = nullptr;
            ~StreamBuffer() {
                if (p) (void)hipFreeAsync(p, s);
            }
        } buf;
        buf.s = s;
        // (where there is no room for it, smaller blocks: the sums are the same for any W)
        hipError_t e = hipMallocAsync(&buf.p, sizeof(double) * (size_t)(W * W), s);
        while (e == hipErrorOutOfMemory && W > GW_T) {
            (void)hipGetLastError();
            W = (W / 2 + GW_T - 1) / GW_T * GW_T;
            e = hipMallocAsync(&buf.p, sizeof(double) * (size_t)(W * W), s);
        }
        if (e != hipSuccess) buf.p = nullptr;
        HIP_CHECK(e);
        G = (n + W - 1) / W;
        double *Dt = static_cast<double *>(buf.p);
        for (int64_t B = 0; B < G; ++B) {
            for (int64_t A = 0; A <= B; ++A) {
                const int64_t a0 = A * W, wa = std::min(W, n - a0), b0 = B * W, wb = std::min(W, n - b0);
                hipLaunchKernelGGL(k_gw_dist, dim3((unsigned)((wa + GW_T - 1) / GW_T), (unsigned)((wb + GW_T - 1) / GW_T)),
                                   dim3(256), 0, s, X, d, ld, a0, wa, b0, wb, W, Dt);
                LAUNCH_CHECK();
                const unsigned ra = (unsigned)((wa + GW_SR - 1) / GW_SR);
                const unsigned rb = A == B ? 0u : (unsigned)((wb + GW_SR - 1) / GW_SR);
                const int first = (B == 0 ? 1 : 0) | (A == 0 ? 2 : 0), last = (B == G - 1 ? 1 : 0);
                auto sum = [&](auto kern) {
                    hipLaunchKernelGGL(kern, dim3(ra + rb), dim3(64 + GW_PT), 0, s, Dt, a0, wa, b0, wb, W, sigma, alpha,
                                       first, last, ra, omega0, p0);
                };
                const bool gauss = phi_kind == ISO_PHI_GAUSS_SQ;
                if (omega0 && p0)
                    sum(gauss ? k_gw_sum<ISO_PHI_GAUSS_SQ, true, true> : k_gw_sum<ISO_PHI_EXP_DIST, true, true>);
                else if (omega0)
                    sum(gauss ? k_gw_sum<ISO_PHI_GAUSS_SQ, true, false> : k_gw_sum<ISO_PHI_EXP_DIST, true, false>);
                else
                    sum(k_gw_sum<ISO_PHI_EXP_DIST, false, true>);
                LAUNCH_CHECK();
            }
        }
    });
}

extern "C" iso_status iso_sigma_median(const int32_t *parent, const double *length, int64_t n, double *sigma,
                                       void *stream) {
    return guarded([&] {
        ISO_REQUIRE(parent && length && sigma, ISO_ERR_INVALID_ARG, "parent, length and sigma must be non-NULL");
        ISO_REQUIRE(n >= 2 && n < (int64_t(1) << 31), ISO_ERR_INVALID_ARG, "n = %lld outside [2, 2^31)", (long long)n);
        require_device();
        hipStream_t s = static_cast<hipStream_t>(stream);
        ScopedWorkspace owned;
        owned.stream = s;
        const size_t need = radix_select_scratch_bytes() + 256;
        HIP_CHECK(hipMallocAsync(&owned.ptr, need, s));
        double *out = static_cast<double *>(owned.ptr);
        void *scratch = static_cast<char *>(owned.ptr) + 256;
        // lower median of the n - 1 edge lengths: rank (n - 2) / 2, the root skipped
        radix_select_f64(length, parent, n, (n - 2) / 2, out, scratch, s);
        HIP_CHECK(hipMemcpyAsync(sigma, out, sizeof(double), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
    });
}
