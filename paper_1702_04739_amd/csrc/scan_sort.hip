// scan_sort.hip -- error state, device check, and the generic primitives the
// pipeline needs: exclusive scan, stable radix sort, radix select.
#include <algorithm>
#include <cstring>

#include "common.hpp"

namespace iso {

// ------------------------------------------------------------------ errors

static thread_local char g_err[512] = "no error";

void set_error(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

const char *get_error() { return g_err; }

void require_device() {
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    ISO_REQUIRE(e == hipSuccess && count > 0, ISO_ERR_NO_DEVICE, "no HIP device available (%s)",
                e == hipSuccess ? "device count is 0" : hipGetErrorString(e));
    int dev = 0;
    HIP_CHECK(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_CHECK(hipGetDeviceProperties(&prop, dev));
    ISO_REQUIRE(std::strncmp(prop.gcnArchName, "gfx950", 6) == 0, ISO_ERR_NO_DEVICE,
                "device %d is %s; this library is built for gfx950 only", dev, prop.gcnArchName);
}

int device_cus() {
    static int cached[64] = {0};
    int dev = 0;
    HIP_CHECK(hipGetDevice(&dev));
    if (dev >= 0 && dev < 64 && cached[dev] > 0) return cached[dev];
    int cus = 0;
    HIP_CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    ISO_REQUIRE(cus > 0, ISO_ERR_HIP, "device %d reports %d compute units", dev, cus);
    if (dev >= 0 && dev < 64) cached[dev] = cus;
    return cus;
}

// ------------------------------------------------------------------ timing

static iso_timing g_timing{};

iso_timing &timing() { return g_timing; }

// ------------------------------------------------------------------ exclusive scan (one workgroup)

constexpr int SCAN_BLOCK = 1024;

__device__ inline int32_t wave_inclusive_scan(int32_t v) {
    const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        int32_t o = __shfl_up(v, off, WAVE);
        if (lane >= off) v += o;
    }
    return v;
}

// Exclusive scan of a tile of up to CH * 4096 elements by one workgroup of 1024
// threads, from `off`; returns off + the tile's sum.  Wave w holds elements
// [w CH 256, (w + 1) CH 256) of the tile, four neighbours per lane and step, so
// every load is in flight before the first is used and one barrier joins the
// waves' totals.  Loads are whole 16-byte groups: `in` is 16-byte aligned and
// its allocation readable to the end of the last group (every array of a
// workspace is padded to 256 bytes).  Latency is what bounds it: 50,000
// elements in one workgroup take 6.5 us (21 to 36 with a strided walk per thread).
constexpr int SCAN_STEP = 256;  // elements of a wave's step

template <int CH>
__device__ __forceinline__ int32_t scan_tile(const int32_t *in, int32_t *out, int64_t n, int64_t tile, int32_t off) {
    __shared__ int32_t wave_sums[SCAN_BLOCK / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int64_t base = tile * (CH * SCAN_STEP * (SCAN_BLOCK / WAVE)) + (int64_t)w * (CH * SCAN_STEP) + 4 * lane;
    const int64_t last = (n - 1) & ~int64_t(3);
    int32_t v[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int4 x = *reinterpret_cast<const int4 *>(in + min(base + c * SCAN_STEP, last));
        v[c][0] = x.x;
        v[c][1] = x.y;
        v[c][2] = x.z;
        v[c][3] = x.w;
    }
    // within the wave: each group's prefix, the groups before it, the steps before
    int32_t run = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        int32_t sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t x = base + c * SCAN_STEP + e < n ? v[c][e] : 0;
            v[c][e] = sum;
            sum += x;
        }
        const int32_t inc = wave_inclusive_scan(sum), before = run + inc - sum;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[c][e] += before;
        run += __shfl(inc, WAVE - 1, WAVE);
    }
    if (lane == 0) wave_sums[w] = run;
    __syncthreads();
    int32_t add = off, all = off;
#pragma unroll
    for (int q = 0; q < SCAN_BLOCK / WAVE; ++q) {
        if (q < w) add += wave_sums[q];
        all += wave_sums[q];
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t i = base + c * SCAN_STEP;
        const int4 x = make_int4(v[c][0] + add, v[c][1] + add, v[c][2] + add, v[c][3] + add);
        if (i + 4 <= n && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
            *reinterpret_cast<int4 *>(out + i) = x;
        } else {
            if (i < n) out[i] = x.x;
            if (i + 1 < n) out[i + 1] = x.y;
            if (i + 2 < n) out[i + 2] = x.z;
            if (i + 3 < n) out[i + 3] = x.w;
        }
    }
    return all;
}

// One workgroup, tile after tile (in may be out: every load of a tile comes
// before its first store).
template <int CH>
__global__ __launch_bounds__(SCAN_BLOCK) void k_exclusive_scan(const int32_t *in, int32_t *out, int64_t n,
                                                               int32_t *total) {
    int32_t all = 0;
    for (int64_t tile = 0; tile * (CH * SCAN_STEP * (SCAN_BLOCK / WAVE)) < n; ++tile) {
        all = scan_tile<CH>(in, out, n, tile, all);
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = all;
}

// Long inputs: tile sums, their exclusive scan, then each tile from its offset.
constexpr int SCAN_CH = 2;
constexpr int64_t SCAN_TILE = (int64_t)SCAN_CH * SCAN_STEP * (SCAN_BLOCK / WAVE);
constexpr int64_t SCAN_ONE = 16 * SCAN_STEP * (SCAN_BLOCK / WAVE);  // most elements left to one workgroup

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_tile_sums(const int32_t *in, int64_t n, int32_t *sums) {
    __shared__ int32_t wave_sums[SCAN_BLOCK / WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + 4 * threadIdx.x;
    const int64_t last = (n - 1) & ~int64_t(3);
    int4 x[SCAN_CH];
#pragma unroll
    for (int c = 0; c < SCAN_CH; ++c) x[c] = *reinterpret_cast<const int4 *>(in + min(base + c * 4 * SCAN_BLOCK, last));
    int32_t v = 0;
#pragma unroll
    for (int c = 0; c < SCAN_CH; ++c) {
        const int64_t i = base + c * 4 * SCAN_BLOCK;
        v += (i < n ? x[c].x : 0) + (i + 1 < n ? x[c].y : 0) + (i + 2 < n ? x[c].z : 0) + (i + 3 < n ? x[c].w : 0);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, WAVE);
    if ((threadIdx.x & (WAVE - 1)) == 0) wave_sums[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x != 0) return;
    int32_t all = 0;
    for (int q = 0; q < SCAN_BLOCK / WAVE; ++q) all += wave_sums[q];
    sums[blockIdx.x] = all;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_tile_apply(const int32_t *in, int32_t *out, int64_t n,
                                                                const int32_t *offsets) {
    (void)scan_tile<SCAN_CH>(in, out, n, blockIdx.x, offsets[blockIdx.x]);
}

static int64_t scan_tiles(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE; }

size_t scan_scratch_bytes(int64_t n) { return 2 * align_up(sizeof(int32_t) * (size_t)scan_tiles(n), 256); }

void exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, int32_t *total, int32_t *scratch,
                        hipStream_t s) {
    if (n <= 0) {
        if (total) HIP_CHECK(hipMemsetAsync(total, 0, sizeof(int32_t), s));
        return;
    }
    ISO_REQUIRE((reinterpret_cast<uintptr_t>(in) & 15) == 0, ISO_ERR_INTERNAL, "scan input is not 16-byte aligned");
    if (n <= SCAN_ONE || scratch == nullptr) {
        const int64_t step = SCAN_ONE / 16;
        auto kern = n <= step       ? k_exclusive_scan<1>
                    : n <= 4 * step ? k_exclusive_scan<4>
                                    : k_exclusive_scan<8>;
        hipLaunchKernelGGL(kern, dim3(1), dim3(SCAN_BLOCK), 0, s, in, out, n, total);
        LAUNCH_CHECK();
        return;
    }
    const int64_t tiles = scan_tiles(n);
    int32_t *sums = scratch, *offs = scratch + align_up(sizeof(int32_t) * (size_t)tiles, 256) / sizeof(int32_t);
    hipLaunchKernelGGL(k_scan_tile_sums, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, in, n, sums);
    LAUNCH_CHECK();
    exclusive_scan_i32(sums, offs, tiles, total, nullptr, s);
    hipLaunchKernelGGL(k_scan_tile_apply, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, in, out, n, offs);
    LAUNCH_CHECK();
}

// ------------------------------------------------------------------ stable radix sort

constexpr int RS_BLOCK = 256;
// Keys per workgroup: 16 per thread, or 4 up to RS_SMALL keys, where 16 leave
// most compute units idle behind a serial walk (n = 50,000, four bytes: 78 us in
// 13 workgroups, 26 in 49).
constexpr int RS_ROUNDS = 16, RS_ROUNDS_SMALL = 4;
constexpr int64_t RS_SMALL = 1 << 18;
static int rs_rounds(int64_t n) { return n <= RS_SMALL ? RS_ROUNDS_SMALL : RS_ROUNDS; }
constexpr int RS_WAVES = RS_BLOCK / WAVE;

__global__ __launch_bounds__(RS_BLOCK) void k_rs_hist(const uint32_t *keys, int64_t n, int shift,
                                                      int32_t *hist, int nblocks, int rounds) {
    __shared__ int32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_BLOCK * rounds;
    for (int r = 0; r < rounds; ++r) {
        int64_t e = base + r * RS_BLOCK + threadIdx.x;
        if (e < n) atomicAdd(&cnt[(keys[e] >> shift) & 0xFF], 1);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(RS_BLOCK) void k_rs_scatter(const uint32_t *keys, const uint32_t *vals,
                                                         uint32_t *okeys, uint32_t *ovals, int64_t n, int shift,
                                                         const int32_t *offsets, int nblocks, int rounds) {
    __shared__ int32_t run[256];
    __shared__ int32_t wcnt[RS_WAVES][256];
    const int lane = threadIdx.x & (WAVE - 1);
    const int w = threadIdx.x / WAVE;
    run[threadIdx.x] = 0;
    for (int q = 0; q < RS_WAVES; ++q) wcnt[q][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    const int64_t base = (int64_t)blockIdx.x * RS_BLOCK * rounds;
    for (int r = 0; r < rounds; ++r) {
        const int64_t e = base + r * RS_BLOCK + threadIdx.x;
        const bool valid = e < n;
        uint32_t key = valid ? keys[e] : 0u;
        uint32_t val = valid ? vals[e] : 0u;
        const int g = (key >> shift) & 0xFF;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint64_t bb = __ballot(valid && ((g >> b) & 1));
            peers &= ((g >> b) & 1) ? bb : ~bb;
        }
        const int rank = __popcll(peers & lt_mask);
        if (valid && rank == 0) wcnt[w][g] = __popcll(peers);
        __syncthreads();
        if (valid) {
            int32_t pos = run[g] + rank;
            for (int q = 0; q < w; ++q) pos += wcnt[q][g];
            int64_t dst = (int64_t)offsets[(int64_t)g * nblocks + blockIdx.x] + pos;
            okeys[dst] = key;
            ovals[dst] = val;
        }
        __syncthreads();
        int32_t add = 0;
        for (int q = 0; q < RS_WAVES; ++q) {
            add += wcnt[q][threadIdx.x];
            wcnt[q][threadIdx.x] = 0;
        }
        run[threadIdx.x] += add;
        __syncthreads();
    }
}

size_t radix_sort_scratch_bytes(int64_t n) {
    const int64_t tile = RS_BLOCK * rs_rounds(n);
    int64_t nblocks = (n + tile - 1) / tile;
    if (nblocks < 1) nblocks = 1;
    return align_up(sizeof(int32_t) * 256 * nblocks, 256);
}

void radix_sort_pairs_u32(uint32_t *keys, uint32_t *vals, uint32_t *tmp_keys, uint32_t *tmp_vals, int64_t n,
                          int key_bits, void *scratch, hipStream_t s) {
    if (n <= 1) return;
    const int rounds = rs_rounds(n);
    const int64_t tile = (int64_t)RS_BLOCK * rounds;
    const int nblocks = (int)((n + tile - 1) / tile);
    int32_t *hist = static_cast<int32_t *>(scratch);
    uint32_t *ka = keys, *va = vals, *kb = tmp_keys, *vb = tmp_vals;
    int passes = 0;
    for (int shift = 0; shift < key_bits; shift += 8) {
        hipLaunchKernelGGL(k_rs_hist, dim3(nblocks), dim3(RS_BLOCK), 0, s, ka, n, shift, hist, nblocks, rounds);
        LAUNCH_CHECK();
        exclusive_scan_i32(hist, hist, (int64_t)256 * nblocks, nullptr, nullptr, s);
        hipLaunchKernelGGL(k_rs_scatter, dim3(nblocks), dim3(RS_BLOCK), 0, s, ka, va, kb, vb, n, shift, hist,
                           nblocks, rounds);
        LAUNCH_CHECK();
        std::swap(ka, kb);
        std::swap(va, vb);
        ++passes;
    }
    if (passes & 1) {
        HIP_CHECK(hipMemcpyAsync(keys, ka, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s));
        HIP_CHECK(hipMemcpyAsync(vals, va, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s));
    }
}

// ------------------------------------------------------------------ radix select (FP64 >= 0)

// Digits of 11 bits from the top (the last one 9 bits): six rounds.  Up to
// SEL_SMALL values one workgroup runs every round in one launch; more take one
// launch per round, in which the workgroup that finishes last (a counter)
// picks the digit, so that no second launch is needed for it.
constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS;
constexpr int64_t SEL_SMALL = 16384;
constexpr int SEL_ROUNDS = 6;

struct SelState {
    uint64_t prefix;
    uint64_t mask;
    int64_t rank;
    int32_t finished, pad;
    int32_t hist[SEL_BINS];
};

__device__ inline void sel_digit(int round, int &shift, int &bits) {
    shift = round + 1 < SEL_ROUNDS ? 64 - SEL_BITS * (round + 1) : 0;
    bits = round + 1 < SEL_ROUNDS ? SEL_BITS : 64 - SEL_BITS * (SEL_ROUNDS - 1);
}

// The digit that holds rank r of the histogram h, by a workgroup of 256; the
// rank within it in *r_out.
__device__ inline int sel_pick(const int32_t *h, int64_t r, int64_t *r_out) {
    __shared__ int32_t part[256];
    __shared__ int s_digit;
    __shared__ int64_t s_rank;
    constexpr int PER = SEL_BINS / 256;
    const int tid = threadIdx.x;
    int32_t x[PER], sum = 0;
    for (int u = 0; u < PER; ++u) {
        x[u] = h[tid * PER + u];
        sum += x[u];
    }
    part[tid] = sum;
    if (tid == 0) {
        s_digit = SEL_BINS - 1;
        s_rank = r;
    }
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int32_t o = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += o;
        __syncthreads();
    }
    int64_t before = (int64_t)part[tid] - sum;
    if (r >= before && r < before + sum) {
        int u = 0;
        while (r >= before + x[u]) before += x[u++];
        s_digit = tid * PER + u;
        s_rank = r - before;
    }
    __syncthreads();
    *r_out = s_rank;
    return s_digit;
}

__global__ __launch_bounds__(256) void k_sel_init(SelState *st, int64_t rank) {
    for (int b = threadIdx.x; b < SEL_BINS; b += 256) st->hist[b] = 0;
    if (threadIdx.x == 0) {
        st->prefix = 0;
        st->mask = 0;
        st->rank = rank;
        st->finished = 0;
    }
}

__device__ inline bool sel_value(const double *vals, const int32_t *skip_if_neg, int64_t i, uint64_t *b) {
    if (skip_if_neg && skip_if_neg[i] < 0) return false;
    *b = (uint64_t)__double_as_longlong(vals[i]);
    return true;
}

__global__ __launch_bounds__(256) void k_sel_round(const double *vals, const int32_t *skip_if_neg, int64_t n,
                                                   int round, SelState *st, double *out) {
    __shared__ int32_t cnt[SEL_BINS];
    __shared__ int s_last;
    int shift, bits;
    sel_digit(round, shift, bits);
    for (int b = threadIdx.x; b < SEL_BINS; b += 256) cnt[b] = 0;
    __syncthreads();
    const uint64_t prefix = st->prefix, mask = st->mask, dm = (1ull << bits) - 1;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        uint64_t b;
        if (sel_value(vals, skip_if_neg, i, &b) && (b & mask) == prefix) atomicAdd(&cnt[(b >> shift) & dm], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < SEL_BINS; b += 256)
        if (cnt[b]) atomicAdd(&st->hist[b], cnt[b]);
    // this workgroup's counts before its arrival, the others' before the reads:
    // one fence per workgroup, between barriers (each writes back the L2), once
    // every wave's atomics have drained
    drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        s_last = atomicAdd(&st->finished, 1) == (int)gridDim.x - 1;
        __threadfence();
    }
    __syncthreads();
    if (!s_last) return;
    for (int b = threadIdx.x; b < SEL_BINS; b += 256) {
        cnt[b] = __hip_atomic_load(&st->hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        st->hist[b] = 0;
    }
    __syncthreads();
    int64_t r;
    const int digit = sel_pick(cnt, st->rank, &r);
    if (threadIdx.x == 0) {
        st->rank = r;
        st->prefix = prefix | (uint64_t)digit << shift;
        st->mask = mask | dm << shift;
        st->finished = 0;
        if (round + 1 == SEL_ROUNDS) *out = __longlong_as_double((long long)(prefix | (uint64_t)digit << shift));
    }
}

__global__ __launch_bounds__(256) void k_sel_small(const double *vals, const int32_t *skip_if_neg, int64_t n,
                                                   int64_t rank, double *out) {
    __shared__ int32_t cnt[SEL_BINS];
    uint64_t prefix = 0, mask = 0;
    for (int round = 0; round < SEL_ROUNDS; ++round) {
        int shift, bits;
        sel_digit(round, shift, bits);
        const uint64_t dm = (1ull << bits) - 1;
        for (int b = threadIdx.x; b < SEL_BINS; b += 256) cnt[b] = 0;
        __syncthreads();
#pragma unroll 8
        for (int64_t i = threadIdx.x; i < n; i += 256) {
            uint64_t b;
            if (sel_value(vals, skip_if_neg, i, &b) && (b & mask) == prefix) atomicAdd(&cnt[(b >> shift) & dm], 1);
        }
        __syncthreads();
        const int digit = sel_pick(cnt, rank, &rank);
        prefix |= (uint64_t)digit << shift;
        mask |= dm << shift;
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = __longlong_as_double((long long)prefix);
}

size_t radix_select_scratch_bytes() { return align_up(sizeof(SelState), 256); }

void radix_select_f64(const double *vals, const int32_t *skip_if_neg, int64_t n, int64_t rank, double *out,
                      void *scratch, hipStream_t s) {
    if (n <= SEL_SMALL) {
        hipLaunchKernelGGL(k_sel_small, dim3(1), dim3(256), 0, s, vals, skip_if_neg, n, rank, out);
        LAUNCH_CHECK();
        return;
    }
    SelState *st = static_cast<SelState *>(scratch);
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, s, st, rank);
    LAUNCH_CHECK();
    const unsigned g = std::min<unsigned>(grid_for(n, 1024), 256u);
    for (int round = 0; round < SEL_ROUNDS; ++round) {
        hipLaunchKernelGGL(k_sel_round, dim3(g), dim3(256), 0, s, vals, skip_if_neg, n, round, st, out);
        LAUNCH_CHECK();
    }
}

// ------------------------------------------------------------------ histogram

namespace {

__global__ __launch_bounds__(256) void k_hist_lds(const int32_t *__restrict__ key, int64_t n, int32_t nbins,
                                                  int32_t *__restrict__ count) {
    __shared__ int32_t h[HIST_LDS_BINS];
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) h[b] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t k = key[i];
        if (k >= 0 && k < nbins) atomicAdd(&h[k], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += blockDim.x)
        if (h[b]) atomicAdd(&count[b], h[b]);
}

__global__ void k_hist_global(const int32_t *__restrict__ key, int64_t n, int64_t nbins, int32_t *__restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t k = key[i];
    if (k >= 0 && k < nbins) atomicAdd(&count[k], 1);
}

}  // namespace

void histogram_i32(const int32_t *key, int64_t n, int64_t nbins, int32_t *count, hipStream_t s) {
    if (n <= 0 || nbins <= 0) return;
    if (nbins <= HIST_LDS_BINS) {
        const unsigned g = std::min<unsigned>(grid_for(n, 256), 4u * (unsigned)device_cus());
        hipLaunchKernelGGL(k_hist_lds, dim3(g), dim3(256), 0, s, key, n, (int32_t)nbins, count);
    } else {
        hipLaunchKernelGGL(k_hist_global, dim3(grid_for(n, 256)), dim3(256), 0, s, key, n, nbins, count);
    }
    LAUNCH_CHECK();
}

}  // namespace iso

extern "C" iso_status iso_timing_enable(int32_t on) {
    iso::g_timing = iso_timing{};
    iso::g_timing.enabled = on ? 1 : 0;
    return ISO_OK;
}

extern "C" iso_status iso_timing_read(iso_timing *out) {
    if (!out) {
        iso::set_error("out is NULL");
        return ISO_ERR_INVALID_ARG;
    }
    *out = iso::g_timing;
    return ISO_OK;
}
