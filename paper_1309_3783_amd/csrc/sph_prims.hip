// Device-wide primitives for the cell build: exclusive scan of uint32 and a
// stable LSD radix sort of (uint64 key, uint32 value) pairs.  Both are
// written for 64-lane wavefronts: the scan uses wave shuffles, the radix
// scatter ranks equal digits inside a wave with eight ballots and across the
// waves of a block through LDS, which keeps the sort stable.
#include "sph_prims.h"

#include <algorithm>

namespace sph {

// ---------------------------------------------------------------------------
// Exclusive scan
// ---------------------------------------------------------------------------
constexpr int SCAN_BS = 256;
constexpr int SCAN_IPT = 8;
constexpr int SCAN_TILE = SCAN_BS * SCAN_IPT;

__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

// Block exclusive scan of one value per thread; returns the block total.
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* s_w, uint32_t& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        uint32_t x = s_w[k];
        if (k < w) base += x;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return base + inc - v;
}

// The scans of a launch: one per blockIdx.y (k_scan_small: per block).  A build
// of few particles is bound by its launches, of which scans were a quarter.
struct ScanJobs {
    ScanJob j[SCAN_JOBS];
    uint32_t* bsum;        // partial sums of a job's tiles, `stride` words per job
    int64_t stride;
};

__global__ __launch_bounds__(SCAN_BS) void k_scan_reduce(ScanJobs a) {
    const ScanJob& J = a.j[blockIdx.y];
    const uint32_t* __restrict__ in = J.in;
    const int64_t n = J.n;
    uint32_t* __restrict__ bsum = a.bsum + blockIdx.y * a.stride;
    if ((int64_t)blockIdx.x * SCAN_TILE >= n) return;
    __shared__ uint32_t s_w[SCAN_BS / 64];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; ++k) {
        int64_t i = base + (int64_t)k * SCAN_BS + threadIdx.x;
        if (i < n) acc += in[i];
    }
    uint32_t tot;
    block_excl_scan(acc, s_w, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Single block: exclusive scan of the block sums, sequential over chunks.
__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* __restrict__ bsum, int64_t nb,
                                                   uint32_t* __restrict__ total) {
    __shared__ uint32_t s_w[16];
    uint32_t carry = 0;
    for (int64_t s = 0; s < nb; s += 1024) {
        int64_t i = s + threadIdx.x;
        uint32_t v = i < nb ? bsum[i] : 0;
        uint32_t tot;
        uint32_t ex = block_excl_scan(v, s_w, tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

__global__ __launch_bounds__(SCAN_BS) void k_scan_apply(const uint32_t* __restrict__ in,
                                                        uint32_t* __restrict__ out, int64_t n,
                                                        const uint32_t* __restrict__ bsum) {
    __shared__ uint32_t s_w[SCAN_BS / 64];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    uint32_t v[SCAN_IPT];
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; ++k) {
        int64_t i = base + k;
        v[k] = i < n ? in[i] : 0;
        acc += v[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan(acc, s_w, tot) + bsum[blockIdx.x];
#pragma unroll
    for (int k = 0; k < SCAN_IPT; ++k) {
        int64_t i = base + k;
        if (i < n) out[i] = ex;
        ex += v[k];
    }
}

// Inputs up to SCAN_SMALL elements: one block stages them in LDS with
// coalesced loads, each thread scans a contiguous run of SCAN_SMALL / 1024,
// and the results go back coalesced (one launch instead of three).
constexpr int64_t SCAN_SMALL = 32768;
// (element i sits at i + i/32 in LDS: a thread's run of consecutive
// elements then spreads over all banks)
__device__ __forceinline__ int scan_pad(int i) { return i + (i >> 5); }
__global__ __launch_bounds__(1024) void k_scan_small(ScanJobs a) {
    const ScanJob& J = a.j[blockIdx.x];
    const uint32_t* in = J.in;
    uint32_t* out = J.out;
    const int64_t n = J.n;
    uint32_t* __restrict__ total = J.total;
    __shared__ uint32_t s_v[SCAN_SMALL + SCAN_SMALL / 32];
    __shared__ uint32_t s_w[16];
#pragma unroll 8
    for (int i = threadIdx.x; i < (int)n; i += 1024) s_v[scan_pad(i)] = in[i];
    __syncthreads();
    constexpr int PER = (int)(SCAN_SMALL / 1024);
    const int base = (int)threadIdx.x * PER;
    uint32_t v[PER];
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        v[k] = base + k < n ? s_v[scan_pad(base + k)] : 0u;
        acc += v[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan(acc, s_w, tot);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (base + k < n) s_v[scan_pad(base + k)] = ex;
        ex += v[k];
    }
    __syncthreads();
#pragma unroll 8
    for (int i = threadIdx.x; i < (int)n; i += 1024) out[i] = s_v[scan_pad(i)];
    if (threadIdx.x == 0 && total) *total = tot;
}

// Up to SCAN_MID_BLOCKS tiles: the apply step sums the partial sums of the
// tiles before its own (two launches instead of three).
__global__ __launch_bounds__(SCAN_BS) void k_scan_apply_mid(ScanJobs a) {
    const ScanJob& J = a.j[blockIdx.y];
    const uint32_t* __restrict__ in = J.in;
    uint32_t* __restrict__ out = J.out;
    const int64_t n = J.n, nb = max((n + SCAN_TILE - 1) / SCAN_TILE, (int64_t)1);
    const uint32_t* __restrict__ bsum = a.bsum + blockIdx.y * a.stride;
    uint32_t* __restrict__ total = J.total;
    if ((int64_t)blockIdx.x >= nb) return;
    if (n == 0) {
        if (threadIdx.x == 0 && total) *total = 0;
        return;
    }
    __shared__ uint32_t s_w[SCAN_BS / 64];
    // offset of this tile: sum of the partial sums of the tiles before it
    uint32_t pre = 0, all = 0;
    for (int64_t k = threadIdx.x; k < nb; k += SCAN_BS) {
        const uint32_t x = bsum[k];
        if (k < (int64_t)blockIdx.x) pre += x;
        all += x;
    }
    uint32_t tp, ta;
    block_excl_scan(pre, s_w, tp);
    block_excl_scan(all, s_w, ta);
    if (blockIdx.x == nb - 1 && threadIdx.x == 0 && total) *total = ta;
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    uint32_t v[SCAN_IPT];
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; ++k) {
        int64_t i = base + k;
        v[k] = i < n ? in[i] : 0;
        acc += v[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan(acc, s_w, tot) + tp;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; ++k) {
        int64_t i = base + k;
        if (i < n) out[i] = ex;
        ex += v[k];
    }
}

size_t scan_tmp_words(int64_t n) { return (size_t)((n + SCAN_TILE - 1) / SCAN_TILE) + 1; }

hipError_t exclusive_scans(const ScanJob* jobs, int njobs, uint32_t* tmp, uint32_t* batch, hipStream_t st) {
    ScanJobs a{};
    int64_t nmax = 0;
    for (int k = 0; k < njobs; ++k) {
        a.j[k] = jobs[k];
        nmax = std::max(nmax, jobs[k].n);
    }
    if (nmax <= SCAN_SMALL) {
        hipLaunchKernelGGL(k_scan_small, dim3((unsigned)njobs), dim3(1024), 0, st, a);
        return hipGetLastError();
    }
    const int64_t nb = (nmax + SCAN_TILE - 1) / SCAN_TILE;
    a.bsum = tmp;
    a.stride = (int64_t)scan_tmp_words(nmax);
    if (nb <= SCAN_MID_BLOCKS) {
        if (njobs > 1) a.bsum = batch;
        const dim3 grid((unsigned)nb, (unsigned)njobs);
        hipLaunchKernelGGL(k_scan_reduce, grid, dim3(SCAN_BS), 0, st, a);
        hipLaunchKernelGGL(k_scan_apply_mid, grid, dim3(SCAN_BS), 0, st, a);
        return hipGetLastError();
    }
    if (njobs > 1) {
        for (int k = 0; k < njobs; ++k) {
            hipError_t e = exclusive_scan(jobs[k].in, jobs[k].out, jobs[k].n, tmp, jobs[k].total, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(SCAN_BS), 0, st, a);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, tmp, nb, jobs[0].total);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(SCAN_BS), 0, st, jobs[0].in, jobs[0].out, nmax, tmp);
    return hipGetLastError();
}

hipError_t exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* tmp, uint32_t* total,
                          hipStream_t st) {
    if (n <= 0) return total ? fill_u32(total, 1, 0, st) : hipSuccess;
    const ScanJob j{in, out, n, total};
    return exclusive_scans(&j, 1, tmp, nullptr, st);
}

// ---------------------------------------------------------------------------
// Radix sort (LSD, 8-bit digits)
// ---------------------------------------------------------------------------
constexpr int RS_BS = 256;
constexpr int RS_ROUNDS = 16;
constexpr int RS_TILE = RS_BS * RS_ROUNDS;

__global__ __launch_bounds__(1024) void k_rs_hist(const uint64_t* __restrict__ key, int64_t n, int shift,
                                                 uint32_t* __restrict__ hist, int64_t nb) {
    // the block's tile of RS_TILE elements, 1024 threads, all loads in flight
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    uint32_t d[RS_TILE / 1024];
#pragma unroll
    for (int r = 0; r < RS_TILE / 1024; ++r) {
        const int64_t i = base + (int64_t)r * 1024 + threadIdx.x;
        d[r] = i < n ? (uint32_t)(key[i] >> shift) & 255u : 256u;
    }
#pragma unroll
    for (int r = 0; r < RS_TILE / 1024; ++r)
        if (d[r] < 256u) atomicAdd(&h[d[r]], 1u);
    __syncthreads();
    if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// The lanes whose digit d equals the lane's own.
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid) {
    uint64_t match = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const uint64_t bal = __ballot(valid && ((d >> bit) & 1u));
        match &= ((d >> bit) & 1u) ? bal : ~bal;
    }
    return match;
}
// The rank of a valid lane's digit d among the equal digits its wave has met
// so far, which cnt (256 words of the wave's own) counts: no block-wide step.
__device__ __forceinline__ uint32_t wave_rank(volatile uint16_t* cnt, uint32_t d, bool valid) {
    const int lane = threadIdx.x & 63;
    const uint64_t match = same_digit(d, valid);
    const uint32_t below = __popcll(match & ~(~0ull << lane));
    uint32_t old = 0;
    if (valid) {
        old = cnt[d];
        if (below == 0) cnt[d] = (uint16_t)(old + __popcll(match));
    }
    return old + below;
}
// From the waves' digit counts c[w][d] to where each wave's run of a digit
// starts in the block's order (digit by digit, within a digit wave by wave):
// thread t stands for digit t / 4 and four of the 16 waves.
__device__ __forceinline__ void digit_starts(uint16_t (*c)[256], uint32_t* s_w) {
    const int d = threadIdx.x >> 2, w0 = 4 * (threadIdx.x & 3);
    uint32_t n[4], sum = 0, tot;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        n[k] = c[w0 + k][d];
        sum += n[k];
    }
    uint32_t at = block_excl_scan(sum, s_w, tot);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[w0 + k][d] = (uint16_t)at;
        at += n[k];
    }
}

// One pass: the tile of RS_TILE elements of this block is first placed in
// LDS in digit order (stable: within a digit, input order), then written
// out, so that runs of one digit go to consecutive addresses.  Each wave ranks
// a run of consecutive elements of its own, so that the block meets only
// between the steps.  FUSED (at most RS_FUSED blocks): hist holds the
// blocks' digit counts and the block adds up where its digits start; else the
// scanned histogram, hist[d * nb + b] = first output position of digit d of
// block b.
constexpr int RS_SBS = 1024;
constexpr int RS_SROUNDS = RS_TILE / RS_SBS;
constexpr int RS_SW = RS_SBS / 64;
constexpr int64_t RS_FUSED = 64;
static_assert(RS_SW == 16 && RS_SBS == 4 * 256, "digit_starts");
template <bool VALS, bool FUSED>
__global__ __launch_bounds__(RS_SBS) void k_rs_scatter(const uint64_t* __restrict__ kin,
                                                       const uint32_t* __restrict__ vin,
                                                       uint64_t* __restrict__ kout,
                                                       uint32_t* __restrict__ vout, int64_t n, int shift,
                                                       const uint32_t* __restrict__ hist, int64_t nb) {
    __shared__ uint64_t s_k[RS_TILE];
    __shared__ uint32_t s_v[VALS ? RS_TILE : 1];
    __shared__ uint32_t g_off[256];
    __shared__ uint16_t c[RS_SW][256];
    __shared__ uint32_t s_w[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t b = blockIdx.x;
    const int64_t base = b * RS_TILE;
    const int tile_n = (int)min((int64_t)RS_TILE, n - base);
    // the whole tile is loaded at once (all loads in flight together)
    uint64_t kr[RS_SROUNDS];
    uint32_t vr[RS_SROUNDS];
#pragma unroll
    for (int r = 0; r < RS_SROUNDS; ++r) {
        const int li = (w * RS_SROUNDS + r) * 64 + lane;
        kr[r] = li < tile_n ? kin[base + li] : 0;
        vr[r] = (VALS && li < tile_n) ? vin[base + li] : 0;
    }
    if (FUSED) {
        const int d = tid >> 2, q = tid & 3;
        uint32_t all = 0, before = 0, tot;
        for (int64_t k = q; k < nb; k += 4) {
            const uint32_t x = hist[(int64_t)d * nb + k];
            all += x;
            before += k < b ? x : 0u;
        }
        for (int m = 1; m < 4; m <<= 1) {
            all += __shfl_xor(all, m, 64);
            before += __shfl_xor(before, m, 64);
        }
        const uint32_t ex = block_excl_scan(q == 0 ? all : 0u, s_w, tot);
        if (q == 0) g_off[d] = ex + before;
    } else if (tid < 256) {
        g_off[tid] = hist[(int64_t)tid * nb + b];
    }
    for (int i = lane; i < 256; i += 64) c[w][i] = 0;
    uint32_t rank[RS_SROUNDS];
#pragma unroll
    for (int r = 0; r < RS_SROUNDS; ++r)
        rank[r] = wave_rank(c[w], (uint32_t)(kr[r] >> shift) & 255u, (w * RS_SROUNDS + r) * 64 + lane < tile_n);
    __syncthreads();
    digit_starts(c, s_w);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_SROUNDS; ++r) {
        if ((w * RS_SROUNDS + r) * 64 + lane < tile_n) {
            const uint32_t pos = c[w][(uint32_t)(kr[r] >> shift) & 255u] + rank[r];
            s_k[pos] = kr[r];
            if (VALS) s_v[pos] = vr[r];
        }
    }
    __syncthreads();
    // write out in digit order: consecutive threads, consecutive addresses
    // within a digit's run (c[0][d]: where the digit starts in the tile)
    for (int i = tid; i < tile_n; i += RS_SBS) {
        const uint64_t k = s_k[i];
        const uint32_t d = (uint32_t)(k >> shift) & 255u;
        const uint32_t pos = g_off[d] + (uint32_t)i - c[0][d];
        kout[pos] = k;
        if (VALS) vout[pos] = s_v[i];
    }
}

// Up to RSB_MAX elements: every pass in one block, keys and values in
// registers and through LDS between the passes (one launch instead of three
// per pass: 10000 keys of 40 bits took 15 launches, 85 us).
constexpr int RSB_ROUNDS = 12;
constexpr int RSB_MAX = RS_SBS * RSB_ROUNDS;
template <bool VALS>
__global__ __launch_bounds__(RS_SBS) void k_rs_block(uint64_t* __restrict__ key, uint32_t* __restrict__ val, int n,
                                                     int lo_bit, int nbits) {
    __shared__ uint64_t s_k[RSB_MAX];
    __shared__ uint32_t s_v[VALS ? RSB_MAX : 1];
    __shared__ uint16_t c[RS_SW][256];
    __shared__ uint32_t s_w[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int rounds = (n + RS_SBS - 1) / RS_SBS;
    const int first = w * rounds * 64 + lane;   // element of round r: first + 64 r
    uint64_t kr[RSB_ROUNDS];
    uint32_t vr[RSB_ROUNDS], rank[RSB_ROUNDS];
#pragma unroll
    for (int r = 0; r < RSB_ROUNDS; ++r) {
        const int li = first + 64 * r;
        const bool on = r < rounds && li < n;
        kr[r] = on ? key[li] : 0;
        vr[r] = VALS && on ? val[li] : 0;
    }
    for (int shift = lo_bit; shift < lo_bit + nbits; shift += 8) {
        for (int i = lane; i < 256; i += 64) c[w][i] = 0;
#pragma unroll
        for (int r = 0; r < RSB_ROUNDS; ++r)
            if (r < rounds) rank[r] = wave_rank(c[w], (uint32_t)(kr[r] >> shift) & 255u, first + 64 * r < n);
        __syncthreads();
        digit_starts(c, s_w);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RSB_ROUNDS; ++r) {
            if (r < rounds && first + 64 * r < n) {
                const uint32_t pos = c[w][(uint32_t)(kr[r] >> shift) & 255u] + rank[r];
                s_k[pos] = kr[r];
                if (VALS) s_v[pos] = vr[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RSB_ROUNDS; ++r) {
            const int li = first + 64 * r;
            if (r < rounds && li < n) {
                kr[r] = s_k[li];
                if (VALS) vr[r] = s_v[li];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RSB_ROUNDS; ++r) {
        const int li = first + 64 * r;
        if (r < rounds && li < n) {
            key[li] = kr[r];
            if (VALS) val[li] = vr[r];
        }
    }
}

static_assert(256 * ((1 << 20) / RS_TILE) >= SCAN_BATCH_WORDS, "the sort scratch of 2^20 elements holds a batch's words");
size_t radix_tmp_words(int64_t n) {
    int64_t nb = (n + RS_TILE - 1) / RS_TILE;
    return (size_t)(256 * nb) + scan_tmp_words(256 * nb) + 8;
}

hipError_t radix_sort(uint64_t* key, uint32_t* val, uint64_t* key_alt, uint32_t* val_alt, int64_t n,
                      int nbits, uint32_t* tmp, hipStream_t st, bool* result_in_alt, int lo_bit) {
    *result_in_alt = false;
    if (n <= 1 || nbits <= 0) return hipSuccess;
    if (lo_bit < 0 || lo_bit + nbits > 64) return hipErrorInvalidValue;
    if (n <= RSB_MAX) {
        if (val) hipLaunchKernelGGL(k_rs_block<true>, dim3(1), dim3(RS_SBS), 0, st, key, val, (int)n, lo_bit, nbits);
        else hipLaunchKernelGGL(k_rs_block<false>, dim3(1), dim3(RS_SBS), 0, st, key, val, (int)n, lo_bit, nbits);
        return hipGetLastError();
    }
    int64_t nb = (n + RS_TILE - 1) / RS_TILE;
    uint32_t* hist = tmp;
    uint32_t* stmp = tmp + 256 * nb;
    uint64_t *ka = key, *kb = key_alt;
    uint32_t *va = val, *vb = val_alt;
    const bool fused = nb <= RS_FUSED;
    auto kern = val ? (fused ? k_rs_scatter<true, true> : k_rs_scatter<true, false>)
                    : (fused ? k_rs_scatter<false, true> : k_rs_scatter<false, false>);
    for (int shift = lo_bit; shift < lo_bit + nbits; shift += 8) {
        hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)nb), dim3(1024), 0, st, ka, n, shift, hist, nb);
        if (!fused) {
            hipError_t e = exclusive_scan(hist, hist, 256 * nb, stmp, nullptr, st);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(RS_SBS), 0, st, ka, va, kb, vb, n, shift, hist, nb);
        std::swap(ka, kb);
        std::swap(va, vb);
        *result_in_alt = !*result_in_alt;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small helpers
// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill2_u32(uint32_t* p, int64_t n, uint32_t v, uint32_t* p2, int64_t n2, uint32_t v2) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
    if (i < n2) p2[i] = v2;
}

hipError_t fill2_u32(uint32_t* p, int64_t n, uint32_t v, uint32_t* p2, int64_t n2, uint32_t v2, hipStream_t st) {
    const int64_t m = std::max(n, n2);
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill2_u32, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, p, n, v, p2, n2, v2);
    return hipGetLastError();
}

hipError_t fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace sph
