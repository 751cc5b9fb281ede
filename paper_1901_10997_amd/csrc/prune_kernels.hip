// Mask updates of the pruning phases on the device (paper Section 4: magnitude-based weight pruning,
// "Msk(w) = 0 iff |w| <= the (100 p_w)-th percentile of |W|"; row/column pruning algorithm: rows / columns whose
// magnitude sum is at or below an order statistic of the row / column sums are removed).
//
// Both need a k-th smallest value of non-negative floating-point numbers, whose bit patterns order like unsigned
// integers, so the selection is a radix select by digits of eleven and ten bits.  Weight pruning: 31-bit keys (the
// magnitudes of the active entries), three passes over weights and mask.  Row/column pruning: 64-bit keys (fp64 sums), a
// few thousand of them, inside one workgroup.  Nothing returns to the host between the passes.
#include "common.h"

#include <mutex>

namespace l355 {

// ---- magnitude pruning of weights ------------------------------------------------------------------------------
// Bound: HBM (three reads of W and mask for the digits, a fourth for the update; the mask bytes that change are written).
// Every pass loads sixteen entries per thread at a time (16-byte loads of W, 4-byte loads of the mask) and counts the
// digit of the keys that match what has been fixed so far in an LDS histogram; a workgroup adds its histogram to the
// global one in order, so that a wave's additions are whole lines.  There is no kernel between the passes: every
// workgroup of a pass scans the finished histogram of the one before (8 KB) for the digit that holds the rank.  One
// workgroup of 1024 threads per compute unit keeps the number of global histogram additions small.
// 6000 x 1500: 400 us for keys, four byte-wide passes and update, -> 51 us (45 MB per pass: 3.6 TB/s).
struct WeightSelect {
    unsigned hist[3][2048];         // digits: bits 30..20, 19..10, 9..0
    unsigned prefix[2], rank[2];    // after the first and second digit: bits fixed so far, rank left among their keys
    unsigned long long active, below[2];   // active entries; entries with a smaller first / second digit
};
constexpr int kSelThreads = 1024;
// digit d = 0, 1, 2 of a key
__device__ __forceinline__ unsigned weight_digit(unsigned key, int d)
{
    return d == 0 ? key >> 20 : d == 1 ? (key >> 10) & 1023u : key & 1023u;
}

struct DigitScan { unsigned digit, below, in; unsigned long long total; };
// The digit of `hist` (2048 bins) that holds rank k (1-based), how many keys lie in smaller bins and in the bin itself.
// from_ratio: k is ceil(ratio * total) instead, at most the total.  Called by all kSelThreads threads.
__device__ __forceinline__ DigitScan scan_digits(const unsigned* __restrict__ hist, unsigned k, bool from_ratio, double ratio, unsigned* rank_out)
{
    __shared__ unsigned long long wtot[16];
    __shared__ unsigned res[3];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const unsigned a = hist[2 * tid], b = hist[2 * tid + 1];
    unsigned long long incl = (unsigned long long)a + b;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
    }
    if (lane == 63) wtot[wv] = incl;
    if (tid == 0) res[0] = res[1] = res[2] = 0u;
    __syncthreads();
    unsigned long long base = 0, total = 0;
    for (int i = 0; i < 16; ++i) {
        if (i < wv) base += wtot[i];
        total += wtot[i];
    }
    if (from_ratio) {
        const double c = (double)total, kk = ceil(ratio * c);
        k = (unsigned)(kk > c ? c : kk);
    }
    const unsigned long long below = base + incl - a - b;
    if (k > below && k <= below + a) { res[0] = 2 * tid; res[1] = (unsigned)below; res[2] = a; }
    else if (k > below + a && k <= below + a + b) { res[0] = 2 * tid + 1; res[1] = (unsigned)below + a; res[2] = b; }
    __syncthreads();
    *rank_out = k;
    const DigitScan d{res[0], res[1], res[2], total};
    __syncthreads();
    return d;
}

// f(index, key) for the active entries among 16 consecutive ones per thread; VEC: both addresses allow the wide loads
template <bool VEC, class F>
__device__ __forceinline__ void for_active_weights(const float* __restrict__ W, const uint8_t* __restrict__ mask, size_t n, F f)
{
    const size_t chunk = (size_t)gridDim.x * kSelThreads * 4;
    for (size_t i0 = ((size_t)blockIdx.x * kSelThreads + threadIdx.x) * 4; i0 < n; i0 += 4 * chunk) {
        float w[4][4];
        uint32_t m[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t i = i0 + u * chunk;
            if (VEC && i + 4 <= n) {
                const float4 v = *reinterpret_cast<const float4*>(W + i);
                w[u][0] = v.x; w[u][1] = v.y; w[u][2] = v.z; w[u][3] = v.w;
                m[u] = *reinterpret_cast<const uint32_t*>(mask + i);
            } else {
                m[u] = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    w[u][j] = 0.f;
                    if (i + j < n) { w[u][j] = W[i + j]; m[u] |= (uint32_t)mask[i + j] << (8 * j); }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            unsigned key[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) key[j] = ((m[u] >> (8 * j)) & 255u) ? (__float_as_uint(w[u][j]) & 0x7FFFFFFFu) : 0xFFFFFFFFu;
            f(i0 + u * chunk, key, m[u]);
        }
    }
}

// pass D (0, 1, 2): histogram of digit D of the keys that match the digits before it
template <int D, bool VEC>
__global__ __launch_bounds__(kSelThreads) void weight_digit_kernel(const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                                                   size_t n, WeightSelect* __restrict__ st, double ratio)
{
    __shared__ unsigned h[2048];
    for (int i = threadIdx.x; i < 2048; i += kSelThreads) h[i] = 0;
    unsigned prefix = 0;
    bool any = true;
    if constexpr (D > 0) {
        unsigned rank = D == 1 ? 0u : st->rank[0];
        const DigitScan d = scan_digits(st->hist[D - 1], rank, D == 1, ratio, &rank);
        any = rank > 0;
        prefix = D == 1 ? d.digit : (st->prefix[0] << 10) | d.digit;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->prefix[D - 1] = prefix;
            st->rank[D - 1] = any ? rank - d.below : 0u;
            st->below[D - 1] = d.below;
            if (D == 1) st->active = d.total;
        }
    }
    __syncthreads();
    if (any)
        for_active_weights<VEC>(W, mask, n, [&](size_t, const unsigned (&key)[4], uint32_t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool match = D == 0 ? key[j] != 0xFFFFFFFFu : D == 1 ? (key[j] >> 20) == prefix : (key[j] >> 10) == prefix;
                if (match) atomicAdd(&h[weight_digit(key[j], D)], 1u);
            }
        });
    __syncthreads();
    for (int i = threadIdx.x; i < 2048; i += kSelThreads)
        if (h[i]) atomicAdd(&st->hist[D][i], h[i]);
}

// mask byte to 0 where the entry is active and its key at or below the selected one (rank 0: nothing).  counts
// (device-visible): active entries before and after.
template <bool VEC>
__global__ __launch_bounds__(kSelThreads) void weight_update_kernel(const float* __restrict__ W, uint8_t* __restrict__ mask,
                                                                    size_t n, const WeightSelect* __restrict__ st,
                                                                    unsigned long long* __restrict__ counts)
{
    unsigned rank = st->rank[1];
    const DigitScan d = scan_digits(st->hist[2], rank, false, 0.0, &rank);
    const unsigned thr = (st->prefix[1] << 10) | d.digit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        counts[0] = st->active;
        counts[1] = rank > 0 ? st->active - st->below[0] - st->below[1] - d.below - d.in : st->active;
    }
    if (rank == 0) return;
    for_active_weights<VEC>(W, mask, n, [&](size_t i, const unsigned (&key)[4], uint32_t m) {
        uint32_t left = m;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (key[j] <= thr) left &= ~(255u << (8 * j));
        if (left == m) return;
        if (VEC && i + 4 <= n) *reinterpret_cast<uint32_t*>(mask + i) = left;
        else
            for (int j = 0; j < 4; ++j)
                if (i + j < n) mask[i + j] = (uint8_t)(left >> (8 * j));
    });
}

size_t prune_weights_scratch_bytes() { return sizeof(WeightSelect); }

template <bool VEC>
static hipError_t prune_weights_passes(const float* W, uint8_t* mask, size_t count, double p_w, WeightSelect* st,
                                       unsigned long long* counts, hipStream_t s)
{
    // sixteen entries per thread and round
    const size_t per = (size_t)kSelThreads * 16;
    const size_t want = (count + per - 1) / per;
    const dim3 grid((unsigned)std::min<size_t>(want, (size_t)device_num_cus())), block(kSelThreads);
    hipLaunchKernelGGL((weight_digit_kernel<0, VEC>), grid, block, 0, s, W, mask, count, st, p_w);
    hipLaunchKernelGGL((weight_digit_kernel<1, VEC>), grid, block, 0, s, W, mask, count, st, p_w);
    hipLaunchKernelGGL((weight_digit_kernel<2, VEC>), grid, block, 0, s, W, mask, count, st, p_w);
    hipLaunchKernelGGL((weight_update_kernel<VEC>), grid, block, 0, s, W, mask, count, st, counts);
    return hipGetLastError();
}

// scratch: prune_weights_scratch_bytes; counts: device-visible, active entries before and after
hipError_t launch_prune_weights(const float* W, uint8_t* mask, size_t count, double p_w, void* scratch,
                                unsigned long long* counts, hipStream_t s)
{
    WeightSelect* st = (WeightSelect*)scratch;
    const hipError_t e = launch_fill_u64((unsigned long long*)st, sizeof(WeightSelect) / 8, 0ull, s);
    if (e != hipSuccess) return e;
    const bool vec = ((uintptr_t)W & 15) == 0 && ((uintptr_t)mask & 3) == 0;
    return vec ? prune_weights_passes<true>(W, mask, count, p_w, st, counts, s) : prune_weights_passes<false>(W, mask, count, p_w, st, counts, s);
}

// ---- row / column pruning -------------------------------------------------------------------------------------
// Importance of a line (row or column) = sum of the magnitudes of its active entries, accumulated in fp64 in index
// order: s = (...((+0 + e_0) + e_1) + ...) + e_last, where e_k = |W| for an active entry and +0 otherwise (adding
// +0 to a non-negative double changes nothing).  The order is part of the definition: an fp64 sum of several
// thousand fp32 magnitudes is not exact in general, and the decision "sum <= threshold" must come out the same on
// every implementation for the masks to be reproducible bit for bit.
//
struct LineThreshold {
    double value;   // the k-th smallest sum
    unsigned any;   // 0: rank 0 was asked for, nothing is removed along this axis
    unsigned count; // lines removed
};

// Row sums.  Bound: one read of the matrix.  The order needs a chain of dependent additions only where an addition rounds,
// and most rows never round: every fp32 magnitude is a multiple of the last place of the smallest one that is not zero
// (2^q), and while the whole sum is below 2^(q + 53) every partial sum in any order is a multiple of 2^q below it, which
// fp64 holds exactly.  So the lanes of a wave sum a row together with its smallest magnitude, and the sum stands if it is
// below 2^(q + 52) (one bit spared: a sum that itself has rounded is off by a few 2^-53 per addition).  Otherwise, also for
// infinities and NaN, the wave sums the row again as the chain.  Weights left by magnitude pruning stop at its threshold and
// pass (6000 of them from a twentieth to four standard deviations: 43 bits); of rows of 1500 normal deviates one in 300
// fails.
// 6000 x 1500 (45 MB), four waves per workgroup: 25.0 -> 8.5 to 11 us against the chain for every row, normal deviates 18, 46
// where every row fails (magnitudes over 15 e-folds); 16384 x 500 22.1 -> 9.9, 3000 x 3000 21.8 -> 8.5 (normal 25.6).
constexpr int kRowWaves = 4;       // waves (rows) per workgroup
constexpr int kChainTile = 384;    // positions of a row in LDS at a time

// One row by a whole wave, in index order.  Lanes fetch a tile of positions (the next one is in flight meanwhile: a tile is
// long enough to cover the latency) and park it as fp64; every lane adds them all, from LDS reads requested a batch ahead.
// buf: the wave's own [kChainTile].
__device__ __forceinline__ double chain_sum(const float* __restrict__ w_row, const uint8_t* __restrict__ mask_row, unsigned len, double* buf)
{
    const int lane = threadIdx.x & 63;
    constexpr int kMine = kChainTile / 64, kBatch = 8, kBatches = kChainTile / 2 / kBatch;
    float w[kMine];
    uint8_t on[kMine];
    auto fetch = [&](unsigned t) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const unsigned pos = t + lane + 64 * i, at = pos < len ? pos : 0;
            w[i] = w_row[at];
            on[i] = pos < len ? mask_row[at] : (uint8_t)0;
        }
    };
    fetch(0);
    double acc = 0.0;
    for (unsigned t = 0; t < len; t += kChainTile) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) buf[lane + 64 * i] = on[i] ? (double)fabsf(w[i]) : 0.0;
        if (t + kChainTile < len) fetch(t + kChainTile);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double2* const src = reinterpret_cast<const double2*>(buf);
        const unsigned left = len - t;                                      // positions behind the end hold +0, which changes nothing
        const int n = left < kChainTile ? (int)(left + 2 * kBatch - 1) / (2 * kBatch) : kBatches;
        double2 cur[kBatch], nxt[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) cur[i] = src[i];
        for (int k = 0; k < n; ++k) {
            const int kn = k + 1 < n ? k + 1 : k;
#pragma unroll
            for (int i = 0; i < kBatch; ++i) nxt[i] = src[kn * kBatch + i];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                acc += cur[i].x;
                acc += cur[i].y;
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) cur[i] = nxt[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    return acc;
}

// Row sums, a wave per row.  VEC: four entries per load (N and both addresses allow it).
template <bool VEC>
__global__ __launch_bounds__(64 * kRowWaves) void row_abs_sum_kernel(const float* __restrict__ W, const uint8_t* __restrict__ mask, int M, int N,
                                                                     double* __restrict__ sums)
{
    __shared__ __attribute__((aligned(16))) double chain[kRowWaves][kChainTile];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = blockIdx.x * kRowWaves + wv;
    if (r >= M) return;
    const size_t first = (size_t)r * N;
    constexpr int kPer = VEC ? 4 : 1, kAhead = VEC ? 4 : 8;
    // sum of magnitudes and the smallest one's bits minus one, which puts zeros (they limit nothing) above all others
    double sum = 0.0;
    unsigned least = 0xFFFFFFFFu;
    const unsigned n = (unsigned)N;                                      // (positions past the end of the longest row fit 32 bits)
    for (unsigned c0 = lane * kPer; c0 < n; c0 += kAhead * 64 * kPer) {
        float w[kAhead][kPer];
        uint32_t on[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const unsigned c = c0 + u * 64 * kPer;
            const size_t idx = first + (c < n ? c : 0);                  // (VEC: N % 4 == 0, a load is in or out as a whole)
            if constexpr (VEC) {
                const float4 v = *reinterpret_cast<const float4*>(W + idx);
                w[u][0] = v.x; w[u][1] = v.y; w[u][2] = v.z; w[u][3] = v.w;
                on[u] = *reinterpret_cast<const uint32_t*>(mask + idx);
            } else {
                w[u][0] = W[idx];
                on[u] = mask[idx];
            }
            if (c >= n) on[u] = 0;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const float v = ((on[u] >> (8 * j)) & 255u) ? fabsf(w[u][j]) : 0.f;
                sum += (double)v;
                least = min(least, __float_as_uint(v) - 1u);
            }
    }
    for (int off = 1; off < 64; off <<= 1) {
        sum += __shfl_xor(sum, off, 64);
        least = min(least, (unsigned)__shfl_xor((int)least, off, 64));
    }
    // the smallest magnitude is a multiple of 2^(exponent - 150)
    const int exponent = (int)((least + 1u) >> 23);
    const bool exact = least == 0xFFFFFFFFu || sum < ldexp(1.0, (exponent > 0 ? exponent : 1) - 150 + 52);
    if (!exact) sum = chain_sum(W + first, mask + first, n, chain[wv]);
    if (lane == 0) sums[r] = sum;
}

// Column sums.  Bound: the chain of dependent fp64 additions down a column (about 8 clocks each: 6000 rows = 20 us), as long
// as nothing else sits on it.  A workgroup sums 16 columns: four waves fetch tiles of 512 positions (the loads of the tile
// after next are in flight while the next one is parked), select by the mask, take magnitudes, widen and park them in LDS as
// fp64, column by column; one wave, a lane per column, does nothing but 16-byte LDS reads, requested a batch ahead, and
// additions.  With 16 columns a 1500-column matrix gives 94 workgroups (64: 24, which cannot pull the matrix in at the rate
// the chain consumes it), and a tile's pitch of 514 doubles puts the 16 lanes of a read on distinct banks.
// 6000 x 1500: 849 -> 39 us (against one wave widening and adding 64 columns).  Summed like the rows 27 us, but a column has
// four times the terms, one in twenty of 6000 normal deviates fails the test, and a wave's chain down a column 70 us.
constexpr int kSumLines = 16, kSumTile = 512, kSumPitch = kSumTile + 2, kSumBatch = 16;
constexpr int kSumThreads = 320;   // one summing wave, four fetching ones
constexpr size_t kSumLds = (size_t)2 * kSumLines * kSumPitch * sizeof(double) + (size_t)2 * kSumTile * sizeof(int);

// VEC: four columns per load (N and both addresses allow it).  AFTER: lanes 16..31 sum the same columns over the rows that
// stay, i.e. those whose sum in `rsums` is above the row threshold, into sums_after.
template <bool VEC, bool AFTER>
__global__ __launch_bounds__(kSumThreads) void col_abs_sum_kernel(const float* __restrict__ W, const uint8_t* __restrict__ mask, int M, int N,
                                                                  double* __restrict__ sums, double* __restrict__ sums_after,
                                                                  const double* __restrict__ rsums,
                                                                  const LineThreshold* __restrict__ row_th)
{
    extern __shared__ __attribute__((aligned(16))) double buf[];   // [2][16][514], then [2][512] ints: row is removed
    int* const gone = reinterpret_cast<int*>(buf + 2 * kSumLines * kSumPitch);
    const int lane = threadIdx.x & 63;
    const int p = (int)threadIdx.x - 64;                     // fetching thread 0..255
    const int line0 = blockIdx.x * kSumLines;
    const int len = M, lines = N;
    const int tiles = (len + kSumTile - 1) / kSumTile;
    constexpr int kPer = VEC ? 4 : 1;                        // columns per load
    constexpr int kLoads = kSumLines * kSumTile / kPer / 256;
    float w[kLoads][kPer];
    uint32_t on[kLoads];
    int gflag[2];
    // (line, position) of load i of this thread; its kPer values run along the columns
    auto place = [&](int i, int& line, int& pos) {
        const int e = p + 256 * i;
        constexpr int kRow = kSumLines / kPer;                   // loads per row of the tile
        line = (e % kRow) * kPer;
        pos = e / kRow;
    };
    auto fetch = [&](int tile) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            int line, pos;
            place(i, line, pos);
            const int r = tile * kSumTile + pos, c = line0 + line;
            const size_t idx = (r < M && c < N) ? (size_t)r * N + c : 0;   // (VEC: N % 4 == 0, a load is in or out as a whole)
            if constexpr (VEC) {
                const float4 v = *reinterpret_cast<const float4*>(W + idx);
                w[i][0] = v.x; w[i][1] = v.y; w[i][2] = v.z; w[i][3] = v.w;
                on[i] = *reinterpret_cast<const uint32_t*>(mask + idx);
            } else {
                w[i][0] = W[idx];
                on[i] = mask[idx];
            }
            if (r >= M || c >= N) on[i] = 0;
        }
        if constexpr (AFTER) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = tile * kSumTile + p + 256 * i;
                gflag[i] = (r < M && rsums[r] <= row_th->value) ? 1 : 0;
            }
        }
    };
    auto park = [&](int tile) {
        double* const b = buf + (tile & 1) * kSumLines * kSumPitch;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            int line, pos;
            place(i, line, pos);
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                b[(line + j) * kSumPitch + pos] = ((on[i] >> (8 * j)) & 255u) ? (double)fabsf(w[i][j]) : 0.0;
        }
        if constexpr (AFTER) {
#pragma unroll
            for (int i = 0; i < 2; ++i) gone[(tile & 1) * kSumTile + p + 256 * i] = gflag[i];
        }
    };
    if (p >= 0) {
        fetch(0);
        park(0);
        if (tiles > 1) fetch(1);
    }
    __syncthreads();
    double acc = 0.0;
    for (int tile = 0; tile < tiles; ++tile) {
        if (p >= 0) {
            if (tile + 1 < tiles) park(tile + 1);
            if (tile + 2 < tiles) fetch(tile + 2);
        } else if (lane < (AFTER ? 2 * kSumLines : kSumLines)) {
            // positions behind the end of the line hold +0, which changes nothing
            const int left = len - tile * kSumTile;
            const int n = (left < kSumTile ? left + kSumBatch - 1 : kSumTile) / kSumBatch;
            const double2* src = reinterpret_cast<const double2*>(buf + ((tile & 1) * kSumLines + (lane & 15)) * kSumPitch);
            const int4* gsrc = reinterpret_cast<const int4*>(gone + (tile & 1) * kSumTile);
            double2 cur[kSumBatch / 2], nxt[kSumBatch / 2];
            int4 gcur[kSumBatch / 4];
#pragma unroll
            for (int i = 0; i < kSumBatch / 2; ++i) cur[i] = src[i];
            for (int k = 0; k < n; ++k) {
                const int kn = k + 1 < n ? k + 1 : k;
#pragma unroll
                for (int i = 0; i < kSumBatch / 2; ++i) nxt[i] = src[kn * (kSumBatch / 2) + i];
                if constexpr (AFTER) {
#pragma unroll
                    for (int i = 0; i < kSumBatch / 4; ++i) gcur[i] = gsrc[k * (kSumBatch / 4) + i];
#pragma unroll
                    for (int i = 0; i < kSumBatch / 4; ++i) {
                        const bool drop = lane >= kSumLines;
                        if (drop && gcur[i].x) cur[2 * i].x = 0.0;
                        if (drop && gcur[i].y) cur[2 * i].y = 0.0;
                        if (drop && gcur[i].z) cur[2 * i + 1].x = 0.0;
                        if (drop && gcur[i].w) cur[2 * i + 1].y = 0.0;
                    }
                }
#pragma unroll
                for (int i = 0; i < kSumBatch / 2; ++i) {
                    acc += cur[i].x;
                    acc += cur[i].y;
                }
#pragma unroll
                for (int i = 0; i < kSumBatch / 2; ++i) cur[i] = nxt[i];
            }
        }
        __syncthreads();
    }
    const int line = line0 + (lane & 15);
    if (p < 0 && line < lines) {
        if (lane < kSumLines) sums[line] = acc;
        else if (AFTER && lane < 2 * kSumLines) sums_after[line] = acc;
    }
}

// The k-th smallest (1-based) of n non-negative doubles, whose bit patterns order like 64-bit unsigned integers, and the
// lines that go with it: those whose value in `judged` is at or below it.  One workgroup: radix select by 11-bit digits
// (LDS histogram, the digit found by a workgroup scan), ended as soon as one sum is left, which with sums of thousands
// of terms is after two or three digits.  out: the threshold; list (may be nullptr): the removed lines in no particular
// order; removed: how many; none (may be nullptr): set to zero, the count of an axis nothing is asked of.
// Bound: latency, of memory and of the barriers.  A thread holds its first kSelKeep sums in registers, requested at once;
// only what is beyond 8192 lines is read again for each digit.  (6000 sums: 26 -> 14.8 us against byte-wide digits walked by
// one thread, 13.1 with the sums held; 256 sums 4.9 -> 5.6; the pruning step of a 6000 x 1500 matrix, where the sums come
// from another XCD's stores, 250 -> 244 with the two launches that set the other axis' count saved.  Adding a wave's equal
// first digits as one: 13.3, nothing in the step.)
constexpr int kSelKeep = 8;
__global__ __launch_bounds__(1024) void select_lines_kernel(const double* __restrict__ sums, int n, unsigned k,
                                                            const double* __restrict__ judged, LineThreshold* __restrict__ out,
                                                            int* __restrict__ list, int* __restrict__ removed, int* __restrict__ none)
{
    __shared__ unsigned hist[2048];
    __shared__ unsigned wtot[16];
    __shared__ unsigned long long found_key;
    __shared__ unsigned found_digit, found_below, found_in, nlist;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    unsigned long long prefix = 0ull;
    unsigned kk = k;
    if (tid == 0) nlist = 0;
    unsigned long long held[kSelKeep];
#pragma unroll
    for (int u = 0; u < kSelKeep; ++u) {
        const int i = tid + 1024 * u;
        held[u] = (unsigned long long)__double_as_longlong(sums[i < n ? i : 0]);
    }
    auto each_key = [&](auto f) {
#pragma unroll
        for (int u = 0; u < kSelKeep; ++u)
            if (tid + 1024 * u < n) f(held[u]);
        for (int i = tid + 1024 * kSelKeep; i < n; i += 1024) f((unsigned long long)__double_as_longlong(sums[i]));
    };
    // digits of bits 63..53, 52..42, 41..31, 30..20, 19..9, 8..0
    for (int top = 64; top > 0 && k > 0;) {
        const int shift = top >= 11 ? top - 11 : 0;
        hist[tid] = 0;
        hist[tid + 1024] = 0;
        __syncthreads();
        each_key([&](unsigned long long key) {
            if (top == 64 || (key >> top) == (prefix >> top)) atomicAdd(&hist[(unsigned)(key >> shift) & ((1u << (top - shift)) - 1u)], 1u);
        });
        __syncthreads();
        // the bin that holds rank kk: inclusive scan over pairs of bins
        const unsigned a = hist[2 * tid], b = hist[2 * tid + 1];
        unsigned incl = a + b;
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        if (lane == 63) wtot[wv] = incl;
        __syncthreads();
        unsigned below = incl - (a + b);
        for (int i = 0; i < wv; ++i) below += wtot[i];
        if (kk > below && kk <= below + a) { found_digit = 2 * tid; found_below = below; found_in = a; }
        else if (kk > below + a && kk <= below + a + b) { found_digit = 2 * tid + 1; found_below = below + a; found_in = b; }
        __syncthreads();
        prefix |= (unsigned long long)found_digit << shift;
        kk -= found_below;
        if (found_in == 1 && shift > 0) {   // one candidate left: it is the answer
            each_key([&](unsigned long long key) {
                if ((key >> shift) == (prefix >> shift)) found_key = key;
            });
            __syncthreads();
            prefix = found_key;
            break;
        }
        top = shift;
        __syncthreads();
    }
    __syncthreads();
    const double value = __longlong_as_double((long long)prefix);
    if (k > 0) {
        auto judge = [&](int i, double sum) {
            if (sum <= value) {
                const unsigned at = atomicAdd(&nlist, 1u);
                if (list) list[at] = i;
            }
        };
        const bool same = judged == sums;
        double other[kSelKeep];
        if (!same) {
#pragma unroll
            for (int u = 0; u < kSelKeep; ++u) {
                const int i = tid + 1024 * u;
                other[u] = judged[i < n ? i : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < kSelKeep; ++u)
            if (tid + 1024 * u < n) judge(tid + 1024 * u, same ? __longlong_as_double((long long)held[u]) : other[u]);
        for (int i = tid + 1024 * kSelKeep; i < n; i += 1024) judge(i, judged[i]);
    }
    __syncthreads();
    if (tid == 0) {
        out->value = value;
        out->any = k > 0 ? 1u : 0u;
        out->count = nlist;
        *removed = (int)nlist;
        if (none) *none = 0;
    }
}

// Mask and weights of the removed lines to zero: a wave per row clears either the whole row or the listed columns of it.
// th[0]: rows, th[1]: columns; an axis with rank 0 removes nothing and its sums are not looked at.
__global__ __launch_bounds__(256) void clear_lines_kernel(float* __restrict__ W, uint8_t* __restrict__ mask, int M, int N,
                                                          const double* __restrict__ rsums, const LineThreshold* __restrict__ th,
                                                          const int* __restrict__ col_list, int by_rows, int by_cols)
{
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= M) return;
    float* const w = W + (size_t)r * N;
    uint8_t* const m = mask + (size_t)r * N;
    if (by_rows && rsums[r] <= th[0].value) {
        for (int c = lane; c < N; c += 64) { m[c] = 0; w[c] = 0.f; }
    } else if (by_cols) {
        const int n = (int)th[1].count;
        for (int i = lane; i < n; i += 64) { m[col_list[i]] = 0; w[col_list[i]] = 0.f; }
    }
}

// scratch (prune_rows_cols_scratch_bytes): row sums [M] f64 | column sums [N] f64 | column sums without the removed rows
// [N] f64 | two thresholds.  The list of removed columns takes the place of the column sums once those have been judged.
size_t prune_rows_cols_scratch_bytes(int M, int N)
{
    return ((size_t)M + 2 * (size_t)N) * sizeof(double) + 2 * sizeof(LineThreshold);
}

__global__ void clear_removed_kernel(int* removed)
{
    if (threadIdx.x < 2) removed[threadIdx.x] = 0;
}

static bool line_loads_fit(const float* W, const uint8_t* mask, int N)
{
    return (N & 3) == 0 && ((uintptr_t)W & 15) == 0 && ((uintptr_t)mask & 3) == 0;
}

static hipError_t launch_row_sums(const float* W, const uint8_t* mask, int M, int N, double* sums, hipStream_t s)
{
    const dim3 grid((M + kRowWaves - 1) / kRowWaves), block(64 * kRowWaves);
    if (line_loads_fit(W, mask, N)) hipLaunchKernelGGL(row_abs_sum_kernel<true>, grid, block, 0, s, W, mask, M, N, sums);
    else hipLaunchKernelGGL(row_abs_sum_kernel<false>, grid, block, 0, s, W, mask, M, N, sums);
    return hipGetLastError();
}

template <bool AFTER>
static hipError_t launch_col_sums(const float* W, const uint8_t* mask, int M, int N, double* sums, double* after,
                                  const double* rsums, const LineThreshold* th, hipStream_t s)
{
    const void* kern = line_loads_fit(W, mask, N) ? (const void*)col_abs_sum_kernel<true, AFTER> : (const void*)col_abs_sum_kernel<false, AFTER>;
    const hipError_t e = allow_dynamic_lds(kern, kSumLds);
    if (e != hipSuccess) return e;
    void* args[] = {&W, &mask, &M, &N, &sums, &after, &rsums, &th};
    return hipLaunchKernel(kern, dim3((N + kSumLines - 1) / kSumLines), dim3(kSumThreads), args, kSumLds, s);
}

// removed: device-visible int[2], receives the number of removed rows and columns
hipError_t launch_prune_rows_cols(float* W, uint8_t* mask, int M, int N, unsigned k_rows, unsigned k_cols, void* scratch,
                                  int* removed, hipStream_t s)
{
    double* rsums = (double*)scratch;
    double* csums = rsums + M;
    double* csums_after = csums + N;
    LineThreshold* th = (LineThreshold*)(csums_after + N);
    int* const list = (int*)csums;
    if (k_rows == 0 && k_cols == 0) {
        hipLaunchKernelGGL(clear_removed_kernel, dim3(1), dim3(64), 0, s, removed);
        return hipGetLastError();
    }
    hipError_t e = hipSuccess;
    // Both thresholds come from the matrix as it came in; rows are removed first and columns judged on what that leaves.
    if (k_rows > 0) {
        e = launch_row_sums(W, mask, M, N, rsums, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(select_lines_kernel, dim3(1), dim3(1024), 0, s, rsums, M, k_rows, rsums, th, (int*)nullptr, removed,
                           k_cols > 0 ? (int*)nullptr : removed + 1);
    }
    if (k_cols > 0) {
        // without removed rows the sums as passed in are also the ones to judge, and one pass reads both
        double* const judged = k_rows > 0 ? csums_after : csums;
        e = k_rows > 0 ? launch_col_sums<true>(W, mask, M, N, csums, csums_after, rsums, th, s)
                       : launch_col_sums<false>(W, mask, M, N, csums, nullptr, nullptr, nullptr, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(select_lines_kernel, dim3(1), dim3(1024), 0, s, csums, N, k_cols, judged, th + 1,
                           k_rows > 0 ? list : (int*)csums_after, removed + 1, k_rows > 0 ? (int*)nullptr : removed);
    }
    hipLaunchKernelGGL(clear_lines_kernel, dim3((M + 3) / 4), dim3(256), 0, s, W, mask, M, N, rsums, th,
                       k_rows > 0 ? list : (int*)csums_after, k_rows > 0 ? 1 : 0, k_cols > 0 ? 1 : 0);
    return hipGetLastError();
}

// ---- the same iteration with no allocation: scratch in a file-scope device array ----------------------------------
// Every device that loads the library holds its own copy of the array, at its own address, until the process ends.
// In host code the array's name is only a handle for hipGetSymbolAddress; the address that call returns for the
// current device is what the kernels get.
constexpr int kStaticMaxLines = 16384;   // largest M and largest N accepted
constexpr size_t kStaticScratchBytes = (size_t)3 * kStaticMaxLines * sizeof(double) + 256;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

int prune_rows_cols_static_max_lines() { return kStaticMaxLines; }

// address of this device's copy of the array, looked up once per device with that device current
static hipError_t static_scratch_for_current_device(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

// the caller has checked M, N <= kStaticMaxLines
hipError_t launch_prune_rows_cols_static(float* W, uint8_t* mask, int M, int N, unsigned k_rows, unsigned k_cols,
                                         int* removed_dev, hipStream_t s)
{
    const size_t need = (prune_rows_cols_scratch_bytes(M, N) + 15) & ~(size_t)15;
    if (need + 2 * sizeof(int) > kStaticScratchBytes) return hipErrorInvalidValue;
    void* ptr = nullptr;
    const hipError_t e = static_scratch_for_current_device(&ptr);
    if (e != hipSuccess) return e;
    // every sum, list entry and threshold that is read has been written by this call, so what the previous one left in
    // the array does not matter
    return launch_prune_rows_cols(W, mask, M, N, k_rows, k_cols, ptr, removed_dev ? removed_dev : (int*)((char*)ptr + need), s);
}

}  // namespace l355
