// Dimension compaction after row/column pruning (paper Section 4, row/column growth & pruning: the pruning shrinks the
// dimensions of the weight matrices; Section 5.1 step (b): each control-gate matrix goes from 1500/400 to 1197/317).
// Rows and columns that have no active connection left leave the matrix; what remains is written out as a smaller
// dense matrix together with the lists of the rows and columns that were kept.
//
// Three kernels, nothing returns to the host between them: one pass over the mask sets a flag per row and per column
// that still has a connection; one workgroup turns the flags into ascending index lists (ballot + popcount per wave,
// wave totals through LDS); a gather writes the compacted matrix and mask.
#include "common.h"

namespace l355 {

// A workgroup covers `rows_per` rows, 1024 columns at a time: its four waves take the rows in turn, a lane sixteen
// columns (VEC = 16: one 16-byte load, 4: four words, 1: bytes, whatever N and the address allow) and keeps their flags
// until the rows are through; the waves' flags meet in LDS, so that a column flag is stored once per workgroup.  Every
// writer of a flag writes the same value.  Bound: HBM, one byte per entry (6000 x 1500: 24 -> 9 us against one byte per load
// and a column flag per 64 rows).
template <int VEC>
__global__ __launch_bounds__(256) void active_flags_kernel(const uint8_t* __restrict__ mask, int M, int N, int rows_per,
                                                           unsigned* __restrict__ rowflag, unsigned* __restrict__ colflag)
{
    __shared__ uint32_t cols[256];   // a byte per column of the chunk
    const int tid = threadIdx.x, lane = tid & 63;
    const int rb = blockIdx.x * rows_per, re = rb + rows_per < M ? rb + rows_per : M;
    for (int cb = 0; cb < N; cb += 1024) {
        const int c0 = cb + lane * 16;
        cols[tid] = 0;
        __syncthreads();
        uint32_t seen[4] = {};
        for (int r = rb + (tid >> 6); r < re; r += 4) {
            const uint8_t* const p = mask + (size_t)r * N + c0;
            uint32_t v[4] = {};
            if (VEC == 16) {
                if (c0 < N) {
                    const uint4 q = *reinterpret_cast<const uint4*>(p);
                    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
                }
            } else if (VEC == 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (c0 + 4 * k < N) v[k] = *reinterpret_cast<const uint32_t*>(p + 4 * k);
            } else {
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (c0 + k < N) v[k >> 2] |= (uint32_t)p[k] << (8 * (k & 3));
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) seen[k] |= v[k];
            const unsigned long long any = __ballot((v[0] | v[1] | v[2] | v[3]) != 0u);
            if (any != 0ull && lane == 0) rowflag[r] = 1u;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (seen[k]) atomicOr(&cols[lane * 4 + k], seen[k]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = tid + 256 * k;
            if (cb + c < N && ((cols[c >> 2] >> (8 * (c & 3))) & 255u)) colflag[cb + c] = 1u;
        }
        __syncthreads();
    }
}

// out[0 .. total) = the indices i in [0, n) with keep(i), ascending; out[total .. n) = -1; *count = total
template <class Keep>
__device__ void ordered_indices(int n, Keep keep, int* __restrict__ out, int* __restrict__ count, int* wave_tot, int* base)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x == 0) *base = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += 1024) {
        const int i = i0 + (int)threadIdx.x;
        const bool on = i < n && keep(i);
        const unsigned long long b = __ballot(on);
        const int before = __popcll(b & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[wv] = __popcll(b);
        __syncthreads();
        int off = *base;
        for (int k = 0; k < wv; ++k) off += wave_tot[k];
        if (on) out[off + before] = i;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int k = 0; k < 16; ++k) t += wave_tot[k];
            *base += t;
        }
        __syncthreads();
    }
    const int total = *base;
    for (int i = total + (int)threadIdx.x; i < n; i += 1024) out[i] = -1;
    if (threadIdx.x == 0) *count = total;
    __syncthreads();
}

// one workgroup of 1024 threads; a unit is kept when any of its `gates` rows has a flag
__global__ __launch_bounds__(1024) void compact_index_kernel(const unsigned* __restrict__ rowflag, const unsigned* __restrict__ colflag,
                                                             int gates, int R, int N, int* __restrict__ row_index,
                                                             int* __restrict__ col_index, int* __restrict__ counts,
                                                             int* __restrict__ counts_out)
{
    __shared__ int wave_tot[16];
    __shared__ int base;
    ordered_indices(R, [&](int u) {
        unsigned any = 0u;
        for (int q = 0; q < gates; ++q) any |= rowflag[(size_t)q * R + u];
        return any != 0u;
    }, row_index, counts, wave_tot, &base);
    ordered_indices(N, [&](int k) { return colflag[k] != 0u; }, col_index, counts + 1, wave_tot, &base);
    if (threadIdx.x < 2) counts_out[threadIdx.x] = counts[threadIdx.x];
}

// Wc[q*Rc + i][j] = the value at (q*R + row_index[i], col_index[j]) where its mask byte is set, +0 otherwise.  A wave
// takes a row of the result, four columns per lane in flight; bound: HBM (6000 x 1500: 24 -> 17 us against one
// 64-bit division per entry).
__global__ __launch_bounds__(256) void compact_gather_kernel(const float* __restrict__ W, const uint8_t* __restrict__ mask, int gates,
                                                             int R, int N, const int* __restrict__ row_index,
                                                             const int* __restrict__ col_index, const int* __restrict__ counts,
                                                             float* __restrict__ Wc, uint8_t* __restrict__ mask_c)
{
    const int Rc = counts[0], Nc = counts[1];
    const int lane = threadIdx.x & 63, stride = gridDim.x * 4;
    for (int row = blockIdx.x * 4 + (threadIdx.x >> 6); row < gates * Rc; row += stride) {
        const int q = row / Rc;
        const size_t src = ((size_t)q * R + row_index[row - q * Rc]) * N, dst = (size_t)row * Nc;
        for (int j0 = lane; j0 < Nc; j0 += 256) {
            float w[4];
            uint8_t on[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + 64 * u;
                const size_t at = src + col_index[j < Nc ? j : j0];
                w[u] = W[at];
                on[u] = mask[at];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + 64 * u;
                if (j >= Nc) continue;
                Wc[dst + j] = on[u] ? w[u] : 0.f;
                if (mask_c) mask_c[dst + j] = on[u] ? 1 : 0;
            }
        }
    }
}

// scratch: flags [gates*R + N] u32 (rounded up to an even count), then counts 2 x int
size_t compact_scratch_bytes(int gates, int R, int N)
{
    const size_t flags = ((size_t)gates * R + N + 1) & ~(size_t)1;
    return flags * sizeof(unsigned) + 2 * sizeof(int);
}

hipError_t launch_compact_rows_cols(const float* W, const uint8_t* mask, int gates, int R, int N, int* row_index,
                                    int* col_index, float* Wc, uint8_t* mask_c, void* scratch, int* counts_out, hipStream_t s)
{
    const int M = gates * R;
    const size_t flags = ((size_t)M + N + 1) & ~(size_t)1;
    unsigned* rowflag = (unsigned*)scratch;
    unsigned* colflag = rowflag + M;
    int* counts = (int*)(rowflag + flags);
    hipError_t e = launch_fill_u64((unsigned long long*)scratch, flags / 2 + 1, 0ull, s);   // flags and both counts
    if (e != hipSuccess) return e;
    // at least four rows (one per wave) and about a workgroup per compute unit
    const int rows_per = std::max(4, (M + device_num_cus() - 1) / device_num_cus());
    const dim3 fgrid((M + rows_per - 1) / rows_per);
    const uintptr_t low = (uintptr_t)N | (uintptr_t)mask;
    if ((low & 15) == 0) hipLaunchKernelGGL(active_flags_kernel<16>, fgrid, dim3(256), 0, s, mask, M, N, rows_per, rowflag, colflag);
    else if ((low & 3) == 0) hipLaunchKernelGGL(active_flags_kernel<4>, fgrid, dim3(256), 0, s, mask, M, N, rows_per, rowflag, colflag);
    else hipLaunchKernelGGL(active_flags_kernel<1>, fgrid, dim3(256), 0, s, mask, M, N, rows_per, rowflag, colflag);
    hipLaunchKernelGGL(compact_index_kernel, dim3(1), dim3(1024), 0, s, rowflag, colflag, gates, R, N, row_index, col_index, counts, counts_out);
    const int g = std::min((M + 3) / 4, 4096);
    hipLaunchKernelGGL(compact_gather_kernel, dim3(g), dim3(256), 0, s, W, mask, gates, R, N, row_index, col_index,
                       counts, Wc, mask_c);
    return hipGetLastError();
}

}  // namespace l355
