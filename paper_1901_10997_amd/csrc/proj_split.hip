// fp32 input projection on the fp16 matrix instruction:  P[m][n] = bias[n] + sum_k X[m][k] * W[n][k]
//
// Every fp32 value of a row is scaled by a power of two that brings the row's largest magnitude into [2^14, 2^15) and kept
// as two fp16 numbers, hi = fp16(v) and lo = fp16(v - hi): 22 to 24 significant bits.  A product is then
// hi.hi + hi.lo + lo.hi (lo.lo is 2^-22 of it at most), three instructions whose products are exact and whose sums are fp32,
// 16 k per 32 clocks each where the fp32 instruction takes 2 k in 64: a tenth of the matrix time.  An element of P is also the
// sum of 3 K / 16 rounded terms instead of K / 2, which more than makes up for the bits the planes drop: error against 64 bits,
// fp32 instruction / here, relative to the product's norm: K 64 1.35e-7 / 1.17e-7, 200 2.5e-7 / 1.8e-7, 640 4.4e-7 / 2.9e-7,
// 1600 7.2e-7 / 4.6e-7 (normal X, uniform W; K 32 9.26e-8 / 9.34e-8, which is why K starts at 64).
//
// Layout: the planes of 32 k lie side by side, 64 bytes hi and 64 bytes lo, so that a slab of 32 k of a row is one 128-byte
// line; slabs go straight into an LDS ring (16-byte chunk c of row r at position c ^ ((r >> 1) & 7): conflict-free reads), and
// a fragment read serves two or one of the three products: two slab bytes per product fewer than a bf16 product needs.
// Bound: the device's power limit under random operands (the issue loop of this instruction reaches 1.7 PFLOP/s there) and
// what a tile's ends leave idle.  4800 x 3200 x 1600 in two directions: fp32 instruction 901 us (109 TFLOP/s), here 311
// (316, 950 counted as fp16 products); x 640: 389 -> 129; 700 x 6000 x 1500: 163 -> 59.
#include <cmath>
#include "common.h"
#include "device_math.h"

namespace l355 {

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kXcds = 8;
constexpr int kGroupM = 4;

// ---- rows into two fp16 planes
// out: per row KB blocks of 128 bytes, 32 hi values then 32 lo values of k = 32 kb ..; unscale: 2^-e of the row's scale 2^e, or a mark
// where the row does not fit (device_math.h).
constexpr int kSplitRowsPerBlock = 4;

__device__ __forceinline__ uint32_t pack_f16x2(_Float16 a, _Float16 b)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

template <int VEC>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ X, int ldx, int M, int K, int KB,
                                                         uint16_t* __restrict__ out, float* __restrict__ unscale)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.x * kSplitRowsPerBlock + wave;
    if (m >= M) return;
    {
        const float* row = X + (size_t)m * ldx;
        unsigned big = 0;   // largest |v| as bits: NaN and infinity come out on top
        for (int k = VEC * lane; k < K; k += VEC * 64) {
            if (VEC == 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(row + k);
                const unsigned a = max(v.x & 0x7fffffffu, v.y & 0x7fffffffu), b = max(v.z & 0x7fffffffu, v.w & 0x7fffffffu);
                big = max(big, max(a, b));
            } else {
                big = max(big, __float_as_uint(row[k]) & 0x7fffffffu);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) big = max(big, (unsigned)__shfl_xor((int)big, o, 64));
        const SplitScale sc = split_scale(big);
        int small = 0, nonzero = 0;
        uint16_t* dst = out + (size_t)m * KB * 64;
        for (int k = VEC * lane; k < 32 * KB; k += VEC * 64) {
            float v[VEC];
            if (VEC == 4) {
                float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k < K) t = *reinterpret_cast<const float4*>(row + k);
                v[0] = t.x; v[1 % VEC] = t.y; v[2 % VEC] = t.z; v[3 % VEC] = t.w;
            } else {
                v[0] = k < K ? row[k] : 0.f;
            }
            _Float16 hi[VEC], lo[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const float s = v[i] * sc.scale;
                nonzero += v[i] != 0.f;
                small += v[i] != 0.f && fabsf(s) < kSplitSmall;
                hi[i] = (_Float16)s;
                lo[i] = (_Float16)(s - (float)hi[i]);
            }
            uint16_t* p = dst + (k >> 5) * 64 + (k & 31);
            if (VEC == 4) {
                *reinterpret_cast<uint2*>(p) = make_uint2(pack_f16x2(hi[0], hi[1 % VEC]), pack_f16x2(hi[2 % VEC], hi[3 % VEC]));
                *reinterpret_cast<uint2*>(p + 32) = make_uint2(pack_f16x2(lo[0], lo[1 % VEC]), pack_f16x2(lo[2 % VEC], lo[3 % VEC]));
            } else {
                p[0] = __builtin_bit_cast(uint16_t, hi[0]);
                p[32] = __builtin_bit_cast(uint16_t, lo[0]);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) { small += __shfl_xor(small, o, 64); nonzero += __shfl_xor(nonzero, o, 64); }
        if (lane == 0) unscale[m] = split_unscale(sc, big, small, nonzero);
    }
}

size_t split_row_halves(int K) { return (size_t)((K + 31) / 32) * 64; }

hipError_t launch_split_rows(const float* X, int ldx, int M, int K, uint16_t* out, float* unscale, hipStream_t s)
{
    const int KB = (K + 31) / 32;
    const dim3 grid((M + kSplitRowsPerBlock - 1) / kSplitRowsPerBlock), block(256);
    if (K % 4 == 0 && ldx % 4 == 0 && ((uintptr_t)X & 15) == 0)
        hipLaunchKernelGGL(split_rows_kernel<4>, grid, block, 0, s, X, ldx, M, K, KB, out, unscale);
    else
        hipLaunchKernelGGL(split_rows_kernel<1>, grid, block, 0, s, X, ldx, M, K, KB, out, unscale);
    return hipGetLastError();
}

// ---- the product
__device__ __forceinline__ u32x4 lds_read_b128(unsigned addr)
{
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory");
    return v;
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "six-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// ---- tiles with rows that have no fp16 form
template <int BM>
__device__ __forceinline__ bool tile_has_marked_rows(const ProjSplitArgs& a, int m0, int lane)
{
    bool marked = false;
#pragma unroll
    for (int i = 0; i < BM / 64; ++i) marked |= !(a.x_unscale[min(m0 + 64 * i + lane, a.M - 1)] < __uint_as_float(kNonFinite));
    return __ballot(marked) != 0;
}

// One wave's TM x TN tiles of 32 x 32 on the fp32 matrix instruction, operands straight from memory, a row of tiles at a
// time (few registers: the split product sets the kernel's count).  A row with a non-finite value is then summed over the
// kept entries where W is held row-compressed: the mask selects, and what it leaves out must not meet an infinity as a zero.
template <int TM, int TN>
__device__ __forceinline__ void f32_tiles(const ProjSplitArgs& a, int dir, int m0, int n0, int lane)
{
    const ProjSplitDir& d = a.d[dir];
    const int M = a.M, N = a.N, K = a.K, fr = lane & 31, fk = lane >> 5;
    constexpr int KU = 4;   // k8 steps requested together
    const float* wrow[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) wrow[j] = d.Wd + (size_t)min(n0 + 32 * j + fr, N - 1) * K;
#pragma unroll 1
    for (int i = 0; i < TM; ++i) {
        const float* xrow = a.X + (size_t)min(m0 + 32 * i + fr, M - 1) * a.ldx;
        f32x16 acc[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += 8 * KU) {   // K % 4 == 0: a lane's four values are all there or none is
            float4 fa[KU], fb[KU][TN];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int k = k0 + 8 * u + 4 * fk;
                fa[u] = k < K ? *reinterpret_cast<const float4*>(xrow + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int j = 0; j < TN; ++j) fb[u][j] = k < K ? *reinterpret_cast<const float4*>(wrow[j] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < KU; ++u)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u].x, fb[u][j].x, acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u].y, fb[u][j].y, acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u].z, fb[u][j].z, acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u].w, fb[u][j].w, acc[j], 0, 0, 0);
                }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + 32 * j + fr;
            if (n >= N) continue;
            const float b = d.bias[n];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + 32 * i + 4 * fk + 8 * (v >> 2) + (v & 3);
                if (m < M) d.P[(size_t)m * N + n] = acc[j][v] + b;
            }
        }
    }
    if (d.row_ptr == nullptr) return;
    for (int m = m0; m < min(m0 + 32 * TM, M); ++m) {
        if (__float_as_uint(a.x_unscale[m]) != kNonFinite) continue;
        const float* x = a.X + (size_t)m * a.ldx;
        for (int n = n0 + lane; n < min(n0 + 32 * TN, N); n += 64) {
            float sum = 0.f;
            for (int e = d.row_ptr[n]; e < d.row_ptr[n + 1]; ++e) sum = fmaf(d.val[e], x[d.col[e]], sum);
            d.P[(size_t)m * N + n] = sum + d.bias[n];
        }
    }
}

// TM x TN: 32 x 32 tiles of a wave; WM x WN waves; NST slabs in the LDS ring; STAGED: sums in two stages.
// STAGED (masked weights): the accumulators are added up and cleared every kStage slabs.  An fp32 sum that meets a mask's zeros
// rounds once per kept term; an instruction over 16 k rounds whether they are zeros or not, 3 K / 16 times in all.  In two
// stages the terms are a small part of the sum when they are rounded: K 1600, 15 % kept, error against 64 bits relative to the
// product's norm: fp32 instruction 2.8e-7, one stage 3.8e-7, two 1.5e-7 (310 us against 271, 4800 x 3200 in two directions; dense
// weights 7.2e-7, 4.6e-7 and 1.7e-7).
constexpr int kStage = 4;
template <int TM, int TN, int WM, int WN, int NST, bool STAGED>
__global__ __launch_bounds__(64 * WM * WN, 2) void proj_split_kernel(ProjSplitArgs a)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, NW = WM * WN;
    constexpr int ROWB = 128;                             // one block of 32 k: 64 bytes hi, 64 bytes lo
    constexpr int STAGE = (BM + BN) * ROWB;
    constexpr int LI = (BM + BN) / 8 / NW;                // direct-load instructions (8 rows each) per wave and slab
    static_assert((BM + BN) % (8 * NW) == 0, "rows divide over the waves");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const int wm = wave / WN, wn = wave % WN;
    const int fr = lane & 31, fk = lane >> 5;
    const int M = a.M, N = a.N, KB = (a.K + 31) >> 5;
    const int rowh = KB * 64;                             // fp16 elements of a row, both planes

    unsigned offa[TM], offb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int rr = (wm * TM + i) * 32 + fr;
        offa[i] = (unsigned)(rr * ROWB + ((fk ^ ((rr >> 1) & 7)) * 16));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int rr = (wn * TN + j) * 32 + fr;
        offb[j] = (unsigned)((BM + rr) * ROWB + ((fk ^ ((rr >> 1) & 7)) * 16));
    }
    for (int pid = blockIdx.x; pid < a.npid; pid += gridDim.x) {
        // consecutive tiles share an XCD; four tile rows at a time walk over all columns of both directions
        const int nblk = a.gm * a.gn * a.ndir;
        const int per_xcd = (nblk + kXcds - 1) / kXcds;
        const int logical = (pid % kXcds) * per_xcd + pid / kXcds;
        if (logical >= nblk) continue;
        const int gnt = a.gn * a.ndir, span = kGroupM * gnt;
        const int group = logical / span, in = logical % span, first = group * kGroupM;
        const int gsz = (a.gm - first) < kGroupM ? (a.gm - first) : kGroupM;
        const int tile_m = first + in % gsz, tn_all = in / gsz;
        const int dir = tn_all >= a.gn ? 1 : 0;
        const int m0 = tile_m * BM, n0 = (tn_all - dir * a.gn) * BN;
        if (pid != (int)blockIdx.x) __builtin_amdgcn_s_barrier();

        f32x16 acc[TM][TN], total[STAGED ? TM : 1][STAGED ? TN : 1];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    acc[i][j][v] = 0.f;
                    if (STAGED) total[STAGED ? i : 0][STAGED ? j : 0][v] = 0.f;
                }

        // direct loads: instruction q of a slab covers LDS rows 8 q .. 8 q + 7 of the combined [X rows | W rows]
        // (eight rows of one operand: scalar base pointer, one 32-bit element offset per instruction and lane)
        const uint16_t* const xbase = a.Xs + (size_t)m0 * rowh;
        const uint16_t* const wbase = a.d[dir].W + (size_t)n0 * rowh;
        unsigned soff[LI];
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const int row0 = (wave_s * LI + i) * 8;
            const int row = row0 + (lane >> 3);
            const int kc = (lane & 7) ^ ((row >> 1) & 7);
            const int r = row0 < BM ? min(row, M - 1 - m0) : min(row - BM, N - 1 - n0);   // rows past the matrix re-read its last
            soff[i] = (unsigned)(r * rowh + 8 * kc);
        }
        auto issue_slab = [&](int kt) {
            unsigned char* st = smem + (size_t)(kt % NST) * STAGE + (size_t)wave_s * LI * 1024;
#pragma unroll
            for (int i = 0; i < LI; ++i) {
                const uint16_t* from = ((wave_s * LI + i) * 8 < BM ? xbase : wbase) + (size_t)kt * 64;
                __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(from + soff[i]),
                                                 (void __attribute__((address_space(3)))*)(st + (size_t)i * 1024), 16, 0, 0);
            }
        };
        // k16 step ks of plane pl (0 hi, 1 lo): chunk 4 pl + 2 ks + fk
        auto read_a = [&](u32x4 (&f)[TM], unsigned st, int ks, int pl) {
#pragma unroll
            for (int i = 0; i < TM; ++i) f[i] = lds_read_b128(st + (offa[i] ^ (unsigned)((ks << 5) | (pl << 6))));
        };
        auto read_b = [&](u32x4 (&f)[TN], unsigned st, int ks, int pl) {
#pragma unroll
            for (int j = 0; j < TN; ++j) f[j] = lds_read_b128(st + (offb[j] ^ (unsigned)((ks << 5) | (pl << 6))));
        };
        auto mma = [&](u32x4 (&fa)[TM], u32x4 (&fb)[TN]) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[i]),
                                                                       __builtin_bit_cast(f16x8, fb[j]), acc[i][j], 0, 0, 0);
        };
        auto arrived_a = [&](u32x4 (&f)[TM]) {
#pragma unroll
            for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(f[i]) : : "memory");
        };
        auto arrived_b = [&](u32x4 (&f)[TN]) {
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(f[j]) : : "memory");
        };
        // slab `target` has landed once only the loads of the (at most NST - 2) younger slabs can still be outstanding
        auto wait_slab = [&](int target) {
            const int y = min(KB - 1 - target, NST - 2);
            if (NST >= 4 && y == 2) wait_vmcnt<NST >= 4 ? 2 * LI : 0>();
            else if (NST >= 3 && y == 1) wait_vmcnt<NST >= 3 ? LI : 0>();
            else wait_vmcnt<0>();
        };
#pragma unroll
        for (int q = 0; q < NST - 1; ++q)
            if (q < KB) issue_slab(q);
        if (tile_has_marked_rows<BM>(a, m0, lane)) {   // the same answer in every wave
            wait_vmcnt<0>();
            f32_tiles<TM, TN>(a, dir, m0 + wm * TM * 32, n0 + wn * TN * 32, lane);
            continue;
        }
        wait_slab(0);
        __builtin_amdgcn_s_barrier();
        if (NST - 1 < KB) issue_slab(NST - 1);
        u32x4 ah[TM], al[TM], bh[TN], bl[TN];
        read_a(ah, lds0, 0, 0);
        read_b(bl, lds0, 0, 1);
        for (int kt = 0; kt < KB; ++kt) {
            const unsigned st = lds0 + (unsigned)((kt % NST) * STAGE);
            const unsigned stn = lds0 + (unsigned)(((kt + 1) % NST) * STAGE);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                // the fragments of each group of products were requested one group ahead or more; the registers a group
                // has read for the last time take the next request
                read_b(bh, st, ks, 0);
                read_a(al, st, ks, 1);
                asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(TM + TN) : "memory");
                arrived_a(ah);
                arrived_b(bl);
                mma(ah, bl);
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(TM) : "memory");
                arrived_b(bh);
                mma(ah, bh);
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                arrived_a(al);
                if (ks == 0) {
                    read_a(ah, st, 1, 0);
                    read_b(bl, st, 1, 1);
                } else if (kt + 1 < KB) {
                    // this wave is done with slab kt; after the barrier its buffer may be refilled and slab kt+1 read
                    wait_slab(kt + 1);
                    __builtin_amdgcn_s_barrier();
                    if (kt + NST < KB) issue_slab(kt + NST);
                    read_a(ah, stn, 0, 0);
                    read_b(bl, stn, 0, 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                mma(al, bh);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (STAGED && (kt % kStage == kStage - 1 || kt == KB - 1)) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            total[STAGED ? i : 0][STAGED ? j : 0][v] += acc[i][j][v];
                            acc[i][j][v] = kt == KB - 1 ? total[STAGED ? i : 0][STAGED ? j : 0][v] : 0.f;
                        }
            }
        }
        // ---- P = acc * 2^-(ex + ew) + bias; accumulator register v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
        const float* bias = a.d[dir].bias;
        float* P = a.d[dir].P;
        float bn[TN], wu[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + (wn * TN + j) * 32 + fr, nc = n < N ? n : N - 1;
            bn[j] = bias[nc];
            wu[j] = a.d[dir].w_unscale[nc];
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = m0 + (wm * TM + i) * 32 + 4 * fk;
            float xu[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = mb + 8 * (v >> 2) + (v & 3);
                xu[v] = a.x_unscale[m < M ? m : M - 1];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = fmaf(acc[i][j][v], xu[v] * wu[j], bn[j]);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + (wn * TN + j) * 32 + fr;
            if (n >= N) continue;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int mb = m0 + (wm * TM + i) * 32 + 4 * fk;
                if (mb - 4 * fk + 32 <= M) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) P[(size_t)(mb + 8 * (v >> 2) + (v & 3)) * N + n] = acc[i][j][v];
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = mb + 8 * (v >> 2) + (v & 3);
                        if (m < M) P[(size_t)m * N + n] = acc[i][j][v];
                    }
                }
            }
        }
    }
}

template <int TM, int TN, int WM, int WN, int NST, bool STAGED>
static hipError_t launch_tiles(ProjSplitArgs a, int per_cu, hipStream_t s)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    a.gm = (a.M + BM - 1) / BM;
    a.gn = (a.N + BN - 1) / BN;
    a.npid = ((a.gm * a.gn * a.ndir + kXcds - 1) / kXcds) * kXcds;
    const int lds = NST * (BM + BN) * 128;
    const hipError_t e = hipFuncSetAttribute((const void*)proj_split_kernel<TM, TN, WM, WN, NST, STAGED>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    const int slots = std::max(kXcds, device_num_cus() * per_cu / kXcds * kXcds);
    hipLaunchKernelGGL((proj_split_kernel<TM, TN, WM, WN, NST, STAGED>), dim3(std::min(a.npid, slots)), dim3(64 * WM * WN), lds, s, a);
    return hipGetLastError();
}

// Tile shapes with what a slab of 32 k costs, in microseconds: alone on a compute unit, and in a full grid; and the end of a
// tile.  (Fits to 19 products of 77 to 19200 rows; the choice they make is within 4 % of the best shape in 17 and 12 % in two.)
// Large tiles move fewer bytes per product: 4800 x 3200 x 1600, both directions, 256 x 256 311 us, 128 x 256 344, 128 x 128 345,
// 64 x 128 401, 64 x 64 442; small ones leave fewer compute units without work: 128 x 4096 x 1024 64 x 64 11.7 us, 128 x 128 24.8.
struct SplitShape {
    int bm, bn, per_cu;
    double full, alone, end;
};
static const SplitShape kSplitShapes[] = {{256, 256, 1, 3.05, 2.0, 5.5}, {128, 256, 1, 1.73, 1.14, 3.6}, {128, 128, 2, 0.93, 0.76, 1.5},
                                          {64, 128, 2, 0.548, 0.55, 1.0}, {64, 64, 2, 0.30, 0.35, 0.8}};
static const double kLaunchUs = 2.5;

// masked: the sums in two stages need twice the accumulators, which the largest tile has no registers for
static int choose_shape(int M, int N, int K, int ndir, bool masked, double* us)
{
    const double cus = device_num_cus();
    const int KB = (K + 31) / 32;
    int best = 1;
    *us = 1e30;
    for (int i = masked ? 1 : 0; i < (int)(sizeof kSplitShapes / sizeof kSplitShapes[0]); ++i) {
        const SplitShape& h = kSplitShapes[i];
        const double tiles = (double)((M + h.bm - 1) / h.bm) * ((N + h.bn - 1) / h.bn) * ndir, r = tiles / cus;
        // two workgroups of a compute unit share it: its second tile is half free
        const double rounds = r <= 1 ? 1 : h.per_cu == 1 ? std::ceil(r) : 0.5 * (r + std::ceil(r));
        const double t = kLaunchUs + rounds * (KB * (r <= 1 ? h.alone : h.full) + h.end);
        if (t < *us) { *us = t; best = i; }
    }
    return best;
}

double proj_split_us(int M, int N, int K, int ndir, bool masked)
{
    double us;
    (void)choose_shape(M, N, K, ndir, masked, &us);
    return us + 3 * kLaunchUs + 8.0 * M * K / 5.4e6;   // the pass over X, its launch and the gaps
}

// More than 64 input rows, K from 64 on (with fewer terms the fp32 instruction's sum is as close to the exact one) and
// large enough that the pass over X is made up for.
bool proj_split_supported(int M, int N, int K, int ndir, bool masked)
{
    if (M <= 64 || K < kSplitMinK || K % 4 != 0) return false;
    const double tiles = (double)((M + 63) / 64) * ((N + 63) / 64) * ndir;
    const double f32_us = 2 * kLaunchUs + (K + 31) / 32 * std::max(0.83, 0.66 * tiles / device_num_cus());   // 64 x 64 tiles, fp32
    return proj_split_us(M, N, K, ndir, masked) < f32_us;
}

hipError_t launch_proj_split(const ProjSplitArgs& a, hipStream_t s)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if (a.K % 4 != 0 || a.ldx % 4 != 0) return hipErrorInvalidValue;
    double us;
    const int shape = choose_shape(a.M, a.N, a.K, a.ndir, a.masked != 0, &us);
    if (a.masked)
        switch (shape) {
            case 1: return launch_tiles<2, 2, 2, 4, 2, true>(a, 1, s);
            case 2: return launch_tiles<2, 2, 2, 2, 2, true>(a, 2, s);
            case 3: return launch_tiles<2, 1, 1, 4, 3, true>(a, 2, s);
            default: return launch_tiles<1, 1, 2, 2, 4, true>(a, 2, s);
        }
    switch (shape) {
        case 0: return launch_tiles<4, 2, 2, 4, 2, false>(a, 1, s);
        case 1: return launch_tiles<2, 2, 2, 4, 2, false>(a, 1, s);
        case 2: return launch_tiles<2, 2, 2, 2, 2, false>(a, 2, s);
        case 3: return launch_tiles<2, 1, 1, 4, 3, false>(a, 2, s);
        default: return launch_tiles<1, 1, 2, 2, 4, false>(a, 2, s);
    }
}

}  // namespace l355
