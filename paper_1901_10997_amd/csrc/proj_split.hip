// fp32 input projection on the fp16 matrix instruction:  P[m][n] = bias[n] + sum_k X[m][k] * W[n][k]
//
// Every fp32 value of a row is scaled by a power of two that brings the row's largest magnitude into [2^14, 2^15) and kept
// as two fp16 numbers, hi = fp16(v) and lo = fp16(v - hi): 22 to 24 significant bits (one value in four is off by half a last
// place).  A product is then hi.hi + hi.lo + lo.hi (lo.lo is 2^-22 of it at most), three instructions whose products are exact
// and whose sums are fp32, 16 k per 32 clocks each where the fp32 instruction takes 2 k in 64: a tenth of the matrix time.  An
// instruction also rounds less often per k, which from some terms on (kSplitMinTerms below) more than makes up for the bits the
// planes drop: error against 64 bits, fp32 instruction / here, relative to the product's norm, dense W: K 64 1.35e-7 / 1.17e-7,
// 200 2.5e-7 / 1.8e-7, 640 4.4e-7 / 2.9e-7, 1600 7.2e-7 / 4.5e-7 (normal X, uniform W; K 32 9.26e-8 / 9.34e-8).
//
// Layout: the planes of 32 k lie side by side, 64 bytes hi and 64 bytes lo, so that a slab of 32 k of a row is one 128-byte
// line; slabs go straight into an LDS ring (16-byte chunk c of row r at position c ^ ((r >> 1) & 7): conflict-free reads), and
// a fragment read serves two or one of the three products: two slab bytes per product fewer than a bf16 product needs.
// Bound: the device's power limit under random operands (the issue loop of this instruction reaches 1.7 PFLOP/s there) and
// what a tile's ends leave idle.  4800 x 3200 x 1600 in two directions, with the split: fp32 instruction 835 to 901 us (109 to
// 118 TFLOP/s), here 279 to 311 (350 to 316; three times that counted as fp16 products); x 640: 348 to 389 -> 127 to 129; 700 x 6000
// x 1500: 163 -> 59.
#include <cmath>
#include "common.h"
#include "device_math.h"

namespace l355 {

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kXcds = 8;
constexpr int kGroupM = 4;

// A sum on the fp32 instruction is off by the rounding of its terms that are not zero, 1.8e-8 sqrt(n) of the product's norm; on planes
// by what the planes drop as well, 0.75e-7 and more whatever n is.  Error against 64 bits, fp32 instruction / planes in stages: 52 of
// 1032 entries kept 1.31e-7 / 0.90e-7, 64 of 640 1.45e-7 / 0.97e-7, 80 of 1600 1.62e-7 / 0.91e-7 (32 of 640 1.03e-7 / 0.9e-7 by a
// model of the sums): level at 25 terms; in one stage (less than two in five are zero) at 46.  Rows of W are judged together (long
// ones count for twice the limit at most), rows of X one by one.
constexpr int kSplitMinTerms = 48, kSplitMinTermsStaged = 32;

// ---- rows into two fp16 planes
// out: per row KB blocks of 128 bytes, 32 hi values then 32 lo values of k = 32 kb ..; unscale: 2^-e of the row's scale 2^e, or a mark
// where the row does not fit (device_math.h; with `marks`, also where it has too few terms).
constexpr int kSplitRowsPerBlock = 4;

__device__ __forceinline__ uint32_t pack_f16x2(_Float16 a, _Float16 b)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

template <int VEC>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ X, int ldx, int M, int K, int KB,
                                                         uint16_t* __restrict__ out, float* __restrict__ unscale,
                                                         SplitMarks* __restrict__ marks, int* __restrict__ terms)
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
        if (lane == 0) {
            float u = split_unscale(sc, big, small, nonzero);
            if (marks && nonzero > 0 && nonzero < kSplitMinTerms && u < __uint_as_float(kNonFinite)) u = __uint_as_float(kTooWide);
            unscale[m] = u;
            if (terms) terms[m] = nonzero;
            if (marks && !(u < __uint_as_float(kNonFinite))) marks->found = ~marks->next;
            if (marks && m == 0) marks->pass = marks->next;
        }
    }
}

size_t split_row_halves(int K) { return (size_t)((K + 31) / 32) * 64; }

hipError_t launch_split_rows(const float* X, int ldx, int M, int K, uint16_t* out, float* unscale, SplitMarks* marks, int* terms,
                             hipStream_t s)
{
    const int KB = (K + 31) / 32;
    const dim3 grid((M + kSplitRowsPerBlock - 1) / kSplitRowsPerBlock), block(256);
    if (K % 4 == 0 && ldx % 4 == 0 && ((uintptr_t)X & 15) == 0)
        hipLaunchKernelGGL(split_rows_kernel<4>, grid, block, 0, s, X, ldx, M, K, KB, out, unscale, marks, terms);
    else
        hipLaunchKernelGGL(split_rows_kernel<1>, grid, block, 0, s, X, ldx, M, K, KB, out, unscale, marks, terms);
    return hipGetLastError();
}

bool split_terms_suffice(const int* terms, int rows, int K, bool* many_zeros)
{
    long long all = 0, capped = 0, some = 0;
    for (int r = 0; r < rows; ++r) all += terms[r];
    *many_zeros = (double)all < 0.6 * (double)rows * (double)K;
    const int least = *many_zeros ? kSplitMinTermsStaged : kSplitMinTerms;
    for (int r = 0; r < rows; ++r) {
        capped += std::min(terms[r], 2 * least);
        some += terms[r] > 0;
    }
    return capped >= least * some;
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

// STAGED (weights with many zeros): sums in stages of kStage slabs.  An fp32 sum that meets a mask's zeros rounds once per kept term;
// an instruction over 16 k rounds whether they are zeros or not, 3 K / 16 times in all.  In stages the terms are a small part of the
// sum when they are rounded; the products with a low plane, a thousandth of the others, have accumulators of their own, and what
// adding a stage rounds off goes into the next.  K 1600, 15 % kept, error against 64 bits relative to the product's norm: fp32
// instruction 2.8e-7, one stage 3.8e-7, stages that lose both 1.5e-7, these 1.0e-7 (4800 x 3200 in two directions, with the split:
// 282 -> 300 us for the last step; in one stage about 245).  Three sets of sums leave no registers for offsets worked out ahead.
constexpr int kStage = 4;
template <bool FIRST, class A, class B>
__device__ __forceinline__ auto& pick(A& a, B& b)
{
    if constexpr (FIRST) return a;
    else return b;
}
__device__ __forceinline__ void end_stage(f32x16& acc, f32x16& total)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float t = total[v] + acc[v];
        acc[v] -= t - total[v];                           // what that sum rounds off: the next stage starts from it
        total[v] = t;
    }
}

// ---- rows that have no fp16 form
// They are summed by the fp32 instruction, and a row's result depends on that row alone: where any is marked the rows are dealt out
// to the tiles by kind, the marked ones to tiles of their own.  A workgroup works that out for itself: a mask of the marked rows
// per 64, their number before each, and the n-th row of a kind from those.  That a row is marked stands in SplitMarks: a product
// without one never comes here.
constexpr int kSortRows = 32768;                          // of one launch (the table's size; more rows are several launches)
constexpr int kRowNonFinite = 1 << 30;
constexpr int kBeforeOff = kSortRows / 64 * 8, kRowOff = kBeforeOff + kSortRows / 64 * 2 + 16, kTableBytes = kRowOff + 256 * 4;
typedef const ProjSplitArgs __attribute__((address_space(4)))* ArgsInMemory;
template <class T>
using InLds = __attribute__((address_space(3))) T*;
struct RowTable {
    InLds<unsigned long long> mask;                       // [kSortRows / 64] marked rows
    InLds<unsigned short> before;                         // [kSortRows / 64 + 1] marked rows before each 64
    InLds<int> row;                                       // [BM] of the present tile; kRowNonFinite beside it
};

// returns the number of marked rows
template <int NW>
__device__ __forceinline__ int sort_rows(const float* x_unscale, int M, const RowTable& t, int tid)
{
    const int lane = tid & 63, chunks = (M + 63) >> 6;
    for (int c = tid >> 6; c < chunks; c += NW) {
        const int m = 64 * c + lane;
        const unsigned long long mask = __ballot(m < M && !(x_unscale[min(m, M - 1)] < __uint_as_float(kNonFinite)));
        if (lane == 0) t.mask[c] = mask;
    }
    __syncthreads();
    if (tid < 64) {
        constexpr int kPer = kSortRows / 64 / 64;
        int mine = 0;
        for (int i = 0; i < kPer; ++i) mine += kPer * lane + i < chunks ? __popcll(t.mask[kPer * lane + i]) : 0;
        int at = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(at, o, 64);
            if (lane >= o) at += up;
        }
        if (lane == 63) t.before[chunks] = (unsigned short)at;   // all of them
        at -= mine;
        for (int i = 0; i < kPer; ++i) {
            const int c = kPer * lane + i;
            if (c < chunks) {
                t.before[c] = (unsigned short)at;
                at += __popcll(t.mask[c]);
            }
        }
    }
    __syncthreads();
    return t.before[chunks];
}

// the n-th row (from 0; there are more than n) that is marked, or that is not
__device__ __forceinline__ int nth_row(const RowTable& t, int chunks, int n, bool marked)
{
    int lo = 0, hi = chunks;                              // the last chunk with at most n of them before it
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1, b = t.before[mid];
        if ((marked ? b : 64 * mid - b) <= n) lo = mid; else hi = mid;
    }
    int k = n - (marked ? (int)t.before[lo] : 64 * lo - (int)t.before[lo]), pos = 0;
    const unsigned long long bits = marked ? t.mask[lo] : ~t.mask[lo];
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const int c = __popcll((bits >> pos) & ((1ull << w) - 1ull));
        if (k >= c) { k -= c; pos += w; }
    }
    return 64 * lo + pos;
}

// All tiles of this workgroup where a row is marked (right where none is, too).
// TS x TN: tiles of a wave, with half the rows of the kernel's, whose registers this shares.  Slabs of 32 k through the LDS ring
// for both kinds (a row's 128 bytes hold both planes of 32 values, or 32 fp32 ones); the fp32 instruction leaves out blocks of
// 32 rows that have none.  A row with a non-finite value is summed over the kept entries where W is held row-compressed: the
// mask selects, and what it leaves out must not meet an infinity as a zero.
// 4800 x 3200 in two directions, K 640 / 1600, microseconds with the split: every row marked 400 / 897 (fp32 kernel of proj_mfma.hip,
// which needs no split, 348 / 835; whole tiles with the operands straight from memory 688 / 1670), every other row 289 / 614
// (684 / 1669), one row 186 / 369 (728 / 1733), none 127 / 279.  Blocks of half a tile: 3.9 waves of them, and what a tile's ends
// leave idle.
template <int TS, int TN, int WM, int WN, int NST, bool STAGED>
__device__ __forceinline__ void sorted_tiles(ArgsInMemory a, unsigned lds0, unsigned table)
{
    constexpr int BM = WM * TS * 32, BN = WN * TN * 32, NW = WM * WN, ROWB = 128, STAGE = (BM + BN) * ROWB, LI = (BM + BN) / 8 / NW;
    static_assert((BM + BN) % (8 * NW) == 0, "rows divide over the waves");
    int tid = threadIdx.x;
    // nothing of this is worked out ahead, in registers of the kernel's loop
    asm volatile("" : "+v"(tid), "+s"(a), "+s"(lds0), "+s"(table));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int fr = lane & 31, fk = lane >> 5;
    const int M = a->M, N = a->N, K = a->K, KB = (K + 31) >> 5, gn = a->gn, gnt = gn * a->ndir;
    RowTable t;
    t.mask = (InLds<unsigned long long>)table;
    t.before = (InLds<unsigned short>)(table + kBeforeOff);
    t.row = (InLds<int>)(table + kRowOff);
    const int marked = __builtin_amdgcn_readfirstlane(sort_rows<NW>(a->x_unscale, M, t, tid));
    // the tiles of marked rows first (each takes several times as long); of each kind consecutive ones share an XCD
    const int gm_f32 = (marked + BM - 1) / BM, gm_planes = (M - marked + BM - 1) / BM;
    const int per_f32 = (gm_f32 * gnt + kXcds - 1) / kXcds, per_planes = (gm_planes * gnt + kXcds - 1) / kXcds;
#pragma unroll 1
    for (int pid = blockIdx.x; pid < kXcds * (per_f32 + per_planes); pid += gridDim.x) {
        const bool f32 = pid < kXcds * per_f32;
        const int q = f32 ? pid : pid - kXcds * per_f32, gm = f32 ? gm_f32 : gm_planes;
        const int logical = (q % kXcds) * (f32 ? per_f32 : per_planes) + q / kXcds;
        if (logical >= gm * gnt) continue;
        const int span = kGroupM * gnt, group = logical / span, in = logical % span, first = group * kGroupM;
        const int gsz = (gm - first) < kGroupM ? (gm - first) : kGroupM;
        const int tn_all = in / gsz, dir = tn_all >= gn ? 1 : 0, n0 = (tn_all - dir * gn) * BN;
        const float* const bias = a->d[dir].bias;
        float* const P = a->d[dir].P;
        const bool by_entries = a->d[dir].row_ptr != nullptr;
        const bool by_hand = f32 && ((uintptr_t)a->X & 15) != 0;   // the caller's rows, at any address: no direct loads
        const int m0 = (first + in % gsz) * BM;           // the first row's number among its kind
        const int rows = min((f32 ? marked : M - marked) - m0, BM);
        __syncthreads();
        for (int r = tid; r < rows; r += 64 * NW) {
            const int m = marked == 0 || marked == M ? m0 + r : nth_row(t, (M + 63) >> 6, m0 + r, f32);
            t.row[r] = f32 && by_entries && __float_as_uint(a->x_unscale[m]) == kNonFinite ? m | kRowNonFinite : m;
        }
        __syncthreads();
        // bytes of this lane's 16 of every direct-load instruction: chunk kc of its row, and eight further on for every slab
        const unsigned char* src[LI];
        int kc[LI];
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const int row0 = (wave * LI + i) * 8, row = row0 + (lane >> 3);
            kc[i] = (lane & 7) ^ ((row >> 1) & 7);
            if (row0 < BM) {
                const size_t m = (size_t)(t.row[row < rows ? row : rows - 1] & ~kRowNonFinite);
                src[i] = f32 ? (const unsigned char*)(a->X + m * a->ldx) : (const unsigned char*)(a->Xs + m * KB * 64);
            } else {
                const size_t n = (size_t)min(n0 + row - BM, N - 1);
                src[i] = f32 ? (const unsigned char*)(a->d[dir].Wd + n * K) : (const unsigned char*)(a->d[dir].W + n * KB * 64);
            }
        }
        const int last = (f32 ? K / 4 : 8 * KB) - 1;      // chunk of a row (past the end the last one: not used)
        auto issue_slab = [&](int kt) {
            const unsigned st = lds0 + (unsigned)((kt % NST) * STAGE + wave * LI * 1024);
#pragma unroll
            for (int i = 0; i < LI; ++i) {
                const unsigned char* const from = src[i] + (size_t)min(8 * kt + kc[i], last) * 16;
                if (by_hand) {
                    const float* const f = (const float*)from;
                    *(InLds<u32x4>)(st + (unsigned)(i * 1024 + lane * 16)) =
                        (u32x4){__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
                } else {
                    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)from,
                                                     (void __attribute__((address_space(3)))*)(st + (unsigned)(i * 1024)), 16, 0, 0);
                }
            }
        };
        f32x16 acc[TS][TN], total[STAGED ? TS : 1][STAGED ? TN : 1], low[STAGED ? TS : 1][STAGED ? TN : 1];
#pragma unroll
        for (int i = 0; i < TS; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    acc[i][j][v] = 0.f;
                    if (STAGED) total[STAGED ? i : 0][STAGED ? j : 0][v] = low[STAGED ? i : 0][STAGED ? j : 0][v] = 0.f;
                }
        // fragments of this lane: chunk c of its rows
        auto read_a = [&](u32x4 (&f)[TS], unsigned st, int c) {
#pragma unroll
            for (int i = 0; i < TS; ++i) {
                const int r = (wm * TS + i) * 32 + fr;
                f[i] = lds_read_b128(st + (unsigned)(r * ROWB + ((c ^ ((r >> 1) & 7)) * 16)));
            }
        };
        auto read_b = [&](u32x4 (&f)[TN], unsigned st, int c) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = BM + (wn * TN + j) * 32 + fr;
                f[j] = lds_read_b128(st + (unsigned)(r * ROWB + ((c ^ ((r >> 1) & 7)) * 16)));
            }
        };
        auto arrived = [&](auto& f) {
#pragma unroll
            for (auto& v : f) asm volatile("" : "+v"(v) : : "memory");
        };
        // slab `target` has landed once only the loads of the (at most NST - 2) younger slabs can still be outstanding
        auto wait_slab = [&](int target) {
            const int younger = min(KB - 1 - target, NST - 2);
            if (NST >= 4 && younger == 2) wait_vmcnt<NST >= 4 ? 2 * LI : 0>();
            else if (NST >= 3 && younger == 1) wait_vmcnt<NST >= 3 ? LI : 0>();
            else wait_vmcnt<0>();
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");   // (by_hand)
            __builtin_amdgcn_s_barrier();
        };
#pragma unroll
        for (int k = 0; k < NST - 1; ++k)
            if (k < KB) issue_slab(k);
        wait_slab(0);
        if (NST - 1 < KB) issue_slab(NST - 1);
        if (f32) {
            u32x4 fa[2][TS], fb[2][TN];
            read_a(fa[0], lds0, fk);
            read_b(fb[0], lds0, fk);
#pragma unroll 1
            for (int kt = 0; kt < KB; ++kt) {
                const unsigned st = lds0 + (unsigned)((kt % NST) * STAGE), stn = lds0 + (unsigned)(((kt + 1) % NST) * STAGE);
#pragma unroll
                for (int u = 0; u < 4; ++u) {         // 8 k each: a lane's four are chunk 2 u + fk of its row; the next ones on their way
                    if (u < 3) {
                        read_a(fa[(u + 1) & 1], st, 2 * (u + 1) + fk);
                        read_b(fb[(u + 1) & 1], st, 2 * (u + 1) + fk);
                        asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(TS + TN) : "memory");
                    } else {
                        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                    }
                    arrived(fa[u & 1]);
                    arrived(fb[u & 1]);
                    if (u == 3 && kt + 1 < KB) {      // done with slab kt: its buffer may be refilled
                        wait_slab(kt + 1);
                        if (kt + NST < KB) issue_slab(kt + NST);
                        read_a(fa[0], stn, fk);
                        read_b(fb[0], stn, fk);
                    }
                    if (32 * kt + 32 > K) {           // K % 4 == 0: a lane's four values are all there or none is
                        const bool there = 32 * kt + 8 * u + 4 * fk < K;
#pragma unroll
                        for (int i = 0; i < TS; ++i) fa[u & 1][i] = there ? fa[u & 1][i] : (u32x4){0, 0, 0, 0};
#pragma unroll
                        for (int j = 0; j < TN; ++j) fb[u & 1][j] = there ? fb[u & 1][j] : (u32x4){0, 0, 0, 0};
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < TS; ++i)
                        if ((wm * TS + i) * 32 < rows)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
#pragma unroll
                                for (int j = 0; j < TN; ++j)
                                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa[u & 1][i][e]),
                                                                                     __uint_as_float(fb[u & 1][j][e]), acc[i][j], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
#pragma unroll 1
            for (int kt = 0; kt < KB; ++kt) {
                const unsigned st = lds0 + (unsigned)((kt % NST) * STAGE);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {      // the order of the products is that of the kernel below: the same bits
                    u32x4 ah[TS], al[TS], bh[TN], bl[TN];
                    read_a(ah, st, 2 * ks + fk);
                    read_b(bl, st, 4 + 2 * ks + fk);
                    read_b(bh, st, 2 * ks + fk);
                    read_a(al, st, 4 + 2 * ks + fk);
                    auto mma = [&](const u32x4 (&fa)[TS], const u32x4 (&fb)[TN], auto& to) {
#pragma unroll
                        for (int i = 0; i < TS; ++i)
#pragma unroll
                            for (int j = 0; j < TN; ++j)
                                to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[i]),
                                                                                  __builtin_bit_cast(f16x8, fb[j]), to[i][j], 0, 0, 0);
                    };
                    auto& lows = pick<STAGED>(low, acc);
                    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(TS + TN) : "memory");
                    arrived(ah);
                    arrived(bl);
                    mma(ah, bl, lows);
                    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                    arrived(bh);
                    arrived(al);
                    if (ks == 1 && kt + 1 < KB) {
                        wait_slab(kt + 1);
                        if (kt + NST < KB) issue_slab(kt + NST);
                    }
                    mma(ah, bh, acc);
                    mma(al, bh, lows);
                }
                if (STAGED && (kt % kStage == kStage - 1 || kt == KB - 1)) {
#pragma unroll
                    for (int i = 0; i < TS; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) end_stage(acc[i][j], total[STAGED ? i : 0][STAGED ? j : 0]);
                }
            }
            if (STAGED) {
#pragma unroll
                for (int i = 0; i < TS; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            acc[i][j][v] = total[STAGED ? i : 0][STAGED ? j : 0][v] + (acc[i][j][v] + low[STAGED ? i : 0][STAGED ? j : 0][v]);
            }
        }
        // accumulator register v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + (wn * TN + j) * 32 + fr, nc = n < N ? n : N - 1;
            const float b = bias[nc], wu = f32 ? 1.f : a->d[dir].w_unscale[nc];
#pragma unroll
            for (int i = 0; i < TS; ++i) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = (wm * TS + i) * 32 + 4 * fk + 8 * (v >> 2) + (v & 3);
                    const int m = t.row[r < rows ? r : rows - 1];
                    const float o = f32 ? acc[i][j][v] + b : fmaf(acc[i][j][v], a->x_unscale[m] * wu, b);
                    if (r < rows && n < N && !(m & kRowNonFinite)) P[(size_t)(m & ~kRowNonFinite) * N + n] = o;
                    if (v % 8 == 7) asm volatile("" : : : "memory");   // (few registers)
                }
            }
        }
        if (!f32 || !by_entries) continue;
        for (int r = wm * TS * 32; r < min((wm + 1) * TS * 32, rows); ++r) {
            const int m = __builtin_amdgcn_readfirstlane(t.row[r]);
            if (!(m & kRowNonFinite)) continue;
            const float* const x = a->X + (size_t)(m & ~kRowNonFinite) * a->ldx;
            for (int n = n0 + wn * TN * 32 + lane; n < min(n0 + (wn + 1) * TN * 32, N); n += 64) {
                float sum = 0.f;
                for (int e = a->d[dir].row_ptr[n]; e < a->d[dir].row_ptr[n + 1]; ++e)
                    sum = fmaf(a->d[dir].val[e], x[a->d[dir].col[e]], sum);
                P[(size_t)(m & ~kRowNonFinite) * N + n] = sum + bias[n];
            }
        }
    }
}

// TM x TN: 32 x 32 tiles of a wave; WM x WN waves; NST slabs in the LDS ring; STAGED: sums in two stages.
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
    // (asked for here, heard behind the first slab)
    const auto marks = (const SplitMarks __attribute__((address_space(4)))*)a.marks;
    const bool look = marks->found == ~marks->pass;
    if (blockIdx.x == 0 && tid == 0) a.marks->next = marks->pass + 1u;
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

        f32x16 acc[TM][TN], total[STAGED ? TM : 1][STAGED ? TN : 1], low[STAGED ? TM : 1][STAGED ? TN : 1];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    acc[i][j][v] = 0.f;
                    if (STAGED) total[STAGED ? i : 0][STAGED ? j : 0][v] = low[STAGED ? i : 0][STAGED ? j : 0][v] = 0.f;
                }

        // direct loads: instruction q of a slab covers LDS rows 8 q .. 8 q + 7 of the combined [X rows | W rows]
        // (eight rows of one operand: scalar base pointer, one 32-bit byte offset per instruction and lane)
        const uint16_t* const xbase = a.Xs + (size_t)m0 * rowh;
        const uint16_t* const wbase = a.d[dir].W + (size_t)n0 * rowh;
        const ptrdiff_t w_off = (const char*)wbase - (const char*)xbase;
        unsigned soff[LI];
        int sl = threadIdx.x & 63;
        asm volatile("" : "+v"(sl));                      // (worked out here, not ahead of the loop in registers of its own)
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const int row0 = (wave_s * LI + i) * 8;
            const int row = row0 + (sl >> 3);
            const int kc = (sl & 7) ^ ((row >> 1) & 7);
            const int r = row0 < BM ? min(row, M - 1 - m0) : min(row - BM, N - 1 - n0);   // rows past the matrix re-read its last
            soff[i] = (unsigned)(r * rowh + 8 * kc) * 2u;
        }
        auto issue_slab = [&](int kt) {
            unsigned char* st = smem + (size_t)(kt % NST) * STAGE + (size_t)wave_s * LI * 1024;
#pragma unroll
            for (int i = 0; i < LI; ++i) {
                const char* const from = (const char*)xbase + (wave_s * LI + i < BM / 8 ? 0 : w_off) + (size_t)kt * 128;
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
        auto mma = [&](u32x4 (&fa)[TM], u32x4 (&fb)[TN], auto& to) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[i]),
                                                                      __builtin_bit_cast(f16x8, fb[j]), to[i][j], 0, 0, 0);
        };
        auto& lows = pick<STAGED>(low, acc);
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
        wait_slab(0);
        if (look) break;
        __builtin_amdgcn_s_barrier();
        if (NST - 1 < KB) issue_slab(NST - 1);
        u32x4 ah[TM], al[TM], bh[TN], bl[TN];
        read_a(ah, lds0, 0, 0);
        read_b(bl, lds0, 0, 1);
        for (int kt = 0; kt < KB; ++kt) {
            if (STAGED) {
#pragma unroll
                for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(offa[i]));
#pragma unroll
                for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(offb[j]));
            }
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
                mma(ah, bl, lows);
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(TM) : "memory");
                arrived_b(bh);
                mma(ah, bh, acc);
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
                mma(al, bh, lows);
                if (STAGED && ks == 1 && (kt % kStage == kStage - 1 || kt == KB - 1)) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) end_stage(acc[i][j], total[STAGED ? i : 0][STAGED ? j : 0]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (STAGED) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] = total[STAGED ? i : 0][STAGED ? j : 0][v] + (acc[i][j][v] + low[STAGED ? i : 0][STAGED ? j : 0][v]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
        }
        // ---- P = acc * 2^-(ex + ew) + bias; accumulator register v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
        int l = threadIdx.x & 63;
        asm volatile("" : "+v"(l));                       // (worked out here, not ahead of the loop in registers of its own)
        const int er = l & 31, ek = l >> 5;
        const float* bias = a.d[dir].bias;
        float* P = a.d[dir].P;
        float bn[TN], wu[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + (wn * TN + j) * 32 + er, nc = n < N ? n : N - 1;
            bn[j] = bias[nc];
            wu[j] = a.d[dir].w_unscale[nc];
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = m0 + (wm * TM + i) * 32 + 4 * ek;
            float xu[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = mb + 8 * (v >> 2) + (v & 3);
                xu[v] = a.x_unscale[m < M ? m : M - 1];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = fmaf(acc[i][j][v], xu[v] * wu[j], bn[j]);
                asm volatile("" : "+v"(acc[i][j]));       // here, not beside the stores: the scales' registers are free again
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + (wn * TN + j) * 32 + er;
            if (n >= N) continue;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int mb = m0 + (wm * TM + i) * 32 + 4 * ek;
                if (mb - 4 * ek + 32 <= M) {
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
    // A row is marked somewhere: no tile is done yet.
    if (look) {
        wait_vmcnt<0>();
        __syncthreads();
        sorted_tiles<(TM + 1) / 2, TN, WM, WN, NST, STAGED>((ArgsInMemory)__builtin_amdgcn_kernarg_segment_ptr(), lds0, lds0 + NST * STAGE);
    }
}

template <int TM, int TN, int WM, int WN, int NST, bool STAGED>
static hipError_t launch_tiles(ProjSplitArgs a, int per_cu, hipStream_t s)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    a.gm = (a.M + BM - 1) / BM;
    a.gn = (a.N + BN - 1) / BN;
    a.npid = ((a.gm * a.gn * a.ndir + kXcds - 1) / kXcds) * kXcds;
    const int lds = NST * (BM + BN) * 128 + kTableBytes;
    const hipError_t e = allow_dynamic_lds((const void*)proj_split_kernel<TM, TN, WM, WN, NST, STAGED>, lds);
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
    return us + 3 * kLaunchUs + 8.0 * M * K / 5.4e6;   // the pass over X, its launch and the gaps (stages: 4 to 8 % over the fits)
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

static hipError_t launch_band(const ProjSplitArgs& a, hipStream_t s)
{
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

hipError_t launch_proj_split(const ProjSplitArgs& all, hipStream_t s)
{
    if (all.M <= 0 || all.N <= 0) return hipSuccess;
    if (all.K % 4 != 0 || all.ldx % 4 != 0 || !all.marks) return hipErrorInvalidValue;
    // rows the table holds, and whose planes a 32-bit offset reaches
    const size_t rowh = split_row_halves(all.K);
    const int band = (int)std::max<size_t>(64, std::min<size_t>(kSortRows, ((size_t)1 << 31) / rowh / 64 * 64));
    for (int m = 0; m < all.M; m += band) {
        ProjSplitArgs a = all;
        a.M = std::min(band, all.M - m);
        a.Xs += (size_t)m * rowh;
        a.x_unscale += m;
        a.X += (size_t)m * a.ldx;
        for (int d = 0; d < a.ndir; ++d) a.d[d].P += (size_t)m * a.N;
        const hipError_t e = launch_band(a, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace l355
