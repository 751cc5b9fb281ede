// Recurrence of a dense fp32 LSTM layer with the time loop on the device, the product on the fp16 matrix instruction:
//     a = P[t] + W_h . h_{t-1};   f,i,o = sigmoid, g = tanh;   c, h            (paper Section 4, cell equations)
// The frame is persist_quad.hip's: one launch per layer, every direction in the grid; a group of workgroups owns some quads
// (four batch columns) of a direction and all units, a workgroup 16 NT packed rows (4 NT units), its eight waves split K, the
// partial sums meet in LDS in a fixed order, and only the workgroups of a group exchange h, through one XCD's L2 where a
// group fits one.
//
// Product.  W_h and h are kept as two fp16 planes each (proj_split.hip): a row of W_h scaled by a power of two, hi + lo; h as
// hi = fp16(h) and lo = fp16((h - hi) 2^12), off by 2^-24 at most (|h| from a half on, one value in four; by less than 2^-36 near
// zero).  The 16x16x32 instruction takes 16 rows of one plane of W_h against 16 columns: the four columns of a quad in both planes
// fill eight of them, two quads (QP = 2) all sixteen, so two instructions give all four products of the planes for 32 k, and a
// column's sum is its hi part plus 2^-12 of its lo part.  fp32 takes four 4x4x1 instructions of 8.8 clocks per 16 k, this 16 per
// 16: less than half, at QP = 2 a quarter, and the instruction sums the 32 k itself, where the other needs a sum over four lane
// groups.
//
// K is dealt out in blocks of 32, KB or KB - 1 to a wave; the last waves, which have the fewest sums to finish, take the longer
// share.  Where KB blocks of weights do not fit the registers the last one is in LDS (XL; 800 units: 25 blocks, one wave with
// four).  An accumulator tile has its 64 sums in the first lanes of each row: moved to one register (DPP bank masks), a wave's
// partial tile is one 256-byte write (as 16-byte writes of sixteen lanes each, 64 of them took a fifth of the step).
//
// Exchange: 8-byte words of four units of a column and plane.  |h| <= 1 leaves bit 14 of a half free: that of the first carries
// the stamp (as in persist_quad.hip: two buffers, step tag g in buffer g & 1 with stamp (g >> 1) & 1), that of the second says
// that a NaN is among the four; a word is taken to arrive whole, also in one half of a 16-byte load (exchange.h).  hx: [quad][buffer]
// [block of 32 k][k / 8 % 4][plane][column][k / 4 % 2], the lanes' order.
// h0 may have any value: a column of it that is not within 1 is multiplied by the fp32 instruction before the first step, into its
// P, and travels as zeros.
#include "common.h"
#include "device_math.h"
#include "exchange.h"

namespace l355 {

namespace {
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned long long u64x2;
constexpr int kSW = 8, kSTH = 512;
constexpr float kLoScale = 4096.f;
constexpr unsigned kStamp = 0x4000u, kOddMark = 0x40000000u;   // in the low 32 bits of an exchange word

template <int CTRL>
__device__ __forceinline__ unsigned dpp_word(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) { return __uint_as_float(dpp_word<CTRL>(__float_as_uint(v))); }
// a, and in the rows' banks (of four lanes) BANKS b moved by CTRL
template <int CTRL, int BANKS>
__device__ __forceinline__ float dpp_bank(float a, float b)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(a), __float_as_int(b), CTRL, 0xF, BANKS, false));
}
__device__ __forceinline__ unsigned half_bits(_Float16 v) { return __builtin_bit_cast(uint16_t, v); }
// a half of more than 1 without its bit 14 is a NaN (in both planes)
__device__ __forceinline__ unsigned long long with_nans(unsigned long long v)
{
    const unsigned long long carried = (v & 0x3FFF3FFF3FFF3FFFull) + 0x03FF03FF03FF03FFull;
    return (v & 0xBFFFBFFFBFFFBFFFull) | (carried & 0x4000400040004000ull);
}
}  // namespace

// NT: tiles of 16 packed rows per workgroup; KB: k blocks of 32 per wave; XL: the last block's weights are in LDS; QP: quads
// per pass (1 or 2)
template <int NT, int KB, bool XL, int QP>
__global__ __launch_bounds__(kSTH) void persist_split_kernel(PersistQuadArgs a)
{
    constexpr int kItems = NT * QP;
    constexpr int kMine = (kItems + kSW - 1) / kSW;
    constexpr int KR = XL ? KB - 1 : KB;                                 // blocks in registers
    constexpr int kPart = kSW * kItems * 64, kAhead = 4;
    static_assert(KR >= 1 && KB >= 2, "layers of more than 256 units");
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* const part = lds;                                             // [2][8][NT][QP * 64]
    float* const cell = part + 2 * kPart;                                // [passes][QP][NT][64]
    const int H = a.H, gn = a.gn;
    int dir, grp, wg;
    if (a.xcd_local) {
        // the workgroups of a group take block ids of one residue modulo 8
        const int jj = blockIdx.x >> 3;
        const int id = (blockIdx.x & 7) + 8 * (jj / gn);
        if (id >= a.ndir * a.groups) return;                             // padding ids take no part in the exchange
        wg = jj % gn; dir = id / a.groups; grp = id - dir * a.groups;
    } else {
        const int id = blockIdx.x / gn;
        wg = blockIdx.x - id * gn; dir = id / a.groups; grp = id - dir * a.groups;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int q_lo = grp * a.mq;
    const int nq = a.quads - q_lo < a.mq ? a.quads - q_lo : a.mq;        // >= 1 (checked by the launcher)
    const int passes = (nq + QP - 1) / QP;

    const PersistQuadDir& D = a.d[dir];
    const float* const h0 = D.h0;
    float* const y = D.y;
    const size_t y_ld = (size_t)D.y_ld;
    float* const hT = D.hT;
    float* const cT = D.cT;
    const int reverse = D.reverse;

    const int NBt = (H + 3) >> 2;                                        // tiles of 16 packed rows = groups of four units
    const int KBt = (H + 31) >> 5;                                       // blocks of 32 k
    const int full = KBt - kSW * (KB - 1);                               // waves with KB blocks, the last ones (1..8: the launcher)
    const bool all_kb = wave >= kSW - full;                              // wave-uniform
    const int kb0 = wave * (KB - 1) + (all_kb ? wave - (kSW - full) : 0);
    f16x8* const wl = reinterpret_cast<f16x8*>(cell + (size_t)passes * kItems * 64) + (size_t)(wave - (kSW - full)) * NT * 128 + lane;   // [full][NT][plane][64]

    // weights: loads from clamped addresses, what lies outside is zeroed afterwards
    f16x8 w[NT][KR][2];
    {
        const f16x8* const Ws = reinterpret_cast<const f16x8*>(D.Ws) + lane;
        const f16x8 zero = {};
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < KB; ++q)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const bool ok = wg * NT + n < NBt && (q < KB - 1 || all_kb);
                    const f16x8 v = Ws[(((size_t)(ok ? wg * NT + n : 0) * KBt + (ok ? kb0 + q : 0)) * 2 + p) * 64];
                    if (q < KR) w[n][q < KR ? q : 0][p] = ok ? v : zero;
                    else if (all_kb) wl[(n * 2 + p) * 64] = ok ? v : zero;
                }
    }

    // This thread's elements of the sums: item i = wave, wave + 8, .. of a pass is tile i % NT of quad i / NT; column lg of
    // the quad, row lr of the tile: row 4 (unit) + gate.  Offsets inside a timestep stay with the lane, the pass and the timestep
    // advance on the scalar side.
    const int gate = lr & 3;
    int unit[kMine], qq[kMine], tl[kMine], col[kMine];
    bool live[kMine];
    float us[kMine];
    unsigned hoff[kMine];
    const size_t hquad = (size_t)KBt * 64;                               // 8-byte words
#pragma unroll
    for (int j = 0; j < kMine; ++j) {
        const int i = wave + kSW * j;
        live[j] = i < kItems;                                            // wave-uniform
        qq[j] = live[j] ? i / NT : 0;
        tl[j] = live[j] ? i - qq[j] * NT : 0;
        const int k4 = wg * NT + tl[j];                                  // group of four units
        unit[j] = 4 * k4 + (lr >> 2);
        us[j] = unit[j] < H ? D.w_unscale[4 * unit[j] + gate] : 0.f;
        col[j] = 4 * (q_lo + qq[j]) + lg;
        hoff[j] = (unsigned)(qq[j] * 2 * hquad) + (unsigned)((((k4 >> 1) * 2 + lr) * 4 + lg) * 2 + (k4 & 1));
    }
    // of a pass that may be short of quads
    auto have_quad = [&](int pass, int j) { return live[j] && pass * QP + qq[j] < nq; };
    auto have_col = [&](int pass, int j) { return have_quad(pass, j) && col[j] + 4 * QP * pass < a.B; };
    for (int pass = 0; pass < passes; ++pass)
#pragma unroll
        for (int j = 0; j < kMine; ++j)
            if (live[j]) {
                const int b = col[j] + 4 * QP * pass;
                cell[(pass * kItems + wave + kSW * j) * 64 + lane] = (D.c0 && have_col(pass, j) && unit[j] < H) ? D.c0[(size_t)b * H + unit[j]] : 0.f;
            }

    // operand lanes: column lr of the instruction is column lr % 4 of a quad in one plane; k 8 (lane / 16) .. + 7 of a block
    const int oc = lr & 3, oq = QP == 1 ? 0 : (lr >> 2) & 1, op_plane = QP == 1 ? (lr >> 2) & 1 : lr >> 3;
    unsigned long long* const hx = reinterpret_cast<unsigned long long*>(a.hx) + ((size_t)dir * a.quads + q_lo) * 2 * hquad;
    const __amdgpu_buffer_rsrc_t words = exchange_buffer(hx, (unsigned)(nq * 2 * hquad * 8));
    const bool tail0 = wave == kSW - 1 && 32 * (KBt - 1) + 8 * lg >= H, tail1 = wave == kSW - 1 && 32 * (KBt - 1) + 8 * lg + 4 >= H;
    const unsigned last0 = all_kb && !tail0 ? ~0u : 0u, last1 = all_kb && !tail1 ? ~0u : 0u;
    // a quad that is not there reads the last one that is: its products are never used
    auto quad_of = [&](int pass, int c) { return pass * QP + c < nq ? pass * QP + c : nq - 1; };

    bool same_xcd = false;
    if (a.xcd_local)
        same_xcd = group_shares_xcd(a.xcc_ids + (size_t)(dir * a.groups + grp) * 64, gn, wg, 1u, part, tid, kSTH,
                                    a.timeout_flag, a.spin_limit) && !a.device_scope_only;

    // columns of h0 that are not within 1 (launch_fill_and_check): any in this group?
    bool beyond = false;
    if (h0)
        for (int c = lane; c < 4 * nq; c += 64) beyond |= 4 * q_lo + c < a.B && D.beyond[4 * q_lo + c] != 0u;
    beyond = __builtin_amdgcn_ballot_w64(beyond) != 0ull;
    auto col_beyond = [&](int pass, int j) { return beyond && D.beyond[col[j] + 4 * QP * pass] != 0u; };
    const ptrdiff_t p_step = (ptrdiff_t)a.Bld * 4 * H * (reverse ? -1 : 1), y_step = (ptrdiff_t)a.Bld * (ptrdiff_t)y_ld * (reverse ? -1 : 1);
    // the timesteps of P and y in the order of the steps
    float* p_t = D.P + (reverse ? (size_t)(a.T - 1) * a.Bld * 4 * H : 0);
    float* y_t = y + (reverse ? (size_t)(a.T - 1) * a.Bld * y_ld : 0);
    // where the sum of this thread's item and row lies in a partial tile (see below)
    const int slot = QP == 1 ? 16 * (lr >> 2) + 4 * gate + lg : 64 * (gate >> 1) + 16 * (lr >> 2) + 8 * (gate & 1) + lg;
    // These columns' product for the first step, by the fp32 instruction over the fp32 weights (launch_to_frag16: tile, block of
    // 16 k, lane 16 (k / 4 % 4) + row, k % 4); operand column c < 4 QP is column c % 4 of quad c / 4.  Added to P by the thread that
    // reads that element below.  No row has a scale here: h0 may be of any size.  Once per layer, microseconds of a one-step recurrence
    // without / with such columns: 800 units 24 / 53, 1500 22 / 59, 2000 19 / 61 (a column of multiply-adds per lane: 226, 588, 503).
    for (int pass = 0; beyond && pass < passes; ++pass) {
        constexpr int kDeep = 4;
        const int KB16 = (H + 15) >> 4;
        const int b16 = 2 * kb0, e16 = min(2 * (kb0 + (all_kb ? KB : KB - 1)), KB16);
        const int c = pass * QP * 4 + lr, b = 4 * q_lo + c;
        const bool to_sum = lr < 4 * QP && c < 4 * nq && b < a.B && D.beyond[b] != 0u;
        if (!__builtin_amdgcn_ballot_w64(to_sum)) continue;              // the same answer in every wave
        const float* const hb = h0 + (size_t)(to_sum ? b : 0) * H;
#pragma unroll 1
        for (int n = 0; n < NT && wg * NT + n < NBt; ++n) {              // (tiles that are not there: never used)
            const f32x4* const Wf = reinterpret_cast<const f32x4*>(D.Wf) + (size_t)(wg * NT + n) * KB16 * 64 + lane;
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int kb = b16; kb < e16; kb += kDeep) {                  // that many blocks requested together
                f32x4 w4[kDeep];
                float h4[kDeep][4];
#pragma unroll
                for (int u = 0; u < kDeep; ++u) {
                    const int at = min(kb + u, e16 - 1);
                    w4[u] = Wf[(size_t)at * 64];
#pragma unroll
                    for (int i = 0; i < 4; ++i) h4[u][i] = hb[min(16 * at + 4 * lg + i, H - 1)];
                }
#pragma unroll
                for (int u = 0; u < kDeep; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        sum = __builtin_amdgcn_mfma_f32_16x16x4f32(w4[u][i], to_sum && kb + u < e16 && 16 * (kb + u) + 4 * lg + i < H ? h4[u][i] : 0.f, sum, 0, 0, 0);
            }
            // rows 4 lg + i of column lr, in the order of the planes' partial tiles
            if (lr < 4 * QP)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    part[(wave * kItems + n * QP) * 64 + 16 * lg + lr + (QP == 1 ? 4 * i : 64 * (i >> 1) + 8 * (i & 1))] = sum[i];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kMine; ++j)
            if (have_col(pass, j) && unit[j] < H && col_beyond(pass, j)) {
                const float* const from = part + tl[j] * QP * 64 + slot + 4 * qq[j];
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < kSW; ++i) sum += from[i * kItems * 64];
                p_t[(size_t)pass * (4 * QP * 4) * H + (unsigned)(col[j] * 4 * H + 4 * unit[j] + gate)] += sum;
            }
        __syncthreads();
    }

    // h of item j as step tag `tag` of its buffers.  Lane 4 u + p of a row: unit u, plane p; the four units of a plane are gathered
    // in lane p.  Columns beyond the batch are published as well (readers wait for every word; what such a column holds is
    // never used).
    auto publish = [&](float h, unsigned tag, int pass, int j) {
        const _Float16 hi = (_Float16)h, lo = (_Float16)((h - (float)hi) * kLoScale);
        const unsigned bits = half_bits(gate == 0 ? hi : lo);
        const unsigned w0 = bits | (dpp_word<0x104>(bits) << 16), w1 = dpp_word<0x108>(bits) | (dpp_word<0x10C>(bits) << 16);
        if (lr < 2 && have_quad(pass, j) && unit[j] < H) {   // (lanes 0 and 1: the first unit of the four)
            const unsigned mark = ((w0 | w1) & 0x40004000u) ? kOddMark : 0u;
            const unsigned lo32 = (w0 & 0xBFFFBFFFu) | mark | (((tag >> 1) & 1u) ? kStamp : 0u);
            exchange_store(hx + ((size_t)pass * QP * 2 + (tag & 1u)) * hquad + hoff[j], ((unsigned long long)(w1 & 0xBFFFBFFFu) << 32) | lo32,
                           same_xcd);
        }
    };
    // the initial state travels like every other (zeros too: a buffer's stamps have to alternate)
    for (int pass = 0; pass < passes; ++pass)
#pragma unroll
        for (int j = 0; j < kMine; ++j)
            if (live[j]) {
                const bool there = h0 && have_col(pass, j) && unit[j] < H && !col_beyond(pass, j);
                publish(there ? h0[(size_t)(col[j] + 4 * QP * pass) * H + unit[j]] : 0.f, 2u, pass, j);
            }

    float p_next[kMine];
    auto load_p = [&](int pass) {
        const float* const Pt = p_t + (size_t)pass * (4 * QP * 4) * H;
#pragma unroll
        for (int j = 0; j < kMine; ++j)
            p_next[j] = have_col(pass, j) && unit[j] < H ? Pt[(unsigned)(col[j] * 4 * H + 4 * unit[j] + gate)] : 0.f;
    };
    load_p(0);
    int buf = 0;                                                         // of the partial tiles
    const float near = gate == 3 ? kTanhNear : -1.f;                     // the candidate's tanh
    float lo_scale;                                                      // in a register: the sum of the planes is one instruction
    asm volatile("v_mov_b32 %0, 0x39800000" : "=v"(lo_scale));           // 2^-12

    for (int s = 0; s < a.T; ++s) {
        const bool last = s == a.T - 1;
        for (int pass = 0; pass < passes; ++pass) {
            float* const part_b = part + buf * kPart;
            // ---- operand words of h_{t-1}: two of four k per lane and block
            u64x2 fr[KB];
            const unsigned tag = (unsigned)s + 2u;
            const unsigned want = ((tag >> 1) & 1u) ? kStamp : 0u;
            const int src = (int)((tag & 1u) * hquad + (QP == 1 ? (size_t)pass * 2 * hquad : 0)) * 8;
            const int loff = (((lg * 2 + op_plane) * 4 + oc) * 2 + (QP == 1 ? 0 : (int)(quad_of(pass, oq) * 2 * hquad))) * 8;
            pace_poll(a.poll_pace);
            unsigned spins = 0, differ;
            for (;;) {
                differ = 0;
                asm volatile("" ::: "memory");                           // read anew in every round
                // a wave without a last block reads its first one twice; a lane without a column multiplies what another reads
                // (never used)
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    const int block = (q < KB - 1 || all_kb ? kb0 + q : kb0) * 512;
                    if constexpr (KB > 2 || NT > 3) {
                        fr[q] = exchange_load16<u64x2>(words, loff, src + block);
                    } else {   // a narrow layer's first round would come before the words do (337 units: 244 us as pairs, 250 so)
                        const unsigned long long* const at = hx + (unsigned)(src + block) / 8u;
                        fr[q].x = __hip_atomic_load(at + (unsigned)loff / 8u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        fr[q].y = __hip_atomic_load(at + (unsigned)loff / 8u + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);                       // all on their way before the first is waited for
                // words of K's last block whose units are all beyond the last one are never written; of a wave without a last block
                // its words are looked at all the same (a load still on its way would make a later wait one for P's too)
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    const unsigned x = (unsigned)fr[q].x ^ want, y = (unsigned)fr[q].y ^ want;
                    if (q < KB - 1) differ |= x | y;
                    else differ |= (x & last0) | (y & last1);
                }
                if (!__builtin_amdgcn_ballot_w64((differ & kStamp) != 0u)) break;
                if (++spins > a.spin_limit) {
                    __hip_atomic_store(a.timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                if ((spins & 63u) == 0 && __hip_atomic_load(a.timeout_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
            }
            const bool odd = __builtin_amdgcn_ballot_w64((differ & kOddMark) != 0u) != 0ull;
            // this step's elements of P were requested a pass ahead; behind the words just waited for they have arrived too
            // (taken over here by hand: at the top of the loop the wait for them would include the stores just issued)
            float p_cur[kMine];
#pragma unroll
            for (int j = 0; j < kMine; ++j) asm volatile("v_mov_b32 %0, %1" : "=v"(p_cur[j]) : "v"(p_next[j]));
            if (pass + 1 < passes) {
                load_p(pass + 1);
            } else if (!last) {
                p_t += p_step;
                load_p(0);
            }
            float* const mine = part_b + wave * kItems * 64 + lane;
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                fr[q].x &= ~(unsigned long long)kStamp;
                fr[q].y &= ~(unsigned long long)kStamp;
            }
            if (odd) {
#pragma unroll
                for (int q = 0; q < KB; ++q) { fr[q].x = with_nans(fr[q].x); fr[q].y = with_nans(fr[q].y); }
            }
            f32x4 acc[NT];
#pragma unroll
            for (int q = 0; q < KR; ++q)
                if (q < KB - 1 || all_kb) {
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[n][q][p], __builtin_bit_cast(f16x8, fr[q]),
                                                                            q + p == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : acc[n], 0, 0, 0);
                }
            if (XL && all_kb) {
                f16x8 x[kAhead];                                     // that many reads ahead of the product
#pragma unroll
                for (int i = 0; i < kAhead; ++i) x[i] = wl[i * 64];
#pragma unroll
                for (int i = 0; i < 2 * NT; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
                    acc[i >> 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[i % kAhead], __builtin_bit_cast(f16x8, fr[KB - 1]), acc[i >> 1], 0, 0, 0);
                    if (i + kAhead < 2 * NT) x[i % kAhead] = wl[(i + kAhead) * 64];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // Accumulator register i of lane 16 g + c: row 4 g + i, column c; columns 4 quad + (column of the quad) of hi, the same of
            // lo four (QP = 2: eight) lanes up.  After the sum of the planes, register i of the first lanes of a row moves to the lanes
            // 4 i (QP = 2: 8 (i % 2)) up.
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = fmaf(dpp_mov<QP == 1 ? 0x104 : 0x108>(acc[n][i]), lo_scale, acc[n][i]);
                if constexpr (QP == 1) {
                    mine[n * 64] = dpp_bank<0x11C, 8>(dpp_bank<0x118, 4>(dpp_bank<0x114, 2>(v[0], v[1]), v[2]), v[3]);
                } else {
                    mine[n * 128] = dpp_bank<0x118, 12>(v[0], v[1]);
                    mine[n * 128 + 64] = dpp_bank<0x118, 12>(v[2], v[3]);
                }
            }
            // one barrier per pass: the partial tiles alternate between two buffers, and a wave that runs ahead reaches
            // the next barrier only after writing the other one
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kMine; ++j)
                if (live[j]) {
                    float* const cp = cell + (pass * kItems + wave + kSW * j) * 64 + lane;
                    const float* const from = part_b + tl[j] * QP * 64 + slot + 4 * qq[j];
                    float v[kSW];
#pragma unroll
                    for (int i = 0; i < kSW; ++i) v[i] = from[i * kItems * 64];
                    const float c_prev = *cp;
                    __builtin_amdgcn_sched_barrier(0);                   // all on their way before the first is waited for
                    const float sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                    const float pre = fmaf(sum, us[j], p_cur[j]);
                    const bool cand = gate == 3;
                    const float rr = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f((cand ? 2.8853900817779268f : -1.4426950408889634f) * pre));
                    float gv = cand ? fmaf(-2.0f, rr, 1.0f) : rr;
                    gv = fabsf(pre) < near ? tanhf_near(pre) : gv;
                    const float f = dpp_mov<0x00>(gv), ig = dpp_mov<0x55>(gv), o = dpp_mov<0xAA>(gv), g = dpp_mov<0xFF>(gv);   // of a lane quad
                    const float c = fmaf(f, c_prev, ig * g);
                    const float h = o * tanhf_exact(c);
                    if (!last) publish(h, (unsigned)s + 3u, pass, j);
                    *cp = c;
                    // outputs after the publication: nothing on the way of h
                    if (have_col(pass, j) && unit[j] < H && gate == 0) {
                        (y_t + (size_t)pass * (4 * QP) * y_ld)[(unsigned)(col[j] * (int)y_ld + unit[j])] = h;
                        if (last) {
                            const size_t at = (size_t)(col[j] + 4 * QP * pass) * H + unit[j];
                            if (hT) hT[at] = h;
                            if (cT) cT[at] = c;
                        }
                    }
                }
            buf ^= 1;
        }
        y_t += y_step;
    }
}

// ---------------------------------------------------------------------------------------------- shapes and launch
namespace {
struct SplitRecShape {
    int nt, kb, qp;
    bool xl;
    const void* kernel;
};
#define S_L(NT_, KB_, XL_, QP_) {NT_, KB_, QP_, XL_, (const void*)persist_split_kernel<NT_, KB_, XL_, QP_>}
// the shapes whose weights (NT KB x 32 bytes per lane), operands and accumulators fit the registers
const SplitRecShape kSplitRecShapes[] = {
    S_L(1, 2, false, 1), S_L(2, 2, false, 1), S_L(3, 2, false, 1),
    S_L(4, 2, false, 1), S_L(6, 2, false, 1), S_L(8, 2, false, 1), S_L(2, 2, false, 2), S_L(3, 2, false, 2),
    S_L(4, 2, false, 2), S_L(6, 2, false, 2), S_L(8, 2, false, 2), S_L(1, 3, false, 1), S_L(2, 3, false, 1),
    S_L(3, 3, false, 1), S_L(5, 3, false, 1), S_L(6, 3, false, 1), S_L(7, 3, false, 1), S_L(2, 3, false, 2),
    S_L(3, 3, false, 2), S_L(5, 3, false, 2), S_L(6, 3, false, 2), S_L(7, 3, false, 2), S_L(1, 4, false, 1),
    S_L(2, 4, false, 1), S_L(3, 4, false, 1), S_L(4, 4, false, 1), S_L(5, 4, false, 1), S_L(2, 4, false, 2),
    S_L(3, 4, false, 2), S_L(4, 4, false, 2), S_L(5, 4, false, 2), S_L(7, 4, true, 1), S_L(7, 4, true, 2),
    S_L(1, 5, false, 1), S_L(2, 5, false, 1), S_L(3, 5, false, 1), S_L(4, 5, false, 1), S_L(2, 5, false, 2),
    S_L(3, 5, false, 2), S_L(4, 5, false, 2), S_L(5, 5, true, 1), S_L(5, 5, true, 2), S_L(1, 6, false, 1),
    S_L(2, 6, false, 1), S_L(3, 6, false, 1), S_L(2, 6, false, 2), S_L(3, 6, false, 2), S_L(4, 6, true, 1),
    S_L(4, 6, true, 2), S_L(1, 7, false, 1), S_L(2, 7, false, 1), S_L(3, 7, false, 1), S_L(2, 7, false, 2),
    S_L(3, 7, false, 2), S_L(1, 8, false, 1), S_L(2, 8, false, 1), S_L(2, 8, false, 2), S_L(3, 8, true, 1),
    S_L(3, 8, true, 2),
};
#undef S_L
constexpr int kSplitRecShapeCount = (int)(sizeof(kSplitRecShapes) / sizeof(kSplitRecShapes[0]));
}  // namespace

// Shape, quads per group and placement of the lowest estimated step time in microseconds; the constants are a fit to 2960
// measured (shape, groups, placement) points over 100 to 2000 units and 4 to 128 columns (standard error 7 %; the choice is
// within 1.3 % of the best point on average).  Microseconds per step, persist_quad.hip / here: 200 units, 16 columns of two
// directions 0.94 / 1.08, 400 1.54 / 1.46, 640 2.08 / 1.58, 800 2.90 / 2.14, 1024 4.35 / 2.35; 64 columns of two directions 400
// 4.1 / 2.6, 800 10.7 / 5.5; 1197, 20 columns 4.75 / 2.8; 1500, 16 columns 5.2 / 3.0.
PersistQuadPlan persist_split_plan(int B, int H, int ndir)
{
    PersistQuadPlan best;
    if (B < 1 || H < 1 || ndir < 1 || ndir > 2) return best;
    const int blocks = (H + 31) / 32, tiles = (H + 3) / 4, quads = (B + 3) / 4, cus = device_num_cus();
    for (int i = 0; i < kSplitRecShapeCount; ++i) {
        const SplitRecShape& sh = kSplitRecShapes[i];
        if ((blocks + kSW - 1) / kSW != sh.kb) continue;
        const int gn = (tiles + sh.nt - 1) / sh.nt;
        for (int groups = 1; groups <= quads && ndir * groups * gn <= cus; ++groups) {
            const int mq = (quads + groups - 1) / groups;
            if ((quads + mq - 1) / mq != groups) continue;   // a group would be left without a quad
            const int passes = (mq + sh.qp - 1) / sh.qp;
            if (sh.qp > 1 && 2 * mq <= sh.qp) continue;      // half of every pass would be empty
            const size_t lds = (((size_t)(2 * kSW + passes) * sh.qp * sh.nt) * 64 + (sh.xl ? (size_t)(blocks - kSW * (sh.kb - 1)) * sh.nt * 512 : 0)) * sizeof(float);
            if (lds > 160 * 1024) continue;
            const int per_xcd = (ndir * groups + 7) / 8;
            const int local = gn <= 64 && per_xcd * gn <= cus / 8;
            const int items = sh.qp * sh.nt;
            const double pass = (local ? 0.604 + 0.034 * sh.qp * per_xcd : 0.838) + 0.0297 * sh.nt * sh.kb + 0.0457 * items +
                                0.0265 * std::max(0, items - 8) + 0.0132 * sh.qp * 16e-3 * H;
            const double us = passes * pass + (passes == 1 ? (local ? 0.25 : 0.51) : 0.0);
            if (us < best.us) {
                best.us = us;
                best.shape = i;
                best.mq = mq; best.groups = groups; best.gn = gn; best.xcd_local = local; best.lds = lds;
            }
        }
    }
    return best;
}

// exchange words of one launch: h, then (8-byte) XCD id slots of the groups
static size_t split_h_words(int B, int H, int ndir) { return (size_t)ndir * ((B + 3) / 4) * 2 * ((H + 31) / 32) * 128; }
size_t persist_split_exchange_words(int B, int H, int ndir) { return split_h_words(B, H, ndir) + (size_t)ndir * ((B + 3) / 4) * 64 * 2; }

void persist_split_describe(const PersistQuadPlan& p, char* buf, size_t n)
{
    const SplitRecShape& sh = kSplitRecShapes[p.shape];
    std::snprintf(buf, n, "(t%d,k%d,q%d,%dx%d%s,split)", sh.nt, sh.kb, sh.qp, p.groups, p.mq, p.xcd_local ? ",xcd" : "");
}

// p: the plan of (a.B, a.H, a.ndir); words: the launch's exchange region, all zero
hipError_t launch_persist_split(PersistQuadArgs& a, const PersistQuadPlan& p, unsigned* words, bool cooperative, hipStream_t s)
{
    if (a.B <= 0 || a.H <= 0 || a.T <= 0) return hipSuccess;
    if (p.shape < 0) return hipErrorInvalidValue;
    const void* const kernel = kSplitRecShapes[p.shape].kernel;
    a.quads = (a.B + 3) / 4;
    a.mq = p.mq; a.groups = p.groups; a.gn = p.gn; a.xcd_local = p.xcd_local;
    // Other passes in between, or an exchange inside an XCD: a short wait there from three k blocks on, as the words are read in half
    // the requests and the first round came too early (800 units, both directions, batch 16, 200 steps: 404 us unpaced, 390, 384, 381,
    // 381 and 394 at 1 to 4 and 6; 640: 314, 301 at 2 and 3; 457, two k blocks: 237, 249 at 1).
    if (p.mq > kSplitRecShapes[p.shape].qp) a.poll_pace = 0;
    else if (p.xcd_local) a.poll_pace = kSplitRecShapes[p.shape].kb > 2 ? 3 : 0;
    a.hx = words;
    a.ux = nullptr;
    a.xcc_ids = (unsigned long long*)(words + split_h_words(a.B, a.H, a.ndir));
    const int grid = p.xcd_local ? 8 * ((a.ndir * p.groups + 7) / 8) * p.gn : a.ndir * p.groups * p.gn;
    // every workgroup must be resident at the same time: at most one per compute unit
    if (grid > device_num_cus()) return hipErrorCooperativeLaunchTooLarge;
    if (p.lds > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(kernel, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    void* kargs[] = {(void*)&a};
    if (cooperative) return hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(kSTH), kargs, (unsigned)p.lds, s);
    return hipLaunchKernel(kernel, dim3(grid), dim3(kSTH), kargs, p.lds, s);
}

// W_h from its fp32 fragment order (launch_to_frag16) as two fp16 planes in the order of the 16x16x32 instruction: tile of 16 rows,
// block of 32 k, plane, lane l: row l % 16, k 8 (l / 16) .. + 7.  A workgroup per tile; unscale as launch_split_rows.
__global__ __launch_bounds__(256) void to_frag_split_kernel(const float4* __restrict__ Wf, int rows, int cols, uint16_t* __restrict__ out,
                                                            float* __restrict__ unscale)
{
    __shared__ unsigned big[16];
    __shared__ int small[16], nonzero[16];
    const int nb = blockIdx.x, KB16 = (cols + 15) >> 4, KB32 = (cols + 31) >> 5;
    const int l = threadIdx.x & 63, r = l & 15;
    if (threadIdx.x < 16) { big[threadIdx.x] = 0; small[threadIdx.x] = 0; nonzero[threadIdx.x] = 0; }
    __syncthreads();
    unsigned mine = 0;
    for (int kb = threadIdx.x >> 6; kb < KB16; kb += 4) {
        const float4 v = Wf[((size_t)nb * KB16 + kb) * 64 + l];
        mine = max(mine, max(max(__float_as_uint(v.x) & 0x7fffffffu, __float_as_uint(v.y) & 0x7fffffffu),
                             max(__float_as_uint(v.z) & 0x7fffffffu, __float_as_uint(v.w) & 0x7fffffffu)));
    }
    atomicMax(&big[r], mine);
    __syncthreads();
    const SplitScale sc = split_scale(big[r]);
    int sm = 0, nz = 0;
    for (int kb = threadIdx.x >> 6; kb < 2 * KB32; kb += 4) {
        const float4 v = kb < KB16 ? Wf[((size_t)nb * KB16 + kb) * 64 + l] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float x[4] = {v.x, v.y, v.z, v.w};
        unsigned hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float t = x[i] * sc.scale;
            const _Float16 a = (_Float16)t;
            nz += x[i] != 0.f;
            sm += x[i] != 0.f && fabsf(t) < kSplitSmall;
            hi[i] = half_bits(a);
            lo[i] = half_bits((_Float16)(t - (float)a));
        }
        const int k = 16 * kb + 4 * (l >> 4);
        uint16_t* const p = out + (((size_t)nb * KB32 + (k >> 5)) * 2 * 64 + r + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
        *reinterpret_cast<uint2*>(p) = make_uint2(hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16));
        *reinterpret_cast<uint2*>(p + 64 * 8) = make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
    }
    atomicAdd(&small[r], sm);
    atomicAdd(&nonzero[r], nz);
    __syncthreads();
    if (threadIdx.x < 16 && 16 * nb + r < rows) unscale[16 * nb + r] = split_unscale(sc, big[r], small[r], nonzero[r]);
}
size_t frag_split_halves(int rows, int cols) { return (size_t)((rows + 15) / 16) * ((cols + 31) / 32) * 1024; }
hipError_t launch_to_frag_split(const float* Wf, int rows, int cols, uint16_t* out, float* unscale, hipStream_t s)
{
    hipLaunchKernelGGL(to_frag_split_kernel, dim3((rows + 15) / 16), dim3(256), 0, s, (const float4*)Wf, rows, cols, out, unscale);
    return hipGetLastError();
}

}  // namespace l355
