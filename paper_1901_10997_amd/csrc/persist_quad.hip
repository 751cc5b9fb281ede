// Recurrence of a dense fp32 layer with the time loop on the device, LSTM and H-LSTM cells (paper Section 4, cell
// equations): the form an unpruned model takes, and the form a row/column-pruned model takes once it has been compacted.
// One launch per layer, every direction in the grid.
//
//   LSTM     a = P[t] + W_h . h_{t-1};                                        f,i,o = sigmoid, g = tanh;  c, h
//   H-LSTM   u_q = relu(P1[t]_q + W1h_q . h_{t-1});  a_q = W2_q . u_q + b2_q;  f,i,o = sigmoid, g = tanh;  c, h
//
// Batch columns are taken four at a time ("quads"): the 4x4x1 fp32 matrix instruction multiplies sixteen independent
// 4x1 by 1x4 blocks at the full fp32 matrix rate, so a batch of 4 wastes nothing, where the 16x16x4 form needs 16 columns
// to fill its rows.  Its first operand (h) can be broadcast over groups of blocks: with four blocks per group one
// instruction covers 16 weight rows x 4 columns x 4 k, one register of h (16 k x 4 columns) serves four instructions, and
// W_h sits in registers in the fragment order of pack time (16 rows x 16 k = 64 lanes x 16 bytes).
//
// A group of workgroups owns `mq` quads of one direction and all units; a workgroup owns 16 NT packed rows (4 NT units),
// its eight waves split K, KB blocks of 16 each, and the partial sums meet in LDS in a fixed order.  Only the workgroups
// of a group exchange data.  Where a group fits the compute units of one XCD (checked in the launch) it publishes
// through that XCD's L2: eight groups of 32 workgroups keep eight copies of W_h in the registers of the chip and no value
// crosses an XCD, which is what makes small column blocks pay.  A group with more than one quad takes them QP at a time,
// so that one exchange, one reduction and one round of gates serve all of them.
//
// Exchange: values carry their own readiness, as 32-bit words with one bit of the step count in a bit the value leaves
// free: |h| <= 1, so bit 30 (a NaN gets it back on reading, see unstamped); u >= 0, so the sign.  h has two buffers per
// quad, step tag g (2 for the first step) in buffer g & 1 with stamp (g >> 1) & 1; u one, stamped (s + 1) & 1.  All
// buffers are zero at launch.  u(s+1) is written only after its producer has received every h of step s, each of which
// was published after its workgroup had read all of u(s); a workgroup without a unit of h (G > H) publishes none that
// anybody could wait for, so it has no second product and never reads u.  (A form of the kernel of its own, SPARE: the
// branch in the loop costs narrow layers up to 2 % where no workgroup takes it, 74 units, both directions, batch 37: 1.99
// -> 2.02 us per step with its projection.)  h of tag g + 2 takes the place of tag g only after its producer has received
// every h of tag g + 1 and every u of that step; each workgroup owns units of at least one of the two and had read tag g
// before it published them.  A wave loads its own K slice straight into operand registers and repeats the load until
// every word is stamped (bounded).  Layouts of a quad, in the order of a wave's lanes (four columns apart in memory, a
// load would touch four times the lines): h [k][column]; u [k / 4][gate][column][k % 4], the operand order of the second
// product, whose sixteen blocks are four gates (each with its own u) x four k.
//
// Bound: the matrix instruction (8.8 clocks with two waves per SIMD issuing) plus one exchange per product plus the
// reduction and the gates.  Microseconds per step of the recurrence, both directions, batch 16: 256 units 1.89 -> 0.85,
// 800 units 4.8 -> 2.9 (against 16-column tiles of the 16x16x4 instruction across the device); H-LSTM 640/640 91 -> 4.4
// (against a launch per product).  LSTM layers of more than 256 units whose weights fit two fp16 planes run in
// persist_split.hip (800 units 2.90 -> 2.14); narrower ones are faster here (200 units 0.94 against 1.08).
#include "common.h"
#include "device_math.h"
#include "exchange.h"

namespace l355 {

namespace {
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
constexpr int kQW = 8, kQTH = 512;
constexpr unsigned kHBit = kHStampBit, kUBit = 0x80000000u;

// one fp32 word of a lane moved inside its 16-lane row
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// acc[i] of lane 16 g + r: column i, row r, k group g.  Returns in lane 16 i + r the sum over the four k groups.
__device__ __forceinline__ float quad_sum(const f32x4& a)
{
    const auto s02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[0]), __float_as_uint(a[2]), false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[1]), __float_as_uint(a[3]), false, false);
    const float k02 = __uint_as_float(s02[0]) + __uint_as_float(s02[1]);
    const float k13 = __uint_as_float(s13[0]) + __uint_as_float(s13[1]);
    const auto sr = __builtin_amdgcn_permlane16_swap(__float_as_uint(k02), __float_as_uint(k13), false, false);
    return __uint_as_float(sr[0]) + __uint_as_float(sr[1]);
}
// Counts a failed round of a bounded wait; true when the wait is to be given up.
__device__ __forceinline__ bool give_up(unsigned& spins, unsigned limit, int* flag)
{
    if (++spins > limit) {
        __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return (spins & 63u) == 0 && __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
}  // namespace

// NT: tiles of 16 packed rows per workgroup; KB: k blocks of 16 per wave; NL: of the NT tiles of the last product, those
// whose weights are in LDS instead of registers (a wave reads its own, 1 KB per tile and block: the shapes that would
// spill otherwise); HL: H-LSTM cell; QP: quads per pass
// SPARE: the last workgroups of a group own no unit of h (H-LSTM, G > H)
template <int NT, int KB, int NL, bool HL, int QP, bool SPARE>
__global__ __launch_bounds__(kQTH) void persist_quad_kernel(PersistQuadArgs a)
{
    constexpr int kItems = NT * QP;                          // (tile, quad) pairs of a pass, evaluated by a wave each
    constexpr int kMine = (kItems + kQW - 1) / kQW;          // ... at most so many by one wave
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float4* const wl = reinterpret_cast<float4*>(lds) + (size_t)(threadIdx.x >> 6) * NL * KB * 64 + (threadIdx.x & 63);   // [8][NL][KB][64]
    float* const part = lds + (size_t)kQW * NL * KB * 256;               // [2][8][QP][NT][64]
    float* const cell = part + 2 * kQW * kItems * 64;                    // [passes][QP][NT][64]
    const int H = a.H, G = a.G, gn = a.gn;
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

    // the direction is chosen by the block index, so its argument block lives in memory: fields copied once
    const PersistQuadDir& D = a.d[dir];
    const float* const Pd = D.P;
    const float* const h0 = D.h0;
    float* const y = D.y;
    const size_t y_ld = (size_t)D.y_ld;
    float* const hT = D.hT;
    float* const cT = D.cT;
    const int reverse = D.reverse;

    const int KBh = (H + 15) >> 4, KBg = (G + 15) >> 4;
    const bool owns_h = !SPARE || 4 * wg * NT < H;                       // of the whole workgroup
    // K blocks: waves 0..3, one per SIMD, take KB each; waves 4..7 KB or, where that covers K, one less
    const int hi = (KBh > KBg ? KBh : KBg) <= 8 * KB - 4 ? KB - 1 : KB;
    const int kb0 = wave < 4 ? wave * KB : 4 * KB + (wave - 4) * hi;
    const bool all_kb = wave < 4 || hi == KB;                            // wave-uniform
    const int rows1 = HL ? 4 * G : 4 * H;                                // packed rows of the first product

    // weights: loads from clamped addresses, what lies outside is zeroed afterwards
    constexpr int N1 = HL ? NT : NT - NL, N2 = HL ? NT - NL : 0;         // tiles of the products in registers
    float4 w1[N1][KB];
    {
        const float4* const Wf = reinterpret_cast<const float4*>(D.Wf);
        const int NB = (rows1 + 15) >> 4;
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const int nb = wg * NT + n, kb = kb0 + q;
                const bool ok = nb < NB && kb < KBh && (q < KB - 1 || all_kb);
                const float4 v = Wf[((size_t)(ok ? nb : 0) * KBh + (ok ? kb : 0)) * 64 + lane];
                const float4 z = ok ? v : make_float4(0.f, 0.f, 0.f, 0.f);
                if (n < N1) w1[n < N1 ? n : 0][q] = z;
                else wl[((n - N1) * KB + q) * 64] = z;
            }
    }
    float4 w2[N2 > 0 ? N2 : 1][HL ? KB : 1];
    if constexpr (HL) {
        const float4* const Wf = reinterpret_cast<const float4*>(D.W2f);
        const int NB = (H + 3) >> 2;
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const int nb = wg * NT + n, kb = kb0 + q;
                const bool ok = nb < NB && kb < KBg && (q < KB - 1 || all_kb);
                float4 v = Wf[((size_t)(ok ? nb : 0) * KBg + (ok ? kb : 0)) * 64 + lane];
                if (!ok) v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (n < N2) w2[n < N2 ? n : 0][q] = v;
                else wl[((n - N2) * KB + q) * 64] = v;
            }
    }

    // This thread's elements of the sums: item i = wave, wave + 8, .. of a pass is tile i % NT of quad i / NT; column lg of
    // the quad, row lr of the tile.  First product (and LSTM cell): row 4 (unit) + gate; H-LSTM gate outputs: row 4 (gate)
    // + unit.
    const int gate = HL ? (lr >> 2) : (lr & 3);
    int unit[kMine], qq[kMine];
    bool live[kMine];
    float b2[kMine];
#pragma unroll
    for (int j = 0; j < kMine; ++j) {
        const int i = wave + kQW * j;
        live[j] = i < kItems;                                            // wave-uniform
        qq[j] = live[j] ? i / NT : 0;
        const int n = live[j] ? i - qq[j] * NT : 0;
        unit[j] = 4 * (wg * NT + n) + (HL ? (lr & 3) : (lr >> 2));
        b2[j] = (HL && live[j] && unit[j] < H) ? D.bias2[4 * unit[j] + gate] : 0.f;
    }
    auto tile_of = [&](int j) { return wave + kQW * j - qq[j] * NT; };
    auto row1_of = [&](int j) { return 16 * (wg * NT + tile_of(j)) + lr; };
    // a pass may be short of quads
    auto have_quad = [&](int pass, int j) { return pass * QP + qq[j] < nq; };
    // batch column of item j; of a quad that the group does not have, none
    auto col_of = [&](int pass, int j) { return have_quad(pass, j) ? 4 * (q_lo + pass * QP + qq[j]) + lg : a.B; };
    // Quad c of a pass as an operand; one that is not there reads the last one that is (a condition on the load would make
    // the compiler wait for each): its products are never used.
    auto quad_of = [&](int pass, int c) { return pass * QP + c < nq ? pass * QP + c : nq - 1; };
    for (int pass = 0; pass < passes; ++pass)
#pragma unroll
        for (int j = 0; j < kMine; ++j)
            if (live[j]) {
                const int b = col_of(pass, j);
                cell[(pass * kItems + wave + kQW * j) * 64 + lane] = (D.c0 && b < a.B && unit[j] < H) ? D.c0[(size_t)b * H + unit[j]] : 0.f;
            }

    const size_t hquad = (size_t)KBh * 64, uquad = (size_t)KBg * 256;
    unsigned* const hx = a.hx + ((size_t)dir * a.quads + q_lo) * 2 * hquad;          // [quad][2][k][column]
    unsigned* const ux = HL ? a.ux + ((size_t)dir * a.quads + q_lo) * uquad : nullptr;
    const __amdgpu_buffer_rsrc_t uwords = exchange_buffer(ux, HL ? (unsigned)(nq * uquad * 4) : 0u);

    bool same_xcd = false;
    if (a.xcd_local)
        same_xcd = group_shares_xcd(a.xcc_ids + (size_t)(dir * a.groups + grp) * 64, gn, wg, 1u, part, tid, kQTH,
                                    a.timeout_flag, a.spin_limit) && !a.device_scope_only;

    // P and y: rows of the batch advance on the scalar side, the thread keeps its offset inside a timestep
    float p_next[kMine];
    auto load_p = [&](int s, int pass) {
        const int t = reverse ? a.T - 1 - s : s;
        const float* const Pt = Pd + (size_t)t * a.Bld * rows1;
#pragma unroll
        for (int j = 0; j < kMine; ++j) {
            const int b = col_of(pass, j), r = row1_of(j);
            p_next[j] = (live[j] && r < rows1 && b < a.B) ? Pt[(unsigned)(b * rows1 + r)] : 0.f;
        }
    };
    load_p(0, 0);
    float* part_w = part + (wave * kItems) * 64 + lane;  // where this wave's partial tiles go
    const float* part_r = part + wave * 64 + lane;       // this thread's first element of the first wave's tiles
    int flip = kQW * kItems * 64;                        // to the other buffer
    auto switch_buffers = [&]() { part_w += flip; part_r += flip; flip = -flip; };
    // sum of the workgroup's eight partial tiles for this thread's item j, after the workgroup's barrier
    auto gather_sum = [&](float start, int j) -> float {
        float sum = start;
#pragma unroll
        for (int w = 0; w < kQW; ++w) sum += part_r[(w * kItems + kQW * j) * 64];
        return sum;
    };
    auto put_partials = [&](const f32x4 (&acc)[QP][NT]) {
#pragma unroll
        for (int c = 0; c < QP; ++c)
#pragma unroll
            for (int n = 0; n < NT; ++n) part_w[(c * NT + n) * 64] = quad_sum(acc[c][n]);
    };
    auto finish_cell = [&](float pre, int s, int pass, int j) {
        const bool cand = gate == 3;
        const float rr = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f((cand ? 2.8853900817779268f : -1.4426950408889634f) * pre));
        const float gv = cand ? fmaf(-2.0f, rr, 1.0f) : rr;
        float f, ig, o, g;
        if constexpr (HL) {        // lanes 0..3 of a row: the gates of their unit are 4, 8 and 12 lanes up
            f = gv; ig = dpp_mov<0x104>(gv); o = dpp_mov<0x108>(gv); g = dpp_mov<0x10C>(gv);
        } else {                   // the four lanes of a quad
            f = dpp_mov<0x00>(gv); ig = dpp_mov<0x55>(gv); o = dpp_mov<0xAA>(gv); g = dpp_mov<0xFF>(gv);
        }
        float* const cp = cell + (pass * kItems + wave + kQW * j) * 64 + lane;
        const float c = fmaf(f, *cp, ig * g);
        const float h = o * tanhf_fast(c);
        const bool last = s == a.T - 1;
        const int b = col_of(pass, j);
        // columns beyond the batch are published as well (readers wait for every word; what such a column holds is never used)
        const bool mine = have_quad(pass, j) && unit[j] < H && (HL ? lr < 4 : gate == 0);
        if (mine && !last) {
            const unsigned tag = (unsigned)s + 2u;
            exchange_store(hx + ((size_t)(pass * QP + qq[j]) * 2 + (tag & 1u)) * hquad + (unsigned)(unit[j] * 4 + lg),
                           (__float_as_uint(h) & ~kHBit) | (((tag >> 1) & 1u) << 30), same_xcd);
        }
        *cp = c;
        // outputs after the publication: nothing on the way of h
        if (mine && b < a.B) {
            const int t = reverse ? a.T - 1 - s : s;
            (y + (size_t)t * a.Bld * y_ld)[(unsigned)(b * y_ld + unit[j])] = h;
            if (last) {
                if (hT) hT[(size_t)b * H + unit[j]] = h;
                if (cT) cT[(size_t)b * H + unit[j]] = c;
            }
        }
    };

    for (int s = 0; s < a.T; ++s) {
        for (int pass = 0; pass < passes; ++pass) {
            // ---- first product: operand words of h_{t-1}, one register per 16 k
            unsigned fr[QP][KB];
            if (s > 0) {
                const unsigned tag = (unsigned)s + 1u;
                const unsigned want = ((tag >> 1) & 1u) << 30;
                const unsigned* src[QP];
#pragma unroll
                for (int c = 0; c < QP; ++c) src[c] = hx + ((size_t)quad_of(pass, c) * 2 + (tag & 1u)) * hquad + lane;
                const bool tail_dead = 16 * (KBh - 1) + (lane >> 2) >= H;   // beyond the last unit: never written, stays zero
                pace_poll(a.poll_pace);
                unsigned spins = 0;
                for (;;) {
                    unsigned differ = 0;
                    // a block beyond K reads the last one again (its weights are zero)
#pragma unroll
                    for (int c = 0; c < QP; ++c)
#pragma unroll
                        for (int q = 0; q < KB; ++q)
                            fr[c][q] = __hip_atomic_load(src[c] + (kb0 + q < KBh ? kb0 + q : KBh - 1) * 64, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int c = 0; c < QP; ++c)
#pragma unroll
                        for (int q = 0; q < KB; ++q)
                            differ |= tail_dead && kb0 + q >= KBh - 1 ? 0u : fr[c][q] ^ want;
                    if (!__builtin_amdgcn_ballot_w64((differ & kHBit) != 0u) || give_up(spins, a.spin_limit, a.timeout_flag)) break;
                }
            } else {
#pragma unroll
                for (int c = 0; c < QP; ++c)
#pragma unroll
                    for (int q = 0; q < KB; ++q) {
                        const int b = 4 * (q_lo + quad_of(pass, c)) + (lane & 3), k = 16 * (kb0 + q) + (lane >> 2);
                        fr[c][q] = (h0 && b < a.B && k < H) ? __float_as_uint(h0[(size_t)b * H + k]) : 0u;
                    }
            }
            // this step's elements of P were requested a product ahead; behind the words just waited for they have arrived too
            // (taken over here by hand: at the top of the loop the wait for them would include the stores just issued)
            float p_cur[kMine];
#pragma unroll
            for (int j = 0; j < kMine; ++j) asm volatile("v_mov_b32 %0, %1" : "=v"(p_cur[j]) : "v"(p_next[j]));
            if (pass + 1 < passes) load_p(s, pass + 1);
            else if (s + 1 < a.T) load_p(s + 1, 0);
            f32x4 acc[QP][NT];
#pragma unroll
            for (int c = 0; c < QP; ++c)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[c][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (s > 0 || h0) {
                const unsigned strip = s > 0 ? kHBit : 0u;               // h0 is taken as it is
#pragma unroll
                for (int q = 0; q < KB; ++q)
                    if (q < KB - 1 || all_kb) {
                        float av[QP];
#pragma unroll
                        for (int c = 0; c < QP; ++c) av[c] = unstamped(fr[c][q], strip);
                        float4 w[NT];
#pragma unroll
                        for (int n = 0; n < NT; ++n) w[n] = n < N1 ? w1[n < N1 ? n : 0][q] : wl[((n - N1) * KB + q) * 64];
#define QUAD_MFMA(E_, A_)                                              \
    _Pragma("unroll") for (int c = 0; c < QP; ++c)                     \
        _Pragma("unroll") for (int n = 0; n < NT; ++n)                 \
            acc[c][n] = __builtin_amdgcn_mfma_f32_4x4x1f32(av[c], w[n].E_, acc[c][n], 2, A_, 0);
                        QUAD_MFMA(x, 0) QUAD_MFMA(y, 1) QUAD_MFMA(z, 2) QUAD_MFMA(w, 3)
#undef QUAD_MFMA
                    }
            }
            put_partials(acc);
            // one barrier per product: the partial tiles alternate between two buffers, and a wave that runs ahead reaches
            // the next barrier only after writing the other one
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kMine; ++j)
                if (live[j]) {
                    const float sum = gather_sum(p_cur[j], j);
                    if constexpr (HL) {
                        const float u = sum > 0.f ? sum : 0.f;
                        const int hu = row1_of(j) >> 2;                  // hidden unit; gate lr & 3
                        if (hu < G && have_quad(pass, j))
                            exchange_store(ux + (size_t)(pass * QP + qq[j]) * uquad + (unsigned)((hu >> 2) * 64 + 16 * (lr & 3) + 4 * lg + (hu & 3)),
                                           (__float_as_uint(u) & ~kUBit) | (((unsigned)s + 1u) << 31), same_xcd);
                    } else {
                        finish_cell(sum, s, pass, j);
                    }
                }
            switch_buffers();
        }
        if constexpr (HL) {
            for (int pass = 0; owns_h && pass < passes; ++pass) {
                // ---- second product: four gates x four k per instruction, one register of u each
                u32x4 fu[QP][KB];
                const unsigned want = ((unsigned)s + 1u) << 31;
                pace_poll(a.poll_pace);
                unsigned spins = 0;
                for (;;) {
                    asm volatile("" ::: "memory");                       // read anew in every round
#pragma unroll
                    for (int c = 0; c < QP; ++c)
#pragma unroll
                        for (int q = 0; q < KB; ++q)
                            fu[c][q] = exchange_load16<u32x4>(uwords, lane * 16, quad_of(pass, c) * (int)uquad * 4 + (kb0 + q < KBg ? kb0 + q : KBg - 1) * 1024);
                    __builtin_amdgcn_sched_barrier(0);                   // all on their way before the first is waited for
                    unsigned differ = 0;
#pragma unroll
                    for (int c = 0; c < QP; ++c)
#pragma unroll
                        for (int q = 0; q < KB; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const bool dead = kb0 + q >= KBg - 1 && 16 * (KBg - 1) + 4 * lg + e >= G;
                                differ |= dead ? 0u : fu[c][q][e] ^ want;
                            }
                    if (!__builtin_amdgcn_ballot_w64((differ & kUBit) != 0u) || give_up(spins, a.spin_limit, a.timeout_flag)) break;
                }
                f32x4 acc[QP][NT];
#pragma unroll
                for (int c = 0; c < QP; ++c)
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[c][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < KB; ++q)
                    if (q < KB - 1 || all_kb) {
                        float4 w[NT];
#pragma unroll
                        for (int n = 0; n < NT; ++n) w[n] = n < N2 ? w2[n < N2 ? n : 0][q] : wl[((n - N2) * KB + q) * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int c = 0; c < QP; ++c) {
                                const float av = __uint_as_float(fu[c][q][e] & ~kUBit);
#pragma unroll
                                for (int n = 0; n < NT; ++n)
                                    acc[c][n] = __builtin_amdgcn_mfma_f32_4x4x1f32(av, e == 0 ? w[n].x : e == 1 ? w[n].y : e == 2 ? w[n].z : w[n].w,
                                                                                   acc[c][n], 0, 0, 0);
                            }
                    }
                put_partials(acc);
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kMine; ++j)
                    if (live[j]) finish_cell(gather_sum(b2[j], j), s, pass, j);
                switch_buffers();
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- shapes and launch
namespace {
struct QuadShape {
    int nt, kb, nl;
    bool hl;
    int qp;
    const void *kernel, *spare_kernel;   // SPARE = false, true
};
#define Q_L(NT_, KB_, NL_, QP_) {NT_, KB_, NL_, false, QP_, (const void*)persist_quad_kernel<NT_, KB_, NL_, false, QP_, false>, nullptr}
#define Q_H(NT_, KB_, NL_, QP_)                                                                       \
    {NT_, KB_, NL_, true, QP_, (const void*)persist_quad_kernel<NT_, KB_, NL_, true, QP_, false>,     \
     (const void*)persist_quad_kernel<NT_, KB_, NL_, true, QP_, true>}
// the shapes whose weights (NT KB float4 per lane and product), operand words and accumulators fit the registers
const QuadShape kQuadShapes[] = {
    Q_L(1, 1, 0, 1), Q_L(1, 2, 0, 1), Q_L(2, 2, 0, 1), Q_L(1, 3, 0, 1), Q_L(2, 3, 0, 1), Q_L(3, 3, 0, 1), Q_L(1, 4, 0, 1),
    Q_L(2, 4, 0, 1), Q_L(4, 4, 0, 1), Q_L(1, 5, 0, 1), Q_L(2, 5, 0, 1), Q_L(3, 5, 0, 1), Q_L(5, 5, 0, 1), Q_L(1, 6, 0, 1),
    Q_L(2, 6, 0, 1), Q_L(3, 6, 0, 1), Q_L(6, 6, 0, 1), Q_L(1, 7, 0, 1), Q_L(2, 7, 0, 1), Q_L(4, 7, 0, 1), Q_L(7, 7, 1, 1),
    Q_L(1, 8, 0, 1), Q_L(2, 8, 0, 1), Q_L(4, 8, 0, 1), Q_L(5, 8, 0, 1), Q_L(2, 10, 0, 1), Q_L(3, 10, 0, 1),
    Q_L(4, 10, 0, 1), Q_L(2, 12, 0, 1), Q_L(3, 12, 0, 1), Q_L(2, 16, 0, 1),
    Q_L(1, 1, 0, 2), Q_L(1, 2, 0, 2), Q_L(2, 2, 0, 2), Q_L(1, 3, 0, 2), Q_L(2, 3, 0, 2), Q_L(3, 3, 0, 2), Q_L(1, 4, 0, 2),
    Q_L(2, 4, 0, 2), Q_L(4, 4, 0, 2), Q_L(1, 5, 0, 2), Q_L(2, 5, 0, 2), Q_L(3, 5, 0, 2), Q_L(5, 5, 0, 2), Q_L(1, 6, 0, 2),
    Q_L(2, 6, 0, 2), Q_L(3, 6, 0, 2), Q_L(1, 7, 0, 2), Q_L(2, 7, 0, 2), Q_L(4, 7, 0, 2), Q_L(1, 8, 0, 2), Q_L(2, 8, 0, 2),
    Q_L(4, 8, 0, 2), Q_L(2, 10, 0, 2), Q_L(3, 10, 0, 2), Q_L(2, 12, 0, 2),
    Q_L(4, 1, 0, 1), Q_L(4, 1, 0, 2), Q_L(4, 1, 0, 4), Q_L(1, 1, 0, 4), Q_L(4, 2, 0, 1), Q_L(4, 2, 0, 2), Q_L(4, 2, 0, 4),
    Q_L(2, 2, 0, 4), Q_L(6, 3, 0, 1), Q_L(6, 3, 0, 2), Q_L(3, 3, 0, 4), Q_L(7, 4, 0, 1), Q_L(4, 4, 0, 4),
    Q_H(1, 1, 0, 1), Q_H(1, 2, 0, 1), Q_H(2, 2, 0, 1), Q_H(1, 3, 0, 1), Q_H(3, 3, 0, 1), Q_H(1, 4, 0, 1), Q_H(2, 4, 0, 1),
    Q_H(4, 4, 0, 1), Q_H(1, 5, 0, 1), Q_H(2, 5, 0, 1), Q_H(5, 5, 2, 1), Q_H(1, 6, 0, 1), Q_H(2, 6, 0, 1), Q_H(3, 6, 0, 1),
    Q_H(1, 7, 0, 1), Q_H(2, 7, 0, 1), Q_H(4, 7, 2, 1), Q_H(1, 8, 0, 1), Q_H(2, 8, 0, 1), Q_H(2, 10, 1, 1),
    Q_H(2, 12, 1, 1), Q_H(1, 16, 1, 1),
    Q_H(1, 1, 0, 2), Q_H(1, 2, 0, 2), Q_H(2, 2, 0, 2), Q_H(1, 3, 0, 2), Q_H(3, 3, 0, 2), Q_H(1, 4, 0, 2), Q_H(2, 4, 0, 2),
    Q_H(4, 4, 0, 2), Q_H(1, 5, 0, 2), Q_H(2, 5, 0, 2), Q_H(1, 6, 0, 2), Q_H(2, 6, 0, 2), Q_H(1, 7, 0, 2), Q_H(2, 7, 0, 2),
    Q_H(1, 8, 0, 2),
};
#undef Q_L
#undef Q_H
constexpr int kQuadShapeCount = (int)(sizeof(kQuadShapes) / sizeof(kQuadShapes[0]));
}  // namespace

// Shape, quads per group and placement of the lowest estimated step time in microseconds: per pass and product a fixed
// part, the matrix instructions, the reduction and gates of a (tile, quad) pair; the operand words; and the part of the
// exchange that other passes would hide.  The constants are a fit to 700 measured (shape, groups, placement) points over
// 100 to 1900 units and batches of 1 to 64 (standard error 12 %, which the choice needs only near ties).
// H-LSTM steps have become shorter since (operand words of the second product sixteen bytes per lane): 0.74 of that fit over 180 layers of
// 64 to 2000 units and batches of 2 to 64, a step of 60 without the 5 us that a launch takes to its first one (0.65 to 0.83 in eight of
// ten), alike inside an XCD and across, so the shapes rank as they did.
PersistQuadPlan persist_quad_plan(int B, int H, int G, int ndir)
{
    PersistQuadPlan best;
    if (B < 1 || H < 1 || G < 0 || ndir < 1 || ndir > 2) return best;
    const bool hl = G > 0;
    const int kblocks = std::max((H + 15) / 16, (G + 15) / 16);
    const int tiles = std::max((H + 3) / 4, (G + 3) / 4);
    const int quads = (B + 3) / 4, cus = device_num_cus();
    const int stages = hl ? 2 : 1;
    for (int i = 0; i < kQuadShapeCount; ++i) {
        const QuadShape& sh = kQuadShapes[i];
        if (sh.hl != hl || sh.kb * kQW < kblocks) continue;
        const int gn = (tiles + sh.nt - 1) / sh.nt;
        // (more groups than that fit neither way, so the loop ends there whatever the batch)
        for (int groups = 1; groups <= quads && ndir * groups * gn <= cus; ++groups) {
            const int mq = (quads + groups - 1) / groups;
            if ((quads + mq - 1) / mq != groups) continue;   // a group would be left without a quad
            const int passes = (mq + sh.qp - 1) / sh.qp;
            if (sh.qp > 1 && 2 * mq <= sh.qp) continue;      // half of every pass would be empty
            const size_t lds = ((size_t)kQW * sh.nl * sh.kb * 256 + (size_t)(2 * kQW + passes) * sh.qp * sh.nt * 64) * sizeof(float);
            if (lds > 160 * 1024) continue;
            const int per_xcd = (ndir * groups + 7) / 8;
            const int local = gn <= 64 && per_xcd * gn <= cus / 8;
            const double words_kb = (16.0 * H + 64.0 * G) / 1e3;             // operand words of a quad and step
            const double pass = stages * ((local ? 0.42 : 0.63) + 0.0097 * sh.qp * sh.nt * sh.kb * 4 + 0.045 * sh.qp * sh.nt) + 0.033 * sh.qp * words_kb;
            const double us = (hl ? 0.74 : 1.0) * (passes * pass + (passes == 1 ? stages * (local ? 0.29 : 0.59) : 0.0));
            if (us < best.us) {
                best.us = us;
                best.shape = i;
                best.mq = mq; best.groups = groups; best.gn = gn; best.xcd_local = local; best.lds = lds;
            }
        }
    }
    return best;
}

// Time of a step of an LSTM plan where many columns meet a narrow layer: a fit to 700 measured points of 16 to 512 units and 80
// to 4096 columns (standard error 8 %), with the terms that the choice of a shape can do without (groups that share an XCD's
// L2, more items of a pass than waves).  persist_quad_plan's own model is up to 40 % low there.
double persist_quad_many_columns_us(const PersistQuadPlan& p, int H, int ndir)
{
    const QuadShape& sh = kQuadShapes[p.shape];
    const int items = sh.qp * sh.nt, passes = (p.mq + sh.qp - 1) / sh.qp;
    const double pass = 0.50 + (p.xcd_local ? 0.0 : 0.10) + 0.0073 * items * sh.kb * 4 + 0.048 * items + 0.023 * std::max(0, items - 8) +
                        0.023 * sh.qp * 16e-3 * H + 0.030 * sh.qp * ((ndir * p.groups + 7) / 8);
    return passes * pass + (passes == 1 ? 0.35 : 0.0);
}

// exchange words of one launch: h, then u, then (8-byte) XCD id slots of the groups
static size_t quad_h_words(int B, int H, int ndir) { return (size_t)ndir * ((B + 3) / 4) * 8 * ((H + 15) / 16) * 16; }
static size_t quad_u_words(int B, int G, int ndir) { return (size_t)ndir * ((B + 3) / 4) * ((G + 15) / 16) * 256; }
size_t persist_quad_exchange_words(int B, int H, int G, int ndir)
{
    return quad_h_words(B, H, ndir) + quad_u_words(B, G, ndir) + (size_t)ndir * ((B + 3) / 4) * 64 * 2;
}

void persist_quad_describe(const PersistQuadPlan& p, char* buf, size_t n)
{
    const QuadShape& sh = kQuadShapes[p.shape];
    std::snprintf(buf, n, "(t%d,k%d,q%d,%dx%d%s)", sh.nt, sh.kb, sh.qp, p.groups, p.mq, p.xcd_local ? ",xcd" : "");
}

// p: the plan of (a.B, a.H, a.G, a.ndir); words: the launch's exchange region, all zero
hipError_t launch_persist_quad(PersistQuadArgs& a, const PersistQuadPlan& p, unsigned* words, bool cooperative, hipStream_t s)
{
    if (a.B <= 0 || a.H <= 0 || a.T <= 0) return hipSuccess;
    if (p.shape < 0) return hipErrorInvalidValue;
    const QuadShape& sh = kQuadShapes[p.shape];
    const void* const kernel = a.G > 0 && 4 * sh.nt * (p.gn - 1) >= a.H ? sh.spare_kernel : sh.kernel;
    a.quads = (a.B + 3) / 4;
    a.mq = p.mq; a.groups = p.groups; a.gn = p.gn; a.xcd_local = p.xcd_local;
    if (p.xcd_local || p.mq > sh.qp) a.poll_pace = 0;   // visible by the time the first read arrives, or other passes in between
    a.hx = words;
    a.ux = words + quad_h_words(a.B, a.H, a.ndir);
    a.xcc_ids = (unsigned long long*)(a.ux + quad_u_words(a.B, a.G, a.ndir));
    const int grid = p.xcd_local ? 8 * ((a.ndir * p.groups + 7) / 8) * p.gn : a.ndir * p.groups * p.gn;
    // every workgroup must be resident at the same time: at most one per compute unit
    if (grid > device_num_cus()) return hipErrorCooperativeLaunchTooLarge;
    if (p.lds > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(kernel, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    void* kargs[] = {(void*)&a};
    if (cooperative) return hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(kQTH), kargs, (unsigned)p.lds, s);
    return hipLaunchKernel(kernel, dim3(grid), dim3(kQTH), kargs, p.lds, s);
}

// A row-major fp32 matrix W[rows][cols] in the fragment order of the 16-row matrix instructions: tile (nb, kb) is 64 lanes x
// 4 values, lane l holding W[16 nb + r][16 kb + 4 (l / 16) .. + 3] with r = l % 16, or, by_gate, r = 4 (l % 4) + (l / 4) % 4
// (rows 4 unit + gate taken gate by gate: the second product of the H-LSTM); zero beyond the matrix.
__global__ __launch_bounds__(256) void to_frag16_kernel(const float* __restrict__ W, int rows, int cols, int by_gate, float4* __restrict__ out)
{
    const int KB = (cols + 15) >> 4;
    const size_t total = (size_t)((rows + 15) >> 4) * KB * 64;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int l = (int)(i & 63);
        const size_t tile = i >> 6;
        const int r = by_gate ? 4 * (l & 3) + ((l >> 2) & 3) : (l & 15);
        const int n = 16 * (int)(tile / KB) + r, k = 16 * (int)(tile % KB) + 4 * (l >> 4);
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = (n < rows && k + c < cols) ? W[(size_t)n * cols + k + c] : 0.f;
        out[i] = make_float4(v[0], v[1], v[2], v[3]);
    }
}
size_t frag16_floats(int rows, int cols) { return (size_t)((rows + 15) / 16) * ((cols + 15) / 16) * 256; }
hipError_t launch_to_frag16(const float* W, int rows, int cols, bool by_gate, float* out, hipStream_t s)
{
    const size_t g = (frag16_floats(rows, cols) / 4 + 255) / 256;
    hipLaunchKernelGGL(to_frag16_kernel, dim3((unsigned)std::min<size_t>(g, 8192)), dim3(256), 0, s, W, rows, cols, by_gate ? 1 : 0, (float4*)out);
    return hipGetLastError();
}

// The same copy of a masked matrix from its row-compressed form: out is zero, a wave per row puts the kept entries in place.
__global__ __launch_bounds__(256) void csr_to_frag16_kernel(const int* __restrict__ row_ptr, const uint16_t* __restrict__ col, const float* __restrict__ val,
                                                            int rows, int KB, int by_gate, float* __restrict__ out)
{
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= rows) return;
    const int r = n & 15, l = by_gate ? (r >> 2) | ((r & 3) << 2) : r;
    for (int e = row_ptr[n] + (threadIdx.x & 63); e < row_ptr[n + 1]; e += 64) {
        const int k = col[e];
        out[(((size_t)(n >> 4) * KB + (k >> 4)) * 64 + 16 * ((k & 15) >> 2) + l) * 4 + (k & 3)] = val[e];
    }
}
hipError_t launch_csr_to_frag16(const int* row_ptr, const uint16_t* col, const float* val, int rows, int cols, bool by_gate, float* out, hipStream_t s)
{
    const hipError_t e = launch_fill_f32(out, frag16_floats(rows, cols), 0.0f, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(csr_to_frag16_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, row_ptr, col, val, rows, (cols + 15) / 16, by_gate ? 1 : 0, out);
    return hipGetLastError();
}

}  // namespace l355
