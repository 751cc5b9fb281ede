// Recurrence of a bf16 dense layer with the time loop on the device, any width up to 2048 and any batch from 2 (paper
// Section 4, cell equations): serving batches, widths that row/column pruning leaves behind, and the wide layers that the
// 32-row tiles of persist_mfma.hip do not take.  One launch per layer, every direction in the grid.
//
//   R[b][n] = sum_k hb[b][k] * W_h[n][k]      (hb = h_{t-1} rounded to bf16, W_h packed rows n = 4 * unit + gate)
//   a = P[t][b][n] + R[b][n];  f,i,o = sigmoid, g = tanh;  c <- f*c + i*g;  h = o*tanh(c)
//
// A group of workgroups owns up to R batch rows of one direction and all units; a workgroup owns 16 NT packed rows (4 NT
// units), its eight waves split K, KB blocks of 32 each, with their slices of W_h in registers in the operand order of the
// 16x16x32 matrix instruction (fragment-ordered at pack time).  Rows are taken 16 at a time; the partial tiles meet in
// LDS and are summed in a fixed order.  Groups are the only workgroups that exchange data; where they fit one XCD each
// they hand h over through its L2 (checked in the launch).  A batch of 2 to 16 rows per group costs the same matrix work,
// so the batch is dealt over as many groups as fit, which makes each group's h, the volume every workgroup reads per step,
// small.
//
// Exchange: |h| <= 1 leaves bit 14 of a bf16 pattern free (a NaN gets it back on reading, see unstamped); it carries one
// bit of the step count (step tag g, 2 for the first step, in buffer g & 1 with stamp (g >> 1) & 1; both buffers zero at
// launch).  h lies in operand order, [k / 8][row][8], so a wave loads 16 bytes per lane straight into operand registers
// and repeats the load until every live element is stamped (bounded); a tile publishes the 4 units of a row as one 8-byte
// word.  A workgroup writes h_t after all of its waves have read h_{t-1} (barrier), and each of those was published after
// its workgroup had read h_{t-2} from the buffer h_t goes to.
//
// A stack (STACK): consecutive layers of one width and direction run in one launch, each with workgroups of its own, so that n layers
// take T + n - 1 steps instead of n T.  A layer above the first keeps W_x beside W_h (the last blocks in LDS where the registers do
// not hold both), multiplies its input while its own h travels and adds its bias; no projection of it is launched.  h of every step
// goes to a buffer of that step as well (device scope, behind the publication: nobody overwrites it, so no layer waits for the one
// above), stamped alike; the words of the next step are requested behind a step's products.
//
// Operand words are read 16 bytes per lane (exchange_load16): as pairs of 8-byte loads every line was asked for twice, and the
// requests bounded the step (1197 units, batch 20 2.33 -> 2.07 us, in a stack 4.7 -> 3.3).
//
// Bound: the exchange and the chain around it.  Microseconds per step of one layer of 1197 units, batch 20: 18.8 with a launch per
// step, 2.1 here; of 1024, batch 64 3.7 with the 32-row tiles, 2.2 here.  Two layers of 1197, batch 20, 70 steps: 388 us one after
// the other with 8-byte loads, 335 with 16, 262 as a stack; four of 512 474 and 186.
#include "common.h"
#include "device_math.h"
#include "exchange.h"

namespace l355 {

namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
constexpr int kRW = 8, kRTH = 512;
constexpr unsigned kStamp = 0x40004000u;                                 // of two values
constexpr unsigned long long kStamps = 0x4000400040004000ull;            // of four

template <int CTRL>
__device__ __forceinline__ float dpp_mov_f(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// Four published values without their stamps.  A NaN has bit 14 set itself and |h| <= 1 else: without that bit a (quiet) NaN is
// a pattern of at least 0x3FC0 (1.5), from which the addition carries into bit 14 again.  The halves apart: 32-bit operations.
// strip: kStamp, or 0 to take the values as they are.
__device__ __forceinline__ unsigned unstamped_pair(unsigned v, unsigned strip)
{
    const unsigned carried = (v & 0x3FFF3FFFu) + 0x00400040u;
    return (v & ~strip) | (carried & strip);
}
__device__ __forceinline__ unsigned long long unstamped(unsigned long long v, unsigned strip)
{
    return (unsigned long long)unstamped_pair((unsigned)(v >> 32), strip) << 32 | unstamped_pair((unsigned)v, strip);
}
// Scalar base and 32-bit lane offset in bytes (an index would be taken for up to 34 bits, and the addresses for lane values).
template <class T>
__device__ __forceinline__ T* at_bytes(T* base, unsigned bytes) { return (T*)((char*)base + bytes); }
template <class T>
__device__ __forceinline__ const T* at_bytes(const T* base, unsigned bytes) { return (const T*)((const char*)base + bytes); }
// Lanes 4j..4j+3 hold gates 0..3 of a unit, v[b] for batch rows b = 0..3: afterwards lane 4j + q holds in v[g] gate g of row q.
__device__ __forceinline__ void quad_transpose(float (&v)[4], int lane)
{
    const bool odd = (lane & 1) != 0, hi = (lane & 2) != 0;
    float r0 = dpp_mov_f<0xB1>(odd ? v[0] : v[1]), r1 = dpp_mov_f<0xB1>(odd ? v[2] : v[3]);
    v[0] = odd ? r0 : v[0];
    v[1] = odd ? v[1] : r0;
    v[2] = odd ? r1 : v[2];
    v[3] = odd ? v[3] : r1;
    r0 = dpp_mov_f<0x4E>(hi ? v[0] : v[2]);
    r1 = dpp_mov_f<0x4E>(hi ? v[1] : v[3]);
    v[0] = hi ? r0 : v[0];
    v[1] = hi ? r1 : v[1];
    v[2] = hi ? v[2] : r0;
    v[3] = hi ? v[3] : r1;
}
}  // namespace

// NT: tiles of 16 packed rows per workgroup; KB: k blocks of 32 per wave; RT: sixteens of batch rows per pass; STACK: the
// "directions" are consecutive layers; XL: k blocks of their W_x per wave that are in LDS
template <int NT, int KB, int RT, bool STACK, int XL>
__global__ __launch_bounds__(kRTH) void persist_rows_bf16_kernel(PersistRowsArgs a)
{
    static_assert(NT * RT <= 8, "one (tile, four rows) item per 16-lane row");
    constexpr int kRows = 16 * RT, kTiles = RT * NT;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    f32x4* const part = reinterpret_cast<f32x4*>(lds);                               // [2][8][RT][NT][64]
    float* const cell = lds + (size_t)2 * kRW * kTiles * 256;                        // [passes][512]
    const int H = a.H, B = a.B, gn = a.gn;
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
    const int R = a.rows;                                                // rows per group (stride of the exchange layout)
    const int b_lo = grp * R;
    const int rows = B - b_lo < R ? B - b_lo : R;                        // >= 1 (checked by the launcher)
    const int passes = (rows + kRows - 1) / kRows;

    // the direction is chosen by the block index, so its argument block lives in memory: fields copied once
    const PersistRowsDir& D = a.d[dir];
    const float* const Pd = D.P;
    float* const y = D.y;
    uint16_t* const yb = D.yb;
    const size_t y_ld = (size_t)D.y_ld, yb_ld = (size_t)D.yb_ld;
    float* const hT = D.hT;
    float* const cT = D.cT;
    const int reverse = D.reverse;

    const int KBt = (H + 31) >> 5, tiles = (H + 3) >> 2;
    const int kb0 = wave * KB;
    // weights: loads from clamped addresses, what lies outside is zeroed afterwards
    auto weight = [&](const uint16_t* from, int n, int q) {
        const int nb = wg * NT + n, kb = kb0 + q;
        const bool ok = nb < tiles && kb < KBt;
        const uint4 v = reinterpret_cast<const uint4*>(from)[((size_t)(ok ? nb : 0) * KBt + (ok ? kb : 0)) * 64 + lane];
        return ok ? v : make_uint4(0u, 0u, 0u, 0u);
    };
    uint4 w[NT][KB];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int q = 0; q < KB; ++q) w[n][q] = weight(D.Wf, n, q);
    const bool upper = STACK && dir > 0, feeds = STACK && dir + 1 < a.ndir;   // of the whole workgroup
    constexpr int KX = KB - XL;                                          // blocks of W_x in registers
    uint4 wx[STACK ? NT : 1][STACK ? KX : 1];
    uint4* const wxl = reinterpret_cast<uint4*>(cell + (size_t)passes * kRTH) + (size_t)wave * XL * NT * 64 + lane;   // [8][XL][NT][64]
    if constexpr (STACK)
        if (upper) {
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    const uint4 v = weight(D.Wxf, n, q);
                    if (q < KX) wx[n][q < KX ? q : 0] = v;
                    else wxl[((q - KX) * NT + n) * 64] = v;
                }
        }

    unsigned long long* const hx = a.hx + ((size_t)dir * a.groups + grp) * 2 * ((size_t)KBt * 8 * R);   // [2][k / 8][row][2] words
    const size_t xbuf = (size_t)KBt * 8 * R;
    const bool has_h0 = D.h0x != nullptr;
    const unsigned long long* const h0x = has_h0 ? D.h0x + grp * xbuf : hx;   // (without h0 the first step's words are not used)
    // h of every step for the layer above, [T] of the same; of the layer below
    unsigned long long* const seq = STACK ? a.seq + ((size_t)dir * a.groups + grp) * a.T * xbuf : nullptr;
    const unsigned long long* const below = STACK ? a.seq + ((size_t)(dir - (upper ? 1 : 0)) * a.groups + grp) * a.T * xbuf : nullptr;

    // This thread's 16-lane row serves tile `tile`, batch rows row4 .. + 3 of a pass: packed row lr of the tile while the sums
    // are gathered, unit lr / 4 and batch row lr % 4 from the cell update on.
    const int item = wave * 4 + lg, tile = item % NT, row4 = 4 * (item / NT);
    const int tl = wg * NT + tile, unit = 4 * tl + (lr >> 2), col = 16 * tl + lr;
    for (int pass = 0; pass < passes; ++pass) {
        const int r = pass * kRows + row4 + (lr & 3);
        cell[pass * kRTH + tid] = (D.c0 && row4 < kRows && r < rows && unit < H) ? D.c0[(size_t)(b_lo + r) * H + unit] : 0.f;
    }

    bool same_xcd = false;
    if (a.xcd_local)
        same_xcd = group_shares_xcd(a.xcc_ids + (size_t)(dir * a.groups + grp) * 64, gn, wg, 1u, lds, tid, kRTH,
                                    a.timeout_flag, a.spin_limit) && !a.device_scope_only;

    // P of the item's four rows: unconditional loads (clamped), requested a pass ahead; an upper layer adds its bias
    float p_next[4];
    if (STACK && upper) {
        const float b = D.P[col < 4 * H ? col : 0];
#pragma unroll
        for (int v = 0; v < 4; ++v) p_next[v] = b;
    }
    auto load_p = [&](int s, int pass) {
        if (STACK && upper) return;
        const int t = reverse ? a.T - 1 - s : s;
        const float* const Pt = Pd + ((size_t)t * B + b_lo) * (size_t)(4 * H);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = pass * kRows + row4 + v;
            p_next[v] = *at_bytes(Pt, (unsigned)((r < rows ? r : rows - 1) * 4 * H + (col < 4 * H ? col : 0)) * 4u);
        }
    };
    load_p(0, 0);
    int buf = 0;
    // operand words from the [k / 8][row][2] words at src, two of four k per lane and block; a row that is not there reads the last
    // one (never used), a block beyond K the last one again (its weights are zero)
    auto fetch = [&](u64x2 (&fr)[RT][KB], const unsigned long long* src, int pass) {
        asm volatile("" ::: "memory");                                   // read anew by every call
        const __amdgpu_buffer_rsrc_t from = exchange_buffer(src, (unsigned)xbuf * 8u);
#pragma unroll
        for (int c = 0; c < RT; ++c) {
            const int r = pass * kRows + 16 * c + lr;
            const int off = (lg * R + (r < rows ? r : rows - 1)) * 16;
#pragma unroll
            for (int q = 0; q < KB; ++q) fr[c][q] = exchange_load16<u64x2>(from, off, (kb0 + q < KBt ? kb0 + q : KBt - 1) * 64 * R);
        }
        __builtin_amdgcn_sched_barrier(0);                               // all on their way before the first is waited for
    };
    // does an element lack the stamp `want`?
    auto stale = [&](const u64x2 (&fr)[RT][KB], unsigned want) {
        unsigned differ = 0;
#pragma unroll
        for (int c = 0; c < RT; ++c)
#pragma unroll
            for (int q = 0; q < KB; ++q)
                differ |= ((unsigned)fr[c][q].x ^ want) | ((unsigned)(fr[c][q].x >> 32) ^ want) | ((unsigned)fr[c][q].y ^ want) |
                          ((unsigned)(fr[c][q].y >> 32) ^ want);
        return __builtin_amdgcn_ballot_w64((differ & kStamp) != 0u) != 0ull;
    };
    // counts a failed round of a bounded wait; true when the wait is to be given up
    auto give_up = [&](unsigned& spins) {
        if (++spins > a.spin_limit) {
            __hip_atomic_store(a.timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        return (spins & 63u) == 0 && __hip_atomic_load(a.timeout_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    };
    auto multiply = [&](f32x4 (&acc)[RT][NT], const u64x2 (&fr)[RT][KB], auto by, unsigned strip) {
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            bf16x8 b[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) b[n] = __builtin_bit_cast(bf16x8, by(n, q));
#pragma unroll
            for (int c = 0; c < RT; ++c) {
                u64x2 v = fr[c][q];
                v.x = unstamped(v.x, strip);
                v.y = unstamped(v.y, strip);
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[c][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), b[n], acc[c][n], 0, 0, 0);
            }
        }
    };
    u64x2 xr[RT][KB];                                                    // upper layers: the next pass's input, requested a pass ahead
    if (STACK && upper) fetch(xr, below, 0);
    // The lanes of a tile's row publish four units of four batch rows in lanes 0..3; behind the last tile the others publish zeros for
    // the units that fill up K's last block, so that readers find a stamp on every word (a store of its own for these made the step
    // of 1197 units 4 % longer).
    const int pad_words = 8 * KBt - tiles;
    const bool puts = lr < 4 ? tl < tiles : tl == tiles - 1 && (lr >> 2) <= pad_words;
    const bool puts_more = tl == tiles - 1 && 4 + (lr >> 2) <= pad_words;
    const int pad0 = 4 * tiles, pads = yb ? (D.yb_width - pad0) >> 2 : 0;   // columns of yb behind the last tile, in fours

    for (int s = 0; s < a.T; ++s) {
        const int t = reverse ? a.T - 1 - s : s;
        const bool last = s == a.T - 1;
        for (int pass = 0; pass < passes; ++pass) {
            f32x4 acc[RT][NT];
#pragma unroll
            for (int c = 0; c < RT; ++c)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[c][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if constexpr (STACK)
                if (upper) {
                    // ---- the input's product, while h_{t-1} travels
                    for (unsigned spins = 0; stale(xr, kStamp) && !give_up(spins);) fetch(xr, below + (size_t)s * xbuf, pass);
                    multiply(acc, xr, [&](int n, int q) { return q < KX ? wx[n][q < KX ? q : 0] : wxl[((q - KX) * NT + n) * 64]; }, kStamp);
                }
            // ---- operand fragments of h_{t-1}
            u64x2 fr[RT][KB];
            const unsigned tag = (unsigned)s + 1u, want = ((tag >> 1) & 1u) ? kStamp : 0u;
            const unsigned long long* const src = s > 0 ? hx + (tag & 1u) * xbuf : h0x;
            if (s > 0 && !upper) pace_poll(a.poll_pace);
            unsigned spins = 0;
            do fetch(fr, src, pass);
            while (stale(fr, want) && s > 0 && !give_up(spins));       // (looked at in the first step too: a load still on its way would make later waits longer)
            // the pass's elements of P were requested a pass ahead; behind the words just waited for they have arrived too
            // (taken over here by hand: at the top of the loop the wait for them would include the stores just issued)
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) asm volatile("v_mov_b32 %0, %1" : "=v"(v[e]) : "v"(p_next[e]));
            if (pass + 1 < passes) load_p(s, pass + 1);
            else if (!last) load_p(s + 1, 0);
            if (s > 0 || has_h0) multiply(acc, fr, [&](int n, int q) { return w[n][q]; }, s > 0 ? kStamp : 0u);   // h0 is taken as it is
            if constexpr (STACK)
            {
                if (upper && !(last && pass + 1 == passes)) {
                    if (pass + 1 < passes) fetch(xr, below + (size_t)s * xbuf, pass + 1);
                    else fetch(xr, below + (size_t)(s + 1) * xbuf, 0);
                } else {
                    // not used any more: without this the old values stay in registers beside h's
#pragma unroll
                    for (int c = 0; c < RT; ++c)
#pragma unroll
                        for (int q = 0; q < KB; ++q) asm volatile("" : "=v"(xr[c][q].x), "=v"(xr[c][q].y));
                }
            }
            // partial tiles -> LDS: lane l of an accumulator holds batch rows 4 (l / 16) .. + 3 of packed row l % 16
            f32x4* const mine = part + ((size_t)(buf * kRW + wave) * kTiles) * 64 + lane;
#pragma unroll
            for (int c = 0; c < RT; ++c)
#pragma unroll
                for (int n = 0; n < NT; ++n) mine[(c * NT + n) * 64] = acc[c][n];
            // one barrier per pass: the partial tiles alternate between two buffers, and a wave that runs ahead reaches the next
            // barrier only after writing the other one
            __syncthreads();
            const int r = pass * kRows + row4 + (lr & 3);
            if (row4 < kRows && pass * kRows + row4 < rows) {
                const f32x4* const from = part + ((size_t)buf * kRW * kTiles + (row4 >> 4) * NT + tile) * 64 + 4 * (row4 & 15) + lr;
                f32x4 q[kRW];
#pragma unroll
                for (int x = 0; x < kRW; ++x) q[x] = from[(size_t)x * kTiles * 64];
                __builtin_amdgcn_sched_barrier(0);                       // all on their way before the first is waited for
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += ((q[0][e] + q[1][e]) + (q[2][e] + q[3][e])) + ((q[4][e] + q[5][e]) + (q[6][e] + q[7][e]));
                const bool cand = (lr & 3) == 3;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float rr = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f((cand ? 2.8853900817779268f : -1.4426950408889634f) * v[e]));
                    v[e] = cand ? fmaf(-2.0f, rr, 1.0f) : rr;
                }
                quad_transpose(v, lane);
                float* const cp = cell + pass * kRTH + tid;
                const float c = fmaf(v[0], *cp, v[1] * v[3]);
                const float h = v[2] * tanhf_fast(c);
                // the four units of this batch row in bf16, gathered in lanes 0..3 of the row
                const unsigned hb = f32_to_bf16_bits(h);
                const unsigned h1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)hb, 0x104, 0xF, 0xF, true);
                const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)hb, 0x108, 0xF, 0xF, true);
                const unsigned h3 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)hb, 0x10C, 0xF, 0xF, true);
                const unsigned long long four = (unsigned long long)(hb | (h1 << 16)) | ((unsigned long long)(h2 | (h3 << 16)) << 32);
                const bool put = lr < 4 && r < rows && tl < tiles;
                const unsigned long long sent = lr < 4 ? four : 0ull;
                const int tw = tl + (lr >> 2);
                const unsigned word = (unsigned)(((tw >> 1) * R + r) * 2 + (tw & 1)) * 8u;
                if (puts && r < rows && !last) {
                    const unsigned tag = (unsigned)s + 2u;
                    const unsigned long long stamp = ((tag >> 1) & 1u) ? kStamps : 0ull;
                    exchange_store(at_bytes(hx + (tag & 1u) * xbuf, word), (sent & ~kStamps) | stamp, same_xcd);
                    if (puts_more) exchange_store(at_bytes(hx + (tag & 1u) * xbuf, word + (unsigned)(4 * R) * 8u), stamp, same_xcd);
                }
                *cp = c;
                // outputs after the publication: nothing on the way of h
                if (STACK && feeds && puts && r < rows) {
                    __hip_atomic_store(at_bytes(seq + (size_t)s * xbuf, word), sent | kStamps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (puts_more) __hip_atomic_store(at_bytes(seq + (size_t)s * xbuf, word + (unsigned)(4 * R) * 8u), kStamps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (put && yb) *reinterpret_cast<unsigned long long*>(at_bytes(yb + ((size_t)t * B + b_lo) * yb_ld, (unsigned)(r * (int)yb_ld + 4 * tl) * 2u)) = four;
                if (r < rows && unit < H) {
                    if (y) *at_bytes(y + ((size_t)t * B + b_lo) * y_ld, (unsigned)(r * (int)y_ld + unit) * 4u) = h;
                    if (last) {
                        if (hT) *at_bytes(hT + (size_t)b_lo * H, (unsigned)(r * H + unit) * 4u) = h;
                        if (cT) *at_bytes(cT + (size_t)b_lo * H, (unsigned)(r * H + unit) * 4u) = c;
                    }
                }
            }
            buf ^= 1;
        }
        // the columns of yb that pad a row to the next product's K blocks
        if (pads > 0 && wg == gn - 1)
            for (int i = tid; i < rows * pads; i += kRTH)
                *reinterpret_cast<unsigned long long*>(yb + ((size_t)t * B + b_lo + i / pads) * yb_ld + pad0 + 4 * (i % pads)) = 0ull;
    }
}

// ---------------------------------------------------------------------------------------------- shapes and launch
namespace {
struct RowsShape {
    int nt, kb, rt, xl;
    const void* kernel;
};
#define R_S(NT_, KB_) {NT_, KB_, 1, 0, (const void*)persist_rows_bf16_kernel<NT_, KB_, 1, false, 0>}
// shapes whose weights (NT KB x 16 bytes per lane), operands and accumulators fit the registers, those that some width and batch takes
const RowsShape kRowsShapes[] = {
    R_S(1, 1), R_S(2, 1), R_S(4, 1), R_S(3, 2), R_S(4, 2), R_S(8, 2), R_S(1, 3), R_S(5, 3), R_S(6, 3), R_S(1, 4), R_S(2, 4),
    R_S(4, 4), R_S(7, 4), R_S(8, 4), R_S(2, 5), R_S(3, 5), R_S(5, 5), R_S(2, 6), R_S(3, 6), R_S(5, 6), R_S(2, 8), R_S(4, 8),
};
#undef R_S
constexpr int kRowsShapeCount = (int)(sizeof(kRowsShapes) / sizeof(kRowsShapes[0]));
// ... and with the input's matrix beside the recurrent one (2 NT KB x 16 bytes)
#define R_K(NT_, KB_, RT_, XL_) {NT_, KB_, RT_, XL_, (const void*)persist_rows_bf16_kernel<NT_, KB_, RT_, true, XL_>}
const RowsShape kStackShapes[] = {
    R_K(1, 1, 1, 0), R_K(2, 1, 1, 0), R_K(4, 1, 1, 0), R_K(8, 1, 1, 0), R_K(4, 2, 1, 0), R_K(6, 2, 1, 0), R_K(8, 2, 1, 0),
    R_K(2, 3, 1, 0), R_K(3, 3, 1, 0), R_K(6, 3, 1, 1), R_K(2, 4, 1, 0), R_K(3, 4, 1, 0), R_K(4, 4, 1, 0), R_K(3, 5, 1, 0),
    R_K(4, 5, 1, 2), R_K(3, 6, 1, 2), R_K(1, 1, 2, 0), R_K(2, 1, 2, 0), R_K(4, 1, 2, 0), R_K(4, 2, 2, 0), R_K(3, 3, 2, 0),
    R_K(4, 3, 2, 0), R_K(3, 4, 2, 0), R_K(3, 5, 2, 2),
};
#undef R_K
constexpr int kStackShapeCount = (int)(sizeof(kStackShapes) / sizeof(kStackShapes[0]));
}  // namespace

// Shape, rows per group and placement of the lowest estimated step time in microseconds: per pass a fixed part, the matrix
// instructions, the tiles' partial sums, the h that is read (KB); and the part of the exchange that other passes would
// hide.  The constants are a fit to 3500 measured (shape, groups, placement) points over 100 to 2000 units and batches of 2
// to 128 (standard error 7 %).
PersistRowsPlan persist_rows_bf16_plan(int B, int H, int ndir)
{
    PersistRowsPlan best;
    if (B < 1 || H < 1 || ndir < 1 || ndir > 2) return best;
    const int kblocks = (H + 31) / 32, tiles = (H + 3) / 4, cus = device_num_cus();
    for (int i = 0; i < kRowsShapeCount; ++i) {
        const RowsShape& sh = kRowsShapes[i];
        if (sh.kb * kRW < kblocks) continue;
        const int gn = (tiles + sh.nt - 1) / sh.nt;
        const int most = std::min(B, 64);
        for (int groups = 1; groups <= most && ndir * groups * gn <= cus; ++groups) {   // (more fit neither way)
            const int rows = (B + groups - 1) / groups;
            if ((B + rows - 1) / rows != groups) continue;   // a group would be left without a row
            const int passes = (rows + 15) / 16;
            const size_t lds = ((size_t)2 * kRW * sh.nt * 256 + (size_t)passes * kRTH) * sizeof(float);
            if (lds > 160 * 1024) continue;
            const int per_xcd = (ndir * groups + 7) / 8;
            const int local = gn <= 64 && per_xcd * gn <= cus / 8;
            const double h_kb = std::min(rows, 16) * H * 2e-3;
            const double pass = (local ? 0.71 : 0.882) + (local ? 0.0022 : 0.0047) * sh.nt * sh.kb + (local ? 0.084 : 0.094) * sh.nt +
                                (local ? 0.0174 : 0.0109) * h_kb;
            const double us = passes * pass + (passes == 1 ? (local ? 0.265 : 0.467) : 0.0);
            if (us < best.us) {
                best.us = us;
                best.shape = i;
                best.rows = rows; best.groups = groups; best.gn = gn; best.xcd_local = local; best.lds = lds;
            }
        }
    }
    return best;
}

// The same for `layers` consecutive layers of one width in a launch: a fit to 1550 points over 100 to 1500 units, 2 to 5 layers and
// batches of 2 to 128 (standard error 6 %).
PersistRowsPlan persist_rows_bf16_stack_plan(int B, int H, int layers)
{
    PersistRowsPlan best;
    if (B < 1 || H < 1 || layers < 2 || layers > kMaxRowsStack) return best;
    const int kblocks = (H + 31) / 32, tiles = (H + 3) / 4, cus = device_num_cus();
    for (int i = 0; i < kStackShapeCount; ++i) {
        const RowsShape& sh = kStackShapes[i];
        if (sh.kb * kRW < kblocks || (sh.kb > 1 && (sh.kb - 1) * kRW >= kblocks)) continue;
        const int gn = (tiles + sh.nt - 1) / sh.nt;
        const int most = std::min(B, 64);
        for (int groups = 1; groups <= most && layers * groups * gn <= cus; ++groups) {
            const int rows = (B + groups - 1) / groups;
            if ((B + rows - 1) / rows != groups) continue;
            if (2 * rows <= 16 * sh.rt && sh.rt > 1) continue;
            const int passes = (rows + 16 * sh.rt - 1) / (16 * sh.rt);
            const size_t lds = ((size_t)2 * kRW * sh.nt * sh.rt * 256 + (size_t)passes * kRTH + (size_t)kRW * sh.xl * sh.nt * 256) * sizeof(float);
            if (lds > 160 * 1024) continue;
            const int per_xcd = (layers * groups + 7) / 8;
            const int local = gn <= 64 && per_xcd * gn <= cus / 8;
            const double h_kb = std::min(rows, 16 * sh.rt) * H * 2e-3;
            const double pass = (local ? 1.30 : 1.45) + (local ? 0.0138 : 0.0103) * sh.nt * sh.kb * sh.rt + (local ? 0.044 : 0.079) * sh.nt * sh.rt +
                                (local ? 0.018 : 0.0098) * h_kb + 0.09 * (sh.rt - 1);
            const double us = passes * pass + (passes == 1 ? (local ? 0.27 : 0.40) : 0.0);
            if (us < best.us) {
                best.us = us;
                best.shape = i;
                best.layers = layers;
                best.rows = rows; best.groups = groups; best.gn = gn; best.xcd_local = local; best.lds = lds;
            }
        }
    }
    return best;
}

// 8-byte words of one launch: h, the XCD id slots of the groups, then (a stack of layers, T steps) what each layer hands up
static size_t rows_h_words(const PersistRowsPlan& p, int H, int ndir) { return (size_t)ndir * p.groups * 2 * ((H + 31) / 32) * 8 * p.rows; }
size_t persist_rows_bf16_exchange_words(const PersistRowsPlan& p, int H, int ndir, int T)
{
    if (p.shape < 0) return 0;
    return rows_h_words(p, H, ndir) + (size_t)ndir * p.groups * 64 + (p.layers > 0 ? (size_t)T * (rows_h_words(p, H, ndir - 1) / 2) : 0);
}
void persist_rows_bf16_describe(const PersistRowsPlan& p, char* buf, size_t n)
{
    const RowsShape& sh = (p.layers > 0 ? kStackShapes : kRowsShapes)[p.shape];
    char rt[8] = "";
    if (sh.rt > 1) std::snprintf(rt, sizeof rt, ",r%d", sh.rt);
    std::snprintf(buf, n, "(t%d,k%d%s,%dx%d%s)", sh.nt, sh.kb, rt, p.groups, p.rows, p.xcd_local ? ",xcd" : "");
}

// p: the plan of (a.B, a.H, a.ndir); words: the launch's exchange region, all zero
hipError_t launch_persist_rows_bf16(PersistRowsArgs& a, const PersistRowsPlan& p, unsigned long long* words, bool cooperative, hipStream_t s)
{
    if (a.B <= 0 || a.H <= 0 || a.T <= 0) return hipSuccess;
    if (p.shape < 0 || (p.layers > 0 && p.layers != a.ndir)) return hipErrorInvalidValue;
    const RowsShape& sh = (p.layers > 0 ? kStackShapes : kRowsShapes)[p.shape];
    const void* const kernel = sh.kernel;
    a.rows = p.rows; a.groups = p.groups; a.gn = p.gn; a.xcd_local = p.xcd_local;
    if (p.xcd_local || p.rows > 16 * sh.rt) a.poll_pace = 0;   // visible by the time the first read arrives, or other passes in between
    a.hx = words;
    a.xcc_ids = words + rows_h_words(p, a.H, a.ndir);
    a.seq = a.xcc_ids + (size_t)a.ndir * p.groups * 64;
    const int grid = p.xcd_local ? 8 * ((a.ndir * p.groups + 7) / 8) * p.gn : a.ndir * p.groups * p.gn;
    // every workgroup must be resident at the same time: at most one per compute unit
    if (grid > device_num_cus()) return hipErrorCooperativeLaunchTooLarge;
    if (p.lds > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(kernel, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    void* kargs[] = {(void*)&a};
    if (cooperative) return hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(kRTH), kargs, (unsigned)p.lds, s);
    return hipLaunchKernel(kernel, dim3(grid), dim3(kRTH), kargs, p.lds, s);
}

// Words of h0 in operand order for one (launch, direction or layer): [group][k / 8][row][2]
size_t rows_bf16_state_words(const PersistRowsPlan& p, int H) { return (size_t)p.groups * ((H + 31) / 32) * 8 * p.rows; }

// The initial states of n (launch, direction or layer) blocks in bf16 and operand order, from `first` on, and `zeros` words of zeros
// behind them.  (Converted inside the recurrence, addresses and conditions of single values took its registers.)
__global__ __launch_bounds__(256) void rows_prepare_kernel(unsigned long long* __restrict__ first, RowsStates st, const float* __restrict__ h0, size_t total)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        unsigned long long v = 0ull;
        if (i < st.at[st.n]) {
            int e = 0;
            while (i >= st.at[e + 1]) ++e;
            const int H = st.H[e], R = st.rows[e], per = ((H + 31) >> 5) * 8 * R;
            const unsigned j = (unsigned)(i - st.at[e]), g = j / per, w = j - g * per;
            const int k8 = w / (2 * R), r = (int)(w - k8 * 2 * R) >> 1, k = 8 * k8 + 4 * (int)(w & 1u), b = (int)g * R + r;
            if (b < st.B && k < H) {
                const float* const from = h0 + st.off[e] + (size_t)b * H;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (k + c < H) v |= (unsigned long long)f32_to_bf16_bits(from[k + c]) << (16 * c);
            }
        }
        first[i] = v;
    }
}
void RowsStates::add(const PersistRowsPlan& p, int H_, size_t off_)
{
    H[n] = H_; rows[n] = p.rows; off[n] = off_;
    at[n + 1] = at[n] + rows_bf16_state_words(p, H_);
    ++n;
}
hipError_t launch_rows_prepare(unsigned long long* first, const RowsStates& st, const float* h0, size_t zeros, hipStream_t s)
{
    const size_t total = st.at[st.n] + zeros;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(rows_prepare_kernel, dim3((unsigned)std::min<size_t>((total + 255) / 256, 2048)), dim3(256), 0, s, first, st, h0, total);
    return hipGetLastError();
}

// A row-major bf16 matrix W[rows][cols] in the operand order of the 16x16x32 matrix instruction: tile (nb, kb) is 64 lanes x
// 8 values, lane l holding W[16 nb + l % 16][32 kb + 8 (l / 16) .. + 7]; zero beyond the matrix.
__global__ __launch_bounds__(256) void to_frag32_kernel(const uint16_t* __restrict__ W, int rows, int cols, uint4* __restrict__ out)
{
    const int KB = (cols + 31) >> 5;
    const size_t total = (size_t)((rows + 15) >> 4) * KB * 64;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int l = (int)(i & 63);
        const size_t tile = i >> 6;
        const int n = 16 * (int)(tile / KB) + (l & 15), k = 32 * (int)(tile % KB) + 8 * (l >> 4);
        uint32_t v[4] = {};
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (n < rows && k + c < cols) v[c >> 1] |= (uint32_t)W[(size_t)n * cols + k + c] << (16 * (c & 1));
        out[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}
size_t frag32_elements(int rows, int cols) { return (size_t)((rows + 15) / 16) * ((cols + 31) / 32) * 512; }
hipError_t launch_to_frag32(const uint16_t* W, int rows, int cols, uint16_t* out, hipStream_t s)
{
    const size_t g = (frag32_elements(rows, cols) / 8 + 255) / 256;
    hipLaunchKernelGGL(to_frag32_kernel, dim3((unsigned)std::min<size_t>(g, 8192)), dim3(256), 0, s, W, rows, cols, (uint4*)out);
    return hipGetLastError();
}

}  // namespace l355
