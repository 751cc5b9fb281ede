// Small-batch row-compressed recurrence with the time loop on the device: one launch per layer, every
// direction of the layer in the same grid.
//
// Per timestep (paper Section 4, cell equations): a = P[t] + W_h.h_{t-1} (P = input projection with bias);
// f,i,o = sigmoid, g = tanh; c_t = f*c_{t-1} + i*g; h_t = o*tanh(c_t).
//
// The grid is a 2-D partition per direction: unit groups x batch groups.  A workgroup owns UPB hidden units
// and BW batch columns; it needs only the h values of its own batch columns (all H of them), which keeps the
// polled volume per workgroup at BW*H slots however large the batch is.  Each wave keeps the kept weights of
// its UPW units in registers in the quarter-wave form: slot s of a unit is one 64-lane gather that serves all
// four gate rows, gate q on lanes 16q..16q+15, so a lane accumulates BW sums per unit, a row's total is a butterfly
// inside its 16 lanes, and lane 16*gate + pair ends up with a gate total (pair = local unit * BW + column).  One
// exp2 and one reciprocal evaluate all gates of all pairs; c and h are updated in lanes 0..pairs-1.  h travels
// between workgroups as 32-bit words that carry their readiness in bit 30 (free in |h| <= 1; a NaN gets it back on reading, see
// unstamped): step tag g, counted over the launches of a forward that share the words (epoch), in buffer g & 1 with stamp (g >> 1) & 1,
// both buffers zero before the first; per (direction, batch group) [buffer][k][BW], the order of the LDS copy, so that the poll is a
// straight copy, sixteen bytes per lane and load.  (As tagged 8-byte slots: two layers of 1500 units, batch 20, 10 % kept,
// 4.4 us per step; 3.7 so, 3.4 with four columns per gather, as planned below.)  Only the workgroups of one (direction, batch group) exchange anything; where the groups
// fit they are placed on one XCD each and, once the launch has verified that from the hardware's XCD ids, publish h
// with workgroup-scope stores that stay in that XCD's L2 (exchange.h).  All waits are bounded.
#include <type_traits>
#include "common.h"
#include "device_math.h"
#include "exchange.h"
#include "quarter_wave.h"

namespace l355 {

// S = slots per unit (16 kept entries of each gate per slot).  Configurations with registers to spare for the
// XCD-local hand-over:
constexpr bool persist_batched_q16_xcd_capable(int s, int upw) { return s * upw <= 84; }

template <int S, int UPW, int BW>
__global__ __launch_bounds__(512) void persist_batched_q16_kernel(PersistBatchedArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];  // hbuf[H][BW] (the BW batch values of one k adjacent; whole 16 bytes) | pub[BW][UPB]
    constexpr int PAIRS = UPW * BW;
    static_assert(PAIRS <= 16, "pairs must fit one 16-lane row");
    static_assert(S % 2 == 0, "slots come in pairs (one per bank half)");
    const int H = a.H, B = a.B;
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthreads >> 6;
    const int upb = nwaves * UPW;
    float* hbuf = lds;
    float* pub = lds + (((size_t)BW * H + 3) & ~(size_t)3);
    constexpr bool kXcd = persist_batched_q16_xcd_capable(S, UPW);
    int dir, bgi, ugi;
    if (kXcd && a.xcd_local) {
        const int j = blockIdx.x >> 3;
        const int g = (blockIdx.x & 7) + 8 * (j / a.ug);
        if (g >= a.ndir * a.bg) return;     // padding ids take no part in the exchange
        ugi = j % a.ug; dir = g / a.bg; bgi = g % a.bg;
    } else {
        const int per_dir = a.ug * a.bg;
        dir = blockIdx.x / per_dir;
        const int rem = blockIdx.x % per_dir;
        bgi = rem / a.ug; ugi = rem % a.ug;
    }
    const PersistBatchedDir& D = a.d[dir];
    const int b0 = bgi * BW;
    const int bw = (B - b0) < BW ? (B - b0) : BW;         // columns actually present (none: 0 or less)
    const int u0 = ugi * upb + wave * UPW;                // first unit of this wave
    // words of this batch group: [buffer][k][BW], i.e. in the order of the LDS copy of h
    unsigned* const xchg = a.xchg + ((size_t)dir * a.bg + bgi) * 2 * a.h_stride;

    // kept weights of this wave's units: values in fp32 registers, columns as 16-bit LDS byte offsets of their h
    // values, two to a register.  Every load is issued whatever the shape (clamped address, zeroed afterwards).
    float wv[UPW][S];
    unsigned wc[UPW][S / 2];
    {
        const int slots = D.q16_slots;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int unit = (u0 + u < H) ? (u0 + u) : (H - 1);
            float tv[S];
            unsigned tk[S];
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const int ii = i < slots ? i : slots - 1;
                const size_t idx = ((size_t)unit * slots + ii) * 64 + lane;
                tv[i] = D.q16_val[idx];
                tk[i] = D.q16_col[idx];
            }
#pragma unroll
            for (int i = 0; i < S / 2; ++i) wc[u][i] = 0u;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const bool live = (u0 + u < H) && i < slots;
                wv[u][i] = live ? tv[i] : 0.f;
                wc[u][i >> 1] |= ((live ? tk[i] : 0u) * (BW * 4u)) << (16 * (i & 1));
            }
        }
    }
    const Q16Extra<kQ16LstmRounds> extra = load_q16_extra<UPW, kQ16LstmRounds>(D.q16_ovf_ptr, D.q16_ovf_ent, D.q16_ovf_val, H, u0, lane, BW * 4u);
    // lane 16*gate + pair: pair = local unit * BW + column
    const int lp = lane & 15, row = lane >> 4;
    const int pu = lp / BW, pb = lp % BW;
    const bool pair_ok = lp < PAIRS && pb < bw && (u0 + pu) < H;
    const int unit_l = u0 + pu;
    float c = 0.f;
    if (lane < 16 && pair_ok && D.c0) c = D.c0[(size_t)(b0 + pb) * H + unit_l];

    // The direction is chosen by the block index, so `D` is addressed through memory: its fields are copied once
    // and the outputs are written after the publication.
    const float* const Pd_c = D.P;
    float* const y_c = D.y;
    const size_t y_ld_c = (size_t)D.y_ld;
    float* const hT_c = D.hT;
    float* const cT_c = D.cT;
    const float* const h0_c = D.h0;
    const int reverse = D.reverse;
    constexpr int kInFlight = S * UPW <= 84 ? 4 : 2;   // 16-byte loads of a thread
    bool same_xcd = false;
    if (kXcd && a.xcd_local)
        same_xcd = group_shares_xcd(a.xcc_ids + ((size_t)dir * a.bg + bgi) * 64, a.ug, ugi, a.tag_base + 1u, hbuf, tid,
                                    nthreads, a.timeout_flag, a.spin_limit) && !a.device_scope_only;
    // P comes from memory (never from a cache: every element is read once), and a wave's loads return in order: a
    // load of P issued in front of the poll would hold back the poll's answer by a memory round trip in every step.
    // So the element for step s+1 is requested right after the poll of step s has been answered.
    auto load_p = [&](int s_) {
        const int t_ = reverse ? (a.T - 1 - s_) : s_;
        return (pair_ok && s_ < a.T) ? Pd_c[((size_t)t_ * a.Bld + b0 + pb) * (4 * (size_t)H) + 4 * unit_l + row] : 0.f;
    };
    float pin_next = load_p(0);
    for (int s = 0; s < a.T; ++s) {
        const int t = reverse ? (a.T - 1 - s) : s;
        if (s == 0) {
            for (int e = tid; e < BW * H; e += nthreads) {
                const int b = e / H, k = e - b * H;
                float v = (h0_c && b < bw) ? h0_c[(size_t)(b0 + b) * H + k] : 0.f;
                if (a.round_h_bf16) v = round_bf16(v);
                hbuf[k * BW + b] = v;
            }
        } else {
            pace_poll(a.poll_pace);   // (set by the launcher)
            const unsigned tag = a.epoch + (unsigned)s + 1u;
            gather_stamped_all<kInFlight>(xchg + (tag & 1u) * a.h_stride, BW * H, kHStampBit, ((tag >> 1) & 1u) ? kHStampBit : 0u, hbuf, tid, nthreads,
                                          a.timeout_flag, a.spin_limit, [](unsigned v) { return unstamped(v, kHStampBit); });
        }
        // (the value is taken over here, behind the poll's own wait, and not at the top of the loop, where waiting for
        // it would also wait for the acknowledgement of the stores just issued, in front of the poll)
        constexpr bool kTight = S * UPW >= 84 || (BW == 4 && S * UPW >= 72);   // near the register limit
        if constexpr (!kTight) asm volatile("" : "+v"(pin_next));   // (near the register limit the pin costs more than it saves)
        const float pin = pin_next;
        pin_next = load_p(s + 1);
        __syncthreads();
        if constexpr (kTight) {
            // near the register limit the offsets stay packed two to a register: the compiler must not unpack all
            // of them ahead of the time loop
#pragma unroll
            for (int u = 0; u < UPW; ++u)
#pragma unroll
                for (int i = 0; i < S / 2; ++i) asm volatile("" : "+v"(wc[u][i]));
        }
        float G = 0.f;
        {
            // The wave's UPW * S gathers as one software-pipelined sequence: PD reads are in flight ahead of the
            // multiply-adds that consume them, whatever unit they belong to.
            using VT = typename std::conditional<BW == 2, float2, float4>::type;
            constexpr int NS = UPW * S;
            constexpr int PDMAX = kTight ? 8 : 12;
            constexpr int PD = NS < PDMAX ? NS : PDMAX;
            auto read_slot = [&](int n) {
                const int u = n / S, i = n % S;
                const unsigned off = (wc[u][i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
                return *reinterpret_cast<const VT*>(reinterpret_cast<const char*>(hbuf) + off);
            };
            VT ring[PD];
#pragma unroll
            for (int n = 0; n < PD; ++n) ring[n] = read_slot(n);
            float acc[2][BW];   // two chains per column
            float tot[16];      // per-lane partial sums of the wave's (unit, column) pairs, pair p = BW u + b
#pragma unroll
            for (int p = PAIRS; p < 16; ++p) tot[p] = 0.f;
#pragma unroll
            for (int n = 0; n < NS; ++n) {
                const int u = n / S, i = n % S;
                if (i == 0) {
#pragma unroll
                    for (int b = 0; b < BW; ++b) acc[0][b] = acc[1][b] = 0.f;
                }
                const float w = wv[u][i];
                const VT x = ring[n % PD];
                acc[i & 1][0] = fmaf(w, x.x, acc[i & 1][0]);
                acc[i & 1][1] = fmaf(w, x.y, acc[i & 1][1]);
                if constexpr (BW == 4) {
                    acc[i & 1][2] = fmaf(w, x.z, acc[i & 1][2]);
                    acc[i & 1][3] = fmaf(w, x.w, acc[i & 1][3]);
                }
                if (n + PD < NS) ring[n % PD] = read_slot(n + PD);
                __builtin_amdgcn_sched_barrier(0);
                if (i == S - 1) {
#pragma unroll
                    for (int b = 0; b < BW; ++b) tot[u * BW + b] = acc[0][b] + acc[1][b];
                }
            }
            add_q16_extra<UPW, BW>(tot, extra, [&](unsigned off) { return *reinterpret_cast<const VT*>(reinterpret_cast<const char*>(hbuf) + off); });
            // all the sums over the 16 lanes of a row at once: lane p of row q ends up with gate q's total of pair p
            G = row16_transpose_sum(tot, lp);
        }
        G += pin;
        const bool cand = row == 3;
        const float sc = cand ? 2.8853900817779268f : -1.4426950408889634f;
        const float rr = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(sc * G));
        const float gate = cand ? fmaf(-2.0f, rr, 1.0f) : rr;
        const float gi = __shfl(gate, 16 + lp, 64), go = __shfl(gate, 32 + lp, 64), gg = __shfl(gate, 48 + lp, 64);
        float h_keep = 0.f;
        if (lane < 16) {
            c = fmaf(gate, c, gi * gg);
            const float h = go * tanhf_fast(c);
            if (lp < PAIRS) pub[(wave * UPW + pu) * BW + pb] = a.round_h_bf16 ? round_bf16(h) : h;
            h_keep = h;
        }
        __syncthreads();
        if (s + 1 < a.T) {
            const unsigned tag = a.epoch + (unsigned)s + 2u, stamp = ((tag >> 1) & 1u) ? kHStampBit : 0u;
            unsigned* const out = xchg + (tag & 1u) * a.h_stride + (size_t)ugi * upb * BW;
            // (columns that a ragged group lacks as well: readers wait for whole groups of words)
            for (int e = tid; e < BW * upb; e += nthreads)
                if (ugi * upb + e / BW < H) exchange_store(out + e, (__float_as_uint(pub[e]) & ~kHStampBit) | stamp, kXcd && same_xcd);
        }
        // outputs after the publication: nothing on the way of h_t
        if (lane < 16 && pair_ok) {
            y_c[((size_t)t * a.Bld + b0 + pb) * y_ld_c + unit_l] = h_keep;
            if (s + 1 == a.T) {
                const size_t ci = (size_t)(b0 + pb) * H + unit_l;
                if (hT_c) hT_c[ci] = h_keep;
                if (cT_c) cT_c[ci] = c;
            }
        }
    }
}

constexpr int kWaves = 8;
static size_t batched_lds_bytes(int H, int upw, int bw) { return ((((size_t)bw * H + 3) & ~(size_t)3) + (size_t)bw * kWaves * upw) * sizeof(float); }

// ------------------------------------------------------------------------------------------------ planning
// Choose (UPW, BW): at most one workgroup per compute unit, within the register budget (1.5 registers per unit and slot; 512-thread
// workgroups leave 256 registers per lane) and PAIRS <= 16.
constexpr int kQ16WeightRegs = 156;
// one XCD holds an eighth of the compute units; its share of the groups must fit there
bool persist_batched_q16_local(int slots, int upw, int ug, int bg, int ndir)
{
    return persist_batched_q16_xcd_capable(slots, upw) && ug <= 64 && ((ndir * bg + 7) / 8) * ug <= device_num_cus() / 8;
}
bool persist_batched_q16_plan(int B, int H, int slots, int ndir, int* upw_out, int* bw_out, int* ug_out, int* bg_out)
{
    if (B < 2 || slots < 2 || slots > 24 || (slots & 1) || H < 1 || H > 4096) return false;
    // The shape of the lowest estimated step: vector issue per gather (bw multiply-adds, the address), what a group outside one XCD
    // pays more for its exchange, the words that are polled (microseconds; the terms that differ between shapes).  Four columns per gather beat
    // two wherever both leave a wave as many multiply-adds (1000 units, batch 20: 1.60 us per step against 1.95; 300 units, both
    // directions, batch 30: 1.9 against 2.2), and a shape inside an XCD pays where a wave does not get many more units for it.
    double least = 1e30;
    for (int bw = 2; bw <= 4; bw *= 2)
        for (int upw = 2; upw <= 8; ++upw) {
            if (upw * bw > 16 || 3 * slots * upw > 2 * kQ16WeightRegs) continue;
            if (batched_lds_bytes(H, upw, bw) > 64 * 1024) continue;
            const int ug = (H + kWaves * upw - 1) / (kWaves * upw), bg = (B + bw - 1) / bw;
            if (ug * bg * ndir > device_num_cus()) continue;
            const bool local = persist_batched_q16_local(slots, upw, ug, bg, ndir);
            const double us = 0.0033 * slots * upw * (bw + 1.5) + (local ? 0.0 : 0.3) + 0.026e-3 * H * bw;
            if (us < least) {
                least = us;
                *upw_out = upw; *bw_out = bw; *ug_out = ug; *bg_out = bg;
            }
        }
    return least < 1e30;
}

// The plan of a run of B batch columns among runs of up to `longest` over the same words.  Where the longest has the same shape and
// placement the run gets as many batch groups, the last one without a column: it writes its words like the others, so the next launch
// finds every word written equally often and none has to be cleared in between.
bool persist_batched_q16_run_plan(int B, int longest, int H, int slots, int ndir, int* upw, int* bw, int* ug, int* bg)
{
    if (!persist_batched_q16_plan(B, H, slots, ndir, upw, bw, ug, bg)) return false;
    int upw_l, bw_l, ug_l, bg_l;
    if (longest > B && persist_batched_q16_plan(longest, H, slots, ndir, &upw_l, &bw_l, &ug_l, &bg_l) && upw_l == *upw && bw_l == *bw &&
        persist_batched_q16_local(slots, upw_l, ug_l, bg_l, ndir) == persist_batched_q16_local(slots, *upw, *ug, *bg, ndir))
        *bg = bg_l;
    return true;
}

// words of a buffer of a (direction, batch group): whole 256-byte blocks
size_t persist_batched_q16_stride(int H, int bw) { return ((size_t)H * bw + 63) / 64 * 64; }

template <int S, int UPW, int BW>
static hipError_t launch_q16_cfg(PersistBatchedArgs& a, int blocks, bool cooperative, hipStream_t s)
{
    const size_t lds = batched_lds_bytes(a.H, UPW, BW);
    void* args[] = {(void*)&a};
    auto kern = persist_batched_q16_kernel<S, UPW, BW>;
    if (cooperative) return hipLaunchCooperativeKernel((const void*)kern, dim3(blocks), dim3(64 * kWaves), args, (unsigned)lds, s);
    return hipLaunchKernel((const void*)kern, dim3(blocks), dim3(64 * kWaves), args, lds, s);
}

template <int S>
static hipError_t launch_q16_s(PersistBatchedArgs& a, int upw, int bw, int blocks, bool coop, hipStream_t s)
{
#define CFG(U, W) if constexpr (3 * S * U <= 2 * kQ16WeightRegs) { if (upw == U && bw == W) return launch_q16_cfg<S, U, W>(a, blocks, coop, s); }
    CFG(2, 2) CFG(3, 2) CFG(4, 2) CFG(5, 2) CFG(6, 2) CFG(7, 2) CFG(8, 2) CFG(2, 4) CFG(3, 4) CFG(4, 4)
#undef CFG
    return hipErrorInvalidValue;
}

hipError_t launch_persist_batched_q16(PersistBatchedArgs& a, int longest, int ndir, int slots, int cooperative, hipStream_t s)
{
    if (a.T <= 0) return hipSuccess;
    int upw, bw, ug, bg;
    if (!persist_batched_q16_run_plan(a.B, longest, a.H, slots, ndir, &upw, &bw, &ug, &bg)) return hipErrorInvalidValue;
    a.ug = ug;
    a.bg = bg;
    const int per_xcd = (ndir * bg + 7) / 8;
    a.ndir = ndir;
    a.h_stride = persist_batched_q16_stride(a.H, bw);
    a.xcd_local = persist_batched_q16_local(slots, upw, ug, bg, ndir) ? 1 : 0;
    const int blocks = a.xcd_local ? 8 * per_xcd * ug : ug * bg * ndir;
    // Inside an XCD a wait costs what it lasts, except where the products are so short that the first round of the poll comes before many
    // workgroups' words do, and a second follows: up to three units per wave and 20 slots in all, two columns, 20 workgroups and more to a group
    // (119 steps unpaced / at 3: 643 units, 8 % kept, batch 14 211 / 202 us, 768, both directions, batch 5 209 / 201, 433, batch 6 182 / 177;
    // but four units per wave, 832 units, batch 3 186 / 190, and nine workgroups, 134 units, batch 8 145 / 149).
    if (a.xcd_local && a.poll_pace > 0) a.poll_pace = bw == 2 && upw <= 3 && slots * upw <= 20 && ug >= 20 ? 3 : 0;
    switch (slots) {
        case 2: return launch_q16_s<2>(a, upw, bw, blocks, cooperative != 0, s);
        case 4: return launch_q16_s<4>(a, upw, bw, blocks, cooperative != 0, s);
        case 6: return launch_q16_s<6>(a, upw, bw, blocks, cooperative != 0, s);
        case 8: return launch_q16_s<8>(a, upw, bw, blocks, cooperative != 0, s);
        case 10: return launch_q16_s<10>(a, upw, bw, blocks, cooperative != 0, s);
        case 12: return launch_q16_s<12>(a, upw, bw, blocks, cooperative != 0, s);
        case 14: return launch_q16_s<14>(a, upw, bw, blocks, cooperative != 0, s);
        case 16: return launch_q16_s<16>(a, upw, bw, blocks, cooperative != 0, s);
        case 18: return launch_q16_s<18>(a, upw, bw, blocks, cooperative != 0, s);
        case 20: return launch_q16_s<20>(a, upw, bw, blocks, cooperative != 0, s);
        case 22: return launch_q16_s<22>(a, upw, bw, blocks, cooperative != 0, s);
        case 24: return launch_q16_s<24>(a, upw, bw, blocks, cooperative != 0, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace l355
