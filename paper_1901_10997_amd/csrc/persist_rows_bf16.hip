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
// Bound: the exchange and the chain around it.  Two layers of 1197 units, batch 20: 18.8 us per step with a launch per
// step and layer, 2.5 here (388 against 3063 us per forward of 70 steps); one layer of 1024: batch 64 3.7 us with the 32-row
// tiles, 2.4 here, batch 128 4.3 and 2.8.
#include "common.h"
#include "device_math.h"
#include "exchange.h"

namespace l355 {

namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
constexpr int kRW = 8, kRTH = 512;
constexpr unsigned long long kStamps = 0x4000400040004000ull;

template <int CTRL>
__device__ __forceinline__ float dpp_mov_f(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// Four published values without their stamps.  A NaN has bit 14 set itself and |h| <= 1 else: without that bit a (quiet) NaN is
// a pattern of at least 0x3FC0 (1.5), from which the addition carries into bit 14 again.  The halves apart: 32-bit operations.
__device__ __forceinline__ unsigned unstamped_pair(unsigned v)
{
    const unsigned carried = (v & 0x3FFF3FFFu) + 0x00400040u;
    return (v & 0xBFFFBFFFu) | (carried & 0x40004000u);
}
__device__ __forceinline__ unsigned long long unstamped(unsigned long long v)
{
    return (unsigned long long)unstamped_pair((unsigned)(v >> 32)) << 32 | unstamped_pair((unsigned)v);
}
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

// NT: tiles of 16 packed rows per workgroup; KB: k blocks of 32 per wave
template <int NT, int KB>
__global__ __launch_bounds__(kRTH) void persist_rows_bf16_kernel(PersistRowsArgs a)
{
    static_assert(NT <= 8, "one (tile, four rows) item per 16-lane row");
    extern __shared__ __attribute__((aligned(16))) float lds[];
    f32x4* const part = reinterpret_cast<f32x4*>(lds);                               // [2][8][NT][64]
    float* const cell = lds + (size_t)2 * kRW * NT * 256;                            // [passes][512]
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
    const int passes = (rows + 15) / 16;

    // the direction is chosen by the block index, so its argument block lives in memory: fields copied once
    const PersistRowsDir& D = a.d[dir];
    const float* const Pd = D.P;
    const float* const h0 = D.h0;
    float* const y = D.y;
    uint16_t* const yb = D.yb;
    const size_t y_ld = (size_t)D.y_ld, yb_ld = (size_t)D.yb_ld;
    float* const hT = D.hT;
    float* const cT = D.cT;
    const int reverse = D.reverse;

    const int KBt = (H + 31) >> 5, tiles = (H + 3) >> 2;
    const int kb0 = wave * KB;
    // weights: loads from clamped addresses, what lies outside is zeroed afterwards
    uint4 w[NT][KB];
    {
        const uint4* const Wf = reinterpret_cast<const uint4*>(D.Wf);
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const int nb = wg * NT + n, kb = kb0 + q;
                const bool ok = nb < tiles && kb < KBt;
                const uint4 v = Wf[((size_t)(ok ? nb : 0) * KBt + (ok ? kb : 0)) * 64 + lane];
                w[n][q] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
            }
    }

    unsigned long long* const hx = a.hx + ((size_t)dir * a.groups + grp) * 2 * ((size_t)KBt * 8 * R);   // [2][k / 8][row][2] words
    const size_t xbuf = (size_t)KBt * 8 * R;

    // This thread's 16-lane row serves tile `tile`, batch rows row4 .. + 3 of a pass: packed row lr of the tile while the sums
    // are gathered, unit lr / 4 and batch row lr % 4 from the cell update on.
    const int item = wave * 4 + lg, tile = item % NT, row4 = 4 * (item / NT);
    const int tl = wg * NT + tile, unit = 4 * tl + (lr >> 2), col = 16 * tl + lr;
    for (int pass = 0; pass < passes; ++pass) {
        const int r = pass * 16 + row4 + (lr & 3);
        cell[pass * kRTH + tid] = (D.c0 && row4 < 16 && r < rows && unit < H) ? D.c0[(size_t)(b_lo + r) * H + unit] : 0.f;
    }

    bool same_xcd = false;
    if (a.xcd_local)
        same_xcd = group_shares_xcd(a.xcc_ids + (size_t)(dir * a.groups + grp) * 64, gn, wg, 1u, lds, tid, kRTH,
                                    a.timeout_flag, a.spin_limit) && !a.device_scope_only;

    // P of the item's four rows: unconditional loads (clamped), requested a pass ahead
    float p_next[4];
    auto load_p = [&](int s, int pass) {
        const int t = reverse ? a.T - 1 - s : s;
        const float* const Pt = Pd + ((size_t)t * B + b_lo) * (size_t)(4 * H);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = pass * 16 + row4 + v;
            p_next[v] = Pt[(unsigned)((r < rows ? r : rows - 1) * 4 * H + (col < 4 * H ? col : 0))];
        }
    };
    load_p(0, 0);
    int buf = 0;
    const int pad0 = 4 * tiles, pads = yb ? (D.yb_width - pad0) >> 2 : 0;   // columns of yb behind the last tile, in fours

    for (int s = 0; s < a.T; ++s) {
        const int t = reverse ? a.T - 1 - s : s;
        const bool last = s == a.T - 1;
        for (int pass = 0; pass < passes; ++pass) {
            // ---- operand fragments of h_{t-1}
            u64x2 fr[KB];
            const int r_op = pass * 16 + lr < rows ? pass * 16 + lr : rows - 1;   // a row that is not there reads the last one (never used)
            if (s > 0) {
                const unsigned tag = (unsigned)s + 1u;
                const unsigned long long want = ((tag >> 1) & 1u) ? kStamps : 0ull;
                const unsigned long long* const src = hx + (tag & 1u) * xbuf + (unsigned)((lg * R + r_op) * 2);
                // units are published in fours: 8-byte words of the last block beyond the last tile are never written
                const int k_last = 32 * (KBt - 1) + 8 * lg;
                const bool dead0 = k_last >= pad0, dead1 = k_last + 4 >= pad0;
                pace_poll(a.poll_pace);
                unsigned spins = 0;
                for (;;) {
                    // a block beyond K reads the last one again (its weights are zero)
#pragma unroll
                    for (int q = 0; q < KB; ++q) {
                        const unsigned long long* const p = src + (size_t)(kb0 + q < KBt ? kb0 + q : KBt - 1) * 8 * R;
                        fr[q].x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        fr[q].y = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    unsigned long long differ = 0;
#pragma unroll
                    for (int q = 0; q < KB; ++q) {
                        const bool tail = kb0 + q >= KBt - 1;                    // wave-uniform
                        differ |= (tail && dead0 ? 0ull : fr[q].x ^ want) | (tail && dead1 ? 0ull : fr[q].y ^ want);
                    }
                    if (!__builtin_amdgcn_ballot_w64((differ & kStamps) != 0ull)) break;
                    if (++spins > a.spin_limit) {
                        __hip_atomic_store(a.timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
                    if ((spins & 63u) == 0 && __hip_atomic_load(a.timeout_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
                }
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    fr[q].x = unstamped(fr[q].x);
                    fr[q].y = unstamped(fr[q].y);
                }
            } else if (h0) {
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    const int k = 32 * (kb0 + q) + 8 * lg;
                    unsigned long long x[2] = {0ull, 0ull};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (k + e < H) x[e >> 2] |= (unsigned long long)f32_to_bf16_bits(h0[(size_t)(b_lo + r_op) * H + k + e]) << (16 * (e & 3));
                    fr[q].x = x[0];
                    fr[q].y = x[1];
                }
            }
            // the pass's elements of P were requested a pass ahead; behind the words just waited for they have arrived too
            // (taken over here by hand: at the top of the loop the wait for them would include the stores just issued)
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) asm volatile("v_mov_b32 %0, %1" : "=v"(v[e]) : "v"(p_next[e]));
            if (pass + 1 < passes) load_p(s, pass + 1);
            else if (!last) load_p(s + 1, 0);
            f32x4 acc[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[n] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (s > 0 || h0) {
#pragma unroll
                for (int q = 0; q < KB; ++q)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fr[q]), __builtin_bit_cast(bf16x8, w[n][q]),
                                                                         acc[n], 0, 0, 0);
            }
            // partial tiles -> LDS: lane l of an accumulator holds batch rows 4 (l / 16) .. + 3 of packed row l % 16
            f32x4* const mine = part + ((size_t)(buf * kRW + wave) * NT) * 64 + lane;
#pragma unroll
            for (int n = 0; n < NT; ++n) mine[n * 64] = acc[n];
            // one barrier per pass: the partial tiles alternate between two buffers, and a wave that runs ahead reaches the next
            // barrier only after writing the other one
            __syncthreads();
            const int r = pass * 16 + row4 + (lr & 3);
            if (row4 < 16 && pass * 16 + row4 < rows) {
                const f32x4* const from = part + ((size_t)buf * kRW * NT + tile) * 64 + 4 * row4 + lr;
#pragma unroll
                for (int x = 0; x < kRW; ++x) {
                    const f32x4 q = from[(size_t)x * NT * 64];
                    v[0] += q[0]; v[1] += q[1]; v[2] += q[2]; v[3] += q[3];
                }
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
                if (put && !last) {
                    const unsigned tag = (unsigned)s + 2u;
                    exchange_store(hx + (tag & 1u) * xbuf + (unsigned)(((tl >> 1) * R + r) * 2 + (tl & 1)),
                                   (four & ~kStamps) | (((tag >> 1) & 1u) ? kStamps : 0ull), same_xcd);
                }
                *cp = c;
                // outputs after the publication: nothing on the way of h
                if (put && yb) *reinterpret_cast<unsigned long long*>(yb + ((size_t)t * B + b_lo) * yb_ld + (unsigned)(r * (int)yb_ld + 4 * tl)) = four;
                if (r < rows && unit < H) {
                    if (y) (y + ((size_t)t * B + b_lo) * y_ld)[(unsigned)(r * (int)y_ld + unit)] = h;
                    if (last) {
                        if (hT) hT[(size_t)(b_lo + r) * H + unit] = h;
                        if (cT) cT[(size_t)(b_lo + r) * H + unit] = c;
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
    int nt, kb;
    const void* kernel;
};
#define R_S(NT_, KB_) {NT_, KB_, (const void*)persist_rows_bf16_kernel<NT_, KB_>}
// the shapes whose weights (NT KB x 16 bytes per lane), operands and accumulators fit the registers
const RowsShape kRowsShapes[] = {
    R_S(1, 1), R_S(2, 1), R_S(4, 1), R_S(1, 2), R_S(2, 2), R_S(3, 2), R_S(4, 2), R_S(8, 2), R_S(1, 3), R_S(2, 3), R_S(3, 3),
    R_S(5, 3), R_S(6, 3), R_S(1, 4), R_S(2, 4), R_S(4, 4), R_S(7, 4), R_S(8, 4), R_S(2, 5), R_S(3, 5), R_S(5, 5), R_S(2, 6),
    R_S(3, 6), R_S(5, 6), R_S(2, 8), R_S(3, 8), R_S(4, 8),
};
#undef R_S
constexpr int kRowsShapeCount = (int)(sizeof(kRowsShapes) / sizeof(kRowsShapes[0]));
}  // namespace

// Shape, rows per group and placement of the lowest estimated step time in microseconds: per pass a fixed part, the matrix
// instructions, the tiles' partial sums, the h that is read (KB); and the part of the exchange that other passes would
// hide.  The constants are a fit to 1200 measured (shape, groups, placement) points over 64 to 2000 units and batches of 3
// to 256 (standard error 10 %).
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
            const double pass = (local ? 0.95 : 1.1) + 0.027 * sh.nt * sh.kb + (local ? 0.02 : 0.04) * sh.nt + (local ? 0.016 : 0.01) * h_kb;
            const double us = passes * pass + (passes == 1 ? (local ? 0.32 : 0.56) : 0.0);
            if (us < best.us) {
                best.us = us;
                best.shape = i;
                best.rows = rows; best.groups = groups; best.gn = gn; best.xcd_local = local; best.lds = lds;
            }
        }
    }
    return best;
}

// 8-byte words of one launch: h, then the XCD id slots of the groups
static size_t rows_h_words(const PersistRowsPlan& p, int H, int ndir) { return (size_t)ndir * p.groups * 2 * ((H + 31) / 32) * 8 * p.rows; }
size_t persist_rows_bf16_exchange_words(const PersistRowsPlan& p, int H, int ndir)
{
    return p.shape >= 0 ? rows_h_words(p, H, ndir) + (size_t)ndir * p.groups * 64 : 0;
}
void persist_rows_bf16_describe(const PersistRowsPlan& p, char* buf, size_t n)
{
    std::snprintf(buf, n, "(t%d,k%d,%dx%d%s)", kRowsShapes[p.shape].nt, kRowsShapes[p.shape].kb, p.groups, p.rows, p.xcd_local ? ",xcd" : "");
}

// p: the plan of (a.B, a.H, a.ndir); words: the launch's exchange region, all zero
hipError_t launch_persist_rows_bf16(PersistRowsArgs& a, const PersistRowsPlan& p, unsigned long long* words, bool cooperative, hipStream_t s)
{
    if (a.B <= 0 || a.H <= 0 || a.T <= 0) return hipSuccess;
    if (p.shape < 0) return hipErrorInvalidValue;
    const void* const kernel = kRowsShapes[p.shape].kernel;
    a.rows = p.rows; a.groups = p.groups; a.gn = p.gn; a.xcd_local = p.xcd_local;
    if (p.xcd_local || p.rows > 16) a.poll_pace = 0;   // visible by the time the first read arrives, or other passes in between
    a.hx = words;
    a.xcc_ids = words + rows_h_words(p, a.H, a.ndir);
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
