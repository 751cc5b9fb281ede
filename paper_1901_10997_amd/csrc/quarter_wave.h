// Row-compressed weights in the quarter-wave form: the entries outside a wave's slots (device side).
#pragma once
#include <hip/hip_runtime.h>
#include "common.h"

namespace l355 {

// Slot s of a unit is one 64-lane gather for all four gate rows, gate q on lanes 16q..16q+15, so the slot count of a matrix would
// be that of its longest row.  The entries that rows have beyond the slots are dealt to the lanes of their own gate instead, sixteen
// of a gate per round whatever unit of the wave they belong to: a round is one gather, and its products join the lanes' partial
// sums of their units.  Lane (q, i) holds entry 16 r + i of gate q in round r.
template <int R>   // most rounds
struct Q16Extra {
    float v[R];
    unsigned at[R];   // LDS offset of the column in `scale`d units; local unit in the high half (no entry: 0xffff)
    int rounds;       // of the wave
};
// ptr: [4][units + 1]; u0: the wave's first unit, of UPW
template <int UPW, int R>
__device__ __forceinline__ Q16Extra<R> load_q16_extra(const int32_t* ptr, const uint32_t* ent, const float* val, int units, int u0, int lane, unsigned scale)
{
    Q16Extra<R> x;
    x.rounds = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) { x.v[r] = 0.f; x.at[r] = 0xffff0000u; }
    if (ptr != nullptr && u0 < units) {
        const int32_t* const gate = ptr + (size_t)(lane >> 4) * (units + 1);
        int from[UPW + 1];
#pragma unroll
        for (int u = 0; u <= UPW; ++u) from[u] = gate[u0 + u < units ? u0 + u : units];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = from[0] + 16 * r + (lane & 15);
            const bool have = e < from[UPW];
            if (have) {
                int local = 0;
#pragma unroll
                for (int u = 1; u < UPW; ++u) local += e >= from[u];
                x.v[r] = val[e];
                x.at[r] = ((unsigned)local << 16) | (ent[e] * scale);
            }
            x.rounds += __builtin_amdgcn_ballot_w64(have) != 0ull;
        }
    }
    x.rounds = __builtin_amdgcn_readfirstlane(x.rounds);
    return x;
}
// tot[u * BW + b]: the lane's partial sums; read(offset) -> the BW values of a column.  (Products of lanes without an entry and sums of
// other units are left out, not multiplied by zero: a value may be infinite.)
template <int UPW, int BW, int R, class Read>
__device__ __forceinline__ void add_q16_extra(float (&tot)[16], const Q16Extra<R>& x, Read read)
{
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (x.rounds > r) {   // wave-uniform
            unsigned at = x.at[r];
            asm volatile("" : "+v"(at));   // unpacked here, not ahead of the time loop
            const auto c = read(at & 0xffffu);
            const unsigned local = at >> 16;
            float t[BW];
            t[0] = x.v[r] * c.x; t[1] = x.v[r] * c.y;
            if constexpr (BW == 4) { t[2] = x.v[r] * c.z; t[3] = x.v[r] * c.w; }
#pragma unroll
            for (int u = 0; u < UPW; ++u)
#pragma unroll
                for (int b = 0; b < BW; ++b) tot[u * BW + b] += local == (unsigned)u ? t[b] : 0.f;
        }
}

}  // namespace l355
