// Small utility kernels: fills (used instead of memset nodes so that callers may capture a forward into a
// graph) and a streaming copy used to quote the achievable memory bandwidth next to the spec-sheet figure.
#include "common.h"

#include <map>
#include <mutex>
#include <utility>

namespace l355 {

__global__ void fill_u64_kernel(unsigned long long* p, size_t n, unsigned long long v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void fill_f32_kernel(float* p, size_t n, float v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ __launch_bounds__(256) void copy_kernel(float4* __restrict__ dst, const float4* __restrict__ src, size_t n16)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

static int grid_for(size_t n, int threads)
{
    size_t g = (n + threads - 1) / threads;
    if (g > 256 * 16) g = 256 * 16;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_fill_u64(unsigned long long* p, size_t n, unsigned long long v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// A wave per row behind the blocks that fill: one launch for both (the check alone 2.5 us of launch, 1 us of work).
__global__ __launch_bounds__(256) void fill_and_check_kernel(unsigned long long* p, size_t n, unsigned fill_blocks, const float* __restrict__ h0,
                                                             StateRows rows, unsigned* __restrict__ beyond)
{
    if (blockIdx.x < fill_blocks) {
        for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)fill_blocks * 256) p[i] = 0ull;
        return;
    }
    const int r = (int)(blockIdx.x - fill_blocks) * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= rows.blocks * rows.B) return;
    const int i = r / rows.B, len = rows.len[i];
    const float* const v = h0 + rows.off[i] + (size_t)(r - i * rows.B) * len;
    bool out = false;
    for (int k = lane; k < len; k += 8 * 64) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = v[min(k + 64 * u, len - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) out |= !(fabsf(x[u]) <= 1.f);
    }
    const bool any = __ballot(out) != 0;   // (lanes past the end leave the loop a round early: false)
    if (lane == 0) beyond[r] = any;
}
hipError_t launch_fill_and_check(unsigned long long* p, size_t n, const float* h0, const StateRows& rows, unsigned* beyond, hipStream_t s)
{
    const unsigned fill_blocks = n > 0 ? (unsigned)grid_for(n, 256) : 0u, checks = (unsigned)((rows.blocks * (size_t)rows.B + 3) / 4);
    hipLaunchKernelGGL(fill_and_check_kernel, dim3(fill_blocks + checks), dim3(256), 0, s, p, n, fill_blocks, h0, rows, beyond);
    return hipGetLastError();
}
hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n16, 256)), dim3(256), 0, s, (float4*)dst, (const float4*)src, n16);
    return hipGetLastError();
}

// rows [rows][parts * part_cols] (pitch src_ld) -> [rows][parts * part_pitch], each part padded with zeros
template <typename E>
__global__ __launch_bounds__(256) void pad_rows_kernel(const E* __restrict__ src, int src_ld, int rows, int parts, int part_cols,
                                                       int part_pitch, E* __restrict__ dst)
{
    const int ld = parts * part_pitch;
    for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += gridDim.x * 4)
        for (int c = threadIdx.x & 63; c < ld; c += 64) {
            const int p = c / part_pitch, k = c - p * part_pitch;
            dst[(size_t)r * ld + c] = k < part_cols ? src[(size_t)r * src_ld + p * part_cols + k] : (E)0;
        }
}
hipError_t launch_pad_rows(const void* src, bool bf16, int src_ld, int rows, int parts, int part_cols, int part_pitch, void* dst, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)std::min((rows + 3) / 4, 8192)), block(256);
    if (bf16)
        hipLaunchKernelGGL(pad_rows_kernel<uint16_t>, grid, block, 0, s, (const uint16_t*)src, src_ld, rows, parts, part_cols, part_pitch, (uint16_t*)dst);
    else
        hipLaunchKernelGGL(pad_rows_kernel<float>, grid, block, 0, s, (const float*)src, src_ld, rows, parts, part_cols, part_pitch, (float*)dst);
    return hipGetLastError();
}

int device_num_cus()
{
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cached = n;
        else
            cached = 256;
    }
    return cached;
}

// The limit belongs to the device as well as the kernel.  It is set once for each pair (or again for a larger size); a call
// that fails leaves nothing behind, so the next one tries again.
hipError_t allow_dynamic_lds(const void* kernel, size_t bytes)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void*>, size_t> allowed;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    const auto it = allowed.find({dev, kernel});
    if (it != allowed.end() && it->second >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) allowed[{dev, kernel}] = bytes;
    return e;
}

// ---- scratch of the calls that have no handle and wait for their result (mask updates, compaction) -----------------
// A hipMalloc / hipFree pair per call costs more than the kernels of a small matrix, so each GPU keeps a few areas in a
// file-scope device array (part of the loaded code object, like the code itself: given back when that is unloaded) and a
// line of pinned host memory per area for the counts a call returns.  A call takes a free area for as long as it runs;
// further concurrent calls, and those that need more than an area holds, allocate their own and free it.
namespace {
constexpr int kAreas = 4, kScratchDevices = 64;
constexpr size_t kAreaBytes = 512 * 1024, kHostLine = 64;
static __device__ __align__(256) unsigned char scratch_areas[kAreas * kAreaBytes];
std::mutex g_areas_mutex;
struct DeviceAreas {
    char* base = nullptr;
    char* host = nullptr;
    bool busy[kAreas] = {};
} g_areas[kScratchDevices];
}  // namespace

hipError_t take_scratch(size_t bytes, ScratchArea* out)
{
    *out = ScratchArea{};
    hipError_t e = hipGetDevice(&out->device);
    if (e != hipSuccess) return e;
    if (bytes <= kAreaBytes && out->device >= 0 && out->device < kScratchDevices) {
        std::lock_guard<std::mutex> lock(g_areas_mutex);
        DeviceAreas& a = g_areas[out->device];
        if (!a.base) {
            void *d = nullptr, *h = nullptr;
            e = hipGetSymbolAddress(&d, HIP_SYMBOL(scratch_areas));
            if (e == hipSuccess) e = hipHostMalloc(&h, kAreas * kHostLine, hipHostMallocDefault);
            if (e != hipSuccess) return e;
            a.base = (char*)d;
            a.host = (char*)h;
        }
        for (int i = 0; i < kAreas; ++i)
            if (!a.busy[i]) {
                a.busy[i] = true;
                out->area = i;
                out->dev = a.base + (size_t)i * kAreaBytes;
                out->host = a.host + (size_t)i * kHostLine;
                return hipSuccess;
            }
    }
    e = hipMalloc(&out->dev, bytes);
    if (e == hipSuccess) e = hipHostMalloc(&out->host, kHostLine, hipHostMallocDefault);
    if (e != hipSuccess) give_scratch(*out);
    return e;
}

// the kernels that use the area have completed
void give_scratch(ScratchArea& a)
{
    if (a.area >= 0) {
        std::lock_guard<std::mutex> lock(g_areas_mutex);
        g_areas[a.device].busy[a.area] = false;
    } else {
        if (a.dev) (void)hipFree(a.dev);
        if (a.host) (void)hipHostFree(a.host);
    }
    a = ScratchArea{};
}

}  // namespace l355
