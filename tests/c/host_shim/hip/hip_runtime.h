// What fmb_device.h needs of the HIP headers, for the CPU: vector types, math names and a wave of 64 lanes
// run as coroutines that meet at every cross-lane operation (host_wave below).
#pragma once
#include <ucontext.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __restrict__

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline int __float_as_int(float x) { int i; memcpy(&i, &x, 4); return i; }
inline unsigned __float_as_uint(float x) { unsigned i; memcpy(&i, &x, 4); return i; }
inline float __int_as_float(int i) { float x; memcpy(&x, &i, 4); return x; }
inline float __uint_as_float(unsigned i) { float x; memcpy(&x, &i, 4); return x; }
inline int __clz(int x) { return x ? __builtin_clz((unsigned)x) : 32; }

namespace hostwave {
constexpr int kLanes = 64, kStack = 256 << 10;
struct Wave {
    ucontext_t back, lane_ctx[kLanes];
    std::vector<char> stacks = std::vector<char>((size_t)kLanes * kStack);
    std::function<void(int)> body;
    int lane = 0;
    bool done[kLanes];
    int values[2][kLanes];
};
inline Wave &wave() { static Wave w; return w; }
inline void entry()
{
    Wave &w = wave();
    const int l = w.lane;
    w.body(l);
    w.done[l] = true;
    swapcontext(&w.lane_ctx[l], &w.back);
}
// Hands x to the wave and returns every lane's value once all lanes have met here.
inline const int *meet(int x)
{
    Wave &w = wave();
    static thread_local int turn[kLanes];
    const int l = w.lane, k = turn[l] ^= 1;
    w.values[k][l] = x;
    swapcontext(&w.lane_ctx[l], &w.back);
    return w.values[k];
}
// Runs body(lane) on 64 lanes in step; every lane takes the same cross-lane operations.
inline void run(std::function<void(int)> body)
{
    Wave &w = wave();
    w.body = std::move(body);
    for (int l = 0; l < kLanes; ++l) {
        getcontext(&w.lane_ctx[l]);
        w.lane_ctx[l].uc_stack.ss_sp = &w.stacks[(size_t)l * kStack];
        w.lane_ctx[l].uc_stack.ss_size = kStack;
        w.lane_ctx[l].uc_link = nullptr;
        makecontext(&w.lane_ctx[l], entry, 0);
        w.done[l] = false;
    }
    for (bool any = true; any;) {
        any = false;
        for (w.lane = 0; w.lane < kLanes; ++w.lane)
            if (!w.done[w.lane]) {
                swapcontext(&w.back, &w.lane_ctx[w.lane]);
                any = any || !w.done[w.lane];
            }
    }
}
// The DPP moves that the reductions use: row shifts right, rotation by 8, broadcasts of lanes 15 and 31.
inline int dpp(int old, int src, int ctrl, int rows, int banks, bool zero)
{
    const int *v = meet(src);
    const int l = wave().lane, row = l / 16, in = l % 16;
    int from = -1;
    if (ctrl >= 0x111 && ctrl <= 0x11F) from = in >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    if (ctrl == 0x142) from = row > 0 ? 16 * row - 1 : -1;
    if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
    if (!((rows >> row) & 1)) return old;
    (void)banks;
    return from >= 0 ? v[from] : zero ? 0 : old;
}
inline unsigned long long ballot(bool p)
{
    const int *v = meet(p);
    unsigned long long m = 0;
    for (int l = 0; l < kLanes; ++l) m |= (unsigned long long)(v[l] != 0) << l;
    return m;
}
struct Pair {
    unsigned a, b;
    unsigned operator[](int i) const { return i ? b : a; }
};
}  // namespace hostwave

#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_sqrtf(x) sqrtf(x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_logf(x) log2f(x)
#define __builtin_amdgcn_ballot_w64(p) hostwave::ballot(p)
#define __builtin_amdgcn_update_dpp(old, src, ctrl, rows, banks, zero) hostwave::dpp(old, src, ctrl, rows, banks, zero)
#define __builtin_amdgcn_readlane(x, l) (hostwave::meet(x)[l])
// (wave_sum16's swaps: compiled, not run here)
#define __builtin_amdgcn_permlane32_swap(a, b, x, y) (hostwave::Pair{a, b})
#define __builtin_amdgcn_permlane16_swap(a, b, x, y) (hostwave::Pair{a, b})

using std::isfinite;
typedef void *hipStream_t;
