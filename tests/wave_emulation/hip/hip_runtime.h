// What csrc/ctf_device.h needs to compile for the host, with the 64 lanes of a
// wave as coroutines: a lane runs until the next wave-wide step (an LDS sync,
// a ballot, a cross-lane read), then the next lane runs.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#define __device__
#define __host__
#define __global__
#define __shared__
#define __forceinline__ inline

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct int2 { int x, y; };
struct int4 { int x, y, z, w; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline int2 make_int2(int x, int y) { return {x, y}; }
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
struct Dim { unsigned x, y, z; };
extern Dim threadIdx, blockIdx, blockDim, gridDim;

namespace wave {
constexpr int kLanes = 64;
extern int lane;              // the running lane
void step();                  // run the other lanes up to here
extern uint64_t slot[kLanes];
template <class V> inline void give(V v) { uint64_t b = 0; memcpy(&b, &v, sizeof v); slot[lane] = b; step(); }
template <class V> inline V of(int l) { V v; memcpy(&v, &slot[l], sizeof v); return v; }
inline uint64_t ballot(bool p)
{
    give<uint64_t>(p);
    uint64_t m = 0;
    for (int l = 0; l < kLanes; ++l) m |= slot[l] << l;
    step();
    return m;
}
inline int read(int v, int l)
{
    give(v);
    const int r = of<int>(l);
    step();
    return r;
}
// DPP: row shifts right (0x111..0x11f) and the row broadcasts 15 and 31
inline int dpp(int old, int v, int ctrl, int rows)
{
    give(v);
    const int row = lane / 16, in = lane % 16;
    int src = -1;
    if (ctrl > 0x110 && ctrl < 0x120) src = in >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
    else if (ctrl == 0x142) src = row > 0 ? 16 * row - 1 : -1;
    else if (ctrl == 0x143) src = row > 1 ? 31 : -1;
    const int r = src >= 0 && (rows >> row & 1) ? of<int>(src) : old;
    step();
    return r;
}
}  // namespace wave

inline int __lane_id() { return wave::lane; }
inline int __popc(uint32_t m) { return __builtin_popcount(m); }
inline int __popcll(uint64_t m) { return __builtin_popcountll(m); }
inline void __syncthreads() {}
inline int __mul24(int a, int b) { return a * b; }
inline float __int_as_float(int v) { float f; memcpy(&f, &v, 4); return f; }
inline int __float_as_int(float f) { int v; memcpy(&v, &f, 4); return v; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint64_t)a * b >> 32; }
template <class T> inline T atomicAdd(T* p, T v) { T o = *p; *p += v; return o; }

#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() wave::step()
#define __builtin_amdgcn_ballot_w64(p) wave::ballot(p)
#define __builtin_amdgcn_inverse_ballot_w64(m) ((m) >> wave::lane & 1)
#define __builtin_amdgcn_readlane(v, l) wave::read(v, l)
#define __builtin_amdgcn_readfirstlane(v) wave::read(v, 0)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) wave::dpp(old, v, ctrl, rows)
#define __builtin_amdgcn_mov_dpp(v, ctrl, rows, banks, bound) wave::dpp(0, v, ctrl, rows)
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t a)
{
    return a + __builtin_popcount(wave::lane < 32 ? m & ((1u << wave::lane) - 1u) : m);
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t a)
{
    return a + (wave::lane < 32 ? 0 : __builtin_popcount(m & (uint32_t)((1ull << (wave::lane - 32)) - 1u)));
}
inline uint32_t __builtin_amdgcn_sad_u8(uint32_t a, uint32_t b, uint32_t c)
{
    for (int i = 0; i < 32; i += 8) c += abs((int)(a >> i & 255) - (int)(b >> i & 255));
    return c;
}
inline uint32_t __builtin_amdgcn_alignbyte(uint32_t hi, uint32_t lo, uint32_t n)
{
    return (uint32_t)((((uint64_t)hi << 32) | lo) >> (8 * n));
}
inline uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    uint32_t r = 0;
    for (int i = 0; i < 4; ++i) {
        const uint32_t s = sel >> (8 * i) & 255;   // 0..7 only
        r |= ((s < 4 ? lo >> (8 * s) : hi >> (8 * (s - 4))) & 255) << (8 * i);
    }
    return r;
}
inline float __builtin_amdgcn_sinf(float x) { return sinf(6.2831853f * x); }
inline float __builtin_amdgcn_fractf(float x) { return x - floorf(x); }
