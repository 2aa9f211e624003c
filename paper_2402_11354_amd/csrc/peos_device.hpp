// Device-side helpers shared by the PEOs kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace peos {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));  // in memory at any float

constexpr int kWave = 64;
constexpr uint32_t kEmpty = 0xFFFFFFFFu;   // empty visited-hash slot

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Ordering point for LDS traffic between the lanes of a one-wave workgroup.
// A wave's LDS operations execute in order, so a compiler-level barrier
// (a wavefront-scope fence) is enough; unlike __syncthreads it does not wait
// for outstanding global loads, which lets prefetches stay in flight.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Ordering point for one wave's own global-memory accesses (the visited
// bitmap and its cleanup list, which only the wave that searches the query
// touches): the fence keeps the compiler from moving accesses across it, and
// the wait holds the wave until those issued before are complete, so that a
// lane reads what another lane's atomic or store put there, whatever order
// the caches serve requests in.  No cache is written back or invalidated (an
// agent-scope fence would write back the whole L2 of the XCD, at every spill).
__device__ __forceinline__ void wave_mem_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt 0; the other counters at their maxima
    __builtin_amdgcn_wave_barrier();
}

// number of lanes of the mask below this one (no lane mask kept in registers)
__device__ __forceinline__ int lanes_before(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ int popc(uint64_t x) { return __popcll(x); }

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t wave_uniform(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ float wave_uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// value of v in lane t (t uniform across the wave), as a scalar
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int t)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, t);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), t);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// 64 bytes a row by four lanes: lane l of the load holds 16-byte chunk l % 4
// of row l / 4 (consecutive lanes share a row, so the 64 bytes are one
// access; with a row per lane of 16 every lane's 16 bytes are an access of
// their own, and the vector caches serve one a cycle).  by_row moves them to
// the matrix cores' layout: lane 16 c + r receives chunk c of row r.
__device__ __forceinline__ float4 by_row(float4 v)
{
    const int l = lane_id();
    const int from = 4 * (4 * (l & 15) + (l >> 4));
    auto move = [&](float x) { return __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(x))); };
    return make_float4(move(v.x), move(v.y), move(v.z), move(v.w));
}

// value of v in lane (this lane xor O), all lanes active: lane swaps within
// quads are DPP moves (no LDS round trip), xor 4 / 8 / 16 a swizzle, wider
// ones a permute through the LDS crossbar
template <int O>
__device__ __forceinline__ float xor_lane(float v)
{
    static_assert(O >= 1 && O < 64 && (O & (O - 1)) == 0, "power of two below 64");
    const int b = __float_as_int(v);
    if (O == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, false));
    if (O == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x4E, 0xF, 0xF, false));
    if (O < 32) return __int_as_float(__builtin_amdgcn_ds_swizzle(b, 0x1F | (O << 10)));
    return __shfl_xor(v, O, kWave);
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += xor_lane<32>(v);
    v += xor_lane<16>(v);
    v += xor_lane<8>(v);
    v += xor_lane<4>(v);
    v += xor_lane<2>(v);
    v += xor_lane<1>(v);
    return v;
}

__device__ __forceinline__ int wave_sum_int(int v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// smallest value of the wave, as a scalar: four steps within rows of 16 lanes
// and two across them, each a DPP move and a minimum (no LDS round trip)
__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    auto step = [&](uint32_t o) { v = o < v ? o : v; };
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x111, 0xF, 0xF, false));  // row_shr:1
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x112, 0xF, 0xF, false));  // row_shr:2
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x114, 0xF, 0xF, false));  // row_shr:4
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x118, 0xF, 0xF, false));  // row_shr:8
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xF, 0xF, false));  // row_bcast:15
    step((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xF, 0xF, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// total order on (distance, id): map a float to an unsigned key that sorts
// like the float (negative values reversed), then append the id.
__device__ __forceinline__ uint32_t order_bits(float f)
{
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float bits_value(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k);
}

__device__ __forceinline__ uint64_t sort_key(float d, uint32_t id)
{
    return (static_cast<uint64_t>(order_bits(d)) << 32) | id;
}

}  // namespace peos
