// Device-side helpers shared by the kernels of libdc_mi355x (gfx950, wave64): 128-bit streaming
// accesses, LDS by integer address, cross-lane primitives.
#ifndef DC_DEVICE_H
#define DC_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dcdev {

constexpr int kMaxDevices = 64; // GPUs that the library keeps something about

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 128-bit streaming accesses for data that is touched once.
__device__ __forceinline__ void store16_stream(void *p, uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    u32x4 v = {a, b, c, d};
    __builtin_nontemporal_store(v, static_cast<u32x4 *>(p));
}
__device__ __forceinline__ u32x4 load16_stream(const void *p)
{
    return __builtin_nontemporal_load(static_cast<const u32x4 *>(p));
}

// `bytes` bytes from an address on (both the same in all lanes) into which 16-byte stores go by offset; a lane that gives kNowhere
// stores nothing, though the instruction is issued.
class StoreWindow {
public:
    static constexpr uint32_t kNowhere = 0x80000000u; // beyond any window
    __device__ __forceinline__ StoreWindow(uint8_t *base, uint32_t bytes)
#ifdef __AMDGCN__
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000)) {} // untyped 32-bit data, no swizzle
#else
        : base(base), bytes(bytes) {}
#endif
    __device__ __forceinline__ void store16(uint32_t offset, const u32x4 &v) const
    {
#ifdef __AMDGCN__
        __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)offset, 0, 0);
#else
        if (offset != kNowhere && offset + 16 <= bytes) *reinterpret_cast<u32x4 *>(base + offset) = v;
#endif
    }

private:
#ifdef __AMDGCN__
    __amdgpu_buffer_rsrc_t rsrc;
#else
    uint8_t *base;
    uint32_t bytes;
#endif
};

// LDS accessed through 32-bit byte addresses, so that address arithmetic stays in one VALU operation.
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
__device__ __forceinline__ uint32_t lds_load32(uint32_t addr) { return *(const lds_u32 *)(uintptr_t)addr; }
__device__ __forceinline__ uint32_t lds_load16(uint32_t addr) { return *(const lds_u16 *)(uintptr_t)addr; }

// The compiler moves no instruction across this place.
__device__ __forceinline__ void keep_order()
{
#ifdef __AMDGCN__
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// The value is taken as a new one: what follows from it is worked out here, not ahead of a loop and kept.
__device__ __forceinline__ void anew(uint32_t &v)
{
#ifdef __AMDGCN__
    asm volatile("" : "+v"(v));
#endif
}

// All of these, the same in all lanes, are in their registers from here on: none is asked for once another has come.
__device__ __forceinline__ void in_registers(const u32x4 &a, uint64_t b, uint32_t c, uint32_t d)
{
#ifdef __AMDGCN__
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
#endif
}

// The value is in its register from here on (SAME: it is the same in all lanes, a scalar register): it is not worked out later, and
// a loop behind this place does not wait for the load that it came from.
template <bool SAME, typename T> __device__ __forceinline__ void in_register(const T &v)
{
#ifdef __AMDGCN__
    if constexpr (SAME) asm volatile("" ::"s"(v));
    else asm volatile("" ::"v"(v));
#endif
}

// Value of another lane through the data-parallel primitives; lanes without a source (and rows that
// the row mask leaves out) read 0.  0x110 + n: n lanes to the right inside a row of 16; 0x142 / 0x143:
// lane 15 of a row to the next row / lane 31 to rows 2 and 3; 0x138: one lane to the right over
// the whole wave.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}

// v with the value of one lane (the same number in all lanes) replaced by w (the same in all lanes).
// (The compiler has no builtin for the instruction, so the intrinsic is taken by its name; a compiler that calls it otherwise ends the build.
// Not an instruction in inline asm: the waits that it may need behind the one that made w scalar are the compiler's to put there.  A comparison and
// a selection in its place are 1 to 2 % of a decode of short chunks: 16000 of 4 KiB 37.7 instead of 36.8 us, 6000 of 8 KiB 21.9 instead of 21.6.)
#ifdef __AMDGCN__
extern "C" __device__ uint32_t dc_llvm_writelane(uint32_t w, uint32_t lane, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
#endif
__device__ __forceinline__ uint32_t with_lane(uint32_t v, uint32_t lane, uint32_t w)
{
#ifdef __AMDGCN__
    return dc_llvm_writelane(w, lane, v);
#else
    return (threadIdx.x & 63u) == lane ? w : v;
#endif
}

// Inclusive prefix sum over the 64 lanes (HALVES: over each half of 32 lanes on its own).
template <bool HALVES> __device__ __forceinline__ uint32_t lanes_prefix_sum(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v);
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    v += dpp_or_zero<0x142, 0xA>(v);
    if (!HALVES) v += dpp_or_zero<0x143, 0xC>(v);
    return v;
}

// For every lane the last non-zero value among the lanes below it (0 if none).
template <bool HALVES> __device__ __forceinline__ uint32_t lanes_last_nonzero_below(uint32_t v)
{
    uint32_t t;
    v = dpp_or_zero<0x138, 0xF>(v);
    t = dpp_or_zero<0x111, 0xF>(v); v = v ? v : t;
    t = dpp_or_zero<0x112, 0xF>(v); v = v ? v : t;
    t = dpp_or_zero<0x114, 0xF>(v); v = v ? v : t;
    t = dpp_or_zero<0x118, 0xF>(v); v = v ? v : t;
    t = dpp_or_zero<0x142, 0xA>(v); v = v ? v : t;
    if (!HALVES) { t = dpp_or_zero<0x143, 0xC>(v); v = v ? v : t; }
    return v;
}

// For every lane the largest value among the lanes below it (0 if none).
template <bool HALVES> __device__ __forceinline__ uint32_t lanes_largest_below(uint32_t v)
{
    auto with = [&](uint32_t t) { v = t > v ? t : v; };
    v = dpp_or_zero<0x138, 0xF>(v);
    if (HALVES) v = threadIdx.x & 31u ? v : 0u;
    with(dpp_or_zero<0x111, 0xF>(v));
    with(dpp_or_zero<0x112, 0xF>(v));
    with(dpp_or_zero<0x114, 0xF>(v));
    with(dpp_or_zero<0x118, 0xF>(v));
    with(dpp_or_zero<0x142, 0xA>(v));
    if (!HALVES) with(dpp_or_zero<0x143, 0xC>(v));
    return v;
}

// Sum over the 64 lanes, result in lane 63.
__device__ __forceinline__ float lanes_sum(float v)
{
#define DC_SUM_STEP(CTRL, MASK) v += __uint_as_float(dpp_or_zero<CTRL, MASK>(__float_as_uint(v)));
    DC_SUM_STEP(0x111, 0xF)
    DC_SUM_STEP(0x112, 0xF)
    DC_SUM_STEP(0x114, 0xF)
    DC_SUM_STEP(0x118, 0xF)
    DC_SUM_STEP(0x142, 0xA)
    DC_SUM_STEP(0x143, 0xC)
#undef DC_SUM_STEP
    return v;
}
__device__ __forceinline__ int32_t lanes_sum(int32_t v)
{
    return __builtin_bit_cast(int32_t, lanes_prefix_sum<false>(__builtin_bit_cast(uint32_t, v)));
}

} // namespace dcdev

// Records the launch status of the calling thread (dc_last_hip_error() reports it); DC_OK or DC_E_HIP.
int dc_launch_status();

#endif // DC_DEVICE_H
