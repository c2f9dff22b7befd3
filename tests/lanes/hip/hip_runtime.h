// Stands in for the HIP runtime header when a device source of the library is compiled for the CPU: a launch runs the
// kernel's workgroups one after the other, in the order the caller chooses for the lanes (first to last, last to first, shuffled),
// every lane as a fiber of its own that runs alone until it has to meet others.
//
// Lanes meet where the source says so: at a barrier, a wave barrier, or an operation that reads other lanes (ballot, DPP,
// shuffle, readlane), which waits for all lanes of the wave that have not returned.  Between two meetings every lane runs
// alone, in an order that the caller chooses, and LDS is filled with arbitrary bytes before every workgroup.  So a value that
// is read before it is written, or an access that is only right because the lanes of a wave keep in step, gives results that
// depend on the order or on the fill.
#ifndef LANES_HIP_RUNTIME_H
#define LANES_HIP_RUNTIME_H

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <setjmp.h>
#include <ucontext.h>
#include <unistd.h>

#include <algorithm>
#include <functional>
#include <random>
#include <vector>

#define __global__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static __attribute__((section("lds_vars")))
extern "C" char __start_lds_vars[], __stop_lds_vars[];

struct dim3 {
    uint32_t x, y, z;
    dim3(uint32_t x_ = 1, uint32_t y_ = 1, uint32_t z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

namespace lanes {

enum Order { kAscending, kDescending, kShuffled };
struct Config { Order order = kAscending; uint64_t seed = 1; int compute_units = 256; };
inline Config config;

enum class Meet { none, wave, block };
struct Lane {
    ucontext_t start;
    jmp_buf at;
    std::vector<char> stack;
    bool started = false, done = false;
    Meet waits = Meet::none;
    const char *op = nullptr; // the operation the lane waits at
    uint32_t meetings = 0;    // of its wave: which half of the exchange is in use
    uint32_t tid = 0;
};
struct Wave {
    uint64_t value[2][64]; // what the lanes bring to a meeting, two meetings in turn
    uint64_t there[2];     // which lanes came
};

inline std::vector<Lane> lane;
inline std::vector<Wave> wave;
inline uint32_t now = 0, threads = 0; // the lane that runs; lanes of the workgroup
inline uint32_t counted = 0;          // __syncthreads_count
inline jmp_buf scheduler;
inline std::function<void()> body;
inline std::mt19937_64 strays;

inline void fail(const char *what)
{
    fprintf(stderr, "%s\n", what);
    _exit(3);
}
inline void wait(Meet kind, const char *op)
{
    lane[now].waits = kind;
    lane[now].op = op;
    if (!_setjmp(lane[now].at)) _longjmp(scheduler, 1);
}
// Brings v to the wave's next meeting and returns the meeting: all values are there.
inline uint32_t meet(uint64_t v, const char *op)
{
    Wave &w = wave[now / 64];
    const uint32_t half = lane[now].meetings++ & 1u;
    w.value[half][now & 63u] = v;
    w.there[half] |= 1ull << (now & 63u);
    wait(Meet::wave, op);
    return half;
}
inline bool came(uint32_t half, uint32_t l) { return wave[now / 64].there[half] >> l & 1u; }
inline uint64_t from(uint32_t half, uint32_t l)
{
    // the register of a lane that has returned holds anything
    return came(half, l) ? wave[now / 64].value[half][l] : strays();
}
inline void run_lane()
{
    body();
    lane[now].done = true;
    _longjmp(scheduler, 1);
}

// Releases the lanes of [first, last) if all of them that have not returned wait for `kind`.
inline bool release(uint32_t first, uint32_t last, Meet kind)
{
    const char *op = nullptr;
    for (uint32_t i = first; i < last; i++) {
        if (lane[i].done) continue;
        if (lane[i].waits != kind) return false;
        if (op && strcmp(op, lane[i].op)) fail("lanes of one wave wait at different operations");
        op = lane[i].op;
    }
    if (!op) return false;
    for (uint32_t i = first; i < last; i++) lane[i].waits = Meet::none;
    if (kind == Meet::wave) { // the other half of the exchange is free now
        for (uint32_t i = first; i < last; i++)
            if (!lane[i].done) {
                wave[first / 64].there[lane[i].meetings & 1u] = 0;
                break;
            }
    }
    return true;
}

inline void run_block(uint32_t n_threads, std::mt19937_64 &rng)
{
    for (char *p = __start_lds_vars; p < __stop_lds_vars; p++) *p = (char)rng();
    threads = n_threads;
    if (lane.size() < n_threads) lane.resize(n_threads);
    wave.assign((n_threads + 63) / 64, Wave{});
    counted = 0;
    std::vector<uint32_t> order(n_threads);
    for (uint32_t i = 0; i < n_threads; i++) {
        Lane &l = lane[i];
        if (l.stack.empty()) l.stack.resize(64 << 10);
        l.started = l.done = false;
        l.waits = Meet::none;
        l.meetings = 0;
        l.tid = i;
        order[i] = config.order == kDescending ? n_threads - 1 - i : i;
    }
    for (;;) {
        if (config.order == kShuffled) std::shuffle(order.begin(), order.end(), rng);
        static volatile uint32_t at, ran, left;
        ran = left = 0;
        for (at = 0; at < n_threads; at = at + 1) {
            Lane &l = lane[order[at]];
            if (l.done) continue;
            left = left + 1;
            if (l.waits != Meet::none) continue;
            ran = ran + 1;
            now = order[at];
            if (!_setjmp(scheduler)) {
                if (l.started) _longjmp(l.at, 1);
                l.started = true;
                getcontext(&l.start);
                l.start.uc_stack.ss_sp = l.stack.data();
                l.start.uc_stack.ss_size = l.stack.size();
                l.start.uc_link = nullptr;
                makecontext(&l.start, run_lane, 0);
                setcontext(&l.start);
            }
        }
        if (!left) return;
        bool released = false;
        for (uint32_t w = 0; w < n_threads; w += 64) released |= release(w, std::min(w + 64, n_threads), Meet::wave);
        if (!released) released = release(0, n_threads, Meet::block);
        if (!released && !ran) fail("no lane can go on");
    }
}

template <typename Kernel, typename... Args> void launch(Kernel kernel, dim3 grid, dim3 block, Args... args);

// ---- operations that read other lanes
inline uint64_t ballot(bool v, const char *op)
{
    const uint32_t h = meet(v, op);
    uint64_t m = 0;
    for (uint32_t l = 0; l < 64; l++) m |= came(h, l) && from(h, l) ? 1ull << l : 0ull;
    return m;
}
// The source lane of a DPP control in a wave of 64, or -1.
inline int dpp_source(int ctrl, int l)
{
    const int row = l & ~15, in = l & 15;
    if (ctrl < 0x100) return (l & ~3) | (ctrl >> 2 * (l & 3) & 3);         // quad_perm
    if (ctrl > 0x110 && ctrl < 0x120) return in >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1; // row_shr
    if (ctrl > 0x120 && ctrl < 0x130) return row | ((in - (ctrl - 0x120)) & 15);            // row_ror
    if (ctrl == 0x130) return l < 63 ? l + 1 : -1;                         // wave_shl
    if (ctrl == 0x138) return l > 0 ? l - 1 : -1;                          // wave_shr
    if (ctrl == 0x142) return l >= 16 ? row - 1 : -1;                      // lane 15 of a row to the next row
    if (ctrl == 0x143) return l >= 32 ? 31 : -1;                           // lane 31 to rows 2 and 3
    fail("a DPP control that is not modelled");
    return -1;
}

} // namespace lanes

#define threadIdx (dim3(lanes::lane[lanes::now].tid))
inline dim3 blockIdx, gridDim;

template <typename Kernel, typename... Args> void lanes::launch(Kernel kernel, dim3 grid, dim3 block, Args... args)
{
    std::mt19937_64 rng(config.seed);
    gridDim = grid;
    body = [&] { kernel(args...); };
    std::vector<uint32_t> order(grid.x);
    for (uint32_t b = 0; b < grid.x; b++) order[b] = config.order == kDescending ? grid.x - 1 - b : b;
    if (config.order == kShuffled) std::shuffle(order.begin(), order.end(), rng);
    for (uint32_t b : order) {
        blockIdx = dim3(b);
        run_block(block.x, rng);
    }
}
namespace lanes { inline std::vector<const char *> launched; } // the kernels' names as the source writes them
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    (lanes::launched.push_back(#kernel), lanes::launch(kernel, grid, block, __VA_ARGS__))

inline void __syncthreads() { lanes::wait(lanes::Meet::block, "__syncthreads"); }
inline int __syncthreads_count(int v)
{
    if (v) lanes::counted++;
    lanes::wait(lanes::Meet::block, "__syncthreads_count");
    const uint32_t n = lanes::counted;
    lanes::wait(lanes::Meet::block, "__syncthreads_count, read");
    lanes::counted = 0;
    lanes::wait(lanes::Meet::block, "__syncthreads_count, cleared");
    return (int)n;
}
#define __builtin_amdgcn_wave_barrier() ((void)lanes::meet(0, "wave barrier"))
#define __builtin_amdgcn_fence(order, scope) ((void)0) // a fence orders a lane's own accesses: they are in order here
inline uint64_t __ballot(int v) { return lanes::ballot(v != 0, "ballot"); }
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int row_mask, int bank_mask, bool bound_ctrl)
{
    const uint32_t h = lanes::meet((uint32_t)v, "dpp");
    const int l = (int)(lanes::now & 63u), from = lanes::dpp_source(ctrl, l);
    if (!(row_mask >> (l / 16) & 1) || !(bank_mask >> (l / 4 % 4) & 1)) return old;
    if (from < 0 || !lanes::came(h, (uint32_t)from)) return bound_ctrl ? 0 : old;
    return (int)lanes::from(h, (uint32_t)from);
}
inline int __builtin_amdgcn_mov_dpp(int v, int ctrl, int row_mask, int bank_mask, bool bound_ctrl)
{
    return __builtin_amdgcn_update_dpp(0, v, ctrl, row_mask, bank_mask, bound_ctrl);
}
inline int __any(int v) { return lanes::ballot(v != 0, "any") != 0; }
inline int __all(int v) { return lanes::ballot(v == 0, "all") == 0; }
inline int __shfl(int v, int l, int width = 64)
{
    const uint32_t h = lanes::meet((uint32_t)v, "shuffle"), base = (lanes::now & 63u) & ~(uint32_t)(width - 1);
    return (int)lanes::from(h, base + ((uint32_t)l & (uint32_t)(width - 1)));
}
inline int __shfl_xor(int v, int mask) { return (int)lanes::from(lanes::meet((uint32_t)v, "shuffle"), (lanes::now ^ (uint32_t)mask) & 63u); }
inline int __builtin_amdgcn_readlane(int v, uint32_t l)
{
    return (int)lanes::from(lanes::meet((uint32_t)v, "readlane"), l & 63u);
}
inline int __builtin_amdgcn_readfirstlane(int v)
{
    const uint32_t h = lanes::meet((uint32_t)v, "readfirstlane");
    uint32_t l = 0;
    while (!lanes::came(h, l)) l++;
    return (int)lanes::from(h, l);
}
struct lanes_pair { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
// rows of 16 lanes: the odd rows of a change places with the even rows of b
inline lanes_pair __builtin_amdgcn_permlane16_swap(uint32_t a, uint32_t b, bool, bool)
{
    const uint32_t h = lanes::meet((uint64_t)b << 32 | a, "row swap"), l = lanes::now & 63u;
    const uint64_t other = lanes::from(h, l ^ 16u);
    if (l & 16u) return {{(uint32_t)(other >> 32), b}};
    return {{a, (uint32_t)other}};
}
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t c)
{
    const uint32_t l = lanes::now & 63u;
    return c + (uint32_t)__builtin_popcount(l < 32 ? m & ((1u << l) - 1u) : m);
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t c)
{
    const uint32_t l = lanes::now & 63u;
    return c + (l <= 32 ? 0u : (uint32_t)__builtin_popcount(m & ((1u << (l - 32)) - 1u)));
}
inline float __builtin_amdgcn_rcpf(float v) { return 1.0f / v; }
template <typename T> T atomicAdd(T *p, T v) { const T old = *p; *p = old + v; return old; }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline uint32_t __brev(uint32_t v)
{
    uint32_t r = 0;
    for (int i = 0; i < 32; i++) r |= (v >> i & 1u) << (31 - i);
    return r;
}
inline uint32_t __float_as_uint(float v) { uint32_t r; memcpy(&r, &v, 4); return r; }
inline float __uint_as_float(uint32_t v) { float r; memcpy(&r, &v, 4); return r; }

// ---- operations of one lane
inline uint32_t __builtin_amdgcn_alignbit(uint32_t hi, uint32_t lo, uint32_t n) { return (uint32_t)(((uint64_t)hi << 32 | lo) >> (n & 31u)); }
inline uint32_t __builtin_amdgcn_alignbyte(uint32_t hi, uint32_t lo, uint32_t n) { return (uint32_t)(((uint64_t)hi << 32 | lo) >> 8 * (n & 3u)); }
inline uint32_t __builtin_amdgcn_ubfe(uint32_t v, uint32_t at, uint32_t width)
{
    return (v >> (at & 31u)) & ((1u << (width & 31u)) - 1u);
}
inline uint32_t __builtin_amdgcn_perm(uint32_t a, uint32_t b, uint32_t select)
{
    const uint64_t both = (uint64_t)a << 32 | b;
    uint32_t r = 0;
    for (int i = 0; i < 4; i++) {
        const uint32_t s = select >> 8 * i & 0xFFu;
        if (s > 7 && s != 12) lanes::fail("a byte selector that is not modelled");
        r |= s == 12 ? 0u : (uint32_t)(both >> 8 * s & 0xFFu) << 8 * i;
    }
    return r;
}
template <typename V> float __builtin_amdgcn_fdot2_f32_bf16(V a, V b, float c, bool)
{
    return (float)a[0] * (float)b[0] + ((float)a[1] * (float)b[1] + c);
}
inline int __builtin_amdgcn_sdot4(int a, int b, int c, bool)
{
    for (int i = 0; i < 4; i++) c += (int)(int8_t)(a >> 8 * i) * (int)(int8_t)(b >> 8 * i);
    return c;
}
inline int __builtin_amdgcn_s_getreg(int) { return 0; }
inline uint64_t wall_clock64() { return 0; }
extern "C" inline __attribute__((used)) __bf16 __truncsfbf2(float v) // to nearest, ties to even
{
    uint32_t b = __float_as_uint(v);
    b += 0x7FFFu + (b >> 16 & 1u);
    const uint16_t h = (uint16_t)(b >> 16);
    __bf16 r;
    memcpy(&r, &h, 2);
    return r;
}

// ---- the host side of a launch
typedef void *hipStream_t;
typedef int hipError_t;
constexpr hipError_t hipSuccess = 0;
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = lanes::config.compute_units; return hipSuccess; }
template <typename T> hipError_t hipGetSymbolAddress(void **p, T &v) { *p = (void *)&v; return hipSuccess; }
#define HIP_SYMBOL(v) v

#endif // LANES_HIP_RUNTIME_H
