// Stand-in for the HIP runtime header that runs a kernel's source on the CPU, for tests of its index arithmetic and of
// its barriers.  A thread of a block is a fiber.  Between two barriers the waves run one after another, in the order
// `emu::wave_order` gives, and within a wave each lane runs on until it meets an operation across lanes: everything a
// barrier does not order happens in an order the hardware may or may not take, so a missing barrier shows as a wrong
// result.  Only what the kernels under test use is here.
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static  // one block at a time

struct dim3 {
    uint32_t x, y, z;
    dim3(uint32_t x_ = 1, uint32_t y_ = 1, uint32_t z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) double2 { double x, y; };
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline double2 make_double2(double x, double y) { return {x, y}; }
inline float __uint_as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
inline uint32_t __float_as_uint(float f) { return __builtin_bit_cast(uint32_t, f); }
typedef void* hipStream_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidConfiguration = 9 };

namespace emu {

constexpr int kLanes = 64;
constexpr size_t kStack = 256 << 10;
enum class Wait { none, lanes, block, over };

struct Fiber {
    ucontext_t ctx;
    std::vector<char> stack;
    dim3 tid;
    Wait wait = Wait::none;
    uint64_t in[4];  // operands of the operation across lanes that the fiber waits in
};

inline std::vector<Fiber> fibers;
inline ucontext_t scheduler;
inline Fiber* self = nullptr;
inline dim3 block_idx, block_dim, grid_dim;
inline std::function<void()> body;
inline std::function<int(int, int)> wave_order = [](int i, int) { return i; };  // the i-th wave to run, of n
inline std::function<bool(dim3)> wanted = [](dim3) { return true; };            // blocks to run

inline void pause(Wait w) {
    self->wait = w;
    swapcontext(&self->ctx, &scheduler);
}
inline int lane() { return (int)(self - fibers.data()) % kLanes; }
inline Fiber* wave() { return self - lane(); }

// every lane's operand; the caller must not pause again before it has read the others'
template <typename T>
void exchange(T v, int slot = 0) {
    static_assert(sizeof(T) <= 16, "two words");
    memcpy(&self->in[slot], &v, sizeof(T));
}
template <typename T>
T operand(int of, int slot = 0) {
    T v;
    memcpy(&v, &wave()[of].in[slot], sizeof(T));
    return v;
}
// the operands may be overwritten once every lane has read them
template <typename F>
auto across(F read) {
    pause(Wait::lanes);
    auto r = read();
    pause(Wait::lanes);
    return r;
}

template <typename T>
T shfl(T v, int from) {
    exchange(v);
    return across([&] { return operand<T>(from & (kLanes - 1)); });
}
template <typename T>
T readfirstlane(T v) { return shfl(v, 0); }
inline uint64_t ballot(bool b) {
    exchange(b);
    return across([] {
        uint64_t m = 0;
        for (int i = 0; i < kLanes; ++i) m |= (uint64_t)operand<bool>(i) << i;
        return m;
    });
}
// 16 products of a 4 x 1 and a 1 x 4 tile, four lanes each: lane = 4 * block + row of A (column of B and D)
template <typename V>
V mfma_4x4x1(float a, float b, V c) {
    exchange(a);
    return across([&] {
        for (int i = 0; i < 4; ++i) c[i] = __builtin_fmaf(operand<float>((lane() & ~3) + i), b, c[i]);
        return c;
    });
}
// 16 x 16 outputs: lane = 16 * lq + li holds row (column) li of A (B), terms E lq .. E lq + E - 1, and rows 4 lq .. 4 lq + 3 of
// column li of the outputs.  The terms and the accumulator round once.
template <int E, typename A, typename V>
V mfma_16x16(A a, A b, V c) {
    struct Row { uint16_t x[E]; };
    exchange(a);
    exchange(b, 2);
    return across([&] {
        auto value = [](uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); };
        for (int r = 0; r < 4; ++r) {
            double s = c[r];
            for (int q = 0; q < 4; ++q) {
                const Row x = operand<Row>(16 * q + 4 * (lane() / 16) + r), y = operand<Row>(16 * q + lane() % 16, 2);
                for (int e = 0; e < E; ++e) s += (double)value(x.x[e]) * (double)value(y.x[e]);
            }
            c[r] = (float)s;
        }
        return c;
    });
}
// 16 lanes address 4 values each, lane i columns 4 (i % 4) on of row i / 4; lane i gets column i of the four rows
template <typename V>
V read_transposed(const void* p) {
    exchange(p);
    return across([&] {
        V v;
        const int l = lane() % 16, base = lane() - l;
        for (int e = 0; e < 4; ++e) v[e] = operand<const short*>(base + 4 * e + l / 4)[l % 4];
        return v;
    });
}

inline void entry() {
    body();
    self->wait = Wait::over;
    swapcontext(&self->ctx, &scheduler);
}

inline void run_block() {
    const int n = (int)(block_dim.x), waves = n / kLanes;
    if ((int)fibers.size() < n) fibers.resize(n);
    for (int t = 0; t < n; ++t) {
        Fiber& f = fibers[t];
        f.stack.resize(kStack);
        f.tid = dim3((uint32_t)t, 0, 0);
        f.wait = Wait::none;
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = f.stack.data();
        f.ctx.uc_stack.ss_size = kStack;
        f.ctx.uc_link = nullptr;
        makecontext(&f.ctx, entry, 0);
    }
    for (bool left = true; left;) {
        left = false;
        for (int i = 0; i < waves; ++i) {
            Fiber* w = &fibers[wave_order(i, waves) * kLanes];
            for (bool going = true; going;) {
                int at_lanes = 0, at_block = 0, over = 0;
                for (int l = 0; l < kLanes; ++l) {
                    if (w[l].wait == Wait::none || w[l].wait == Wait::lanes) {
                        self = &w[l];
                        swapcontext(&scheduler, &w[l].ctx);
                    }
                    at_lanes += w[l].wait == Wait::lanes;
                    at_block += w[l].wait == Wait::block;
                    over += w[l].wait == Wait::over;
                }
                if (at_lanes != 0 && at_lanes != kLanes) abort();  // an operation across lanes that not all lanes reach
                going = at_lanes != 0;
            }
            left |= w[0].wait != Wait::over;
        }
        for (int t = 0; t < n; ++t)
            if (fibers[t].wait == Wait::block) fibers[t].wait = Wait::none;
    }
}

inline hipError_t launch(dim3 grid, dim3 block, std::function<void()> call) {
    if ((uint64_t)grid.x * block.x > 0xffffffffu) return hipErrorInvalidConfiguration;
    block_dim = block;
    grid_dim = grid;
    body = call;
    for (uint32_t y = 0; y < grid.y; ++y)
        for (uint32_t x = 0; x < grid.x; ++x) {
            block_idx = dim3(x, y, 0);
            if (wanted(block_idx)) run_block();
        }
    return hipSuccess;
}

}  // namespace emu

#define threadIdx (emu::self->tid)
#define blockIdx (emu::block_idx)
#define gridDim (emu::grid_dim)
#define __syncthreads() emu::pause(emu::Wait::block)
#define __shfl(v, from) emu::shfl(v, from)
#define __builtin_amdgcn_readfirstlane(v) emu::readfirstlane(v)
#define __builtin_amdgcn_readlane(v, from) emu::shfl(v, from)
#define __builtin_amdgcn_ballot_w64(b) emu::ballot(b)
#define __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, x, y, z) emu::mfma_4x4x1(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) emu::mfma_16x16<8>(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, x, y, z) emu::mfma_16x16<4>(a, b, c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(p) emu::read_transposed<s16x4_t>((const void*)(p))
#define __builtin_amdgcn_wave_barrier() emu::pause(emu::Wait::lanes)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __umul24(a, b) (((uint32_t)(a) & 0xffffffu) * ((uint32_t)(b) & 0xffffffu))
// the launch of `kernel` with `args`, the names they have in hy_launch.hpp
#define hipLaunchKernel(fn, grid, block, ptrs, shared, st) ((void)(ptrs), emu::launch(grid, block, [&] { kernel(args...); }))
