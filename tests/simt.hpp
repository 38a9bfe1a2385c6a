/*
 * Device code on the CPU, one workgroup at a time: a fiber per thread, wavefronts of 64.
 *
 * A thread runs until it needs another one.  An operation over the wavefront is carried out once every
 * thread of it that still runs waits for something, among those that wait for it: the
 * threads that have left a loop, and stand at the barrier behind it, take no part, as on the GPU.  (Code in
 * which they would stand at another operation over the wavefront instead cannot be run here.)  A
 * barrier is passed once every thread of the workgroup has come to it or has ended.
 * Only what the sources under test use is here.
 */
#ifndef SIMT_HPP
#define SIMT_HPP

#include <math.h>
#include <setjmp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <type_traits>
#include <vector>

struct dim3 { uint32_t x, y, z; dim3(uint32_t x_ = 1, uint32_t y_ = 1, uint32_t z_ = 1) : x(x_), y(y_), z(z_) {} };
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

namespace simt {

enum State { READY, WAVE, BARRIER, DONE };
struct Fiber {
    dim3 tid;
    State state;
    int line;                    /* where the operation over the wavefront stands */
    uint64_t in, out, mask;      /* its operand; its result: another lane's operand, or who takes part */
    bool started;
    ucontext_t ctx;
    jmp_buf at;
};
inline std::vector<Fiber> fibers;
inline char *stacks;
inline Fiber *cur;
inline jmp_buf scheduler;
inline ucontext_t home;
inline std::function<void()> body;
inline dim3 block, grid;
constexpr size_t STACK = 256 * 1024;

inline void entry()
{
    body();
    cur->state = DONE;
    _longjmp(scheduler, 1);
}
__attribute__((noinline)) inline void yield()
{
    if (!_setjmp(cur->at)) _longjmp(scheduler, 1);
}
__attribute__((noinline)) inline void resume(Fiber *f)
{
    if (_setjmp(scheduler)) return;
    cur = f;
    if (f->started) _longjmp(f->at, 1);
    f->started = true;
    setcontext(&f->ctx);
}

/* One workgroup of `threads`. */
inline void run(uint32_t threads, dim3 block_, dim3 grid_, std::function<void()> f)
{
    if (fibers.size() < threads) { fibers.resize(threads); stacks = static_cast<char *>(realloc(stacks, threads * STACK)); }
    body = f; block = block_; grid = grid_;
    for (uint32_t i = 0; i < threads; ++i) {
        Fiber &b = fibers[i];
        b.tid = dim3(i, 0, 0); b.state = READY; b.started = false;
        getcontext(&b.ctx);
        b.ctx.uc_stack.ss_sp = &stacks[i * STACK];
        b.ctx.uc_stack.ss_size = STACK;
        b.ctx.uc_link = &home;
        makecontext(&b.ctx, entry, 0);
    }
    while (true) {
        for (uint32_t w0 = 0; w0 < threads; w0 += 64)
            while (true) {
                int line = 0;
                uint64_t group = 0;
                for (uint32_t i = 0; i < 64; ++i) {
                    Fiber &f = fibers[w0 + i];
                    while (f.state == READY) resume(&f);
                    if (f.state != WAVE) continue;
                    if (line && f.line != line) { fprintf(stderr, "lanes at lines %d and %d: who waits for whom is not known here\n", line, f.line); abort(); }
                    line = f.line;
                    group |= 1ull << i;
                }
                if (!line) break;
                for (uint32_t i = 0; i < 64; ++i)
                    if ((group >> i) & 1ull) { fibers[w0 + i].mask = group; fibers[w0 + i].state = READY; }
            }
        uint32_t done = 0;
        for (uint32_t i = 0; i < threads; ++i) {
            if (fibers[i].state == BARRIER) fibers[i].state = READY;
            else ++done;
        }
        if (done == threads) return;
    }
}

/* ---- operations over the wavefront: every lane leaves its operand, then reads the others' */
inline uint32_t lane() { return cur->tid.x & 63u; }
inline Fiber *wave0() { return &fibers[cur->tid.x & ~63u]; }
inline uint64_t meet(uint64_t x, int line)       /* -> the lanes that take part */
{
    /* two meetings, so that nobody leaves its next operand before all have read this one */
    cur->in = x; cur->line = line; cur->state = WAVE;
    yield();
    const uint64_t group = cur->mask;
    return group;
}
inline void leave(int line) { cur->line = line; cur->state = WAVE; yield(); }
inline uint64_t ballot(bool p, int line)
{
    const uint64_t g = meet(p, line);
    uint64_t r = 0;
    for (int i = 0; i < 64; ++i) if (((g >> i) & 1ull) && wave0()[i].in) r |= 1ull << i;
    leave(line);
    return r;
}
inline bool all(bool p, int line)
{
    const uint64_t g = meet(p, line);
    bool r = true;
    for (int i = 0; i < 64; ++i) if (((g >> i) & 1ull) && !wave0()[i].in) r = false;
    leave(line);
    return r;
}
template <typename T> T read(T x, int from, int line)
{
    static_assert(sizeof(T) <= 8, "an operand");
    uint64_t v = 0;
    memcpy(&v, &x, sizeof x);
    const uint64_t g = meet(v, line);
    const int src = from < 0 ? __builtin_ctzll(g) : from;
    if ((g >> src) & 1ull) v = wave0()[src].in;
    leave(line);
    memcpy(&x, &v, sizeof x);
    return x;
}
template <typename T> T shfl_up(T x, int d, int line) { const int l = (int)lane(); return read(x, l >= d ? l - d : l, line); }
/* data-parallel moves: shifts inside a row of 16 lanes, the last lane of a row or of the first half to the rows behind it,
 * permutations of four; lanes of rows outside `rows`, and without `zero` those that get nothing, keep old */
inline int dpp(int old, int x, uint32_t ctrl, uint32_t rows, bool zero, int line)
{
    const int l = (int)lane(), row = l / 16;
    int src = -1;
    if (ctrl < 0x100) src = (l & ~3) | (int)((ctrl >> (2 * (l & 3))) & 3u);
    else if (ctrl > 0x100 && ctrl < 0x110) src = l + (int)(ctrl - 0x100);
    else if (ctrl > 0x110 && ctrl < 0x120) src = l - (int)(ctrl - 0x110);
    else if (ctrl == 0x142) src = row ? row * 16 - 1 : -1;
    else if (ctrl == 0x143) src = row >= 2 ? 31 : -1;
    else { fprintf(stderr, "dpp %x\n", ctrl); abort(); }
    if (ctrl > 0x100 && ctrl < 0x120 && (src < row * 16 || src >= row * 16 + 16)) src = -1;
    const uint64_t g = meet((uint32_t)x, line);
    int v = src >= 0 && ((g >> src) & 1ull) ? (int)(uint32_t)wave0()[src].in : zero ? 0 : old;
    if (!((rows >> row) & 1u)) v = old;
    leave(line);
    return v;
}
inline uint32_t mbcnt(uint32_t mask, uint32_t below, uint32_t add) { return add + (uint32_t)__builtin_popcount(mask & below); }
inline void barrier() { cur->state = BARRIER; yield(); }
[[noreturn]] inline void missing(const char *what) { fprintf(stderr, "%s is not emulated\n", what); abort(); }

}  // namespace simt

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define threadIdx (simt::cur->tid)
#define blockIdx simt::block
#define gridDim simt::grid
#define __syncthreads() simt::barrier()
#define __ballot(p) simt::ballot(p, __LINE__)
#define __all(p) simt::all(p, __LINE__)
#define __shfl_up(x, d, w) simt::shfl_up(x, d, __LINE__)
#define __shfl_xor(x, d, w) simt::read(x, (int)(simt::lane() ^ (uint32_t)(d)), __LINE__)
#define __builtin_amdgcn_readfirstlane(x) simt::read(x, -1, __LINE__)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __shfl(x, l, w) simt::read(x, (int)(l), __LINE__)
#define __any(p) (simt::ballot(p, __LINE__) != 0)
#define __builtin_amdgcn_readlane(x, l) simt::read((int)(x), (int)(l), __LINE__)
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, zero) simt::dpp(old, x, ctrl, rows, zero, __LINE__)
#define __builtin_amdgcn_mov_dpp(x, ctrl, rows, banks, zero) simt::dpp(0, x, ctrl, rows, zero, __LINE__)
#define __builtin_amdgcn_mbcnt_lo(m, add) simt::mbcnt(m, simt::lane() < 32 ? (1u << simt::lane()) - 1u : ~0u, add)
#define __builtin_amdgcn_mbcnt_hi(m, add) simt::mbcnt(m, simt::lane() < 32 ? 0u : (1u << (simt::lane() - 32)) - 1u, add)
#define __builtin_amdgcn_s_sleep(x) ((void)0)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __syncthreads_or(p) (simt::missing("__syncthreads_or"), 0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_fetch_add(p, x, order, scope) atomicAdd(p, x)
#define __hip_atomic_load(p, order, scope) (*(p))
#define __threadfence() ((void)0)
#define wall_clock64() 0ull
#define __builtin_nontemporal_load(p) (*(p))
#define __builtin_nontemporal_store(v, p) ((void)(*(p) = (v)))

inline uint32_t atomicAdd(uint32_t *p, uint32_t x) { const uint32_t old = *p; *p += x; return old; }
inline uint32_t atomicMax(uint32_t *p, uint32_t x) { const uint32_t old = *p; *p = old > x ? old : x; return old; }
inline uint32_t atomicOr(uint32_t *p, uint32_t x) { const uint32_t old = *p; *p |= x; return old; }
inline int __popc(uint32_t x) { return __builtin_popcount(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline uint32_t __float_as_uint(float x) { uint32_t u; memcpy(&u, &x, 4); return u; }
inline float __uint_as_float(uint32_t u) { float x; memcpy(&x, &u, 4); return x; }
inline int __float_as_int(float x) { return (int)__float_as_uint(x); }
inline float __int_as_float(int u) { return __uint_as_float((uint32_t)u); }
typedef _Float16 __half;
inline __half __float2half_rn(float x) { return (__half)x; }
inline float __half2float(__half x) { return (float)x; }
inline unsigned short __half_as_ushort(__half x) { unsigned short u; memcpy(&u, &x, 2); return u; }
inline long long __double_as_longlong(double x) { long long u; memcpy(&u, &x, 8); return u; }
inline double __longlong_as_double(long long u) { double x; memcpy(&x, &u, 8); return x; }
inline float __fadd_rn(float a, float b) { return a + b; }
inline float __fsub_rn(float a, float b) { return a - b; }
inline float __fdiv_rn(float a, float b) { return a / b; }
inline float __fmul_rn(float a, float b) { return a * b; }
inline float __fmaf_rn(float a, float b, float c) { return fmaf(a, b, c); }
template <typename A, typename B> std::common_type_t<A, B> min(A a, B b) { std::common_type_t<A, B> x = a, y = b; return x < y ? x : y; }
template <typename A, typename B> std::common_type_t<A, B> max(A a, B b) { std::common_type_t<A, B> x = a, y = b; return x > y ? x : y; }

#endif
