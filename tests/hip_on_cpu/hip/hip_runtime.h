// Runs a kernel's source on the CPU: a lane is a fiber, a workgroup's waves run one after the other up to the next barrier, in ascending
// or descending order.  A wave that reads shared memory which a wave ahead of it may already have written, with no barrier between,
// therefore reads the wrong value every time in one of the two orders.  Operations over lanes (and fences, where the lanes' shared-memory
// accesses are in order on the GPU) wait for the 64 lanes of the wave; they must not stand in divergent code.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <memory>
#include <vector>

#define __global__
#define __device__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)

typedef int hipError_t;
typedef void* hipStream_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidDevice = 1;
constexpr int hipFuncAttributeMaxDynamicSharedMemorySize = 0;
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct float4 {
    float x, y, z, w;
};
inline dim3 threadIdx, blockIdx, blockDim;

namespace emu {
enum State { READY, BARRIER, DONE };
struct Lane {
    ucontext_t context;
    std::unique_ptr<char[]> stack{new char[1 << 17]};
    State state = READY;
    int ops = 0;   // operations over lanes that it has begun
    int vote = 1;  // at its barrier
};
struct Wave {
    uint64_t posted[2][64];
    int arrived[2] = {0, 0}, finished = 0;  // of the two newest operations; operations that all lanes have begun
};
inline std::vector<Lane>* lanes;
inline std::vector<Wave>* waves;
inline ucontext_t scheduler;
inline bool backwards;     // the order of the waves
inline int64_t operations;  // over lanes, of all waves so far
inline const void* kernel;  // launched last
inline int votes;          // of all lanes at the last barrier
inline std::function<void()> body;
extern unsigned char* const shared;
extern const size_t shared_bytes;

inline Lane& lane() { return (*lanes)[threadIdx.x]; }
inline void yield() { swapcontext(&lane().context, &scheduler); }
// every lane's value, once all lanes of the wave have begun the operation
inline const uint64_t* exchange(uint64_t v) {
    Wave& w = (*waves)[threadIdx.x / 64];
    const int op = lane().ops++, turn = op & 1;
    w.posted[turn][threadIdx.x & 63] = v;
    if (++w.arrived[turn] == 64) {
        w.arrived[turn] = 0;
        ++w.finished;
        ++operations;
    }
    while (w.finished <= op) yield();
    return w.posted[turn];
}
inline int barrier(int vote) {
    lane().vote = vote;
    lane().state = BARRIER;
    yield();
    return votes;
}
inline void run_lane() {
    body();
    lane().state = DONE;
    yield();
}

template <typename K, typename... A>
void launch(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t, A... args) {
    if (lds > shared_bytes) abort();
    emu::kernel = (const void*)kernel;
    blockDim = block;
    body = [=] { kernel(args...); };
    for (unsigned b = 0; b < grid.x; ++b) {
        blockIdx = dim3(b, 0, 0);
        memset(shared, 0xFF, shared_bytes);
        std::vector<Lane> ls(block.x);
        std::vector<Wave> ws((block.x + 63) / 64);  // (a last wave of fewer than 64 lanes cannot take an operation over lanes)
        lanes = &ls;
        waves = &ws;
        for (Lane& l : ls) {
            getcontext(&l.context);
            l.context.uc_stack.ss_sp = l.stack.get();
            l.context.uc_stack.ss_size = 1 << 17;
            l.context.uc_link = nullptr;
            makecontext(&l.context, run_lane, 0);
        }
        for (bool live = true; live;) {
            for (size_t i = 0; i < ws.size(); ++i) {
                const size_t w = backwards ? ws.size() - 1 - i : i;
                for (bool ready = true; ready;) {
                    ready = false;
                    for (size_t t = 64 * w; t < 64 * w + 64 && t < ls.size(); ++t)
                        if (ls[t].state == READY) {
                            threadIdx = dim3((unsigned)t, 0, 0);
                            swapcontext(&scheduler, &ls[t].context);
                            ready = ready || ls[t].state == READY;
                        }
                }
            }
            live = false;
            votes = 1;
            for (Lane& l : ls)
                if (l.state == BARRIER) {
                    votes &= l.vote;
                    l.state = READY;
                    live = true;
                }
        }
    }
}

template <typename T>
T of(const uint64_t* all, int l) {
    T v;
    memcpy(&v, &all[l], sizeof v);
    return v;
}
template <typename T>
uint64_t bits(T v) {
    uint64_t u = 0;
    memcpy(&u, &v, sizeof v);
    return u;
}
struct Pair {
    uint32_t v[2];
    uint32_t operator[](int i) const { return v[i]; }
};
}  // namespace emu
#define hipLaunchKernelGGL(kernel, ...) emu::launch(kernel, __VA_ARGS__)

inline void __syncthreads() { emu::barrier(1); }
inline int __syncthreads_and(int p) { return emu::barrier(p != 0); }
inline uint64_t __ballot(int p) {
    const uint64_t* all = emu::exchange(p != 0);
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l) m |= all[l] << l;
    return m;
}
inline int __any(int p) { return __ballot(p) != 0; }
inline int __all(int p) { return __ballot(p) == ~0ull; }
inline void __builtin_amdgcn_fence(int, const char*) { emu::exchange(0); }
inline int __builtin_amdgcn_readlane(int v, int l) { return emu::of<int>(emu::exchange(emu::bits(v)), l); }
inline int __builtin_amdgcn_readfirstlane(int v) { return __builtin_amdgcn_readlane(v, 0); }
inline int __builtin_amdgcn_update_dpp(int, int v, int ctrl, int, int, bool) {
    const uint64_t* all = emu::exchange(emu::bits(v));
    const int l = threadIdx.x & 63, row = l & ~15, i = l & 15;
    if (ctrl < 0x100) return emu::of<int>(all, (l & ~3) + ((ctrl >> (2 * (l & 3))) & 3));
    if (ctrl == 0x140) return emu::of<int>(all, row + 15 - i);
    if (ctrl == 0x141) return emu::of<int>(all, (l & ~7) + 7 - (l & 7));
    const int n = ctrl & 15;
    if (ctrl >> 4 == 0x12) return emu::of<int>(all, row + ((i - n) & 15));
    if (ctrl >> 4 == 0x11) return i >= n ? emu::of<int>(all, l - n) : 0;
    abort();
}
inline emu::Pair __builtin_amdgcn_permlane16_swap(uint32_t a, uint32_t b, bool, bool) {
    const uint64_t* all = emu::exchange((uint64_t)a << 32 | b);
    const int l = threadIdx.x & 63;
    if (l & 16) return {{(uint32_t)all[l - 16], b}};
    return {{a, (uint32_t)(all[l + 16] >> 32)}};
}
inline emu::Pair __builtin_amdgcn_permlane32_swap(uint32_t a, uint32_t b, bool, bool) {
    const uint64_t* all = emu::exchange((uint64_t)a << 32 | b);
    const int l = threadIdx.x & 63;
    if (l & 32) return {{(uint32_t)all[l - 32], b}};
    return {{a, (uint32_t)(all[l + 32] >> 32)}};
}
inline uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    const uint64_t both = (uint64_t)hi << 32 | lo;
    uint32_t r = 0;
    for (int b = 0; b < 4; ++b) r |= (uint32_t)((both >> (8 * ((sel >> (8 * b)) & 7))) & 0xFF) << (8 * b);
    return r;
}
inline float __builtin_amdgcn_fmed3f(float a, float b, float c) { return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c)); }

inline uint32_t __float_as_uint(float f) { return (uint32_t)emu::bits(f); }
inline float __uint_as_float(uint32_t u) {
    const uint64_t v = u;
    return emu::of<float>(&v, 0);
}
inline long long __double_as_longlong(double d) { return (long long)emu::bits(d); }
inline int __double2hiint(double d) { return (int)(emu::bits(d) >> 32); }
inline int __double2loint(double d) { return (int)emu::bits(d); }
inline double __hiloint2double(int hi, int lo) {
    const uint64_t v = (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo;
    return emu::of<double>(&v, 0);
}
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int atomicAdd(int* p, int v) { return (*p += v) - v; }
