// Launch helpers shared by the device translation units.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <string>

#include "internal.hpp"

namespace dgmg {

#define HIPCHK(expr)                                                                       \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            fail(DGMG_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_));            \
    } while (0)

#define DISPATCH_B(bval, ...)                                                          \
    switch (bval) {                                                                    \
        case 4: { constexpr int BV = 4; __VA_ARGS__; } break;                          \
        case 8: { constexpr int BV = 8; __VA_ARGS__; } break;                          \
        case 9: { constexpr int BV = 9; __VA_ARGS__; } break;                          \
        case 16: { constexpr int BV = 16; __VA_ARGS__; } break;                        \
        case 25: { constexpr int BV = 25; __VA_ARGS__; } break;                        \
        case 27: { constexpr int BV = 27; __VA_ARGS__; } break;                        \
        case 64: { constexpr int BV = 64; __VA_ARGS__; } break;                        \
        default: fail(DGMG_EUNSUPPORTED, "unsupported block size");                    \
    }

// Event pair of one timed launch (null: the launch is not timed).
struct LaunchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};

// A graph under construction: kernels in the order in which they are added.
// Its nodes are built from the launches' arguments and not by capturing a
// stream: while one is captured, in whatever mode, calls of other threads on the
// legacy stream fail.
struct GraphRecorder {
    hipGraph_t graph = nullptr;
    hipGraphNode_t last = nullptr;
    template <typename... KA>
    void add(void (*k)(KA...), dim3 grid, dim3 block, KA... a) {
        void* args[] = {(void*)&a...};
        hipKernelNodeParams q{};
        q.func = reinterpret_cast<void*>(k);
        q.gridDim = grid;
        q.blockDim = block;
        q.kernelParams = args;
        hipGraphNode_t n = nullptr;
        HIPCHK(hipGraphAddKernelNode(&n, graph, last ? &last : nullptr, last ? 1 : 0, &q));
        last = n;
    }
};
// Set while the calling thread records a graph (record_graph in solver.hip):
// klaunch then adds to it instead of launching.
extern thread_local GraphRecorder* t_recorder;

// Launches kernel k on st.  When the launch is timed, the start and stop
// events ride on the kernel's own dispatch (hipExtLaunchKernelGGL), so their
// interval is the kernel's execution alone, without the dispatch gaps that
// separately recorded events would add.
template <typename... KA, typename... A>
static void klaunch(const LaunchEvents& ev, void (*k)(KA...), dim3 grid, dim3 block, hipStream_t st, A&&... a) {
    if (t_recorder) {
        t_recorder->add<KA...>(k, grid, block, static_cast<KA>(a)...);
        return;
    }
    if (!ev.start) {
        hipLaunchKernelGGL(k, grid, block, 0, st, static_cast<KA>(a)...);
        return;
    }
    hipExtLaunchKernelGGL(k, grid, block, 0, st, ev.start, ev.stop, 0, static_cast<KA>(a)...);
}
template <typename... KA, typename... A>
static void klaunch(void (*k)(KA...), dim3 grid, dim3 block, hipStream_t st, A&&... a) {
    klaunch(LaunchEvents{}, k, grid, block, st, static_cast<KA>(a)...);
}

}  // namespace dgmg
