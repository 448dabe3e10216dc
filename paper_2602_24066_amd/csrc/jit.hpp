// Run-time specialised kernels (see jit.cpp).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>
#include <vector>

#include "wordset.hpp"

namespace sig {

struct JitKernel {
    std::vector<char> code;        // code object produced by hiprtc
    std::string name;              // kernel symbol
    std::string log;               // compiler log (warnings or errors)
    std::string cache_file;        // set when the code object came from the disk cache
    hipModule_t mod = nullptr;
    hipFunction_t fn = nullptr;
    // further kernels of the module and their wavefronts per workgroup; one that does not fit its launch stays nullptr
    struct More { const char* name; int nw; hipFunction_t fn; };
    std::vector<More> more;
    int dev = -1;                  // device the module was loaded on
    int nw = 0;                    // wavefronts (units) per workgroup
    int tile = 0;                  // segments per LDS tile
    bool tried = false;
    bool ok = false;
    std::mutex m;                  // compilation and loading of this kernel; calls on other kernels do not wait for it
};

std::string jit_forward_source(const WordSet& ws, const Plan& plan, int NW, int T);
// flush_rounds: the sum of a gradient tile as a function (0), or inlined in that many rounds; own_set: reconstruction from intermediates
// of its own
std::string jit_backward_source(const WordSet& ws, const Plan& plan, int NW, int T, int flush_rounds, bool own_set);
// hiprtc: source -> gfx950 code object.  0 on success; the log is kept either way.  Needs no device.
// With SIG_JIT_CACHE naming a directory the code object is looked up there first (use_cache) and stored after a
// compilation; use_cache = false removes a cached file and compiles afresh.
int jit_compile(const std::string& src, const char* kernel_name, JitKernel& out, bool use_cache = true);
// Loads the code object on the current device (first use) and checks what it declares against the launch shape:
// nw * 64 threads per workgroup, static LDS within the 64 KB a kernel may declare, the registers of nw / 4 wavefronts
// per SIMD.  A code object that does not fit is refused here (hipErrorLaunchFailure is never risked at dispatch).
hipError_t jit_load(JitKernel& k);
// the check alone, on the numbers hipFuncGetAttribute reports (host only; for tests)
bool jit_launch_shape_fits(int nw, int max_threads_per_block, int static_lds_bytes, int num_regs);
void jit_release(JitKernel& k);

// Full truncations with lanes = words (jit_lanes.cpp): a lane holds a word of length depth - R and the R levels below
// it, `lanes` = d^(depth - R) of them per path in `waves` wavefronts, nwb wavefronts per workgroup, T segments per
// gradient tile, TS segments of increments staged at a time.
struct LanesShape {
    bool ok, msum;                 // msum: gradient sums as matrix products
    bool shares;                   // backward: a wavefront's LDS holds a chunk signature over the words shorter than the depth
    int R, T, TS, nwb;
    int split;                     // wavefronts that share the children of 64 words (forward, R = 2: 1 or 2)
    int64_t lanes, waves;
    double fit;                    // wavefronts a SIMD holds by the LDS they take
    int chain;                     // multiply-adds of a lane's chain per segment
    double per_lane;               // instructions of a lane per segment, for comparing shapes
};
// the form for a batch of B paths; levels = 1 or 2 asks for that R (0: the cheaper one)
LanesShape lanes_shape(int d, int depth, bool backward, int64_t B, int levels);
// Time chunks of those truncations: products of the chunk signatures over all words (one workgroup per path and first
// letter; the forward call), over the words shorter than the depth in both directions (two per path and letter; the
// backward call), and the adjoints at the chunk boundaries (one per boundary and first letter).
enum LanesChunkPart { kLanesScanFull = 0, kLanesScanLow = 1, kLanesAdjoint = 2, kLanesDisplacement = 3 };
int lanes_chunk_threads(int d, int depth, LanesChunkPart part);   // of a workgroup
LanesShape lanes_low_shape(int d, int depth);                 // forward kernel over the words shorter than the depth
bool lanes_chunks_available(int d, int depth);
// source of sig_fwd_lanes (backward = false) or sig_bwd_lanes for that shape and, where time chunks are available, of the
// kernels they take: sig_scan_lanes, and backward sig_low_lanes (forward) and sig_adjoint_lanes as well
// arrays: backward with the kernels that write products and boundary adjoints of time chunks to arrays
std::string lanes_source(int d, int depth, const LanesShape& s, bool backward, bool arrays);
constexpr int kLanesChunkCounts[] = {2, 3, 4, 6, 8, 12, 16, 24, 32};
// time chunks for B paths of L segments: the count with the shortest modelled time, 1 where none gains a tenth
int lanes_chunk_count(int d, int depth, bool backward, int64_t B, int64_t L, int levels);

}  // namespace sig
