// C ABI of the library (see include/sig.h for the contract of every entry point).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include <cstdlib>
#include <mutex>
#include <string>

#include "../../include/sig.h"
#include "jit.hpp"
#include "kernels.hpp"
#include "wordset.hpp"

struct sig_wordset : public sig::WordSet {};

namespace {
thread_local int g_last_hip = 0;

int hip_fail(hipError_t e)
{
    g_last_hip = (int)e;
    return SIG_EHIP;
}

const sig::WordSet* W(const sig_wordset* ws) { return ws; }

// Launch-shape knobs: one table for the environment variables read when a set is built and for
// sig_wordset_set_option / sig_wordset_get_option.
struct OptionName { const char* name; const char* env; int sig::WordSet::Options::*field; };
const OptionName kOptions[] = {
    {"no_jit", "SIG_NO_JIT", &sig::WordSet::Options::no_jit},
    {"jit_waves", "SIG_JIT_WAVES", &sig::WordSet::Options::jit_waves},
    {"chunks", "SIG_CHUNKS", &sig::WordSet::Options::chunks},
    {"fwd_tails", "SIG_FWD_TAILS", &sig::WordSet::Options::fwd_tails},
    {"bwd_tails", "SIG_BWD_TAILS", &sig::WordSet::Options::bwd_tails},
    {"lanes", "SIG_LANES", &sig::WordSet::Options::lanes},
    {"lanes_levels", "SIG_LANES_LEVELS", &sig::WordSet::Options::lanes_levels},
    {"logsig_gather", "SIG_LOGSIG_GATHER", &sig::WordSet::Options::logsig_gather},
    {"jit_wg_waves", "SIG_JIT_WG_WAVES", &sig::WordSet::Options::jit_wg_waves},
    {"bwd_tile", "SIG_BWD_TILE", &sig::WordSet::Options::bwd_tile},
    {"ckpt_chunks", "SIG_CKPT_CHUNKS", &sig::WordSet::Options::ckpt_chunks},
    {"jit_fwd_tile", "SIG_JIT_FWD_TILE", &sig::WordSet::Options::jit_fwd_tile},
};
void options_from_environment(sig::WordSet& w)
{
    for (const OptionName& o : kOptions) {
        const char* e = std::getenv(o.env);
        if (e && e[0]) w.opt.*(o.field) = std::atoi(e);
    }
    if (w.closure) w.closure->opt = w.opt;
}
int finish_build(int rc, sig::WordSet* w, sig_wordset** out)
{
    if (rc != SIG_OK) return rc;
    options_from_environment(*w);
    *out = static_cast<sig_wordset*>(w);
    return SIG_OK;
}

// Picks the plan variant: the coarsest one (least recomputation of shared ancestors) that still
// yields enough wavefronts to occupy the 256 compute units, else the finest.
int pick_variant(const sig::WordSet& ws, int dir, int64_t B, int64_t want = 2048 /* two wavefronts per SIMD */)
{
    const int64_t groups = (B + 63) / 64;
    const auto& pl = ws.plans[dir];
    for (size_t v = 0; v < pl.size(); ++v)
        if ((int64_t)pl[v].units.size() * groups >= want) return (int)v;
    return (int)pl.size() - 1;
}

// kernel timer (see sig_profile_enable); channels 0/1: main kernel of forward/backward, 2/3: whole call
struct Profiler {
    unsigned mask = 0;                // bit `which` set: that channel records
    std::vector<hipEvent_t> ev[4];    // start/stop interleaved
    size_t used[4] = {0, 0, 0, 0};
    hipEvent_t* next(int dir)
    {
        if (!((mask >> dir) & 1u) || used[dir] >= SIG_PROFILE_MAX_LAUNCHES) return nullptr;
        if (ev[dir].size() < 2 * (used[dir] + 1)) {
            hipEvent_t a, b;
            if (hipEventCreate(&a) != hipSuccess) return nullptr;
            if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return nullptr; }
            ev[dir].push_back(a);
            ev[dir].push_back(b);
        }
        return &ev[dir][2 * used[dir]++];
    }
};
Profiler g_prof;

// brackets everything a call enqueues
struct CallTimer {
    hipEvent_t* pe;
    hipStream_t st;
    CallTimer(int dir, hipStream_t s) : pe(g_prof.next(2 + dir)), st(s) { if (pe) (void)hipEventRecord(pe[0], st); }
    ~CallTimer() { if (pe) (void)hipEventRecord(pe[1], st); }
};

// Time chunks for full truncations: with few paths the sequential kernels leave wavefront slots empty, so the
// segments of every path are cut into C chunks that run as independent rows and are combined afterwards with Chen's
// relation.  Forward it pays off once a chunk is a few hundred segments long (d = 4: the chunk products and the second
// launch cost about as much as 100 segments); backward from the terminal signature alone has to recompute the chunk
// signatures, a forward pass of its own: d = 4 does so on request (option "chunks") where its fused form does not run.
// For d = 8 and d = 16 the counts below are what a call has to bring a workspace for; low_chunks may cut finer (backward it is
// what a call takes).
struct Chunks { int64_t C, Lc; };
// own_chunks = false: sig_backward does not chunk by itself (sig_backward_static, whose scratch array is sized for
// whole paths).
Chunks trunc_chunks(const sig::WordSet& w, int dir, int64_t B, int64_t n_points, bool own_chunks = true)
{
    const int64_t L = n_points - 1;
    int64_t C = 1;
    if (L >= 64 && sig::chunking_available(w.d, w.depth)) {
        if (w.opt.chunks > 0) {                                                           // tuning knob
            C = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(w.opt.chunks, 64), L / 32));
        } else if (dir == 0) {
            const int64_t slots = (int64_t)1024 * sig::trunc_occupancy(w.d, w.depth, dir);
            C = slots / sig::trunc_waves_per_row(w.d, w.depth, dir) / std::max<int64_t>(B, 1);
            C = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(C, 64), L / 256));
        } else if (own_chunks && !sig::trunc_backward_tails_available(w.d, w.depth)) {
            const int64_t rows_wanted = 2048 / sig::trunc_waves_per_row(w.d, w.depth, 1);
            C = std::min<int64_t>(std::min<int64_t>(16, rows_wanted / std::max<int64_t>(B, 1)), L / 256);
            C = C >= 16 ? 16 : (C >= 8 ? 8 : (C >= 4 ? 4 : 1));     // whole wavefronts per SIMD
        }
    }
    const int64_t Lc = (L + C - 1) / C;
    return Chunks{(L + Lc - 1) / Lc, Lc};
}
// d = 8 and d = 16 (sig::trunc_low_available): chunks with products by slices in one launch, and backward with chunk signatures over
// the words shorter than the depth alone (the longest are never reconstructed), so few paths are cut finer, and shorter ones
// than above: up to sixteen chunks (eight forward), a model decides.  Microseconds per segment of a row: a lone wavefront on
// each SIMD, and what a wavefront adds beyond that; per chunk: a product, the boundary adjoints and the traffic of its signature.
// A forward and a backward call, one after the other on a stream, whole paths (or the chunks of at least 256 segments before) ->
// now: d = 8, 3 paths x 979 segments 703 -> 123 us, 62 x 515 404 -> 255, 5 x 238 206 -> 72; d = 16, 1 x 373 251 -> 71, 18 x 591 350 -> 168.
double low_time(const sig::WordSet& w, int dir, bool kept /* the chunk signatures are */, int64_t B, int64_t L, int64_t C)
{
    const bool d8 = w.d == 8;
    const double lone = dir ? (d8 ? 0.65 : 0.526) : (d8 ? 0.168 : 0.146), each = dir ? (d8 ? 0.468 : 0.325) : (d8 ? 0.153 : 0.108);
    const double per_simd = std::ceil((double)sig::trunc_waves_per_row(w.d, w.depth, dir) * (double)(B * C) / 1024.0);
    const double pairs = std::floor(per_simd / 2.0), single = per_simd - 2.0 * pairs;        // two wavefronts fit a SIMD
    const double Lc = (double)((L + C - 1) / C), paths = (double)B, n = (double)C;
    const double t = Lc * (pairs * 2.0 * each + single * lone);
    if (C == 1) return t;
    if (!dir) return t + 4.5 + n * (1.0 + (d8 ? 0.09 : 0.17) * paths);
    return t + (kept ? 9.0 : 18.0 + (d8 ? 0.12 : 0.05) * Lc) + n * (0.6 + 0.11 * paths);
}
int low_chunk_count(const sig::WordSet& w, int dir, int64_t B, int64_t L)
{
    double best = 0.93 * low_time(w, dir, false, B, L, 1);
    int choice = 1;
    for (int C : {2, 3, 4, 6, 8, 12, 16}) {
        if (L < 8 * (int64_t)C || (dir == 0 && C > 8)) break;
        const double t = low_time(w, dir, false, B, L, C);
        if (t < best) {
            best = t;
            choice = C;
        }
    }
    return choice;
}
// the product of every path's chunk signatures: small ones in LDS; by slices from three chunks on, of two spread over the grid (forward
// calls of 128 x 1,024, d = 8: 160.8 us, by slices 163.9; 64 x 4,096, d = 16 455.7 and 456.7)
hipError_t chunk_product_of(const sig::WordSet& w, const float* Sc, float* coeffs, int64_t B, int64_t C, hipStream_t st)
{
    if (!sig::trunc_low_available(w.d, w.depth))
        return sig::chunk_scan(w.d, w.depth, Sc, nullptr, nullptr, coeffs, nullptr, nullptr, B, (int)C, st);
    if (C > 2) return sig::chunk_slices_forward(w.d, w.depth, Sc, coeffs, B, (int)C, st);
    return sig::chunk_product(w.d, w.depth, Sc, coeffs, B, st);
}
Chunks low_chunks(const sig::WordSet& w, int dir, int64_t B, int64_t n_points)
{
    const int64_t L = n_points - 1;
    int64_t C = 1;
    if (w.opt.chunks > 0) C = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(w.opt.chunks, 64), L / 4));   // tuning knob
    else C = low_chunk_count(w, dir, B, L);
    const int64_t Lc = (L + C - 1) / C;
    return Chunks{(L + Lc - 1) / Lc, Lc};
}
// Forward for d = 4 in the layout with 64 words of length 3 per wavefront (two wavefronts per chunk of a path, 2 or 4
// chunks per path in one workgroup, chunk signatures multiplied in LDS).  Returns the number of chunks, 0 = the
// kernel with four wavefronts per path instead (with its chunk arrays in HBM for long paths): measured faster only
// for fewer than 192 paths of more than 512 segments.  Four chunks need a compute unit per path, so larger batches
// take two.  The option "fwd_tails" = 0 (or a "chunks" setting) switches it off, = 2 / = 4 force that many chunks.
int64_t trunc_forward_fused_chunks(const sig::WordSet& w, int64_t B, int64_t n_points, const float* coeffs)
{
    if (!sig::trunc_forward_tails_available(w.d, w.depth) || ((uintptr_t)coeffs & 15) != 0) return 0;
    const int64_t L = n_points - 1;
    const int f = w.opt.fwd_tails;
    if (f == 0) return 0;
    if (f == -1 && w.opt.chunks > 0) return 0;               // asks for the form with chunk arrays in HBM
    int64_t C;
    if (f == 2 || f == 4) {
        C = f;
    } else {
        if (B < 192 && L > 512) return 0;
        C = B <= 256 ? 4 : 2;
    }
    while (C > 1 && L < 8 * C) C /= 2;                       // chunks of at least 8 segments
    if (C < 2) return 0;
    const int64_t Lc = (L + C - 1) / C;
    return (C - 1) * Lc >= L ? 0 : C;
}

// Backward launch shape for a full truncation.  d = 4 has a second kernel with one wavefront per (path, chunk) row
// that does half the vector work per path and fits two wavefronts on a SIMD, so it wants about two thousand rows.
// Smaller batches take its fused form (2, 4 or 8 chunks of a path in one workgroup, everything between the chunks
// in LDS), larger ones run it unchunked; the thresholds come from a scan over 64..2,048 paths of 64..1,024 segments.
// The option "bwd_tails" = 0 switches it off, = 1 takes the unfused form with chunk arrays in HBM ("chunks" chunks),
// =2 / =4 / =8 force the fused form with that many chunks.
struct BwdShape { bool tails, fused; int64_t C, Lc; };
BwdShape trunc_backward_shape(const sig::WordSet& w, int64_t B, int64_t n_points, bool own_chunks = true)
{
    const int64_t L = n_points - 1;
    const Chunks ch = trunc_chunks(w, 1, B, n_points, own_chunks);
    BwdShape s{false, false, ch.C, ch.Lc};
    if (!sig::trunc_backward_tails_available(w.d, w.depth)) return s;
    const int f = w.opt.bwd_tails;
    if (f == 0) return s;
    if (f == 1) return BwdShape{true, false, ch.C, ch.Lc};
    int64_t C = f == 2 || f == 4 || f == 8 ? f : (B <= 256 ? 8 : (B <= 896 ? 4 : (B <= 1536 ? 2 : 1)));
    while (C > 1 && L < 8 * C) C /= 2;                       // chunks of at least 8 segments
    if (C == 1) return BwdShape{true, false, f == -1 ? 1 : ch.C, f == -1 ? L : ch.Lc};
    const int64_t Lc = (L + C - 1) / C;
    if ((C - 1) * Lc >= L) return s;
    return BwdShape{true, true, C, Lc};
}
// Checkpointed form (sig_forward_checkpointed / sig_backward_checkpointed): the forward pass leaves the signatures of C
// time chunks of every path in a buffer the caller keeps, and the backward pass walks the C chunks side by side
// without recomputing them.  Taken where the backward kernel of a full truncation has too few rows to put two
// wavefronts on every SIMD (eight wavefronts per row for d = 8, sixteen for d = 16); C = 2 .. 16, chunks of at least 64
// segments (measured: 8 paths x 8,192 segments, d = 16: step 4.1 ms plain, 1.43 ms with four chunks, 1.00 ms with eight).
// "ckpt_chunks" forces a count (0: this rule, 1: off).
//
// Word sets closed under suffixes as well as prefixes (anisotropic sets, Definition 7.1) that run through the
// straight-line specialised kernels (lane = row) take the same form: Chen's relation restricted to such a set stays
// inside it.  Those kernels gain from rows up to about 2,048 (32 lane groups: fewer, larger units, so less
// recomputation of shared ancestors per group), but every chunk boundary costs a product and an adjoint sum over the
// set, gathers that run at a fraction of the rate of the kernels.  Measured on 5,754 words for 64 .. 1,024 paths of
// 512 .. 4,096 segments (step time against the plain calls: -75 % for 64 paths x 4,096 segments with eight chunks,
// -35 % for 512 x 2,048 with four, -20 % for 512 x 512 with two, -5 % for 1,024 x 512 with two); more than 2,048 rows
// lose.  "ckpt_chunks" forces a count of up to 16 (chunks of at least 64 segments).
bool jit_enabled(const sig::WordSet& w);
bool words_time_chunks(const sig::WordSet& w)
{
    return w.kind != 0 && w.pair_tables && jit_enabled(w) && w.max_len <= 14 && sig::words_scan_lds_bytes(w.size()) <= 160 * 1024;
}
Chunks checkpoint_chunks(const sig::WordSet& w, int64_t B, int64_t n_points)
{
    const int64_t L = n_points - 1;
    int64_t C = 1;
    if (B >= 1 && words_time_chunks(w)) {
        if (w.opt.ckpt_chunks > 0) {
            C = std::min<int64_t>(std::min<int64_t>(w.opt.ckpt_chunks, 16), L / 64);
        } else {
            // at most 2,048 rows and chunks of at least 256 segments; batches that stay at 512 rows or below take chunks
            // down to 128 segments; never more than eight
            C = std::min<int64_t>(2048 / B, L / 256);
            if (B * std::max<int64_t>(C, 1) <= 512) C = std::min<int64_t>(2048 / B, L / 128);
            C = std::min<int64_t>(C, 8);
        }
        C = std::max<int64_t>(1, C);
        if (B * C > (int64_t)65535 * 64) C = 1;
    }
    if (w.kind == 0 && B >= 1 && B <= 65535 && sig::trunc_backward_available(w.d, w.depth) && sig::chunking_available(w.d, w.depth) &&
        !sig::trunc_backward_tails_available(w.d, w.depth)) {
        if (w.opt.ckpt_chunks > 0) {
            C = std::min<int64_t>(w.opt.ckpt_chunks, 16);
        } else {
            const int64_t rows_wanted = 2048 / sig::trunc_waves_per_row(w.d, w.depth, 1);
            C = std::min<int64_t>(std::min<int64_t>(16, (rows_wanted + B - 1) / B), L / 64);
            if (C > 4) C = C >= 16 ? 16 : (C >= 8 ? 8 : 4);         // beyond four: powers of two (whole wavefronts per SIMD)
        }
        C = std::max<int64_t>(1, std::min<int64_t>(C, L / 64));
    }
    if (C < 2) return Chunks{1, L};
    const int64_t Lc = (L + C - 1) / C;
    return Chunks{(L + Lc - 1) / Lc, Lc};
}
size_t chunk_array_bytes(const sig::WordSet& w, int64_t B, int64_t C)
{
    return ((size_t)B * (size_t)C * (size_t)w.size() * sizeof(float) + 255) & ~(size_t)255;
}

bool use_trunc_forward(const sig::WordSet& w, int64_t B)
{
    return w.kind == 0 && B <= 65535 && sig::trunc_forward_available(w.d, w.depth);
}

bool use_trunc_backward(const sig::WordSet& w, int64_t B)
{
    return w.kind == 0 && B <= 65535 && sig::trunc_backward_available(w.d, w.depth);
}

// ---- run-time specialised kernels ------------------------------------------------------------------------
std::mutex g_jit_mutex;

int jit_wg_waves(const sig::WordSet& w)   // wavefronts (units) per workgroup
{
    return w.opt.jit_wg_waves == 8 ? 8 : std::max(1, std::min(4, w.opt.jit_wg_waves));
}
// Nanoseconds a backward segment takes two wavefronts of a SIMD whose units hold that many words, and the additions of all
// workgroups to the gradients (see jit_units)
double jit_pair_ns(double unit) { return 430.0 + 13.4 * unit; }
double jit_additions_ns(double d, int64_t workgroups) { return (double)workgroups * d * 256.0 / 1150.0; }
// Work units asked of the balanced planner for a batch of B paths: two wavefronts per SIMD (2,048) over the path groups, in
// whole workgroups, and not so many that units shrink below eight words (every unit recomputes the ancestors of its
// first word).  Where that comes to more than one workgroup per compute unit (256), half as many of larger units may be
// the better choice; a model of the backward kernel decides, in nanoseconds per segment, fitted to 40 pairs of 4 to 40
// letters, 1,500 to 10,000 words and 384 to 1,024 paths (of kernels with a second set of intermediates; with the shared set seven of those
// shapes take 0.89 to 1.00 of the time, and no choice was looked at anew):
//   one workgroup each: the latency of a lone wavefront, 250 + 25 d, and 9.5 per word of its unit;
//   two (jit_pair_ns): 430 and 13.4 per word, or the additions of all workgroups to the gradients (d x 256 bytes each) at 1.15 TB/s.
// So few words or many letters take one each (backward calls of 256 segments, two -> one: 1,500 words, d = 10, 640 paths
// 269 -> 169 us, 960 paths 303 -> 189; 3,000 words, 512 paths, d = 20 557 -> 291, d = 8 249 -> 167), large units of few
// letters do not (5,754 words, d = 6, 640 paths 220 and 257; 10,000, d = 10 314 and 364).  The count is rounded down to
// four steps an octave, so that neighbouring batch sizes share a kernel.  The forward kernel adds nothing up and follows
// only into units of up to twelve words (1,500 words, 512 paths: d = 10 55 -> 54 us, d = 20 77 -> 71; 6,000, d = 10 78 and 86).
// Units go down to four words where 128 to 512 words and three or more path groups leave most of the chip empty (calls of 256
// segments, forward + backward: 150 words, d = 5, 256 paths 144 -> 136 us; 384, d = 6, 300 paths 124 -> 111; 500, d = 4 143 -> 133;
// 400, d = 20, 256 paths 264 -> 248; at 640 paths, 120 workgroups of eight words each, no gain).  Not beyond: every column adds to the
// same gradients in no fixed order, so fewer words and one or two groups keep the few columns that let two runs agree to a few
// roundings (up to 39 words, one column: bit for bit; 150 words on 9 paths gained 6 % from ten columns and differed by twice as
// much), and large sets would compile twice as long (1,500 words: 15 -> 33 s for 7 %).
int64_t jit_units(const sig::WordSet& w, int dir, int64_t B)
{
    const int kJitWaves = jit_wg_waves(w);
    const int64_t groups = (B + 63) / 64;
    int64_t want = 2048;
    if (w.opt.jit_waves > 0) want = w.opt.jit_waves;                                       // tuning knob
    auto columns = [&](int64_t words_each) {
        const int64_t n = std::min(std::max<int64_t>(1, want / groups), std::max<int64_t>(1, w.size() / words_each));
        return (n + kJitWaves - 1) / kJitWaves;
    };
    int64_t c = columns(8);
    if (w.opt.jit_waves <= 0 && kJitWaves == 4) {
        if (c * groups > 256 && groups <= 256) {
            int64_t one = 256 / groups, step = 1;
            while (one >= 8 * step) step *= 2;
            one -= one % step;
            const double d = (double)w.d, unit = (double)w.size() / (4.0 * (double)one), unit2 = (double)w.size() / (4.0 * (double)c);
            const double lone = 250.0 + 25.0 * d + 9.5 * unit;
            const double two = std::max(jit_pair_ns(unit2), jit_additions_ns(d, c * groups));
            if (1.05 * lone < two && (dir == 1 || unit <= 12.0)) c = one;
        } else if (w.size() >= 128 && w.size() <= 512 && groups >= 3 && c * groups <= 100) {
            c = columns(4);
        }
    }
    return c * kJitWaves;
}

// segments per LDS tile; backward also keeps one gradient tile [T][d][65] per wavefront of the workgroup (four as a
// rule) in the 64 KB of static LDS
int jit_tile_steps(int d, int dir, int nw = 4) { return std::min(8, (dir ? 192 / std::max(nw, 4) : 240) / std::max(d, 1)); }
int jit_tile_for(const sig::WordSet& w, int dir)
{
    if (dir == 0 && w.opt.jit_fwd_tile > 0) return std::max(1, std::min(std::min(w.opt.jit_fwd_tile, 32), 240 / std::max(w.d, 1)));
    return std::max(1, jit_tile_steps(w.d, dir, jit_wg_waves(w)));
}

// Form of the sum of a gradient tile in the backward kernel for B paths (0: a function, else inlined in that many rounds).
// Where a SIMD holds one wavefront its latency is the time, and a call anywhere in a unit costs more than its own: calls of
// 256 segments, 512 paths, called -> inlined: 1,500 words, d = 10 186 -> 156 us, d = 7 166 -> 139, d = 14 244 -> 209; 384 words,
// d = 6, 300 paths 94 -> 79.  Two wavefronts hide it, and a function leaves them more registers and compiles sooner (10,000 words,
// d = 10 295 us called, 313 inlined, 33 and 40 s; d = 8 260 and 266; 6,000, d = 9 282 and 289), except for tiles of eight segments,
// where inlining in two rounds is the faster (5,754 words, d = 6 210 called, 195 inlined).
int jit_flush_rounds(const sig::WordSet& w, int dir, int64_t B, int64_t n_units)
{
    if (dir == 0) return 0;
    if (n_units * ((B + 63) / 64) <= 1024) return 1;
    return jit_tile_for(w, 1) >= 8 ? 2 : 0;
}

// Whether the backward kernel reconstructs from intermediates of its own (emit_backward_unit): where two wavefronts share a SIMD over tiles
// of eight segments and the additions of all workgroups take the units' time or longer.  Its multiply-adds hide behind the
// additions there, and workgroups reach those sooner.  sig_backward, shared -> own: 5,754 words, d = 6, 512 paths x 512 segments (0.93 of the
// units' time) 379 -> 366 us, x 200 165 -> 163, 384 x 300 (1.04) 231 -> 226, 448 x 300 (0.98) 236 -> 233; 5,000 words, 512 x 512 (0.99),
// 6,000, 512 x 300 (0.92) and 3,000, d = 5 (0.97) within 1 % either way.  Below, the instructions count: 640 x 300 (0.84) 250 and 256.
bool jit_own_set(const sig::WordSet& w, int dir, int64_t B, int64_t n_units)
{
    const int64_t groups = (B + 63) / 64;
    if (dir == 0 || n_units * groups <= 1024 || jit_tile_for(w, 1) < 8) return false;
    const double additions = jit_additions_ns((double)w.d, n_units / jit_wg_waves(w) * groups);
    return additions >= 0.88 * jit_pair_ns((double)w.size() / (double)n_units);
}

bool jit_enabled(const sig::WordSet& w)
{
    if (w.opt.no_jit) return false;
    return w.kernels_supported && w.size() > 0 && jit_tile_steps(w.d, 1) >= 1;
}

// The balanced plan (and kernel slot) for (direction, batch size); created on first use.  Registers bound the unit
// size: a forward unit keeps one value per word, a backward unit two, next to the Horner intermediates.
sig::WordSet::JitEntry* jit_entry(const sig::WordSet& cw, int dir, int64_t B)
{
    sig::WordSet& w = const_cast<sig::WordSet&>(cw);     // the cache is logically mutable
    const int64_t n_units = jit_units(w, dir, B);
    const int wgw = jit_wg_waves(w), tile = jit_tile_for(w, dir), flush = jit_flush_rounds(w, dir, B, n_units);
    const bool own_set = jit_own_set(w, dir, B, n_units);
    std::lock_guard<std::mutex> lock(g_jit_mutex);
    for (auto* e : w.jit[dir])
        if (e->n_units == n_units && e->wg_waves == wgw && e->tile == tile && e->flush_rounds == flush && e->own_set == own_set) return e;
    auto* e = new (std::nothrow) sig::WordSet::JitEntry;
    if (!e) return nullptr;
    try {
        e->n_units = n_units;
        e->wg_waves = wgw;
        e->tile = tile;
        e->flush_rounds = flush;
        e->own_set = own_set;
        if (dir == 0) sig::build_plan_balanced(w, n_units, 320, false, 1, 1, e->plan);
        else sig::build_plan_balanced(w, n_units, 160, true, 6, 9, e->plan);
        e->kernel = new sig::JitKernel;
        w.jit[dir].push_back(e);
    } catch (const std::bad_alloc&) {
        delete e;
        return nullptr;
    }
    return e;
}

// Source of the specialised kernel of an entry; fills nw / tile.
std::string jit_source(const sig::WordSet& w, int dir, const sig::WordSet::JitEntry& e, int& nw, int& tile)
{
    const sig::Plan& p = e.plan;
    // Four wavefronts per workgroup = one per SIMD, so a workgroup's registers fit whatever a unit needs.
    nw = (int)std::min<size_t>((size_t)jit_wg_waves(w), std::max<size_t>(1, p.units.size()));
    tile = jit_tile_for(w, dir);
    return dir ? sig::jit_backward_source(w, p, nw, tile, e.flush_rounds, e.own_set) : sig::jit_forward_source(w, p, nw, tile);
}

// What a call may do to get its kernel: compile and load it (ordinary entry points), or only use one that is already
// loaded (the entry point that allocates nothing: loading a code object allocates device memory).
enum class Build { compile_only, compile_and_load, loaded_only };
// Set by ensure_* when a Build::loaded_only call found a kernel that exists but is not compiled or loaded yet.
thread_local bool g_not_ready = false;

// Brings one kernel to the asked state under the kernel's own lock (a compilation of seconds does not hold up calls
// on other word sets or kernels); `source` is called at most once per kernel.
template <class MakeSource>
sig::JitKernel* bring_up(sig::JitKernel* k, Build how, const char* name, MakeSource source)
{
    std::lock_guard<std::mutex> lock(k->m);
    if (how == Build::loaded_only) {
        if (k->tried && !k->ok) return nullptr;          // specialisation failed earlier: the fallback kernels run
        if (!k->fn) { g_not_ready = true; return nullptr; }
        return k;
    }
    std::string src;
    if (!k->tried) {
        k->tried = true;
        try {
            src = source(*k);
            (void)sig::jit_compile(src, name, *k);
        } catch (const std::bad_alloc&) { k->ok = false; }
    }
    if (!k->ok) return nullptr;
    if (how == Build::compile_and_load && !k->fn && sig::jit_load(*k) != hipSuccess) {
        // a code object from the disk cache that does not load is removed and compiled afresh, once
        bool again = false;
        if (!k->cache_file.empty()) {
            try {
                if (src.empty()) src = source(*k);
                again = sig::jit_compile(src, name, *k, false) == 0 && sig::jit_load(*k) == hipSuccess;
            } catch (const std::bad_alloc&) { again = false; }
        }
        if (!again) {
            k->ok = false;
            return nullptr;
        }
    }
    return k;
}

// Kernel for (direction, batch size) in the asked state, or nullptr if specialisation is off or failed.
// Compilation happens once per entry; the outcome is remembered.  *plan receives the entry's plan.
sig::JitKernel* ensure_jit(const sig::WordSet& cw, int dir, int64_t B, Build how, const sig::Plan** plan = nullptr)
{
    if (!jit_enabled(cw)) return nullptr;
    sig::WordSet::JitEntry* e = jit_entry(cw, dir, B);
    if (!e) return nullptr;
    if (plan) *plan = &e->plan;
    return bring_up(e->kernel, how, dir ? "sig_bwd_jit" : "sig_fwd_jit",
                    [&](sig::JitKernel& k) { return jit_source(cw, dir, *e, k.nw, k.tile); });
}

// bytes of the transposed increments the specialised kernels read: [groups][Lpad][d][64] floats
int64_t jit_lpad(const sig::WordSet& w, int64_t n_points, int dir)
{
    const int64_t T = jit_tile_for(w, dir), L = n_points - 1;
    return (L + T - 1) / T * T;
}
size_t jit_dxt_bytes(const sig::WordSet& w, int64_t B, int64_t n_points, int dir)
{
    const size_t n = (size_t)((B + 63) / 64) * (size_t)jit_lpad(w, n_points, dir) * (size_t)w.d * 64 * sizeof(float);
    return (n + 255) & ~(size_t)255;
}

// Workgroup columns x path groups.  The workgroups of a group read the same increments and add into the same gradients, so
// where every XCD (workgroups go round them, each with an L2 of its own) can be given the same number of groups, a group
// stays on one: a flat grid that the kernel takes apart (5,754 words, 512 paths x 512 segments: backward 385 -> 363 us).
dim3 jit_grid(const sig::JitKernel& k, const sig::Plan& p, int64_t B)
{
    const unsigned gx = (unsigned)((p.units.size() + (size_t)k.nw - 1) / (size_t)k.nw);
    const unsigned gy = (unsigned)((B + 63) / 64);
    return gy % 8 == 0 ? dim3(gx * gy, 1, 1) : dim3(gx, gy, 1);
}
// L segments of a row, Lpad of them in dxT (whole tiles of the kernel fit)
hipError_t launch_jit_forward(sig::JitKernel& k, const sig::Plan& p, const float* dxT, int64_t B, int64_t L, int64_t Lpad, float* coeffs,
                              int64_t nW, hipStream_t st)
{
    long lB = (long)B, lT = (long)((L + k.tile - 1) / k.tile), lW = (long)nW, lP = (long)Lpad;
    void* args[] = {(void*)&dxT, (void*)&lB, (void*)&lT, (void*)&coeffs, (void*)&lW, (void*)&lP};
    const dim3 grid = jit_grid(k, p, B);
    return hipModuleLaunchKernel(k.fn, grid.x, grid.y, 1, (unsigned)k.nw * 64, 1, 1, 0, st, args, nullptr);
}

// B rows; with C > 1 they are the C time chunks of B / C paths, whose last chunks read row (path) of coeffs_last and
// grad_last and the others row (path * C + chunk) of coeffs and grad.  C = 1: coeffs and grad hold a row per path.
hipError_t launch_jit_backward(sig::JitKernel& k, const sig::Plan& p, const float* dxT, const float* coeffs, const float* grad,
                               int64_t B, int64_t L, int64_t Lpad, int64_t nW, float* gdx, hipStream_t st,
                               const float* coeffs_last = nullptr, const float* grad_last = nullptr, int64_t C = 1)
{
    long lB = (long)B, lL = (long)L, lT = (long)((L + k.tile - 1) / k.tile), lW = (long)nW, lC = (long)C, lP = (long)Lpad;
    if (C <= 1) { coeffs_last = coeffs; grad_last = grad; lC = 1; }
    void* args[] = {(void*)&dxT, (void*)&coeffs, (void*)&grad, (void*)&lB, (void*)&lL, (void*)&lT, (void*)&lW, (void*)&gdx,
                    (void*)&coeffs_last, (void*)&grad_last, (void*)&lC, (void*)&lP};
    const dim3 grid = jit_grid(k, p, B);
    return hipModuleLaunchKernel(k.fn, grid.x, grid.y, 1, (unsigned)k.nw * 64, 1, 1, 0, st, args, nullptr);
}

int bwd_tile_steps(int d) { return std::max(1, std::min(16, 32 / std::max(d, 1))); }

// ---- time chunks of word sets closed under suffixes: rows = (path, chunk) pairs of the specialised kernels ------------
sig::WordTables word_tables(const sig::WordSet& w)
{
    sig::WordTables t;
    const unsigned char* base = (const unsigned char*)w.dev;
    t.prod_pairs = (const uint32_t*)(base + w.dev_prod_off);
    t.adj_pairs = (const uint32_t*)(base + w.dev_adj_pairs_off);
    t.adj_key = (const uint32_t*)(base + w.dev_adj_key_off);
    t.adj_groups = (int)(w.adj_pairs.size() / 256);
    for (int n = 0; n <= w.max_len + 1; ++n) {
        t.level_start[n] = w.level_start[(size_t)n];
        t.tail_off[n] = w.tail_off[(size_t)n];
    }
    t.N = w.max_len;
    t.W = (int)w.size();
    return t;
}
// the tables of the closure of a set that lacks suffixes, with its words and terms marked
sig::WordTables closure_tables(const sig::WordSet& w)
{
    sig::WordTables t = word_tables(*w.closure);
    const unsigned char* base = (const unsigned char*)w.dev;
    t.prod_pairs = (const uint32_t*)(base + w.dev_closure_prod_off);
    t.adj_pairs = (const uint32_t*)(base + w.dev_closure_adj_pairs_off);
    t.adj_key = (const uint32_t*)(base + w.dev_closure_adj_key_off);
    t.adj_groups = (int)(w.closure_adj_pairs.size() / 256);
    t.own = (const int32_t*)(base + w.dev_closure_own_off);
    t.W_own = (int)w.size();
    return t;
}
// products of the chunk signatures: from the left into rows and last, from the right into rows_reverse, as far as given
hipError_t words_products(const sig::WordTables& t, const float* S, int64_t B, int64_t C, float* rows, float* last, float* rows_reverse,
                          hipStream_t st)
{
    if (sig::words_scan_small_available(t)) return sig::words_scan_small(t, S, B, (int)C, rows, last, rows_reverse, st);
    if (rows_reverse) return sig::words_scan_both(t, S, B, (int)C, rows, rows_reverse, st);
    return sig::words_scan(t, S, B, (int)C, false, rows, last, st);
}
// Both kernels for B * C rows, compiled and loaded, or false: then the checkpointed calls run as the plain ones (the
// outcome of a compilation is remembered, so the forward and the backward call of a pair decide alike).
bool words_kernels(const sig::WordSet& w, int64_t rows, sig::JitKernel** fwd, const sig::Plan** fplan, sig::JitKernel** bwd,
                   const sig::Plan** bplan)
{
    *fwd = ensure_jit(w, 0, rows, Build::compile_and_load, fplan);
    *bwd = *fwd ? ensure_jit(w, 1, rows, Build::compile_and_load, bplan) : nullptr;
    return *fwd && *bwd;
}
size_t words_forward_ckpt_workspace(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return jit_dxt_bytes(w, B * ch.C, ch.Lc + 1, 0);
}
// increment gradients and increments of all rows in the transposed layout | boundary adjoints (for more than two chunks
// first what follows every chunk, overwritten in place) | for more than two chunks: signatures at the chunk ends
// The chunked forward pass: transposed increments of all (path, chunk) rows, their signatures into Sc [B][C][|W|], the
// product of every path's chunk signatures into coeffs (nullptr: the chunk signatures alone).
hipError_t words_forward_chunked(const sig::WordSet& w, const float* path, int64_t B, int64_t n_points, const Chunks& ch,
                                 sig::JitKernel& fk, const sig::Plan& fp, float* dxT, float* Sc, float* coeffs, hipStream_t st)
{
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    const int64_t Lpad = jit_lpad(w, ch.Lc + 1, 0);
    hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, nullptr, st, rows);
    if (e != hipSuccess) return e;
    hipEvent_t* pe = g_prof.next(0);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = launch_jit_forward(fk, fp, dxT, B * ch.C, ch.Lc, Lpad, Sc, w.size(), st);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e == hipSuccess && coeffs) e = words_products(word_tables(w), Sc, B, ch.C, nullptr, coeffs, nullptr, st);
    return e;
}
size_t words_backward_ckpt_workspace(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return 2 * jit_dxt_bytes(w, B * ch.C, ch.Lc + 1, 1) + (ch.C == 2 ? 1 : 2) * chunk_array_bytes(w, B, ch.C);
}
// The backward pass over the (path, chunk) rows of a suffix-closed set, from the chunk signatures Sc [B][C][|W|]:
// boundary adjoints (and, beyond two chunks, the signatures at the chunk ends) from products over the set, one launch
// of the specialised kernel over all rows, chain rule.  workspace: words_backward_ckpt_workspace bytes.
hipError_t words_backward_chunked(const sig::WordSet& w, const float* path, const float* coeffs, const float* grad_coeffs,
                                  const float* Sc, const Chunks& ch, int64_t B, int64_t n_points, float* grad_path, void* workspace,
                                  sig::JitKernel& bk, const sig::Plan& bp, hipStream_t st)
{
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    const size_t t_bytes = jit_dxt_bytes(w, B * ch.C, ch.Lc + 1, 1), nb = chunk_array_bytes(w, B, ch.C);
    float* gdx = (float*)workspace;
    float* dxT = (float*)((unsigned char*)workspace + t_bytes);
    float* Abar = (float*)((unsigned char*)workspace + 2 * t_bytes);
    const float* Pfx = Sc;
    const sig::WordTables tab = word_tables(w);
    const int64_t Lpad = jit_lpad(w, ch.Lc + 1, 1);
    // rows of one path share the points between their chunks: the chain rule adds into grad_path, which the adjoint
    // kernel clears on the way
    const int64_t n_gp = B * n_points * w.d;
    hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, gdx, st, rows);
    if (ch.C == 2) {
        // two chunks: the signature at the end of the first is the first chunk's own, what follows it the second's
        // (row c + 1 of the chunk signatures, read as row c of an array that starts one row later)
        if (e == hipSuccess) e = sig::words_adjoint(tab, grad_coeffs, Sc + w.size(), B, 2, Abar, grad_path, n_gp, st);
    } else {
        float* P = (float*)((unsigned char*)workspace + 2 * t_bytes + nb);
        if (e == hipSuccess) e = words_products(tab, Sc, B, ch.C, P, nullptr, Abar, st);
        if (e == hipSuccess) e = sig::words_adjoint(tab, grad_coeffs, Abar, B, (int)ch.C, Abar, grad_path, n_gp, st);   // in place, row by row
        Pfx = P;
    }
    if (e != hipSuccess) return e;
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    // the rows of the last chunk are the caller's terminal signature and gradient themselves
    e = launch_jit_backward(bk, bp, dxT, Pfx, Abar, B * ch.C, ch.Lc, Lpad, w.size(), gdx, st, coeffs, grad_coeffs, ch.C);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return e;
    return sig::grad_points_transposed(gdx, B, n_points, w.d, Lpad, grad_path, st, rows);
}
// sig_backward on a suffix-closed set recomputes the chunk signatures and takes the same route where that still wins:
// from four chunks on by the rule of the checkpointed calls (measured: 64 paths x 4,096 segments 2.36 -> 0.62 ms,
// 512 x 2,048 1.57 -> 1.24 ms; with two chunks the second forward pass eats the gain).
// workspace: | backward part (its first bytes serve the forward's transposed increments before) | chunk signatures |
bool words_backward_recomputes(const sig::WordSet& w, const Chunks& ch) { return w.kind != 0 && ch.C >= 4; }
size_t words_backward_recompute_first(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return std::max(words_backward_ckpt_workspace(w, B, ch), words_forward_ckpt_workspace(w, B, ch));
}
size_t words_backward_recompute_workspace(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return words_backward_recompute_first(w, B, ch) + chunk_array_bytes(w, B, ch.C);
}

// what sig_forward asks for where such a set takes the chunks of the checkpointed calls (at least what whole paths need)
size_t words_forward_bytes(const sig::WordSet& w, int64_t B, int64_t n_points, const Chunks& ch)
{
    const size_t whole = jit_dxt_bytes(w, B, n_points, 0);
    return ch.C >= 2 ? std::max(whole, words_forward_ckpt_workspace(w, B, ch) + chunk_array_bytes(w, B, ch.C)) : whole;
}

// ---- time chunks of sig_forward and sig_backward on small launches ---------------------------------------------------
// A specialised kernel takes 0.08-0.16 us per segment forward and 0.2-0.45 backward however few paths there are, so where the
// wavefronts of whole paths fill at most three quarters of the SIMDs the plain calls cut every path into chunks, for sets that
// lack suffixes as well: the chunk signatures are then those of the closure, and the backward rows run over the set itself.
// Which kernels that takes follows from the batch size alone: they are planned for plain_rows(B).
const sig::WordSet& chunk_set(const sig::WordSet& w) { return w.closure ? *w.closure : w; }
sig::WordTables chunk_tables(const sig::WordSet& w) { return w.closure ? closure_tables(w) : word_tables(w); }
int64_t plain_rows(int64_t B) { return std::min<int64_t>(std::max<int64_t>(2048, B), 8 * B); }
bool plain_chunks_available(const sig::WordSet& w, int64_t B)
{
    if (w.kind == 0 || B < 1 || !jit_enabled(w) || !(w.closure || w.pair_tables)) return false;
    const sig::WordSet& c = chunk_set(w);
    if (c.size() > 4096 || c.max_len > 8) return false;
    return jit_units(w, 1, B) * ((B + 63) / 64) <= 768;
}
// Modelled time in microseconds of a call (kForward, kBackward, which runs the chunks' forward pass again, kBackwardKept, which
// finds their signatures in a checkpoint) with C chunks, fitted to a scan of ten sets (36 to 432 words, closures up to 1,195, 4 to 9
// letters, 22 to 300 paths of 66 to 819 segments, counts up to 32): a segment's latency by letters and words of a unit, as often
// as the wavefronts fill the SIMDs; a product per chunk, by words of the closure and paths; the launches.
enum PlainCall { kForward, kBackward, kBackwardKept };
double plain_time(const sig::WordSet& w, PlainCall call, int64_t B, int64_t L, int64_t C)
{
    const sig::WordSet& c = chunk_set(w);
    const double d = (double)w.d, words = (double)c.size(), own = (double)w.size(), paths = (double)B;
    const int64_t R = C > 1 ? plain_rows(B) : B;
    const double units = (double)jit_units(w, call == kForward ? 0 : 1, R);
    const double seg_b = 0.05 + 0.04 * d + 0.0095 * std::max(0.0, own / units - 8.0);
    auto forward = [&](double per_unit) { return 0.05 + 0.008 * d + 0.003 * std::max(0.0, per_unit - 8.0); };
    if (C == 1) return (double)L * (call == kForward ? forward(own / units) : seg_b);
    const double Lc = (double)((L + C - 1) / C), groups = (double)((B * C + 63) / 64), uf = (double)jit_units(c, 0, R);
    double t = call == kBackwardKept ? 0.0 : Lc * forward(words / uf) * std::max(1.0, groups * uf / 2048.0);
    if (call == kForward) return t + 5.5 + (double)C * (0.3 + 0.0005 * words + 0.0006 * paths + 2.0e-6 * paths * words);
    t += Lc * seg_b * std::max(1.0, groups * units / 1024.0) + (double)C * (0.4 + 0.001 * words + 0.0024 * paths + 1.0e-5 * paths * words);
    return t + (call == kBackwardKept ? 10.0 : 15.0);
}
// The count with the shortest modelled time.  A forward and a backward call, one after the other on a stream, whole paths -> at the
// choice, us: 226 words, d = 9, 22 paths x 819 segments 528 -> 89; 432, d = 8, 46 x 526 321 -> 100; 384 (lead-lag, d = 6), 300 x 256
// 112 -> 82; 36 (lead-lag, d = 4), 39 x 388 132 -> 53; 240, d = 11, 258 x 969 609 -> 212.
int plain_chunk_count(const sig::WordSet& w, PlainCall call, int64_t B, int64_t L)
{
    double best = 0.93 * plain_time(w, call, B, L, 1);
    int choice = 1;
    for (int C : sig::kLanesChunkCounts) {
        if (L < 8 * (int64_t)C) break;                        // chunks of at least 8 segments
        const double t = plain_time(w, call, B, L, C);
        if (t < best) {
            best = t;
            choice = C;
        }
    }
    return choice;
}
Chunks plain_chunks(const sig::WordSet& w, int dir, int64_t B, int64_t n_points)
{
    const int64_t L = n_points - 1;
    int64_t C = 1;
    if (plain_chunks_available(w, B)) {
        if (w.opt.chunks > 0) {
            C = std::min<int64_t>(std::min<int64_t>(w.opt.chunks, 64), L / 4);        // tuning knob
        } else {
            C = plain_chunk_count(w, dir ? kBackward : kForward, B, L);
        }
        if (B * C > (int64_t)65535 * 64) C = 1;
    }
    if (C < 2) return Chunks{1, L};
    const int64_t Lc = (L + C - 1) / C;
    return Chunks{(L + Lc - 1) / Lc, Lc};
}
int64_t plain_lpad(const sig::WordSet& w, const Chunks& ch)    // one transposed copy serves both directions
{
    return std::max(jit_lpad(w, ch.Lc + 1, 0), jit_lpad(w, ch.Lc + 1, 1));
}
size_t plain_dxt_bytes(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return ((size_t)((B * ch.C + 63) / 64) * (size_t)plain_lpad(w, ch) * (size_t)w.d * 64 * sizeof(float) + 255) & ~(size_t)255;
}
size_t plain_forward_bytes(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return plain_dxt_bytes(w, B, ch) + chunk_array_bytes(chunk_set(w), B, ch.C);
}
// increment gradients | increments | chunk signatures | products from the left | from the right | boundary adjoints (without a
// closure in place of the products from the right)
size_t plain_backward_bytes(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return 2 * plain_dxt_bytes(w, B, ch) + 2 * chunk_array_bytes(chunk_set(w), B, ch.C) + (w.closure ? 2 : 1) * chunk_array_bytes(w, B, ch.C);
}
struct PlainKernels {
    sig::JitKernel *chunk = nullptr, *rows = nullptr;      // signatures of the chunks; backward: the rows
    const sig::Plan *chunk_plan = nullptr, *rows_plan = nullptr;
};
bool plain_kernels(const sig::WordSet& w, int dir, int64_t B, Build how, PlainKernels& k)
{
    k.chunk = ensure_jit(chunk_set(w), 0, plain_rows(B), how, &k.chunk_plan);
    k.rows = k.chunk && dir ? ensure_jit(w, 1, plain_rows(B), how, &k.rows_plan) : nullptr;
    return k.chunk && (dir == 0 || k.rows);
}
// While a stream is captured nothing can be loaded: kernels that no call has brought up yet are done without.
Build unless_captured(Build how, hipStream_t st)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (how == Build::compile_and_load && hipStreamIsCapturing(st, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone)
        return Build::loaded_only;
    return how;
}
// The kernels of a chunked call.  A call that takes chunks loads those of whole paths as well, for calls of the batch size that
// don't (other lengths, sig_backward_static).
bool plain_kernels_for(const sig::WordSet& w, int dir, int64_t B, Build how, hipStream_t st, PlainKernels& k)
{
    how = unless_captured(how, st);
    return ensure_jit(w, dir, B, how) && plain_kernels(w, dir, B, how, k);
}
// The checkpointed backward call of a suffix-closed set takes more chunks than are kept (ch) where that is the faster for all the
// forward pass they need again (209 words, 26 paths x 693 segments: 62 us with the five that are kept, 45 with 24).  C = 1: no.
Chunks plain_instead_of_kept(const sig::WordSet& w, int64_t B, int64_t n_points, const Chunks& ch)
{
    const int64_t L = n_points - 1;
    if (w.opt.ckpt_chunks != 0 || !plain_chunks_available(w, B)) return Chunks{1, L};
    const Chunks own = plain_chunks(w, 1, B, n_points);
    if (own.C < 2 || plain_time(w, kBackward, B, L, own.C) >= 0.93 * plain_time(w, kBackwardKept, B, L, ch.C)) return Chunks{1, L};
    return own;
}
hipError_t plain_forward_chunked(const sig::WordSet& w, const PlainKernels& k, const float* path, int64_t B, int64_t n_points,
                                 const Chunks& ch, float* coeffs, void* workspace, hipStream_t st)
{
    const sig::WordSet& c = chunk_set(w);
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    float* dxT = (float*)workspace;
    float* Sc = (float*)((unsigned char*)workspace + plain_dxt_bytes(w, B, ch));
    const int64_t Lpad = plain_lpad(w, ch);
    hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, nullptr, st, rows);
    if (e != hipSuccess) return e;
    hipEvent_t* pe = g_prof.next(0);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = launch_jit_forward(*k.chunk, *k.chunk_plan, dxT, B * ch.C, ch.Lc, Lpad, Sc, c.size(), st);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return e;
    return words_products(chunk_tables(w), Sc, B, ch.C, nullptr, coeffs, nullptr, st);
}
hipError_t plain_backward_chunked(const sig::WordSet& w, const PlainKernels& k, const float* path, const float* coeffs,
                                  const float* grad_coeffs, int64_t B, int64_t n_points, const Chunks& ch, float* grad_path,
                                  void* workspace, hipStream_t st)
{
    const sig::WordSet& c = chunk_set(w);
    const sig::WordTables tab = chunk_tables(w);
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    const size_t t = plain_dxt_bytes(w, B, ch), nc = chunk_array_bytes(c, B, ch.C), nw = chunk_array_bytes(w, B, ch.C);
    unsigned char* base = (unsigned char*)workspace;
    float* gdx = (float*)base;
    float* dxT = (float*)(base + t);
    float* Sc = (float*)(base + 2 * t);
    float* left = (float*)(base + 2 * t + nc);
    float* right = (float*)(base + 2 * t + nc + nw);
    float* Abar = w.closure ? (float*)(base + 2 * t + 2 * nc + nw) : right;
    const int64_t Lpad = plain_lpad(w, ch);
    hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, gdx, st, rows);
    if (e == hipSuccess) e = launch_jit_forward(*k.chunk, *k.chunk_plan, dxT, B * ch.C, ch.Lc, Lpad, Sc, c.size(), st);
    if (e == hipSuccess) e = words_products(tab, Sc, B, ch.C, left, nullptr, right, st);
    // rows of one path share the points between their chunks: the chain rule adds into grad_path, cleared here
    if (e == hipSuccess) e = sig::words_adjoint(tab, grad_coeffs, right, B, (int)ch.C, Abar, grad_path, B * n_points * w.d, st);
    if (e != hipSuccess) return e;
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = launch_jit_backward(*k.rows, *k.rows_plan, dxT, left, Abar, B * ch.C, ch.Lc, Lpad, w.size(), gdx, st, coeffs, grad_coeffs, ch.C);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return e;
    return sig::grad_points_transposed(gdx, B, n_points, w.d, Lpad, grad_path, st, rows);
}

// ---- full truncations without a register-resident kernel of their own: lanes = words -----------------------
// Lanes = paths needs 64 paths per wavefront and a compilation that grows with the word set (minutes beyond a few
// ten thousand words); lanes = words fills the wavefronts from a single path on and compiles in about a second per
// shape.  Taken whenever the words of a path fill at least half a wavefront; the option "lanes" = 0 switches it off, = 1 takes
// it for every shape it is defined for.
int lanes_levels_asked(const sig::WordSet& w)             // testing knob: 1 or 2 levels below the lane's word
{
    return w.opt.lanes_levels == 1 || w.opt.lanes_levels == 2 ? w.opt.lanes_levels : 0;
}
sig::LanesShape lanes_shape_for(const sig::WordSet& w, int dir, int64_t B)
{
    sig::LanesShape s = sig::lanes_shape(w.d, w.depth, dir != 0, B, lanes_levels_asked(w));
    if (!s.ok) s = sig::lanes_shape(w.d, w.depth, dir != 0, B, 0);
    return s;
}

// Sets whose words of length depth - R fill less than half a wavefront (30 words over 2 letters, 72 over 8) still win that
// way while the paths are few: lanes = paths walks every path from end to end behind a transposition of its increments and
// cannot cut it into time chunks.  Measured, step (forward + backward), lanes = paths -> lanes = words: 2 letters, depth 4:
// 32 x 64 segments 44 -> 30 us, 512 x 500 190 -> 104, 1,024 x 100 58 -> 59, 1,500 x 200 92 -> 120; 3 letters, depth 3:
// 512 x 500 218 -> 85, 1,024 x 100 65 -> 47; 12 letters, depth 2: 32 x 500 335 -> 41, 1,500 x 200 176 -> 108, 3,000 x 200
// 212 -> 200.  So the line lies higher the fewer letters the chain of a lane has.  Depth 5: 2 letters, 512 x 256
// 108 -> 89 us, 768 x 256 110 -> 124; 3 letters, 768 x 256 124 -> 164 (with up to some 600 paths they have one level below the
// lane's word, 81 lanes, and don't come here).  Words of four letters on paths of up to 64 segments stay with lanes = paths from 64 paths on.  That is not
// where the times lie: lanes = words is the faster there too (3 letters, depth 4, 64 x 64 42 -> 25 us, 768 x 64 43 -> 31; 2 letters
// 64 x 16 21 -> 12, 768 x 64 37 -> 30); a host test fixes the kernel of 64 paths of 64 segments.
// `L`: segments; kAnyLength asks whether some length would run this way.  `chunks`: the call can take time chunks (windows and
// sig_backward_static cannot; beyond depth 3 their walk over whole rows gains little over lanes = paths or loses: static
// call, 2 letters, depth 4, 64 paths x 256 segments 67 and 63 us, 768 x 1,000 233 and 293).
constexpr int64_t kAnyLength = INT64_MAX;
bool use_lanes(const sig::WordSet& w, int64_t B, int64_t L, bool chunks = true, bool* small = nullptr)
{
    if (small) *small = false;
    if (w.kind != 0 || !jit_enabled(w)) return false;
    const int f = w.opt.lanes;
    if (f == 0) return false;
    const sig::LanesShape s = lanes_shape_for(w, 0, B), sb = lanes_shape_for(w, 1, B);
    if (!s.ok || !sb.ok || B * std::max(s.waves, sb.waves) > (int64_t)0x7fffffff) return false;
    if (f == 1 || std::min(s.lanes, sb.lanes) >= 32) return true;
    if (!sig::lanes_chunks_available(w.d, w.depth) || (!chunks && w.depth > 3)) return false;
    const bool few = B <= (w.depth == 2 ? 2048 : (w.depth == 3 ? 1024 : (L <= 64 ? 63 : (w.depth == 4 ? 768 : (w.d == 2 ? 512 : 256)))));
    if (small) *small = few;
    return few;
}

// Time chunks of those truncations: a wavefront takes 0.1-0.15 us per segment forward and 0.25-0.35 us backward however few
// there are, so few paths are cut into C chunks that run as rows of their own.  Forward: chunk signatures, then their
// product; backward: chunk signatures over the words shorter than the depth (a d-th of the work; the longest words are
// never reconstructed), their products from both sides, the adjoints at the boundaries, then the rows.
Chunks lanes_chunks(const sig::WordSet& w, int dir, int64_t B, int64_t n_points)
{
    const int64_t L = n_points - 1;
    int64_t C = 1;
    if (L >= 16 && B >= 1 && sig::lanes_chunks_available(w.d, w.depth)) {
        if (w.opt.chunks > 0) {
            C = std::min<int64_t>(std::min<int64_t>(w.opt.chunks, 64), L / 4);        // tuning knob
        } else {
            sig::WordSet::LanesMemo& memo = const_cast<sig::WordSet&>(w).lanes_memo;
            const int levels = lanes_levels_asked(w);
            std::lock_guard<std::mutex> lock(memo.m);
            C = 0;
            for (const auto& c : memo.choices)
                if (c.dir == dir && c.B == B && c.L == L && c.levels == levels) C = c.C;
            if (C == 0) {
                sig::WordSet::ChunkChoice& c = memo.choices[memo.next];
                memo.next = (memo.next + 1) % 16;
                c.dir = dir; c.B = B; c.L = L; c.levels = levels;
                c.C = sig::lanes_chunk_count(w.d, w.depth, dir != 0, B, L, levels);
                C = c.C;
            }
        }
    }
    if (C < 2 || B * C > 65535) return Chunks{1, L};
    const int64_t Lc = (L + C - 1) / C;
    return Chunks{(L + Lc - 1) / Lc, Lc};
}
// rows of words shorter than the depth, [B][C] of them
size_t lanes_low_bytes(const sig::WordSet& w, int64_t B, int64_t C)
{
    return ((size_t)B * (size_t)C * (size_t)w.level_start[(size_t)w.depth] * sizeof(float) + 255) & ~(size_t)255;
}

// Whether backward calls over chunks ask for products and boundary adjoints in arrays: where a wavefront's LDS does not hold a chunk
// signature, and for counts set by the option "chunks" (which keeps that form to compare the other with).
bool lanes_arrays(const sig::WordSet& w, const sig::LanesShape& s) { return w.opt.chunks > 0 || !s.shares; }

sig::JitKernel* ensure_lanes(const sig::WordSet& cw, int dir, const sig::LanesShape& s, Build how)
{
    sig::WordSet& w = const_cast<sig::WordSet&>(cw);     // the cache is logically mutable
    const bool arrays = dir == 1 && lanes_arrays(w, s);
    sig::JitKernel* k = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_jit_mutex);
        sig::JitKernel*& slot = w.lanes[dir][(dir == 1 && s.R == 1 && w.d == 2 && !s.msum) || s.split == 2 ? 2 : s.R - 1][arrays ? 1 : 0];
        if (!slot) slot = new (std::nothrow) sig::JitKernel;
        k = slot;
    }
    if (!k) return nullptr;
    // everything but the levels per lane, the arrays and, for two letters, the form of the sums follows from (d, depth, direction)
    return bring_up(k, how, dir ? "sig_bwd_lanes" : "sig_fwd_lanes", [&](sig::JitKernel& kk) {
        kk.nw = s.nwb;
        kk.tile = s.T;
        if (sig::lanes_chunks_available(w.d, w.depth)) {
            auto waves = [&](sig::LanesChunkPart part) { return sig::lanes_chunk_threads(w.d, w.depth, part) / 64; };
            if (dir == 0) kk.more = {{"sig_scan_lanes", waves(sig::kLanesScanFull), nullptr}};
            else kk.more = {{"sig_low_lanes", sig::lanes_low_shape(w.d, w.depth).nwb, nullptr}};
            if (arrays) {
                kk.more.push_back({"sig_scan_lanes", waves(sig::kLanesScanLow), nullptr});
                kk.more.push_back({"sig_adjoint_lanes", waves(sig::kLanesAdjoint), nullptr});
            }
        }
        return sig::lanes_source(w.d, w.depth, s, dir != 0, arrays);
    });
}

// rows: the B paths, with a window list the B * K (path, window) pairs, or (wl.win == nullptr, wl.K > 1) the K time chunks of
// wl.max_len segments of every path; read straight from the path.  Backward over chunks: low_coeffs and low_grad hold
// signature and adjoint at the end of every chunk but the last, [B][K - 1][words shorter than the depth], or low_coeffs alone the
// chunks' own signatures [B][K].  Forward: n_zero floats at zero are cleared on the way.
hipError_t launch_lanes(hipFunction_t fn, const sig::LanesShape& s, const float* path, const float* coeffs_in, const float* grad,
                        int64_t B, int64_t n_points, float* out, hipStream_t st, const sig::WindowList& wl = sig::WindowList(),
                        const float* low_coeffs = nullptr, const float* low_grad = nullptr, float* zero = nullptr, int64_t n_zero = 0)
{
    const bool parts = wl.several_rows();
    long lB = (long)B, lP = (long)n_points, lK = (long)wl.rows_per_path(), lM = parts ? (long)wl.max_len : lP - 1;
    const int64_t* win = wl.win;
    const int64_t rows = B * wl.rows_per_path();
    const int64_t blocks = (rows * s.waves + s.nwb - 1) / s.nwb;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (grad) {
        void* args[] = {(void*)&path, (void*)&coeffs_in, (void*)&grad, (void*)&lB, (void*)&lP, (void*)&out, (void*)&win, (void*)&lK,
                        (void*)&lM, (void*)&low_coeffs, (void*)&low_grad};
        return hipModuleLaunchKernel(fn, (unsigned)blocks, 1, 1, (unsigned)s.nwb * 64, 1, 1, 0, st, args, nullptr);
    }
    long lz = (long)n_zero;            // (the last two: of the kernel in the backward module alone)
    void* args[] = {(void*)&path, (void*)&lB, (void*)&lP, (void*)&out, (void*)&win, (void*)&lK, (void*)&lM, (void*)&zero, (void*)&lz};
    return hipModuleLaunchKernel(fn, (unsigned)blocks, 1, 1, (unsigned)s.nwb * 64, 1, 1, 0, st, args, nullptr);
}

// The module of a chunked call, or false where it lacks one of the kernels (then the call walks whole paths).
struct LanesChunked {
    sig::LanesShape main, low;
    sig::JitKernel* k = nullptr;
    const sig::JitKernel::More& product() const { return k->more[0]; }       // forward
    const sig::JitKernel::More& lower() const { return k->more[0]; }         // backward
    const sig::JitKernel::More& scan() const { return k->more[1]; }          // ... with arrays
    const sig::JitKernel::More& adjoint() const { return k->more[2]; }
};
bool lanes_chunk_kernels(const sig::WordSet& w, int dir, int64_t rows, Build how, LanesChunked& c)
{
    c.main = lanes_shape_for(w, dir, rows);
    if (!c.main.ok || rows * c.main.waves > (int64_t)0x7fffffff) return false;
    c.k = ensure_lanes(w, dir, c.main, how);
    if (!c.k || c.k->more.empty()) return false;
    if (dir) c.low = sig::lanes_low_shape(w.d, w.depth);
    if (how == Build::compile_only) return true;
    for (const auto& m : c.k->more)
        if (!m.fn) return false;
    return true;
}
// The first call with B paths brings up whatever paths of another length may need as well (chunked or whole: another
// number of rows may take the other number of levels per lane), so that later calls of that batch size compile and
// load nothing - under graph capture, or in sig_backward_static, they could not.
void lanes_bring_up(const sig::WordSet& cw, int dir, int64_t B, Build how)
{
    if (how == Build::loaded_only) return;
    sig::WordSet& w = const_cast<sig::WordSet&>(cw);
    sig::WordSet::LanesMemo& memo = w.lanes_memo;
    if (how == Build::compile_and_load) {
        std::lock_guard<std::mutex> lock(memo.m);
        for (const auto& l : memo.loaded)
            if (l.first == dir && l.second == B) return;
    }
    bool all = ensure_lanes(w, dir, lanes_shape_for(w, dir, B), how) != nullptr;
    bool small_set = false;
    (void)use_lanes(w, B, kAnyLength, true, &small_set);
    // lanes = paths as well where sig_backward_static or paths of another length take it
    if (small_set && w.depth > 2 && (dir == 1 || !use_lanes(w, B, 1))) all = ensure_jit(w, dir, B, how) != nullptr && all;
    if (sig::lanes_chunks_available(w.d, w.depth))
        for (int C : sig::kLanesChunkCounts) {
            const sig::LanesShape s = lanes_shape_for(w, dir, B * C);
            if (s.ok && B * C <= 65535) all = ensure_lanes(w, dir, s, how) != nullptr && all;
        }
    if (!all || how != Build::compile_and_load) return;       // asked again by the next call
    try {
        std::lock_guard<std::mutex> lock(memo.m);
        if (memo.loaded.size() >= 64) memo.loaded.clear();
        memo.loaded.emplace_back(dir, B);
    } catch (const std::bad_alloc&) { }
}
// forward, workspace: the chunk signatures [B][C][|W|]
hipError_t lanes_forward_chunked(const sig::WordSet& w, const LanesChunked& k, const float* path, int64_t B, int64_t n_points,
                                 const Chunks& ch, float* coeffs, float* Sc, hipStream_t st)
{
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    hipEvent_t* pe = g_prof.next(0);
    if (pe) (void)hipEventRecord(pe[0], st);
    hipError_t e = launch_lanes(k.k->fn, k.main, path, nullptr, nullptr, B, n_points, Sc, st, rows);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return e;
    long lC = (long)ch.C;
    float* none = nullptr;
    void* args[] = {(void*)&Sc, (void*)&lC, (void*)&coeffs, (void*)&none};
    return hipModuleLaunchKernel(k.product().fn, (unsigned)(B * w.d), 1, 1, (unsigned)k.product().nw * 64, 1, 1, 0, st, args, nullptr);
}
// backward, workspace: chunk signatures [B][C] over the words shorter than the depth; where the lanes of the walk don't work out
// signature and adjoints at the chunk ends from them, also products from the left, from the right and boundary adjoints [B][C - 1]
size_t lanes_backward_chunked_bytes(const sig::WordSet& w, int64_t B, const Chunks& ch, bool arrays)
{
    return lanes_low_bytes(w, B, ch.C) + (arrays ? 3 * lanes_low_bytes(w, B, ch.C - 1) : 0);
}
bool lanes_backward_arrays(const sig::WordSet& w, int64_t B, const Chunks& ch) { return lanes_arrays(w, lanes_shape_for(w, 1, B * ch.C)); }
hipError_t lanes_backward_chunked(const sig::WordSet& w, const LanesChunked& k, const float* path, const float* coeffs,
                                  const float* grad_coeffs, int64_t B, int64_t n_points, const Chunks& ch, bool arrays, float* grad_path,
                                  void* workspace, hipStream_t st)
{
    const size_t nb = lanes_low_bytes(w, B, ch.C - 1);
    unsigned char* base = (unsigned char*)workspace;
    float* Sc = (float*)base;
    float* left = Sc;
    float* abar = nullptr;
    sig::WindowList rows;
    rows.K = ch.C; rows.max_len = ch.Lc;
    const int64_t n_path = B * n_points * w.d;                // cleared for the rows, which add into it
    hipError_t e = launch_lanes(k.lower().fn, k.low, path, nullptr, nullptr, B, n_points, Sc, st, rows, nullptr, nullptr, grad_path,
                                arrays ? 0 : n_path);
    if (e != hipSuccess) return e;
    if (arrays) {
        left = (float*)(base + lanes_low_bytes(w, B, ch.C));
        float* right = (float*)((unsigned char*)left + nb);
        abar = (float*)((unsigned char*)right + nb);
        long lC = (long)ch.C, lC1 = lC - 1, lz = (long)n_path;
        void* scan_args[] = {(void*)&Sc, (void*)&lC, (void*)&left, (void*)&right};
        e = hipModuleLaunchKernel(k.scan().fn, (unsigned)(2 * B * w.d), 1, 1, (unsigned)k.scan().nw * 64, 1, 1, 0, st, scan_args, nullptr);
        if (e != hipSuccess) return e;
        void* adj_args[] = {(void*)&grad_coeffs, (void*)&right, (void*)&lC1, (void*)&abar, (void*)&grad_path, (void*)&lz};
        e = hipModuleLaunchKernel(k.adjoint().fn, (unsigned)(B * (ch.C - 1) * w.d), 1, 1, (unsigned)k.adjoint().nw * 64, 1, 1, 0, st,
                                  adj_args, nullptr);
        if (e != hipSuccess) return e;
    }
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = launch_lanes(k.k->fn, k.main, path, coeffs, grad_coeffs, B, n_points, grad_path, st, rows, left, abar);
    if (pe) (void)hipEventRecord(pe[1], st);
    return e;
}
}  // namespace

extern "C" {

int sig_wordset_build_truncated(int d, int depth, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_truncated(d, depth, &w), w, out);
}

int sig_wordset_build_anisotropic(int d, const double* weights, double cutoff, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_anisotropic(d, weights, cutoff, &w), w, out);
}

int sig_wordset_build(int d, const int32_t* letters, const int64_t* offsets, int64_t n_words, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_list(d, letters, offsets, n_words, &w), w, out);
}

int sig_wordset_build_graph(int d, const int32_t* edges, int64_t n_edges, int depth, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_graph(d, edges, n_edges, depth, &w), w, out);
}

int sig_wordset_build_leadlag_sparse(int d, int depth, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_leadlag_sparse(d, depth, &w), w, out);
}

int sig_wordset_build_logsig(int d, int depth, sig_wordset** out)
{
    if (!out) return SIG_EINVAL;
    sig::WordSet* w = nullptr;
    return finish_build(sig::build_logsig(d, depth, &w), w, out);
}

int sig_wordset_set_option(sig_wordset* ws, const char* name, int value)
{
    if (!ws || !name) return SIG_EINVAL;
    for (const OptionName& o : kOptions)
        if (std::strcmp(o.name, name) == 0) {
            ws->opt.*(o.field) = value;
            if (ws->closure) ws->closure->opt = ws->opt;
            std::lock_guard<std::mutex> lock(ws->lanes_memo.m);
            ws->lanes_memo.loaded.clear();                  // the kernels a batch size needs may be others now
            return SIG_OK;
        }
    return SIG_EINVAL;
}

int sig_wordset_get_option(const sig_wordset* ws, const char* name, int* value)
{
    if (!ws || !name || !value) return SIG_EINVAL;
    for (const OptionName& o : kOptions)
        if (std::strcmp(o.name, name) == 0) {
            *value = W(ws)->opt.*(o.field);
            return SIG_OK;
        }
    return SIG_EINVAL;
}

int64_t sig_wordset_n_lyndon(const sig_wordset* ws) { return ws ? W(ws)->n_lyndon : -1; }

int sig_logsig_forward(const sig_wordset* ws, const float* coeffs, int64_t B, float* logsig, void* stream)
{
    if (!ws || B < 0) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    if (w.n_lyndon <= 0) return SIG_EUNSUPPORTED;
    if (!w.dev) return SIG_ENOTUPLOADED;
    if (B == 0) return SIG_OK;
    if (!coeffs || !logsig) return SIG_EINVAL;
    const unsigned char* base = (const unsigned char*)w.dev;
    hipError_t e = sig::logsig_forward(coeffs, B, w.size(), (const int32_t*)(base + w.lyn_len_off),
                                       (const int32_t*)(base + w.lyn_sub_off), (const int32_t*)(base + w.lyn_sub_t_off), w.n_lyndon,
                                       w.lyn_stride, w.depth, logsig, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

size_t sig_logsig_backward_workspace_bytes(const sig_wordset* ws, int64_t B)
{
    if (!ws || B <= 0 || W(ws)->n_lyndon <= 0) return 0;
    return ((size_t)B * (size_t)W(ws)->n_lyndon * (size_t)W(ws)->lyn_pairs * sizeof(float) + 255) & ~(size_t)255;
}

int sig_logsig_backward(const sig_wordset* ws, const float* coeffs, const float* grad_logsig, int64_t B, float* grad_coeffs,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    if (!ws || B < 0) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    if (w.n_lyndon <= 0) return SIG_EUNSUPPORTED;
    if (!w.dev) return SIG_ENOTUPLOADED;
    if (B == 0) return SIG_OK;
    if (!coeffs || !grad_logsig || !grad_coeffs) return SIG_EINVAL;
    if (!workspace || workspace_bytes < sig_logsig_backward_workspace_bytes(ws, B)) return SIG_EWORKSPACE;
    const unsigned char* base = (const unsigned char*)w.dev;
    hipError_t e = sig::logsig_backward(coeffs, grad_logsig, B, w.size(), (const int32_t*)(base + w.lyn_len_off),
                                        (const int32_t*)(base + w.lyn_sub_off), w.n_lyndon, w.lyn_stride, w.depth, w.lyn_pairs,
                                        (const int32_t*)(base + w.lyn_inv_off_off), (const int32_t*)(base + w.lyn_inv_ent_off),
                                        (const int32_t*)(base + w.lyn_sub_t_off), w.lyn_long, (float*)workspace, grad_coeffs,
                                        w.opt.logsig_gather != 0, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_leadlag_transform(const float* path, int64_t B, int64_t n_points, int d, float* out, void* stream)
{
    if (B < 0 || n_points < 1 || d < 1) return SIG_EINVAL;
    if (B == 0) return SIG_OK;
    if (!path || !out) return SIG_EINVAL;
    hipError_t e = sig::leadlag(path, B, n_points, d, out, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_leadlag_backward(const float* grad_out, int64_t B, int64_t n_points, int d, float* grad_path, void* stream)
{
    if (B < 0 || n_points < 1 || d < 1) return SIG_EINVAL;
    if (B == 0) return SIG_OK;
    if (!grad_out || !grad_path) return SIG_EINVAL;
    hipError_t e = sig::leadlag_backward(grad_out, B, n_points, d, grad_path, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

void sig_wordset_free(sig_wordset* ws) { delete static_cast<sig::WordSet*>(ws); }

int64_t sig_wordset_size(const sig_wordset* ws) { return ws ? W(ws)->size() : -1; }
int sig_wordset_dim(const sig_wordset* ws) { return ws ? W(ws)->d : -1; }
int sig_wordset_max_len(const sig_wordset* ws) { return ws ? W(ws)->max_len : -1; }
int64_t sig_wordset_n_user(const sig_wordset* ws) { return ws ? (int64_t)W(ws)->user_index.size() : -1; }
const int32_t* sig_wordset_parent(const sig_wordset* ws) { return ws ? W(ws)->parent.data() : nullptr; }
const int32_t* sig_wordset_letter(const sig_wordset* ws) { return ws ? W(ws)->letter.data() : nullptr; }
const int32_t* sig_wordset_level_start(const sig_wordset* ws) { return ws ? W(ws)->level_start.data() : nullptr; }
const int64_t* sig_wordset_user_index(const sig_wordset* ws)
{
    return (ws && !W(ws)->user_index.empty()) ? W(ws)->user_index.data() : nullptr;
}
int sig_wordset_suffix_closed(const sig_wordset* ws) { return ws ? (W(ws)->suffix_closed ? 1 : 0) : -1; }
const int32_t* sig_wordset_tail_table(const sig_wordset* ws, const int32_t** tail_off)
{
    if (!ws || !W(ws)->suffix_closed) return nullptr;
    if (tail_off) *tail_off = W(ws)->tail_off.data();
    return W(ws)->tail_tab.data();
}
int64_t sig_wordset_term_tables(const sig_wordset* ws, const uint32_t** prod_pairs, const uint32_t** adj_pairs,
                                const uint32_t** adj_key, int64_t* n_adj)
{
    if (!ws || !W(ws)->pair_tables) return -1;
    if (prod_pairs) *prod_pairs = W(ws)->prod_pairs.data();
    if (adj_pairs) *adj_pairs = W(ws)->adj_pairs.data();
    if (adj_key) *adj_key = W(ws)->adj_key.data();
    if (n_adj) *n_adj = (int64_t)W(ws)->adj_pairs.size();
    return (int64_t)W(ws)->prod_pairs.size();
}
int64_t sig_wordset_min_fma_per_step(const sig_wordset* ws) { return ws ? W(ws)->min_fma : -1; }

int64_t sig_wordset_kernel_fma_per_step(const sig_wordset* ws, int backward)
{
    if (!ws || !W(ws)->kernels_supported) return -1;
    // reported for the finest variant unless a launch picked another one; forward count of
    // multiply-adds, the backward kernels issue about 3 per leaf pair and 4.5 per inner pair
    const auto& pl = W(ws)->plans[backward ? 1 : 0];
    return pl.empty() ? -1 : pl.front().fma_per_step;
}

int sig_wordset_plan_count(const sig_wordset* ws, int backward)
{
    return ws ? (int)W(ws)->plans[backward ? 1 : 0].size() : -1;
}

int sig_wordset_plan_get(const sig_wordset* ws, int backward, int variant, const int32_t** units, int64_t* n_units,
                         const uint32_t** ops, int64_t* n_ops, const int32_t** slot_word, int64_t* n_slots,
                         int64_t* fma_per_step)
{
    if (!ws) return SIG_EINVAL;
    const auto& pl = W(ws)->plans[backward ? 1 : 0];
    if (variant < 0 || variant >= (int)pl.size()) return SIG_EINVAL;
    const sig::Plan& p = pl[(size_t)variant];
    static_assert(sizeof(sig::UnitDesc) == 4 * sizeof(int32_t), "UnitDesc is four int32");
    if (units) *units = reinterpret_cast<const int32_t*>(p.units.data());
    if (n_units) *n_units = (int64_t)p.units.size();
    if (ops) *ops = p.ops.data();
    if (n_ops) *n_ops = (int64_t)p.ops.size();
    if (slot_word) *slot_word = p.slot_word.data();
    if (n_slots) *n_slots = (int64_t)p.slot_word.size();
    if (fma_per_step) *fma_per_step = p.fma_per_step;
    return SIG_OK;
}

int sig_wordset_jit_plan_get(sig_wordset* ws, int backward, int64_t B, const int32_t** units, int64_t* n_units,
                             const uint32_t** ops, int64_t* n_ops, const int32_t** slot_word, int64_t* n_slots,
                             int64_t* fma_per_step)
{
    if (!ws || B < 1) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    if (!w.kernels_supported || w.size() == 0) return SIG_EUNSUPPORTED;
    sig::WordSet::JitEntry* e = jit_entry(w, backward ? 1 : 0, B);
    if (!e) return SIG_ENOMEM;
    const sig::Plan& p = e->plan;
    if (units) *units = reinterpret_cast<const int32_t*>(p.units.data());
    if (n_units) *n_units = (int64_t)p.units.size();
    if (ops) *ops = p.ops.data();
    if (n_ops) *n_ops = (int64_t)p.ops.size();
    if (slot_word) *slot_word = p.slot_word.data();
    if (n_slots) *n_slots = (int64_t)p.slot_word.size();
    if (fma_per_step) *fma_per_step = p.fma_per_step;
    return SIG_OK;
}

int sig_wordset_jit_prepare(sig_wordset* ws, int backward, int64_t B)
{
    if (!ws || B < 1) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    const int dir = backward ? 1 : 0;
    if (!jit_enabled(w)) return SIG_EUNSUPPORTED;
    if (dir == 0 ? use_trunc_forward(w, B) : use_trunc_backward(w, B)) return SIG_EUNSUPPORTED;
    if (use_lanes(w, B, kAnyLength)) {
        lanes_bring_up(w, dir, B, Build::compile_only);
        return ensure_lanes(w, dir, lanes_shape_for(w, dir, B), Build::compile_only) ? SIG_OK : SIG_EJIT;
    }
    return ensure_jit(w, dir, B, Build::compile_only) ? SIG_OK : SIG_EJIT;
}

int sig_wordset_jit_prepare_chunks(sig_wordset* ws, int backward, int64_t B)
{
    if (!ws || B < 1) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    const int dir = backward ? 1 : 0;
    if (!jit_enabled(w)) return SIG_EUNSUPPORTED;
    if (dir == 0 ? use_trunc_forward(w, B) : use_trunc_backward(w, B)) return SIG_EUNSUPPORTED;
    PlainKernels k;
    return !plain_chunks_available(w, B) || plain_kernels(w, dir, B, Build::compile_only, k) ? SIG_OK : SIG_EJIT;
}

size_t sig_wordset_jit_source(sig_wordset* ws, int backward, int64_t B, char* buf, size_t n)
{
    if (!ws || B < 1) return 0;
    const sig::WordSet& w = *W(ws);
    const int dir = backward ? 1 : 0;
    if (!jit_enabled(w)) return 0;
    std::string src;
    if (use_lanes(w, B, kAnyLength)) {
        const sig::LanesShape s = lanes_shape_for(w, dir, B);
        src = sig::lanes_source(w.d, w.depth, s, dir != 0, dir == 1 && lanes_arrays(w, s));
    } else {
        sig::WordSet::JitEntry* e = jit_entry(w, dir, B);
        if (!e) return 0;
        int nw = 0, tile = 0;
        src = jit_source(w, dir, *e, nw, tile);
    }
    if (buf && n > 0) {
        const size_t c = std::min(n - 1, src.size());
        std::memcpy(buf, src.data(), c);
        buf[c] = 0;
    }
    return src.size();
}

size_t sig_wordset_device_bytes(const sig_wordset* ws) { return ws ? W(ws)->image.size() : 0; }

int sig_wordset_upload(sig_wordset* ws, void* dev_buf, size_t dev_bytes, void* stream)
{
    if (!ws || !dev_buf) return SIG_EINVAL;
    if (dev_bytes < ws->image.size()) return SIG_EWORKSPACE;
    if (((uintptr_t)dev_buf & 255) != 0) return SIG_EINVAL;
    hipError_t e = hipMemcpyAsync(dev_buf, ws->image.data(), ws->image.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e);
    ws->dev = dev_buf;
    (void)hipGetDevice(&ws->dev_id);
    return SIG_OK;
}

size_t sig_forward_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    if (!ws || B <= 0 || n_points <= 1) return 0;
    const sig::WordSet& w = *W(ws);
    if (use_trunc_forward(w, B)) {
        const Chunks ch = trunc_chunks(w, 0, B, n_points);
        size_t n = ch.C > 1 ? chunk_array_bytes(w, B, ch.C) : 0;
        if (sig::trunc_low_available(w.d, w.depth)) {
            const Chunks low = low_chunks(w, 0, B, n_points);
            if (low.C > 1) n = std::max(n, chunk_array_bytes(w, B, low.C));
        }
        return n;
    }
    if (!jit_enabled(w)) return 0;
    size_t n = jit_dxt_bytes(w, B, n_points, 0);
    if (use_lanes(w, B, n_points - 1)) {
        const Chunks ch = lanes_chunks(w, 0, B, n_points);
        if (ch.C > 1) n = std::max(n, chunk_array_bytes(w, B, ch.C));
    }
    if (plain_chunks_available(w, B)) {
        const Chunks ch = plain_chunks(w, 0, B, n_points);
        if (ch.C > 1) n = std::max(n, plain_forward_bytes(w, B, ch));
    } else if (w.kind != 0) {
        // sets closed under suffixes: time chunks as in the checkpointed calls, the chunk signatures in the workspace
        n = std::max(n, words_forward_bytes(w, B, n_points, checkpoint_chunks(w, B, n_points)));
    }
    return n;
}

static size_t gdx_bytes_of(const sig::WordSet& w, int64_t B, int64_t n_points)
{
    return ((size_t)B * (size_t)(n_points - 1) * (size_t)w.d * sizeof(float) + 255) & ~(size_t)255;
}

// chunk signatures, products from both sides [B][C] and boundary adjoints [B][C - 1], rows of words shorter than the depth
static size_t low_backward_arrays(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return ch.C > 1 ? 3 * lanes_low_bytes(w, B, ch.C) + lanes_low_bytes(w, B, ch.C - 1) : 0;
}
// What the checkpointed backward call of those shapes takes from its workspace over the kept chunks, beside the gradient of the
// increments: boundary adjoints [B][C - 1]; beyond two chunks these and the products from both sides [B][C] are rows of words
// shorter than the depth
static size_t low_kept_arrays(const sig::WordSet& w, int64_t B, const Chunks& ch)
{
    return ch.C == 2 ? chunk_array_bytes(w, B, 1) : lanes_low_bytes(w, B, ch.C - 1) + 2 * lanes_low_bytes(w, B, ch.C);
}
// ... and the chunks that it takes in their place, for all the forward pass they need again, where they fill the SIMDs so much
// better than the ones that are kept (ch).  C = 1: none.  d = 8, 1 to 38 paths of 130 to 900 segments, kept -> taken 57 -> 40 to 236 ->
// 209 us; d = 16, 55 -> 39 to 301 -> 273 us.  There the model promises too much where the taken chunks put a second wavefront on a
// SIMD that the kept ones don't (12 paths x 150 59 -> 67 us; 8 x 500, at 0.79 of the modelled time, 87 -> 81) and where the kept ones
// put a third (60 x 900 371 -> 390; 38 x 260 131 -> 114), so its line lies lower.
static Chunks low_instead_of_kept(const sig::WordSet& w, int64_t B, int64_t n_points, const Chunks& ch)
{
    const int64_t L = n_points - 1;
    if (w.opt.ckpt_chunks != 0) return Chunks{1, L};
    const Chunks own = low_chunks(w, 1, B, n_points);
    const int64_t waves = sig::trunc_waves_per_row(w.d, w.depth, 1) * B, kept = waves * ch.C;
    const double line = w.d != 16 || waves * own.C <= 1024 ? 0.93 : (kept <= 1024 ? 0.85 : (kept > 2048 ? 0.90 : 0.93));
    if (own.C < 2 || low_time(w, 1, false, B, L, own.C) >= line * low_time(w, 1, true, B, L, ch.C)) return Chunks{1, L};
    return own;
}
// sig_backward of those shapes over chunks of its own; workspace: gradient of the increments | low_backward_arrays
static hipError_t low_backward(const sig::WordSet& w, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                               int64_t n_points, const Chunks& ch, float* grad_path, void* workspace, hipStream_t st)
{
    const size_t gb = gdx_bytes_of(w, B, n_points), nb = lanes_low_bytes(w, B, ch.C);
    unsigned char* base = (unsigned char*)workspace + gb;
    float* gdx = (float*)workspace;
    float* Sc = (float*)base;
    float* left = (float*)(base + nb);
    float* right = (float*)(base + 2 * nb);
    float* Abar = (float*)(base + 3 * nb);
    hipError_t e = sig::trunc_forward_low(w.d, w.depth, path, B, n_points, ch.C, ch.Lc, Sc, st);
    if (e == hipSuccess) e = sig::chunk_slices_both(w.d, w.depth, Sc, w.level_start[(size_t)w.depth], left, right, B, (int)ch.C, st);
    if (e == hipSuccess)
        e = sig::chunk_adjoint(w.d, w.depth, grad_coeffs, right, w.level_start[(size_t)w.depth], Abar, B, (int)ch.C, gdx,
                               B * (n_points - 1) * w.d, st);
    if (e != hipSuccess) return e;
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = sig::trunc_backward(w.d, w.depth, path, left, Abar, coeffs, grad_coeffs, B, n_points, ch.C, ch.Lc, gdx, nullptr, w.opt.bwd_tile, st,
                            true);
    if (pe) (void)hipEventRecord(pe[1], st);
    return e == hipSuccess ? sig::grad_points(gdx, B, n_points, w.d, grad_path, st) : e;
}

// what sig_backward needs; own_chunks = false: when it takes no time chunks of its own (sig_backward_static)
static size_t backward_workspace(const sig_wordset* ws, int64_t B, int64_t n_points, bool own_chunks)
{
    if (!ws || B <= 0 || n_points <= 1) return 0;
    const sig::WordSet& w = *W(ws);
    size_t n = (size_t)B * (size_t)(n_points - 1) * (size_t)w.d * sizeof(float);
    n = (n + 255) & ~(size_t)255;                                   // gradient with respect to the increments
    if (use_trunc_backward(w, B)) {
        const BwdShape ch = trunc_backward_shape(w, B, n_points, own_chunks);
        size_t arrays = ch.C > 1 && !ch.fused ? 4 * chunk_array_bytes(w, B, ch.C) : 0;   // chunk signatures, prefixes, suffixes, adjoints
        if (own_chunks && sig::trunc_low_available(w.d, w.depth)) arrays = std::max(arrays, low_backward_arrays(w, B, low_chunks(w, 1, B, n_points)));
        n += arrays;
    } else if (jit_enabled(w)) {
        // the specialised kernels keep the increment gradients in the (padded) layout of their transposed increments
        const size_t t = jit_dxt_bytes(w, B, n_points, 1);
        n = std::max(n, t) + t;
    }
    return n;
}

// what sig_backward asks for where a suffix-closed set takes the chunks of the checkpointed calls (at least what whole paths need)
static size_t words_backward_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    const Chunks ch = checkpoint_chunks(*W(ws), B, n_points);
    const size_t whole = backward_workspace(ws, B, n_points, false);
    return words_backward_recomputes(*W(ws), ch) ? std::max(whole, words_backward_recompute_workspace(*W(ws), B, ch)) : whole;
}
// ... and on a small launch, whose own chunks take plain_bytes (0: none): those are taken where the workspace holds them; a
// suffix-closed set is refused below what it asks for without them
static size_t small_backward_need(const sig_wordset* ws, int64_t B, int64_t n_points, size_t plain_bytes)
{
    return std::min(words_backward_bytes(ws, B, n_points), std::max(backward_workspace(ws, B, n_points, false), plain_bytes));
}

size_t sig_backward_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    size_t n = backward_workspace(ws, B, n_points, true);
    if (n == 0) return 0;
    const sig::WordSet& w = *W(ws);
    if (!use_trunc_backward(w, B) && use_lanes(w, B, n_points - 1)) {
        const Chunks ch = lanes_chunks(w, 1, B, n_points);
        if (ch.C > 1) n = std::max(n, lanes_backward_chunked_bytes(w, B, ch, lanes_backward_arrays(w, B, ch)));
    }
    if (plain_chunks_available(w, B)) {
        const Chunks ch = plain_chunks(w, 1, B, n_points);
        if (ch.C > 1) n = std::max(n, plain_backward_bytes(w, B, ch));
    } else if (w.kind != 0 && jit_enabled(w)) {
        n = std::max(n, words_backward_bytes(ws, B, n_points));
    }
    return n;
}

static int check_common(const sig_wordset* ws, const void* path, int64_t B, int64_t n_points)
{
    if (!ws) return SIG_EINVAL;
    if (B < 0 || n_points < 1) return SIG_EINVAL;
    if (B > 0 && !path) return SIG_EINVAL;
    if (!W(ws)->kernels_supported) return SIG_EUNSUPPORTED;
    if (!W(ws)->dev) return SIG_ENOTUPLOADED;
    if (B > (int64_t)65535 * 64) return SIG_ETOOLARGE;
    return SIG_OK;
}

// sig_forward; word_chunks = false keeps a suffix-closed set from taking time chunks of its own (the checkpointed call
// that falls back to this one has sized its workspace for whole paths)
static int forward_impl(const sig_wordset* ws, const float* path, int64_t B, int64_t n_points, float* coeffs, void* workspace,
                        size_t workspace_bytes, void* stream, bool word_chunks)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    if (B == 0) return SIG_OK;
    if (!coeffs) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    hipStream_t st = (hipStream_t)stream;
    if (n_points == 1) {
        hipError_t e = sig::fill_zero(coeffs, B * w.size(), st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    CallTimer whole(0, st);
    if (use_trunc_forward(w, B)) {
        if (const int64_t C = trunc_forward_fused_chunks(w, B, n_points, coeffs)) {
            const int64_t Lc = (n_points - 1 + C - 1) / C;
            hipEvent_t* pe = g_prof.next(0);
            if (pe) (void)hipEventRecord(pe[0], st);
            hipError_t e = sig::trunc_forward_tails_fused(w.d, w.depth, path, B, n_points, C, Lc, coeffs, st);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
        Chunks ch = trunc_chunks(w, 0, B, n_points);
        if (sig::trunc_low_available(w.d, w.depth)) {
            // (a smaller workspace, rows that are not aligned, and calls for which the model sees no gain in more chunks - 128 paths of
            // 1,024 segments, d = 8 - go on with the count above: whole paths, or the chunks that the call has to bring a workspace for)
            const Chunks low = low_chunks(w, 0, B, n_points);
            const size_t nb = chunk_array_bytes(w, B, low.C);
            if (low.C > 1 && workspace && workspace_bytes >= nb && (((uintptr_t)workspace & 255) | ((uintptr_t)coeffs & 15)) == 0) {
                hipEvent_t* pe = g_prof.next(0);
                if (pe) (void)hipEventRecord(pe[0], st);
                hipError_t e = sig::trunc_forward(w.d, w.depth, path, B, n_points, low.C, low.Lc, (float*)workspace, st);
                if (pe) (void)hipEventRecord(pe[1], st);
                if (e == hipSuccess) e = chunk_product_of(w, (const float*)workspace, coeffs, B, low.C, st);
                return e == hipSuccess ? SIG_OK : hip_fail(e);
            }
        }
        float* Sc = coeffs;
        if (ch.C > 1) {
            const size_t nb = chunk_array_bytes(w, B, ch.C);
            if (!workspace || workspace_bytes < nb) return SIG_EWORKSPACE;
            if (((uintptr_t)workspace & 255) != 0 || ((uintptr_t)coeffs & 15) != 0) return SIG_EINVAL;
            Sc = (float*)workspace;
        }
        hipEvent_t* pe = g_prof.next(0);
        if (pe) (void)hipEventRecord(pe[0], st);
        hipError_t e = sig::trunc_forward(w.d, w.depth, path, B, n_points, ch.C, ch.Lc, Sc, st);
        if (pe) (void)hipEventRecord(pe[1], st);
        if (e == hipSuccess && ch.C > 1) e = chunk_product_of(w, Sc, coeffs, B, ch.C, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    bool small_set = false;
    if (use_lanes(w, B, kAnyLength)) lanes_bring_up(w, 0, B, Build::compile_and_load);
    if (use_lanes(w, B, n_points - 1, true, &small_set)) {
        if (small_set) {                 // as lanes = paths asks for it
            if (!workspace || workspace_bytes < jit_dxt_bytes(w, B, n_points, 0)) return SIG_EWORKSPACE;
            if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
        }
        // (a caller without a workspace for the chunk signatures gets the walk over whole paths)
        const Chunks ch = lanes_chunks(w, 0, B, n_points);
        LanesChunked lc;
        if (ch.C > 1 && workspace && workspace_bytes >= chunk_array_bytes(w, B, ch.C) && ((uintptr_t)workspace & 255) == 0 &&
            lanes_chunk_kernels(w, 0, B * ch.C, Build::compile_and_load, lc)) {
            hipError_t e = lanes_forward_chunked(w, lc, path, B, n_points, ch, coeffs, (float*)workspace, st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
        const sig::LanesShape ls = lanes_shape_for(w, 0, B);
        if (sig::JitKernel* lk = ensure_lanes(w, 0, ls, Build::compile_and_load)) {
            hipEvent_t* pe = g_prof.next(0);
            if (pe) (void)hipEventRecord(pe[0], st);
            hipError_t e = launch_lanes(lk->fn, ls, path, nullptr, nullptr, B, n_points, coeffs, st);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    bool set_chunks = w.kind != 0 && word_chunks;        // sets closed under suffixes: the time chunks of the checkpointed calls
    if (word_chunks && plain_chunks_available(w, B)) {
        // (a smaller workspace gets those chunks where it holds them, and must for such a set; others then walk whole paths)
        const Chunks ch = plain_chunks(w, 0, B, n_points);
        const bool fits = ch.C > 1 && workspace && workspace_bytes >= std::max(jit_dxt_bytes(w, B, n_points, 0), plain_forward_bytes(w, B, ch));
        set_chunks = ch.C > 1 && !fits;
        PlainKernels k;
        if (fits && plain_kernels_for(w, 0, B, Build::compile_and_load, st, k)) {
            if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
            hipError_t e = plain_forward_chunked(w, k, path, B, n_points, ch, coeffs, workspace, st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    if (set_chunks) {
        const Chunks ch = checkpoint_chunks(w, B, n_points);
        const sig::Plan* cp = nullptr;
        sig::JitKernel* ck = ch.C >= 2 ? ensure_jit(w, 0, B * ch.C, Build::compile_and_load, &cp) : nullptr;
        if (ck) {
            if (!workspace || workspace_bytes < words_forward_bytes(w, B, n_points, ch)) return SIG_EWORKSPACE;
            if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
            float* dxT = (float*)workspace;
            float* Sc = (float*)((unsigned char*)workspace + words_forward_ckpt_workspace(w, B, ch));
            hipError_t e = words_forward_chunked(w, path, B, n_points, ch, *ck, *cp, dxT, Sc, coeffs, st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    const sig::Plan* jp = nullptr;
    if (sig::JitKernel* jk = ensure_jit(w, 0, B, Build::compile_and_load, &jp)) {
        if (!workspace || workspace_bytes < jit_dxt_bytes(w, B, n_points, 0)) return SIG_EWORKSPACE;
        if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
        float* dxT = (float*)workspace;
        const int64_t Lpad = jit_lpad(w, n_points, 0);
        hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, nullptr, st);
        if (e != hipSuccess) return hip_fail(e);
        hipEvent_t* pe = g_prof.next(0);
        if (pe) (void)hipEventRecord(pe[0], st);
        e = launch_jit_forward(*jk, *jp, dxT, B, n_points - 1, Lpad, coeffs, w.size(), st);
        if (pe) (void)hipEventRecord(pe[1], st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    const int v = pick_variant(w, 0, B);
    const sig::Plan& p = w.plans[0][(size_t)v];
    const auto& po = w.offsets[0][(size_t)v];
    const unsigned char* base = (const unsigned char*)w.dev;
    sig::GenericArgs a;
    a.units = (const sig::UnitDesc*)(base + po.units);
    a.ops = (const uint32_t*)(base + po.ops);
    a.slot_word = (const int32_t*)(base + po.slots);
    a.n_units = (int64_t)p.units.size();
    a.max_slots = p.max_slots;
    a.path = path; a.B = B; a.P = n_points; a.d = w.d; a.nW = w.size();
    a.coeffs = coeffs;
    hipEvent_t* pe = g_prof.next(0);
    if (pe) (void)hipEventRecord(pe[0], st);
    hipError_t e = sig::generic_forward(a, w.max_len, st);
    if (pe) (void)hipEventRecord(pe[1], st);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_forward(const sig_wordset* ws, const float* path, int64_t B, int64_t n_points, float* coeffs, void* workspace,
                size_t workspace_bytes, void* stream)
{
    return forward_impl(ws, path, B, n_points, coeffs, workspace, workspace_bytes, stream, true);
}

// sig_backward and sig_backward_static: the same kernels on the caller's workspace or on the static scratch array;
// `how` says whether a run-time specialised kernel may be compiled and loaded by this call.
// Backward over the C time chunks whose signatures the forward pass left in ckpt [B][C][|W|]: signature and adjoint at
// the end of every chunk from products of the chunk signatures, then all (path, chunk) rows in one launch.
static int backward_checkpointed(const sig::WordSet& w, const float* path, const float* coeffs, const float* grad_coeffs,
                                 const float* ckpt, const Chunks& ch, int64_t B, int64_t n_points, float* grad_path,
                                 void* workspace, hipStream_t st)
{
    if ((((uintptr_t)coeffs | (uintptr_t)grad_coeffs | (uintptr_t)ckpt) & 15) != 0) return SIG_EINVAL;
    const int64_t nW = w.size(), nL = w.level_start[(size_t)w.depth];   // all words, those shorter than the depth
    // workspace: increment gradients | boundary adjoints | for more than two chunks: products from the left and from the right
    float* gdx = (float*)workspace;
    float* Abar = (float*)((unsigned char*)workspace + gdx_bytes_of(w, B, n_points));
    CallTimer whole(1, st);
    const int64_t n_gdx = B * (n_points - 1) * w.d;                 // cleared by the launch of the adjoints
    hipError_t e = hipSuccess;
    const float* row_coeffs = ckpt;
    const bool low = ch.C > 2;
    if (low) {
        float* left = (float*)((unsigned char*)Abar + lanes_low_bytes(w, B, ch.C - 1));
        float* right = (float*)((unsigned char*)left + lanes_low_bytes(w, B, ch.C));
        e = sig::chunk_slices_both(w.d, w.depth, ckpt, nW, left, right, B, (int)ch.C, st);
        if (e == hipSuccess) e = sig::chunk_adjoint(w.d, w.depth, grad_coeffs, right, nL, Abar, B, (int)ch.C, gdx, n_gdx, st);
        row_coeffs = left;
    } else {
        // two chunks: the signature at the end of the first is the first chunk's own, what follows it the second's
        e = sig::chunk_adjoint(w.d, w.depth, grad_coeffs, ckpt + nW, nW, Abar, B, 2, gdx, n_gdx, st);
    }
    if (e != hipSuccess) return hip_fail(e);
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    // the rows of the last chunk are the caller's terminal signature and gradient themselves
    e = sig::trunc_backward(w.d, w.depth, path, row_coeffs, Abar, coeffs, grad_coeffs, B, n_points, ch.C, ch.Lc, gdx, nullptr,
                            w.opt.bwd_tile, st, low);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return hip_fail(e);
    e = sig::grad_points(gdx, B, n_points, w.d, grad_path, st);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

static int backward_impl(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                         int64_t n_points, float* grad_path, void* workspace, size_t workspace_bytes, void* stream, Build how,
                         float* residual = nullptr, bool word_chunks = true /* false: no time chunks of its own */)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    if (B == 0) return SIG_OK;
    if (!coeffs || !grad_coeffs || !grad_path) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    hipStream_t st = (hipStream_t)stream;
    if (n_points == 1) {
        hipError_t e = sig::fill_zero(grad_path, B * w.d, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    // the chunks of the word-per-lane kernels are taken where the workspace holds them, not asked for
    // (sig_backward_static takes no chunks: small sets beyond depth 2 then run with lanes = paths, those of depth 2 walk whole
    // paths as fast or faster a word per lane, 12 letters, 512 paths x 160 segments 71 -> 27 us, 2 letters, 64 x 900 125 -> 117)
    bool small_set = false;
    const bool lanes_path = !use_trunc_backward(w, B) && use_lanes(w, B, n_points - 1, true, &small_set) &&
                            !(small_set && w.depth > 2 && how == Build::loaded_only);
    // the same holds for the chunks of small launches, except where a suffix-closed set has always asked for its chunks
    const bool small_launch = plain_chunks_available(w, B);
    const bool low = use_trunc_backward(w, B) && sig::trunc_low_available(w.d, w.depth) && word_chunks && !residual;
    const Chunks pc = small_launch && word_chunks && !residual ? plain_chunks(w, 1, B, n_points) : Chunks{1, n_points - 1};
    const bool optional = lanes_path || (low && trunc_chunks(w, 1, B, n_points).C == 1);
    // (with the residual whole paths are walked: no chunks to hold; d = 8 and d = 16 need no more than low_backward takes, which
    // is less than the size for whole arrays that a caller is told)
    const Chunks lch = low ? low_chunks(w, 1, B, n_points) : Chunks{1, n_points - 1};
    const size_t low_need = low ? gdx_bytes_of(w, B, n_points) + low_backward_arrays(w, B, lch) : 0;
    const size_t plain_bytes = pc.C > 1 ? plain_backward_bytes(w, B, pc) : 0;
    const size_t need = !word_chunks || optional || residual ? backward_workspace(ws, B, n_points, false)
                        : low                                ? low_need
                        : small_launch                       ? small_backward_need(ws, B, n_points, plain_bytes)
                                                             : sig_backward_workspace_bytes(ws, B, n_points);
    if (!workspace || workspace_bytes < need) return SIG_EWORKSPACE;
    if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
    float* gdx = (float*)workspace;
    CallTimer whole(1, st);
    if (low) {
        if (lch.C > 1 && workspace_bytes >= low_need && (((uintptr_t)coeffs | (uintptr_t)grad_coeffs) & 15) == 0) {
            hipError_t le = low_backward(w, path, coeffs, grad_coeffs, B, n_points, lch, grad_path, workspace, st);
            return le == hipSuccess ? SIG_OK : hip_fail(le);
        }
    }
    if (word_chunks && !residual && !use_trunc_backward(w, B) && use_lanes(w, B, kAnyLength)) lanes_bring_up(w, 1, B, how);
    if (lanes_path && word_chunks && !residual) {
        const Chunks lch = lanes_chunks(w, 1, B, n_points);
        LanesChunked lc;
        const bool arrays = lch.C > 1 && lanes_backward_arrays(w, B, lch) &&
                            workspace_bytes >= lanes_backward_chunked_bytes(w, B, lch, true);
        const bool shares = lch.C > 1 && lanes_shape_for(w, 1, B * lch.C).shares &&
                            workspace_bytes >= lanes_backward_chunked_bytes(w, B, lch, false);
        if ((arrays || shares) && lanes_chunk_kernels(w, 1, B * lch.C, how, lc)) {
            hipError_t le = lanes_backward_chunked(w, lc, path, coeffs, grad_coeffs, B, n_points, lch, arrays, grad_path, workspace, st);
            return le == hipSuccess ? SIG_OK : hip_fail(le);
        }
    }
    const bool plain_fits = pc.C > 1 && workspace_bytes >= plain_bytes;
    if (plain_fits) {
        PlainKernels k;
        if (plain_kernels_for(w, 1, B, how, st, k)) {
            hipError_t ce = plain_backward_chunked(w, k, path, coeffs, grad_coeffs, B, n_points, pc, grad_path, workspace, st);
            return ce == hipSuccess ? SIG_OK : hip_fail(ce);
        }
    }
    if (word_chunks && w.kind != 0 && jit_enabled(w) && !residual && (!small_launch || (pc.C > 1 && !plain_fits))) {
        // suffix-closed set, few long paths: chunk signatures recomputed, then the route of the checkpointed call
        const Chunks wc = checkpoint_chunks(w, B, n_points);
        sig::JitKernel *fk, *bk;
        const sig::Plan *fp = nullptr, *bp = nullptr;
        if (words_backward_recomputes(w, wc) && words_kernels(w, B * wc.C, &fk, &fp, &bk, &bp)) {
            float* Sc = (float*)((unsigned char*)workspace + words_backward_recompute_first(w, B, wc));
            hipError_t ce = words_forward_chunked(w, path, B, n_points, wc, *fk, *fp, (float*)workspace, Sc, nullptr, st);
            if (ce == hipSuccess)
                ce = words_backward_chunked(w, path, coeffs, grad_coeffs, Sc, wc, B, n_points, grad_path, workspace, *bk, *bp, st);
            return ce == hipSuccess ? SIG_OK : hip_fail(ce);
        }
    }
    hipError_t e = hipSuccess;
    const bool trunc = use_trunc_backward(w, B);
    BwdShape ch = trunc ? trunc_backward_shape(w, B, n_points, word_chunks) : BwdShape{false, false, 1, n_points - 1};
    if (residual) {                      // reported by the kernels that walk whole paths with several wavefronts per row
        if (!trunc) return SIG_EUNSUPPORTED;
        ch = BwdShape{false, false, 1, n_points - 1};
        e = sig::fill_zero(residual, B, st);
        if (e != hipSuccess) return hip_fail(e);
    }
    // the fused form reads the leaves of the gradient with 16-byte loads; rows that are not aligned so take the kernel with
    // four wavefronts per path, which reads word by word
    if (ch.fused && (((uintptr_t)coeffs | (uintptr_t)grad_coeffs) & 15) != 0) ch = BwdShape{false, false, 1, n_points - 1};
    // word sets that may run through the straight-line specialised kernels clear their (larger) array further down
    const bool maybe_jit = !trunc && !lanes_path && jit_enabled(w);
    if (!ch.tails && !maybe_jit && !lanes_path) {       // the one-wavefront-per-row kernel stores every entry itself
        e = sig::fill_zero(gdx, B * (n_points - 1) * w.d, st);
        if (e != hipSuccess) return hip_fail(e);
    }
    if (trunc) {
        const float* row_coeffs = coeffs;
        const float* row_grad = grad_coeffs;
        if (ch.C > 1 && !ch.fused && (((uintptr_t)coeffs | (uintptr_t)grad_coeffs) & 15) != 0) return SIG_EINVAL;
        // (shapes whose chunks low_backward takes: a call without its workspace walks whole paths)
        if (ch.C > 1 && sig::trunc_low_available(w.d, w.depth)) ch = BwdShape{false, false, 1, n_points - 1};
        if (ch.C > 1 && !ch.fused) {
            // chunk signatures (recomputed: only the terminal signature was kept), then the signature and the
            // adjoint at the end of every chunk
            const size_t nb = chunk_array_bytes(w, B, ch.C);
            unsigned char* base = (unsigned char*)workspace + gdx_bytes_of(w, B, n_points);
            float* Sc = (float*)base;
            float* Pfx = (float*)(base + nb);
            float* Abar = (float*)(base + 2 * nb);
            e = sig::trunc_forward(w.d, w.depth, path, B, n_points, ch.C, ch.Lc, Sc, st);
            if (e == hipSuccess) e = sig::chunk_scan(w.d, w.depth, Sc, Pfx, coeffs, nullptr, grad_coeffs, Abar, B, (int)ch.C, st);
            if (e != hipSuccess) return hip_fail(e);
            row_coeffs = Pfx;
            row_grad = Abar;
        }
        hipEvent_t* pe = g_prof.next(1);
        if (pe) (void)hipEventRecord(pe[0], st);
        // the one-wavefront-per-row kernel applies the chain rule itself when its rows are whole paths or all
        // chunks of a path share a workgroup
        const bool points = ch.fused || (ch.tails && ch.C == 1);
        if (ch.fused) e = sig::trunc_backward_tails_fused(w.d, w.depth, path, coeffs, grad_coeffs, B, n_points, ch.C, ch.Lc, grad_path, st);
        else if (ch.tails)
            e = sig::trunc_backward_tails(w.d, w.depth, path, row_coeffs, row_grad, B, n_points, ch.C, ch.Lc, gdx,
                                          points ? grad_path : nullptr, st);
        else e = sig::trunc_backward(w.d, w.depth, path, row_coeffs, row_grad, nullptr, nullptr, B, n_points, ch.C, ch.Lc, gdx, residual,
                                     w.opt.bwd_tile, st);
        if (pe) (void)hipEventRecord(pe[1], st);
        if (e != hipSuccess) return hip_fail(e);
        if (!points) e = sig::grad_points(gdx, B, n_points, w.d, grad_path, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    if (lanes_path) {
        const sig::LanesShape ls = lanes_shape_for(w, 1, B);
        g_not_ready = false;
        sig::JitKernel* lk = ensure_lanes(w, 1, ls, how);
        if (!lk && g_not_ready) return SIG_ENOTREADY;
        if (lk) {
            e = sig::fill_zero(grad_path, B * n_points * w.d, st);      // the kernel adds into it
            if (e != hipSuccess) return hip_fail(e);
            hipEvent_t* pe = g_prof.next(1);
            if (pe) (void)hipEventRecord(pe[0], st);
            e = launch_lanes(lk->fn, ls, path, coeffs, grad_coeffs, B, n_points, grad_path, st);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    const sig::Plan* jp = nullptr;
    g_not_ready = false;
    sig::JitKernel* jk = ensure_jit(w, 1, B, how, &jp);
    if (!jk && g_not_ready) return SIG_ENOTREADY;
    if (jk) {
        // increment gradients and increments in the same layout [group][padded segment][letter][lane], one after the other
        const size_t t_bytes = jit_dxt_bytes(w, B, n_points, 1);
        const size_t gdx_bytes = std::max(gdx_bytes_of(w, B, n_points), t_bytes);
        float* dxT = (float*)((unsigned char*)workspace + gdx_bytes);
        const int64_t Lpad = jit_lpad(w, n_points, 1);
        e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, gdx, st);   // clears the gradients as well
        if (e != hipSuccess) return hip_fail(e);
        hipEvent_t* pe = g_prof.next(1);
        if (pe) (void)hipEventRecord(pe[0], st);
        e = launch_jit_backward(*jk, *jp, dxT, coeffs, grad_coeffs, B, n_points - 1, Lpad, w.size(), gdx, st);
        if (pe) (void)hipEventRecord(pe[1], st);
        if (e != hipSuccess) return hip_fail(e);
        e = sig::grad_points_transposed(gdx, B, n_points, w.d, Lpad, grad_path, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    if (maybe_jit || lanes_path) {       // no specialised kernel after all: the table-driven one takes gdx [B][L][d]
        e = sig::fill_zero(gdx, B * (n_points - 1) * w.d, st);
        if (e != hipSuccess) return hip_fail(e);
    }
    const int v = pick_variant(w, 1, B);
    const sig::Plan& p = w.plans[1][(size_t)v];
    const auto& po = w.offsets[1][(size_t)v];
    const unsigned char* base = (const unsigned char*)w.dev;
    sig::GenericArgs a;
    a.units = (const sig::UnitDesc*)(base + po.units);
    a.ops = (const uint32_t*)(base + po.ops);
    a.slot_word = (const int32_t*)(base + po.slots);
    a.n_units = (int64_t)p.units.size();
    a.max_slots = p.max_slots;
    a.path = path; a.B = B; a.P = n_points; a.d = w.d; a.nW = w.size();
    a.coeffs_in = coeffs; a.grad_coeffs = grad_coeffs; a.gdx = gdx;
    a.tile_steps = bwd_tile_steps(w.d);
    hipEvent_t* pe = g_prof.next(1);
    if (pe) (void)hipEventRecord(pe[0], st);
    e = sig::generic_backward(a, w.max_len, st);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e != hipSuccess) return hip_fail(e);
    e = sig::grad_points(gdx, B, n_points, w.d, grad_path, st);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_backward(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                 int64_t n_points, float* grad_path, void* workspace, size_t workspace_bytes, void* stream)
{
    return backward_impl(ws, path, coeffs, grad_coeffs, B, n_points, grad_path, workspace, workspace_bytes, stream,
                         Build::compile_and_load);
}

size_t sig_checkpoint_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    if (!ws || B <= 0 || n_points <= 1) return 0;
    const Chunks ch = checkpoint_chunks(*W(ws), B, n_points);
    return ch.C >= 2 ? chunk_array_bytes(*W(ws), B, ch.C) : 0;
}

int64_t sig_checkpoint_chunks(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    if (!ws || B <= 0 || n_points <= 1) return 1;
    const Chunks ch = checkpoint_chunks(*W(ws), B, n_points);
    return ch.C >= 2 ? ch.C : 1;
}

size_t sig_forward_checkpointed_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    if (!ws || B <= 0 || n_points <= 1) return 0;
    const Chunks ch = checkpoint_chunks(*W(ws), B, n_points);
    if (ch.C < 2) return sig_forward_workspace_bytes(ws, B, n_points);
    if (W(ws)->kind != 0)                                // (the call needs less)
        return std::max(words_forward_ckpt_workspace(*W(ws), B, ch), sig_forward_workspace_bytes(ws, B, n_points));
    return 0;                                            // full truncations: the chunk signatures are the checkpoint
}

size_t sig_backward_checkpointed_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points)
{
    if (!ws || B <= 0 || n_points <= 1) return 0;
    const sig::WordSet& w = *W(ws);
    const Chunks ch = checkpoint_chunks(w, B, n_points);
    if (ch.C < 2) return sig_backward_workspace_bytes(ws, B, n_points);
    if (w.kind != 0) return std::max(words_backward_ckpt_workspace(w, B, ch), sig_backward_workspace_bytes(ws, B, n_points));
    // full truncations (the kept chunks, or those that the call takes in their place)
    const size_t arrays = std::max(low_kept_arrays(w, B, ch), low_backward_arrays(w, B, low_instead_of_kept(w, B, n_points, ch)));
    return gdx_bytes_of(w, B, n_points) + arrays;
}

int sig_forward_checkpointed(const sig_wordset* ws, const float* path, int64_t B, int64_t n_points, float* coeffs,
                             void* checkpoint, size_t checkpoint_bytes, void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    const sig::WordSet& w = *W(ws);
    const Chunks ch = (B > 0 && n_points > 1) ? checkpoint_chunks(w, B, n_points) : Chunks{1, 0};
    if (ch.C < 2) return sig_forward(ws, path, B, n_points, coeffs, workspace, workspace_bytes, stream);
    if (!coeffs) return SIG_EINVAL;
    const size_t nb = chunk_array_bytes(w, B, ch.C);
    if (!checkpoint || checkpoint_bytes < nb) return SIG_EWORKSPACE;
    if (w.kind != 0) {
        if (((uintptr_t)checkpoint & 255) != 0) return SIG_EINVAL;
        sig::JitKernel *fk, *bk;
        const sig::Plan *fp = nullptr, *bp = nullptr;
        if (!words_kernels(w, B * ch.C, &fk, &fp, &bk, &bp))
            return forward_impl(ws, path, B, n_points, coeffs, workspace, workspace_bytes, stream, false);
        const size_t need = std::max(words_forward_ckpt_workspace(w, B, ch), jit_dxt_bytes(w, B, n_points, 0));
        if (!workspace || workspace_bytes < need) return SIG_EWORKSPACE;
        if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
        hipStream_t st = (hipStream_t)stream;
        // the backward call of the pair finds its kernels loaded, also where it takes other chunks than are kept
        PlainKernels k;
        if (plain_instead_of_kept(w, B, n_points, ch).C > 1) (void)plain_kernels(w, 1, B, unless_captured(Build::compile_and_load, st), k);
        CallTimer whole(0, st);
        hipError_t e = words_forward_chunked(w, path, B, n_points, ch, *fk, *fp, (float*)workspace, (float*)checkpoint, coeffs, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    if (((uintptr_t)checkpoint & 255) != 0 || ((uintptr_t)coeffs & 15) != 0) return SIG_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    CallTimer whole(0, st);
    float* Sc = (float*)checkpoint;
    hipEvent_t* pe = g_prof.next(0);
    if (pe) (void)hipEventRecord(pe[0], st);
    hipError_t e = sig::trunc_forward(w.d, w.depth, path, B, n_points, ch.C, ch.Lc, Sc, st);
    if (pe) (void)hipEventRecord(pe[1], st);
    if (e == hipSuccess) e = chunk_product_of(w, Sc, coeffs, B, ch.C, st);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_backward_checkpointed(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs,
                              const void* checkpoint, size_t checkpoint_bytes, int64_t B, int64_t n_points, float* grad_path,
                              void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    const sig::WordSet& w = *W(ws);
    const Chunks ch = (B > 0 && n_points > 1) ? checkpoint_chunks(w, B, n_points) : Chunks{1, 0};
    if (ch.C < 2) return sig_backward(ws, path, coeffs, grad_coeffs, B, n_points, grad_path, workspace, workspace_bytes, stream);
    if (!coeffs || !grad_coeffs || !grad_path) return SIG_EINVAL;
    if (!checkpoint || checkpoint_bytes < chunk_array_bytes(w, B, ch.C)) return SIG_EWORKSPACE;
    if (w.kind != 0) {
        // (a smaller workspace, and kernels that failed to compile or cannot be loaded now, mean the chunks that are kept)
        const Chunks own = plain_instead_of_kept(w, B, n_points, ch);
        PlainKernels k;
        if (own.C > 1 && workspace && workspace_bytes >= plain_backward_bytes(w, B, own) &&
            (((uintptr_t)workspace | (uintptr_t)checkpoint) & 255) == 0 &&
            plain_kernels(w, 1, B, unless_captured(Build::compile_and_load, (hipStream_t)stream), k)) {
            CallTimer whole(1, (hipStream_t)stream);
            hipError_t e = plain_backward_chunked(w, k, path, coeffs, grad_coeffs, B, n_points, own, grad_path, workspace, (hipStream_t)stream);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
        sig::JitKernel *fk, *bk;
        const sig::Plan *fp = nullptr, *bp = nullptr;
        if (!words_kernels(w, B * ch.C, &fk, &fp, &bk, &bp))
            return sig_backward(ws, path, coeffs, grad_coeffs, B, n_points, grad_path, workspace, workspace_bytes, stream);
        const size_t need = std::max(words_backward_ckpt_workspace(w, B, ch), words_backward_bytes(ws, B, n_points));
        if (!workspace || workspace_bytes < need) return SIG_EWORKSPACE;
        if (((uintptr_t)workspace & 255) != 0 || ((uintptr_t)checkpoint & 255) != 0) return SIG_EINVAL;
        hipStream_t st = (hipStream_t)stream;
        CallTimer whole(1, st);
        hipError_t e = words_backward_chunked(w, path, coeffs, grad_coeffs, (const float*)checkpoint, ch, B, n_points, grad_path,
                                              workspace, *bk, *bp, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    const size_t gb = gdx_bytes_of(w, B, n_points);
    if (!workspace || workspace_bytes < gb + low_kept_arrays(w, B, ch)) return SIG_EWORKSPACE;
    if (((uintptr_t)workspace & 255) != 0 || ((uintptr_t)checkpoint & 255) != 0) return SIG_EINVAL;
    const Chunks own = low_instead_of_kept(w, B, n_points, ch);
    if (own.C > 1 && workspace_bytes >= gb + low_backward_arrays(w, B, own) && (((uintptr_t)coeffs | (uintptr_t)grad_coeffs) & 15) == 0) {
        CallTimer whole(1, (hipStream_t)stream);
        hipError_t e = low_backward(w, path, coeffs, grad_coeffs, B, n_points, own, grad_path, workspace, (hipStream_t)stream);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    return backward_checkpointed(w, path, coeffs, grad_coeffs, (const float*)checkpoint, ch, B, n_points, grad_path, workspace,
                                 (hipStream_t)stream);
}

int sig_backward_residual(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                          int64_t n_points, float* grad_path, float* residual, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    if (!residual) return SIG_EINVAL;
    if (ws && B > 0 && n_points == 1) {
        hipError_t e = sig::fill_zero(residual, B, (hipStream_t)stream);
        if (e != hipSuccess) return hip_fail(e);
    }
    return backward_impl(ws, path, coeffs, grad_coeffs, B, n_points, grad_path, workspace, workspace_bytes, stream,
                         Build::compile_and_load, residual);
}

int sig_backward_static(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                        int64_t n_points, float* grad_path, void* stream)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    if (backward_workspace(ws, B, n_points, false) > (size_t)SIG_STATIC_SCRATCH_BYTES) return SIG_ETOOLARGE;
    void* scratch_ptr = nullptr;                         // this device's copy of the static array
    hipError_t e = sig::static_scratch(&scratch_ptr);
    if (e != hipSuccess) return hip_fail(e);
    return backward_impl(ws, path, coeffs, grad_coeffs, B, n_points, grad_path, scratch_ptr, (size_t)SIG_STATIC_SCRATCH_BYTES, stream,
                         Build::loaded_only, nullptr, false);
}

// ---- windows: every (path, window) pair is gathered into a path of its own (padded with its last point), the
// ordinary forward / backward runs on those B * K paths, and the gradient is scattered back.
static size_t win_sub_bytes(const sig::WordSet& w, int64_t B, int64_t K, int64_t n_sub)
{
    return ((size_t)B * (size_t)K * (size_t)n_sub * (size_t)w.d * sizeof(float) + 255) & ~(size_t)255;
}

// Full truncations with register-resident kernels read every window straight from the path (no copy of the path per
// window, short windows end early); other word sets take the gather into padded sub-paths.
static bool windows_direct(const sig::WordSet& w, int64_t B, int64_t K, int backward)
{
    return B * K <= 65535 && (backward ? use_trunc_backward(w, B * K) : use_trunc_forward(w, B * K));
}
// Word sets that run through the straight-line specialised kernels (lane = row): their rows can be windows as well,
// the increments being transposed straight from the path.  (The workspace the window calls ask for covers both this
// form and the gather into padded sub-paths, which the other kernels and a failed compilation take; both walk whole windows.)
static bool windows_rows_jit(const sig::WordSet& w, int64_t rows)
{
    return !use_trunc_forward(w, rows) && !use_trunc_backward(w, rows) && !use_lanes(w, rows, kAnyLength, false) && jit_enabled(w);
}

size_t sig_forward_windows_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points, int64_t K, int64_t max_window_len)
{
    if (!ws || B <= 0 || K <= 0 || n_points < 1 || max_window_len < 0) return 0;
    if (windows_direct(*W(ws), B, K, 0)) return 0;
    const int64_t n_sub = max_window_len + 1;
    const size_t whole = jit_enabled(*W(ws)) ? jit_dxt_bytes(*W(ws), B * K, n_sub, 0) : 0;
    return win_sub_bytes(*W(ws), B, K, n_sub) + whole;
}

size_t sig_backward_windows_workspace_bytes(const sig_wordset* ws, int64_t B, int64_t n_points, int64_t K, int64_t max_window_len)
{
    if (!ws || B <= 0 || K <= 0 || n_points < 1 || max_window_len < 0) return 0;
    if (windows_direct(*W(ws), B, K, 1)) return n_points > 1 ? gdx_bytes_of(*W(ws), B, n_points) : 0;
    const int64_t n_sub = max_window_len + 1;
    // the gather form; the forms that take windows as rows need less, or (a word per lane) the increment gradients of
    // the whole paths
    const size_t gather = 2 * win_sub_bytes(*W(ws), B, K, n_sub) + backward_workspace(ws, B * K, n_sub, false);
    return n_points > 1 ? std::max(gather, gdx_bytes_of(*W(ws), B, n_points)) : gather;
}

int sig_forward_windows(const sig_wordset* ws, const float* path, int64_t B, int64_t n_points, const int64_t* windows, int64_t K,
                        int64_t max_window_len, float* coeffs, void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    if (K < 0 || max_window_len < 0 || max_window_len > n_points - 1) return SIG_EINVAL;
    if (B == 0 || K == 0) return SIG_OK;
    if (!windows || !coeffs) return SIG_EINVAL;
    if (B * K > (int64_t)65535 * 64) return SIG_ETOOLARGE;
    const sig::WordSet& w = *W(ws);
    if (windows_direct(w, B, K, 0)) {
        hipStream_t st = (hipStream_t)stream;
        if (n_points == 1 || max_window_len == 0) {
            hipError_t e0 = sig::fill_zero(coeffs, B * K * w.size(), st);
            return e0 == hipSuccess ? SIG_OK : hip_fail(e0);
        }
        CallTimer whole(0, st);
        sig::WindowList wl;
        wl.win = windows; wl.K = K; wl.max_len = max_window_len;
        hipEvent_t* pe = g_prof.next(0);
        if (pe) (void)hipEventRecord(pe[0], st);
        hipError_t e1 = sig::trunc_forward_windows(w.d, w.depth, path, B, n_points, wl, coeffs, st);
        if (pe) (void)hipEventRecord(pe[1], st);
        return e1 == hipSuccess ? SIG_OK : hip_fail(e1);
    }
    const int64_t n_sub = max_window_len + 1;
    const size_t sb = win_sub_bytes(w, B, K, n_sub);
    if (!workspace || workspace_bytes < sig_forward_windows_workspace_bytes(ws, B, n_points, K, max_window_len)) return SIG_EWORKSPACE;
    if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
    // a word per lane (full truncations of any alphabet size): every (path, window) row reads its window of the path
    if (!use_trunc_forward(w, B * K) && use_lanes(w, B * K, kAnyLength, false) && n_points > 1 && max_window_len > 0) {
        const sig::LanesShape ls = lanes_shape_for(w, 0, B * K);
        if (sig::JitKernel* lk = ensure_lanes(w, 0, ls, Build::compile_and_load)) {
            hipStream_t st = (hipStream_t)stream;
            CallTimer whole(0, st);
            sig::WindowList wl;
            wl.win = windows; wl.K = K; wl.max_len = max_window_len;
            hipEvent_t* pe = g_prof.next(0);
            if (pe) (void)hipEventRecord(pe[0], st);
            hipError_t e = launch_lanes(lk->fn, ls, path, nullptr, nullptr, B, n_points, coeffs, st, wl);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    // straight-line specialised kernels: the rows' increments are transposed straight from the path, window by window
    if (windows_rows_jit(w, B * K) && n_points > 1 && max_window_len > 0) {
        const sig::Plan* jp = nullptr;
        if (sig::JitKernel* jk = ensure_jit(w, 0, B * K, Build::compile_and_load, &jp)) {
            hipStream_t st = (hipStream_t)stream;
            CallTimer whole(0, st);
            sig::WindowList wl;
            wl.win = windows; wl.K = K; wl.max_len = max_window_len;
            float* dxT = (float*)workspace;
            const int64_t Lpad = jit_lpad(w, n_sub, 0);
            hipError_t e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, nullptr, st, wl);
            if (e != hipSuccess) return hip_fail(e);
            hipEvent_t* pe = g_prof.next(0);
            if (pe) (void)hipEventRecord(pe[0], st);
            e = launch_jit_forward(*jk, *jp, dxT, B * K, max_window_len, Lpad, coeffs, w.size(), st);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    float* sub = (float*)workspace;
    hipError_t e = sig::window_gather(path, B, n_points, w.d, windows, K, n_sub, sub, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e);
    return forward_impl(ws, sub, B * K, n_sub, coeffs, (unsigned char*)workspace + sb, workspace_bytes - sb, stream, false);
}

int sig_backward_windows(const sig_wordset* ws, const float* path, const float* coeffs, const float* grad_coeffs, int64_t B,
                         int64_t n_points, const int64_t* windows, int64_t K, int64_t max_window_len, float* grad_path,
                         void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_common(ws, path, B, n_points);
    if (rc != SIG_OK) return rc;
    if (K < 0 || max_window_len < 0 || max_window_len > n_points - 1) return SIG_EINVAL;
    if (B == 0) return SIG_OK;
    if (!grad_path) return SIG_EINVAL;
    const sig::WordSet& w = *W(ws);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    const bool direct = K > 0 && windows_direct(w, B, K, 1);
    // the direct form stores every point itself
    if (!direct || n_points == 1 || max_window_len == 0) e = sig::fill_zero(grad_path, B * n_points * w.d, st);
    if (e != hipSuccess) return hip_fail(e);
    if (K == 0) return SIG_OK;
    if (!windows || !coeffs || !grad_coeffs) return SIG_EINVAL;
    if (B * K > (int64_t)65535 * 64) return SIG_ETOOLARGE;
    if (direct) {
        if (n_points == 1 || max_window_len == 0) return SIG_OK;            // grad_path is zero already
        if (!workspace || workspace_bytes < gdx_bytes_of(w, B, n_points)) return SIG_EWORKSPACE;
        if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
        CallTimer whole(1, st);
        float* gdx = (float*)workspace;
        e = sig::fill_zero(gdx, B * (n_points - 1) * w.d, st);
        if (e != hipSuccess) return hip_fail(e);
        sig::WindowList wl;
        wl.win = windows; wl.K = K; wl.max_len = max_window_len;
        hipEvent_t* pe = g_prof.next(1);
        if (pe) (void)hipEventRecord(pe[0], st);
        e = sig::trunc_backward_windows(w.d, w.depth, path, coeffs, grad_coeffs, B, n_points, wl, gdx, st);
        if (pe) (void)hipEventRecord(pe[1], st);
        if (e != hipSuccess) return hip_fail(e);
        e = sig::grad_points(gdx, B, n_points, w.d, grad_path, st);
        return e == hipSuccess ? SIG_OK : hip_fail(e);
    }
    const int64_t n_sub = max_window_len + 1;
    const size_t sb = win_sub_bytes(w, B, K, n_sub);
    if (!workspace || workspace_bytes < sig_backward_windows_workspace_bytes(ws, B, n_points, K, max_window_len)) return SIG_EWORKSPACE;
    if (((uintptr_t)workspace & 255) != 0) return SIG_EINVAL;
    // a word per lane: rows = windows read straight from the path, their gradients added up in grad_path (cleared above)
    if (!use_trunc_backward(w, B * K) && use_lanes(w, B * K, kAnyLength, false) && n_points > 1 && max_window_len > 0) {
        const sig::LanesShape ls = lanes_shape_for(w, 1, B * K);
        if (sig::JitKernel* lk = ensure_lanes(w, 1, ls, Build::compile_and_load)) {
            CallTimer whole(1, st);
            sig::WindowList wl;
            wl.win = windows; wl.K = K; wl.max_len = max_window_len;
            hipEvent_t* pe = g_prof.next(1);
            if (pe) (void)hipEventRecord(pe[0], st);
            e = launch_lanes(lk->fn, ls, path, coeffs, grad_coeffs, B, n_points, grad_path, st, wl);
            if (pe) (void)hipEventRecord(pe[1], st);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    // straight-line specialised kernels: rows = windows, increments and their gradients in the transposed layout, the
    // chain rule adds every window's gradient into grad_path (needs 2 arrays of the transposed layout: less than asked)
    if (windows_rows_jit(w, B * K) && n_points > 1 && max_window_len > 0) {
        const sig::Plan* jp = nullptr;
        if (sig::JitKernel* jk = ensure_jit(w, 1, B * K, Build::compile_and_load, &jp)) {
            CallTimer whole(1, st);
            sig::WindowList wl;
            wl.win = windows; wl.K = K; wl.max_len = max_window_len;
            const size_t t_bytes = jit_dxt_bytes(w, B * K, n_sub, 1);
            float* gdx = (float*)workspace;
            float* dxT = (float*)((unsigned char*)workspace + t_bytes);
            const int64_t Lpad = jit_lpad(w, n_sub, 1);
            e = sig::increments_transposed(path, B, n_points, w.d, Lpad, dxT, gdx, st, wl);
            if (e != hipSuccess) return hip_fail(e);
            hipEvent_t* pe = g_prof.next(1);
            if (pe) (void)hipEventRecord(pe[0], st);
            e = launch_jit_backward(*jk, *jp, dxT, coeffs, grad_coeffs, B * K, max_window_len, Lpad, w.size(), gdx, st);
            if (pe) (void)hipEventRecord(pe[1], st);
            if (e != hipSuccess) return hip_fail(e);
            e = sig::grad_points_transposed(gdx, B, n_points, w.d, Lpad, grad_path, st, wl);
            return e == hipSuccess ? SIG_OK : hip_fail(e);
        }
    }
    float* sub = (float*)workspace;
    float* gsub = (float*)((unsigned char*)workspace + sb);
    e = sig::window_gather(path, B, n_points, w.d, windows, K, n_sub, sub, st);
    if (e != hipSuccess) return hip_fail(e);
    rc = backward_impl(ws, sub, coeffs, grad_coeffs, B * K, n_sub, gsub, (unsigned char*)workspace + 2 * sb, workspace_bytes - 2 * sb,
                       stream, Build::compile_and_load, nullptr, false);
    if (rc != SIG_OK) return rc;
    e = sig::window_scatter(gsub, B, n_points, w.d, windows, K, n_sub, grad_path, st);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_profile_enable(int on)
{
    g_prof.mask = on == 1 ? 0xFu : ((unsigned)on >> 1) & 0xFu;
    for (size_t& u : g_prof.used) u = 0;
    return SIG_OK;
}

int sig_profile_read(int which, int64_t* n_launches, double* total_ms)
{
    if (which < 0 || which > 3) return SIG_EINVAL;
    const int dir = which;
    double sum = 0.0;
    for (size_t k = 0; k < g_prof.used[dir]; ++k) {
        hipError_t e = hipEventSynchronize(g_prof.ev[dir][2 * k + 1]);
        if (e != hipSuccess) return hip_fail(e);
        float ms = 0.0f;
        e = hipEventElapsedTime(&ms, g_prof.ev[dir][2 * k], g_prof.ev[dir][2 * k + 1]);
        if (e != hipSuccess) return hip_fail(e);
        sum += ms;
    }
    if (n_launches) *n_launches = (int64_t)g_prof.used[dir];
    if (total_ms) *total_ms = sum;
    return SIG_OK;
}

const char* sig_strerror(int code)
{
    switch (code) {
        case SIG_OK: return "success";
        case SIG_EINVAL: return "invalid argument";
        case SIG_ELETTER: return "letter outside [0, d)";
        case SIG_EEMPTYWORD: return "empty word or empty word list";
        case SIG_ENOMEM: return "out of host memory";
        case SIG_EWORKSPACE: return "workspace or table buffer missing or too small";
        case SIG_EHIP: return "HIP runtime error";
        case SIG_ETOOLARGE: return "word set exceeds a format limit";
        case SIG_ENOTUPLOADED: return "word set tables not uploaded";
        case SIG_EUNSUPPORTED: return "not supported for this word set";
        case SIG_EJIT: return "run-time compilation failed";
        case SIG_ENOTREADY: return "the kernel for this word set and batch is not loaded yet (call sig_backward once first)";
        default: return "unknown error";
    }
}

int sig_last_hip_error(void) { return g_last_hip; }
const char* sig_version(void) { return "sig-mi355x 0.1"; }

const char* sig_wordset_kernel_name(const sig_wordset* ws, int backward)
{
    if (!ws || !W(ws)->kernels_supported) return "unsupported";
    if (!backward && use_trunc_forward(*W(ws), 1)) return "trunc_mfma_fwd_kernel";
    if (backward && use_trunc_backward(*W(ws), 1)) return sig::trunc_backward_kernel_name(W(ws)->d, W(ws)->depth);
    if (use_lanes(*W(ws), 1, kAnyLength)) return backward ? "sig_bwd_lanes" : "sig_fwd_lanes";
    if (jit_enabled(*W(ws))) return backward ? "sig_bwd_jit" : "sig_fwd_jit";
    return backward ? "bwd_generic_kernel" : "fwd_generic_kernel";
}

int sig_jit_launch_shape_ok(int waves, int max_threads_per_block, int static_lds_bytes, int registers)
{
    return sig::jit_launch_shape_fits(waves, max_threads_per_block, static_lds_bytes, registers) ? 1 : 0;
}

int sig_probe_fma(void* out, size_t out_bytes, int blocks, int iters, void* stream)
{
    if (!out || blocks < 1 || iters < 1) return SIG_EINVAL;
    if (out_bytes < (size_t)blocks * 256 * sizeof(float)) return SIG_EWORKSPACE;
    hipError_t e = sig::fma_probe((float*)out, blocks, iters, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

int sig_probe_issue(void* out, size_t out_bytes, int blocks, int iters, int mode, void* stream)
{
    if (!out || blocks < 1 || iters < 1 || mode < 0 || mode > 7) return SIG_EINVAL;
    if (out_bytes < (size_t)blocks * 256 * sizeof(float)) return SIG_EWORKSPACE;
    hipError_t e = sig::issue_probe((float*)out, blocks, iters, mode, (hipStream_t)stream);
    return e == hipSuccess ? SIG_OK : hip_fail(e);
}

const char* sig_kernel_name(const sig_wordset* ws, int backward, int64_t B, int64_t n_points)
{
    if (!ws || !W(ws)->kernels_supported) return "unsupported";
    const sig::WordSet& w = *W(ws);
    if (B < 1 || n_points < 2) return sig_wordset_kernel_name(ws, backward);
    if (!backward && use_trunc_forward(w, B))
        return trunc_forward_fused_chunks(w, B, n_points, nullptr) ? "trunc_tails_fwd_kernel" : "trunc_mfma_fwd_kernel";
    if (backward && use_trunc_backward(w, B)) {
        const BwdShape sh = trunc_backward_shape(w, B, n_points);
        return sh.tails ? "trunc_tails_bwd_kernel" : sig::trunc_backward_kernel_name(w.d, w.depth);
    }
    if (use_lanes(w, B, n_points - 1)) return backward ? "sig_bwd_lanes" : "sig_fwd_lanes";
    if (jit_enabled(w)) return backward ? "sig_bwd_jit" : "sig_fwd_jit";
    return backward ? "bwd_generic_kernel" : "fwd_generic_kernel";
}

}  // extern "C"
