// Full truncations of any alphabet size with lanes = words: kernels compiled at run time (hiprtc) from one fixed
// source with the shape (d, N) as macros, because the register arrays below are sized by d.
//
// Layout (the one of trunc_node_bwd_kernel, without its power-of-two assumptions): a lane holds a word u of length
// K = N - R together with everything below it, R = 1 (the d leaves under u) or R = 2 (d children and d^2 leaves).
// The coefficients of u's prefixes (the chain) are recomputed in every lane that shares them and stored by one.
// The letters below u are the same in every lane, so those levels are multiply-adds with lane-uniform increments
// (Section 3.1, eq. (3) and Algorithm 1, with the Horner intermediates shared between words).  ceil(d^K / 64)
// wavefronts serve a path; lanes past d^K carry a copy of the last word with zero adjoints and store nothing.
// Against lanes = paths this fills the wavefronts for any batch size and needs one short compilation per shape
// instead of one that grows with the word set.
#include <algorithm>
#include <cmath>
#include <sstream>
#include <string>

#include "jit.hpp"

namespace sig {
namespace {

const char* const kLanesSource = R"SRC(
#define K (N - R)
#define NC ((N + 3) / 4 * 4)
#define DP ((D + 3) / 4 * 4)
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int ipow(int b, int e)
{
    int r = 1;
    for (int q = 0; q < e; ++q) r *= b;
    return r;
}
// first canonical index of the words of length n >= 1
constexpr long level_start(int n)
{
    long r = 0;
    for (int m = 1; m < n; ++m) r += ipow(D, m);
    return r;
}
constexpr float inv1(int t) { return 1.0f / (float)(t + 1); }
// chain positions k = 1 .. NU whose letter takes at most three values inside a wavefront (runs of D^(K-k) >= 32 lanes)
constexpr int count_wide()
{
    int n = 0;
    for (int k = 1; k <= K; ++k) n += ipow(D, K - k) >= 32 ? 1 : 0;
    return n;
}

#define NL ipow(D, K)                       /* words of length K = lanes per path */
#define WAVES ((NL + 63) / 64)
#define NWORDS (level_start(N) + ipow(D, N))
#define NU count_wide()

static_assert(K >= 1 && (R == 1 || R == 2), "a lane holds a word of length N - R and one or two levels below it");
// MSUM: backward with the leaves alone below u, gradient sums over the lanes as matrix products (see there)
static_assert((MSUM || !BACKWARD || T * D <= 64) && TS % T == 0, "one lane per (letter, segment) of a tile; whole tiles per staging tile");

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Increments are staged TS segments at a time (a multiple of T; the global loads of the next staging tile are in
// flight while this one is worked on, and a longer tile hides their latency when a SIMD has a single wavefront).
// Element e = lane + 64 q of a staging tile is (segment j0 + e / D, letter e % D); zero outside [0, L).
#define EPL ((TS * D + 63) / 64)
__device__ __forceinline__ void fetch_increments(const float* __restrict__ X, long j0, long L, int lane, float (&dx)[EPL])
{
    // points are rows of D floats, so element e of the tile is X[j0 D + e + D] - X[j0 D + e]
    const long base = j0 * D, lim = L * D;
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
        long idx = base + lane + 64 * q;
        const bool ok = idx >= 0 && idx < lim;
        idx = idx < 0 ? 0 : (idx < lim ? idx : lim - 1);
        const float x1 = X[idx + D], x0 = X[idx];
        dx[q] = ok ? x1 - x0 : 0.0f;
    }
}
// LDS of a staging tile: Ec[segment][letter][t] = dX / (t + 1) for the chain (a lane reads the row of its own
// letter), and E0[segment][letter] = dX as contiguous rows for the levels below u (every lane reads all
// letters)
#define TILE_F (TS * D * NC + TS * DP)
__device__ __forceinline__ void stage_increments(float* Ec, const float (&dx)[EPL], int lane)
{
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
        const int e = lane + 64 * q;
        if (e < TS * D) {
#pragma unroll
            for (int t = 0; t < N; ++t) Ec[e * NC + t] = dx[q] * inv1(t);
            float* E0 = Ec + TS * D * NC;
            E0[(e / D) * DP + e % D] = dx[q];
        }
    }
}
// the D increments of a segment from one of the contiguous rows
__device__ __forceinline__ void load_row(const float* row, float (&e)[DP])
{
#pragma unroll
    for (int q = 0; q < DP / 4; ++q) {
        const f4 v = ((const f4*)row)[q];
        e[4 * q] = v[0]; e[4 * q + 1] = v[1]; e[4 * q + 2] = v[2]; e[4 * q + 3] = v[3];
    }
}

// What a lane reads of a segment: all letters' increments, and the scaled increments of its chain letters.
struct Segment {
    float e0[DP], ec[K][NC];
    __device__ __forceinline__ void read(const float* Ec, const float* E0, int at, const int (&letter)[K])
    {
        load_row(E0 + at * DP, e0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float* src = Ec + (at * D + letter[k]) * NC;
#pragma unroll
            for (int t = 0; t <= N - (k + 1) + (BACKWARD && k > 0 ? 1 : 0); ++t) ec[k][t] = src[t];
        }
    }
};
// Segments are worked on in groups whose reads are issued together: a lone wavefront otherwise waits for LDS in every
// segment (forward, one path of 199 segments, d = 10, depth 4: 39 -> 23 us; 8 x 1,000, d = 3, depth 5: 168 -> 84).  A tile's
// last group may reach past the end of the row, where the staged increments are zero: such a segment changes nothing.
// Two levels below u fill the registers with their own state: one segment after the other there, and forward, beyond 48
// values (LAZY), every read where it is used (256 x 199 segments, 10 letters, depth 4: 58 us against 64 in pairs; 16 x 100, 6
// letters, depth 6: 34 against 30).
#define LAZY (R == 2 && (D + SP - 1) / SP * (D + 1) > 48)
#define GROUP (LAZY || TS % 2 ? 1 : (R == 1 && TS % 4 == 0 && DP + K * NC <= 32 ? 4 : 2))
// Two letters and a chain of seven or more: the addresses of the 190 predicated reads that sum the short runs do not change
// from tile to tile, and held in registers over the loop they cost half the speed, as do two segments or two row sums in flight
// (100 segments, two wavefronts per SIMD: depth 9 446 -> 163 us, depth 10 553 -> 211, 12 823 -> 304).  So there they are formed
// anew, and one thing is done after the other.
#define ONE_BY_ONE (!MSUM && D == 2 && K >= 7)
#define BGROUP (R == 2 || T % 2 ? 1 : (MSUM && DP + K * NC <= 32 ? 4 : 2))

// Row r is part k = r % KW of path r / KW, read straight from the path: with win == nullptr time chunk k, max_len segments
// from segment k * max_len on (KW = 1 and max_len = P - 1: the whole path); otherwise window k, between the points
// win[2 k] and win[2 k + 1] clamped to the path, at most max_len segments.
__device__ __forceinline__ void row_of(const long* __restrict__ win, long KW, long max_len, long r, long P, long& b, long& k,
                                       long& first, long& L)
{
    b = r / KW;
    k = r - b * KW;
    if (win == nullptr) {
        first = k * max_len;
        L = P - 1 - first < max_len ? P - 1 - first : max_len;
    } else {
        long l = win[2 * k], e = win[2 * k + 1];
        l = l < 0 ? 0 : (l > P - 1 ? P - 1 : l);
        e = e < l ? l : (e > P - 1 ? P - 1 : e);
        first = l;
        L = e - l < max_len ? e - l : max_len;
    }
}

#if !BACKWARD
// SP = 2 (two levels below u): two wavefronts share 64 words, each with half of the children and what lies below them, both with
// the whole chain.  For batches that would leave SIMDs without a wavefront otherwise: the halves cost a chain more, time chunks
// their signatures' traffic (256 paths x 199 segments, d = 10, depth 4: 60 us in two chunks -> 48 us whole).
#define DJ ((D + SP - 1) / SP)
extern "C" __global__ __launch_bounds__(64 * NWB) void FORWARD_NAME(const float* __restrict__ path, long B, long P,
                                                                      float* __restrict__ coeffs, const long* __restrict__ win,
                                                                      long KW, long max_len
#if CLEARS
                                                                      , float* __restrict__ zero, long n_zero
#endif
                                                                      )
{
#if CLEARS
    // n_zero floats at `zero` are cleared on the way for the kernel that runs next (backward; two more arguments cost a forward
    // call 0.2 us of launch)
    for (long e = (long)blockIdx.x * (64 * NWB) + threadIdx.x; e < n_zero; e += (long)gridDim.x * (64 * NWB)) zero[e] = 0.0f;
#endif
    __shared__ __attribute__((aligned(16))) float smem[NWB * TILE_F];
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long wave = (long)blockIdx.x * NWB + wib;
    if (wave >= B * KW * WAVES * SP) return;             // wavefronts share nothing: no barrier is skipped
    float* Ec = smem + wib * TILE_F;
    const float* E0 = Ec + TS * D * NC;
    const long row = wave / (WAVES * SP);
    long b, part, first, L;
    row_of(win, KW, max_len, row, P, b, part, first, L);
    const int in_row = __builtin_amdgcn_readfirstlane((int)(wave - row * (WAVES * SP)));
    const int p0 = in_row / SP * 64, j0 = in_row % SP * DJ;          // first word, first child
    const bool valid = p0 + lane < NL;
    const int p = valid ? p0 + lane : NL - 1;
    int letter[K];
    {
        int q = p;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) { letter[k] = q % D; q /= D; }
    }
    const float* X = path + (b * P + first) * D;

    float Sc[K], S1[DJ];
#pragma unroll
    for (int k = 0; k < K; ++k) Sc[k] = 0.0f;
#pragma unroll
    for (int j = 0; j < DJ; ++j) S1[j] = 0.0f;
#if R == 2
    float S2[DJ][D];
#pragma unroll
    for (int j = 0; j < DJ; ++j)
#pragma unroll
        for (int jj = 0; jj < D; ++jj) S2[j][jj] = 0.0f;
#endif

    const long ntiles = (L + TS - 1) / TS;
    float dxn[EPL];
#pragma unroll
    for (int q = 0; q < EPL; ++q) dxn[q] = 0.0f;
    if (L > 0) fetch_increments(X, 0, L, lane, dxn);     // an empty window reads nothing and stores the zero signature
    for (long n = 0; n < ntiles; ++n) {
        wave_lds_fence();
        stage_increments(Ec, dxn, lane);
        wave_lds_fence();
        fetch_increments(X, (n + 1) * TS, L, lane, dxn); // past the end: zeros, and a zero increment changes nothing
#if LAZY
#pragma unroll 2
        for (int tt = 0; tt < TS; ++tt) {
            const float* Et = Ec + tt * D * NC;
            float e0[DP];
            load_row(E0 + tt * DP, e0);
          {
#else
        const int steps = L - n * TS < TS ? (int)(L - n * TS) : TS;
#pragma unroll 1
        for (int t0 = 0; t0 < steps; t0 += GROUP) {
          Segment xs[GROUP];
#pragma unroll
          for (int u = 0; u < GROUP; ++u) xs[u].read(Ec, E0, t0 + u, letter);
#pragma unroll
          for (int u = 0; u < GROUP; ++u) {
            const int tt = t0 + u;
            const float (&e0)[DP] = xs[u].e0;
#endif
            float ap[K + 1][N + 2];
#pragma unroll
            for (int t = 0; t < N + 2; ++t) ap[0][t] = 1.0f;
#pragma unroll
            for (int k = 1; k <= K; ++k) {
#if LAZY
                const float* src = Et + letter[k - 1] * NC;
#else
                const float (&src)[NC] = xs[u].ec[k - 1];
#endif
#pragma unroll
                for (int t = 1; t <= N - k; ++t) ap[k][t] = __builtin_fmaf(src[t], ap[k - 1][t + 1], Sc[k - 1]);
                Sc[k - 1] = __builtin_fmaf(src[0], ap[k - 1][1], Sc[k - 1]);
            }
#if R == 2
            // the increments of the wavefront's own children (of half of an odd alphabet the last is none: its place is padding).  A child's
            // intermediate S1 + dX / 2 A takes dX and half of A: halving is exact, and there is no second row of increments to read.
            const float half = 0.5f * ap[K][2];
#if SP == 1
            const float (&own)[DP] = e0;
#else
            float own[DJ];
#pragma unroll
            for (int j = 0; j < DJ; ++j) own[j] = E0[tt * DP + j0 + j];
#endif
#else
            const float (&own)[DP] = e0;
#endif
#pragma unroll
            for (int j = 0; j < DJ; ++j) {
#if R == 2
                const float Gp = __builtin_fmaf(own[j], half, S1[j]);
#pragma unroll
                for (int jj = 0; jj < D; ++jj) S2[j][jj] = __builtin_fmaf(e0[jj], Gp, S2[j][jj]);
#endif
                S1[j] = __builtin_fmaf(own[j], ap[K][1], S1[j]);
            }
          }
        }
    }

    if (!valid) return;
    float* out = coeffs + row * NWORDS;
#pragma unroll
    for (int k = 1; k <= K; ++k)
        if (j0 == 0 && p % ipow(D, K - k) == 0) out[level_start(k) + p / ipow(D, K - k)] = Sc[k - 1];
#pragma unroll
    for (int j = 0; j < DJ; ++j) {
        if (SP > 1 && j0 + j >= D) break;
        out[level_start(K + 1) + (long)p * D + j0 + j] = S1[j];
#if R == 2
#pragma unroll
        for (int jj = 0; jj < D; ++jj) out[level_start(K + 2) + ((long)p * D + j0 + j) * D + jj] = S2[j][jj];
#endif
    }
}
#else
// Backward (Section 4: reconstruction, Proposition 4.6; gradient of Proposition 4.1 in its adjoint form).
// Per segment a lane produces one gradient contribution per letter below u (all lanes to the same letter) and one
// per chain position (to the lane's own letter at that position).  They go to LDS rows [source][segment][lane] for
// the segments of a tile and are summed per tile:
//   - rows of the letters below u: lane j T + t adds up row (j, t);
//   - chain positions whose letter runs over fewer than 32 lanes: the same lane adds the members of its letter;
//   - chain positions with longer runs (at most three of them reach into a wavefront): a lane writes to the row of
//     its run, and these rows are summed like the rows of the first kind by a second group of lanes, whose sums the
//     lane of the letter then picks up.
// The chain rule from increments to points (a point is the end of one segment and the start of the next) is applied to
// the sums of a wavefront: the point after segment s gets its gradient less that of segment s + 1, which is the
// neighbouring lane's or, at the end of a tile, the first of the tile walked before.  So there is one floating-point
// atomic into grad_path (zeroed by the caller) per letter and segment and no array of increment gradients.
// With one level below u and up to 16 letters the sums are instead one matrix product per tile of 16 segments,
//   g(j, s) = sum_p G(p j) A+_p(s)[1] + sum_k sum_p [letter k of p is j] c_k(p, s),
// letters x (1 + K) 64 words times (1 + K) 64 words x segments on 16x16x4 instructions: the leaf adjoints G and the 0/1
// indicators are constant (16 registers each), the right factor goes through LDS, one value per lane, segment and
// source.  The sums by rows of LDS above took two thirds of a wavefront's time (D + K writes and D products a segment,
// 64 chained additions and up to 28 predicated reads a tile): one path of 199 segments, d = 10, depth 4, walked whole:
// 125 -> 59 us; 8 x 1,000, d = 3, depth 5: 603 -> 315.
#if MSUM
#define VROW 68                              /* 64 lanes and a shift of four banks per segment */
#define BW_PER_WAVE (TILE_F + (K + 1) * 16 * VROW)
#else
#define NSRC (D + K + 2 * NU)
#define BW_PER_WAVE (TILE_F + NSRC * T * 64 + (3 * NU * T + 3) / 4 * 4)
#endif
// row of chain position k (1-based): three rows for each of the first NU positions, one for the others
constexpr int chain_row(int k) { return k <= NU ? D + 3 * (k - 1) : D + 3 * NU + (k - NU - 1); }

__device__ __forceinline__ float row_sum(const float* row, int lane)
{
    // rows lie 256 bytes apart: every lane starts at another 16-byte piece of its row
    const f4* r = (const f4*)row;
    f4 acc = r[lane & 15];
#pragma unroll
    for (int i = 1; i < 16; ++i) acc += r[(i + lane) & 15];
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

#if MSUM
// The sums of one segment for letters j0 .. j0 + 3 lane by lane: of the wavefront's words (the first is p0) every letter takes
// the products with its leaf adjoints and the chain values of the words that have it at the position.  v: the segment's row
// of the first source.  Rolled loops: it runs only where a sum is not finite.
__device__ __forceinline__ void letter_sums(const float* v, const float* __restrict__ leaves, int p0, int j0, f4& sum)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = j0 + r;
        float acc = 0.0f;
        if (j < D) {
#pragma unroll 1
            for (int i = 0; i < 64; ++i) {
                const bool in = p0 + i < NL;
                int q = in ? p0 + i : NL - 1;                  // lanes past the last word hold a copy of it
                acc = __builtin_fmaf(in ? leaves[(long)q * D + j] : 0.0f, v[i], acc);
#pragma unroll 1
                for (int k = K; k >= 1; --k) {
                    acc += q % D == j ? v[k * 16 * VROW + i] : 0.0f;
                    q /= D;
                }
            }
        }
        sum[r] = acc;
    }
}
#endif

// Signature and adjoints at the end of chunk `part` of a path, from the signatures S_0 .. S_{C-1} of its chunks over the words
// shorter than N (rows), for the lane's words alone: what a kernel for the products and one for the adjoints would write to arrays.
//   - S_0 S_1 .. S_part on the lane's chain needs the chain itself and infixes of the lane's word;
//   - the adjoints at the end of the path, taken back over chunks C - 1 .. part + 1: Abar(u) += sum_v Abar(u v) S_c(v).  The walk is
//     linear in them and a chain word's may be spread over the lanes that share it, so a lane adds the terms whose word u v is its
//     own (in its registers) to its share of Abar(u), nothing exchanged between the chunks.
// In the end the shares of a wavefront are summed: those of a gradient whose terms cancel (that of a log-signature) are larger than
// their sum, and the walk would round them.  Error of such a gradient, shares -> sums -> one value per word (arrays): 27 and 64 lanes
// a path (3 and 4 letters, depth 4) 1.25, 1.37 -> 1.00 -> 1; a word whose lanes lie in several wavefronts keeps that many shares,
// 1,000 lanes (10 letters) 1.38 -> 1.30 -> 1 (256 paths 0.99: two levels a lane, 100 lanes), still below the walk over whole
// paths, 1.8.  Backward calls of 12 to 33 us take 0.1 to 0.8 us for it; the arrays cost 5 to 15.
// The rows pass through the wavefront's LDS one after the other, each loaded while the one before is used.
// Bound by the latency of a row (0.3-0.6 us); two launches of 5 us and the arrays' traffic saved (256 paths x 199 segments, d = 10,
// depth 4: 30 us of 181).
__device__ __forceinline__ void chunk_boundary(const float* __restrict__ rows, int part, int C, int p0, int p, int lane, float* st,
                                               float (&Sc)[K], float (&Ac)[K], float (&A1)[D]
#if R == 2
                                               , float (&S1)[D], float (&An)[D][D]
#endif
                                               )
{
    constexpr int NLOW = (int)level_start(N), NQ = (NLOW + 63) / 64;
    // Two levels: lanes read the words of length N - 1 in runs of D^2 from run to run; where those lie in a few banks (D a multiple of four)
    // a run is a float longer (backward calls, 4 letters, depth 5, 90 paths x 130 segments 27.6 -> 19.7 us, 8 letters, depth 4, 90 x 130
    // 35.3 -> 27.4, with chunks of whole tiles; 12 letters have no register for the places).
    constexpr bool PADDED = R == 2 && D % 4 == 0 && D <= 10 && NLOW + ipow(D, K - 1) <= BW_PER_WAVE;
    auto place = [&](int e) { return PADDED && e >= level_start(N - 1) ? e + (e - (int)level_start(N - 1)) / (D * D) : e; };
    float ahead[NQ];
    auto fetch = [&](int c) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) ahead[q] = rows[(long)c * NLOW + (lane + 64 * q < NLOW ? lane + 64 * q : 0)];
    };
    fetch(0);
#pragma unroll 1
    for (int i = 0; i < C; ++i) {
        wave_lds_fence();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (lane + 64 * q < NLOW) st[place(lane + 64 * q)] = ahead[q];
        wave_lds_fence();
        if (i + 1 < C) fetch(i + 1 <= part ? i + 1 : C - (i + 1 - part));       // up to `part`, then back from the last
        if (i <= part) {
#if R == 2
#pragma unroll
            for (int j = 0; j < D; ++j) {                       // longer words first: a word reads the chain as it was
                float v = st[level_start(K + 1) + p * D + j + (PADDED ? p / D : 0)];
                if (i > 0) {
                    v += S1[j];
#pragma unroll
                    for (int m = 1; m <= K; ++m)
                        v = __builtin_fmaf(Sc[m - 1], st[level_start(K + 1 - m) + (p % ipow(D, K - m)) * D + j], v);
                }
                S1[j] = v;
            }
#endif
#pragma unroll
            for (int k = K; k >= 1; --k) {
                const int u = p / ipow(D, K - k);
                float v = st[level_start(k) + u];
                if (i > 0) {
                    v += Sc[k - 1];
#pragma unroll
                    for (int m = 1; m < k; ++m) v = __builtin_fmaf(Sc[m - 1], st[level_start(k - m) + u % ipow(D, k - m)], v);
                }
                Sc[k - 1] = v;
            }
        } else {
#pragma unroll
            for (int k = 1; k <= K; ++k) {
                const int after = p % ipow(D, K - k);           // the lane's word without its first k letters
                float v = Ac[k - 1];
#pragma unroll
                for (int n = k + 1; n <= K; ++n)
                    v = __builtin_fmaf(Ac[n - 1], st[level_start(n - k) + (p / ipow(D, K - n)) % ipow(D, n - k)], v);
#pragma unroll
                for (int j = 0; j < D; ++j) v = __builtin_fmaf(A1[j], st[level_start(K - k + 1) + after * D + j], v);
#if R == 2
#pragma unroll
                for (int j = 0; j < D; ++j)
#pragma unroll
                    for (int jj = 0; jj < D; ++jj) v = __builtin_fmaf(An[j][jj], st[level_start(K - k + 2) + (after * D + j) * D + jj + (PADDED && k == 1 ? after : 0)], v);
#endif
                Ac[k - 1] = v;
            }
#if R == 2
#pragma unroll
            for (int j = 0; j < D; ++j)
#pragma unroll
                for (int jj = 0; jj < D; ++jj) A1[j] = __builtin_fmaf(An[j][jj], st[jj], A1[j]);
#endif
        }
    }
    // (the lanes that share a word are consecutive; the sum lies in the first of them)
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const int m = ipow(D, K - k), in_run = (p0 + lane) % m;
        float v = Ac[k - 1];
#pragma unroll
        for (int off = 1; off < 64 && off < m; off *= 2) {
            const float other = __shfl_down(v, off);
            if (lane + off < 64 && in_run + off < m) v += other;
        }
        Ac[k - 1] = lane == 0 || in_run == 0 ? v : 0.0f;
    }
}

// Two levels of eleven and twelve letters take the registers that two wavefronts of a SIMD have each, if addresses that do not change from
// tile to tile are formed anew and segments taken one by one: depth 3 and 4 fit (233 to 255 registers, none spilled), longer chains
// spill 19 to 48 of them (80 to 196 bytes of scratch a lane).  One level walks with ten times the wavefronts.  Backward calls, one
// level -> two: depth 4, 11 letters 256 x 400 494 -> 153 us, 64 x 150 72 -> 54; 12 letters 128 x 300 278 -> 133; depth 5, 11 letters
// 16 x 100 196 -> 158, 64 x 100 583 -> 180, 256 x 40 1,125 -> 261; 12 letters 16 x 100 296 -> 184, 256 x 40 1,744 -> 444; depth 6, 11
// letters 2 x 60 504 -> 133, 16 x 60 1,630 -> 321.  Without that bound depth 5 spills nothing and has a SIMD to itself: 16 x 100 134, but
// 64 x 100 270, 256 x 40 353.
#define TWO_A_SIMD (R == 2 && D > 10)
#if TWO_A_SIMD
#define WAVES_PER_SIMD __attribute__((amdgpu_waves_per_eu(2)))
#else
#define WAVES_PER_SIMD
#endif
extern "C" __global__ __launch_bounds__(64 * NWB) WAVES_PER_SIMD void sig_bwd_lanes(const float* __restrict__ path,
        const float* __restrict__ coeffs, const float* __restrict__ grad, long B, long P, float* grad_path,
        const long* __restrict__ win, long KW, long max_len, const float* __restrict__ low_coeffs, const float* __restrict__ low_grad)
{
    __shared__ __attribute__((aligned(16))) float smem[NWB * BW_PER_WAVE];
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long wave = (long)blockIdx.x * NWB + wib;
    if (wave >= B * KW * WAVES) return;
    float* Ec = smem + wib * BW_PER_WAVE;
    const float* E0 = Ec + TS * D * NC;
    float* Vb = Ec + TILE_F;
#if !MSUM
    float* Wide = Vb + NSRC * T * 64;                    // [3 NU][T] sums over long runs
#endif
    const long row = wave / WAVES;
    long b, part, first, L;
    row_of(win, KW, max_len, row, P, b, part, first, L);
    const int p0 = __builtin_amdgcn_readfirstlane((int)(wave - row * WAVES) * 64);
    const bool valid = p0 + lane < NL;
    const int p = valid ? p0 + lane : NL - 1;
    int letter[K];
    {
        int q = p;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) { letter[k] = q % D; q /= D; }
    }
    if (L <= 0) return;                                  // an empty window: no gradient (wavefronts share no barrier)
    const float* X = path + (b * P + first) * D;
    // Whole paths and windows have a row of their own in coeffs and grad.  A time chunk takes the adjoints of the words of
    // length N, constant in time, from its path's row, and so does a path's last chunk with all others; for the chunks
    // before it, signature and adjoints at the end of the chunk (words shorter than N, the longest are never
    // reconstructed) are rows of low_coeffs and low_grad [B][KW - 1].  Without low_grad the rows of low_coeffs [B][KW] are the
    // chunks' own signatures, from which a lane works out what it needs (below).
    const long whole = win == nullptr ? b : row;
    const bool inner = win == nullptr && part + 1 < KW, given = inner && low_grad != nullptr;
    const float* gr = grad + whole * NWORDS;
    const float* cf = given ? low_coeffs + (b * (KW - 1) + part) * level_start(N) : coeffs + whole * NWORDS;
    const float* gl = given ? low_grad + (b * (KW - 1) + part) * level_start(N) : gr;
    float* const gp_row = grad_path + (b * P + first) * D;      // the gradients of overlapping windows add up here

    // signature and adjoints at the end of the path; a word shared by several lanes has its adjoint in the first
    float Sc[K], Ac[K], A1[D];
#pragma unroll
    for (int k = 1; k <= K; ++k) {
        const long w = level_start(k) + p / ipow(D, K - k);
        Sc[k - 1] = cf[w];
        Ac[k - 1] = valid && p % ipow(D, K - k) == 0 ? gl[w] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < D; ++j) A1[j] = valid ? (R == 1 ? gr : gl)[level_start(K + 1) + (long)p * D + j] : 0.0f;
#if R == 2
    float S1[D], An[D][D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        S1[j] = cf[level_start(K + 1) + (long)p * D + j];
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
#pragma unroll
        for (int jj = 0; jj < D; ++jj) An[j][jj] = 0.0f;
    // The leaf adjoints under a wavefront's words are one contiguous run of memory, but a lane's are D^2 floats from the next
    // lane's: read lane by lane every load touches 64 cache lines, which the wavefronts of a compute unit push out of its 32 KB
    // before their next load comes back to them (256 paths x 199 segments, d = 10, depth 4: 93 us, 80 this way).  So they come
    // through the wavefront's LDS, a word a load into rows of an odd number of floats, as many words at a time as fit.
    // (Forward stores that way: 4 us slower on the same case, whose wavefronts are alone on their SIMDs.)
    {
        constexpr int LR = (D * D) | 1, PER = (D * D + 63) / 64;
        constexpr int NW = 64 * LR <= BW_PER_WAVE ? 64 : (32 * LR <= BW_PER_WAVE ? 32 : (16 * LR <= BW_PER_WAVE ? 16 : 8));
        static_assert(NW * LR <= BW_PER_WAVE, "eight words at least");
        const float* src = gr + level_start(K + 2);
#pragma unroll
        for (int w0 = 0; w0 < 64; w0 += NW) {
            wave_lds_fence();
#pragma unroll 1
            for (int w = 0; w < NW; w += 8) {                  // loads of eight words in flight, from clamped addresses
                float v[8][PER];
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int q = 0; q < PER; ++q) {
                        const int word = p0 + w0 + w + u, i = lane + 64 * q;
                        v[u][q] = src[(long)(word < NL ? word : NL - 1) * (D * D) + (i < D * D ? i : 0)];
                    }
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int q = 0; q < PER; ++q)
                        if (lane + 64 * q < D * D) Ec[(w + u) * LR + lane + 64 * q] = v[u][q];
            }
            wave_lds_fence();
            if (lane / NW == w0 / NW && valid) {
#pragma unroll
                for (int j = 0; j < D; ++j)
#pragma unroll
                    for (int jj = 0; jj < D; ++jj) An[j][jj] = Ec[lane % NW * LR + j * D + jj];
            }
        }
        wave_lds_fence();
    }
#endif
    if constexpr (level_start(N) <= BW_PER_WAVE) {
        if (inner && !given) chunk_boundary(low_coeffs + b * KW * level_start(N), (int)part, (int)KW, p0, p, lane, Ec, Sc, Ac, A1
#if R == 2
                                            , S1, An
#endif
                                            );
    }
#if MSUM
    // left factors: lane (16 g + j) holds row j, words p0 + 16 g + i, i = 0 .. 15
    const int col = lane & 15, grp = lane >> 4;
    // (the loads from clamped addresses, all in flight at once; the letters through LDS instead of sixteen times K divisions)
    float leaf_rows[16], chain_rows[K][16], later[4];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int q = p0 + grp * 16 + i;
        leaf_rows[i] = gr[level_start(N) + (long)(q < NL ? q : NL - 1) * D + (col < D ? col : 0)];
    }
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < K; ++k) Vb[k * 64 + lane] = (float)letter[k];
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f4 v = *(const f4*)(Vb + k * 64 + grp * 16 + 4 * i);
#pragma unroll
            for (int r = 0; r < 4; ++r) chain_rows[k][4 * i + r] = v[r] == (float)col ? 1.0f : 0.0f;
        }
#pragma unroll
    for (int i = 0; i < 16; ++i) leaf_rows[i] = p0 + grp * 16 + i < NL && col < D ? leaf_rows[i] : 0.0f;   // (words past the last: zeros)
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) later[r] = 0.0f;
#else
    // chain positions with long runs: the run of this lane among those that reach into the wavefront (0, 1 or 2),
    // how many do, and the letter of the first
    int my_run[NU + 1], runs[NU + 1], first_letter[NU + 1];
#pragma unroll
    for (int k = 1; k <= NU; ++k) {
        const int s = ipow(D, K - k);
        my_run[k] = (p0 + lane) / s - p0 / s;
        runs[k] = (p0 + 63) / s - p0 / s + 1;
        first_letter[k] = (p0 / s) % D;
    }

    float later = 0.0f;                                        // lane (j, T - 1): gradient of the segment after this tile
#endif
    const long nstage = (L + TS - 1) / TS;
    float dxn[EPL];
    fetch_increments(X, (nstage - 1) * TS, L, lane, dxn);
    for (long ns = nstage - 1; ns >= 0; --ns) {
        wave_lds_fence();
        stage_increments(Ec, dxn, lane);
        wave_lds_fence();
        fetch_increments(X, (ns - 1) * TS, L, lane, dxn);
      for (int sub = TS / T - 1; sub >= 0; --sub) {          // tiles of T segments: the unit of the gradient sums
        const long n = ns * (TS / T) + sub;
        // (the last tile may be a partial one: what the rows hold for the segments that it lacks is summed and dropped)
        const int steps = (MSUM || R == 2) && L - n * T < T ? (int)(L - n * T) : T;
#pragma unroll (BGROUP == 1 && !ONE_BY_ONE && !TWO_A_SIMD ? 2 : 1)
        for (int t1 = (steps + BGROUP - 1) / BGROUP * BGROUP; t1 > 0; t1 -= BGROUP) {
          Segment xs[BGROUP];
#pragma unroll
          for (int u = 0; u < BGROUP; ++u) xs[u].read(Ec, E0, sub * T + t1 - 1 - u, letter);
#pragma unroll
          for (int u = 0; u < BGROUP; ++u) {
            const int tt = t1 - 1 - u;
            const Segment& x = xs[u];
            const float (&e0)[DP] = x.e0;
            const float (&ec)[K][NC] = x.ec;
            // Reconstruction by solving the forward step for the signature it started from: a word needs of the shorter ones only
            // the Horner intermediates with +dX, formed word by word on the way down the chain.
            float ap[K + 1][N + 2];
#pragma unroll
            for (int t = 0; t < N + 2; ++t) ap[0][t] = 1.0f;
#pragma unroll
            for (int k = 1; k <= K; ++k) {
                Sc[k - 1] = __builtin_fmaf(-ec[k - 1][0], ap[k - 1][1], Sc[k - 1]);
#pragma unroll
                for (int t = 1; t <= N - k; ++t) ap[k][t] = __builtin_fmaf(ec[k - 1][t], ap[k - 1][t + 1], Sc[k - 1]);
            }
#if MSUM
            float* vb = Vb + tt * VROW + lane;
            vb[0] = ap[K][1];
#else
            float* vb = Vb + tt * 64 + lane;
#endif
            float g1 = 0.0f;
#if R == 1
            // the leaves: constant adjoints
#pragma unroll
            for (int j = 0; j < D; ++j) {
#if !MSUM
                vb[j * T * 64] = A1[j] * ap[K][1];
#endif
                g1 = __builtin_fmaf(e0[j], A1[j], g1);
            }
#else
            float y[D];
#pragma unroll
            for (int j = 0; j < D; ++j) y[j] = 0.0f;
            const float hp2 = 0.5f * ap[K][2];
            float g2 = 0.0f;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                S1[j] = __builtin_fmaf(-e0[j], ap[K][1], S1[j]);
                const float Gp = __builtin_fmaf(e0[j], hp2, S1[j]);
                float h = 0.0f;
#pragma unroll
                for (int jj = 0; jj < D; ++jj) {
                    h = __builtin_fmaf(e0[jj], An[j][jj], h);
                    y[jj] = __builtin_fmaf(An[j][jj], Gp, y[jj]);
                }
                const float q0 = A1[j];
                A1[j] = q0 + h;
                y[j] = __builtin_fmaf(q0, ap[K][1], y[j]);
                y[j] = __builtin_fmaf(h, hp2, y[j]);
                g1 = __builtin_fmaf(e0[j], q0, g1);
                g2 = __builtin_fmaf(e0[j], h, g2);               // (of halved increments: the factor comes below)
            }
#pragma unroll
            for (int j = 0; j < D; ++j) vb[j * T * 64] = y[j];
#endif
            // The chain, with the pushed adjoints gbar_k[t] kept as h[t] = gbar_k[t] / (t + 1): the gradient takes them so, the push
            // to the parent, gbar_{k-1}[t + 1] = dX / (t + 1) gbar_k[t], is h'[t + 1] = dX / (t + 2) h[t], and the sum of what is
            // pushed is dX times the sum of h: three operations a pair instead of four.
            float h[N + 2], pushed;
            h[1] = 0.5f * g1;
#if R == 2
            h[2] = (1.0f / 6.0f) * g2;
            pushed = __builtin_fmaf(0.5f, g2, g1);
#else
            pushed = g1;
#endif
#pragma unroll
            for (int k = K; k >= 1; --k) {
                h[0] = Ac[k - 1];
                Ac[k - 1] += pushed;
                float gc = h[0] * ap[k - 1][1], sum = h[0];
#pragma unroll
                for (int t = 1; t <= N - k; ++t) {
                    gc = __builtin_fmaf(h[t], ap[k - 1][t + 1], gc);
                    sum += h[t];
                }
                pushed = ec[k - 1][0] * sum;
                if (k > 1) {
#pragma unroll
                    for (int t = N - k; t >= 0; --t) h[t + 1] = ec[k - 1][t + 1] * h[t];
                }
#if MSUM
                vb[k * 16 * VROW] = gc;
#else
                if (k <= NU) {
                    const int kk = k <= NU ? k : 0;
                    vb[chain_row(k) * T * 64] = my_run[kk] == 0 ? gc : 0.0f;
                    if (runs[kk] > 1) vb[(chain_row(k) + 1) * T * 64] = my_run[kk] == 1 ? gc : 0.0f;
                    if (runs[kk] > 2) vb[(chain_row(k) + 2) * T * 64] = my_run[kk] == 2 ? gc : 0.0f;
                } else {
                    vb[chain_row(k) * T * 64] = gc;
                }
#endif
            }
          }
        }
#if MSUM
        // columns of segments past the end hold leftovers, each in its own column of the result, and are dropped
        wave_lds_fence();
        f4 sum[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int k = 0; k <= K; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f4 v = *(const f4*)(Vb + (k * 16 + col) * VROW + grp * 16 + 4 * q);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sum[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(k == 0 ? leaf_rows[4 * q + i] : chain_rows[k > 0 ? k - 1 : 0][4 * q + i],
                                                                      v[i], sum[i & 1], 0, 0, 0);
            }
        const long sg = n * T + col;
        sum[0] += sum[1];
        // The indicators multiply every lane's value, so a NaN or an infinity from one word would reach all letters.  It shows
        // in the sums; they are then formed anew from the values of each letter's own lanes.
        float zero = 0.0f;                                     // NaN as soon as one of the four is not finite
#pragma unroll
        for (int r = 0; r < 4; ++r) zero = __builtin_fmaf(sum[0][r], 0.0f, zero);
        if (__builtin_amdgcn_ballot_w64(sg < L && !(zero == 0.0f)) != 0) letter_sums(Vb + col * VROW, gr + level_start(N), p0, grp * 4, sum[0]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float acc = sg < L ? sum[0][r] : 0.0f;
            // the next segment's in the lane to the right; lane 15 of a row receives lane 0's, kept for the next tile
            const float next = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(acc), 0x12f, 0xf, 0xf, true));   // row_ror:15
            const int j = grp * 4 + r;
            if (j < D && sg < L)
                __hip_atomic_fetch_add(gp_row + (sg + 1) * D + j, acc - (col == 15 ? later[r] : next), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            if (n == 0 && col == 0 && j < D)
                __hip_atomic_fetch_add(gp_row + j, -acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            later[r] = next;
        }
#else
        wave_lds_fence();
        const int j = lane / T, t = lane % T;
        const long sg = n * T + t;
#if ONE_BY_ONE
        float acc = 0.0f;
        if (lane < T * D) acc = row_sum(Vb + lane * 64, lane);
#pragma unroll
        for (int base = 0; base < 3 * NU * T; base += 64) {
            const int o = base + lane;
            if (o < 3 * NU * T) Wide[o] = row_sum(Vb + (D * T + o) * 64, lane);
        }
        int jr = j;
        asm volatile("" : "+v"(jr));                           // keeps what follows from it inside the loop
#else
        // rows of both kinds are summed together, from clamped addresses: their reads overlap
        float acc = row_sum(Vb + (lane < T * D ? lane : 0) * 64, lane);
#pragma unroll
        for (int base = 0; base < 3 * NU * T; base += 64) {
            const int o = base + lane;                                    // row D + o / T: position o / T / 3 + 1, run o / T % 3
            const bool in = o < 3 * NU * T;
            const float sum = row_sum(Vb + (in ? D * T + o : 0) * 64, lane);
            if (in) Wide[o] = sum;                                        // rows of runs that do not reach here are not read below
        }
        int jr = j;
#if TWO_A_SIMD
        asm volatile("" : "+v"(jr));
#endif
#endif
        if (NU > 0) wave_lds_fence();
        // (for two letters segments past the end are summed too: behind a condition that changes from tile to tile the reads took
        // 78 registers more; depth 8, two wavefronts per SIMD 110 -> 96 us.  Three letters and more are faster with it.)
        if (lane < T * D && ((D == 2 && !ONE_BY_ONE) || sg < L)) {
            // chain position k with runs of s < 32 lanes: the lanes whose k-th letter is j, s of them every s D
#pragma unroll
            for (int k = NU + 1; k <= K; ++k) {
                const int s = ipow(D, K - k), period = s * D;
                const float* V = Vb + (chain_row(k) * T + t) * 64;
                const int rs0 = (p0 / period) * period + jr * s - p0;     // first run that can reach this wavefront
#pragma unroll
                for (int r = 0; r < (64 + period - 1) / period + 1; ++r)
#pragma unroll
                    for (int u = 0; u < s; ++u) {
                        const int q = rs0 + r * period + u;
                        const bool in = q >= 0 && q < 64;
                        const float v = V[in ? q : 0];
                        acc += in ? v : 0.0f;
                    }
            }
#pragma unroll
            for (int k = 1; k <= NU; ++k) {
                const int q = (j - first_letter[k] + D) % D;             // the run whose letter is j
                if (q < runs[k]) acc += Wide[(3 * (k - 1) + q) * T + t];
            }
        }
        if (sg >= L) acc = 0.0f;
        const float next = __shfl_down(acc, 1);
        if (lane < T * D && sg < L)
            __hip_atomic_fetch_add(gp_row + (sg + 1) * D + j, acc - (t == T - 1 ? later : next), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        later = __shfl(acc, j * T);
        if (n == 0 && lane < T * D && t == 0)
            __hip_atomic_fetch_add(gp_row + j, -acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#endif
        wave_lds_fence();                                      // the rows are rewritten by the next tile
      }
    }
}
#endif
)SRC";

// Time chunks (Chen's relation, eq. (2)): products of the chunk signatures S_0 .. S_{C-1} of a path, and the adjoints
// at the chunk boundaries, for any alphabet size.
const char* const kLanesChunkSource = R"SRC(
constexpr int ipow(int b, int e)
{
    int r = 1;
    for (int q = 0; q < e; ++q) r *= b;
    return r;
}
// first canonical index of the words of length n >= 1 (= how many are shorter), and the same inside a slice, which has
// D^(n - 1) words of length n
constexpr int level_start(int n)
{
    int r = 0;
    for (int m = 1; m < n; ++m) r += ipow(D, m);
    return r;
}
constexpr int slice_start(int n)
{
    int r = 0;
    for (int m = 1; m < n; ++m) r += ipow(D, m - 1);
    return r;
}

#if PART < 2
// Products over words of length <= M.  A workgroup keeps one slice of the running product for one path: the words with
// first letter i of S_0 S_1 .. S_c, whose factors on the left stay inside the slice, or with last letter i of
// S_c .. S_{C-1}, whose factors on the right do.  So the D slices (and both directions) advance side by side and only
// the words shorter than M of the next chunk signature are shared, staged in LDS.  The words of length M are never read
// again and live in registers.  Bound by the latency of one chunk after the other (two barriers each; the loads of the
// next chunk are in flight meanwhile).
// PART 0: from the left, the full product to `left` [B][level_start(M + 1)].
// PART 1: both directions, every product: left [B][C - 1] receives S_0 .. S_c, right [B][C - 1] S_{c+1} .. S_{C-1}.
#define NS level_start(M)                   /* words shorter than M */
#define NTOP ipow(D, M - 1)                 /* words of length M in a slice */
#define QS ((NS + NT - 1) / NT)
#define QT ((NTOP + NT - 1) / NT)
#define ROW level_start(M + 1)

// word e of length n of slice i
__device__ __forceinline__ int word_of(bool from_left, int i, int n, int e)
{
    return level_start(n) + (from_left ? i * ipow(D, n - 1) + e : e * D + i);
}
// sum over the cuts of word e of length n of the slice, x the slice's lower levels and s the next chunk's
template <int n>
__device__ __forceinline__ float cuts(bool from_left, const float* x, const float* s, int e)
{
    float acc = 0.0f;
    const unsigned u = (unsigned)e;
    if (from_left) {
#pragma unroll
        for (int m = 1; m < n; ++m)
            acc = __builtin_fmaf(x[slice_start(m) + u / (unsigned)ipow(D, n - m)], s[level_start(n - m) + u % (unsigned)ipow(D, n - m)], acc);
    } else {
#pragma unroll
        for (int m = 1; m < n; ++m)
            acc = __builtin_fmaf(s[level_start(m) + u / (unsigned)ipow(D, n - 1 - m)],
                                 x[slice_start(n - m) + u % (unsigned)ipow(D, n - m - 1)], acc);
    }
    return acc;
}
// the words of length n <= M - 1: y = x times the next chunk, stored to out where the product is asked for
template <int n>
__device__ __forceinline__ void lower_level(bool from_left, int i, const float* x, const float* s, float* y, float* __restrict__ out)
{
    if constexpr (n < M) {
        for (int e = threadIdx.x; e < ipow(D, n - 1); e += NT) {
            const int w = word_of(from_left, i, n, e);
            const float v = x[slice_start(n) + e] + s[w] + cuts<n>(from_left, x, s, e);
            y[slice_start(n) + e] = v;
            if (out) out[w] = v;
        }
        lower_level<n + 1>(from_left, i, x, s, y, out);
    }
}

extern "C" __global__ __launch_bounds__(NT) void sig_scan_lanes(const float* __restrict__ chunk_sigs, long C, float* __restrict__ left,
                                                                float* __restrict__ right)
{
    __shared__ float s[NS > 0 ? NS : 1], x[2][M > 1 ? slice_start(M) : 1];
    const int tid = threadIdx.x;
#if PART == 0
    const bool from_left = true;
    const int i = blockIdx.x % D;
    const long b = blockIdx.x / D;
#else
    const bool from_left = blockIdx.x % 2 == 0;
    const int i = blockIdx.x / 2 % D;
    const long b = blockIdx.x / (2 * D);
#endif
    const float* rows = chunk_sigs + b * C * ROW;
    const int n_chunks = (int)(PART == 0 ? C : C - 1);          // PART 1 needs no product over all chunks
    // chunk number and output row of step n: forwards from the first chunk, or backwards from the last
    const long c0 = from_left ? 0 : C - 1;
    const long dc = from_left ? 1 : -1;
    float top[QT], next_top[QT], next_s[QS > 0 ? QS : 1];
    {
        const float* S0 = rows + c0 * ROW;
        float* out = PART == 0 ? nullptr : (from_left ? left + b * (C - 1) * ROW : right + (b * (C - 1) + C - 2) * ROW);
#pragma unroll
        for (int n = 1; n < M; ++n)
            for (int e = tid; e < ipow(D, n - 1); e += NT) {
                const int w = word_of(from_left, i, n, e);
                const float v = S0[w];
                x[0][slice_start(n) + e] = v;
                if (out) out[w] = v;
            }
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const int e = tid + q * NT;
            top[q] = 0.0f;
            if (e < NTOP) {
                const int w = word_of(from_left, i, M, e);
                top[q] = S0[w];
                if (out) out[w] = top[q];
            }
        }
    }
    auto fetch = [&](long c) {
        const float* S = rows + c * ROW;
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            next_s[q] = S[e < NS ? e : 0];
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const int e = tid + q * NT;
            next_top[q] = S[word_of(from_left, i, M, e < NTOP ? e : NTOP - 1)];
        }
    };
    if (n_chunks > 1) fetch(c0 + dc);
    for (int n = 1; n < n_chunks; ++n) {
        float mine[QT];
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            if (e < NS) s[e] = next_s[q];
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) mine[q] = next_top[q];
        __syncthreads();
        fetch(c0 + dc * (n + 1 < n_chunks ? n + 1 : n));
        float* out = PART == 0 ? nullptr : (from_left ? left + (b * (C - 1) + n) * ROW : right + (b * (C - 1) + C - 2 - n) * ROW);
        const float* xo = x[(n - 1) & 1];
        lower_level<1>(from_left, i, xo, s, x[n & 1], out);
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const int e = tid + q * NT;
            if (e < NTOP) {
                top[q] += mine[q] + cuts<M>(from_left, xo, s, e);
                if (out) out[word_of(from_left, i, M, e)] = top[q];
            }
        }
        __syncthreads();
    }
#if PART == 0
    if (n_chunks == 1) __syncthreads();
    const float* xo = x[(n_chunks - 1) & 1];
    float* out = left + b * ROW;
#pragma unroll
    for (int n = 1; n < M; ++n)
        for (int e = tid; e < ipow(D, n - 1); e += NT) out[word_of(true, i, n, e)] = xo[slice_start(n) + e];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int e = tid + q * NT;
        if (e < NTOP) out[word_of(true, i, M, e)] = top[q];
    }
#endif
}
#elif PART == 3
// Depth 2: the chunk signatures over the words shorter than the depth are the chunks' displacements (a wavefront per row).
extern "C" __global__ __launch_bounds__(256) void sig_low_lanes(const float* __restrict__ path, long B, long P, float* __restrict__ coeffs,
                                                                const long* __restrict__, long KW, long max_len,
                                                                float* __restrict__ zero, long n_zero)
{
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n_zero; e += (long)gridDim.x * 256) zero[e] = 0.0f;
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= B * KW || lane >= D) return;
    const long b = row / KW, first = (row - b * KW) * max_len;
    const long last = first + max_len < P - 1 ? first + max_len : P - 1;
    coeffs[row * D + lane] = path[(b * P + last) * D + lane] - path[(b * P + first) * D + lane];
}
#else
// Adjoint at the boundary after chunk c: Abar(u) = grad(u) + sum_v grad(u v) Q_c(v) for the words u shorter than N
// (Proposition 4.1 with the right factor Q_c = S_{c+1} .. S_{C-1}).  A workgroup takes one boundary of one path and the
// words with one first letter: D^(N-1) products for every length of u, so each length gets as many lanes per word as
// the workgroup has (all of it for the single word of length 1).  Q_c sits in LDS; the gradient row comes from L2.
// On the way the workgroups clear n_zero floats at `zero` for the kernel that runs next.
#define NLOW level_start(N)
template <int n>
__device__ __forceinline__ void length_n(int i, const float* __restrict__ g, const float* q, float* __restrict__ out, float* part)
{
    if constexpr (n < N) {
        constexpr int U = ipow(D, n - 1);
        constexpr int each = NT / U;
        constexpr int G = U == 1 || each >= 64 ? 64 : (each >= 32 ? 32 : (each >= 16 ? 16 : (each >= 8 ? 8 : (each >= 4 ? 4 : (each >= 2 ? 2 : 1)))));
        constexpr int stride = U == 1 ? NT : G;                // lanes that share a word
        const int lane = U == 1 ? threadIdx.x : threadIdx.x % G;
        for (int u0 = 0; u0 < U; u0 += NT / stride) {
            const int e = u0 + (U == 1 ? 0 : threadIdx.x / G);
            float acc = 0.0f;
            if (e < U) {
                const int u = i * U + e;
#pragma unroll
                for (int m = 1; m <= N - n; ++m) {
                    const float* gb = g + level_start(n + m) + u * ipow(D, m);
#pragma unroll 4
                    for (int v = lane; v < ipow(D, m); v += stride) acc = __builtin_fmaf(gb[v], q[level_start(m) + v], acc);
                }
            }
#pragma unroll
            for (int w = 1; w < G; w *= 2) acc += __shfl_xor(acc, w);
            if (U == 1) {
                if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = acc;
            } else if (e < U && lane == 0) {
                const int w = level_start(n) + i * U + e;
                out[w] = g[w] + acc;
            }
        }
        length_n<n + 1>(i, g, q, out, part);
    }
}

extern "C" __global__ __launch_bounds__(NT) void sig_adjoint_lanes(const float* __restrict__ grad, const float* __restrict__ after, long C1,
                                                                   float* __restrict__ abar, float* __restrict__ zero, long n_zero)
{
    __shared__ float q[NLOW], part[NT / 64];
    const long bc = blockIdx.x / D;
    const int i = blockIdx.x % D;
    const float* Q = after + bc * NLOW;
    const float* g = grad + bc / C1 * (long)level_start(N + 1);
    float* out = abar + bc * NLOW;
    for (int e = threadIdx.x; e < NLOW; e += NT) q[e] = Q[e];
    for (long e = (long)blockIdx.x * NT + threadIdx.x; e < n_zero; e += (long)gridDim.x * NT) zero[e] = 0.0f;
    __syncthreads();
    length_n<1>(i, g, q, out, part);
    __syncthreads();
    if (threadIdx.x == 0) {
        float acc = g[i];
        for (int w = 0; w < NT / 64; ++w) acc += part[w];
        out[i] = acc;
    }
}
#endif
)SRC";

}  // namespace

namespace {
int64_t words_up_to(int d, int n)
{
    int64_t r = 0, p = 1;
    for (int m = 1; m <= n; ++m) { p *= d; r += p; }
    return r;
}
}  // namespace

namespace {
// Modelled time of a forward segment in microseconds, `waves` wavefronts to a SIMD: the latency of the chain and the issue of a
// lone wavefront's instructions (and, where the halves of a word's children begin at an odd place, their increments read one by
// one: 5, 6 and 10 letters 0.03 us).  A second wavefront fills the gaps of the first: 1.4 times the time, not twice, and 0.7 for each
// from there on (8 letters, depth 4, one level: 0.070 us a segment alone, 0.109 with two, 0.202 with four).
double forward_segment(const LanesShape& s, int d, double waves)
{
    const bool odd = s.split > 1 && (d + 1) / 2 % 2 != 0;
    const double lone = 0.0013 * s.chain + 0.005 + (s.R == 1 ? 0.0019 : 0.0021) * s.per_lane + (odd ? 0.033 : 0.0);
    return waves <= 1.0 ? lone : lone * std::max(1.4, 0.7 * waves);
}
}  // namespace

LanesShape lanes_shape(int d, int depth, bool backward, int64_t B, int levels)
{
    LanesShape best{};
    if (d < 2 || d > 64 || depth < 2 || depth > 12) return best;
    const int NC = (depth + 3) / 4 * 4, DP = (d + 3) / 4 * 4;
    double best_cost = 0.0;
    // Two levels per lane while their state fits the registers (forward d + d^2 values, backward twice that and the
    // per-letter sums).  Between the admissible forms: the time of a segment is the instructions of a lane times the
    // wavefronts a SIMD has to run one after the other (1,024 SIMDs); two levels per lane share more work between
    // words but leave few wavefronts for small batches, where one level per lane then has the shorter segment.
    // (forms: one level, two levels, and forward two levels with the children of a word halved between two wavefronts)
    for (int form = 1; form <= (backward ? 2 : 3); ++form) {
        const int R = form == 1 ? 1 : 2, split = form == 3 ? 2 : 1;
        if (levels != 0 && R != levels) continue;
        if (depth - R < 1) continue;
        if (R == 2 && d > 12) continue;
        LanesShape s{};
        s.R = R;
        s.split = split;
        s.T = 64 / d < 8 ? 64 / d : 8;
        const int K = depth - R;
        double lanes = 1.0;
        for (int k = 0; k < K; ++k) lanes *= d;
        if (lanes > 1.0e9) continue;
        s.lanes = (int64_t)lanes;
        if (split > 1 && s.lanes < 32) continue;           // small sets keep the kernels they have
        s.waves = (s.lanes + 63) / 64 * split;
        int chain = 0, wide = 0;
        double run = lanes;
        for (int k = 1; k <= K; ++k) {
            chain += depth - k + 1;
            run /= d;                                      // d^(K - k)
            wide += run >= 32.0 ? 1 : 0;
        }
        const double per_lane = 2.0 * chain + (R == 2 ? ((double)d * d + 3.0 * d) / split : 2.0 * d);
        s.chain = chain;
        s.per_lane = per_lane;
        const double rounds = (double)std::max<int64_t>(B, 1) * (double)s.waves / 1024.0;
        const double cost = backward ? per_lane * (rounds < 1.0 ? 1.0 : rounds) : forward_segment(s, d, rounds);
        if (best.ok && cost >= best_cost) continue;            // (every call asks, several times)
        // LDS of a wavefront: the increments of a staging tile and, backward, the gradient rows of the segments of a
        // tile; eight wavefronts of 20 KB fit a compute unit, so longer tiles are cut down to that.  The staging
        // tile is as many tiles as fit (up to 32 segments and three increments per lane): its global loads are issued
        // one staging tile ahead.
        // gradient sums as matrix products, tiles of 16 segments: 4.4 KB of LDS for every source.  Two letters and depth 7 and
        // more are then left with one wavefront per SIMD, so batches of more than that sum rows (depth 7, 100 segments: 1,024
        // paths 57 us as products, 72 as rows; 2,048 111 and 85; 8,192 434 and 366)
        const bool msum = backward && R == 1 && d <= 16 && !(d == 2 && K >= 6 && rounds > 1.0);
        s.msum = msum;
        auto lds_bytes = [&](int T, int TS) {
            const size_t tile = (size_t)TS * ((size_t)d * NC + (size_t)DP);
            if (msum) return (tile + (size_t)(K + 1) * 16 * 68) * sizeof(float);
            return (tile + (backward ? (size_t)(d + K + 2 * wide) * T * 64 + (size_t)((3 * wide * T + 3) / 4 * 4) : 0)) * sizeof(float);
        };
        // (a lane carries its share of the next staging tile in registers: one increment where the state of two
        // levels already fills them)
        const int staged = (R == 2 && (d + split - 1) / split * (d + 1) > 48) ? 64 : 192;
        if (msum) {
            s.T = s.TS = 16;
        } else if (backward) {
            while (s.T > 1 && lds_bytes(s.T, s.T) > 20 * 1024) --s.T;
            s.TS = s.T;
            while (s.TS + s.T <= 32 && (s.TS + s.T) * d <= staged && lds_bytes(s.T, s.TS + s.T) <= 20 * 1024) s.TS += s.T;
        } else {
            s.T = 1;                                       // no gradient tiles: only the staging tile matters
            s.TS = 32;
            while (s.TS > 2 && (s.TS * d > staged || s.TS % (R == 1 && s.TS > 4 ? 4 : 2) != 0 || lds_bytes(1, s.TS) > 8 * 1024)) --s.TS;
            if (s.TS * d > 64 && s.TS * d > staged) s.TS = 1;
        }
        const size_t per_wave = lds_bytes(s.T, s.TS);
        s.shares = backward && words_up_to(d, depth - 1) * sizeof(float) <= per_wave;
        s.nwb = (int)(per_wave * 4 <= 64 * 1024 ? 4 : (per_wave * 2 <= 64 * 1024 ? 2 : (per_wave <= 64 * 1024 ? 1 : 0)));
        s.ok = s.nwb > 0;
        if (s.ok) s.fit = std::max(1.0, std::floor(160.0 * 1024.0 / ((double)per_wave * s.nwb))) * s.nwb / 4.0;
        if (s.ok) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

namespace {
// words of length `top` that a slice holds, over the threads of a workgroup
int scan_threads(int64_t n_top) { return n_top <= 2048 ? 256 : (n_top <= 8192 ? 512 : 1024); }
}  // namespace

// The products over all words need the words shorter than the depth of one chunk and two copies of a slice in the
// 64 KB of LDS a kernel may declare, and the words of full length of a slice in registers (at most 16 a thread).
bool lanes_chunks_available(int d, int depth)
{
    if (d < 2 || d > 64 || depth < 2 || depth > 12) return false;
    double top = 1.0;
    for (int k = 1; k < depth; ++k) top *= d;
    if (top > 16.0 * 1024.0) return false;
    return (words_up_to(d, depth - 1) + 2 * (words_up_to(d, depth - 2) + 1)) * 4 <= 62 * 1024;
}

// Times in microseconds, fitted to a scan of 33 shapes (2..40 letters, depth 2..9, 1..512 paths of 17..500 segments, every form and
// count: 1,828 calls each way); the choice of form and count costs 1.7 % over the best forward and 1 % backward on average.  A
// segment takes the latency of a lane's chain and the issue of its instructions, as often as wavefronts share a SIMD, in as many
// rounds as the chip holds the wavefronts; chunks cost their launches, a product per chunk and the traffic of the chunk signatures
// forward, and backward what a wavefront needs to pass the chunk signatures.  Whole paths -> the choice: forward 37 x 301
// segments, d = 7, depth 4: 29.5 -> 15.1 us, 8 x 1,000, d = 3, depth 5: 83.5 -> 17.6; backward 67.5 -> 27.9 and 294 -> 26.2.
int lanes_chunk_count(int d, int depth, bool backward, int64_t B, int64_t L, int levels)
{
    const double words = (double)words_up_to(d, depth), low_words = (double)words_up_to(d, depth - 1), k = words / 1000.0;
    const double low_waves = (double)lanes_low_shape(d, depth).waves;
    const double low_exponent = backward ? 0.4 : 0.07, scan_exponent = backward ? -0.12 : 0.21;
    // two more launches backward: at least their host time
    const double launches = backward ? std::max(5.0, 4.1 * std::pow(k, low_exponent)) : 3.0 * std::pow(k, low_exponent);
    const double product = (backward ? 0.78 : 0.48) * std::pow(k, scan_exponent) + (backward ? 4.5e-6 : 1.9e-6) * (double)B * words;
    auto time = [&](int64_t C) {
        LanesShape s = lanes_shape(d, depth, backward, B * C, levels);
        if (!s.ok) s = lanes_shape(d, depth, backward, B * C, 0);
        const double waves = (double)(B * C) * (double)s.waves / 1024.0, Lc = (double)((L + C - 1) / C);
        if (!backward) {
            const double t = 3.7 + Lc * forward_segment(s, d, waves);
            return C == 1 ? t : t + launches + (double)C * product;
        }
        // Two wavefronts of 18 to 20 KB of LDS at a time, and those with sums as matrix products by the room that there is (16 letters,
        // whose factors fill the registers: one): 10 letters, depth 4, 1,000 lanes a path, 0.23 us a segment alone, 0.30 with one on
        // every SIMD, 0.63 with two.  Two levels of two or four letters have fewer rows to sum where the runs of equal letters fall into
        // rows of sixteen lanes (4 letters, depth 5, 64 lanes 0.38 us, 5 letters 0.76).
        double latency, issue, rounds = std::ceil(waves / 2.0);
        if (s.msum) {
            latency = 0.0034 * s.chain;
            issue = 0.008 + 0.0039 * (6.0 * (depth - s.R + 1) + (s.shares ? 2.0 * (s.chain + std::min(d, 10)) : s.per_lane));
            if (s.shares) rounds = std::max(rounds, std::ceil(waves / (d > 12 ? 1.0 : s.fit)));
        } else if (s.R == 1 && d == 2) {
            latency = 0.59;                                  // sums by rows: the chip is full, more rows gain nothing
            issue = 0.13;
            if (C > 1) return 1.0e9;
        } else if (s.R == 1) {
            latency = 1.1;
            issue = 0.0002 * s.per_lane;
        } else {
            const double rows = s.shares && (d == 2 || d == 4) && s.lanes <= 64 ? 0.55 : 1.0;
            latency = rows * (0.206 + 0.023 * s.chain);
            issue = rows * (0.132 + 0.0018 * s.per_lane);
        }
        // The sums of a tile take the same however few segments it has, counted here against the average tile (as products a third of a full
        // tile's time, but a fifth fits the calls; paths of under 32 segments are too short to choose between tiles).
        const double share = L < 32 ? 0.0 : (s.msum ? 0.2 : (s.R == 2 ? 0.25 : 1.0)), pad = std::ceil(Lc / s.T) * s.T - Lc;
        const double t = 8.5 + (Lc + share * (pad - 0.3 * (s.T - 1))) * rounds * (latency + issue * std::max(1.0, waves / rounds));
        if (C == 1) return t;
        const double low = 0.08 * Lc * std::max(1.0, (double)(B * C) * low_waves / 2048.0);
        if (!s.shares) return t + launches + (double)C * product + low;
        // without arrays at the boundaries: one launch in place of the clearing one, and every wavefront passes the chunk signatures.
        // Not on paths of a few segments once wavefronts share SIMDs: what they read first takes longer than the segments saved.  Two
        // levels, which read more, only up to a wavefront on each SIMD, if a path has several (one sums its tile cheaply) over three to
        // nine letters (two: the sums of a tile take the same time however few its segments are).  128 to 512 paths, whole -> two
        // chunks: 5 letters, depth 5, x 17 segments 27 -> 24 us, 9 letters, depth 4 26 -> 23, but 4 letters, depth 5, x 24 17 -> 21,
        // 10 letters, depth 4, x 17 23 -> 27.  (Two letters, depth 9, 128 x 24 stay whole because a host test fixes that: 23 us, 20 in two chunks
        // since four wavefronts' sums fit a compute unit.)
        const bool few = s.R == 1 ? waves < (d == 2 ? 1.0 : 1.5) : waves < 0.75 || (waves <= 1.0 && s.lanes > 64 && d > 2 && d < 10);
        if (L < 32 && !few) return 1.0e9;
        const double terms = (double)(depth - s.R) * (s.R == 1 ? 0.002 * d : (d > 10 ? 0.006 : 0.0035) * (d + (double)d * d));
        return t + 1.0 + (double)C * rounds * (0.2 + 0.0004 * low_words + terms) + low;
    };
    double best = 0.93 * time(1);
    int choice = 1;
    auto consider = [&](int64_t C) {
        const double t = time(C);
        if (t < best) {
            best = t;
            choice = (int)C;
        }
    };
    for (int C : kLanesChunkCounts) {
        if (L < 8 * (int64_t)C) break;                        // chunks of at least 8 segments
        consider(C);
        if (!backward || L < 32) continue;
        // and the count near it whose chunks are whole tiles.  Backward calls, with that and partial tiles of two levels: 1 path x 199
        // segments, 10 letters, depth 4, 13 chunks of one tile of 16 instead of 12 of two, 20.4 -> 18.7 us; 32 x 99, 6 letters, depth 5,
        // 35.1 -> 28.9; 186 x 160, 3 letters, depth 5, 29.8 -> 24.9; 47 shapes 0.95 on geometric average, the slowest 1.01
        LanesShape s = lanes_shape(d, depth, true, B * C, levels);
        if (!s.ok) s = lanes_shape(d, depth, true, B * C, 0);
        const int64_t tiles = std::max<int64_t>(1, (L / C + s.T / 2) / s.T), whole = (L + tiles * s.T - 1) / (tiles * s.T);
        if (whole >= 2 && whole <= 32 && L >= 8 * whole) consider(whole);
    }
    return choice;
}

int lanes_chunk_threads(int d, int depth, LanesChunkPart part)
{
    int64_t top = 1;                                          // words of the longest length in a slice
    for (int k = 1; k < (part == kLanesScanLow ? depth - 1 : depth); ++k) top *= d;
    return scan_threads(top);
}

// One shape for every batch: the words shorter than the depth are a d-th of the work.
LanesShape lanes_low_shape(int d, int depth)
{
    if (depth > 2) return lanes_shape(d, depth - 1, false, 256, 0);
    LanesShape s{};
    s.ok = true;
    s.lanes = d;
    s.waves = 1;
    s.nwb = 4;
    return s;
}

// The kernels of a module share their text, with other shapes: a namespace each, the shape macros set anew in front of it.
std::string lanes_source(int d, int depth, const LanesShape& s, bool backward, bool arrays)
{
    std::ostringstream o;
    auto lanes = [&](const char* ns, int n, const LanesShape& q, bool bwd, const char* forward_name) {
        o << "#define N " << n << "\n#define R " << q.R << "\n#define SP " << q.split << "\n#define T " << q.T << "\n#define TS " << q.TS
          << "\n#define NWB " << q.nwb << "\n#define BACKWARD " << (bwd ? 1 : 0) << "\n#define MSUM " << (bwd && q.msum ? 1 : 0)
          << "\n#define FORWARD_NAME " << forward_name << "\n#define CLEARS " << (backward ? 1 : 0) << "\nnamespace " << ns << " {\n"
          << kLanesSource << "}\n#undef N\n#undef R\n#undef SP\n#undef T\n#undef TS\n#undef NWB\n#undef BACKWARD\n#undef MSUM\n"
          << "#undef FORWARD_NAME\n#undef CLEARS\n";
    };
    auto chunk = [&](const char* ns, LanesChunkPart part) {
        o << "#define N " << depth << "\n#define M " << (part == kLanesScanLow ? depth - 1 : depth)
          << "\n#define NT " << lanes_chunk_threads(d, depth, part) << "\n#define PART " << (int)part << "\nnamespace " << ns << " {\n"
          << kLanesChunkSource << "}\n#undef N\n#undef M\n#undef NT\n#undef PART\n";
    };
    o << "#define D " << d << "\n";
    lanes("rows", depth, s, backward, "sig_fwd_lanes");
    if (lanes_chunks_available(d, depth)) {
        if (!backward) {
            chunk("scan", kLanesScanFull);
        } else {
            if (depth > 2) lanes("low", depth - 1, lanes_low_shape(d, depth), false, "sig_low_lanes");
            else chunk("low", kLanesDisplacement);
            if (arrays) {
                chunk("scan", kLanesScanLow);
                chunk("adjoint", kLanesAdjoint);
            }
        }
    }
    return o.str();
}

}  // namespace sig
