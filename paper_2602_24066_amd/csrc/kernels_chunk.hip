// Time chunks for full truncations.
//
// Chen's relation (Section 3, eq. 2) is associative, so a path may be cut into C consecutive chunks whose
// signatures S_1 .. S_C are computed independently (C times as many wavefronts for the sequential kernels) and
// multiplied afterwards:  S_{0,T} = S_1 (x) S_2 (x) .. (x) S_C,  where in the word basis
//     (a (x) b)(w) = sum_{k=0..n} a(w_1..w_k) b(w_{k+1}..w_n),   a(empty) = b(empty) = 1        (Section 2.1).
// The backward pass of chunk c needs the signature up to the end of the chunk, P_c = S_1 (x) .. (x) S_c, and the
// adjoint there, Abar_c(u) = sum_v grad(u v) Q_c(v) with Q_c = S_{c+1} (x) .. (x) S_C the signature of the rest
// of the path (Proposition 4.1 with the right factor taken at a chunk boundary).
//
// All arrays are [B][C][W] floats (W = d + d^2 + .. + d^N coefficients, levels concatenated, each row-major);
// d is a power of two so that prefixes and suffixes of a word index are shifts and masks.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace sig {
namespace {

struct Levels {
    int N;            // depth
    int lb;           // log2(d), >= 2
    int W;            // coefficients (a multiple of 4)
    int ls[14];       // ls[n] = index of the first word of length n, n = 1..N (multiples of 4); ls[N + 1] = W
};

typedef float f4 __attribute__((ext_vector_type(4)));

// Four consecutive coefficients (word length n, indices i .. i + 3 inside the level, i a multiple of 4) of a (x) b.
// The four words differ in their last letter only, so every prefix is shared and the suffixes are contiguous.
__device__ __forceinline__ f4 quad_product(const float* a, const float* b, const Levels& g, int n, int i)
{
    f4 acc = *(const f4*)(a + g.ls[n] + i) + *(const f4*)(b + g.ls[n] + i);
    for (int k = 1; k < n; ++k) {
        const int sh = g.lb * (n - k);
        const float av = a[g.ls[k] + (i >> sh)];
        const f4 bv = *(const f4*)(b + g.ls[n - k] + (i & ((1 << sh) - 1)));
        acc += av * bv;
    }
    return acc;
}

// out = a (x) b by the whole workgroup; out2 (may be null) receives a second copy.  Level by level, so that the
// level offsets and shifts are uniform.
__device__ __forceinline__ void tensor_product(const float* a, const float* b, float* out, float* out2, const Levels& g)
{
    for (int n = 1; n <= g.N; ++n) {
        const int quads = (g.ls[n + 1] - g.ls[n]) >> 2;
        for (int qd = threadIdx.x; qd < quads; qd += blockDim.x) {
            const f4 r = quad_product(a, b, g, n, 4 * qd);
            *(f4*)(out + g.ls[n] + 4 * qd) = r;
            if (out2) *(f4*)(out2 + g.ls[n] + 4 * qd) = r;
        }
    }
}

__device__ __forceinline__ void copy_row(const float* src, float* dst, int W)
{
    for (int o = 4 * threadIdx.x; o < W; o += 4 * blockDim.x) *(f4*)(dst + o) = *(const f4*)(src + o);
}

// out(u) = gr(u) + sum_{m >= 1} sum_{|v| = m} gr(u v) q(v) for every word u, by the whole workgroup.  The words of
// one length k are spread over the workgroup, with blockDim / d^k threads (at most 64, at least 1) sharing the
// inner sums of a word; for a fixed m the terms of a word are contiguous in gr and in q.
__device__ __forceinline__ void adjoint_contract(const float* gr, const float* q, float* __restrict__ out, const Levels& g)
{
    const int N = g.N;
    copy_row(gr + g.ls[N], out + g.ls[N], g.W - g.ls[N]);               // words of length N
    for (int k = 1; k < N; ++k) {
        const int nk = g.ls[k + 1] - g.ls[k];                           // words of length k
        int tpw = (int)blockDim.x / nk;                                 // threads per word (power of two)
        tpw = tpw > 64 ? 64 : (tpw < 1 ? 1 : tpw);
        const int wpp = (int)blockDim.x / tpw;                          // words per pass
        const int t = threadIdx.x % tpw;
        for (int i0 = 0; i0 < nk; i0 += wpp) {
            const int i = i0 + threadIdx.x / tpw;
            float acc = 0.0f;
            if (i < nk)
                for (int m = 1; m <= N - k; ++m) {
                    const int cnt = 1 << (g.lb * m);
                    const float* src = gr + g.ls[k + m] + (i << (g.lb * m));
                    const float* qv = q + g.ls[m];
                    for (int v = t; v < cnt; v += tpw) acc = fmaf(src[v], qv[v], acc);
                }
            for (int off = tpw >> 1; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
            if (i < nk && t == 0) out[g.ls[k] + i] = gr[g.ls[k] + i] + acc;
        }
    }
}

// Signatures that fit LDS three times, a workgroup per path: the running product and the next factor are staged in three
// rotating buffers of W floats.  Forward (Abar == nullptr): coeffs_out[b] = S_1 (x) .. (x) S_C.  Backward, two workgroups per
// path side by side: Pfx[c] = S_1 (x) .. (x) S_c for c < C and Pfx[C] = terminal[b] (the signature the caller kept); and, from
// the suffix products Q_c = S_{c+1} (x) .. (x) S_C, the adjoints at the chunk boundaries, Abar[c](u) = sum_v grad(u v) Q_c(v)
// (grad is read from global memory: consecutive threads read consecutive coefficients).
__global__ __launch_bounds__(1024) void chunk_scan_kernel(const float* __restrict__ Sc, float* Pfx, const float* __restrict__ terminal,
                                                          float* coeffs_out, const float* __restrict__ grad, float* Abar, int C, Levels g)
{
    extern __shared__ f4 smem4[];
    float* sm = (float*)smem4;
    const int64_t b = blockIdx.x;
    const int64_t W = g.W;
    const float* S = Sc + b * C * W;
    const bool bwd = Abar != nullptr;
    float* buf[3] = {sm, sm + W, sm + 2 * W};
    int cur = 0;
    if (blockIdx.y == 0) {
        float* P = bwd ? Pfx + b * C * W : nullptr;
        copy_row(S, buf[0], (int)W);
        if (bwd) copy_row(S, P, (int)W);
        const int lastp = bwd ? C - 2 : C - 1;
        for (int s = 1; s <= lastp; ++s) {
            const int nb = (cur + 1) % 3, no = (cur + 2) % 3;
            copy_row(S + (int64_t)s * W, buf[nb], (int)W);
            __syncthreads();
            float* dst = (!bwd && s == C - 1) ? coeffs_out + b * W : (bwd ? P + (int64_t)s * W : nullptr);
            tensor_product(buf[cur], buf[nb], buf[no], dst, g);
            cur = no;
            __syncthreads();
        }
        if (bwd) copy_row(terminal + b * W, P + (int64_t)(C - 1) * W, (int)W);
    } else {
        const float* const gb = grad + b * W;
        float* const Ab = Abar + b * C * W;
        copy_row(gb, Ab + (int64_t)(C - 1) * W, (int)W);                // the last chunk's adjoint is grad
        copy_row(S + (int64_t)(C - 1) * W, buf[0], (int)W);
        __syncthreads();
        adjoint_contract(gb, buf[0], Ab + (int64_t)(C - 2) * W, g);
        for (int q = C - 3; q >= 0; --q) {
            const int nb = (cur + 1) % 3, no = (cur + 2) % 3;
            copy_row(S + (int64_t)(q + 1) * W, buf[nb], (int)W);
            __syncthreads();
            tensor_product(buf[nb], buf[cur], buf[no], nullptr, g);
            cur = no;
            __syncthreads();
            adjoint_contract(gb, buf[cur], Ab + (int64_t)q * W, g);
        }
    }
}

// ---- products by slices: a workgroup keeps one slice of the running product of a path.  The words with first letter i of
// S_0 S_1 .. S_c have their left factors inside the slice, those with last letter i of S_c .. S_{C-1} their right ones, so the D
// slices (and both directions) advance side by side, all chunks in one launch; only the shorter words of the next chunk
// signature are shared, staged in LDS a product ahead.  Bound by the latency of one product after the other (two barriers
// each).  A grid-wide launch per product instead cost 4.5-5 us each: 3 paths x 979 segments, d = 8, eight chunks, 35 us forward.
template <int B, int E> struct Ipow { static constexpr int v = B * Ipow<B, E - 1>::v; };
template <int B> struct Ipow<B, 0> { static constexpr int v = 1; };
template <int D, int n> struct LevelAt { static constexpr int v = LevelAt<D, n - 1>::v + Ipow<D, n - 1>::v; };    // words shorter than n
template <int D> struct LevelAt<D, 1> { static constexpr int v = 0; };
template <int D, int n> constexpr int kLevel = LevelAt<D, n>::v;
template <int D, int n> constexpr int kSlice = LevelAt<D, n>::v / D;                                          // the same inside a slice
template <int B, int E> constexpr int kPow = Ipow<B, E>::v;

// ---- two chunks: their product, and the boundary adjoints of large signatures.  Sizes are template constants: with the level table as
// a kernel argument every look into it was a load that the next instruction waited for.

template <int D, int n, int m>
__device__ __forceinline__ void product_cuts(const float* __restrict__ a, const float* __restrict__ b, unsigned i, f4& acc)
{
    if constexpr (m < n) {
        constexpr unsigned below = kPow<D, n - m>;
        acc += a[kLevel<D, m> + i / below] * *(const f4*)(b + kLevel<D, n - m> + i % below);
        product_cuts<D, n, m + 1>(a, b, i, acc);
    }
}
// coefficients o .. o + 3 (words of length n or more, one length: D is a multiple of four) of a (x) b
template <int D, int N, int n>
__device__ __forceinline__ f4 product_quad(const float* __restrict__ a, const float* __restrict__ b, unsigned o)
{
    if constexpr (n < N) {
        if (o >= (unsigned)kLevel<D, n + 1>) return product_quad<D, N, n + 1>(a, b, o);
    }
    f4 acc = *(const f4*)(a + o) + *(const f4*)(b + o);
    product_cuts<D, n, 1>(a, b, o - kLevel<D, n>, acc);
    return acc;
}
// out[b] = S[b][0] (x) S[b][1] for every path, spread over the whole grid: blockIdx.y = path, blockIdx.x covers the quads of all levels.
// Bound by memory: 128 paths, d = 8, depth 5 15.7 -> 12.6 us for 57 MB, 64 paths, d = 16, depth 4 13.4 -> 11.0.
template <int D, int N>
__global__ __launch_bounds__(256) void chunk_product_kernel(const float* __restrict__ S, float* __restrict__ out)
{
    constexpr int W = kLevel<D, N + 1>;
    const unsigned o = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (o >= (unsigned)W) return;
    const float* a = S + (int64_t)blockIdx.y * 2 * W;
    *(f4*)(out + (int64_t)blockIdx.y * W + o) = product_quad<D, N, 1>(a, a + W, o);
}

// Sum over groups of LANES consecutive lanes, in every lane of the group.
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int LANES>
__device__ __forceinline__ float group_sum(float v)
{
    if constexpr (LANES > 1) v += dpp<0xB1>(v);                          // lane ^ 1
    if constexpr (LANES > 2) v += dpp<0x4E>(v);                          // lane ^ 2
    if constexpr (LANES > 4) v += dpp<0x141>(v);                         // mirrored in eight lanes: the other four
    if constexpr (LANES > 8) v += dpp<0x140>(v);                         // mirrored in sixteen
    if constexpr (LANES > 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (LANES > 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

constexpr int kAdjointThreads = 512;
// sum over |v| = m .. N - k of grad(a u' v) Q(v), the share of thread t of the TPW threads of u = a u' (u' the iw-th word of length k - 1)
template <int D, int N, int k, int m>
__device__ __forceinline__ float adjoint_terms(const float* sg, const float* sq, unsigned iw, unsigned t, float acc)
{
    if constexpr (m <= N - k) {
        constexpr unsigned words = kPow<D, k - 1>, TPW = kAdjointThreads / words, CNT = kPow<D, m>;
        const float* src = sg + kLevel<D, k - 1 + m> + iw * CNT;
        const float* qv = sq + kLevel<D, m>;
        if constexpr (CNT > TPW) {
            // every word starts its sum at another place: the terms of neighbouring words lie a power of two apart, in the same banks
            const unsigned shift = ((iw * CNT >> 6) * TPW) & (CNT - 1);
#pragma unroll
            for (unsigned q = 0; q < CNT / TPW; ++q) {
                const unsigned r = (t + q * TPW + shift) & (CNT - 1);
                acc = fmaf(src[r], qv[r], acc);
            }
        } else {
            const unsigned r = t & (CNT - 1);
            const float term = src[r] * qv[r];
            acc += t < CNT ? term : 0.0f;
        }
        acc = adjoint_terms<D, N, k, m + 1>(sg, sq, iw, t, acc);
    }
    return acc;
}
template <int D, int N, int k>
__device__ __forceinline__ void adjoint_lengths(const float* sg, const float* sq, unsigned a, float* out)
{
    if constexpr (k < N) {
        constexpr unsigned words = kPow<D, k - 1>, TPW = kAdjointThreads / words;
        static_assert(words <= kAdjointThreads && TPW <= 64, "a word's threads lie in one wavefront");
        const unsigned iw = threadIdx.x / TPW, t = threadIdx.x % TPW;
        const float acc = group_sum<TPW>(adjoint_terms<D, N, k, 1>(sg, sq, iw, t, 0.0f));
        if (t == 0) out[kLevel<D, k> + a * words + iw] = sg[kLevel<D, k - 1> + iw] + acc;
        adjoint_lengths<D, N, k + 1>(sg, sq, a, out);
    }
}
// level of the words that o lies among (o < kLevel<D, N>), times what `grad` holds further on for the words with first letter a
template <int D, int N, int m>
__device__ __forceinline__ unsigned below_letter(unsigned o, unsigned a)
{
    if constexpr (m + 1 < N) {
        if (o >= (unsigned)kLevel<D, m + 1>) return below_letter<D, N, m + 1>(o, a);
    }
    return o - kLevel<D, m> + kLevel<D, m + 1> + a * (unsigned)kPow<D, m>;
}

// The boundary adjoints, one workgroup per (path, chunk but the last, first letter a): every word u that begins with a gets
// Abar(u) = grad(u) + sum_v grad(u v) Q(v).  The words u v all begin with a too, so workgroups share no output, and what a workgroup
// reads - the gradients of the words a v and Q(v) for |v| < N, 2 (d + .. + d^(N-1)) floats - is staged in LDS once: sg[level m + v] =
// grad(a v), sq[level m + v] = Q(v) for |v| = m.  All threads work on one word length at a time and split the sums of a word between 512 /
// (words of that length) of them (those of the letter itself add up through LDS), so that short words, whose sums run over thousands of
// terms, take as few rounds as long ones.  The adjoints of the words of length N are the gradient itself, in every chunk: the backward
// kernels read them there and their places in Abar stay unwritten.  On the way n_zero floats at `zero` (16-byte aligned) are cleared for
// those kernels.  Bound by the latency of its loads, the sums and the launch: two chunks, 128 paths, d = 8, depth 5 28 -> 7.2 us, 64 paths,
// d = 16, depth 4 22 -> 7.1 (before, with the level table as an argument, loops of unknown length and workgroups for last chunks).
template <int D, int N>
__global__ __launch_bounds__(kAdjointThreads) void chunk_adjoint_subtree_kernel(const float* __restrict__ grad, const float* __restrict__ Q,
                                                                                float* __restrict__ Abar, int C, float* __restrict__ zero,
                                                                                int64_t n_zero, int64_t row_words)
{
    constexpr unsigned below = kLevel<D, N>, NT = kAdjointThreads, PER = (below / 4 + NT - 1) / NT;
    static_assert(D % 4 == 0, "a quad's words have one length");
    __shared__ __attribute__((aligned(16))) float sq[below], sg[below];
    __shared__ float red[NT / 64];
    const unsigned tid = threadIdx.x, a = blockIdx.y;
    const int64_t b = blockIdx.x / (unsigned)(C - 1), row = b * C + (blockIdx.x - b * (C - 1));
    const float* gr = grad + b * kLevel<D, N + 1>;
    const float* q = Q + row * row_words;
    float* out = Abar + (int64_t)blockIdx.x * row_words;                 // [B][C - 1]: the last chunk has no row
    f4 vq[PER], vg[PER];
#pragma unroll
    for (unsigned r = 0; r < PER; ++r) {
        const unsigned o = 4 * (tid + r * NT) < below ? 4 * (tid + r * NT) : 0;
        vq[r] = *(const f4*)(q + o);
        vg[r] = *(const f4*)(gr + below_letter<D, N, 1>(o, a));
    }
    const float own = gr[a];
    {
        const int64_t step = (int64_t)gridDim.x * gridDim.y * NT;
        int64_t i = ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * NT + tid;
        if (i < (n_zero & 3)) zero[(n_zero & ~(int64_t)3) + i] = 0.0f;
        for (; i < n_zero / 4; i += step) ((f4*)zero)[i] = (f4){0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (unsigned r = 0; r < PER; ++r) {
        const unsigned o = 4 * (tid + r * NT);
        if (o < below) {
            *(f4*)(sq + o) = vq[r];
            *(f4*)(sg + o) = vg[r];
        }
    }
    __syncthreads();
    // the letter itself: all of the staged products, a wavefront's sum each
    float acc = 0.0f;
#pragma unroll
    for (unsigned r = 0; r < (below + NT - 1) / NT; ++r) {
        const unsigned o = tid + r * NT;
        const float term = sg[o < below ? o : 0] * sq[o < below ? o : 0];
        acc += o < below ? term : 0.0f;
    }
    acc = group_sum<64>(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    adjoint_lengths<D, N, 2>(sg, sq, a, out);
    __syncthreads();
    if (tid == 0) {
        float sum = own;
        for (unsigned w = 0; w < NT / 64; ++w) sum += red[w];
        out[a] = sum;
    }
}

// word e of length n of the slice of letter i
template <int D, int n>
__device__ __forceinline__ int slice_word(bool from_left, int i, int e)
{
    return kLevel<D, n> + (from_left ? i * kPow<D, n - 1> + e : e * D + i);
}
// sum over the cuts m .. n - 1 of word e of length n of the slice; x: the slice's shorter words, s: those of the next chunk
template <int D, int n, int m>
__device__ __forceinline__ float slice_cuts(bool from_left, const float* x, const float* s, unsigned e, float acc)
{
    if constexpr (m < n) {
        constexpr unsigned below = kPow<D, n - m>, below_right = kPow<D, n - m - 1>;      // suffixes of a cut, those of the slice
        acc = from_left ? fmaf(x[kSlice<D, m> + e / below], s[kLevel<D, n - m> + e % below], acc)
                        : fmaf(s[kLevel<D, m> + e / below_right], x[kSlice<D, n - m> + e % below_right], acc);
        acc = slice_cuts<D, n, m + 1>(from_left, x, s, e, acc);
    }
    return acc;
}
// the same for four words that share all prefixes (the first is e), from the left
template <int D, int n, int m>
__device__ __forceinline__ void quad_cuts(const float* x, const float* s, unsigned e, f4& acc)
{
    if constexpr (m < n) {
        constexpr unsigned below = kPow<D, n - m>;
        acc += x[kSlice<D, m> + e / below] * *(const f4*)(s + kLevel<D, n - m> + e % below);
        quad_cuts<D, n, m + 1>(x, s, e, acc);
    }
}
// y = x times the next chunk for the words of length n .. LAST, also to out where it is given
template <int D, int n, int LAST, int NT>
__device__ __forceinline__ void slice_levels(bool from_left, int i, const float* x, const float* s, float* y, float* __restrict__ out)
{
    if constexpr (n <= LAST) {
        for (int e = threadIdx.x; e < kPow<D, n - 1>; e += NT) {
            const int w = slice_word<D, n>(from_left, i, e);
            const float v = x[kSlice<D, n> + e] + s[w] + slice_cuts<D, n, 1>(from_left, x, s, (unsigned)e, 0.0f);
            y[kSlice<D, n> + e] = v;
            if (out) out[w] = v;
        }
        slice_levels<D, n + 1, LAST, NT>(from_left, i, x, s, y, out);
    }
}
// the words of length n .. LAST of a slice of one signature, to LDS and where it is given to out
template <int D, int n, int LAST, int NT>
__device__ __forceinline__ void slice_copy(bool from_left, int i, const float* __restrict__ S, float* y, float* __restrict__ out)
{
    if constexpr (n <= LAST) {
        for (int e = threadIdx.x; e < kPow<D, n - 1>; e += NT) {
            const int w = slice_word<D, n>(from_left, i, e);
            const float v = S[w];
            y[kSlice<D, n> + e] = v;
            if (out) out[w] = v;
        }
        slice_copy<D, n + 1, LAST, NT>(from_left, i, S, y, out);
    }
}

// coeffs[b] = S_0 .. S_{C-1}.  The words of length N are never read again: a thread keeps its quads of them (four words that
// share all prefixes) in registers.
template <int D, int N, int NT>
__global__ __launch_bounds__(NT) void chunk_slices_forward_kernel(const float* __restrict__ Sc, int C, float* __restrict__ coeffs)
{
    constexpr int W = kLevel<D, N + 1>, NS = kLevel<D, N>, XS = kSlice<D, N>, TOP = kPow<D, N - 1> / 4, QT = (TOP + NT - 1) / NT;
    constexpr int QS = (NS / 4 + NT - 1) / NT;
    static_assert(D % 4 == 0 && TOP % NT == 0, "whole quads of a word's siblings; every thread has quads of the longest words");
    __shared__ __attribute__((aligned(16))) float s[NS];
    __shared__ float x[2][XS];
    const int tid = (int)threadIdx.x, i = (int)(blockIdx.x % D);
    const int64_t b = blockIdx.x / D;
    const float* rows = Sc + b * C * (int64_t)W;
    f4 top[QT], next_top[QT], next_s[QS];
    constexpr int T0 = kLevel<D, N>;
    const int t0 = T0 + i * kPow<D, N - 1>;
    slice_copy<D, 1, N - 1, NT>(true, i, rows, x[0], nullptr);
#pragma unroll
    for (int q = 0; q < QT; ++q) top[q] = *(const f4*)(rows + t0 + 4 * (tid + q * NT));
    auto fetch = [&](int c) {
        const float* S = rows + (int64_t)c * W;
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            next_s[q] = *(const f4*)(S + 4 * (e < NS / 4 ? e : 0));
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) next_top[q] = *(const f4*)(S + t0 + 4 * (tid + q * NT));
    };
    fetch(1);                                            // (two chunks at least)
    for (int c = 1; c < C; ++c) {
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            if (e < NS / 4) *(f4*)(s + 4 * e) = next_s[q];
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) top[q] += next_top[q];
        __syncthreads();
        fetch(c + 1 < C ? c + 1 : c);
        const float* xo = x[(c - 1) & 1];
        slice_levels<D, 1, N - 1, NT>(true, i, xo, s, x[c & 1], nullptr);
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const unsigned e = 4u * (unsigned)(tid + q * NT);
            quad_cuts<D, N, 1>(xo, s, e, top[q]);
        }
        __syncthreads();
    }
    float* out = coeffs + b * (int64_t)W;
    const float* xo = x[(C - 1) & 1];
#pragma unroll
    for (int q = 0; q < QT; ++q) *(f4*)(out + t0 + 4 * (tid + q * NT)) = top[q];
    int w = 0;                                           // the shorter words of the slice, level by level
    for (int n = 1, size = 1; n < N; ++n, size *= D) {
        for (int e = tid; e < size; e += NT) out[w + i * size + e] = xo[(size - 1) / (D - 1) + e];
        w += size * D;
    }
}

// Over the words of length <= M, Sc [B][C] rows of sc_words floats, left and right [B][C] rows of those words:
// left[c] = S_0 .. S_c, right[c] = S_{c+1} .. S_{C-1} for c <= C - 2.
// Workgroup (path, letter, direction).
template <int D, int M, int NT>
__global__ __launch_bounds__(NT) void chunk_slices_both_kernel(const float* __restrict__ Sc, int64_t sc_words, int C,
                                                               float* __restrict__ left, float* __restrict__ right)
{
    constexpr int W = kLevel<D, M + 1>, XS = kSlice<D, M + 1>, QS = (W / 4 + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) float s[W];
    __shared__ float x[2][XS];
    const int tid = (int)threadIdx.x;
    const bool from_left = blockIdx.x % 2 == 0;
    const int i = (int)(blockIdx.x / 2 % D);
    const int64_t b = blockIdx.x / (2 * D);
    const float* rows = Sc + b * C * sc_words;
    float* out_rows = (from_left ? left : right) + b * C * (int64_t)W;
    // step n multiplies with chunk c0 + n dc; its product ends (from the right: begins) there
    const int c0 = from_left ? 0 : C - 1, dc = from_left ? 1 : -1, steps = C - 1;
    auto out_row = [&](int n) { return out_rows + (int64_t)(from_left ? n : C - 2 - n) * W; };
    slice_copy<D, 1, M, NT>(from_left, i, rows + c0 * sc_words, x[0], out_row(0));
    f4 next[QS];
    auto fetch = [&](int c) {
        const float* S = rows + c * sc_words;
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            next[q] = *(const f4*)(S + 4 * (e < W / 4 ? e : 0));
        }
    };
    if (steps > 1) fetch(c0 + dc);
    for (int n = 1; n < steps; ++n) {
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            const int e = tid + q * NT;
            if (e < W / 4) *(f4*)(s + 4 * e) = next[q];
        }
        __syncthreads();
        fetch(c0 + dc * (n + 1 < steps ? n + 1 : n));
        slice_levels<D, 1, M, NT>(from_left, i, x[(n - 1) & 1], s, x[n & 1], out_row(n));
        __syncthreads();
    }
}

constexpr size_t kMaxChunkLds = 96 * 1024;       // three signatures of up to 8,192 coefficients

bool make_levels(int d, int depth, Levels& g)
{
    if (d < 4 || (d & (d - 1)) != 0 || depth < 2 || depth > 12) return false;
    g.N = depth;
    g.lb = 0;
    while ((1 << g.lb) < d) ++g.lb;
    if (g.lb * depth > 30) return false;
    int64_t off = 0;
    g.ls[0] = 0;
    for (int n = 1; n <= depth; ++n) {
        g.ls[n] = (int)off;
        off += (int64_t)1 << (g.lb * n);
    }
    if (off > 0x7fffffff) return false;
    g.ls[depth + 1] = (int)off;
    g.W = (int)off;
    return true;
}

}  // namespace

bool chunking_available(int d, int depth)
{
    Levels g;
    return make_levels(d, depth, g);
}

hipError_t chunk_scan(int d, int depth, const float* Sc, float* Pfx, const float* terminal, float* coeffs_out, const float* grad,
                      float* Abar, int64_t B, int C, hipStream_t stream)
{
    Levels g;
    if (!make_levels(d, depth, g) || C < 2 || B < 1 || B > 0x7fffffff) return hipErrorInvalidValue;
    const bool bwd = Abar != nullptr;
    if (bwd ? !Pfx || !terminal || !grad || coeffs_out : !coeffs_out) return hipErrorInvalidValue;
    const size_t lds = 3 * (size_t)g.W * sizeof(float);
    if (lds > kMaxChunkLds) return hipErrorInvalidValue;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&chunk_scan_kernel), (int)kMaxChunkLds);
    if (e != hipSuccess) return e;
    chunk_scan_kernel<<<dim3((unsigned)B, bwd ? 2 : 1), 1024, lds, stream>>>(Sc, Pfx, terminal, coeffs_out, grad, Abar, C, g);
    return hipGetLastError();
}

hipError_t chunk_product(int d, int depth, const float* Sc, float* coeffs, int64_t B, hipStream_t stream)
{
    if (B < 1 || B > 65535) return hipErrorInvalidValue;
    auto grid = [&](int W) { return dim3((unsigned)((W / 4 + 255) / 256), (unsigned)B); };
    if (d == 8 && depth == 5) chunk_product_kernel<8, 5><<<grid(kLevel<8, 6>), 256, 0, stream>>>(Sc, coeffs);
    else if (d == 16 && depth == 4) chunk_product_kernel<16, 4><<<grid(kLevel<16, 5>), 256, 0, stream>>>(Sc, coeffs);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t chunk_slices_forward(int d, int depth, const float* Sc, float* coeffs, int64_t B, int C, hipStream_t stream)
{
    if (B < 1 || C < 2 || B * d > 0x7fffffff) return hipErrorInvalidValue;
    if (d == 8 && depth == 5) chunk_slices_forward_kernel<8, 5, 512><<<(unsigned)(B * 8), 512, 0, stream>>>(Sc, C, coeffs);
    else if (d == 16 && depth == 4) chunk_slices_forward_kernel<16, 4, 512><<<(unsigned)(B * 16), 512, 0, stream>>>(Sc, C, coeffs);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t chunk_slices_both(int d, int depth, const float* Sc, int64_t sc_words, float* left, float* right, int64_t B, int C,
                             hipStream_t stream)
{
    if (B < 1 || C < 2 || 2 * B * d > 0x7fffffff) return hipErrorInvalidValue;
    if (d == 8 && depth == 5) chunk_slices_both_kernel<8, 4, 512><<<(unsigned)(B * 16), 512, 0, stream>>>(Sc, sc_words, C, left, right);
    else if (d == 16 && depth == 4) chunk_slices_both_kernel<16, 3, 512><<<(unsigned)(B * 32), 512, 0, stream>>>(Sc, sc_words, C, left, right);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t chunk_adjoint(int d, int depth, const float* grad, const float* Q, int64_t row_words, float* Abar, int64_t B, int C,
                         float* zero, int64_t n_zero, hipStream_t stream)
{
    if (C < 2 || B < 1 || B * C > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(B * (C - 1)), (unsigned)d);
    if (d == 8 && depth == 5 && row_words >= kLevel<8, 5>)
        chunk_adjoint_subtree_kernel<8, 5><<<grid, kAdjointThreads, 0, stream>>>(grad, Q, Abar, C, zero, n_zero, row_words);
    else if (d == 16 && depth == 4 && row_words >= kLevel<16, 4>)
        chunk_adjoint_subtree_kernel<16, 4><<<grid, kAdjointThreads, 0, stream>>>(grad, Q, Abar, C, zero, n_zero, row_words);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sig
