// Offline weight preparation: dense 4-bit base, residual block scores, top-K
// block selection and the sparse 4-bit residual (Section 3 Eq. (4);
// Section 4.1 and Alg. 1).
//
// The three passes over W are bound by reading it (4 bytes an element against
// half a byte written) and, close behind, by the quantiser's VALU work.  They
// share one split: a workgroup of 256 threads owns a 128 x 128 block of W,
// eight adjacent lanes own a row's 128 values (64 contiguous bytes, one 16-code
// chunk, each), so a wave reads eight whole 512-byte row segments, row maxima
// are three lane exchanges, and W is read once where the base and its score
// are both wanted.  (A thread per row and group, reading 512 bytes alone, and a
// second pass for the score took 242 + 590 us on 14336 x 4096; this takes
// 69 us.)
#include "mq_device.h"

namespace mq {

constexpr int kPrepThreads = 256;
constexpr int kRowLanes = kGroup / 16;                      // lanes per row: one 16-code chunk each
constexpr int kRowsPerPass = kPrepThreads / kRowLanes;      // 32 rows of the block at a time
constexpr int kPrepPasses = kGroup / kRowsPerPass;

struct Chunk16 {
    float v[16];
};

__device__ __forceinline__ Chunk16 load_chunk(const float* p) {
    Chunk16 c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 f = reinterpret_cast<const float4*>(p)[i];
        c.v[4 * i + 0] = f.x;
        c.v[4 * i + 1] = f.y;
        c.v[4 * i + 2] = f.z;
        c.v[4 * i + 3] = f.w;
    }
    return c;
}

// Largest |v| of the row (over its eight lanes; every lane gets it).
__device__ __forceinline__ float row_absmax(const Chunk16& c) {
    float m = 0.0f;
#pragma unroll
    for (int e = 0; e < 16; ++e) m = fmaxf(m, fabsf(c.v[e]));
#pragma unroll
    for (int off = 1; off < kRowLanes; off <<= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    return m;
}

// Codes of 16 values for a scale s, as floats.
__device__ __forceinline__ void quant_chunk16(const Chunk16& c, float s, float (&q)[16]) {
    const float inv_s = 1.0f / s;
#pragma unroll
    for (int e = 0; e < 16; ++e) q[e] = s == 0.0f ? 0.0f : (float)quant_code(c.v[e], s, inv_s);
}

__device__ __forceinline__ uint2 fold_chunk16(const float (&q)[16]) {
    int qi[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) qi[e] = (int)q[e];
    return fold_codes(qi);
}

// R = W - s q in fp32: s * q is exact (11-bit significand times |q| <= 8), so
// the difference is rounded once.
__device__ __forceinline__ float residual_at(float w, float s, float q) {
    const float deq = s * q;
    return w - deq;
}

// Residual of 16 values from their stored chunk and scale.
__device__ __forceinline__ Chunk16 residual_chunk(const Chunk16& w, const uint2 ch, float s) {
    Chunk16 r;
#pragma unroll
    for (int e = 0; e < 16; ++e) r.v[e] = residual_at(w.v[e], s, (float)chunk_code(ch.x, ch.y, e));
    return r;
}

// Sum of the workgroup's per-thread fp64 values, in a fixed order (lanes by
// halves, then waves); the result is thread 0's.
__device__ __forceinline__ double block_sum(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = red[0];
    for (int w = 1; w < kPrepThreads / 64; ++w) t += red[w];
    return t;
}

// ---------------------------------------------------------------------------
// Base quantisation, Eq. (1) over 128 values, and (SCORE) ||R_B||_F^2 of the
// block in fp64.  Workgroup = block (nb, kb), kb fastest.
// ---------------------------------------------------------------------------
template <bool SCORE>
__global__ __launch_bounds__(kPrepThreads) void quant_base_kernel(
    const float* __restrict__ W, int N, int K, int ldw,
    uint8_t* __restrict__ Wq, uint16_t* __restrict__ s_w, double* __restrict__ score) {
    __shared__ double red[kPrepThreads / 64];
    const int KB = K / kGroup;
    const int nb = blockIdx.x / KB, kb = blockIdx.x % KB;
    const int c = threadIdx.x % kRowLanes;
    double acc = 0.0;
#pragma unroll
    for (int p = 0; p < kPrepPasses; ++p) {
        const int n = nb * kGroup + p * kRowsPerPass + (int)threadIdx.x / kRowLanes;
        const Chunk16 w = load_chunk(W + (int64_t)n * ldw + (int64_t)kb * kGroup + 16 * c);
        const uint16_t sb = scale_bits_from_amax(row_absmax(w));
        const float s = half_bits_to_float(sb);
        float q[16];
        quant_chunk16(w, s, q);
        if (c == 0) s_w[wscale_index(N, n, kb)] = sb;
        *reinterpret_cast<uint2*>(Wq + piece_offset(N, n, kb) + 8 * c) = fold_chunk16(q);
        if constexpr (SCORE) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const double r = residual_at(w.v[e], s, q[e]);
                acc += r * r;
            }
        }
    }
    if constexpr (SCORE) {
        const double t = block_sum(acc, red);
        if (threadIdx.x == 0) score[blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// Diagonal Hessian h_j = (2/T) sum_t X[t,j]^2, fp64, each channel's tokens
// added in order (a fixed result whatever the split).  That chain of T
// dependent additions is what bounds the kernel, so a workgroup of eight waves
// owns 64 channels: all waves fetch the next kHessRows tokens (two steps ahead,
// whole 128-byte lines) and put their squares -- exact in fp32 -- into LDS,
// and wave 0 adds the rows of the step before, one channel a lane.  (One thread
// per channel, each load waited for: 484 us at T = 2048, K = 4096; this takes
// 19 us.)
// ---------------------------------------------------------------------------
constexpr int kHessThreads = 512, kHessCols = 64, kHessRows = 256;
constexpr int kHessVecs = kHessRows * kHessCols / 8 / kHessThreads;   // 8-channel pieces a thread and step
__host__ __device__ constexpr int hess_steps(int T) { return (T - 1) / kHessRows + 1; }   // T >= 1
static_assert(hess_steps(1) == 1 && hess_steps(kHessRows + 1) == 2 && hess_steps(0x7fffffff) == 1 << 23,
              "no token count overflows the step count");

template <bool VEC>
__global__ __launch_bounds__(kHessThreads) void hessian_diag_kernel(
    const uint16_t* __restrict__ X, int T, int K, int ldx, double* __restrict__ h) {
    __shared__ __attribute__((aligned(16))) float sq[2][kHessRows][kHessCols];
    const int t = threadIdx.x, lane = t & 63;
    const int j0 = blockIdx.x * kHessCols;
    const int cc = (t % (kHessCols / 8)) * 8, r0 = t / (kHessCols / 8);   // channels cc .. cc + 7 of rows r0 + 64 i
    constexpr int kRowStep = kHessThreads / (kHessCols / 8);
    struct Piece {
        uint32_t w[4];
    };
    auto fetch = [&](int step, Piece (&d)[kHessVecs]) {
#pragma unroll
        for (int i = 0; i < kHessVecs; ++i) {
            const int64_t row = (int64_t)step * kHessRows + r0 + i * kRowStep;
            d[i] = Piece{{0u, 0u, 0u, 0u}};
            if (row >= T) continue;
            const uint16_t* src = X + row * ldx + j0 + cc;
            if constexpr (VEC) {
                if (j0 + cc < K) {                        // K % 8 == 0
                    const uint4 v = *reinterpret_cast<const uint4*>(src);
                    d[i] = Piece{{v.x, v.y, v.z, v.w}};
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (j0 + cc + e < K) d[i].w[e / 2] |= (uint32_t)src[e] << (16 * (e & 1));
            }
        }
    };
    auto put = [&](int buf, const Piece (&d)[kHessVecs]) {
#pragma unroll
        for (int i = 0; i < kHessVecs; ++i) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = half_bits_to_float((uint16_t)(d[i].w[e / 2] >> (16 * (e & 1))));
                f[e] = x * x;
            }
            float4* dst = reinterpret_cast<float4*>(&sq[buf][r0 + i * kRowStep][cc]);
            dst[0] = make_float4(f[0], f[1], f[2], f[3]);
            dst[1] = make_float4(f[4], f[5], f[6], f[7]);
        }
    };
    const int steps = hess_steps(T);
    Piece d[kHessVecs];
    fetch(0, d);
    put(0, d);
    fetch(1, d);
    __syncthreads();
    double acc = 0.0;
    for (int s = 0; s < steps; ++s) {
        if (s + 1 < steps) {
            put((s + 1) & 1, d);
            fetch(s + 2, d);
        }
        if (t < 64) {
            // sixteens of rows that hold tokens (all 256 rows of the last step took 3.9 us at T = 1
            // instead of 2.4, 6.5 instead of 4.8 at T = 257); rows past T are zeros, which change nothing
            const int rows = s + 1 < steps ? kHessRows : T - s * kHessRows;
            for (int r0 = 0; r0 < rows; r0 += 16)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc += (double)sq[s & 1][r0 + r][lane];
        }
        __syncthreads();
    }
    if (t < 64 && j0 + lane < K) h[j0 + lane] = 2.0 / (double)T * acc;
}

// ---------------------------------------------------------------------------
// Delta-Hessian score (Alg. 1): per block, sum_B h_j R^2 - sum_B h_j (R - Q(R))^2,
// clamped at 0; Q(R) with one scale per block row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kPrepThreads) void score_dhessian_kernel(
    const float* __restrict__ W, int N, int K, int ldw,
    const uint8_t* __restrict__ Wq, const uint16_t* __restrict__ s_w,
    const double* __restrict__ h, double* __restrict__ score) {
    __shared__ double red[2][kPrepThreads / 64];
    const int KB = K / kGroup;
    const int nb = blockIdx.x / KB, kb = blockIdx.x % KB;
    const int c = threadIdx.x % kRowLanes;
    double hj[16];                                        // the lane's 16 columns in every pass
#pragma unroll
    for (int e = 0; e < 16; ++e) hj[e] = h[kb * kGroup + 16 * c + e];
    double before = 0.0, after = 0.0;
#pragma unroll 2
    for (int p = 0; p < kPrepPasses; ++p) {
        const int n = nb * kGroup + p * kRowsPerPass + (int)threadIdx.x / kRowLanes;
        const Chunk16 w = load_chunk(W + (int64_t)n * ldw + (int64_t)kb * kGroup + 16 * c);
        const uint2 ch = *reinterpret_cast<const uint2*>(Wq + piece_offset(N, n, kb) + 8 * c);
        const Chunk16 r = residual_chunk(w, ch, half_bits_to_float(s_w[wscale_index(N, n, kb)]));
        const float sr = half_bits_to_float(scale_bits_from_amax(row_absmax(r)));
        float q[16];
        quant_chunk16(r, sr, q);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const double rv = (double)r.v[e], d = rv - (double)sr * (double)q[e];
            before += hj[e] * (rv * rv);
            after += hj[e] * (d * d);
        }
    }
    const double b = block_sum(before, red[0]), a = block_sum(after, red[1]);
    if (threadIdx.x == 0) {
        const double d = b - a;
        score[blockIdx.x] = d > 0.0 ? d : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Top-K selection: the nnzb blocks of largest score, ties to the lower linear
// index, as a CSR.  One workgroup:
//   1. a most-significant-digit radix search over order-preserving 64-bit keys
//      (digits of log2(2 kSelThreads) bits, from the first bit in which the keys
//      differ) narrows [lo, lo + 2^bits) to the keys that hold the nnzb-th
//      largest, and stops as soon as all of them are taken;
//   2. one pass in linear order (block rows are consecutive): a block is
//      selected when its key is above that range, or in it and among the first
//      `need` of those; a block-wide scan of both counts gives every selected
//      block its place and every block row its start.
// It reads the scores once when they fit in registers (kSelItems a thread),
// else once per digit.  Bound by one CU's instruction issue and a few barriers
// a digit (typical scores take two or three digits), so few blocks take
// threads and code for no more items than they have: with 1024 threads of 16
// items for every size, 1 block took 9.9 us against 2.5 with <64, 1>, 1024
// blocks 12.6 against 8.0 with <1024, 1>, 3584 14.2 against 9.7 with <1024, 4>.
// (Counting each block's rank against all scores, twice, takes 4.9, 174 and
// 600 us for these.)
// ---------------------------------------------------------------------------
// order-preserving key of a finite score (-0 as +0)
__device__ __forceinline__ uint64_t score_key(double s) {
    const uint64_t u = (uint64_t)__double_as_longlong(s + 0.0);
    return (u >> 63) ? ~u : u | (1ull << 63);
}

template <int kSelThreads, int kSelItems>
__global__ __launch_bounds__(kSelThreads) void select_kernel(
    const double* __restrict__ score, int NB, int KB, int nnzb,
    int32_t* __restrict__ rowptr, int32_t* __restrict__ kb_out) {
    constexpr int kSelBins = 2 * kSelThreads, kSelWaves = kSelThreads / 64;
    constexpr int kSelDigit = 31 - __builtin_clz(kSelBins);
    __shared__ int hist[kSelBins];
    __shared__ uint64_t lo_sh[kSelWaves], hi_sh[kSelWaves];
    __shared__ int wsum[2][kSelWaves];
    __shared__ int pick_bin, pick_above;
    const int n = NB * KB, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (nnzb == 0) {
        for (int i = t; i <= NB; i += kSelThreads) rowptr[i] = 0;
        return;
    }
    // item i < items of tile b: linear index (b kSelThreads + t) items + i
    const int items = min(kSelItems, (n + kSelThreads - 1) / kSelThreads);
    const int tiles = (n + kSelThreads * items - 1) / (kSelThreads * items);
    auto index = [&](int b, int i) { return (b * kSelThreads + t) * items + i; };      // below 2^24 + 2^14
    auto valid = [&](int b, int i) { return i < items && index(b, i) < n; };
    uint64_t key[kSelItems];
    auto load_tile = [&](int b) {
#pragma unroll
        for (int i = 0; i < kSelItems; ++i) key[i] = valid(b, i) ? score_key(score[index(b, i)]) : 0;
    };

    // smallest and largest key
    uint64_t kmin = ~0ull, kmax = 0;
    for (int b = 0; b < tiles; ++b) {
        load_tile(b);
#pragma unroll
        for (int i = 0; i < kSelItems; ++i)
            if (valid(b, i)) {
                kmin = key[i] < kmin ? key[i] : kmin;
                kmax = key[i] > kmax ? key[i] : kmax;
            }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t a = __shfl_xor((unsigned long long)kmin, off, 64), c = __shfl_xor((unsigned long long)kmax, off, 64);
        kmin = a < kmin ? a : kmin;
        kmax = c > kmax ? c : kmax;
    }
    if (lane == 0) {
        lo_sh[wv] = kmin;
        hi_sh[wv] = kmax;
    }
    __syncthreads();
    for (int w = 0; w < kSelWaves; ++w) {
        kmin = lo_sh[w] < kmin ? lo_sh[w] : kmin;
        kmax = hi_sh[w] > kmax ? hi_sh[w] : kmax;
    }
    // keys in [lo, lo + 2^bits) hold the nnzb-th largest; `need` of them are
    // taken, and all keys above
    int bits = kmin == kmax ? 0 : 64 - __builtin_clzll(kmin ^ kmax);
    uint64_t lo = bits == 64 ? 0 : (kmin >> bits) << bits;
    int need = nnzb, inside = n;
    while (bits > 0 && need < inside) {
        const int d = bits < kSelDigit ? bits : kSelDigit, sh = bits - d;
        for (int u = t; u < kSelBins; u += kSelThreads) hist[u] = 0;
        __syncthreads();
        for (int b = 0; b < tiles; ++b) {
            if (tiles > 1) load_tile(b);
#pragma unroll
            for (int i = 0; i < kSelItems; ++i) {
                const uint64_t off = key[i] - lo;
                if (valid(b, i) && key[i] >= lo && (bits == 64 || (off >> bits) == 0)) atomicAdd(&hist[(int)(off >> sh)], 1);
            }
        }
        __syncthreads();
        // counts from the top bin down: thread t takes the two bins
        // top = kSelBins - 1 - 2 t and top - 1
        const int top = kSelBins - 1 - 2 * t;
        const int h0 = hist[top], h1 = hist[top - 1];
        int pre = h0 + h1;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(pre, off, 64);
            if (lane >= off) pre += o;
        }
        if (lane == 63) wsum[0][wv] = pre;
        __syncthreads();
        for (int w = 0; w < wv; ++w) pre += wsum[0][w];
        const int above1 = pre - h1, above0 = above1 - h0;    // keys above each of the two bins
        if (above0 < need && need <= above0 + h0) {
            pick_bin = top;
            pick_above = above0;
        }
        if (above1 < need && need <= above1 + h1) {
            pick_bin = top - 1;
            pick_above = above1;
        }
        __syncthreads();
        lo += (uint64_t)pick_bin << sh;
        need -= pick_above;
        inside = hist[pick_bin];
        bits = sh;
        __syncthreads();
    }
    // placement
    int base_gt = 0, base_eq = 0;                             // before this tile
    for (int b = 0; b < tiles; ++b) {
        if (tiles > 1) load_tile(b);
        int gt = 0, eq = 0;
        uint32_t gtm = 0, eqm = 0;
#pragma unroll
        for (int i = 0; i < kSelItems; ++i) {
            if (!valid(b, i) || key[i] < lo) continue;
            const uint64_t off = key[i] - lo;
            const bool in = bits == 64 || (off >> bits) == 0;
            if (in) { eqm |= 1u << i; ++eq; }
            else { gtm |= 1u << i; ++gt; }
        }
        int sg = gt, se = eq;
        for (int off = 1; off < 64; off <<= 1) {
            const int a = __shfl_up(sg, off, 64), c = __shfl_up(se, off, 64);
            if (lane >= off) { sg += a; se += c; }
        }
        __syncthreads();
        if (lane == 63) {
            wsum[0][wv] = sg;
            wsum[1][wv] = se;
        }
        __syncthreads();
        int g0 = base_gt + sg - gt, e0 = base_eq + se - eq;
        for (int w = 0; w < kSelWaves; ++w) {
            if (w < wv) {
                g0 += wsum[0][w];
                e0 += wsum[1][w];
            }
            base_gt += wsum[0][w];
            base_eq += wsum[1][w];
        }
        const int idx0 = index(b, 0);
        int row = idx0 / KB, col = idx0 - row * KB;
#pragma unroll
        for (int i = 0; i < kSelItems; ++i) {
            if (valid(b, i)) {
                const int pos = g0 + min(e0, need);           // selected before this block
                if (col == 0) rowptr[row] = pos;
                const bool g = (gtm >> i) & 1, e = (eqm >> i) & 1;
                if ((g || (e && e0 < need)) && pos < nnzb) kb_out[pos] = col;
                g0 += g;
                e0 += e;
                if (++col == KB) {
                    col = 0;
                    ++row;
                }
            }
        }
    }
    if (t == 0) rowptr[NB] = nnzb;
}

// ---------------------------------------------------------------------------
// Residual quantisation on the selected blocks: workgroup = block p, all 128
// rows at once (few blocks and little work each: one trip to memory instead of
// one per 32 rows, 14.9 -> 12.8 us for 358 blocks, 11.5 -> 7.5 us for 102).
// ---------------------------------------------------------------------------
constexpr int kResThreads = kGroup * kRowLanes;
__global__ __launch_bounds__(kResThreads) void quant_residual_kernel(
    const float* __restrict__ W, int N, int K, int ldw,
    const uint8_t* __restrict__ Wq, const uint16_t* __restrict__ s_w,
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ res_kb, int NB,
    uint8_t* __restrict__ Rq, uint16_t* __restrict__ s_r) {
    const int p = blockIdx.x;
    // block row of entry p: largest nb with rowptr[nb] <= p
    int lo = 0, hi = NB - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (rowptr[mid] <= p) lo = mid; else hi = mid - 1;
    }
    const int nb = lo, kb = res_kb[p];
    const int c = threadIdx.x % kRowLanes, r = (int)threadIdx.x / kRowLanes, n = nb * kGroup + r;
    const Chunk16 w = load_chunk(W + (int64_t)n * ldw + (int64_t)kb * kGroup + 16 * c);
    const uint2 ch = *reinterpret_cast<const uint2*>(Wq + piece_offset(N, n, kb) + 8 * c);
    const Chunk16 res = residual_chunk(w, ch, half_bits_to_float(s_w[wscale_index(N, n, kb)]));
    const uint16_t srb = scale_bits_from_amax(row_absmax(res));
    float q[16];
    quant_chunk16(res, half_bits_to_float(srb), q);
    if (c == 0) s_r[(int64_t)p * kGroup + r] = srb;
    *reinterpret_cast<uint2*>(Rq + ((int64_t)p * kGroup + r) * kGroupBytes + 8 * c) = fold_chunk16(q);
}

}  // namespace mq

using namespace mq;

static mq_status check_weight_args(const float* W, int N, int K, int ldw,
                                   const void* Wq, const void* s_w) {
    if (N < 0 || K < 0) return MQ_ERR_INVALID_ARG;
    if (!mq_host::shape_ok(N, K) || ldw < K || ldw % 4 != 0) return MQ_ERR_UNSUPPORTED_SHAPE;
    if (!W || !Wq || !s_w) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(W, 16) || !mq_host::aligned(Wq, 16) || !mq_host::aligned(s_w, 2))
        return MQ_ERR_MISALIGNED;
    return MQ_OK;
}

extern "C" mq_status mq_quantize_weight(const float* W, int N, int K, int ldw,
                                        uint8_t* Wq, void* s_w, double* score,
                                        hipStream_t stream) {
    mq_status st = check_weight_args(W, N, K, ldw, Wq, s_w);
    if (st != MQ_OK) return st;
    if (score && !mq_host::aligned(score, 8)) return MQ_ERR_MISALIGNED;
    const unsigned nblk = (unsigned)((int64_t)(N / kGroup) * (K / kGroup));
    if (score)
        hipLaunchKernelGGL(quant_base_kernel<true>, dim3(nblk), dim3(kPrepThreads), 0, stream,
                           W, N, K, ldw, Wq, static_cast<uint16_t*>(s_w), score);
    else
        hipLaunchKernelGGL(quant_base_kernel<false>, dim3(nblk), dim3(kPrepThreads), 0, stream,
                           W, N, K, ldw, Wq, static_cast<uint16_t*>(s_w), score);
    return mq_host::launch_status();
}

extern "C" mq_status mq_hessian_diag(const void* X, int T, int K, int ldx, double* h,
                                     hipStream_t stream) {
    if (T <= 0 || K <= 0 || ldx < K) return MQ_ERR_INVALID_ARG;
    if (!X || !h) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(X, 2) || !mq_host::aligned(h, 8)) return MQ_ERR_MISALIGNED;
    // 16-byte loads where every row piece is aligned (K % 8: no piece straddles the last channel)
    const bool vec = mq_host::aligned(X, 16) && ldx % 8 == 0 && K % 8 == 0;
    const dim3 grid((unsigned)(((int64_t)K + kHessCols - 1) / kHessCols)), block(kHessThreads);
    if (vec)
        hipLaunchKernelGGL(hessian_diag_kernel<true>, grid, block, 0, stream, static_cast<const uint16_t*>(X), T, K,
                           ldx, h);
    else
        hipLaunchKernelGGL(hessian_diag_kernel<false>, grid, block, 0, stream, static_cast<const uint16_t*>(X), T, K,
                           ldx, h);
    return mq_host::launch_status();
}

extern "C" mq_status mq_block_scores_dhessian(const float* W, int N, int K, int ldw,
                                              const uint8_t* Wq, const void* s_w,
                                              const double* h, double* score,
                                              hipStream_t stream) {
    mq_status st = check_weight_args(W, N, K, ldw, Wq, s_w);
    if (st != MQ_OK) return st;
    if (!h || !score) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(h, 8) || !mq_host::aligned(score, 8)) return MQ_ERR_MISALIGNED;
    const int nblk = (N / kGroup) * (K / kGroup);
    hipLaunchKernelGGL(score_dhessian_kernel, dim3(nblk), dim3(kPrepThreads), 0, stream,
                       W, N, K, ldw, Wq, static_cast<const uint16_t*>(s_w), h, score);
    return mq_host::launch_status();
}

extern "C" mq_status mq_select_blocks(const double* score, int NB, int KB, int nnzb,
                                      int32_t* res_rowptr, int32_t* res_kb,
                                      hipStream_t stream) {
    if (NB <= 0 || KB <= 0 || nnzb < 0) return MQ_ERR_INVALID_ARG;
    if ((int64_t)NB * KB > (1 << 24)) return MQ_ERR_UNSUPPORTED_SHAPE;
    if ((int64_t)nnzb > (int64_t)NB * KB) return MQ_ERR_INVALID_ARG;
    if (!score || !res_rowptr || (nnzb > 0 && !res_kb)) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(score, 8) || !mq_host::aligned(res_rowptr, 4) ||
        (res_kb && !mq_host::aligned(res_kb, 4)))
        return MQ_ERR_MISALIGNED;
    const int n = NB * KB;
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, stream, score, NB, KB, nnzb, res_rowptr, res_kb);
    };
    if (n <= 64) run(select_kernel<64, 1>, 64);
    else if (n <= 1024) run(select_kernel<1024, 1>, 1024);
    else if (n <= 4096) run(select_kernel<1024, 4>, 1024);
    else run(select_kernel<1024, 16>, 1024);
    return mq_host::launch_status();
}

extern "C" mq_status mq_quantize_residual(const float* W, int N, int K, int ldw,
                                          const uint8_t* Wq, const void* s_w,
                                          const int32_t* res_rowptr, const int32_t* res_kb,
                                          int nnzb, uint8_t* Rq, void* s_r,
                                          hipStream_t stream) {
    mq_status st = check_weight_args(W, N, K, ldw, Wq, s_w);
    if (st != MQ_OK) return st;
    if (nnzb < 0 || (int64_t)nnzb > (int64_t)(N / kGroup) * (K / kGroup)) return MQ_ERR_INVALID_ARG;
    if (nnzb == 0) return MQ_OK;
    if (!res_rowptr || !res_kb || !Rq || !s_r) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(res_rowptr, 4) || !mq_host::aligned(res_kb, 4) ||
        !mq_host::aligned(Rq, 16) || !mq_host::aligned(s_r, 2))
        return MQ_ERR_MISALIGNED;
    hipLaunchKernelGGL(quant_residual_kernel, dim3(nnzb), dim3(kResThreads), 0, stream,
                       W, N, K, ldw, Wq, static_cast<const uint16_t*>(s_w),
                       res_rowptr, res_kb, N / kGroup, Rq, static_cast<uint16_t*>(s_r));
    return mq_host::launch_status();
}
