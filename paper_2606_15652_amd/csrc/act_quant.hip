// Per-token symmetric activation quantisation fused with code packing
// (Section 2, Eq. (1) applied per row; Section 4.2 "Kernel Fusion": layout
// packing is fused with quantisation): INT4 codes in the matrix instruction's
// operand form, or (W4A8) INT8 codes as an e4m3 high plane and a folded 4-bit
// low plane.
//
// One workgroup per token row, one thread per quarter of a group (32 codes,
// 64 bytes of X) or half of one, up to 1024 threads: a row of up to 65536 values
// is read once, in one trip to memory, and stays in registers.  The row maximum of |x| is
// taken on the fp16 bit patterns with the sign cleared (an order-preserving
// integer max for finite values, packed 16-bit maxima), reduced across the wave
// by DPP and across the waves through LDS.  Large inputs are bound by memory
// and, close behind, by the VALU work per code: a code is five fp32 operations
// and a clamp, and one conversion instruction turns the thread's codes into
// their operand dwords.  Few rows are bound by latency.  (256 threads of up
// to 16 chunks of 16 codes, packed with integer operations, against this: INT4
// 4096 x 4096 10.8 -> 9.6 us, 8192 x 8192 34.0 -> 28.8; INT8 2048 x 4096
// 11.0 -> 7.0, 16 x 14336 10.8 -> 3.9.)
#include "mq_device.h"

namespace mq {

constexpr int kActMaxThreads = 1024;

// Row of workgroup b.  Workgroups go to the eight XCDs in turn (b % 8), and
// neighbouring rows share the 128-byte lines of the operand planes (a row
// writes 64 and 32 bytes of each group's main and tail pieces), so each XCD
// takes a contiguous range of rows: the lines are then written whole from one
// L2.  A bijection on [0, M): XCD x holds rows x per + min(x, rem) on.
__device__ __forceinline__ int xcd_row(int b, int M) {
    const int x = b % 8, k = b / 8, per = M / 8, rem = M % 8;
    return x * per + min(x, rem) + k;
}

// C: values a thread takes at a time; P: such pieces it keeps in registers
// (0: longer rows, read a second time for the codes).
template <bool A8, int C, int P>
__global__ __launch_bounds__(kActMaxThreads) void act_quant_kernel(
    const uint16_t* __restrict__ X, int M, int K, int ldx,
    uint8_t* __restrict__ Xq, uint16_t* __restrict__ s_x) {
    __shared__ uint32_t red[kActMaxThreads / 64];
    const int m = xcd_row(blockIdx.x, M);
    const int t = threadIdx.x, threads = blockDim.x;
    const uint16_t* row = X + (int64_t)m * ldx;
    const int pieces = K / C, G = K / kGroup;

    Halves<C> v[P > 0 ? P : 1] = {};
    uint32_t amax = 0;
    if constexpr (P > 0) {
#pragma unroll
        for (int i = 0; i < P; ++i)
            if (t + i * threads < pieces) v[i] = load_halves<C>(row + C * (t + i * threads));
#pragma unroll
        for (int i = 0; i < P; ++i) amax = max(amax, absmax_bits(v[i]));
    } else {
        for (int c = t; c < pieces; c += threads) amax = max(amax, absmax_bits(load_halves<C>(row + C * c)));
    }
    amax = wave_max_dpp(amax);
    if (threads > 64) {
        if ((t & 63) == 0) red[t >> 6] = amax;
        __syncthreads();
        for (int w = 0; w < threads / 64; ++w) amax = max(amax, red[w]);
    }

    constexpr int qmax = A8 ? kQmax8 : kQmax;
    const uint16_t sb = scale_bits_from_amax(half_bits_to_float((uint16_t)amax), qmax);
    const float s = A8 && sb == kHalfInf ? 0.0f : half_bits_to_float(sb);
    const float inv_s = s == 0.0f ? 0.0f : 1.0f / s;        // a zero scale: all codes 0
    if (t == 0) s_x[m] = sb;
    const uint32_t keep = amax < kHalfInf ? ~0u : 0u;       // INT4: a row that is not finite has codes 0

    auto store = [&](const Halves<C>& x, int c) {
        float q[C];
        quant_codes(x, s, inv_s, (float)qmax, q);
        const int g = c / (kGroup / C), j = c % (kGroup / C);   // piece j of group g
        if constexpr (A8) {
            // x = 8 h + l: the e4m3 bytes of h = floor(x / 8) in the high plane (piece (row, group)
            // of 128 bytes at (g M + m) 128, chunks placed by hi_chunk_offset), the folded 4-bit
            // codes l in [0, 7] in the low plane (M K bytes on, the W4A4 group order)
            uint32_t hb[C / 4];
#pragma unroll
            for (int i = 0; i < C / 4; ++i) {
                float h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    h[e] = floorf(q[4 * i + e] * 0.125f);
                    q[4 * i + e] = __builtin_fmaf(-8.0f, h[e], q[4 * i + e]);
                }
                int b = __builtin_amdgcn_cvt_pk_fp8_f32(h[0], h[1], 0, false);
                hb[i] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(h[2], h[3], b, true);
            }
            const u32x6 d = operand_dwords(q);
            uint8_t* hi = Xq + ((int64_t)g * M + m) * 128;
#pragma unroll
            for (int k = 0; k < C / 16; ++k)
                *reinterpret_cast<uint4*>(hi + hi_chunk_offset(C / 16 * j + k)) =
                    make_uint4(hb[4 * k], hb[4 * k + 1], hb[4 * k + 2], hb[4 * k + 3]);
            uint8_t* lo = Xq + (int64_t)M * K + piece_offset(M, m, g) + C / 2 * j;
            const uint2 l0 = make_uint2(d[0] | (d[2] & kFoldA), d[1] | (d[2] & kFoldB));
            if constexpr (C == 32)
                *reinterpret_cast<uint4*>(lo) = make_uint4(l0.x, l0.y, d[3] | (d[5] & kFoldA), d[4] | (d[5] & kFoldB));
            else
                *reinterpret_cast<uint2*>(lo) = l0;
        } else {
            const u32x6 d = operand_dwords(q) & keep;
            uint8_t* main = Xq + act_main_offset(M, m, g);
            if constexpr (C == 32) {
                *reinterpret_cast<uint4*>(main + 16 * j) = make_uint4(d[0], d[1], d[2], d[3]);
                *reinterpret_cast<uint2*>(Xq + act_tail_offset(M, G, m, g, j)) = make_uint2(d[4], d[5]);
            } else {
                // the threads of a quarter's halves (both here: K / 16 is even): the even one
                // writes the main plane's 16 bytes, with the odd one's d0 as d3, the odd one the tail's 8
                const uint32_t d3 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d[0], 0xF5, 0xf, 0xf, true);   // quad_perm 1, 1, 3, 3
                if ((j & 1) == 0) *reinterpret_cast<uint4*>(main + 8 * j) = make_uint4(d[0], d[1], d[2], d3);
                else *reinterpret_cast<uint2*>(Xq + act_tail_offset(M, G, m, g, j / 2)) = make_uint2(d[1], d[2]);
            }
        }
    };
    if constexpr (P > 0) {
#pragma unroll
        for (int i = 0; i < P; ++i)
            if (t + i * threads < pieces) store(v[i], t + i * threads);
    } else {
        for (int c = t; c < pieces; c += threads) {
            v[0] = load_halves<C>(row + C * c);
            store(v[0], c);
        }
    }
}

template <bool A8>
static mq_status quantize_rows(const void* X, int M, int K, int ldx, uint8_t* Xq, void* s_x, hipStream_t stream) {
    if (M < 0 || K < 0) return MQ_ERR_INVALID_ARG;
    if (M > (1 << 24) || K < 128 || K % 128 != 0 || K > (1 << 20) || ldx < K || ldx % 8 != 0)
        return MQ_ERR_UNSUPPORTED_SHAPE;
    if (M == 0) return MQ_OK;
    if (!X || !Xq || !s_x) return MQ_ERR_INVALID_ARG;
    if (!mq_host::aligned(X, 16) || !mq_host::aligned(Xq, 16) || !mq_host::aligned(s_x, 2))
        return MQ_ERR_MISALIGNED;
    const auto* x = static_cast<const uint16_t*>(X);
    auto* s = static_cast<uint16_t*>(s_x);
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(M), dim3(threads), 0, stream, x, M, K, ldx, Xq, s);
    };
    auto whole_waves = [](int n) { return (n + 63) / 64 * 64; };
    // Few workgroups a CU are bound by how long a thread's codes take one wave
    // (two workgroups' single waves met on one SIMD: 4096-value rows at M = 512
    // 3.2 us by quarters, 2.8 by halves; 512-value rows 3.0 and 2.1), so threads
    // take halves where rows are few, and always where that leaves a row in one
    // wave (K <= 1024: 8192 rows of 1024 values 7.0 and 5.2 us).  Rows up to
    // 2048 values need a second wave for it: only up to one workgroup a CU
    // (M = 256 2.3 and 2.2 us, M = 512 2.45 and 2.55).  Beyond, quarters are
    // cheaper (8192 values equal at M = 1024; 14336 at M = 1024 8.9 and 9.8).
    const int most_rows_by_halves = K <= 1024 ? M : K <= 2048 ? 256 : K <= 8192 ? 1024 : 0;
    if (M <= most_rows_by_halves) run(act_quant_kernel<A8, 16, 1>, whole_waves(K / 16));
    else if (K <= 32 * kActMaxThreads) run(act_quant_kernel<A8, 32, 1>, whole_waves(K / 32));
    else if (K <= 64 * kActMaxThreads) run(act_quant_kernel<A8, 32, 2>, kActMaxThreads);
    else run(act_quant_kernel<A8, 32, 0>, kActMaxThreads);
    return mq_host::launch_status();
}

}  // namespace mq

using namespace mq;

extern "C" mq_status mq_quantize_act8(const void* X, int M, int K, int ldx,
                                      uint8_t* Xq8, void* s_x, hipStream_t stream) {
    return quantize_rows<true>(X, M, K, ldx, Xq8, s_x, stream);
}

extern "C" mq_status mq_quantize_act(const void* X, int M, int K, int ldx,
                                     uint8_t* Xq, void* s_x, hipStream_t stream) {
    return quantize_rows<false>(X, M, K, ldx, Xq, s_x, stream);
}
