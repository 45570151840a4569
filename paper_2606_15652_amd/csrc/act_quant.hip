// Per-token symmetric activation quantisation fused with code packing
// (Section 2, Eq. (1) applied per row; Section 4.2 "Kernel Fusion": layout
// packing is fused with quantisation): INT4 codes in the matrix instruction's
// operand form, or (W4A8) INT8 codes as an e4m3 high plane and a folded 4-bit
// low plane.
//
// One workgroup per token row, one thread per quarter of a group (32 codes,
// 64 bytes of X), up to 1024 threads: a row of up to 32768 values is read once,
// in one trip to memory, and stays in registers.  The row maximum of |x| is
// taken on the fp16 bit patterns with the sign cleared (an order-preserving
// integer max for finite values, packed 16-bit maxima), reduced across the wave
// by DPP and across the waves through LDS.  Large inputs are bound by memory
// and, close behind, by the VALU work per code: a code is five fp32 operations
// and a clamp, and one conversion instruction turns the thread's 32 codes into
// their six operand dwords.  Few rows are bound by latency.  (256 threads of up
// to 16 chunks of 16 codes, packed with integer operations, against this: INT4
// 4096 x 4096 11.0 -> 9.4 us, 8192 x 8192 33.0 -> 27.3; INT8 2048 x 4096
// 11.2 -> 7.4, 16 x 14336 11.0 -> 4.1.)
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

// LOOP: rows longer than 32 codes a thread, read a second time for the codes.
template <bool A8, bool LOOP>
__global__ __launch_bounds__(kActMaxThreads) void act_quant_kernel(
    const uint16_t* __restrict__ X, int M, int K, int ldx,
    uint8_t* __restrict__ Xq, uint16_t* __restrict__ s_x) {
    __shared__ uint32_t red[kActMaxThreads / 64];
    const int m = xcd_row(blockIdx.x, M);
    const int t = threadIdx.x, threads = blockDim.x;
    const uint16_t* row = X + (int64_t)m * ldx;
    const int nq = K / 32, G = K / kGroup;

    Quarter v = {};
    uint32_t amax = 0;
    for (int c = t; c < nq; c += threads) {
        v = load_quarter(row + 32 * c);
        const uint32_t cm = quarter_absmax_bits(v);
        amax = cm > amax ? cm : amax;
        if constexpr (!LOOP) break;
    }
    amax = wave_max_dpp(amax);
    if ((t & 63) == 0) red[t >> 6] = amax;
    __syncthreads();
    for (int w = 0; w < threads / 64; ++w) amax = red[w] > amax ? red[w] : amax;

    constexpr int qmax = A8 ? kQmax8 : kQmax;
    const uint16_t sb = scale_bits_from_amax(half_bits_to_float((uint16_t)amax), qmax);
    float s = half_bits_to_float(sb);
    float inv_s = s == 0.0f ? 0.0f : 1.0f / s;              // a zero scale: all codes 0
    if (t == 0) s_x[m] = sb;
    const bool finite = amax < kHalfInf;
    if (!finite) nonfinite_scale<A8>(s, inv_s);

    for (int c = t; c < nq; c += threads) {
        if constexpr (LOOP) v = load_quarter(row + 32 * c);
        if (!finite) nonfinite_quarter<A8>(v, amax);
        float q[32];
        quarter_codes(v, s, inv_s, (float)qmax, q);
        const int g = c >> 2, j = c & 3;                    // quarter j of group g
        if constexpr (A8) {
            // x = 8 h + l: the e4m3 bytes of h = floor(x / 8) in the high plane (piece (row, group)
            // of 128 bytes at (g M + m) 128, chunks placed by hi_chunk_offset), the folded 4-bit
            // codes l in [0, 7] in the low plane (M K bytes on, the W4A4 group order)
            uint32_t hb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
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
            *reinterpret_cast<uint4*>(hi + hi_chunk_offset(2 * j)) = make_uint4(hb[0], hb[1], hb[2], hb[3]);
            *reinterpret_cast<uint4*>(hi + hi_chunk_offset(2 * j + 1)) = make_uint4(hb[4], hb[5], hb[6], hb[7]);
            *reinterpret_cast<uint4*>(Xq + (int64_t)M * K + piece_offset(M, m, g) + 16 * j) =
                make_uint4(d[0] | (d[2] & kFoldA), d[1] | (d[2] & kFoldB), d[3] | (d[5] & kFoldA), d[4] | (d[5] & kFoldB));
        } else {
            const u32x6 d = operand_dwords(q);
            *reinterpret_cast<uint4*>(Xq + act_main_offset(M, m, g) + 16 * j) = make_uint4(d[0], d[1], d[2], d[3]);
            *reinterpret_cast<uint2*>(Xq + act_tail_offset(M, G, m, g, j)) = make_uint2(d[4], d[5]);
        }
        if constexpr (!LOOP) break;
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
    const int quarters = K / 32, threads = (quarters + 63) / 64 * 64;
    if (threads <= kActMaxThreads)
        hipLaunchKernelGGL((act_quant_kernel<A8, false>), dim3(M), dim3(threads), 0, stream, x, M, K, ldx, Xq, s);
    else
        hipLaunchKernelGGL((act_quant_kernel<A8, true>), dim3(M), dim3(kActMaxThreads), 0, stream, x, M, K, ldx, Xq, s);
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
