// W4A8 GEMM for large M over weights in the tiled layout (which tile_weights.hip produces).
//
// Why another layout: for large M the kernel is bound by how fast a compute unit can pull its operand tiles out of
// L2.  A wave-wide 16-byte-per-lane load that touches 16 or 32 different cache lines (what a k slice of a row-major
// operand amounts to) moves well under half the bytes per cycle of one that touches 8 whole lines.  The activations
// can be read in whole lines as they are (a stage is 128 k = one 128-byte line per row).  The packed weights cannot
// (128 k of a row are 64 bytes), but they are static, so they are reordered once, after quantisation (the paper also
// fixes the weight format offline, Sec. 5.3), into 2 KB blocks that a stage consumes whole:
//
//   block (nb, kb) = output channels 32 nb .. 32 nb + 31, k = 128 kb .. 128 kb + 127, at byte ((nb * KB) + kb) * 2048,
//                    KB = ceil(K / 128); rows past N and k past K hold zero codes;
//   inside a block: 16-byte chunk (c, r), c = 0..3, r = 0..31, at (c * 32 + r) * 16 holds the 32 codes
//                    k = 128 kb + 32 c .. + 31 of channel 32 nb + r;
//   inside a dword (8 codes k0..k7): nibbles, low to high, hold k0 k4 k1 k5 k2 k6 k3 k7, so that
//                    (w << 4) & 0xF0F0F0F0 is {16 k0 .. 16 k3} and w & 0xF0F0F0F0 is {16 k4 .. 16 k7} as int8:
//                    the conversion of Fig. 4(c) then lands in the activations' natural k order and the
//                    activation bytes need no shuffling at all.
//
// The 16 lanes of a K group of an MFMA operand read 256 consecutive bytes of a block: no LDS bank conflicts, no swizzle.
//
// Matrix instruction: v_mfma_i32_16x16x64_i8.  At large M the chip holds its clock to a power limit, and per operation
// the 16x16x64 form touches half the accumulator registers of the 32x32x32 form: a register-resident loop on random
// int8 activations and multiples of 16 as weights runs at 4.5 POP/s with it and at 3.6 with 32x32x32 (4.8 and 4.6 on
// constant operands, where power does not bind).  In this kernel, N = 8192, K = 28672, M = 2048: 326 us before (32x32x32),
// 278 us now; N = 27648, K = 5120, M = 1024: 123 before, 102 now.  What bounds it then: in the 256 x 256 tile the matrix
// cores, 80 % busy at 2.1 GHz; in the smaller tiles the vector issue slots of the conversion (6 operations per weight
// fragment and wave, for MT MFMAs of four issue slots each) and the LDS reads.
//
// Kernel structure: a ring of STAGES stages of 128 k in LDS, filled by LDS-direct buffer loads (1 KB per wave
// instruction: 8 activation rows x 128 B, or half a weight block).  Stage t + STAGES is requested as soon as every
// wave has taken its last fragment of stage t, so STAGES - 1 stages are in flight while one is being multiplied.
// One workgroup barrier per stage; fragments are always read a block of MFMAs ahead of their use.
#include "gemm_prefill_ring.hpp"

namespace w4a8 {

namespace {

// The fused SiLU * up form of a tile: one launch covers the problem (byte offsets below 2^32 are the caller's check).
template <int MT, int NT, int WM, int WN, int STAGES>
hipError_t launch_tile_swiglu(PrefillArgs p, hipStream_t stream) {
    constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    const int total = p.tiles_m * p.tiles_n;
    return launch_one<MT, NT, WM, WN, STAGES, false, 4, false, false, 1, true>(p, dim3(8 * ((total + 7) / 8)), stream);
}

}  // namespace

// Second half of a GEMM whose K was split over workgroups: adds the slabs of raw sums and applies Eq. (6),(7).
// Integer addition in any order gives the same sum, so the result has the bits of the unsplit kernel.
// What bounds it is latency: a thread has four channels of a row, one load from each slab.  SPLITS slabs, known at compile time, are
// asked for at once; 0: any number, one behind the other (a loop that waits at every slab, which this kernel was for any number, with a
// 64-bit division per thread in front: GEMM and sum of N = 5120, K = 13824, M = 128 in six slices 21.0 -> 20.8 us, of N = 1502,
// K = 12032, M = 50, whose channels are read one by one, 10.7 -> 9.4).  A row takes whole workgroups of 1024 channels: a narrow output leaves
// most of one idle and is no slower for it (before and now, with the GEMM: N = 64, K = 16736, M = 123 11.4 us and 10.2, N = 1232,
// K = 29376, M = 499 30.4 and 29.5, N = 1056, K = 13824, M = 16 level).
template <int SPLITS>
__global__ __launch_bounds__(256) void splitk_epilogue_kernel(const int *__restrict__ part, const float *__restrict__ s_a,
                                                              const float *__restrict__ s_w, unsigned short *__restrict__ out, int M, int N,
                                                              int splits) {
    const int n = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;
    if (n >= N) return;
    const size_t slab = (size_t)M * N;
    for (int m = blockIdx.y; m < M; m += gridDim.y) {
        const size_t at = (size_t)m * N + n;
        const float sa = s_a[m];
        if ((N & 3) == 0) {
            const float4 sw = *(const float4 *)(s_w + n);
            v4i s = *(const v4i *)(part + at);
            if constexpr (SPLITS > 0) {
                v4i t[SPLITS];
#pragma unroll
                for (int i = 1; i < SPLITS; ++i) t[i] = *(const v4i *)(part + i * slab + at);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 1; i < SPLITS; ++i) s += t[i];
            } else {
                for (int i = 1; i < splits; ++i) s += *(const v4i *)(part + i * slab + at);
            }
            v2u o;
            o.x = pack_f16x2((float)s.x * (sa * sw.x), (float)s.y * (sa * sw.y));
            o.y = pack_f16x2((float)s.z * (sa * sw.z), (float)s.w * (sa * sw.w));
            *(v2u *)(out + at) = o;
        } else {
            const int count = SPLITS > 0 ? SPLITS : splits;
            for (int j = 0; j < 4 && n + j < N; ++j) {
                int s = 0;
#pragma unroll SPLITS > 0 ? SPLITS : 1
                for (int i = 0; i < count; ++i) s += part[i * slab + at + j];
                out[at + j] = f32_to_f16_bits((float)s * (sa * s_w[n + j]));
            }
        }
    }
}

hipError_t launch_splitk_epilogue(const int *part, int splits, const float *s_a, const float *s_w, void *out, int M, int N,
                                  hipStream_t stream) {
    const dim3 grid(((unsigned)N + 1023) / 1024, (unsigned)(M < 65535 ? M : 65535));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, part, s_a, s_w, (unsigned short *)out, M, N, splits);
        return hipGetLastError();
    };
    switch (splits) {  // the library's own choice goes up to eight
        case 2: return launch(splitk_epilogue_kernel<2>);
        case 3: return launch(splitk_epilogue_kernel<3>);
        case 4: return launch(splitk_epilogue_kernel<4>);
        case 5: return launch(splitk_epilogue_kernel<5>);
        case 6: return launch(splitk_epilogue_kernel<6>);
        case 7: return launch(splitk_epilogue_kernel<7>);
        case 8: return launch(splitk_epilogue_kernel<8>);
        default: return launch(splitk_epilogue_kernel<0>);
    }
}

hipError_t launch_gemm_prefill_tiled(const PrefillArgs &p, bool acc_out, int tile, hipStream_t stream, int wbits) {
    // slices keep every byte offset inside the kernel below 2^32; slices of N start on a 32-channel block
    const long long kMaxBytes = 0xF0000000ll;
    const long long kb_total = (p.K + kTiledBlockK - 1) / kTiledBlockK;
    const long long block_bytes = (long long)kTiledBlockBytes * (wbits == 8 ? 2 : 1);
    if (wbits == kWeightsFineGrained4 && (p.K % kTiledBlockK != 0 || p.ldg < p.N || (p.ldg & 3) != 0 ||
                                          kb_total * (long long)p.ldg * 4 > kMaxBytes))
        return hipErrorInvalidValue;
    long long m_rows = kMaxBytes / p.K, n_rows = kMaxBytes / (kb_total * (block_bytes / 32));
    m_rows -= m_rows % 256;
    n_rows -= n_rows % 3840;  // a multiple of every tile width
    for (long long n0 = 0; n0 < p.N; n0 += n_rows) {
        for (long long m0 = 0; m0 < p.M; m0 += m_rows) {
            PrefillArgs q = p;
            q.M = (int)((p.M - m0) < m_rows ? (p.M - m0) : m_rows);
            q.N = (int)((p.N - n0) < n_rows ? (p.N - n0) : n_rows);
            q.xq = p.xq + (size_t)m0 * p.K;
            q.wp = p.wp + (size_t)(n0 / 32) * (size_t)kb_total * (size_t)block_bytes;
            if (p.s_a) q.s_a = p.s_a + m0;
            if (p.s_w) q.s_w = p.s_w + n0;
            if (p.out) q.out = (unsigned short *)p.out + (size_t)m0 * p.ldc + n0;
            if (p.acc_out) q.acc_out = p.acc_out + (size_t)m0 * p.ldc + n0;
            if (p.splits > 1 && (q.M != p.M || q.N != p.N)) return hipErrorInvalidValue;  // slabs are whole problems
            hipError_t e;
            if (wbits == 4) {
                switch (tile) {
                    case kTiled256x256: e = launch_tile<8, 4, 2, 4, 3>(q, acc_out, stream); break;
                    case kTiled256x256Square: e = launch_tile<4, 8, 4, 2, 3>(q, acc_out, stream); break;
                    case kTiled128x256: e = launch_tile<8, 4, 1, 4, 2>(q, acc_out, stream); break;
                    case kTiled128x160: e = launch_tile<2, 10, 4, 1, 3>(q, acc_out, stream); break;
                    case kTiled128x128: e = launch_tile<4, 4, 2, 2, 3>(q, acc_out, stream); break;
                    case kTiled64x128: e = launch_tile<2, 2, 2, 4, 4>(q, acc_out, stream); break;
                    case kTiled64x64: e = launch_tile<2, 2, 2, 2, 4>(q, acc_out, stream); break;
                    case kTiled32x128: e = launch_tile<2, 2, 1, 4, 4>(q, acc_out, stream); break;
                    case kTiled128x160K2: e = launch_tile<2, 10, 4, 1, 3, 4, false, false, 2>(q, acc_out, stream); break;
                    case kTiled128x128K2: e = launch_tile<4, 4, 2, 2, 3, 4, false, false, 2>(q, acc_out, stream); break;
                    case kTiled256x192: e = launch_tile<4, 6, 4, 2, 3>(q, acc_out, stream); break;
                    case kTiled128x256W8: e = launch_tile<8, 2, 1, 8, 4>(q, acc_out, stream); break;
                    case kTiled64x256: e = launch_tile<4, 2, 1, 8, 4>(q, acc_out, stream); break;
                    case kTiled128x384: e = launch_tile<8, 3, 1, 8, 3>(q, acc_out, stream); break;
                    case kTiled128x192: e = launch_tile<4, 3, 2, 4, 4>(q, acc_out, stream); break;
                    case kTiled64x192: e = launch_tile<2, 3, 2, 4, 4>(q, acc_out, stream); break;
                    case kTiled128x320: e = launch_tile<4, 5, 2, 4, 4>(q, acc_out, stream); break;
                    case kTiled192x320: e = launch_tile<6, 5, 2, 4, 3>(q, acc_out, stream); break;
                    case kTiled192x256: e = launch_tile<6, 4, 2, 4, 3>(q, acc_out, stream); break;
                    case kTiled192x192: e = launch_tile<6, 3, 2, 4, 4>(q, acc_out, stream); break;
                    case kTiled256x320: e = launch_tile<8, 5, 2, 4, 3>(q, acc_out, stream); break;
                    case kTiled192x384: e = launch_tile<6, 6, 2, 4, 3>(q, acc_out, stream); break;
                    default: e = hipErrorInvalidConfiguration;
                }
            } else if (wbits == 8) {
                // int8 weight stages are twice as large: shallower rings for the same LDS
                switch (tile) {
                    case kTiled256x256: e = launch_tile<8, 4, 2, 4, 2, 8>(q, acc_out, stream); break;
                    case kTiled256x256Square: e = launch_tile<4, 8, 4, 2, 2, 8>(q, acc_out, stream); break;
                    case kTiled128x256: e = launch_tile<8, 4, 1, 4, 2, 8>(q, acc_out, stream); break;
                    case kTiled128x160: e = launch_tile<2, 10, 4, 1, 2, 8>(q, acc_out, stream); break;
                    case kTiled128x128: e = launch_tile<4, 4, 2, 2, 2, 8>(q, acc_out, stream); break;
                    case kTiled64x128: e = launch_tile<2, 4, 2, 2, 3, 8>(q, acc_out, stream); break;
                    case kTiled64x64: e = launch_tile<2, 2, 2, 2, 4, 8>(q, acc_out, stream); break;
                    case kTiled32x128: e = launch_tile<2, 2, 1, 4, 3, 8>(q, acc_out, stream); break;
                    case kTiled128x256W8: e = launch_tile<8, 2, 1, 8, 3, 8>(q, acc_out, stream); break;
                    case kTiled128x192: e = launch_tile<4, 3, 2, 4, 3, 8>(q, acc_out, stream); break;
                    case kTiled64x192: e = launch_tile<2, 3, 2, 4, 4, 8>(q, acc_out, stream); break;
                    case kTiled192x192: e = launch_tile<6, 3, 2, 4, 3, 8>(q, acc_out, stream); break;
                    default: e = hipErrorInvalidConfiguration;
                }
            } else if (wbits == kWeightsUnsigned4) {
                switch (tile) {
                    case kTiled256x256: e = launch_tile<8, 4, 2, 4, 3, 4, true>(q, acc_out, stream); break;
                    case kTiled256x256Square: e = launch_tile<4, 8, 4, 2, 3, 4, true>(q, acc_out, stream); break;
                    case kTiled128x256: e = launch_tile<8, 4, 1, 4, 2, 4, true>(q, acc_out, stream); break;
                    case kTiled128x160: e = launch_tile<2, 10, 4, 1, 3, 4, true>(q, acc_out, stream); break;
                    case kTiled128x128: e = launch_tile<4, 4, 2, 2, 3, 4, true>(q, acc_out, stream); break;
                    case kTiled64x128: e = launch_tile<2, 4, 2, 2, 4, 4, true>(q, acc_out, stream); break;
                    case kTiled64x64: e = launch_tile<2, 2, 2, 2, 4, 4, true>(q, acc_out, stream); break;
                    case kTiled32x128: e = launch_tile<2, 2, 1, 4, 4, 4, true>(q, acc_out, stream); break;
                    default: e = hipErrorInvalidConfiguration;
                }
            } else if (wbits == kWeightsFineGrained4) {
                // one problem, one launch: the group scales are addressed with the whole problem's pitch
                if (q.M != p.M || q.N != p.N) return hipErrorInvalidValue;
                switch (tile) {
                    case kFine128x256: e = launch_tile<4, 4, 2, 4, 3, 4, false, true>(q, acc_out, stream); break;
                    case kFine256x128: e = launch_tile<4, 4, 4, 2, 3, 4, false, true>(q, acc_out, stream); break;
                    case kFine128x128: e = launch_tile<4, 4, 2, 2, 3, 4, false, true>(q, acc_out, stream); break;
                    case kFine64x128: e = launch_tile<2, 4, 2, 2, 4, 4, false, true>(q, acc_out, stream); break;
                    case kFine64x64: e = launch_tile<2, 2, 2, 2, 4, 4, false, true>(q, acc_out, stream); break;
                    case kFine32x128: e = launch_tile<2, 2, 1, 4, 4, 4, false, true>(q, acc_out, stream); break;
                    default: e = hipErrorInvalidConfiguration;
                }
            } else {
                e = hipErrorInvalidConfiguration;
            }
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_gemm_prefill_tiled_swiglu(const PrefillArgs &p, int tile, hipStream_t stream) {
    // p.N interleaved channels (even), p.out = h with pitch p.ldc (a multiple of 4 elements: the 8-byte stores of four
    // values are aligned)
    const long long kMaxBytes = 0xF0000000ll;
    const long long kb_total = (p.K + kTiledBlockK - 1) / kTiledBlockK;
    if ((p.N & 1) || (p.ldc & 3) || (long long)p.M * p.K > kMaxBytes ||
        (long long)((p.N + 31) / 32) * kb_total * kTiledBlockBytes > kMaxBytes)
        return hipErrorInvalidValue;
    switch (tile) {
        case kTiled256x256: return launch_tile_swiglu<8, 4, 2, 4, 3>(p, stream);
        case kTiled128x256: return launch_tile_swiglu<8, 4, 1, 4, 2>(p, stream);
        case kTiled64x128: return launch_tile_swiglu<2, 2, 2, 4, 4>(p, stream);
        case kTiled64x64: return launch_tile_swiglu<2, 2, 2, 2, 4>(p, stream);
        case kTiled32x128: return launch_tile_swiglu<2, 2, 1, 4, 4>(p, stream);
        case kTiled128x256W8: return launch_tile_swiglu<8, 2, 1, 8, 4>(p, stream);
        case kTiled64x256: return launch_tile_swiglu<4, 2, 1, 8, 4>(p, stream);
        case kTiled128x384: return launch_tile_swiglu<8, 3, 1, 8, 3>(p, stream);
        case kTiled128x192: return launch_tile_swiglu<4, 3, 2, 4, 4>(p, stream);
        case kTiled64x192: return launch_tile_swiglu<2, 3, 2, 4, 4>(p, stream);
        case kTiled128x320: return launch_tile_swiglu<4, 5, 2, 4, 4>(p, stream);
        case kTiled192x320: return launch_tile_swiglu<6, 5, 2, 4, 3>(p, stream);
        case kTiled192x256: return launch_tile_swiglu<6, 4, 2, 4, 3>(p, stream);
        case kTiled192x192: return launch_tile_swiglu<6, 3, 2, 4, 4>(p, stream);
        case kTiled256x320: return launch_tile_swiglu<8, 5, 2, 4, 3>(p, stream);
        case kTiled192x384: return launch_tile_swiglu<6, 6, 2, 4, 3>(p, stream);
        default: return hipErrorInvalidConfiguration;
    }
}

hipError_t prepare_tiled_kernels() {
    PrefillArgs a{};
    a.M = 32; a.N = 32; a.K = kTiledBlockK; a.ldc = 32; a.ldg = 32;
    a.prepare_only = true;
    for (int tile : {kTiled256x256, kTiled128x256, kTiled64x128, kTiled64x64, kTiled32x128, kTiled128x256W8, kTiled64x256, kTiled128x384,
                     kTiled128x192, kTiled64x192, kTiled128x320, kTiled192x320, kTiled192x256, kTiled192x192, kTiled256x320, kTiled192x384})
        if (const hipError_t e = launch_gemm_prefill_tiled_swiglu(a, tile, nullptr); e != hipSuccess) return e;
    for (int tile : {kTiled128x256W8, kTiled128x192, kTiled64x192, kTiled192x192})  // int8 weights, beside 1 .. kTiledTileMax
        for (int acc = 0; acc <= 1; ++acc)
            if (const hipError_t e = launch_gemm_prefill_tiled(a, acc != 0, tile, nullptr, 8); e != hipSuccess) return e;
    for (int tile : {kTiled256x320, kTiled192x384})  // int4 weights, beside 1 .. kTiledTileLast
        for (int acc = 0; acc <= 1; ++acc)
            if (const hipError_t e = launch_gemm_prefill_tiled(a, acc != 0, tile, nullptr, 4); e != hipSuccess) return e;
    struct Format { int wbits, tiles; bool acc; };
    const Format formats[] = {{4, kTiledTileLast, true}, {8, kTiledTileMax, true}, {kWeightsUnsigned4, kTiledTileMax, true},
                              {kWeightsFineGrained4, kFineTileMax, false}};
    for (const Format &f : formats)
        for (int tile = 1; tile <= f.tiles; ++tile)
            for (int acc = 0; acc <= (f.acc ? 1 : 0); ++acc) {
                const hipError_t e = launch_gemm_prefill_tiled(a, acc != 0, tile, nullptr, f.wbits);
                if (e != hipSuccess) return e;
            }
    return hipSuccess;
}

size_t tiled_weight_bytes(int N, int K, int wbits) {
    return (size_t)((N + 31) / 32) * (size_t)((K + kTiledBlockK - 1) / kTiledBlockK) * (size_t)(kTiledBlockBytes * wbits / 4);
}

}  // namespace w4a8
