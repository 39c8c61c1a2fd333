// The GEMM kernel over tiled weights for medium M and for outputs too small to fill the chip with the large-M kernel's tiles:
// the waves of a workgroup split K, weights go from memory to registers, one barrier per 512 or 1024 k.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace w4a8 {

namespace {

typedef __attribute__((address_space(3))) void *medium_lds_t;

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_medium_loads() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// LDS: two stages of the activations, or the exchange of the k groups' sums that takes their place
constexpr int medium_lds_bytes(int mt, int nt, int nw, int kg) {
    const int stages = 2 * kg * mt * 2048, exchange = (kg - 1) * nw * mt * nt * 1024;
    return stages > exchange ? stages : exchange;
}

}  // namespace

// NW x KG waves: NW side by side along N, each 16 MT tokens x 16 NT channels, and KG groups along K: k step (128 k) number
// KG s + kg of stage s is multiplied by group kg, and the groups' integer sums meet in LDS at the end.
//
// Why: with 64-row tiles the large-M kernel spends its time per stage of 128 k on the handover between stages, and on every
// weight byte twice in LDS.  Here a stage is KG times as long, so there are KG times fewer barriers; a weight fragment is
// loaded into the registers of the one wave that uses it (a lane's 16 bytes of a tiled block are an operand of both MFMA
// steps of a k step), its successor being requested as soon as it has been converted; and an output too narrow for a tile
// per compute unit is cut finer instead of along K over workgroups, which costs slabs of sums and a second launch.
// What bounds it: the bytes a compute unit brings in, (BM + BN / 2) K, at 56 to 77 KB/us while the weights come from memory and 79 to
// 90 from the memory-side cache, which is the reason for the shapes (near square in bytes, one per compute unit); and 3 to 5 us of
// launch, exchange and epilogue.  That rate is no limit of the memory (3.3 TB/s): a fragment is requested one stage ahead of its
// use, and a stage, 64 KB for 64 x 128, lasts as long as its loads take to arrive, 1.17 us.
template <int MT, int NT, int NW, int KG, bool ACC_OUT, int WBITS, bool SWIGLU, bool NOT_KEPT>
__global__ __launch_bounds__(64 * NW * KG, MT * NT <= 12 && WBITS == 4 ? 4 : 2) void gemm_medium_kernel(W4A8_PREFILL_PARAMS) {
    const PrefillArgs p = prefill_args<16 * MT, 16 * NT * NW>(W4A8_PREFILL_PARAM_NAMES);
    static_assert(!SWIGLU || (WBITS == 4 && !ACC_OUT), "fused SiLU * up: int4 weights, fp16 output");
    constexpr bool W8 = WBITS == 8;
    constexpr int WAVES = NW * KG, BM = 16 * MT, BN = 16 * NT * NW;
    constexpr int kBlock = kTiledBlockK * 32 * WBITS / 8;
    constexpr int WV = W8 ? 2 : 1;  // 16-byte pieces of a lane's weight fragment per k step
    constexpr int kStep = MT * 2048, kStage = KG * kStep;
    constexpr int A_LOADS = KG * MT * 2 / WAVES, W_LOADS = NT * WV;
    static_assert(A_LOADS * WAVES == KG * MT * 2, "every wave issues the same number of activation loads: the waits count on it");
    static_assert(WAVES * 64 >= BM && WAVES * 64 >= BN, "one thread per row and per channel of the tile");
    constexpr int kWeightPolicy = NOT_KEPT ? 2 : 0;  // non-temporal, where launch_medium_one says so
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int idx = lane & 15;  // row of a 16-row operand tile
    const int g = lane >> 4;    // K group
    const int kg = wave / NW, wn = wave % NW;

    // XCD-aware tile order, as in the large-M kernel: consecutive tiles of one XCD share their weights
    const int total = p.tiles_m * p.tiles_n;
    const int per_xcd = (total + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= total) return;
    const int tile_n = logical / p.tiles_m;
    const int bm0 = (logical - tile_n * p.tiles_m) * BM;
    const int bn0 = tile_n * BN;

    // the epilogue's scales ride in two registers through the main loop
    float sa_mine = 0.f, sw_mine = 0.f;
    if (!ACC_OUT) {
        if (tid < BM && bm0 + tid < p.M) sa_mine = p.s_a[bm0 + tid];
        if (tid < BN && bn0 + tid < p.N) sw_mine = p.s_w[bn0 + tid];
    }

    const int steps = (p.K + kTiledBlockK - 1) / kTiledBlockK;
    const int nb_total = (p.N + 31) >> 5;
    const unsigned w_bytes = (unsigned)((size_t)nb_total * steps * kBlock);
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)p.xq, 0, (unsigned)((size_t)p.M * p.K), 0x00020000);

    // Activation wave load L of a stage: rows 8 l .. 8 l + 7 of its k step L / (2 MT), l = L % (2 MT), whole 128-byte lines;
    // lane -> row 8 l + lane / 8, 16-byte slot lane % 8, which receives the row's piece slot ^ fx(row),
    // fx(row) = (row & 7) ^ ((row >> 3) & 1).  Rows past M, k past K and steps past the last one have offsets beyond the buffer
    // (the launcher sees to M K < 2^30): such a lane fetches nothing and delivers zeros.
    constexpr unsigned kNoRow = 0x40000000u, kNoStep = 0x80000000u, kNowhere = 0xFFFFFFF0u;
    unsigned x_off[A_LOADS];
    bool x_last_ok[2];  // of the two pieces a lane ever loads, by the parity of l
#pragma unroll
    for (int i = 0; i < 2; ++i) x_last_ok[i] = (steps - 1) * kTiledBlockK + ((lane & 7) ^ (lane >> 3) ^ i) * 16 < p.K;
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) {
        const int l = (j * WAVES + wave) % (2 * MT);
        const int m = bm0 + 8 * l + (lane >> 3);
        x_off[j] = m < p.M ? (unsigned)m * (unsigned)p.K + ((lane & 7) ^ (lane >> 3) ^ (l & 1)) * 16 : kNoRow;
    }
    auto stage = [&](int s, int slot) {
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {
            const int L = j * WAVES + wave, step = s * KG + L / (2 * MT);
            const unsigned k0 = step < steps ? (unsigned)step * kTiledBlockK : kNoStep;
            const bool cut = step + 1 == steps && !x_last_ok[(L % (2 * MT)) & 1];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (medium_lds_t)(lds + slot * kStage + L * 1024), 16,
                                                     (int)(cut ? kNowhere : x_off[j] + k0), 0, 0, 0);
        }
    };
    // A lane's weights of a k step: chunk g of its channel's row of the block (int4: the codes of both MFMA steps), or chunks
    // 2 g and 2 g + 1 (int8).  Step h of the two multiplies k = 32 g + 16 h .. + 15, piece 2 g + h of an activation row.
    // Channels that do not exist lie beyond the buffer with either piece's offset added.
    constexpr unsigned kNoChannel = kNowhere - 512u * (WV - 1);
    static_assert(kNoChannel + 512u * (WV - 1) + 15u >= kNoChannel && kNoChannel >= kMediumMaxWeights, "offsets must not come round to the buffer's start");
    unsigned w_off[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = bn0 + 16 * (wn * NT + t), nb = n >> 5;
        w_off[t] = nb < nb_total ? (unsigned)nb * (unsigned)(steps * kBlock) + (unsigned)((n & 16) + idx) * 16u + (unsigned)g * (512u * WV)
                                 : kNoChannel;
    }
    v4u wreg[NT][WV];
    auto w_load = [&](int s, int t) {
        const int step = s * KG + kg;
        // a step past the last one fetches nothing and delivers zeros: its buffer has no bytes
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, step < steps ? w_bytes : 0u, 0x00020000);
#pragma unroll
        for (int h = 0; h < WV; ++h)
            wreg[t][h] = __builtin_amdgcn_raw_buffer_load_b128(rs, w_off[t] + h * 512, step < steps ? step * kBlock : 0, kWeightPolicy);
    };

    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mt][t] = v4i{0, 0, 0, 0};

    auto lds_barrier = [] {  // orders LDS only: the loads in flight stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    __builtin_amdgcn_sched_barrier(0);
    stage(0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) w_load(0, t);
    __builtin_amdgcn_sched_barrier(0);
    const int fxr = (idx & 7) ^ (idx >> 3);
    const int stages = (steps + KG - 1) / KG;
    for (int s = 0; s < stages; ++s) {
        // Outstanding, in this order: the stage's activations, the stage's weights.  Loads return in order, so with the
        // weights allowed to be outstanding this wave's part of the activations is in; behind the barrier everyone's is, and
        // everyone has multiplied the stage before, whose slot takes the next one.
        wait_medium_loads<W_LOADS>();
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        stage(s + 1, (s + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t *const rows = lds + (s & 1) * kStage + kg * kStep + idx * 128;
        v4u x[MT][2];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int h = 0; h < 2; ++h) x[mt][h] = *(const v4u *)(rows + mt * 2048 + (((2 * g + h) ^ fxr) << 4));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            v4i w[2];
            if constexpr (W8) {
                w[0] = __builtin_bit_cast(v4i, wreg[t][0]);
                w[1] = __builtin_bit_cast(v4i, wreg[t][WV - 1]);
            } else {
                // convert first, refill second: the old register is dead when the load that replaces it is issued
                w[0] = w_operand_tiled(wreg[t][0].x, wreg[t][0].y);
                w[1] = w_operand_tiled(wreg[t][0].z, wreg[t][0].w);
                __builtin_amdgcn_sched_barrier(0);
                w_load(s + 1, t);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][t] = mfma_i8_16x16x64(w[h], __builtin_bit_cast(v4i, x[mt][h]), acc[mt][t]);
            if constexpr (W8) {  // the fragment is the operand: it is replaced behind its MFMAs
                __builtin_amdgcn_sched_barrier(0);
                w_load(s + 1, t);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // The groups' sums meet: unit u = MT t + mt (16 x 16 outputs) of a wave's part is finished by group u % KG.
    float *const sa_lds = (float *)(lds + medium_lds_bytes(MT, NT, NW, KG));
    float *const sw_lds = sa_lds + BM;
    if (!ACC_OUT) {
        if (tid < BM) sa_lds[tid] = sa_mine;
        if (tid < BN) sw_lds[tid] = sw_mine;
    }
    constexpr int kUnits = MT * NT;
    v4i *const part = (v4i *)lds;  // [wn][unit][KG - 1][lane]
    wait_medium_loads<0>();        // the zeros of the stage past the last one
    lds_barrier();                 // the stages' memory is free
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const int at = (kg + KG - u % KG) % KG - 1;
        if (at >= 0) part[((wn * kUnits + u) * (KG - 1) + at) * 64 + lane] = acc[u % MT][u / MT];
    }
    lds_barrier();
    const bool vec_ok = (p.ldc & 3) == 0;
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        if (u % KG != kg) continue;
        const int t = u / MT, mt = u % MT;
        v4i s = acc[mt][t];
#pragma unroll
        for (int w = 0; w < KG - 1; ++w) s += part[((wn * kUnits + u) * (KG - 1) + w) * 64 + lane];
        const int m = bm0 + 16 * mt + idx, nl = 16 * (wn * NT + t) + 4 * g, n = bn0 + nl;
        if (m >= p.M || n >= p.N) continue;
        if constexpr (ACC_OUT) {
            int *dst = p.acc_out + (size_t)m * p.ldc + n;
            constexpr int kShift = W8 ? 0 : 4;  // int4: exact, every sum is a multiple of 16
            const v4i v = v4i{s.x >> kShift, s.y >> kShift, s.z >> kShift, s.w >> kShift};
            if (vec_ok && n + 3 < p.N) {
                *(v4i *)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < p.N) dst[e] = v[e];
            }
        } else {
            // Eq. (6),(7)
            const float sa = sa_lds[16 * mt + idx];
            const float4 sw = *(const float4 *)(sw_lds + nl);
            auto deq = [&](int a, float s_w) { return W8 ? (float)a * (sa * s_w) : dequant(a, sa, s_w); };
            const float o[4] = {deq(s.x, sw.x), deq(s.y, sw.y), deq(s.z, sw.z), deq(s.w, sw.w)};
            if constexpr (SWIGLU) {  // two (gate, up) pairs: N is a multiple of 4 and p.ldc of 2
                const unsigned gu0 = pack_f16x2(o[0], o[1]), gu1 = pack_f16x2(o[2], o[3]);
                unsigned short *dst = (unsigned short *)p.out + (size_t)m * p.ldc + (n >> 1);
                *(unsigned *)dst = pack_f16x2(silu_mul_f32(lo_half(gu0), hi_half(gu0)), silu_mul_f32(lo_half(gu1), hi_half(gu1)));
            } else {
                unsigned short *dst = (unsigned short *)p.out + (size_t)m * p.ldc + n;
                if (vec_ok && n + 3 < p.N) {
                    *(v2u *)dst = v2u{pack_f16x2(o[0], o[1]), pack_f16x2(o[2], o[3])};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < p.N) dst[e] = f32_to_f16_bits(o[e]);
                }
            }
        }
    }
}

namespace {

template <int MT, int NT, int NW, int KG, bool ACC_OUT, int WBITS, bool SWIGLU, bool NOT_KEPT>
hipError_t launch_medium_as(const PrefillArgs &p, hipStream_t stream) {
    constexpr int kLds = medium_lds_bytes(MT, NT, NW, KG) + 4 * (16 * MT + 16 * NT * NW);
    static_assert(kLds <= 160 * 1024, "a workgroup's stages and exchange must fit the compute unit's LDS");
    constexpr auto kernel = gemm_medium_kernel<MT, NT, NW, KG, ACC_OUT, WBITS, SWIGLU, NOT_KEPT>;
    if (const hipError_t e = allow_lds<kernel>(kLds); e != hipSuccess) return e;
    if (p.prepare_only) return hipSuccess;
    const int total = p.tiles_m * p.tiles_n;
    hipLaunchKernelGGL(kernel, dim3(8 * ((total + 7) / 8)), dim3(64 * NW * KG), kLds, stream, W4A8_PREFILL_LAUNCH_ARGS(p, ACC_OUT));
    return hipGetLastError();
}

template <int MT, int NT, int NW, int KG, bool ACC_OUT, int WBITS, bool SWIGLU>
hipError_t launch_medium_one(PrefillArgs p, hipStream_t stream) {
    constexpr int BM = 16 * MT, BN = 16 * NT * NW;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    // With eight k groups the weights are loaded with the non-temporal hint where the tile rows of a column all lie on one XCD, which
    // then fetches them once for its own L2 alone; a column that is cut between two XCDs is wanted again by the second.  Cold weights,
    // hint and none: N = 4351, K = 9888, M = 25 (one tile row) 10.4 us and 11.1; N = 1519, K = 12160, M = 53 (two, whole columns) 10.9 and
    // 11.5; N = 2076, K = 10528, M = 41 (two, cut) 11.2 and 10.65; N = 1082, K = 11104, M = 161 (six, cut) 11.2 and 10.75.  Over 260 shapes with one
    // to sixteen tile rows, int4 and int8, the rule takes the faster of the two each time (within 1 %).  The shapes with four k groups serve
    // larger M, where the hint costs up to 20 %.
    if constexpr (KG == 8) {
        if (p.prepare_only) {
            if (const hipError_t e = launch_medium_as<MT, NT, NW, KG, ACC_OUT, WBITS, SWIGLU, true>(p, stream); e != hipSuccess) return e;
        } else if ((p.tiles_m * p.tiles_n + 7) / 8 % p.tiles_m == 0) {
            return launch_medium_as<MT, NT, NW, KG, ACC_OUT, WBITS, SWIGLU, true>(p, stream);
        }
    }
    return launch_medium_as<MT, NT, NW, KG, ACC_OUT, WBITS, SWIGLU, false>(p, stream);
}

}  // namespace

}  // namespace w4a8
