// The large-M W4A8 GEMM kernel: output tiles fed through a ring of LDS-direct loads.  Included by gemm_prefill_tiled.hip
// (weights in the tiled layout, every format) and gemm_prefill_row.hip (int4 weights in the row-major storage format).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace w4a8 {

namespace {

typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kStageK = kTiledBlockK;

// Swizzle of the eight 16-byte slots of a 128-byte activation row in LDS: 8 as well as 16 consecutive rows reading
// the same logical slot fall into different banks.
__device__ __forceinline__ int fx(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// ROW: the same for the four 16-byte slots of a channel's 64 bytes (four channels span all the banks)
__device__ __forceinline__ int fw(int row) { return (row >> 2) & 3; }

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The same for the unsigned storage: each nibble holds u = w + 8 and the subtraction happens here, on four bytes at
// a time: (u + 0x78) ^ 0x80 is u - 8 as a two's-complement byte, and u + 0x78 <= 0x87 never carries into the next byte.
__device__ __forceinline__ v4i u_operand_tiled(unsigned w0, unsigned w1) {
    auto minus8 = [](unsigned bytes) { return (int)((bytes + 0x78787878u) ^ 0x80808080u); };
    v4i r;
    r.x = minus8(w0 & 0x0F0F0F0Fu);
    r.y = minus8((w0 >> 4) & 0x0F0F0F0Fu);
    r.z = minus8(w1 & 0x0F0F0F0Fu);
    r.w = minus8((w1 >> 4) & 0x0F0F0F0Fu);
    return r;
}

}  // namespace

// WBITS = 4: the W4A8 kernel over the tiled layout.  WBITS = 8: the W8A8 comparison variant (the paper's Table 4 sets its
// W4A8 against W8A8): int8 weight codes in blocks of 32 channels x 128 k = 4 KB, chunk (c, r), c = 0..7, at
// (c * 32 + r) * 16 holding k = 128 kb + 16 c .. + 15 of channel 32 nb + r; a fragment is an MFMA operand as it is.
// UNS (with WBITS = 4): the "vanilla" unsigned storage the paper measures FastGEMM against (Sec. 5.3, App. A.1,
// Fig. 4(b), "Asym GEMM" of Sec. 7.2): the nibbles hold u = w + 8 and 8 is subtracted from every byte after
// unpacking, 7 VALU operations per 8 weights instead of 3; the sums are then true sums, not sixteen-fold ones.
// FG (with WBITS = 4, signed): the fine-grained recipe the paper argues against (Eq. (5), Fig. 2(b), Sec. 7.2): one
// weight scale per group of 128 k and channel, p.s_w = s_g[K / 128][p.ldg].  A stage of the ring is exactly one
// group, so every stage starts its integer sums from zero and ends by folding them, converted to fp32 and multiplied
// by the group's scales, into a second, floating-point set of accumulators: per MFMA 8 extra VALU operations, twice
// the accumulator registers (which rules out the 256 x 256 tile), and one more 16-byte load per wave and stage (each
// wave brings in the 16 NT scales it needs itself, next to its share of the operands).
// KS = 2 (signed int4, per-channel scales only): two sets of WM x WN waves share the output tile and split every
// stage's k between them (set ks takes MFMA step ks); their
// integer sums meet in LDS before the epilogue.  For tiles that a compute unit holds only once (N too small for
// more workgroups) this doubles the waves per SIMD without shrinking the tile.
// SWIGLU (signed int4, per-channel scales, fp16 output): the channels are gate and up projections interleaved
// (channel 2 i = gate_i, 2 i + 1 = up_i) and the epilogue stores h_i = fp16(silu(fp16 gate_i) * fp16 up_i) instead of the
// two values: the glue between the gate+up and the down projection done where its inputs are produced (the fusion
// across operators of Sec. 6.1).  p.out is then h [M][p.ldc], p.ldc = channels / 2; same bits as silu_mul_kernel
// gives on the unfused output.
// ROW (signed int4, per-channel scales): p.wp is the packed row-major array [N][K / 2].  128 k of a channel are 64
// contiguous bytes, so a wave load takes 16 channels x 64 B; in LDS a channel keeps its 64 bytes, the four 16-byte chunks
// swizzled by the channel (fw, applied on the global side) so that the 16 channels of a K group fall into different banks.
// Chunk g holds the 32 codes of K group g as in a tiled block, but with even and odd k in the low and high nibbles: the
// conversion is the same bit operations, and the activation fragments are brought into that k order in registers
// (x_operand, four byte permutations each), behind the MFMAs of the channel tile before their first use.
// What bounds it: as over the tiled layout, plus the address unit, since a weight load touches 16 half lines where a
// block's touches 8 whole ones.  Measured, N = 15360, K = 5120, M = 777: 60.6 us (192 x 320 tile) against 80 with 128 x 256
// tiles of 32x32x32 MFMAs staged through registers; N = 26688, K = 6944, M = 43: 35 us against 80 for weight streaming.
template <int MT, int NT, int WM, int WN, int STAGES, bool ACC_OUT, int WBITS = 4, bool UNS = false, bool FG = false,
          int KS = 1, bool SWIGLU = false, bool ROW = false>
__global__ __launch_bounds__(64 * WM * WN * KS, 2) void gemm_prefill_tiled_kernel(W4A8_PREFILL_PARAMS) {
    const PrefillArgs p = prefill_args<16 * MT * WM, 16 * NT * WN>(W4A8_PREFILL_PARAM_NAMES);
    static_assert(!SWIGLU || (WBITS == 4 && !UNS && !FG && !ACC_OUT), "fused SiLU * up: the plain W4A8 kernel, fp16 output");
    static_assert(KS == 1 || (KS == 2 && WBITS == 4 && !UNS && !FG && STAGES == 3), "k split: the plain W4A8 kernel only");
    static_assert(!ROW || (WBITS == 4 && !UNS && !FG && !SWIGLU && KS == 1), "row-major storage: the plain W4A8 kernel");
    static_assert(WBITS == 4 || WBITS == 8, "int4 or int8 weight codes");
    static_assert(!UNS || WBITS == 4, "the unsigned storage is a 4-bit format");
    static_assert(!FG || (WBITS == 4 && !UNS && !ACC_OUT), "group scales: signed int4 codes, fp16 output");
    constexpr bool W8 = WBITS == 8;
    constexpr bool kTrueSums = W8 || UNS;  // else every sum is sixteen times the true one
    constexpr int kBlock = kTiledBlockK * 32 * WBITS / 8;  // bytes of a weight block: 2 KB or 4 KB
    constexpr int kParts = kBlock / 1024;                  // wave loads per block
    constexpr int kOutWaves = WM * WN;     // waves that own a part of the output tile
    constexpr int kWaves = kOutWaves * KS;
    constexpr int BM = 16 * MT * WM;
    constexpr int BN = 16 * NT * WN;
    static_assert(BM % 32 == 0 && BN % 32 == 0, "the tile is whole weight blocks wide");
    constexpr int A_TOTAL = BM / 8;                 // wave loads (8 rows x 128 B) of an activation stage
    constexpr int B_TOTAL = (BN / 32) * kParts;     // wave loads (1 KB of a weight block) of a weight stage
    static_assert(A_TOTAL % kWaves == 0 && (kWaves & 1) == 0, "activation loads must split evenly over an even wave count");
    constexpr int A_LOADS = A_TOTAL / kWaves;
    constexpr int B_LOADS = (B_TOTAL + kWaves - 1) / kWaves;
    constexpr bool kRagged = B_LOADS * kWaves != B_TOTAL;
    constexpr int kLoads = A_LOADS + B_LOADS + (FG ? 1 : 0);  // per wave and stage, the same for every wave: the waits count on it
    constexpr int A_STAGE = BM * 128;
    constexpr int B_STAGE = (BN / 32) * kBlock;
    constexpr int kBBase = STAGES * A_STAGE;
    constexpr int kSpare = STAGES * (A_STAGE + B_STAGE);  // 1 KB that absorbs the surplus loads of an uneven split
    constexpr int kScaleBase = kSpare + 1024;             // FG: per ring slot and wave, 16 NT group scales
    constexpr int kScaleWave = NT * 64;
    constexpr int kSlabRows = MT % 2 == 0 ? 32 : 16;      // rows that a wave turns around in LDS at a time in the epilogue
    // behind everything else: the tile's s_a and s_w for the epilogue (see below); mirrors launch_one's layout
    constexpr int kRingBytes = STAGES * (A_STAGE + B_STAGE) + 1024 + (FG ? STAGES * kOutWaves * NT * 64 + 1024 : 0);
    constexpr int kMeetBytes = KS == 2 ? kOutWaves * (kSlabRows * (32 * NT + 16) + MT * NT * 4 * 256) : 0;
    constexpr int kEpiScales = kRingBytes > kMeetBytes ? kRingBytes : kMeetBytes;
    static_assert(kWaves * 64 >= BM && kWaves * 64 >= BN, "one thread per row and per channel of the tile");
    static_assert(STAGES >= 2 && (STAGES - 1) * kLoads < 64, "outstanding loads must fit the counter");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: keeps LDS addresses in scalar registers
    const int ks = wave / kOutWaves;       // which half of every stage's k this wave multiplies (KS = 2)
    const int wsub = wave % kOutWaves;
    const int wm = wsub / WN;
    const int wn = wsub % WN;
    const int idx = lane & 15;  // row of a 16-row operand tile
    const int g = lane >> 4;    // K group

    // XCD-aware tile order: workgroup ids go round-robin over the 8 XCDs, and an XCD takes a run of consecutive tiles, column of tiles
    // by column within a group of tile rows: those that it has in flight share weight panels and activation rows in its L2.  A
    // panel is fetched once per group.
    const int total = p.tiles_m * p.tiles_n;
    const int per_xcd = (total + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= total) return;
    // An XCD works on some kAtOnce tiles at a time, m tile rows by n columns of them, and pulls in m BM bytes of activations and
    // n BN WBITS / 8 of weights per k: least for m near kBestRows.  With more tile rows than that they are taken in groups.  Bytes
    // from the memory-side cache cost the clock at the power limit about three times what bytes from L2 do: N = 57344, K = 8192, M = 2048
    // 1175 MB and 940, N = 10240 319 and 151 (with the taller tile), N = 5120, M = 1024 as 128 x 192 108 and 93; the 70B layer 1207 us and
    // 1197.  kAtOnce: what the LDS of 32 compute units holds, three of the smallest tiles each.  (With two for every workgroup of
    // four waves 64 x 64 tiles of unsigned weights took nine tile rows in two groups: N = 3679, K = 6720, M = 521 32.1 us before there were
    // groups, then 37.8, now 31.8.)
    constexpr int kAtOnce = 32 * (160 * 1024 / (kEpiScales + 4 * (BM + BN)));
    constexpr int kBestRows = [] {
        int m = 1;
        while (m * m * BM * 8 < kAtOnce * BN * WBITS) ++m;
        return m;
    }();
    int rows = p.tiles_m, row0 = 0, in_group = logical;
    const int groups = (p.tiles_m + kBestRows / 2) / kBestRows;
    if (groups > 1) {
        rows = (p.tiles_m + groups - 1) / groups;
        const int group = logical / (rows * p.tiles_n);
        in_group -= group * rows * p.tiles_n;
        row0 = group * rows;
        rows = min(rows, p.tiles_m - row0);
    }
    const int tile_n = in_group / rows;
    const int tile_m = row0 + in_group - tile_n * rows;
    const int bm0 = tile_m * BM;
    const int bn0 = tile_n * BN;

    // The epilogue needs s_a of the tile's rows and s_w of its channels.  Fetched there, each of its passes would
    // start with a trip to memory (measured: 5 to 10 us of epilogue per tile).  So they are requested here, ahead of
    // everything, ride in two registers through the main loop and are parked in LDS when the ring has gone idle.
    float sa_mine = 0.f, sw_mine = 0.f;
    if (!ACC_OUT) {
        if (tid < BM && bm0 + tid < p.M) sa_mine = p.s_a[bm0 + tid];
        if (!FG && tid < BN && bn0 + tid < p.N) sw_mine = p.s_w[bn0 + tid];
    }

    // Split of K across workgroups (p.splits > 1, raw sums only): blockIdx.y takes the stages
    // [st_begin, st_begin + st_total) and writes its partial sums to its own M x ldc slab of acc_out.
    const int st_all = (p.K + kStageK - 1) / kStageK;
    const int st_begin = ACC_OUT && p.splits > 1 ? (int)blockIdx.y * p.stages_per_split : 0;
    const int st_total = ACC_OUT && p.splits > 1 ? min(st_all - st_begin, p.stages_per_split) : st_all;
    const int k_last = (st_all - 1) * kStageK;
    const int nb_total = (p.N + 31) >> 5;

    constexpr unsigned kNowhere = 0xFFFFFFF0u;  // beyond every buffer: such a lane fetches nothing and delivers zeros
    auto make_rsrc = [](const void *base, size_t bytes) {
        const unsigned long long b = (unsigned long long)base;
        v4i r;
        r.x = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
        r.y = __builtin_amdgcn_readfirstlane((int)(unsigned)((b >> 32) & 0xFFFFu));
        r.z = __builtin_amdgcn_readfirstlane((int)(unsigned)bytes);
        r.w = 0x00020000;
        return r;
    };
    const v4i a_rsrc = make_rsrc(p.xq, (size_t)p.M * p.K);
    const v4i b_rsrc = make_rsrc(p.wp, ROW ? (size_t)p.N * (p.K >> 1) : (size_t)nb_total * st_all * kBlock);

    // Activation wave load L covers rows 8L .. 8L+7: lane -> row 8L + lane/8, physical slot lane%8, which receives
    // the logical chunk slot ^ fx(row).  With an even wave count fx(row) is the same for all loads of a lane.
    const int a_chunk = (lane & 7) ^ fx(8 * wave + (lane >> 3));
    const bool a_last_ok = k_last + a_chunk * 16 < p.K;
    unsigned a_off[A_LOADS], b_off[B_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        const int m = bm0 + 8 * (i * kWaves + wave) + (lane >> 3);
        a_off[i] = m < p.M ? (unsigned)m * (unsigned)p.K + a_chunk * 16 : kNowhere;
    }
    // Weight wave load L covers the 1 KB part L % kParts of the tile's 32-channel block L / kParts; ROW: channels
    // 16 L .. 16 L + 15, lane -> channel 16 L + lane / 4, physical slot lane % 4, the swizzle being the same for all L.
    const int b_chunk = (lane & 3) ^ fw(lane >> 2);
    const bool b_last_ok = !ROW || k_last + b_chunk * 32 < p.K;
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
        const int L = i * kWaves + wave;
        if constexpr (ROW) {
            const int n = bn0 + 16 * L + (lane >> 2);
            b_off[i] = (L < B_TOTAL && n < p.N) ? (unsigned)n * (unsigned)(p.K >> 1) + b_chunk * 16 : kNowhere;
            continue;
        }
        const int nb = (bn0 >> 5) + L / kParts;
        b_off[i] = (L < B_TOTAL && nb < nb_total)
                       ? ((unsigned)nb * (unsigned)st_all * kParts + (L % kParts)) * 1024u + lane * 16
                       : kNowhere;
    }
    // FG: lane L < 4 NT of every wave fetches the scales of channels n_wave + 4 L .. + 3 of the stage's group
    // (p.ldg is a multiple of 4, so a 16-byte run lies wholly inside a row of s_g or wholly outside)
    const v4i g_rsrc = FG ? make_rsrc(p.s_w, (size_t)st_all * (size_t)p.ldg * 4) : v4i{0, 0, 0, 0};
    const int g_n = bn0 + wn * (16 * NT) + 4 * lane;
    const unsigned g_off = (FG && g_n < p.ldg) ? (unsigned)g_n * 4u : kNowhere;

    // The load is written in assembly on purpose: the compiler orders LDS reads after every LDS-writing load it knows
    // of (it cannot tell the ring slots apart) and would wait for the stage just requested before each fragment read.
    // Here the ordering is explicit instead: wait_vmcnt + barrier before a slot is read, barrier before it is refilled.
    auto dma16 = [](const v4i &rsrc, unsigned lds_addr, unsigned voffset, int soffset) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset)
                     : "memory", "m0");
    };
    const unsigned lds_base = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(lds_ptr_t)lds);
    // loads j = part, part + parts, ... of the kLoads loads of stage st (activation loads first), into ring slot `slot`
    auto issue = [&](int st_local, int slot, int part, int parts) {
        const int st = st_begin + st_local;  // position along K
        const bool last = st + 1 >= st_all;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            if (j % parts != part) continue;
            if (j < A_LOADS) {
                dma16(a_rsrc, lds_base + slot * A_STAGE + (j * kWaves + wave) * 1024,
                      (last && !a_last_ok) ? kNowhere : a_off[j], st * kStageK);
            } else if (j < A_LOADS + B_LOADS) {
                const int i = j - A_LOADS;
                const int L = i * kWaves + wave;
                const unsigned dst = (kRagged && L >= B_TOTAL) ? kSpare : kBBase + slot * B_STAGE + L * 1024;
                if constexpr (ROW)
                    dma16(b_rsrc, lds_base + dst, (last && !b_last_ok) ? kNowhere : b_off[i], st * (kStageK / 2));
                else
                    dma16(b_rsrc, lds_base + dst, b_off[i], st * kBlock);
            } else if (lane < 4 * NT) {  // FG: the other lanes are masked off and write nothing
                dma16(g_rsrc, lds_base + kScaleBase + (slot * kWaves + wave) * kScaleWave, g_off, st * p.ldg * 4);
            }
        }
    };

    // The wave's part of the output tile: MT x NT tiles of 16 rows of X x 16 channels.
    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mt][t] = v4i{0, 0, 0, 0};
    // FG: sum over the groups of float(integer sum of the group) * group scale, sixteen-fold like the integer sums
    float facc[FG ? MT : 1][FG ? NT : 1][4];
    if (FG) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) facc[FG ? mt : 0][FG ? t : 0][v] = 0.f;
    }

    // LDS offsets of this lane's fragments inside a stage.  A stage is two MFMA steps h = 0, 1 of 64 k.  int4: K group g of
    // step h is k = 32 g + 16 h .. + 15, so that the 16 bytes of weight chunk g hold a lane's codes of both steps (dwords
    // 2 h, 2 h + 1), and the activation chunk is 2 g + h.  int8: k = 64 h + 16 g .. + 15, chunk 4 h + g of both operands.
    int xa[2];
    {
        const int row = wm * (16 * MT) + idx;  // the other m tiles lie multiples of 16 rows further: same swizzle
#pragma unroll
        for (int h = 0; h < 2; ++h) xa[h] = row * 128 + (((W8 ? 4 * h + g : 2 * g + h) ^ fx(row)) << 4);
    }
    // channel tile t of the wave is tile T = wn NT + t of the output tile, half T % 2 of weight block T / 2
    const int tile0 = wn * NT;
    const int wa_even = kBBase + (tile0 >> 1) * kBlock + (tile0 & 1) * 256 + (g * 32 + idx) * 16;
    const int wa_odd = wa_even + ((tile0 & 1) ? kBlock - 256 : 256);
    const int wa_row = kBBase + tile0 * 1024 + idx * 64 + ((g ^ fw(idx)) << 4);
    auto wa = [&](int t) {
        if constexpr (ROW) return wa_row + t * 1024;
        return (NT % 2 == 0 ? wa_even + (t & 1) * 256 : (t & 1) ? wa_odd : wa_even) + (t >> 1) * kBlock;
    };
    // A block of MFMAs takes at most four m tiles, so that its fragments and those of the next one fit the registers.
    constexpr int XF = MT > 4 ? MT / 2 : MT;
    constexpr int kBlocksPerStep = MT / XF;
    constexpr int kBlocks = 2 * kBlocksPerStep;  // per stage
    static_assert(MT % XF == 0, "m tiles must split evenly over the blocks");
    auto read_x = [&](v4u(&dst)[XF], int slot, int h, int m0) {
#pragma unroll
        for (int i = 0; i < XF; ++i) dst[i] = *(const v4u *)(&lds[slot * A_STAGE + xa[h] + (m0 + i) * 2048]);
    };
    // ROW: the k order of the weight codes, in place
    auto order_x = [&](v4u(&x)[XF]) {
        if constexpr (ROW) {
#pragma unroll
            for (int i = 0; i < XF; ++i) x[i] = __builtin_bit_cast(v4u, x_operand(x[i]));
        }
    };
    // weight fragment of channel tile t: int4 -> both steps of the stage; int8 -> step h
    auto read_w = [&](v4u &dst, int slot, int t, int h) {
        dst = *(const v4u *)(&lds[slot * B_STAGE + wa(t) + (W8 ? h * 2048 : 0)]);
    };
    // the scales of this wave's channels for the group in ring slot `slot`, in accumulator order:
    // register v of tile t belongs to channel 16 t + 4 g + v
    auto read_sg = [&](float(&dst)[NT][4], int slot) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 v = *(const float4 *)(&lds[kScaleBase + (slot * kWaves + wave) * kScaleWave + (16 * t + 4 * g) * 4]);
            dst[t][0] = v.x;
            dst[t][1] = v.y;
            dst[t][2] = v.z;
            dst[t][3] = v.w;
        }
    };
    auto w_op = [&](const v4u &w, int h) {
        return W8    ? v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w}
               : UNS ? (h == 0 ? u_operand_tiled(w.x, w.y) : u_operand_tiled(w.z, w.w))
                     : (h == 0 ? w_operand_tiled(w.x, w.y) : w_operand_tiled(w.z, w.w));
    };
    // MFMAs of m tiles m0 .. m0 + XF - 1 with every channel tile, step h.  fresh = true (FG, first step of a stage): the
    // group's integer sums start from zero.  behind(t) is issued behind the MFMAs of channel tile t.
    // wk[t] holds the operands of channel tile t.  While the MFMAs of a tile run, the codes of the next tile are converted
    // (CONVERT: the block is the first of its step; in the others the operands are there already), two vector operations
    // to an MFMA, which issue while the matrix core is busy (N = 5120, K = 13824, M = 1024, tile 128 x 256: 67 us against 75
    // with the conversion right in front of the MFMAs that use it); behind the last tile of a step (hn >= 0) those of the
    // first tile of the next step, hn.  xn: the activation fragments of the next block, requested in front of this one.
    v4i wk[NT];
    auto mfma_block = [&](const v4u(&x)[XF], v4u(&xn)[XF], v4u(&w)[NT], int h, int m0, bool fresh, bool convert, int hn, auto behind) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            static_assert(NT >= 2, "the next step's first operand is converted before its fragment is replaced");
            const v4i wop = wk[t];
            if (convert && t + 1 < NT) wk[t + 1] = w_op(w[t + 1], h);
            if (t + 1 == NT && hn >= 0) wk[0] = w_op(w[0], hn);
            if (t + 1 == NT) order_x(xn);
#pragma unroll
            for (int i = 0; i < XF; ++i)
                acc[m0 + i][t] = mfma_i8_16x16x64(wop, v4i{(int)x[i].x, (int)x[i].y, (int)x[i].z, (int)x[i].w},
                                                  fresh ? v4i{0, 0, 0, 0} : acc[m0 + i][t]);
            behind(t);
#pragma unroll
            for (int i = 0; i < XF; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (ROW && t + 1 == NT)
                    __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // those of order_x as well
                else
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Two schedules.  Ring of two: stage st + 2 can only be requested once stage st has been read, i.e. in one burst
    // behind the barrier of stage st.  Ring of three or more (kSpread): the slot freed by the barrier of stage st - 1
    // is refilled with stage st + STAGES - 1 load by load, between the MFMAs up to the next barrier; a burst of loads right
    // behind the barrier holds up the issuing wave for as long as the address unit needs to take them (measured: a
    // fifth of the loop time), spread out they cost an issue slot each.
    // Loads return in order, so "at most n outstanding" means all but the youngest n have landed; waiting for fewer
    // than could be allowed is always safe, which is what happens near the end of K.
    // Measured: spreading pays for the 8-wave tiles (3-4 %); the 4-wave tiles with a ring of three lose 5-15 % to
    // the shorter look-ahead it implies, so they keep the burst.
    constexpr bool kSpread = STAGES >= 3 && kWaves >= 8;
    constexpr int kAhead = kSpread ? STAGES - 1 : STAGES;  // stages requested before the loop starts
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
        if (s < st_total) issue(s, s, 0, 1);
    if (st_total >= kAhead)
        wait_vmcnt<(kAhead - 1) * kLoads>();
    else
        wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();

    v4u x0[XF], x1[XF], w[NT];
    int slot = 0;
    auto handover = [&](bool count_outstanding) {
        if (count_outstanding)
            wait_vmcnt<(STAGES - 2) * kLoads>();  // the stages behind st + 1 may still be in flight
        else
            wait_vmcnt<0>();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's last fragment reads of the slot have returned
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    if constexpr (KS == 2) {
        // Wave set ks multiplies step ks of every stage, whose fragments it reads one stage ahead.
        static_assert(kSpread && XF == MT, "the k split uses the spread schedule and one block per step");
        auto read_half = [&](v4u &dst, int slot, int t) {  // the eight bytes of step ks
            const v2u v = *(const v2u *)(&lds[slot * B_STAGE + wa(t) + 8 * ks]);
            dst.x = v.x;
            dst.y = v.y;
        };
        read_x(x0, 0, ks, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t) read_half(w[t], 0, t);
        wk[0] = w_op(w[0], 0);
        for (int st = 0; st < st_total; ++st) {
            const int next = slot + 1 == STAGES ? 0 : slot + 1;
            const int prev = slot == 0 ? STAGES - 1 : slot - 1;
            const int target = st + STAGES - 1;  // into the slot whose fragments every wave had before the last barrier
            if (target < st_total) issue(target, prev, 0, 1);
            handover(target < st_total);
            const bool more = st + 1 < st_total;
            if (more) read_x(x1, next, ks, 0);
            __builtin_amdgcn_sched_barrier(0);
            mfma_block(x0, x1, w, 0, 0, false, true, 0, [&](int t) {
                if (more) read_half(w[t], next, t);
            });
#pragma unroll
            for (int i = 0; i < XF; ++i) x0[i] = x1[i];
            slot = next;
        }
    } else {
        read_x(x0, 0, 0, 0);
        order_x(x0);
#pragma unroll
        for (int t = 0; t < NT; ++t) read_w(w[t], 0, t, 0);
        wk[0] = w_op(w[0], 0);
        float sg[FG ? NT : 1][4];
        // One stage: kBlocks blocks of MFMAs, each reading the activation fragments of the block behind it; the scheduling
        // fences keep those reads in front of the MFMAs they overlap with (left alone the compiler sinks them next to
        // their first use and every block then starts with an exposed LDS wait).  A weight fragment is replaced by its
        // successor right behind its last MFMAs.  TARGET: there is a stage left to request; EARLY: behind the barrier, one more.
        // Where load j of a target stage is issued: places 0 .. NT - 1 are the channel tiles of the last block, behind the barrier,
        // then come those of the other blocks.  With two blocks both take loads (N = 5120, K = 13824, M = 1024 as 128 x 192: 71.5 us
        // with all of them in the first, 69.2 so; N = 15360, K = 5120, M = 128 as 64 x 128: 17.5 and 16.7); with four, three are enough
        // (256 x 256 level, 192 x 320 over row-major weights 1 % slower), and so is one with row-major weights and two loads a stage
        // (64 x 128: over 33 shapes both blocks take 2.3 % longer, up to 7; N = 2796, K = 13504, M = 583: 42.2 us and 39.6 so).
        constexpr int kFirstPlace = kBlocks == 2 && !(ROW && kLoads == 2) ? 0 : NT;
        constexpr auto place = [](int j) { return kFirstPlace + j * (kBlocks * NT - kFirstPlace) / kLoads; };
        auto stage = [&](int st, auto target_c, auto early_c) {
            constexpr bool TARGET = decltype(target_c)::value, EARLY = decltype(early_c)::value;
            const int next = slot + 1 == STAGES ? 0 : slot + 1;
            const int prev = slot == 0 ? STAGES - 1 : slot - 1;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) {
                const int h = b / kBlocksPerStep, m0 = (b % kBlocksPerStep) * XF;
                const bool last = b + 1 == kBlocks;
                v4u(&x)[XF] = (b & 1) ? x1 : x0;
                v4u(&xn)[XF] = (b & 1) ? x0 : x1;
                const bool more = TARGET || st + 1 < st_total;
                if (!last) {
                    read_x(xn, slot, (b + 1) / kBlocksPerStep, ((b + 1) % kBlocksPerStep) * XF);
                    if constexpr (FG)
                        if (b + 2 == kBlocks) read_sg(sg, slot);  // before the barrier that lets the slot be refilled
                } else {
                    // Every fragment of this stage is in registers once the reads above have returned, so after the
                    // barrier the slot can be refilled; stage st + 1 must be in LDS for every wave.
                    handover(TARGET || (!kSpread && st + STAGES <= st_total));
                    if (!kSpread && TARGET) issue(st + STAGES, slot, 0, 1);
                    if (more) read_x(xn, next, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                const bool step_ends = m0 + XF == MT;
                mfma_block(x, xn, w, h, m0, FG && h == 0, m0 == 0, step_ends ? 1 - h : -1, [&](int t) {
                    // Loads of a target stage, evenly between two barriers: the last block's has freed this stage's slot.
                    if constexpr (kSpread) {
#pragma unroll
                        for (int j = 0; j < kLoads; ++j) {
                            if (last ? EARLY && place(j) == t : TARGET && place(j) == (b + 1) * NT + t)
                                issue(last ? st + STAGES : st + STAGES - 1, last ? slot : prev, j, kLoads);
                        }
                    }
                    if (step_ends) {
                        if (last) {
                            if (more) read_w(w[t], next, t, 0);
                        } else if (W8) {
                            read_w(w[t], slot, t, 1);
                        }
                    }
                });
            }
            if constexpr (FG) {
                // Dq of Eq. (5) for this group: a group's sums are below 2^24 in magnitude, so the conversion is exact
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            facc[mt][t][v] = __builtin_fmaf((float)acc[mt][t][v], sg[t][v], facc[mt][t][v]);
            }
            slot = next;
        };
        const int with_target = st_total - (kSpread ? STAGES - 1 : STAGES);
        int st = 0;
        if constexpr (kSpread) {
            if (with_target > 0) {  // what a stage before the first would have requested behind its barrier
#pragma unroll
                for (int j = 0; j < kLoads; ++j)
                    if (place(j) < NT) issue(STAGES - 1, STAGES - 1, j, kLoads);
            }
            for (; st + 1 < with_target; ++st) stage(st, std::true_type{}, std::true_type{});
        }
        for (; st < with_target; ++st) stage(st, std::true_type{}, std::false_type{});
        for (; st < st_total; ++st) stage(st, std::false_type{}, std::false_type{});
    }
    wait_vmcnt<0>();

    // The ring is idle: the last barrier of the loop lies behind every wave's last fragment read and every load has
    // landed.  Park the scales behind it; the barrier that makes them visible is the one of the k halves' meeting
    // where there is one.
    float *const sa_lds = (float *)(lds + kEpiScales);
    float *const sw_lds = sa_lds + BM;
    if (!ACC_OUT) {
        if (tid < BM) sa_lds[tid] = sa_mine;
        if (tid < BN) sw_lds[tid] = sw_mine;
        if constexpr (KS == 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        }
    }

    if constexpr (KS == 2) {
        // The two k halves meet: the ring is idle (the last barrier lies behind every wave's last fragment read and
        // every load has landed), the upper set parks its sums behind the area the epilogue's slabs will use and leaves.
        constexpr int kRedBase = kOutWaves * kSlabRows * (32 * NT + 16);
        int *part = (int *)(lds + kRedBase) + wsub * (MT * NT * 4 * 64) + lane;
        if (ks == 1) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) part[((mt * NT + t) * 4 + v) * 64] = acc[mt][t][v];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (ks == 1) return;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[mt][t][v] += part[((mt * NT + t) * 4 + v) * 64];
    }

    // Epilogue (Eq. (6),(7)).  A lane holds, per tile, four consecutive n of one m, so storing from the
    // accumulator layout writes 32 bytes into each of 16 different rows per instruction.  Instead every wave turns
    // its 32-row slabs around in LDS (the ring is idle now: the last barrier of the loop lies behind every wave's
    // last fragment read and every load has landed) and stores whole 16-byte runs of 8 channels, 8 or more lanes per
    // row, i.e. whole cache lines.
    // int4 sums are sixteen times the true sums (the nibbles sat in the high half of their bytes); int8 sums are true
    auto deq = [](int a, float s_a, float s_w) { return kTrueSums ? (float)a * (s_a * s_w) : dequant(a, s_a, s_w); };
    // FG: the sixteen-fold fp32 sum times s_a / 16 (both scalings by a power of two are exact): one rounding, as in
    // f * s_a on the true sum
    auto value = [&](int mt, int t, int v, float s_a, float s_w) {
        if constexpr (FG)
            return facc[mt][t][v] * (s_a * 0.0625f);
        else
            return deq(acc[mt][t][v], s_a, s_w);
    };
    if (!ACC_OUT && (SWIGLU || (p.ldc & 7) == 0)) {  // the fused form is only launched with a pitch that allows this path
        constexpr int kRowBytes = 32 * NT;         // fp16 bytes of a slab row (16 NT channels)
        constexpr int kPitch = kRowBytes + 16;     // padded: rows 16 apart, not 1 apart, share banks
        constexpr int kChunksPerRow = 2 * NT;      // 16-byte chunks
        constexpr int kReads = (kSlabRows * kChunksPerRow + 63) / 64;
        constexpr int kSlabTiles = kSlabRows / 16;
        static_assert(kOutWaves * kSlabRows * kPitch <= STAGES * (A_STAGE + B_STAGE), "slabs must fit the ring");
        uint8_t *slab = lds + wsub * (kSlabRows * kPitch);
        const int n_wave = bn0 + wn * (16 * NT);
#pragma unroll
        for (int mt = 0; mt < MT; mt += kSlabTiles) {
            const int m_slab = bm0 + wm * (16 * MT) + 16 * mt;
            float sa[kSlabTiles];  // 0 for rows past M
#pragma unroll
            for (int e = 0; e < kSlabTiles; ++e) sa[e] = sa_lds[wm * (16 * MT) + 16 * (mt + e) + idx];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int nl = 16 * t + 4 * g;
                // channels past N carry scale 0: their values are formed but never stored
                const float4 sw = FG ? float4{0.f, 0.f, 0.f, 0.f} : *(const float4 *)(sw_lds + wn * (16 * NT) + nl);
#pragma unroll
                for (int e = 0; e < kSlabTiles; ++e) {
                    v2u o;
                    o.x = pack_f16x2(value(mt + e, t, 0, sa[e], sw.x), value(mt + e, t, 1, sa[e], sw.y));
                    o.y = pack_f16x2(value(mt + e, t, 2, sa[e], sw.z), value(mt + e, t, 3, sa[e], sw.w));
                    *(v2u *)(slab + (16 * e + idx) * kPitch + nl * 2) = o;
                }
            }
#pragma unroll
            for (int j = 0; j < kReads; ++j) {
                const int c = j * 64 + lane;
                const int row = c / kChunksPerRow, col = c - row * kChunksPerRow;
                if (kSlabRows * kChunksPerRow % 64 != 0 && row >= kSlabRows) continue;
                const v4u v = *(const v4u *)(slab + row * kPitch + col * 16);
                const int mm = m_slab + row, n = n_wave + col * 8;
                if (mm >= p.M || n >= p.N) continue;
                if constexpr (SWIGLU) {
                    // eight channels = four (gate, up) pairs -> four values of h
                    const v2u hv = silu_mul_pairs4(v);
                    unsigned short *dst = (unsigned short *)p.out + (size_t)mm * p.ldc + (n >> 1);
                    if (n + 8 <= p.N) {
                        *(v2u *)dst = hv;
                    } else {
                        const unsigned w[2] = {hv.x, hv.y};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + 2 * e + 1 < p.N) dst[e] = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
                    }
                    continue;
                }
                unsigned short *dst = (unsigned short *)p.out + (size_t)mm * p.ldc + n;
                if (n + 8 <= p.N) {
                    *(v4u *)dst = v;
                } else {
                    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (n + e < p.N) dst[e] = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        return;
    }

    // general epilogue: raw sums, or an output pitch that rules out 16-byte stores
    const bool vec_ok = (p.ldc & 3) == 0;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = bm0 + wm * (16 * MT) + 16 * mt + idx;
        if (m >= p.M) continue;
        const float sa = ACC_OUT ? 0.f : sa_lds[wm * (16 * MT) + 16 * mt + idx];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int n = bn0 + wn * (16 * NT) + 16 * t + 4 * g;
            if (n >= p.N) continue;
            if (ACC_OUT) {
                int *dst = p.acc_out + (size_t)m * p.ldc + n;
                if (p.splits > 1) dst += (size_t)blockIdx.y * (size_t)p.M * (size_t)p.ldc;
                constexpr int kShift = kTrueSums ? 0 : 4;  // signed int4: exact, every sum is a multiple of 16
                const v4i s = acc[mt][t];
                const v4i v = v4i{s.x >> kShift, s.y >> kShift, s.z >> kShift, s.w >> kShift};
                if (vec_ok && n + 3 < p.N) {
                    *(v4i *)dst = v;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (n + j < p.N) dst[j] = v[j];
                }
            } else {
                unsigned short *dst = (unsigned short *)p.out + (size_t)m * p.ldc + n;
                if (vec_ok && n + 3 < p.N) {
                    const float4 sw = FG ? float4{0.f, 0.f, 0.f, 0.f} : *(const float4 *)(sw_lds + (n - bn0));
                    v2u o;
                    o.x = pack_f16x2(value(mt, t, 0, sa, sw.x), value(mt, t, 1, sa, sw.y));
                    o.y = pack_f16x2(value(mt, t, 2, sa, sw.z), value(mt, t, 3, sa, sw.w));
                    *(v2u *)dst = o;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (n + j < p.N) dst[j] = f32_to_f16_bits(value(mt, t, j, sa, FG ? 0.f : sw_lds[n + j - bn0]));
                }
            }
        }
    }
}

namespace {

template <int MT, int NT, int WM, int WN, int STAGES, bool ACC_OUT, int WBITS, bool UNS, bool FG, int KS, bool SWIGLU = false, bool ROW = false>
hipError_t launch_one(const PrefillArgs &p, dim3 grid, hipStream_t stream) {
    constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
    // ring + spare KB; group scales: 64 NT bytes per wave and ring slot, and a KB of slack behind them
    constexpr int kRing = STAGES * (BM * 128 + BN * 16 * WBITS) + 1024 + (FG ? STAGES * WM * WN * NT * 64 + 1024 : 0);
    // k split: the epilogue's slabs and, behind them, the parked sums of the upper wave set
    constexpr int kMeet = KS == 2 ? WM * WN * ((MT % 2 == 0 ? 32 : 16) * (32 * NT + 16) + MT * NT * 4 * 256) : 0;
    constexpr int kLdsBytes = (kRing > kMeet ? kRing : kMeet) + (BM + BN) * 4;  // + the epilogue's s_a and s_w
    static_assert(kLdsBytes <= 160 * 1024, "a workgroup's ring must fit the compute unit's LDS");
    constexpr auto kernel = gemm_prefill_tiled_kernel<MT, NT, WM, WN, STAGES, ACC_OUT, WBITS, UNS, FG, KS, SWIGLU, ROW>;
    if (const hipError_t e = allow_lds<kernel>(kLdsBytes); e != hipSuccess) return e;
    if (p.prepare_only) return hipSuccess;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WM * WN * KS), kLdsBytes, stream, W4A8_PREFILL_LAUNCH_ARGS(p, ACC_OUT));
    return hipGetLastError();
}

template <int MT, int NT, int WM, int WN, int STAGES, int WBITS = 4, bool UNS = false, bool FG = false, int KS = 1, bool ROW = false>
hipError_t launch_tile(PrefillArgs p, bool acc_out, hipStream_t stream) {
    constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    const int total = p.tiles_m * p.tiles_n;
    const dim3 grid(8 * ((total + 7) / 8), p.splits > 1 ? p.splits : 1);
    if (p.splits > 1 && (!acc_out || FG)) return hipErrorInvalidValue;  // a split of K returns raw partial sums
    if constexpr (FG) {
        if (acc_out) return hipErrorInvalidValue;  // there is no single integer sum to return
        return launch_one<MT, NT, WM, WN, STAGES, false, WBITS, UNS, true, 1>(p, grid, stream);
    } else {
        return acc_out ? launch_one<MT, NT, WM, WN, STAGES, true, WBITS, UNS, false, KS, false, ROW>(p, grid, stream)
                       : launch_one<MT, NT, WM, WN, STAGES, false, WBITS, UNS, false, KS, false, ROW>(p, grid, stream);
    }
}

}  // namespace

}  // namespace w4a8
