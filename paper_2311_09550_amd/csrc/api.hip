// C ABI of the W4A8 library: argument validation, tiling choice, launches.
// Nothing here touches the data; every step of the path runs in the kernels.
#include "../../include/w4a8.h"
#include "../../include/w4a8_tuning.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <iterator>
#include <mutex>

#include "kernels.hpp"

namespace {

using namespace w4a8;

constexpr int kDecodeMaxM = 64;

// What HIP said when an entry point last returned W4A8_ERR_LAUNCH on this thread (hipSuccess if it never did).
thread_local hipError_t last_hip_error = hipSuccess;

inline int launched(hipError_t e) {
    if (e == hipSuccess) return W4A8_OK;
    last_hip_error = e;
    (void)hipGetLastError();  // a rejected launch leaves its error in the runtime's per-thread slot: take it out
    return W4A8_ERR_LAUNCH;
}

inline bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

inline int check_gemm_shape(int M, int N, int K) {
    if (M < 1 || N < 1 || K < 32 || (K % 32) != 0 || K > W4A8_MAX_K) return W4A8_ERR_SHAPE;
    return W4A8_OK;
}

// Compute units of the current device (256 on MI355X); queried once per device.
int compute_units() {
    static std::atomic<int> cus[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Scratch memory of the entry point that allocates nothing (w4a8_gemm_tiled_splitk_static): the slabs of raw sums
// that the K slices of one GEMM exchange.  One array per GPU, held from the moment the library is loaded until the
// process ends.  `scratch` is only the host-side name of the symbol; the device address is looked up once per device
// and every use below goes through that address.
constexpr size_t kStaticScratchBytes = W4A8_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device (NULL and an error code if the lookup fails).
int static_scratch(void **ptr) {
    static void *addr[kMaxDevices];
    static std::atomic<bool> known[kMaxDevices];
    static std::mutex lookup_lock;
    int dev = 0;
    *ptr = nullptr;
    if (int e = launched(hipGetDevice(&dev))) return e;
    if (dev < 0 || dev >= kMaxDevices) return launched(hipErrorInvalidDevice);
    if (!known[dev].load(std::memory_order_acquire)) {
        std::lock_guard<std::mutex> hold(lookup_lock);
        if (!known[dev].load(std::memory_order_relaxed)) {
            void *p = nullptr;
            if (int e = launched(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)))) return e;
            if (p == nullptr) return launched(hipErrorInvalidSymbol);
            addr[dev] = p;
            known[dev].store(true, std::memory_order_release);
        }
    }
    *ptr = addr[dev];
    return W4A8_OK;
}

struct Plan {
    int tiling;
    DecodeShape decode;
    int prefill_tile;
};

bool resident_shape(int M, int N, int K, int waves, int grid, int prefetch, bool whole16, int aux, bool tiled, DecodeShape *out,
                    int k_slices = 1, bool x_window = false);

// Shape of the persistent weight-streaming kernel for (M, N, K).  Returns false when a wave's share of the
// activations would not fit in registers (then the general streaming kernel takes over).
//   waves    : 8 or 16, 0 = library's choice (8 wherever a wave's k steps fit its registers, see below);
//   grid     : workgroups wanted, 0 = library's choice.  A workgroup's range is N / grid rounded up to whole cache
//              lines of the weight array (8 channels in the tiled array, 4 in the row-major one).  The library's own
//              choice is one workgroup per compute unit with the range rounded up to whole 16-channel chunks
//              (measured on LLaMA-7B/13B/70B shapes, cold weights: within 4 % of the best grid everywhere; ranges of
//              20 or 24 channels, i.e. chunks of 12, lose up to 13 % to ranges of 32 on fewer compute units);
//   prefetch : chunks of weight loads a wave keeps in flight, 0 = library's choice: one, since a compute unit takes
//              only some 40 to 50 outstanding wave-wide loads and one chunk per wave mostly is that many; two by
//              two_chunks_ahead, among others where a range is exactly two chunks and M <= 8 (everything is then requested at
//              once: 4 to 5 % on 13B's O; level at 16 tokens);
//   whole16  : chunks of 16 channels even where the range does not divide evenly;
//   aux      : cache policy of the weight loads, -1 = library's choice (non-temporal: 5 to 10 % faster);
//   k_slices : workgroups along K (raw sums only when more than one);
//   x_window : every wave stages its own k steps (tiled weights, 17 to 64 tokens).  Then waves = 0 means 16 waves for
//              two column tiles when their k steps fit, else 8.
// Whether a wave asks for two chunks ahead.  One chunk of all waves should be the 32 or more loads that keep a compute unit
// busy; where it is fewer, a second one is worth the slot that it wastes at the end of an odd number of chunks, but not where one is
// nearly enough.  Cold, one chunk ahead and two: tiled weights, one token, 32768 x 1024 8.06 us and 5.66, 32000 x 2048 9.17 and 7.35,
// 24576 x 3072 8.50 and 7.93, 22016 x 4096 (six chunks) 9.29 and 9.08; but 20480 x 4096 (five) 8.70 and 8.96, with 32 tokens 10.1 and 10.5,
// 12288 x 4096 (three) 6.12 and 6.49, 27648 x 5120 12.96 and 13.54.  Row-major 32768 x 1024 8.75 and 6.07, 32000 x 2048 10.3 and 8.3, but
// 17216 x 4000 11.5 and 11.9; with 17 to 32 tokens, whose rows then no longer fit LDS beside the sums and are read in operand order,
// still 11.1 and 8.4, 13.1 and 10.7.  With three and four column tiles 64 tokens of 24576 x 3072 take 11.4 and 12.6, 32000 x 2048 12.4 and 11.1.
// The norm in front takes long enough for two chunks to arrive: 12288 x 4096 7.70 and 7.30, 22016 x 4096 10.8 and 9.9 (10240 x 8192, eight
// steps a wave: 10.6 and 11.4).
bool two_chunks_ahead(const DecodeShape &s, int chunks, int M, int mt) {
    const int loads = s.waves * s.x_steps;
    if (chunks == 2 && M <= 8) return true;
    if (chunks >= 2 && (loads <= 8 || (s.norm && loads <= 32))) return true;
    const int few = !s.tiled || mt > 2 ? 16 : chunks % 2 != 0 ? 24 : 32;
    return chunks >= 4 && loads <= few;
}

bool resident_shape(int M, int N, int K, int waves, int grid, int prefetch, bool whole16, int aux, bool tiled, DecodeShape *out,
                    int k_slices, bool x_window) {
    const int mt = (M + 15) / 16;
    DecodeShape s{};
    s.resident = true;
    s.tiled = tiled;
    s.fused_quant = out->fused_quant;  // set by the caller that wants the kernel to quantise its own activations
    s.swiglu = out->swiglu;            // ... or to apply SiLU * up to interleaved gate / up channels
    s.norm = out->norm;                // ... or to add the residual and normalise in front of its quantiser
    s.aux = aux < 0 ? 2 : aux;
    s.x_window = x_window;
    const int ks_all = (K + 127) / 128, want = k_slices < 1 ? 1 : k_slices;
    const int ks_total = (ks_all + want - 1) / want;           // k steps of a slice
    s.k_slices = (ks_all + ks_total - 1) / ks_total;           // no empty slice
    // 8 waves wherever their k steps fit the registers (measured 4 to 13 % faster than 16): up to 14 steps per wave
    // for one column tile (K <= 14336), 7 for two with per-wave staging, 5 for three and four
    if (waves == 0) {
        if (mt == 1)
            waves = ks_total <= 112 ? 8 : 16;
        else if (x_window)
            waves = (mt == 2 && ks_total > 56) ? 16 : 8;
        else
            waves = 16;
    }
    s.waves = waves;
    s.x_steps = (ks_total + waves - 1) / waves;
    // beyond 8 steps per wave only 11 and 14 are instantiated; a wave's surplus steps load nothing and multiply zeros
    if (mt == 1 && waves == 8 && s.x_steps > 8) s.x_steps = s.x_steps <= 11 ? 11 : 14;
    // In the tiled array a 128-byte line holds 16 bytes of each of 8 consecutive channels: ranges that start on
    // multiples of 8 channels never share a line with a neighbour (which would fetch it a second time).
    const int unit = tiled ? 8 : 4;
    int rows;
    if (grid <= 0) {
        const long long per_wg = ((long long)N * s.k_slices + compute_units() - 1) / compute_units();
        rows = per_wg > kResidentMaxRows ? kResidentMaxRows : (int)((per_wg + 15) / 16 * 16);
    } else {
        rows = ((N + grid - 1) / grid + unit - 1) / unit * unit;
    }
    if (rows < unit) rows = unit;
    s.rows_per_wg = rows;
    const int chunks = (rows + 15) / 16;
    s.chunk_rows = whole16 ? 16 : (((rows + chunks - 1) / chunks + 3) & ~3);
    s.prefetch = prefetch;
    if (prefetch == 0) {
        s.prefetch = two_chunks_ahead(s, chunks, M, mt) ? 2 : 1;
        if (s.prefetch == 2 && !decode_resident_supported(M, N, K, s)) s.prefetch = 1;
    }
    if (!decode_resident_supported(M, N, K, s)) return false;
    *out = s;
    return true;
}

// Price of a launch of the large-M kernel over tiled int4 weights, in microseconds, for every output tile the library
// chooses from.  A launch runs in rounds of as many workgroups as the chip holds at once (per_cu to a compute unit):
//   launch + round * rounds + stages of 128 k * (stage * full rounds + last + share * part - lone * [part <= half]),
// part = filled share of the last round (the last three terms only where there is one; lone: a compute unit then holds one
// workgroup instead of several).  The coefficients are least-squares fits over 280 random shapes (N 1024 .. 32768,
// K 1024 .. 16384, M 17 .. 1400, up to six K slices; every tile timed on every shape from HIP graphs, weights cold); the
// fits are within 5 to 8 % of the measured times, and choosing among tiles, K slices and the weight-streaming kernel by
// them costs 1.2 % on average over always choosing the fastest.  (Rounds times area over an efficiency on nine tiles, the
// rule before, cost 8 %.)  Of 32 tile shapes tried, these are the ones whose removal costs anything.
struct TileCost {
    int id, bm, bn, per_cu;
    float launch, round, stage, last, share, lone;
};
constexpr TileCost kTileCosts[] = {
    {kTiled256x256, 256, 256, 1, 7.43f, 0.00f, 1.064f, 0.967f, 0.163f, 0.000f},
    {kTiled128x256, 128, 256, 2, 6.07f, 0.00f, 1.198f, 1.005f, 0.436f, 0.337f},
    {kTiled64x128, 64, 128, 2, 3.33f, 0.42f, 0.537f, 0.401f, 0.181f, 0.144f},
    {kTiled64x64, 64, 64, 3, 3.35f, 0.17f, 0.531f, 0.214f, 0.363f, 0.034f},
    {kTiled32x128, 32, 128, 3, 3.45f, 0.17f, 0.520f, 0.230f, 0.337f, 0.036f},
    {kTiled128x256W8, 128, 256, 1, 5.67f, 0.00f, 0.779f, 0.505f, 0.173f, 0.000f},
    {kTiled64x256, 64, 256, 1, 3.18f, 1.24f, 0.485f, 0.343f, 0.142f, 0.000f},
    {kTiled128x384, 128, 384, 1, 6.67f, 0.02f, 1.022f, 0.732f, 0.193f, 0.000f},
    {kTiled128x192, 128, 192, 1, 4.17f, 0.88f, 0.635f, 0.466f, 0.150f, 0.000f},
    {kTiled64x192, 64, 192, 1, 2.53f, 1.62f, 0.413f, 0.333f, 0.120f, 0.000f},
    {kTiled128x320, 128, 320, 1, 5.80f, 0.66f, 0.904f, 0.662f, 0.168f, 0.000f},
    {kTiled192x320, 192, 320, 1, 7.19f, 0.00f, 1.112f, 0.976f, 0.111f, 0.000f},
    {kTiled192x256, 192, 256, 1, 6.43f, 0.00f, 0.927f, 0.767f, 0.129f, 0.000f},
    {kTiled192x192, 192, 192, 1, 5.91f, 0.00f, 0.802f, 0.620f, 0.141f, 0.000f},
};

// The same for more than 512 tokens with K >= 1024, where the prices above are extrapolated for the most part: a round costs some
// 5 to 8 us beside its stages, and the chip is at its power limit.  Fits over 600 shapes (380 random, 220 of whole tiles, the models' linears
// among them; M 513 .. 2300, N 1024 .. 65536, K 1024 .. 28672; weights cold, the chip warm; about 9 % off, but alike for all tiles), their
// shares and shorter terms then moved by hand towards the choices that measured best.  On 870 other random shapes (M 513 .. 2300, K from
// 1024; every weight byte cold) choosing by them costs 0.7 % on average over always taking the fastest of the sixteen, the prices above on
// fourteen tiles 1.3 %; 4 of the 870 take over 3 % longer than by those, by 6 % at most.  (64 x 256 had been fitted cheaper than
// 64 x 192 where both take one round: N = 4224, K = 15808, M = 689 56.8 us, 51.8 as 64 x 192.)  Two tiles are in here alone, worth 0.3 %
// each: 256 x 320 (N = 10240, K = 8192, M = 2048, one round where 192 x 256 takes two: 126.8 -> 111.2 us) and 192 x 384 (N = 21888,
// K = 13184, M = 718: 169 -> 148).
// More of the output per operand byte is what counts at the power limit:
// the matrix instructions alone hold 2.35 GHz, with the LDS reads of 256 x 256 2.1, with operands coming from L2 as well 1.9.
constexpr int kManyTokens = 512, kManyTokensMinK = 1024;
constexpr TileCost kManyTokensTileCosts[] = {
    {kTiled256x256, 256, 256, 1, 2.318f, 6.822f, 1.311f, 0.866f, 0.424f, 0.000f},
    {kTiled128x256, 128, 256, 2, 1.304f, 7.124f, 1.324f, 1.017f, 0.430f, 0.468f},
    {kTiled64x128, 64, 128, 2, 3.274f, 1.665f, 0.513f, 0.297f, 0.265f, 0.096f},
    {kTiled64x64, 64, 64, 3, 4.730f, 0.000f, 0.543f, 0.136f, 0.399f, 0.000f},
    {kTiled32x128, 32, 128, 3, 4.842f, 0.291f, 0.481f, 0.152f, 0.359f, 0.000f},
    {kTiled128x256W8, 128, 256, 1, 2.584f, 4.417f, 0.736f, 0.482f, 0.216f, 0.000f},
    {kTiled64x256, 64, 256, 1, 2.946f, 2.444f, 0.466f, 0.318f, 0.136f, 0.000f},
    {kTiled128x384, 128, 384, 1, 2.736f, 5.661f, 1.040f, 0.682f, 0.301f, 0.000f},
    {kTiled128x192, 128, 192, 1, 2.613f, 4.036f, 0.597f, 0.398f, 0.166f, 0.000f},
    {kTiled64x192, 64, 192, 1, 2.677f, 2.228f, 0.444f, 0.317f, 0.108f, 0.000f},
    {kTiled128x320, 128, 320, 1, 2.233f, 5.860f, 0.915f, 0.622f, 0.240f, 0.000f},
    {kTiled192x320, 192, 320, 1, 2.277f, 6.877f, 1.261f, 0.866f, 0.368f, 0.000f},
    {kTiled192x256, 192, 256, 1, 2.536f, 5.834f, 0.995f, 0.690f, 0.279f, 0.000f},
    {kTiled192x192, 192, 192, 1, 2.271f, 5.243f, 0.823f, 0.570f, 0.214f, 0.000f},
    {kTiled256x320, 256, 320, 1, 1.885f, 9.544f, 1.574f, 1.090f, 0.474f, 0.000f},
    {kTiled192x384, 192, 384, 1, 2.258f, 8.945f, 1.373f, 1.054f, 0.421f, 0.000f},
};

// What K slices add: a second launch, and the slabs written and read
double slab_us(int M, int N, int slices) { return 2.0 + 0.34e-6 * 4.0 * M * (double)N * slices; }

// lone_slots: up to how many workgroups of the last round each has a compute unit for itself; 0: half of what the chip holds
double tile_us(const TileCost &t, int M, int N, int stages, int cus, int slices = 1, long long lone_slots = 0) {
    const long long n = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * slices;
    const long long slots = (long long)cus * t.per_cu;
    const long long full = n / slots, rest = n % slots;
    double us = t.launch + t.round * (double)(full + (rest != 0)) + t.stage * (double)(full * stages);
    if (rest != 0) {
        const double part = (double)rest / (double)slots;
        us += (t.last + t.share * part - (t.per_cu > 1 && rest <= (lone_slots ? lone_slots : slots / 2) ? t.lone : 0.f)) * stages;
    }
    return us;
}

struct TileCosts {
    const TileCost *first, *last;
    const TileCost *begin() const { return first; }
    const TileCost *end() const { return last; }
};
TileCosts signed_tile_costs(int M, int K) {
    if (M > kManyTokens && K >= kManyTokensMinK) return {std::begin(kManyTokensTileCosts), std::end(kManyTokensTileCosts)};
    return {std::begin(kTileCosts), std::end(kTileCosts)};
}

int cheapest_tile(TileCosts costs, int M, int N, int K, double *price = nullptr) {
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK, cus = compute_units();
    int best = 0;
    double best_us = 0;
    for (const TileCost &t : costs) {
        const double us = tile_us(t, M, N, stages, cus);
        if (best == 0 || us < best_us) best = t.id, best_us = us;
    }
    if (price) *price = best_us;
    return best;
}

int choose_tiled_tile(int M, int N, int K) { return cheapest_tile(signed_tile_costs(M, K), M, N, K); }

// The unsigned storage has prices of its own: it lacks the tiles above kTiledTileMax, converts a weight fragment in 14
// vector operations instead of 6, which the taller tiles spread over more MFMAs, and runs 64 x 128 on 4 waves.  Fits over 428
// shapes (260 random, M 1 .. 2048, and the models' linears; weights cold) within 3 to 6 %; choosing by them costs 0.6 % on
// average over always taking the fastest of the eight tiles, the signed prices 3.0 %, rounds times area over an efficiency
// 4.0 %.  (N = K = 5120, M = 1024: 128 x 256 at 39.8 us, 64 x 128 at 47.6; N = 4096, K = 11008, M = 1024: 128 x 128 at 58.7, 64 x 128
// at 67.7.)  The second 256 x 256 and 128 x 160 would gain nothing.
constexpr TileCost kUnsignedTileCosts[] = {
    {kTiled256x256, 256, 256, 1, 1.28f, 5.73f, 1.604f, 1.096f, 0.287f, 0.000f},
    {kTiled128x256, 128, 256, 2, 1.96f, 4.34f, 1.607f, 1.283f, 0.308f, 0.503f},
    {kTiled128x128, 128, 128, 2, 2.87f, 2.35f, 1.046f, 0.882f, 0.129f, 0.354f},
    {kTiled64x128, 64, 128, 2, 3.32f, 1.21f, 0.681f, 0.621f, 0.090f, 0.175f},
    {kTiled64x64, 64, 64, 3, 2.48f, 1.44f, 0.555f, 0.305f, 0.272f, 0.039f},
    {kTiled32x128, 32, 128, 3, 2.95f, 1.19f, 0.546f, 0.353f, 0.226f, 0.078f},
};

int choose_unsigned_tile(int M, int N, int K) { return cheapest_tile({std::begin(kUnsignedTileCosts), std::end(kUnsignedTileCosts)}, M, N, K); }

// The same kernel over row-major weights.  Its stages take longer, a weight stage being half a cache line of every
// channel: 1.2 times the prices above up to 64 tokens, 1.1 at large M, much the same for every tile.  So the prices serve
// to choose among its tiles as they are (within 0.6 % of always taking the fastest on 200 random shapes).
int choose_row_tile(int M, int N, int K) {
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK, cus = compute_units();
    int best = 0;
    double best_us = 0;
    for (const TileCost &t : kTileCosts) {
        bool there = false;
        for (const int id : kRowTiles) there |= id == t.id;
        if (!there) continue;
        const double us = tile_us(t, M, N, stages, cus);
        if (best == 0 || us < best_us) best = t.id, best_us = us;
    }
    return best;
}

// Over row-major weights: a weight-streaming kernel, or the tiles.  Measured on 900 shapes (M 1 .. 64, 730 of them random),
// every byte of the weights cold, as a model's layers find them; a rule of sizes, since where K is no multiple of 128 (rows
// that start inside a cache line) no price of the tiles comes nearer than 30 %:
//   up to 16 tokens streaming is the faster one on 94 % of the shapes, and taking it always costs 0.8 % on average (prices
//   that took the tiles for wide N cost 3.7 %: N = 27648, K = 5120, M = 1: 18.8 us tiled, 16.8 streaming; 57344 x 8192: 51 and
//   41; only copies that stay in the memory-side cache gain from the tiles, 14.2 against 16.5);
//   17 to 32 tokens, the persistent kernel where it has a shape (K <= 8192): 1.6 %, the prices 3.4 % (N = 33061, K = 5376,
//   M = 17: 24.9 us and 31.8 tiled; N = 27648, K = 5120, M = 32: 22.2 and 19.9);
//   else the general kernel, whose workgroups walk all of K once for every 32 channels of a compute unit: one round up to 32
//   channels per compute unit, two beyond (N = 8478, K = 15648, M = 47: 86.7 us and 40.2 tiled).  In one round it is the faster
//   one up to 32 tokens (N = 5120, K = 13824, M = 32: 26.9 and 36.0), with more only on a short K (N = 3746, M = 59: K = 1824 8.0
//   and 9.1; N = 5948, K = 7488, M = 36: 22.3 and 19.7).  0.1 and 0.3 %.
bool row_major_streams(int M, int N, int K, bool persistent) {
    constexpr int kShortK = 2048;
    if (M <= 16 || persistent) return true;
    if (N > 32 * compute_units()) return false;
    return M <= 32 || (M <= kDecodeMaxM && K <= kShortK);
}

// Whether one launch of the large-M kernel reaches every byte of both operands (32-bit byte offsets)
bool one_launch_covers(int M, int N, int K) {
    return (long long)M * K <= 0xF0000000ll && (long long)tiled_weight_bytes(N, K, 4) <= 0xF0000000ll;
}

// Price of the medium-M kernel in microseconds: as above, k steps of 128 in place of stages (rounded up to whole stages of `groups`
// steps), and three terms more: deep, for the share of a compute unit's workgroups that the fullest one holds in the last
// round; weights, per MB of int4 codes (what the memory needs beside them); ragged, where rows of activations do not begin on
// a cache line (K % 128 != 0).
struct StepCost {
    int id, bm, bn, groups, per_cu;
    float launch, round, step, last, share, deep, weights, ragged;
};

double step_us(const StepCost &t, int M, int N, int K, int cus) {
    const long long n = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const long long slots = (long long)cus * t.per_cu, full = n / slots, rest = n % slots;
    const double part = (double)rest / (double)slots, deep = (double)((rest + cus - 1) / cus) / t.per_cu;
    const int steps = ((K + kTiledBlockK - 1) / kTiledBlockK + t.groups - 1) / t.groups * t.groups;
    double us = t.launch + t.round * (double)(full + (rest != 0)) + t.weights * 0.5e-6 * (double)N * K;
    us += steps * (t.step * (double)full + (rest != 0 ? t.last + t.share * part + t.deep * deep : 0.0));
    if (K % kTiledBlockK != 0) us += t.ragged * ((double)full + part) * steps;
    return us;
}

bool medium_covers(int M, int N, int K, int wbits) {
    return (long long)M * K < kMediumMaxActivations && tiled_weight_bytes(N, K, wbits) <= kMediumMaxWeights;
}

// Its tiles over int4 weights: of eighteen tried, those without which the choice would cost more than 0.3 % on average.  Fits
// over 552 shapes (420 random, M 17 .. 1024, N 1024 .. 32768, K 1024 .. 16384, and the models' linears; weights cold) within 6 to 9 %.
// A medium tile is taken where it is priced that much lower than the large-M kernel (below): 1.7 % on average over always taking the fastest, 3 of
// 216 shapes that were not fitted to are more than 3 % slower than without the kernel, by 9 % at most, and all together take 0.93 of
// the time: 0.87 from 65 to 512 tokens (N = K = 5120, M = 128: 14.7 us in three slices of K, 10.3 as 32 x 96 tiles; N = 4096, K = 11008:
// M = 50 17.7 and 11.9, M = 333 28.2 and 24).  Of 903 more shapes with 65 to 512 tokens 21 take over 3 % longer than without it, all
// with K up to 3072 and priced close to the large-M kernel (N = 16320, K = 1888, M = 167: 13.15 us, 12.0 without).  Below 17 tokens the weight-streaming kernel holds the activations in registers.
constexpr StepCost kMediumCosts[] = {
    {kMedium32x32, 32, 32, 8, 2, 2.018f, 1.159f, 0.142f, 0.000f, 0.016f, 0.138f, 0.066f, 0.010f},
    {kMedium32x64, 32, 64, 4, 4, 1.504f, 1.200f, 0.359f, 0.037f, 0.059f, 0.292f, 0.086f, 0.022f},
    {kMedium32x64K8, 32, 64, 8, 2, 2.420f, 1.089f, 0.209f, 0.000f, 0.008f, 0.207f, 0.061f, 0.028f},
    {kMedium32x96, 32, 96, 4, 3, 1.018f, 1.981f, 0.337f, 0.021f, 0.032f, 0.332f, 0.085f, 0.016f},
    {kMedium48x128, 48, 128, 4, 2, 0.578f, 3.335f, 0.318f, 0.000f, 0.051f, 0.333f, 0.067f, 0.032f},
    {kMedium64x96, 64, 96, 4, 2, 0.713f, 3.345f, 0.338f, 0.000f, 0.078f, 0.321f, 0.053f, 0.013f},
    {kMedium64x128, 64, 128, 4, 1, 1.315f, 3.121f, 0.218f, 0.191f, 0.041f, 0.000f, 0.054f, 0.006f},
    {kMedium64x160, 64, 160, 4, 1, 0.963f, 3.888f, 0.258f, 0.230f, 0.045f, 0.000f, 0.054f, 0.005f},
};
// How much lower it has to be priced than the large-M kernel.  Beyond 512 tokens 15 %: it brings in more bytes per operation, which
// prices taken from short runs don't show.  N = 5120, K = 13824, M = 1024, as 64 x 160 tiles: 73.5 us against 75.3 by itself, but the
// layer around it 306 us instead of 299, at the power limit.  (On 60 shapes beyond 512 tokens it then gives 7.0 %, with 3 % 7.1.)
double medium_over_tiles(int M) { return M <= 512 ? 1.03 : 1.15; }
// Over int4 weights beyond 512 tokens 12 %, and against the prices of kTileCosts, not those of kManyTokensTileCosts, which ask more for few and
// small tiles and less for a long K.  On the same 870 shapes the choice among all tiles then costs 1.2 % on average over always taking the
// fastest, and 4 shapes take over 3 % longer than by kTileCosts and 15 % alone (2.0 %), by 5 % at most; 15 % cost 1.4 %.  Against
// kManyTokensTileCosts 15 % cost 1.1 %, but 13 shapes take over 3 % longer (N = 3072, K = 1024, M = 586 7.3 us as 32 x 64 tiles, 5.8 as
// 64 x 128; N = 3264, K = 3680, M = 768 17.1 as 64 x 256, 14.1 as 64 x 160).
constexpr double kMediumOverManyTokens = 1.12;

// Against weight streaming: 10 % lower than its price, preference included (streaming_preferred), where that takes one slice
// (the two are level there: N = 8544, K = 1824, M = 63 6.44 us and 6.43); 7 % lower than sliced_us where it takes several.  (By the price
// of one slice and 8 % more for the slabs it was taken for N = 1600, K = 11264, M = 59, 10.8 us, where three slices take 9.4; of 715
// shapes with several slices 22 took over 3 % longer than without the medium-M kernel, by up to 15 %, now 3.)
constexpr double kMediumOverStreaming = 1.10, kMediumOverSlices = 1.07;

// How a GEMM over tiled int4 weights with more than 16 tokens is run: by the weight-streaming kernel with per-wave
// staging, K cut into slices, by the large-M kernel, K cut into slices, or by the medium-M kernel.  All are priced and the
// cheapest one is taken, near ties by weight streaming.
struct TiledPlan {
    bool wide;          // weight-streaming kernel, else the large-M kernel
    DecodeShape shape;  // wide: its shape
    int tile;           // else: output tile, of the large-M or the medium-M kernel, and K slices
    int splits, stages_per_split;
};

// Price of the weight-streaming kernel in microseconds: what every compute unit brings in (the activations and its
// weights), a fixed part per chunk of 16 channels, more of it where a wave has more than 8 k steps, and the slabs.  Fitted
// like the tiles' prices, within 5 % of those shapes; on 346 others, with up to 65536 channels, within 9 % with one slice and
// 13 % too low on average with several.  Older than two_chunks_ahead: where that asks for two, the kernel takes 2 to 30 % less.
double wide_us(const DecodeShape &s, int M, int N, int K) {
    const double steps = ((K + 127) / 128 + s.k_slices - 1) / s.k_slices;
    const double chunks = (s.rows_per_wg + 15) / 16, mt = (M + 15) / 16, long_walk = s.x_steps > 8 ? s.x_steps - 8 : 0;
    const double x_kb = M * steps * 0.125, w_kb = s.rows_per_wg * steps * 0.0625;
    double us = 2.215 + 0.01676 * x_kb + 0.01376 * w_kb + chunks * (0.630 + 0.0551 * mt + 0.1122 * long_walk);
    if (s.k_slices > 1) us += slab_us(M, N, s.k_slices);
    return us;
}

// The same for several slices, where the medium-M kernel is set against them: fitted over 4275 such launches (17 to 64 tokens, N
// up to 32768, two to four slices, weights cold) within 6.2 %.  It knows two things more: ranges rounded to whole chunks can make more
// workgroups than there are compute units, and the few beyond take a round of their own (N = 4096, K = 11008, M = 50: 86 ranges
// in three slices, 16.5 us); and the slabs of an N that is no multiple of four are stored and read value by value.
double sliced_us(const DecodeShape &s, int M, int N, int K, int cus) {
    const int ranges = (N + s.rows_per_wg - 1) / s.rows_per_wg, rounds = (ranges * s.k_slices + cus - 1) / cus;
    const double steps = ((K + 127) / 128 + s.k_slices - 1) / s.k_slices, mt = (M + 15) / 16, slab_mb = 4e-6 * M * (double)N * s.k_slices;
    const double x_kb = M * steps * 0.125, w_kb = s.rows_per_wg * steps * 0.0625, chunks = (s.rows_per_wg + 15) / 16;
    return 3.603 + rounds * (0.00901 * x_kb + 0.03258 * w_kb + 0.0757 * chunks) + 0.2753 * mt + 0.2278 * s.k_slices +
           (N % 4 ? 1.445 : 0.6046) * slab_mb;
}

// The tiles' prices are too low where K is no multiple of 128 and where N is wide, and streaming is the form
// that such shapes hurt less, so near ties are its own: a tile is taken where it is priced 15 % lower, 10 % where K is cut
// into two or three slices, and simply lower beyond, where streaming's own price is the one that is too low (N = 8192, K =
// 28672, M = 64: 41.0 us in six slices, priced 30.1; 32.7 with tiles, priced 27.8).  On 522 shapes with 17 to 64 tokens
// (weights cold) that loses 0.5 % on average over always taking the faster with one slice and 1.7 % with several, 1.4 and 2.4 %
// without the preference; 6 shapes are more than 3 % slower than always streaming, 34 without it.
// (M = 64: N = 27648, K = 5120 17.9 us streaming, 19.8 tiled; N = 22016, K = 4096 14.0 and 15.3; N = 8544, K = 1824, M = 63 6.6
// and 7.5.)
double streaming_preferred(int slices) { return slices == 1 ? 0.85 : slices <= 3 ? 0.9 : 1.0; }

constexpr int kMaxSlices = 8;
constexpr int kSplitMaxM = 512;  // the large-M kernel is not split beyond: there its tiles fill the chip or the slabs cost more

// max_slab: bytes of slabs allowed (0: one slice only).
TiledPlan plan_tiled(int M, int N, int K, size_t max_slab, bool swiglu, int cus) {
    TiledPlan best{};
    double best_us = -1;
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK;
    const size_t slab = (size_t)M * (size_t)N * sizeof(int32_t);
    const int max_slices = max_slab / slab < 2 ? 1 : (int)(max_slab / slab < (size_t)kMaxSlices ? max_slab / slab : kMaxSlices);
    const int ring_slices = M <= kSplitMaxM && one_launch_covers(M, N, K) ? max_slices : 1;
    for (const TileCost &t : signed_tile_costs(M, K)) {
        for (int s = 1; s <= ring_slices; ++s) {
            const int per = (stages + s - 1) / s, n = (stages + per - 1) / per;
            if (n != s) continue;  // the same as fewer slices
            double us = tile_us(t, M, N, per, cus, s);
            if (s > 1) us += slab_us(M, N, s);
            if (best_us < 0 || us < best_us) {
                best_us = us;
                best.tile = t.id;
                best.splits = s;
                best.stages_per_split = per;
            }
        }
    }
    if (M <= kResidentMaxM) {
        for (int s = 1; s <= (swiglu ? 1 : max_slices); ++s) {
            DecodeShape shape{};
            shape.swiglu = swiglu;
            if (!resident_shape(M, N, K, 0, 0, 0, false, -1, true, &shape, s, true) || shape.k_slices != s) continue;
            const double us = streaming_preferred(s) * wide_us(shape, M, N, K);
            if (us < best_us) {
                best_us = us;
                best.wide = true;
                best.shape = shape;
            }
        }
    }
    if (medium_covers(M, N, K, 4)) {
        if (M > kManyTokens) cheapest_tile({std::begin(kTileCosts), std::end(kTileCosts)}, M, N, K, &best_us);
        const double bar = !best.wide                  ? best_us / (M > kManyTokens ? kMediumOverManyTokens : medium_over_tiles(M))
                           : best.shape.k_slices == 1 ? best_us / kMediumOverStreaming
                                                      : sliced_us(best.shape, M, N, K, cus) / kMediumOverSlices;
        double medium_us = bar;
        for (const StepCost &t : kMediumCosts) {
            const double us = step_us(t, M, N, K, cus);
            if (us < medium_us) {
                medium_us = us;
                best = TiledPlan{};
                best.tile = t.id;
                best.splits = 1;
                best.stages_per_split = stages;
            }
        }
    }
    best.splits = best.wide ? best.shape.k_slices : best.splits;
    return best;
}

// What the entries over tiled weights do with a shape: the plan, and what w4a8_gemm_tiled_splitk asks of its caller.
struct Route {
    TiledPlan plan;
    size_t need;      // bytes of workspace, 0 when one slice is asked for
    bool one_launch;  // refused where one launch cannot address the problem (slabs are whole M x N matrices)
};
enum RouteKind { kUnsliced, kSliced, kSwiglu, kInt8 };  // kInt8: over int8 weights, a tile

Route make_route(int M, int N, int K, RouteKind kind, int cus);

thread_local unsigned long long plans_made = 0;

// The library's own choice for more than 16 tokens, over int8 weights for any number (pricing its tiles takes longer than the rest
// of a call's checks: 0.5 us), remembered per thread: it is a pure function of its arguments (and of the
// device's compute units), and a loop over a model's layers asks for the same few again and again.  16 sets of four, the
// oldest of a set replaced; the set comes from all bits of the shape (a sum or XOR of products with its top bits taken put
// two linears of one layer into one place for every M).
Route tiled_route(int M, int N, int K, RouteKind kind) {
    struct Entry { int M, N, K, cus; RouteKind kind; Route route; };
    constexpr unsigned kSets = 16, kWays = 4;
    static thread_local Entry entries[kSets][kWays];
    static thread_local unsigned char oldest[kSets];
    const int cus = compute_units();
    unsigned long long h = 0;
    for (const unsigned v : {(unsigned)M, (unsigned)N, (unsigned)K, (unsigned)kind}) {
        h = (h ^ v) * 0x9E3779B97F4A7C15ull;
        h ^= h >> 29;
    }
    const unsigned set = (unsigned)(h >> 8) % kSets;
    for (const Entry &e : entries[set])
        if (e.M == M && e.N == N && e.K == K && e.cus == cus && e.kind == kind) return e.route;
    Entry &e = entries[set][oldest[set]];
    oldest[set] = (unsigned char)((oldest[set] + 1) % kWays);
    ++plans_made;
    return (e = Entry{M, N, K, cus, kind, make_route(M, N, K, kind, cus)}).route;
}

TiledPlan tiled_plan(int M, int N, int K, bool swiglu) { return tiled_route(M, N, K, swiglu ? kSwiglu : kUnsliced).plan; }

// a: one launch's worth of the problem; tile: of either kernel
hipError_t launch_tile(const PrefillArgs &a, bool acc_out, bool swiglu, int tile, hipStream_t st, int wbits) {
    if (tile >= kMediumFirst && tile <= kMediumLast) return launch_gemm_medium(a, acc_out, swiglu, tile, st, wbits);
    return swiglu ? launch_gemm_prefill_tiled_swiglu(a, tile, st) : launch_gemm_prefill_tiled(a, acc_out, tile, st, wbits);
}

// d: pointers only
hipError_t launch_wide(DecodeArgs d, int M, int N, int K, const DecodeShape &s, bool acc_out, hipStream_t st) {
    d.M = M; d.N = N; d.K = K;
    d.rows_per_wg = s.rows_per_wg;
    d.chunk_rows = s.chunk_rows;
    return launch_gemm_decode(d, acc_out, s, st);
}

// The choice among the fine-grained variant's tiles (measured on LLaMA-13B shapes at M = 1024 and 4096: two
// 128 x 128 workgroups per compute unit are never slower than one 128 x 256 workgroup of 8 waves).
int choose_fine_tile(int M, int N) {
    const int cus = compute_units();
    auto count = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (M <= 32) return kFine32x128;
    if (M <= 64 || count(128, 128) * 4 < (long long)cus * 3)
        return count(64, 128) * 4 >= (long long)cus * 3 ? kFine64x128 : kFine64x64;
    struct Option { int id, bm, bn, per_cu; double eff; };
    const Option options[] = {{kFine128x256, 128, 256, 1, 0.95}, {kFine128x128, 128, 128, 2, 1.00}};
    int best = kFine128x256;
    double best_cost = 0;
    for (const Option &o : options) {
        const long long tiles = count(o.bm, o.bn);
        const long long slots = (long long)cus * o.per_cu;
        const long long full = tiles / slots, rest = tiles % slots;
        const double last = rest == 0 ? 0.0 : (o.per_cu == 1 || rest * 2 > slots ? 1.0 : 0.5);
        const double cost = ((double)full + last) * o.bm * o.bn * o.per_cu / o.eff;
        if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = o.id; }
    }
    return best;
}

// The large-M kernel's tile for the int8-weight variant.  Its stages bring in twice the weight bytes, through rings one stage shallower,
// and convert nothing: a launch takes 1.06 to 1.42 times the price of the same tile over int4 weights, most where the weight
// stream is most of the work.  The factors are geometric means over 36 shapes (29 random, M 1 .. 1024; weights cold).
// Choosing by them costs 0.6 % on average over always taking the fastest of fourteen tiles; rounds times area over an
// efficiency on seven tiles, the rule before, cost 11 % (N = 5120, K = 13824, M = 512: 64 x 128 at 81 us, now 64 x 192 at 61;
// N = 11722, K = 15648, M = 1: 54 us, now 38).  128 x 256 of 4 waves, 128 x 160 and 128 x 128 were never the fastest,
// 64 x 256 and 192 x 256 neither.
int choose_ring_tile8(int M, int N, int K) {
    struct Factor { int id; double over_int4; };
    const Factor factors[] = {{kTiled256x256, 1.195}, {kTiled64x128, 1.333},  {kTiled64x64, 1.217},  {kTiled32x128, 1.411},
                              {kTiled128x256W8, 1.252}, {kTiled128x192, 1.173}, {kTiled64x192, 1.277}, {kTiled192x192, 1.060}};
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK, cus = compute_units();
    int best = 0;
    double best_us = 0;
    for (const Factor &f : factors)
        for (const TileCost &t : kTileCosts) {
            if (t.id != f.id) continue;
            // a compute unit with two workgroups streams twice the weights: no discount for a lone one then
            const double us = f.over_int4 * tile_us(t, M, N, stages, cus, 1, cus);
            if (best == 0 || us < best_us) best = t.id, best_us = us;
        }
    return best;
}

// Over int8 weights the medium-M kernel is set against the large-M kernel's tile of the rule above, both by prices of one form:
// fits over 216 shapes (150 random, M 1 .. 1024, and the models' linears; weights cold) within 8 to 12 %.  It is taken where it is
// priced lower by medium_over_tiles: 0.5 % on average over always taking the fastest of the fourteen tiles, one of the 216 shapes is more than 3 %
// slower than without it (by 5 %), and all together take 0.81 of the time: 0.68 up to 16 tokens, 0.79 from 33 to 64, 0.92 from 257
// to 512 (N = 5120, K = 13824, M = 512: 64 x 192 at 60 us, now 96 x 128 at 46).  By these prices for every tile seven shapes are slower.
constexpr StepCost kTileCosts8[] = {
    {kTiled256x256, 256, 256, 1, 1, 0.000f, 5.779f, 1.546f, 1.150f, 0.396f, 0.000f, 0.000f, 0.000f},
    {kTiled64x128, 64, 128, 1, 2, 2.516f, 0.337f, 0.683f, 0.071f, 0.126f, 0.566f, 0.105f, 0.027f},
    {kTiled64x64, 64, 64, 1, 2, 2.149f, 0.662f, 0.439f, 0.021f, 0.123f, 0.365f, 0.078f, 0.014f},
    {kTiled32x128, 32, 128, 1, 2, 1.582f, 0.547f, 0.552f, 0.106f, 0.025f, 0.467f, 0.131f, 0.000f},
    {kTiled128x256W8, 128, 256, 1, 1, 1.047f, 2.977f, 0.830f, 0.620f, 0.332f, 0.000f, 0.046f, 0.000f},
    {kTiled128x192, 128, 192, 1, 1, 0.715f, 2.903f, 0.719f, 0.528f, 0.257f, 0.000f, 0.034f, 0.000f},
    {kTiled64x192, 64, 192, 1, 1, 0.000f, 2.870f, 0.486f, 0.436f, 0.107f, 0.000f, 0.108f, 0.028f},
    {kTiled192x192, 192, 192, 1, 1, 0.473f, 4.555f, 0.874f, 0.579f, 0.214f, 0.000f, 0.006f, 0.009f},
    {kMedium16x16, 16, 16, 8, 4, 2.768f, 0.031f, 0.206f, 0.011f, 0.000f, 0.179f, 0.134f, 0.000f},
    {kMedium16x32, 16, 32, 8, 4, 2.813f, 0.000f, 0.333f, 0.000f, 0.043f, 0.291f, 0.128f, 0.000f},
    {kMedium32x32, 32, 32, 8, 2, 2.503f, 0.642f, 0.216f, 0.000f, 0.051f, 0.172f, 0.086f, 0.002f},
    {kMedium32x64, 32, 64, 4, 4, 1.661f, 1.038f, 0.544f, 0.000f, 0.012f, 0.568f, 0.180f, 0.000f},
    {kMedium64x96, 64, 96, 4, 2, 0.000f, 3.414f, 0.463f, 0.021f, 0.091f, 0.440f, 0.150f, 0.000f},
    {kMedium96x128, 96, 128, 4, 1, 0.000f, 4.544f, 0.355f, 0.337f, 0.075f, 0.000f, 0.100f, 0.041f},
};

int choose_tiled_tile8(int M, int N, int K) {
    int best = choose_ring_tile8(M, N, K);
    if (!medium_covers(M, N, K, 8)) return best;
    const int cus = compute_units();
    double best_us = 0;
    for (const StepCost &t : kTileCosts8)
        if (t.id == best) best_us = step_us(t, M, N, K, cus) / medium_over_tiles(M);
    for (const StepCost &t : kTileCosts8) {
        if (t.id < kMediumFirst) continue;
        const double us = step_us(t, M, N, K, cus);
        if (us < best_us) best = t.id, best_us = us;
    }
    return best;
}

// Tiling choice.  Small M streams the weights once (HBM bound); large M goes to the LDS-staged tiling
// (matrix-core bound).  `variant` refines a forced tiling (see w4a8.h); 0 lets the library choose.
int choose_plan(int M, int N, int K, int tiling, int variant, Plan *pl) {
    pl->tiling = tiling;
    if (tiling == W4A8_TILING_AUTO_TILED) {
        // one weight array for every M: the weight-streaming kernels up to M = 16; up to M = 64, where all of K fits a
        // wave's registers, these or the large-M kernel, by price; the large-M kernel above
        if (M > 16) {
            const TiledPlan t = tiled_plan(M, N, K, false);
            pl->decode = t.shape;
            pl->prefill_tile = t.tile;
            pl->tiling = t.wide ? W4A8_TILING_DECODE_RESIDENT : W4A8_TILING_PREFILL_TILED;
            return W4A8_OK;
        }
        pl->tiling = (resident_shape(M, N, K, 0, 0, 0, false, -1, true, &pl->decode, 1, true) ||
                      resident_shape(M, N, K, 0, 0, 0, false, -1, true, &pl->decode))
                         ? W4A8_TILING_DECODE_RESIDENT_TILED
                         : W4A8_TILING_DECODE_STREAM_TILED;
    }
    const bool decode_tiled = pl->tiling == W4A8_TILING_DECODE_RESIDENT_TILED || pl->tiling == W4A8_TILING_DECODE_STREAM_TILED;
    if (pl->tiling == W4A8_TILING_DECODE_RESIDENT_TILED) pl->tiling = W4A8_TILING_DECODE_RESIDENT;
    if (pl->tiling == W4A8_TILING_DECODE_STREAM_TILED) pl->tiling = W4A8_TILING_DECODE_STREAM;
    if (tiling == W4A8_TILING_AUTO) {
        const bool resident = M <= 32 && resident_shape(M, N, K, 0, 0, 0, false, -1, false, &pl->decode);
        pl->tiling = !row_major_streams(M, N, K, resident) ? W4A8_TILING_PREFILL
                     : resident                            ? W4A8_TILING_DECODE_RESIDENT
                                                           : W4A8_TILING_DECODE_STREAM;
    }
    if (pl->tiling == W4A8_TILING_DECODE_RESIDENT) {
        if (M > kResidentMaxM) return W4A8_ERR_ARG;
        const int flags = variant / 100000000, prefetch = variant / 10000000 % 10, waves = variant / 100000 % 100;
        // The library's own choice over the tiled array: per-wave staging from five tokens on (measured on LLaMA-13B
        // shapes: level with the whole-row staging at 5 or 6 tokens, 6 to 20 % faster at 16, where the whole rows crowd
        // or overflow LDS; below five tokens its extra round trip per window costs up to 8 % on a long K).
        const bool want_window = (flags & 16) != 0 || (tiling == W4A8_TILING_AUTO_TILED && M >= 5);
        auto shape = [&](bool window) {
            return resident_shape(M, N, K, waves, variant % 100000, prefetch, (flags & 1) != 0,
                                  (flags & 2) ? 2 : (flags & 8) ? 0 : -1, decode_tiled, &pl->decode, 1, window);
        };
        if (!(want_window && shape(true)) && !((flags & 16) == 0 && shape(false))) return W4A8_ERR_ARG;
        pl->decode.x_direct = (flags & 4) != 0;
    } else if (pl->tiling == W4A8_TILING_DECODE_STREAM) {
        if (M > kDecodeMaxM) return W4A8_ERR_ARG;
        const int mt = (M + 15) / 16;
        DecodeShape s{};
        s.resident = false;
        s.tiled = decode_tiled;
        // K beyond the resident kernel's reach at token-generation sizes (70B down, K = 28672): two row tiles on four
        // waves stream 7 % faster than the general default (measured, cold weights)
        const bool long_k_decode = mt == 1 && K > 16384;
        s.row_tiles = variant ? variant / 100 : ((M <= 8 && !long_k_decode) ? 1 : 2);
        s.waves = variant ? variant % 100 : (((mt >= 4 && s.row_tiles == 2) || long_k_decode) ? 4 : 8);
        if ((s.row_tiles != 1 && s.row_tiles != 2) || (s.waves != 4 && s.waves != 8)) return W4A8_ERR_ARG;
        if (mt == 4 && s.row_tiles == 2 && s.waves == 8) return W4A8_ERR_ARG;  // would not fit in LDS
        pl->decode = s;
    } else if (pl->tiling == W4A8_TILING_PREFILL_TILED) {
        if (variant < 0 || variant > kTiledTileMax4) return W4A8_ERR_ARG;
        pl->prefill_tile = variant ? variant : choose_tiled_tile(M, N, K);
    } else {
        if (variant < 0 || variant > kPrefillTileMax) return W4A8_ERR_ARG;
        pl->prefill_tile = variant ? kRowTiles[variant - 1] : choose_row_tile(M, N, K);
    }
    return W4A8_OK;
}

int run_gemm(const int8_t *xq, const float *s_a, const uint8_t *wp, const float *s_w, void *out_fp16, int32_t *acc_i32,
             int M, int N, int K, int tiling, int variant, void *stream) {
    const bool want_acc = acc_i32 != nullptr;
    if ((out_fp16 != nullptr) == want_acc) return W4A8_ERR_NULL;  // exactly one output
    if (!xq || !wp) return W4A8_ERR_NULL;
    if (!want_acc && (!s_a || !s_w)) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (tiling < W4A8_TILING_AUTO || tiling > W4A8_TILING_AUTO_TILED || variant < 0) return W4A8_ERR_ARG;
    if (misaligned(xq) || misaligned(wp) || misaligned(out_fp16) || misaligned(acc_i32) || (s_w && misaligned(s_w)))
        return W4A8_ERR_ALIGN;

    Plan pl{};
    if (int e = choose_plan(M, N, K, tiling, variant, &pl)) return e;
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t err;
    if (pl.tiling == W4A8_TILING_PREFILL_TILED) {
        PrefillArgs a{};
        a.xq = xq; a.s_a = s_a; a.wp = wp; a.s_w = s_w;
        a.out = out_fp16; a.acc_out = acc_i32;
        a.M = M; a.N = N; a.K = K; a.ldc = N;
        err = launch_tile(a, want_acc, false, pl.prefill_tile, st, 4);
    } else if (pl.tiling != W4A8_TILING_PREFILL) {
        DecodeArgs a{};
        a.xq = xq; a.s_a = s_a; a.wp = wp; a.s_w = s_w;
        a.out = out_fp16; a.acc_out = acc_i32;
        a.M = M; a.N = N; a.K = K;
        a.rows_per_wg = pl.decode.rows_per_wg;
        a.chunk_rows = pl.decode.chunk_rows;
        a.x_direct = pl.decode.x_direct;
        err = launch_gemm_decode(a, want_acc, pl.decode, st);
    } else {
        PrefillArgs a{};
        a.xq = xq; a.s_a = s_a; a.wp = wp; a.s_w = s_w;
        a.out = out_fp16; a.acc_out = acc_i32;
        a.M = M; a.N = N; a.K = K; a.ldc = N;
        err = launch_gemm_prefill_row(a, want_acc, pl.prefill_tile, st);
    }
    return launched(err);
}

}  // namespace

extern "C" {

int w4a8_version(void) { return 100; }

const char *w4a8_last_hip_error(void) { return hipGetErrorName(last_hip_error); }

const char *w4a8_strerror(int err) {
    switch (err) {
        case W4A8_OK: return "ok";
        case W4A8_ERR_NULL: return "a required pointer is NULL (or both / neither output given)";
        case W4A8_ERR_SHAPE: return "shape outside the contract: M,N >= 1, 32 <= K <= 65536, K % 32 == 0";
        case W4A8_ERR_ALIGN: return "device pointer not 16-byte aligned";
        case W4A8_ERR_WORKSPACE: return "workspace smaller than w4a8_gemm_workspace_bytes reports";
        case W4A8_ERR_LAUNCH: return "HIP rejected the kernel launch";
        case W4A8_ERR_VALUE: return "weight code outside [-8, 7]";
        case W4A8_ERR_ARG: return "tiling id or variant not available for this shape";
        default: return "unknown w4a8 error code";
    }
}

int w4a8_quantize_act(const void *x_fp16, int8_t *xq, float *s_a, int M, int K, void *stream) {
    if (!x_fp16 || !xq || !s_a) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, 1, K)) return e;
    if (misaligned(x_fp16) || misaligned(xq)) return W4A8_ERR_ALIGN;
    return launched(launch_quantize_act(x_fp16, K, xq, s_a, M, K, static_cast<hipStream_t>(stream)));
}

int w4a8_quantize_act_strided(const void *x_fp16, long long ldx, int8_t *xq, float *s_a, int M, int K, void *stream) {
    if (!x_fp16 || !xq || !s_a) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, 1, K)) return e;
    if (ldx < K || (ldx & 7) != 0) return W4A8_ERR_SHAPE;  // rows must not overlap and must start 16-byte aligned
    if (misaligned(x_fp16) || misaligned(xq)) return W4A8_ERR_ALIGN;
    return launched(launch_quantize_act(x_fp16, ldx, xq, s_a, M, K, static_cast<hipStream_t>(stream)));
}

size_t w4a8_gemm_workspace_bytes(int M, int N, int K) {
    (void)M; (void)N; (void)K;
    return 0;  // no tiling needs scratch memory: partial sums meet in LDS
}

int w4a8_gemm(const int8_t *xq, const float *s_a, const uint8_t *wp, const float *s_w, void *out_fp16, int M, int N, int K,
              void *workspace, size_t workspace_bytes, void *stream) {
    (void)workspace; (void)workspace_bytes;
    if (!out_fp16) return W4A8_ERR_NULL;
    return run_gemm(xq, s_a, wp, s_w, out_fp16, nullptr, M, N, K, W4A8_TILING_AUTO, 0, stream);
}

int w4a8_gemm_acc_i32(const int8_t *xq, const uint8_t *wp, int32_t *acc, int M, int N, int K, void *workspace,
                      size_t workspace_bytes, void *stream) {
    (void)workspace; (void)workspace_bytes;
    if (!acc) return W4A8_ERR_NULL;
    return run_gemm(xq, nullptr, wp, nullptr, nullptr, acc, M, N, K, W4A8_TILING_AUTO, 0, stream);
}

int w4a8_gemm_tuned(const int8_t *xq, const float *s_a, const uint8_t *wp, const float *s_w, void *out_fp16,
                    int32_t *acc_i32, int M, int N, int K, int tiling, int variant, void *workspace, size_t workspace_bytes,
                    void *stream) {
    (void)workspace; (void)workspace_bytes;
    return run_gemm(xq, s_a, wp, s_w, out_fp16, acc_i32, M, N, K, tiling, variant, stream);
}

size_t w4a8_tiled_weight_bytes(int N, int K) {
    if (check_gemm_shape(1, N, K)) return 0;
    return tiled_weight_bytes(N, K);
}

int w4a8_tile_weights(const uint8_t *wp, uint8_t *wt, int N, int K, void *stream) {
    if (!wp || !wt) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(1, N, K)) return e;
    if (misaligned(wp) || misaligned(wt)) return W4A8_ERR_ALIGN;
    return launched(launch_tile_weights(wp, wt, N, K, static_cast<hipStream_t>(stream)));
}

int w4a8_gemm_tiled(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16, int M, int N,
                    int K, void *stream) {
    if (!out_fp16) return W4A8_ERR_NULL;
    return run_gemm(xq, s_a, wt, s_w, out_fp16, nullptr, M, N, K, W4A8_TILING_AUTO_TILED, 0, stream);
}

int w4a8_gemm_tiled_swiglu(const int8_t *xq, const float *s_a, const uint8_t *wt_gu, const float *s_w_gu, void *h_fp16, int M,
                           int I, int K, void *stream) {
    if (!xq || !s_a || !wt_gu || !s_w_gu || !h_fp16) return W4A8_ERR_NULL;
    if (I < 32 || (I % 32) != 0 || I > W4A8_MAX_K) return W4A8_ERR_SHAPE;  // I follows the K contract, as in w4a8_silu_mul
    const int N = 2 * I;
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (misaligned(xq) || misaligned(wt_gu) || misaligned(h_fp16) || misaligned(s_w_gu)) return W4A8_ERR_ALIGN;
    if (!one_launch_covers(M, N, K)) return W4A8_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const TiledPlan pl = tiled_plan(M, N, K, true);
    if (pl.wide) {
        DecodeArgs d{};
        d.xq = xq; d.s_a = s_a; d.wp = wt_gu; d.s_w = s_w_gu; d.out = h_fp16;
        return launched(launch_wide(d, M, N, K, pl.shape, false, st));
    }
    PrefillArgs a{};
    a.xq = xq; a.s_a = s_a; a.wp = wt_gu; a.s_w = s_w_gu; a.out = h_fp16;
    a.M = M; a.N = N; a.K = K; a.ldc = I;
    return launched(launch_tile(a, false, true, pl.tile, st, 4));
}

// ---- K split over workgroups for shapes whose tiles alone leave most of the chip idle (medium M, small N)

namespace {

// What w4a8_gemm_tiled_splitk asks of its caller for a shape: how many slabs of raw sums the workspace has to hold, and by
// that which calls are refused.  Callers size buffers by it (w4a8_gemm_tiled_workspace_bytes) and the static entry refuses by
// it, so it is a rule of its own that does not move with the prices of plan_tiled; the library's choice stays within it and
// often needs less.
//   17 to 64 tokens: as few slices as let a slice of K fit the registers of the weight-streaming kernel, up to 8;
//   else, and up to 512 tokens: where the tiles fill up to half the compute units (all of them on a long K), as many slices
//   as bring two workgroups to every compute unit, at least 12 stages each and at most 6.  The tiles are those of a rule by
//   rounds and area; a forced tile is cut by the same rule.
struct SlabRule {
    int slices;
    bool ring;  // slices of the large-M kernel, whose one launch must cover the problem
};

long long tile_count(int M, int N, int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

struct TileShape { int bm, bn; };
constexpr TileShape kForcedTiles[] = {{0, 0},     {256, 256}, {256, 256}, {128, 256}, {128, 160}, {128, 128}, {64, 128},
                                      {64, 64},   {32, 128},  {128, 160}, {128, 128}, {256, 192}, {128, 256}};
static_assert(sizeof kForcedTiles / sizeof kForcedTiles[0] == kTiledTileMax4 + 1, "one shape per tile that can be forced");

TileShape slab_rule_tile(int M, int N, bool long_k, int cus) {
    auto count = [&](int bm, int bn) { return tile_count(M, N, bm, bn); };
    if (M <= 32) return {32, 128};
    if (M <= 64) return count(64, 128) * 4 >= cus * 3ll ? TileShape{64, 128} : TileShape{64, 64};
    if (count(128, 128) * 4 < cus * 3ll) return long_k ? TileShape{128, 128} : TileShape{64, 128};
    struct Option { int bm, bn, per_cu; double eff, alone; };
    const Option options[] = {{256, 256, 1, 1.00, 1.0},  {256, 192, 1, 0.97, 1.0},  {128, 256, 2, 0.93, 0.73}, {128, 256, 1, 0.85, 1.0},
                              {128, 160, 2, 0.66, 0.63}, {128, 128, 2, 0.75, 0.67}, {64, 128, 2, 0.60, 0.75},  {128, 128, 1, 0.60, 1.0}};
    TileShape best{256, 256};
    double best_cost = 0;
    for (const Option &o : options) {
        const long long tiles = count(o.bm, o.bn), slots = (long long)cus * o.per_cu, full = tiles / slots, rest = tiles % slots;
        const double last = rest == 0 ? 0.0 : ((o.per_cu > 1 && rest <= cus) ? o.alone : 1.0);
        const double cost = ((double)full + last) * o.bm * o.bn * o.per_cu / o.eff;
        if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = {o.bm, o.bn}; }
    }
    if (best.bm == 64 && long_k && count(128, 128) <= cus) best = {128, 128};
    return best;
}

SlabRule slab_rule(int M, int N, int K, int variant, int cus) {
    if (variant == 0 && M <= kResidentMaxM)
        for (int s = 1; s <= kMaxSlices; ++s) {
            DecodeShape t{};
            if (resident_shape(M, N, K, 0, 0, 0, false, -1, true, &t, s, true)) return {s, false};
        }
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK;
    const bool long_k = stages >= 64;
    if (M > kSplitMaxM) return {1, true};
    const TileShape t = variant ? kForcedTiles[variant] : slab_rule_tile(M, N, long_k, cus);
    const long long tiles = tile_count(M, N, t.bm, t.bn);
    if (tiles > (long_k ? cus : cus / 2)) return {1, true};
    int s = (int)((2ll * cus + tiles / 2) / tiles);
    if (s > 6) s = 6;
    if (s > stages / 12) s = stages / 12;
    if (s < 1) s = 1;
    const int per = (stages + s - 1) / s;
    return {(stages + per - 1) / per, true};  // no empty slice
}

Route make_route(int M, int N, int K, RouteKind kind, int cus) {
    Route r{};
    if (kind == kInt8) {
        r.plan.tile = choose_tiled_tile8(M, N, K);
        return r;
    }
    if (kind == kSliced) {
        const SlabRule rule = slab_rule(M, N, K, 0, cus);
        r.need = rule.slices > 1 ? rule.slices * ((size_t)M * (size_t)N * sizeof(int32_t)) : 0;
        r.one_launch = rule.ring && rule.slices > 1;
    }
    r.plan = plan_tiled(M, N, K, r.need, kind == kSwiglu, cus);
    return r;
}

// What w4a8_gemm_tiled_splitk does with a shape and a forced tile or slice count, if any.  stream: token generation (up to 16
// tokens, nothing forced), the entry without slices.
struct SplitRoute : Route {
    bool stream;
};

SplitRoute split_route(int M, int N, int K, int variant, int splits) {
    if (variant == 0 && splits == 0) return M <= 16 ? SplitRoute{{}, true} : SplitRoute{tiled_route(M, N, K, kSliced), false};
    SplitRoute r{};
    const size_t slab = (size_t)M * (size_t)N * sizeof(int32_t);
    const int stages = (K + kTiledBlockK - 1) / kTiledBlockK;
    TiledPlan &pl = r.plan;
    if (variant == 0 && M > 16 && M <= kResidentMaxM && splits <= stages &&
        resident_shape(M, N, K, 0, 0, 0, false, -1, true, &pl.shape, splits, true)) {
        // a forced count without a tile: slices of the weight-streaming kernel where it has a shape for them
        pl.wide = true;
        pl.splits = pl.shape.k_slices;
        r.need = splits > 1 ? splits * slab : 0;
        return r;
    }
    if (splits == 0) splits = slab_rule(M, N, K, variant, compute_units()).slices;
    if (splits > stages) splits = stages;
    pl.tile = variant ? variant : choose_tiled_tile(M, N, K);
    pl.stages_per_split = (stages + splits - 1) / splits;
    pl.splits = (stages + pl.stages_per_split - 1) / pl.stages_per_split;  // no empty slice
    r.one_launch = pl.splits > 1;
    r.need = pl.splits > 1 ? pl.splits * slab : 0;
    return r;
}

}  // namespace

size_t w4a8_gemm_tiled_workspace_bytes(int M, int N, int K) {
    if (check_gemm_shape(M, N, K)) return 0;
    return split_route(M, N, K, 0, 0).need;  // a forced count is checked against the buffer at the call
}

static int splitk_on_route(const SplitRoute &route, const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16,
                           int M, int N, int K, void *workspace, size_t workspace_bytes, void *stream) {
    if (route.stream)  // token generation: the weight-streaming kernels over the same array
        return run_gemm(xq, s_a, wt, s_w, out_fp16, nullptr, M, N, K, W4A8_TILING_AUTO_TILED, 0, stream);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const TiledPlan &pl = route.plan;
    const bool sliced = pl.splits > 1;
    if (route.need) {
        if (route.one_launch && !one_launch_covers(M, N, K)) return W4A8_ERR_SHAPE;
        if (!workspace) return W4A8_ERR_NULL;
        if (workspace_bytes < route.need) return W4A8_ERR_WORKSPACE;
    }
    int32_t *const slabs = sliced ? static_cast<int32_t *>(workspace) : nullptr;
    void *const out = sliced ? nullptr : out_fp16;
    hipError_t e;
    if (pl.wide) {
        DecodeArgs d{};
        d.xq = xq; d.s_a = s_a; d.wp = wt; d.s_w = s_w; d.out = out; d.acc_out = slabs;
        e = launch_wide(d, M, N, K, pl.shape, sliced, st);
    } else {
        PrefillArgs a{};
        a.xq = xq; a.s_a = s_a; a.wp = wt; a.s_w = s_w; a.out = out; a.acc_out = slabs;
        a.M = M; a.N = N; a.K = K; a.ldc = N;
        a.splits = pl.splits;
        a.stages_per_split = pl.stages_per_split;
        e = launch_tile(a, sliced, false, pl.tile, st, 4);
    }
    if (int err = launched(e); err || !sliced) return err;
    return launched(launch_splitk_epilogue(slabs, pl.splits, s_a, s_w, out_fp16, M, N, st));
}

static int check_splitk(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, const void *out_fp16, int M, int N, int K,
                        int variant, int splits) {
    if (!xq || !s_a || !wt || !s_w || !out_fp16) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (variant < 0 || variant > kTiledTileMax4 || splits < 0 || splits > 64) return W4A8_ERR_ARG;
    if (misaligned(xq) || misaligned(wt) || misaligned(out_fp16) || misaligned(s_w)) return W4A8_ERR_ALIGN;
    return W4A8_OK;
}

int w4a8_gemm_tiled_splitk(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16, int M,
                           int N, int K, int variant, int splits, void *workspace, size_t workspace_bytes, void *stream) {
    if (int e = check_splitk(xq, s_a, wt, s_w, out_fp16, M, N, K, variant, splits)) return e;
    if (misaligned(workspace)) return W4A8_ERR_ALIGN;
    return splitk_on_route(split_route(M, N, K, variant, splits), xq, s_a, wt, s_w, out_fp16, M, N, K, workspace,
                           workspace_bytes, stream);
}

// what the norm in front of the fused quantiser needs (gamma == NULL: no norm)
struct NormArgs {
    const void *res;
    long long ldres;
    const void *gamma;
    float eps;
    void *r_out, *y_out;
};

// quantiser + GEMM in one launch; swiglu: N = 2 I interleaved gate / up channels, out = h
static int linear_tiled(const void *x_fp16, long long ldx, const uint8_t *wt, const float *s_w, void *out_fp16, float *s_a_out,
                        int M, int N, int K, bool swiglu, void *stream, const NormArgs *norm = nullptr) {
    if (!x_fp16 || !wt || !s_w || !out_fp16) return W4A8_ERR_NULL;
    if (norm) {
        if (!norm->gamma) return W4A8_ERR_NULL;
        if (!(norm->eps >= 0.0f) || !(norm->eps < 3.0e38f)) return W4A8_ERR_ARG;
        if (norm->res && (norm->ldres < K || (norm->ldres & 7) != 0)) return W4A8_ERR_SHAPE;
        if (misaligned(norm->res) || misaligned(norm->gamma) || misaligned(norm->r_out) || misaligned(norm->y_out)) return W4A8_ERR_ALIGN;
        if (norm->res && ((unsigned long long)(M > 0 ? M - 1 : 0) * (unsigned long long)norm->ldres + (unsigned long long)K) * 2ull > 0xFFFF0000ull)
            return W4A8_ERR_SHAPE;
    }
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (ldx < K || (ldx & 7) != 0) return W4A8_ERR_SHAPE;  // rows must not overlap and must start 16-byte aligned
    if (misaligned(x_fp16) || misaligned(wt) || misaligned(out_fp16) || misaligned(s_w)) return W4A8_ERR_ALIGN;
    if (M > 4) return W4A8_ERR_ARG;
    if (((unsigned long long)(M - 1) * (unsigned long long)ldx + (unsigned long long)K) * 2ull > 0xFFFF0000ull) return W4A8_ERR_SHAPE;
    DecodeShape shape{};
    shape.fused_quant = true;
    shape.swiglu = swiglu;
    shape.norm = norm != nullptr;
    if (!resident_shape(M, N, K, 0, 0, 0, false, -1, true, &shape)) return W4A8_ERR_ARG;
    // both copies of the rows (fp16 and int8, padded to the 1 KB pieces of the copy; with the norm the residual rows as
    // well) must fit in LDS beside the slots of the partial sums
    const long long row_bytes = ((K + 1023) / 1024) * 1024 + 16 + (norm ? 2 : 1) * ((2ll * K + 1023) / 1024) * 1024;
    if (row_bytes * M + 3 * 1024 + 2ll * shape.prefetch * shape.waves * 1024 > 160 * 1024) return W4A8_ERR_ARG;
    DecodeArgs a{};
    a.x16 = static_cast<const uint16_t *>(x_fp16);
    a.ldx = ldx;
    a.s_a_out = s_a_out;
    a.wp = wt; a.s_w = s_w; a.out = out_fp16;
    a.M = M; a.N = N; a.K = K;
    a.rows_per_wg = shape.rows_per_wg;
    a.chunk_rows = shape.chunk_rows;
    if (norm) {
        a.res16 = static_cast<const uint16_t *>(norm->res);
        a.ldres = norm->ldres;
        a.gamma = static_cast<const uint16_t *>(norm->gamma);
        a.eps = norm->eps;
        a.r_out = static_cast<uint16_t *>(norm->r_out);
        a.y_out = static_cast<uint16_t *>(norm->y_out);
    }
    return launched(launch_gemm_decode(a, false, shape, static_cast<hipStream_t>(stream)));
}

int w4a8_linear_tiled_norm_fp16(const void *x_fp16, long long ldx, const void *res_fp16, long long ldres, const void *gamma_fp16,
                                float eps, void *r_out_fp16, void *y_out_fp16, const uint8_t *wt, const float *s_w, void *out_fp16,
                                float *s_a_out, int M, int N, int K, int swiglu, void *stream) {
    if (swiglu != 0 && swiglu != 1) return W4A8_ERR_ARG;
    if (swiglu && ((N & 63) != 0 || N / 2 > W4A8_MAX_K)) return W4A8_ERR_SHAPE;  // N = 2 I, I follows the K contract
    const NormArgs norm{res_fp16, ldres, gamma_fp16, eps, r_out_fp16, y_out_fp16};
    return linear_tiled(x_fp16, ldx, wt, s_w, out_fp16, s_a_out, M, N, K, swiglu != 0, stream, &norm);
}

int w4a8_linear_tiled_fp16(const void *x_fp16, long long ldx, const uint8_t *wt, const float *s_w, void *out_fp16,
                           float *s_a_out, int M, int N, int K, void *stream) {
    return linear_tiled(x_fp16, ldx, wt, s_w, out_fp16, s_a_out, M, N, K, false, stream);
}

int w4a8_linear_tiled_swiglu_fp16(const void *x_fp16, long long ldx, const uint8_t *wt_gu, const float *s_w_gu, void *h_fp16,
                                  float *s_a_out, int M, int I, int K, void *stream) {
    if (I < 32 || (I % 32) != 0 || I > W4A8_MAX_K) return W4A8_ERR_SHAPE;
    return linear_tiled(x_fp16, ldx, wt_gu, s_w_gu, h_fp16, s_a_out, M, 2 * I, K, true, stream);
}

int w4a8_gemm_tiled_splitk_static(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16,
                                  int M, int N, int K, int variant, int splits, void *stream) {
    if (int e = check_splitk(xq, s_a, wt, s_w, out_fp16, M, N, K, variant, splits)) return e;
    const SplitRoute route = split_route(M, N, K, variant, splits);
    if (route.need > kStaticScratchBytes) return W4A8_ERR_WORKSPACE;
    void *ws = nullptr;
    if (int e = static_scratch(&ws)) return e;
    return splitk_on_route(route, xq, s_a, wt, s_w, out_fp16, M, N, K, ws, kStaticScratchBytes, stream);
}

int w4a8_route(int entry, int M, int N, int K, int variant, int splits, int *tiling, int *tile, int *slices) {
    if (!tiling || !tile || !slices) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, N, K)) return e;
    *tile = 0;
    *slices = 1;
    auto report = [&](const TiledPlan &pl) {
        *tiling = pl.wide ? W4A8_TILING_DECODE_RESIDENT_TILED : W4A8_TILING_PREFILL_TILED;
        *tile = pl.wide ? 0 : pl.tile;
        *slices = pl.splits > 1 ? pl.splits : 1;
        return (int)W4A8_OK;
    };
    auto plan = [&](int auto_tiling) {
        Plan pl{};
        if (int e = choose_plan(M, N, K, auto_tiling, 0, &pl)) return e;
        const bool tiled = auto_tiling == W4A8_TILING_AUTO_TILED;
        *tiling = !tiled                                      ? pl.tiling
                  : pl.tiling == W4A8_TILING_DECODE_RESIDENT ? W4A8_TILING_DECODE_RESIDENT_TILED
                  : pl.tiling == W4A8_TILING_DECODE_STREAM   ? W4A8_TILING_DECODE_STREAM_TILED
                                                              : pl.tiling;
        if (pl.tiling == W4A8_TILING_PREFILL || pl.tiling == W4A8_TILING_PREFILL_TILED) *tile = pl.prefill_tile;
        return (int)W4A8_OK;
    };
    switch (entry) {
        case W4A8_ROUTE_GEMM: return plan(W4A8_TILING_AUTO);
        case W4A8_ROUTE_GEMM_TILED: return plan(W4A8_TILING_AUTO_TILED);
        case W4A8_ROUTE_SPLITK:
        case W4A8_ROUTE_SPLITK_STATIC: {
            if (variant < 0 || variant > kTiledTileMax4 || splits < 0 || splits > 64) return W4A8_ERR_ARG;
            const SplitRoute r = split_route(M, N, K, variant, splits);
            if (entry == W4A8_ROUTE_SPLITK_STATIC && r.need > kStaticScratchBytes) return W4A8_ERR_WORKSPACE;
            if (r.one_launch && !one_launch_covers(M, N, K)) return W4A8_ERR_SHAPE;
            return r.stream ? plan(W4A8_TILING_AUTO_TILED) : report(r.plan);
        }
        case W4A8_ROUTE_SWIGLU:
            if (N % 64 != 0 || !one_launch_covers(M, N, K)) return W4A8_ERR_SHAPE;
            return report(tiled_plan(M, N, K, true));
        case W4A8_ROUTE_W8A8:
        case W4A8_ROUTE_UNSIGNED:
            *tiling = W4A8_TILING_PREFILL_TILED;
            *tile = entry == W4A8_ROUTE_W8A8 ? tiled_route(M, N, K, kInt8).plan.tile : choose_unsigned_tile(M, N, K);
            return W4A8_OK;
        default: return W4A8_ERR_ARG;
    }
}

unsigned long long w4a8_plans_made(void) { return plans_made; }

int w4a8_init(void) {
    // some four hundred kernels, each asked for once per device: a caller may call this before every set-up of a layer
    static std::atomic<bool> done[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices && done[dev].load(std::memory_order_acquire)) return W4A8_OK;
    void *ws = nullptr;
    if (int e = static_scratch(&ws)) return e;
    (void)compute_units();
    if (int e = launched(prepare_tiled_kernels())) return e;
    if (int e = launched(prepare_row_kernels())) return e;
    if (int e = launched(prepare_medium_kernels())) return e;
    if (int e = launched(prepare_decode_kernels())) return e;
    done[dev].store(true, std::memory_order_release);  // static_scratch has seen to the device's number
    return W4A8_OK;
}

// ---- W8A8 comparison variant: int8 weight codes in the tiled layout, the same kernels without the int4 conversion

size_t w8a8_tiled_weight_bytes(int N, int K) {
    if (check_gemm_shape(1, N, K)) return 0;
    return tiled_weight_bytes(N, K, 8);
}

int w8a8_tile_weights(const int8_t *w8, uint8_t *wt, int N, int K, void *stream) {
    if (!w8 || !wt) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(1, N, K)) return e;
    if (misaligned(w8) || misaligned(wt)) return W4A8_ERR_ALIGN;
    return launched(launch_tile_weights8(w8, wt, N, K, static_cast<hipStream_t>(stream)));
}

static int gemm_tiled_variant(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16,
                              int32_t *acc_i32, int M, int N, int K, int variant, void *stream, int wfmt);

int w8a8_gemm_tiled(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16,
                    int32_t *acc_i32, int M, int N, int K, int variant, void *stream) {
    return gemm_tiled_variant(xq, s_a, wt, s_w, out_fp16, acc_i32, M, N, K, variant, stream, 8);
}

// ---- ablation: the vanilla unsigned storage (u = w + 8 in the nibbles, 8 subtracted in registers), same tiled layout

int w4a8_gemm_tiled_unsigned(const int8_t *xq, const float *s_a, const uint8_t *ut, const float *s_w, void *out_fp16,
                             int32_t *acc_i32, int M, int N, int K, int variant, void *stream) {
    return gemm_tiled_variant(xq, s_a, ut, s_w, out_fp16, acc_i32, M, N, K, variant, stream, kWeightsUnsigned4);
}

// ---- ablation: fine-grained (group-wise) weight scales, Eq. (5)

int w4a8_gemm_fine_grained(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_g, int ldg, void *out_fp16,
                           int M, int N, int K, int variant, void *stream) {
    if (!xq || !s_a || !wt || !s_g || !out_fp16) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (K % kTiledBlockK != 0 || ldg < N || (ldg & 3) != 0) return W4A8_ERR_SHAPE;
    // one launch covers the problem: every byte offset inside the kernel stays below 2^32
    const long long kMaxBytes = 0xF0000000ll;
    if ((long long)M * K > kMaxBytes || (long long)tiled_weight_bytes(N, K, 4) > kMaxBytes ||
        (long long)(K / kTiledBlockK) * ldg * 4 > kMaxBytes)
        return W4A8_ERR_SHAPE;
    if (variant < 0 || variant > kFineTileMax) return W4A8_ERR_ARG;
    if (misaligned(xq) || misaligned(wt) || misaligned(out_fp16) || misaligned(s_g)) return W4A8_ERR_ALIGN;
    PrefillArgs a{};
    a.xq = xq; a.s_a = s_a; a.wp = wt; a.s_w = s_g;
    a.out = out_fp16;
    a.M = M; a.N = N; a.K = K; a.ldc = N; a.ldg = ldg;
    const int tile = variant ? variant : choose_fine_tile(M, N);
    return launched(launch_gemm_prefill_tiled(a, false, tile, static_cast<hipStream_t>(stream), kWeightsFineGrained4));
}

static int gemm_tiled_variant(const int8_t *xq, const float *s_a, const uint8_t *wt, const float *s_w, void *out_fp16,
                              int32_t *acc_i32, int M, int N, int K, int variant, void *stream, int wfmt) {
    const bool want_acc = acc_i32 != nullptr;
    if ((out_fp16 != nullptr) == want_acc) return W4A8_ERR_NULL;  // exactly one output
    if (!xq || !wt) return W4A8_ERR_NULL;
    if (!want_acc && (!s_a || !s_w)) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, N, K)) return e;
    if (variant < 0 || variant > kTiledTileMax) return W4A8_ERR_ARG;
    if (misaligned(xq) || misaligned(wt) || misaligned(out_fp16) || misaligned(acc_i32) || (s_w && misaligned(s_w)))
        return W4A8_ERR_ALIGN;
    PrefillArgs a{};
    a.xq = xq; a.s_a = s_a; a.wp = wt; a.s_w = s_w;
    a.out = out_fp16; a.acc_out = acc_i32;
    a.M = M; a.N = N; a.K = K; a.ldc = N;
    const int tile = variant ? variant
                             : wfmt == 8 ? tiled_route(M, N, K, kInt8).plan.tile : choose_unsigned_tile(M, N, K);
    return launched(launch_tile(a, want_acc, false, tile, static_cast<hipStream_t>(stream), wfmt));
}

int w4a8_quantize_weights(const void *w_fp16, uint8_t *wp, float *s_w, int N, int K, void *stream) {
    if (!w_fp16 || !wp || !s_w) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(1, N, K)) return e;
    if (misaligned(w_fp16) || misaligned(wp)) return W4A8_ERR_ALIGN;
    return launched(launch_quantize_weights(w_fp16, wp, s_w, N, K, static_cast<hipStream_t>(stream)));
}

int w4a8_quantize_weights_clipped(const void *w_fp16, const float *gamma, const float *beta, uint8_t *wp, float *s_w, int N,
                                  int K, void *stream) {
    if (!w_fp16 || !wp || !s_w) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(1, N, K)) return e;
    if (misaligned(w_fp16) || misaligned(wp)) return W4A8_ERR_ALIGN;
    return launched(launch_quantize_weights_clip(w_fp16, gamma, beta, wp, s_w, N, K, static_cast<hipStream_t>(stream)));
}

int w4a8_silu_mul(const void *gate_up_fp16, void *h_fp16, int M, int I, void *stream) {
    if (!gate_up_fp16 || !h_fp16) return W4A8_ERR_NULL;
    if (M < 1 || I < 8 || (I % 8) != 0 || M > 65535) return W4A8_ERR_SHAPE;
    if (misaligned(gate_up_fp16) || misaligned(h_fp16)) return W4A8_ERR_ALIGN;
    return launched(launch_silu_mul(gate_up_fp16, h_fp16, M, I, static_cast<hipStream_t>(stream)));
}

int w4a8_silu_mul_quantize(const void *gate_up_fp16, int8_t *xq, float *s_a, int M, int I, void *stream) {
    if (!gate_up_fp16 || !xq || !s_a) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, 1, I)) return e;  // I is the K of the GEMM that consumes xq
    if (misaligned(gate_up_fp16) || misaligned(xq)) return W4A8_ERR_ALIGN;
    return launched(launch_silu_mul_quantize(gate_up_fp16, xq, s_a, M, I, static_cast<hipStream_t>(stream)));
}

// ---- probes of what the chip sustains (context for the measurements, no part of the path)

int w4a8_add_rmsnorm_quantize(const void *x_fp16, const void *res_fp16, const void *gamma_fp16, float eps, void *r_out_fp16,
                              void *y_out_fp16, int8_t *xq, float *s_a, int M, int K, void *stream) {
    if (!x_fp16 || !gamma_fp16 || !xq || !s_a) return W4A8_ERR_NULL;
    if (int e = check_gemm_shape(M, 1, K)) return e;
    if (!(eps >= 0.0f) || !(eps < 3.0e38f)) return W4A8_ERR_ARG;  // also refuses NaN
    if (misaligned(x_fp16) || misaligned(res_fp16) || misaligned(gamma_fp16) || misaligned(r_out_fp16) || misaligned(y_out_fp16) ||
        misaligned(xq))
        return W4A8_ERR_ALIGN;
    return launched(launch_add_rmsnorm_quantize(x_fp16, res_fp16, gamma_fp16, eps, r_out_fp16, y_out_fp16, xq, s_a, M, K,
                                                static_cast<hipStream_t>(stream)));
}

int w4a8_probe_stream_read(const void *buf, size_t bytes, void *sink, void *stream) {
    if (!buf || !sink) return W4A8_ERR_NULL;
    if (bytes < 16) return W4A8_ERR_SHAPE;
    if (misaligned(buf)) return W4A8_ERR_ALIGN;
    return launched(launch_probe_stream_read(buf, bytes, static_cast<unsigned *>(sink), 8 * compute_units(), static_cast<hipStream_t>(stream)));
}

int w4a8_probe_read_pattern(const void *buf, size_t bytes, void *sink, int pattern, int loads, int workgroups_per_cu,
                            void *stream) {
    if (!buf || !sink) return W4A8_ERR_NULL;
    if (bytes < 16 || bytes > 0xFFFFFFF0ull) return W4A8_ERR_SHAPE;
    if (misaligned(buf)) return W4A8_ERR_ALIGN;
    if (pattern < 0 || pattern > 5 || (loads != 4 && loads != 8 && loads != 16) || workgroups_per_cu < 1 || workgroups_per_cu > 64)
        return W4A8_ERR_ARG;
    return launched(launch_probe_read_pattern(buf, bytes, static_cast<unsigned *>(sink), pattern, loads, workgroups_per_cu * compute_units(), static_cast<hipStream_t>(stream)));
}

int w4a8_probe_mixed_read(const void *cold, size_t cold_bytes, const void *hot, size_t hot_bytes, void *sink, int mode,
                          void *stream) {
    if (!cold || !hot || !sink) return W4A8_ERR_NULL;
    if (misaligned(cold) || misaligned(hot)) return W4A8_ERR_ALIGN;
    if (mode < 0 || mode > 3) return W4A8_ERR_ARG;
    const int cus = compute_units();
    const size_t per_iter = (mode == 2 ? 4096u : 2048u) * 16u;               // cold bytes a workgroup reads per iteration
    if (hot_bytes < 16 || hot_bytes > 0xFFFFFFF0ull || cold_bytes < per_iter * (size_t)cus) return W4A8_ERR_SHAPE;
    size_t per_wg = cold_bytes / (size_t)cus / per_iter * per_iter;           // whole iterations, within the buffer
    if (per_wg > 0x0FFFFFF0ull) per_wg = 0x0FFFFFF0ull / per_iter * per_iter;
    return launched(launch_probe_mixed_read(cold, (unsigned)(per_wg / 16), hot, (unsigned)(hot_bytes / 16), static_cast<unsigned *>(sink),
                                            mode, cus, static_cast<hipStream_t>(stream)));
}

int w4a8_probe_mfma_int8(void *sink, int iters, int pattern, void *stream) {
    if (!sink) return W4A8_ERR_NULL;
    if (iters < 1 || iters > (1 << 24) || pattern < 0 || pattern > 1) return W4A8_ERR_ARG;
    return launched(launch_probe_mfma_i8(static_cast<int *>(sink), 2 * compute_units(), iters, pattern, static_cast<hipStream_t>(stream)));
}

int w4a8_pack_weights_host(const int8_t *wq_host, uint8_t *wp_host, int N, int K) {
    if (!wq_host || !wp_host) return W4A8_ERR_NULL;
    if (N < 1 || K < 2 || (K & 1)) return W4A8_ERR_SHAPE;
    const size_t total = (size_t)N * (size_t)(K / 2);
    for (size_t i = 0; i < total; ++i) {
        const int even = wq_host[2 * i], odd = wq_host[2 * i + 1];
        if (even < -8 || even > 7 || odd < -8 || odd > 7) return W4A8_ERR_VALUE;
    }
    for (size_t i = 0; i < total; ++i) {
        const unsigned even = (unsigned)wq_host[2 * i] & 15u, odd = (unsigned)wq_host[2 * i + 1] & 15u;
        wp_host[i] = (uint8_t)(even | (odd << 4));
    }
    return W4A8_OK;
}

}  // extern "C"
