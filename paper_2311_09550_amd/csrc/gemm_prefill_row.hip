// W4A8 GEMM for large M over int4 weights in the packed row-major storage format: the instantiations of the ring kernel
// (gemm_prefill_ring.hpp, ROW) and their launch.
#include "gemm_prefill_ring.hpp"

namespace w4a8 {

namespace {

template <int MT, int NT, int WM, int WN, int STAGES>
hipError_t launch_row_tile(const PrefillArgs &p, bool acc_out, hipStream_t stream) {
    return launch_tile<MT, NT, WM, WN, STAGES, 4, false, false, 1, true>(p, acc_out, stream);
}

hipError_t launch_slice(const PrefillArgs &p, bool acc_out, int tile, hipStream_t stream) {
    switch (tile) {
        case kTiled256x256: return launch_row_tile<8, 4, 2, 4, 3>(p, acc_out, stream);
        case kTiled128x256: return launch_row_tile<8, 4, 1, 4, 2>(p, acc_out, stream);
        case kTiled64x128: return launch_row_tile<2, 2, 2, 4, 4>(p, acc_out, stream);
        case kTiled64x64: return launch_row_tile<2, 2, 2, 2, 4>(p, acc_out, stream);
        case kTiled32x128: return launch_row_tile<2, 2, 1, 4, 4>(p, acc_out, stream);
        case kTiled64x256: return launch_row_tile<4, 2, 1, 8, 4>(p, acc_out, stream);
        case kTiled128x192: return launch_row_tile<4, 3, 2, 4, 4>(p, acc_out, stream);
        case kTiled64x192: return launch_row_tile<2, 3, 2, 4, 4>(p, acc_out, stream);
        case kTiled192x320: return launch_row_tile<6, 5, 2, 4, 3>(p, acc_out, stream);
        case kTiled192x256: return launch_row_tile<6, 4, 2, 4, 3>(p, acc_out, stream);
        case kTiled192x192: return launch_row_tile<6, 3, 2, 4, 4>(p, acc_out, stream);
        default: return hipErrorInvalidConfiguration;
    }
}

}  // namespace

// The kernel addresses its operands with 32-bit byte offsets; a problem whose activation or weight matrix is
// larger than that is cut into row slices of M and N, one launch each (the slices write disjoint parts of the output).
hipError_t launch_gemm_prefill_row(const PrefillArgs &p, bool acc_out, int tile, hipStream_t stream) {
    const long long kMaxBytes = 0xF0000000ll;
    long long m_rows = kMaxBytes / p.K, n_rows = kMaxBytes / (p.K >> 1);
    m_rows -= m_rows % 768;   // multiples of every tile height and width
    n_rows -= n_rows % 3840;
    for (long long n0 = 0; n0 < p.N; n0 += n_rows) {
        for (long long m0 = 0; m0 < p.M; m0 += m_rows) {
            PrefillArgs q = p;
            q.M = (int)((p.M - m0) < m_rows ? (p.M - m0) : m_rows);
            q.N = (int)((p.N - n0) < n_rows ? (p.N - n0) : n_rows);
            q.xq = p.xq + (size_t)m0 * p.K;
            q.wp = p.wp + (size_t)n0 * (p.K >> 1);
            if (p.s_a) q.s_a = p.s_a + m0;
            if (p.s_w) q.s_w = p.s_w + n0;
            if (p.out) q.out = (unsigned short *)p.out + (size_t)m0 * p.ldc + n0;
            if (p.acc_out) q.acc_out = p.acc_out + (size_t)m0 * p.ldc + n0;
            const hipError_t e = launch_slice(q, acc_out, tile, stream);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t prepare_row_kernels() {
    PrefillArgs a{};
    a.M = 32; a.N = 32; a.K = kTiledBlockK; a.ldc = 32;
    a.prepare_only = true;
    for (int tile : kRowTiles)
        for (int acc = 0; acc <= 1; ++acc)
            if (const hipError_t e = launch_gemm_prefill_row(a, acc != 0, tile, nullptr); e != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace w4a8
