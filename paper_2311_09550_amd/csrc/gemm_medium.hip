// The medium-M kernel's instantiations over int4 and int8 weights and their launch.
#include "gemm_medium.hpp"

namespace w4a8 {

namespace {

template <int MT, int NT, int NW, int KG>
hipError_t launch_medium4(const PrefillArgs &p, bool acc_out, bool swiglu, hipStream_t stream) {
    return swiglu    ? launch_medium_one<MT, NT, NW, KG, false, 4, true>(p, stream)
           : acc_out ? launch_medium_one<MT, NT, NW, KG, true, 4, false>(p, stream)
                     : launch_medium_one<MT, NT, NW, KG, false, 4, false>(p, stream);
}

template <int MT, int NT, int NW, int KG>
hipError_t launch_medium8(const PrefillArgs &p, bool acc_out, hipStream_t stream) {
    return acc_out ? launch_medium_one<MT, NT, NW, KG, true, 8, false>(p, stream)
                   : launch_medium_one<MT, NT, NW, KG, false, 8, false>(p, stream);
}

}  // namespace

hipError_t launch_gemm_medium(const PrefillArgs &p, bool acc_out, bool swiglu, int tile, hipStream_t stream, int wbits) {
    if (p.splits > 1 || (swiglu && (acc_out || wbits != 4 || (p.N & 3) || (p.ldc & 1)))) return hipErrorInvalidValue;
    if ((long long)p.M * p.K >= kMediumMaxActivations || tiled_weight_bytes(p.N, p.K, wbits) > kMediumMaxWeights) return hipErrorInvalidValue;
    if (wbits == 4) {
        switch (tile) {
            case kMedium32x32: return launch_medium4<2, 2, 1, 8>(p, acc_out, swiglu, stream);
            case kMedium32x64: return launch_medium4<2, 2, 2, 4>(p, acc_out, swiglu, stream);
            case kMedium32x64K8: return launch_medium4<2, 4, 1, 8>(p, acc_out, swiglu, stream);
            case kMedium32x96: return launch_medium4<2, 3, 2, 4>(p, acc_out, swiglu, stream);
            case kMedium48x128: return launch_medium4<3, 4, 2, 4>(p, acc_out, swiglu, stream);
            case kMedium64x96: return launch_medium4<4, 3, 2, 4>(p, acc_out, swiglu, stream);
            case kMedium64x128: return launch_medium4<4, 4, 2, 4>(p, acc_out, swiglu, stream);
            case kMedium64x160: return launch_medium4<4, 5, 2, 4>(p, acc_out, swiglu, stream);
            default: return hipErrorInvalidConfiguration;
        }
    }
    if (wbits != 8) return hipErrorInvalidConfiguration;
    switch (tile) {
        case kMedium16x16: return launch_medium8<1, 1, 1, 8>(p, acc_out, stream);
        case kMedium16x32: return launch_medium8<1, 2, 1, 8>(p, acc_out, stream);
        case kMedium32x32: return launch_medium8<2, 2, 1, 8>(p, acc_out, stream);
        case kMedium32x64: return launch_medium8<2, 2, 2, 4>(p, acc_out, stream);
        case kMedium64x96: return launch_medium8<4, 3, 2, 4>(p, acc_out, stream);
        case kMedium96x128: return launch_medium8<6, 4, 2, 4>(p, acc_out, stream);
        default: return hipErrorInvalidConfiguration;
    }
}

hipError_t prepare_medium_kernels() {
    PrefillArgs a{};
    a.M = 32; a.N = 32; a.K = kTiledBlockK; a.ldc = 32;
    a.prepare_only = true;
    for (int tile = kMediumFirst; tile <= kMediumLast; ++tile)
        for (const int wbits : {4, 8})
            for (int form = 0; form < (wbits == 4 ? 3 : 2); ++form) {
                const hipError_t e = launch_gemm_medium(a, form == 1, form == 2, tile, nullptr, wbits);
                if (e != hipSuccess && e != hipErrorInvalidConfiguration) return e;  // not every tile serves both formats
            }
    return hipSuccess;
}

}  // namespace w4a8
