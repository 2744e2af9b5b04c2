// Instances of the fused z pass, compiled once per group of grid sides
// (LC_FUSED_SET = 0 .. 5): one unit of them all takes minutes to compile.
#include "lc_fused_device.h"

#ifndef LC_FUSED_SET
#error "compile with -DLC_FUSED_SET=0..5"
#endif

namespace lc {

#if LC_FUSED_SET == 0
#define LC_EACH_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96)
#elif LC_FUSED_SET == 1
#define LC_EACH_N(X) X(128)
#elif LC_FUSED_SET == 2
#define LC_EACH_N(X) X(192)
#elif LC_FUSED_SET == 3
#define LC_EACH_N(X) X(256)
#elif LC_FUSED_SET == 4
#define LC_EACH_N(X) X(384)
#else
#define LC_EACH_N(X) X(512)
#endif

template <> hipError_t fused_set_launch<LC_FUSED_SET>(int n, FusedForm form, const FusedArgs &a, const void *tw_full,
                                                      hipStream_t st) {
    switch (n) {
#define X_(N)                                                                                                    \
    case N:                                                                                                      \
        return form == FusedForm::fp32 ? fused_t<N>(a, tw_full, st)                                              \
               : form == FusedForm::plain64 ? fused_plain_t<double, N>(a, tw_full, st)                           \
                                            : fused_plain_t<float, N>(a, tw_full, st);
        LC_EACH_N(X_)
#undef X_
        default: return hipErrorInvalidValue;
    }
}

#if LC_FUSED_SET == 0
template <int N> static int64_t tiles_t() {
    ColSet s0, s1;
    fused_sets<N>(s0, s1);
    return (int64_t)s0.n_wgs + s1.n_wgs;
}

int64_t fused_tiles(int n) {
    switch (n) {
#define X_(N) case N: return tiles_t<N>();
        X_(8) X_(12) X_(16) X_(24) X_(32) X_(48) X_(64) X_(96) X_(128) X_(192) X_(256) X_(384) X_(512)
#undef X_
        default: return 0;
    }
}

int fused_cpw(int n) {
    switch (n) {
#define X_(N) case N: return FusedShape<float, N, FusedTiling<N>>::CPW;
        X_(8) X_(12) X_(16) X_(24) X_(32) X_(48) X_(64) X_(96) X_(128) X_(192) X_(256) X_(384) X_(512)
#undef X_
        default: return 0;
    }
}
#endif

}  // namespace lc
