// Kernels and dispatch of the MFMA contraction (tile code in tcol_gemm_tile.h).
#include "tcol_gemm_tile.h"
#include "tcol_launch.h"

namespace tcol {

template <int PREC, int BM, int NTW, int MODE>
__device__ __forceinline__ void gemm_body(const GraphDev* __restrict__ gd, int G, int total_tiles, int honor_stop,
                                          int passes, int cstage) {
    const int tile = batch_remap(blockIdx.x, total_tiles, G);
    int g, tm, tn;
    decode_tile<MODE>(gd, G, tile, g, tm, tn);
    gemm_tile<PREC, BM, NTW, MODE>(gd, g, tm, tn, honor_stop, passes, cstage);
}

// ------------------------------------------------------------- dispatch ------

constexpr int kMaxLds = 160 * 1024;

template <int BM, int NTW, int MODE>
static size_t lds_bytes(int cstage) {
    using T = Tile<BM, NTW>;
    const size_t sweep = T::NB * T::STAGE;
    if (MODE == 0) return sweep;
    const size_t epi = (size_t)(BM < 128 ? BM : 128) * (T::BN + 4) * sizeof(float) + (size_t)cstage;
    return sweep > epi ? sweep : epi;
}

// The contraction kernel.  Tiles that run two waves per SIMD (a second 4-wave block
// per CU, or one 8-wave block) are compiled for at most 256 registers per lane, so
// that the second wave can actually be resident.
template <int PREC, int BM, int NTW, int MODE>
__global__ __launch_bounds__(tile_threads(BM)) void k_gemm(const GraphDev* __restrict__ gd, int G,
                                                                 int total_tiles, int honor_stop, int passes,
                                                                 int cstage) {
    gemm_body<PREC, BM, NTW, MODE>(gd, G, total_tiles, honor_stop, passes, cstage);
}
template <int PREC, int BM, int NTW, int MODE>
__global__ __launch_bounds__(tile_threads(BM)) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_x2(
    const GraphDev* __restrict__ gd, int G, int total_tiles, int honor_stop, int passes, int cstage) {
    gemm_body<PREC, BM, NTW, MODE>(gd, G, total_tiles, honor_stop, passes, cstage);
}
template <int BM, int NTW, int MODE>
constexpr bool two_per_simd() {
    return MODE == 0 && Tile<BM, NTW>::TWO_PER_SIMD;
}

template <int PREC, int BM, int NTW, int MODE>
static hipError_t prep_one() {
    const void* f;
    if constexpr (two_per_simd<BM, NTW, MODE>())
        f = (const void*)k_gemm_x2<PREC, BM, NTW, MODE>;
    else
        f = (const void*)k_gemm<PREC, BM, NTW, MODE>;
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
}

template <int PREC, int BM, int NTW, int MODE>
static hipError_t launch_one(const GraphDev* gd, int G, int total_tiles, int honor_stop, int passes, int cstage,
                             hipStream_t s) {
    const size_t shm = lds_bytes<BM, NTW, MODE>(cstage);
    if (shm > (size_t)kMaxLds) return hipErrorInvalidValue;
    constexpr int threads = Tile<BM, NTW>::THREADS;
    if constexpr (two_per_simd<BM, NTW, MODE>())
        k_gemm_x2<PREC, BM, NTW, MODE><<<dim3(total_tiles), dim3(threads), shm, s>>>(gd, G, total_tiles, honor_stop,
                                                                                    passes, cstage);
    else
        k_gemm<PREC, BM, NTW, MODE><<<dim3(total_tiles), dim3(threads), shm, s>>>(gd, G, total_tiles, honor_stop,
                                                                                 passes, cstage);
    return hipGetLastError();
}

// instantiated tile shapes: (BM, NTW)
#define TCOL_GEMM_SHAPES(X, PREC, MODE) \
    X(PREC, 64, 2, MODE) X(PREC, 64, 4, MODE) X(PREC, 128, 4, MODE) X(PREC, 128, 6, MODE) X(PREC, 128, 8, MODE) \
    X(PREC, 64, 9, MODE) X(PREC, 128, 9, MODE) X(PREC, 256, 4, MODE) X(PREC, 256, 6, MODE)

#define TCOL_GEMM_CASE(PREC, BM, NTW, MODE)                                                             \
    if (s.prec == PREC && s.bm == BM && s.ntw == NTW && s.mode == MODE) {                               \
        if (op == 0) return hipSuccess;                                                                 \
        if (op == 1) return prep_one<PREC, BM, NTW, MODE>();                                             \
        if (op == 3) { *lds_out = lds_bytes<BM, NTW, MODE>(cstage); return hipSuccess; }                 \
        return launch_one<PREC, BM, NTW, MODE>(gd, G, total_tiles, honor_stop, passes, cstage, st);     \
    }

static hipError_t gemm_dispatch(int op, const GemmShape& s, const GraphDev* gd, int G, int total_tiles,
                                int honor_stop, int passes, int cstage, hipStream_t st, size_t* lds_out) {
    TCOL_GEMM_SHAPES(TCOL_GEMM_CASE, kPrecFP32, 0)
    TCOL_GEMM_SHAPES(TCOL_GEMM_CASE, kPrecFP4, 0)
    TCOL_GEMM_SHAPES(TCOL_GEMM_CASE, kPrecFP32, 1)
    TCOL_GEMM_SHAPES(TCOL_GEMM_CASE, kPrecFP4, 1)
    return hipErrorInvalidValue;
}

bool gemm_supported(const GemmShape& s) {
    return gemm_dispatch(0, s, nullptr, 0, 0, 0, 0, 0, nullptr, nullptr) == hipSuccess;
}
hipError_t gemm_prepare(const GemmShape& s) { return gemm_dispatch(1, s, nullptr, 0, 0, 0, 0, 0, nullptr, nullptr); }
hipError_t launch_gemm(const GemmShape& s, const GraphDev* gd, int G, int total_tiles, int honor_stop, int passes,
                       int cstage, hipStream_t st) {
    if (total_tiles <= 0) return hipSuccess;
    return gemm_dispatch(2, s, gd, G, total_tiles, honor_stop, passes, cstage, st, nullptr);
}
size_t gemm_lds_bytes(const GemmShape& s, int cstage) {
    size_t b = 0;
    if (gemm_dispatch(3, s, nullptr, 0, 0, 0, 0, cstage, nullptr, &b) != hipSuccess) return 0;
    return b;
}
int gemm_bn(int ntw) { return 32 * ntw; }

}  // namespace tcol
