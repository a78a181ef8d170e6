// The contraction of a merged iteration with the row update in its epilogue.
//
// For a graph with gfuse the column tiles hold whole members (gr_mpb of them), so once the K-sweeps
// are done a block holds the gradient rows of its 64 or 128 vertices in those members and updates
// them itself, in place: the first launch of the iteration has already answered the stop rule.  G
// (8 bytes per weight written and read back) and the update launch fall away.  Other graphs of the
// context store G for the update launch as in tcol_gemm.hip.
//
// The epilogue takes 64 rows at a time through LDS, one member after the other: 16 lanes per row, four
// rows per group of lanes.  Its weights come from HBM, so the four rows of the next member (KPL <= 8) or
// of this one are loaded before they are needed, 64 rows x 4 k bytes in flight per block; the arithmetic is
// the row-update kernel's, in its order, so the results keep their bits.
// Planted n = 1000, k = 28, D = 128 (64 x 64 tiles): the iteration 55 -> 47 us; ECP n = 1000, k = 90,
// D = 256 (128 x 192): 145 -> 132 us; n = 500, k = 50, D = 64 (64 x 64): 28.5 -> 22.4 us.
#include "tcol_gemm_tile.h"
#include "tcol_launch.h"
#include "tcol_rows.h"

namespace tcol {

template <int BM, int NTW>
constexpr size_t rows_lds() {
    using T = Tile<BM, NTW>;
    const size_t sweep = (size_t)T::NB * T::STAGE, epi = (size_t)64 * (T::BN + 4) * sizeof(float);
    return sweep > epi ? sweep : epi;
}

template <int BM, int NTW, int KPL, int VAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_rows(
    const GraphDev* __restrict__ gd, int G, int total_tiles) {
    using T = Tile<BM, NTW>;
    constexpr int MT = T::MT, BN = T::BN;
    static_assert(T::WAVES == 4, "four waves");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int g, tm, tn;
    decode_tile<2>(gd, G, batch_remap(blockIdx.x, total_tiles, G), g, tm, tn);
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (st->stopped) return;
    const long long t = st->tc;
    const bool stop = merged_stop(d, st, t);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // graphs without gfuse end in the update launch
    const bool fuse = d.gfuse != 0;
    if (fuse && tm == 0 && tn == 0 && tid < 64) merged_end(d, st, t, stop, tid, 64);
    if (stop) return;
    const float tf = (float)t;
    const bool pen = (d.lambda * tf != 0.0f) || (d.mu * tf != 0.0f);
    const uint32_t sign = prob_partition(d.problem) ? 0x80000000u : 0u;
    const int n = d.n, k = d.k;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = tm * BM;
    const int d0 = tn * d.gr_mpb;
    const int n0 = fuse ? d0 * k : tn * BN;
    const int pS = st->pS;

    f32x4 acc[MT][NTW];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const size_t ld = op_row_bytes(kPrecFP4, d.n_pad), ld2 = (size_t)d.n_pad * 2;
    const uint8_t* S = (const uint8_t*)d.Sop[pS] + (size_t)n0 * ld;
    gemm_sweep<kPrecFP4, BM, NTW>(acc, (const uint8_t*)d.Aop + (size_t)m0 * ld, S, ld, ceil_div(n, 256), lds);
    if (pen) {
        __syncthreads();
        pen_sweep<BM, NTW>(acc, (const uint8_t*)d.Pop + (size_t)m0 * ld2, S, ld2, ld, ceil_div(n, 64), lds);
    }
    if (!fuse) {
        const int ncol_end = min(d.ncols, n0 + BN);
        float* __restrict__ Gg = d.G;
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
            const int col = n0 + wn * (NTW * 16) + nt * 16 + (lane & 15);
            if (col < ncol_end) {
                const int cm = col / k, cl = col - cm * k;
                float* __restrict__ o = Gg + ((size_t)cm * n + m0) * k + cl;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = wm * T::RW + mt * 16 + (lane >> 4) * 4 + r;
                        if (m0 + row < n) o[(size_t)row * k] = flip_sign(acc[mt][nt][r], sign);
                    }
            }
        }
        return;
    }
    // ---- row update
    constexpr int LDG = BN + 4;         // rows four apart fall on other banks, for the writes and the reads below
    constexpr bool NEXT = KPL <= 8;     // the next member's rows in flight too
    float* Gt = (float*)lds;
    const RowCtx x = row_ctx(d, t);
    const int nmem = min(d.gr_mpb, d.D - d0);
    const int l16 = tid & 15;
    const int r0 = ((tid >> 4) & 3) * 4 + wave;   // the group's first row; the others 16 apart
    float* __restrict__ W = d.W[0];
    float* __restrict__ vel = d.vel;
    const int32_t* __restrict__ V = d.V[pS];
    int16_t* __restrict__ cn = d.c[pS];
    const int cs = d.cs;
    // the loads of stages past the end still write LDS
    wait_vm<0>();
#pragma unroll 1
    for (int h = 0; h < BM / 64; ++h) {
        const int ib = m0 + h * 64 + r0;
        RowRegs<KPL, VAR> R[NEXT ? 2 : 1][4];
        float none[KPL];
        auto load = [&](RowRegs<KPL, VAR>(&Q)[4], int dm) {
            const size_t ro = ((size_t)(d0 + dm) * n + ib) * k;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (ib + 16 * u < n)
                    row_load<KPL, VAR>(Q[u], none, x, W + ro + (size_t)16 * u * k, nullptr,
                                       vel ? vel + ro + (size_t)16 * u * k : nullptr, 0, l16);
        };
        auto update = [&](RowRegs<KPL, VAR>(&Q)[4], int dm) {
            const size_t ro = ((size_t)(d0 + dm) * n + ib) * k;
            RowClasses<KPL, VAR> C;
            classes_load<KPL, VAR>(C, x, V + (size_t)(d0 + dm) * k, l16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (ib + 16 * u >= n) continue;
                const float* gr = Gt + (r0 + 16 * u) * LDG + dm * k;
                float gv[KPL];
#pragma unroll
                for (int q = 0; q < KPL; ++q)
                    if (16 * q < k) gv[q] = flip_sign(gr[min(l16 + 16 * q, k - 1)], sign);
                const int c = row_step<KPL, VAR>(Q[u], C, gv, x, W + ro + (size_t)16 * u * k,
                                                 vel ? vel + ro + (size_t)16 * u * k : nullptr, 0, nullptr, nullptr, l16);
                if (l16 == 0) {
                    if (c < 0) atomicExch(&st->next_bad, 1);
                    cn[(size_t)(d0 + dm) * cs + ib + 16 * u] = (int16_t)max(c, 0);
                }
            }
        };
        load(R[0], 0);
        stage_barrier();
        if (BM == 64 || wm == h) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = (BM == 64 ? wm * T::RW : 0) + mt * 16 + (lane >> 4) * 4 + r;
                        Gt[row * LDG + wn * (NTW * 16) + nt * 16 + (lane & 15)] = acc[mt][nt][r];
                    }
        }
        stage_barrier();
        if constexpr (NEXT) {
            for (int dm = 0; dm < nmem; dm += 2) {
                if (dm + 1 < nmem) load(R[1], dm + 1);
                update(R[0], dm);
                if (dm + 1 >= nmem) break;
                if (dm + 2 < nmem) load(R[0], dm + 2);
                update(R[1], dm + 1);
            }
        } else {
            for (int dm = 0; dm < nmem; ++dm) {
                if (dm) load(R[0], dm);
                update(R[0], dm);
            }
        }
    }
}

// instantiations (BM, NTW, KPL, VAR), where they were the fastest way for some k and D: k <= 16 KPL, two
// members and more to a column tile at small k, one at k of 97 to 128 and 193 to 256.  Momentum variants
// (VAR 3, with the added fitness term's registers too) only where they do not spill.  Others are not built: those
// graphs take the update launch.
#define TCOL_GR_KERNELS(X) \
    TCOL_GR_PLAIN(X, 0) TCOL_GR_PLAIN(X, 1) \
    X(64, 2, 2, 3) X(64, 2, 4, 3) X(64, 4, 4, 3) X(64, 4, 6, 3) X(128, 4, 4, 3) X(128, 4, 6, 3)
#define TCOL_GR_PLAIN(X, V) \
    X(64, 2, 2, V) X(64, 2, 4, V) X(64, 4, 2, V) X(64, 4, 4, V) X(64, 4, 6, V) X(64, 4, 8, V) X(64, 6, 6, V) \
    X(64, 8, 16, V) X(128, 4, 2, V) X(128, 4, 4, V) X(128, 4, 6, V) X(128, 4, 8, V) X(128, 6, 6, V)

static int rows_kpl(int kmax) {
    for (int kpl : {2, 4, 6, 8, 12, 16})
        if (16 * kpl >= kmax) return kpl;
    return 0;
}
static int rows_var(int var) { return var & 2 ? 3 : var; }

bool gemm_rows_built(int bm, int ntw, int kmax, int var) {
    const int kpl = rows_kpl(kmax), vr = rows_var(var);
#define TCOL_GR_HAS(BM, NTW, KP, VR) \
    if (bm == BM && ntw == NTW && kpl == KP && vr == VR) return true;
    TCOL_GR_KERNELS(TCOL_GR_HAS)
#undef TCOL_GR_HAS
    return false;
}

hipError_t gemm_rows_prepare(int bm, int ntw, int kmax, int var) {
    const int kpl = rows_kpl(kmax), vr = rows_var(var);
#define TCOL_GR_PREP(BM, NTW, KP, VR)                                                          \
    if (bm == BM && ntw == NTW && kpl == KP && vr == VR)                                       \
        return hipFuncSetAttribute((const void*)k_gemm_rows<BM, NTW, KP, VR>,                  \
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    TCOL_GR_KERNELS(TCOL_GR_PREP)
#undef TCOL_GR_PREP
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_rows(int bm, int ntw, int kmax, int var, const GraphDev* gd, int G, int total_tiles,
                            hipStream_t s) {
    if (total_tiles <= 0) return hipSuccess;
    const int kpl = rows_kpl(kmax), vr = rows_var(var);
    bool done = false;
#define TCOL_GR_LAUNCH(BM, NTW, KP, VR)                                                                       \
    if (!done && bm == BM && ntw == NTW && kpl == KP && vr == VR) {                                           \
        k_gemm_rows<BM, NTW, KP, VR><<<total_tiles, 256, rows_lds<BM, NTW>(), s>>>(gd, G, total_tiles);       \
        done = true;                                                                                          \
    }
    TCOL_GR_KERNELS(TCOL_GR_LAUNCH)
#undef TCOL_GR_LAUNCH
    return done ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace tcol
