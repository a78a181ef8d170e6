// The row update on 16 lanes (softmax, straight-through gradient, update, smoothing, argmax) and the
// end of a merged iteration: device code shared by the row-update kernel, the class-row sums and the
// contraction with the row update.
#pragma once

#include "tcol_internal.h"

#include <math.h>

namespace tcol {

__device__ inline bool finite_f(float x) { return (__float_as_uint(x) & 0x7F800000u) != 0x7F800000u; }

// global-address-space views: loads through them are not ordered against LDS
// operations (a flat pointer may alias LDS, which pins every flat load behind
// the LDS atomics and barriers before it)
template <typename T>
__device__ inline const __attribute__((address_space(1))) T* gview(const T* p) {
    return (const __attribute__((address_space(1))) T*)p;
}
// x with the sign bits of `sign` flipped in.  Not a product with +-1: the compiler could contract that, and not
// the added fitness term's product, with the addition that follows in row_step, and change its rounding
__device__ __forceinline__ float flip_sign(float x, uint32_t sign) { return __uint_as_float(__float_as_uint(x) ^ sign); }

// the stop rule's answer for the update launch of a merged iteration: uniform over the launch
// (legal_min of this iteration is complete, and the entry cleared here is the next one's)
__device__ __forceinline__ bool merged_stop(const GraphDev& d, const GraphState* st, long long t) {
    return d.stop_on_legal && st->legal_min[t & 1] != 0x7FFFFFFF;
}

// End of a merged iteration, by one wave-sized group of lanes (lane of `lanes`) of the launch that
// updates the weights: the route counters, then either the stop (lowest legal member, its colouring)
// or t <- t + 1.  The launch's other blocks read st->tc, not t.
__device__ __forceinline__ void merged_end(const GraphDev& d, GraphState* st, long long t, bool stop, int lane, int lanes) {
    int ld = stop && d.cmax == 1 ? st->legal_min[t & 1] : -1;
    if (stop && d.cmax > 1) {
        // multicolouring: the lowest member without conflicts, and its selection as [i][s]
        while (d.f2[++ld] != 0) {}
        for (int e = lane; e < d.n * d.cmax; e += lanes) {
            const int i = e / d.cmax, sl = e - i * d.cmax;
            d.snap[e] = d.sel[((size_t)ld * d.cmax + sl) * d.cs + i];
        }
    } else if (stop) {
        const int16_t* c = d.c[st->pS] + (size_t)ld * d.cs;
        for (int i = lane; i < d.n; i += lanes) d.snap[i] = c[i];
    }
    if (lane != 0) return;
    const float tf = (float)t;
    if (d.lambda * tf != 0.0f || d.mu * tf != 0.0f) st->it_dense += 1;
    else st->it_nopen += 1;
    if (stop) {
        st->legal_d = ld;
        st->stopped = 1;
        return;
    }
    st->legal_min[(t + 1) & 1] = 0x7FFFFFFF;
    st->t = t + 1;
    st->steps_done += 1;
}

// Step 4 with the row held in registers, one (member, vertex) row per 16-lane
// group, k <= 16 KPL: softmax along k (max subtracted), straight-through
// gradient gW = s^ (G - sum_l s^_l G_l), update, smoothing, and in mode 0 the
// argmax colouring of the updated row for the next iteration (written over
// this iteration's colours).  Mode 1 writes gS and gW instead.
// VAR bit 0: some graph of the launch has an added fitness term (equity or colour
// cost), bit 1: some graph takes heavy-ball steps, bit 2: some graph is a multicolouring whose next
// colours are selected from the row; the plain variant carries none of their registers.
struct RowCtx {
    float nut, eta, rho, gam;
    int problem, c1, c2, k;
    bool smooth;
};

__device__ __forceinline__ RowCtx row_ctx(const GraphDev& d, long long t) {
    RowCtx x;
    x.nut = prob_added(d.problem) ? d.nu * (float)t : 0.0f;
    x.eta = d.eta;
    x.rho = d.rho;
    x.gam = d.momentum;
    x.problem = d.problem;
    x.c1 = d.c1;
    x.c2 = d.c2;
    x.k = d.k;
    x.smooth = d.nb_iter > 0 && ((t + 1) % d.nb_iter) == 0;
    return x;
}

// loads of a row's weights and, where present, velocity (indices clamped into the row inside the last
// group of 16 instead of per-lane branches, so they are all in flight together).  Groups of 16 past the row's end are
// skipped whole: KPL is sized for the largest k of the launch, and a row of a graph with fewer
// colours would otherwise issue every group's loads.
template <int KPL, int VAR>
struct RowRegs {
    float wv[KPL], vv[(VAR & 2) ? KPL : 1];
};

// the class sizes of a row's member at the lane's colours (the same for all rows of a member; read only with an
// added fitness term)
template <int KPL, int VAR>
struct RowClasses {
    int32_t cv[(VAR & 1) ? KPL : 1];
};

template <int KPL, int VAR>
__device__ __forceinline__ void classes_load(RowClasses<KPL, VAR>& C, const RowCtx& x, const int32_t* V, int l16) {
    if constexpr ((VAR & 1) != 0) {
        if (x.nut != 0.0f) {
#pragma unroll
            for (int q = 0; q < KPL; ++q)
                if (16 * q < x.k) C.cv[q] = gview(V)[min(l16 + 16 * q, x.k - 1)];
        }
    }
}

// gs: the row of G, unless null, into gv.
template <int KPL, int VAR>
__device__ __forceinline__ void row_load(RowRegs<KPL, VAR>& R, float (&gv)[KPL], const RowCtx& x, const float* w,
                                         const float* gs, const float* vel, int mode, int l16) {
    const int k = x.k;
#pragma unroll
    for (int q = 0; q < KPL; ++q)
        if (16 * q < k) {
            const int l = min(l16 + 16 * q, k - 1);
            R.wv[q] = gview(w)[l];
            if (gs) gv[q] = gview(gs)[l];
        }
    if constexpr ((VAR & 2) != 0) {
        if (vel && mode != 1) {
#pragma unroll
            for (int q = 0; q < KPL; ++q)
                if (16 * q < k) R.vv[q] = gview(vel)[min(l16 + 16 * q, k - 1)];
        }
    }
}

// the row's arithmetic; gv: the lane's entries of gS without the added-fitness term.  w, vel: the row's
// memory (written in mode 0); gS_out, gW_out: the row's outputs (mode 1).  Returns the row's next colour
// (mode 0), or -1 where the updated row is not finite; with VAR bit 2 the updated weights stay in R.wv.
template <int KPL, int VAR>
__device__ __forceinline__ int row_step(RowRegs<KPL, VAR>& R, const RowClasses<KPL, VAR>& C, float (&gv)[KPL],
                                        const RowCtx& x, float* __restrict__ w,
                                        float* __restrict__ vel, int mode, float* __restrict__ gS_out,
                                        float* __restrict__ gW_out, int l16) {
    constexpr bool ADD = (VAR & 1) != 0, MOM = (VAR & 2) != 0;
    const int k = x.k;
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        const int l = l16 + 16 * q;
        if (l < k) {
            if constexpr (ADD) {
                // one rounding, by name: contracted or not, the rows of a block must not differ
                if (x.nut != 0.0f) gv[q] = __builtin_fmaf(x.nut, added_grad(x.problem, C.cv[q], l, x.c1, x.c2), gv[q]);
            }
        } else {
            R.wv[q] = -INFINITY;
            gv[q] = 0.0f;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < KPL; ++q) mx = fmaxf(mx, R.wv[q]);
    mx = row16_max(mx);
    float ev[KPL];
    float z = 0.0f, qs = 0.0f;
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        ev[q] = (l16 + 16 * q < k) ? exp_soft(R.wv[q] - mx) : 0.0f;
        z += ev[q];
        qs += ev[q] * gv[q];
    }
    z = row16_sum(z);
    qs = row16_sum(qs);
    const float rz = 1.0f / z;
    const float rq = qs * rz;
    if (mode == 1) {
#pragma unroll
        for (int q = 0; q < KPL; ++q) {
            const int l = l16 + 16 * q;
            if (l < k) {
                if (gS_out) gS_out[l] = gv[q];
                if (gW_out) gW_out[l] = ev[q] * rz * (gv[q] - rq);
            }
        }
        return 0;
    }
    float best = -INFINITY;
    int bi = 0x7FFFFFFF, bad = 0;
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        const int l = l16 + 16 * q;
        if (l < k) {
            float step = ev[q] * rz * (gv[q] - rq);
            if constexpr (MOM) {
                if (vel) {
                    step = x.gam * R.vv[q] + step;  // heavy-ball velocity
                    vel[l] = step;
                }
            }
            float nw = R.wv[q] - x.eta * step;
            if (x.smooth) nw = nw / x.rho;
            w[l] = nw;
            if constexpr ((VAR & 4) != 0) R.wv[q] = nw;
            if (!finite_f(nw)) bad = 1;
            if (nw > best) { best = nw; bi = l; }
        }
    }
    // the argmax over the row: the largest value, then the lowest colour holding it
    const int bo = f32_ord(best);
    const int bmax = row16_max_i(bo);
    bi = row16_min_i(bo == bmax ? bi : 0x7FFFFFFF);
    bad = row16_max_i(bad);
    return bad || bi >= k ? -1 : bi;
}

// Multicolouring: the row's demand of colours from its updated weights (-INFINITY past k) in registers, as the colour
// kernel's selection: one after the other the largest weight not yet taken, the lowest colour on ties (adding zero
// makes -0 and 0 tie as they compare).  Slots past the demand take -1; slot 0 is also the vertex's colour.
template <int KPL>
__device__ __forceinline__ void row_select(const GraphDev& d, const float (&wv)[KPL], int m, int i, int l16, int16_t* c) {
    const int k = d.k, CM = d.cmax, ci = d.dem[i];
    unsigned long long taken = 0;
    for (int sl = 0; sl < CM; ++sl) {
        float best = -INFINITY;
        int bi = 0x7FFFFFFF;
#pragma unroll
        for (int q = 0; q < KPL; ++q)
            if (l16 + 16 * q < k && !((taken >> q) & 1ull) && wv[q] > best) {
                best = wv[q];
                bi = l16 + 16 * q;
            }
        const int bo = f32_ord(best + 0.0f);
        const int bmax = row16_max_i(bo);
        bi = row16_min_i(bo == bmax ? bi : 0x7FFFFFFF);
        const int pick = (sl < ci && bi < k) ? bi : -1;
        if (pick >= 0 && (pick & 15) == l16) taken |= 1ull << (pick >> 4);
        if (l16 == 0) {
            d.sel[((size_t)m * CM + sl) * d.cs + i] = (int16_t)pick;
            if (sl == 0) c[i] = (int16_t)pick;
        }
    }
}

}  // namespace tcol
