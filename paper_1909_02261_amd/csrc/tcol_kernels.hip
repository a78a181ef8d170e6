// gfx950 kernels of the TensCol population step other than the MFMA contraction:
// graph validation and packing, argmax colouring, class sizes, one-hot S^T
// expansion, group concentration with the penalty operand, fitness and stop
// rule, softmax straight-through update, loss reduction, state updates.
//
// Every kernel takes the descriptor array of all graphs of a context and a
// flattened work index, so one launch serves a batch of graphs of uneven sizes.
#include "tcol_internal.h"
#include "tcol_launch.h"
#include "tcol_rows.h"

#include <math.h>

namespace tcol {

// ---------------------------------------------------------------- helpers ----

__device__ inline uint16_t f32_to_bf16_rne(float x) {
    // round to nearest even on the upper 16 bits (inputs here are finite)
    uint32_t u = __float_as_uint(x);
    uint32_t lsb = (u >> 16) & 1u;
    u += 0x7FFFu + lsb;
    return (uint16_t)(u >> 16);
}


__device__ inline int graph_of_row(const GraphDev* gd, int G, int w) {
    return find_graph(gd, G, w, [](const GraphDev& x) { return x.row_begin; });
}

// ---------------------------------------------------- shared device helpers --

__device__ inline bool pen_active(const GraphDev& d, const GraphState* st) {
    const float tf = (float)st->t;
    return (d.lambda * tf != 0.0f) || (d.mu * tf != 0.0f);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// equal 16-bit halves of a and b among those whose top bit is set in `valid`
// (0x8000 for the low half, 0x80000000 for the high half): a half of a ^ b is zero
// exactly when subtracting one inside that half sets its top bit while the half
// itself does not have it set (colours are < 2^15)
__device__ inline int equal_halves_in(uint32_t a, uint32_t b, uint32_t valid) {
    const uint32_t x = a ^ b;
    u16x2 h = __builtin_bit_cast(u16x2, x);
    const u16x2 one = {1, 1};
    const uint32_t y = __builtin_bit_cast(uint32_t, (u16x2)(h - one));
    return __builtin_popcount(y & ~x & valid);
}

typedef unsigned int u32x4n __attribute__((ext_vector_type(4)));
// order this wave's LDS accesses across lanes (LDS executes a wave's operations in issue order)
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// 16-byte global load (p 16-byte aligned)
__device__ inline u32x4n gload16(const void* p) { return *(const __attribute__((address_space(1))) u32x4n*)p; }

// ------------------------------------------------------ validation, packing --

// Checks A (n x n, row-major 0/1, symmetric, zero diagonal; unless A8 is null) and writes the
// zero-padded byte copy A8, the bit copy Ab and the operand copy Aop (each unless null;
// Aop [n_pad][n_pad], in fp4 two entries per byte, the lower column in the low nibble, 1.0 = 0x2).
// One block per 64 x 64 tile: a wave reads 64 bytes of a row at a time (A's rows have any
// alignment) and turns them into one ballot, from which every copy is written; the mirrored tile's
// ballots go to LDS for the symmetry check.
__global__ __launch_bounds__(256) void k_pack_graph(const uint8_t* __restrict__ A, int n, int n_pad, int op,
                                                    uint8_t* __restrict__ A8, unsigned long long* __restrict__ Ab,
                                                    void* __restrict__ Aop, int* __restrict__ bad,
                                                    unsigned long long* __restrict__ ones) {
    __shared__ unsigned long long mir[64];
    __shared__ unsigned int wcount[4];
    const int T = n_pad / 64;
    const int ti = blockIdx.x / T, tj = blockIdx.x - ti * T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = ti * 64, j0 = tj * 64;
    const bool check = A8 != nullptr;
    uint8_t own[16], oth[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int r = wave * 16 + u;
        own[u] = i0 + r < n && j0 + lane < n ? A[(size_t)(i0 + r) * n + j0 + lane] : (uint8_t)0;
        oth[u] = check && j0 + r < n && i0 + lane < n ? A[(size_t)(j0 + r) * n + i0 + lane] : (uint8_t)0;
    }
    if (check) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const unsigned long long m = __ballot(oth[u] != 0);
            if (lane == 0) mir[wave * 16 + u] = m;
        }
    }
    __syncthreads();
    const unsigned long long mcol = check ? mir[lane] : 0ull;   // bit r: A[j0 + lane][i0 + r]
    unsigned int count = 0;   // ones of A seen by this wave (2 |E| over all waves of a valid graph)
    bool wrong = false;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int r = wave * 16 + u, i = i0 + r;
        const bool a = own[u] != 0;
        const unsigned long long m = __ballot(a);
        count += (unsigned)__popcll(m);
        if (check) wrong |= own[u] > 1 || a != (bool)((mcol >> r) & 1ull) || (a && i == j0 + lane);
        const size_t e = (size_t)i * n_pad + j0 + lane;
        if (A8) A8[e] = a ? 1 : 0;
        if (Ab && lane == 0) Ab[(size_t)tj * n_pad + i] = m;
        if (!Aop) continue;
        if (op == kPrecFP32) {
            ((float*)Aop)[e] = a ? 1.0f : 0.0f;
        } else if (lane < 32) {
            const unsigned int two = (unsigned int)(m >> (2 * lane)) & 3u;
            ((uint8_t*)Aop)[((size_t)i * n_pad + j0) / 2 + lane] = (uint8_t)(((two & 1u) << 1) | ((two & 2u) << 4));
        }
    }
    if (check && __any(wrong) && lane == 0) atomicOr(bad, 1);
    // one atomic per block
    if (lane == 0) wcount[wave] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long c = (unsigned long long)wcount[0] + wcount[1] + wcount[2] + wcount[3];
        if (c) atomicAdd(ones, c);
    }
}

// ------------------------------------------------------------ step 1 -----------

// Multicolouring, step 1 for row r = (member m, vertex i): the dem[i] colours of largest weight,
// one after the other (each the argmax of the colours not yet taken, lowest l on ties), into
// sel[m][s][i] for s < dem[i] and -1 for the other slots; slot 0 also into c[pS].  16 lanes per
// row; lane l16 keeps a bit per colour l16 + 16 q it holds that has been taken (k <= 1024).
__device__ inline void select_row(const GraphDev& d, GraphState* st, int r, const float* w, int l16) {
    const int k = d.k, n = d.n, CM = d.cmax;
    const int m = r / n, i = r - m * n;
    const int ci = d.dem[i];
    int bad = 0;
    for (int l = l16; l < k; l += 16)
        if (!finite_f(w[l])) bad = 1;
    for (int sh = 8; sh >= 1; sh >>= 1) bad |= __shfl_xor(bad, sh, 16);
    if (bad) {
        if (l16 == 0) {
            atomicExch(&st->error, -5);
            atomicExch(&st->stopped, 1);
            d.c[st->pS][(size_t)m * d.cs + i] = 0;
        }
        return;
    }
    unsigned long long taken = 0;
    for (int sl = 0; sl < CM; ++sl) {
        float best = -INFINITY;
        int bi = 0x7FFFFFFF;
        int q = 0;
        for (int l = l16; l < k; l += 16, ++q)
            if (!((taken >> q) & 1ull) && w[l] > best) {
                best = w[l];
                bi = l;
            }
        for (int sh = 8; sh >= 1; sh >>= 1) {
            const float ob = __shfl_xor(best, sh, 16);
            const int oi = __shfl_xor(bi, sh, 16);
            if (ob > best || (ob == best && oi < bi)) {
                best = ob;
                bi = oi;
            }
        }
        const int pick = (sl < ci && bi < k) ? bi : -1;
        if (pick >= 0 && (pick & 15) == l16) taken |= 1ull << (pick >> 4);
        if (l16 == 0) {
            d.sel[((size_t)m * CM + sl) * d.cs + i] = (int16_t)pick;
            if (sl == 0) d.c[st->pS][(size_t)m * d.cs + i] = (int16_t)pick;
        }
    }
}

// c_d(i) = argmax_l W[d,i,l], lowest l on ties; 16 lanes per row, or from 129 colours a wave per row (longer pieces of
// a row per load: k = 211, n = 2999, D = 25 21.5 -> 18 us; k = 280,
// n = 4000, D = 32 40 -> 28 us), four rows in flight per wave either way.
__global__ __launch_bounds__(256) void k_colors(const GraphDev* __restrict__ gd, int G, int total_rows,
                                                int honor_stop) {
    {
        // the wave's four rows, when they belong to one graph with long rows
        const int r0 = blockIdx.x * 16 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 4;
        if (r0 >= total_rows) return;
        const GraphDev& d = gd[graph_of_row(gd, G, r0)];
        const int k = d.k, lane = threadIdx.x & 63;
        if (d.cmax == 1 && k > 128 && r0 + 3 < d.row_begin + d.D * d.n) {
            GraphState* st = d.st;
            if (honor_stop && st->stopped) return;
            const float* __restrict__ w = d.W[st->pW] + (size_t)(r0 - d.row_begin) * k;
            int16_t* __restrict__ c = d.c[st->pS];
            float best[4];
            int bi[4];
            bool bad = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                best[q] = -INFINITY;
                bi[q] = 0x7FFFFFFF;
            }
            constexpr int U = 4;
            for (int l0 = 0; l0 < k; l0 += 64 * U) {
                float x[4][U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (l0 + 64 * u < k) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) x[q][u] = gview(w)[(size_t)q * k + min(l0 + 64 * u + lane, k - 1)];
                    }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (l0 + 64 * u < k) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (!finite_f(x[q][u])) bad = true;
                            if (x[q][u] > best[q]) { best[q] = x[q][u]; bi[q] = min(l0 + 64 * u + lane, k - 1); }
                        }
                    }
            }
            if (__any(bad) && lane == 0) {
                atomicExch(&st->error, -5);
                atomicExch(&st->stopped, 1);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int bo = f32_ord(best[q] + 0.0f);
                const int arg = wave_min_i(bo == wave_max_i(bo) ? bi[q] : 0x7FFFFFFF);
                const int r = r0 + q - d.row_begin, m = r / d.n;
                // (a row of NaN has no maximum; the graph is stopped then)
                if (lane == 0) c[(size_t)m * d.cs + (r - m * d.n)] = (int16_t)(arg < k ? arg : 0);
            }
            return;
        }
    }
    const int l16 = threadIdx.x & 15;
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
    if (row >= total_rows) return;
    const GraphDev& d = gd[graph_of_row(gd, G, row)];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    const int r = row - d.row_begin;
    const float* w = d.W[st->pW] + (size_t)r * d.k;
    if (d.cmax > 1) {
        select_row(d, st, r, w, l16);
        return;
    }
    // eight loads in flight per lane (indices clamped into the row: a repeated last value changes neither the
    // maximum nor, by the strict comparison, its colour)
    constexpr int U = 8;
    const int k = d.k;
    float best = -INFINITY;
    int bi = 0x7FFFFFFF;
    int bad = 0;
    for (int l = l16; l < k; l += 16 * U) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (l - l16 + 16 * u < k) x[u] = gview(w)[min(l + 16 * u, k - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (l - l16 + 16 * u < k) {
                if (!finite_f(x[u])) bad = 1;
                if (x[u] > best) { best = x[u]; bi = min(l + 16 * u, k - 1); }
            }
    }
    // the largest value of the 16 lanes, then the lowest colour holding it
    // (adding zero makes -0 and 0 tie across lanes as they compare)
    const int bo = f32_ord(best + 0.0f);
    const int bmax = row16_max_i(bo);
    bi = row16_min_i(bo == bmax ? bi : 0x7FFFFFFF);
    bad = row16_max_i(bad);
    if (l16 == 0) {
        if (bad || bi >= d.k) {
            bi = 0;
            atomicExch(&st->error, -5);
            atomicExch(&st->stopped, 1);
        }
        const int m = r / d.n, i = r - m * d.n;
        d.c[st->pS][(size_t)m * d.cs + i] = (int16_t)bi;
    }
}

// Per-iteration penalty choice of graphs on the sparse rows (ps_mode 2): row i has at
// most sum_d |class of c_d(i)| nonzeros in P, and over all rows that is
// w = sum_d sum_l #V_{d,l}^2.  While its average over the rows stays within n the
// iteration takes the sparse rows; beyond (the population collapsing into a few large
// classes) the dense pass, whose cost does not depend on the classes.  Partitioning
// keeps the sparse rows: its operand over D - Mt has nonzeros wherever Mt < D, so its
// rows are dense anyway and the sparse kernel is the faster on them.  Returns pdense.
__device__ inline int penalty_choice(const GraphDev& d, long long w) {
    // n: on k-colouring of G(4000, .5) with k = 280, D = 32 (fp4) the step took 0.326 ms against
    // 0.334 (0.4 n), 0.324 (1.5 n), 0.330 (2 n), 0.340 (3 n)
    return d.ps_mode == 2 && !prob_partition(d.problem) && w > (long long)d.n * d.n ? 1 : 0;
}

// Class sizes #V_{d,l} of member d, its added fitness (equity or colour cost) and
// the vertex-major copy of its colours.
// For a graph on the sparse penalty also the member's vertices grouped by colour
// (counting sort) and, for each vertex, the start and size of its class; with `decide`
// the last of the graph's member blocks then takes the iteration's penalty choice
// (penalty_choice).  One block per member.
// Dynamic LDS: k counts, and with the class lists 4 k per-wave cursors, k class starts
// and n entries.
// block b of the S^T expansion (the expansion kernel's body; the fast path runs it in
// extra blocks of the class-size launch, since both read only the colours)
// (adv: the launch also ends the previous iteration, so a pending non-finite update counts as
// a stop)
__device__ __forceinline__ void expand_block(const GraphDev* __restrict__ gd, int G, int b, int honor_stop, int next, int gate,
                             int adv);

// end of an iteration for a running graph: t <- t + 1, and a non-finite weight from the
// update stops the graph with an error
__device__ inline void advance_graph(GraphState* st) {
    if (st->stopped) return;
    st->t += 1;
    st->steps_done += 1;
    if (st->next_bad) {
        st->error = -5;
        st->stopped = 1;
    }
}

constexpr int kPrepScratch = 288;   // words of the class-size block's LDS scratch

// the class-size kernel's block for member `mem` (flattened over the graphs)
constexpr int kPrepBatch = 8;   // colours loaded per lane before the class-size atomics use them

__device__ __forceinline__ void prep_member(const GraphDev* __restrict__ gd, int G, int mem, int honor_stop, int next, int decide,
                            int advance_prev) {
    // dynamic LDS (prep_lds): a scratch of kPrepScratch words (the scan's run sums, two
    // four-wave reductions, the ticket result), then the counts and class lists
    extern __shared__ int prep_dyn[];
    int* part = prep_dyn;                                     // [257]
    long long* fsum = (long long*)(prep_dyn + 260);           // [4]
    long long* qsum = fsum + 4;                               // [4]
    int* last_block_p = prep_dyn + 276;
    int* prep_sh = prep_dyn + kPrepScratch;
    const GraphDev& d = gd[find_graph(gd, G, mem, [](const GraphDev& x) { return x.mem_begin; })];
    GraphState* st = d.st;
    // Whether the graph is stopped for this iteration, read before anything in this launch
    // writes the state: advance_graph below can only turn `stopped` on, and exactly when
    // next_bad is set, so every thread of every member block (and of the expansion blocks)
    // takes the same decision whether it reads `stopped` before or after that write.  A
    // graph's member blocks therefore all run or all return, and the ticket of the penalty
    // choice below counts all of them.
    const bool stop_now = honor_stop && (st->stopped || (advance_prev && st->next_bad));
    // the previous iteration's end (its own launch otherwise), by the graph's first member
    // block: nothing in this launch reads t
    if (advance_prev && mem == d.mem_begin && threadIdx.x == 0) advance_graph(st);
    if (stop_now) return;
    const int p = next ? st->pS ^ 1 : st->pS;
    const int m = mem - d.mem_begin;
    const int k = d.k, n = d.n, tid = threadIdx.x;
    const int16_t* __restrict__ c = d.c[p] + (size_t)m * d.cs;
    int16_t* __restrict__ cT = d.cT;
    const size_t cTs = d.cTs;
    int* cnt = prep_sh;
    const bool lists = d.psparse != 0;              // uniform over the block
    // with the class lists each wave counts its own quarter of the vertices
    constexpr int NW = 4;
    const int wv = tid >> 6, lane = tid & 63;
    const int Q = ((n + NW - 1) / NW + 63) & ~63;
    int* cw = prep_sh + k;                          // [NW][k]
    for (int l = tid; l < k; l += 256) cnt[l] = 0;
    if (lists)
        for (int l = tid; l < NW * k; l += 256) cw[l] = 0;
    __syncthreads();
    // the vertex loops load kPrepBatch colours per lane before using any of them (one round
    // of load latency per batch instead of one per vertex)
    if (lists) {
        const int e = min(n, (wv + 1) * Q);
        for (int i0 = wv * Q + lane; i0 < e; i0 += 64 * kPrepBatch) {
            int16_t xs[kPrepBatch];
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) xs[u] = i0 + 64 * u < e ? gview(c)[i0 + 64 * u] : (int16_t)0;
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) {
                const int i = i0 + 64 * u;
                if (i < e) {
                    atomicAdd(&cnt[xs[u]], 1);
                    atomicAdd(&cw[wv * k + xs[u]], 1);
                    cT[(size_t)i * cTs + m] = xs[u];
                }
            }
        }
    } else if (d.cmax > 1) {
        // multicolouring: every selected colour of the vertex counts in its class
        for (int i = tid; i < n; i += 256) {
            for (int sl = 0; sl < d.cmax; ++sl) {
                const int16_t x = d.sel[((size_t)m * d.cmax + sl) * d.cs + i];
                if (x >= 0) atomicAdd(&cnt[x], 1);
            }
            cT[(size_t)i * cTs + m] = gview(c)[i];
        }
    } else {
        for (int i0 = tid; i0 < n; i0 += 256 * kPrepBatch) {
            int16_t xs[kPrepBatch];
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) xs[u] = i0 + 256 * u < n ? gview(c)[i0 + 256 * u] : (int16_t)0;
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) {
                const int i = i0 + 256 * u;
                if (i < n) {
                    atomicAdd(&cnt[xs[u]], 1);
                    cT[(size_t)i * cTs + m] = xs[u];
                }
            }
        }
    }
    __syncthreads();
    int32_t* V = d.V[p] + (size_t)m * k;
    for (int l = tid; l < k; l += 256) V[l] = cnt[l];
    // added fitness of the member from the counts: f_eq = sum_l min(|#V - c1|, |#V - c2|),
    // or the colour cost sum_l (l + 1) #V_l (the fitness kernel of this iteration reads it)
    if (prob_added(d.problem)) {
        const int c1 = d.c1, c2 = d.c2;
        long long fe = 0;
        for (int l = tid; l < k; l += 256) {
            const long long v = cnt[l];
            if (d.problem == kProbMSCP) {
                fe += (long long)(l + 1) * v;
            } else {
                const long long x = v > c1 ? v - c1 : c1 - v;
                const long long y = v > c2 ? v - c2 : c2 - v;
                fe += x < y ? x : y;
            }
        }
        for (int sh = 32; sh >= 1; sh >>= 1) fe += __shfl_xor(fe, sh);
        if ((tid & 63) == 0) fsum[tid >> 6] = fe;
        __syncthreads();
        if (tid == 0) d.feq[m] = fsum[0] + fsum[1] + fsum[2] + fsum[3];
    }
    if (!lists) return;
    {
        // sum_l #V_l^2: the class-mate increments of all rows for this member
        long long q2 = 0;
        for (int l = tid; l < k; l += 256) q2 += (long long)cnt[l] * cnt[l];
        for (int sh = 32; sh >= 1; sh >>= 1) q2 += __shfl_xor(q2, sh);
        if ((tid & 63) == 0) qsum[tid >> 6] = q2;
        __syncthreads();
        if (tid == 0) d.sq[m] = qsum[0] + qsum[1] + qsum[2] + qsum[3];
        if (decide) {
            // the last member block to get here sums every member's value (a ticket
            // counter after a release fence; the last block reads the others' values
            // with atomic loads after an acquire fence) and resets the counter
            int& last_block = *last_block_p;
            if (tid == 0) {
                __threadfence();
                last_block = atomicAdd(&st->prep_ticket, 1) == d.D - 1;
            }
            __syncthreads();
            if (last_block && tid < 64) {
                __threadfence();
                long long w = 0;
                for (int mm = tid; mm < d.D; mm += 64) w += __atomic_load_n(d.sq + mm, __ATOMIC_RELAXED);
                for (int sh = 32; sh >= 1; sh >>= 1) w += __shfl_xor(w, sh);
                if (tid == 0) {
                    st->pdense = penalty_choice(d, w);
                    st->prep_ticket = 0;
                }
            }
        }
    }
    int* offl = cw + NW * k;                        // [k] class starts
    int16_t* lst = (int16_t*)(offl + k);            // [n]
    int32_t* __restrict__ off = d.cls_off + (size_t)m * (k + 1);
    int16_t* __restrict__ cv = d.cls_v + (size_t)m * d.cs;
    // exclusive scan of the counts: runs of `per` classes per thread, the 256 run sums
    // scanned by wave 0 (four per lane, then across lanes)
    const int per = (k + 255) / 256;
    const int lb = min(k, tid * per), le = min(k, lb + per);
    int run = 0;
    for (int l = lb; l < le; ++l) run += cnt[l];
    part[tid] = run;
    __syncthreads();
    if (tid < 64) {
        const int v0 = part[4 * tid], v1 = part[4 * tid + 1], v2 = part[4 * tid + 2], v3 = part[4 * tid + 3];
        const int sum = v0 + v1 + v2 + v3;
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if (tid >= o) incl += y;
        }
        const int ex = incl - sum;
        part[4 * tid] = ex;
        part[4 * tid + 1] = ex + v0;
        part[4 * tid + 2] = ex + v0 + v1;
        part[4 * tid + 3] = ex + v0 + v1 + v2;
    }
    __syncthreads();
    // class l starts at its offset; within it the quarters follow in order, so each
    // wave's cursor for l starts after the earlier quarters' vertices of colour l
    int acc = part[tid];
    for (int l = lb; l < le; ++l) {
        off[l] = acc;
        offl[l] = acc;
        int q = acc;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int x = cw[w * k + l];
            cw[w * k + l] = q;
            q += x;
        }
        acc += cnt[l];
    }
    if (tid == 0) off[k] = n;
    __syncthreads();
    // placement: each vertex takes the next slot of its colour in its wave's range (the
    // order inside a class is not used: the penalty counts do not depend on it), and
    // records its class's start and size for this member
    {
        int* cur = cw + wv * k;
        int2* __restrict__ cinfo = d.cinfo;
        const int qb = wv * Q, qe = min(n, (wv + 1) * Q);
        for (int i0 = qb + lane; i0 < qe; i0 += 64 * kPrepBatch) {
            int xs[kPrepBatch];
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) xs[u] = i0 + 64 * u < qe ? (int)gview(c)[i0 + 64 * u] : 0;
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) {
                const int i = i0 + 64 * u;
                if (i < qe) {
                    const int x = xs[u];
                    const int pos = atomicAdd(&cur[x], 1);
                    lst[pos] = (int16_t)i;
                    cinfo[(size_t)m * d.cs + i] = make_int2(offl[x], cnt[x]);
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < n; i += 256) cv[i] = lst[i];
}

__global__ __launch_bounds__(256) void k_prep(const GraphDev* __restrict__ gd, int G, int total_mem, int honor_stop,
                                              int next, int decide, int ex_blocks, int advance_prev) {
    const int mem = blockIdx.x;
    if (mem >= total_mem) {
        // blocks past the members: the expansion of the current colours (gate 1), with the
        // same stop decision as the member blocks
        if (mem - total_mem < ex_blocks) expand_block(gd, G, mem - total_mem, honor_stop, next, 1, advance_prev);
        return;
    }
    prep_member(gd, G, mem, honor_stop, next, decide, advance_prev);
}

// -------------------------------------------------------- sparse penalty rows ----

// Penalty rows from the nonzeros of P.  The penalty operand
//   P_ij = t * (a_ij ? 2 alpha lambda x^(alpha-1) : -[i != j or bonus_diag] 2 beta mu x^(beta-1)),
// x = Mt_ij (D - Mt_ij for partitioning), enters the gradient as (P.S_d)[i, l], and
// with one-hot S_d that is the sum of P_ij over the vertices j of colour l in member
// d.  For colouring P_ij vanishes unless j shares row i's colour in some member
// (alpha, beta > 1 give 0^(alpha-1) = 0): a few hundred of the n entries of a row
// in a typical iteration.  One block of NT threads per row i:
//   1. Mt_ij from the class lists: j shares i's colour in member d exactly when j is
//      in the class of c_d(i), so each member adds one to the count of every vertex
//      of that class; the sum_d |class| increments are spread over the whole block.
//      When the classes are large (more than n D / 8 increments: the population
//      briefly collapses into a few giant classes after each smoothing) every j
//      compares its vertex-major colours with row i's instead (n D comparisons);
//   2. the counts become table indices of P_ij, and the nonzero entries go to a list
//      (j, index);
//   3. members are taken PM at a time: every listed j adds P_ij to the accumulator
//      of (d, c_d(j)) for each member d of the group (c_d(j) from the vertex-major
//      colours; consecutive lanes take consecutive members, so the atomics of one
//      instruction hit different accumulators even when a class holds most of the
//      vertices), then the group's sums go to G[d][i][l], added to the contraction's
//      A.S_d (accumulate 1) or written for the contraction's epilogue (accumulate 0).
// A graph choosing per iteration (ps_mode 2) takes these rows only in the iterations
// where the class-size kernel found its classes small; otherwise the contraction's dense pass.
// Steps 1 and 3 issue the loads of their next batch before the atomics of the current
// one.  The sums are taken in 64-bit fixed point: every table value times 2^sc, with sc
// chosen so that n max|P| stays below 2^62, is an integer whenever the table's binary
// exponents span at most 38 - bits(n) (every setting of the paper's parameter grid up
// to n = 4000; beyond, each term is rounded at 2^-sc, at most 2^-30 of max|P| over a
// row), and integer sums do not depend on the order of the additions, so the LDS
// atomics give the same bits on every run.  The result is the sum of the FP32 values
// P_ij, exact in those cases, rounded once to FP32.
// Dynamic LDS (penalty_sparse_lds): table [2 (D + 1) + 1] i64 (the last entry 0, for
// an excluded diagonal), class starts and the prefix of the class sizes [D + 1] i32
// each, the list length, row i's colours [cTs] i16, list [n_pad] u32, then counts
// [n_pad] u32 overlaid by the group's accumulators [PM][k] i64.
// the fitness of one graph (the fitness kernel's body; the fast path runs it in extra
// blocks of the sparse penalty launch, since both follow the contraction)
__device__ __forceinline__ void fitness_graph(const GraphDev* __restrict__ gd, int g, int honor_stop, int flags, int* best);

__host__ __device__ inline size_t ps_tab_words(int D) { return ((size_t)2 * (D + 1) + 1 + 1) & ~(size_t)1; }
__host__ __device__ inline size_t ps_int_words(int D) { return ((size_t)D + 1 + 3) & ~(size_t)3; }
constexpr int kPsBatch = 4;     // entries per thread per batch in steps 1 and 3 (48 registers: eight waves per SIMD)
constexpr int kPsA8 = 2;        // adjacency words per thread loaded at the start

// ---- the row update on the sparse-rows launch (fast path, graphs with pfuse) ----
//
// One wave per (member d, vertex i) row, lane j holding colours j, j + 64, ... (KW of them):
// the added-fitness term, softmax along k (max subtracted), the straight-through gradient
// gW = s^ (gS - sum_l s^_l gS_l), W' = W - eta gW (divided by rho in the smoothing
// iterations) written to the other weight buffer, and the argmax of W' (lowest colour on
// ties) to the other colour buffer.  The arithmetic of the row-update kernel, with the row's
// sums taken over 64 lanes.  The fitness launch that follows accepts the update by flipping
// the buffers, unless the graph stops in this iteration (the stop rule comes before the update).
struct FuseCtx {
    const float* Wc;          // current weights
    float* Wn;                // the other buffer, written
    int16_t* cn;              // the other colour buffer, written
    const int32_t* V;         // class sizes of this iteration (added fitness term)
    float nut, eta, rho;
    bool smooth;
};

__device__ inline FuseCtx fuse_ctx(const GraphDev& d, GraphState* st) {
    FuseCtx f;
    const int pW = st->pW, pS = st->pS;
    const long long t = st->t;
    f.Wc = d.W[pW];
    f.Wn = d.W[pW ^ 1];
    f.cn = d.c[pS ^ 1];
    f.V = d.V[pS];
    f.nut = prob_added(d.problem) ? d.nu * (float)t : 0.0f;
    f.eta = d.eta;
    f.rho = d.rho;
    f.smooth = d.nb_iter > 0 && ((t + 1) % d.nb_iter) == 0;
    return f;
}

// loads of row (dd, i): weights and the raw G entries (fp32 bits, or the uint16 A.S count) of
// the lane's colours below k; one base address per row, so the loads take immediate offsets
template <int KW>
__device__ inline void fuse_row_load(const GraphDev& d, const FuseCtx& f, int dd, int i, int lane, bool g16,
                                     float (&wv)[KW], uint32_t (&gr)[KW]) {
    const int k = d.k;
    const size_t row = ((size_t)dd * d.n + i) * k + lane;
    const auto* __restrict__ w = gview(f.Wc) + row;
    const auto* __restrict__ g32 = gview((const float*)d.G) + row;
    const auto* __restrict__ g16p = gview((const uint16_t*)d.G) + row;
#pragma unroll
    for (int q = 0; q < KW; ++q) {
        wv[q] = 0.0f;
        gr[q] = 0u;
        if (lane + 64 * q < k) {
            wv[q] = w[64 * q];
            gr[q] = g16 ? (uint32_t)g16p[64 * q] : __float_as_uint(g32[64 * q]);
        }
    }
}

// gv: the lane's entries of gS without the added-fitness term (entries past k are ignored)
template <int KW, int ADD>
__device__ inline void fuse_row_update(const GraphDev& d, GraphState* st, const FuseCtx& f, int dd, int i, int lane,
                                       const float (&wv)[KW], float (&gv)[KW]) {
    const int k = d.k;
    if (ADD && f.nut != 0.0f) {
        const auto* __restrict__ V = gview(f.V) + (size_t)dd * k + lane;
#pragma unroll
        for (int q = 0; q < KW; ++q)
            if (lane + 64 * q < k) gv[q] += f.nut * added_grad(d.problem, V[64 * q], lane + 64 * q, d.c1, d.c2);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < KW; ++q)
        if (lane + 64 * q < k) mx = fmaxf(mx, wv[q]);
    mx = wave_max(mx);
    float e[KW];
    float z = 0.0f, qs = 0.0f;
#pragma unroll
    for (int q = 0; q < KW; ++q) {
        e[q] = (lane + 64 * q < k) ? exp_soft(wv[q] - mx) : 0.0f;
        z += e[q];
        qs += e[q] * gv[q];
    }
    z = wave_sum(z);
    qs = wave_sum(qs);
    const float rz = 1.0f / z;
    const float rq = qs * rz;
    float* __restrict__ wo = f.Wn + ((size_t)dd * d.n + i) * k + lane;
    float best = -INFINITY;
    int bi = 0x7FFFFFFF;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < KW; ++q) {
        const int l = lane + 64 * q;
        if (l < k) {
            const float step = e[q] * rz * (gv[q] - rq);
            float nw = wv[q] - f.eta * step;
            if (f.smooth) nw = nw / f.rho;
            wo[64 * q] = nw;
            if (!finite_f(nw)) bad = true;
            if (nw > best) { best = nw; bi = l; }
        }
    }
    // the argmax: the largest value, then the lowest colour holding it
    const int bo = f32_ord(best);
    const int bmax = wave_max_i(bo);
    const int arg = wave_min_i(bo == bmax ? bi : 0x7FFFFFFF);
    const bool any_bad = __any(bad);
    if (lane == 0) {
        int c = arg;
        if (any_bad || c >= k) {
            c = 0;
            atomicExch(&st->next_bad, 1);
        }
        f.cn[(size_t)dd * d.cs + i] = (int16_t)c;
    }
}

// the row update alone for every member of vertex i (iterations of a pfuse graph whose penalty
// took the dense pass, or without a penalty): G holds the whole fp32 gradient; each wave takes
// members wave, wave + NT/64, ... (the launch's blocks per CU keep enough rows in flight)
template <int NT, int KW, int ADD>
__device__ __forceinline__ void fuse_update_only(const GraphDev& d, GraphState* st, int i) {
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const FuseCtx f = fuse_ctx(d, st);
    for (int dd = wave; dd < d.D; dd += NW) {
        float wv[KW], gv[KW];
        uint32_t gr[KW];
        fuse_row_load<KW>(d, f, dd, i, lane, false, wv, gr);
#pragma unroll
        for (int q = 0; q < KW; ++q) gv[q] = __uint_as_float(gr[q]);
        fuse_row_update<KW, ADD>(d, st, f, dd, i, lane, wv, gv);
    }
}

// The fused variants with at most five values per lane are held to 64 registers (eight waves per
// SIMD): with their 35 KB of LDS at n = 4000, k = 280, D = 32 that runs four 512-thread blocks per
// CU instead of three (the step 0.321 -> 0.310 ms there; two registers spill in the variant with
// an added fitness term).
template <int NT, int KW, int ADD>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 512 && KW > 0 && KW <= 5 ? 8 : 1))) void
k_pen_sparse(const GraphDev* __restrict__ gd, int G, int total_blocks, int honor_stop, int PM, int accumulate) {
    extern __shared__ __attribute__((aligned(16))) uint8_t ps_sh[];
    constexpr int B = KW > 0 ? 2 : kPsBatch;
    const int b = blockIdx.x;
    if (b >= total_blocks) return;
    const GraphDev& d = gd[find_graph(gd, G, b, [](const GraphDev& x) { return x.ps_begin; })];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    const bool sparse_now = d.psparse && !st->pdense && pen_active(d, st);
    // graphs whose row update rides on this launch (the fast path's sparse graphs)
    const bool fuse = KW > 0 && d.pfuse && accumulate;
    if constexpr (KW > 0) {
        if (fuse && !sparse_now) {
            fuse_update_only<NT, KW, ADD>(d, st, b - d.ps_begin);
            return;
        }
    }
    if (!sparse_now) return;
    const int n = d.n, k = d.k, D = d.D, cs = d.cs;
    const int n_pad = d.n_pad;
    const size_t cTs = d.cTs;
    const int i = b - d.ps_begin;
    const int tid = threadIdx.x, lane = tid & 63;
    const int T = 2 * (D + 1) + 1, zslot = T - 1;
    long long* tab = (long long*)ps_sh;                       // [ps_tab_words(D)]
    int* cbeg = (int*)(tab + ps_tab_words(D));                 // [ps_int_words(D)]
    int* pre = cbeg + ps_int_words(D);                         // [ps_int_words(D)]
    int* nzc = pre + ps_int_words(D);                          // [4]: list length, max-exponent
    int16_t* ci = (int16_t*)(nzc + 4);                         // [cTs]
    uint32_t* list = (uint32_t*)(ci + cTs);                    // [n_pad]
    uint32_t* cnt = list + n_pad;                              // [n_pad], steps 1-2
    unsigned long long* acc = (unsigned long long*)cnt;        // [PM][k], step 3
    const float tf = (float)st->t;
    const bool diag = d.bonus_diag != 0;
    const int16_t* __restrict__ cT = d.cT;
    // partitioning: the values are those of the dense operand, whose product the
    // contraction negates along with A.S
    const float sgn = prob_partition(d.problem) ? -1.0f : 1.0f;

    // 0. the adjacency bytes of step 2's first passes, the row's colours and classes,
    // the value table (one round of loads); counts cleared; the table's largest magnitude
    constexpr int TV = (2 * (kMaxD + 1) + 1 + NT - 1) / NT;   // table entries per thread
    float tv[TV];
#pragma unroll
    for (int u = 0; u < TV; ++u) {
        const int vi = tid + u * NT;
        tv[u] = 0.0f;
        if (vi < T - 1) tv[u] = vi <= D ? -(tf * gview(d.lut_bon)[vi]) : tf * gview(d.lut_pen)[vi - D - 1];
    }
    const uint8_t* __restrict__ arow = d.A8 + (size_t)i * n_pad;
    uint32_t a4pre[kPsA8];
#pragma unroll
    for (int u = 0; u < kPsA8; ++u) {
        const int j0 = 4 * (tid + u * NT);
        a4pre[u] = j0 < n ? gview((const uint32_t*)(arow + j0))[0] : 0u;
    }
    for (int dm = tid; dm < (int)cTs; dm += NT) {
        ci[dm] = gview(cT)[(size_t)i * cTs + dm];
        if (dm < D) {
            // (start, size) as one 8-byte load: start in the low word
            const unsigned long long cl = gview((const unsigned long long*)d.cinfo)[(size_t)dm * d.cs + i];
            cbeg[dm] = (int)(uint32_t)cl;
            pre[dm + 1] = (int)(uint32_t)(cl >> 32);
        }
    }
    for (int e = tid; e < n_pad / 4; e += NT) ((u32x4n*)cnt)[e] = u32x4n{0u, 0u, 0u, 0u};
    if (tid == 0) { nzc[0] = 0; nzc[1] = 0; pre[0] = 0; }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < TV; ++u) {
        if (tv[u] != 0.0f) {
            int ex;
            frexpf(tv[u], &ex);
            // exponents are compared as ex + 256 > 0 (the counter starts at 0 = none)
            atomicMax(&nzc[1], ex + 256);
        }
    }
    // prefix of the class sizes (wave 0, 64 members at a time)
    if (tid < 64) {
        int carry = 0;
        for (int base = 0; base < D; base += 64) {
            const int dm = base + lane;
            int x = dm < D ? pre[dm + 1] : 0;
#pragma unroll
            for (int sh = 1; sh < 64; sh <<= 1) {
                const int y = __shfl_up(x, sh);
                if (lane >= sh) x += y;
            }
            if (dm < D) pre[dm + 1] = carry + x;
            carry += __shfl(x, 63);
        }
    }
    __syncthreads();
    // fixed-point scale: |P_ij| < 2^E1 and n < 2^E2, so sums stay below 2^(E1 + E2) <= 2^62
    const int emax = nzc[1];
    const int sc = 62 - ((emax > 0 ? emax - 256 : 0) + (32 - __builtin_clz((unsigned)n)));
#pragma unroll
    for (int u = 0; u < TV; ++u) {
        const int vi = tid + u * NT;
        if (vi < T) tab[vi] = (long long)rint(ldexp((double)tv[u], sc));
    }
    // 1. Mt_ij
    const int W1 = pre[D];
    if ((long long)W1 * 8 <= (long long)n * D) {
        // from the class lists: entry q of the concatenated classes belongs to member dm
        // with pre[dm] <= q < pre[dm + 1] (found once by bisection, then advanced)
        int dm = 0;
        if (tid < W1) {
            int lo = 0, hi = D - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= tid) lo = mid; else hi = mid - 1;
            }
            dm = lo;
        }
        int js[B];
        auto fetch = [&](int q0) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int q = q0 + u * NT;
                js[u] = -1;
                if (q < W1) {
                    while (pre[dm + 1] <= q) ++dm;
                    js[u] = gview(d.cls_v)[(size_t)dm * cs + cbeg[dm] + (q - pre[dm])];
                }
            }
        };
        fetch(tid);
        for (int q0 = tid; q0 < W1; q0 += B * NT) {
            int cur[B];
#pragma unroll
            for (int u = 0; u < B; ++u) cur[u] = js[u];
            if (q0 + B * NT < W1) fetch(q0 + B * NT);
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (cur[u] >= 0) atomicAdd(&cnt[cur[u]], 1u);
        }
    } else {
        // by comparison: eight members per 16-byte word of a vertex-major row; members
        // beyond D (the row padding) are masked out
        const int nw = (int)(cTs / 8);
        for (int j0 = tid; j0 < n; j0 += 2 * NT) {
            int m2[2] = {0, 0};
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j = j0 + u * NT;
                if (j >= n) continue;
                const int16_t* row = cT + (size_t)j * cTs;
                for (int w = 0; w < nw; ++w) {
                    const u32x4n x = gload16(row + 8 * w);
                    const u32x4n y = *(const u32x4n*)(ci + 8 * w);
                    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        const int m0 = 8 * w + 2 * h;
                        const uint32_t valid = (m0 < D ? 0x8000u : 0u) | (m0 + 1 < D ? 0x80000000u : 0u);
                        m2[u] += equal_halves_in(xs[h], ys[h], valid);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (j0 + u * NT < n) cnt[j0 + u * NT] = (uint32_t)m2[u];
        }
    }
    __syncthreads();
    // 2. table index of P_ij for every j; the nonzero entries go to the list
    for (int base = 0, pass = 0; base < n; base += 4 * NT, ++pass) {
        const int j0 = base + 4 * tid;
        int vi[4];
        bool nz[4];
        if (j0 < n) {
            uint32_t a4 = 0;
            if (pass < kPsA8) {
#pragma unroll
                for (int u = 0; u < kPsA8; ++u)
                    if (u == pass) a4 = a4pre[u];
            } else {
                a4 = gview((const uint32_t*)(arow + j0))[0];
            }
            const u32x4n c4 = *(const u32x4n*)(cnt + j0);
            const uint32_t cw[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + u;
                const bool edge = ((a4 >> (8 * u)) & 0xFFu) != 0;
                const bool excl = !edge && !diag && j == i;
                vi[u] = excl ? zslot : (edge ? D + 1 + (int)cw[u] : (int)cw[u]);
                nz[u] = j < n && tab[vi[u]] != 0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) { vi[u] = zslot; nz[u] = false; }
        }
        unsigned long long bal[4];
        int tot = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bal[u] = __ballot(nz[u]);
            tot += __popcll(bal[u]);
        }
        int off = 0;
        if (lane == 0 && tot > 0) off = atomicAdd(&nzc[0], tot);
        off = __shfl(off, 0);
        const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (nz[u]) list[off + __popcll(bal[u] & below)] = (uint32_t)(j0 + u) | ((uint32_t)vi[u] << 16);
            off += __popcll(bal[u]);
        }
    }
    __syncthreads();
    const int nnz = nzc[0];
    // 3. members PM (= 8) at a time
    __attribute__((address_space(1))) float* Gg = (__attribute__((address_space(1))) float*)d.G;
    const double inv = ldexp(1.0, -sc);
    constexpr int KWF = KW > 0 ? KW : 1;
    FuseCtx fc{};
    if constexpr (KW > 0)
        if (fuse) fc = fuse_ctx(d, st);
    const int wave = tid >> 6;
    for (int d0 = 0; d0 < D; d0 += PM) {
        const int pm = min(PM, D - d0);
        // fused: wave w < pm loads row (d0 + w, i) of the weights and of the uint16 A.S counts
        // now, behind the accumulation below (PM is at most the block's wave count)
        float wv[KWF];
        uint32_t gr[KWF];
        if constexpr (KW > 0)
            if (fuse && wave < pm) fuse_row_load<KW>(d, fc, d0 + wave, i, lane, true, wv, gr);
        // f_color (fast path): thread dd < pm loads the contraction's (A.S)[i, c_d(i)] of member
        // d0 + dd now, behind the accumulation below, and adds it to the slots before the barrier
        // that precedes this group's read-modify-write of G (or its row updates)
        float own = 0.0f;
        if (accumulate && tid < pm) {
            const size_t o = ((size_t)(d0 + tid) * n + i) * k + ci[d0 + tid];
            own = fuse ? (float)gview((const uint16_t*)d.G)[o] : sgn * Gg[o];
        }
        // the accumulators start at zero: cleared here before the first group (they share their
        // words with the counts of steps 1-2), and by the fused row updates, which clear each
        // member's row once they have read it, before the later groups
        if (!fuse || d0 == 0) {
            for (int e = tid; e < pm * k / 2; e += NT) ((u32x4n*)acc)[e] = u32x4n{0u, 0u, 0u, 0u};
            if ((pm * k) & 1)
                if (tid == 0) acc[pm * k - 1] = 0ull;
            __syncthreads();
        }
        // one list entry per thread: the colours of its vertex j in the group's (at most eight)
        // members come in one 16-byte word of the vertex-major colours (rows padded to a multiple
        // of eight), and each member's accumulator of that colour takes P_ij.  The next entry's
        // word is loaded before this entry's LDS atomics.
        const auto* __restrict__ cTg = gview(cT);
        auto word = [&](int e, u32x4n& w, int& vi) {
            vi = 0;
            if (e < nnz) {
                const uint32_t ent = list[e];
                w = *(const __attribute__((address_space(1))) u32x4n*)(cTg + (size_t)(ent & 0xFFFFu) * cTs + d0);
                vi = (int)(ent >> 16);
            }
        };
        u32x4n wn = {0u, 0u, 0u, 0u};
        int vn;
        word(tid, wn, vn);
        for (int e = tid; e < nnz; e += NT) {
            const u32x4n wc = wn;
            const int vc = vn;
            word(e + NT, wn, vn);
            const unsigned long long v = (unsigned long long)tab[vc];
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                if (h < pm) {
                    const int c = (int)((wc[h >> 1] >> (16 * (h & 1))) & 0xFFFFu);
                    atomicAdd(&acc[h * k + c], v);
                }
            }
        }
        // the number of row i's neighbours sharing its colour (the gather of 2 f_color)
        if (accumulate && tid < pm)
            atomicAdd(&d.f2p[(size_t)(d0 + tid) * kF2Slots + (i & (kF2Slots - 1))], (int)own);
        __syncthreads();
        if constexpr (KW > 0) {
            if (fuse) {
                // gS = sgn (A.S + P.S) for row (d0 + wave, i): the member's sums to FP32 (sgn P.S)
                // and added to the A.S counts, rounded as the unfused path rounds the stored G;
                // the row's accumulators are cleared for the next group; then the row update
                if (wave < pm) {
                    float gv[KW];
                    unsigned long long* __restrict__ ar = acc + wave * k + lane;
#pragma unroll
                    for (int q = 0; q < KW; ++q) {
                        gv[q] = 0.0f;
                        if (lane + 64 * q < k) {
                            gv[q] = sgn * (float)gr[q] + sgn * (float)((double)(long long)ar[64 * q] * inv);
                            ar[64 * q] = 0ull;
                        }
                    }
                    fuse_row_update<KW, ADD>(d, st, fc, d0 + wave, i, lane, wv, gv);
                }
                __syncthreads();
                continue;
            }
        }
        for (int e0 = tid; e0 < pm * k; e0 += 4 * NT) {
            float prev[4];
            size_t off[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * NT;
                prev[u] = 0.0f;
                off[u] = 0;
                if (e < pm * k) {
                    const int dd = e / k, l = e - dd * k;
                    off[u] = ((size_t)(d0 + dd) * n + i) * k + l;
                    if (accumulate) prev[u] = Gg[off[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * NT;
                if (e < pm * k) Gg[off[u]] = prev[u] + sgn * (float)((double)(long long)acc[e] * inv);
            }
        }
        __syncthreads();
    }
}


// One-hot S^T [rows (d,l)][cols j] in the operand format; 16 columns per thread
// (fp4: two columns per byte, the lower in the low nibble, 1.0 = 0x2; both contraction
// passes read it).
__device__ __forceinline__ void expand_block(const GraphDev* __restrict__ gd, int G, int b, int honor_stop, int next, int gate,
                             int adv) {
    const GraphDev& d = gd[find_graph(gd, G, b, [](const GraphDev& x) { return x.ex_begin; })];
    GraphState* st = d.st;
    if (honor_stop && (st->stopped || (adv && st->next_bad))) return;
    const int p = next ? st->pS ^ 1 : st->pS;
    // a thread takes 16 columns of kExpandRows consecutive colour rows of one member: their
    // colours are loaded once for all of its rows
    const int cgs = d.n_pad / 16;
    const int kr = (d.k + kExpandRows - 1) / kExpandRows;   // row groups per member
    const long long item = (long long)(b - d.ex_begin) * 256 + threadIdx.x;
    const long long rg = item / cgs;
    const int cg = (int)(item - rg * cgs);
    if (rg >= (long long)d.D * kr) return;
    const int dm = (int)(rg / kr);
    const int l0 = (int)(rg - (long long)dm * kr) * kExpandRows;
    const int j0 = cg * 16;
    const int CM = d.cmax;
    uint32_t w1[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};   // the member's 16 colours (one colour per vertex)
    if (CM == 1 && j0 < d.n) {
        // 16 colours in two 16-byte loads (rows are padded to 64 entries)
        const int16_t* c = d.c[p] + (size_t)dm * d.cs;
        const uint4 a = *(const uint4*)(c + j0);
        const uint4 bb = *(const uint4*)(c + j0 + 8);
        w1[0] = a.x; w1[1] = a.y; w1[2] = a.z; w1[3] = a.w;
        w1[4] = bb.x; w1[5] = bb.y; w1[6] = bb.z; w1[7] = bb.w;
    }
#pragma unroll 1
    for (int rr = 0; rr < kExpandRows; ++rr) {
    const int l = l0 + rr;
    if (l >= d.k) break;
    const int row = dm * d.k + l;
    uint32_t mask = 0;   // bit q set when column j0+q has colour l (one of its colours: multicolouring)
    if (j0 < d.n) {
        if (CM == 1) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int col = (int)((w1[q >> 1] >> (16 * (q & 1))) & 0xFFFFu);
                if (j0 + q < d.n && col == l) mask |= 1u << q;
            }
        } else {
            for (int sl = 0; sl < CM; ++sl) {
                const int16_t* c = d.sel + ((size_t)dm * CM + sl) * d.cs;
                const uint4 a = *(const uint4*)(c + j0);
                const uint4 bb = *(const uint4*)(c + j0 + 8);
                const uint32_t w[8] = {a.x, a.y, a.z, a.w, bb.x, bb.y, bb.z, bb.w};
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int col = (int)((w[q >> 1] >> (16 * (q & 1))) & 0xFFFFu);
                    if (j0 + q < d.n && col == l) mask |= 1u << q;
                }
            }
        }
    }
    const size_t off = (size_t)row * d.n_pad + j0;
    if (d.op == kPrecFP32) {
        float4* o = (float4*)((float*)d.Sop[p] + off);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float4 x;
            x.x = (mask >> (4 * v + 0)) & 1 ? 1.0f : 0.0f;
            x.y = (mask >> (4 * v + 1)) & 1 ? 1.0f : 0.0f;
            x.z = (mask >> (4 * v + 2)) & 1 ? 1.0f : 0.0f;
            x.w = (mask >> (4 * v + 3)) & 1 ? 1.0f : 0.0f;
            o[v] = x;
        }
    } else {
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if ((mask >> q) & 1) w[q >> 3] |= 0x2u << (4 * (q & 7));
        *(uint2*)((uint8_t*)d.Sop[p] + (off >> 1)) = make_uint2(w[0], w[1]);
    }
    }
}

__global__ __launch_bounds__(256) void k_expand(const GraphDev* __restrict__ gd, int G, int total_blocks,
                                                int honor_stop, int next, int gate) {
    const int b = blockIdx.x;
    if (b >= total_blocks) return;
    expand_block(gd, G, b, honor_stop, next, gate, 0);
}

// ------------------------------------------------------------ step 3 -----------

// Group concentration Mt_ij = #{d : c_d(i) = c_d(j)} over TS x TS tiles of the
// upper triangle (mirrored; TS = 64, or 32 when n_pad <= 2048 so small graphs still
// give every CU work), and from it the penalty operand
//   P_ij = t * (a_ij ? 2 alpha lambda m^(alpha-1) : -[i != j or bonus_diag] 2 beta mu m^(beta-1)).
// Optional: Mt to mt_out (int32 [n][n]) and kappa / varpi partial sums.  Each of the
// 256 threads owns a PT x PT block of the tile (PT = TS / 16).
//
// The compares are the work (n^2 D / 2 of them, VALU), so colours are compared packed: the tile's
// vertices get their colours in LDS vertex-major, four members to a word (BYTES: colours below
// 126) or two, and for a pair of words (x ^ y) + 0x7f7f7f7f (0x7fff7fff) sets the top bit of
// every field that differs, which a masked population count adds to the pair's count: three
// instructions per four (two) members.  Members past D and unselected slots hold 0x7f on the i side and
// 0x7e on the j side (0x7fff, 0x7ffe), which differ from each other and from every colour.  16-byte
// pieces of a row are swizzled so that the lanes of a read fall on different banks.
// G(1000, .5), k = 90, D = 256: 20.8 us with the member and expansion blocks in the same launch,
// against 30.9 us (16-bit compares, one pair at a time) and 14.6 us for two launches.
constexpr int kMtWords = 32;    // words per vertex and LDS chunk (over the slots of a multicolouring)
constexpr int kMtLds = 2 * 64 * kMtWords * 4 + 2 * 256 * 8;   // both sides of a tile, the loss reduction

template <int PT, int BYTES>
__device__ __forceinline__ void mtilde_tile(const GraphDev& d, GraphState* st, int b, int flags, int32_t* __restrict__ mt_out,
                            uint8_t* lds) {
    constexpr int TS = 16 * PT;
    constexpr int PW = BYTES ? 4 : 2;   // members per word
    constexpr uint32_t kLow = BYTES ? 0x7f7f7f7fu : 0x7fff7fffu;
    uint32_t* sw = (uint32_t*)lds;      // [2][TS][kMtWords]
    double(*red)[256] = (double(*)[256])(lds + 2 * 64 * kMtWords * 4);
    const float tf = (float)st->t;
    const bool pen = !(flags & kFlagMtOut) && ((d.lambda * tf != 0.0f) || (d.mu * tf != 0.0f));
    const int p = st->pS;
    // upper-triangle tile (ti <= tj)
    int u = b - d.mt_begin, ti = 0, T = d.mt_T;
    while (u >= T - ti) { u -= T - ti; ++ti; }
    const int tj = ti + u;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int i0 = ti * TS, j0 = tj * TS;
    int cnt[PT][PT];
#pragma unroll
    for (int a = 0; a < PT; ++a)
#pragma unroll
        for (int q = 0; q < PT; ++q) cnt[a][q] = 0;
    // planes of colours: the members' (one colour per vertex), or for multicolouring the slots of
    // the selection, every slot against every slot of the same member
    const int CM = d.cmax;
    const int16_t* __restrict__ base = CM > 1 ? d.sel : d.c[p];
    const int cs = d.cs, D = d.D, nv = d.n;
    const int W = (D + PW - 1) / PW;
    const int wp = CM == 1 ? kMtWords : (kMtWords / CM) & ~3;   // words per plane and chunk
    int total = 0;      // compares per pair
    for (int w0 = 0; w0 < W; w0 += wp) {
        const int wn = (min(wp, W - w0) + 3) & ~3;
        total += wn * PW * CM * CM;
        __syncthreads();
        const int per = CM * wn;        // words per vertex
        for (int e = threadIdx.x; e < 2 * per * TS; e += 256) {
            const int x = e & (TS - 1);
            int r = e / TS;
            const int side = r >= per ? 1 : 0;
            r -= side * per;
            const int pl = CM == 1 ? 0 : r / wn, w = r - pl * wn;
            const int v = (side ? j0 : i0) + x;
            int16_t cv[PW];
#pragma unroll
            for (int h = 0; h < PW; ++h) {
                const int dm = (w0 + w) * PW + h;
                cv[h] = v < nv && dm < D ? gview(base)[(size_t)(dm * CM + pl) * cs + v] : (int16_t)-1;
            }
            uint32_t word = 0;
#pragma unroll
            for (int h = 0; h < PW; ++h) {
                const uint32_t f = cv[h] < 0 ? (BYTES ? 0x7fu : 0x7fffu) - (uint32_t)side : (uint32_t)cv[h];
                word |= f << (h * (32 / PW));
            }
            const int slot = (pl * wn + w) >> 2;
            sw[(side * TS + x) * kMtWords + (((slot ^ (x / PT)) & 7) << 2) + (w & 3)] = word;
        }
        __syncthreads();
        auto piece = [&](int side, int r, int slot) {
            return *(const uint4*)(sw + (side * TS + r) * kMtWords + (((slot ^ (r / PT)) & 7) << 2));
        };
        const int np = wn >> 2;
        for (int s1 = 0; s1 < CM; ++s1)
            for (int s2 = 0; s2 < CM; ++s2)
                for (int c4 = 0; c4 < np; ++c4) {
                    uint4 av[PT], bv[PT];
#pragma unroll
                    for (int a = 0; a < PT; ++a) {
                        av[a] = piece(0, ty * PT + a, s1 * np + c4);
                        bv[a] = piece(1, tx * PT + a, s2 * np + c4);
                    }
#pragma unroll
                    for (int a = 0; a < PT; ++a)
#pragma unroll
                        for (int q = 0; q < PT; ++q) {
                            cnt[a][q] += __builtin_popcount(((av[a].x ^ bv[q].x) + kLow) & ~kLow);
                            cnt[a][q] += __builtin_popcount(((av[a].y ^ bv[q].y) + kLow) & ~kLow);
                            cnt[a][q] += __builtin_popcount(((av[a].z ^ bv[q].z) + kLow) & ~kLow);
                            cnt[a][q] += __builtin_popcount(((av[a].w ^ bv[q].w) + kLow) & ~kLow);
                        }
                }
    }
    // the fields that agree
#pragma unroll
    for (int a = 0; a < PT; ++a)
#pragma unroll
        for (int q = 0; q < PT; ++q) cnt[a][q] = total - cnt[a][q];
    if (flags & kFlagMtOut) {
        // the counts alone, through LDS, so that the tile and its mirror leave in whole rows (n = 2999, D = 25: the
        // launch 37.7 -> 22.5 us)
        if (!mt_out) return;
        const int n = d.n;
        const bool mirror = ti != tj;
        constexpr int LT = TS + 1;
        static_assert(TS * LT * 4 <= kMtLds, "count tile fits");
        int* ct = (int*)lds;
        __syncthreads();
#pragma unroll
        for (int a = 0; a < PT; ++a)
#pragma unroll
            for (int q = 0; q < PT; ++q) ct[(ty * PT + a) * LT + tx * PT + q] = cnt[a][q];
        __syncthreads();
        const int x = threadIdx.x & (TS - 1);
        for (int y = threadIdx.x / TS; y < TS; y += 256 / TS) {
            if (i0 + y < n && j0 + x < n) mt_out[(size_t)(i0 + y) * n + j0 + x] = ct[y * LT + x];
            if (mirror && j0 + y < n && i0 + x < n) mt_out[(size_t)(j0 + y) * n + i0 + x] = ct[x * LT + y];
        }
        return;
    }
    const bool mirror = ti != tj;
    double ka = 0.0, vb = 0.0;
    const bool fp32 = d.op == kPrecFP32;
    // fields used between the stores below stay in registers (no reload through gd)
    const int n = d.n;
    const size_t n_pad = d.n_pad;
    const uint8_t* __restrict__ A8 = d.A8;
    const float* __restrict__ lut_pen = d.lut_pen;
    const float* __restrict__ lut_bon = d.lut_bon;
    const double* __restrict__ lut_ka = d.lut_ka;
    const double* __restrict__ lut_vb = d.lut_vb;
    const bool bdiag = d.bonus_diag != 0;
    void* __restrict__ Pop = d.Pop;
    // the thread's block: rows i0 + PT ty + a, columns j0 + PT tx + q; the adjacency of a
    // row's PT columns is one load (A8 rows are n_pad bytes, PT | j), and the operand goes
    // out as one vector store per row of the block and per row of its mirror
    const int ib = i0 + ty * PT, jb = j0 + tx * PT;
    float val[PT][PT];
#pragma unroll
    for (int a = 0; a < PT; ++a) {
        const int i = ib + a;
        uint32_t arow;
        if constexpr (PT == 4)
            arow = gview((const uint32_t*)(A8 + (size_t)i * n_pad + jb))[0];
        else
            arow = gview((const uint16_t*)(A8 + (size_t)i * n_pad + jb))[0];
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int j = jb + q;
            // the sign of an fp32 entry tells edges (+) from the others (-), also where it is zero: the
            // class-row sums count by it (their graphs' tables are finite and not negative, -0 included)
            float v = -0.0f;
            if (i < n && j < n) {
                const int m = cnt[a][q];
                const bool edge = ((arow >> (8 * q)) & 0xFFu) != 0;
                const bool bon = !edge && (i != j || bdiag);
                if (edge) v = tf * lut_pen[m];
                else if (bon) v = -(tf * lut_bon[m]);
                if (flags & kFlagLoss) {
                    const double wgt = mirror ? 2.0 : 1.0;
                    if (edge) ka += wgt * lut_ka[m];
                    else if (bon) vb += wgt * lut_vb[m];
                }
            }
            val[a][q] = v;
        }
    }
    if (pen || (flags & kFlagForcePen)) {
        if (fp32) {
#pragma unroll
            for (int a = 0; a < PT; ++a) {
                float* o = (float*)Pop + (size_t)(ib + a) * n_pad + jb;
                if constexpr (PT == 4) *(float4*)o = make_float4(val[a][0], val[a][1], val[a][2], val[a][3]);
                else *(float2*)o = make_float2(val[a][0], val[a][1]);
            }
            if (mirror) {
#pragma unroll
                for (int q = 0; q < PT; ++q) {
                    float* o = (float*)Pop + (size_t)(jb + q) * n_pad + ib;
                    if constexpr (PT == 4) *(float4*)o = make_float4(val[0][q], val[1][q], val[2][q], val[3][q]);
                    else *(float2*)o = make_float2(val[0][q], val[1][q]);
                }
            }
        } else {
            // the penalty pass multiplies by 2 S (cheaper to widen from fp4), so the operand is
            // stored halved, exactly
#pragma unroll
            for (int a = 0; a < PT; ++a)
#pragma unroll
                for (int q = 0; q < PT; ++q) val[a][q] *= 0.5f;
#pragma unroll
            for (int a = 0; a < PT; ++a) {
                uint16_t* o = (uint16_t*)Pop + (size_t)(ib + a) * n_pad + jb;
                const uint32_t lo = f32_to_bf16_rne(val[a][0]) | ((uint32_t)f32_to_bf16_rne(val[a][1]) << 16);
                if constexpr (PT == 4) {
                    const uint32_t hi = f32_to_bf16_rne(val[a][2]) | ((uint32_t)f32_to_bf16_rne(val[a][3]) << 16);
                    *(uint2*)o = make_uint2(lo, hi);
                } else {
                    *(uint32_t*)o = lo;
                }
            }
            if (mirror) {
#pragma unroll
                for (int q = 0; q < PT; ++q) {
                    uint16_t* o = (uint16_t*)Pop + (size_t)(jb + q) * n_pad + ib;
                    const uint32_t lo = f32_to_bf16_rne(val[0][q]) | ((uint32_t)f32_to_bf16_rne(val[1][q]) << 16);
                    if constexpr (PT == 4) {
                        const uint32_t hi = f32_to_bf16_rne(val[2][q]) | ((uint32_t)f32_to_bf16_rne(val[3][q]) << 16);
                        *(uint2*)o = make_uint2(lo, hi);
                    } else {
                        *(uint32_t*)o = lo;
                    }
                }
            }
        }
    }
    if (flags & kFlagLoss) {
        red[0][threadIdx.x] = ka;
        red[1][threadIdx.x] = vb;
        __syncthreads();
        for (int s = 128; s >= 1; s >>= 1) {
            if (threadIdx.x < s) {
                red[0][threadIdx.x] += red[0][threadIdx.x + s];
                red[1][threadIdx.x] += red[1][threadIdx.x + s];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            d.part[2 * (b - d.mt_begin) + 0] = red[0][0];
            d.part[2 * (b - d.mt_begin) + 1] = red[1][0];
        }
    }
}

// tile b (flattened over the graphs) of the group-concentration kernel (lds: kMtLds bytes); adv:
// the launch also ends the previous iteration (a pending non-finite update counts as a stop)
__device__ __forceinline__ void mtilde_block(const GraphDev* __restrict__ gd, int G, int b, int honor_stop, int flags, int gsel,
                             int32_t* __restrict__ mt_out, uint8_t* lds, int adv = 0) {
    const int g = find_graph(gd, G, b, [](const GraphDev& x) { return x.mt_begin; });
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (honor_stop && (st->stopped || (adv && st->next_bad))) return;
    if (gsel >= 0 && g != gsel) return;
    const float tf = (float)st->t;
    const bool pen = (d.lambda * tf != 0.0f) || (d.mu * tf != 0.0f);
    if (!pen && !(flags & (kFlagForcePen | kFlagLoss | kFlagMtOut))) return;
    if ((flags & kFlagGate) && d.psparse && !st->pdense) return;
    if (d.mt_ts == 32) {
        if (d.k <= 126) mtilde_tile<2, 1>(d, st, b, flags, mt_out, lds);
        else mtilde_tile<2, 0>(d, st, b, flags, mt_out, lds);
    } else {
        if (d.k <= 126) mtilde_tile<4, 1>(d, st, b, flags, mt_out, lds);
        else mtilde_tile<4, 0>(d, st, b, flags, mt_out, lds);
    }
}
__global__ __launch_bounds__(256) void k_mtilde(const GraphDev* __restrict__ gd, int G, int total_tiles,
                                                int honor_stop, int flags, int gsel, int32_t* __restrict__ mt_out) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kMtLds];
    const int b = blockIdx.x;
    if (b >= total_tiles) return;
    mtilde_block(gd, G, b, honor_stop, flags, gsel, mt_out, lds);
}

// ------------------------------------------------ merged first launch -----------

// Position q of the order in which the fp32 contraction sums the vertices of a class (components
// of 16-byte chunks, then chunks, within each 16 vertices) -> vertex.  The class-row sums follow it,
// so they give the contraction's bits.
__device__ __forceinline__ int vertex_at(int q) { return (q & ~15) | ((q & 3) << 2) | ((q >> 2) & 3); }

// words of the member block's dynamic LDS: scratch, counts, per-wave cursors, per-wave 64-bit batch
// masks, class starts, then the list (each class padded to a multiple of four entries)
__host__ __device__ inline size_t member_lds_bytes(int k, int n) {
    return sizeof(int) * ((size_t)kPrepScratch + 14 * (size_t)k + 2) + sizeof(int16_t) * (((size_t)n + 3 * (size_t)k + 1) & ~(size_t)1);
}

// One part's answer to whether member m is illegal: the parts of a member (the blocks of its conflict search and,
// with an added fitness, its member block) add to one word, and the last of them, which sees that all have answered,
// clears it and lists a member that none found illegal.  The word is the member's first conflict slot, which is zero
// between the launches that use it.
__device__ __forceinline__ void legal_vote(const GraphDev& d, GraphState* st, int m, int parts, bool bad) {
    int* word = d.f2p + (size_t)m * kF2Slots;
    const int add = bad ? 0x10000 : 1;
    const int all = atomicAdd(word, add) + add;
    if ((all & 0xFFFF) + (all >> 16) != parts) return;
    atomicExch(word, 0);
    if ((all >> 16) == 0) atomicMin(&st->legal_min[st->t & 1], m);
}

// whether an iteration asks for the members' legality (minimum sum colouring always has a colour cost; a
// multicolouring graph's conflicts come from the contraction)
__device__ __forceinline__ bool asks_legal(const GraphDev& d, int want) {
    return (want & 1) && d.stop_on_legal && d.problem != kProbMSCP && d.cmax == 1;
}

// Member `mem` of the merged first launch (one colour per vertex): class sizes and the added
// fitness where the problem has one, with want & 2 the class lists in summation order for graphs on the
// class-row sums, and with want & 4 its conflict counter cleared.
__device__ __forceinline__ void member_block(const GraphDev* __restrict__ gd, int G, int mem, int honor_stop, int adv,
                                             int want, int* sh) {
    const GraphDev& d = gd[find_graph(gd, G, mem, [](const GraphDev& x) { return x.mem_begin; })];
    GraphState* st = d.st;
    // read before this launch writes the state; the write below only turns `stopped` on, exactly when
    // next_bad is set, so every block of the launch takes the same decision (see prep_member)
    const bool stop_now = honor_stop && (st->stopped || (adv && st->next_bad));
    const int tid = threadIdx.x;
    if (mem == d.mem_begin && tid == 0) {
        if (adv && !st->stopped && st->next_bad) {
            st->error = -5;
            st->stopped = 1;
        }
        st->tc = st->t;
    }
    const int m = mem - d.mem_begin;
    // a gather follows: its counters start at zero
    if ((want & 4) && !stop_now && tid == 0) d.f2[m] = 0;
    if (stop_now || d.cmax > 1) return;
    const int k = d.k, n = d.n;
    const bool added = prob_added(d.problem);
    const bool lists = d.rows && (want & 2);
    if (!lists && !added) return;
    const int16_t* __restrict__ c = d.c[st->pS] + (size_t)m * d.cs;
    int* part_sum = sh;                                       // [257]
    long long* fsum = (long long*)(sh + 260);                 // [4]
    int* cnt = sh + kPrepScratch;                             // [k]
    int* cw = cnt + k;                                        // [4][k]
    unsigned long long* msk = (unsigned long long*)(cw + 4 * k + (k & 1));   // [4][k] (8-byte aligned)
    int* offl = (int*)(msk + 4 * (size_t)k);                  // [k]
    int16_t* lst = (int16_t*)(offl + k + (k & 1));            // [n + 3 k at most]
    constexpr int NW = 4;
    const int wv = tid >> 6, lane = tid & 63;
    const int Q = ((n + NW - 1) / NW + 63) & ~63;             // positions per wave
    for (int l = tid; l < k; l += 256) cnt[l] = 0;
    if (lists)
        for (int l = tid; l < NW * k; l += 256) {
            cw[l] = 0;
            msk[l] = 0ull;
        }
    __syncthreads();
    const int np16 = (n + 15) & ~15;                          // positions (those of vertices >= n are skipped)
    const int e0 = wv * Q, e1 = min(np16, (wv + 1) * Q);
    for (int i0 = e0 + lane; i0 < e1; i0 += 64 * kPrepBatch) {
        int xs[kPrepBatch];
#pragma unroll
        for (int u = 0; u < kPrepBatch; ++u) {
            const int q = i0 + 64 * u, v = vertex_at(q);
            xs[u] = q < e1 && v < n ? (int)gview(c)[v] : -1;
        }
#pragma unroll
        for (int u = 0; u < kPrepBatch; ++u)
            if (xs[u] >= 0) {
                atomicAdd(&cnt[xs[u]], 1);
                if (lists) atomicAdd(&cw[wv * k + xs[u]], 1);
            }
    }
    __syncthreads();
    if (added) {
        int32_t* V = d.V[st->pS] + (size_t)m * k;
        const int c1 = d.c1, c2 = d.c2;
        long long fe = 0;
        for (int l = tid; l < k; l += 256) {
            const long long v = cnt[l];
            V[l] = cnt[l];
            if (d.problem == kProbMSCP) {
                fe += (long long)(l + 1) * v;
            } else {
                const long long x = v > c1 ? v - c1 : c1 - v;
                const long long y = v > c2 ? v - c2 : c2 - v;
                fe += x < y ? x : y;
            }
        }
        for (int o = 32; o >= 1; o >>= 1) fe += __shfl_xor(fe, o);
        if (lane == 0) fsum[wv] = fe;
        __syncthreads();
        if (tid == 0) {
            const long long f = fsum[0] + fsum[1] + fsum[2] + fsum[3];
            d.feq[m] = f;
            // with an added fitness the member is legal only if that is 0 too
            if (asks_legal(d, want)) legal_vote(d, st, m, d.lg_parts + 1, f != 0);
        }
    }
    if (lists) {
        // exclusive scan of the padded counts (as in prep_member); the padding entries are -1
        const int per = (k + 255) / 256;
        const int lb = min(k, tid * per), le = min(k, lb + per);
        int run = 0;
        for (int l = lb; l < le; ++l) run += (cnt[l] + 3) & ~3;
        part_sum[tid] = run;
        __syncthreads();
        if (tid < 64) {
            const int v0 = part_sum[4 * tid], v1 = part_sum[4 * tid + 1], v2 = part_sum[4 * tid + 2],
                      v3 = part_sum[4 * tid + 3];
            const int sum = v0 + v1 + v2 + v3;
            int incl = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (tid >= o) incl += y;
            }
            const int ex = incl - sum;
            part_sum[4 * tid] = ex;
            part_sum[4 * tid + 1] = ex + v0;
            part_sum[4 * tid + 2] = ex + v0 + v1;
            part_sum[4 * tid + 3] = ex + v0 + v1 + v2;
            if (tid == 63) part_sum[256] = incl;
        }
        __syncthreads();
        const int total = part_sum[256];
        int acc = part_sum[tid];
        for (int l = lb; l < le; ++l) {
            const int pads = -cnt[l] & 3;
            offl[l] = acc;
            // start (a multiple of four) and padding in one word
            d.cls_off[(size_t)m * (k + 1) + l] = acc | pads;
            int q = acc;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int x = cw[w * k + l];
                cw[w * k + l] = q;
                q += x;
            }
            for (int e = 0; e < pads; ++e) lst[q + e] = (int16_t)-1;
            acc = q + pads;
        }
        if (tid == 0) d.cls_off[(size_t)m * (k + 1) + k] = total;
        __syncthreads();
        // placement in summation order: each wave walks its positions 64 at a time; lanes of one
        // colour find their rank among the batch in the colour's batch mask, and the last of them
        // moves the wave's cursor and clears the mask
        int* cur = cw + wv * k;
        unsigned long long* mw = msk + (size_t)wv * k;
        for (int i0 = e0 + lane; i0 - lane < e1; i0 += 64) {
            const int v = vertex_at(i0);
            const bool in = i0 < e1 && v < n;
            const int x = in ? (int)gview(c)[v] : 0;
            if (in) atomicOr(&mw[x], 1ull << lane);
            wave_sync();
            unsigned long long same = 0;
            int at = 0;
            if (in) {
                same = mw[x];
                at = cur[x];
            }
            wave_sync();
            if (in) {
                const int rank = __popcll(same & ((1ull << lane) - 1ull));
                lst[at + rank] = (int16_t)v;
                if ((same >> lane) == 1ull) {
                    cur[x] = at + rank + 1;
                    mw[x] = 0ull;
                }
            }
            wave_sync();
        }
        __syncthreads();
        // the entries as byte offsets of the vertices' rows of P; padding takes the row past the last, which is zero
        uint32_t* __restrict__ cj = d.cls_j + (size_t)m * d.js;
        const uint32_t rb = 4u * (uint32_t)d.n_pad;
        for (int q = tid; q < total; q += 256) cj[q] = (lst[q] < 0 ? (uint32_t)d.n_pad : (uint32_t)lst[q]) * rb;
    }
}

// words of 64 vertices per piece of the class masks below, and their row stride (odd: rows on different banks), for
// the LDS of a group-concentration tile; at least one word
struct ScanShape {
    int words, stride;
};
constexpr int kScanHead = 16;   // ints before the masks
__host__ __device__ inline ScanShape scan_shape(int n, int k) {
    constexpr int room = (kMtLds - 4 * kScanHead) / 8;
    const int all = (n + 63) / 64;
    if (k * (all | 1) <= room) return {all, all | 1};
    int w = room / k;
    if (w > 1 && !(w & 1) && k * (w + 1) > room) --w;
    if (w < 1) w = 1;
    return {w, w | 1};
}
__host__ __device__ inline size_t scan_lds_bytes(int n, int k) {
    return 4 * kScanHead + 8 * (size_t)k * scan_shape(n, k).stride;
}

// The conflict counts by these masks or by compares.  A piece of masks takes a block about 0.85 us whatever it holds;
// the compares take about 0.07 us per 10^6 pairs, and more blocks.  tcol_conflicts, masks and compares, fp4:
// n = 2000, k = 900, D = 16 (32 pieces) 58 and 34 us; k = 500 (7 pieces) 27.7 and 26.2, at D = 64 55 and 67;
// n = 1000, k = 500, D = 16 (4 pieces) 18.3 and 16.8, at D = 64 33 and 35; n = 4000, k = 200, D = 16 (6 pieces) 30 and
// 42.  One piece: n = 2000, k = 60, D = 64 26 and 44; n = 71, D = 16 3.9 and 3.4 (the launch).
inline bool count_by_masks(int n, int D, ScanShape ss) {
    return 2 * ceil_div(n, 64) <= ss.words * (1 + (long long)n * n * D / 6000000);
}

// the class masks of words [s0, s1) of the vertices with colours c, by the block's 256 threads (which have read the
// last ones before): msk[l * stride + w] holds the vertices of class l in word s0 + w
template <typename C>
__device__ __forceinline__ void class_masks(C c, int n, int k, ScanShape ss, int s0, int s1, unsigned long long* msk) {
    const int tid = threadIdx.x;
    const int end = min(n, 64 * s1);
    int x[4];
    auto load = [&](int v0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = c[min(v0 + 256 * u, end - 1)];
    };
    load(64 * s0 + tid);    // in flight while the masks are cleared
    for (int e = tid; e < k * ss.stride; e += 256) msk[e] = 0ull;
    __syncthreads();
    for (int v0 = 64 * s0 + tid; v0 < end; v0 += 256 * 4) {
        if (v0 >= 64 * s0 + 256 * 4) load(v0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + 256 * u;
            if (v < end) atomicOr((uint32_t*)(msk + x[u] * ss.stride + (v >> 6) - s0) + ((v >> 5) & 1), 1u << (v & 31));
        }
    }
    __syncthreads();
}

// The stop rule's question for one part of a member: whether some pair of its vertices conflicts (partitioning: is
// cut). The member's classes are bit masks in LDS, 64 vertices to a word, a piece of the words at a time, and vertex
// i's adjacency to 64 vertices is one word (A is symmetric, so a wave reads 64 rows' words in one load): i conflicts
// with those of them that both words hold.  n^2 / 128 words a member whatever its classes are, and a search that finds
// a pair ends at once, which in all but the last iterations is in the first words.
// Eight iterations with members one conflict from legal, D = 8 (fp4): n = 2700, k = 2 412 us, 384 without the stop
// rule; n = 5000, k = 3 647 and 643.  A scan of the pairs of each class, byte by byte, took 9350 and 22040 there.
__device__ __forceinline__ void legal_block(const GraphDev* __restrict__ gd, int G, int b, int honor_stop, int adv, int want,
                                            int* sh) {
    const GraphDev& d = gd[find_graph(gd, G, b, [](const GraphDev& x) { return x.lg_begin; })];
    GraphState* st = d.st;
    if (honor_stop && (st->stopped || (adv && st->next_bad))) return;
    if (!asks_legal(d, want)) return;
    const int n = d.n, k = d.k, parts = d.lg_parts;
    const int loc = b - d.lg_begin;
    const int m = loc / parts, part = loc - m * parts;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strips = (n + 63) / 64;
    const ScanShape ss = scan_shape(n, k);
    volatile int* found = sh;
    unsigned long long* msk = (unsigned long long*)(sh + kScanHead);
    const auto* __restrict__ c = gview((const int16_t*)d.c[st->pS]) + (size_t)m * d.cs;
    const size_t n_pad = d.n_pad;
    const unsigned long long flip = prob_partition(d.problem) ? ~0ull : 0ull;
    if (tid == 0) *found = 0;
    for (int s0 = 0; s0 < strips; s0 += ss.words) {
        const int s1 = min(strips, s0 + ss.words);
        class_masks(c, n, k, ss, s0, s1, msk);
        // this part's strips, the longest rows first; vertex i looks at the words up to its own
        for (int q = (strips - 1 - part) / parts - wave; q >= 0; q -= 4) {
            const int strip = part + q * parts;
            if (strip < s0 || *found) break;
            const int i = strip * 64 + lane;
            const unsigned long long* row = msk + (i < n ? (int)c[i] : 0) * ss.stride - s0;
            const auto* __restrict__ a = gview(d.Ab) + i;
            const int e = min(s1, strip + 1);
            for (int s = s0; s < e && !*found; s += 8) {
                unsigned long long w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = s + u < e ? a[(size_t)(s + u) * n_pad] : 0ull;
                unsigned long long hit = 0;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (s + u < e) hit |= w[u] & (row[s + u] ^ flip);
                if (__any(hit != 0ull)) *found = 1;
            }
        }
        __syncthreads();
        if (*found) break;      // no wave writes it before the next piece's barriers: the same answer for all
    }
    if (tid == 0) legal_vote(d, st, m, parts + (prob_added(d.problem) ? 1 : 0), *found != 0);
}

// 2 f_color without a contraction (one colour per vertex): each wave of a block takes 64 vertices of one member and
// counts, as the search above looks, the vertices that a word of A and the class's word of masks both hold.  Words
// before the vertices' own count twice, for the pair's other end.
// Launch with the member blocks: n = 2999, k = 211, D = 25 12.2 us, n = 1000, k = 90, D = 64 5.1 us (the compares of
// every pair of colours, below, 25 and 10.7; the contraction and its expansion 50 and 24).
__device__ __forceinline__ int count_masks(const GraphDev& d, int m, int part, ScanShape ss, int* sh) {
    const int n = d.n, k = d.k, strips = (n + 63) / 64, parts = count_parts(n);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned long long* msk = (unsigned long long*)(sh + kScanHead);
    const auto* __restrict__ c = gview((const int16_t*)d.c[d.st->pS]) + (size_t)m * d.cs;
    const size_t n_pad = d.n_pad;
    const int last = part + (strips - 1 - part) / parts * parts;    // the block's last strip
    const int strip = part + wave * parts;                          // past the last: none
    const int i = strip * 64 + lane;
    const int ci = i < n ? (int)c[i] : 0;
    const auto* __restrict__ a = gview(d.Ab) + min(strip, strips - 1) * 64 + lane;
    int below = 0, own = 0;
    for (int s0 = 0; s0 <= last; s0 += ss.words) {
        const int s1 = min(strips, s0 + ss.words);
        if (s0) __syncthreads();
        // the first words are in flight while the masks are made (past the strip's own they are not counted)
        unsigned long long w[8];
        auto load = [&](int s) {
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = a[(size_t)min(s + u, strips - 1) * n_pad];
        };
        load(s0);
        class_masks(c, n, k, ss, s0, s1, msk);
        if (strip > last) continue;
        const unsigned long long* row = msk + ci * ss.stride - s0;
        const int e = min(s1, strip);
        for (int s = s0; s < e; s += 8) {
            if (s > s0) load(s);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s + u < e) below += __popcll(w[u] & row[s + u]);
        }
        if (strip >= s0 && strip < s1) own = __popcll(a[(size_t)strip * n_pad] & row[strip]);
    }
    return 2 * below + own;
}

// even bits of x to the low half, odd bits to the high half
__device__ __forceinline__ uint32_t unshuffle(uint32_t x) {
    uint32_t t = (x ^ (x >> 1)) & 0x22222222u;
    x ^= t ^ (t << 1);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu;
    x ^= t ^ (t << 2);
    t = (x ^ (x >> 4)) & 0x00F000F0u;
    x ^= t ^ (t << 4);
    t = (x ^ (x >> 8)) & 0x0000FF00u;
    return x ^ t ^ (t << 8);
}

// The same by compares, as fast for any number of classes: a block takes one strip of 64 vertices i, one per lane, and
// each of its waves a quarter of the vertices j.  Lane i's adjacency to 64 vertices is one word, their colours come two
// to a scalar word; a pair of colours takes four instructions: (c_i ^ c_j) + 0x7fff7fff sets bits 15 and 31 where they
// differ, the complemented adjacency bits of the two vertices are shifted onto the same bits, and a masked population
// count adds the pairs that are no conflict.
__device__ __forceinline__ int count_compares(const GraphDev& d, int m, int strip) {
    const int n = d.n, strips = (n + 63) / 64;
    const int quarter = (strips + 3) / 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int s0 = min(strips, wave * quarter), s1 = min(strips, s0 + quarter);
    const int i = strip * 64 + (threadIdx.x & 63);
    const int16_t* __restrict__ c = d.c[d.st->pS] + (size_t)m * d.cs;
    const uint32_t ci = (uint16_t)gview(c)[i];      // rows are padded to 64 entries
    const uint32_t ci2 = ci | (ci << 16);
    const unsigned long long* __restrict__ Ab = d.Ab + i;
    const size_t n_pad = d.n_pad;
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
    int none = 0;
    unsigned long long a = s0 < s1 ? gview(Ab)[(size_t)s0 * n_pad] : 0ull;
    for (int s = s0; s < s1; ++s) {
        const unsigned long long an = s + 1 < s1 ? gview(Ab)[(size_t)(s + 1) * n_pad] : 0ull;
        const uint32_t lo = ~unshuffle((uint32_t)a), hi = ~unshuffle((uint32_t)(a >> 32));
        const scalar_ptr cw = (scalar_ptr)(c + 64 * s);
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t y = ((ci2 ^ cw[w]) + 0x7fff7fffu) | (lo << (15 - w));
            const uint32_t z = ((ci2 ^ cw[16 + w]) + 0x7fff7fffu) | (hi << (15 - w));
            none += __builtin_popcount(y & 0x80008000u);
            none += __builtin_popcount(z & 0x80008000u);
        }
        a = an;
    }
    return i < n ? 64 * (s1 - s0) - none : 0;
}

__device__ __forceinline__ void conflict_block(const GraphDev* __restrict__ gd, int G, int b, int gsel, int* sh) {
    const int g = find_graph(gd, G, b, [](const GraphDev& x) { return x.cf_begin; });
    if (gsel >= 0 && g != gsel) return;
    const GraphDev& d = gd[g];
    const int words = d.cf_words;
    const bool masks = words != 0;
    const int parts = masks ? count_parts(d.n) : (d.n + 63) / 64;
    const int loc = b - d.cf_begin;
    const int m = loc / parts, part = loc - m * parts;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int f = masks ? count_masks(d, m, part, {words, words | 1}, sh) : count_compares(d, m, part);
    for (int o = 32; o >= 1; o >>= 1) f += __shfl_xor(f, o);
    // one add per block, spread over the member's slots (the fitness folds them): adds of every wave to the
    // members' counters, a few cache lines, took longer than the counting
    if (lane == 0) sh[wave] = f;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&d.f2p[(size_t)m * kF2Slots + (part & (kF2Slots - 1))], sh[0] + sh[1] + sh[2] + sh[3]);
}

// First launch of a merged iteration: everything that depends only on the colours, in blocks of
// several kinds: the members (class sizes, lists), the search for legal members, the group-concentration tiles with the
// penalty operand, the expansion of S^T, and (where they are asked for) the conflict counts.  As three launches of 4-5
// us each they were most of a small graph's iteration.  t stays as it is here (the launch that updates the weights
// advances it), so the tiles may read it; a pending non-finite update ends the graph (adv).
// Held to 64 registers (eight waves per SIMD, no spills; 95 without): the blocks of the later kinds start
// beside the tiles instead of after them (16 graphs, 10 iterations: 4608 -> 4538 us).  The search for legal members
// (contexts with a stop rule) and the counts (calls that report) are variants, since their code costs the tiles
// registers (eight iterations of n = 2000, k = 28, D = 20 without a stop rule: 341 us, 349 with the search in the same
// kernel); the search takes seven waves (n = 1000, k = 28, D = 128: 398.5 us for eight iterations, 401.7 at eight).
constexpr int kPhase1Plain = 0, kPhase1Legal = 1, kPhase1Count = 2;
template <int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KIND == kPhase1Legal ? 7 : 8))) void k_phase1(
    const GraphDev* __restrict__ gd, int G, int total_mem, int total_mt, int total_ex, int total_cf, int total_lg,
    int honor_stop, int adv, int want, int mt_flags, int gsel) {
    extern __shared__ __attribute__((aligned(16))) int p1_sh[];
    int b = blockIdx.x;
    if (b < total_mem) {
        member_block(gd, G, b, honor_stop, adv, want, p1_sh);
        return;
    }
    b -= total_mem;
    if constexpr (KIND == kPhase1Legal) {
        if (b < total_lg) {
            legal_block(gd, G, b, honor_stop, adv, want, p1_sh);
            return;
        }
        b -= total_lg;
    }
    if (b < total_mt) {
        mtilde_block(gd, G, b, honor_stop, mt_flags, gsel, nullptr, (uint8_t*)p1_sh, adv);
        return;
    }
    b -= total_mt;
    if (b < total_ex) {
        expand_block(gd, G, b, honor_stop, 0, 1, adv);
        return;
    }
    if constexpr (KIND == kPhase1Count) {
        b -= total_ex;
        if (b < total_cf) conflict_block(gd, G, b, gsel, p1_sh);
    }
}

// ------------------------------------------------------- step 2, stop rule -----

// One block per graph: f_color = f2 / 2 (f2 gathered from A.S); the main
// fitness f_color, or |E| - f_color for partitioning; the added fitness (f_eq, or
// the colour cost sum_l (l + 1) #V_l) as the class-size kernel left it; f = main + added;
// lowest legal member; stop rule.  Clears f2.  With kFlagReport only the fitness
// arrays are written.
__device__ __forceinline__ void fitness_graph(const GraphDev* __restrict__ gd, int g, int honor_stop, int flags, int* best_sh) {
    int& best = *best_sh;
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    const bool sparse_now = d.psparse && !st->pdense && pen_active(d, st);
    const int p = st->pS;
    if (threadIdx.x == 0) best = 0x7FFFFFFF;
    if (((flags & kFlagFoldSparse) && sparse_now) || (flags & kFlagFoldCounts)) {
        // the sparse rows of this iteration (or the conflict counts) gathered 2 f_color into slots: fold and clear them
        for (int m = threadIdx.x; m < d.D; m += blockDim.x) {
            int sum = 0;
            for (int sl = 0; sl < kF2Slots; ++sl) {
                sum += d.f2p[(size_t)m * kF2Slots + sl];
                d.f2p[(size_t)m * kF2Slots + sl] = 0;
            }
            d.f2[m] = sum;
        }
    }
    __syncthreads();
    // the added fitness (equity or colour cost) was reduced by the class-size kernel
    const bool added = prob_added(d.problem);
    for (int m = threadIdx.x; m < d.D; m += blockDim.x) {
        long long fc = d.f2[m] / 2;
        if (prob_partition(d.problem)) fc = (d.ones_dev ? (long long)(*d.ones_dev / 2) : d.edges) - fc;
        const long long fe = added ? d.feq[m] : 0;
        d.fcol[m] = fc;
        d.feq[m] = fe;
        d.f[m] = fc + fe;
        d.f2[m] = 0;
        if (fc + fe == 0) atomicMin(&best, m);
    }
    __syncthreads();
    if (flags & kFlagReport) return;
    if (threadIdx.x == 0) {
        // the route this iteration's penalty product took (the contraction and the sparse
        // rows read the same state)
        if (!pen_active(d, st)) st->it_nopen += 1;
        else if ((flags & kFlagPlainPen) || !d.psparse || st->pdense) st->it_dense += 1;
        else st->it_sparse += 1;
    }
    const int ld = best == 0x7FFFFFFF ? -1 : best;
    const bool stop = ld >= 0 && d.stop_on_legal;
    if (stop) {
        if (d.cmax > 1) {
            // multicolouring: the legal member's selection as [i][s]
            for (int e = threadIdx.x; e < d.n * d.cmax; e += blockDim.x) {
                const int i = e / d.cmax, sl = e - i * d.cmax;
                d.snap[e] = d.sel[((size_t)ld * d.cmax + sl) * d.cs + i];
            }
        } else {
            const int16_t* c = d.c[p] + (size_t)ld * d.cs;
            for (int i = threadIdx.x; i < d.n; i += blockDim.x) d.snap[i] = c[i];
        }
        if (threadIdx.x == 0) {
            st->legal_d = ld;
            st->stopped = 1;
        }
    }
    if ((flags & kFlagFlipFused) && d.pfuse && threadIdx.x == 0 && !stop) {
        // the sparse-rows launch wrote this iteration's update into the other buffers
        st->pW ^= 1;
        st->pS ^= 1;
    }
    if ((flags & kFlagFused) && threadIdx.x == 0 && !stop) {
        // fused path: the contraction kernel wrote the update into the other buffers
        st->pW ^= 1;
        st->pS ^= 1;
        st->t += 1;
        st->steps_done += 1;
        if (st->next_bad) {
            st->error = -5;
            st->stopped = 1;
        }
    }
}

__global__ __launch_bounds__(256) void k_fitness(const GraphDev* __restrict__ gd, int G, int honor_stop,
                                                 int flags, int gsel) {
    __shared__ int best;
    const int g = blockIdx.x;
    if (g >= G || (gsel >= 0 && g != gsel)) return;
    fitness_graph(gd, g, honor_stop, flags, &best);
}

// Separate-kernel path, step 4: softmax along k, straight-through gradient,
// update and smoothing (mode 0), or gradient output without update (mode 1,
// one graph).  16 lanes per row (d, i).
__global__ __launch_bounds__(256) void k_update(const GraphDev* __restrict__ gd, int G, int total_rows,
                                                int honor_stop, int mode, int gsel,
                                                float* __restrict__ gS_out, float* __restrict__ gW_out) {
    const int l16 = threadIdx.x & 15;
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
    if (row >= total_rows) return;
    const int g = graph_of_row(gd, G, row);
    if (gsel >= 0 && g != gsel) return;
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    const int r = row - d.row_begin;
    const int m = r / d.n;
    const int k = d.k;
    float* w = d.W[0] + (size_t)r * k;
    const float* gs = d.G + (size_t)r * k;
    const long long t = st->t;
    const float nut = prob_added(d.problem) ? d.nu * (float)t : 0.0f;
    const int prob = d.problem;
    const int32_t* V = d.V[st->pS] + (size_t)m * k;
    const float gam = d.momentum;
    float* vel = d.vel ? d.vel + (size_t)r * k : nullptr;
    float mx = -INFINITY;
    for (int l = l16; l < k; l += 16) mx = fmaxf(mx, w[l]);
    mx = row16_max(mx);
    float z = 0.0f, q = 0.0f;
    for (int l = l16; l < k; l += 16) {
        float e = exp_soft(w[l] - mx);
        float gv = gs[l];
        if (nut != 0.0f) gv += nut * added_grad(prob, V[l], l, d.c1, d.c2);
        z += e;
        q += e * gv;
    }
    z = row16_sum(z);
    q = row16_sum(q);
    const float rz = 1.0f / z;
    const float rr = q * rz;
    const bool smooth = d.nb_iter > 0 && ((t + 1) % d.nb_iter) == 0;
    for (int l = l16; l < k; l += 16) {
        float e = exp_soft(w[l] - mx) * rz;
        float gv = gs[l];
        if (nut != 0.0f) gv += nut * added_grad(prob, V[l], l, d.c1, d.c2);
        float gw = e * (gv - rr);
        if (mode == 0) {
            float step = gw;
            if (vel) {
                step = gam * vel[l] + gw;       // heavy-ball velocity
                vel[l] = step;
            }
            float nw = w[l] - d.eta * step;
            if (smooth) nw = nw / d.rho;
            w[l] = nw;
        } else {
            if (gS_out) gS_out[(size_t)r * k + l] = gv;
            if (gW_out) gW_out[(size_t)r * k + l] = gw;
        }
    }
}

// merged: the row belongs to a merged iteration (its t is st->tc, the stop rule is answered by the
// first launch, and the graph's first row also ends the iteration)
template <int KPL, int VAR>
__device__ __forceinline__ void update_row(const GraphDev* __restrict__ gd, int G, int row, int honor_stop, int mode,
                                           int gsel, float* __restrict__ gS_out, float* __restrict__ gW_out, int merged) {
    const int l16 = threadIdx.x & 15;
    int g = 0;
    if (merged) {
        while (g + 1 < G && (row < gd[g].ur_begin || row >= gd[g].ur_begin + gd[g].ur_rows)) ++g;
    } else {
        g = graph_of_row(gd, G, row);
    }
    if (gsel >= 0 && g != gsel) return;
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    // the fast path's sparse graphs take their row update in the sparse-rows launch
    if (mode == 0 && d.pfuse) return;
    const int r = row - (merged ? d.ur_begin : d.row_begin);
    const long long t = merged ? st->tc : st->t;
    if (merged) {
        bool stop = false;
        if ((VAR & 4) != 0 && d.cmax > 1) {
            // the contraction's gather has counted the conflicts
            int legal = 0;
            if (d.stop_on_legal)
                for (int x = l16; x < d.D; x += 16) legal |= d.f2[x] == 0;
            stop = row16_max_i(legal) != 0;
        } else {
            stop = merged_stop(d, st, t);
        }
        if (r == 0) merged_end(d, st, t, stop, l16, 16);
        if (stop) return;
    }
    const int k = d.k;
    const int m = r / d.n, i = r - m * d.n;
    float* w = d.W[0] + (size_t)r * k;
    const float* gs = d.G + (size_t)r * k;
    const RowCtx x = row_ctx(d, t);
    float* vel = d.vel ? d.vel + (size_t)r * k : nullptr;
    int16_t* __restrict__ cnext = d.c[st->pS] + (size_t)m * d.cs;
    RowRegs<KPL, VAR> R;
    float gv[KPL];
    RowClasses<KPL, VAR> C;
    row_load<KPL, VAR>(R, gv, x, w, gs, vel, mode, l16);
    classes_load<KPL, VAR>(C, x, d.V[st->pS] + (size_t)m * k, l16);
    const int c = row_step<KPL, VAR>(R, C, gv, x, w, vel, mode, gS_out ? gS_out + (size_t)r * k : nullptr,
                                     gW_out ? gW_out + (size_t)r * k : nullptr, l16);
    if constexpr ((VAR & 4) != 0) {
        if (mode == 0 && merged && d.cmax > 1 && c >= 0) {
            row_select<KPL>(d, R.wv, m, i, l16, cnext);
            return;
        }
    }
    if (mode == 0 && l16 == 0) {
        if (c < 0) atomicExch(&st->next_bad, 1);
        cnext[i] = (int16_t)max(c, 0);
    }
}

template <int KPL, int VAR>
__global__ __launch_bounds__(256) void k_update_rows(const GraphDev* __restrict__ gd, int G, int row0, int total_rows,
                                                     int honor_stop, int mode, int gsel, float* __restrict__ gS_out,
                                                     float* __restrict__ gW_out, int merged) {
    const int row = row0 + blockIdx.x * 16 + (threadIdx.x >> 4);
    if (row >= row0 + total_rows) return;
    update_row<KPL, VAR>(gd, G, row, honor_stop, mode, gsel, gS_out, gW_out, merged);
}

// ------------------------------------------------------------- class-row sums ----

// Steps 2-4 of a graph in fp32 operands, without a contraction: with one-hot S_d,
//   G[d, i, l] = sum_{j in class (d, l)} (a_ij + P_ij),
// so a wave takes 64 vertices i of member d (one per lane) and walks the member's vertices j
// grouped by colour: P is symmetric, so row j gives its 64 entries in one load, whose sign bits are the
// adjacency (mtilde_tile).  n^2 D additions instead of the contraction's n^2 D k multiply-adds at
// the 157 TFLOP/s of the fp32 matrix instructions (rows_preferred says where the additions win).  The counts
// come first, exactly, then the P_ij in FP32 one after the other in the order of the member's list, which is
// the order of the fp32 contraction's accumulation: the same bits.  The list holds row offsets, read into scalar
// registers, and each class is padded to a multiple of four with a row of zeros, so an entry costs one
// load, two instructions to count and one to add; the next class is loaded while one is summed.  The block's
// eight waves share the colours by eighths of the work; the 64 gradient rows meet in LDS and the same block takes the
// row update (or writes the gradients).
// With all vertices in one class (n = 1000, k = 85, D = 48) an iteration takes 82 us, 172 before a wave's walks of a
// long class were pipelined and the block counted a large one together.
// n = 500, k = 50, D = 64: 16 us per launch against 44 us (contraction) + 8 us (row update) before, n = 125, k = 18,
// D = 8 7.6 against 16 + 3.7 us; gradients at n = 1000, k = 85, D = 48 36 against 162 + 11 us.  (A first form, with the
// adjacency from bit masks and lists in LDS, two walks and a check per entry, took 26, 10.6 and 49 us.)
//
// mode 0: step (merged iteration); 1: gS / gW of graph gsel and 2 f_color.
constexpr int kCrThreads = 512;
// entries of a class's list beyond which its walks are pipelined through the list, and beyond which, when that is half
// as much again as a wave's share, the block counts it together (a class within the share is counted by its wave, whose
// sum then finds its rows in the caches: n = 8000, k = 14, D = 4 367 us an iteration against 459); and the entries that
// walking a class costs by itself
constexpr int kCrLong = 144, kCrLarge = 256, kCrClass = 16;
template <int KPL, int VAR>
__global__ __launch_bounds__(kCrThreads) __attribute__((amdgpu_waves_per_eu(KPL <= 8 ? 4 : 2))) void k_class_rows(
    const GraphDev* __restrict__ gd, int G, int total_blocks, int honor_stop, int mode, int gsel,
    float* __restrict__ gS_out, float* __restrict__ gW_out) {
    extern __shared__ __attribute__((aligned(16))) uint8_t cr_sh[];
    constexpr int NW = kCrThreads / 64;
    if ((int)blockIdx.x >= total_blocks) return;
    // where P is larger than an XCD's L2 each XCD takes a contiguous range of strips (n = 1000, D = 48: 41 -> 36.5 us;
    // at n = 500 the hardware's order is 3 % faster)
    const int b = G == 1 && gd[0].n_pad >= 1024 ? xcd_remap(blockIdx.x, total_blocks) : (int)blockIdx.x;
    const int g = find_graph(gd, G, b, [](const GraphDev& x) { return x.cr_begin; });
    if (gsel >= 0 && g != gsel) return;
    const GraphDev& d = gd[g];
    GraphState* st = d.st;
    if (honor_stop && st->stopped) return;
    const long long t = st->tc;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (mode == 0) {
        const bool stop = merged_stop(d, st, t);
        if (b == d.cr_begin && tid < 64) merged_end(d, st, t, stop, tid, 64);
        if (stop) return;
    }
    const int n = d.n, k = d.k, D = d.D;
    const int loc = b - d.cr_begin;
    const int strip = loc / D, m = loc - strip * D;      // the members of a strip are neighbours: they share P's columns in L2
    const int KS = k | 1;                                // odd row stride: the lanes of a column on different banks
    int* fsum = (int*)cr_sh;                             // [NW]
    float* Gt = (float*)(cr_sh + 64);                    // [64][KS]
    const float tf = (float)t;
    const bool pen = (d.lambda * tf != 0.0f) || (d.mu * tf != 0.0f);
    const uint32_t sign = prob_partition(d.problem) ? 0x80000000u : 0u;
    // the row update's rows: 16 lanes each, two rows per group of lanes; where they fit in registers
    // their loads go out now, behind the sums (at KPL = 4 they spill: n = 500, k = 50, D = 64 211 us for eight
    // iterations, 204.5 without)
    constexpr bool AHEAD = KPL <= 2 && VAR == 0;
    const RowCtx x = row_ctx(d, t);
    const int l16 = tid & 15, g16 = tid >> 4;
    constexpr int NG = kCrThreads / 16, NR = 64 / NG;
    const int32_t* V = d.V[st->pS] + (size_t)m * k;
    int16_t* __restrict__ cnext = d.c[st->pS] + (size_t)m * d.cs;
    const size_t ro0 = ((size_t)m * n + strip * 64 + g16) * k;
    RowRegs<KPL, VAR> ahead[AHEAD ? NR : 1];
    if constexpr (AHEAD) {
        float none[KPL];
#pragma unroll
        for (int u = 0; u < NR; ++u)
            if (strip * 64 + g16 + NG * u < n)
                row_load<KPL, VAR>(ahead[u], none, x, d.W[0] + ro0 + (size_t)NG * u * k, nullptr,
                                   d.vel ? d.vel + ro0 + (size_t)NG * u * k : nullptr, mode, l16);
    }
    // the member's list (scalar loads: written by the launch before)
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
    const int32_t* __restrict__ co = d.cls_off + (size_t)m * (k + 1);
    const scalar_ptr off = (scalar_ptr)co;
    const scalar_ptr lst = (scalar_ptr)(d.cls_j + (size_t)m * d.js);
    const char* __restrict__ Pc = (const char*)d.Pop + (size_t)strip * 256;
    // this wave's colours: those with their middle in its eighth of the work (the entries of the lists, and for each
    // class what kCrClass entries cost); and whether some class is large
    int l0 = 0, l1 = 0;
    bool large = false;
    const int large_from = max(kCrLarge, 3 * (int)off[k] / (2 * NW));
    {
        const int T = (int)off[k] + kCrClass * k;
        for (int lb = 0; lb < k; lb += 64) {
            const int l = lb + lane;
            const int o0 = gview(co)[min(l, k)] & ~3, o1 = gview(co)[min(l + 1, k)] & ~3;
            const int o = l < k ? NW / 2 * (o0 + o1 + kCrClass * (2 * l + 1)) : 1 << 30;
            l0 += __popcll(__ballot(o < wave * T));
            l1 += __popcll(__ballot(o < (wave + 1) * T));
            large |= __any(o1 - o0 > large_from);
        }
        l0 = __builtin_amdgcn_readfirstlane(l0);
        l1 = __builtin_amdgcn_readfirstlane(l1);
    }
    const int i = strip * 64 + lane;
    const int own_c = mode != 0 && i < n ? (int)gview(cnext)[i] : -1;
    int own = 0;
    float* __restrict__ Gl = Gt + lane * KS;
    // up to 16 entries of the list, in groups of four: loads, count of edges (entries whose sign is clear), sum in
    // order
    auto load = [&](float (&v)[16], int p, int ng) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < ng) {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[4 * q + u] = gview((const float*)(Pc + lst[p + 4 * q + u]))[lane];
            }
    };
    auto edges = [&](const float (&v)[16], int ng, int c) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < ng) {
#pragma unroll
                for (int u = 0; u < 4; ++u) c += __float_as_int(v[4 * q + u]) >= 0 ? 1 : 0;
            }
        return c;
    };
    auto add = [&](const float (&v)[16], int ng, float acc) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < ng) {
#pragma unroll
                for (int u = 0; u < 4; ++u) acc += v[4 * q + u];
            }
        return acc;
    };
    // the same 16 loads in a long class, whose list entries come 64 at a time, a lane each, ahead of their use (lv:
    // those from the walk's position on; past its end the row of zeros, which stays in the caches).  Without
    // conditions, so that a wait for one piece leaves the next in flight
    const uint32_t* __restrict__ cj = d.cls_j + (size_t)m * d.js;
    const uint32_t zero_row = 4u * (uint32_t)d.n_pad * (uint32_t)d.n_pad;
    auto entries = [&](int q, int e) {
        const uint32_t x = gview(cj)[min(q + lane, e - 1)];
        return q + lane < e ? x : zero_row;
    };
    auto load_at = [&](float (&v)[16], uint32_t lv, int at) {
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v[u] = gview((const float*)(Pc + (uint32_t)__builtin_amdgcn_readlane((int)lv, at + u)))[lane];
    };
    auto groups = [](int entries) { return max(0, min(4, entries >> 2)); };
    // edges of the entries [p, e), by this wave
    auto count_walk = [&](int p, int e) {
        float v[16], w[16];
        int c = 0;
        if (p >= e) return c;
        uint32_t lv = entries(p, e);
        load_at(v, lv, 0);
        for (int q = p; q < e; q += 64) {
            const uint32_t next = entries(q + 64, e);
            load_at(w, lv, 16);
            c = edges(v, groups(e - q), c);
            load_at(v, lv, 32);
            c = edges(w, groups(e - q - 16), c);
            load_at(w, lv, 48);
            c = edges(v, groups(e - q - 32), c);
            load_at(v, next, 0);
            c = edges(w, groups(e - q - 48), c);
            lv = next;
        }
        return c;
    };
    if (large) {
        // the block's waves count a large class together, a piece each, into its place among the gradient rows
        auto each_large = [&](auto f) {
            for (int lb = 0; lb < k; lb += 64) {
                const int l = lb + lane;
                unsigned long long b = __ballot((gview(co)[min(l + 1, k)] & ~3) - (gview(co)[min(l, k)] & ~3) > large_from);
                for (; b; b &= b - 1) f(lb + __builtin_ctzll(b));
            }
        };
        if (wave == 0) each_large([&](int l) { ((int*)Gl)[l] = 0; });
        __syncthreads();
        each_large([&](int l) {
            const int p = (int)off[l] & ~3, e = (int)off[l + 1] & ~3;
            const int piece = ((e - p) / 4 + NW - 1) / NW * 4;
            const int q = p + wave * piece;
            atomicAdd((int*)Gl + l, count_walk(min(q, e), min(q + piece, e)));
        });
        __syncthreads();
    }
    // class l in v (its first 16 entries), entries [p, e), of which the last `pads` are padding (counted as edges
    // by their sign, so taken off)
    auto finish = [&](float (&v)[16], int l, int p, int e, int pads) {
        if (e - p > kCrLong) {
            const int c = (e - p > large_from ? ((const int*)Gl)[l] : count_walk(p, e)) - pads;
            if (mode != 0 && own_c == l) own = c;
            float acc = (float)c;
            if (pen) {
                float w[16];
                uint32_t lv = entries(p, e);
                for (int q = p; q < e; q += 64) {
                    const uint32_t next = entries(q + 64, e);
                    load_at(w, lv, 16);
                    acc = add(v, groups(e - q), acc);
                    load_at(v, lv, 32);
                    acc = add(w, groups(e - q - 16), acc);
                    load_at(w, lv, 48);
                    acc = add(v, groups(e - q - 32), acc);
                    load_at(v, next, 0);
                    acc = add(w, groups(e - q - 48), acc);
                    lv = next;
                }
            }
            Gl[l] = acc;
            return;
        }
        int c = edges(v, min(4, (e - p) >> 2), -pads);
        if (e - p <= 16) {
            if (mode != 0 && own_c == l) own = c;
            Gl[l] = pen ? add(v, (e - p) >> 2, (float)c) : (float)c;
            return;
        }
        // both walks two pieces deep
        float w[16];
        for (int q = p + 16; q < e; q += 32) {
            load(v, q, min(4, (e - q) >> 2));
            const int n2 = q + 16 < e ? min(4, (e - q - 16) >> 2) : 0;
            load(w, q + 16, n2);
            c = edges(v, min(4, (e - q) >> 2), c);
            c = edges(w, n2, c);
        }
        if (mode != 0 && own_c == l) own = c;
        float acc = (float)c;
        if (pen) {
            load(v, p, 4);
            for (int q = p; q < e; q += 32) {
                const int n2 = q + 16 < e ? min(4, (e - q - 16) >> 2) : 0;
                load(w, q + 16, n2);
                acc = add(v, min(4, (e - q) >> 2), acc);
                if (q + 32 < e) load(v, q + 32, min(4, (e - q - 32) >> 2));
                acc = add(w, n2, acc);
            }
        }
        Gl[l] = acc;
    };
    if (l0 < l1) {
        float va[16], vb[16];
        int ra = (int)off[l0], rb = (int)off[l0 + 1];
        load(va, ra & ~3, min(4, ((rb & ~3) - (ra & ~3)) >> 2));
        for (int l = l0; l < l1; l += 2) {
            const int rc = l + 1 < l1 ? (int)off[l + 2] : rb;
            if (l + 1 < l1) load(vb, rb & ~3, min(4, ((rc & ~3) - (rb & ~3)) >> 2));
            finish(va, l, ra & ~3, rb & ~3, ra & 3);
            if (l + 1 >= l1) break;
            const int rd = l + 2 < l1 ? (int)off[l + 3] : rc;
            if (l + 2 < l1) load(va, rc & ~3, min(4, ((rd & ~3) - (rc & ~3)) >> 2));
            finish(vb, l + 1, rb & ~3, rc & ~3, rb & 3);
            ra = rc;
            rb = rd;
        }
    }
    if (mode != 0) {
        // 2 f_color: the counts at the vertices' own colours
        for (int o = 32; o >= 1; o >>= 1) own += __shfl_xor(own, o);
        if (lane == 0) fsum[wave] = own;
    }
    __syncthreads();
    if (mode != 0 && tid == 0) {
        int f = 0;
        for (int w = 0; w < NW; ++w) f += fsum[w];
        atomicAdd(&d.f2p[(size_t)m * kF2Slots + (strip & (kF2Slots - 1))], f);
    }
    // row update, 16 lanes per row
    RowClasses<KPL, VAR> C;
    classes_load<KPL, VAR>(C, x, V, l16);
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        const int rr = g16 + NG * u;
        const int iv = strip * 64 + rr;
        if (iv >= n) break;
        float* w = d.W[0] + ro0 + (size_t)NG * u * k;
        float* vel = d.vel ? d.vel + ro0 + (size_t)NG * u * k : nullptr;
        RowRegs<KPL, VAR> R;
        float gv[KPL];
        if constexpr (AHEAD) {
            R = ahead[u];
        } else {
            row_load<KPL, VAR>(R, gv, x, w, nullptr, vel, mode, l16);
        }
#pragma unroll
        for (int q = 0; q < KPL; ++q)
            if (16 * q < k) gv[q] = flip_sign(Gt[rr * KS + min(l16 + 16 * q, k - 1)], sign);
        const size_t ro = ro0 + (size_t)NG * u * k;
        const int c = row_step<KPL, VAR>(R, C, gv, x, w, vel, mode, gS_out ? gS_out + ro : nullptr,
                                         gW_out ? gW_out + ro : nullptr, l16);
        if (mode == 0 && l16 == 0) {
            if (c < 0) atomicExch(&st->next_bad, 1);
            cnext[iv] = (int16_t)max(c, 0);
        }
    }
}

// t <- t + 1 for every graph still running.
__global__ void k_advance(const GraphDev* __restrict__ gd, int G) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    advance_graph(gd[g].st);
}

// Fitness report of every graph (one block each), then (unless out is null) graph g's FP64 loss: L = sum main fitness +
// nu t sum added fitness + lambda t kappa - mu t varpi (kappa, varpi from the group-concentration kernel's partials).
// fold: kFlagFoldCounts where the conflicts are in the slots, else 0.
__global__ __launch_bounds__(256) void k_loss(const GraphDev* __restrict__ gd, int G, int g, int ntiles, int fold,
                                              double* __restrict__ out) {
    __shared__ double red[4][256];
    __shared__ int best;
    fitness_graph(gd, blockIdx.x, 0, kFlagReport | fold, &best);
    if ((int)blockIdx.x != g || !out) return;
    __syncthreads();
    const GraphDev& d = gd[g];
    double ka = 0, vb = 0, sf = 0, se = 0;
    for (int u = threadIdx.x; u < ntiles; u += 256) {
        ka += d.part[2 * u];
        vb += d.part[2 * u + 1];
    }
    for (int m = threadIdx.x; m < d.D; m += 256) {
        sf += (double)d.fcol[m];
        se += (double)d.feq[m];
    }
    red[0][threadIdx.x] = ka; red[1][threadIdx.x] = vb;
    red[2][threadIdx.x] = sf; red[3][threadIdx.x] = se;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (threadIdx.x < s)
            for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double t = (double)d.st->t;
        const double eq = prob_added(d.problem) ? red[3][0] : 0.0;
        out[0] = red[2][0] + (double)d.nu * t * eq + (double)d.lambda * t * red[0][0] - (double)d.mu * t * red[1][0];
        out[1] = red[2][0];
        out[2] = eq;
        out[3] = red[0][0];
        out[4] = red[1][0];
    }
}

// Report of one graph for tcol_conflicts: the first G blocks take the fitness of a graph each (kFlagReport; fold as in
// k_loss), graph g's copies it out, the others copy its colours.
__global__ __launch_bounds__(256) void k_report(const GraphDev* __restrict__ gd, int G, int g, int fold, int16_t* colors,
                                                int64_t* fcol, int64_t* feq) {
    __shared__ int best;
    const GraphDev& d = gd[g];
    if ((int)blockIdx.x < G) {
        fitness_graph(gd, blockIdx.x, 0, kFlagReport | fold, &best);
        if ((int)blockIdx.x != g) return;
        __syncthreads();
        for (int m = threadIdx.x; m < d.D; m += 256) {
            if (fcol) fcol[m] = d.fcol[m];
            if (feq) feq[m] = d.feq[m];
        }
        return;
    }
    if (!colors) return;
    const int16_t* __restrict__ c = d.c[d.st->pS];
    const size_t total = (size_t)d.D * d.n, step = (size_t)(gridDim.x - G) * 256;
    for (size_t e = (size_t)(blockIdx.x - G) * 256 + threadIdx.x; e < total; e += step) {
        const size_t m = e / d.n;
        colors[e] = c[m * d.cs + (e - m * d.n)];
    }
}

// graph g's selection as [d][i][s]: the cmax colours of each vertex (slot 0 the argmax, -1 past
// the demand), or the argmax colouring when cmax = 1
__global__ void k_copy_selection(const GraphDev* __restrict__ gd, int g, int16_t* __restrict__ out) {
    const GraphDev& d = gd[g];
    const int CM = d.cmax, n = d.n;
    const int16_t* c = d.c[d.st->pS];
    const size_t total = (size_t)d.D * n * CM;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t mi = e / CM;
        const int sl = (int)(e - mi * CM);
        const size_t m = mi / n, i = mi - m * n;
        out[e] = CM > 1 ? d.sel[((size_t)m * CM + sl) * d.cs + i] : c[m * d.cs + i];
    }
}

__global__ void k_state(const GraphDev* __restrict__ gd, int G, int op, int g_only, long long t) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G || (g_only >= 0 && g != g_only)) return;
    GraphState* st = gd[g].st;
    if (op == 0) {            // reset run state (keeps t and the route counters)
        st->stopped = 0; st->error = 0; st->legal_d = -1; st->steps_done = 0; st->next_bad = 0;
        st->prep_ticket = 0;
        st->legal_min[0] = st->legal_min[1] = 0x7FFFFFFF;
    } else if (op == 1) {     // set t
        st->t = t;
        st->legal_min[0] = st->legal_min[1] = 0x7FFFFFFF;
    } else if (op == 2) {     // clear steps counter only
        st->steps_done = 0; st->legal_d = -1;
    } else if (op == 3) {     // the caller's buffer holds the weights again
        st->pW = 0;
    } else if (op == 4) {     // clear the conflict accumulators (after timing repeated contractions)
        for (int m = 0; m < gd[g].D; ++m) gd[g].f2[m] = 0;
    } else if (op == 5) {     // the sparse rows' route for this iteration (timing of its contraction form)
        st->pdense = 0;
    }
}

// ------------------------------------------------------------ initial weights -

// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC'11), from its published round
// function and constants: ten rounds of two 32x32->64 multiplies, with the key
// bumped by the Weyl constants between rounds.
__device__ inline void philox4x32_10(uint32_t (&x)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)x[0] * 0xD2511F53ull;
        const uint64_t p1 = (uint64_t)x[2] * 0xCD9E8D57ull;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ x[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ x[3] ^ k1;
        x[0] = n0;
        x[1] = (uint32_t)p1;
        x[2] = n2;
        x[3] = (uint32_t)p0;
    }
}

// two 32-bit words to a uniform in (0, 1] with 53 bits
__device__ inline double uniform53(uint32_t hi, uint32_t lo) {
    return ((double)(hi >> 5) * 67108864.0 + (double)(lo >> 6) + 1.0) * (1.0 / 9007199254740992.0);
}

// W[e] ~ N(0, sigma0^2), e < count: counter block b = (b mod 2^32, b / 2^32, stream 1, 0)
// under key = seed gives two uniforms (u1, u2) and, by Box-Muller in FP64, the normals
// r cos(2 pi u2) and r sin(2 pi u2), r = sqrt(-2 ln u1), for entries 2b and 2b+1,
// scaled by sigma0 and rounded to fp32.  One thread per block b.
__global__ __launch_bounds__(256) void k_init_weights(float* __restrict__ W, long long count, uint32_t key0,
                                                      uint32_t key1, double sigma0) {
    const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (2 * b >= count) return;
    uint32_t x[4] = {(uint32_t)b, (uint32_t)((unsigned long long)b >> 32), 1u, 0u};
    philox4x32_10(x, key0, key1);
    const double u1 = uniform53(x[0], x[1]), u2 = uniform53(x[2], x[3]);
    const double r = sqrt(-2.0 * log(u1));
    const double th = 6.283185307179586 * u2;
    // one range reduction for both (the same values as cos and sin by themselves): 36 M weights 165 -> 137 us
    double sn, cn;
    sincos(th, &sn, &cn);
    W[2 * b] = (float)(r * cn * sigma0);
    if (2 * b + 1 < count) W[2 * b + 1] = (float)(r * sn * sigma0);
}

// ------------------------------------------------ class-conflict matrix ---------

// C_d = S_d^T (A.S_d) for one graph: row l of C_d is the sum of the rows of A.S_d (the contraction's G,
// [D][n][k]) of the vertices of colour l.  A block takes 16 columns of member d and up to kCcRows
// colours l, whose sums it holds in LDS: each 16 lanes of it read rows of G (one column per lane, eight rows in
// flight) and add them to the row of the vertex's colour.  The integers are exact in FP32 and in
// int32.  G is read once per kCcRows colours, so its bytes bound the kernel: n = 2999, k = 211, D = 25 196 us
// (a product with the one-hot S_d on fp32 matrix instructions, one row tile at a time) -> 33 us.
// out is [D][k][k] int32.
constexpr int kCcRows = 2048, kCcThreads = 1024;

__global__ __launch_bounds__(kCcThreads) void k_class_conflicts(const GraphDev* __restrict__ gd, int g, int row_blocks,
                                                                int32_t* __restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) int cc_sh[];     // [rows][16]
    const GraphDev& d = gd[g];
    const int k = d.k, n = d.n;
    const int cols = (k + 15) / 16;
    int b = blockIdx.x;
    const int rb = b % row_blocks;
    b /= row_blocks;
    const int dm = b / cols, c0 = (b - dm * cols) * 16;
    const int l0 = rb * kCcRows, rows = min(kCcRows, k - l0);
    const int l16 = threadIdx.x & 15, grp = threadIdx.x >> 4;
    constexpr int NG = kCcThreads / 16, U = 8;
    for (int e = threadIdx.x; e < rows * 16; e += kCcThreads) cc_sh[e] = 0;
    __syncthreads();
    const int16_t* __restrict__ col = d.c[d.st->pS] + (size_t)dm * d.cs;
    const bool in = c0 + l16 < k;
    const float* __restrict__ Gd = d.G + (size_t)dm * n * k + (in ? c0 + l16 : 0);
    for (int i0 = grp; i0 < n; i0 += NG * U) {
        float x[U];
        int l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + NG * u, n - 1);
            x[u] = gview(Gd)[(size_t)i * k];
            l[u] = (int)gview(col)[i] - l0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + NG * u < n && in && l[u] >= 0 && l[u] < rows) atomicAdd(&cc_sh[l[u] * 16 + l16], (int)x[u]);
    }
    __syncthreads();
    // G holds -A.S for partitioning
    const int sg = prob_partition(d.problem) ? -1 : 1;
    if (!in) return;
    for (int l = grp; l < rows; l += NG) out[((size_t)dm * k + l0 + l) * k + c0 + l16] = sg * cc_sh[l * 16 + l16];
}

// ------------------------------------------- descriptors from kernel arguments --

// Writes one graph's descriptor and a fresh state (the values travel as kernel arguments,
// so a captured launch carries them; no host buffer has to outlive the call).
// The conflict counts and the number of ones of A, which the call's kernels add to, start at zero.
__global__ void k_put_desc(GraphDev d, GraphDev* __restrict__ gd, GraphState* __restrict__ st,
                           unsigned long long* __restrict__ ones) {
    for (int e = threadIdx.x; e < d.D * kF2Slots; e += blockDim.x) d.f2p[e] = 0;
    if (threadIdx.x != 0) return;
    *ones = 0ull;
    *gd = d;
    GraphState s{};
    s.legal_d = -1;
    *st = s;
}

// p[0 .. words) = 0 (16-byte stores; p 16-byte aligned)
__global__ __launch_bounds__(256) void k_zero16(uint4* __restrict__ p, size_t words) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < words; e += (size_t)gridDim.x * blockDim.x)
        p[e] = make_uint4(0u, 0u, 0u, 0u);
}

// ------------------------------------------------------------- launchers -----

#define TCOL_LAUNCH_CHECK() do { hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return e_; } while (0)

hipError_t launch_init_weights(float* W, long long count, unsigned long long seed, double sigma0, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const long long blocks = ((count + 1) / 2 + 255) / 256;
    hipLaunchKernelGGL(k_init_weights, dim3((unsigned)blocks), dim3(256), 0, s, W, count, (uint32_t)seed,
                       (uint32_t)(seed >> 32), sigma0);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_pack_graph(const uint8_t* A, int n, int n_pad, int op, uint8_t* A8, unsigned long long* Ab, void* Aop,
                             int* bad, unsigned long long* ones, hipStream_t s) {
    const int T = n_pad / 64;
    hipLaunchKernelGGL(k_pack_graph, dim3(T * T), dim3(256), 0, s, A, n, n_pad, op, A8, Ab, Aop, bad, ones);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_colors(const GraphDev* gd, int G, int total_rows, int honor_stop, hipStream_t s) {
    if (total_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_colors, dim3(ceil_div(total_rows, 16)), dim3(256), 0, s, gd, G, total_rows, honor_stop);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

size_t prep_lds(int kmax, int nmax, int lists) {
    size_t b = sizeof(int) * ((size_t)kPrepScratch + (size_t)kmax);
    if (lists) b += sizeof(int) * 5 * (size_t)kmax + sizeof(int16_t) * (size_t)nmax;
    return (b + 15) / 16 * 16;
}

hipError_t launch_prep(const GraphDev* gd, int G, int total_mem, size_t lds, int honor_stop, int next, int decide,
                       int ex_blocks, int advance_prev, hipStream_t s) {
    if (total_mem <= 0) return hipSuccess;
    if (lds > 150 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prep, dim3(total_mem + ex_blocks), dim3(256), lds, s, gd, G, total_mem, honor_stop, next,
                       decide, ex_blocks, advance_prev);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

// instantiations of the sparse rows: KW = 0 (no row update), or the row update's values per lane
// (k <= 64 KW) for graphs whose update rides on the launch, with (ADD = 1) or without the added
// fitness term (the equity or colour-cost gradient, whose class-size loads take registers)
#define TCOL_PS_KERNELS(X) \
    X(256, 0, 0) X(512, 0, 0) X(1024, 0, 0) \
    X(512, 2, 0) X(512, 3, 0) X(512, 5, 0) X(512, 7, 0) X(512, 9, 0) \
    X(512, 2, 1) X(512, 3, 1) X(512, 5, 1) X(512, 7, 1) X(512, 9, 1) \
    X(1024, 2, 0) X(1024, 3, 0) X(1024, 5, 0) X(1024, 7, 0) X(1024, 9, 0) \
    X(1024, 2, 1) X(1024, 3, 1) X(1024, 5, 1) X(1024, 7, 1) X(1024, 9, 1)

int penalty_sparse_kw(int kmax) {
    for (int kw : {2, 3, 5, 7, 9})
        if (64 * kw >= kmax) return kw;
    return -1;
}

hipError_t penalty_sparse_prepare() {
#define TCOL_PS_ATTR(NT, KW, ADD)                                                                            \
    {                                                                                                        \
        const hipError_t e = hipFuncSetAttribute((const void*)k_pen_sparse<NT, KW, ADD>,                     \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);    \
        if (e != hipSuccess) return e;                                                                       \
    }
    TCOL_PS_KERNELS(TCOL_PS_ATTR)
#undef TCOL_PS_ATTR
    // k_prep also holds 1 KB of static LDS
    return hipFuncSetAttribute((const void*)k_prep, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
}

size_t penalty_sparse_lds(int PM, int kmax, int dmax, int nmax) {
    const size_t n_pad = (size_t)round_up(nmax, kPadN);
    const size_t acc = 8 * (size_t)PM * (size_t)kmax;
    const size_t work = acc > 4 * n_pad ? acc : 4 * n_pad;
    const size_t b = 8 * ps_tab_words(dmax) + 2 * 4 * ps_int_words(dmax) + 16 + 2 * (size_t)round_up(dmax, 8) +
                     4 * n_pad + work;
    return (b + 15) / 16 * 16;
}

hipError_t launch_penalty_sparse(const GraphDev* gd, int G, int blocks, int PM, int threads, int kw, int add,
                                 size_t lds, int honor_stop, int accumulate, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    const int grid = blocks;
    if (PM != 8 || lds > 160 * 1024) return hipErrorInvalidValue;
    // the fused row update takes one wave per member of a group
    if (kw > 0 && PM > threads / 64) return hipErrorInvalidValue;
    bool done = false;
    if (kw == 0) add = 0;
#define TCOL_PS_LAUNCH(NT, KW, ADD)                                                                         \
    if (!done && threads == NT && kw == KW && add == ADD) {                                                 \
        k_pen_sparse<NT, KW, ADD><<<grid, NT, lds, s>>>(gd, G, blocks, honor_stop, PM, accumulate);         \
        done = true;                                                                                        \
    }
    TCOL_PS_KERNELS(TCOL_PS_LAUNCH)
#undef TCOL_PS_LAUNCH
    if (!done) return hipErrorInvalidValue;
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_expand(const GraphDev* gd, int G, int total_blocks, int honor_stop, int next, int gate,
                         hipStream_t s) {
    if (total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand, dim3(total_blocks), dim3(256), 0, s, gd, G, total_blocks, honor_stop, next, gate);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_mtilde(const GraphDev* gd, int G, int total_tiles, int honor_stop, int flags, int gsel,
                         int32_t* mt_out, hipStream_t s) {
    if (total_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mtilde, dim3(total_tiles), dim3(256), 0, s, gd, G, total_tiles, honor_stop, flags, gsel,
                       mt_out);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_fitness(const GraphDev* gd, int G, int honor_stop, int flags, int gsel, hipStream_t s) {
    hipLaunchKernelGGL(k_fitness, dim3(G), dim3(256), 0, s, gd, G, honor_stop, flags, gsel);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_update(const GraphDev* gd, int G, int total_rows, int honor_stop, int mode, int gsel,
                         float* gS_out, float* gW_out, hipStream_t s) {
    if (total_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_update, dim3(ceil_div(total_rows, 16)), dim3(256), 0, s, gd, G, total_rows, honor_stop,
                       mode, gsel, gS_out, gW_out);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

int update_rows_kpl(int kmax) {
    const int need = (kmax + 15) / 16;
    for (int kpl : {2, 4, 6, 8, 12, 18, 24, 36})
        if (kpl >= need) return kpl;
    return 0;
}

hipError_t launch_update_rows(const GraphDev* gd, int G, int row0, int total_rows, int kmax, int var, int honor_stop, int mode,
                              int gsel, float* gS_out, float* gW_out, int merged, hipStream_t s) {
    if (total_rows <= 0) return hipSuccess;
    if (var < 0 || var > 7) return hipErrorInvalidValue;
    if (var & 4) var |= 1;   // the multicolouring variants carry the added fitness term too
    const dim3 grid(ceil_div(total_rows, 16)), blk(256);
#define TCOL_UR(KP)                                                                                                  \
    switch (var) {                                                                                                   \
        case 0: hipLaunchKernelGGL((k_update_rows<KP, 0>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break;                                                           \
        case 1: hipLaunchKernelGGL((k_update_rows<KP, 1>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break;                                                           \
        case 2: hipLaunchKernelGGL((k_update_rows<KP, 2>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break;                                                           \
        case 3: hipLaunchKernelGGL((k_update_rows<KP, 3>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break; \
        case 5: hipLaunchKernelGGL((k_update_rows<KP, 5>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break; \
        default: hipLaunchKernelGGL((k_update_rows<KP, 7>), grid, blk, 0, s, gd, G, row0, total_rows, honor_stop, mode, gsel, \
                                   gS_out, gW_out, merged); break; \
    }
    switch (update_rows_kpl(kmax)) {
        case 2: TCOL_UR(2) break;
        case 4: TCOL_UR(4) break;
        case 6: TCOL_UR(6) break;
        case 8: TCOL_UR(8) break;
        case 12: TCOL_UR(12) break;
        case 18: TCOL_UR(18) break;
        case 24: TCOL_UR(24) break;
        case 36: TCOL_UR(36) break;
        default: return hipErrorInvalidValue;
    }
#undef TCOL_UR
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

size_t phase1_lds(int kmax, int nmax, int lists) {
    // without lists only the scratch and the counts are used
    size_t b = lists ? member_lds_bytes(kmax, nmax) : sizeof(int) * ((size_t)kPrepScratch + kmax);
    if (b < (size_t)kMtLds) b = kMtLds;
    if (b < scan_lds_bytes(nmax, kmax)) b = scan_lds_bytes(nmax, kmax);
    return (b + 15) / 16 * 16;
}

hipError_t phase1_prepare() {
    for (const void* f : {(const void*)k_phase1<kPhase1Plain>, (const void*)k_phase1<kPhase1Legal>,
                          (const void*)k_phase1<kPhase1Count>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxBlockLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Blocks per member of the search for legal members: 1024 vertices each (n = 1000: one block's search to the end takes
// about 6 us, less than the tiles of the same launch), 256, a strip a wave, where the masks take several pieces, each of
// which waits for its loads (eight iterations with members one conflict from legal, D = 8, fp4: n = 1000, k = 300
// 366 -> 322 us, 314 without the stop rule; n = 2000, k = 300 653 -> 590, 576).
int search_parts(int n, int k) { return ceil_div(n, scan_shape(n, k).words < ceil_div(n, 64) ? 256 : 1024); }

int conflict_words(int D, int n, int k) {
    const ScanShape ss = scan_shape(n, k);
    return count_by_masks(n, D, ss) ? ss.words : 0;
}

hipError_t launch_phase1(const GraphDev* gd, int G, int total_mem, int total_mt, int total_ex, int total_cf, int total_lg,
                         size_t lds, int honor_stop, int adv, int want, int mt_flags, int gsel, hipStream_t s) {
    // no sequence both searches and counts
    if (lds > (size_t)kMaxBlockLds || (total_lg > 0 && total_cf > 0)) return hipErrorInvalidValue;
    const dim3 grid(total_mem + total_lg + total_mt + total_ex + total_cf), blk(256);
#define TCOL_P1(KIND) \
    hipLaunchKernelGGL(k_phase1<KIND>, grid, blk, lds, s, gd, G, total_mem, total_mt, total_ex, total_cf, total_lg, \
                       honor_stop, adv, want, mt_flags, gsel)
    if (total_lg > 0) TCOL_P1(kPhase1Legal);
    else if (total_cf > 0) TCOL_P1(kPhase1Count);
    else TCOL_P1(kPhase1Plain);
#undef TCOL_P1
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

size_t class_rows_lds(int k) { return 64 + ((size_t)64 * (k | 1) * 4 + 15) / 16 * 16; }

#define TCOL_CR_KPL(X, V) X(2, V) X(4, V) X(6, V) X(8, V) X(12, V) X(18, V) X(24, V) X(36, V)

hipError_t class_rows_prepare(int kmax, int var) {
#define TCOL_CR_ATTR(KP, VR)                                                                                   \
    if (update_rows_kpl(kmax) == KP && var == VR)                                                              \
        return hipFuncSetAttribute((const void*)k_class_rows<KP, VR>,                                          \
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kMaxBlockLds);
    TCOL_CR_KPL(TCOL_CR_ATTR, 0) TCOL_CR_KPL(TCOL_CR_ATTR, 1) TCOL_CR_KPL(TCOL_CR_ATTR, 2) TCOL_CR_KPL(TCOL_CR_ATTR, 3)
#undef TCOL_CR_ATTR
    return hipErrorInvalidValue;
}

hipError_t launch_class_rows(const GraphDev* gd, int G, int blocks, size_t lds, int kmax, int var, int honor_stop,
                             int mode, int gsel, float* gS_out, float* gW_out, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    if (lds > (size_t)kMaxBlockLds) return hipErrorInvalidValue;
    bool done = false;
#define TCOL_CR_LAUNCH(KP, VR)                                                                                 \
    if (!done && update_rows_kpl(kmax) == KP && var == VR) {                                                   \
        k_class_rows<KP, VR><<<blocks, kCrThreads, lds, s>>>(gd, G, blocks, honor_stop, mode, gsel, gS_out, gW_out);  \
        done = true;                                                                                           \
    }
    TCOL_CR_KPL(TCOL_CR_LAUNCH, 0) TCOL_CR_KPL(TCOL_CR_LAUNCH, 1) TCOL_CR_KPL(TCOL_CR_LAUNCH, 2) TCOL_CR_KPL(TCOL_CR_LAUNCH, 3)
#undef TCOL_CR_LAUNCH
    if (!done) return hipErrorInvalidValue;
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_advance(const GraphDev* gd, int G, hipStream_t s) {
    hipLaunchKernelGGL(k_advance, dim3(ceil_div(G, 64)), dim3(64), 0, s, gd, G);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_loss(const GraphDev* gd, int G, int g, int ntiles, int fold, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_loss, dim3(G), dim3(256), 0, s, gd, G, g, ntiles, fold, out);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_report(const GraphDev* gd, int G, int g, int fold, int16_t* colors, int64_t* fcol, int64_t* feq, hipStream_t s) {
    hipLaunchKernelGGL(k_report, dim3(G + 256), dim3(256), 0, s, gd, G, g, fold, colors, fcol, feq);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_class_conflicts(const GraphDev* gd, int g, int D, int k, int32_t* out, hipStream_t s) {
    if (D <= 0 || k <= 0) return hipSuccess;
    const int rb = ceil_div(k, kCcRows);
    const size_t lds = (size_t)std::min(k, kCcRows) * 16 * 4;
    const hipError_t e = hipFuncSetAttribute((const void*)k_class_conflicts, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             kMaxBlockLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_class_conflicts, dim3(D * ceil_div(k, 16) * rb), dim3(kCcThreads), lds, s, gd, g, rb, out);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_put_desc(const GraphDev& d, GraphDev* gd, GraphState* st, unsigned long long* ones, hipStream_t s) {
    hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(256), 0, s, d, gd, st, ones);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (((uintptr_t)p & 15) || (bytes & 15)) return hipErrorInvalidValue;
    const size_t words = bytes / 16;
    const int blocks = (int)std::min<size_t>((words + 255) / 256, 2048);
    hipLaunchKernelGGL(k_zero16, dim3(blocks), dim3(256), 0, s, (uint4*)p, words);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_copy_selection(const GraphDev* gd, int g, int16_t* out, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_selection, dim3(512), dim3(256), 0, s, gd, g, out);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_state(const GraphDev* gd, int G, int op, int g_only, long long t, hipStream_t s) {
    hipLaunchKernelGGL(k_state, dim3(ceil_div(G, 64)), dim3(64), 0, s, gd, G, op, g_only, t);
    TCOL_LAUNCH_CHECK();
    return hipSuccess;
}

}  // namespace tcol
