// asora_fwd.hip -- forward ray-tracing kernels for gfx950.
//
// One work-group sweeps one piece of one source (see asora_dev.h): shell by
// shell in L1 distance q (Section 3.3), with the exit columns of the last
// four shells in an LDS ring (FP64), the photoionization table in LDS, and
// the rate of every owned cell added to an FP64 N^3 accumulator with one
// hardware atomic per source-cell.  The persistent kernel pulls
// (source, piece) items from a global counter, largest radius first.
#include <stddef.h>

#include <type_traits>

#include "asora_dev.h"
#include "asora_internal.h"
#include "asora_sweep.h"

namespace asora {

constexpr int kWG = 256;

struct FwdArgs {
    int N;
    Extent ex;
    double alpha, sigma0;
    float tau_w;            // weight floor, <= 0: geometric weights
    int reading;            // 0: directional source half path, 1: scalar
    TabParams tp;
    const TabNode *tab;
    const double *nHI;
    double *gacc;
    double *coldens;
    const int32_t *ijk;
    const double *Q;
    const float *R;         // may be NULL: every source has R = R_cap
    float R_cap;
    const int *order;       // sources sorted by piece kind, then spatially (Morton blocks)
    const int *seg;         // seg[t] .. seg[t+1]: sources of type t in order[]
    int type, n_pieces;
    int *counter;
    int *err;
    int ring_cap, row_cap;
    int plain_src;          // >= 0: non-persistent launch for this source
    int src0, items;         // layer pieces, direct: the first source, the number of pyramids (0: from the counters)
    int region_bytes;       // per-wave LDS region (wave kernels)
    GroupClasses grp;       // group pieces
    int grp_shared;         // bytes of their work-group tables
    double coef_unit;       // sigma0 / (4 pi alpha^2)
    const double *nHI_T;    // n_HI in the [k][i][j] layout (layer pieces with d = k)
    double *gacc_T;         // Gamma accumulator in the [k][i][j] layout
    int lay_S;              // row stride of the per-wave layer buffer (layer pieces)
    char *keep;             // layer pieces: column records, per (source, pyramid); NULL = none
    size_t keep_piece_bytes;
    long keep_cap;          // cells per pyramid record
    int keep_Mcap;          // largest layer of the plan
    const Node64 *n64;      // the table in FP64 (the rate of a forward that keeps records)
    int early_exit;         // layer pieces: stop after the first opaque layer
    const TabNode *tab_h;   // photo-heating table on the same node grid (read through the
                            // caches), or NULL: no heating
    double *hacc, *hacc_T;  // heating accumulators, in the layouts of gacc and gacc_T
    float dP0_h;            // dH/dtau at the first node (slope of the heating table's continuation)
    LayerConst lc;
    int sq_n;               // layer pieces: entries of the work-group's LDS table of sqrt(r^2)
                            // (r^2 < sq_n); 0: roots computed per cell
};

// The node grid's parameters with the heating table's end slope.
__device__ __forceinline__ TabParams heat_params(const FwdArgs &A)
{
    TabParams t = A.tp;
    t.dP0 = A.dP0_h;
    return t;
}

// Heating of one cell, added to hacc: the heating table's divided difference
// over the cell's optical depths, with the rate's coefficient (the same
// formula with H in place of P).
__device__ __forceinline__ void add_heating(const FwdArgs &A, double *hacc, uint32_t cp, double ta,
                                            double dt, int r2, double coef)
{
    const float nd = neg_divdiff(A.tab_h, heat_params(A), ta, dt);
    if (nd > 0.f) unsafeAtomicAdd(&hacc[cp], coef * (double)(nd * rcp_approx((float)r2)));
}

struct Lds {
    const TabNode *tab;   // read through the caches
    double *ring;      // [4][ring_cap]
    int *rowbase;      // [4][row_cap]: slot of (row, B) = rowbase[row] + B
    int *rowstart;     // [row_cap + 1] of the current shell
};

// Sweep one piece of one source.  Called by all threads of the work-group.
__device__ void sweep_piece(const FwdArgs &A, const Lds &L, int src, int p, int *sh_total)
{
    const int tid = threadIdx.x;
    const int N = A.N;
    const int si = A.ijk[3 * src], sj = A.ijk[3 * src + 1], sk = A.ijk[3 * src + 2];
    const float R = A.R ? A.R[src] : A.R_cap;
    if (!(R >= 0.f && R <= A.R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 ||
        sk >= N) {
        if (tid == 0) atomicOr(A.err, 1);
        return;
    }
    const double Q = A.Q[src];
    const int Rsq = (int)floor((double)R * (double)R);
    const Piece pc = make_piece(A.type, p);
    const int Qmax = max_shell(Rsq, A.ex);
    const long cs = ((long)si * N + sj) * N + sk;
    const double n_s = A.nHI[cs];

    CellCtx X;
    X.pc = pc;
    X.N = N;
    X.si = si;
    X.sj = sj;
    X.sk = sk;
    X.reading = A.reading;
    X.tau_w = A.tau_w;
    X.sigma0 = A.sigma0;
    X.alpha = A.alpha;
    X.half_col = n_s * A.alpha * 0.5;
    X.coef = Q * A.coef_unit;
    X.tab = L.tab;
    X.m64 = nullptr;
    X.tp = A.tp;
    X.ring = L.ring;
    X.rowbase = L.rowbase;
    X.ring_cap = A.ring_cap;
    X.row_cap = A.row_cap;
    X.nHI = A.nHI;

    const bool src_owner = (pc.kind == 0) || (pc.oct == 0 && (pc.dom < 0 || pc.dom == 2));
    if (src_owner && tid == 0) {
        const double G = source_cell_rate(L.tab, A.tp, A.sigma0, A.alpha, Q, n_s);
        if (G != 0.0) unsafeAtomicAdd(&A.gacc[cs], G);
        if (A.coldens) A.coldens[cs] = 0.0;
        if (A.hacc) {
            const double H = source_cell_rate(A.tab_h, heat_params(A), A.sigma0, A.alpha, Q, n_s);
            if (H != 0.0) unsafeAtomicAdd(&A.hacc[cs], H);
        }
    }

    for (int q = 1; q <= Qmax; ++q) {
        const int slot = q & 3;
        const int nrows = pc.n_oct * (q + 1);
        // ---- row table of shell q (wave 0): counts, exclusive scan, bases
        if (tid < 64) {
            const int c = (nrows + 63) >> 6;
            const int r0 = tid * c;
            int sum = 0;
            for (int k = 0; k < c; ++k) {
                const int r = r0 + k;
                if (r < nrows) {
                    int blo, cnt;
                    row_range(pc, A.ex, Rsq, q, r, &blo, &cnt);
                    sum += cnt;
                }
            }
            int incl = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(incl, off, 64);
                if (tid >= off) incl += t;
            }
            int run = incl - sum;
            for (int k = 0; k < c; ++k) {
                const int r = r0 + k;
                if (r < nrows) {
                    int blo, cnt;
                    row_range(pc, A.ex, Rsq, q, r, &blo, &cnt);
                    L.rowstart[r] = run;
                    L.rowbase[slot * A.row_cap + r] = run - blo;
                    run += cnt;
                }
            }
            if (tid == 63) {
                L.rowstart[nrows] = incl;
                *sh_total = incl;
            }
        }
        __syncthreads();
        const int total = *sh_total;
        const int *rb_q = L.rowbase + slot * A.row_cap;
        double *ring_q = L.ring + slot * A.ring_cap;
        for (int g = tid; g < total; g += kWG) {
            const int row = find_row(L.rowstart, nrows, g);
            CellOut co;
            cell_update(X, q, g, row, rb_q[row], co);
            ring_q[g] = co.Nout;
            if (co.owned) {
                if (co.G != 0.0) unsafeAtomicAdd(&A.gacc[co.cp], co.G);
                if (A.coldens) A.coldens[co.cp] = co.Nin;
                if (A.hacc)
                    add_heating(A, A.hacc, co.cp, A.sigma0 * co.Nin, A.sigma0 * co.dN, co.r2, X.coef);
            }
        }
        __syncthreads();
    }
}

static FwdArgs make_args(const FwdLaunch &F);

// Per-wave queue of pending rate evaluations (structure of arrays in LDS).
constexpr int kQueue = 128;
struct RateQueue {
    double *ta;     // entry optical depth
    float *dt;      // in-cell optical depth
    uint32_t *cp;   // cell index
    int *r2;        // squared distance (cells)
};

template <bool HEAT>
__device__ __forceinline__ void rate_batch(const FwdArgs &A, const TabNode *T, const RateQueue &Qa,
                                           int head, int lane, double coef, double *acc)
{
    const int pos = (head + lane) & (kQueue - 1);
    const double ta = Qa.ta[pos];
    const float nd = neg_divdiff(T, A.tp, ta, (double)Qa.dt[pos]);
    if (nd > 0.f) {
        const double G = coef * (double)(nd * rcp_approx((float)Qa.r2[pos]));
        unsafeAtomicAdd(&acc[Qa.cp[pos]], G);
    }
    if (HEAT) add_heating(A, A.hacc, Qa.cp[pos], ta, (double)Qa.dt[pos], Qa.r2[pos], coef);
}

template <int TYPE, bool HEAT>
__device__ void sweep_piece_wave(const FwdArgs &A, const TabNode *T, double *ring, int *rowbase,
                                 int *rowstart, const RateQueue &Qa, int src, int p, int lane)
{
    const int N = A.N;
    const int si = A.ijk[3 * src], sj = A.ijk[3 * src + 1], sk = A.ijk[3 * src + 2];
    const float R = A.R ? A.R[src] : A.R_cap;
    if (!(R >= 0.f && R <= A.R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 ||
        sk >= N) {
        if (lane == 0) atomicOr(A.err, 1);
        return;
    }
    const double Q = A.Q[src];
    const int Rsq = (int)floor((double)R * (double)R);
    const Piece pc = make_piece(TYPE, p);
    const int Qmax = max_shell(Rsq, A.ex);
    const long cs = ((long)si * N + sj) * N + sk;
    const double n_s = A.nHI[cs];

    CellCtx X;
    X.pc = pc;
    X.N = N;
    X.si = si;
    X.sj = sj;
    X.sk = sk;
    X.reading = A.reading;
    X.tau_w = A.tau_w;
    X.sigma0 = A.sigma0;
    X.alpha = A.alpha;
    X.half_col = n_s * A.alpha * 0.5;
    X.coef = Q * A.coef_unit;
    X.tab = T;
    X.m64 = nullptr;
    X.tp = A.tp;
    X.ring = ring;
    X.rowbase = rowbase;
    X.ring_cap = A.ring_cap;
    X.row_cap = A.row_cap;
    X.nHI = A.nHI;

    const bool src_owner = (pc.kind == 0) || (pc.oct == 0 && (pc.dom < 0 || pc.dom == 2));
    if (src_owner && lane == 0) {
        const double G = source_cell_rate(T, A.tp, A.sigma0, A.alpha, Q, n_s);
        if (G != 0.0) unsafeAtomicAdd(&A.gacc[cs], G);
        if (A.coldens) A.coldens[cs] = 0.0;
        if (HEAT) {
            const double H = source_cell_rate(A.tab_h, heat_params(A), A.sigma0, A.alpha, Q, n_s);
            if (H != 0.0) unsafeAtomicAdd(&A.hacc[cs], H);
        }
    }
    int head = 0, tail = 0;   // rate queue positions (wave-uniform)

    for (int q = 1; q <= Qmax; ++q) {
        const int slot = q & 3;
        const int nrows = pc.n_oct * (q + 1);
        int *rb_q = rowbase + slot * A.row_cap;
        const int total = wave_build_rows(pc, A.ex, Rsq, q, lane, rowstart, rb_q);
        wave_sync();
        double *ring_q = ring + slot * A.ring_cap;
        // columns for 64 cells at a time; cells whose rate is non-zero (owned,
        // entry optical depth below the table end) go to the wave's queue, and
        // every full 64 queued rates are evaluated by all lanes together
        for (int g0 = 0; g0 < total; g0 += 64) {
            const int g = g0 + lane;
            bool want = false;
            CellOut co;
            co.Nin = 0.0;
            if (g < total) {
                const int row = find_row(rowstart, nrows, g);
                cell_update<false>(X, q, g, row, rb_q[row], co);
                ring_q[g] = co.Nout;
                if (co.owned) {
                    if (A.coldens) A.coldens[co.cp] = co.Nin;
                    want = A.sigma0 * co.Nin < A.tp.tau_hi;
                }
            }
            const uint64_t mask = __ballot(want);
            if (want) {
                const int pos = (tail + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))) & (kQueue - 1);
                Qa.ta[pos] = A.sigma0 * co.Nin;
                Qa.dt[pos] = A.sigma0 * co.dN;
                Qa.cp[pos] = co.cp;
                Qa.r2[pos] = co.r2;
            }
            tail += __popcll(mask);
            if (tail - head >= 64) {
                wave_sync();
                rate_batch<HEAT>(A, T, Qa, head, lane, X.coef, A.gacc);
                head += 64;
                wave_sync();
            }
        }
        wave_sync();
    }
    // the rates still queued
    if (tail > head) {
        wave_sync();
        if (lane < tail - head) rate_batch<HEAT>(A, T, Qa, head, lane, X.coef, A.gacc);
        wave_sync();
    }
}

// One wave per piece; the work-group only shares the table.  Persistent
// (items from the global counter) or plain (item = wave index).
template <int TYPE, bool HEAT>
__device__ __forceinline__ void fwd_wave_body(const FwdArgs &A, char *smem)
{
    constexpr int npieces0 = TYPE == 0 ? 1 : (TYPE == 1 ? 8 : 24);
    if (A.plain_src < 0 && A.seg[TYPE + 1] == A.seg[TYPE]) return;   // no sources of this kind
    (void)npieces0;
    const TabNode *T = A.tab;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    char *region = smem + (size_t)wave * A.region_bytes;
    double *ring = (double *)region;
    RateQueue Qa;
    Qa.ta = ring + 4 * (size_t)A.ring_cap;
    Qa.dt = (float *)(Qa.ta + kQueue);
    Qa.cp = (uint32_t *)(Qa.dt + kQueue);
    Qa.r2 = (int *)(Qa.cp + kQueue);
    int *rowbase = Qa.r2 + kQueue;
    int *rowstart = rowbase + 4 * A.row_cap;
    constexpr int npieces = TYPE == 0 ? 1 : (TYPE == 1 ? 8 : 24);
    if (A.plain_src >= 0) {
        const int item = blockIdx.x * waves + wave;
        if (item < npieces)
            sweep_piece_wave<TYPE, HEAT>(A, T, ring, rowbase, rowstart, Qa, A.plain_src, item, lane);
        return;
    }
    const int base = A.seg[TYPE];
    const int nitems = (A.seg[TYPE + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (;;) {
        const int item = next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = A.order[base + item / npieces];
        sweep_piece_wave<TYPE, HEAT>(A, T, ring, rowbase, rowstart, Qa, src, item % npieces, lane);
    }
}

template <int TYPE>
__global__ __launch_bounds__(1024) void fwd_wave(FwdArgs A)
{
    extern __shared__ __align__(16) char smem[];
    fwd_wave_body<TYPE, false>(A, smem);
}

// The same sweep, adding the photo-heating of every cell to hacc.
template <int TYPE>
__global__ __launch_bounds__(1024) void fwd_wave_heat(FwdArgs A)
{
    extern __shared__ __align__(16) char smem[];
    fwd_wave_body<TYPE, true>(A, smem);
}

// ---- layer pieces --------------------------------------------------------
// One wave sweeps one pyramid layer by layer (sweep_layers).  Cells whose rate
// is non-zero (owned, entry optical depth below the table end) go to the
// wave's queue, and every full 64 queued rates are evaluated by all lanes
// together.  With KEEP the sweep also writes the pyramid's column record (the
// cells' layer-buffer entries and the chunks' masks of cells with a rate) for a
// later adjoint.
//
// The queue, in LDS (byte offsets): per cell its entry optical depth as an
// entry (entry_tau), the cell index, the in-cell optical depth and the squared
// distance in 16 bits (a layer buffer that fits the LDS bounds the radius: R^2
// stays below 2^16, which the plan checks).  The in-cell optical depth is
// rounded to FP32 as in RateQueue (a relative change of 6e-8 in one argument of
// the rate), except with KEEP, whose rate is evaluated in FP64.
template <bool KEEP>
struct LayerQueue {
    using dt_t = typename std::conditional<KEEP, double, float>::type;
    static constexpr int kBytes = kQueue * (int)(sizeof(double) + sizeof(dt_t) + sizeof(uint32_t) + sizeof(uint16_t));
    int e, dt, cp, r2;
    __device__ __forceinline__ explicit LayerQueue(int base)
        : e(base), dt(base + 8 * kQueue), cp(dt + (int)sizeof(dt_t) * kQueue), r2(cp + 4 * kQueue)
    {
    }
};

// One batch of queued cells, from ring position head: the rate added to Gamma,
// from the FP32 divided difference, with KEEP from the FP64 one.
// BOTH: cells marked kQueueT belong to the transposed accumulators.
constexpr int kQueueT = 0x8000;
template <bool KEEP, bool HEAT, bool EXTRA, bool BOTH = false>
__device__ __forceinline__ void layer_rate_batch(const FwdArgs &A, const LayerQueue<KEEP> &Qa, int head, int lane,
                                                 double coef, double *acc, double *hacc)
{
    const int pos = (head + lane) & (kQueue - 1);
    const double ta = entry_tau(lds<double>(Qa.e + 8 * pos));
    const double dt = (double)lds<typename LayerQueue<KEEP>::dt_t>(Qa.dt + (int)sizeof(typename LayerQueue<KEEP>::dt_t) * pos);
    const uint32_t cp = lds<uint32_t>(Qa.cp + 4 * pos);
    int r2 = lds<uint16_t>(Qa.r2 + 2 * pos);
    if (BOTH) {
        if (r2 & kQueueT) {
            acc = A.gacc_T;
            hacc = A.hacc_T;
        }
        r2 &= kQueueT - 1;
    }
    // (the heating is evaluated before the first atomic: a table's nodes that
    // are loaded after it arrive after it)
    float nh = 0.f;
    if (HEAT) nh = EXTRA ? neg_divdiff(A.tab_h, heat_params(A), ta, dt) : neg_divdiff_fine(A.tab_h, heat_params(A), ta, dt);
    double G;
    if (!KEEP) {
        const float nd = EXTRA ? neg_divdiff(A.tab, A.tp, ta, dt) : neg_divdiff_fine(A.tab, A.tp, ta, dt);
        G = coef * (double)(nd * rcp_approx((float)r2));
    } else {
        const TabParams tp = reload_arg<TabParams>(offsetof(FwdArgs, tp));
        G = coef * rcp_f64((double)r2) * neg_divdiff64<!EXTRA>(NodeArray{A.n64}, tp, ta, dt);
    }
    if (HEAT) asm volatile("" : "+v"(nh), "+v"(G));
    if (G > 0.0) unsafeAtomicAdd(&acc[cp], G);
    if (HEAT && nh > 0.f) unsafeAtomicAdd(&hacc[cp], coef * (double)(nh * rcp_approx((float)r2)));
}

// EXTRA: with the entry-column output, the early exit or a coarse table;
// without, those are compiled out (fewer registers for the common sweep).
// TEAM: swept by the work-group's waves together, each with its own queue; not
// with the early exit, which would have to agree across the waves.
template <bool KEEP, bool HEAT, bool EXTRA, bool TEAM>
__device__ __forceinline__ void sweep_layer_piece(const FwdArgs &A, const SweepLds &W, const LayerQueue<KEEP> &Qa,
                                                  Team team, int src, int p, int lane)
{
    const bool first = (!TEAM || team.w == 0) && lane == 0;
    const int N = A.N;
    const int si = uniform(A.ijk[3 * src]), sj = uniform(A.ijk[3 * src + 1]), sk = uniform(A.ijk[3 * src + 2]);
    const float R = A.R ? A.R[src] : A.R_cap;
    if (!(R >= 0.f && R <= A.R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 ||
        sk >= N) {
        if (first) atomicOr(A.err, 1);
        return;
    }
    const double Q = uniform(A.Q[src]);
    const int Rsq = uniform((int)floor((double)R * (double)R));
    const LayerPiece L = make_layer_piece(p, si, sj, sk, N, A.ex);
    const uint32_t cs = ((uint32_t)si * (uint32_t)N + (uint32_t)sj) * (uint32_t)N + (uint32_t)sk;
    const double n_s = uniform(A.nHI[cs]);
    LayerX X;
    X.N = N;
    X.reading = A.reading;
    X.tau_w = A.tau_w;
    X.sigma0 = A.sigma0;
    X.alpha = A.alpha;
    layer_x_source(X, A.lc, n_s);
    X.nHI = L.transposed ? A.nHI_T : A.nHI;
    double *acc = L.transposed ? A.gacc_T : A.gacc;
    double *hacc = HEAT ? (L.transposed ? A.hacc_T : A.hacc) : nullptr;
    const double coef = uniform(Q * A.coef_unit);
    LayerRecord rec;
    if (KEEP)
        rec = layer_record_at(A.keep + ((size_t)src * 24 + p) * A.keep_piece_bytes, A.keep_cap, 0);

    if (p == 3 * 0 + 2 && first) {   // the source cell, once per source
        const double G = source_cell_rate<!EXTRA>(A.tab, A.tp, A.sigma0, A.alpha, Q, n_s);
        if (G != 0.0) unsafeAtomicAdd(&A.gacc[cs], G);
        if (EXTRA && A.coldens) A.coldens[cs] = 0.0;
        if (HEAT) {
            const double H = source_cell_rate<!EXTRA>(A.tab_h, heat_params(A), A.sigma0, A.alpha, Q, n_s);
            if (H != 0.0) unsafeAtomicAdd(&A.hacc[cs], H);
        }
    }
    const int Mx = min(uniform(isqrt_floor(Rsq)), L.ext_d);
    // the last layer swept, recorded and visited by the adjoint: every layer,
    // unless the early exit stops the pyramid at its first opaque layer
    int m_last = Mx;
    if (Mx >= 1) {
        sweep_index_terms<TEAM>(L, N, W, team, lane);
        // the rate queue: `pend` cells from ring position `head`
        int head = 0, pend = 0;
        long off = 0, choff = 0;   // first cell and chunk of layer m in the record
        bool opq = true;           // every cell of layer m so far leaves opaque
        sweep_layers<TEAM>(
            L, X, W, team, Rsq, Mx, m_last, A.tp.tau_hi, A.lc.inv_hi, lane,
            [&](const SweepChunk &k) {
                const bool owned = k.in & layer_owned(L, k.m, k.u, k.v);
                const bool want = owned & k.below;
                if (KEEP && k.in) rec.h[off + k.c * 64 + lane] = k.h;
                if (EXTRA && A.coldens && owned)
                    A.coldens[layer_std_index(L, N, k.m, k.u, k.v)] = entry_tau(k.e_in) * X.inv_s0;
                const uint64_t mask = ballot(want);
                if (KEEP && lane == 0 && k.any) rec.lit[choff + k.c] = mask;
                if (EXTRA && !TEAM && A.early_exit)
                    opq = opq && ballot(k.in && entry_below(k.h, A.lc.opaque, A.lc.inv_opq)) == 0;
                if (want) {
                    const int q = (head + pend + rank_in(mask)) & (kQueue - 1);
                    lds<double>(Qa.e + 8 * q) = k.e_in;
                    lds<typename LayerQueue<KEEP>::dt_t>(Qa.dt + (int)sizeof(typename LayerQueue<KEEP>::dt_t) * q) =
                        (typename LayerQueue<KEEP>::dt_t)k.dt;
                    lds<uint32_t>(Qa.cp + 4 * q) = k.cell;
                    lds<uint16_t>(Qa.r2 + 2 * q) = (uint16_t)k.r2;
                }
                pend += __popcll(mask);
                if (pend >= 64) {
                    wave_sync();
                    layer_rate_batch<KEEP, HEAT, EXTRA>(A, Qa, head, lane, coef, acc, hacc);
                    head = (head + 64) & (kQueue - 1);
                    pend -= 64;
                }
            },
            [&](int m, int total) {
                off += total;
                choff += (total + 63) / 64;
                if (EXTRA && !TEAM && A.early_exit && opq) m_last = m;   // every later cell has a zero rate
                opq = true;
            });
        wave_sync();
        if (lane < pend) layer_rate_batch<KEEP, HEAT, EXTRA>(A, Qa, head, lane, coef, acc, hacc);
        wave_sync();
    }
    if (KEEP && first) rec.lit[A.keep_cap / 64 + A.keep_Mcap] = (uint64_t)m_last;
}

// The work-group shares only the table of square roots, when the launch gives
// one (sq_n > 0: the plan adds it only where it costs no wave); every wave
// has its own region (rate queue, layer buffer, table of factors).  The rate
// tables are read through the caches: 32-byte nodes in LDS would take the room
// of three to six waves.
// KEEP: writes the column records; HEAT: adds the photo-heating of every cell
// to hacc / hacc_T.
template <bool KEEP, bool HEAT, bool EXTRA>
__global__ __launch_bounds__(1024) void fwd_layer(FwdArgs A)
{
    constexpr int TYPE = 3, npieces = 24;
    const bool direct = A.items > 0;
    if (!direct && A.seg[TYPE + 1] == A.seg[TYPE]) return;   // no sources of this kind
    for (int k = threadIdx.x; k < A.sq_n; k += blockDim.x) lds<double>(8 * k) = sqrt((double)k);
    __syncthreads();
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    const int region = (A.sq_n ? (int)layer_sqrt_bytes(A.sq_n - 1) : 0) + wave * A.region_bytes;
    const LayerQueue<KEEP> Qa(region);
    SweepLds W;
    W.S = A.lay_S;
    W.sq = 0;
    W.sq_n = A.sq_n;
    W.lay = region + LayerQueue<KEEP>::kBytes;
    W.geo = W.lay + 8 * (W.S + 1) * (W.S + 1);
    // persistent: items from the counters; direct: one item per wave, pyramids
    // of the sources from src0 on
    const int base = direct ? 0 : A.seg[TYPE];
    const int nitems = direct ? A.items : (A.seg[TYPE + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (;;) {
        const int item = direct ? (int)blockIdx.x * waves + wave : next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = direct ? A.src0 + item / npieces : uniform(A.order[base + item / npieces]);
        sweep_layer_piece<KEEP, HEAT, EXTRA, false>(A, W, Qa, Team{0, 1}, src, item % npieces, lane);
        if (direct) break;
    }
}

// One work-group per pyramid, its waves a team: for calls with so few pyramids
// that one wave each would leave the chip idle.  Bound by the latency of a
// layer: its chunks and one barrier (32^3, one source of radius 15: 20 us for
// 15 layers with two waves to a pyramid, where the shell sweep of eight octants
// took 127; 128^3, 85 sources of radius 30: 190 us with one wave, 116 with two).
template <bool KEEP, bool HEAT, bool EXTRA>
__global__ __launch_bounds__(1024) void fwd_team(FwdArgs A)
{
    const Team team{uniform((int)threadIdx.x >> 6), (int)blockDim.x >> 6};
    const int lane = threadIdx.x & 63;
    SweepLds W;
    W.S = A.lay_S;
    W.sq = 0;
    W.sq_n = 0;
    W.lay = 0;
    W.geo = 2 * 8 * (W.S + 1) * (W.S + 1);
    const LayerQueue<KEEP> Qa((W.geo + 2 * (int)sizeof(GeoRow) * W.S + 15 & ~15) + team.w * LayerQueue<KEEP>::kBytes);
    const int item = blockIdx.x;
    sweep_layer_piece<KEEP, HEAT, EXTRA, true>(A, W, Qa, team, A.src0 + item / 24, item % 24, lane);
}

// ---- group pieces --------------------------------------------------------
// One wave sweeps W.G pyramids of a source together (sweep_group), for sources
// too small for a pyramid's layers to fill a wave.
template <bool HEAT, bool EXTRA>
__device__ __forceinline__ void sweep_group_piece(const FwdArgs &A, const GroupLds &W, const LayerQueue<false> &Qa,
                                                  float R_cap, int src, int part, int lane)
{
    const int N = A.N;
    const int si = uniform(A.ijk[3 * src]), sj = uniform(A.ijk[3 * src + 1]), sk = uniform(A.ijk[3 * src + 2]);
    const float R = A.R ? A.R[src] : R_cap;
    if (!(R >= 0.f && R <= R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 ||
        sk >= N) {
        if (lane == 0) atomicOr(A.err, 1);
        return;
    }
    const double Q = uniform(A.Q[src]);
    const int Rsq = uniform((int)floor((double)R * (double)R));
    const uint32_t cs = ((uint32_t)si * (uint32_t)N + (uint32_t)sj) * (uint32_t)N + (uint32_t)sk;
    const double n_s = uniform(A.nHI[cs]);
    LayerX X;
    X.N = N;
    X.reading = A.reading;
    X.tau_w = A.tau_w;
    X.sigma0 = A.sigma0;
    X.alpha = A.alpha;
    layer_x_source(X, A.lc, n_s);
    X.nHI = A.nHI;
    const double coef = uniform(Q * A.coef_unit);
    if (part == 0 && lane == 0) {   // the source cell, once per source
        const double G = source_cell_rate<!EXTRA>(A.tab, A.tp, A.sigma0, A.alpha, Q, n_s);
        if (G != 0.0) unsafeAtomicAdd(&A.gacc[cs], G);
        if (EXTRA && A.coldens) A.coldens[cs] = 0.0;
        if (HEAT) {
            const double H = source_cell_rate<!EXTRA>(A.tab_h, heat_params(A), A.sigma0, A.alpha, Q, n_s);
            if (H != 0.0) unsafeAtomicAdd(&A.hacc[cs], H);
        }
    }
    const int Mx = uniform(isqrt_floor(Rsq));   // within the box: see radii_of
    if (Mx < 1) return;
    group_tables(W, part * W.G, si, sj, sk, N, lane);
    int head = 0, pend = 0;   // the rate queue
    sweep_group(X, A.nHI_T, W, Rsq, Mx, A.tp.tau_hi, A.lc.inv_hi, lane, [&](const GroupChunk &k) {
        const bool owned = k.in & group_owned(k.flags, k.m, k.u, k.v);
        const bool want = owned & k.below;
        if (EXTRA && A.coldens && owned) {
            uint32_t c = k.cell;
            if (k.flags & kGroupT) {   // [k][i][j] to [i][j][k]
                const uint32_t n = (uint32_t)N, ck = c / (n * n), cij = c % (n * n);
                c = cij * n + ck;
            }
            A.coldens[c] = entry_tau(k.e_in) * X.inv_s0;
        }
        const uint64_t mask = ballot(want);
        if (want) {
            const int q = (head + pend + rank_in(mask)) & (kQueue - 1);
            lds<double>(Qa.e + 8 * q) = k.e_in;
            lds<float>(Qa.dt + 4 * q) = (float)k.dt;
            lds<uint32_t>(Qa.cp + 4 * q) = k.cell;
            lds<uint16_t>(Qa.r2 + 2 * q) = (uint16_t)(k.r2 | (k.flags & kGroupT ? kQueueT : 0));
        }
        pend += __popcll(mask);
        if (pend >= 64) {
            wave_sync();
            layer_rate_batch<false, HEAT, EXTRA, true>(A, Qa, head, lane, coef, A.gacc, A.hacc);
            head = (head + 64) & (kQueue - 1);
            pend -= 64;
        }
    });
    wave_sync();
    if (lane < pend) layer_rate_batch<false, HEAT, EXTRA, true>(A, Qa, head, lane, coef, A.gacc, A.hacc);
    wave_sync();
}

// Bytes of the work-group's tables and of one wave's region.
static size_t group_shared_bytes(const GroupClasses &c)
{
    const int Rsq = c.Rsq[c.n - 1], M = isqrt_floor(Rsq), S = c.S[c.n - 1];
    return ((size_t)(Rsq + 1) * sizeof(double) + (size_t)M * S * sizeof(Geo) + 15) & ~(size_t)15;
}
static size_t group_wave_bytes(const GroupClasses &c)
{
    size_t most = 0;
    for (int t = 0; t < c.n; ++t) {
        const size_t b = (size_t)c.G[t] * ((size_t)(c.S[t] + 1) * (c.S[t] + 1) * sizeof(double) + sizeof(GroupRow)) +
                         12 * (size_t)(isqrt_floor(c.Rsq[t]) + 1) * sizeof(uint32_t);
        most = b > most ? b : most;
    }
    return ((size_t)LayerQueue<false>::kBytes + most + 31) & ~(size_t)15;
}
size_t group_lds_bytes(const GroupClasses &c, int waves)
{
    return group_shared_bytes(c) + (size_t)waves * group_wave_bytes(c);
}

// The classes of a call in one launch, the largest radii first: a class's last
// sources run beside the next one's first.  Bound by latency: nearly every
// chunk of highly ionized gas fills a batch of rates, whose additions the next
// chunk's fields queue behind (125^3, 20000 sources of radii 1 to 10, 505 us at
// 52 % of VALU issue with 57 of 64 lanes active; without the additions 358,
// without the rates 285; by shells 1003).
template <bool HEAT, bool EXTRA>
__global__ __launch_bounds__(1024) void fwd_group(FwdArgs A)
{
    const bool direct = A.items > 0;
    if (!direct && A.seg[A.grp.n] == A.seg[0]) return;   // no sources of these kinds
    const int Rsq = A.grp.Rsq[A.grp.n - 1], M = isqrt_floor(Rsq), S0 = A.grp.S[A.grp.n - 1];
    GroupLds W;
    W.sq = 0;
    W.geo = 8 * (Rsq + 1);
    W.geo_S = S0;
    for (int k = threadIdx.x; k <= Rsq; k += blockDim.x) lds<double>(8 * k) = sqrt((double)k);
    for (int k = threadIdx.x; k < M * S0; k += blockDim.x) {
        const int m = k / S0 + 1;
        lds<Geo>(W.geo + (int)sizeof(Geo) * k) = layer_geo(m, rcp_f64((double)m), k % S0);
    }
    __syncthreads();
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    const LayerQueue<false> Qa(A.grp_shared + wave * A.region_bytes);
    W.lay = Qa.e + LayerQueue<false>::kBytes;
    const int home = (int)(blockIdx.x % kXcds);
    for (int t = A.grp.n - 1; t >= 0; --t) {
        W.S = A.grp.S[t];
        W.K = isqrt_floor(A.grp.Rsq[t]) + 1;
        W.G = A.grp.G[t];
        W.row = (W.lay + W.G * 8 * (W.S + 1) * (W.S + 1) + 15) & ~15;
        W.term = W.row + W.G * (int)sizeof(GroupRow);
        const int npieces = 24 / W.G;
        const int base = direct ? 0 : A.seg[t];
        const int nitems = direct ? A.items : (A.seg[t + 1] - base) * npieces;
        int chunk = home;
        for (;;) {
            const int item = direct ? (int)blockIdx.x * waves + wave
                                    : next_item(A.counter + kXcds * kCounterPad * t, nitems, home, chunk, lane);
            if (item >= nitems) break;
            const int src = direct ? A.src0 + item / npieces : uniform(A.order[base + item / npieces]);
            sweep_group_piece<HEAT, EXTRA>(A, W, Qa, A.grp.R[t], src, item % npieces, lane);
            if (direct) break;
        }
        if (direct) break;
    }
}

static const void *group_fn(bool heat, bool extra)
{
    return heat ? (extra ? (const void *)fwd_group<true, true> : (const void *)fwd_group<true, false>)
                : (extra ? (const void *)fwd_group<false, true> : (const void *)fwd_group<false, false>);
}

hipError_t group_occupancy(int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, group_fn(false, false), waves * 64, lds);
}

size_t layer_region_bytes(int S, bool keep)
{
    const size_t b = (size_t)(keep ? LayerQueue<true>::kBytes : LayerQueue<false>::kBytes) +
                     (size_t)(S + 1) * (S + 1) * sizeof(double) + (size_t)S * sizeof(GeoRow);
    return (b + 15) & ~(size_t)15;
}

size_t team_bytes(int S, bool keep, int T)
{
    const size_t shared = 2 * ((size_t)(S + 1) * (S + 1) * sizeof(double) + (size_t)S * sizeof(GeoRow));
    return ((shared + 15) & ~(size_t)15) +
           (size_t)T * (keep ? LayerQueue<true>::kBytes : LayerQueue<false>::kBytes);
}

static const void *layer_fn(bool keep, bool heat, bool extra, bool team = false)
{
    static const void *const f[16] = {
        (const void *)fwd_layer<false, false, false>, (const void *)fwd_layer<false, false, true>,
        (const void *)fwd_layer<false, true, false>,  (const void *)fwd_layer<false, true, true>,
        (const void *)fwd_layer<true, false, false>,  (const void *)fwd_layer<true, false, true>,
        (const void *)fwd_layer<true, true, false>,   (const void *)fwd_layer<true, true, true>,
        (const void *)fwd_team<false, false, false>,  (const void *)fwd_team<false, false, true>,
        (const void *)fwd_team<false, true, false>,   (const void *)fwd_team<false, true, true>,
        (const void *)fwd_team<true, false, false>,   (const void *)fwd_team<true, false, true>,
        (const void *)fwd_team<true, true, false>,    (const void *)fwd_team<true, true, true>};
    return f[(team ? 8 : 0) + (keep ? 4 : 0) + (heat ? 2 : 0) + (extra ? 1 : 0)];
}

hipError_t layer_occupancy(bool keep, int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, layer_fn(keep, false, false), waves * 64, lds);
}

// The instance a layer launch needs beyond its outputs: see EXTRA.
static bool layer_extra(const FwdArgs &A)
{
    return A.coldens || A.early_exit || !A.tp.fine || (A.keep && !A.tp.tame);
}

hipError_t launch_fwd_layer(hipStream_t st, const FwdLaunch &F, int S, int waves, int grid,
                            int plain_src)
{
    FwdArgs A = make_args(F);
    if (plain_src >= 0) {
        A.src0 = plain_src;
        A.items = 24;
        grid = (24 + waves - 1) / waves;
    }
    A.lay_S = S;
    A.region_bytes = (int)layer_region_bytes(S, A.keep != nullptr);
    const int Rsq = (int)floor((double)F.R_cap * (double)F.R_cap);
    const size_t sqb = F.sq_table ? layer_sqrt_bytes(Rsq) : 0;
    A.sq_n = sqb ? Rsq + 1 : 0;
    const size_t lds = sqb + (size_t)waves * A.region_bytes;
    void *args[] = {&A};
    return hipLaunchKernel(layer_fn(A.keep != nullptr, F.hacc != nullptr, layer_extra(A)), dim3(grid), dim3(64 * waves),
                           args, lds, st);
}

// Group pieces; plain_src: the source is of the largest class.
hipError_t launch_fwd_group(hipStream_t st, const FwdLaunch &F, const GroupClasses &grp, int waves, int grid,
                            int plain_src)
{
    FwdArgs A = make_args(F);
    A.grp = grp;
    if (plain_src >= 0) {
        A.src0 = plain_src;
        A.items = 24 / grp.G[grp.n - 1];
        grid = (A.items + waves - 1) / waves;
    }
    A.counter = F.ctl + kCtlCounter;   // of class 0
    A.region_bytes = (int)group_wave_bytes(grp);
    A.grp_shared = (int)group_shared_bytes(grp);
    void *args[] = {&A};
    return hipLaunchKernel(group_fn(F.hacc != nullptr, F.coldens || !F.tp.fine), dim3(grid), dim3(64 * waves), args,
                           group_lds_bytes(grp, waves), st);
}

// Every pyramid of the n_src sources at once, by T waves each.
hipError_t launch_fwd_direct(hipStream_t st, const FwdLaunch &F, int S, int T, int n_src)
{
    FwdArgs A = make_args(F);
    A.items = 24 * n_src;
    A.lay_S = S;
    const bool keep = A.keep != nullptr;
    A.region_bytes = (int)layer_region_bytes(S, keep);
    const size_t lds = T > 1 ? team_bytes(S, keep, T) : (size_t)A.region_bytes;
    void *args[] = {&A};
    return hipLaunchKernel(layer_fn(keep, F.hacc != nullptr, layer_extra(A), T > 1), dim3(A.items), dim3(64 * T), args, lds, st);
}

size_t wave_region_bytes(int ring_cap, int row_cap)
{
    const size_t b = 4 * (size_t)ring_cap * sizeof(double) +
                     (size_t)kQueue * (sizeof(double) + sizeof(float) + sizeof(uint32_t) + sizeof(int)) +
                     (4 * (size_t)row_cap + row_cap + 1) * sizeof(int);
    return (b + 15) & ~(size_t)15;
}

hipError_t wave_occupancy(int type, int waves, size_t lds, int *blocks_per_cu)
{
    const void *f = type == 0 ? (const void *)fwd_wave<0> : (type == 1 ? (const void *)fwd_wave<1> : (const void *)fwd_wave<2>);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, waves * 64, lds);
}

hipError_t launch_fwd_wave(hipStream_t st, const FwdLaunch &F, int waves, int grid, int plain_src)
{
    FwdArgs A = make_args(F);
    A.plain_src = plain_src;
    A.region_bytes = (int)wave_region_bytes(F.ring_cap, F.row_cap);
    const size_t lds = (size_t)waves * A.region_bytes;
    if (plain_src >= 0) grid = (pieces_of_type(F.type) + waves - 1) / waves;
    if (F.hacc) {
        switch (F.type) {
        case 0: hipLaunchKernelGGL(fwd_wave_heat<0>, dim3(grid), dim3(64 * waves), lds, st, A); break;
        case 1: hipLaunchKernelGGL(fwd_wave_heat<1>, dim3(grid), dim3(64 * waves), lds, st, A); break;
        default: hipLaunchKernelGGL(fwd_wave_heat<2>, dim3(grid), dim3(64 * waves), lds, st, A); break;
        }
        return hipGetLastError();
    }
    switch (F.type) {
    case 0: hipLaunchKernelGGL(fwd_wave<0>, dim3(grid), dim3(64 * waves), lds, st, A); break;
    case 1: hipLaunchKernelGGL(fwd_wave<1>, dim3(grid), dim3(64 * waves), lds, st, A); break;
    default: hipLaunchKernelGGL(fwd_wave<2>, dim3(grid), dim3(64 * waves), lds, st, A); break;
    }
    return hipGetLastError();
}

__device__ Lds carve_lds(char *smem, const FwdArgs &A)
{
    Lds L;
    L.tab = A.tab;
    L.ring = (double *)smem;
    L.rowbase = (int *)(L.ring + 4 * (size_t)A.ring_cap);
    L.rowstart = L.rowbase + 4 * A.row_cap;
    return L;
}

__global__ __launch_bounds__(kWG) void fwd_persistent(FwdArgs A)
{
    extern __shared__ __align__(16) char smem[];
    __shared__ int sh_item, sh_total;
    const Lds L = carve_lds(smem, A);
    const int base = A.seg[A.type];
    const long nitems = (long)(A.seg[A.type + 1] - base) * A.n_pieces;
    __syncthreads();
    for (;;) {
        if (threadIdx.x == 0) sh_item = atomicAdd(A.counter, 1);
        __syncthreads();
        const long item = sh_item;
        if (item >= nitems) break;
        const int src = A.order[base + (int)(item / A.n_pieces)];
        const int p = (int)(item % A.n_pieces);
        sweep_piece(A, L, src, p, &sh_total);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kWG) void fwd_plain(FwdArgs A)
{
    extern __shared__ __align__(16) char smem[];
    __shared__ int sh_total;
    const Lds L = carve_lds(smem, A);
    __syncthreads();
    sweep_piece(A, L, A.plain_src, blockIdx.x, &sh_total);
}

// ---- small kernels: n_HI, accumulators, bucketing, final conversion --------

__global__ void prologue_kernel(const float *__restrict__ nH, const float *__restrict__ xHI,
                                double *__restrict__ nHI, double *__restrict__ gacc,
                                double *__restrict__ coldens, long n3, int *ctl, int nctl)
{
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < n3; c += stride) {
        nHI[c] = (double)nH[c] * (double)xHI[c];   // exact
        gacc[c] = 0.0;
        if (coldens) coldens[c] = 0.0;
    }
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < nctl; k += blockDim.x) ctl[k] = 0;
}

// Morton index of the 16^3 block that holds cell (i, j, k).
__device__ __forceinline__ int block_morton(int i, int j, int k, int N)
{
    const int bi = (int)((long)i * 16 / N), bj = (int)((long)j * 16 / N), bk = (int)((long)k * 16 / N);
    int m = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        m |= (((bi >> b) & 1) << (3 * b + 2)) | (((bj >> b) & 1) << (3 * b + 1)) | (((bk >> b) & 1) << (3 * b));
    return m;
}

// Source pre-pass: piece kind by radius, then the spatial block of the source
// in Morton order, so that sources swept at the same time lie close together
// and share cached field and accumulator lines.
__global__ void classify_kernel(const float *R, const int32_t *ijk, long nsrc, int N, float R_max,
                                Radii radii, int big_type, int *keys, int *hist, int *err)
{
    const long s = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (s >= nsrc) return;
    const float r = R ? R[s] : R_max;
    const int i = ijk[3 * s], j = ijk[3 * s + 1], k = ijk[3 * s + 2];
    int key;
    if (!(r >= 0.f && r <= R_max) || i < 0 || i >= N || j < 0 || j >= N || k < 0 || k >= N) {
        atomicOr(err, 1);
        key = kTypes * kSBins;   // not scheduled
    } else {
        const int type = r <= radii.r[0] ? 0 : (r <= radii.r[1] ? 1 : (r <= radii.r[2] ? 2 : big_type));
        key = type * kSBins + block_morton(i, j, k, N);
        atomicAdd(&hist[key], 1);
    }
    keys[s] = key;
}

// Exclusive scan of the kTypes*kSBins histogram by one work-group of kScanThreads
// threads (each owns a run of consecutive bins); offsets and per-kind segment
// starts.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void scan_kernel(const int *hist, int *offs, int *seg)
{
    constexpr int n = kTypes * kSBins;
    constexpr int per = (n + kScanThreads - 1) / kScanThreads;
    __shared__ int wsum[kScanThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int v[per];
    int sum = 0;
#pragma unroll
    for (int u = 0; u < per; ++u) {
        const int b = t * per + u;
        v[u] = b < n ? hist[b] : 0;
        sum += v[u];
    }
    int incl = sum;   // inclusive scan over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(incl, off, 64);
        if (lane >= off) incl += x;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    int run = before + incl - sum;
#pragma unroll
    for (int u = 0; u < per; ++u) {
        const int b = t * per + u;
        if (b < n) {
            offs[b] = run;
            if (b % kSBins == 0) seg[b / kSBins] = run;
        }
        run += v[u];
    }
    if (t == kScanThreads - 1) seg[kTypes] = run;
}

__global__ void scatter_kernel(const int *keys, long nsrc, int *offs, int *order)
{
    const long s = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (s >= nsrc) return;
    const int key = keys[s];
    if (key >= kTypes * kSBins) return;
    const int pos = atomicAdd(&offs[key], 1);
    order[pos] = (int)s;
}

// What a call with layer pieces starts from, in one pass over the fields: n_HI
// and the zeroed accumulators (the rate's, with hacc the heating's) in the
// standard layout and in the [k][i][j] layout of the pieces whose dominant
// axis is k, the cleared entry columns, the cleared control block.  One 32 x 32
// (j, k) tile of one i plane per work-group, staged through LDS so that both
// the reads (along k) and the transposed writes (along j) are contiguous; the
// work-groups share the control block.  The planes of a second absorber's field
// follow those of the first.
constexpr int kTile = 32;
__global__ __launch_bounds__(256) void layer_prologue_kernel(FieldPair F, int *ctl, int nctl, int N)
{
    __shared__ double tile[kTile][kTile + 1];
    const int k0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile, s = blockIdx.z >= N ? 1 : 0;
    const int i = blockIdx.z - s * N;
    const float *__restrict__ nH = F.n[s], *__restrict__ xHI = F.x[s];
    const FieldBufs B = F.b[s];
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;   // 32 x 8
    for (int jj = ty; jj < kTile; jj += 8) {
        const int j = j0 + jj, k = k0 + tx;
        if (j < N && k < N) {
            const size_t c = ((size_t)i * N + j) * N + k;
            const double n = (double)nH[c] * (double)xHI[c];   // exact
            tile[jj][tx] = n;
            B.nHI[c] = n;
            B.gacc[c] = 0.0;
            if (B.hacc) B.hacc[c] = 0.0;
            if (B.coldens) B.coldens[c] = 0.0;
        }
    }
    const long block = ((long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const long threads = (long)gridDim.x * gridDim.y * gridDim.z * 256;
    for (long k = block * 256 + threadIdx.x; k < nctl; k += threads) ctl[k] = 0;
    __syncthreads();
    for (int kk = ty; kk < kTile; kk += 8) {
        const int k = k0 + kk, j = j0 + tx;
        if (j < N && k < N) {
            const size_t t = ((size_t)k * N + i) * N + j;
            B.nHI_T[t] = tile[tx][kk];
            B.gacc_T[t] = 0.0;
            if (B.hacc_T) B.hacc_T[t] = 0.0;
        }
    }
}

// Gamma = accumulator + transposed accumulator, in the standard layout; the
// planes of a second output follow those of the first.
__global__ __launch_bounds__(256) void transpose_finalize_kernel(FinalPair F, int N, int accumulate)
{
    __shared__ double tile[kTile][kTile + 1];
    const int k0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile, s = blockIdx.z >= N ? 1 : 0;
    const int i = blockIdx.z - s * N;
    const double *__restrict__ gacc = F.acc[s], *__restrict__ gacc_T = F.acc_T[s];
    float *__restrict__ gamma = F.out[s];
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;
    for (int kk = ty; kk < kTile; kk += 8) {
        const int k = k0 + kk, j = j0 + tx;
        if (j < N && k < N) tile[kk][tx] = gacc_T[((size_t)k * N + i) * N + j];
    }
    __syncthreads();
    for (int jj = ty; jj < kTile; jj += 8) {
        const int j = j0 + jj, k = k0 + tx;
        if (j < N && k < N) {
            const size_t c = ((size_t)i * N + j) * N + k;
            const float v = (float)(gacc[c] + tile[tx][jj]);
            gamma[c] = accumulate ? gamma[c] + v : v;
        }
    }
}

// Clears an accumulator (a kernel: no memset node where the caller records
// the launch into a graph).
__global__ void zero_kernel(double *__restrict__ p, long n)
{
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < n; c += stride) p[c] = 0.0;
}

__global__ void finalize_kernel(const double *__restrict__ gacc, float *__restrict__ gamma, long n3,
                                int accumulate)
{
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < n3; c += stride) {
        const float v = (float)gacc[c];
        gamma[c] = accumulate ? gamma[c] + v : v;
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers (called from the C ABI in asora_api.hip)
// ---------------------------------------------------------------------------
hipError_t launch_prologue(hipStream_t st, const float *nH, const float *xHI, double *nHI,
                           double *gacc, double *coldens, long n3, int *ctl, int nctl, int n_cu)
{
    const int blocks = n_cu * 8;
    hipLaunchKernelGGL(prologue_kernel, dim3(blocks), dim3(256), 0, st, nH, xHI, nHI, gacc,
                       coldens, n3, ctl, nctl);
    return hipGetLastError();
}

hipError_t launch_layer_prologue(hipStream_t st, const FieldPair &F, int *ctl, int nctl, int N)
{
    const dim3 grid((N + kTile - 1) / kTile, (N + kTile - 1) / kTile, F.n[1] ? 2 * N : N);
    hipLaunchKernelGGL(layer_prologue_kernel, grid, dim3(256), 0, st, F, ctl, nctl, N);
    return hipGetLastError();
}

hipError_t launch_transpose_finalize(hipStream_t st, const FinalPair &F, int N, int accumulate)
{
    const dim3 grid((N + kTile - 1) / kTile, (N + kTile - 1) / kTile, F.out[1] ? 2 * N : N);
    hipLaunchKernelGGL(transpose_finalize_kernel, grid, dim3(256), 0, st, F, N, accumulate);
    return hipGetLastError();
}

hipError_t launch_bucketing(hipStream_t st, const float *R, const int32_t *ijk, long nsrc, int N,
                            float R_max, const Radii &radii, int big_type, int *keys, int *ctl, int *order, int *err)
{
    int *hist = ctl + kCtlHist, *offs = ctl + kCtlOffs, *seg = ctl + kCtlSeg;
    const int b = (int)((nsrc + 255) / 256);
    if (nsrc > 0) {
        hipLaunchKernelGGL(classify_kernel, dim3(b), dim3(256), 0, st, R, ijk, nsrc, N, R_max,
                           radii, big_type, keys, hist, err);
    }
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanThreads), 0, st, hist, offs, seg);
    if (nsrc > 0)
        hipLaunchKernelGGL(scatter_kernel, dim3(b), dim3(256), 0, st, keys, nsrc, offs, order);
    return hipGetLastError();
}

static FwdArgs make_args(const FwdLaunch &F)
{
    FwdArgs A;
    A.N = F.N;
    A.ex = make_extent(F.N);
    A.alpha = F.alpha;
    A.sigma0 = F.sigma0;
    A.tau_w = F.tau_w;
    A.reading = F.reading;
    A.tp = F.tp;
    A.tab = F.tab;
    A.nHI = F.nHI;
    A.gacc = F.gacc;
    A.coldens = F.coldens;
    A.nHI_T = F.nHI_T;
    A.gacc_T = F.gacc_T;
    A.lay_S = 0;
    A.keep = F.keep;
    A.keep_piece_bytes = F.keep_piece_bytes;
    A.keep_cap = F.keep_cap;
    A.keep_Mcap = F.keep_Mcap;
    A.n64 = F.n64;
    A.early_exit = F.early_exit ? 1 : 0;
    A.tab_h = F.tab_h;
    A.hacc = F.hacc;
    A.hacc_T = F.hacc_T;
    A.dP0_h = F.dP0_h;
    A.ijk = F.ijk;
    A.Q = F.Q;
    A.R = F.R;
    A.R_cap = F.R_cap;
    A.order = F.order;
    A.seg = F.ctl + kCtlSeg;
    A.type = F.type;
    A.n_pieces = pieces_of_type(F.type);
    A.counter = F.ctl + kCtlCounter + kXcds * kCounterPad * F.type;
    A.err = F.err;
    A.ring_cap = F.ring_cap;
    A.row_cap = F.row_cap;
    A.plain_src = -1;
    A.src0 = 0;
    A.items = 0;
    A.grp = GroupClasses();
    A.region_bytes = 0;
    A.coef_unit = F.sigma0 / (4.0 * M_PI * F.alpha * F.alpha);
    A.lc = make_layer_const(F.sigma0, F.alpha, F.tau_w, F.tp.tau_hi);
    A.sq_n = 0;
    return A;
}

size_t fwd_lds_bytes(int ring_cap, int row_cap)
{
    return 4 * (size_t)ring_cap * sizeof(double) +
           (4 * (size_t)row_cap + row_cap + 1) * sizeof(int);
}

hipError_t fwd_configure(size_t max_lds)
{
    // Best effort: the dynamic LDS limit of a kernel defaults to what the device
    // offers; raising it explicitly is only an opt-in where a runtime needs it.
    const int dyn = (int)max_lds - 64;   // leave room for the static LDS words
    (void)hipFuncSetAttribute((const void *)fwd_persistent,
                              hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_plain, hipFuncAttributeMaxDynamicSharedMemorySize,
                              dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave<0>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave<1>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave<2>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave_heat<0>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave_heat<1>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipFuncSetAttribute((const void *)fwd_wave_heat<2>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    for (int f = 0; f < 4; ++f)
        (void)hipFuncSetAttribute(group_fn(f & 2, f & 1), hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    for (int f = 0; f < 16; ++f)
        (void)hipFuncSetAttribute(layer_fn(f & 4, f & 2, f & 1, f & 8), hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipGetLastError();
    return hipSuccess;
}

hipError_t fwd_occupancy(size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)fwd_persistent,
                                                        kWG, lds);
}

hipError_t launch_fwd_persistent(hipStream_t st, const FwdLaunch &F, int grid)
{
    const FwdArgs A = make_args(F);
    const size_t lds = fwd_lds_bytes(F.ring_cap, F.row_cap);
    hipLaunchKernelGGL(fwd_persistent, dim3(grid), dim3(kWG), lds, st, A);
    return hipGetLastError();
}

hipError_t launch_fwd_plain(hipStream_t st, const FwdLaunch &F, int src)
{
    FwdArgs A = make_args(F);
    A.plain_src = src;
    const size_t lds = fwd_lds_bytes(F.ring_cap, F.row_cap);
    hipLaunchKernelGGL(fwd_plain, dim3(A.n_pieces), dim3(kWG), lds, st, A);
    return hipGetLastError();
}

hipError_t launch_zero(hipStream_t st, double *p, long n, int n_cu)
{
    hipLaunchKernelGGL(zero_kernel, dim3(n_cu * 8), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_finalize(hipStream_t st, const double *gacc, float *gamma, long n3, int accumulate,
                           int n_cu)
{
    hipLaunchKernelGGL(finalize_kernel, dim3(n_cu * 8), dim3(256), 0, st, gacc, gamma, n3,
                       accumulate);
    return hipGetLastError();
}

}  // namespace asora
