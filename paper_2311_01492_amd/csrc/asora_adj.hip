// asora_adj.hip -- adjoint (reverse-mode) ray-tracing kernels for gfx950.
//
// Shell pieces (adj_wave): one wave per source piece, like the forward wave
// kernels.  For each piece
// the wave first recomputes the exit column of every cell, shell by shell
// (the forward sweep without the rate), keeping the last four shells in an
// LDS ring and storing every shell to the wave's own scratch in global
// memory together with its in-cell columns (so that the reverse pass reads
// them back in order instead of gathering n_HI again).  It then sweeps the
// shells from the outermost inward: the exit
// columns of shells q-1..q-3 (the neighbours of shell q) come back from the
// scratch into the LDS ring, and the adjoints of the exit columns of shells
// q..q-3 live in a second LDS ring that the cells of shell q update with LDS
// atomics when they push their entry-column adjoint to their neighbours.
// dL/dn_HI goes to an FP64 N^3 accumulator with hardware atomics; dL/dQ is
// reduced over the wave and added once per piece.
#include <stddef.h>

#include "asora_dev.h"
#include "asora_internal.h"
#include "asora_sweep.h"

namespace asora {

struct AdjArgs {
    int N;
    Extent ex;
    double alpha, sigma0, coef_unit;
    float tau_w;
    int reading;
    TabParams tp;
    const TabNode *tab;
    const Node64 *n64;       // the table in FP64
    const double *nHI;
    const double *gbar;      // dL/dGamma, N^3
    double *nbar;            // dL/dn_HI accumulator, N^3
    double *qbar;            // dL/dQ, n_src
    const int32_t *ijk;
    const double *Q;
    const float *R;
    float R_cap;
    const int *order;
    const int *seg;
    int *counter;
    int *err;
    int ring_cap, row_cap, shell_cap;
    int region_bytes;
    double *store;           // per wave: stored exit columns, then in-cell columns
    long store_stride;       // doubles per wave (twice the largest piece's cell count)
    // layer pieces
    const double *nHI_T;     // [k][i][j] copies for pyramids with dominant axis k
    const double *gbar_T;
    double *nbar_T;
    int Mcap, lay_S;         // largest layer index, row stride of the layer buffers
    const char *kept;        // column records kept by the forward (per source and pyramid), or NULL
    size_t rec_piece_bytes;  // bytes of one pyramid's column record
    long rec_cap;            // cells per pyramid record
    int early_exit;          // layer pieces: stop at the first opaque layer
    LayerConst lc;
    int sq_n;                // layer pieces: entries of the work-group's LDS table of sqrt(r^2); 0: none
    int items;               // layer pieces, direct: the number of pyramids (0: from the counters)
    int type;
    GroupClasses grp;        // group pieces: one class
    int grp_shared;          // bytes of their work-group tables
};

template <int TYPE>
__device__ void adjoint_piece_wave(const AdjArgs &A, const TabNode *T, char *region, double *store,
                                   int src, int p, int lane)
{
    double *store_dN = store + A.store_stride / 2;   // in-cell columns, same indexing as store
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
    const uint32_t cs = ((uint32_t)si * (uint32_t)N + (uint32_t)sj) * (uint32_t)N + (uint32_t)sk;
    const double n_s = A.nHI[cs];

    // LDS region of this wave
    double *ring = (double *)region;                        // [4][ring_cap] exit columns
    double *abar = ring + 4 * (size_t)A.ring_cap;           // [4][ring_cap] their adjoints
    int *rowbase = (int *)(abar + 4 * (size_t)A.ring_cap);  // [4][row_cap]
    int *rowstart = rowbase + 4 * A.row_cap;                // [4][row_cap + 1]
    int *shoff = rowstart + 4 * (A.row_cap + 1);            // [shell_cap + 2] offsets in store

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
    X.n64 = A.n64;
    X.tp = A.tp;
    X.ring = ring;
    X.rowbase = rowbase;
    X.ring_cap = A.ring_cap;
    X.row_cap = A.row_cap;
    X.nHI = A.nHI;

    // ---- forward: exit columns of every shell, kept and stored
    if (lane == 0) shoff[1] = 0;
    wave_sync();
    for (int q = 1; q <= Qmax; ++q) {
        const int slot = q & 3;
        int *rs_q = rowstart + slot * (A.row_cap + 1);
        int *rb_q = rowbase + slot * A.row_cap;
        const int total = wave_build_rows(pc, A.ex, Rsq, q, lane, rs_q, rb_q);
        wave_sync();
        const int off = shoff[q];
        const int nrows = pc.n_oct * (q + 1);
        double *ring_q = ring + slot * (size_t)A.ring_cap;
        for (int g = lane; g < total; g += 64) {
            const int row = find_row(rs_q, nrows, g);
            CellOut co;
            cell_update<false>(X, q, g, row, rb_q[row], co);
            ring_q[g] = co.Nout;
            store[off + g] = co.Nout;
            store_dN[off + g] = co.dN;
        }
        if (lane == 0) shoff[q + 1] = off + total;
        wave_sync();
    }

    // ---- reverse
    for (int k = lane; k < 4 * A.ring_cap; k += 64) abar[k] = 0.0;
    wave_sync();
    double nb_src = 0.0, qb = 0.0;
    for (int q = Qmax; q >= 1; --q) {
        const int slot = q & 3;
        if (q < Qmax && q - 3 >= 1) {
            // shell q-3 enters the rings (its slot held shell q+1, finished)
            const int q3 = q - 3, s3 = q3 & 3;
            const int t3 = wave_build_rows(pc, A.ex, Rsq, q3, lane, rowstart + s3 * (A.row_cap + 1),
                                           rowbase + s3 * A.row_cap);
            const int off3 = shoff[q3];
            for (int g = lane; g < t3; g += 64) {
                ring[s3 * (size_t)A.ring_cap + g] = store[off3 + g];
                abar[s3 * (size_t)A.ring_cap + g] = 0.0;
            }
            wave_sync();
        }
        const int *rs_q = rowstart + slot * (A.row_cap + 1);
        const int *rb_q = rowbase + slot * A.row_cap;
        const int nrows = pc.n_oct * (q + 1);
        const int total = shoff[q + 1] - shoff[q];
        for (int g = lane; g < total; g += 64) {
            const int row = find_row(rs_q, nrows, g);
            CellAdj ca;
            cell_adjoint(X, q, g, row, rb_q[row], abar[slot * (size_t)A.ring_cap + g],
                         store_dN[shoff[q] + g], A.gbar, ca);
            if (ca.nbar != 0.0) unsafeAtomicAdd(&A.nbar[ca.cp], ca.nbar);
            nb_src += ca.nbar_src;
            qb += ca.qbar;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (ca.slot[k] >= 0)
                    atomicAdd(&abar[(ca.qn[k] & 3) * (size_t)A.ring_cap + ca.slot[k]], ca.Mbar[k]);
        }
        wave_sync();
    }
    const bool src_owner = (pc.kind == 0) || (pc.oct == 0 && (pc.dom < 0 || pc.dom == 2));
    if (src_owner && lane == 0) {
        double nb, q1;
        source_cell_adjoint_nodes<false>(NodeArray{A.n64}, A.tp, A.sigma0, A.alpha, Q, n_s, A.gbar[cs], &nb, &q1);
        nb_src += nb;
        qb += q1;
    }
    // wave sums
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        nb_src += __shfl_xor(nb_src, off, 64);
        qb += __shfl_xor(qb, off, 64);
    }
    if (lane == 0) {
        if (nb_src != 0.0) unsafeAtomicAdd(&A.nbar[cs], nb_src);
        if (qb != 0.0) unsafeAtomicAdd(&A.qbar[src], qb / Q);
    }
}

template <int TYPE>
__global__ __launch_bounds__(512) void adj_wave(AdjArgs A)
{
    extern __shared__ __align__(16) char smem[];
    if (A.seg[TYPE + 1] == A.seg[TYPE]) return;   // no sources of this kind
    const TabNode *T = A.tab;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    char *region = smem + (size_t)wave * A.region_bytes;
    double *store = A.store + (size_t)(blockIdx.x * waves + wave) * A.store_stride;
    constexpr int npieces = TYPE == 0 ? 1 : (TYPE == 1 ? 8 : 24);
    const int base = A.seg[TYPE];
    const int nitems = (A.seg[TYPE + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (;;) {
        const int item = next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = A.order[base + item / npieces];
        adjoint_piece_wave<TYPE>(A, T, region, store, src, item % npieces, lane);
    }
}

// ---- layer pieces --------------------------------------------------------
// One wave per pyramid, in two passes.
//  (F) Unless the forward kept the pyramid's column record: the columns layer
//      by layer, in place in the LDS buffer as in the forward kernel, every
//      cell's layer-buffer entry written to the record in the wave's scratch
//      together with each chunk's mask of cells with a rate.
//  (R) Layers from the outermost inward, each layer's rectangle in chunks
//      from the first to the last: every cell takes and clears its slot in
//      the LDS adjoint buffer (the adjoint of its exit column, pushed by its
//      consumers).  The cells with work (an adjoint, or a rate) are gathered
//      into full batches of 64 by an LDS queue.  A batch recomputes the cells'
//      interpolation from the record's entries of layer m - 1, evaluates the
//      FP64 rate derivatives of those with a rate, adds alpha ds times the
//      total adjoint to dL/dn_HI with one atomic, and pushes the entry
//      column's adjoint through the interpolation weights to the neighbours'
//      slots with LDS atomics.  A neighbour slot precedes the pushing cell in
//      (u, v) order, so it was already taken in this layer.  A layer without
//      a rate that no cell pushed to is left out at once: no rate depends on
//      its cells.
// Evaluating the rate's terms where the interpolation is at hand needs one
// evaluation and one atomic per cell (250^3, 10^5 sources of radii 5 to 40: 141
// ms -> 103 with the column pass in its new form and the cells with work
// gathered; about 44 in (F), 42 in (R) without the derivatives, 17 for them);
// evaluating them in (F) or in the forward took a second queue, a second atomic, and 8 (in the forward: 24)
// more bytes per cell with a rate out and back.
// The tables are read through the caches (only cells with a rate use them),
// which leaves the LDS to the per-wave buffers.
__device__ __forceinline__ void wave_sync_global()
{
    // this wave's global stores complete before its later global loads by
    // other lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <bool TEAM>
__device__ __forceinline__ void team_sync_global()
{
    if (TEAM) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
        wave_sync_global();
    }
}

constexpr int kAdjQueue = 128;   // queue entries per wave

// The rate masks of chunks c0 .. c0 + 63 of a layer (first chunk at choff),
// one per lane, held in registers.
__device__ __forceinline__ uint64_t load_masks(const LayerRecord &rec, long choff, int c0, int nch, int lane)
{
    uint32_t lo = 0, hi = 0;
    if (c0 + lane < nch) {
        const uint64_t mk = rec.lit[choff + c0 + lane];
        lo = (uint32_t)mk;
        hi = (uint32_t)(mk >> 32);
    }
    // without this the compiler turns every readlane of the masks back into
    // a global load per chunk
    asm volatile("" : "+v"(lo), "+v"(hi));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t mask_of_chunk(uint64_t masks, int c)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(masks >> 32), c & 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)masks, c & 63);
}

// Bytes of a team's buffers, geometry and flags (the queues follow).
__host__ __device__ constexpr size_t adj_team_shared_bytes(int S)
{
    return (2 * ((size_t)(S + 1) * (S + 1) * sizeof(double) + (size_t)S * sizeof(GeoRow)) + 3 * sizeof(int) + 15) & ~(size_t)15;
}

// LDS of a wave: one buffer (the columns in (F), the adjoint slots in (R)),
// the queue of cells with work, the table of factors and index terms; sq: the
// work-group's table of roots.
struct AdjLds {
    SweepLds sweep;
    const double *sq;
    double *buf;
    double *qT;     // adjoint of the cell's exit column
    int *quv;       // u | v << 8, bit 16: the cell has a rate
    GeoRow *geo;
    int *flag;      // TEAM: see adjoint_layer_piece
};

// The reverse pass of one cell: the adjoint Tin of its exit column and, with gb
// = dL/dGamma (0: no rate), its rate's terms; what it pushes to its neighbours
// in layer m - 1 (entries e0 .. e3), its entry column's and its own adjoint and
// its share of dL/dQ.
struct AdjCell {
    double b0, b1, b2, b3;   // pushes
    double Tin, Tn, q;
};

template <bool FAST>
__device__ __forceinline__ void adjoint_cell(const AdjArgs &A, const LayerX &X, const NodeArray &nodes, int m,
                                             double coef, double ads, int r2, const Geo &gu, const Geo &gv, double e0,
                                             double e1, double e2, double e3, double gb, double nhi, double Tin,
                                             AdjCell &C)
{
    C.q = 0.0;
    const double s0 = gu.om * gv.om, s1 = gu.a * gv.om, s2 = gu.om * gv.a, s3 = gu.a * gv.a;
    // t_in, and the derivatives b_n of t_in by the neighbours' t
    double t, b0, b1, b2, b3;
    if (m == 1) {
        t = X.reading == 0 ? X.half_n * (X.sigma0 * ads) : X.half_tau;
        b0 = b1 = b2 = b3 = 0.0;
    } else if (__ballot(!all_thick(e0, e1, e2, e3)) == 0) {
        // all thick: t_in = 1 / W, W = sum s e; b = s e^2 / W^2
        b0 = s0 * e0;
        b1 = s1 * e1;
        b2 = s2 * e2;
        b3 = s3 * e3;
        t = rcp_f64((b0 + b1) + (b2 + b3));
        const double k = t * t;
        b0 *= e0 * k;
        b1 *= e1 * k;
        b2 *= e2 * k;
        b3 *= e3 * k;
    } else {
        // f = e or 1 / tau_w; b = s f / W, for a thick neighbour times t_in f
        const double f0 = e0 > 0.0 ? e0 : X.inv_tw, f1 = e1 > 0.0 ? e1 : X.inv_tw;
        const double f2 = e2 > 0.0 ? e2 : X.inv_tw, f3 = e3 > 0.0 ? e3 : X.inv_tw;
        b0 = s0 * f0;
        b1 = s1 * f1;
        b2 = s2 * f2;
        b3 = s3 * f3;
        const double iW = rcp_f64((b0 + b1) + (b2 + b3));
        t = iW * (s0 * (e0 > 0.0 ? 1.0 : -e0 * X.inv_tw) + s1 * (e1 > 0.0 ? 1.0 : -e1 * X.inv_tw) +
                  s2 * (e2 > 0.0 ? 1.0 : -e2 * X.inv_tw) + s3 * (e3 > 0.0 ? 1.0 : -e3 * X.inv_tw));
        b0 *= iW * (e0 > 0.0 ? t * e0 : 1.0);
        b1 *= iW * (e1 > 0.0 ? t * e1 : 1.0);
        b2 *= iW * (e2 > 0.0 ? t * e2 : 1.0);
        b3 *= iW * (e3 > 0.0 ? t * e3 : 1.0);
    }
    // N_out = N_in + dN: both receive the exit column's adjoint,
    // and the rate adds its own parts
    double Tn = Tin;
    if (gb != 0.0) {
        double D, Da, Ddt;
        const TabParams tp = reload_arg<TabParams>(offsetof(AdjArgs, tp));
        rate_derivs_nodes<FAST>(nodes, tp, t, nhi * (X.sigma0 * ads), &D, &Da, &Ddt);
        const double k = -gb * coef * rcp_f64((double)r2);
        C.q = k * D;
        Tin += k * Da * X.sigma0;
        Tn += k * Ddt * X.sigma0;
    }
    C.b0 = Tin * b0;
    C.b1 = Tin * b1;
    C.b2 = Tin * b2;
    C.b3 = Tin * b3;
    C.Tin = Tin;
    C.Tn = Tn;
}

// TEAM: the work-group's waves take a layer's chunks in turn, in both passes.
// In (R) a layer's slots are taken from one buffer and the pushes go to the
// other; W.flag[3] tells all waves that a layer had a push, in turn (a flag is
// cleared a layer before it is used and two after it was read).
template <bool KEPT, bool FAST, bool TEAM>
__device__ __forceinline__ void adjoint_layer_piece(const AdjArgs &A, const AdjLds &W, Team team, char *scratch,
                                                    int src, int p, int lane)
{
    const int w0 = TEAM ? team.w : 0, T = TEAM ? team.T : 1;
    const int tid = w0 * 64 + lane, nt = T * 64;
    const bool first = w0 == 0 && lane == 0;
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
    const double *gbar = L.transposed ? A.gbar_T : A.gbar;
    double *nbar = L.transposed ? A.nbar_T : A.nbar;
    const double coef = uniform(Q * A.coef_unit);
    const int S = A.lay_S;
    const LayerRecord rec = layer_record_at(
        KEPT ? (char *)A.kept + ((size_t)src * 24 + p) * A.rec_piece_bytes : scratch, A.rec_cap, 0);
    const int Mx = min(uniform(isqrt_floor(Rsq)), L.ext_d);
    double *buf = W.buf;
    GeoRow *geo = W.geo;
    sweep_index_terms<TEAM>(L, N, W.sweep, team, lane);   // (every pass)

    // ---- (F), every layer; with the early exit only up to the first layer
    // whose cells all leave opaque (layer_opaque): later layers have no rate
    // and no adjoint.  Kept records hold the layers their forward swept.
    double nb_src = 0.0, qb = 0.0;
    long off = 0, choff = 0;   // the record's cells and chunks of layers 1 .. Mt
    int Mt = Mx;   // the last layer (R) visits
    if (KEPT) {
        const int ml = uniform((int)rec.lit[A.rec_cap / 64 + A.Mcap]);
        Mt = ml < Mx ? ml : Mx;
        for (int m = 1; m <= Mt; ++m) {
            const int t = layer_rect_uniform(L.ext_u, L.ext_v, Rsq, m).total;
            off += t;
            choff += (t + 63) / 64;
        }
    } else if (Mx >= 1) {
        bool opq = true;   // every cell of layer m so far leaves opaque
        sweep_layers<TEAM>(
            L, X, W.sweep, team, Rsq, Mx, Mt, A.tp.tau_hi, A.lc.inv_hi, lane,
            [&](const SweepChunk &k) {
                if (k.in) rec.h[off + k.c * 64 + lane] = k.h;
                const uint64_t mask = ballot(k.in & k.below & layer_owned(L, k.m, k.u, k.v));
                if (lane == 0 && k.any) rec.lit[choff + k.c] = mask;
                if (!TEAM && A.early_exit) opq = opq && ballot(k.in && entry_below(k.h, A.lc.opaque, A.lc.inv_opq)) == 0;
            },
            [&](int m, int total) {
                off += total;
                choff += (total + 63) / 64;
                if (!TEAM && A.early_exit && opq) Mt = m;
                opq = true;
            });
        team_sync_global<TEAM>();
    }
    const int P2 = (S + 1) * (S + 1);
    for (int k = tid; k < (TEAM ? 2 * P2 : S * S); k += nt) buf[k] = 0.0;   // the adjoint slots
    if (TEAM && tid < 3) W.flag[tid] = 0;
    int turn = 0;   // of the flags
    team_sync_global<TEAM>();

    // ---- (R)
    const NodeArray nodes{A.n64};
    bool pushed = false;   // a cell of layer m + 1 pushed to layer m's slots
    for (int m = Mt; m >= 1; --m) {
        const LayerRect r = layer_rect_uniform(L.ext_u, L.ext_v, Rsq, m);
        const int nch = (r.total + 63) / 64;
        off -= r.total;    // first cell of layer m in the record
        choff -= nch;      // its first chunk
        uint64_t masks = load_masks(rec, choff, 0, nch, lane);
        if (!pushed && nch <= 64 && __ballot(masks != 0) == 0) continue;   // no rate depends on this layer
        // entries of layer m - 1 (its rectangle precedes layer m's)
        const LayerRect rp = layer_rect_uniform(L.ext_u, L.ext_v, Rsq, m >= 2 ? m - 1 : 1);
        const double *Hprev = rec.h + (m >= 2 ? off - rp.total : 0);
        // this layer's geometry (the previous layer's readers are done)
        const double inv_m = rcp_f64((double)m), am = X.alpha * inv_m;
        const int m2 = m * m;
        const uint32_t idx_d = layer_idx_d(L, N, m);
        for (int k = tid; k < S; k += nt) geo[k].g = layer_geo(m, inv_m, k);
        double *take = TEAM && (m & 1) ? buf + P2 : buf, *give = TEAM && !(m & 1) ? buf + P2 : buf;
        const int next = turn == 2 ? 0 : turn + 1;
        if (TEAM && tid == 0) W.flag[next] = 0;
        team_sync<TEAM>();
        int qh = 0, qn = 0;   // the queue: qn cells from ring position qh
        bool any = false;
        RectWalk w;
        w.init(r, tid, nt);
        // the wave's chunks, then a last round for the cells left in the queue
        int mbase = 0;   // masks: of chunks mbase .. mbase + 63
        for (int c = w0, last = 0; !last; c += T) {
            last = c >= nch;
            if (!last) {
                if (c >= mbase + 64) {
                    mbase = c & ~63;
                    masks = load_masks(rec, choff, mbase, nch, lane);
                }
                const int u = w.u, v = w.v;
                const bool act = (u < r.nu) & (mul24(u, u) + mul24(v, v) <= r.rem);
                const bool lit = act && ((mask_of_chunk(masks, c) >> lane) & 1);
                double Tin = 0.0;
                if (pushed && act) {
                    double *slot = take + mul24(u, S) + v;
                    Tin = *slot;
                    *slot = 0.0;
                }
                w.up();
                const uint64_t need = __ballot(lit || Tin != 0.0);
                if (need == 0) continue;
                any = true;
                wave_sync();
                if (lit || Tin != 0.0) {
                    const unsigned k = (unsigned)(qh + qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u))) &
                                       (unsigned)(kAdjQueue - 1);
                    W.qT[k] = Tin;
                    W.quv[k] = u | (v << 8) | (lit ? 1 << 16 : 0);
                }
                qn += __popcll(need);
                wave_sync();
                if (qn < 64) continue;
            }
            const int cnt = qn < 64 ? qn : 64;
            const bool run = lane < cnt;
            double Tin = 0.0;
            int u = 0, v = 0;
            bool lit = false;
            if (run) {
                const unsigned k = (unsigned)(qh + lane) & (unsigned)(kAdjQueue - 1);
                const int uv = W.quv[k];
                Tin = W.qT[k];
                u = uv & 0xff;
                v = (uv >> 8) & 0xff;
                lit = (uv >> 16) != 0;
            }
            qh = (qh + cnt) & (kAdjQueue - 1);
            qn -= cnt;
            if (run) {
                const int r2 = m2 + mul24(u, u) + mul24(v, v);
                const double ads = (A.sq_n ? W.sq[r2] : sqrt_fast((double)r2)) * am;   // alpha ds
                const uint32_t cp = idx_d + geo[u].iu + geo[v].iv;
                const Geo gu = geo[u].g, gv = geo[v].g;
                // the neighbours (u, v), (u - 1, v), (u, v - 1), (u - 1, v - 1) of
                // layer m - 1; one of zero weight may lie outside it and is
                // replaced by the one next to it
                const int ua = u < m ? u : m - 1, ub = u > 0 ? u - 1 : 0;
                const int va = v < m ? v : m - 1, vb = v > 0 ? v - 1 : 0;
                double e0 = 0.0, e1 = 0.0, e2 = 0.0, e3 = 0.0;
                if (m >= 2) {
                    const double *ra = Hprev + mul24(ua, rp.wv), *rb = Hprev + mul24(ub, rp.wv);
                    e0 = ra[va];
                    e1 = rb[va];
                    e2 = ra[vb];
                    e3 = rb[vb];
                }
                double gb = 0.0, nhi = 0.0;
                if (lit) {
                    gb = gbar[cp];
                    nhi = X.nHI[cp];
                }
                AdjCell C;
                adjoint_cell<FAST>(A, X, nodes, m, coef, ads, r2, gu, gv, e0, e1, e2, e3, gb, nhi, Tin, C);
                qb += C.q;
                if (m >= 2) {
                    double *ra = give + mul24(ua, S), *rb = give + mul24(ub, S);
                    atomicAdd(&ra[va], C.b0);
                    atomicAdd(&rb[va], C.b1);
                    atomicAdd(&ra[vb], C.b2);
                    atomicAdd(&rb[vb], C.b3);
                } else {
                    nb_src += C.Tin * (X.reading == 0 ? ads * 0.5 : X.alpha * 0.5);
                }
                const double nb = C.Tn * ads;
                if (nb != 0.0) unsafeAtomicAdd(&nbar[cp], nb);
            }
            wave_sync();
        }
        if (TEAM) {
            if (any && lane == 0) W.flag[turn] = 1;
            __syncthreads();
            any = uniform(W.flag[turn]) != 0;
            turn = next;
        }
        pushed = any;
    }
    if (p == 3 * 0 + 2 && first) {   // the source cell, once per source
        double nb, q1;
        source_cell_adjoint_nodes<FAST>(nodes, A.tp, A.sigma0, A.alpha, Q, n_s, A.gbar[cs], &nb, &q1);
        nb_src += nb;
        qb += q1;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        nb_src += __shfl_xor(nb_src, o, 64);
        qb += __shfl_xor(qb, o, 64);
    }
    if (lane == 0) {
        if (nb_src != 0.0) unsafeAtomicAdd(&A.nbar[cs], nb_src);
        if (qb != 0.0) unsafeAtomicAdd(&A.qbar[src], qb / Q);
    }
}

template <bool KEPT, bool FAST>
__global__ __launch_bounds__(64 * kAdjLayerWaves) void adj_layer(AdjArgs A)
{
    extern __shared__ __align__(16) char smem[];
    constexpr int TYPE = 3, npieces = 24;
    const bool direct = A.items > 0;   // the pyramids in turn, else from the counters
    if (!direct && A.seg[TYPE + 1] == A.seg[TYPE]) return;   // no sources of this kind
    // the work-group's table of square roots, when the launch gives one
    // (every pass takes a cell's root from it)
    double *sq = (double *)smem;
    for (int k = threadIdx.x; k < A.sq_n; k += blockDim.x) sq[k] = sqrt((double)k);
    __syncthreads();
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    AdjLds W;
    W.sq = sq;
    W.sweep.S = A.lay_S;
    W.sweep.sq = 0;
    W.sweep.sq_n = A.sq_n;
    W.sweep.lay = (A.sq_n ? (int)layer_sqrt_bytes(A.sq_n - 1) : 0) + wave * A.region_bytes;
    W.sweep.geo = W.sweep.lay + 8 * (A.lay_S + 1) * (A.lay_S + 1) + kAdjQueue * (int)(sizeof(double) + sizeof(int));
    W.buf = (double *)(smem + W.sweep.lay);
    W.qT = W.buf + (size_t)(A.lay_S + 1) * (A.lay_S + 1);
    W.quv = (int *)(W.qT + kAdjQueue);
    W.geo = (GeoRow *)(W.quv + kAdjQueue);
    W.flag = nullptr;
    char *scratch = (char *)(A.store + (size_t)(blockIdx.x * waves + wave) * A.store_stride);
    const int base = direct ? 0 : A.seg[TYPE];
    const int nitems = direct ? A.items : (A.seg[TYPE + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (int turn = 0;; ++turn) {
        const int item = direct ? (turn * (int)gridDim.x + (int)blockIdx.x) * waves + wave
                                : next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = direct ? item / npieces : uniform(A.order[base + item / npieces]);
        adjoint_layer_piece<KEPT, FAST, false>(A, W, Team{0, 1}, scratch, src, item % npieces, lane);
    }
}

// One work-group per pyramid (see fwd_team): 64^3, 64 sources of radius 20 with
// kept records, two waves to a pyramid, 83 us against 130 by one wave each.
template <bool KEPT, bool FAST>
__global__ __launch_bounds__(64 * kAdjLayerWaves) void adj_team(AdjArgs A)
{
    extern __shared__ __align__(16) char smem[];
    const Team team{uniform((int)threadIdx.x >> 6), (int)blockDim.x >> 6};
    AdjLds W;
    W.sq = nullptr;
    W.sweep.S = A.lay_S;
    W.sweep.sq = 0;
    W.sweep.sq_n = 0;
    W.sweep.lay = 0;
    W.sweep.geo = 2 * 8 * (A.lay_S + 1) * (A.lay_S + 1);
    W.buf = (double *)smem;
    W.geo = (GeoRow *)(smem + W.sweep.geo);
    W.flag = (int *)(W.geo + 2 * A.lay_S);
    char *queues = smem + adj_team_shared_bytes(A.lay_S);
    W.qT = (double *)queues + team.w * kAdjQueue;
    W.quv = (int *)((double *)queues + team.T * kAdjQueue) + team.w * kAdjQueue;
    char *scratch = (char *)(A.store + (size_t)blockIdx.x * A.store_stride);
    const int item = blockIdx.x;
    adjoint_layer_piece<KEPT, FAST, true>(A, W, team, scratch, item / 24, item % 24, threadIdx.x & 63);
}

// ---- group pieces --------------------------------------------------------
// Several pyramids of a small source by one wave, as sweep_group: both passes
// of adjoint_layer_piece over layers whose rectangles follow each other, slots
// and record entries numbered alike.  Never with kept records (the forward
// keeps none of these sources).
template <bool FAST>
__device__ __forceinline__ void adjoint_group_piece(const AdjArgs &A, const GroupLds &W, int qT, int quv, char *scratch,
                                                    int src, int part, int lane)
{
    const int N = A.N;
    const int si = uniform(A.ijk[3 * src]), sj = uniform(A.ijk[3 * src + 1]), sk = uniform(A.ijk[3 * src + 2]);
    const float R = A.R ? A.R[src] : A.R_cap;
    if (!(R >= 0.f && R <= A.R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 ||
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
    const LayerRecord rec = layer_record_at(scratch, A.rec_cap, 0);
    const int Mx = uniform(isqrt_floor(Rsq));   // within the box: see radii_of
    const int P = W.S + 1, P8 = 8 * P, PP8 = P8 * P;
    const NodeArray nodes{A.n64};
    double nb_src = 0.0, qb = 0.0;
    if (Mx >= 1) {
        group_tables(W, part * W.G, si, sj, sk, N, lane);
        // ---- (F)
        long off = 0, choff = 0;
        sweep_group(X, A.nHI_T, W, Rsq, Mx, A.tp.tau_hi, A.lc.inv_hi, lane, [&](const GroupChunk &k) {
            if (k.in) rec.h[off + k.c * 64 + lane] = k.h;
            const uint64_t mask = ballot(k.in & k.below & group_owned(k.flags, k.m, k.u, k.v));
            if (lane == 0) rec.lit[choff + k.c] = mask;
            if (k.c == 0) {
                off += k.cells;
                choff += (k.cells + 63) / 64;
            }
        });
        wave_sync_global();
        for (int k = lane; k < W.G * P * P; k += 64) lds<double>(W.lay + 8 * k) = 0.0;   // the adjoint slots
        wave_sync_global();
        // ---- (R)
        bool pushed = false;   // a cell of layer m + 1 pushed to layer m's slots
        for (int m = Mx; m >= 1; --m) {
            const LayerRect r = layer_rect_uniform(Mx, Mx, Rsq, m);
            const int cells = W.G * r.total, nch = (cells + 63) / 64;   // at most 16 chunks (kGroup)
            off -= cells;
            choff -= nch;
            const uint64_t masks = load_masks(rec, choff, 0, nch, lane);
            if (!pushed && __ballot(masks != 0) == 0) continue;   // no rate depends on this layer
            const LayerRect rp = layer_rect_uniform(Mx, Mx, Rsq, m >= 2 ? m - 1 : 1);
            const double *Hprev = rec.h + (m >= 2 ? off - W.G * rp.total : 0);
            const float inv_t = rcp_approx((float)r.total), inv_w = rcp_approx((float)r.wv);
            const double am = X.alpha * rcp_f64((double)m);
            const int m2 = m * m, geo = W.geo + (int)sizeof(Geo) * W.geo_S * (m - 1);
            int qh = 0, qn = 0;   // the queue: qn cells from ring position qh
            bool any = false;
            // chunks 0 .. nch - 1, then a last round for the cells left in the queue
            for (int c = 0; c <= nch; ++c) {
                if (c < nch) {
                    const int g = c * 64 + lane;
                    const int pl = (int)(((float)g + 0.5f) * inv_t), l = g - mul24(pl, r.total);
                    const int u = (int)(((float)l + 0.5f) * inv_w), v = l - mul24(u, r.wv);
                    const bool act = (g < cells) & (mul24(u, u) + mul24(v, v) <= r.rem);
                    const bool lit = act && ((mask_of_chunk(masks, c) >> lane) & 1);
                    double Tin = 0.0;
                    if (pushed && act) {
                        const int slot = W.lay + mul24(pl, PP8) + mul24(u, P8) + 8 * v;
                        Tin = lds<double>(slot);
                        lds<double>(slot) = 0.0;
                    }
                    const uint64_t need = __ballot(lit || Tin != 0.0);
                    if (need == 0) continue;
                    any = true;
                    wave_sync();
                    if (lit || Tin != 0.0) {
                        const int k = (qh + qn + rank_in(need)) & (kAdjQueue - 1);
                        lds<double>(qT + 8 * k) = Tin;
                        lds<int>(quv + 4 * k) = u | (v << 8) | (pl << 16) | (lit ? 1 << 24 : 0);
                    }
                    qn += __popcll(need);
                    wave_sync();
                    if (qn < 64) continue;
                }
                const int cnt = qn < 64 ? qn : 64;
                const int at = (qh + lane) & (kAdjQueue - 1);
                qh = (qh + cnt) & (kAdjQueue - 1);
                qn -= cnt;
                if (lane < cnt) {
                    const int uv = lds<int>(quv + 4 * at);
                    double Tin = lds<double>(qT + 8 * at);
                    const int u = uv & 0xff, v = (uv >> 8) & 0xff, pl = (uv >> 16) & 0xff;
                    const bool lit = (uv >> 24) != 0;
                    const GroupRow row = lds<GroupRow>(W.row + (int)sizeof(GroupRow) * pl);
                    const bool tr = (row.flags & kGroupT) != 0;
                    const uint32_t cp = lds<uint32_t>(row.d + 4 * m) + lds<uint32_t>(row.u + 4 * u) +
                                        lds<uint32_t>(row.v + 4 * v);
                    const int r2 = m2 + mul24(u, u) + mul24(v, v);
                    const double ads = lds<double>(W.sq + 8 * r2) * am;   // alpha ds
                    const Geo gu = lds<Geo>(geo + (int)sizeof(Geo) * u), gv = lds<Geo>(geo + (int)sizeof(Geo) * v);
                    const int ua = u < m ? u : m - 1, ub = u > 0 ? u - 1 : 0;
                    const int va = v < m ? v : m - 1, vb = v > 0 ? v - 1 : 0;
                    double e0 = 0.0, e1 = 0.0, e2 = 0.0, e3 = 0.0;
                    if (m >= 2) {
                        const double *base = Hprev + mul24(pl, rp.total);
                        const double *ra = base + mul24(ua, rp.wv), *rb = base + mul24(ub, rp.wv);
                        e0 = ra[va];
                        e1 = rb[va];
                        e2 = ra[vb];
                        e3 = rb[vb];
                    }
                    double gb = 0.0, nhi = 0.0;
                    if (lit) {
                        gb = (tr ? A.gbar_T : A.gbar)[cp];
                        nhi = (tr ? A.nHI_T : A.nHI)[cp];
                    }
                    AdjCell C;
                    adjoint_cell<FAST>(A, X, nodes, m, coef, ads, r2, gu, gv, e0, e1, e2, e3, gb, nhi, Tin, C);
                    qb += C.q;
                    if (m >= 2) {
                        const int base = W.lay + mul24(pl, PP8);
                        const int ra = base + mul24(ua, P8), rb = base + mul24(ub, P8);
                        atomicAdd(&lds<double>(ra + 8 * va), C.b0);
                        atomicAdd(&lds<double>(rb + 8 * va), C.b1);
                        atomicAdd(&lds<double>(ra + 8 * vb), C.b2);
                        atomicAdd(&lds<double>(rb + 8 * vb), C.b3);
                    } else {
                        nb_src += C.Tin * (X.reading == 0 ? ads * 0.5 : X.alpha * 0.5);
                    }
                    const double nb = C.Tn * ads;
                    if (nb != 0.0) unsafeAtomicAdd(&(tr ? A.nbar_T : A.nbar)[cp], nb);
                }
                wave_sync();
            }
            pushed = any;
        }
    }
    if (part == 0 && lane == 0) {   // the source cell, once per source
        double nb, q1;
        source_cell_adjoint_nodes<FAST>(nodes, A.tp, A.sigma0, A.alpha, Q, n_s, A.gbar[cs], &nb, &q1);
        nb_src += nb;
        qb += q1;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        nb_src += __shfl_xor(nb_src, o, 64);
        qb += __shfl_xor(qb, o, 64);
    }
    if (lane == 0) {
        if (nb_src != 0.0) unsafeAtomicAdd(&A.nbar[cs], nb_src);
        if (qb != 0.0) unsafeAtomicAdd(&A.qbar[src], qb / Q);
    }
}

// Bytes of the work-group's tables and of a wave's region (one class).
static size_t adj_group_shared_bytes(const GroupClasses &c)
{
    return ((size_t)(c.Rsq[0] + 1) * sizeof(double) + (size_t)isqrt_floor(c.Rsq[0]) * c.S[0] * sizeof(Geo) + 15) & ~(size_t)15;
}
static size_t adj_group_wave_bytes(const GroupClasses &c)
{
    return ((size_t)c.G[0] * ((size_t)(c.S[0] + 1) * (c.S[0] + 1) * sizeof(double) + sizeof(GroupRow)) +
            12 * (size_t)(isqrt_floor(c.Rsq[0]) + 1) * sizeof(uint32_t) + kAdjQueue * (sizeof(double) + sizeof(int)) + 31) &
           ~(size_t)15;
}
size_t adj_group_lds_bytes(const GroupClasses &c, int waves)
{
    return adj_group_shared_bytes(c) + (size_t)waves * adj_group_wave_bytes(c);
}

template <bool FAST>
__global__ __launch_bounds__(1024) void adj_group(AdjArgs A)
{
    if (A.seg[A.type + 1] == A.seg[A.type]) return;   // no sources of this kind
    const int Rsq = A.grp.Rsq[0], M = isqrt_floor(Rsq);
    GroupLds W;
    W.S = W.geo_S = A.grp.S[0];
    W.K = M + 1;
    W.G = A.grp.G[0];
    W.sq = 0;
    W.geo = 8 * (Rsq + 1);
    for (int k = threadIdx.x; k <= Rsq; k += blockDim.x) lds<double>(8 * k) = sqrt((double)k);
    for (int k = threadIdx.x; k < M * W.S; k += blockDim.x) {
        const int m = k / W.S + 1;
        lds<Geo>(W.geo + (int)sizeof(Geo) * k) = layer_geo(m, rcp_f64((double)m), k % W.S);
    }
    __syncthreads();
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    const int qT = A.grp_shared + wave * A.region_bytes, quv = qT + 8 * kAdjQueue;
    W.lay = quv + 4 * kAdjQueue;
    W.row = (W.lay + W.G * 8 * (W.S + 1) * (W.S + 1) + 15) & ~15;
    W.term = W.row + W.G * (int)sizeof(GroupRow);
    char *scratch = (char *)(A.store + (size_t)(blockIdx.x * waves + wave) * A.store_stride);
    const int npieces = 24 / W.G, base = A.seg[A.type], nitems = (A.seg[A.type + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (;;) {
        const int item = next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = uniform(A.order[base + item / npieces]);
        adjoint_group_piece<FAST>(A, W, qT, quv, scratch, src, item % npieces, lane);
    }
}

// What an adjoint with layer pieces starts from, in one pass over the fields.
// dL/dn_HI of the pieces with dominant axis k is accumulated in the [k][i][j]
// layout: that layout's n_HI and dL/dGamma, the zeroed accumulators of both
// layouts, and the cleared dL/dQ and control block (one 32 x 32 (j, k) tile of
// one i plane per work-group; the work-groups share the last two).
constexpr int kTile = 32;
__global__ __launch_bounds__(256) void adj_layer_prologue_kernel(
    const float *__restrict__ nH, const float *__restrict__ xHI, const double *__restrict__ gbar, AdjBufs B, long nsrc,
    int *ctl, int nctl, int N)
{
    __shared__ double tn[kTile][kTile + 1], tg[kTile][kTile + 1];
    const int k0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile, i = blockIdx.z;
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;
    for (int jj = ty; jj < kTile; jj += 8) {
        const int j = j0 + jj, k = k0 + tx;
        if (j < N && k < N) {
            const size_t c = ((size_t)i * N + j) * N + k;
            if (B.nHI_T) {   // NULL: both layouts still in place from the forward
                const double n = (double)nH[c] * (double)xHI[c];
                tn[jj][tx] = n;
                B.nHI[c] = n;
            }
            tg[jj][tx] = gbar[c];
            B.nbar[c] = 0.0;
        }
    }
    const long block = ((long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const long threads = (long)gridDim.x * gridDim.y * gridDim.z * 256, me = block * 256 + threadIdx.x;
    for (long k = me; k < nctl; k += threads) ctl[k] = 0;
    if (B.qbar)
        for (long k = me; k < nsrc; k += threads) B.qbar[k] = 0.0;
    __syncthreads();
    for (int kk = ty; kk < kTile; kk += 8) {
        const int k = k0 + kk, j = j0 + tx;
        if (j < N && k < N) {
            const size_t t = ((size_t)k * N + i) * N + j;
            if (B.nHI_T) B.nHI_T[t] = tn[tx][kk];
            B.gbar_T[t] = tg[tx][kk];
            B.nbar_T[t] = 0.0;
        }
    }
}

// dL/dn_H = x_HI g, dL/dx_HI = n_H g with g = dL/dn_HI from both layouts.
__global__ __launch_bounds__(256) void adj_transpose_finalize_kernel(
    const double *__restrict__ nbar, const double *__restrict__ nbar_T, const float *__restrict__ nH,
    const float *__restrict__ xHI, float *__restrict__ dnH, float *__restrict__ dxHI, int N,
    int accumulate)
{
    __shared__ double tile[kTile][kTile + 1];
    const int k0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile, i = blockIdx.z;
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;
    for (int kk = ty; kk < kTile; kk += 8) {
        const int k = k0 + kk, j = j0 + tx;
        if (j < N && k < N) tile[kk][tx] = nbar_T[((size_t)k * N + i) * N + j];
    }
    __syncthreads();
    for (int jj = ty; jj < kTile; jj += 8) {
        const int j = j0 + jj, k = k0 + tx;
        if (j < N && k < N) {
            const size_t c = ((size_t)i * N + j) * N + k;
            const double g = nbar[c] + tile[tx][jj];
            const float a = (float)(g * (double)xHI[c]);
            const float b = (float)(g * (double)nH[c]);
            dnH[c] = accumulate ? dnH[c] + a : a;
            dxHI[c] = accumulate ? dxHI[c] + b : b;
        }
    }
}

__global__ void adj_prologue_kernel(const float *__restrict__ nH, const float *__restrict__ xHI,
                                    double *__restrict__ nHI, double *__restrict__ nbar, long n3,
                                    double *__restrict__ qbar, long nsrc, int zero_q, int *ctl,
                                    int nctl)
{
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < n3; c += stride) {
        if (nHI) nHI[c] = (double)nH[c] * (double)xHI[c];   // NULL: still in place from the forward
        nbar[c] = 0.0;
    }
    if (zero_q)
        for (long s = blockIdx.x * (long)blockDim.x + threadIdx.x; s < nsrc; s += stride) qbar[s] = 0.0;
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < nctl; k += blockDim.x) ctl[k] = 0;
}

// dL/dn_H = x_HI dL/dn_HI, dL/dx_HI = n_H dL/dn_HI
__global__ void adj_finalize_kernel(const double *__restrict__ nbar, const float *__restrict__ nH,
                                    const float *__restrict__ xHI, float *__restrict__ dnH,
                                    float *__restrict__ dxHI, long n3, int accumulate)
{
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = blockIdx.x * (long)blockDim.x + threadIdx.x; c < n3; c += stride) {
        const double g = nbar[c];
        const float a = (float)(g * (double)xHI[c]);
        const float b = (float)(g * (double)nH[c]);
        dnH[c] = accumulate ? dnH[c] + a : a;
        dxHI[c] = accumulate ? dxHI[c] + b : b;
    }
}

// ---------------------------------------------------------------------------
size_t adj_region_bytes(int ring_cap, int row_cap, int shell_cap)
{
    const size_t b = 8 * (size_t)ring_cap * sizeof(double) +
                     (4 * (size_t)row_cap + 4 * ((size_t)row_cap + 1) + (size_t)shell_cap + 2) *
                         sizeof(int);
    return (b + 15) & ~(size_t)15;
}

static const void *adj_fn(int type)
{
    return type == 0 ? (const void *)adj_wave<0>
                     : (type == 1 ? (const void *)adj_wave<1> : (const void *)adj_wave<2>);
}

// fast: a fine and tame table (the general evaluations compiled out)
static const void *adj_layer_fn(bool kept, bool fast, bool team = false)
{
    if (team)
        return kept ? (fast ? (const void *)adj_team<true, true> : (const void *)adj_team<true, false>)
                    : (fast ? (const void *)adj_team<false, true> : (const void *)adj_team<false, false>);
    return kept ? (fast ? (const void *)adj_layer<true, true> : (const void *)adj_layer<true, false>)
                : (fast ? (const void *)adj_layer<false, true> : (const void *)adj_layer<false, false>);
}

hipError_t adj_configure(size_t max_lds)
{
    const int dyn = (int)max_lds - 64;
    for (int t = 0; t < 3; ++t)
        (void)hipFuncSetAttribute(adj_fn(t), hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    for (int f = 0; f < 2; ++f)
        (void)hipFuncSetAttribute(f ? (const void *)adj_group<true> : (const void *)adj_group<false>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    for (int f = 0; f < 8; ++f)
        (void)hipFuncSetAttribute(adj_layer_fn(f & 2, f & 1, f & 4), hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    (void)hipGetLastError();
    return hipSuccess;
}

hipError_t adj_occupancy(int type, int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, adj_fn(type), waves * 64, lds);
}

hipError_t launch_adj_prologue(hipStream_t st, const float *nH, const float *xHI, double *nHI,
                               double *nbar, long n3, double *qbar, long nsrc, int zero_q, int *ctl,
                               int nctl, int n_cu)
{
    hipLaunchKernelGGL(adj_prologue_kernel, dim3(n_cu * 8), dim3(256), 0, st, nH, xHI, nHI, nbar,
                       n3, qbar, nsrc, zero_q, ctl, nctl);
    return hipGetLastError();
}

static AdjArgs make_adj_args(const AdjLaunch &L)
{
    AdjArgs A;
    A.N = L.N;
    A.ex = make_extent(L.N);
    A.alpha = L.alpha;
    A.sigma0 = L.sigma0;
    A.coef_unit = L.sigma0 / (4.0 * M_PI * L.alpha * L.alpha);
    A.tau_w = L.tau_w;
    A.reading = L.reading;
    A.tp = L.tp;
    A.tab = L.tab;
    A.n64 = L.n64;
    A.nHI = L.nHI;
    A.gbar = L.gbar;
    A.nbar = L.nbar;
    A.qbar = L.qbar;
    A.ijk = L.ijk;
    A.Q = L.Q;
    A.R = L.R;
    A.R_cap = L.R_cap;
    A.order = L.order;
    A.seg = L.ctl + kCtlSeg;
    A.counter = L.ctl + kCtlCounter + kXcds * kCounterPad * L.type;
    A.err = L.err;
    A.ring_cap = L.ring_cap;
    A.row_cap = L.row_cap;
    A.shell_cap = L.shell_cap;
    A.region_bytes = 0;
    A.store = L.store;
    A.store_stride = L.store_stride;
    A.nHI_T = L.nHI_T;
    A.gbar_T = L.gbar_T;
    A.nbar_T = L.nbar_T;
    A.Mcap = 0;
    A.lay_S = 0;
    A.kept = L.kept;
    A.rec_piece_bytes = L.rec_piece_bytes;
    A.rec_cap = L.rec_cap;
    A.early_exit = L.early_exit ? 1 : 0;
    A.lc = make_layer_const(L.sigma0, L.alpha, L.tau_w, L.tp.tau_hi);
    A.sq_n = 0;
    A.items = 0;
    A.type = L.type;
    A.grp = L.grp;
    A.grp_shared = 0;
    return A;
}

hipError_t launch_adj_wave(hipStream_t st, const AdjLaunch &L)
{
    AdjArgs A = make_adj_args(L);
    A.region_bytes = (int)adj_region_bytes(L.ring_cap, L.row_cap, L.shell_cap);
    const size_t lds = (size_t)L.waves * A.region_bytes;
    switch (L.type) {
    case 0: hipLaunchKernelGGL(adj_wave<0>, dim3(L.grid), dim3(64 * L.waves), lds, st, A); break;
    case 1: hipLaunchKernelGGL(adj_wave<1>, dim3(L.grid), dim3(64 * L.waves), lds, st, A); break;
    default: hipLaunchKernelGGL(adj_wave<2>, dim3(L.grid), dim3(64 * L.waves), lds, st, A); break;
    }
    return hipGetLastError();
}

// Per-wave LDS of the layer adjoint: the buffer (the padded (S + 1) x (S + 1)
// layer buffer in (F), the S x S adjoint slots in (R)), the queue of cells
// with work, the table of factors and index terms.
size_t adj_layer_region_bytes(int S)
{
    return ((size_t)(S + 1) * (S + 1) * sizeof(double) + kAdjQueue * (sizeof(int) + sizeof(double)) +
            (size_t)S * sizeof(GeoRow) + 15) &
           ~(size_t)15;
}

hipError_t adj_layer_occupancy(bool kept, int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, adj_layer_fn(kept, true), waves * 64, lds);
}

hipError_t launch_adj_layer(hipStream_t st, const AdjLaunch &L, int Mcap, int S)
{
    AdjArgs A = make_adj_args(L);
    A.Mcap = Mcap;
    A.lay_S = S;
    A.region_bytes = (int)adj_layer_region_bytes(S);
    const int Rsq = (int)floor((double)L.R_cap * (double)L.R_cap);
    const size_t sqb = L.sq_table ? layer_sqrt_bytes(Rsq) : 0;
    A.sq_n = sqb ? Rsq + 1 : 0;
    const size_t lds = sqb + (size_t)L.waves * A.region_bytes;
    void *args[] = {&A};
    return hipLaunchKernel(adj_layer_fn(A.kept != nullptr, A.tp.fine && A.tp.tame), dim3(L.grid), dim3(64 * L.waves), args, lds, st);
}

static const void *adj_group_fn(bool fast) { return fast ? (const void *)adj_group<true> : (const void *)adj_group<false>; }

hipError_t adj_group_occupancy(int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, adj_group_fn(true), waves * 64, lds);
}

hipError_t launch_adj_group(hipStream_t st, const AdjLaunch &L)
{
    AdjArgs A = make_adj_args(L);
    A.region_bytes = (int)adj_group_wave_bytes(L.grp);
    A.grp_shared = (int)adj_group_shared_bytes(L.grp);
    void *args[] = {&A};
    return hipLaunchKernel(adj_group_fn(A.tp.fine && A.tp.tame), dim3(L.grid), dim3(64 * L.waves), args,
                           adj_group_lds_bytes(L.grp, L.waves), st);
}

size_t adj_team_bytes(int S, int T)
{
    return adj_team_shared_bytes(S) + (size_t)T * kAdjQueue * (sizeof(int) + sizeof(double));
}

// Every pyramid of the n_src sources, by T waves each: L.grid work-groups, one
// each if T > 1.
hipError_t launch_adj_direct(hipStream_t st, const AdjLaunch &L, int Mcap, int S, int T, int n_src)
{
    AdjArgs A = make_adj_args(L);
    A.Mcap = Mcap;
    A.lay_S = S;
    A.items = 24 * n_src;
    A.region_bytes = (int)adj_layer_region_bytes(S);
    const size_t lds = T > 1 ? adj_team_bytes(S, T) : (size_t)A.region_bytes;
    void *args[] = {&A};
    return hipLaunchKernel(adj_layer_fn(A.kept != nullptr, A.tp.fine && A.tp.tame, T > 1), dim3(L.grid), dim3(64 * T),
                           args, lds, st);
}

hipError_t launch_adj_layer_prologue(hipStream_t st, const float *nH, const float *xHI, const double *gbar,
                                     const AdjBufs &B, long nsrc, int *ctl, int nctl, int N)
{
    const dim3 grid((N + kTile - 1) / kTile, (N + kTile - 1) / kTile, N);
    hipLaunchKernelGGL(adj_layer_prologue_kernel, grid, dim3(256), 0, st, nH, xHI, gbar, B, nsrc, ctl, nctl, N);
    return hipGetLastError();
}

hipError_t launch_adj_transpose_finalize(hipStream_t st, const double *nbar, const double *nbar_T,
                                         const float *nH, const float *xHI, float *dnH, float *dxHI,
                                         int N, int accumulate)
{
    const dim3 grid((N + kTile - 1) / kTile, (N + kTile - 1) / kTile, N);
    hipLaunchKernelGGL(adj_transpose_finalize_kernel, grid, dim3(256), 0, st, nbar, nbar_T, nH, xHI,
                       dnH, dxHI, N, accumulate);
    return hipGetLastError();
}

hipError_t launch_adj_finalize(hipStream_t st, const double *nbar, const float *nH, const float *xHI,
                               float *dnH, float *dxHI, long n3, int accumulate, int n_cu)
{
    hipLaunchKernelGGL(adj_finalize_kernel, dim3(n_cu * 8), dim3(256), 0, st, nbar, nH, xHI, dnH,
                       dxHI, n3, accumulate);
    return hipGetLastError();
}

}  // namespace asora
