// asora_he.hip -- forward sweep with two absorbers, hydrogen and helium (the
// extension the paper plans, Sections 2 and 6), for gfx950.
//
// Every source is swept as layer pyramids (asora_dev.h), one wave per
// pyramid.  The layer buffer holds two columns per cell: the HI column as its
// layer-buffer entry (the optical-depth weights of the hydrogen method, on
// the HI column at the HI threshold) and the HeI column itself; both are
// interpolated with the same weights.  The spectrum is split into bands:
// band b has its own table (its photons that survive an optical depth taken
// at its lower edge, on its own node grid) and the cross-sections sH[b],
// sHe[b] of HI and HeI there, so that its optical depth is
// sH[b] N_HI + sHe[b] N_HeI.  A cell's rate of species i is
// Q sum_b s_i,b (-D_b) / (4 pi alpha^2 r^2), D_b the divided difference of
// band b's table over the cell's optical depths (eq. sugg for each band, the
// band's absorbed photons shared between the species in proportion to their
// in-cell optical depths).  Rates are accumulated in FP64 like the hydrogen
// rate; the tables are read through the caches.
#include "asora_dev.h"
#include "asora_internal.h"
#include "asora_sweep.h"

namespace asora {

struct HeArgs {
    int N;
    Extent ex;
    double alpha, sigma0;
    float tau_w;
    int reading;
    int nb;                     // bands
    const TabNode *tab;         // nb x n_tab nodes
    int n_tab;
    TabParams tp[kMaxBands];    // node grid (and end slope) of each band's table
    double sH[kMaxBands], sHe[kMaxBands];
    const double *nHI, *nHeI;       // [i][j][k]
    const double *nHI_T, *nHeI_T;   // [k][i][j]
    double *gH, *gHe, *gH_T, *gHe_T;
    const int32_t *ijk;
    const double *Q;
    const float *R;
    float R_cap;
    const int *order;
    const int *seg;
    int *counter;
    int *err;
    int src0, items;    // direct: the first source, the number of pyramids (0: from the counters)
    int lay_S;
    int region_bytes;
    LayerConst lc;
    int sq_n;
    double coef_unit;   // 1 / (4 pi alpha^2)
};

// Per-wave queue of cells with a rate: both entry columns, the cell index
// and (m << 16) | r^2 (r^2 < 2^16: the plan checks it).  The in-cell columns
// are recomputed by the batch exactly as the sweep formed them, which keeps
// the queue, and so the LDS per wave, small.
constexpr int kHeQueue = 128;

// LDS byte offsets of a wave: the queue's entry HI optical depth (as a
// layer-buffer entry), entry HeI column, cell index and mr; the two layer
// buffers; the table of GeoRows; the work-group's roots (at 0).
struct HeLds {
    int e, NinHe, cp, mr;
    int lay, layHe, geo;
    int S, sq_n;
};

__host__ __device__ constexpr int he_queue_bytes() { return kHeQueue * (int)(2 * sizeof(double) + 2 * sizeof(uint32_t)); }

// Rates of one queued cell (one lane): every band's divided difference,
// shared between the species by their cross-sections.  nH, nHe: the fields
// in the piece's layout.  FINE: every band's table is.
template <bool FINE>
__device__ __forceinline__ void he_rate(const HeArgs &A, const HeLds &W, int pos, double coef, const double *nH,
                                        const double *nHe, double inv_s0, double *gH, double *gHe)
{
    const double NH = entry_tau(lds<double>(W.e + 8 * pos)) * inv_s0, NHe = lds<double>(W.NinHe + 8 * pos);
    const uint32_t cp = lds<uint32_t>(W.cp + 4 * pos), mr = lds<uint32_t>(W.mr + 4 * pos);
    const int r2 = (int)(mr & 0xffffu), m = (int)(mr >> 16);
    const double n1 = nH[cp], n2 = nHe[cp];
    const double ds = (W.sq_n ? lds<double>(8 * r2) : sqrt_fast((double)r2)) * rcp_f64((double)m);
    const double dH = n1 * A.alpha * ds, dHe = n2 * A.alpha * ds;
    double sumH = 0.0, sumHe = 0.0;
    for (int b = 0; b < A.nb; ++b) {
        const double T = A.sH[b] * NH + A.sHe[b] * NHe;
        const double dT = A.sH[b] * dH + A.sHe[b] * dHe;
        const TabNode *tab = A.tab + (size_t)b * A.n_tab;
        const double nd = (double)(FINE ? neg_divdiff_fine(tab, A.tp[b], T, dT) : neg_divdiff(tab, A.tp[b], T, dT));
        sumH += A.sH[b] * nd;
        sumHe += A.sHe[b] * nd;
    }
    const double k = coef * (double)rcp_approx((float)r2);
    if (sumH > 0.0) unsafeAtomicAdd(&gH[cp], k * sumH);
    if (sumHe > 0.0) unsafeAtomicAdd(&gHe[cp], k * sumHe);
}

// The source cell: entry column 0, path half a cell, volume alpha^3.
__device__ void he_source_cell(const HeArgs &A, uint32_t cs, double Q)
{
    const double nH = A.nHI[cs], nHe = A.nHeI[cs];
    double GH = 0.0, GHe = 0.0;
    for (int b = 0; b < A.nb; ++b) {
        const double dT = (A.sH[b] * nH + A.sHe[b] * nHe) * A.alpha * 0.5;
        const double nd = (double)neg_divdiff(A.tab + (size_t)b * A.n_tab, A.tp[b], 0.0, dT);
        GH += A.sH[b] * nd;
        GHe += A.sHe[b] * nd;
    }
    const double k = Q / (2.0 * A.alpha * A.alpha);
    if (GH != 0.0) unsafeAtomicAdd(&A.gH[cs], k * GH);
    if (GHe != 0.0) unsafeAtomicAdd(&A.gHe[cs], k * GHe);
}

// As sweep_layers, with the helium field and buffer beside the hydrogen ones:
// by one wave in place, or by a team (layers of odd m use the second of each
// buffer and table, `odd` bytes further on).
template <bool FINE, bool TEAM>
__device__ __forceinline__ void sweep_layer_piece_he(const HeArgs &A, const HeLds &W, Team team, int src, int p, int lane)
{
    const int w0 = TEAM ? team.w : 0, T = TEAM ? team.T : 1, tid = w0 * 64 + lane, nt = T * 64;
    const bool first = w0 == 0 && lane == 0;
    const int N = A.N;
    const int si = uniform(A.ijk[3 * src]), sj = uniform(A.ijk[3 * src + 1]), sk = uniform(A.ijk[3 * src + 2]);
    const float R = A.R ? A.R[src] : A.R_cap;
    if (!(R >= 0.f && R <= A.R_cap) || si < 0 || si >= N || sj < 0 || sj >= N || sk < 0 || sk >= N) {
        if (first) atomicOr(A.err, 1);
        return;
    }
    const double Q = uniform(A.Q[src]);
    const int Rsq = uniform((int)floor((double)R * (double)R));
    const LayerPiece L = make_layer_piece(p, si, sj, sk, N, A.ex);
    const uint32_t cs = ((uint32_t)si * (uint32_t)N + (uint32_t)sj) * (uint32_t)N + (uint32_t)sk;
    LayerX X;
    X.N = N;
    X.reading = A.reading;
    X.tau_w = A.tau_w;
    X.sigma0 = A.sigma0;
    X.alpha = A.alpha;
    layer_x_source(X, A.lc, uniform(A.nHI[cs]));
    X.nHI = L.transposed ? A.nHI_T : A.nHI;
    const double half_he = uniform(A.nHeI[cs]) * A.alpha * 0.5;
    const double *nHe = L.transposed ? A.nHeI_T : A.nHeI;
    double *gH = L.transposed ? A.gH_T : A.gH;
    double *gHe = L.transposed ? A.gHe_T : A.gHe;
    const double coef = uniform(Q * A.coef_unit);
    if (p == 3 * 0 + 2 && first) he_source_cell(A, cs, Q);   // once per source
    const int Mx = min(uniform(isqrt_floor(Rsq)), L.ext_d);
    if (Mx < 1) return;
    const int S = W.S, P = S + 1, P8 = 8 * P, He = W.layHe - W.lay;
    const int odd = 2 * P8 * P, geo_odd = (int)sizeof(GeoRow) * S;   // HI and HeI buffers of odd layers
    for (int k = tid; k < (TEAM ? 4 : 2) * P * P; k += nt) lds<double>(W.lay + 8 * k) = 0.0;
    const SweepLds G{W.lay, W.geo, 0, W.sq_n, S};
    sweep_index_terms<TEAM>(L, N, G, team, lane);
    auto factors = [&](int m, double inv_m) {
        const int base = W.geo + (TEAM && (m & 1) ? geo_odd : 0);
        for (int k = tid; k < S; k += nt) lds<Geo>(base + mul24(k, (int)sizeof(GeoRow))) = layer_geo(m, inv_m, k);
    };
    auto rounds = [&](int total) { return TEAM ? ((total + 63) / 64 + T - 1) / T : (total + 63) / 64; };
    LayerRect r;
    RectWalk w;
    uint32_t idx_d = 0, cp = 0;
    int m2 = 0, u = 0, v = 0, r2 = 0, gu = 0, gv = 0, gbase = W.geo;
    bool act = false;
    double n1 = 0.0, n2 = 0.0;
    auto enter = [&](int m) {
        r = layer_rect_uniform(L.ext_u, L.ext_v, Rsq, m);
        m2 = m * m;
        idx_d = layer_idx_d(L, N, m);
        if (TEAM) gbase = W.geo + (m & 1 ? geo_odd : 0);
        w.init(r, ((rounds(r.total) - 1) * T + w0) * 64 + lane, nt);
    };
    auto fetch = [&]() {
        const int uv2 = mul24(w.u, w.u) + mul24(w.v, w.v);
        act = (w.u < r.nu) & (uv2 <= r.rem);
        u = act ? w.u : 0;
        v = act ? w.v : 0;
        r2 = m2 + (act ? uv2 : 0);
        gu = mul24(u, (int)sizeof(GeoRow)) + gbase;
        gv = mul24(v, (int)sizeof(GeoRow)) + gbase;
        cp = idx_d + lds<uint32_t>(gu + (int)offsetof(GeoRow, iu)) + lds<uint32_t>(gv + (int)offsetof(GeoRow, iv));
        n1 = X.nHI[cp];
        n2 = nHe[cp];
    };
    enter(1);
    fetch();
    if (TEAM) {
        factors(1, 1.0);
        __syncthreads();
    }
    int head = 0, pend = 0;   // the rate queue
    for (int m = 1; m <= Mx; ++m) {
        const double inv_m = rcp_f64((double)m);
        if (TEAM) {
            if (m < Mx) factors(m + 1, rcp_f64((double)(m + 1)));
        } else {
            factors(m, inv_m);
            wave_sync();
        }
        const int from = W.lay + (TEAM && !(m & 1) ? odd : 0), to = W.lay + (TEAM && (m & 1) ? odd : 0);
        for (int c = rounds(r.total) - 1; c >= 0; --c) {
            const bool in = act;
            const int ku = gu, kv = gv, r2c = r2, uc = u, vc = v;
            const uint32_t cell = cp;
            const double d1 = n1, d2 = n2;
            if (c > 0) {
                w.down();
                fetch();
            } else if (m < Mx) {
                enter(m + 1);
                fetch();
            }
            const int s = mul24(uc, P8) + 8 * vc, q = s + from, q1 = q + P8;
            const double h3 = lds<double>(q), h1 = lds<double>(q + 8);
            const double h2 = lds<double>(q1), h0 = lds<double>(q1 + 8);
            const double M3 = lds<double>(q + He), M1 = lds<double>(q + He + 8);
            const double M2 = lds<double>(q1 + He), M0 = lds<double>(q1 + He + 8);
            const Geo fu = lds<Geo>(ku), fv = lds<Geo>(kv);
            const double ds = (W.sq_n ? lds<double>(8 * r2c) : sqrt_fast((double)r2c)) * inv_m;
            const double ads = X.sa * ds;
            const bool thick = ballot(!all_thick(h0, h1, h2, h3)) == 0;
            double e_in, hout, NinHe;
            layer_cell_core(X, m, thick, fu, fv, ads, d1 * ads, h0, h1, h2, h3, 0.0, INFINITY, &e_in, &hout);
            // the helium column with the same weights: N_He = sum s f M_He / sum s f
            if (m == 1) {
                NinHe = X.reading == 0 ? half_he * ds : half_he;
            } else {
                const double w0 = fu.om * fv.om * (h0 > 0.0 ? h0 : X.inv_tw);
                const double w1 = fu.a * fv.om * (h1 > 0.0 ? h1 : X.inv_tw);
                const double w2 = fu.om * fv.a * (h2 > 0.0 ? h2 : X.inv_tw);
                const double w3 = fu.a * fv.a * (h3 > 0.0 ? h3 : X.inv_tw);
                NinHe = (w0 * M0 + w1 * M1 + w2 * M2 + w3 * M3) * rcp_f64(w0 + w1 + w2 + w3);
            }
            if (in) {
                lds<double>(s + to + P8 + 8) = hout;
                lds<double>(s + to + P8 + He + 8) = NinHe + d2 * A.alpha * ds;
            }
            const double Nin = entry_tau(e_in) * X.inv_s0;
            bool below = false;
            for (int b = 0; b < A.nb; ++b) below |= A.sH[b] * Nin + A.sHe[b] * NinHe < A.tp[b].tau_hi;
            const bool want = in & below & layer_owned(L, m, uc, vc);
            asm volatile("" : "+v"(n1), "+v"(n2));   // see sweep_layers
            const uint64_t mask = ballot(want);
            if (want) {
                const int k = (head + pend + rank_in(mask)) & (kHeQueue - 1);
                lds<double>(W.e + 8 * k) = e_in;
                lds<double>(W.NinHe + 8 * k) = NinHe;
                lds<uint32_t>(W.cp + 4 * k) = cell;
                lds<uint32_t>(W.mr + 4 * k) = ((uint32_t)m << 16) | (uint32_t)r2c;
            }
            pend += __popcll(mask);
            if (pend >= 64) {
                wave_sync();
                he_rate<FINE>(A, W, (head + lane) & (kHeQueue - 1), coef, X.nHI, nHe, X.inv_s0, gH, gHe);
                head = (head + 64) & (kHeQueue - 1);
                pend -= 64;
            }
            wave_sync();
        }
        if (TEAM) __syncthreads();
    }
    wave_sync();
    if (lane < pend) he_rate<FINE>(A, W, (head + lane) & (kHeQueue - 1), coef, X.nHI, nHe, X.inv_s0, gH, gHe);
    wave_sync();
}

template <bool FINE>
__global__ __launch_bounds__(1024) void fwd_layer_he(HeArgs A)
{
    constexpr int TYPE = 3, npieces = 24;
    const bool direct = A.items > 0;
    if (!direct && A.seg[TYPE + 1] == A.seg[TYPE]) return;   // no sources
    for (int k = threadIdx.x; k < A.sq_n; k += blockDim.x) lds<double>(8 * k) = sqrt((double)k);
    __syncthreads();
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    HeLds W;
    W.S = A.lay_S;
    W.sq_n = A.sq_n;
    W.e = (A.sq_n ? (int)layer_sqrt_bytes(A.sq_n - 1) : 0) + wave * A.region_bytes;
    W.NinHe = W.e + 8 * kHeQueue;
    W.cp = W.NinHe + 8 * kHeQueue;
    W.mr = W.cp + 4 * kHeQueue;
    W.lay = W.e + he_queue_bytes();
    W.layHe = W.lay + 8 * (W.S + 1) * (W.S + 1);
    W.geo = W.layHe + 8 * (W.S + 1) * (W.S + 1);
    const int base = direct ? 0 : A.seg[TYPE];
    const int nitems = direct ? A.items : (A.seg[TYPE + 1] - base) * npieces;
    const int home = (int)(blockIdx.x % kXcds);
    int chunk = home;
    for (;;) {
        const int item = direct ? (int)blockIdx.x * waves + wave : next_item(A.counter, nitems, home, chunk, lane);
        if (item >= nitems) break;
        const int src = direct ? A.src0 + item / npieces : uniform(A.order[base + item / npieces]);
        sweep_layer_piece_he<FINE, false>(A, W, Team{0, 1}, src, item % npieces, lane);
        if (direct) break;
    }
}

// Bytes of a team's buffers and tables (the queues follow).
__host__ __device__ constexpr size_t he_team_shared_bytes(int S)
{
    return (2 * (2 * (size_t)(S + 1) * (S + 1) * sizeof(double) + (size_t)S * sizeof(GeoRow)) + 15) & ~(size_t)15;
}

// One work-group per pyramid, its waves a team (see fwd_team).
template <bool FINE>
__global__ __launch_bounds__(1024) void fwd_team_he(HeArgs A)
{
    const Team team{uniform((int)threadIdx.x >> 6), (int)blockDim.x >> 6};
    HeLds W;
    W.S = A.lay_S;
    W.sq_n = 0;
    W.lay = 0;
    W.layHe = 8 * (W.S + 1) * (W.S + 1);
    W.geo = 4 * 8 * (W.S + 1) * (W.S + 1);
    W.e = (int)he_team_shared_bytes(W.S) + team.w * he_queue_bytes();
    W.NinHe = W.e + 8 * kHeQueue;
    W.cp = W.NinHe + 8 * kHeQueue;
    W.mr = W.cp + 4 * kHeQueue;
    const int item = blockIdx.x;
    sweep_layer_piece_he<FINE, true>(A, W, team, A.src0 + item / 24, item % 24, threadIdx.x & 63);
}

size_t he_team_bytes(int S, int T) { return he_team_shared_bytes(S) + (size_t)T * he_queue_bytes(); }

size_t he_region_bytes(int S)
{
    const size_t b = (size_t)he_queue_bytes() + 2 * (size_t)(S + 1) * (S + 1) * sizeof(double) +
                     (size_t)S * sizeof(GeoRow);
    return (b + 15) & ~(size_t)15;
}

hipError_t he_configure(size_t max_lds)
{
    (void)hipFuncSetAttribute((const void *)fwd_layer_he<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)max_lds - 64);
    for (const void *f : {(const void *)fwd_team_he<false>, (const void *)fwd_team_he<true>})
        (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds - 64);
    (void)hipFuncSetAttribute((const void *)fwd_layer_he<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)max_lds - 64);
    (void)hipGetLastError();
    return hipSuccess;
}

hipError_t he_occupancy(int waves, size_t lds, int *blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)fwd_layer_he<true>, waves * 64, lds);
}

// n_direct > 0: the pyramids of that many sources from src0 on (by `team` waves
// each if that is more than 1), else all sources of the call from the counters.
hipError_t launch_fwd_layer_he(hipStream_t st, const HeLaunch &H, int S, int waves, int grid, int src0, int n_direct,
                               int team)
{
    HeArgs A;
    A.N = H.N;
    A.ex = make_extent(H.N);
    A.alpha = H.alpha;
    A.sigma0 = H.sigma0;
    A.tau_w = H.tau_w;
    A.reading = H.reading;
    A.nb = H.nb;
    A.tab = H.tab;
    A.n_tab = H.n_tab;
    for (int b = 0; b < kMaxBands; ++b) {
        A.tp[b] = H.tp[b < H.nb ? b : 0];
        A.sH[b] = b < H.nb ? H.sH[b] : 0.0;
        A.sHe[b] = b < H.nb ? H.sHe[b] : 0.0;
    }
    A.nHI = H.nHI;
    A.nHeI = H.nHeI;
    A.nHI_T = H.nHI_T;
    A.nHeI_T = H.nHeI_T;
    A.gH = H.gH;
    A.gHe = H.gHe;
    A.gH_T = H.gH_T;
    A.gHe_T = H.gHe_T;
    A.ijk = H.ijk;
    A.Q = H.Q;
    A.R = H.R;
    A.R_cap = H.R_cap;
    A.order = H.order;
    A.seg = H.ctl + kCtlSeg;
    A.counter = H.ctl + kCtlCounter + kXcds * kCounterPad * 3;
    A.err = H.err;
    A.src0 = src0;
    A.items = 24 * n_direct;
    A.lc = make_layer_const(H.sigma0, H.alpha, H.tau_w, 1.0);   // (every band has its own tau_hi)
    A.lay_S = S;
    A.region_bytes = (int)he_region_bytes(S);
    const int Rsq = (int)floor((double)H.R_cap * (double)H.R_cap);
    const size_t sqb = H.sq_table ? layer_sqrt_bytes(Rsq) : 0;
    A.sq_n = sqb ? Rsq + 1 : 0;
    A.coef_unit = 1.0 / (4.0 * M_PI * H.alpha * H.alpha);
    const size_t lds = sqb + (size_t)waves * A.region_bytes;
    bool fine = true;
    for (int b = 0; b < H.nb; ++b) fine = fine && H.tp[b].fine;
    void *args[] = {&A};
    if (team > 1)
        return hipLaunchKernel(fine ? (const void *)fwd_team_he<true> : (const void *)fwd_team_he<false>, dim3(A.items),
                               dim3(64 * team), args, he_team_bytes(S, team), st);
    if (n_direct > 0) grid = (A.items + waves - 1) / waves;
    return hipLaunchKernel(fine ? (const void *)fwd_layer_he<true> : (const void *)fwd_layer_he<false>, dim3(grid),
                           dim3(64 * waves), args, lds, st);
}

}  // namespace asora
