// asora_sweep.h -- the column sweep of a layer pyramid by one wave or by the
// waves of a work-group together, shared by the forward kernels and the
// adjoint's column pass.
#pragma once
#include "asora_dev.h"

namespace asora {

// The lanes of the wave where p holds.
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Lanes below this one that are set in mask.
__device__ __forceinline__ int rank_in(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// LDS by byte offset: the offsets of a wave's arrays are scalars, and an
// element's address is one multiply-add or shift-add away from them.
template <class T>
__device__ __forceinline__ T &lds(int offset)
{
    extern __shared__ __align__(16) char smem[];
    return *(T *)(smem + offset);
}

// Byte offsets of a sweep's arrays: the layer buffer of (S + 1)^2 doubles
// (layer_slot), the table of GeoRows, the work-group's table of roots (sq_n
// entries, none if 0).  A team has two layer buffers and two tables of
// GeoRows, one after the other: layers of odd m use the second of each.
struct SweepLds {
    int lay, geo, sq, sq_n;
    int S;
};

// The waves of a team: the work-group's T waves, of which this is wave w.
struct Team {
    int w, T;
};

template <bool TEAM>
__device__ __forceinline__ void team_sync()
{
    if (TEAM)
        __syncthreads();
    else
        wave_sync();
}

// The pyramid's index terms along u and v, kept for all layers.
template <bool TEAM>
__device__ __forceinline__ void sweep_index_terms(const LayerPiece &L, int N, const SweepLds &W, Team team, int lane)
{
    const int nt = TEAM ? team.T * 64 : 64;
    for (int k = (TEAM ? team.w * 64 : 0) + lane; k < W.S; k += nt) {
        const uint32_t iu = layer_idx_u(L, N, k), iv = layer_idx_v(L, N, k);
        for (int b = 0; b < (TEAM ? 2 : 1); ++b) {
            const int row = W.geo + (int)sizeof(GeoRow) * (k + b * W.S);
            lds<uint32_t>(row + (int)offsetof(GeoRow, iu)) = iu;
            lds<uint32_t>(row + (int)offsetof(GeoRow, iv)) = iv;
        }
    }
    team_sync<TEAM>();
}

// One chunk of a layer: 64 cells, one per lane.
struct SweepChunk {
    int m, c;           // layer, chunk
    bool in;            // the lane has a cell (the others hold values of cell (0, 0))
    int u, v, r2;
    uint32_t cell;      // index in the piece's layout
    double dt;          // in-cell optical depth
    double e_in, h;     // entry and exit optical depths, as entries (tau_entry)
    bool below;         // entry optical depth below tau_hi
    bool any;           // the chunk has cells (a team's last round may be short)
};

// Sweeps layers 1 .. m_last (m_last may be lowered by layer_end) of pyramid L:
// chunk(SweepChunk) after each chunk, layer_end(m, total) after each layer's.
//
// Layer m is the rectangle of LayerRect, covered in chunks of 64 consecutive
// cells.
//
// One wave (!TEAM): the previous layer lives in the wave's LDS buffer and is
// overwritten in place: chunks go from the last to the first, and a cell reads
// only slots at or before its own (u, v) in lexicographic order, so every slot
// a chunk reads still holds layer m - 1 (its own writes follow its reads, and
// LDS operations of a wave run in order).
//
// A team (TEAM): the work-group's waves take the chunks of a layer in turn,
// read the previous layer from one buffer and write the other, with one
// barrier a layer.  The waves run the same number of rounds in every layer; a
// round past the last chunk has no active lane.
//
// The sweep is bound by instruction issue, then by the latency of a chunk's
// dependent chain (250^3, 40000 sources of radii 5 to 40, forward: 24.9 ms with
// columns converted to optical depths in every cell and fields loaded where
// they are used, 17.5 ms in this form; 12.4 ms of it without the rates).  So
// the chunks of all layers form one sequence, a chunk's
// field values are fetched one chunk ahead, and lanes without a cell repeat
// cell (0, 0) instead of being masked off (only the writes are masked).
template <bool TEAM, class Chunk, class LayerEnd>
__device__ __forceinline__ void sweep_layers(const LayerPiece &L, const LayerX &X, const SweepLds &W, Team team,
                                             int Rsq, int Mx, int &m_last, double tau_hi, double inv_hi, int lane,
                                             Chunk chunk, LayerEnd layer_end)
{
    const int S = W.S, P = S + 1, P8 = 8 * P;
    const int w0 = TEAM ? team.w : 0, T = TEAM ? team.T : 1;
    const int lay_bytes = P8 * P, geo_bytes = (int)sizeof(GeoRow) * S;
    const int tid = w0 * 64 + lane, nt = T * 64;
    for (int k = tid; k < (TEAM ? 2 : 1) * P * P; k += nt) lds<double>(W.lay + 8 * k) = 0.0;   // finite everywhere it is read
    // the bilinear factors of a layer's offsets
    auto factors = [&](int m, double inv_m) {
        const int base = W.geo + (TEAM && (m & 1) ? geo_bytes : 0);
        for (int k = tid; k < S; k += nt) lds<Geo>(base + mul24(k, (int)sizeof(GeoRow))) = layer_geo(m, inv_m, k);
    };
    LayerRect r;      // the layer of the chunk fetched last
    RectWalk w;       // its cells
    uint32_t idx_d = 0, cp = 0;
    int m2 = 0, u = 0, v = 0, r2 = 0, gu = 0, gv = 0, gbase = W.geo;
    bool act = false;
    double nhi = 0.0;
    auto rounds = [&](int total) { return TEAM ? ((total + 63) / 64 + T - 1) / T : (total + 63) / 64; };
    auto enter = [&](int m) {
        r = layer_rect_uniform(L.ext_u, L.ext_v, Rsq, m);
        m2 = m * m;
        idx_d = layer_idx_d(L, X.N, m);
        if (TEAM) gbase = W.geo + (m & 1 ? geo_bytes : 0);
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
        nhi = X.nHI[cp];
    };
    enter(1);
    fetch();
    if (TEAM) {
        factors(1, 1.0);
        __syncthreads();
    }
    for (int m = 1; m <= m_last; ++m) {
        const double inv_m = rcp_f64((double)m), am = X.sa * inv_m;
        if (TEAM) {
            // the next layer's, in the table whose readers passed the last barrier
            if (m < Mx) factors(m + 1, rcp_f64((double)(m + 1)));
        } else {
            factors(m, inv_m);   // (every chunk ends with a wave barrier)
            wave_sync();
        }
        const int total = r.total;
        // where layers m - 1 and m are
        const int from = W.lay + (TEAM && !(m & 1) ? lay_bytes : 0), to = W.lay + (TEAM && (m & 1) ? lay_bytes : 0);
        for (int c = rounds(total) - 1; c >= 0; --c) {
            SweepChunk k;
            k.m = m;
            k.c = c * T + w0;
            k.any = !TEAM || k.c * 64 < total;
            k.in = act;
            k.u = u;
            k.v = v;
            k.r2 = r2;
            k.cell = cp;
            const int ku = gu, kv = gv;
            const double dens = nhi;
            // the next chunk, and its fields
            if (c > 0) {
                w.down();
                fetch();
            } else if (m < Mx) {
                enter(m + 1);
                fetch();
            }
            // slot (u - 1, v - 1) and the same one row up: the four neighbours
            // are two adjacent pairs, the cell's own slot the last
            const int s = mul24(k.u, P8) + 8 * k.v, q = s + from, q1 = q + P8;
            const double h3 = lds<double>(q), h1 = lds<double>(q + 8);
            const double h2 = lds<double>(q1), h0 = lds<double>(q1 + 8);
            const Geo fu = lds<Geo>(ku), fv = lds<Geo>(kv);
            const double rt = W.sq_n ? lds<double>(W.sq + 8 * k.r2) : sqrt_fast((double)k.r2);   // r2 <= Rsq < sq_n
            const double ads = rt * am;
            k.dt = dens * ads;
            const bool thick = ballot(!all_thick(h0, h1, h2, h3)) == 0;
            k.below = layer_cell_core(X, m, thick, fu, fv, ads, k.dt, h0, h1, h2, h3, tau_hi, inv_hi, &k.e_in, &k.h);
            if (k.in) lds<double>(s + to + P8 + 8) = k.h;
            // the fetched value is waited for here: after the rate batch that
            // may follow, the wait would include the batch's atomics
            asm volatile("" : "+v"(nhi));
            chunk(k);
            wave_sync();
        }
        layer_end(m, total);
        if (TEAM) __syncthreads();
    }
}

// ---- groups of pyramids ---------------------------------------------------
// A layer of a small pyramid has fewer cells than a wave has lanes, so a wave
// sweeps G pyramids of a source (G a divisor of 24) together: a group's layer
// is the G rectangles one after the other, in chunks of 64 cells across their
// borders.  The radius is within the box on every side, so that the rectangles
// are alike.
//
// What differs from pyramid to pyramid is looked up per lane: GroupRow, and
// the index terms of the axes.  What depends on the layer alone (the factors,
// the roots) is the same for every source and held once per work-group.
struct alignas(16) GroupRow {
    int d, u, v;   // byte offsets of the pyramid's index terms along d, u, v
    int flags;     // kGroup...
};
constexpr int kGroupNegU = 1, kGroupNegV = 2, kGroupTieU = 4, kGroupTieV = 8, kGroupT = 16;

// Byte offsets: G layer buffers of (S + 1)^2 doubles, G GroupRows, twelve
// tables of K index terms (axis, sign, layout); shared: the factors of layers
// 1 .. M (geo_S each), the roots of r^2.
struct GroupLds {
    int lay, row, term, geo, sq;
    int S, K, G;
    int geo_S;   // row stride of the table of factors
};

struct GroupChunk {
    int m, c, cells;    // layer, chunk, the layer's cells
    bool in;
    int u, v, r2, flags;
    uint32_t cell;      // index in the pyramid's layout
    double dt, e_in, h;
    bool below;
};

// The index terms of a source's axes and the rows of pyramids p0 .. p0 + G - 1.
__device__ __forceinline__ void group_tables(const GroupLds &W, int p0, int si, int sj, int sk, int N, int lane)
{
    const uint32_t n = (uint32_t)N, nn = n * n;
    for (int k = lane; k < W.K; k += 64) {
        for (int a = 0; a < 6; ++a) {   // axis, sign
            const int ax = a >> 1, s = ax == 0 ? si : (ax == 1 ? sj : sk);
            const uint32_t w = (uint32_t)wrap(a & 1 ? s - k : s + k, N);
            // standard [i][j][k], transposed [k][i][j]
            lds<uint32_t>(W.term + 4 * (W.K * (2 * a) + k)) = w * (ax == 0 ? nn : (ax == 1 ? n : 1u));
            lds<uint32_t>(W.term + 4 * (W.K * (2 * a + 1) + k)) = w * (ax == 0 ? n : (ax == 1 ? 1u : nn));
        }
    }
    if (lane < W.G) {
        const int p = p0 + lane, oct = p / 3, d = p % 3, au = d == 0 ? 1 : 0, av = d == 2 ? 1 : 2, t = d == 2 ? 1 : 0;
        auto base = [&](int ax) { return W.term + 4 * W.K * (2 * (2 * ax + ((oct >> ax) & 1)) + t); };
        GroupRow r;
        r.d = base(d);
        r.u = base(au);
        r.v = base(av);
        // as in make_layer_piece
        r.flags = ((oct >> au) & 1 ? kGroupNegU : 0) | ((oct >> av) & 1 ? kGroupNegV : 0) | (d == 0 ? kGroupTieU : 0) |
                  (d != 2 ? kGroupTieV : 0) | (t ? kGroupT : 0);
        lds<GroupRow>(W.row + (int)sizeof(GroupRow) * lane) = r;
    }
}

// layer_owned of a cell of a group.
__device__ __forceinline__ bool group_owned(int flags, int m, int u, int v)
{
    const int u0 = flags & kGroupNegU, v0 = (flags & kGroupNegV) >> 1;
    return ((unsigned)(u - u0) < (unsigned)(m + 1 - u0 - ((flags & kGroupTieU) >> 2))) &
           ((unsigned)(v - v0) < (unsigned)(m + 1 - v0 - ((flags & kGroupTieV) >> 3)));
}

// Sweeps layers 1 .. Mx of a group; nHI_T: X.nHI in the transposed layout.  In
// place, as one wave's sweep_layers: a pyramid's cells follow each other in
// (u, v) order, and chunks go from the last to the first.
template <class Chunk>
__device__ __forceinline__ void sweep_group(const LayerX &X, const double *nHI_T, const GroupLds &W, int Rsq, int Mx,
                                            double tau_hi, double inv_hi, int lane, Chunk chunk)
{
    const int P = W.S + 1, P8 = 8 * P, PP8 = P8 * P;
    for (int k = lane; k < W.G * P * P; k += 64) lds<double>(W.lay + 8 * k) = 0.0;
    wave_sync();
    LayerRect r;
    float inv_t = 0.f, inv_w = 0.f;
    int cells = 0, m2 = 0, mf = 0, gbase = 0;   // of the layer of the chunk fetched last
    int p8 = 0, u = 0, v = 0, r2 = 0, flags = 0;
    uint32_t cp = 0;
    bool act = false;
    double nhi = 0.0;
    auto enter = [&](int m) {
        r = layer_rect_uniform(Mx, Mx, Rsq, m);
        inv_t = rcp_approx((float)r.total);
        inv_w = rcp_approx((float)r.wv);
        cells = W.G * r.total;
        m2 = m * m;
        mf = 4 * m;
        gbase = W.geo + (int)sizeof(Geo) * W.geo_S * (m - 1);
    };
    // (the quotients are exact as in RectWalk::init: at most 24 rectangles)
    auto fetch = [&](int c) {
        const int g = c * 64 + lane;
        int pl = (int)(((float)g + 0.5f) * inv_t);
        const int l = g - mul24(pl, r.total);
        u = (int)(((float)l + 0.5f) * inv_w);
        v = l - mul24(u, r.wv);
        int uv2 = mul24(u, u) + mul24(v, v);
        act = (g < cells) & (uv2 <= r.rem);
        pl = act ? pl : 0;
        u = act ? u : 0;
        v = act ? v : 0;
        uv2 = act ? uv2 : 0;
        r2 = m2 + uv2;
        p8 = mul24(pl, PP8);
        const GroupRow row = lds<GroupRow>(W.row + (int)sizeof(GroupRow) * pl);
        flags = row.flags;
        cp = lds<uint32_t>(row.d + mf) + lds<uint32_t>(row.u + 4 * u) + lds<uint32_t>(row.v + 4 * v);
        nhi = (flags & kGroupT ? nHI_T : X.nHI)[cp];
    };
    enter(1);
    fetch((cells + 63) / 64 - 1);
    for (int m = 1; m <= Mx; ++m) {
        const double am = X.sa * rcp_f64((double)m);
        const int total = cells;
        for (int c = (total + 63) / 64 - 1; c >= 0; --c) {
            GroupChunk k;
            k.m = m;
            k.c = c;
            k.cells = total;
            k.in = act;
            k.u = u;
            k.v = v;
            k.r2 = r2;
            k.flags = flags;
            k.cell = cp;
            const int s = p8 + mul24(u, P8) + 8 * v + W.lay, s1 = s + P8;
            const int ku = gbase + (int)sizeof(Geo) * u, kv = gbase + (int)sizeof(Geo) * v;
            const double dens = nhi;
            if (c > 0) {
                fetch(c - 1);
            } else if (m < Mx) {
                enter(m + 1);
                fetch((cells + 63) / 64 - 1);
            }
            const double h3 = lds<double>(s), h1 = lds<double>(s + 8);
            const double h2 = lds<double>(s1), h0 = lds<double>(s1 + 8);
            const Geo fu = lds<Geo>(ku), fv = lds<Geo>(kv);
            const double ads = lds<double>(W.sq + 8 * k.r2) * am;
            k.dt = dens * ads;
            const bool thick = ballot(!all_thick(h0, h1, h2, h3)) == 0;
            k.below = layer_cell_core(X, m, thick, fu, fv, ads, k.dt, h0, h1, h2, h3, tau_hi, inv_hi, &k.e_in, &k.h);
            if (k.in) lds<double>(s1 + 8) = k.h;
            asm volatile("" : "+v"(nhi));   // see sweep_layers
            chunk(k);
            wave_sync();
        }
    }
}

}  // namespace asora
