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
// dependent chain.  So the chunks of all layers form one sequence, a chunk's
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

}  // namespace asora
