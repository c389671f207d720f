// rd_march.hpp -- K time steps per launch: a z march that keeps its planes in
// registers (temporal blocking; section 2's step, Eq. (5), taken K times between
// one read and one write of every species).
//
// What bounds a step is memory first: one read and one write of every species.
// A launch of K steps moves them once, so the bound becomes the vector
// arithmetic, repeated in the halos of the tiles; K, the rows of a lane and the
// waves of a workgroup trade one against the other.
//
// A lane owns four cells of a row (one 16-byte load in FP32) in RY rows; L lanes
// make a tile row and the T = 64 W threads of a workgroup T / L groups of RY
// rows, so rows of any length fill the waves (a wave is not a row).  A tile
// stores K rows less on each side than it loads, K cells less at an inner x
// edge (one halo lane), and marches K planes more: level l of plane p - l + 1
// (level 0: the planes loaded) is formed in iteration p, all levels one after
// the other, so an iteration loads one plane and stores one plane K steps on.
//   z neighbours: registers -- three planes of level 0 and one in flight, two
//     of each further level (a new value takes the place of the oldest);
//   y neighbours: registers inside a lane; the lane's first and last row pass
//     through LDS, every level and field in one exchange per iteration (two
//     buffers by parity, so one barrier);
//   x neighbours: the next lane by DPP; at the ends of a wave through LDS in the
//     same exchange (XEX; not needed where rows lie inside a wave).
// Loads and stores are buffer accesses of one plane, 32-bit offsets per lane
// formed once; a lane that stores nothing has an offset out of the plane, which
// the hardware drops, so the loop has no branch around its stores and the
// counts of accesses in flight stay exact.
//
// Face rules.  Along y and z a mirror face is the reflection of the rows
// (planes) at it: the reflected rows, computed as any other, come out equal to
// the rows they mirror bit for bit, since a row's two neighbours are added to
// each other first; a periodic face wraps.  So rows and planes outside the grid
// need no code but the index they are loaded from.  Along x the rule is applied
// at use, at every level: mirror, periodic, or a fixed ghost value.  Held layers
// and fixed ghosts along y and z are left to the other plans.
// Values between levels are rounded to the storage type, as a step that stored
// them would; every cell goes through the model's own cell function, so K steps
// give the bits of K launches of one.
//
// Measured (us per step, launches one after the other; one step per launch, the
// best plan before, tuned, against the default plan here): diffusion 512^3 FP32
// 189 -> 79 (K 4: 1700 Gcell/s, 1.7 times what the bytes of single steps would
// allow at 8 TB/s), BF16 121 -> 79 (72 tuned); Brusselator 256^3 FP32 44.3 ->
// 28.5, BF16 42.3 -> 28.8; pollutant 512x512x128 FP32 218 -> 124; small grids,
// where a launch is the latency of its chain of loads: diffusion 64^3 6.1 -> 2.2,
// Brusselator 101x90x77 10.2 -> 4.8.  (A profiler's trace, which runs launches
// apart, has 82 to 86 for diffusion 512^3 and 32 for the Brusselator.)  By counters,
// of the issue slots for vector instructions (four clocks each, at 2.4 GHz) the
// FP32 launches fill: diffusion 512^3, K 4, 76 to 79 %, moving 1.10 times the
// fields in and out at 3.5 TB/s; Brusselator, K 2, 61 %, 1.10 times at 4.6 TB/s;
// pollutant, K 2, 58 %, 1.06 times at 4.5 TB/s.
// Non-temporal stores gained diffusion 512^3 2 % and cost the Brusselator, whose
// fields stay in the last cache, 20 %.
//
// Point sources: a plane that has any in the tile's rows takes a second copy of
// the cell code; the others have neither a branch per cell nor its waits (with
// them, and the wind and the source rows looked up plane by plane, the pollutant
// took 171 us where it took 131 without, 256x256x64 37.8 and 28.1).
#pragma once

#include "rd_march_cfg.hpp"
#include "rd_tiles.hpp"

namespace rdk {

#ifdef __HIP_DEVICE_COMPILE__
typedef unsigned march_u4 __attribute__((ext_vector_type(4)));
typedef unsigned march_u2 __attribute__((ext_vector_type(2)));
typedef float march_f4 __attribute__((ext_vector_type(4)));
#endif

// Index of grid row / plane q, at most n beyond either face of a periodic or
// mirror axis of n cells: wrapped, or reflected (-1 is 0, -2 is 1, ..).
__device__ __forceinline__ int march_index(int q, int n, bool periodic) {
    const int lo = periodic ? q + n : -1 - q, hi = periodic ? q - n : 2 * n - 1 - q;
    return q < 0 ? lo : q >= n ? hi : q;
}

// Element e (0 .. 2) of a lane's cells, by value: a select, not an address.
__device__ __forceinline__ float march_elem(int e, float c0, float c1, float c2) {
    return e == 0 ? c0 : e == 1 ? c1 : c2;
}

// A value held in a scalar register that the compiler cannot form again by
// reloading it.
__device__ __forceinline__ float scopy(float x) {
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+s"(x));
#endif
    return x;
}

#ifdef __HIP_DEVICE_COMPILE__
// Four loaded cells as FP32, and four results as stored (offset ~0: dropped).
template <class S, class Raw>
__device__ __forceinline__ void march_unpack(const Raw& q, float (&v)[4]) {
    using T = typename S::T;
    if constexpr (sizeof(T) == 4) {
        v[0] = __uint_as_float(q.x);
        v[1] = __uint_as_float(q.y);
        v[2] = __uint_as_float(q.z);
        v[3] = __uint_as_float(q.w);
    } else {
        v[0] = S::up(T(q.x & 0xffffu));
        v[1] = S::up(T(q.x >> 16));
        v[2] = S::up(T(q.y & 0xffffu));
        v[3] = S::up(T(q.y >> 16));
    }
}
template <class S>
__device__ __forceinline__ void march_store(const float (&o)[4], __amdgpu_buffer_rsrc_t ws, unsigned so) {
    if constexpr (sizeof(typename S::T) == 4) {
        march_u4 d;
        d.x = __float_as_uint(o[0]);
        d.y = __float_as_uint(o[1]);
        d.z = __float_as_uint(o[2]);
        d.w = __float_as_uint(o[3]);
        __builtin_amdgcn_raw_buffer_store_b128(d, ws, so, 0, 0);
    } else {
        march_u2 d;
        d.x = S::down2(o[0], o[1]);
        d.y = S::down2(o[2], o[3]);
        __builtin_amdgcn_raw_buffer_store_b64(d, ws, so, 0, 0);
    }
}
#endif

// f(row) for every row of a lane: inner rows first, then the first and last.
template <int RY, int I = 0, class F>
__device__ __forceinline__ void march_rows(F&& f) {
    if constexpr (I < RY) {
        f(std::integral_constant<int, (I < RY - 2 ? I + 1 : I == RY - 1 ? RY - 1 : 0)>{});
        march_rows<RY, I + 1>(f);
    }
}

// N contiguous floats to / from LDS (scalar accesses, which the compiler
// merges: vectors built here from single cells kept the planes they come from
// in memory).
template <int N>
__device__ __forceinline__ void march_lds_put(RD_LDS float* p, const float (&e)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = e[i];
}
template <int N>
__device__ __forceinline__ void march_lds_get(const RD_LDS float* p, float (&e)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) e[i] = p[i];
}

template <int NF> struct MarchConst {
    float kx[NF], ky[NF], kz[NF], kc[1];
    float p[3];
    float dt;
    __device__ __forceinline__ explicit MarchConst(const StepArgs& a) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            kx[f] = scopy(a.kx[f]);
            ky[f] = scopy(a.ky[f]);
            kz[f] = scopy(a.kz[f]);
        }
        kc[0] = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) p[i] = scopy(a.p[i]);
        dt = scopy(a.dt);
    }
};

// LDS of a march of NF fields and K levels, in floats: the boundary rows of
// every thread and the edge cells, each twice (by parity).
template <int NF, int RY, int W, int K>
struct MarchLds {
    static constexpr int T = 64 * W;
    static constexpr int NR = RY == 1 ? 1 : 2;       // boundary rows of a lane
    static constexpr int NE = K * NF;                // values of an edge slot: by level, then field
    static constexpr int NX = (W + T / kMarchMinLanes) * RY + 1;   // edge slots of one side, the last the face values
    static constexpr int ROWS = 2 * K * NF * NR * T * 4, EDGES = 2 * 2 * NX * NE;
};

// One workgroup's march: K steps of planes z0 .. z1-1 of the rows stored from
// yb on (a tile leaves KG rows on each side, KG >= K) in x tile tx.
template <class M, class S, int RY, int W, int K, int KG, bool XEX, int RAG, bool MIR>
__device__ __forceinline__ void march_tile_steps(const StepArgs& a, RD_LDS float* rows_l, RD_LDS float* edge_l, int tx,
                                                 int yb, int z0, int z1) {
#ifdef __HIP_DEVICE_COMPILE__
    using R = MarchLds<M::NF, RY, W, K>;
    constexpr int NF = M::NF, T = R::T, ES = int(sizeof(typename S::T));
    constexpr int NR = R::NR, NE = R::NE, NX = R::NX;
    static_assert(M::NO == NF && KG >= K, "every field is stored, from a tile that is deep enough");
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);

    // ---- the tile ---------------------------------------------------------
    const int L = a.mg[MG_LANES], halo = a.mg[MG_HALO], G = T / L;
    const int BY = G * RY - 2 * KG;                  // rows stored
    const int yg = t / L, x4 = t - yg * L;
    const bool perx = a.bck[0][0] == BC_PERIODIC, pery = a.bck[0][2] == BC_PERIODIC,
               perz = a.bck[0][4] == BC_PERIODIC;
    const int x = (tx * (L - 2 * halo) + x4 - halo) * 4;
    int xm = x;                                      // column loaded
    if (perx && halo) xm = x < 0 ? x + a.nx : x >= a.nx ? x - a.nx : x;
    xm = min(max(xm, 0), a.pitch - 4);
    const bool wrap = perx && !halo;                 // the row's ends meet through LDS
    const int e_last = (a.nx - 1) & 3;               // element of the row's last cell
    const bool first = x == 0 && !(perx && halo), last = x <= a.nx - 1 && x > a.nx - 5 && !(perx && halo);
    const bool rot = !XEX && perx;                  // rows of one wave: the lane rotation wraps them
    const bool own_l = first && a.bck[0][0] == BC_MIRROR, in_l = first && a.bck[0][0] != BC_MIRROR && !rot;
    const bool mir_r = a.bck[0][1] == BC_MIRROR;
    // the last lane is full (RAG 0: always, 1: never, 2: of any grid)
    const bool full = RAG == 0 || (RAG == 2 && e_last == 3);
    const bool own_r = last && mir_r && full, in_r = last && !mir_r && full && !rot;
    // a row that ends inside its last lane: the cell after the row's last then
    // holds what is beyond the face
    bool after[3];
#pragma unroll
    for (int i = 1; i < 4; ++i) after[i - 1] = last && e_last + 1 == i;
    const bool stored_x = x4 >= halo && x4 < L - halo && x >= 0 && x < a.nx && yg < G;

    unsigned lo[RY], so[RY];                         // byte offsets in a plane: loaded, stored (~0: not stored)
    int yr[M::SOURCES ? RY : 1];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int yl = yg * RY + r, y = yb - KG + yl;
        const int ym = march_index(min(max(y, -KG), a.ny - 1 + KG), a.ny, pery);
        lo[r] = unsigned(ym * a.pitch + xm) * ES;
        so[r] = stored_x && yl >= KG && yl < KG + BY && y < a.ny ? unsigned(y * a.pitch + x) * ES : 0x80000000u;
        if constexpr (M::SOURCES) yr[r] = ym;
    }

    // rows ys0 .. ys1 - 1 hold every source of the tile (rows beyond a mirror
    // face reflect into the tile, those beyond a periodic one wrap out of it)
    const bool all_rows = pery && (yb < KG || yb + BY + KG > a.ny);
    const int ys0 = all_rows ? 0 : max(yb - KG, 0), ys1 = all_rows ? a.ny : min(yb + BY + KG, a.ny);

    // ---- exchange slots ------------------------------------------------------
    // boundary rows: slot t; the rows above and below are those of t -+ L
    const int up_t = max(t - L, 0), dn_t = min(t + L, T - 1);
    auto row_at = [&](int par, int l, int f, int k, int th) __attribute__((always_inline)) {
        return rows_l + ((((par * K + l) * NF + f) * NR + k) * T + th) * 4;
    };
    // x edges: where this lane's first / last cell goes (-1: nowhere) and where
    // its outer neighbours come from -- the next wave, the row's other end
    // (slot W + row group) or the face's value (the last slot)
    constexpr int FACE = MIR ? 0 : NX - 1;            // (mirror faces take no value)
    int ef = -1, el = -1, rf = 0, rl = 0;
    if (lane == 0 && x4 != 0) ef = rf = w * RY;
    if (lane == 63 && x4 != L - 1) el = rl = (w + 1) * RY;
    if (first) {
        if (wrap) ef = (W + yg) * RY;
        rf = wrap ? (W + yg) * RY : FACE;
    }
    if (last) {
        if (wrap) el = (W + yg) * RY;
        rl = wrap ? (W + yg) * RY : FACE;
    }
    if (yg >= G || (w == W - 1 && lane == 63 && !last)) {
        el = -1;
        rl = FACE;
    }
    if (yg >= G) {
        ef = -1;
        rf = FACE;
    }
    // side 0 holds first cells (read as a right neighbour), side 1 last cells
    auto edge_at = [&](int par, int side, int slot) __attribute__((always_inline)) {
        return edge_l + ((par * 2 + side) * NX + slot) * NE;
    };
    if constexpr (XEX && !MIR) {
        if (t < 4 * NE) {                            // written before the first barrier, read after it
            const int f = t % NF, side = (t / NE) & 1;
            edge_at(t / (2 * NE), side, FACE)[t % NE] = side ? a.bcv[f][0] : a.bcv[f][1];
        }
    }

    const MarchConst<NF> k(a);
    float cl[NF], cr[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        cl[f] = scopy(a.bcv[f][0]);
        cr[f] = scopy(a.bcv[f][1]);
    }

    // ---- planes ------------------------------------------------------------
    const long long pbytes = a.plane * ES;
    float V[4][NF][RY][4];                           // level 0: planes p-1, p, p+1
    float Q[K > 1 ? K - 1 : 1][2][NF][RY][4];        // levels 1 .. K-1: two planes each
    using Raw = std::conditional_t<ES == 4, march_u4, march_u2>;
    Raw P[NF][RY];                                   // the plane in flight
    auto issue = [&](int p) __attribute__((always_inline)) {
        const int pz = march_index(min(p, z1 - 1 + K), a.nz, perz);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)((const char*)a.in[f] + pz * pbytes), 0, int(pbytes), 0x00027000);
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                if constexpr (ES == 4) P[f][r] = __builtin_amdgcn_raw_buffer_load_b128(rs, lo[r], 0, 0);
                else P[f][r] = __builtin_amdgcn_raw_buffer_load_b64(rs, lo[r], 0, 0);
            }
        }
    };
    auto take = [&](float (&v)[NF][RY][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int r = 0; r < RY; ++r) march_unpack<S>(P[f][r], v[f][r]);
    };
#pragma unroll
    for (int l = 0; l < (K > 1 ? K - 1 : 1); ++l)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int r = 0; r < RY; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) Q[l][j][f][r][i] = 0.f;

    const int pa_ = z0 - (K - 1), pb_ = z1 - 1 + (K - 1);   // centre planes of level 1
    issue(pa_ - 1);
    take(V[0]);
    issue(pa_);
    take(V[1]);
    issue(pa_ + 1);

    auto export_plane = [&](int par, int l, const float (&v)[NF][RY][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                const float(&c)[4] = v[f][j == 0 ? 0 : RY - 1];
                lds_st4(row_at(par, l, f, j, t), c[0], c[1], c[2], c[3]);
            }
    };
    // the last cell of a row in this lane
    auto end_cell = [&](const float (&c)[4]) __attribute__((always_inline)) {
        if constexpr (RAG == 0) return c[3];
        const float ce = march_elem(e_last, c[0], c[1], c[2]);
        return last && !full ? ce : c[3];
    };
    // the row ends of every level and field, one vector per slot and row
    auto export_edges = [&](int par, const float (&v0)[NF][RY][4], auto par_c) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_c)::value;
        if constexpr (XEX) {
            if (ef >= 0) {
                march_rows<RY>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    float e[NE];
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        e[f] = v0[f][r][0];
#pragma unroll
                        for (int l = 1; l < K; ++l) e[l * NF + f] = Q[l - 1][PAR][f][r][0];
                    }
                    march_lds_put<NE>(edge_at(par, 0, ef + r), e);
                });
            }
            if (el >= 0) {
                march_rows<RY>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    float e[NE];
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        e[f] = end_cell(v0[f][r]);
#pragma unroll
                        for (int l = 1; l < K; ++l) e[l * NF + f] = end_cell(Q[l - 1][PAR][f][r]);
                    }
                    march_lds_put<NE>(edge_at(par, 1, el + r), e);
                });
            }
        }
    };
    struct Halo {
        float up[NF][4], dn[NF][4];
    };
    auto import_plane = [&](int par, int l, Halo& h) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            lds_ld4(row_at(par, l, f, NR - 1, up_t), h.up[f]);
            lds_ld4(row_at(par, l, f, 0, dn_t), h.dn[f]);
        }
    };

    // one row of the level above: centre plane v, planes vm and vp
    auto row = [&](int r, const float (&vm)[NF][RY][4], const float (&v)[NF][RY][4], const float (&vp)[NF][4],
                   const Halo& h, const float (&xl)[NF], const float (&xr)[NF], float wind, int src_row,
                   float (&o)[NF][4]) __attribute__((always_inline)) {
        float c[NF][4], left[NF], right[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c[f][i] = v[f][r][i];
            if constexpr (RAG != 0) {
                const float ce = march_elem(e_last, c[f][0], c[f][1], c[f][2]);
                const float fr = MIR || mir_r ? ce : xr[f];
#pragma unroll
                for (int i = 1; i < 4; ++i) c[f][i] = after[i - 1] ? fr : c[f][i];
            }
            if constexpr (XEX) {
                left[f] = lane_from_left(c[f][3], xl[f]);
                right[f] = lane_from_right(c[f][0], xr[f]);
            } else {
                left[f] = lane_from_left_wrap(c[f][3]);
                right[f] = lane_from_right_wrap(c[f][0]);
            }
            left[f] = own_l ? c[f][0] : left[f];
            if constexpr (RAG != 1) right[f] = own_r ? c[f][3] : right[f];
            if constexpr (!MIR) {
                left[f] = in_l ? (XEX ? xl[f] : cl[f]) : left[f];
                if constexpr (RAG != 1) right[f] = in_r ? (XEX ? xr[f] : cr[f]) : right[f];
            }
        }
        auto cells = [&](auto src) __attribute__((always_inline)) {
            // emissions of the lane's cells; where there are none -0, which
            // leaves a sum as it is
            float e[NF][4];
            if constexpr (src.value) {
                const int s0 = cload_ptr<int>(a.src_row)[src_row + yr[r]];
                const int s1 = cload_ptr<int>(a.src_row)[src_row + yr[r] + 1];
                bool any[4] = {};
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) e[f][i] = 0.f;
                for (int q = s0; q < s1; ++q) {
                    const int d = cload_ptr<int>(a.src_x)[q] - xm, sp = cload_ptr<int>(a.src_sp)[q] - a.sp0;
                    const float rate = cload_ptr<float>(a.src_rate)[q];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        any[i] = any[i] || d == i;
#pragma unroll
                        for (int f = 0; f < NF; ++f) e[f][i] = d == i && sp == f ? rate : e[f][i];
                    }
                }
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) e[f][i] = any[i] ? e[f][i] : -0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                Nb n[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    n[f].c = c[f][i];
                    n[f].xm = i > 0 ? c[f][i - 1] : left[f];
                    n[f].xp = i < 3 ? c[f][i + 1] : right[f];
                    n[f].ym = r > 0 ? v[f][r > 0 ? r - 1 : 0][i] : h.up[f][i];
                    n[f].yp = r < RY - 1 ? v[f][r < RY - 1 ? r + 1 : 0][i] : h.dn[f][i];
                    n[f].zm = vm[f][r][i];
                    n[f].zp = vp[f][i];
                }
                float ei[NF], oi[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) ei[f] = src.value ? e[f][i] : 0.f;
                M::cell(k, n, wind, src.value, ei, oi);
#pragma unroll
                for (int f = 0; f < NF; ++f) o[f][i] = oi[f];
            }
        };
        // (src_row is the same for every lane, so rows of no source take a path
        // without a branch per cell)
        if constexpr (M::SOURCES) {
            if (src_row >= 0) {
                cells(std::true_type{});
                return;
            }
        }
        cells(std::false_type{});
    };

    // The wind of the next 64 centre planes of level 1, one per lane, and which
    // of them hold a source in the tile's rows, one per bit: looked up a plane at a time they
    // would each put a scalar load's latency before that plane's barrier.
    float wind_t = 0.f;
    unsigned long long srow_t = 0;
    auto tables = [&](int p) __attribute__((always_inline)) {
        if constexpr (M::WIND == WIND_PLANE || M::SOURCES) {
            const int pz = march_index(min(p + lane, a.nz + K - 2), a.nz, perz);
            wind_t = plane_wind<M>(a, pz);
            if constexpr (M::SOURCES) {
                const int q = pz * a.ny;
                srow_t = __ballot(cload_ptr<int>(a.src_row)[q + ys0] < cload_ptr<int>(a.src_row)[q + ys1]);
            }
        }
    };
    float wind[K];
    int srow[K];
#pragma unroll
    for (int l = 0; l < K; ++l) {
        wind[l] = 0.f;
        srow[l] = -1;
    }

    auto plane = [&](int p, auto jc) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value;
        constexpr int par = J & 1, I0 = J & 3, I1 = (J + 1) & 3, I2 = (J + 2) & 3;
        take(V[I2]);
        issue(p + 2);
        export_edges(par, V[I1], std::integral_constant<int, par>{});
        export_plane(par, 0, V[I1]);
#pragma unroll
        for (int l = 1; l < K; ++l) export_plane(par, l, Q[l - 1][par]);
        // wind and sources of the planes the levels compute: level l's are those
        // of level l - 1 a plane ago
#pragma unroll
        for (int l = K - 1; l > 0; --l) {
            wind[l] = wind[l - 1];
            srow[l] = srow[l - 1];
        }
        if constexpr (M::WIND == WIND_PLANE)
            wind[0] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wind_t), (p - pa_) & 63));
        if constexpr (M::SOURCES)
            srow[0] = (srow_t >> ((p - pa_) & 63)) & 1 ? march_index(min(p, a.nz + K - 2), a.nz, perz) * a.ny : -1;
        lds_done();
        ring_barrier();
        Halo h[K];
#pragma unroll
        for (int l = 0; l < K; ++l) import_plane(par, l, h[l]);
        const int zo = p - (K - 1);
        const bool put = zo >= z0 && zo < z1;
        __amdgpu_buffer_rsrc_t ws[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f)
            ws[f] = __builtin_amdgcn_make_buffer_rsrc((void*)((char*)a.out[f] + zo * pbytes), 0,
                                                      put ? int(pbytes) : 0, 0x00027000);
        // inner rows first: they need no row of another lane
        march_rows<RY>([&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value;
            float xl[NE], xr[NE];
            if constexpr (XEX) {
                march_lds_get<NE>(edge_at(par, 1, !MIR && rf == FACE ? FACE : rf + r), xl);
                march_lds_get<NE>(edge_at(par, 0, !MIR && rl == FACE ? FACE : rl + r), xr);
            }
            float n[NF][4], o[NF][4];
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < 4; ++i) n[f][i] = V[I2][f][r][i];
            float el_[NF], er_[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                el_[f] = XEX ? xl[f] : 0.f;
                er_[f] = XEX ? xr[f] : 0.f;
            }
            row(r, V[I0], V[I1], n, h[0], el_, er_, wind[0], srow[0], o);
#pragma unroll
            for (int l = 1; l < K; ++l) {
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) n[f][i] = ES == 4 ? o[f][i] : S::up(S::down(o[f][i]));
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    el_[f] = XEX ? xl[l * NF + f] : 0.f;
                    er_[f] = XEX ? xr[l * NF + f] : 0.f;
                }
                row(r, Q[l - 1][par ^ 1], Q[l - 1][par], n, h[l], el_, er_, wind[l], srow[l], o);
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) Q[l - 1][par ^ 1][f][r][i] = n[f][i];
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) march_store<S>(o[f], ws[f], so[r]);
        });
    };
    for (int p = pa_; p <= pb_; p += 4) {
        if (((p - pa_) & 63) == 0) tables(p);
        plane(p, std::integral_constant<int, 0>{});
        if (p + 1 > pb_) break;
        plane(p + 1, std::integral_constant<int, 1>{});
        if (p + 2 > pb_) break;
        plane(p + 2, std::integral_constant<int, 2>{});
        if (p + 3 > pb_) break;
        plane(p + 3, std::integral_constant<int, 3>{});
    }
#else
    (void)a, (void)rows_l, (void)edge_l, (void)tx, (void)yb, (void)z0, (void)z1;
#endif
}

template <class M, class S, int RY, int W, int K, bool XEX, int RAG, bool MIR>
__global__ __launch_bounds__(64 * W) void march_kernel(const StepArgs* __restrict__ pa) {
    using R = MarchLds<M::NF, RY, W, K>;
    __shared__ __attribute__((aligned(16))) float rows_s[R::ROWS];
    __shared__ __attribute__((aligned(16))) float edge_s[R::EDGES];
    const StepArgs& a = *pa;
    const int by = R::T / a.mg[MG_LANES] * RY - 2 * K;
    const bool left_over = a.mg[MG_STEPS] != K;
    const int cz = left_over ? a.mg[MG_LEFT_CZ] : a.cz, chunks = left_over ? a.mg[MG_LEFT_CHUNKS] : a.chunks_z;
    const int tiles_y = (a.ny + by - 1) / by;
    const MarchTile t = march_tile(xcd_tile(blockIdx.x, gridDim.x), a.tiles_x, tiles_y, chunks, a.zfast != 0);
    const int z0 = t.z * cz;
    march_tile_steps<M, S, RY, W, K, K, XEX, RAG, MIR>(a, (RD_LDS float*)&rows_s[0], (RD_LDS float*)&edge_s[0], t.x,
                                                       t.y * by, z0, min(z0 + cz, a.nz));
}

// The batched form (served grids of diffusion or the Brusselator): a persistent
// launch walks the batch's (grid, tile) items, two steps of each grid that has
// as many left, one of a grid with one (the same tiles).  The items are listed
// by falling cost and dealt to the workgroups there and back (b, 2n-1-b, 2n+b,
// ..), without a counter: claiming them from one, atomics of every workgroup on
// one address, took longer than short items do (64 grids of 32^3 to 128^3, 20 to
// 200 steps each, from start to end: 14.4 ms claimed, 11.4 ms dealt).  `launch`
// counts the tick's launches.
//
// Against one step a launch on the tiled LDS ring (batched_tr_kernel, which
// still takes batches with a grid this kernel does not): 22.2 -> 11.4 ms on that
// batch, a launch of all 64 grids 150 -> 66 us a step.  Rows of short grids
// leave a third to a half of the lanes in halos and past the grid.
template <class S, int RY, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 2, W / 2))) void batched_march_kernel(
    const int* __restrict__ meta, const BatchEntry* __restrict__ ents, int launch) {
    using R = MarchLds<2, RY, W, 2>;                 // serves both models and both step counts
    __shared__ __attribute__((aligned(16))) float rows_s[R::ROWS];
    __shared__ __attribute__((aligned(16))) float edge_s[R::EDGES];
    const int ng = meta[0];
    const int total = meta[1];
    const int* first = meta + 4;
    RD_LDS float* rows_l = (RD_LDS float*)&rows_s[0];
    RD_LDS float* edge_l = (RD_LDS float*)&edge_s[0];
    const int n = gridDim.x, b = xcd_tile(blockIdx.x, n);
    for (int round = 0; (long long)round * n < total; ++round) {
        const long long item_l = (long long)round * n + (round & 1 ? n - 1 - b : b);
        if (item_l >= total) continue;
        const int item = int(item_l);
        int lo = 0, hi = ng - 1;                 // last grid with first_item <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first[mid] <= item) lo = mid; else hi = mid - 1;
        }
        const BatchEntry& en = ents[lo];
        const long long left = en.steps_left - 2LL * launch;
        if (left <= 0) continue;                 // this grid already finished
        const StepArgs& a = en.args[(en.parity + launch) & 1];
        const TileXYZ tc = tile_coords(a, item - first[lo]);
        const int z0 = tc.z * a.cz, z1 = min(z0 + a.cz, a.nz);
        const int yb = tc.y * (R::T / a.mg[MG_LANES] * RY - 4);
        // rows inside a wave with whole lanes, or any
        const bool plain = a.mg[MG_VARIANT] == MARCH_PLAIN, two = left >= 2;
#define RD_BATCH_TILE(M, K, X, RG) march_tile_steps<M, S, RY, W, K, 2, X, RG, false>(a, rows_l, edge_l, tc.x, yb, z0, z1)
#define RD_BATCH_MODEL(M)                                                                                      \
    if (two) {                                                                                                 \
        if (plain) RD_BATCH_TILE(M, 2, false, 0);                                                          \
        else RD_BATCH_TILE(M, 2, true, 2);                                                                  \
    } else {                                                                                                   \
        RD_BATCH_TILE(M, 1, true, 2);                                                                       \
    }
        if (en.model == 1) {
            RD_BATCH_MODEL(Brusselator)
        } else {
            RD_BATCH_MODEL(Diffusion<1>)
        }
#undef RD_BATCH_MODEL
#undef RD_BATCH_TILE
        __syncthreads();                         // the next item refills the exchange
    }
}

}  // namespace rdk
