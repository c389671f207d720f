// rd_march19.hpp -- the register march (rd_march.hpp) for the 19-point Laplacian.
//
// The LDS ring that 19-point grids ran on before stages whole rows of 256 cells
// a chunk (a quarter of the lanes idle at nx = 192) and takes one step a launch:
// Turing 192^3 FP32 44.5 us a step, where its bytes alone take 17.
// Here a lane keeps four cells of its row in three planes, and of the rows
// above and below, in registers, so that a plane costs each lane one row
// written to LDS and two read; the row's ends come from the next lanes.  That
// every edge neighbour lies in a cross of four values per x position (s, q
// below) leaves two lane moves per field and side.
//
// Rows stay inside a wave (16, 32 or 64 lanes), so no cell crosses waves but by
// the rows.  The boundary rows are exchanged for the newest plane of each
// level, so a level is two planes behind the one below it, and one barrier a
// plane serves all.  More than two steps do not fit the registers of two fields
// (185 at two).  What bounds it is vector issue: by counters, at Turing 192^3
// 73 to 75 % of the slots (four clocks an instruction, at 2.4 GHz) by 93
// instructions a cell and step, of which about 50 are the cell's and the rest those of rows
// and planes that only lead to it; 8 waves per CU.  Measured, us a step of Turing
// FP32, launches one after the other (a workgroup for every CU, where the grid
// has chunks enough): 192^3 20.7 (in a profiler's trace 22.5), 256^3 42.2, 64^3
// 5.6, 128^3 9.6, 130x101x77 8.4 (direct 59.6); single steps at 192^3 23.4.
#pragma once

#include "rd_march.hpp"

namespace rdk {

// K steps per launch; a lane holds four cells of one row.  Rows lie inside a
// wave (L divides 64), so x neighbours are the next lane's in every plane.
template <class M, class S, int W, int K, bool RAG>
__global__ __launch_bounds__(64 * W) void march19_kernel(const StepArgs* __restrict__ pa) {
    constexpr int NF = M::NF, T = 64 * W;
    static_assert(M::NO == NF && !M::SOURCES && M::WIND == WIND_NONE, "every field is stored; no directed term");
    __shared__ __attribute__((aligned(16))) float rows_s[2 * K * NF * T * 4];
#ifdef __HIP_DEVICE_COMPILE__
    constexpr int ES = int(sizeof(typename S::T));
    const StepArgs& a = *pa;
    RD_LDS float* rows_l = (RD_LDS float*)&rows_s[0];
    const int t = threadIdx.x;

    // ---- the tile ---------------------------------------------------------
    const int L = a.mg[MG_LANES], halo = a.mg[MG_HALO], G = T / L, BY = G - 2 * K;
    const bool left_over = a.mg[MG_STEPS] != K;
    const int cz = left_over ? a.mg[MG_LEFT_CZ] : a.cz, chunks = left_over ? a.mg[MG_LEFT_CHUNKS] : a.chunks_z;
    const int tiles_y = (a.ny + BY - 1) / BY;
    const MarchTile tile = march_tile(xcd_tile(blockIdx.x, gridDim.x), a.tiles_x, tiles_y, chunks, a.zfast != 0);
    const int yb = tile.y * BY, z0 = tile.z * cz, z1 = min(z0 + cz, a.nz);
    const int yg = t / L, x4 = t - yg * L;
    const bool perx = a.bck[0][0] == BC_PERIODIC, pery = a.bck[0][2] == BC_PERIODIC,
               perz = a.bck[0][4] == BC_PERIODIC;
    const int x = (tile.x * (L - 2 * halo) + x4 - halo) * 4;
    int xm = x;
    if (perx && halo) xm = x < 0 ? x + a.nx : x >= a.nx ? x - a.nx : x;
    xm = min(max(xm, 0), a.pitch - 4);
    // face rules along x: a periodic axis wraps by its halo lanes, or, in rows
    // of a whole wave, by the lane rotation
    const int e_last = (a.nx - 1) & 3;
    const bool first = x == 0 && !perx, last = x <= a.nx - 1 && x > a.nx - 5 && !perx;
    const bool mir_l = a.bck[0][0] == BC_MIRROR, mir_r = a.bck[0][1] == BC_MIRROR;
    const bool own_l = first && mir_l, in_l = first && !mir_l;
    const bool own_r = last && mir_r && !RAG, in_r = last && !mir_r && !RAG;
    bool after[3];
#pragma unroll
    for (int i = 1; i < 4; ++i) after[i - 1] = last && e_last + 1 == i;
    const int y = yb - K + yg, ym = march_index(min(max(y, -K), a.ny - 1 + K), a.ny, pery);
    const unsigned lo = unsigned(ym * a.pitch + xm) * ES;
    const bool st = x4 >= halo && x4 < L - halo && x >= 0 && x < a.nx && yg >= K && yg < K + BY && y < a.ny;
    const unsigned so = st ? unsigned(y * a.pitch + x) * ES : 0x80000000u;
    const int up_t = max(t - L, 0), dn_t = min(t + L, T - 1);
    auto row_at = [&](int par, int l, int f, int th) __attribute__((always_inline)) {
        return rows_l + (((par * K + l) * NF + f) * T + th) * 4;
    };
    const MarchConst<NF> k(a);
    float cl[NF], cr[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        cl[f] = scopy(a.bcv[f][0]);
        cr[f] = scopy(a.bcv[f][1]);
    }

    // ---- planes ------------------------------------------------------------
    const long long pbytes = a.plane * ES;
    using Raw = std::conditional_t<ES == 4, march_u4, march_u2>;
    Raw P[2][NF];                                    // two planes in flight
    float V[K][4][NF][4];                            // level l: three planes, the fourth slot the next
    float U[K][4][NF][4], D[K][4][NF][4];            // the rows above and below of the same planes
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < 4; ++i) V[l][j][f][i] = U[l][j][f][i] = D[l][j][f][i] = 0.f;
    auto issue = [&](int p, Raw (&q)[NF]) __attribute__((always_inline)) {
        const int pz = march_index(min(p, z1 - 1 + K), a.nz, perz);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)((const char*)a.in[f] + pz * pbytes), 0, int(pbytes), 0x00027000);
            if constexpr (ES == 4) q[f] = __builtin_amdgcn_raw_buffer_load_b128(rs, lo, 0, 0);
            else q[f] = __builtin_amdgcn_raw_buffer_load_b64(rs, lo, 0, 0);
        }
    };
    const int p0 = z0 - K, p1 = z1 + 2 * K - 2;      // newest plane of level 0 in the first and last iteration
    issue(p0, P[0]);
    issue(p0 + 1, P[1]);

    // one level up: the cells of the middle plane
    auto level = [&](int I0, int I1, int I2, const float (&v)[4][NF][4], const float (&u)[4][NF][4],
                     const float (&d)[4][NF][4], float (&o)[NF][4]) __attribute__((always_inline)) {
        Nb19 n[4][NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            float c[4], s[4], q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c[i] = v[I1][f][i];
                s[i] = (u[I1][f][i] + d[I1][f][i]) + (v[I0][f][i] + v[I2][f][i]);
                q[i] = (u[I0][f][i] + d[I0][f][i]) + (u[I2][f][i] + d[I2][f][i]);
            }
            if constexpr (RAG) {
                const float ce = march_elem(e_last, c[0], c[1], c[2]), se = march_elem(e_last, s[0], s[1], s[2]);
                const float gc = mir_r ? ce : cr[f], gs = mir_r ? se : 4.f * cr[f];
#pragma unroll
                for (int i = 1; i < 4; ++i) {
                    c[i] = after[i - 1] ? gc : c[i];
                    s[i] = after[i - 1] ? gs : s[i];
                }
            }
            auto ends = [&](const float (&r)[4], float kk, float& left, float& right) __attribute__((always_inline)) {
                left = lane_from_left_wrap(r[3]);
                right = lane_from_right_wrap(r[0]);
                left = own_l ? r[0] : left;
                left = in_l ? kk * cl[f] : left;
                if constexpr (!RAG) {
                    right = own_r ? r[3] : right;
                    right = in_r ? kk * cr[f] : right;
                }
            };
            float left, right, sl, sr;
            ends(c, 1.f, left, right);
            ends(s, 4.f, sl, sr);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                Nb19& m = n[i][f];
                m.c = c[i];
                m.xm = i > 0 ? c[i - 1] : left;
                m.xp = i < 3 ? c[i + 1] : right;
                m.ym = u[I1][f][i];
                m.yp = d[I1][f][i];
                m.zm = v[I0][f][i];
                m.zp = v[I2][f][i];
                m.s = s[i];
                m.sxm = i > 0 ? s[i - 1] : sl;
                m.sxp = i < 3 ? s[i + 1] : sr;
                m.q = q[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e[NF] = {};
            float oi[NF];
            M::cell(k, n[i], 0.f, false, e, oi);
#pragma unroll
            for (int f = 0; f < NF; ++f) o[f][i] = oi[f];
        }
    };

    auto plane = [&](int p, auto jc) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value;
        constexpr int par = J & 1, I0 = J & 3, I1 = (J + 1) & 3, I2 = (J + 2) & 3, I3 = (J + 3) & 3;
#pragma unroll
        for (int f = 0; f < NF; ++f) march_unpack<S>(P[par][f], V[0][I2][f]);
        issue(p + 2, P[par]);
#pragma unroll
        for (int l = 0; l < K; ++l)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const float(&c)[4] = V[l][I2][f];
                lds_st4(row_at(par, l, f, t), c[0], c[1], c[2], c[3]);
            }
        lds_done();
        ring_barrier();
#pragma unroll
        for (int l = 0; l < K; ++l)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                lds_ld4(row_at(par, l, f, up_t), U[l][I2][f]);
                lds_ld4(row_at(par, l, f, dn_t), D[l][I2][f]);
            }
        const int zo = p - (2 * K - 1);
        const bool put = zo >= z0;
        float o[NF][4];
#pragma unroll
        for (int l = 0; l < K; ++l) {
            level(I0, I1, I2, V[l], U[l], D[l], o);
            if (l < K - 1) {
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        V[l + 1 < K ? l + 1 : 0][I3][f][i] = ES == 4 ? o[f][i] : S::up(S::down(o[f][i]));
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(
                (void*)((char*)a.out[f] + zo * pbytes), 0, put ? int(pbytes) : 0, 0x00027000);
            march_store<S>(o[f], ws, so);
        }
    };
    for (int p = p0; p <= p1; p += 4) {
        plane(p, std::integral_constant<int, 0>{});
        if (p + 1 > p1) break;
        plane(p + 1, std::integral_constant<int, 1>{});
        if (p + 2 > p1) break;
        plane(p + 2, std::integral_constant<int, 2>{});
        if (p + 3 > p1) break;
        plane(p + 3, std::integral_constant<int, 3>{});
    }
#else
    (void)pa, (void)rows_s;
#endif
}

}  // namespace rdk
