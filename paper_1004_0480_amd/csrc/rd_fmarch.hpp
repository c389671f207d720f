// rd_fmarch.hpp -- the front model's step in one pass, its planes in registers:
// the register march (rd_march.hpp: lanes, tiles, exchange, reflected faces)
// with the chemical potential as its first level and the update as its second.
//
// Iteration p loads plane p + 2 of C and p + 1 of A and B, forms mu of plane p
// from C, and updates plane p - 1 of A, B and C from A, B and the mu planes
// p - 2, p - 1, p; a tile therefore loses two rows on each side.  The boundary
// rows of C, mu, A and B pass through LDS in one exchange per plane.  mu takes
// mirror ghosts on every face: with mirror faces of C the reflected rows give
// them by themselves.  A and B may be held or fixed beyond the z faces: the
// values of a whole plane are replaced then, outside the usual planes' path.
// The values are those of the two passes and of the LDS form (rd_fused.hpp):
// the same ChemPotential::mu, lapf and FrontCH::rates.
//
// The LDS form reads some 25 LDS values per two cells and keeps a wave for the
// loads; here it is 8 exchanged vectors per eight cells, and the loads in flight
// are registers.  Measured (us per step, tuned plans): 384x384x512 FP32 398 ->
// 371, BF16 307 -> 232 and with stochastic rounding (one generator call per
// species and lane, which holds exactly its four cells) 369 -> 295; 248x200x180
// BF16 29; default plans: 384x384x512 FP32 427 -> 371, BF16 381 -> 254, with
// rounding 295, 248x200x180 FP32 62 -> 42, BF16 65 -> 32, 64^3 26 -> 7.3.  At
// 384x384x512 FP32 it is bound by memory: 1.97 GB of traffic a step (1.09 times
// the fields: the tiles' halos) at 5.3 TB/s, a third of the issue slots of the
// vector units filled.  In BF16 it is half of them (1.03 GB at 4 TB/s), with
// rounding 79 %, 43 % of the instructions for the generator.
#pragma once

#include "rd_march.hpp"

namespace rdk {

// LDS of the register-march front kernel: by plane parity, the boundary rows
// of C, mu, A and B of every thread and the x-edge cells (the four fields of a
// row side by side).
template <int RY, int W>
struct Fmarch {
    static constexpr int T = 64 * W, NR = RY == 1 ? 1 : 2, NX = (W + T / kMarchMinLanes) * RY;
    static constexpr int ROWS = 2 * 4 * NR * T * 4, EDGES = 2 * 2 * NX * 4;   // floats
};

template <class S, int RY, int W, bool CD, bool SR, bool RAG>
__global__ __launch_bounds__(64 * W) void fmarch_kernel(const StepArgs* __restrict__ pa) {
    using F = Fmarch<RY, W>;
    constexpr int T = F::T, NR = F::NR, NX = F::NX, ES = int(sizeof(typename S::T));
    static_assert(!SR || (ES == 2 && !RAG), "stochastic stores: BF16, rows of whole lanes");
    __shared__ __attribute__((aligned(16))) float rows_s[F::ROWS];
    __shared__ __attribute__((aligned(16))) float edge_s[F::EDGES];
    if (SR) tick_clock<FrontCH>(*pa, (blockIdx.x | threadIdx.x) == 0);
#ifdef __HIP_DEVICE_COMPILE__
    const StepArgs& a = *pa;
    RD_LDS float* rows_l = (RD_LDS float*)&rows_s[0];
    RD_LDS float* edge_l = (RD_LDS float*)&edge_s[0];
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);

    const int L = a.mg[MG_LANES], halo = a.mg[MG_HALO], G = T / L;
    const int BY = G * RY - 4;
    const TileXYZ tc = tile_coords(a, xcd_tile(blockIdx.x, gridDim.x));
    const int yb = tc.y * BY, z0 = tc.z * a.cz, z1 = min(z0 + a.cz, a.nz);
    const int yg = t / L, x4 = t - yg * L;
    const int x = (tc.x * (L - 2 * halo) + x4 - halo) * 4;
    const int xm = min(max(x, 0), a.pitch - 4);
    const int e_last = (a.nx - 1) & 3;
    const bool first = x == 0, last = x <= a.nx - 1 && x > a.nx - 5;
    bool after[3];
#pragma unroll
    for (int i = 1; i < 4; ++i) after[i - 1] = last && e_last + 1 == i;
    const bool stored_x = x4 >= halo && x4 < L - halo && x >= 0 && x < a.nx && yg < G;
    unsigned lo[RY], so[RY], pc[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int yl = yg * RY + r, y = yb - 2 + yl;
        const int ym = march_index(min(max(y, -2), a.ny + 1), a.ny, false);
        lo[r] = unsigned(ym * a.pitch + xm) * ES;
        so[r] = stored_x && yl >= 2 && yl < 2 + BY && y < a.ny ? unsigned(y * a.pitch + x) * ES : 0x80000000u;
        // stochastic rounding: the counter of the lane's four cells on plane 0
        pc[r] = unsigned(((long long)ym * a.nx + xm) >> 2);
    }
    const unsigned dpc = unsigned((unsigned long long)unsigned(a.nx) * unsigned(a.ny) >> 2);
    const unsigned sr_n = SR ? unsigned(cload_ptr<StepClock>(a.clk_in)->n) : 0u;
    const unsigned sr_key = a.sr_key + unsigned(a.sp0);

    const int up_t = max(t - L, 0), dn_t = min(t + L, T - 1);
    auto row_at = [&](int par, int f, int k, int th) __attribute__((always_inline)) {
        return rows_l + (((par * 4 + f) * NR + k) * T + th) * 4;
    };
    // cross-wave x neighbours: the slot of this lane's outer cell, -1 if the
    // neighbour lane is in the wave (or there is none)
    int el = -1, er = -1;
    if (lane == 0 && x4 != 0 && !first) el = w;
    if (lane == 63 && x4 != L - 1 && !last && w < W - 1) er = w + 1;
    if (yg >= G) el = er = -1;
    auto edge_at = [&](int par, int side, int slot, int r) __attribute__((always_inline)) {
        return edge_l + ((par * 2 + side) * NX + slot * RY + r) * 4;
    };

    // the coefficients, in scalar registers
    struct Const {
        float kx[4], ky[4], kz[4], kc[4], p[6], dt;
    } k;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        k.kx[f] = scopy(a.kx[f]);
        k.ky[f] = scopy(a.ky[f]);
        k.kz[f] = scopy(a.kz[f]);
        k.kc[f] = scopy(a.kc[f]);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) k.p[i] = scopy(a.p[i]);
    k.dt = scopy(a.dt);

    const long long pbytes = a.plane * ES;
    using Raw = std::conditional_t<ES == 4, march_u4, march_u2>;
    using Plane = float[RY][4];
    Plane VA[4], VB[4], VC[4], Q[2];
    Raw PA[RY], PB[RY], PC[RY];
    auto issue = [&](int f, int p, Raw (&P)[RY]) __attribute__((always_inline)) {
        const int pz = march_index(p, a.nz, false);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)((const char*)a.in[f] + pz * pbytes), 0, int(pbytes), 0x00027000);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if constexpr (ES == 4) P[r] = __builtin_amdgcn_raw_buffer_load_b128(rs, lo[r], 0, 0);
            else P[r] = __builtin_amdgcn_raw_buffer_load_b64(rs, lo[r], 0, 0);
        }
    };
    auto take = [&](const Raw (&P)[RY], Plane& v) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RY; ++r) march_unpack<S>(P[r], v[r]);
    };
    // planes on and beyond a z face whose rule fixes A or B there
    auto fix_plane = [&](int f, int p, Plane& v) __attribute__((always_inline)) {
        if (p <= 0 || p >= a.nz - 1) {
            const Src s = resolve_axis(p, a.nz, a.bck[f][4], a.bck[f][5], a.bcv[f][4], a.bcv[f][5]);
            if (s.cst) {
#pragma unroll
                for (int r = 0; r < RY; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[r][i] = s.v;
            }
        }
    };
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) VA[j][r][i] = VB[j][r][i] = Q[j][r][i] = 0.f;
    issue(2, z0 - 2, PC);
    take(PC, VC[0]);
    issue(2, z0 - 1, PC);
    take(PC, VC[1]);
    issue(2, z0, PC);
    issue(0, z0 - 1, PA);
    issue(1, z0 - 1, PB);

    // a row's cells with its x neighbours: c patched beyond a ragged end
    auto xnb = [&](const float (&v)[4], float xl, float xr, float (&c)[4], float& left, float& right)
                   __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = v[i];
        if constexpr (RAG) {
            const float ce = march_elem(e_last, c[0], c[1], c[2]);
#pragma unroll
            for (int i = 1; i < 4; ++i) c[i] = after[i - 1] ? ce : c[i];
        }
        left = lane_from_left(c[3], xl);
        right = lane_from_right(c[0], xr);
        left = first ? c[0] : left;
        if constexpr (!RAG) right = last ? c[3] : right;
    };

    auto plane = [&](int p, auto jc) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value;
        constexpr int par = J & 1, I0 = J & 3, I1 = (J + 1) & 3, I2 = (J + 2) & 3;
        take(PC, VC[I2]);
        take(PA, VA[I2]);
        take(PB, VB[I2]);
        // (the last planes are read again rather than branched around)
        issue(2, min(p + 2, z1 + 1), PC);
        issue(0, min(p + 1, z1), PA);
        issue(1, min(p + 1, z1), PB);
        fix_plane(0, p, VA[I2]);
        fix_plane(1, p, VB[I2]);
        // centre planes: C of p, mu of p-1, A and B of p-1
        const Plane& c1 = VC[I1];
        const Plane& m1 = Q[par];
        const Plane& a1 = VA[I1];
        const Plane& b1 = VB[I1];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int r = j == 0 ? 0 : RY - 1;
            lds_st4(row_at(par, 0, j, t), c1[r][0], c1[r][1], c1[r][2], c1[r][3]);
            lds_st4(row_at(par, 1, j, t), m1[r][0], m1[r][1], m1[r][2], m1[r][3]);
            lds_st4(row_at(par, 2, j, t), a1[r][0], a1[r][1], a1[r][2], a1[r][3]);
            lds_st4(row_at(par, 3, j, t), b1[r][0], b1[r][1], b1[r][2], b1[r][3]);
        }
        if (el >= 0) {
#pragma unroll
            for (int r = 0; r < RY; ++r) lds_st4(edge_at(par, 0, el, r), c1[r][0], m1[r][0], a1[r][0], b1[r][0]);
        }
        if (er >= 0) {
#pragma unroll
            for (int r = 0; r < RY; ++r) lds_st4(edge_at(par, 1, er, r), c1[r][3], m1[r][3], a1[r][3], b1[r][3]);
        }
        lds_done();
        ring_barrier();
        float cu[4], cd[4], mu[4], md[4], au[4], ad[4], bu[4], bd[4];
        lds_ld4(row_at(par, 0, NR - 1, up_t), cu);
        lds_ld4(row_at(par, 0, 0, dn_t), cd);
        lds_ld4(row_at(par, 1, NR - 1, up_t), mu);
        lds_ld4(row_at(par, 1, 0, dn_t), md);
        lds_ld4(row_at(par, 2, NR - 1, up_t), au);
        lds_ld4(row_at(par, 2, 0, dn_t), ad);
        lds_ld4(row_at(par, 3, NR - 1, up_t), bu);
        lds_ld4(row_at(par, 3, 0, dn_t), bd);
        float xl[RY][4], xr[RY][4];
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int f = 0; f < 4; ++f) xl[r][f] = xr[r][f] = 0.f;
        if (el >= 0) {
#pragma unroll
            for (int r = 0; r < RY; ++r) lds_ld4(edge_at(par, 1, el, r), xl[r]);
        }
        if (er >= 0) {
#pragma unroll
            for (int r = 0; r < RY; ++r) lds_ld4(edge_at(par, 0, er, r), xr[r]);
        }
        const int zo = p - 1;
        const bool put = zo >= z0;
        __amdgpu_buffer_rsrc_t ws[3];
#pragma unroll
        for (int f = 0; f < 3; ++f)
            ws[f] = __builtin_amdgcn_make_buffer_rsrc((void*)((char*)a.out[f] + zo * pbytes), 0,
                                                      put ? int(pbytes) : 0, 0x00027000);
        // held outputs of the z faces
        const int hz = zo == 0 ? 16 : 0, hz1 = zo == a.nz - 1 ? 32 : 0;
        const bool held = ((a.out_held[0] | a.out_held[1]) & (hz | hz1)) != 0;
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            auto around = [&](const Plane& vm, const Plane& v, const float (&vp)[4], const float (&u)[4],
                              const float (&d)[4], float fl, float fr, Nb (&n)[4]) __attribute__((always_inline)) {
                float c[4], left, right;
                xnb(v[r], fl, fr, c, left, right);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    n[i].c = c[i];
                    n[i].xm = i > 0 ? c[i - 1] : left;
                    n[i].xp = i < 3 ? c[i + 1] : right;
                    n[i].ym = r > 0 ? v[r > 0 ? r - 1 : 0][i] : u[i];
                    n[i].yp = r < RY - 1 ? v[r < RY - 1 ? r + 1 : 0][i] : d[i];
                    n[i].zm = vm[r][i];
                    n[i].zp = vp[i];
                }
            };
            Nb nb[4];
            // mu of plane p
            around(VC[I0], VC[I1], VC[I2][r], cu, cd, xl[r][0], xr[r][0], nb);
            float mp[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) mp[i] = ChemPotential::mu(k, nb[i].c, lapf(nb[i], k, 3));
            // the update of plane p-1
            float la[4], lb[4], lm[4];
            around(Q[par ^ 1], Q[par], mp, mu, md, xl[r][1], xr[r][1], nb);
#pragma unroll
            for (int i = 0; i < 4; ++i) lm[i] = lapf(nb[i], k, 3);
            around(VA[I0], VA[I1], VA[I2][r], au, ad, xl[r][2], xr[r][2], nb);
#pragma unroll
            for (int i = 0; i < 4; ++i) la[i] = lapf(nb[i], k, 0);
            around(VB[I0], VB[I1], VB[I2][r], bu, bd, xl[r][3], xr[r][3], nb);
#pragma unroll
            for (int i = 0; i < 4; ++i) lb[i] = lapf(nb[i], k, 1);
            float o[3][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float A = VA[I1][r][i], B = VB[I1][r][i], C = VC[I0][r][i];
                const float q = CD ? (k.p[5] * A) * C : 0.f;
                float oi[3];
                FrontCH::rates(k, A, B, C, la[i], lb[i], -0.f, lm[i], q, oi);
#pragma unroll
                for (int f = 0; f < 3; ++f) o[f][i] = oi[f];
            }
            if (held) {
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[f][i] = held_out(a, f, -1, -1, zo, o[f][i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) Q[par ^ 1][r][i] = mp[i];
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                if constexpr (SR) {
                    const PhiloxOut q = philox2x32_10(pc[r] + unsigned(zo) * dpc, sr_n, sr_key + unsigned(f));
                    march_u2 d;
                    d.x = unsigned(bf16_stochastic(o[f][0], q.w0 & 0xffffu)) |
                          (unsigned(bf16_stochastic(o[f][1], q.w0 >> 16)) << 16);
                    d.y = unsigned(bf16_stochastic(o[f][2], q.w1 & 0xffffu)) |
                          (unsigned(bf16_stochastic(o[f][3], q.w1 >> 16)) << 16);
                    __builtin_amdgcn_raw_buffer_store_b64(d, ws[f], so[r], 0, 0);
                } else {
                    march_store<S>(o[f], ws[f], so[r]);
                }
            }
        }
    };
    for (int p = z0 - 1; p <= z1; p += 4) {
        plane(p, std::integral_constant<int, 0>{});
        if (p + 1 > z1) break;
        plane(p + 1, std::integral_constant<int, 1>{});
        if (p + 2 > z1) break;
        plane(p + 2, std::integral_constant<int, 2>{});
        if (p + 3 > z1) break;
        plane(p + 3, std::integral_constant<int, 3>{});
    }
#else
    (void)pa, (void)rows_s, (void)edge_s;
#endif
}

}  // namespace rdk
