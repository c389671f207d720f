// rd_march_cfg.hpp -- shapes of the register-march kernel (rd_march.hpp), its
// lane geometry, and the models and storage types it is compiled for.
#pragma once

#include "rd_internal.hpp"

namespace rdk {

// Rows per lane (four cells each), waves per workgroup, and the time steps a
// launch advances (every shape also takes fewer: one, and two where it takes
// more, for what is left of a count).
struct MarchCfg { int ry, w, k; };
constexpr MarchCfg kMarchCfgs[] = {{1, 8, 2}, {1, 16, 2}, {2, 8, 2}, {1, 8, 3}, {1, 16, 3}, {1, 8, 4}};
constexpr int kNumMarchCfgs = sizeof(kMarchCfgs) / sizeof(kMarchCfgs[0]);

constexpr int kMarchVX = 4;        // cells per lane and row
constexpr int kMarchMinLanes = 8;  // lanes of a tile row, at least (the LDS edge slots count on it)

// StepArgs.mg: lanes of a tile row, halo lanes on each side of it, steps of the
// plan's launches, and the z chunks of launches of fewer steps (which need not
// spread their z halo over as many planes)
// and in a batch's table the lane exchange (MARCH_*)
enum { MG_LANES = 0, MG_HALO = 1, MG_STEPS = 2, MG_LEFT_CZ = 3, MG_LEFT_CHUNKS = 4, MG_VARIANT = 5 };

// LDS bytes of shape i for nf fields: two buffers (by plane parity) of the
// boundary rows of every thread, and of the x-edge cells, at each level.
constexpr long long march_lds_bytes(int nf, int i) {
    const MarchCfg c = kMarchCfgs[i];
    const int t = 64 * c.w, rows = c.ry == 1 ? 1 : 2;
    return 2LL * c.k * nf * (16LL * rows * t + 8LL * (c.w + t / kMarchMinLanes) * c.ry);
}

// Fields of a pass model the kernel takes, 0 for the others: every field is
// stored, in the storage type, and no term but the x wind has a direction.
constexpr int march_fields(int pm) {
    switch (pm) {
    case PM_DIFF1: return 1;
    case PM_BRUSS: return 2;
    case PM_POLL1: return 1;
    case PM_POLL2: return 2;
    case PM_POLL2U: return 2;
    default: return 0;
    }
}

// Shape i is compiled for this storage and pass model.  More than two steps a
// launch pay for one field only: with two the arithmetic, repeated in the
// halos, already takes as long as the memory (Brusselator 256^3 FP32: 28.5 us
// a step at two steps, 35.2 at four).  For one field FP32 it is the reverse
// (diffusion 512^3: 104 us at two, 112 at three, 79 at four); two rows per lane
// never won there.
constexpr bool march_ok(int storage, int pm, int i) {
    if (i < 0 || i >= kNumMarchCfgs || (storage != ST_F32 && storage != ST_BF16)) return false;
    const int nf = march_fields(pm);
    const MarchCfg c = kMarchCfgs[i];
    return (nf == 1 ? c.ry == 1 : nf == 2 && c.k == 2) && march_lds_bytes(nf, i) <= 160 * 1024;
}

// Shapes of the register-march front kernel (rd_fmarch.hpp): rows per lane,
// waves per workgroup.  One step per launch; its tiles lose two rows on each
// side, as those of two steps of the others do (mu, then its Laplacian).
struct FmarchCfg { int ry, w; };
constexpr FmarchCfg kFmarchCfgs[] = {{2, 8}, {1, 8}, {1, 16}};
constexpr int kNumFmarchCfgs = sizeof(kFmarchCfgs) / sizeof(kFmarchCfgs[0]);
constexpr bool fmarch_ok(int storage, int i) {
    return (storage == ST_F32 || storage == ST_BF16) && i >= 0 && i < kNumFmarchCfgs;
}
// Variants: C with a redissolution term, stochastic rounding, rows that end
// inside a lane.
hipError_t launch_fmarch(int storage, int cfg, bool cd, bool sr, bool ragged, const StepArgs* d, long long blocks,
                         hipStream_t s);
hipError_t launch_fmarch_f32(int cfg, bool cd, bool sr, bool ragged, const StepArgs* d, long long blocks, hipStream_t s);
hipError_t launch_fmarch_bf16(int cfg, bool cd, bool sr, bool ragged, const StepArgs* d, long long blocks, hipStream_t s);

// The 19-point register march (rd_march19.hpp): eight waves a workgroup, one
// row of four cells per lane, one or two steps a launch.
constexpr int kMarch19Waves = 8, kMarch19MaxSteps = 2;
constexpr int march19_fields(int pm) {
    return pm == PM_DIFF1 ? 1 : pm == PM_BRUSS || pm == PM_TURING ? 2 : 0;
}
hipError_t launch_march19(int storage, int pm, int k, bool ragged, const StepArgs* d, long long blocks, hipStream_t s);
hipError_t launch_march19_f32(int pm, int k, bool ragged, const StepArgs* d, long long blocks, hipStream_t s);
hipError_t launch_march19_bf16(int pm, int k, bool ragged, const StepArgs* d, long long blocks, hipStream_t s);

// The lane exchange a geometry needs: none (rows lie inside a wave and end at
// whole lanes), through LDS, or through LDS with a last lane that is not full.
// MARCH_MIRROR is added where both x faces are mirrors.
enum { MARCH_PLAIN = 0, MARCH_EDGES = 1, MARCH_RAGGED = 2, MARCH_MIRROR = 4 };

// Tiles of the batched launch: rows per lane, waves.
struct BatchMarchCfg { int ry, w; };
constexpr BatchMarchCfg kBatchMarch = {1, 8};

// One batched launch of up to two steps per grid; workgroups a CU holds.
hipError_t launch_batched_march(int storage, const int* meta, const BatchEntry* ents, int launch, int blocks, hipStream_t s);
int batched_march_blocks_per_cu(int storage);
hipError_t launch_batched_march_f32(const int* meta, const BatchEntry* ents, int launch, int blocks, hipStream_t s);
hipError_t launch_batched_march_bf16(const int* meta, const BatchEntry* ents, int launch, int blocks, hipStream_t s);
int batched_march_blocks_per_cu_f32();
int batched_march_blocks_per_cu_bf16();

// One launch of k steps (1, 2 or the shape's) of shape cfg; `variant` MARCH_*.
hipError_t launch_march(int storage, int pm, int cfg, int k, int variant, const StepArgs* d, long long blocks,
                        hipStream_t s);
#define RD_DECLARE_MARCH(sfx)                                                                     \
    hipError_t launch_march_##sfx(int pm, int cfg, int k, int variant, const StepArgs* d, long long blocks, \
                                  hipStream_t s);
RD_DECLARE_MARCH(f32_diff)
RD_DECLARE_MARCH(f32_react)
RD_DECLARE_MARCH(f32_poll)
RD_DECLARE_MARCH(bf16_diff)
RD_DECLARE_MARCH(bf16_react)
RD_DECLARE_MARCH(bf16_poll)
#undef RD_DECLARE_MARCH

}  // namespace rdk
