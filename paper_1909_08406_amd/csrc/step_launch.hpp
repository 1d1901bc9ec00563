// Launch description of one collide-and-stream step and the launchers of
// the step kernels, one per storage form and rounding mode. Each launcher
// lives in its own translation unit (step_*.hip), so the many template
// instances of the step kernel compile in parallel; the host side of the
// library (lbm.hip) fills a StepLaunch and calls the launcher of its form.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"

namespace lbm {

// Block sizes of the step-kernel variants; the batched launch keeps one
// (box, tile) list per block size.
constexpr int NBLK = 4;
constexpr int BLK_SIZES[NBLK] = {128, 256, 512, 1024};
constexpr int blk_index(int blk) { return blk == 128 ? 0 : blk == 256 ? 1 : blk == 512 ? 2 : 3; }

// Cache-policy hints of a variant.
constexpr int FL_NT_LOAD = 1;   // non-temporal loads (streamed once)
constexpr int FL_NT_STORE = 2;  // non-temporal stores
// Stage each tile's source rows in LDS (k_step_lds): 16-bit storage, per-box
// launches of boxes whose x-rows hold whole tiles; elsewhere the variant
// runs the plain kernel of its block size.
constexpr int FL_LDS = 4;

// Step-kernel launch variants: block size and cache-policy hints. Every
// variant computes the same per-node arithmetic.
struct VariantDesc {
    int blk;
    int fl;
};
constexpr VariantDesc VARIANTS[] = {
    {256, 0}, {256, FL_NT_LOAD | FL_NT_STORE}, {512, 0}, {128, 0}, {256, FL_NT_STORE}, {1024, 0}, {256, FL_LDS},
};
constexpr int NVARIANTS = int(sizeof(VARIANTS) / sizeof(VARIANTS[0]));

struct BatchBox;

// How a launch's tiles lie on the 8 XCDs: dispatch order; one contiguous
// eighth of the tiles per XCD; or runs of XCD_RUN consecutive tiles, one run
// per XCD in turn, so that all XCDs stay near one another in every one of the
// step's 82 streams.
constexpr uint32_t XCD_DISPATCH = 0, XCD_EIGHTHS = 1, XCD_RUNS = 2;
constexpr uint32_t XCD_RUN_LOG2 = 4, XCD_RUN = 1u << XCD_RUN_LOG2;

// The mapping of a launch with lbm_tuning.xcd_remap on. block, stride: bytes
// of a q-block and from one to the next (0: many boxes); held: bytes of both
// population buffers. Times below are us per step of dispatch order / eighths
// / runs.
//   Runs by default: HBM serves the 82 streams faster when they advance
// together than as 8 x 82 streams an eighth apart, and a run keeps the lines
// that its tiles share in one L2. FP32 256^3 2075 / 2188 / 2071, 512^3 15022 /
// 14320 / 14291; FP64 192^3 1844 eighths, 1805 runs, 256x256x512 9136 / 8677 /
// 8640; FP16+SR 251x183x130 386 / 395 / 384, 512x512x480 8347 / 8209 / 8188,
// 512^3 8878 / 8813 / 8831 (0.5% behind eighths among other work); 256 uneven
// boxes FP32 4734 / 4765 / 4424, FP16+SR 2361 / 2693 / 2351; 64 boxes of 64^3
// FP64 5480 / 4260 / 4229. Dispatch order is within 1% of runs for most boxes,
// ahead by up to 3% for FP64 batches and up to 30% behind elsewhere (the lines
// that tiles share are fetched by both of their XCDs). Runs of 64 are within 1%
// of runs of 16 for one box up to 1 GiB q-blocks and up to 4% behind for FP32
// batches; runs of 8 fall behind by 8-18% at q-blocks of 128-512 MiB.
//   Eighths while both buffers fit in the last-level cache of 256 MiB: HBM
// then serves little, and an XCD finds much of its part of the last step in
// its own L2 (4 MiB each). 34 MiB FP16+SR 12.1 / 11.5 / 12.1; 106 MiB FP32
// 21.4 / 19.3 / 19.5; 154 MiB FP16+SR 33.5 / 31.0 / 31.4, with walls BF16 37.3
// / 32.8 / 33.6; 207 MiB isothermal FP16+SR 42.4 / 36.5 / 38.3; 246 MiB FP32
// 39.7 all three. (At 176 MiB 16-bit forms of E2 alone gain 3% from runs.)
// Just beyond, 263 MiB FP32 49.5 / 51.5 / 48.8.
//   And eighths where those meet fewer of the same memory channels at a time
// than runs do: q-blocks within 1/64 of 16 MiB, in every width (15.75, 15.88,
// 16, 16.12, 16.25 MiB FP32: runs 1.03, 1.05, 1.03, 1.03, 1.03 of eighths,
// FP16+SR 1.01, 1.06, 1.04, 1.08, 1.01, FP64 16 MiB 1.04; at 15.5 and 16.5 MiB
// 0.97-0.99), and q-blocks exactly 4 or 8 MiB apart, for any shape (8 MiB FP32
// 1.03, FP64 1.03-1.06; 4 MiB FP64 1.00-1.05, FP32 0.96-1.01 from box to box;
// at 3.75, 4.25, 7.75 and 8.25 MiB 0.93-0.99; 16-bit blocks are padded apart
// and gain from runs at 8 MiB, 0.98).
inline uint32_t xcd_map(uint32_t remap, uint64_t block, uint64_t stride, uint64_t held)
{
    if (!remap) return XCD_DISPATCH;
    constexpr uint64_t MiB = 1u << 20;
    const bool near16 = block >= 16 * MiB - MiB / 4 && block <= 16 * MiB + MiB / 4;
    return held <= 256 * MiB || stride == 4 * MiB || stride == 8 * MiB || near16 ? XCD_EIGHTHS : XCD_RUNS;
}

// Everything one step launch needs. Pointers are device pointers unless
// noted; the per-box arrays are host arrays of nboxes entries.
struct StepLaunch {
    const void* in;          // current population buffer (all boxes)
    void* out;               // the other buffer
    int newton;              // Newton steps of the equilibrium solve, 1..4
    int schedule;            // LBM_SCHEDULE_PER_BOX (0) or LBM_SCHEDULE_BATCHED (1)
    int variant;             // 0 .. NVARIANTS-1 (energy-conserving model only)
    uint32_t model;          // MODEL_* bits
    uint32_t xcd_remap;      // runs of consecutive tiles per XCD (xcd_map)
    uint32_t step;           // step count seeding the stochastic rounding
    const uint32_t* step_base;  // device counter added to step (graph replays), or null
    hipStream_t stream;
    // batched schedule
    const BatchBox* table;   // per-box parameters
    const uint2* tiles[NBLK];  // (box, tile) lists per block size
    uint64_t ntiles[NBLK];
    uint64_t held;           // bytes of both population buffers
    // per-box schedule (host arrays)
    int nboxes;
    const StepParams* params;  // kernel parameters of each box (step fields set by the launcher)
    const uint64_t* offset;    // element offset of each box in a buffer
    const uint64_t* nodes;     // nodes of each box
};

// Launchers: queue one step and return 0, or a negative lbm_error.
int enqueue_step_f64(const StepLaunch& L);
int enqueue_step_f32(const StepLaunch& L);
int enqueue_step_f32_sr(const StepLaunch& L);
int enqueue_step_f32s(const StepLaunch& L);
int enqueue_step_f16s(const StepLaunch& L);
int enqueue_step_f16s_sr(const StepLaunch& L);
int enqueue_step_bf16s(const StepLaunch& L);
int enqueue_step_bf16s_sr(const StepLaunch& L);

}  // namespace lbm
