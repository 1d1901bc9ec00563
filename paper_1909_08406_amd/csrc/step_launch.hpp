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
// eighth of the tiles per XCD; or XCD_RUNS + 4 lg: runs of 2^lg consecutive
// tiles, one run per XCD in turn, so that all XCDs stay near one another in
// every one of the step's 82 streams.
constexpr uint32_t XCD_DISPATCH = 0, XCD_EIGHTHS = 1, XCD_RUNS = 2;

// The mapping of a launch with lbm_tuning.xcd_remap on. q_bytes: bytes of a
// q-block (0: many boxes); held: bytes of both population buffers.
//   Runs by default: HBM serves the 82 streams faster when they advance
// together than as 8 x 82 streams an eighth apart, and a run keeps the lines
// that its tiles share in one L2. Runs of 16 against eighths, us per step:
// FP32 256^3 2071 / 2182, 251x183x130 734 / 769; FP64 192^3 1805 / 1844;
// FP16 256^3 1045 / 1082, FP16+SR 1085 / 1091; BF16+SR E1 251x183x130 383 /
// 400. Runs of 64 for many boxes (256 uneven ones FP32 3635 / 3756, FP16+SR
// 1889 / 1913) and where a q-block has 128 MiB or more: shorter runs fall
// behind there (FP32 512 MiB 1.18x of eighths with runs of 8, FP16 384 MiB
// 1.08x, 1.03x with runs of 16), runs of 64 do not (0.94-1.00x from 128 to
// 1024 MiB).
//   Eighths where the q-blocks lie a power of two up to 16 MiB apart: the
// streams then meet in the same memory channels wherever they advance
// together (FP32 4, 8, 16 MiB: runs of 16 1.01x, 1.06x, 1.03x; FP64 1.05x,
// 1.03x, 1.04x; at 6, 10, 12, 14 MiB 0.91-0.98x; 16-bit blocks are padded
// apart and show it at 16 MiB only, 1.04x against 0.91-0.98x around it).
// 16-bit blocks of 384 MiB and more gained nothing from any run (512^3
// FP16+SR 8.74 / 8.78 ms alone, 0.3-0.7% the other way among other work).
//   And eighths while both buffers hold up to 128 MiB: an XCD then finds much
// of its part of the last step in its own L2 (4 MiB each; 48^3 FP16+SR, 36 MB:
// 12.2 against 13.5 us; FP32, 72 MB: 14.6 / 14.9; 800x400x1, 105 MB: 33.8 /
// 34.0, with walls 33.2 / 36.2; otherwise equal from 86 to 172 MB; FP16 258 MB
// 0.89 of eighths).
inline uint32_t xcd_map(uint32_t remap, uint64_t q_bytes, int elem_bytes, uint64_t held)
{
    if (!remap) return XCD_DISPATCH;
    const bool pow2 = q_bytes != 0 && (q_bytes & (q_bytes - 1)) == 0 && q_bytes <= (16u << 20);
    if (held <= (128u << 20) || (pow2 && (elem_bytes > 2 || q_bytes == (16u << 20))) ||
        (elem_bytes == 2 && q_bytes >= (384u << 20)))
        return XCD_EIGHTHS;
    return XCD_RUNS + 4 * (q_bytes == 0 || q_bytes >= (128u << 20) ? 6 : 4);
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
