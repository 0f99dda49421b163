// m2c_kernels.h -- launch interfaces of the device kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "m2c_internal.h"

namespace m2c {

// Device buffers of one run of a batch (the kernels pick the state buffers
// from the run's device-side parity sc->cur).
struct RunDesc {
    Grid g;
    double* W[2];
    double* W1;
    uint8_t* chi[2];
    int32_t* queue;
    int32_t* fslot;
    double* fluxF;
    double* star;
    int32_t* flips;
    int32_t* blockcnt;
    DevScalars* sc;
    long long qcap;
    int nblk_compact;
    int tiles_x, tiles_y, tiles_z, kz;
};

// Arguments of one bulk Runge-Kutta stage launch.
struct StageArgs {
    Grid g;
    const double* Win;             // stage input state [6][N]
    const double* W0;              // start-of-step state [6][N] (blended stages)
    double* Wout;                  // stage output [6][N]
    const uint8_t* chi;            // material ids frozen for the step
    uint8_t* chi_next;             // last stage: ids of the new level set
    int32_t* flips;                // last stage: flipped cells (append)
    const int32_t* fslot;          // [3N] face -> queue slot or -1
    const double* fluxF;           // [qcap][10] one-sided interface fluxes
    long long qcap;
    DevScalars* sc;
    int tiles_x, tiles_y, tiles_z, kz;
    double c0, c1;                 // blend of the stage: c0 W0 + c1 (Win + dt R)
};

// Interface work-queue arguments (compaction, FIVER, phase update).
struct IfaceArgs {
    Grid g;
    const double* Win;             // stage input state [6][N]
    const uint8_t* chi;            // ids frozen for the step
    int32_t* queue;
    int32_t* fslot;
    double* fluxF;                 // [qcap][10]
    double* star;                  // [8][qcap]
    int32_t* blockcnt;
    long long qcap;
    int nblk;                      // compaction blocks
    DevScalars* sc;
};

struct PhaseArgs {
    Grid g;
    double* W;                     // new state [6][N] (updated in place at flipped cells)
    const uint8_t* chi_old;        // ids of the step
    const uint8_t* chi_new;        // ids of the new level set
    const int32_t* flips;
    const int32_t* fslot;
    const double* star;
    long long qcap;
    DevScalars* sc;
};

bool stage_tile_supported(int tx, int ty);
// FP64 stage blocks resident on the chip at once: two per CU, which is what
// the registers of every tuned FP64 stage kernel allow (their build test holds
// them to it).
int stage_slots();
// Planes per stage block, from the number of blocks at a given number of
// planes (blocks: int -> long long).  Three regimes:
//   at least 4096 blocks with 32 or 16 planes (16 rounds of two blocks per
//     CU): that many, so that the prologue of a block's march and the
//     re-read halo planes are amortised (32 measured 1.5% faster than 16 on
//     384^3, where the line was drawn; it costs the grids just below it: 256^3
//     gets 16 planes, 794 us per stage launch, where 32 take 755, and 200^3
//     gets 8, 466 us, where 15 take 450);
//   grids whose blocks of fewer than 8 planes all fit on the chip at once:
//     the fewest planes that still fit.  There the launch lasts as long as
//     one block's march, so fewer planes are a shorter launch until the
//     blocks no longer run side by side (per stage launch, 8 planes -> this
//     rule: 32^3 47 -> 14 us, 50x43x37 54 -> 18 us, 64^3 52 -> 31 us; one
//     plane fewer than fits: 64^3 36 us, 80^3 58 against 46 us).  FP64 only
//     (slots 0: not at all): the face below a block's first plane is
//     evaluated in the march's prologue, by code that rounds differently from
//     that for the faces inside it, so results depend on where a grid is
//     split: at 1e-12 in FP64, at 3e-9 in the mixed form, which keeps to
//     blocks of 8;
//   otherwise 8 (128^3: 128 us; 4, 6, 10 and 16 planes: 143, 142, 131, 149).
template <class Blocks>
int stage_planes(Blocks blocks, int slots)
{
    if (blocks(32) >= 4096) return 32;
    if (blocks(16) >= 4096) return 16;
    for (int kz = 1; kz < 8; ++kz)
        if (blocks(kz) <= slots) return kz;
    return 8;
}
// stage: kind 1 (first), 2 (last, blended), 3 (middle of RK3), 4 (forward
// Euler); the batched kernel has kinds 1 and 2 (TVD-RK2)
hipError_t launch_stage(int stage, bool mixed, int tx, int ty, const StageArgs& a, hipStream_t s);
// the same with the configured limiter and flux (any, including MC + HLLC)
hipError_t launch_stage_opts(int stage, bool mixed, int tx, int ty, const StageArgs& a, hipStream_t s);
// general-EOS stage kernels (FP64; tiles 16x15 and 64x2)
bool stage_tile_supported_eos(int tx, int ty);
hipError_t launch_stage_eos(int stage, int tx, int ty, const StageArgs& a, hipStream_t s);
// the default scheme on the 16x15 tile for fs, the set of the two
// materials' families (eos::fam_set): sets with NASG, and the others
hipError_t launch_stage_eos_nasg(int stage, int fs, const StageArgs& a, hipStream_t s);
hipError_t launch_stage_eos_other(int stage, int fs, const StageArgs& a, hipStream_t s);
// items: (run, tile) pairs over all runs of a batch
hipError_t launch_stage_batch(int stage, bool mixed, int tx, int ty, const RunDesc* runs, const int2* items,
                              int nitems, hipStream_t s);

// Interface kernels (k_interface.hip).
constexpr int COMPACT_THREADS = 256;
constexpr int COMPACT_CELLS_PER_THREAD = 16;
constexpr int COMPACT_CELLS_PER_BLOCK = COMPACT_THREADS * COMPACT_CELLS_PER_THREAD;
// The compaction blocks of a grid are taken in chunks of consecutive ones, a
// launch block and a count of faces per chunk; one compaction block each up
// to COMPACT_CHUNKS.  The limit bounds the counts that each chunk adds up and
// the blocks that a kept queue launches to no purpose; where it lies matters
// little (384^3 with 13824 compaction blocks and a moving interface: steps
// of 5.01, 4.93, 4.96, 4.94 and 4.97 ms at 1024, 2048, 4096, 8192 and 16384
// chunks).
constexpr int COMPACT_CHUNKS = 4096;
__host__ __device__ constexpr int compact_per_chunk(int nblk) { return (nblk - 1) / COMPACT_CHUNKS + 1; }
__host__ __device__ constexpr int compact_chunks(int nblk) { return (nblk - 1) / compact_per_chunk(nblk) + 1; }
// What the launch after k_step_begin does to open a step: end the previous
// one of the same call, form dt and clear the accumulators (dt_imposed > 0:
// that dt).
struct StepOpen {
    int end_prev, begin;
    double dt_imposed;
};
// start of a single-grid step: the previous step's phase update (prev_phase,
// nullable) and the counts of the interface queue
hipError_t launch_step_begin(const IfaceArgs& a, const PhaseArgs* prev_phase, hipStream_t s);
// opens the step and writes a rebuilt queue without solving it
hipError_t launch_scatter(const IfaceArgs& a, const StepOpen& o, hipStream_t s);
hipError_t launch_end_step(DevScalars* sc, int stages, hipStream_t s);
// whether the first FIVER launch of a step opens it and writes a rebuilt queue
// (else launch_scatter does, before it)
bool fiver_opens(const IfaceArgs& a, const MlpDev* mlp);
// open (nullable): this launch opens the step; mlp: the learned guess (null:
// acoustic)
hipError_t launch_fiver(const IfaceArgs& a, bool record, const StepOpen* open, const MlpDev* mlp, hipStream_t s);
hipError_t launch_phase(const PhaseArgs& a, hipStream_t s);
// Batched forms: cmap lists the compaction chunks as (run, chunk of run); the
// compaction also opens every run's step.
hipError_t launch_compact_batch(const RunDesc* runs, const int2* cmap, int ncblocks, hipStream_t s);
hipError_t launch_fiver_batch(const RunDesc* runs, int nruns, int stage, hipStream_t s);
hipError_t launch_phase_batch(const RunDesc* runs, int nruns, hipStream_t s);

// Learned star-pressure guess (k_mlp.hip).
struct MlpDev;
hipError_t launch_mlp_features(long long n, const double* in, const double* eos, const double* ps, float* X,
                               float* tg, hipStream_t s);
hipError_t launch_mlp_forward(long long n, const float* X, const MlpDev& m, float* y, hipStream_t s);
// gradient of samples [i0, i0 + cnt) as partial sums, one per block of
// mlp_grad_blocks(cnt), at part[block][GRAD_STRIDE]
int mlp_grad_blocks(long long cnt);
hipError_t launch_mlp_grad(long long i0, long long cnt, long long ntot, float invB, const float* X, const float* T,
                           const MlpDev& m, float* part, hipStream_t s);
hipError_t launch_grad_sum(const float* part, int nblk, float* grad, hipStream_t s);
hipError_t launch_fill_f32(float* p, long long n, float v, hipStream_t s);
hipError_t launch_adam(const MlpDev& md, float* m, float* v, const float* part, int nblk, float* sse, float lr,
                       float b1, float b2, float eps, int step, hipStream_t s);
hipError_t launch_mlp_sync(const MlpDev& m, hipStream_t s);
hipError_t launch_points_guess(long long n, const double* in, const double* eos, const MlpDev& m, double* guess,
                               hipStream_t s);

// Per-step bookkeeping and state conversion (k_misc.hip).
hipError_t launch_end_batch(const RunDesc* runs, int nruns, int stages, hipStream_t s);
hipError_t launch_lambda(const Grid& g, const double* W, const uint8_t* chi, DevScalars* sc, hipStream_t s);
hipError_t launch_accept_lambda(DevScalars* sc, hipStream_t s);
// lam: the state's CFL maximum to lam_set as well
hipError_t launch_prim_to_cons(const Grid& g, const double* prim6, double* W, uint8_t* chi,
                               DevScalars* sc, bool lam, hipStream_t s);
hipError_t launch_cons_to_prim(const Grid& g, const double* W, const uint8_t* chi, double* prim6,
                               hipStream_t s);
hipError_t launch_chi_from_phi(const Grid& g, const double* W, uint8_t* chi, hipStream_t s);
hipError_t launch_fill_i32(int32_t* p, long long n, int32_t v, hipStream_t s);
hipError_t launch_hllc_points(long long n, const double* qL, const double* qR, double gamma, double pc,
                              bool mixed, double* F, hipStream_t s);
// guess (nullable): candidate initial pressures, judged against the
// acoustic guess; nfb (nullable) counts problems that started from the
// acoustic guess although a candidate was given.
hipError_t launch_riemann_points(long long n, const double* in, const double* eos, const double* guess,
                                 double rtol, int maxit, double* out, int32_t* iters, int32_t* vac,
                                 unsigned long long* nfb, hipStream_t s);

}  // namespace m2c
