// Host-callable launchers of the UGKWP kernels (kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.hpp"

namespace ugkwp {

// scan partial slots needed for an exclusive scan over n integers
long long scan_partials_needed(long long n);
long long count_partials_needed(long long nc, long long nff);

// Dev::long_from of a batch of nc cells whose instances have at most per_cell reference particles (the
// larger of n_ref and n_min)
int long_from(long long nc, long long per_cell);
// rows of waves over which the lists of such a batch are spread
int list_split(long long nc, bool sparse, long long per_cell);

// measurement hook: called around each group of launches of a step (no-op by default)
enum ProfSlot : int {
    kSlotPrim = 0,      // k_prim_dt
    kSlotCellPrep,      // k_cell_prep (with the counts of entering particles)
    kSlotScan,          // k_offsets
    kSlotFlux,          // k_flux
    kSlotSample,        // k_sample
    kSlotStream,        // k_stream, k_stream_long, k_stream_in, k_track
    kSlotStreamWall,    // (no kernels: k_track re-emits at walls)
    kSlotCount,         // (no kernels: k_track counts)
    kSlotScan2,         // scan of the bucket counts
    kSlotScatter,       // k_scatter
    kSlotGather,        // k_gather, k_gather_long, k_update, k_heat
    kSlotFinal,         // (the averaging kernels when averaging is on)
    kNumSlots
};
struct Prof {
    virtual ~Prof() {}
    virtual void begin(int) {}
    virtual void end(int) {}
};

// launch shapes of the kernels whose shape is tunable; every choice gives the same results
struct LaunchCfg {
    int stream_bs = 256;  // k_stream block size: 128, 256 or 512 (a wave per cell)
    int stream_ilp = 1;   // k_stream runs of 64 particles loaded together: 1 or 2
    int sample_wpb = 4;   // k_sample waves per block: 1, 2, 4 or 8
    int flux_bs = 128;    // k_flux and k_flux2 block size: 64, 128 or 256 (k_flux2_axes has one shape)
};
bool launch_cfg_valid(const LaunchCfg &c);

void launch_fill_f64(double *p, long long n, double v, hipStream_t s);
// a new state from W0 [nc][5] in device memory; *worst: its first non-physical cell, which leaves the
// state before as it is, or LLONG_MAX
void launch_take_state(const Dev &D, const double *W0, long long *worst, hipStream_t s);
// one full time step on stream s; particles are read from pa[buf] and left in pa[buf ^ 1]
void launch_step(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s, Prof *pr);
// a wave-only step when no particle exists anywhere (the same results as launch_step)
void launch_step_wave_only(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s, Prof *pr);
// Shakhov model: each cell's heat flux from the particles in pa[buf]
void launch_heat(const Dev &D, int buf, hipStream_t s);
// [nc][5] field (0 W, 1 W^p, 2 W^h, 3 primitives) into device memory out
void launch_moments(const Dev &D, int which, double *out, hipStream_t s);
// the particles of pa[buf] in their order, one after the other, into pa[buf ^ 1] (between steps)
void launch_pack(const Dev &D, int buf, hipStream_t s);
// Wbar = A / D of the time averaging, [nc][5] in out
void launch_avg_out(const Dev &D, double *out, hipStream_t s);

}  // namespace ugkwp
