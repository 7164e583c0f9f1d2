// Half-steps of the long-range paths driven by their low Philox draws
// (kmc_draws.hip), shared with the host library.  Not part of the public ABI.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "kmc_internal.h"

namespace kmc {

constexpr int kDrawBlock = 1024;      // threads per workgroup
constexpr int kDrawMaxGrid = 256;     // workgroups per launch, at most
constexpr int kDrawSlots = 512;       // entries of a generating workgroup's list (slot 0: its count)
constexpr int kDrawList = 256;        // draws of one resolving workgroup, at most
constexpr int kDrawTableEntries = 65536;  // (step, device) entries of the threshold table, at least one step
constexpr int kDrawMaxSteps = 1024;   // steps per threshold table
constexpr double kDrawMaxMean = 8192.0;   // expected draws per half-step, at most

// First rail of part i of n of the generating workgroups' rails.
__host__ __device__ inline int64_t draw_share(int64_t rails, int64_t i, int64_t n) { return rails * i / n; }

struct DrawArgs {
    const DevInfo *devs;
    const int32_t *rail_dev;             // global rail -> device
    int64_t rails_total;
    int32_t n_devices;
    const uint32_t *thr;                 // [steps + 1][D] stage-0 threshold of a device's words
    const double *volt;                  // [steps + 1][D] bias
    double beta, c0, alpha, ea_scalar;
    const void *ea;
    uint32_t key0, key1;
    int32_t cutoff, rail_range;
    const int8_t *plane;                 // state before the previous half-step's hops
    int8_t *other;                       // the other plane: receives the hops of the last two half-steps
    // lists, by the half-step's index since the call began (launch); entries
    // of draws (row, site, device, rail), of hops (row, site << 1 | dir, device,
    // rail), dir 0 moving the ion at the site up
    int64_t launch;
    uint4 *draws;                        // [2][kDrawMaxGrid][kDrawSlots]
    uint4 *hops;                         // [4][hop_cap]
    int64_t hop_cap;
    uint32_t *n_hops;                    // [4]
    int32_t n_bins, per_bin;             // resolving workgroups: per_bin for each column block
    int32_t *status;                     // raised when a list is too short
    int32_t resolve, generate;           // what this launch does
    int32_t k;                           // threshold-table row of the resolved half-step's step
    int64_t n;                           // its step; the generated half-step is the one after it
    int64_t tally_row;
    int32_t *tally_net, *tally_dec;
    HopArgs::LogBuf log;
    // dense: the kernel's MFMA fragments for the parity's column blocks
    const void *ktiles;
    int32_t nb, rows;                    // 32-site blocks per rail; survivors per product (32 or 16)
    int32_t pitch;
    float k10;
    // fixed: the potential, in two planes like the state
    const int64_t *phi;
    int64_t *phi_other;
    const int64_t *kfix;
    int64_t k10fix;
    int32_t frac_bits;
};

hipError_t launch_draws(const DrawArgs &a, bool dense, int h, int grid, size_t lds, hipStream_t st);
hipError_t launch_draw_table(uint32_t *thr, double *volt, const DevInfo *devs, int n_devices, const double *knot_t,
                             const double *knot_v, int64_t n_base, int rows, double dt, double beta, double c0,
                             double alpha, uint32_t *clear, hipStream_t st);
// The hops of the last two half-steps into the planes that miss them.
hipError_t launch_draw_settle(const DrawArgs &a, bool dense, hipStream_t st);
size_t draws_lds_bytes(bool dense, int rail_range, int nb, int rows, int cutoff);
hipError_t set_draws_lds_limit(bool dense, size_t lds);

}  // namespace kmc
