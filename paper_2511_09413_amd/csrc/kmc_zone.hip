// The paper's own zone model (SI S2.1, "Step-by-Step Explanation of the
// Markov Chain Monte Carlo Framework"), declared in include/kmc.h as the
// kmc_zone_* calls.
//
// State: the ion-position matrix X [rails][ions] (1-based columns, uint16,
// strictly increasing along a rail).  Up to 4096 steps per launch with every
// ion in registers (zone_run) for up to 131072 rails; beyond, one launch per
// step (zone_step).  A step:
//   * the step's table comes from the zone populations before the step: the
//     bias V(t_n), the net drop with the implicit space charge
//     dV_net(z) = V - f (sum_{z'<z} rho_z' - sum_{z'>z} rho_z'),
//     rho_z = N_z - N/Z, the energy gap of Eq. S1, the Boltzmann factor of
//     Eq. S2 and the directional probabilities of Eqs. S3-S4, in binary64
//     (computed by the previous step's last workgroup, or after a state or
//     protocol change by a one-workgroup kernel);
//   * a wavefront takes two rails, a lane two neighbouring ions of a rail:
//     one Philox4x32-10 block gives the lane's four uniforms (right and left
//     trial of each ion), the neighbours' columns come from the adjacent
//     lanes, a move is M_right - M_left with the gap tests of SI S2.1, and two
//     ions aiming at one column both stay;
//   * the new zone populations (added at zone boundaries only: the columns of
//     a rail stay increasing) and the net hops are summed per workgroup in
//     LDS, then into 64 bucket rows by device atomics; the last workgroup to
//     finish (counted per bucket, then over the buckets) sums the buckets
//     into the populations, writes the step's output row, clears the buckets
//     and evaluates the next step's table.
#include "../../include/kmc.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "kmc_device.h"
#include "kmc_internal.h"
#include "kmc_philox.h"
#include "kmc_queue.h"

namespace kmc {
kmc_status record_error(kmc_status s, const std::string &msg);
}

namespace {

using kmc::record_error;
using kmc::kMaxKnots;
using kmc::philox4x32_10;
using kmc::philox_lane;
using kmc::philox_step;
using kmc::philox_words;
using kmc::PhiloxLane;
using kmc::PhiloxStep;
using kmc::protocol_voltage;

constexpr int kZoneMaxZones = 64;
constexpr int kZoneMaxIons = 64;      // two per lane of a 32-lane half-wavefront
constexpr int kZoneBuckets = 64;
constexpr int kZoneBucketStride = 128;  // int64 per bucket row (zones, then net)
constexpr int kZoneBlock = 256;
constexpr int kZoneMaxGrid = 2048;

constexpr int32_t kZoneNoTally = -2147483647 - 1;  // tally rows of launches after a timed-out wait
constexpr int kZonePairsPerIter = 4;  // rail pairs a wavefront loads before computing them

struct ZoneArgs {
    uint16_t *X;                // [rails][ions]
    int32_t rails, ions, sites, zones;
    double p0, kT, hot, v_factor, dt;
    uint32_t key0, key1;
    const double *knot_t, *knot_v;
    int32_t n_knots;
    int64_t n_set;
    int64_t n;                  // absolute step of the launch
    int64_t row;                // output row of the step (n - first step of the call)
    const double *table;        // [2][Z] P_left, P_right of this step
    double *table_next;         // [2][Z] of the next step (written by the last workgroup)
    int64_t *pop_next;          // [Z] zone populations after the step (written by the last workgroup)
    int64_t *bucket;            // [kZoneBuckets][kZoneBucketStride], zero on entry
    uint32_t *ticket;           // [kZoneBuckets + 1] counters, 32 uint32 apart
    int32_t *net_out;           // caller [n_steps] or null
    int32_t *zone_out;          // caller [n_steps][Z] or null
    int64_t *net_total;         // running total of the net hops
    const int32_t *bad;         // raised by a timed-out wait of an earlier launch: nothing is run
};

__device__ __forceinline__ int zone_of(int x, int sites, int zones) {
    return (int)(((int64_t)x * zones + sites - 1) / sites);  // 1-based
}

// The same zone without an integer division: q = (x zones + sites - 1) /
// sites with n = x zones + sites - 1 < 2^23, from a binary32 reciprocal (n is
// exact in binary32 and the product is within one unit of the quotient),
// corrected by one integer test each way.
__device__ __forceinline__ int zone_fast(uint32_t x, uint32_t sites, uint32_t zones, float inv_sites) {
    const uint32_t n = x * zones + sites - 1u;
    uint32_t q = (uint32_t)((float)n * inv_sites);
    q -= q * sites > n ? 1u : 0u;
    q += (q + 1u) * sites <= n ? 1u : 0u;
    return (int)q;
}

// The accept test u <= p of a uniform u = w 2^-32 is w <= floor(p 2^32) for
// the integer w (p 2^32 is exact in binary64): one threshold per zone and
// direction, 0xFFFFFFFF when p >= 1 (every word accepts).
__device__ __forceinline__ uint32_t word_threshold(double p) {
    const double t = floor(p * 4294967296.0);
    return t >= 4294967295.0 ? 0xFFFFFFFFu : (t <= 0.0 ? 0u : (uint32_t)t);
}

// Directional probabilities of a zone with the excess populations below and
// above it (Eqs. S1-S4), binary64, the operations in the order of the text.
__device__ __forceinline__ void zone_probabilities(double below, double above, double V, double p0, double kT, double hot,
                                                   double v_factor, double *pl_out, double *pr_out) {
    const double dv = V - v_factor * (below - above);
    const double dE = dv * hot;
    const double B = exp(-dE / kT);
    const double pl = p0 / (1.0 + B);
    *pl_out = pl;
    *pr_out = B * pl;
}

// Table entry of zone z for bias V and populations pop (Eqs. S1-S4 with the
// space-charge drop), binary64, the operations in the order of the text.
__device__ inline void zone_entry(int z, int Z, const int64_t *pop, double V, double p0, double kT, double hot,
                                  double v_factor, double *pl_out, double *pr_out) {
    double total = 0.0;
    for (int y = 0; y < Z; ++y) total += (double)pop[y];
    const double mean = total / (double)Z;
    double below = 0.0, above = 0.0;
    for (int y = 0; y < z; ++y) below += (double)pop[y] - mean;
    for (int y = z + 1; y < Z; ++y) above += (double)pop[y] - mean;
    zone_probabilities(below, above, V, p0, kT, hot, v_factor, pl_out, pr_out);
}

__global__ __launch_bounds__(kZoneBlock) void zone_step(ZoneArgs a) {
    __shared__ uint32_t s_tl[kZoneMaxZones], s_tr[kZoneMaxZones];
    __shared__ int32_t s_pop[kZoneMaxZones];
    __shared__ int64_t s_fin[kZoneMaxZones + 1];
    __shared__ int32_t s_net;
    __shared__ double s_v;
    __shared__ uint32_t s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int Z = a.zones;
    if (*a.bad != 0) {
        if (blockIdx.x == 0 && tid == 0 && a.net_out) a.net_out[a.row] = kZoneNoTally;
        if (blockIdx.x == 0 && tid < Z && a.zone_out) a.zone_out[a.row * Z + tid] = kZoneNoTally;
        return;
    }
    if (tid < Z) {
        s_tl[tid] = word_threshold(a.table[tid]);
        s_tr[tid] = word_threshold(a.table[Z + tid]);
        s_pop[tid] = 0;
    }
    if (tid == 0) s_net = 0;
    __syncthreads();
    const uint32_t sites = (uint32_t)a.sites, zones = (uint32_t)Z;
    const float inv_sites = 1.0f / (float)a.sites;

    // ions: a half-wavefront per rail, a lane per two neighbouring ions; a
    // wavefront loads kZonePairsPerIter rail pairs before computing them
    const int half = lane >> 5, l = lane & 31;
    const int j0 = 2 * l, j1 = 2 * l + 1;
    const int64_t pairs = ((int64_t)a.rails + 1) / 2;
    const int64_t tw = (int64_t)gridDim.x * (kZoneBlock / 64), gw = (int64_t)blockIdx.x * (kZoneBlock / 64) + wave;
    int net = 0;
    for (int64_t it = 0; it * kZonePairsPerIter * tw < pairs; ++it) {
        int x0[kZonePairsPerIter], x1[kZonePairsPerIter];
        int64_t rail[kZonePairsPerIter];
#pragma unroll
        for (int k = 0; k < kZonePairsPerIter; ++k) {
            const int64_t pr = (it * kZonePairsPerIter + k) * tw + gw;
            rail[k] = 2 * pr + half;
            const bool ok = pr < pairs && rail[k] < a.rails;
            const uint16_t *row = a.X + rail[k] * a.ions;
            x0[k] = ok && j0 < a.ions ? (int)row[j0] : 0;
            x1[k] = ok && j1 < a.ions ? (int)row[j1] : 0;
        }
#pragma unroll
        for (int k = 0; k < kZonePairsPerIter; ++k) {
            const int64_t pr = (it * kZonePairsPerIter + k) * tw + gw;
            const bool rail_ok = pr < pairs && rail[k] < a.rails;
            const bool h0 = rail_ok && j0 < a.ions, h1 = rail_ok && j1 < a.ions;
            // neighbours: the previous lane's second ion, the next lane's first
            // ion (a virtual ion at column 0 before the first ion and at
            // sites + 1 after the last)
            const int prev_x1 = __shfl_up(x1[k], 1, 32);
            const int next_x0 = __shfl_down(x0[k], 1, 32);
            const bool has_next = j1 + 1 < a.ions && l < 31;
            const int left0 = l == 0 ? 0 : prev_x1;
            const int right0 = h1 ? x1[k] : a.sites + 1;
            const int right1 = has_next ? next_x0 : a.sites + 1;
            // the lane's four uniforms: right and left trial of ions j0 and j1
            const uint4 w = philox4x32_10((uint32_t)l, (uint32_t)rail[k], (uint32_t)a.n, 2u << 1, a.key0, a.key1);
            int m0 = 0, m1 = 0;
            if (h0) {
                const int z = zone_fast((uint32_t)x0[k], sites, zones, inv_sites) - 1;
                const int mr = (w.x <= s_tr[z]) && (right0 - x0[k] > 1);
                const int ml = (w.y <= s_tl[z]) && (x0[k] - left0 > 1);
                m0 = mr - ml;
            }
            if (h1) {
                const int z = zone_fast((uint32_t)x1[k], sites, zones, inv_sites) - 1;
                const int mr = (w.z <= s_tr[z]) && (right1 - x1[k] > 1);
                const int ml = (w.w <= s_tl[z]) && (x1[k] - x0[k] > 1);
                m1 = mr - ml;
            }
            // two ions aiming at one column both stay (such pairs are disjoint)
            const int prev_m1 = __shfl_up(m1, 1, 32);
            const int next_m0 = __shfl_down(m0, 1, 32);
            const bool in_pair = h0 && h1 && m0 == 1 && m1 == -1 && x1[k] - x0[k] == 2;
            const bool with_prev = h0 && l > 0 && prev_m1 == 1 && m0 == -1 && x0[k] - prev_x1 == 2;
            const bool with_next = h1 && has_next && m1 == 1 && next_m0 == -1 && next_x0 - x1[k] == 2;
            if (in_pair || with_prev) m0 = 0;
            if (in_pair || with_next) m1 = 0;
            const int y0 = x0[k] + m0, y1 = x1[k] + m1;
            uint16_t *row = a.X + rail[k] * a.ions;
            if (h0) row[j0] = (uint16_t)y0;
            if (h1) row[j1] = (uint16_t)y1;
            net -= m0 + m1;
            // zone populations after the move: the columns stay increasing, so
            // the ions of a zone are consecutive; zone z holds (index after its
            // last ion) - (index of its first ion), added at the boundaries only
            const int zz0 = h0 ? zone_fast((uint32_t)y0, sites, zones, inv_sites) : 0;
            const int zz1 = h1 ? zone_fast((uint32_t)y1, sites, zones, inv_sites) : 0;
            const int prev_zz1 = __shfl_up(zz1, 1, 32);
            const int next_zz0 = __shfl_down(zz0, 1, 32);
            if (h0) {
                if (j0 > 0 && prev_zz1 != zz0) atomicAdd(&s_pop[zz0 - 1], -j0);
                if (!h1 || zz1 != zz0) atomicAdd(&s_pop[zz0 - 1], j0 + 1);
            }
            if (h1) {
                if (zz0 != zz1) atomicAdd(&s_pop[zz1 - 1], -j1);
                if (!has_next || next_zz0 != zz1) atomicAdd(&s_pop[zz1 - 1], j1 + 1);
            }
        }
    }
    // the workgroup's net hops
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) net += __shfl_xor(net, off, 64);
    if (lane == 0 && net != 0) atomicAdd(&s_net, net);
    __syncthreads();

    // workgroup sums into its bucket row; the last workgroup ends the step
    const int b = blockIdx.x % kZoneBuckets;
    int64_t *brow = a.bucket + (int64_t)b * kZoneBucketStride;
    if (tid < Z && s_pop[tid] != 0) atomicAdd((unsigned long long *)&brow[tid], (unsigned long long)(int64_t)s_pop[tid]);
    if (tid == Z && s_net != 0) atomicAdd((unsigned long long *)&brow[Z], (unsigned long long)(int64_t)s_net);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
        const uint32_t nb = (uint32_t)min((int)gridDim.x, kZoneBuckets);
        const uint32_t members = gridDim.x / kZoneBuckets + ((uint32_t)b < gridDim.x % kZoneBuckets ? 1u : 0u);
        uint32_t last = 0;
        uint32_t *cb = a.ticket + b * 32;
        uint32_t *ct = a.ticket + kZoneBuckets * 32;
        if (__hip_atomic_fetch_add(cb, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1u) {
            __hip_atomic_store(cb, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (__hip_atomic_fetch_add(ct, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1u) {
                __hip_atomic_store(ct, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = 1;
            }
        }
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    // the last workgroup: populations after the step, the output row, and the
    // next step's table
    if (tid == 0) s_v = protocol_voltage(a.knot_t, a.knot_v, a.n_knots, (double)(a.n + 1 - a.n_set) * a.dt);
    if (tid <= Z) s_fin[tid] = 0;
    __syncthreads();
    // every thread takes some of the kZoneBuckets x (Z + 1) bucket entries
    for (int e = tid; e < kZoneBuckets * (Z + 1); e += kZoneBlock) {
        const int bb = e / (Z + 1), q = e - bb * (Z + 1);
        int64_t *p = a.bucket + (int64_t)bb * kZoneBucketStride + q;
        const int64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v != 0) {
            __hip_atomic_store(p, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            atomicAdd((unsigned long long *)&s_fin[q], (unsigned long long)v);
        }
    }
    __syncthreads();
    if (tid <= Z) {
        const int64_t sum = s_fin[tid];
        if (tid < Z) {
            a.pop_next[tid] = sum;
            if (a.zone_out) a.zone_out[a.row * Z + tid] = (int32_t)sum;
        } else {
            if (a.net_out) a.net_out[a.row] = (int32_t)sum;
            *a.net_total += sum;
        }
    }
    __syncthreads();
    if (tid < Z) {
        double pl, pr;
        zone_entry(tid, Z, s_fin, s_v, a.p0, a.kT, a.hot, a.v_factor, &pl, &pr);
        a.table_next[tid] = pl;
        a.table_next[Z + tid] = pr;
    }
}

// ---------------------------------------------------------------------------
// zone_run: up to kZoneRunSteps steps in one launch, every ion in registers.
//
// One launch per step left the step's time to everything but its work: at
// 128,000 x 60 ions 33 us (15 MB read and written again, the division-free zone
// index four times per lane, 250 VALU per rail pair) and at 500 rails 12 us, all
// of it launch, ticket chain and table latency.  Here a wavefront owns P rail
// pairs for the launch and keeps each ion's column and zone in registers, so a
// step touches no memory but the zone sums, and its VALU work is mostly the
// Philox block (34 instructions: what depends on the lane or on the step alone
// is computed once) and the compares; trials, gap tests and conflicts are
// wavefront masks combined by the scalar unit.  Thresholds are looked up by the
// ion's zone (LDS), the zone by its column (a byte table in LDS), and only ions
// that change zone touch the populations.
//
// Between two steps the workgroups add their population changes and net hops
// to kZoneAcc accumulator rows (64-bit words: arrivals in the upper 24 bits, the
// biased sum below) and every workgroup polls those rows until all members of
// a row have arrived.  Rows alternate by the step's parity: a workgroup adds to
// a row again only after every workgroup has added the step in between, hence
// after all have read it.  Every workgroup then evaluates the table itself.
// Measured, us per step: 500 rails x 200 12.2 -> 2.7 (two round trips between
// workgroups and the table's serial binary64), 128,000 rails 32.7 -> 13.7 (VALU,
// about 120 instructions per rail pair).
//
// The launch needs all its workgroups resident at once.  It is sized for an
// idle GPU; where other work holds CUs its workgroups leave at the gate
// (kmc_queue.h) and zone_queue, launched behind it, takes the same steps tile by
// tile with the ions in memory, on whatever part of the GPU is free.
constexpr int kZoneAcc = 8;               // accumulator rows (workgroup index modulo 8: one XCD each)
constexpr int kZoneAccStride = 72;        // 64-bit words per row (zones, then net)
constexpr int kZoneRunSteps = 4096;       // steps per launch (the biased sums stay below 2^40)
constexpr int kZoneRunMaxPairs = 16;      // rail pairs per wavefront
constexpr int64_t kZoneBias = 1 << 20;    // above any workgroup's change in one step

struct ZoneRunArgs {
    uint16_t *X;                // [rails][ions]
    int32_t rails, ions, sites, zones;
    double p0, kT, hot, v_factor, dt;
    uint32_t key0, key1;
    const double *knot_t, *knot_v;
    int32_t n_knots, n_steps;
    int64_t n_set;
    int64_t n0;                 // absolute step of the launch's first step
    int64_t row0;               // its output row
    double *table;              // [2][Z] of the first step; replaced by the one after the last step
    int64_t *pop;               // [Z] zone populations, replaced likewise
    unsigned long long *acc;    // [2][kZoneAcc][kZoneAccStride], zero on entry
    kmc::QueueWords *queue;     // zero on entry
    unsigned long long *acc_next;   // the following launch's, cleared by this one
    kmc::QueueWords *queue_next;
    int32_t tile_pairs, n_tiles;    // zone_queue: rail pairs per tile, tiles
    int32_t *bad;               // raised when a wait of the loop timed out; while it is, launches leave at once
    int32_t *net_out, *zone_out;
    int64_t *net_total;
    int32_t gate_ticks;         // 10 ns ticks a workgroup waits at the gate
    int32_t wait_limit;         // polls of a step's sums before the wait counts as hung
};

// The kernel arguments, read again from the argument segment where a step's
// end needs them (scalar loads): held across the pairs' work they would fill
// the scalar registers.
typedef const __attribute__((address_space(4))) ZoneRunArgs *ZoneKArgs;
__device__ __forceinline__ ZoneKArgs zone_kargs() {
    ZoneKArgs p = (ZoneKArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// LDS of one workgroup; the zone byte of every column follows it.
struct ZoneLds {
    uint32_t thr[2][kZoneMaxZones];    // right, left thresholds of the zones
    int32_t dpop[2][kZoneMaxZones];    // the workgroup's population changes, by the step's parity
    int32_t dnet[2];
    int32_t sum[2][kZoneMaxZones + 1]; // the lattice's changes, by the step's parity
    int32_t pop[kZoneMaxZones];
    int64_t before[2][kZoneAcc * (kZoneMaxZones + 1)];  // the accumulators' sums when last read
    double kt[kMaxKnots], kv[kMaxKnots];
    int64_t net;
    int32_t go;
    uint32_t ticket, last;             // zone_queue
};

constexpr uint64_t kFirstLanes = 0x0000000100000001ull, kLastLanes = 0x8000000080000000ull;

// One step of a rail pair: lane l of each half holds ions 2l and 2l + 1 of its
// rail (columns x0, x1; absent ions at sites + 1; z0, z1: four times the
// zero-based zone).  v0, v1: the lanes whose ions exist.  Returns the pair's net
// hops (left moves minus right moves).
__device__ __forceinline__ int zone_pair(uint32_t &x0, uint32_t &x1, uint32_t &z0, uint32_t &z1, const uint4 &w,
                                         uint64_t v0, uint64_t v1, uint32_t wall, bool last_lane, const uint32_t *thr,
                                         int32_t *dpop, const uint8_t *zone_at) {
    auto at = [](const uint32_t *p, uint32_t z) { return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(p) + z); };
    // gaps to the right neighbours; the left gap of a lane's first ion is the
    // previous lane's right gap (or the wall)
    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)wall, (int)x0, 0x130, 0xf, 0xf, false);  // lane + 1
    const uint32_t gn = (last_lane ? wall : next) - x1;
    const uint32_t gi = x1 - x0;
    const uint64_t gn_free = __ballot(gn > 1u), gi_free = __ballot(gi > 1u);
    const uint64_t gn_two = __ballot(gn == 2u) & ~kLastLanes, gi_two = __ballot(gi == 2u);
    const uint64_t gp_free = ((gn_free << 1) & ~kFirstLanes) | (__ballot(x0 > 1u) & kFirstLanes);
    const uint64_t right0 = __ballot(w.x <= at(thr, z0)) & gi_free & v0;
    const uint64_t left0 = __ballot(w.y <= at(thr + kZoneMaxZones, z0)) & gp_free & v0;
    const uint64_t right1 = __ballot(w.z <= at(thr, z1)) & gn_free & v1;
    const uint64_t left1 = __ballot(w.w <= at(thr + kZoneMaxZones, z1)) & gi_free & v1;
    // a move is M_right - M_left; two ions aiming at one column both stay
    uint64_t r0 = right0 & ~left0, l0 = left0 & ~right0, r1 = right1 & ~left1, l1 = left1 & ~right1;
    const uint64_t in = r0 & l1 & gi_two, out = r1 & (l0 >> 1) & gn_two;
    r0 &= ~in;
    l1 &= ~in;
    r1 &= ~out;
    l0 &= ~(out << 1);
    x0 += __builtin_amdgcn_inverse_ballot_w64(r0) ? 1u : 0u;
    x0 -= __builtin_amdgcn_inverse_ballot_w64(l0) ? 1u : 0u;
    x1 += __builtin_amdgcn_inverse_ballot_w64(r1) ? 1u : 0u;
    x1 -= __builtin_amdgcn_inverse_ballot_w64(l1) ? 1u : 0u;
    const uint32_t y0 = zone_at[x0], y1 = zone_at[x1];
    auto cross = [&](uint32_t &z, uint32_t y) {
        if (z != y) {
            atomicAdd(reinterpret_cast<int32_t *>(reinterpret_cast<char *>(dpop) + y), 1);
            atomicAdd(reinterpret_cast<int32_t *>(reinterpret_cast<char *>(dpop) + z), -1);
            z = y;
        }
    };
    cross(z0, y0);
    cross(z1, y1);
    return (__popcll(l0) + __popcll(l1)) - (__popcll(r0) + __popcll(r1));
}

// The workgroup's tables, before the first step (ends with a barrier).
__device__ inline void zone_setup(const ZoneRunArgs &a, ZoneLds &s, uint8_t *zone_at) {
    const int tid = threadIdx.x, Z = a.zones;
    for (int i = tid; i < kZoneMaxZones; i += blockDim.x) {
        s.thr[0][i] = i < Z ? word_threshold(a.table[Z + i]) : 0u;
        s.thr[1][i] = i < Z ? word_threshold(a.table[i]) : 0u;
        s.dpop[0][i] = s.dpop[1][i] = 0;
        s.pop[i] = i < Z ? (int32_t)a.pop[i] : 0;
    }
    for (int i = tid; i < kMaxKnots; i += blockDim.x) {
        s.kt[i] = a.knot_t[i];
        s.kv[i] = a.knot_v[i];
    }
    for (int i = tid; i <= kZoneMaxZones; i += blockDim.x) s.sum[0][i] = s.sum[1][i] = 0;
    if (tid < 2) s.dnet[tid] = 0;
    if (tid == 0) s.net = 0;
    const float inv_sites = 1.0f / (float)a.sites;
    for (int x = tid; x < a.sites + 2; x += blockDim.x)
        zone_at[x] = x >= 1 && x <= a.sites ? (uint8_t)(4 * (zone_fast((uint32_t)x, (uint32_t)a.sites, (uint32_t)Z, inv_sites) - 1)) : 0;
    __syncthreads();
}

// The end of step k in the first wavefront: populations, the output row (one
// workgroup), the thresholds of step k + 1; V is the bias at that step.  kEach:
// the workgroup ends this step alone, so its populations, table and net hops go
// to memory now, else after the launch's last step.
template <bool kEach>
__device__ inline void zone_end_step(ZoneLds &s, int k, double V, bool writer) {
    const ZoneKArgs ap = zone_kargs();
    const auto &a = *ap;
    const int tid = threadIdx.x, Z = a.zones, par = k & 1;
    if (tid >= 64) return;
    int64_t pop = 0;
    if (tid < Z) {
        pop = s.pop[tid] + s.sum[par][tid];
        s.pop[tid] = (int32_t)pop;
    }
    const int32_t net = s.sum[par][Z];
    s.sum[par ^ 1][tid] = 0;
    if (tid == 0) s.sum[par ^ 1][kZoneMaxZones] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (tid < Z) {
        // the table's space-charge sums in the order of zone_entry (the total
        // is the ion count, exact in binary64)
        const double mean = (double)((int64_t)a.rails * a.ions) / (double)Z;
        double below = 0.0, above = 0.0;
#pragma unroll 4
        for (int y = 0; y < Z; ++y) {
            const double rho = (double)s.pop[y] - mean;
            if (y < tid) below += rho;
            if (y > tid) above += rho;
        }
        double pl, pr;
        zone_probabilities(below, above, V, a.p0, a.kT, a.hot, a.v_factor, &pl, &pr);
        s.thr[0][tid] = word_threshold(pr);
        s.thr[1][tid] = word_threshold(pl);
        if (writer) {
            if (a.zone_out) a.zone_out[(a.row0 + k) * Z + tid] = (int32_t)pop;
            if (kEach) {
                kmc::queue_store(a.pop + tid, pop);
                kmc::queue_store(a.table + tid, pl);
                kmc::queue_store(a.table + Z + tid, pr);
            } else if (k == a.n_steps - 1) {
                a.pop[tid] = pop;
                a.table[tid] = pl;
                a.table[Z + tid] = pr;
            }
        }
    }
    if (writer && tid == 0) {
        s.net += net;
        if (a.net_out) a.net_out[a.row0 + k] = net;
        if (kEach) atomicAdd(reinterpret_cast<unsigned long long *>(a.net_total), (unsigned long long)(int64_t)net);
        else if (k == a.n_steps - 1) *a.net_total += s.net;
    }
}

// The accumulators and queue words of one launch, by one workgroup.
__device__ inline void zone_clear(unsigned long long *acc, kmc::QueueWords *queue) {
    for (int i = threadIdx.x; i < 2 * kZoneAcc * kZoneAccStride; i += blockDim.x) acc[i] = 0;
    for (int i = threadIdx.x; i < kmc::kQueueWords; i += blockDim.x) reinterpret_cast<uint32_t *>(queue)[i] = 0u;
}

template <int P>
__global__ __launch_bounds__(1024) void zone_run(ZoneRunArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    ZoneLds &s = *reinterpret_cast<ZoneLds *>(smem);
    uint8_t *zone_at = smem + sizeof(ZoneLds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6;
    // all workgroups are resident, or none runs
    if (tid == 0)
        s.go = kmc::queue_gate(a.queue->gate, gridDim.x, a.gate_ticks) &&
               !__hip_atomic_load(a.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (blockIdx.x == 0) zone_clear(a.acc_next, a.queue_next);
    zone_setup(a, s, zone_at);
    if (!s.go) return;

    // the wavefront's ions
    const int half = lane >> 5, l = lane & 31, j0 = 2 * l, j1 = 2 * l + 1;
    const int64_t pairs = ((int64_t)a.rails + 1) / 2;
    const int64_t pair0 = ((int64_t)blockIdx.x * waves + wave) * P;
    const uint32_t wall = (uint32_t)a.sites + 1u;
    const bool last_lane = l == 31;
    const uint64_t has0 = __ballot(j0 < a.ions), has1 = __ballot(j1 < a.ions);
    uint32_t x0[P], x1[P], z0[P], z1[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int64_t rail = 2 * (pair0 + k) + half;
        const bool ok = rail < a.rails;
        const uint16_t *row = a.X + rail * a.ions;
        x0[k] = ok && j0 < a.ions ? row[j0] : wall;
        x1[k] = ok && j1 < a.ions ? row[j1] : wall;
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        z0[k] = zone_at[x0[k]];
        z1[k] = zone_at[x1[k]];
    }
    const uint32_t rail0 = (uint32_t)(2 * pair0 + half);
    const int mine = (int)(pairs - pair0 < P ? (pairs - pair0 > 0 ? pairs - pair0 : 0) : P);  // pairs of this wavefront
    const int odd_at = (a.rails & 1) ? (int)(pairs - 1 - pair0 < P ? pairs - 1 - pair0 : P) : P;  // the pair without a second rail
    const PhiloxLane lc = philox_lane((uint32_t)l, 2u << 1, a.key0, a.key1);
    for (int i = tid; i < 2 * kZoneAcc * (kZoneMaxZones + 1); i += blockDim.x) (&s.before[0][0])[i] = 0;  // (the first step's barrier precedes their use)
    for (int k = 0; k < a.n_steps; ++k) {
        const int par = k & 1;
        // opaque: what is derived from these for every pair is not held over the steps
        uint32_t rail_k = rail0;
        int mine_k = __builtin_amdgcn_readfirstlane(mine), odd_k = __builtin_amdgcn_readfirstlane(odd_at);
        asm volatile("" : "+v"(rail_k), "+s"(mine_k), "+s"(odd_k));
        const uint32_t key0 = zone_kargs()->key0, key1 = zone_kargs()->key1;
        const PhiloxStep sc = philox_step(lc, (uint32_t)zone_kargs()->n0 + (uint32_t)k, key0, key1);
        int net = 0;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            if (q < mine_k) {
                const uint4 w = philox_words(lc, sc, rail_k + 2u * (uint32_t)q, key0, key1);
                const uint64_t v = q == odd_k ? 0xFFFFFFFFull : ~0ull;
                net += zone_pair(x0[q], x1[q], z0[q], z1[q], w, has0 & v, has1 & v, wall, last_lane, &s.thr[0][0],
                                 s.dpop[par], zone_at);
            }
            // no mixing of pairs: their words would spill
            __builtin_amdgcn_sched_barrier(0);
        }
        if (lane == 0 && net != 0) atomicAdd(&s.dnet[par], net);
        kmc::lds_barrier();
        const ZoneKArgs ka = zone_kargs();
        const int Z = ka->zones;
        unsigned long long *rows_at = ka->acc + par * kZoneAcc * kZoneAccStride;
        if (tid <= Z) {
            int32_t *at = tid < Z ? &s.dpop[par][tid] : &s.dnet[par];
            const int64_t v = *at;
            *at = 0;
            __hip_atomic_fetch_add(rows_at + (blockIdx.x % kZoneAcc) * kZoneAccStride + tid,
                                   (1ull << 40) + (unsigned long long)(v + kZoneBias), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        // the bias of the next step, while the sums travel
        double V = 0.0;
        if (tid < 64) V = protocol_voltage(s.kt, s.kv, ka->n_knots, (double)(ka->n0 + k + 1 - ka->n_set) * ka->dt);
        const int words = min((int)gridDim.x, kZoneAcc) * (Z + 1);
        // (after a hung wait the remaining steps run through without waiting,
        // and nothing of them is used)
        const int limit = s.go ? ka->wait_limit : 0;
        for (int e = tid; e < words; e += blockDim.x) {
            const int row = e / (Z + 1), q = e - row * (Z + 1);
            const int64_t members = ((int)gridDim.x - row + kZoneAcc - 1) / kZoneAcc;
            const uint64_t want = (uint64_t)(members * (k / 2 + 1));
            uint64_t v = 0;
            int spins = 0;
            while (((v = __hip_atomic_load(rows_at + row * kZoneAccStride + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >>
                    40) != want) {
                if (++spins > limit) {
                    s.go = 0;
                    __hip_atomic_store(zone_kargs()->bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            const int64_t low = (int64_t)(v & ((1ull << 40) - 1ull));
            atomicAdd(&s.sum[par][q], (int32_t)(low - s.before[par][e] - members * kZoneBias));
            s.before[par][e] = low;
        }
        kmc::lds_barrier();
        // (16 pairs: leaving here costs nothing and takes 3 % off the loop, whose
        // registers it changes, 13.47 -> 13.12 us per step; with fewer pairs the
        // test would be 0.1 us of the first wavefront's chain)
        if (P == 16 && !s.go) return;
        zone_end_step<false>(s, k, V, blockIdx.x == 0);
        kmc::lds_barrier();
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int64_t rail = 2 * (pair0 + k) + half;
        uint16_t *row = a.X + rail * a.ions;
        if (rail < a.rails) {
            if (j0 < a.ions) row[j0] = (uint16_t)x0[k];
            if (j1 < a.ions) row[j1] = (uint16_t)x1[k];
        }
    }
}

// Behind every zone_run: the same steps when the launch left them undone, from
// a queue of tiles (kmc_queue.h) with the ions in memory.  The workgroup that
// completes a step's last tile sums the step's changes, writes its output row
// and the next step's table, and publishes the step.  After a timed-out wait
// nothing is run, and the tally rows of the launch read kZoneNoTally.
__global__ __launch_bounds__(1024) void zone_queue(ZoneRunArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    if (*a.bad != 0) {
        if (blockIdx.x != 0) return;
        for (int i = tid; a.net_out && i < a.n_steps; i += blockDim.x) a.net_out[a.row0 + i] = kZoneNoTally;
        for (int i = tid; a.zone_out && i < a.n_steps * a.zones; i += blockDim.x)
            a.zone_out[a.row0 * a.zones + i] = kZoneNoTally;
        return;
    }
    if ((a.queue->gate[0] & kmc::kQueueAbort) == 0) return;
    ZoneLds &s = *reinterpret_cast<ZoneLds *>(smem);
    uint8_t *zone_at = smem + sizeof(ZoneLds);
    const int lane = tid & 63, half = lane >> 5, l = lane & 31, j0 = 2 * l, j1 = 2 * l + 1, Z = a.zones;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    zone_setup(a, s, zone_at);
    const int pairs = (a.rails + 1) / 2;
    const uint32_t wall = (uint32_t)a.sites + 1u;
    const PhiloxLane lc = philox_lane((uint32_t)l, 2u << 1, a.key0, a.key1);
    unsigned long long *row_of_wg = a.acc + (blockIdx.x % kZoneAcc) * kZoneAccStride;
    int at_step = -1;  // whose thresholds the LDS holds
    bool ended = false;  // the workgroup has ended the step before at_step
    for (;;) {
        // (one block of thread 0 between two barriers: with two of them and only
        // the back edge between, the compiler may send the other lanes on alone)
        if (tid == 0) {
            if (ended) __hip_atomic_store(a.queue->ready, (uint32_t)at_step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t v = __hip_atomic_fetch_add(a.queue->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s.ticket = v;
            s.go = v < (uint32_t)a.n_steps * (uint32_t)a.n_tiles &&
                   kmc::queue_wait(a.queue->ready, v / (uint32_t)a.n_tiles, a.bad, a.wait_limit);
        }
        __syncthreads();
        const uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.ticket);
        if (!__builtin_amdgcn_readfirstlane(s.go)) return;
        ended = false;
        const int k = (int)(ticket / (uint32_t)a.n_tiles), tile = (int)(ticket - (uint32_t)k * (uint32_t)a.n_tiles);
        if (k != at_step && tid < Z) {
            s.thr[0][tid] = word_threshold(kmc::queue_load(a.table + Z + tid));
            s.thr[1][tid] = word_threshold(kmc::queue_load(a.table + tid));
        }
        at_step = k;
        __syncthreads();
        const PhiloxStep sc = philox_step(lc, (uint32_t)(a.n0 + k), a.key0, a.key1);
        int net = 0;
        const int end = min(pairs, (tile + 1) * a.tile_pairs);
        for (int pr = tile * a.tile_pairs + wave; pr < end; pr += blockDim.x >> 6) {
            const int rail = 2 * pr + half;
            const bool h0 = rail < a.rails && j0 < a.ions, h1 = rail < a.rails && j1 < a.ions;
            uint16_t *row = a.X + (int64_t)rail * a.ions;
            uint32_t x0 = h0 ? kmc::queue_load(row + j0) : wall, x1 = h1 ? kmc::queue_load(row + j1) : wall;
            uint32_t z0 = zone_at[x0], z1 = zone_at[x1];
            const uint4 w = philox_words(lc, sc, (uint32_t)rail, a.key0, a.key1);
            net += zone_pair(x0, x1, z0, z1, w, __ballot(h0), __ballot(h1), wall, l == 31, &s.thr[0][0], s.dpop[0], zone_at);
            if (h0) kmc::queue_store(row + j0, (uint16_t)x0);
            if (h1) kmc::queue_store(row + j1, (uint16_t)x1);
        }
        if (lane == 0 && net != 0) atomicAdd(&s.dnet[0], net);
        __syncthreads();
        unsigned long long *sums = a.acc + (k & 1) * kZoneAcc * kZoneAccStride;
        if (tid <= Z) {
            int32_t *at = tid < Z ? &s.dpop[0][tid] : &s.dnet[0];
            const int64_t v = *at;
            *at = 0;
            if (v != 0) atomicAdd(row_of_wg + (k & 1) * kZoneAcc * kZoneAccStride + tid, (unsigned long long)v);
        }
        kmc::queue_stores_done();
        if (tid == 0)
            s.last = __hip_atomic_fetch_add(a.queue->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                     (uint32_t)(k + 1) * (uint32_t)a.n_tiles;
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane((int)s.last)) continue;
        // every tile of step k is done
        if (tid < Z) s.pop[tid] = (int32_t)kmc::queue_load(a.pop + tid);
        if (tid <= Z) {
            int64_t sum = 0;
            for (int r = 0; r < kZoneAcc; ++r) {
                unsigned long long *p = sums + r * kZoneAccStride + tid;
                sum += (int64_t)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(p, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s.sum[k & 1][tid] = (int32_t)sum;
        }
        __syncthreads();
        const double V = protocol_voltage(s.kt, s.kv, a.n_knots, (double)(a.n0 + k + 1 - a.n_set) * a.dt);
        zone_end_step<true>(s, k, V, true);
        kmc::queue_stores_done();
        at_step = k + 1;  // zone_end_step left its thresholds in the LDS
        ended = true;
    }
}

// The table of the step n from the populations pop (one workgroup).
__global__ void zone_make_table(const int64_t *pop, int Z, const double *knot_t, const double *knot_v, int n_knots,
                                int64_t n, int64_t n_set, double dt, double p0, double kT, double hot,
                                double v_factor, double *table) {
    __shared__ double s_v;
    __shared__ int64_t s_pop[kZoneMaxZones];
    const int tid = threadIdx.x;
    if (tid == 0) s_v = protocol_voltage(knot_t, knot_v, n_knots, (double)(n - n_set) * dt);
    if (tid < Z) s_pop[tid] = pop[tid];
    __syncthreads();
    if (tid < Z) {
        double pl, pr;
        zone_entry(tid, Z, s_pop, s_v, p0, kT, hot, v_factor, &pl, &pr);
        table[tid] = pl;
        table[Z + tid] = pr;
    }
}

// Ion-position matrix from the caller's occupancy (one wavefront per rail):
// the k-th occupied site of a rail becomes column X[k] (1-based).  Rails
// whose ion count differs from `ions` raise *bad.  The populations of the
// zones are added to pop.
__global__ __launch_bounds__(256) void zone_import(const int8_t *occ, uint16_t *X, int rails, int sites, int ions,
                                                  int zones, int64_t *pop, int32_t *bad, int write) {
    __shared__ int32_t s_pop[kZoneMaxZones];
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < kZoneMaxZones) s_pop[threadIdx.x] = 0;
    __syncthreads();
    const int64_t rail = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (rail < rails) {
        const int8_t *src = occ + rail * sites;
        int base = 0;
        for (int s0 = 0; s0 < sites; s0 += 64) {
            const int s = s0 + lane;
            const bool occd = s < sites && src[s] != 0;
            const uint64_t m = __ballot(occd);
            const int rank = base + __popcll(m & ((1ull << lane) - 1ull));
            if (write && occd && rank < ions) {
                X[rail * ions + rank] = (uint16_t)(s + 1);
                atomicAdd(&s_pop[zone_of(s + 1, sites, zones) - 1], 1);
            }
            base += __popcll(m);
        }
        if (lane == 0 && base != ions) atomicExch(bad, 1);
    }
    __syncthreads();
    if (write && threadIdx.x < zones && s_pop[threadIdx.x] != 0)
        atomicAdd((unsigned long long *)&pop[threadIdx.x], (unsigned long long)(int64_t)s_pop[threadIdx.x]);
}

// Caller occupancy from the ion-position matrix (one wavefront per rail).
// The first workgroup clears the words of the call's multi-step launches.
__global__ __launch_bounds__(256) void zone_export(const uint16_t *X, int8_t *occ, int rails, int sites, int ions,
                                                  unsigned long long *acc, kmc::QueueWords *queue) {
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0)
        for (int i = 0; i < 2; ++i) zone_clear(acc + i * 2 * kZoneAcc * kZoneAccStride, queue + i);
    const int64_t rail = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (rail >= rails) return;
    int8_t *dst = occ + rail * sites;
    for (int s = lane; s < sites; s += 64) dst[s] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int j = lane; j < ions; j += 64) dst[(int)X[rail * ions + j] - 1] = 1;
}

__global__ void zone_fill_i64(int64_t *p, int64_t n, int64_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

struct ZoneKnots {
    double t[kMaxKnots], v[kMaxKnots];
};
__global__ void zone_set_knots(double *kt, double *kv, ZoneKnots k) {
    const int i = threadIdx.x;
    if (i < kMaxKnots) {
        kt[i] = k.t[i];
        kv[i] = k.v[i];
    }
}

}  // namespace

struct kmc_zone_ctx {
    kmc_zone_params p{};
    int32_t ions = 0;
    unsigned char *ws = nullptr;
    int8_t *occ_user = nullptr;
    hipStream_t stream = nullptr;
    bool poisoned = false;
    int64_t n = 0;              // step counter
    int64_t n_set = 0;          // step of the protocol install
    int32_t n_knots = 1;
    int cur = 0;                // population buffer holding the current state
    // workspace layout
    int cus = 0;                // compute units of the GPU (0: the runs go step by step)
    int32_t gate_ticks = 10000000;  // 0.1 s
    int32_t wait_limit = 1 << 22;
    size_t off_X, off_pop, off_table, off_bucket, off_ticket, off_knots, off_total, off_bad, off_acc, off_queue, total;
    template <typename T>
    T *at(size_t off) { return reinterpret_cast<T *>(ws + off); }
};

namespace {

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

kmc_status zone_validate(const kmc_zone_params *p) {
    if (!p) return record_error(KMC_EINVAL, "params is NULL");
    if (p->rails < 1) return record_error(KMC_EINVAL, "rails must be >= 1");
    if (p->sites < 2 || p->sites > 65534) return record_error(KMC_EUNSUPPORTED, "sites must be in [2, 65534]");
    if (p->zones < 1 || p->zones > kZoneMaxZones) return record_error(KMC_EUNSUPPORTED, "zones must be in [1, 64]");
    if (p->ions_per_rail < 0 || p->ions_per_rail > kZoneMaxIons || p->ions_per_rail > p->sites)
        return record_error(KMC_EUNSUPPORTED, "ions_per_rail must be in [0, min(64, sites)]");
    if (!(std::isfinite(p->p0) && p->p0 >= 0.0 && p->p0 <= 1.0)) return record_error(KMC_EINVAL, "p0 must be in [0, 1]");
    if (!(std::isfinite(p->kT_ev) && p->kT_ev > 0.0)) return record_error(KMC_EINVAL, "kT_ev must be > 0");
    if (!std::isfinite(p->hop_over_thickness)) return record_error(KMC_EINVAL, "hop_over_thickness must be finite");
    if (!std::isfinite(p->v_factor)) return record_error(KMC_EINVAL, "v_factor must be finite");
    if (!(std::isfinite(p->dt_s) && p->dt_s > 0.0)) return record_error(KMC_EINVAL, "dt_s must be > 0");
    if ((int64_t)p->rails * p->ions_per_rail > ((int64_t)1 << 31) - 1)
        return record_error(KMC_EUNSUPPORTED, "more than 2^31 - 1 ions");
    return KMC_OK;
}

void zone_layout(kmc_zone_ctx *c) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align256(off + bytes);
        return at;
    };
    c->off_X = take(sizeof(uint16_t) * (size_t)c->p.rails * (size_t)std::max(c->p.ions_per_rail, 1));
    c->off_pop = take(sizeof(int64_t) * 2 * kZoneMaxZones);
    c->off_table = take(sizeof(double) * 2 * 2 * kZoneMaxZones);
    c->off_bucket = take(sizeof(int64_t) * kZoneBuckets * kZoneBucketStride);
    c->off_ticket = take(sizeof(uint32_t) * (kZoneBuckets + 1) * 32);
    c->off_knots = take(sizeof(double) * 2 * kMaxKnots);
    c->off_total = take(sizeof(int64_t));
    c->off_bad = take(sizeof(int32_t) * 4);  // rejected occupancy, -, timed-out wait, -
    // (two sets, used in turn by the launches of a call)
    c->off_acc = take(sizeof(uint64_t) * 2 * 2 * kZoneAcc * kZoneAccStride);
    c->off_queue = take(sizeof(kmc::QueueWords) * 2);
    c->total = off;
}

kmc_status zone_hip(kmc_zone_ctx *c, hipError_t e, const char *what) {
    if (e == hipSuccess) return KMC_OK;
    if (c) c->poisoned = true;
    return record_error(KMC_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define ZONE_HIP(c, expr)                                     \
    do {                                                      \
        kmc_status s_ = zone_hip((c), (expr), #expr);         \
        if (s_ != KMC_OK) return s_;                          \
    } while (0)

kmc_status zone_usable(kmc_zone_ctx *c) {
    if (!c) return record_error(KMC_EINVAL, "context is NULL");
    if (c->poisoned) return record_error(KMC_ESTATE, "context poisoned by an earlier HIP error");
    return KMC_OK;
}

hipError_t zone_fill(int64_t *p, int64_t n, int64_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zone_fill_i64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// The table of the current step from the current populations (after a
// state or protocol change; otherwise each step's last workgroup writes it).
kmc_status zone_refresh_table(kmc_zone_ctx *c) {
    const int Z = c->p.zones;
    hipLaunchKernelGGL(zone_make_table, dim3(1), dim3(64), 0, c->stream,
                       c->at<int64_t>(c->off_pop) + c->cur * kZoneMaxZones, Z, c->at<double>(c->off_knots),
                       c->at<double>(c->off_knots) + kMaxKnots, c->n_knots, c->n, c->n_set, c->p.dt_s, c->p.p0,
                       c->p.kT_ev, c->p.hop_over_thickness, c->p.v_factor,
                       c->at<double>(c->off_table) + c->cur * 2 * kZoneMaxZones);
    ZONE_HIP(c, hipGetLastError());
    return KMC_OK;
}

size_t zone_run_lds(int sites) { return sizeof(ZoneLds) + (((size_t)sites + 2 + 15) & ~(size_t)15); }

const void *zone_run_fn(int pairs) {
    switch (pairs) {
        case 1: return (const void *)zone_run<1>;
        case 2: return (const void *)zone_run<2>;
        case 4: return (const void *)zone_run<4>;
        case 8: return (const void *)zone_run<8>;
        default: return (const void *)zone_run<16>;
    }
}

// Launch shape of zone_run: rail pairs per wavefront, workgroups, threads.  At
// most one workgroup per compute unit, so that all are resident; small lattices
// take four wavefronts per workgroup (one per SIMD) and one pair each, larger
// ones sixteen and as few pairs as fit.  Beyond 16 pairs per wavefront the ions'
// registers would spill: no pairs, and zone_step runs step by step (its 33 us
// per step at 128,000 rails are memory passes that grow with the lattice).
struct ZoneShape {
    int pairs;
    unsigned grid, block;
};
ZoneShape zone_shape(const kmc_zone_ctx *c) {
    const int64_t pairs = ((int64_t)c->p.rails + 1) / 2;
    if (c->cus < 1) return {0, 0, 0};
    if (pairs <= 4 * (int64_t)c->cus) return {1, (unsigned)((pairs + 3) / 4), 256};
    for (int per = 1; per <= kZoneRunMaxPairs; per *= 2) {
        const int64_t grid = (pairs + 16 * per - 1) / (16 * per);
        if (grid <= c->cus) return {per, (unsigned)grid, 1024};
    }
    return {0, 0, 0};
}

// Compute units on which every shape of zone_run is resident with a workgroup
// each (0 when one does not fit).
int zone_run_cus(int sites) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    const size_t lds = zone_run_lds(sites);
    if (hipFuncSetAttribute((const void *)zone_queue, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return 0;
    for (int per = 1; per <= kZoneRunMaxPairs; per *= 2) {
        int blocks = 0;
        if (hipFuncSetAttribute(zone_run_fn(per), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, zone_run_fn(per), 1024, lds) != hipSuccess || blocks < 1)
            return 0;
    }
    return cus;
}

// Whether a wait between workgroups of the runs enqueued so far timed out
// (synchronises).  The state is then invalid and the context of no use.
kmc_status zone_check(kmc_zone_ctx *c) {
    int32_t timed_out = 0;
    ZONE_HIP(c, hipMemcpyAsync(&timed_out, c->at<int32_t>(c->off_bad) + 2, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    ZONE_HIP(c, hipStreamSynchronize(c->stream));
    if (!timed_out) return KMC_OK;
    c->poisoned = true;
    return record_error(KMC_EHIP, "zone kernel: a wait between workgroups timed out; state is invalid");
}

// The caller's occupancy after a run of n_steps.
kmc_status zone_export_state(kmc_zone_ctx *c, int64_t n_steps) {
    hipLaunchKernelGGL(zone_export, dim3((unsigned)((c->p.rails + 3) / 4)), dim3(256), 0, c->stream,
                       c->at<uint16_t>(c->off_X), c->occ_user, c->p.rails, c->p.sites, c->p.ions_per_rail,
                       c->at<unsigned long long>(c->off_acc), c->at<kmc::QueueWords>(c->off_queue));
    ZONE_HIP(c, hipGetLastError());
    c->n += n_steps;
    return KMC_OK;
}

// Read the caller's occupancy into X and the populations of the current
// buffer.  A first pass only counts the ions of every rail (and synchronises),
// so a rejected occupancy leaves the context's state as it was.
kmc_status zone_load(kmc_zone_ctx *c) {
    const int Z = c->p.zones;
    int64_t *pop = c->at<int64_t>(c->off_pop) + c->cur * kZoneMaxZones;
    const dim3 grid((unsigned)((c->p.rails + 3) / 4));
    ZONE_HIP(c, zone_fill(reinterpret_cast<int64_t *>(c->at<int32_t>(c->off_bad)), 1, 0, c->stream));
    hipLaunchKernelGGL(zone_import, grid, dim3(256), 0, c->stream, c->occ_user, c->at<uint16_t>(c->off_X), c->p.rails,
                       c->p.sites, c->p.ions_per_rail, Z, pop, c->at<int32_t>(c->off_bad), 0);
    ZONE_HIP(c, hipGetLastError());
    int32_t bad = 0;
    ZONE_HIP(c, hipMemcpyAsync(&bad, c->at<int32_t>(c->off_bad), sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    ZONE_HIP(c, hipStreamSynchronize(c->stream));
    if (bad) return record_error(KMC_EINVAL, "a rail of the occupancy does not hold ions_per_rail ions");
    ZONE_HIP(c, zone_fill(pop, Z, 0, c->stream));
    hipLaunchKernelGGL(zone_import, grid, dim3(256), 0, c->stream, c->occ_user, c->at<uint16_t>(c->off_X), c->p.rails,
                       c->p.sites, c->p.ions_per_rail, Z, pop, c->at<int32_t>(c->off_bad), 1);
    ZONE_HIP(c, hipGetLastError());
    return zone_refresh_table(c);
}

}  // namespace

extern "C" {

kmc_status kmc_zone_workspace_bytes(const kmc_zone_params *params, size_t *bytes) {
    kmc_status s = zone_validate(params);
    if (s != KMC_OK) return s;
    if (!bytes) return record_error(KMC_EINVAL, "bytes is NULL");
    kmc_zone_ctx c;
    c.p = *params;
    zone_layout(&c);
    *bytes = c.total;
    return KMC_OK;
}

kmc_status kmc_zone_init(const kmc_zone_params *params, int8_t *occ_dev, void *workspace_dev, size_t ws_bytes,
                         void *stream, kmc_zone_ctx **out) {
    kmc_status s = zone_validate(params);
    if (s != KMC_OK) return s;
    if (!out || !occ_dev || !workspace_dev) return record_error(KMC_EINVAL, "out, occ_dev and workspace_dev must not be NULL");
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 256 != 0)
        return record_error(KMC_EINVAL, "workspace_dev must be 256-byte aligned");
    kmc_zone_ctx *c = new kmc_zone_ctx();
    c->p = *params;
    zone_layout(c);
    if (ws_bytes < c->total) {
        const size_t need = c->total;
        delete c;
        return record_error(KMC_ETOOSMALL, "workspace too small: need " + std::to_string(need) + " bytes");
    }
    c->ws = static_cast<unsigned char *>(workspace_dev);
    c->occ_user = occ_dev;
    c->stream = static_cast<hipStream_t>(stream);
    auto fail_init = [&](kmc_status st) {
        delete c;
        return st;
    };
    if ((s = zone_hip(c, zone_fill(c->at<int64_t>(c->off_bucket), kZoneBuckets * kZoneBucketStride, 0, c->stream),
                      "clear buckets")) != KMC_OK)
        return fail_init(s);
    if ((s = zone_hip(c, zone_fill(reinterpret_cast<int64_t *>(c->at<uint32_t>(c->off_ticket)), (kZoneBuckets + 1) * 16,
                                   0, c->stream),
                      "clear counters")) != KMC_OK)
        return fail_init(s);
    if ((s = zone_hip(c, zone_fill(c->at<int64_t>(c->off_total), 1, 0, c->stream), "clear total")) != KMC_OK)
        return fail_init(s);
    if ((s = zone_hip(c, zone_fill(c->at<int64_t>(c->off_bad), 2, 0, c->stream), "clear flags")) != KMC_OK) return fail_init(s);
    if ((s = zone_hip(c, zone_fill(c->at<int64_t>(c->off_acc), (int64_t)(c->total - c->off_acc) / 8, 0, c->stream),
                      "clear accumulators and queue words")) != KMC_OK)
        return fail_init(s);
    c->cus = zone_run_cus(c->p.sites);
    ZoneKnots k{};
    hipLaunchKernelGGL(zone_set_knots, dim3(1), dim3(64), 0, c->stream, c->at<double>(c->off_knots),
                       c->at<double>(c->off_knots) + kMaxKnots, k);
    if ((s = zone_hip(c, hipGetLastError(), "install 0 V")) != KMC_OK) return fail_init(s);
    if ((s = zone_load(c)) != KMC_OK) return fail_init(s);
    *out = c;
    return KMC_OK;
}

kmc_status kmc_zone_load_occupancy(kmc_zone_ctx *c) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if ((s = zone_check(c)) != KMC_OK) return s;
    return zone_load(c);
}

kmc_status kmc_zone_set_bias_protocol(kmc_zone_ctx *c, const double *t_s, const double *v_volt, int32_t n_knots) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if (n_knots < 1 || n_knots > kMaxKnots) return record_error(KMC_EINVAL, "n_knots must be in [1, 64]");
    if (!t_s || !v_volt) return record_error(KMC_EINVAL, "knot arrays are NULL");
    ZoneKnots k{};
    for (int i = 0; i < n_knots; ++i) {
        if (!std::isfinite(t_s[i]) || !std::isfinite(v_volt[i])) return record_error(KMC_EINVAL, "knots must be finite");
        if (i > 0 && t_s[i] < t_s[i - 1]) return record_error(KMC_EINVAL, "knot times must be nondecreasing");
        k.t[i] = t_s[i];
        k.v[i] = v_volt[i];
    }
    hipLaunchKernelGGL(zone_set_knots, dim3(1), dim3(64), 0, c->stream, c->at<double>(c->off_knots),
                       c->at<double>(c->off_knots) + kMaxKnots, k);
    ZONE_HIP(c, hipGetLastError());
    c->n_knots = n_knots;
    c->n_set = c->n;
    return zone_refresh_table(c);
}

kmc_status kmc_zone_run_steps(kmc_zone_ctx *c, int64_t n_steps, int32_t *net_dev, int32_t *zone_dev) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if (n_steps < 0) return record_error(KMC_EINVAL, "n_steps < 0");
    if (c->n + n_steps > (int64_t)0xffffffffLL) return record_error(KMC_EUNSUPPORTED, "step counter would reach 2^32");
    if (n_steps == 0) return KMC_OK;
    ZoneArgs a{};
    a.X = c->at<uint16_t>(c->off_X);
    a.rails = c->p.rails;
    a.ions = c->p.ions_per_rail;
    a.sites = c->p.sites;
    a.zones = c->p.zones;
    a.p0 = c->p.p0;
    a.kT = c->p.kT_ev;
    a.hot = c->p.hop_over_thickness;
    a.v_factor = c->p.v_factor;
    a.dt = c->p.dt_s;
    a.key0 = (uint32_t)(c->p.seed & 0xffffffffu);
    a.key1 = (uint32_t)(c->p.seed >> 32);
    a.knot_t = c->at<double>(c->off_knots);
    a.knot_v = a.knot_t + kMaxKnots;
    a.n_knots = c->n_knots;
    a.n_set = c->n_set;
    a.bucket = c->at<int64_t>(c->off_bucket);
    a.ticket = c->at<uint32_t>(c->off_ticket);
    a.net_out = net_dev;
    a.zone_out = zone_dev;
    a.net_total = c->at<int64_t>(c->off_total);
    a.bad = c->at<int32_t>(c->off_bad) + 2;
    const int64_t pairs = ((int64_t)c->p.rails + 1) / 2;
    const ZoneShape shape = zone_shape(c);
    // One step of a large lattice goes by zone_step: loading the ions to
    // registers and the launch behind cost more than its passes over memory
    // (128,000 rails: 77 us for the call against 69; 32,000: 39 and 37; 4000: 27
    // and 29; two steps 91 and 103, 44 and 53, 30 and 42).
    if (shape.pairs > 0 && (n_steps > 1 || c->p.rails <= 16384)) {
        ZoneRunArgs r{};
        r.X = a.X;
        r.rails = a.rails;
        r.ions = a.ions;
        r.sites = a.sites;
        r.zones = a.zones;
        r.p0 = a.p0;
        r.kT = a.kT;
        r.hot = a.hot;
        r.v_factor = a.v_factor;
        r.dt = a.dt;
        r.key0 = a.key0;
        r.key1 = a.key1;
        r.knot_t = a.knot_t;
        r.knot_v = a.knot_v;
        r.n_knots = a.n_knots;
        r.n_set = a.n_set;
        r.table = c->at<double>(c->off_table) + c->cur * 2 * kZoneMaxZones;
        r.pop = c->at<int64_t>(c->off_pop) + c->cur * kZoneMaxZones;
        r.bad = c->at<int32_t>(c->off_bad) + 2;
        r.net_out = net_dev;
        r.zone_out = zone_dev;
        r.net_total = a.net_total;
        r.wait_limit = c->wait_limit;
        r.tile_pairs = (int32_t)std::max<int64_t>((pairs + shape.grid - 1) / shape.grid, 16);
        r.n_tiles = (int32_t)((pairs + r.tile_pairs - 1) / r.tile_pairs);
        const size_t lds = zone_run_lds(c->p.sites);
        for (int64_t k = 0; k < n_steps; k += kZoneRunSteps) {
            r.n0 = c->n + k;
            r.row0 = k;
            r.n_steps = (int32_t)std::min<int64_t>(kZoneRunSteps, n_steps - k);
            r.gate_ticks = (int32_t)std::min<int64_t>(c->gate_ticks, kmc::kGateTicks * std::max(r.n_steps, 16));
            unsigned long long *acc = c->at<unsigned long long>(c->off_acc);
            kmc::QueueWords *queue = c->at<kmc::QueueWords>(c->off_queue);
            const int set = (int)(k / kZoneRunSteps) & 1;
            r.acc = acc + set * 2 * kZoneAcc * kZoneAccStride;
            r.queue = queue + set;
            r.acc_next = acc + (1 - set) * 2 * kZoneAcc * kZoneAccStride;
            r.queue_next = queue + (1 - set);
            void *kargs[] = {&r};
            ZONE_HIP(c, hipLaunchKernel(zone_run_fn(shape.pairs), dim3(shape.grid), dim3(shape.block), kargs, lds, c->stream));
            ZONE_HIP(c, hipLaunchKernel((const void *)zone_queue, dim3((unsigned)std::min<int64_t>(r.n_tiles, shape.grid)),
                                        dim3(1024), kargs, lds, c->stream));
        }
        return zone_export_state(c, n_steps);
    }
    const int64_t per_wg = (int64_t)(kZoneBlock / 64) * kZonePairsPerIter;
    const unsigned grid = (unsigned)std::min<int64_t>((pairs + per_wg - 1) / per_wg, kZoneMaxGrid);
    int64_t *pop = c->at<int64_t>(c->off_pop);
    double *table = c->at<double>(c->off_table);
    for (int64_t k = 0; k < n_steps; ++k) {
        a.n = c->n + k;
        a.row = k;
        a.table = table + c->cur * 2 * kZoneMaxZones;
        a.table_next = table + (1 - c->cur) * 2 * kZoneMaxZones;
        a.pop_next = pop + (1 - c->cur) * kZoneMaxZones;
        hipLaunchKernelGGL(zone_step, dim3(grid), dim3(kZoneBlock), 0, c->stream, a);
        ZONE_HIP(c, hipGetLastError());
        c->cur = 1 - c->cur;
    }
    return zone_export_state(c, n_steps);
}

kmc_status kmc_zone_read_positions(kmc_zone_ctx *c, int32_t *X_host, size_t count) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if (!X_host) return record_error(KMC_EINVAL, "X_host is NULL");
    const size_t n = (size_t)c->p.rails * (size_t)c->p.ions_per_rail;
    if (count < n) return record_error(KMC_ETOOSMALL, "X_host holds fewer than rails * ions_per_rail entries");
    if ((s = zone_check(c)) != KMC_OK) return s;
    std::vector<uint16_t> tmp(n);
    if (n > 0) {
        ZONE_HIP(c, hipMemcpyAsync(tmp.data(), c->at<uint16_t>(c->off_X), sizeof(uint16_t) * n, hipMemcpyDeviceToHost,
                                   c->stream));
    }
    ZONE_HIP(c, hipStreamSynchronize(c->stream));
    for (size_t i = 0; i < n; ++i) X_host[i] = tmp[i];
    return KMC_OK;
}

kmc_status kmc_zone_set_gate_limit(kmc_zone_ctx *c, int32_t microseconds) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if (microseconds < 0 || microseconds > 10000000) return record_error(KMC_EINVAL, "microseconds must be in [0, 10^7]");
    c->gate_ticks = microseconds * 100;
    return KMC_OK;
}

kmc_status kmc_zone_set_wait_limit(kmc_zone_ctx *c, int32_t polls) {
    kmc_status s = zone_usable(c);
    if (s != KMC_OK) return s;
    if (polls < 0) return record_error(KMC_EINVAL, "polls must be >= 0");
    c->wait_limit = polls;
    return KMC_OK;
}

kmc_status kmc_zone_check(kmc_zone_ctx *c) {
    kmc_status s = zone_usable(c);
    return s != KMC_OK ? s : zone_check(c);
}

kmc_status kmc_zone_get_step(kmc_zone_ctx *c, int64_t *step) {
    if (!c || !step) return record_error(KMC_EINVAL, "NULL argument");
    *step = c->n;
    return KMC_OK;
}

void kmc_zone_destroy(kmc_zone_ctx *c) {
    if (!c) return;
    if (!c->poisoned) (void)hipStreamSynchronize(c->stream);
    delete c;
}

}  // extern "C"
