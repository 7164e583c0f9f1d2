// Half-steps of the long-range paths (KMC_BF16X2 and KMC_PHI_FIXED) driven by
// their low Philox draws.
//
// A candidate can hop only when its word is at most the step's stage-0
// threshold (class_threshold of the lowest barrier class: an exact bound, with
// the potential's own error bound added where it is computed in binary32).
// That test needs no state, so the words of the next half-step are drawn and
// tested while the present one is resolved, and only the few low draws (about
// 500 of 1.7e7 words at 0.3 eV) ever look at the lattice:
//
//   launch j resolves the low draws of half-step j and generates those of
//   half-step j + 1.
//
// Resolving reads the draws' bonds, keeps the candidates (one site of the two
// occupied) and needs the potential at their two sites only.
//   * dense: 32 survivors of one 32-site column block make one 32 x 32 MFMA
//     tile: row i of the left operand is the occupancy of survivor i's own
//     neighbour rails, so the tile's element (i, s) is the potential of
//     survivor i's rail at site s, the products and their order being those of
//     dense_phi (same instruction, same k order; rows and columns of a tile do
//     not interact), hence the same bits.  The odd parity's column blocks start
//     one site later (a second set of kernel fragments), so that no bond
//     straddles two blocks.
//   * fixed: the potential kept hop by hop is read at the two sites.
//
// Snapshots.  Every decision must see the state before the half-step, while
// accepted hops change it.  Two planes alternate: launch j reads a plane that
// holds the hops up to half-step j - 2, adds those of half-step j - 1 from their
// list (to the bytes or potentials it read), and brings the other plane, which
// nobody reads in this launch, to half-step j - 1.  Nothing therefore waits
// inside a launch, and one launch per half-step does.
//
// What bounds it (64 x 1024 x 512 at 0.3 eV, 1900 draws and 63 hops per
// half-step): the latency of a resolving workgroup, about 18 us in the dense
// form (reading the draws 1.8, their sites 0.9, the rails 4, kernel fragments
// and the previous hops 2, the chain of 320 dependent products 7.5 at about 60
// cycles each, the decision 1.5); beside it the generator's 10 us (its Philox
// blocks alone 4.7 at the VALU's rate), followed in the fixed form by the other
// plane's potential.  22 us per half-step dense (the whole potential and its
// decisions: 280) and 16 fixed (decisions and update launches: 26).
#include "kmc_draws.h"

#include <algorithm>

#include "kmc_device.h"
#include "kmc_philox.h"

namespace kmc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Eight occupancy-sum bytes (values 0..2) -> eight BF16 values (0, 1.0, 2.0).
__device__ __forceinline__ u32x4 sums_to_bf16(uint2 v) {
    const uint32_t t_lo = 0x00008000u, t_hi = 0x00403F00u;  // low and high bytes of BF16 0, 1, 2
    const uint32_t l0 = __builtin_amdgcn_perm(0u, t_lo, v.x), h0 = __builtin_amdgcn_perm(0u, t_hi, v.x);
    const uint32_t l1 = __builtin_amdgcn_perm(0u, t_lo, v.y), h1 = __builtin_amdgcn_perm(0u, t_hi, v.y);
    u32x4 r;
    r.x = __builtin_amdgcn_perm(h0, l0, 0x05010400u);
    r.y = __builtin_amdgcn_perm(h0, l0, 0x07030602u);
    r.z = __builtin_amdgcn_perm(h1, l1, 0x05010400u);
    r.w = __builtin_amdgcn_perm(h1, l1, 0x07030602u);
    return r;
}

constexpr int kStaged = 256;         // hops of the previous half-step looked at together
constexpr int kDenseBatch = 32;      // survivors of one MFMA tile
constexpr int kFixedBatch = 64;
constexpr int kChain = 4;            // k-steps of the dense tile per wavefront and turn

struct DrawLds {
    uint4 draw[kDrawList];               // resolving: the workgroup's draws; generating: see gen
    uint4 hop[kStaged];
    uint32_t flip[kDrawList];            // bit 0, 1: the draw's sites changed by the previous half-step
    int64_t rise[kDrawList];             // fixed: its hops' contributions to phi(s + 1) - phi(s)
    uint4 surv[kDrawList];               // survivors (site << 1 | ion at the lower site)
    int64_t surv_rise[kDrawList];
    int32_t surv_rails[kDrawList];       // rails of its device
    int32_t n_draws, n_surv;
    float4 acc[4][64];                   // dense: the tile's accumulator, passed from wavefront to wavefront
    int32_t nbr_off[2 * kMaxRailRange + 1], nbr_dist[2 * kMaxRailRange + 1];  // fixed: of a hop's device
    uint4 gen[kDrawSlots];               // generating: the workgroup's low draws, from slot 1
    uint32_t n_gen;
};

__device__ __forceinline__ int ring_distance(int a, int b, int R) {
    const int x = a < b ? b - a : a - b;
    return x < R - x ? x : R - x;
}

// A hop into a state plane: the two bytes' occupancy bits change (atomically: a
// byte may take a hop of each of two lists).
__device__ void flip_sites(int8_t *plane, const DevInfo *devs, uint4 hop) {
    const DevInfo &dv = devs[hop.z];
    const int64_t at = dv.off_pad + (int64_t)hop.w * dv.pitch + (hop.y >> 1);
    for (int e = 0; e < 2; ++e) {
        const uintptr_t p = reinterpret_cast<uintptr_t>(plane) + (uintptr_t)(at + e);
        atomicXor(reinterpret_cast<unsigned int *>(p & ~(uintptr_t)3), 1u << (8 * (p & 3)));
    }
}

// A hop's change of the fixed-point potential: K(x - t) - K(x - o) on every
// distinct rail within rail_range, one workgroup, integer atomics (see
// kmc_phifix.hip).  kt: the kernel table, in LDS; off, dist: LDS for the
// device's neighbour rails.
__device__ void add_hop_potential(const DrawArgs &a, const int64_t *kt, int64_t *phi, uint4 hop, int32_t *off, int32_t *dist) {
    const DevInfo &dv = a.devs[hop.z];
    __syncthreads();
    if (threadIdx.x < 2 * kMaxRailRange + 1) {
        off[threadIdx.x] = dv.nbr_off[threadIdx.x];
        dist[threadIdx.x] = dv.nbr_dist[threadIdx.x];
    }
    __syncthreads();
    const int r = (int)hop.w, s = (int)(hop.y >> 1);
    const int o = hop.y & 1u ? s + 1 : s, t = hop.y & 1u ? s : s + 1;
    const int L = dv.sites, R = dv.rails, cut = a.cutoff, cs = cut + 1;
    int lo = s - cut, hi = s + 1 + cut;
    lo = lo < 0 ? 0 : lo;
    hi = hi > L - 1 ? L - 1 : hi;
    const int span = hi - lo + 1, work = span * dv.n_nbr;
    unsigned long long *base = reinterpret_cast<unsigned long long *>(phi) + dv.off_pad;
    for (int i = threadIdx.x; i < work; i += blockDim.x) {
        const int k = i / span, x = lo + i - k * span;
        int rr = r + off[k];
        if (rr < 0 || rr >= R) rr = ((rr % R) + R) % R;
        const int64_t *ktr = kt + dist[k] * cs;
        const int dt_ = abs(x - t), do_ = abs(x - o);
        const int64_t delta = (dt_ <= cut ? ktr[dt_] : 0) - (do_ <= cut ? ktr[do_] : 0);
        if (delta != 0) atomicAdd(base + (int64_t)rr * dv.pitch + x, (unsigned long long)delta);
    }
}

// Draws the words of the half-step of parity H, step n, on the workgroup's
// share of the rails (part `first` of `stride`, device by device) and lists the
// low ones in the workgroup's own list (one counter for all workgroups' draws
// serialised them: 25 us of the launch).
template <int H>
__device__ void generate(const DrawArgs &a, DrawLds &w, int64_t n, int k, int64_t list, int first, int stride) {
    const int tid = threadIdx.x;
    if (tid == 0) w.n_gen = 0u;
    __syncthreads();
    const int64_t end = draw_share(a.rails_total, first + 1, stride);
    for (int64_t row = draw_share(a.rails_total, first, stride); row < end;) {
        const int d = a.rail_dev[row];
        const DevInfo &dv = a.devs[d];
        const uint32_t thr = a.thr[(int64_t)k * a.n_devices + d];
        const int bpr = dv.pitch / 8, per_pass = kDrawBlock / bpr;
        const int slot = tid / bpr, b = tid - slot * bpr;
        const int r0 = (int)(row - dv.row0);
        const int r1 = (int)min((int64_t)dv.rails, end - dv.row0);
        row = dv.row0 + r1;
        if (slot >= per_pass) continue;
        const int last = dv.sites - 2 - 8 * b;  // bond (8b + q, 8b + q + 1) exists iff q <= last
        const PhiloxLane lc = philox_lane((uint32_t)b, ((uint32_t)d << 4) | (uint32_t)H, a.key0, a.key1);
        const PhiloxStep sc = philox_step(lc, (uint32_t)n, a.key0, a.key1);
        for (int r = r0 + slot; r < r1; r += per_pass) {
            const uint4 x = philox_words(lc, sc, (uint32_t)r, a.key0, a.key1);
            if (min(min(x.x, x.y), min(x.z, x.w)) <= thr) {
                for (int i = 0; i < 4; ++i) {
                    const int q = H + 2 * i;
                    if (word_of(x, i) > thr || q > last) continue;
                    const uint32_t at = atomicAdd(&w.n_gen, 1u) + 1u;
                    if (at < kDrawSlots)
                        w.gen[at] = make_uint4((uint32_t)(dv.row0 + r), (uint32_t)(8 * b + q), (uint32_t)d, (uint32_t)r);
                }
            }
        }
    }
    __syncthreads();
    uint4 *out = a.draws + ((list & 1) * kDrawMaxGrid + blockIdx.x) * kDrawSlots;
    uint32_t m = w.n_gen;
    if (m >= kDrawSlots) {
        if (tid == 0) __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        m = kDrawSlots - 1;
    }
    if (tid == 0) out[0] = make_uint4(m, 0u, 0u, 0u);
    else if (tid <= (int)m) out[tid] = w.gen[tid];
}

// Loads and products of the dense tile: element (i, c) is the potential of row
// i of x at site c of column block `bin`.  x: [m + 1][rows][rs] sums of the
// rails at each distance.  The accumulator's chain of products (its order is
// dense_phi's) goes from wavefront to wavefront, kChain k-steps each, so that
// every wavefront's kernel fragments are in its registers before its turn: one
// wavefront with four k-steps of loads in flight waited for each (about 20 us).
struct DenseFragments {
    u32x4 t[kChain][2][2];
};
__device__ __forceinline__ void load_fragments(const DrawArgs &a, int bin, int turn, DenseFragments &f) {
    const int lane = threadIdx.x & 63, nb = a.nb, nd = 2 * nb - 1;
    const int dd = turn * kChain / nb, jb = turn * kChain - dd * nb;
    if (dd > a.rail_range) return;
    // a uniform base and a lane offset; opaque, so that the addresses are not
    // held in registers from batch to batch
    const char *base = reinterpret_cast<const char *>(a.ktiles) + ((int64_t)dd * nd + (jb - bin + nb - 1)) * 4096;
    uint32_t at = 16u * (uint32_t)lane;
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int u = 0; u < kChain; ++u)  // [m+1][nd][part][q][64]
#pragma unroll
        for (int x = 0; x < 4; ++x)
            f.t[u][x >> 1][x & 1] = *reinterpret_cast<const u32x4 *>(base + u * 4096 + x * 1024 + (size_t)at);
}
// The left operand of a wavefront's k-steps, from the sums in LDS.
__device__ __forceinline__ void load_rows(const DrawArgs &a, const unsigned char *x, int rs, int turn, u32x4 (&xa)[kChain][2]) {
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    // (nb is a multiple of kChain: a turn stays at one distance)
    const int dd = turn * kChain / a.nb, jb = turn * kChain - dd * a.nb;
    if (dd > a.rail_range) return;
    const unsigned char *xd = x + (dd * a.rows + (col & (a.rows - 1))) * rs + half * 8 + jb * 32;
#pragma unroll
    for (int u = 0; u < kChain; ++u)
#pragma unroll
        for (int q = 0; q < 2; ++q) xa[u][q] = sums_to_bf16(*reinterpret_cast<const uint2 *>(xd + u * 32 + q * 16));
}
__device__ __forceinline__ void dense_turn(int turn, const DenseFragments &f, const u32x4 (&xa)[kChain][2], float4 (*acc_lds)[64]) {
    const int lane = threadIdx.x & 63;
    f32x16 acc = f32x16{};
    if (turn > 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float4 v = acc_lds[r][lane];
            acc[4 * r] = v.x;
            acc[4 * r + 1] = v.y;
            acc[4 * r + 2] = v.z;
            acc[4 * r + 3] = v.w;
        }
#pragma unroll
    for (int u = 0; u < kChain; ++u)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int part = 0; part < 2; ++part)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa[u][q]),
                                                              __builtin_bit_cast(bf16x8, f.t[u][part][q]), acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc_lds[r][lane] = make_float4(acc[4 * r], acc[4 * r + 1], acc[4 * r + 2], acc[4 * r + 3]);
}

// Resolves the half-step of parity H on the draws of column block `bin` (fixed:
// 0) in the lists of the generating workgroups `part`, part + per_bin, ...
template <bool Dense, int H>
__device__ void resolve(const DrawArgs &a, DrawLds &w, unsigned char *smem, int bin, int part) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t list = a.launch;
    const uint4 *prev = a.hops + ((list + 3) & 3) * a.hop_cap;   // hops of half-step j - 1
    const int n_prev = list > 0 ? (int)min((int64_t)a.n_hops[(list + 3) & 3], a.hop_cap) : 0;
    if (tid == 0) w.n_draws = 0;
    if (tid < kDrawList) {
        w.flip[tid] = 0u;
        w.rise[tid] = 0;
    }
    auto stage = [&](int h0) {  // hops h0 .. h0 + kStaged - 1 of the previous half-step
        if (tid < kStaged && h0 + tid < n_prev) w.hop[tid] = prev[h0 + tid];
    };
    if (tid < kStaged) w.hop[tid] = prev[tid];  // (the lists are longer; beyond the count: not used)
    __syncthreads();
    // the draws: four threads per list, its first 16 slots (the count among
    // them) in one round of loads
    {
        const int segments = gridDim.x;
        const int seg = tid >> 2, sub = tid & 3;
        const bool mine = seg < segments && seg % a.per_bin == part;
        const uint4 *from = a.draws + ((list & 1) * kDrawMaxGrid + seg) * kDrawSlots;
        uint4 e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = mine ? from[4 * sub + i] : make_uint4(0u, 0u, 0u, 0u);
        const int count = __shfl((int)e[0].x, lane & ~3, 64);
        auto take = [&](uint4 v) {
            if (Dense && (((int)v.y - H) >> 5) != bin) return;
            const int at = atomicAdd(&w.n_draws, 1);
            if (at < kDrawList) w.draw[at] = v;
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int slot = 4 * sub + i;
            if (slot >= 1 && slot <= count) take(e[i]);
        }
        for (int slot = 16 + sub; slot <= count; slot += 4) take(from[slot]);
    }
    __syncthreads();
    int n_draws = w.n_draws;
    if (n_draws > kDrawList) {
        if (tid == 0) __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        n_draws = kDrawList;
    }
    if (n_draws == 0) return;
    // the state of their bonds, before the previous half-step's hops
    uint4 own = make_uint4(0u, 0u, 0u, 0u);
    uint32_t b0 = 0, b1 = 0;
    int own_rails = 0;
    if (tid < n_draws) {
        own = w.draw[tid];
        own_rails = a.devs[own.z].rails;
        const int8_t *at = a.plane + own.y;
        if (Dense) at += (int64_t)own.x * a.pitch;
        else at += a.devs[own.z].off_pad + (int64_t)own.w * a.devs[own.z].pitch;
        b0 = (uint32_t)at[0] & 1u;
        b1 = (uint32_t)at[1] & 1u;
    }
    for (int h0 = 0; h0 < n_prev; h0 += kStaged) {
        if (h0 > 0) {
            __syncthreads();
            stage(h0);
            __syncthreads();
        }
        const int m = min(kStaged, n_prev - h0);
        for (int q = tid; q < m * n_draws; q += kDrawBlock) {
            const int h = q / n_draws, i = q - h * n_draws;
            const uint4 e = w.hop[h], x = w.draw[i];
            const int s = (int)x.y, hs = (int)(e.y >> 1);
            if (e.x == x.x && (hs == s - 1 || hs == s + 1)) atomicXor(&w.flip[i], hs == s - 1 ? 1u : 2u);
            if (!Dense && e.z == x.z) {
                const int dist = ring_distance((int)e.w, (int)x.w, a.devs[x.z].rails);
                if (dist <= a.rail_range) {
                    const int cut = a.cutoff;
                    const int64_t *ktr = a.kfix + (int64_t)dist * (cut + 1);
                    auto K = [&](int y) { y = abs(y); return y <= cut ? ktr[y] : (int64_t)0; };
                    const int ho = e.y & 1u ? hs + 1 : hs, ht = e.y & 1u ? hs : hs + 1;
                    const int64_t up = K(s + 1 - ht) - K(s + 1 - ho), low = K(s - ht) - K(s - ho);
                    atomicAdd(reinterpret_cast<unsigned long long *>(&w.rise[i]), (unsigned long long)(up - low));
                }
            }
        }
    }
    if (tid == 0) w.n_surv = 0;
    __syncthreads();
    if (tid < n_draws) {
        // the candidates among them
        b0 ^= w.flip[tid] & 1u;
        b1 ^= w.flip[tid] >> 1;
        if (b0 != b1) {
            const int to = atomicAdd(&w.n_surv, 1);
            w.surv[to] = make_uint4(own.x, own.y << 1 | b0, own.z, own.w);
            w.surv_rise[to] = w.rise[tid];
            w.surv_rails[to] = own_rails;
        }
    }
    __syncthreads();
    const int n_surv = w.n_surv;
    const int batch = Dense ? a.rows : kFixedBatch;
    for (int i0 = 0; i0 < n_surv; i0 += batch) {
        const int here = min(batch, n_surv - i0);
        // (opaque: what follows from the thread's index is not held in
        // registers from batch to batch)
        int me_tid = tid;
        asm volatile("" : "+v"(me_tid));
        // the decisions are the last wavefront's (whose turn in the dense tile
        // comes last); their own inputs are loaded before that
        const int me = me_tid - (kDrawBlock - 64);
        const bool decider = me >= 0 && me < here;
        uint4 x = make_uint4(0u, 0u, 0u, 0u);
        double V = 0.0, ea = 0.0;
        int64_t rise = 0;
        int L = 2;
        auto load_inputs = [&]() {
            if (decider) {
                x = w.surv[i0 + me];
                const DevInfo &dv = a.devs[x.z];
                const int s = (int)(x.y >> 1), o = x.y & 1u ? s : s + 1;
                L = dv.sites;
                V = a.volt[(int64_t)a.k * a.n_devices + x.z];
                const int64_t at = dv.off + (int64_t)x.w * L + o;
                ea = !a.ea ? a.ea_scalar
                           : (Dense ? (double)reinterpret_cast<const float *>(a.ea)[at] : reinterpret_cast<const double *>(a.ea)[at]);
                if constexpr (!Dense) {
                    const int64_t prow = dv.off_pad + (int64_t)x.w * dv.pitch + s;
                    rise = a.phi[prow + 1] - a.phi[prow] + w.surv_rise[i0 + me];
                }
            }
        };
        if constexpr (Dense) {
            // the rows of the left operand: for every survivor, the sums of the
            // rails at each distance
            const int Lp = a.nb * 32, rs = Lp + 8, pieces = Lp / 16;
            // 16 sites per thread and turn: rails of up to 512 sites take one
            // turn, longer ones two where more than half a tile has survivors.
            // (The rows of a tile do not interact: those without a survivor
            // are neither staged nor looked at.  The second turn is straight
            // code off the common path: as a loop it took 0.5 us of the 46 per
            // step of 64 x 1024 x 512, which has no second turn.)
            static_assert(kDenseBatch * (kDenseMaxSites / 16) <= 2 * kDrawBlock, "two turns stage a tile");
            auto put_piece = [&](int p) {
                const int i = p / pieces, c = p - i * pieces;
                // (every load is issued before the first is used, so the
                // rails that are not wanted are read as the survivor's own)
                const bool have = c * 16 < a.pitch;
                const uint4 v = w.surv[i0 + i];
                const int rr = (int)v.w, R = w.surv_rails[i0 + i];
                const int8_t *base = a.plane + (int64_t)(v.x - v.w) * a.pitch + (have ? c * 16 : 0);
                // (two groups of loads: all nine rails would not fit the
                // registers)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    constexpr int kFirst[3] = {0, 3, kMaxRailRange + 1};
                    uint4 raw[2][3];
#pragma unroll
                    for (int dd = kFirst[g]; dd < kFirst[g + 1]; ++dd)
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            int y = k ? rr - dd : rr + dd;
                            y = y >= R ? y - R : (y < 0 ? y + R : y);
                            if (dd > a.rail_range || 2 * dd > R) y = rr;
                            if (dd > 0 || k == 0)
                                raw[k][dd - kFirst[g]] = *reinterpret_cast<const uint4 *>(base + (int64_t)y * a.pitch);
                        }
#pragma unroll
                    for (int dd = kFirst[g]; dd < kFirst[g + 1]; ++dd)
                        if (dd <= a.rail_range) {
                            // one rail at distance 0 and at half the ring, else two; none beyond
                            const uint32_t m1 = have && 2 * dd <= R ? 0x01010101u : 0u;
                            const uint32_t m2 = have && dd > 0 && 2 * dd < R ? 0x01010101u : 0u;
                            const uint4 x1 = raw[0][dd - kFirst[g]], x2 = raw[dd > 0][dd - kFirst[g]];
                            unsigned char *to = smem + (dd * a.rows + i) * rs + c * 16;
                            *reinterpret_cast<uint2 *>(to) = make_uint2((x1.x & m1) + (x2.x & m2), (x1.y & m1) + (x2.y & m2));
                            *reinterpret_cast<uint2 *>(to + 8) = make_uint2((x1.z & m1) + (x2.z & m2), (x1.w & m1) + (x2.w & m2));
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (me_tid < here * pieces) put_piece(me_tid);
            if (__builtin_expect(here * pieces > kDrawBlock, 0)) {
                if (me_tid + kDrawBlock < here * pieces) put_piece(me_tid + kDrawBlock);
            }
            DenseFragments f;
            load_fragments(a, bin, wave, f);
            if (n_prev > kStaged) {
                __syncthreads();
                stage(0);
            }
            __syncthreads();
            // the previous half-step's hops, added where they touch those rails
            for (int h0 = 0; h0 < n_prev; h0 += kStaged) {
                if (h0 > 0) {
                    __syncthreads();
                    stage(h0);
                    __syncthreads();
                }
                const int m = min(kStaged, n_prev - h0);
                for (int p = me_tid; p < m * kDenseBatch; p += kDrawBlock) {
                    const int i = p % kDenseBatch;
                    const uint4 e = w.hop[p / kDenseBatch];
                    if (i < here && e.z == w.surv[i0 + i].z) {
                        const int dist = ring_distance((int)e.w, (int)w.surv[i0 + i].w, w.surv_rails[i0 + i]);
                        if (dist <= a.rail_range) {
                            const int hs = (int)(e.y >> 1), o = e.y & 1u ? hs + 1 : hs, t = e.y & 1u ? hs : hs + 1;
                            const int at = (dist * a.rows + i) * rs;
                            auto add = [&](int b, uint32_t v) {
                                atomicAdd(reinterpret_cast<unsigned int *>(smem) + ((at + b) >> 2), v << (8 * ((at + b) & 3)));
                            };
                            add(t, 1u);
                            add(o, 0xFFFFFFFFu);
                        }
                    }
                }
            }
            load_inputs();
            const int turns = (a.rail_range + 1) * a.nb / kChain;
            for (int turn0 = 0; turn0 < turns; turn0 += kDrawBlock / 64) {
                if (turn0 == 0) __syncthreads();  // the rows are complete
                u32x4 xa[kChain][2];
                load_rows(a, smem, rs, turn0 + wave, xa);
                for (int turn = turn0; turn < min(turns, turn0 + kDrawBlock / 64); ++turn) {
                    lds_barrier();
                    if (wave == turn - turn0) {
                        dense_turn(turn, f, xa, w.acc);
                        load_fragments(a, bin, turn + kDrawBlock / 64, f);
                    }
                }
            }
            __syncthreads();
        }
        if constexpr (!Dense) load_inputs();
        bool acc = false;
        const int s = (int)(x.y >> 1);
        const bool up = (x.y & 1u) != 0u;
        const int o = up ? s : s + 1, t = up ? s + 1 : s;
        if (decider) {
            const uint4 blk = philox4x32_10((uint32_t)s >> 3, x.w, (uint32_t)a.n, (x.z << 4) | (uint32_t)H, a.key0, a.key1);
            const uint32_t word = word_of(blk, (s >> 1) & 3);
            if constexpr (Dense) {
                // element (me, c) of the tile: register 4 (me / 8) + me % 4 of lane 32 ((me / 4) % 2) + c
                const float *row = &w.acc[me >> 3][32 * ((me >> 2) & 1) + (s - H - 32 * bin)].x + (me & 3);
                const float lower = row[0], upper = row[4];
                const float phi_o = up ? lower : upper, phi_t = up ? upper : lower;
                const float alpha_r = (float)a.alpha, V_r = (float)V, beta_r = (float)a.beta, c0_r = (float)a.c0;
                const float e_coul = (phi_t - a.k10) - phi_o;
                const float e_app = ((alpha_r * V_r) * (float)(t - o)) / (float)L;
                acc = decide_hop<float>(e_app + e_coul, (float)ea, word, beta_r, c0_r, a.log, (int)x.z, H, a.n, (int)x.w, s);
            } else {
                const int64_t diff = (up ? rise : -rise) - a.k10fix;
                const double e_coul = ldexp((double)diff, -a.frac_bits);
                const double e_app = ((a.alpha * V) * (double)(t - o)) / (double)L;
                acc = decide_hop<double>(e_app + e_coul, ea, word, a.beta, a.c0, a.log, (int)x.z, H, a.n, (int)x.w, s);
            }
        }
        if (wave == kDrawBlock / 64 - 1) {
            // one reservation for the wavefront's hops
            const uint64_t m = __ballot(acc);
            uint32_t base = 0;
            if (m && lane == 0) base = atomicAdd(&a.n_hops[list & 3], (uint32_t)__popcll(m));
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (acc) {
                const int64_t at = (int64_t)base + __popcll(m & ((1ull << lane) - 1ull));
                if (at >= a.hop_cap) __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else a.hops[(list & 3) * a.hop_cap + at] = make_uint4(x.x, (uint32_t)s << 1 | (up ? 0u : 1u), x.z, x.w);
                const int64_t row = a.tally_row * a.n_devices + x.z;
                atomicAdd(&a.tally_net[row], t < o ? 1 : -1);
                const int qo = (10 * o) / L, qt = (10 * t) / L;
                if (qo != qt) {
                    atomicAdd(&a.tally_dec[row * kDeciles + qo], -1);
                    atomicAdd(&a.tally_dec[row * kDeciles + qt], 1);
                }
            }
        }
        __syncthreads();
    }
}

// One launch: the first n_bins x per_bin workgroups resolve the half-step, the
// others bring the other plane up to date and generate the next half-step's
// draws.
template <bool Dense, int H>
__global__ __launch_bounds__(kDrawBlock) void half_step_draws(DrawArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ DrawLds w;
    const int tid = threadIdx.x;
    const int64_t j = a.launch;
    const int resolvers = a.resolve ? a.n_bins * a.per_bin : 0;
    if ((int)blockIdx.x < resolvers) {
        // (an empty list of the next half-step's draws)
        if (tid == 0 && a.generate)
            a.draws[(((j + 1) & 1) * kDrawMaxGrid + blockIdx.x) * kDrawSlots] = make_uint4(0u, 0u, 0u, 0u);
        resolve<Dense, H>(a, w, smem, (int)blockIdx.x / a.per_bin, (int)blockIdx.x % a.per_bin);
        return;
    }
    const int first = (int)blockIdx.x - resolvers, stride = (int)gridDim.x - resolvers;
    if (a.resolve) {
        // the hops of half-steps j - 2 and j - 1 into the other plane
        const int64_t m2 = j >= 2 ? min((int64_t)a.n_hops[(j - 2) & 3], a.hop_cap) : 0;
        const int64_t m1 = j >= 1 ? min((int64_t)a.n_hops[(j - 1) & 3], a.hop_cap) : 0;
        auto hop_at = [&](int64_t i) {
            return i < m2 ? a.hops[((j - 2) & 3) * a.hop_cap + i] : a.hops[((j - 1) & 3) * a.hop_cap + i - m2];
        };
        if constexpr (!Dense) {
            if (first < m1 + m2) {
                int64_t *kt = reinterpret_cast<int64_t *>(smem);
                for (int q = tid; q < (a.rail_range + 1) * (a.cutoff + 1); q += kDrawBlock) kt[q] = a.kfix[q];
                __syncthreads();
                for (int64_t i = first; i < m1 + m2; i += stride) add_hop_potential(a, kt, a.phi_other, hop_at(i), w.nbr_off, w.nbr_dist);
            }
        }
        if (first == stride - 1) {
            for (int64_t i = tid; i < m1 + m2; i += kDrawBlock) flip_sites(a.other, a.devs, hop_at(i));
            if (tid == 0) a.n_hops[(j + 1) & 3] = 0u;  // the next launch's list (nobody reads it now)
        }
    }
    if (a.generate) {
        const int64_t n_gen = a.resolve ? a.n + (H == 1 ? 1 : 0) : a.n;
        const int k_gen = a.resolve ? a.k + (H == 1 ? 1 : 0) : a.k;
        generate<1 - H>(a, w, n_gen, k_gen, a.resolve ? j + 1 : j, first, stride);
    }
}

// After the call's last launch J - 1: the plane it read misses the hops of
// half-steps J - 2 and J - 1, the other those of J - 1.
template <bool Dense>
__global__ __launch_bounds__(256) void settle_hops(DrawArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t off[2 * kMaxRailRange + 1], dist[2 * kMaxRailRange + 1];
    int64_t *kt = reinterpret_cast<int64_t *>(smem);
    if constexpr (!Dense) {
        for (int q = threadIdx.x; q < (a.rail_range + 1) * (a.cutoff + 1); q += blockDim.x) kt[q] = a.kfix[q];
        __syncthreads();
    }
    for (int back = 2; back >= 1; --back) {
        const int64_t j = a.launch - back;
        if (j < 0) continue;
        const int64_t m = min((int64_t)a.n_hops[j & 3], a.hop_cap);
        const uint4 *hops = a.hops + (j & 3) * a.hop_cap;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
            flip_sites(const_cast<int8_t *>(a.plane), a.devs, hops[i]);
            if (back == 1) flip_sites(a.other, a.devs, hops[i]);
        }
        if constexpr (!Dense)
            for (int64_t i = blockIdx.x; i < m; i += gridDim.x) {
                add_hop_potential(a, kt, const_cast<int64_t *>(a.phi), hops[i], off, dist);
                if (back == 1) add_hop_potential(a, kt, a.phi_other, hops[i], off, dist);
            }
    }
}

// Stage-0 threshold and bias of every device at steps n_base .. n_base + rows - 1.
__global__ __launch_bounds__(256) void draw_table(uint32_t *thr, double *volt, const DevInfo *devs, int n_devices,
                                                  const double *knot_t, const double *knot_v, int64_t n_base, int rows,
                                                  double dt, double beta, double c0, double alpha, uint32_t *clear) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (clear && i < 4) clear[i] = 0u;
    if (i >= (int64_t)rows * n_devices) return;
    const int d = (int)(i % n_devices);
    const int64_t n = n_base + i / n_devices;
    const DevInfo &dv = devs[d];
    const double V = protocol_voltage(knot_t + d * kMaxKnots, knot_v + d * kMaxKnots, dv.n_knots, (double)(n - dv.n_set) * dt);
    thr[i] = class_threshold(c0, beta, alpha, V, dv.sites, dv.ea_min, dv.ea_step, dv.coul_bound, 0);
    volt[i] = V;
}

const void *draws_fn(bool dense, int h) {
    if (dense) return h == 0 ? (const void *)half_step_draws<true, 0> : (const void *)half_step_draws<true, 1>;
    return h == 0 ? (const void *)half_step_draws<false, 0> : (const void *)half_step_draws<false, 1>;
}

}  // namespace

size_t draws_lds_bytes(bool dense, int rail_range, int nb, int rows, int cutoff) {
    if (dense) return (size_t)(rail_range + 1) * rows * (nb * 32 + 8);
    return sizeof(int64_t) * (size_t)(rail_range + 1) * (cutoff + 1);
}

hipError_t set_draws_lds_limit(bool dense, size_t lds) {
    for (int h = 0; h < 2; ++h) {
        const hipError_t e = hipFuncSetAttribute(draws_fn(dense, h), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return dense ? hipSuccess
                 : hipFuncSetAttribute((const void *)settle_hops<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

hipError_t launch_draws(const DrawArgs &a, bool dense, int h, int grid, size_t lds, hipStream_t st) {
    DrawArgs args = a;
    void *kargs[] = {&args};
    return hipLaunchKernel(draws_fn(dense, h), dim3((unsigned)grid), dim3(kDrawBlock), kargs, lds, st);
}

hipError_t launch_draw_table(uint32_t *thr, double *volt, const DevInfo *devs, int n_devices, const double *knot_t,
                             const double *knot_v, int64_t n_base, int rows, double dt, double beta, double c0,
                             double alpha, uint32_t *clear, hipStream_t st) {
    const int64_t n = std::max<int64_t>((int64_t)rows * n_devices, 4);
    hipLaunchKernelGGL(draw_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, thr, volt, devs, n_devices, knot_t,
                       knot_v, n_base, rows, dt, beta, c0, alpha, clear);
    return hipGetLastError();
}

hipError_t launch_draw_settle(const DrawArgs &a, bool dense, hipStream_t st) {
    if (dense) hipLaunchKernelGGL(settle_hops<true>, dim3(16), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(settle_hops<false>, dim3(256), dim3(256), draws_lds_bytes(false, a.rail_range, 0, 0, a.cutoff), st, a);
    return hipGetLastError();
}

}  // namespace kmc
