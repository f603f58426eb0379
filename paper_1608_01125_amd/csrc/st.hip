// Statistical (ST) regime: photon macro-particles as clouds (the paper's rate picture,
// Sec. 2.2, "statistical regime": collision rate n_I n_II <sigma v> between two clouds).
//
// Each macro-particle i is a uniform cloud filling an axis-aligned box of the binning
// grid's cell size c = (c_x, c_y, c_z), centred on its position, with number density
// n_i = w_i / V, V = c_x c_y c_z. Over step k (mid-step time t_m = k dt + dt/2) the pair
// (i, j) yields
//     Y_ij,k = n_i n_j sigma_BW(s_ij) (1 - u_i.u_j) dt V_ov(t_m),
// V_ov the intersection volume of the two clouds at t_m (product over axes of
// max(0, c_a - |X_i,a - X_j,a|)); (1 - u_i.u_j) c is the rate factor the paper's
// reactivity gives for two photons; sigma = 0 at and below threshold.
// Evaluation order: ((((w_i w_j) / (V V)) sigma) (1 - u_i.u_j)) dt V_ov.
//
// Broad phase: the clouds' boxes, swept from the first to the last mid-step of a window of up to
// 32 steps (rounded outward), in the same hierarchy as the exact path. A wave descends it once for
// eight neighbouring queries, queues the pairs whose boxes meet and sums Y in FP64 over the
// window's steps in which the two clouds overlap (k_st_traverse); sparse clouds that move many
// edges per step descend step by step, a lane per query (k_st_lanes). The sums go to a bin-pair
// table: key = bin(query) * n_target_bins + bin(target), open addressing with linear probing,
// keys claimed by compare-and-swap, values added atomically, neighbouring pairs of one key first
// added up across the wave.
//
// Depletion (the rate equation of Sec. 2.2 with the loss of collision partners): in
// exposure mode the traversal adds, per cloud pair (key = i * n_target + j), the pair's
// exposure S_k = sigma (1 - u_i.u_j) dt V_ov(t_m) / V, evaluated in the order
// (((sigma (1 - u_i.u_j)) dt) V_ov) / V; afterwards every pair gets the closed-form pair
// density at its summed exposure (k tau -> S, k = sigma c (1 - cos phi)): with
// n0 = a + b, a = w_i / V, b = w_j / V,
//     a == b:  (n0/2)^2 S / (1 + (n0/2) S)
//     a != b:  (alpha - 1) alpha n0 (-expm1(X)) / (alpha expm1(X) + 2 alpha - 1),
//              alpha = min(a, b) / n0, X = n0 (2 alpha - 1) S <= 0,
// and the depleted yield V n(S) replaces the pair's exposure in its slot and is added to
// the bin-pair table.
//
// Binning: 3-D cell of the position at the grid time t_bin, log-spaced energy bin,
// polar-angle bin of the direction about the beam axis; values outside a range go to
// its edge bin; bin = (((ix ny + iy) nz + iz) n_e + ie) n_th + ith.
#include <cmath>

#include "tril_internal.h"

namespace tril {

namespace {

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ int cell_of(double v, int n) {
    // v: position in units of the range, scaled by n; floor then clamp (NaN -> 0)
    const double f = floor(v);
    if (!(f >= 0.0)) return 0;
    if (f >= (double)(n - 1)) return n - 1;
    return (int)f;
}

__global__ void __launch_bounds__(256) k_st_bin(BeamDev b, StGridDev g, int32_t *__restrict__ bins,
                                                double *__restrict__ sums) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= b.n) return;
    const double E = b.E[i], w = b.w[i];
    const double px = b.px[i], py = b.py[i], pz = b.pz[i];
    const double x = b.x[i], y = b.y[i], z = b.z[i];
    const bool ok = isfinite(E) && isfinite(w) && isfinite(px) && isfinite(py) && isfinite(pz) &&
                    isfinite(x) && isfinite(y) && isfinite(z) && E > 0.0 && w >= 0.0;
    if (!ok) {
        bins[i] = -1;
        return;
    }
    const double ux = px / E, uy = py / E, uz = pz / E;
    const double X[3] = {x + g.t_bin * ux, y + g.t_bin * uy, z + g.t_bin * uz};
    int ip[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        ip[a] = cell_of(((X[a] - g.lo[a]) / (g.hi[a] - g.lo[a])) * (double)g.n_pos[a], g.n_pos[a]);
    const int ie = cell_of((log(E / g.e_lo) / log(g.e_hi / g.e_lo)) * (double)g.n_e, g.n_e);
    const double uu = (ux * ux + uy * uy) + uz * uz;
    double cth = ((ux * g.axis[0] + uy * g.axis[1]) + uz * g.axis[2]) / sqrt(uu);
    cth = fmin(fmax(cth, -1.0), 1.0);
    const int ith = cell_of((acos(cth) / g.th_max) * (double)g.n_th, g.n_th);
    const int64_t bin =
        ((((int64_t)ip[0] * g.n_pos[1] + ip[1]) * g.n_pos[2] + ip[2]) * g.n_e + ie) * g.n_th + ith;
    bins[i] = (int32_t)bin;
    if (sums) {
        double *s = sums + kStSums * bin;
        atomicAdd(s + 0, w);
        atomicAdd(s + 1, w * E);
        atomicAdd(s + 2, w * ux);
        atomicAdd(s + 3, w * uy);
        atomicAdd(s + 4, w * uz);
        atomicAdd(s + 5, w * X[0]);
        atomicAdd(s + 6, w * X[1]);
        atomicAdd(s + 7, w * X[2]);
    }
}

__global__ void k_st_clear(long long *__restrict__ keys, double *__restrict__ vals, int64_t cap,
                           double *__restrict__ slots) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k < cap) {
        keys[k] = -1ll;
        vals[k] = 0.0;
    }
    if (k < kCounterSlots) slots[k] = 0.0;
}

__device__ __forceinline__ uint64_t mix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

// Linear probing gives up (and flags a full table) after this many slots: a table that
// holds its keys at moderate load never gets near it.
constexpr uint64_t kMaxProbe = 1024;

// Adds v under key. The slots of a probe are read kProbe at a time: a wave waits for the longest
// probe of its 64 lanes, about 20 slots at a load of 0.6, and each slot read by itself is a
// round trip to memory (the cloud traversal took 2.5 ms per exact pass of 2e4 clouds per beam
// that way). The reads (relaxed atomics, whole words beside other lanes' compare-and-swaps) may be
// stale: a slot's key never changes once it is set, so a key that is seen is there, and an empty
// slot is claimed by the compare-and-swap, which sees the truth. So they may come from the
// nearest cache: with reads at the device's scope the training rows take 4.58 ms instead of 4.30,
// the audit of 2e5 clouds 17.6 instead of 16.6.
constexpr int kProbe = 8;
__device__ __forceinline__ void table_add(long long *keys, double *vals, uint64_t mask,
                                          long long key, double v, unsigned int *err) {
    uint64_t h = mix64((uint64_t)key) & mask;
    for (uint64_t probe = 0; probe <= mask && probe < kMaxProbe; probe += kProbe) {
        long long cur[kProbe];
#pragma unroll
        for (int r = 0; r < kProbe; ++r)
            cur[r] = __hip_atomic_load(keys + ((h + r) & mask), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
        __builtin_amdgcn_sched_barrier(0);  // all on their way before the first is looked at
        int at = kProbe;  // first slot that holds the key or is free
#pragma unroll
        for (int r = kProbe - 1; r >= 0; --r)
            if (cur[r] == key || cur[r] == -1ll) at = r;
        while (at < kProbe) {
            const uint64_t slot = (h + at) & mask;
            long long prev = key;
            bool known = false;
#pragma unroll
            for (int r = 0; r < kProbe; ++r) known |= r == at && cur[r] == key;
            if (!known)
                prev = (long long)atomicCAS(reinterpret_cast<unsigned long long *>(keys + slot),
                                            ~0ull, (unsigned long long)key);
            if (prev == -1ll || prev == key) {
                atomicAdd(vals + slot, v);
                return;
            }
            int next = kProbe;  // taken meanwhile: the next candidate of this batch
#pragma unroll
            for (int r = kProbe - 1; r >= 0; --r)
                if (r > at && (cur[r] == key || cur[r] == -1ll)) next = r;
            at = next;
        }
        h = (h + kProbe) & mask;
    }
    atomicOr(err, kErrTableFull);
}

__device__ __forceinline__ bool set_has(const long long *keys, uint64_t mask, long long key) {
    uint64_t h = mix64((uint64_t)key) & mask;
    for (uint64_t probe = 0; probe <= mask && probe < kMaxProbe; ++probe) {
        const long long cur = keys[h];
        if (cur == key) return true;
        if (cur == -1ll) return false;
        h = (h + 1) & mask;
    }
    return false;
}

// One photon as the cloud traversal reads it: its position at t = 0, direction p / E, energy,
// weight and bin, in one 80-B record (the pair test would gather ten scattered words, and
// divide, from the beam's arrays).
__global__ void __launch_bounds__(256) k_st_pack(BeamDev b, const int32_t *__restrict__ bins,
                                                 StRec *__restrict__ rec) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= b.n) return;
    const double E = b.E[i];
    StRec r;
    r.x[0] = b.x[i]; r.x[1] = b.y[i]; r.x[2] = b.z[i];
    r.u[0] = b.px[i] / E; r.u[1] = b.py[i] / E; r.u[2] = b.pz[i] / E;
    r.E = E;
    r.w = b.w[i];
    r.bin = bins[i];
    r.pad = 0;
    rec[i] = r;
}

// What the cloud traversal adds per overlapping pair and step.
enum : int { kStYield = 0, kStOverlap = 1, kStExposure = 2, kStMeet = 3 };

// First and last step (clamped to [k0, k1]) in which two clouds at distance d + t v (per
// axis, t the mid-step time) can overlap along one axis of edge c; sl is far above the FP64
// rounding of the positions, so no overlapping step falls outside. The quotients are those of
// a refined reciprocal: their error, relative 1e-15, is covered by the rounding outward to
// whole steps.
__device__ __forceinline__ void axis_steps(double d, double v, double c, double sl, double t_end,
                                           double inv_dt, double &lo, double &hi) {
    const double h = c + sl;
    if (fabs(v) * t_end <= 0.5 * sl) {  // no motion beyond the slack: all steps or none
        if (fabs(d) > h) lo = INFINITY;
        return;
    }
    double r = __builtin_amdgcn_rcp(v);
    r = r * (2.0 - v * r);
    r = r * (2.0 - v * r);
    const double t1 = (-h - d) * r, t2 = (h - d) * r;
    lo = fmax(lo, floor(fmin(t1, t2) * inv_dt - 0.5));
    hi = fmin(hi, ceil(fmax(t1, t2) * inv_dt - 0.5));
}

// The cross-section as bw_sigma's formula has it, with one reciprocal of s and, well above
// threshold, one logarithm: 2 log1p(b) + ln s = ln((1 + b)^2 s), whose rounded argument costs
// an absolute 3e-16 of a logarithm above 1 (closer to threshold the two logarithms stay).
__device__ __forceinline__ double st_sigma(double s) {
    if (!(s > 2.0)) return bw_sigma(s);
    const double r = 1.0 / s;
    const double b2 = (s - 1.0) * r;
    const double b = sqrt(b2);
    const double L = log(((1.0 + b) * (1.0 + b)) * s);
    return (((0.5 * M_PI) * (kRe * kRe)) * r) * ((3.0 - b2 * b2) * L - (2.0 * b) * (2.0 - b2));
}

// One query photon and leaf whose hulls met: the sum over the steps of [k0, k1] in which the
// two clouds overlap, under its key (-1: nothing). Pair quantities (s, sigma, 1 - u_i.u_j, the weights) do not depend on the step and are
// formed once. cnt: the steps with a positive value.
__device__ __forceinline__ long long st_pair(const StRec &q, int64_t i, int32_t k0, int32_t k1,
                                             const StRec *__restrict__ trec, int64_t j, int64_t n_t,
                                             double dt, double inv_dt, double inv_vv,
                                             const StCell &cell, int mode, int64_t n_t_bins,
                                             const long long *__restrict__ filter, uint64_t fmask,
                                             double &sum, uint32_t &cnt) {
    sum = 0.0;
    cnt = 0;
    const StRec t = trec[j];
    if (t.bin < 0) return -1ll;
    // bin-pair key, or in exposure and swarm mode the cloud pair (caller rows)
    const long long key = mode >= kStExposure ? (long long)i * n_t + j
                                              : (long long)q.bin * n_t_bins + t.bin;
    if (filter != nullptr && !set_has(filter, fmask, key)) return -1ll;
    const double cphi = (q.u[0] * t.u[0] + q.u[1] * t.u[1]) + q.u[2] * t.u[2];
    const double s = ((q.E * t.E) * (1.0 - cphi)) / (2.0 * kMe * kMe);
    if (!(s > 1.0)) return -1ll;
    if (mode == kStMeet) {  // swarms: the swept clouds meet, above threshold
        sum = 1.0;
        cnt = 1;
        return key;
    }
    const double t_end = ((double)k1 + 1.0) * dt;
    double lo = (double)k0, hi = (double)k1;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        axis_steps(q.x[a] - t.x[a], q.u[a] - t.u[a], cell.c[a],
                   1e-11 * (1.0 + fabs(q.x[a]) + fabs(t.x[a]) + t_end), t_end, inv_dt, lo, hi);
    if (!(lo <= hi)) return -1ll;
    const double V = (cell.c[0] * cell.c[1]) * cell.c[2];
    double f = dt;
    if (mode == kStYield)
        f = (((q.w * t.w) * inv_vv) * st_sigma(s)) * (1.0 - cphi) * dt;
    else if (mode == kStExposure)
        f = (st_sigma(s) * (1.0 - cphi)) * dt / V;
    // The overlap along each axis from the pair's distance. The definition takes it from the
    // two positions, whose rounding is below 4e-16 of their magnitude: an overlap of more than
    // 1e-5 of that magnitude differs by less than 1e-10 of itself, a smaller one is formed,
    // and the step decided, as the definition has it.
    const double d0 = q.x[0] - t.x[0], d1 = q.x[1] - t.x[1], d2 = q.x[2] - t.x[2];
    const double v0 = q.u[0] - t.u[0], v1 = q.u[1] - t.u[1], v2 = q.u[2] - t.u[2];
    const double near = 1e-5 * (1.0 + fmax(fmax(fabs(q.x[0]) + fabs(t.x[0]), fabs(q.x[1]) + fabs(t.x[1])),
                                            fabs(q.x[2]) + fabs(t.x[2])) + t_end);
    const int32_t ka = (int32_t)lo, steps = (int32_t)(hi - lo);
    double vol = 0.0;
    for (int32_t r = 0; r <= steps; ++r) {
        const double tm = (double)(ka + r) * dt + 0.5 * dt;
        double ox = cell.c[0] - fabs(fma(tm, v0, d0));
        double oy = cell.c[1] - fabs(fma(tm, v1, d1));
        double oz = cell.c[2] - fabs(fma(tm, v2, d2));
        const double o = fmin(fmin(ox, oy), oz);
        if (fabs(o) <= near) {
            ox = cell.c[0] - fabs((q.x[0] + tm * q.u[0]) - (t.x[0] + tm * t.u[0]));
            oy = cell.c[1] - fabs((q.x[1] + tm * q.u[1]) - (t.x[1] + tm * t.u[1]));
            oz = cell.c[2] - fabs((q.x[2] + tm * q.u[2]) - (t.x[2] + tm * t.u[2]));
            if (!(ox > 0.0 && oy > 0.0 && oz > 0.0)) continue;
        } else if (!(o > 0.0)) {
            continue;
        }
        const double vov = (ox * oy) * oz;
        vol += vov;
        if (f * vov > 0.0) ++cnt;
    }
    sum = f * vol;
    return cnt > 0 ? key : -1ll;
}

__device__ __forceinline__ bool st_overlap(const float q[6], float4 lo, float4 hi) {
    return (q[0] <= hi.x) & (q[3] >= lo.x) & (q[1] <= hi.y) & (q[4] >= lo.y) & (q[2] <= hi.z) &
           (q[5] >= lo.z);
}

constexpr int kStQueries = 8;   // query photons of one wave
constexpr int kStStack = 1024;  // pending nodes of a wave
constexpr int kStDepth = 128;   // deeper than any radix tree over (key, index) pairs
// A wave's hull of more than this many times its widest query box's volume is loose (its nodes
// are tested against the boxes too). Training rows of 2e4 clouds per beam and the audit of 2e5:
// 4.27 and 16.5 ms with the hull alone, 3.95 and 15.9 so (with the boxes' tests in a loop: 4.17 and
// 16.7 always, 4.13 and 16.6 above 4 volumes, 4.05 and 16.3 above 16, 4.04 and 16.3 above 64, 4.09
// and 16.3 above 512).
constexpr float kStLoose = 16.0f;
// Waves of one launch: a grid holds at most 2^32 - 1 threads, and eight per query and window
// pass that from 2^29 queries times windows (the windows of one build times the query beam).
constexpr int64_t kStLaunch = (int64_t)1 << 25;

// Cloud traversal: one wave per kStQueries neighbouring query photons (in Morton order) and
// window of win consecutive steps. The boxes hold the clouds swept over the window, so one
// descent reaches every pair that overlaps in any of its steps, and the pair's quantities are
// formed and its key added once per window instead of once per step: two head-on clouds of
// 1.25 um overlap for 12 steps of 0.1 um/c.
//   * Clouds are larger than the photons' spacing (a query meets tens of targets per window),
//     so its neighbours reach nearly the same leaves: the wave descends once, with the hull of
//     its queries' boxes, 64 pending nodes at a time (lane = node; one load per internal node,
//     both children tested from it). Where the boxes fill little of their hull (clouds smaller
//     than their spacing, the outskirts of a beam, where neighbours along the curve are far
//     apart), a node that the hull meets must meet one of the boxes as well: one wave that
//     walks through most of the tree holds up its launch (3e4 sparse clouds per beam, a step
//     each in 40 launches, 47 ms with the hull alone, 9.2 so; one step of 2e4 dense ones in a
//     call 1.03 and 0.42 ms).
//   * A leaf that passes is tested against the queries' own boxes, eight leaves at a time; the
//     pairs that meet are queued in LDS and evaluated 64 at a time, so that every lane of the
//     long FP64 pair code works, however unequal the queries are.
//   * Neighbouring pairs of one bin pair are added up across the wave before the table.
// Bound by the pair code's FP64 chain and the table's atomics, and by the heaviest waves: the
// queries of a wave are few so that their hull stays tight and no wave holds too many of the
// dense core (training rows of 2e4 clouds per beam: 10.7 ms with 32 queries per wave, 9.5 with
// 16, 8.9 with 8 or 4, at windows of 16 steps). The exact pass of that instance took 20.7 ms with
// a descent and an evaluation per step, 2.4 ms with one lane per query and window of 16 steps
// (each with a descent of its own), 1.8 ms with 16 queries per wave. Four waves per SIMD (128
// VGPRs, some of the pair code's constants spilled) against two unspilled: 9.5 against 9.8 ms
// for the rows; five: 11.0 ms. (The rows' times include about 4.5 ms of allocations and row forming
// that have gone since; they take 3.95 ms now.)
__global__ void __launch_bounds__(64, 4) k_st_traverse(
    const Node *__restrict__ nodes, int32_t n_int, const PBox *__restrict__ root_box,
    const PBox *__restrict__ qbox, const uint32_t *__restrict__ qorder, int64_t nq, int64_t groups,
    int64_t first, const int32_t *__restrict__ inst_root, int64_t n_t, const StRec *__restrict__ qrec,
    const StRec *__restrict__ trec, int64_t n_t_bins, double dt, int32_t win, int32_t k_begin,
    int32_t k_last, StCell cell, int mode, const long long *__restrict__ filter, uint64_t fmask,
    long long *keys, double *vals, uint64_t mask, double *__restrict__ slots, DevCounters *c) {
    __shared__ int32_t s_node[kStStack];
    __shared__ int32_t s_leaf[192];          // queued pairs: target row
    __shared__ uint8_t s_owner[192];         //               and query lane
    __shared__ int32_t s_row[kStQueries];
    __shared__ float4 s_box[kStQueries][2];
    const int lane = threadIdx.x, ql = lane & (kStQueries - 1), grp = lane / kStQueries;
    const int64_t wave = first + blockIdx.x;
    const int64_t so = wave / groups;  // window of the hierarchy
    const int64_t qi = (wave - so * groups) * kStQueries + ql;
    int32_t root = -1, tag = -1;
    float qb[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (qi < nq) {
        const int32_t row = (int32_t)qorder[qi];
        const float4 *bp = reinterpret_cast<const float4 *>(qbox + so * nq + row);
        const float4 a = bp[0], b = bp[1];
        qb[0] = a.x; qb[1] = a.y; qb[2] = a.z;
        qb[3] = b.x; qb[4] = b.y; qb[5] = b.z;
        tag = __float_as_int(a.w);
        if (tag >= 0 && qrec[row].bin >= 0) root = inst_root[tag];
        if (grp == 0) s_row[ql] = row;
    }
    // the steps of this (aligned) window
    const int64_t ws = ((int64_t)c->step + so) * win;
    const int32_t k0 = (int32_t)max((int64_t)k_begin, ws);
    const int32_t k1 = (int32_t)min((int64_t)k_last, ws + win - 1);
    const double V = (cell.c[0] * cell.c[1]) * cell.c[2];
    const double inv_dt = 1.0 / dt, inv_vv = 1.0 / (V * V);
    double total = 0.0;
    uint32_t visits = 0, n_pairs = 0;
    int queued = 0;  // uniform over the wave
    // Evaluates the last `cnt` queued pairs (at most 64).
    auto evaluate = [&](int cnt) {
        __syncthreads();
        const int x = queued - cnt + lane;
        long long key = -1ll;
        double sum = 0.0;
        if (lane < cnt) {
            const int32_t row = s_row[s_owner[x]];
            uint32_t n;
            key = st_pair(qrec[row], row, k0, k1, trec, s_leaf[x], n_t, dt, inv_dt, inv_vv, cell,
                          mode, n_t_bins, filter, fmask, sum, n);
            n_pairs += n;
            total += sum;
        }
        queued -= cnt;
        // a run of equal keys is added up into its first lane
        const long long prev = __shfl_up(key, 1);
        const bool head = lane == 0 || prev != key;
        unsigned long long heads = __ballot(head);
        if (heads != ~0ull) {
            heads = (heads >> lane) >> 1;
            const int last = heads ? lane + (int)__ffsll(heads) - 1 : 63;  // of this run
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double v = __shfl_down(sum, off);
                if (lane + off <= last) sum += v;
            }
        }
        if (head && key >= 0) table_add(keys, vals, mask, key, sum, &c->err);
        __syncthreads();
    };
    const unsigned long long below = (1ull << lane) - 1ull;
    auto queue_pair = [&](bool meets, int32_t leaf_row) {
        const unsigned long long b = __ballot(meets);
        if (meets) {
            const int at = queued + (int)__popcll(b & below);
            s_leaf[at] = leaf_row;
            s_owner[at] = (uint8_t)ql;
        }
        queued += (int)__popcll(b);
    };
    // one descent per hierarchy that the queries belong to (one per instance; nearly always
    // one for the wave)
    for (unsigned long long todo = __ballot(root != -1); todo != 0ull;) {
        const int32_t r0 = __shfl(root, (int)__ffsll(todo) - 1);
        const bool mine = root == r0;
        todo &= ~__ballot(mine);
        if (r0 <= -2) {  // an instance of one row: its root is that leaf
            bool meets = false;
            if (mine && grp == 0) {
                const float4 *lp = reinterpret_cast<const float4 *>(root_box + tag);
                ++visits;
                meets = st_overlap(qb, lp[0], lp[1]);
            }
            // (at most kStQueries of these in all: one per query)
            queue_pair(meets, (int32_t)(link_elem(r0) - so * n_t));
            continue;
        }
        float hull[6];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            hull[a] = mine ? qb[a] : INFINITY;
            hull[3 + a] = mine ? qb[3 + a] : -INFINITY;
#pragma unroll
            for (int off = kStQueries / 2; off >= 1; off >>= 1) {
                hull[a] = fminf(hull[a], __shfl_xor(hull[a], off));
                hull[3 + a] = fmaxf(hull[3 + a], __shfl_xor(hull[3 + a], off));
            }
        }
        // loose: the hull is mostly empty space between the queries' boxes
        float full = 1.0f, own = 1.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float w = mine ? qb[3 + a] - qb[a] : 0.0f;
#pragma unroll
            for (int off = kStQueries / 2; off >= 1; off >>= 1) w = fmaxf(w, __shfl_xor(w, off));
            full *= hull[3 + a] - hull[a];
            own *= w;
        }
        const bool loose = !(full <= kStLoose * own);
        if (grp == 0) {
            s_box[ql][0] = mine ? make_float4(qb[0], qb[1], qb[2], 0.0f)
                                : make_float4(INFINITY, INFINITY, INFINITY, 0.0f);
            s_box[ql][1] = mine ? make_float4(qb[3], qb[4], qb[5], 0.0f)
                                : make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
        }
        if (lane == 0) s_node[0] = r0;
        int top = 1;  // uniform over the wave
        uint32_t seen = 0;
        while (top > 0) {
            __syncthreads();
            // 64 nodes at a time add at most 64 to the stack per level; when it is nearly full,
            // one at a time adds one per level
            const int take = top > kStStack - 128 - kStDepth ? 1 : min(top, 64);
            top -= take;
            seen += (uint32_t)take;
            if (seen > (uint32_t)n_int + 2u || top > kStStack - 130) {
                if (lane == 0) atomicOr(&c->err, kErrSpin);
                break;
            }
            float4 l0{}, l1{}, r0v{}, r1{};
            int32_t lc = -1, rc = -1;
            bool ovl = false, ovr = false;
            if (lane < take) {
                const float4 *np = reinterpret_cast<const float4 *>(nodes + s_node[top + lane]);
                l0 = np[0]; l1 = np[1]; r0v = np[2]; r1 = np[3];
                ++visits;
                lc = __float_as_int(l0.w);
                rc = __float_as_int(r0v.w);
                ovl = st_overlap(hull, l0, l1);
                ovr = st_overlap(hull, r0v, r1);
                if (loose && (ovl || ovr)) {
                    bool al = false, ar = false;
#pragma unroll  // (in a loop, the boxes' reads wait for one another: rows 4.05 ms, audit 16.2)
                    for (int j = 0; j < kStQueries; ++j) {
                        const float4 a = s_box[j][0], b = s_box[j][1];
                        const float q[6] = {a.x, a.y, a.z, b.x, b.y, b.z};
                        al |= st_overlap(q, l0, l1);
                        ar |= st_overlap(q, r0v, r1);
                    }
                    ovl &= al;
                    ovr &= ar;
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int side = 0; side < 2; ++side) {
                const int32_t ch = side ? rc : lc;
                const bool ov = side ? ovr : ovl;
                const unsigned long long in = __ballot(ov && ch >= 0);
                if (ov && ch >= 0) s_node[top + (int)__popcll(in & below)] = ch;
                top += (int)__popcll(in);
                // leaves: each group of kStQueries lanes takes one
                for (unsigned long long lv = __ballot(ov && ch < 0); lv != 0ull;) {
                    int src = -1;
#pragma unroll
                    for (int g = 0; g < 64 / kStQueries; ++g) {
                        const int at = (int)__ffsll(lv) - 1;  // -1: none left
                        if (g == grp) src = at;
                        lv &= lv - 1ull;
                    }
                    const int from = src < 0 ? lane : src;
                    float4 lo, hi;
                    lo.x = __shfl(side ? r0v.x : l0.x, from);
                    lo.y = __shfl(side ? r0v.y : l0.y, from);
                    lo.z = __shfl(side ? r0v.z : l0.z, from);
                    hi.x = __shfl(side ? r1.x : l1.x, from);
                    hi.y = __shfl(side ? r1.y : l1.y, from);
                    hi.z = __shfl(side ? r1.z : l1.z, from);
                    const int32_t link = __shfl(ch, from);
                    queue_pair(src >= 0 && mine && st_overlap(qb, lo, hi),
                               (int32_t)(link_elem(link) - so * n_t));
                    if (queued >= 64) evaluate(64);
                }
            }
        }
        __syncthreads();
    }
    while (queued > 0) evaluate(min(queued, 64));
    // per-wave sums into spread slots
    unsigned long long v = visits, np_ = n_pairs;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        v += __shfl_xor(v, off);
        np_ += __shfl_xor(np_, off);
        total += __shfl_xor(total, off);
    }
    if (lane == 0) {
        const int slot = blockIdx.x & (kCounterSlots - 1);
        if (v) atomicAdd(&c->visits[slot], v);
        if (np_) atomicAdd(&c->st_pairs[slot], np_);
        if (total != 0.0) atomicAdd(&slots[slot], total);
    }
}

// The cloud traversal of windows of one step by a lane per query and step, which descends by
// itself, one load per overlapped internal node, both children tested from it, pending right
// children on the lane's stack, and evaluates its leaves' pairs one after another. It is the
// better one where most descents end after a few nodes without a leaf: there is little that
// neighbours could share, and a wave per kStQueries queries (k_st_traverse) pays its latency for
// eight lanes' work. Swarms (their table's values count the steps in which two clouds meet): 3e4
// macro-particles per beam over 400 steps 7.7 ms by waves, 0.8 ms so. Yields: 1e5 clouds of 0.02
// um per beam at 90 degrees, steps of 50 edges, 3.4 ms by waves (1.8 in windows of 4 steps), 0.9
// ms so. Where all those waves are on the chip at once (kMeetWaves), their latency is the whole
// time, and a lane that adds up its pairs one after another the slower: 24 macro-particles that
// all meet over 10 steps 22 us by waves, 80 by lanes.
constexpr int64_t kMeetWaves = 4096;  // 256 CUs of 16
template <bool kMeets>
__global__ void __launch_bounds__(256) k_st_lanes(
    const Node *__restrict__ nodes, int32_t n_int, const PBox *__restrict__ root_box,
    const PBox *__restrict__ qbox, const uint32_t *__restrict__ qorder, int64_t nq, int64_t m,
    const int32_t *__restrict__ inst_root, int64_t n_t, const StRec *__restrict__ qrec,
    const StRec *__restrict__ trec, int64_t n_t_bins, double dt, StCell cell, int mode,
    const long long *__restrict__ filter, uint64_t fmask, long long *keys, double *vals,
    uint64_t mask, double *__restrict__ slots, DevCounters *c) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t so = e / nq;  // step of the launch
    int64_t i = 0;
    int32_t node = -1, tag = -1;
    float qb[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (so < m) {
        i = qorder[e - so * nq];
        const float4 *bp = reinterpret_cast<const float4 *>(qbox + so * nq + i);
        const float4 a = bp[0], b = bp[1];
        qb[0] = a.x; qb[1] = a.y; qb[2] = a.z;
        qb[3] = b.x; qb[4] = b.y; qb[5] = b.z;
        tag = __float_as_int(a.w);
        if (tag >= 0 && qrec[i].bin >= 0) node = inst_root[tag];
    }
    const int32_t k = (int32_t)(c->step + so);
    const double V = (cell.c[0] * cell.c[1]) * cell.c[2];
    const double inv_dt = 1.0 / dt, inv_vv = 1.0 / (V * V);
    double total = 0.0;
    uint32_t visits = 0, n_pairs = 0;
    auto leaf = [&](int32_t link) {
        double sum;
        uint32_t n;
        const long long key =
            st_pair(qrec[i], i, k, k, trec, link_elem(link) - so * n_t, n_t, dt, inv_dt, inv_vv, cell,
                    kMeets ? (int)kStMeet : mode, n_t_bins, kMeets ? nullptr : filter, fmask, sum, n);
        n_pairs += n;
        total += sum;
        if (key >= 0) table_add(keys, vals, mask, key, sum, &c->err);
    };
    if (node <= -2) {  // an instance of one row: its root is that leaf
        const float4 *lp = reinterpret_cast<const float4 *>(root_box + tag);
        ++visits;
        if (st_overlap(qb, lp[0], lp[1])) leaf(node);
        node = -1;
    }
    int32_t stack[kStDepth];
    int32_t depth = 0;
    const uint32_t max_visits = (uint32_t)n_int + 2u;
    while (node >= 0) {
        if (visits > max_visits) {
            atomicOr(&c->err, kErrSpin);
            break;
        }
        const float4 *np = reinterpret_cast<const float4 *>(nodes + node);
        const float4 l0 = np[0], l1 = np[1], r0 = np[2], r1 = np[3];
        ++visits;
        const int32_t lc = __float_as_int(l0.w), rc = __float_as_int(r0.w);
        const bool ovl = st_overlap(qb, l0, l1), ovr = st_overlap(qb, r0, r1);
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            const int32_t ch = side ? rc : lc;
            if ((side ? ovr : ovl) && ch < 0) leaf(ch);
        }
        const bool gol = ovl && lc >= 0, gor = ovr && rc >= 0;
        if (gol) {
            if (gor) {
                if (depth >= kStDepth) {
                    atomicOr(&c->err, kErrSpin);
                    break;
                }
                stack[depth++] = rc;
            }
            node = lc;
        } else if (gor) {
            node = rc;
        } else {
            node = depth > 0 ? stack[--depth] : -1;
        }
    }
    // per-wave sums into spread slots
    unsigned long long v = visits, np_ = n_pairs;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        v += __shfl_xor(v, off);
        np_ += __shfl_xor(np_, off);
        total += __shfl_xor(total, off);
    }
    if ((threadIdx.x & 63) == 0) {
        const int slot = blockIdx.x & (kCounterSlots - 1);
        if (v) atomicAdd(&c->visits[slot], v);
        if (np_) atomicAdd(&c->st_pairs[slot], np_);
        if (total != 0.0) atomicAdd(&slots[slot], total);
    }
}

// Closed-form pair density of two clouds of densities a, b at exposure S (file comment).
__device__ __forceinline__ double depleted_density(double a, double b, double S) {
    if (!(a > 0.0) || !(b > 0.0) || !(S > 0.0)) return 0.0;
    const double n0 = a + b;
    if (a == b) {
        const double h = n0 / 2.0;
        return ((h * h) * S) / (1.0 + h * S);
    }
    const double alpha = fmin(a, b) / n0;
    const double X = (n0 * (2.0 * alpha - 1.0)) * S;
    const double E = expm1(X);
    return ((((alpha - 1.0) * alpha) * n0) * (-E)) / (alpha * E + (2.0 * alpha - 1.0));
}

// Every occupied slot of the cloud-pair table: exposure -> depleted yield (in place), added
// to the bin-pair table; per-wave totals into the slots.
__global__ void __launch_bounds__(256) k_st_deplete(long long *__restrict__ pkeys,
                                                    double *__restrict__ pvals, int64_t pcap,
                                                    BeamDev q, BeamDev t,
                                                    const int32_t *__restrict__ q_bins,
                                                    const int32_t *__restrict__ t_bins,
                                                    int64_t n_t_bins, StCell cell,
                                                    long long *keys, double *vals, uint64_t mask,
                                                    double *__restrict__ slots, DevCounters *c) {
    const double V = (cell.c[0] * cell.c[1]) * cell.c[2];
    double tot = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t h = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; h < pcap; h += stride) {
        const long long key = pkeys[h];
        if (key < 0) continue;
        const int64_t i = key / t.n, j = key - i * t.n;
        const double Y = V * depleted_density(q.w[i] / V, t.w[j] / V, pvals[h]);
        pvals[h] = Y;
        tot += Y;
        table_add(keys, vals, mask, (long long)q_bins[i] * n_t_bins + t_bins[j], Y, &c->err);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) tot += __shfl_xor(tot, off);
    if ((threadIdx.x & 63) == 0 && tot != 0.0) atomicAdd(&slots[blockIdx.x & (kCounterSlots - 1)], tot);
}

// ---- IP regime: swarms of real photons -------------------------------------------------
// A macro-particle of weight w is floor(w + 1/2) real photons with its momentum, at the
// centres of the cells of a level-L octree over its cloud box (8^L >= n, L smallest): real
// photon k takes, at level l, the octant given by base-8 digit l of k (lowest digit = top
// level; digit bits 2, 1, 0 = upper half along x, y, z), which spreads any n evenly.
// The octree needs no storage: the node at level l whose octants are the low l digits of
// `base` holds the real photons base, base + 8^l, base + 2 8^l, ... below n.
// Real photons p (of the query's swarm) and q (of the target's) collide when their
// time-synchronous distance over the run window [T0, T0 + Tw] comes within r,
// r^2 = sigma(s) / pi (weight 1 each), as the narrow phase evaluates it in FP64 over a step
// window (swarm_hit).
//
// A wave takes the 64 real photons p of one block (an octree node two levels above the
// photons), one per lane, and descends the target's octree with the block's hull, 64 nodes at
// a time. All pairs of a swarm pair share one relative velocity v, so as long as no pair's
// closest approach is cut off by the window, distances are those of the two coordinates across
// v: node against block, a pair of rectangles.
//   * No pair can collide: the node is dropped.
//   * Every pair collides: the node's photons are counted without being visited.
//   * Otherwise its children follow; a node of at most 64 photons is tested pair by pair, two
//     subtractions, a product and a fused multiply-add each.
// Positions are of magnitude M (micrometres) and r of 1e-9 um, so the rounding of the
// definition's own positions (below 1e-15 M) is what a decision has to clear: pairs within
// `band` of r^2, and pairs whose approach the window cuts off, take swarm_hit itself. The
// counts are therefore the definition's.
// 24 x 24 swarms of 4096 real photons: 2.2 to 2.3 ms per call, pair finding included, against
// 184 ms with one lane per photon walking the octree down to every colliding photon, six FP64
// divisions per node. Bound by FP64 issue in the pair loop (5.2 ms while each photon pair
// branched on the band by itself); four waves per SIMD (128 VGPRs) against two unspilled: 5.2
// against 7.7 ms then; five and six 2.6 and 4.8 ms where four took 2.45.
constexpr int64_t kSwarmMax = (int64_t)1 << 30;  // real photons per macro-particle

__device__ __forceinline__ int swarm_level(int64_t n) {
    int L = 0;
    int64_t cells = 1;
    while (cells < n) {
        cells *= 8;
        ++L;
    }
    return L;
}

// Integer cell coordinates, at level `lvl`, of the octants in the low lvl digits of k.
__device__ __forceinline__ void swarm_cell(int64_t k, int lvl, int64_t c[3]) {
    c[0] = c[1] = c[2] = 0;
    for (int l = 0; l < lvl; ++l) {
        const int d = (int)((k >> (3 * l)) & 7);
        c[0] = 2 * c[0] + ((d >> 2) & 1);
        c[1] = 2 * c[1] + ((d >> 1) & 1);
        c[2] = 2 * c[2] + (d & 1);
    }
}

__device__ __forceinline__ void swarm_offset(int64_t k, int L, const StCell &cell, double o[3]) {
    int64_t c[3];
    swarm_cell(k, L, c);
    const double cells = (double)((int64_t)1 << L);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double h = cell.c[a] / cells;
        o[a] = ((double)c[a] + 0.5) * h - 0.5 * cell.c[a];
    }
}

// Orders the wave's LDS accesses before it with those after it, between its lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The definition: closest approach of two real photons at distance d at T0 (each component the
// difference of the two FP64 positions), relative velocity v, over [0, Tw].
__device__ __forceinline__ bool swarm_hit(double dx, double dy, double dz, const double v[3],
                                          double Tw, double r2) {
    const double vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    const double dv = (dx * v[0] + dy * v[1]) + dz * v[2];
    double tau = -dv / vv;
    if (!(tau > 0.0)) tau = 0.0;
    if (tau > Tw) tau = Tw;
    const double ex = dx + tau * v[0], ey = dy + tau * v[1], ez = dz + tau * v[2];
    return (ex * ex + ey * ey) + ez * ez <= r2;
}

// Slots of (a piece of) the pair table that hold a pair: their count starts at zero, and their
// numbers go to list, in no order: from its front where the query's swarm has several blocks of
// 64 photons, from its end where it has one (listed: how many of each). Workgroups that looked for
// the pairs themselves read the slots one after another, 5.5 ms for 2^22 slots with few pairs.
__global__ void __launch_bounds__(256) k_swarm_list(const long long *__restrict__ pkeys,
                                                    double *__restrict__ pvals, int64_t pcap,
                                                    const double *__restrict__ q_w, int64_t n_t,
                                                    uint32_t *__restrict__ list, uint32_t *listed) {
    __shared__ uint32_t s_n[2][4], s_base[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const long long key = k < pcap ? pkeys[k] : -1ll;
    bool one = false, several = false;
    if (key >= 0) {
        pvals[k] = 0.0;
        several = (int64_t)floor(q_w[key / n_t] + 0.5) > 64;
        one = !several;
    }
    const unsigned long long b[2] = {__ballot(several), __ballot(one)};
    if (lane < 2) s_n[lane][wave] = (uint32_t)__popcll(lane ? b[1] : b[0]);
    __syncthreads();
    if (threadIdx.x < 2) {
        const uint32_t *c = s_n[threadIdx.x], all = (c[0] + c[1]) + (c[2] + c[3]);
        s_base[threadIdx.x] = all ? atomicAdd(listed + threadIdx.x, all) : 0u;
    }
    __syncthreads();
    if (key < 0) return;
    const int which = one ? 1 : 0;
    int64_t at = (int64_t)s_base[which] + __popcll((one ? b[1] : b[0]) & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) at += s_n[which][w];
    list[one ? pcap - 1 - at : at] = (uint32_t)k;
}

constexpr int kSwarmWaves = 4;
constexpr int kSwarmSplit = 4;  // workgroups that share one pair's blocks
// pending nodes of a wave: eight at a time leave room for 56 more per level, at most eight
// levels above the blocks of 64
constexpr int kSwarmStack = 576;

__global__ void __launch_bounds__(64 * kSwarmWaves, 4) k_swarm(
    const long long *__restrict__ pkeys, double *__restrict__ pvals, int64_t pcap,
    const uint32_t *__restrict__ list, const uint32_t *__restrict__ listed, BeamDev q, BeamDev t,
    StCell cell, double T0, double Tw, DevCounters *c) {
    __shared__ uint2 s_node[kSwarmWaves][kSwarmStack];  // (octant digits, level)
    __shared__ double2 s_ab[kSwarmWaves][64];
    __shared__ unsigned long long s_part[kSwarmWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t n_multi = listed[0], n = blockIdx.y == 0 ? n_multi + listed[1] : n_multi;
    for (int64_t at = blockIdx.x; at < n; at += gridDim.x) {
        const int64_t slot = list[at < n_multi ? at : pcap - 1 - (at - n_multi)];
        const long long key = pkeys[slot];
        const int64_t i = key / t.n, j = key - i * t.n;
        const int64_t ni = (int64_t)floor(q.w[i] + 0.5), nj = (int64_t)floor(t.w[j] + 0.5);
        const double Ei = q.E[i], Ej = t.E[j];
        const double ui[3] = {q.px[i] / Ei, q.py[i] / Ei, q.pz[i] / Ei};
        const double uj[3] = {t.px[j] / Ej, t.py[j] / Ej, t.pz[j] / Ej};
        const double cphi = (ui[0] * uj[0] + ui[1] * uj[1]) + ui[2] * uj[2];
        const double s = ((Ei * Ej) * (1.0 - cphi)) / (2.0 * kMe * kMe);
        const bool big = ni > kSwarmMax || nj > kSwarmMax;
        if (big && threadIdx.x == 0) atomicOr(&c->err, kErrData);
        unsigned long long cnt = 0;  // of this lane
        if (s > 1.0 && ni > 0 && nj > 0 && !big) {
            const double r2 = bw_sigma(s) / M_PI, r = sqrt(r2);
            const int Li = swarm_level(ni), Lj = swarm_level(nj);
            const int Bi = max(Li - 2, 0), Bj = max(Lj - 2, 0);  // level of the blocks of 64
            const double v[3] = {ui[0] - uj[0], ui[1] - uj[1], ui[2] - uj[2]};
            const double xi[3] = {q.x[i], q.y[i], q.z[i]}, xj[3] = {t.x[j], t.y[j], t.z[j]};
            // distance of the clouds' centres at T0, and the frame across v
            double D[3], M = 1.0 + 2.0 * Tw;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                D[a] = (xi[a] + T0 * ui[a]) - (xj[a] + T0 * uj[a]);
                M += fabs(xi[a]) + fabs(xj[a]) + 2.0 * T0 + cell.c[a];
            }
            const double vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
            // two photons of one direction can be above threshold (|p| and E agree to 1e-12): no
            // motion, every approach is cut off, and any axis will do
            const bool still = !(vv > 1e-200);
            const double vn = sqrt(vv), iv = still ? 0.0 : 1.0 / vn;
            const double w[3] = {v[0] * iv, v[1] * iv, still ? 1.0 : v[2] * iv};
            // e1 across v and the axis v leans on least, e2 across both
            const double aw[3] = {fabs(w[0]), fabs(w[1]), fabs(w[2])};
            const int ax = aw[0] <= aw[1] ? (aw[0] <= aw[2] ? 0 : 2) : (aw[1] <= aw[2] ? 1 : 2);
            const double m[3] = {ax == 0 ? 1.0 : 0.0, ax == 1 ? 1.0 : 0.0, ax == 2 ? 1.0 : 0.0};
            double e1[3] = {w[1] * m[2] - w[2] * m[1], w[2] * m[0] - w[0] * m[2],
                            w[0] * m[1] - w[1] * m[0]};
            const double n1 = 1.0 / sqrt((e1[0] * e1[0] + e1[1] * e1[1]) + e1[2] * e1[2]);
#pragma unroll
            for (int a = 0; a < 3; ++a) e1[a] *= n1;
            const double e2[3] = {w[1] * e1[2] - w[2] * e1[1], w[2] * e1[0] - w[0] * e1[2],
                                  w[0] * e1[1] - w[1] * e1[0]};
            auto dot = [](const double x[3], const double y[3]) {
                return (x[0] * y[0] + x[1] * y[1]) + x[2] * y[2];
            };
            // half extents of a whole cloud in the frame (a node's: divided by its cells)
            double ha = 0.0, hb = 0.0, hw = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                ha += 0.5 * cell.c[a] * fabs(e1[a]);
                hb += 0.5 * cell.c[a] * fabs(e2[a]);
                hw += 0.5 * cell.c[a] * aw[a];
            }
            const double slack = 2e-14 * M, band = 4.0 * r * slack + 1e-12 * r2 + slack * slack;
            const double Da = dot(e1, D), Db = dot(e2, D), Dw = dot(w, D);
            const double fi = 1.0 / (double)((int64_t)1 << Bi);
            const int64_t n_blocks = (int64_t)1 << (3 * Bi);
            for (int64_t pb = blockIdx.y * kSwarmWaves + wave; pb < n_blocks && pb < ni;
                 pb += (int64_t)gridDim.y * kSwarmWaves) {
                // this lane's photon, and the hull of the block's
                const int64_t p = pb + ((int64_t)lane << (3 * Bi));
                const bool has = p < ni;
                const unsigned long long np = (unsigned long long)__popcll(__ballot(has));
                double op[3] = {0.0, 0.0, 0.0};
                if (has) swarm_offset(p, Li, cell, op);
                const double pa = Da + dot(e1, op), pc = Db + dot(e2, op);
                int64_t cc[3];
                swarm_cell(pb, Bi, cc);
                const double oc[3] = {(((double)cc[0] + 0.5) * fi - 0.5) * cell.c[0],
                                      (((double)cc[1] + 0.5) * fi - 0.5) * cell.c[1],
                                      (((double)cc[2] + 0.5) * fi - 0.5) * cell.c[2]};
                const double Ba = Da + dot(e1, oc), Bb = Db + dot(e2, oc), Bw = Dw + dot(w, oc);
                int top = 0;
                bool first = true;
                while (first || top > 0) {
                    // candidates: the root, or the children of the last eight pending nodes
                    uint32_t base = 0;
                    int lvl = 0;
                    bool cand = false;
                    if (first) {
                        cand = lane == 0;
                    } else {
                        const int take = min(top, 8), at = lane >> 3;
                        if (at < take) {
                            const uint2 nd = s_node[wave][top - take + at];
                            const uint64_t ch =
                                (uint64_t)nd.x + ((uint64_t)(lane & 7) << (3 * nd.y));
                            cand = ch < (uint64_t)nj;
                            base = (uint32_t)ch;
                            lvl = (int)nd.y + 1;
                        }
                        top -= take;
                        wave_lds_sync();  // the nodes are read before their places are filled
                    }
                    first = false;
                    bool mixed = false, cut = false;
                    if (cand) {
                        int64_t qc[3];
                        swarm_cell((int64_t)base, lvl, qc);
                        const double f = 1.0 / (double)((int64_t)1 << lvl);
                        const double oq[3] = {(((double)qc[0] + 0.5) * f - 0.5) * cell.c[0],
                                              (((double)qc[1] + 0.5) * f - 0.5) * cell.c[1],
                                              (((double)qc[2] + 0.5) * f - 0.5) * cell.c[2]};
                        const double h = fi + f;
                        const double da = fabs(Ba - dot(e1, oq)), db = fabs(Bb - dot(e2, oq));
                        const double na = fmax(da - ha * h, 0.0), nb = fmax(db - hb * h, 0.0);
                        const double xa = da + ha * h, xb = db + hb * h;
                        // distances along v at T0 that the pairs have to go: [-lo, -hi]
                        const double along = -(Bw - dot(w, oq)), hl = hw * h + slack;
                        const double lo = along - hl, hi = along + hl, end = vn * Tw;
                        const double late = fmax(fmax(-hi, lo - end), 0.0);
                        const double far = r + slack, in = r - slack;
                        cut = lo < 0.0 || hi > end;
                        const bool miss = (na * na + nb * nb) + late * late > far * far;
                        const bool all = !cut && in > 0.0 && xa * xa + xb * xb < in * in;
                        if (all)
                            cnt += np * (unsigned long long)((((uint64_t)nj - 1 - base) >> (3 * lvl)) + 1);
                        mixed = !miss && !all;
                    }
                    const unsigned long long down = __ballot(mixed && lvl < Bj);
                    if (mixed && lvl < Bj)
                        s_node[wave][top + (int)__popcll(down & below)] =
                            uint2{base, (uint32_t)lvl};
                    top += (int)__popcll(down);
                    wave_lds_sync();
                    for (unsigned long long lv = __ballot(mixed && lvl >= Bj); lv != 0ull;
                         lv &= lv - 1ull) {
                        const int src = (int)__ffsll(lv) - 1;
                        const uint32_t qb = (uint32_t)__shfl((int)base, src);
                        const bool cutoff = __shfl((int)cut, src) != 0;
                        const int64_t qk = (int64_t)qb + ((int64_t)lane << (3 * Bj));
                        const int nq = (int)min((int64_t)64, ((nj - 1 - (int64_t)qb) >> (3 * Bj)) + 1);
                        double oq[3] = {0.0, 0.0, 0.0};
                        if (lane < nq) swarm_offset(qk, Lj, cell, oq);
                        wave_lds_sync();
                        s_ab[wave][lane] = double2{dot(e1, oq), dot(e2, oq)};
                        wave_lds_sync();
                        // eight photons at a time (the list is padded to 64)
                        uint32_t hits = 0;
                        for (int k0 = 0; k0 < nq; k0 += 8) {
                            uint32_t hit = 0, near = 0;
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const double2 ab = s_ab[wave][k0 + e];
                                const double da = pa - ab.x, db = pc - ab.y;
                                const double d2 = fma(da, da, fma(db, db, -r2));
                                hit |= (d2 <= 0.0 ? 1u : 0u) << e;
                                near |= (fabs(d2) <= band ? 1u : 0u) << e;
                            }
                            const uint32_t used = nq - k0 >= 8 ? 0xffu : (1u << (nq - k0)) - 1u;
                            // near r, or cut off by the window: the definition
                            if (cutoff) near |= hit;
                            hit &= used & ~near;
                            for (near = has ? near & used : 0u; near != 0u; near &= near - 1u) {
                                const int e = __ffs((int)near) - 1;
                                double ok[3], d[3];
                                swarm_offset((int64_t)qb + ((int64_t)(k0 + e) << (3 * Bj)), Lj, cell,
                                             ok);
#pragma unroll
                                for (int a = 0; a < 3; ++a)
                                    d[a] = ((xi[a] + op[a]) + T0 * ui[a]) -
                                           ((xj[a] + ok[a]) + T0 * uj[a]);
                                if (swarm_hit(d[0], d[1], d[2], v, Tw, r2)) hit |= 1u << e;
                            }
                            hits += (uint32_t)__popc(hit);
                        }
                        if (has) cnt += hits;
                    }
                }
            }
        }
        // workgroup sum of the lanes' counts
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off);
        if (lane == 0) s_part[wave] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long tot = 0;
            for (int k = 0; k < kSwarmWaves; ++k) tot += s_part[k];
            if (tot) atomicAdd(reinterpret_cast<unsigned long long *>(pvals) + slot, tot);
        }
        __syncthreads();
    }
}

// The listed pairs' counts, whole numbers so far (up to 2^60: a sum of doubles would depend on the
// order above 2^53), as doubles, into the bin-pair table and into *total. The first few bins that
// a wave's pairs fall in are added up across it: 9e4 pairs of one bin, each an addition to the
// same address, took 1.1 ms.
constexpr int kBinRounds = 4;
__global__ void __launch_bounds__(256) k_swarm_bins(
    const long long *__restrict__ pkeys, double *__restrict__ pvals, int64_t pcap,
    const uint32_t *__restrict__ list, const uint32_t *__restrict__ listed, int64_t n_t,
    const int32_t *__restrict__ q_bins, const int32_t *__restrict__ t_bins, int64_t n_t_bins,
    long long *keys, double *vals, uint64_t mask, unsigned long long *total, DevCounters *c) {
    const int lane = threadIdx.x & 63;
    const int64_t n_multi = listed[0], n = n_multi + listed[1];
    unsigned long long all = 0;
    for (int64_t a0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x - lane; a0 < n;
         a0 += (int64_t)gridDim.x * blockDim.x) {  // a wave's 64 pairs
        const int64_t at = a0 + lane;
        unsigned long long tot = 0;
        long long key = -1ll;
        if (at < n) {
            const int64_t slot = list[at < n_multi ? at : pcap - 1 - (at - n_multi)];
            tot = (unsigned long long)__double_as_longlong(pvals[slot]);
            if (tot) {
                pvals[slot] = (double)tot;
                const int64_t i = pkeys[slot] / n_t, j = pkeys[slot] - i * n_t;
                key = (long long)q_bins[i] * n_t_bins + t_bins[j];
            }
        }
        all += tot;
        unsigned long long todo = __ballot(key >= 0);
        for (int r = 0; r < kBinRounds && todo != 0ull; ++r) {
            const int first = (int)__ffsll(todo) - 1;
            const bool mine = key == __shfl(key, first);
            unsigned long long sum = mine ? tot : 0ull;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == first) table_add(keys, vals, mask, key, (double)sum, &c->err);
            todo &= ~__ballot(mine);
        }
        if (todo >> lane & 1ull) table_add(keys, vals, mask, key, (double)tot, &c->err);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) all += __shfl_xor(all, off);
    if (lane == 0 && all) atomicAdd(total, all);
}

// One cloud per occupied bin: weighted-mean energy, direction and position (at the grid
// time, carried back to t = 0 along the mean direction), weight = the bin's total.
// Appended in arbitrary order; rec_bin[r] is the bin of record r.
__global__ void k_st_records(const double *__restrict__ sums, int64_t n_bins, double t_bin,
                             double *__restrict__ soa, int64_t cap, int32_t *__restrict__ rec_bin,
                             unsigned long long *__restrict__ count) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b >= n_bins) return;
    const double *s = sums + kStSums * b;
    const double w = s[0];
    if (!(w > 0.0)) return;
    const unsigned long long r = atomicAdd(count, 1ull);
    if ((int64_t)r >= cap) return;
    const double E = s[1] / w;
    const double u[3] = {s[2] / w, s[3] / w, s[4] / w};
    const double X[3] = {s[5] / w, s[6] / w, s[7] / w};
    for (int a = 0; a < 3; ++a) {
        soa[a * cap + r] = X[a] - t_bin * u[a];
        soa[(3 + a) * cap + r] = E * u[a];
    }
    soa[6 * cap + r] = E;
    soa[7 * cap + r] = w;
    rec_bin[r] = (int32_t)b;
}

// Occupied slots of the overlap table, in no order: key, overlap integral and row number (the
// value the rows are sorted with). Slots are taken kCompactSlots per thread and a workgroup
// claims its rows with one atomic: with one per row, the counter's address was the whole
// kernel (3.2 ms per 2^22 slots). Rows beyond cap are counted, not written.
constexpr int kCompactSlots = 4;
__global__ void __launch_bounds__(256) k_st_compact(const long long *__restrict__ keys,
                                                    const double *__restrict__ vals, int64_t n_slots,
                                                    unsigned long long *__restrict__ key_out,
                                                    uint32_t *__restrict__ row_out,
                                                    double *__restrict__ om_out, int64_t cap,
                                                    unsigned long long *__restrict__ count) {
    __shared__ unsigned int s_wave[4];
    __shared__ unsigned long long s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k0 = blockIdx.x * (int64_t)(256 * kCompactSlots) + threadIdx.x;
    long long key[kCompactSlots];
    double om[kCompactSlots];
    unsigned int rank[kCompactSlots];
    unsigned int n = 0;  // rows of this wave so far
#pragma unroll
    for (int r = 0; r < kCompactSlots; ++r) {
        const int64_t k = k0 + 256 * r;
        key[r] = k < n_slots ? keys[k] : -1ll;
        om[r] = key[r] >= 0 ? vals[k] : 0.0;
        const bool has = om[r] > 0.0;
        const unsigned long long b = __ballot(has);
        rank[r] = n + (unsigned int)__popcll(b & ((1ull << lane) - 1ull));
        if (!has) key[r] = -1ll;
        n += (unsigned int)__popcll(b);
    }
    if (lane == 0) s_wave[wave] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int all = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
        s_base = all ? atomicAdd(count, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    unsigned long long base = s_base;
    for (int w = 0; w < wave; ++w) base += s_wave[w];
#pragma unroll
    for (int r = 0; r < kCompactSlots; ++r) {
        const int64_t row = (int64_t)(base + rank[r]);
        if (key[r] < 0 || row >= cap) continue;
        key_out[row] = (unsigned long long)key[r];
        row_out[row] = (uint32_t)row;
        om_out[row] = om[r];
    }
}

// Feature rows in ascending key order (key, the compacted rows' numbers in that order and their
// overlap integrals Omega; bin pair a, b): log E_a, log E_b, log(1 - cos theta_ab) (theta between
// the mean directions), log rho_a, log rho_b, log Omega (rho = bin total / cell volume); and the
// bin-level yield Y0 = rho_a rho_b sigma(s_ab) (1 - cos theta_ab) Omega. Formed in their final
// places: neighbouring rows share bin a, and no permutation of finished rows follows (forming
// them from the table's slots and moving them took 1.7 ms for 8e6 rows).
__global__ void __launch_bounds__(256) k_st_features(
    const unsigned long long *__restrict__ key, const uint32_t *__restrict__ rows,
    const double *__restrict__ om_in, int64_t n, int64_t n_t_bins,
    const double *__restrict__ q_sums, const double *__restrict__ t_sums, double vol,
    float *__restrict__ x, double *__restrict__ y0, long long *__restrict__ key_out) {
    const int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (row >= n) return;
    const int64_t k = (int64_t)key[row];
    const double om = om_in[rows[row]];
    const int64_t a = k / n_t_bins, b = k - a * n_t_bins;
    const double *sa = q_sums + kStSums * a, *sb = t_sums + kStSums * b;
    const double Ea = sa[1] / sa[0], Eb = sb[1] / sb[0];
    const double ua[3] = {sa[2], sa[3], sa[4]}, ub[3] = {sb[2], sb[3], sb[4]};
    const double na = sqrt((ua[0] * ua[0] + ua[1] * ua[1]) + ua[2] * ua[2]);
    const double nb = sqrt((ub[0] * ub[0] + ub[1] * ub[1]) + ub[2] * ub[2]);
    const double cth = ((ua[0] * ub[0] + ua[1] * ub[1]) + ua[2] * ub[2]) / (na * nb);
    const double qf = fmax(1.0 - cth, 1e-300);
    const double s = ((Ea * Eb) * qf) / (2.0 * kMe * kMe);
    const double ra = sa[0] / vol, rb = sb[0] / vol;
    float *f = x + kMlpIn * row;
    f[0] = (float)log(Ea);
    f[1] = (float)log(Eb);
    f[2] = (float)log(qf);
    f[3] = (float)log(ra);
    f[4] = (float)log(rb);
    f[5] = (float)log(om);
    y0[row] = ((ra * rb) * bw_sigma(s)) * qf * om;
    key_out[row] = k;
}

// Training targets log((Y + eps Y0) / Y0), Y the exact yield of the row's bin pair (0 when
// the pair is absent from the exact table).
__global__ void k_st_targets(const long long *__restrict__ key, const double *__restrict__ y0,
                             int64_t n, const long long *__restrict__ tkeys,
                             const double *__restrict__ tvals, uint64_t tmask, double eps,
                             float *__restrict__ target, double *__restrict__ y_exact) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double Y = 0.0;
    uint64_t h = mix64((uint64_t)key[i]) & tmask;
    for (uint64_t probe = 0; probe <= tmask && probe < kMaxProbe; ++probe) {
        const long long cur = tkeys[h];
        if (cur == key[i]) {
            Y = tvals[h];
            break;
        }
        if (cur == -1ll) break;
        h = (h + 1) & tmask;
    }
    const double z = y0[i];
    target[i] = z > 0.0 ? (float)log((Y + eps * z) / z) : 0.0f;
    if (y_exact) y_exact[i] = Y;
}

__device__ __forceinline__ double st_pred(const double *y0, const float *mean, int64_t i,
                                          double eps, double scale) {
    return scale * fmax(y0[i] * (exp((double)mean[i]) - eps), 0.0);
}

// Bucket of an uncertainty contribution u > 0 on a log2 scale, 16 buckets per octave.
__device__ __forceinline__ int unc_bucket(double u) {
    if (!(u > 0.0)) return 0;
    const int b = (int)floor(log2(u) * 16.0) + kUncBuckets / 2;
    return b < 1 ? 1 : (b >= kUncBuckets ? kUncBuckets - 1 : b);
}

// Histogram of the rows' uncertainty contributions u_i = Yhat_i sd_i (absolute spread of
// the predicted yield): per bucket the sum of u_i^2; and the predicted total in slots.
__global__ void k_st_unc(const double *__restrict__ y0, const float *__restrict__ mean,
                         const float *__restrict__ sdev, int64_t n, double eps, double scale,
                         double *__restrict__ var_hist, double *__restrict__ slots) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double yh = 0.0;
    if (i < n) {
        yh = st_pred(y0, mean, i, eps, scale);
        const double u = yh * (double)sdev[i];
        if (u > 0.0) atomicAdd(&var_hist[unc_bucket(u)], u * u);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) yh += __shfl_xor(yh, off);
    if ((threadIdx.x & 63) == 0 && yh != 0.0) atomicAdd(&slots[blockIdx.x & (kCounterSlots - 1)], yh);
}

// Gate: a row goes to the exact path (key into the filter set, bins marked) when its
// ensemble spread exceeds `gate` (per-pair mode, cut < 0) or its uncertainty bucket lies
// above `cut` (budget mode); the others add their predicted yield.
__global__ void k_st_gate(const long long *__restrict__ key, const double *__restrict__ y0,
                          const float *__restrict__ mean, const float *__restrict__ sdev, int64_t n,
                          double eps, double gate, double scale, int cut, int64_t n_t_bins,
                          long long *filter, uint64_t fmask, uint8_t *__restrict__ qmark,
                          uint8_t *__restrict__ tmark, double *__restrict__ slots,
                          unsigned long long *__restrict__ n_flag, unsigned int *err) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double add = 0.0;
    unsigned long long fl = 0;
    if (i < n) {
        const double yh = st_pred(y0, mean, i, eps, scale);
        const bool flag = cut < 0 ? (sdev[i] > gate) : (unc_bucket(yh * (double)sdev[i]) > cut);
        if (flag) {
            fl = 1;
            const long long k = key[i];
            const int64_t a = k / n_t_bins;
            qmark[a] = 1;
            tmark[k - a * n_t_bins] = 1;
            uint64_t h = mix64((uint64_t)k) & fmask;
            bool done = false;
            for (uint64_t probe = 0; probe <= fmask && probe < kMaxProbe && !done; ++probe) {
                const long long prev = (long long)atomicCAS(
                    reinterpret_cast<unsigned long long *>(filter + h), ~0ull, (unsigned long long)k);
                if (prev == -1ll || prev == k) done = true;
                else h = (h + 1) & fmask;
            }
            if (!done) atomicOr(err, kErrTableFull);
        } else {
            add = yh;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        add += __shfl_xor(add, off);
        fl += __shfl_xor(fl, off);
    }
    if ((threadIdx.x & 63) == 0) {
        if (add != 0.0) atomicAdd(&slots[blockIdx.x & (kCounterSlots - 1)], add);
        if (fl) atomicAdd(n_flag, fl);
    }
}

// Photons whose bin is not marked get bin -1 (skipped by the exact pass).
__global__ void k_st_mask_bins(const int32_t *__restrict__ bins, int64_t n,
                               const uint8_t *__restrict__ mark, int32_t *__restrict__ out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t b = bins[i];
    out[i] = (b >= 0 && mark[b]) ? b : -1;
}

__global__ void k_fill_i64v(long long *p, long long v, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

void launch_st_records(const double *sums, int64_t n_bins, double t_bin, double *soa, int64_t cap,
                       int32_t *rec_bin, unsigned long long *count, hipStream_t st) {
    if (n_bins <= 0) return;
    hipLaunchKernelGGL(k_st_records, dim3(grid_for(n_bins, 256)), dim3(256), 0, st, sums, n_bins,
                       t_bin, soa, cap, rec_bin, count);
}

void launch_st_compact(const long long *keys, const double *vals, int64_t n_slots,
                       unsigned long long *key, uint32_t *row, double *om, int64_t cap,
                       unsigned long long *count, hipStream_t st) {
    hipLaunchKernelGGL(k_st_compact, dim3(grid_for(n_slots, 256 * kCompactSlots)), dim3(256), 0, st,
                       keys, vals, n_slots, key, row, om, cap, count);
}

void launch_st_features(const unsigned long long *key, const uint32_t *rows, const double *om,
                        int64_t n, int64_t n_t_bins, const double *q_sums, const double *t_sums,
                        double vol, float *x, double *y0, long long *key_out, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_st_features, dim3(grid_for(n, 256)), dim3(256), 0, st, key, rows, om, n,
                       n_t_bins, q_sums, t_sums, vol, x, y0, key_out);
}

void launch_st_targets(const long long *key, const double *y0, int64_t n, const long long *tkeys,
                       const double *tvals, int64_t tcap, double eps, float *target, double *y_exact,
                       hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_st_targets, dim3(grid_for(n, 256)), dim3(256), 0, st, key, y0, n, tkeys,
                       tvals, (uint64_t)(tcap - 1), eps, target, y_exact);
}

void launch_st_gate(const long long *key, const double *y0, const float *mean, const float *sdev,
                    int64_t n, double eps, double gate, double scale, int cut, int64_t n_t_bins,
                    long long *filter, int64_t fcap, uint8_t *qmark, uint8_t *tmark, double *slots,
                    unsigned long long *n_flag, unsigned int *err, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_st_gate, dim3(grid_for(n, 256)), dim3(256), 0, st, key, y0, mean, sdev, n,
                       eps, gate, scale, cut, n_t_bins, filter, (uint64_t)(fcap - 1), qmark, tmark, slots,
                       n_flag, err);
}

void launch_st_unc(const double *y0, const float *mean, const float *sdev, int64_t n, double eps,
                   double scale, double *var_hist, double *slots, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_st_unc, dim3(grid_for(n, 256)), dim3(256), 0, st, y0, mean, sdev, n, eps,
                       scale, var_hist, slots);
}

void launch_st_mask_bins(const int32_t *bins, int64_t n, const uint8_t *mark, int32_t *out,
                         hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_st_mask_bins, dim3(grid_for(n, 256)), dim3(256), 0, st, bins, n, mark, out);
}

void launch_fill_keys(long long *p, int64_t n, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill_i64v, dim3(grid_for(n, 256)), dim3(256), 0, st, p, -1ll, n);
}

void launch_st_bin(const BeamDev &b, const StGridDev &g, int32_t *bins, double *sums,
                   hipStream_t st) {
    if (b.n <= 0) return;
    hipLaunchKernelGGL(k_st_bin, dim3(grid_for(b.n, 256)), dim3(256), 0, st, b, g, bins, sums);
}

void launch_st_deplete(long long *pkeys, double *pvals, int64_t pcap, const BeamDev &q,
                       const BeamDev &t, const int32_t *q_bins, const int32_t *t_bins,
                       int64_t n_t_bins, const StCell &cell, long long *keys, double *vals,
                       int64_t cap, double *slots, DevCounters *c, hipStream_t st) {
    if (pcap <= 0 || t.n <= 0) return;
    const unsigned grid = (unsigned)std::min<int64_t>(grid_for(pcap, 256), 4096);
    hipLaunchKernelGGL(k_st_deplete, dim3(grid), dim3(256), 0, st, pkeys, pvals, pcap, q, t,
                       q_bins, t_bins, n_t_bins, cell, keys, vals, (uint64_t)(cap - 1), slots, c);
}

void launch_swarm(const long long *pkeys, double *pvals, int64_t pcap, const BeamDev &q,
                  const BeamDev &t, const int32_t *q_bins, const int32_t *t_bins,
                  int64_t n_t_bins, const StCell &cell, double T0, double Tw, long long *keys,
                  double *vals, int64_t cap, uint32_t *list, unsigned long long *total,
                  DevCounters *c, hipStream_t st) {
    if (pcap <= 0 || t.n <= 0) return;
    uint32_t *listed = reinterpret_cast<uint32_t *>(total + 1);
    for (int64_t a = 0; a < pcap; a += kSwarmList) {  // pieces of the table
        const int64_t n = std::min(pcap - a, kSwarmList);
        if (a > 0) launch_au_zero(reinterpret_cast<double *>(listed), 1, st);
        hipLaunchKernelGGL(k_swarm_list, dim3(grid_for(n, 256)), dim3(256), 0, st, pkeys + a,
                           pvals + a, n, q.w, t.n, list, listed);
        hipLaunchKernelGGL(k_swarm, dim3((unsigned)std::min<int64_t>(n, 16384), kSwarmSplit),
                           dim3(64 * kSwarmWaves), 0, st, pkeys + a, pvals + a, n, list, listed, q,
                           t, cell, T0, Tw, c);
        hipLaunchKernelGGL(k_swarm_bins, dim3((unsigned)std::min<int64_t>(grid_for(n, 256), 512)),
                           dim3(256), 0, st, pkeys + a, pvals + a, n, list, listed, t.n, q_bins,
                           t_bins, n_t_bins, keys, vals, (uint64_t)(cap - 1), total, c);
    }
}

void launch_st_clear(long long *keys, double *vals, int64_t cap, double *slots, hipStream_t st) {
    const int64_t n = cap > kCounterSlots ? cap : kCounterSlots;
    hipLaunchKernelGGL(k_st_clear, dim3(grid_for(n, 256)), dim3(256), 0, st, keys, vals, cap, slots);
}

void launch_st_pack(const BeamDev &b, const int32_t *bins, StRec *rec, hipStream_t st) {
    if (b.n <= 0) return;
    hipLaunchKernelGGL(k_st_pack, dim3(grid_for(b.n, 256)), dim3(256), 0, st, b, bins, rec);
}

void launch_st_traverse(const Node *nodes, int64_t n_int64, const PBox *root_box, const PBox *qbox,
                        const uint32_t *qorder, int64_t nq, int32_t m, const int32_t *inst_root,
                        int64_t n_t, const StRec *qrec, const StRec *trec, int64_t n_t_bins,
                        double dt, int32_t win, int32_t k_begin, int32_t k_last,
                        const StCell &cell, int mode, const long long *filter,
                        int64_t filter_cap, long long *keys, double *vals, int64_t cap,
                        double *slots, DevCounters *c, hipStream_t st) {
    if (nq <= 0 || m <= 0 || n_int64 < 0) return;
    const int64_t groups = (nq + kStQueries - 1) / kStQueries, waves = groups * m;
    for (int64_t first = 0; first < waves; first += kStLaunch)
        hipLaunchKernelGGL(k_st_traverse, dim3((unsigned)std::min(waves - first, kStLaunch)),
                           dim3(64), 0, st, nodes, (int32_t)n_int64, root_box, qbox, qorder, nq,
                           groups, first, inst_root, n_t, qrec, trec, n_t_bins, dt, win, k_begin,
                           k_last, cell, mode, filter, (uint64_t)(filter ? filter_cap - 1 : 0),
                           keys, vals, (uint64_t)(cap - 1), slots, c);
}

void launch_st_lanes(const Node *nodes, int64_t n_int, const PBox *root_box, const PBox *qbox,
                     const uint32_t *qorder, int64_t nq, int32_t m, const int32_t *inst_root,
                     int64_t n_t, const StRec *qrec, const StRec *trec, int64_t n_t_bins, double dt,
                     int32_t k_begin, int32_t k_last, const StCell &cell, int mode,
                     const long long *filter, int64_t filter_cap, long long *keys, double *vals,
                     int64_t cap, double *slots, DevCounters *c, hipStream_t st) {
    if (nq <= 0 || m <= 0 || n_int < 0) return;
    if ((nq + kStQueries - 1) / kStQueries * m <= kMeetWaves) {
        launch_st_traverse(nodes, n_int, root_box, qbox, qorder, nq, m, inst_root, n_t, qrec, trec,
                           n_t_bins, dt, 1, k_begin, k_last, cell, mode, filter, filter_cap, keys,
                           vals, cap, slots, c, st);
        return;
    }
    const dim3 grid(grid_for(nq * m, 256)), block(256);
    const uint64_t fmask = filter ? (uint64_t)(filter_cap - 1) : 0;
    if (mode == kStMeet)
        hipLaunchKernelGGL(k_st_lanes<true>, grid, block, 0, st, nodes, (int32_t)n_int, root_box, qbox,
                           qorder, nq, (int64_t)m, inst_root, n_t, qrec, trec, n_t_bins, dt, cell,
                           mode, filter, fmask, keys, vals, (uint64_t)(cap - 1), slots, c);
    else
        hipLaunchKernelGGL(k_st_lanes<false>, grid, block, 0, st, nodes, (int32_t)n_int, root_box,
                           qbox, qorder, nq, (int64_t)m, inst_root, n_t, qrec, trec, n_t_bins, dt,
                           cell, mode, filter, fmask, keys, vals, (uint64_t)(cap - 1), slots, c);
}

}  // namespace tril
