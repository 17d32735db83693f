// rpdla_batched.hpp -- parameter sweeps in one pass per atom chunk: sampling
// and ionization over every configuration's atoms, then the push of every
// configuration's electrons together (in the order of their step counts, or,
// where the workspace has no room for that, in one persistent launch with a
// work counter per configuration), then one binning pass over the chunk's
// final momenta into per-configuration energy-angle histograms.
#pragma once

#include "rpdla_kernels.hpp"

namespace rpdla {

constexpr int kMaxCfg = 64;

struct BatchCtl {
    unsigned long long chunk;            // index of the chunk being processed
    unsigned long long queue[kMaxCfg];   // per-configuration push work counters
};

struct BatchArgs {
    const DevCfg* cfgs;        // device table [n_cfg]
    const double* geo;         // [n_cfg][2]: sampling radius, half length [m]
    int32_t n_cfg;
    uint64_t seed;
    uint32_t cfg_base;         // RNG key of configuration c is (seed, cfg_base + c)
    int64_t atoms_per_cfg, apc;  // atoms per configuration, atoms per chunk
    int32_t k_first, K;
    double* x; double* y; double* z;  // [n_cfg * apc]
    double* tb;                       // [n_cfg * apc * K]
    double* ux; double* uy; double* uz;  // final momenta [n_cfg * apc * K]
    BatchCtl* ctl;
    HistArgs H;
    unsigned long long* counts;       // [n_cfg][2 nE nA]
    unsigned long long* tallies;      // [n_cfg][6]
    unsigned long long* steps;        // [n_cfg] electron-steps taken, or null
};

__global__ void batch_set_cfg_kernel(DevCfg c, double r_max, double z_half, DevCfg* table,
                                     double* geo, int idx)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        table[idx] = c;
        geo[2 * idx] = r_max;
        geo[2 * idx + 1] = z_half;
    }
}

__global__ void batch_reset_kernel(BatchCtl* ctl, unsigned long long first_chunk)
{
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) ctl->chunk = first_chunk;
        if (threadIdx.x < kMaxCfg) ctl->queue[threadIdx.x] = 0ull;
    }
}

__global__ void batch_zero_queue_kernel(BatchCtl* ctl)
{
    if (blockIdx.x == 0 && threadIdx.x < kMaxCfg) ctl->queue[threadIdx.x] = 0ull;
}

__global__ void batch_advance_kernel(BatchCtl* ctl)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) ctl->chunk += 1ull;
}

// Atoms of this chunk for every configuration, configuration-major.
__global__ void __launch_bounds__(256) batch_sample_kernel(BatchArgs A)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)A.n_cfg * A.apc) return;
    const int c = (int)(i / A.apc);
    const int64_t a = i - (int64_t)c * A.apc;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    if (first + a >= A.atoms_per_cfg) return;
    const U64x4 r = philox4x64((uint64_t)(first + a), 0, 0, 0, A.seed, (uint64_t)(A.cfg_base + c));
    const double rad = A.geo[2 * c] * sqrt(u01(r.v[0]));
    double sn, cs;
    sincos(kTwoPi * u01(r.v[1]), &sn, &cs);
    A.x[i] = rad * cs;
    A.y[i] = rad * sn;
    A.z[i] = A.geo[2 * c + 1] * (2.0 * u01(r.v[2]) - 1.0);
}

// One wave per atom, as ionize_kernel, for atoms i0, i0 + 1, ... of the chunk;
// the wave's configuration is uniform and read with scalar loads.
template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) batch_ionize_kernel(
    BatchArgs A, const DevCfg* __restrict__ cfgs, int64_t i0)
{
    const int64_t i = i0 + wave_index();
    if (i >= (int64_t)A.n_cfg * A.apc) return;
    const int c = (int)(i / A.apc);
    const int64_t a = i - (int64_t)c * A.apc;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    if (first + a >= A.atoms_per_cfg) return;
    const DevCfg& cf = cfgs[c];
    const RateRegs R(cf);
    ionize_atom<FIELD>(cf, R, A.seed, A.cfg_base + (uint32_t)c, (uint64_t)(first + a),
                       A.x[i] * cf.k, A.y[i] * cf.k, A.z[i] * cf.k, A.k_first, A.K,
                       A.tb + i * A.K);
}

// The other forms (see ionize_form), a configuration per blockIdx.y.
template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) batch_ionize_few_kernel(
    BatchArgs A, const DevCfg* __restrict__ cfgs, int32_t per_wave)
{
    const int c = blockIdx.y, lane = __lane_id();
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    const int64_t n = A.atoms_per_cfg - first < A.apc ? A.atoms_per_cfg - first : A.apc;
    const int64_t a0 = wave_index() * per_wave, base = (int64_t)c * A.apc;
    if (a0 >= n) return;
    const DevCfg& cf = cfgs[c];
    const int64_t a = a0 + lane;
    double X = 0.0, Y = 0.0, Z = 0.0;
    bool open = false;
    if (lane < per_wave && a < n) {
        X = A.x[base + a] * cf.k; Y = A.y[base + a] * cf.k; Z = A.z[base + a] * cf.k;
        open = atom_open<FIELD>(cf, A.seed, A.cfg_base + (uint32_t)c, (uint64_t)(first + a), X, Y, Z,
                                A.k_first);
        if (!open)
            for (int s = 0; s < A.K; ++s) A.tb[(base + a) * A.K + s] = __builtin_inf();
    }
    uint64_t todo = __ballot(open);
    if (todo == 0) return;
    const RateRegs R(cf);
#pragma unroll 1
    while (todo) {
        const int l = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        ionize_atom<FIELD>(cf, R, A.seed, A.cfg_base + (uint32_t)c, (uint64_t)(first + a0 + l),
                           lane_value(X, l), lane_value(Y, l), lane_value(Z, l), A.k_first, A.K,
                           A.tb + (base + a0 + l) * A.K);
    }
}

template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) batch_ionize_lane_kernel(
    BatchArgs A, const DevCfg* __restrict__ cfgs)
{
    const int c = blockIdx.y;
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    if (a >= A.apc || first + a >= A.atoms_per_cfg) return;
    const DevCfg& cf = cfgs[c];
    const int64_t i = (int64_t)c * A.apc + a;
    const RateRegs R(cf);
    ionize_atom_lane<FIELD>(cf, R, A.seed, A.cfg_base + (uint32_t)c, (uint64_t)(first + a),
                            A.x[i] * cf.k, A.y[i] * cf.k, A.z[i] * cf.k, A.k_first, A.K,
                            A.tb + i * A.K);
}

// The queue push: one persistent launch over n_cfg * apc * K slots.  Slot j belongs to
// configuration j / (apc K) and atom (j / K) % apc of the chunk.  Every
// configuration has its own work counter, and a wave works on ONE
// configuration at a time: it starts on configuration (wave id mod n_cfg),
// refills its lanes from that configuration's counter, and when the counter
// is exhausted lets its lanes finish and moves on to the next configuration
// that still has work.  The wave's configuration index is therefore uniform,
// and its constants are read from the configuration table (a separate
// read-only kernel argument) with scalar loads at a uniform address, so they
// never occupy vector registers and the compiler can reload instead of
// spilling them.  The step's vector registers hold electron state only.  Final
// momenta go to the chunk's u arrays (NaN for invalid births; unborn and
// inactive slots are not written).
// Register budgets of the queue push: as the single push, except that the mixed
// form keeps 6 waves (its queue switching needs a few more registers than 7 waves
// leave).  The ordered push below has the single push's.
template <class E, int FIELD>
struct BatchWaves { static constexpr int value = ElecWaves<E, FIELD>::value; };
template <int FIELD> struct BatchWaves<ElecMixed, FIELD> { static constexpr int value = 6; };

template <int FIELD, class ELEC>
__global__ void __launch_bounds__(256, (BatchWaves<ELEC, FIELD>::value)) batch_push_kernel(
    BatchArgs A, const DevCfg* __restrict__ cfgs)
{
    extern __shared__ unsigned long long s_steps[];   // [n_cfg] steps taken in this block
    const int ncfg = A.n_cfg;
    for (int w = threadIdx.x; w < ncfg; w += blockDim.x) s_steps[w] = 0ull;
    __syncthreads();

    const int64_t per_cfg = A.apc * A.K;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    const int wave = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    int cw = __builtin_amdgcn_readfirstlane(wave % ncfg);
    int64_t idx = -1;
    bool draining = false;
    ELEC e;
    e.left = 0;
    while (true) {
        if (!draining) {
            while (true) {
                const bool need = idx < 0;
                if (__ballot(need) == 0) break;
                const int64_t j = queue_take(&A.ctl->queue[cw], need);
                bool dry = false;
                if (need) {
                    if (j >= per_cfg) {
                        dry = true;
                    } else {
                        const int64_t a = j / A.K;
                        const int64_t js = (int64_t)cw * per_cfg + j;
                        const double t0 = A.tb[js];
                        if (first + a < A.atoms_per_cfg && t0 < __builtin_inf()) {
                            const int64_t ia = (int64_t)cw * A.apc + a;
                            if (elec_init(cfgs[cw], e, t0, A.x[ia], A.y[ia], A.z[ia])) {
                                if (e.left > 0) {
                                    idx = js;
                                    atomicAdd(&s_steps[cw], (unsigned long long)e.left);
                                } else {
                                    double ux, uy, uz, xf, yf, zf;
                                    elec_final(cfgs[cw], e, ux, uy, uz, xf, yf, zf);
                                    A.ux[js] = ux; A.uy[js] = uy; A.uz[js] = uz;
                                }
                            } else {
                                const double q = __builtin_nan("");
                                A.ux[js] = q; A.uy[js] = q; A.uz[js] = q;
                            }
                        }
                    }
                }
                if (__ballot(dry) != 0) { draining = true; break; }
            }
        }
        if (__ballot(idx >= 0) == 0) {
            if (!draining) continue;
            // this configuration is exhausted: move to the next one with work
            int next = -1;
            for (int k = 1; k <= ncfg && next < 0; ++k) {
                const int c2 = (cw + k) % ncfg;
                const unsigned long long taken = atomicAdd(&A.ctl->queue[c2], 0ull);
                if ((int64_t)taken < per_cfg) next = c2;
            }
            if (next < 0) break;
            cw = __builtin_amdgcn_readfirstlane(next);
            draining = false;
            continue;
        }
        if (idx >= 0) {
            elec_step<FIELD, false, true>(cfgs[cw], e, fm::kCoef);
            if (e.left == 0) {
                double ux, uy, uz, xf, yf, zf;
                elec_final(cfgs[cw], e, ux, uy, uz, xf, yf, zf);
                A.ux[idx] = ux; A.uy[idx] = uy; A.uz[idx] = uz;
                idx = -1;
            }
        }
    }
    if (A.steps) {
        __syncthreads();
        for (int w = threadIdx.x; w < ncfg; w += blockDim.x)
            if (s_steps[w]) atomicAdd(&A.steps[w], s_steps[w]);
    }
}

// ---------------------------------------------------------------------------
// Ordered push of a chunk (see push_group_kernel): each configuration's born
// slots in the order of their step counts, in groups of 64 of one configuration
// (the last one of each part empty), and the groups of all configurations in
// the order of theirs, dealt to the waves in whole rounds and time slices.  A
// wave's configuration is uniform for a group and read with scalar loads.
// With the queues above a wave serves one configuration until that runs dry,
// every time down to its last electron: a sweep of 64 configurations of 10,240
// slots took 13.6% longer (both timed against a third form on two chips, 0.889
// and 0.782 of its time).
// ---------------------------------------------------------------------------
constexpr int kBatchBins = 512;

struct BatchPlan {
    PlanSplit split;
    uint32_t slice_steps, pad;
    uint32_t born[kMaxCfg], base[kMaxCfg];   // born slots; first place in the order
    uint32_t cursor[kMaxCfg * kBatchBins];   // counts, then the next free place
};

struct BatchGroup { uint32_t cfg, first; };  // first: place in its configuration's order

struct BatchPlanArgs {
    BatchPlan* plan;
    uint32_t* order;             // slot of its configuration
    BatchGroup* groups;
    uint64_t* state;
    uint32_t simds, max_waves;
    double n_max;                // bound of the step counts of all configurations
};

__device__ inline uint32_t batch_bin(const DevCfg& c, const BatchPlanArgs& P, double t0, double z)
{
    const double taue = (c.window == 0 ? z * c.k : 0.0) + c.ta_n;
    const double f = (taue - t0 * c.omega) / c.hn * ((double)kBatchBins / P.n_max);
    const double g = fmin(fmax(f, 0.0), (double)(kBatchBins - 1));
    return (uint32_t)(kBatchBins - 1) - (uint32_t)g;
}

// One configuration per blockIdx.y, kPlanChunk of its slots per block.
template <bool PLACE>
__global__ void __launch_bounds__(kPlanBlock) batch_plan_kernel(BatchArgs A,
                                                                const DevCfg* __restrict__ cfgs,
                                                                BatchPlanArgs P)
{
    __shared__ uint32_t bins[kBatchBins], base[kBatchBins];
    constexpr int kPer = kPlanChunk / kPlanBlock;
    const int c = blockIdx.y;
    const int64_t per_cfg = A.apc * A.K;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    for (int b = threadIdx.x; b < kBatchBins; b += kPlanBlock) bins[b] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kPlanChunk;
    uint32_t bin[kPer], rank[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int64_t j = lo + i * kPlanBlock + threadIdx.x;
        bin[i] = kBatchBins;
        if (j < per_cfg) {
            const int64_t a = j / A.K;
            const double t0 = A.tb[(int64_t)c * per_cfg + j];
            if (first + a < A.atoms_per_cfg && t0 < __builtin_inf()) {
                bin[i] = batch_bin(cfgs[c], P, t0, A.z[(int64_t)c * A.apc + a]);
                rank[i] = atomicAdd(&bins[bin[i]], 1u);
            }
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kBatchBins; b += kPlanBlock)
        if (bins[b]) base[b] = atomicAdd(&P.plan->cursor[c * kBatchBins + b], bins[b]);
    if constexpr (PLACE) {
        __syncthreads();
        uint32_t* order = P.order + P.plan->base[c];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (bin[i] < kBatchBins)
                order[base[bin[i]] + rank[i]] = (uint32_t)(lo + i * kPlanBlock + threadIdx.x);
    }
}

// Inclusive sum over the block's threads.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* part)
{
    part[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < kPlanBlock; d *= 2) {
        const uint32_t add = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    const uint32_t r = part[threadIdx.x];
    __syncthreads();
    return r;
}

// Places of the bins, the groups in order, and the plan (one block).
__global__ void __launch_bounds__(kPlanBlock) batch_plan_scan_kernel(int n_cfg, BatchPlanArgs P)
{
    __shared__ uint32_t part[kPlanBlock], born[kMaxCfg], first_bin;
    // each configuration's bins, one after another; threads past kBatchBins add nothing
    for (int c = 0; c < n_cfg; ++c) {
        const bool mine = threadIdx.x < kBatchBins;
        const uint32_t n = mine ? P.plan->cursor[c * kBatchBins + threadIdx.x] : 0;
        const uint32_t up = block_scan(n, part);
        if (mine) P.plan->cursor[c * kBatchBins + threadIdx.x] = up - n;
        if (threadIdx.x == kPlanBlock - 1) born[c] = up;
    }
    if (threadIdx.x == 0) first_bin = 0;
    __syncthreads();
    const int tc = (int)threadIdx.x;
    const uint32_t total = block_scan(tc < n_cfg ? born[tc] : 0, part);
    if (tc < n_cfg) {
        P.plan->born[tc] = born[tc];
        P.plan->base[tc] = total - born[tc];
    }
    // a group starts in each place that is a multiple of 64: groups in the
    // order of (bin, configuration)
    const int cells = n_cfg * kBatchBins, per = (cells + kPlanBlock - 1) / kPlanBlock;
    auto starts = [&](int cell, uint32_t& lo) {
        const int b = cell / n_cfg, c = cell - b * n_cfg;
        const uint32_t* off = P.plan->cursor + c * kBatchBins;
        lo = groups_of(off[b]);
        const uint32_t hi = groups_of(b + 1 < kBatchBins ? off[b + 1] : born[c]);
        return hi - lo;
    };
    uint32_t sum = 0, lo;
    for (int i = 0; i < per; ++i) {
        const int cell = tc * per + i;
        if (cell < cells) sum += starts(cell, lo);
    }
    const uint32_t up = block_scan(sum, part);
    if (tc == kPlanBlock - 1) part[0] = up;
    __syncthreads();
    const PlanSplit split = plan_split(part[0], P.simds, P.max_waves);
    const uint32_t whole = split.whole;
    uint32_t at = up - sum;
    for (int i = 0; i < per; ++i) {
        const int cell = tc * per + i;
        if (cell >= cells) break;
        const uint32_t n = starts(cell, lo);
        const int b = cell / n_cfg, c = cell - b * n_cfg;
        if (n && at <= whole && whole < at + n) first_bin = (uint32_t)b;
        for (uint32_t g = 0; g < n; ++g) P.groups[at + g] = BatchGroup{(uint32_t)c, (lo + g) * 64u};
        at += n;
    }
    __syncthreads();
    if (tc == 0) {
        BatchPlan& p = *P.plan;
        p.split = split;
        p.slice_steps = plan_slice_steps(
            (double)(kBatchBins - first_bin) * (P.n_max / (double)kBatchBins), split.slices);
    }
}

template <int FIELD, class ELEC>
__global__ void __launch_bounds__(256, (ElecWaves<ELEC, FIELD>::value)) batch_group_kernel(
    BatchArgs A, const DevCfg* __restrict__ cfgs, BatchPlanArgs P, int32_t slice)
{
    const BatchPlan* plan = P.plan;
    const uint32_t W = plan->split.waves, whole = plan->split.whole, rest = plan->split.rest;
    const uint32_t wave = (uint32_t)wave_index();
    if (wave >= W) return;
    uint32_t group = wave, end = whole;
    int32_t steps = 0x7fffffff;
    bool first = true;
    if (slice >= 0) {
        const uint32_t slices = plan->split.slices;
        const PlanTurn t = plan_turn((uint32_t)slice, wave, W, rest, slices);
        if (!t.any) return;
        group = whole + t.index;
        end = group + 1;
        first = t.turn == 0;
        if (t.turn + 1 < slices) steps = (int32_t)plan->slice_steps;
    }
    StepRegs<FIELD, ELEC> R;
    const int64_t per_cfg = A.apc * A.K;
    for (; group < end; group += W) {
        // what each lane needs before the step loop and after it, formed anew
        const uint32_t c = P.groups[group].cfg;
        const size_t stride = (size_t)rest * 64;
        auto state = [&]() { return P.state + (size_t)(group - whole) * 64 + fresh_lane(); };
        auto slot = [&]() -> int64_t {       // -1 for a lane without one
            const uint32_t at = P.groups[group].first + fresh_lane();
            return at < plan->born[c] ? (int64_t)c * per_cfg + (int64_t)P.order[plan->base[c] + at]
                                      : -1;
        };
        ELEC e;
        e.left = 0;
        if (!first) {
            get_state(state(), stride, e);
        } else {
            const int64_t js = slot();
            if (js >= 0) {
                const int64_t ia = (int64_t)c * A.apc + (js - (int64_t)c * per_cfg) / A.K;
                if (!elec_init(cfgs[c], e, A.tb[js], A.x[ia], A.y[ia], A.z[ia])) {
                    const double q = __builtin_nan("");
                    A.ux[js] = q; A.uy[js] = q; A.uz[js] = q;
                } else if (e.left <= 0) {
                    double ux, uy, uz, xf, yf, zf;
                    elec_final(cfgs[c], e, ux, uy, uz, xf, yf, zf);
                    A.ux[js] = ux; A.uy[js] = uy; A.uz[js] = uz;
                }
            }
            if (A.steps) {
                unsigned long long n = e.left > 0 ? (unsigned long long)e.left : 0ull;
                for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
                if (fresh_lane() == 0 && n) atomicAdd(&A.steps[c], n);
            }
        }
        const bool runs = e.left > 0;
        R.set(cfgs[c]);
        run_steps<FIELD, true>(R.c, e, R.k, steps);
        if (runs && e.left == 0) {
            const int64_t js = slot();
            double ux, uy, uz, xf, yf, zf;
            elec_final(cfgs[c], e, ux, uy, uz, xf, yf, zf);
            A.ux[js] = ux; A.uy[js] = uy; A.uz[js] = uz;
        }
        if (steps != 0x7fffffff) put_state(state(), stride, e);
    }
}

// Bin the chunk's electrons into their configuration's histogram: one lane
// per slot; bins and tallies merged across the wave (one atomic per distinct
// key).  Tallies as in rpdla_histogram; inactive atoms of a partial chunk are
// skipped.
__global__ void __launch_bounds__(256) batch_hist_kernel(BatchArgs A)
{
    const int64_t per_cfg = A.apc * A.K;
    const int64_t n_slots = (int64_t)A.n_cfg * per_cfg;
    const int64_t first = (int64_t)A.ctl->chunk * A.apc;
    const int64_t nbins = 2ll * A.H.nE * A.H.nA;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t base0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63);
    for (int64_t b = base0; b < n_slots; b += stride) {
        const int64_t j = b + __lane_id();
        int64_t key = -1, tkey = -1, dkey = -1;
        if (j < n_slots) {
            const int c = (int)(j / per_cfg);
            const int64_t a = (j - (int64_t)c * per_cfg) / A.K;
            if (first + a < A.atoms_per_cfg) {
                int tally = -1, dir = -1;
                const double t0 = A.tb[j];
                const bool born = t0 < __builtin_inf();
                key = bin_key(A.H, t0, born ? A.ux[j] : 0.0, born ? A.uy[j] : 0.0,
                              born ? A.uz[j] : 0.0, tally, dir);
                if (key >= 0) key += (int64_t)c * nbins;
                if (tally >= 2) tkey = (int64_t)c * 6 + tally;
                if (dir >= 0) dkey = (int64_t)c * 6 + dir;
            }
        }
        wave_merge_add(key, A.counts);
        wave_merge_add(tkey, A.tallies);
        wave_merge_add(dkey, A.tallies);
    }
}

}  // namespace rpdla
