// optimize.hpp -- k_optimize, the branch-length smoothing loop of a tree, and
// the launch templates of one (precision, block size); each pair is compiled
// in a source of its own (optimize_f32_256.hip and so on), which build in
// parallel.
#pragma once
#include "partials.hpp"

namespace pt {
namespace {

// Log density of independent Exponential(rate) priors on the E lengths in
// LDS, sum_e (log rate - rate t_e); 0 for rate 0.  Every thread reads all
// lengths in the same order, so all hold the same value.
__device__ inline double log_prior(const double *tl, int E, double rate) {
    if (!(rate > 0.0)) return 0.0;
    const double lr = log(rate);
    double s = 0.0;
    for (int e = 0; e < E; ++e) s += lr - rate * tl[e];
    return s;
}

// Branch-length optimisation: one block owns one tree at a time, taken from
// a work counter in the order given (largest trees first), and runs the
// whole smoothing loop -- partial updates, per-edge Newton iterations with
// block reductions, pass-level convergence -- without leaving the kernel.
// Every wave exits once the counter passes the number of trees.
// With a.groups = G > 1 (a small batch: G blocks per tree, all resident at
// once), G blocks on one XCD own tree order[q] instead (see below), each
// over its own contiguous share of the patterns, and every reduction spans the G blocks
// (group_sum3); they take identical decisions, and block 0 of the group
// writes the tree's outputs.
// Each thread owns patterns tid + j*BS, j < ni, of its block's share
// (ni*BS >= the share of every tree).  TAB_LDS: the per-edge eigenbasis
// table lives in LDS after the transition matrices; otherwise in a
// per-block slice of a.tab.  GRP: compiled for a.groups > 1 (the
// one-block-per-tree instantiations carry none of the cross-block code).
//
// What bounds it: a serial chain.  An edge step is an update or two, a table,
// one to two row passes with a block sum each, and the edge's new matrices,
// each a few hundred instructions on one or two waves per SIMD that wait for
// the last.  Clocks per edge step, 48 trees of 27 taxa on 4 blocks each: FP32
// 16.7k when every product was scalar code (updates 7.8k, row passes 7.0k),
// 14.9k with the products on the matrix cores, the sides of two steps fetched
// at once and the exponentials taken while they arrive, 14.5k with the sums'
// exponentials by row broadcast, 14.2k with the tree's descriptor in scalar
// registers (updates 5.4k, row passes 6.8k); FP64 22.1k, then 19.0k with the
// matrix entries by row broadcast (updates 12.6k -> 9.4k), 18.2k with the
// exponentials and 18.1k now.  The slowest of 256 mixed trees, one block of 512
// threads: 28.7k, 24.6k, 24.3k, 24.0k.  Reading the ops ahead of the loop (26
// scalar registers more) cost 5% instead.
// FP32 with up to four categories is held to two waves per SIMD, which keeps
// the matrix results out of the accumulation registers.
template <typename T, int BS, int KP, bool TAB_LDS, bool GRP>
__global__ void __launch_bounds__(BS, sizeof(T) == 4 && KP <= 4 ? 2 : 1) k_optimize(const BatchArgs a, double *brlen, const OptParams opt, int ni,
                                                 int pm_lds_doubles, double *lnl_out, int32_t *passes_out,
                                                 int32_t *status_out) {
    extern __shared__ __attribute__((aligned(16))) double lds[];  // rows of 16 and 32 bytes are read whole
    __shared__ double red[2 * (BS / 64) * 3];
    __shared__ double wxs[(BS / 64) * kWx];
    __shared__ ModelS model;
    __shared__ int q_sh;
    __shared__ GroupS gsh;
    __shared__ double pm_ex[4 * kMaxCats];
    const int tid = threadIdx.x;
    const int G = GRP ? a.groups : 1;
    // grouped: the hardware deals blocks to the XCDs in turn, so block i
    // runs on XCD i % kXcds; the G blocks of a tree are taken from one XCD
    // (trees x, x + kXcds, ... on XCD x), keeping their cross-block traffic
    // within one L2
    const unsigned xcd = blockIdx.x % (unsigned)kXcds, xslot = blockIdx.x / (unsigned)kXcds;
    const int g = GRP ? (int)(xslot % (unsigned)G) : 0;
    GroupS *gs = GRP ? &gsh : nullptr;
    double *wx = wxs + (tid >> 6) * kWx;
    // per block: the table [KP][BS*ni][4] of T, then the weights [BS*ni]
    const size_t tab_bytes = (size_t)BS * ni * KP * 4 * sizeof(T);
    char *tab_base = TAB_LDS ? reinterpret_cast<char *>(lds + pm_lds_doubles)
                             : reinterpret_cast<char *>(a.tab) + (size_t)blockIdx.x * (tab_bytes + (size_t)BS * ni * 8);
    T *tab = reinterpret_cast<T *>(tab_base);
    double *wrow = reinterpret_cast<double *>(tab_base + tab_bytes);
    for (int round = 0;; ++round) {
        int q;
        if (GRP) {
            q = (int)((xslot / (unsigned)G) * (unsigned)kXcds + xcd);
            if (round > 0 || q >= a.n_trees) break;
        } else {
            if (tid == 0) q_sh = atomicAdd(a.queue, 1);
            __syncthreads();
            q = __builtin_amdgcn_readfirstlane(q_sh);
            if (q >= a.n_trees) break;
        }
        // The tree's descriptor is wave-uniform and no launch writes it: scalar
        // loads.  (In vector registers it was also a hazard: with eight
        // categories in FP64 the compiler copied td.edge_off to accumulation
        // registers at the end of a divergent loop, before the instruction that
        // restores the execution mask, so that no lane was copied, and the
        // final lengths went to an address of leftover values.)
        const int b = ((const __attribute__((address_space(4))) int32_t *)a.order)[q];
        const TreeDev td = load_tree(a.trees, b);
        const AlnDev *aln = a.alns + td.aln;
        const int E = td.n_edges;
        // FP64 partials: the matrices, then the lengths, in LDS.  FP32
        // partials: the lengths, then (16-byte aligned) the matrices in FP32
        // (so a 64-taxon tree's table still fits in LDS beside them).
        constexpr bool kF32 = std::is_same<T, float>::value;
        constexpr bool kFuseUpd = GRP && TAB_LDS && FuseFirst<KP>::value && BS == 256;
        double *pm = kF32 ? nullptr : lds;
        double *tl = kF32 ? lds : lds + (size_t)E * KP * 16;
        float *pmf = reinterpret_cast<float *>(lds + (((size_t)E + 1) & ~(size_t)1));
        for (int e = tid; e < E; e += BS) tl[e] = fmin(fmax(brlen[td.edge_off + e], opt.t_min), opt.t_max);
        model_to_lds(aln, &model);
        if (GRP && tid == 0) {
            unsigned long long *base = a.gsync + (size_t)b * kGroupSyncWords;
            gsh.G = G;
            gsh.g = g;
            gsh.seq = 0;
            gsh.is_broken = 0;
            gsh.broken = base;
            gsh.slots = base + 1;
            gsh.wait = a.wait_cycles > 0 ? a.wait_cycles : kGroupWaitCycles;
        }
        __syncthreads();
        for (int x = tid; x < E * KP * 16; x += BS) {
            const int e = x / (KP * 16), r = x % (KP * 16);
            const double pe = pm_entry(&model, r >> 4, r & 15, tl[e]);
            if (kF32) pmf[x] = (float)pe;
            else pm[x] = pe;
        }
        __syncthreads();
        TreeView<T> v = make_view<T>(td, aln, a, &model, pm);
        v.pmf = pmf;
        // this block's share of the patterns
        const int chunk = (v.P + G - 1) / G;
        const int lo = min(v.P, g * chunk);
        v.np = min(v.P - lo, chunk);
        v.tips += lo;
        v.w += lo;
        v.clv += (size_t)lo * 4;
        v.cnt += lo;
        const double tol_gain = opt.tol_lnl / E;
        const double accept = fmax(sqrt(opt.tol_newton), kNewtonAccept);
        int parity = 0;
        double prev = -INFINITY, cur = -INFINITY;
        int passes = 0;
        bool converged = false;
        long long pc[PROF_FIELDS] = {0, 0, 0, 0, 0, 0, 0, 0};
        const long long t_start = clock64();
        for (;;) {
            const bool first = passes == 0;
            const int o0 = first ? td.op_first : td.op_steady;
            const int no = first ? td.n_first : td.n_steady;
            double max_rel = 0.0;
            double pass_gain = 0.0;  // the steps' predicted gains (FP32 partials)
            EdgePre pre;
            bool have_pre = false;
            for (int o = 0; o < no; ++o) {
                const Op op = load_op(a.ops, o0 + o);
                if (op.code == OP_UPDATE) {
                    const long long u0 = a.prof ? clock64() : 0;
                    bool fused = false;
                    // (256 threads per block only: with two waves per SIMD
                    // the extra registers would spill)
                    if constexpr (kFuseUpd) {
                        // an update making one side of the next edge step:
                        // build that edge's table from it directly
                        if (ni == 1 && o + 1 < no) {
                            const Op nx = load_op(a.ops, o0 + o + 1);
                            if (nx.code == OP_NEWTON && (nx.a == op.dst || nx.b == op.dst)) {
                                pre = update_and_table<T, BS, KP, OptPm<T, KP>::value>(
                                    v, op, nx.a == op.dst ? nx.b : nx.a, tl[nx.dst], tab, wrow, wx);
                                have_pre = fused = true;
                            }
                        }
                    }
                    if (!fused) do_update<T, BS, KP, OptPm<T, KP>::value>(v, op, 0, ni);
                    if (a.prof) {
                        pc[PROF_UPDATES] += 1;
                        pc[PROF_CYC_UPDATE] += clock64() - u0;
                    }
                    continue;
                }
                const int e = op.dst;
                const double t0 = tl[e];
                if constexpr (kPassLnl<T>) {
                    if (op.code == OP_EVAL) {
                        const Sums3 r = eval_edge<T, BS, KP>(v, op.a, op.b, 0, ni, t0, red, wx, parity, gs);
                        parity = r.parity;
                        cur = r.l0;
                        continue;
                    }
                }
                // the pass's lnL comes from its last edge step (op.ea = 1)
                const EdgeResult r =
                    newton_edge<T, BS, KP, !kFuseUpd>(v, op.a, op.b, t0, op.ea != 0, opt, tab, wrow, ni, red, wx, parity,
                                                      gs, passes >= 1 ? kRelax : 1.0, accept, have_pre ? &pre : nullptr);
                have_pre = false;
                parity = r.parity;
                if (op.ea) cur = r.lnl;
                pc[PROF_EDGE_STEPS] += 1;
                pc[PROF_NEWTON_ITERS] += r.iters;
                pc[PROF_CYC_TABLE] += r.cyc_table;
                pc[PROF_CYC_ITERS] += r.cyc_iters;
                // A step counts against convergence when it moves the length
                // by more than tol_t relative, unless it starts or ends at a
                // bound and its gain by the quadratic model at the start is
                // negligible (below tol_lnl / E; the bound is then optimal to
                // within that gain).  With FP32 partials a length whose
                // optimum lies at t_min otherwise never settles: the
                // derivative there is at the noise level, and Newton keeps
                // moving the length on and off the bound by amounts tiny in
                // absolute terms but large relative to the 1e-6 floor of the
                // relative change, for no gain.
                //
                // With FP32 partials the same holds away from the bounds: a
                // pass's lnL is resolved only to about 1e-4 (rounding of the
                // stored partials; measured on the 27-taxon trees), above
                // tol_lnl, and a short length keeps moving by about tol_t
                // relative on derivative noise for gains near 1e-9.  There a
                // step counts against convergence only when its gain is not
                // negligible, and the pass's lnL increase is taken as the sum
                // over its steps of the quadratic model's value (which sees
                // no rounding noise) instead of the difference of two noisy
                // lnL values.  A step not concave at its start still counts
                // its model value there (a flat long length settles with a
                // second derivative at the noise level, of either sign), and
                // always counts against convergence by its length change.
                const bool at_bound = t0 <= opt.t_min || t0 >= opt.t_max || r.t <= opt.t_min || r.t >= opt.t_max;
                if (!((kF32 || at_bound) && r.gain < tol_gain))
                    max_rel = fmax(max_rel, fabs(r.t - t0) / fmax(t0, 1e-6));
                pass_gain += r.rise;
                if (r.t != t0) {
                    if (tid == 0) tl[e] = r.t;
                    if constexpr (KP * 16 <= 64) {
                        // the edge's matrices are one wave's work: its first
                        // 4 KP lanes take the exponentials, then every lane
                        // one entry (LDS operations of a wave complete in order)
                        if (tid < 4 * KP) pm_ex[tid] = exp(model.lam[tid & 3] * model.rate[tid >> 2] * r.t);
                        __builtin_amdgcn_wave_barrier();
                        if (tid < KP * 16) {
                            const double pe = pm_entry_ex(&model, pm_ex, tid >> 4, tid & 15);
                            if (kF32) pmf[(size_t)e * KP * 16 + tid] = (float)pe;
                            else pm[(size_t)e * KP * 16 + tid] = pe;
                        }
                    } else {
                        if (tid < KP * 16) {
                            const double pe = pm_entry(&model, tid >> 4, tid & 15, r.t);
                            if (kF32) pmf[(size_t)e * KP * 16 + tid] = (float)pe;
                            else pm[(size_t)e * KP * 16 + tid] = pe;
                        }
                    }
                    __syncthreads();
                }
            }
            ++passes;
            if constexpr (kPassLnl<T>) cur += log_prior(tl, E, opt.prior_rate);
            const double rise = kF32 ? pass_gain : cur - prev;
            if (td.n_steady == 0 || (rise < opt.tol_lnl && max_rel < opt.tol_t)) {
                converged = true;
                break;
            }
            if (passes >= opt.max_passes) break;
            prev = cur;
        }
        if (g == 0) {
            for (int e = tid; e < E; e += BS) brlen[td.edge_off + e] = tl[e];
            if (tid == 0 && a.prof) {
                pc[PROF_PASSES] = passes;
                pc[PROF_CYC_TOTAL] = clock64() - t_start;
                for (int f = 0; f < PROF_FIELDS; ++f) a.prof[(size_t)b * PROF_FIELDS + f] = pc[f];
            }
            if (tid == 0) {
                // a timed-out wait anywhere in the group: status 2, lnL NaN
                const bool broken = GRP && load_agent((GlobalU64 *)gsh.broken) != 0ull;
                lnl_out[b] = broken ? NAN : kPassLnl<T> ? cur : 0.0;
                if (passes_out) passes_out[b] = passes;
                if (status_out) status_out[b] = broken ? 2 : (converged ? 0 : 1);
            }
        }
        __syncthreads();
    }
}

template <typename T, int BS, int KP, bool L, bool GRP>
hipError_t launch_opt_t(int grid, const BatchArgs &a, double *brlen, const OptParams &opt, int ni, int pm_doubles,
                        double *lnl, int32_t *passes, int32_t *status, size_t lds, hipStream_t s) {
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_optimize<T, BS, KP, L, GRP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_optimize<T, BS, KP, L, GRP>), dim3(grid), dim3(BS), lds, s, a, brlen, opt, ni,
                       pm_doubles, lnl, passes, status);
    return hipGetLastError();
}

template <typename T, int BS, int KP, bool L, bool GRP>
int occ_opt_t(size_t lds) {
    int n = 0;
    if (lds > 65536 && hipFuncSetAttribute(reinterpret_cast<const void *>(k_optimize<T, BS, KP, L, GRP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_optimize<T, BS, KP, L, GRP>, BS, lds) != hipSuccess)
        return 0;
    return n;
}

template <typename T, int BS, int KP, bool L, bool GRP>
size_t spill_opt_t() {
    hipFuncAttributes at;
    if (hipFuncGetAttributes(&at, reinterpret_cast<const void *>(k_optimize<T, BS, KP, L, GRP>)) != hipSuccess)
        return ~size_t(0);
    return at.localSizeBytes;
}

// Runtime (padded categories, table placement, grouped) to the matching
// instantiation of FN.  There is none of 512 threads for eight categories:
// two waves per SIMD leave it 256 registers, and it spilled (44 to 176 bytes
// per lane), so such plans take 256 threads.
#define PT_OPT_CALL(FN, T, BSZ, ...)                                                                             \
    PT_KP_SWITCH(if constexpr (KP * BSZ <= 2048) {                                                               \
        if (grouped) return tab_lds ? FN<T, BSZ, KP, true, true>(__VA_ARGS__) : FN<T, BSZ, KP, false, true>(__VA_ARGS__); \
        return tab_lds ? FN<T, BSZ, KP, true, false>(__VA_ARGS__) : FN<T, BSZ, KP, false, false>(__VA_ARGS__);   \
    })

}  // namespace

// The functions of OptimizeShape (kernels.hpp) for partials of type T and
// blocks of BSZ threads.
#define PT_DEFINE_OPTIMIZE(NAME, T, BSZ)                                                                         \
    namespace {                                                                                                  \
    int NAME##_occupancy(int kp, bool tab_lds, bool grouped, size_t lds) {                                       \
        PT_OPT_CALL(occ_opt_t, T, BSZ, lds);                                                                     \
        return 0;                                                                                                \
    }                                                                                                            \
    size_t NAME##_spill(int kp, bool tab_lds, bool grouped) {                                                    \
        PT_OPT_CALL(spill_opt_t, T, BSZ);                                                                        \
        return ~size_t(0);                                                                                       \
    }                                                                                                            \
    hipError_t NAME##_launch(int kp, int items, bool tab_lds, int pm_doubles, int grid, const BatchArgs &a,      \
                             double *brlen, const OptParams &opt, double *lnl, int32_t *passes, int32_t *status, \
                             size_t lds, hipStream_t s) {                                                        \
        const bool grouped = a.groups > 1;                                                                       \
        PT_OPT_CALL(launch_opt_t, T, BSZ, grid, a, brlen, opt, items, pm_doubles, lnl, passes, status, lds, s);  \
        return hipErrorInvalidValue;                                                                             \
    }                                                                                                            \
    }                                                                                                            \
    OptimizeShape NAME() { return {NAME##_occupancy, NAME##_spill, NAME##_launch}; }

}  // namespace pt
