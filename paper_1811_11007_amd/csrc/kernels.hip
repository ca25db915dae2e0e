// kernels.hip -- CDNA4 (gfx950) kernels of the tree likelihood.
//
// Work decomposition.  One thread owns one site pattern at a time and
// handles all of its rate categories, so the per-pattern scaling decision,
// the sum over categories and the logarithm stay inside the thread.  Partials
// are stored category-major per slot, [slot][Kp][P][4], so for a fixed
// category a wavefront's 64 patterns are one contiguous 1 KiB (FP32) or
// 2 KiB (FP64) block: every load and store is fully coalesced.  Transition
// matrices sit in LDS and are read with wave-uniform addresses (broadcast).
//
// Numerics.  Partials may be stored in FP32; every product, transition
// matrix, logarithm and sum over patterns is FP64.  Per-pattern scaling
// multiplies a new partial by 2^S (S = 64 for FP32 storage, 256 for FP64)
// when its largest entry over categories and states falls below 2^-S, and
// counts the event in a per-pattern scaler; scaling by a power of two is
// exact, so it changes no value.
//
// Sums over patterns are fixed-order: butterfly within a wavefront, then the
// per-wave partials in wave order, then the tiles of a tree in tile order (or,
// for a tree optimised by several blocks, the blocks in block order), so a
// rerun is bit-identical.
//
// Kernels: k_pmat (transition matrices), k_tiles32 / k_tiles64 (a tree's
// stored post-order pass over one pattern tile), k_reduce (tile sums in
// order); in optimize.hpp k_optimize (the whole branch-length smoothing loop
// of a tree, one block per tree or one tree split over several blocks).  The
// likelihood that stores nothing and the gradient are in prune.hip and
// grad.hip.
#include "partials.hpp"

namespace pt {
namespace {

// ----------------------------------------------------------------- kernels

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Transition matrices of every edge, P_k(t) = U diag(exp(lambda r_k t)) U^-1:
// one block per tree, so that the tree's descriptor and model constants are
// wave-uniform and arrive by scalar loads (neither is written by any kernel),
// and one thread per (edge, category k) of the tree.  The four exponentials
// serve the matrix's 16 entries, written as 16-byte stores.
__global__ void k_pmat(const BatchArgs a, const double *brlen) {
    using CD = const __attribute__((address_space(4))) double;
    const __attribute__((address_space(4))) TreeDev *td =
        (const __attribute__((address_space(4))) TreeDev *)(a.trees + blockIdx.x);
    const __attribute__((address_space(4))) AlnDev *aln =
        (const __attribute__((address_space(4))) AlnDev *)(a.alns + td->aln);
    const int kp = a.kp, n = td->n_edges * kp;
    const int64_t edge_off = td->edge_off, pm_off = td->pm_off;
    for (int x = threadIdx.x; x < n; x += blockDim.x) {
        const int e = x / kp, k = x - e * kp;
        const double t = brlen[edge_off + e];
        CD *U = aln->U, *V = aln->Uinv;
        double ex[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) ex[m] = exp(aln->lam[m] * aln->rate[k] * t);
        double2 *out = reinterpret_cast<double2 *>(a.pmat + pm_off + (int64_t)x * 16);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            double s2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = (2 * q + h) >> 2, j = (2 * q + h) & 3;
                double s = 0.0;
#pragma unroll
                for (int m = 0; m < 4; ++m) s += U[i * 4 + m] * ex[m] * V[m * 4 + j];
                s2[h] = s;
            }
            out[q] = make_double2(s2[0], s2[1]);
        }
    }
}

// OP_UPDATE for one pattern per thread whose side `fwd_b ? b : a` is the
// partial the previous update of this thread made, still in registers
// (`last`): only the other side is loaded.  The new partial is stored and
// kept in `last` for the next update.  The same expressions as
// update_sides, so the partials are identical.
template <typename T, int KP, bool TO, int PM>
__device__ inline void update_forwarded(const TreeView<T> &v, const Op &op, bool fwd_b, int p,
                                        Side<T, KP, false> &last) {
    Side<T, KP, TO> so;
    so.fetch(v, fwd_b ? op.a : op.b, p);
    double o[KP][4];
    const int c = fwd_b ? update_pattern<T, KP, PM>(v, op, so, last, o) : update_pattern<T, KP, PM>(v, op, last, so, o);
#pragma unroll
    for (int k = 0; k < KP; ++k) last.r[k] = Store<T>::pack(o[k]);
    last.c = c;
#pragma unroll
    for (int k = 0; k < KP; ++k)
        if (k < v.K) Store<T>::store_raw(slot_ptr<T, KP>(v, op.dst, k, p), last.r[k]);
    v.cnt[(size_t)op.dst * v.P + p] = (uint16_t)c;
}

// OP_UPDATE for one pattern per thread with both sides loaded, keeping the
// new partial in `last` (update_sides with the result kept).
template <typename T, int KP, bool TA, bool TB, int PM>
__device__ inline void update_keep(const TreeView<T> &v, const Op &op, int p, Side<T, KP, false> &last) {
    Side<T, KP, TA> sa;
    Side<T, KP, TB> sb;
    sa.fetch(v, op.a, p);
    sb.fetch(v, op.b, p);
    double o[KP][4];
    last.c = update_pattern<T, KP, PM>(v, op, sa, sb, o);
#pragma unroll
    for (int k = 0; k < KP; ++k) last.r[k] = Store<T>::pack(o[k]);
#pragma unroll
    for (int k = 0; k < KP; ++k)
        if (k < v.K) Store<T>::store_raw(slot_ptr<T, KP>(v, op.dst, k, p), last.r[k]);
    v.cnt[(size_t)op.dst * v.P + p] = (uint16_t)last.c;
}

// Requests one update's transition matrices (edges ea and eb, KP categories
// each) into the L2 ahead of use: one 16-byte LDS DMA per lane of the calling
// wave into `row`, which nobody reads.  The FP32 tile kernel reads the
// matrices by scalar loads, which its register budget serialises in pairs
// per update; issued one op early, these requests let those loads find the
// lines in the L2 instead of going out to memory one pair after another.
template <int KP>
__device__ inline void prefetch_pm(const double *pm, int ea, int eb, float4 *row) {
    constexpr int kChunks = KP * 8;  // 16-byte pieces of one edge's KP matrices
    const int lane = threadIdx.x & 63;
    if (lane < 2 * kChunks) {
        const double *src = pm + ((size_t)(lane < kChunks ? ea : eb) * KP) * 16 + (lane % kChunks) * 2;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                         (__attribute__((address_space(3))) void *)row, 16, 0, 0);
    }
}

// Pattern-tile kernels (k_tiles32 / k_tiles64 below): each block runs its tree's LOGLIK program, which ends in one
// EVAL, over one tile of BS * kTileItems patterns.  Output: part[tile] = lnL.
template <typename T, int BS, int KP>
__device__ inline void tiles_body(const BatchArgs &a, const double *brlen) {
    extern __shared__ double lds[];
    __shared__ double red[2 * (BS / 64) * 3];
    __shared__ double wxs[(BS / 64) * kWx];
    __shared__ ModelS model;
    __shared__ float4 pf_row[64];  // target of prefetch_pm, never read
    // FP32 partials: the updates read the tree's transition matrices (written
    // by k_pmat before this launch) in place by scalar loads (see PmPtr);
    // FP64 partials: from a copy in LDS, which measured faster there.
    constexpr bool kConstPm = std::is_same<T, float>::value;
    const int tile = blockIdx.x;
    const TreeDev td = a.trees[a.tile_tree[tile]];
    const AlnDev *aln = a.alns + td.aln;
    if (!kConstPm) {
        // 16-byte loads, four in flight per thread (indices clamped into
        // range, so no branch separates the loads)
        const int n2 = td.n_edges * KP * 8;
        const double2 *src = reinterpret_cast<const double2 *>(a.pmat + td.pm_off);
        double2 *dst = reinterpret_cast<double2 *>(lds);
        for (int i = threadIdx.x; i < n2; i += 4 * BS) {
            double2 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = src[min(i + u * BS, n2 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * BS < n2) dst[i + u * BS] = q[u];
        }
    }
    model_to_lds(aln, &model);
    __syncthreads();
    const TreeView<T> v = make_view<T>(td, aln, a, &model, kConstPm ? a.pmat + td.pm_off : lds);
    double *wx = wxs + (threadIdx.x >> 6) * kWx;
    const int base = (tile - td.tile_begin) * BS * kTileItems;
    int parity = 0;
    // FP64 partials, one pattern per thread: a partial the previous update
    // made is taken from registers when this update reads it (a post-order
    // pass reads most partials right after making them), saving that load's
    // round trip.  With FP32 partials the extra live registers cost more than
    // the load (measured), so those updates load both sides.
    constexpr int PMK = kConstPm ? kPmConst : kPmLds;
    constexpr bool kForward = !kConstPm;
    static_assert(kTileItems == 1, "partials are forwarded for one pattern per thread");
    const int p = base + threadIdx.x;
    const bool live_p = p < v.np;
    Side<T, KP, false> last;
    int last_dst = -1;
    // FP32 partials: the first wave requests each update's matrices into the
    // L2 one op ahead of the update
    if constexpr (kConstPm) {
        if (threadIdx.x < 64 && td.n_first > 0) {
            const Op nx = load_op(a.ops, td.op_first);
            if (nx.code == OP_UPDATE) prefetch_pm<KP>(a.pmat + td.pm_off, nx.ea, nx.eb, pf_row);
        }
    }
    for (int o = 0; o < td.n_first; ++o) {
        const Op op = load_op(a.ops, td.op_first + o);
        if constexpr (kConstPm) {
            if (threadIdx.x < 64 && o + 1 < td.n_first) {
                const Op nx = load_op(a.ops, td.op_first + o + 1);
                if (nx.code == OP_UPDATE) prefetch_pm<KP>(a.pmat + td.pm_off, nx.ea, nx.eb, pf_row);
            }
        }
        if (op.code == OP_UPDATE && !kForward) {
            do_update<T, BS, KP, PMK>(v, op, base, kTileItems);
            continue;
        }
        if (op.code == OP_UPDATE) {
            if (live_p) {
                if (op.b >= 0 && op.b == last_dst) {
                    if (op.a < 0) update_forwarded<T, KP, true, PMK>(v, op, true, p, last);
                    else update_forwarded<T, KP, false, PMK>(v, op, true, p, last);
                } else if (op.a >= 0 && op.a == last_dst) {
                    if (op.b < 0) update_forwarded<T, KP, true, PMK>(v, op, false, p, last);
                    else update_forwarded<T, KP, false, PMK>(v, op, false, p, last);
                } else if (op.a < 0) {
                    if (op.b < 0) update_keep<T, KP, true, true, PMK>(v, op, p, last);
                    else update_keep<T, KP, true, false, PMK>(v, op, p, last);
                } else {
                    if (op.b < 0) update_keep<T, KP, false, true, PMK>(v, op, p, last);
                    else update_keep<T, KP, false, false, PMK>(v, op, p, last);
                }
            }
            last_dst = op.dst;
            continue;
        }
        const Sums3 r = eval_edge<T, BS, KP>(v, op.a, op.b, base, kTileItems, brlen[td.edge_off + op.dst], red, wx,
                                             parity);
        parity = r.parity;
        if (threadIdx.x == 0) a.part[tile] = r.l0;
    }
}

// The tile kernels.  With FP32 partials the kernel is held to 128 VGPRs
// (four blocks per CU), which measured 7 % faster despite a 48-byte spill
// outside the update loop; with FP64 partials the LDS copy of the matrices
// already limits a CU to two blocks.
template <int BS, int KP>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4)))
k_tiles32(const BatchArgs a, const double *brlen) {
    tiles_body<float, BS, KP>(a, brlen);
}

template <int BS, int KP>
__global__ void __launch_bounds__(BS) k_tiles64(const BatchArgs a, const double *brlen) {
    tiles_body<double, BS, KP>(a, brlen);
}

// lnL of every tree from its tiles, in tile order.
__global__ void k_reduce(const BatchArgs a, double *lnl) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_trees) return;
    const TreeDev &td = a.trees[i];
    double s = 0.0;
    for (int t = 0; t < td.n_tiles; ++t) s += a.part[td.tile_begin + t];
    lnl[i] = s;
}

// ------------------------------------------------------------- dispatch

template <typename T, int BS, int KP>
hipError_t launch_tiles_t(const BatchArgs &a, const double *brlen, size_t lds, hipStream_t s) {
    if (std::is_same<T, float>::value) {
        hipLaunchKernelGGL((k_tiles32<BS, KP>), dim3(a.n_tiles), dim3(BS), 0, s, a, brlen);
        return hipGetLastError();
    }
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_tiles64<BS, KP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_tiles64<BS, KP>), dim3(a.n_tiles), dim3(BS), lds, s, a, brlen);
    return hipGetLastError();
}

}  // namespace

bool optimize_shape_supported(int block, int items) {
    return (block == 256 || block == 512) && items >= 1 && items <= 64;
}

namespace {

// The instantiations for a precision and block size (256 or 512, see
// optimize_shape_supported).
OptimizeShape optimize_shape(int precision, int block) {
    if (block == 256) return precision == PT_FP32 ? optimize_f32_256() : optimize_f64_256();
    return precision == PT_FP32 ? optimize_f32_512() : optimize_f64_512();
}

}  // namespace

int optimize_blocks_per_cu(int precision, int block, int kp, bool tab_lds, bool grouped, size_t lds) {
    return optimize_shape(precision, block).occupancy(kp, tab_lds, grouped, lds);
}

size_t optimize_spill_bytes(int precision, int block, int kp, bool tab_lds, bool grouped) {
    return optimize_shape(precision, block).spill(kp, tab_lds, grouped);
}

hipError_t launch_optimize(int precision, int block, int kp, int items, bool tab_lds, int pm_doubles, int grid,
                           const BatchArgs &a, double *brlen, const OptParams &opt, double *lnl, int32_t *passes,
                           int32_t *status, size_t lds, hipStream_t s) {
    return optimize_shape(precision, block).launch(kp, items, tab_lds, pm_doubles, grid, a, brlen, opt, lnl, passes,
                                                   status, lds, s);
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_pmat(const BatchArgs &a, const double *brlen, hipStream_t s) {
    if (a.n_edges <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pmat, dim3((unsigned)a.n_trees), dim3(256), 0, s, a, brlen);
    return hipGetLastError();
}

bool tile_patterns_supported(int pats) { return pats == 64 || pats == 128 || pats == 256; }

hipError_t launch_tiles(int precision, int kp, int tile_pats, const BatchArgs &a, const double *brlen, size_t lds,
                        hipStream_t s) {
    if (a.n_tiles <= 0) return hipSuccess;
#define PT_TILES_BS(BSZ)                                                                             \
    PT_KP_SWITCH(return precision == PT_FP32 ? launch_tiles_t<float, BSZ, KP>(a, brlen, lds, s) \
                                             : launch_tiles_t<double, BSZ, KP>(a, brlen, lds, s))
    if (tile_pats == 64) PT_TILES_BS(64);
    if (tile_pats == 128) PT_TILES_BS(128);
    if (tile_pats == 256) PT_TILES_BS(256);
#undef PT_TILES_BS
    return hipErrorInvalidValue;
}

hipError_t launch_reduce(const BatchArgs &a, double *lnl, hipStream_t s) {
    if (a.n_trees <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce, dim3((unsigned)((a.n_trees + 255) / 256)), dim3(256), 0, s, a, lnl);
    return hipGetLastError();
}

}  // namespace pt
