// prune.hip -- the likelihood with no partial stored, on the matrix cores.
//
// Felsenstein's post-order pass with every partial of a pattern in registers
// (see lanes.hpp for the layout).  A wave owns NI items of Lanes<KP>::kCols
// patterns, all categories of them, and runs its tree's register program
// alone: no barrier until the tile's sum.
//
// Bound: FP64 arithmetic (68 flops per pattern, category and update; the
// matrix cores run FP64 at the vector rate, and do not overlap with it).
// What the layout buys is everything around the products: a transition
// matrix is one coalesced 512-byte load for all categories, made one op
// ahead, and no entry is broadcast to lanes or passes through scalar
// registers.  A tip's product is no product at all: the wave writes the
// matrix's columns to LDS once and every lane reads the entry its pattern's
// code selects, which replaces half of a tree's products.
//
// Measured against the kernel that multiplied on the vector units, a category
// per wave with every matrix entry read by scalar loads (whole likelihood
// call, MI355X): 48 trees of 27 taxa x 976 patterns 45.0 -> 18.3 us; 512
// trees over four alignments 271 -> 140 us (21 -> 41 TFLOP/s).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "lanes.hpp"

namespace pt {
namespace {

constexpr double kLn2 = 0.69314718055994530942;
constexpr int kPruneWaves = 4;             // waves per block, each on its own patterns of one tree
constexpr int kRow = 136;                  // bytes of a tip table's row: 16 codes, 8 bytes of padding

// LDS bytes of a wave: the two tip tables of an op, then the tip codes.
template <int KP>
constexpr size_t table_bytes() {
    return (size_t)Lanes<KP>::NQ * Lanes<KP>::CB * 4 * kRow;
}

// Transition matrices of every edge in lane order (see mat_index): one thread
// per (edge, category), a block per kPmatChunk of them, all of one tree, so
// that the tree's descriptor and model arrive by scalar loads.  The entries
// are those of k_pmat, by the same expressions.
// (128 threads in several blocks per tree: 10.7 us on the 512 trees of the
// header, against 12.9 with one block of 256 per tree.)
constexpr int kPmatChunk = 128;

template <int KP>
__global__ void __launch_bounds__(kPmatChunk) k_pmat_lanes(const BatchArgs a, const double *brlen, int chunks) {
    using CD = const __attribute__((address_space(4))) double;
    constexpr int CB = Lanes<KP>::CB;
    const __attribute__((address_space(4))) TreeDev *td =
        (const __attribute__((address_space(4))) TreeDev *)(a.trees + blockIdx.x / chunks);
    const __attribute__((address_space(4))) AlnDev *aln =
        (const __attribute__((address_space(4))) AlnDev *)(a.alns + td->aln);
    const int x = (int)(blockIdx.x % chunks) * kPmatChunk + threadIdx.x;
    if (x >= td->n_edges * KP) return;
    const int e = x / KP, k = x % KP;
    const double t = brlen[td->edge_off + e];
    CD *U = aln->U, *V = aln->Uinv;
    double ex[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) ex[m] = exp(aln->lam[m] * aln->rate[k] * t);
    double *out = a.pmat + td->pm_off + (size_t)e * KP * 16 + (size_t)(k / CB) * Lanes<KP>::kMat + k % CB * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < 4; ++m) s += U[i * 4 + m] * ex[m] * V[m * 4 + j];
            p[i] = s;
        }
        double2 *o = reinterpret_cast<double2 *>(out + j * CB * 4);
        o[0] = make_double2(p[0], p[1]);
        o[1] = make_double2(p[2], p[3]);
    }
}

typedef uint32_t __attribute__((aligned(1))) UnalignedWord;

// One wave's view of its tile.
template <int KP, int NI>
struct Wave {
    static constexpr int NR = NI * Lanes<KP>::NQ;           // registers of one partial
    static constexpr int kPats = NI * Lanes<KP>::kCols;     // patterns
    static constexpr int kWords = (NI + 3) / 4;             // 32-bit words of a column's codes
};

// The tip codes of a wave's patterns into LDS, [taxon][kPats] bytes of
// 8 * code (a row offset of the tip tables); a pattern past the end reads
// as state A.  Column c of item it is pattern c * NI + it, so a lane's codes
// of one taxon are NI consecutive bytes.  Returns whether any code stands for
// more than one state.
template <int KP, int NI>
__device__ inline bool stage_tips(const uint8_t *tips, int n, int P, int p0, uint8_t *lds) {
    constexpr int WP = Wave<KP, NI>::kPats, kCol = WP / 4, kStep = 64 / kCol;  // words of a row; rows of one step
    static_assert(WP % 4 == 0 && 64 % kCol == 0, "rows of whole words");
    constexpr int kDeep = kCol < 8 ? kCol : 8;  // steps whose loads are in flight together: 64 taxa or more
    const int lane = threadIdx.x & 63, p = p0 + lane % kCol * 4;
    const uint8_t *src = tips + p;
    uint32_t *dst = reinterpret_cast<uint32_t *>(lds) + lane;
    uint32_t many = 0;
    for (int t0 = lane / kCol; t0 < n; t0 += kDeep * kStep, dst += kDeep * 64) {
        uint32_t w[kDeep];
        if (p + 4 <= P) {
            // the row's start has any alignment; a row past the last is read
            // from the last
#pragma unroll
            for (int u = 0; u < kDeep; ++u)
                w[u] = *(const __attribute__((address_space(1))) UnalignedWord *)(src + (size_t)min(t0 + u * kStep, n - 1) * P);
        } else {
            for (int u = 0; u < kDeep; ++u) {
                w[u] = 0x01010101u;
                const uint8_t *r = src + (size_t)min(t0 + u * kStep, n - 1) * P;
                for (int b = 0; b < 4; ++b)
                    if (p + b < P) w[u] = (w[u] & ~(0xffu << (8 * b))) | ((uint32_t)r[b] << (8 * b));
            }
        }
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            many |= w[u] & (w[u] - 0x01010101u);
            if (t0 + u * kStep < n) dst[u * 64] = w[u] << 3;
        }
    }
    wave_lds_fence();
    return __builtin_amdgcn_readfirstlane(__any(many != 0));
}

// Writes the products of a matrix register with the 16 codes' vectors as a
// tip table: row (i, category), entry `code`.  With `many` unset only the
// one-state codes are read, whose products are the matrix's columns.
template <int KP>
__device__ inline void write_table(const double *A, char *tab, bool many) {
    using L = Lanes<KP>;
    const int lane = threadIdx.x & 63, hi = lane >> 4, blk = (lane >> 2) & 3, lo = lane & 3;
#pragma unroll
    for (int q = 0; q < L::NQ; ++q) {
        char *t = tab + q * (L::CB * 4 * kRow) + blk % L::CB * kRow;
        if (!many) {
            *reinterpret_cast<double *>(t + lo * (L::CB * kRow) + (8 << hi)) = A[q];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double bit = (double)(((4 * c + lo) >> hi) & 1);
                *reinterpret_cast<double *>(t + hi * (L::CB * kRow) + (4 * c + lo) * 8) = mfma4(A[q], bit);
            }
        }
    }
    wave_lds_fence();
}

// The entries of a tip table that this lane's codes select, item by item:
// y[it * NQ + q].
template <int KP, int NI>
__device__ inline void read_table(const char *tab, const uint32_t *w, double *y) {
    using L = Lanes<KP>;
    const int lane = threadIdx.x & 63;
    const char *t = tab + (lane >> 4) * (L::CB * kRow) + ((lane >> 2) & 3) % L::CB * kRow;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const uint32_t off = (w[it / 4] >> (8 * (it % 4))) & 0xffu;
#pragma unroll
        for (int q = 0; q < L::NQ; ++q)
            y[it * L::NQ + q] = *reinterpret_cast<const double *>(t + q * (L::CB * 4 * kRow) + off);
    }
}

// This lane's column's codes of one taxon.
template <int KP, int NI>
__device__ inline void read_codes(const uint8_t *tips, int taxon, uint32_t *w) {
    using L = Lanes<KP>;
    const int lane = threadIdx.x & 63, col = ((lane >> 2) & 3) / L::CB * 4 + (lane & 3);
    const uint8_t *p = tips + (size_t)taxon * Wave<KP, NI>::kPats + col * NI;
    if constexpr (NI == 8) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        w[0] = v.x;
        w[1] = v.y;
    } else if constexpr (NI == 4) {
        w[0] = *reinterpret_cast<const uint32_t *>(p);
    } else {
        static_assert(NI == 2, "two, four or eight items");
        w[0] = *reinterpret_cast<const uint16_t *>(p);
    }
}

// Scaling per pattern and category: a partial whose largest entry is below
// 2^-256 (and not zero) is multiplied by 2^256 and the event counted.  The
// common case is settled for all items at once on the high words, compared as
// signed numbers: an entry below zero (a matrix has its zeros to a rounding of
// either sign) is small, as zero is.  Only when some entry of the wave is below
// the threshold are the largest entries looked at, by folding lane masks.
template <int NR>
__device__ inline void scale_partials(double *y, int *cnt) {
    constexpr int kThr = (1023 - 256) << 20;  // high word of 2^-256
    int m = __double2hiint(y[0]);
#pragma unroll
    for (int r = 1; r < NR; ++r) m = min(m, __double2hiint(y[r]));
    if (!__any(m < kThr)) return;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        // bit (b, j): some entry of that category and column
        unsigned long long big = __ballot(y[r] >= 0x1p-256), any = __ballot(y[r] > 0.0);
        big |= big >> 32;
        big |= big >> 16;
        any |= any >> 32;
        any |= any >> 16;
        const uint32_t need = (uint32_t)(any & ~big) >> (lane & 15) & 1u;
        y[r] *= need ? 0x1p256 : 1.0;
        cnt[r] += need;
    }
}

// x = the partial in stack slot `slot`, times the matrix m unless m is null.
template <int RS, int NR, int NQ, int S = 0>
__device__ __attribute__((always_inline)) inline void from_slot(int slot, const double (&stk)[RS][NR], const double *m,
                                                                double *x) {
    if (S == RS - 1 || slot == S) {
#pragma unroll
        for (int r = 0; r < NR; ++r) x[r] = m ? mfma4(m[r % NQ], stk[S][r]) : stk[S][r];
        asm volatile("; slot %0" ::"n"(S));  // see the stores
    } else if constexpr (S < RS - 1) {
        from_slot<RS, NR, NQ, S + 1>(slot, stk, m, x);
    }
}

// k_prune: lnL of a tile of kPruneWaves * kPats patterns of one tree.
// Programs come from compile_loglik_reg: OP_RUPDATE with side forms (tip,
// tip), (accumulator, tip), (stack, accumulator), its dst the stack slot the
// result is kept in (-1: it stays the accumulator); OP_REVAL ends it.  The
// stack is in registers, a slot chosen by wave-uniform branches; RS slots.
// Waves per SIMD asked of the compiler, the most that need no scratch memory
// (also two or more let it keep the products in ordinary registers).  A deep
// stack of the most items takes one: only a no-allocation batch that would not
// fit its workspace otherwise runs it, and at two it spilled 8 to 24 bytes a lane.
template <int KP, int NI, int RS>
constexpr int prune_waves() {
    constexpr bool kMost = NI * Lanes<KP>::NQ == 8;
    return RS > 3 ? (kMost ? 1 : 2) : kMost ? 3 : 5;
}

template <int KP, int NI, int RS>
__global__ void __launch_bounds__(64 * kPruneWaves) __attribute__((amdgpu_waves_per_eu(prune_waves<KP, NI, RS>())))
k_prune(const BatchArgs a) {
    using L = Lanes<KP>;
    using Wv = Wave<KP, NI>;
    constexpr int NR = Wv::NR, NQ = L::NQ;
    extern __shared__ char lds[];
    __shared__ double sums[kPruneWaves];
    // a tree's descriptors have its index: both load at once
    const int b = a.tile_tree[blockIdx.x], sub_of = a.tile_of ? a.tile_of[blockIdx.x] : 0;
    const TreeDev td = a.trees[b];
    const AlnDev *aln = a.alns + b;
    const int sub = a.tile_of ? sub_of : (int)blockIdx.x - td.tile_begin;
    const int P = aln->P, n = aln->n_taxa, K = aln->K;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int p0 = sub * (kPruneWaves * Wv::kPats) + wave * Wv::kPats;
    double term = 0.0;
    if (p0 < P) {
        constexpr size_t kTab = table_bytes<KP>();
        char *tab = lds + (size_t)wave * (2 * kTab + (size_t)a.reg_taxa * Wv::kPats);
        uint8_t *tips = reinterpret_cast<uint8_t *>(tab + 2 * kTab);
        const bool many = stage_tips<KP, NI>(aln->tips, n, P, p0, tips);
        const MatRows<KP> pm(a.pmat + td.pm_off, td.n_edges, lane);
        double acc[NR], stk[RS][NR];
        int cnt[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            acc[r] = 0.0;
            cnt[r] = 0;
        }
        auto tip_side = [&](const uint32_t *w, const double *m, char *t, double *y) __attribute__((always_inline)) {
            write_table<KP>(m, t, many);
            read_table<KP, NI>(t, w, y);
        };
        // The next op's matrices and tip codes are loaded while this one runs,
        // and the op after it, so that their addresses are known in time.
        // (The op read past the root's, which ends the program, is not used.)
        const Op *prog = a.ops + td.op_first;
        Op op = load_op(prog, 0), nx = load_op(prog, 1);
        double ma[NQ], mb[NQ];
        uint32_t wa[Wv::kWords], wb[Wv::kWords];
        auto fetch = [&](const Op &f, double *fa, double *fb, uint32_t *ca, uint32_t *cb) __attribute__((always_inline)) {
            pm.load(f.ea, fa);
            pm.load(f.eb, fb);
            read_codes<KP, NI>(tips, f.tip_a, ca);
            read_codes<KP, NI>(tips, f.tip_b, cb);
        };
        fetch(op, ma, mb, wa, wb);
        for (int o = td.n_first - 1; o > 0; --o) {
            double na[NQ], nb[NQ];
            uint32_t va[Wv::kWords], vb[Wv::kWords];
            fetch(nx, na, nb, va, vb);
            const Op nn = load_op(prog, 2);
            ++prog;
            double xa[NR], xb[NR];
            if (op.b >= 0) {  // side b is a tip, side a a tip or the accumulator
                tip_side(wb, mb, tab + kTab, xb);
                if (op.a >= 0) {
                    tip_side(wa, ma, tab, xa);
                } else {
#pragma unroll
                    for (int r = 0; r < NR; ++r) xa[r] = mfma4(ma[r % NQ], acc[r]);
                }
            } else {  // side a is a stack slot, side b the accumulator
                from_slot<RS, NR, NQ>(REF_STACK0 - op.a, stk, ma, xa);
#pragma unroll
                for (int r = 0; r < NR; ++r) xb[r] = mfma4(mb[r % NQ], acc[r]);
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = xa[r] * xb[r];
            scale_partials<NR>(acc, cnt);
            if (op.dst >= 0) {
#pragma unroll
                for (int s = 0; s < RS; ++s)
                    if (s == op.dst) {
#pragma unroll
                        for (int r = 0; r < NR; ++r) stk[s][r] = acc[r];
                        // keeps the branches apart: merged, they would store
                        // through a pointer and send the stack to scratch memory
                        asm volatile("; slot %0" ::"n"(s));
                    }
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                ma[q] = na[q];
                mb[q] = nb[q];
            }
#pragma unroll
            for (int q = 0; q < Wv::kWords; ++q) {
                wa[q] = va[q];
                wb[q] = vb[q];
            }
            op = nx;
            nx = nn;
        }
        {   // the root edge: side a as it is, side b across the edge
            double xa[NR], xb[NR];
            if (op.b >= 0) {
                tip_side(wb, mb, tab + kTab, xb);
                if (op.a >= 0) {
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        xa[r] = (double)((wa[r / NQ / 4] >> (8 * (r / NQ % 4) + 3 + (lane >> 4))) & 1u);
                } else {
#pragma unroll
                    for (int r = 0; r < NR; ++r) xa[r] = acc[r];
                }
            } else {
                from_slot<RS, NR, NQ>(REF_STACK0 - op.a, stk, nullptr, xa);
#pragma unroll
                for (int r = 0; r < NR; ++r) xb[r] = mfma4(mb[r % NQ], acc[r]);
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = xa[r] * xb[r];
        }
        // L of every pattern and category: the sum over states weighted by
        // the frequencies, in every row of the result
        const double freq = aln->freqs[lane >> 4];
        double Lk[NI];
        int ck[NI];
        const int blk = (lane >> 2) & 3;
        int scaled = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) scaled |= cnt[r];
        const bool any_scaled = __any(scaled != 0);
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            double v[NQ];
            int cm = 0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[q] = mfma4(freq, acc[it * NQ + q]);
            if (any_scaled) {
                // to the least scaled of the pattern's categories
                cm = 0x7fffffff;
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (q * L::CB + blk % L::CB < K) cm = min(cm, cnt[it * NQ + q]);
#pragma unroll
                for (int x = 4; x < 4 * L::CB; x <<= 1) cm = min(cm, __shfl_xor(cm, x));
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (q * L::CB + blk % L::CB < K) v[q] = ldexp(v[q], -256 * (cnt[it * NQ + q] - cm));
            }
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q * L::CB + blk % L::CB < K) s += v[q];
            // over the row's lanes of the same column: rotations by 8 and 4
            if constexpr (L::CB == 4) s += row_ror<8>(s);
            if constexpr (L::CB == 2) s += __shfl_xor(s, 4);
            if constexpr (L::CB == 4) s += row_ror<4>(s);
            Lk[it] = s;
            ck[it] = cm;
        }
        // every row and category lane of a column holds its NI values: each
        // takes the logarithm of its own share of them
        constexpr int kShare = 4 * L::CB;
        const int mine = (lane >> 4) * L::CB + blk % L::CB, col = blk / L::CB * 4 + (lane & 3);
#pragma unroll
        for (int r = 0; r < (NI + kShare - 1) / kShare; ++r) {
            double v = 1.0;
            int c = 0;
#pragma unroll
            for (int it = r * kShare; it < NI && it < (r + 1) * kShare; ++it)
                if (it == r * kShare + mine) {
                    v = Lk[it];
                    c = ck[it];
                }
            const int it = r * kShare + mine, p = p0 + col * NI + it;
            if (it < NI && p < P)
                term += *(const __attribute__((address_space(1))) double *)(aln->w + p) *
                        (log(v) - aln->log_k - (double)c * 256.0 * kLn2);
        }
    }
    term = wave_sum(term);
    if (lane == 0) sums[wave] = term;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kPruneWaves; ++w) s += sums[w];
        a.part[td.tile_begin + sub] = s;
    }
}

// lnL of every tree from its tiles, in tile order.
__global__ void k_tile_sums(const BatchArgs a, double *lnl) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.n_trees) return;
    const int n = a.trees[b].n_tiles;
    const double *p = a.part + a.trees[b].tile_begin;
    double s = 0.0;
    int t = 0;
    for (; t + 8 <= n; t += 8) {  // eight loads in flight, added in order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[t + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; t < n; ++t) s += p[t];
    if (a.keep_nan && isnan(lnl[b])) return;
    if (a.prior_rate > 0.0) {
        // independent Exponential(rate) priors: sum_e (log rate - rate t_e)
        const double lr = log(a.prior_rate);
        double q = 0.0;
        for (int e = 0; e < a.trees[b].n_edges; ++e) q += lr - a.prior_rate * a.brlen[a.trees[b].edge_off + e];
        s += q;
    }
    lnl[b] = s;
}

#define PT_KP_SWITCH(...)                                   \
    switch (kp) {                                           \
    case 1: { constexpr int KP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int KP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int KP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int KP = 8; __VA_ARGS__; } break;   \
    default: break;                                         \
    }
#define PT_NI_SWITCH(...)                                   \
    switch (items) {                                        \
    case 2: { constexpr int NI = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int NI = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int NI = KP < 8 ? 8 : 4; __VA_ARGS__; } break; \
    default: break;                                         \
    }

template <int KP, int NI, int RS>
hipError_t launch_prune_t(const BatchArgs &a, size_t lds, hipStream_t s) {
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_prune<KP, NI, RS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_prune<KP, NI, RS>), dim3(a.n_tiles), dim3(64 * kPruneWaves), lds, s, a);
    return hipGetLastError();
}

}  // namespace

int prune_tile_patterns(int kp, int items) {
    PT_KP_SWITCH(return kPruneWaves * items * Lanes<KP>::kCols);
    return 0;
}

int prune_max_items(int kp) { return kp < 8 ? 8 : 4; }

size_t prune_lds(int kp, int items, int n) {
    PT_KP_SWITCH(return kPruneWaves * (2 * table_bytes<KP>() + (size_t)n * items * Lanes<KP>::kCols));
    return 0;
}

hipError_t launch_pmat_lanes(const BatchArgs &a, const double *brlen, int max_edges, hipStream_t s) {
    if (a.n_edges <= 0) return hipSuccess;
    const int kp = a.kp, chunks = (max_edges * kp + kPmatChunk - 1) / kPmatChunk;
    PT_KP_SWITCH({
        hipLaunchKernelGGL((k_pmat_lanes<KP>), dim3((unsigned)a.n_trees * chunks), dim3(kPmatChunk), 0, s, a, brlen,
                           chunks);
        return hipGetLastError();
    });
    return hipErrorInvalidValue;
}

hipError_t launch_prune(const BatchArgs &a, int items, double *lnl, hipStream_t s) {
    if (a.n_tiles <= 0) return hipSuccess;
    const int kp = a.kp;
    const size_t lds = prune_lds(kp, items, a.reg_taxa);
    hipError_t e = hipErrorInvalidValue;
    PT_KP_SWITCH(PT_NI_SWITCH(e = a.reg_depth <= 3   ? launch_prune_t<KP, NI, 3>(a, lds, s)
                                  : launch_prune_t<KP, NI, kRegStack>(a, lds, s)));
    if (e != hipSuccess || !lnl) return e;
    hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)((a.n_trees + 63) / 64)), dim3(64), 0, s, a, lnl);
    return hipGetLastError();
}

}  // namespace pt
