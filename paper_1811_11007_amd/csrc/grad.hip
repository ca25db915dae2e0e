// grad.hip -- lnL and every edge derivative of a batch of trees on the matrix
// cores: one post-order and one pre-order sweep per wave (layout: lanes.hpp).
//
// Everything is kept in the eigenbasis of the rate matrix, P(t) = U e(t) U^-1:
// a side's coefficients b = U^-1 x are what an edge's derivatives need (lnL =
// sum e a b over the two sides a, b; each derivative one more factor lam r),
// and what the product P(t) x = U (e b) needs, so an edge's only operand is
// its exponentials, 4 per category, and the matrices U and U^-1 stay in
// registers.  Per internal node the post-order sweep stores one partial and
// the pre-order sweep reads it back; the partials of the rest of the tree
// seen from a node (its outer partials) live in registers along the descent,
// one of two stored where it branches.  (The dependency program this replaces
// stored all 3 (n - 2) directional partials and re-read each up to four
// times.)
//
// With FP32 partials every directional partial, inner or outer, is rounded to
// FP32 under the stored pass's scaling rule where that pass would store it,
// so both compute the same derivatives; products and sums are FP64.
//
// Bound: FP64 arithmetic (matrix and vector instructions share the issue),
// then the partials' traffic: one write and one read per internal node.
// Measured against that dependency program (MI355X, a whole call): 256 trees of
// 50 taxa x 1250 patterns, FP32 partials 2214 -> 1214 us; 48 of 64 x 1711, FP64,
// through torch forward and backward 1414 -> 602 us; one of 27 x 976 with
// second derivatives, from host arrays 448 -> 194 us.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"
#include "lanes.hpp"
#include "pt.h"

namespace pt {
namespace {

constexpr double kLn2 = 0.69314718055994530942;
constexpr int kGradWaves = 4;  // waves per block, each on its own patterns of one tree
constexpr int kGradItems = 4;  // items per wave
constexpr int kBuf = 8;        // edges whose sums over a wave's lanes are formed together
constexpr int kTipRow = 17;    // doubles of a row of the tips' coefficients (16 codes)

typedef uint32_t __attribute__((aligned(1))) UnalignedWord;

template <typename T>
struct Round;  // what storing a partial does to it

template <>
struct Round<float> {
    static constexpr int kThr = (1023 - 64) << 20;  // high word of 2^-64
    static constexpr double kUp = 0x1p64;
    static constexpr int kExp = 64;
    // x to 24 bits in FP64, whatever its exponent (Veltkamp's splitting)
    __device__ static inline double value(double x) {
#pragma clang fp contract(off)
        const double c = x * 0x1.00000008p29;
        return c - (c - x);
    }
};

template <>
struct Round<double> {
    static constexpr int kThr = (1023 - 256) << 20;
    static constexpr double kUp = 0x1p256;
    static constexpr int kExp = 256;
    __device__ static inline double value(double x) { return x; }
};

// One entry of a tile through its descriptor.
template <typename T>
__device__ inline T load_entry(__amdgpu_buffer_rsrc_t rows, uint32_t at) {
    if constexpr (std::is_same<T, float>::value) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, at, 0, 0));
    } else {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(rows, at, 0, 0);
        return __hiloint2double((int)v.y, (int)v.x);
    }
}

template <typename T>
__device__ inline void store_entry(__amdgpu_buffer_rsrc_t rows, uint32_t at, T x) {
    if constexpr (std::is_same<T, float>::value) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rows, at, 0, 0);
    } else {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        const u2 v = {(uint32_t)__double2loint(x), (uint32_t)__double2hiint(x)};
        __builtin_amdgcn_raw_buffer_store_b64(v, rows, at, 0, 0);
    }
}

// The exponentials exp(lam_m r_k t) of every edge, [edge][q][m][category]
// (0 for padded categories): one thread each, a block of one tree.
constexpr int kExpChunk = 256;

template <int KP>
__global__ void __launch_bounds__(kExpChunk) k_exps(const BatchArgs a, const double *brlen, int chunks) {
    constexpr int CB = Lanes<KP>::CB;
    const __attribute__((address_space(4))) TreeDev *td =
        (const __attribute__((address_space(4))) TreeDev *)(a.trees + blockIdx.x / chunks);
    const __attribute__((address_space(4))) AlnDev *aln =
        (const __attribute__((address_space(4))) AlnDev *)(a.alns + blockIdx.x / chunks);
    const int x = (int)(blockIdx.x % chunks) * kExpChunk + threadIdx.x;
    if (x >= td->n_edges * KP * 4) return;
    const int e = x / (KP * 4), r = x % (KP * 4), k = r / (4 * CB) * CB + r % CB, m = r / CB % 4;
    const double t = brlen[td->edge_off + e];
    a.pmat[td->pm_off + x] = k < aln->K ? exp(aln->lam[m] * aln->rate[k] * t) : 0.0;
}

// Scaling of a partial by the stored pass's rule: per pattern, over its
// categories and states, when the largest entry is below 2^-S (and not zero)
// all are multiplied by 2^S.  Returns whether any pattern of the wave was
// scaled; cnt (null: not wanted) counts the events per item.  High words are
// compared as signed numbers: an entry below zero (a product has its zeros to
// a rounding of either sign) is small, as zero is.
template <typename T, int KP, int NI>
__device__ __attribute__((always_inline)) inline bool scale_joint(double *y, int *cnt) {
    using L = Lanes<KP>;
    constexpr int NQ = L::NQ;
    int m = __double2hiint(y[0]);
#pragma unroll
    for (int r = 1; r < NI * NQ; ++r) m = min(m, __double2hiint(y[r]));
    if (!__any(m < Round<T>::kThr)) return false;
    // (keeps what follows in its branch: the compiler would run it every time)
#pragma unroll
    for (int r = 0; r < NI * NQ; ++r) asm volatile("" : "+v"(y[r]));
    auto fold = [](unsigned long long v) __attribute__((always_inline)) {
        v |= v >> 32;
        v |= v >> 16;
        if (L::CB == 4) v |= v >> 8;
        if (L::CB >= 2) v |= v >> 4;
        return (uint32_t)v;
    };
    // bits of the columns, at lane & 15 with the category bits cleared
    constexpr uint32_t kCols = L::CB == 4 ? 0x000fu : L::CB == 2 ? 0x0f0fu : 0xffffu;
    unsigned long long big[NI], both = ~0ull;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        big[it] = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) big[it] |= __ballot(__double2hiint(y[it * NQ + q]) >= Round<T>::kThr);
        both &= big[it];
    }
    if ((~fold(both) & kCols) == 0) return false;  // one lane of each column is large enough in every item
    asm volatile("" : "+s"(big[0]));
    uint32_t low[NI], all = 0;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        low[it] = ~fold(big[it]) & kCols;
        all |= low[it];
    }
    if (all == 0) return false;
    const int lane = threadIdx.x & 63, col = lane & 15 & ~((L::CB - 1) << 2);
    bool scaled = false;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        unsigned long long any = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) any |= __ballot(y[it * NQ + q] > 0.0);
        const uint32_t cols = low[it] & fold(any);
        const uint32_t need = cols >> col & 1u;
        scaled |= cols != 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) y[it * NQ + q] *= need ? Round<T>::kUp : 1.0;
        if (cnt) cnt[it] += need;
    }
    return scaled;
}

// Programs come from compile_grad.  Each side reference is a leaf's
// tip (>= 0), the accumulator (REF_ACC) or the partial in slot REF_STACK0 - ref:
//   OP_GUP    acc = b of the node over sides a (edge ea) and b (edge eb), also
//             stored in slot dst;
//   OP_GROOT  the root edge eb between sides a and b: lnL, its derivatives;
//   OP_GDOWN  the node whose outer partial is side dst, across edge tip_a: the
//             derivatives at its children's edges ea and eb (children a and
//             b); child a, unless a tip, is the next accumulator, child b's
//             outer partial, unless a tip, replaces its inner one in its slot.
// Each wave writes its sums over patterns to a row of a.part: d1 of the edges,
// (HESS) d2 of the edges, lnL.
template <typename T, int KP, bool HESS>
__global__ void __launch_bounds__(64 * kGradWaves) __attribute__((amdgpu_waves_per_eu(KP > 4 ? 2 : 3)))
k_grad(const BatchArgs a, int stride) {
    using L = Lanes<KP>;
    constexpr int NI = kGradItems, NQ = L::NQ, NR = NI * NQ, CB = L::CB, WP = NI * L::kCols;
    constexpr bool kF32 = std::is_same<T, float>::value;
    __shared__ double tip_tab[4 * kTipRow];
    __shared__ double buf_s[kGradWaves][kBuf][64];
    __shared__ int ids_s[kGradWaves][2 * kBuf];
    const int bt = a.tile_tree[blockIdx.x];
    const TreeDev td = a.trees[bt];
    const AlnDev *aln = a.alns + bt;
    const int P = aln->P, K = aln->K, E = td.n_edges;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int hi = lane >> 4, blk = (lane >> 2) & 3, lo = lane & 3;
    // the tips' coefficients U^-1 x: row m, entry `code`
    if (threadIdx.x < 64) {
        double s = 0.0;
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (lane >> x & 1) s += aln->Uinv[hi * 4 + x];
        tip_tab[hi * kTipRow + (lane & 15)] = s;
    }
    __syncthreads();
    const int wt = ((int)blockIdx.x - td.tile_begin) * kGradWaves + wave;  // the wave's tile of the tree
    const int p0 = wt * WP;
    if (p0 >= P) return;
    double(*buf)[64] = buf_s[wave];
    int *ids = ids_s[wave];
    double *out = a.part + ((size_t)td.tile_begin * kGradWaves + wt) * stride;

    // constant operands: U, U^-1, and the rows 1, lam r, (lam r)^2 (HESS) or
    // the rows 1, lam r of two edges, one in rows 0 and 1, one in rows 2 and 3
    const double mU = aln->U[lo * 4 + hi], mW = aln->Uinv[lo * 4 + hi];
    double mR[NQ], mS[NQ], lr[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        lr[q] = aln->lam[hi] * aln->rate[q * CB + blk % CB];
        mR[q] = lo == 0 ? 1.0 : lo == 1 ? lr[q] : HESS && lo == 2 ? lr[q] * lr[q] : 0.0;
        mS[q] = lo == 2 ? 1.0 : lo == 3 ? lr[q] : 0.0;
    }
    // column c of item it is pattern p0 + c * NI + it
    const int col = blk / CB * 4 + lo;
    const bool full = p0 + WP <= P;
    const int left = P - p0 - col * NI;  // this lane's patterns
    // A lane's codes of one taxon are the word of its NI patterns, wherever the
    // row starts; past the end the row's last word, shifted (no state: code 0).
    const __attribute__((address_space(1))) uint8_t *tips = (const __attribute__((address_space(1))) uint8_t *)aln->tips;
    const uint32_t tip_at = left >= NI ? p0 + col * NI : max(P - 4, 0);
    const uint32_t tip_shift = left >= NI || left <= 0 ? 0 : 8 * (NI - left), tip_mask = left > 0 ? ~0u : 0u;
    // A slot holds the tiles one after the other (KP * 4 entries per pattern);
    // a full tile register after register, 64 lanes each, the last one
    // [category][pattern][state].  Accesses go through a descriptor of the
    // tile, whose bounds drop what is not there: nothing branches around a
    // load, so that loads are waited for by count and never for the stores
    // behind them.
    const uint32_t tile_bytes = sizeof(T) * KP * 4 * min(WP, P - p0);
    uint32_t place[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int k = r % NQ * CB + blk % CB, it = r / NQ;
        place[r] = full ? lane + 64 * r : it < left && k < K ? (k * (P - p0) + col * NI + it) * 4 + hi : 0x10000000;
        place[r] *= sizeof(T);
    }
    char *const slots = reinterpret_cast<char *>(reinterpret_cast<T *>(a.clv) + td.clv_off + (size_t)p0 * (KP * 4));
    const size_t slot_size = sizeof(T) * KP * 4 * (size_t)P;
    auto slot_rows = [&](int slot) __attribute__((always_inline)) {  // < 0: none
        return __builtin_amdgcn_make_buffer_rsrc(slots + (size_t)max(slot, 0) * slot_size, 0, slot < 0 ? 0 : tile_bytes,
                                                 0x00020000);
    };
    const __attribute__((address_space(1))) char *ex = (const __attribute__((address_space(1))) char *)(a.pmat + td.pm_off);
    const uint32_t ex_at = 8 * (hi * CB + blk % CB);

    auto exps = [&](int e, double *x) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            x[q] = *(const __attribute__((address_space(1))) double *)(ex + (size_t)(e * NQ + q) * (32 * CB) + ex_at);
    };
    // A side as loaded: a tip's codes of the lane's column, or a slot's entries.
    struct Raw {
        uint32_t w;
        T x[NR];
    };
    auto fetch_slot = [&](int ref, Raw &f) __attribute__((always_inline)) {
        const auto rows = slot_rows(REF_STACK0 - ref);
#pragma unroll
        for (int r = 0; r < NR; ++r) f.x[r] = load_entry<T>(rows, place[r]);
    };
    auto fetch_tip = [&](int ref, Raw &f) __attribute__((always_inline)) {
        const __attribute__((address_space(1))) uint8_t *s = tips + (size_t)max(ref, 0) * P;
        if (P >= NI) {
            f.w = *(const __attribute__((address_space(1))) UnalignedWord *)(s + tip_at);
        } else {
            f.w = 0;
            for (int x = 0; x < P; ++x) f.w |= (uint32_t)s[x] << (8 * (NI - P + x));
        }
    };
    auto fetch = [&](int ref, Raw &f) __attribute__((always_inline)) {
        fetch_tip(ref, f);
        fetch_slot(ref, f);
    };
    // its coefficients
    auto side = [&](int ref, const Raw &f, const double *acc, double *b) __attribute__((always_inline)) {
        if (ref >= 0) {
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const uint32_t w = (f.w >> tip_shift & tip_mask) << 3;
                const double v = *(const double *)((const char *)(tip_tab + hi * kTipRow) + (w >> (8 * it) & 0xffu));
#pragma unroll
                for (int q = 0; q < NQ; ++q) b[it * NQ + q] = v;
            }
        } else if (ref == REF_ACC) {
#pragma unroll
            for (int r = 0; r < NR; ++r) b[r] = acc[r];
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) b[r] = kF32 ? mfma4(mW, (double)f.x[r]) : (double)f.x[r];
        }
    };
    // the coefficients of a directional partial, rounded as stored (`stored`:
    // in the range of T)
    auto coeffs = [&](double *y, double *b, bool stored) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            y[r] = stored ? (double)(T)y[r] : Round<T>::value(y[r]);
            b[r] = mfma4(mW, y[r]);
        }
    };
    // what a slot holds: FP32 the partial, FP64 its coefficients
    auto store = [&](int slot, const double *y, const double *b) __attribute__((always_inline)) {
        const auto rows = slot_rows(slot);
#pragma unroll
        for (int r = 0; r < NR; ++r) store_entry<T>(rows, place[r], (T)(kF32 ? y[r] : b[r]));
    };

    // Rows of 64 lanes wait in LDS for their sums: an edge's terms in all lanes,
    // or (pairs) in rows 1 and 3 those of two edges, or (HESS) in rows 1 and 2
    // those of an edge's two derivatives.
    int n_buf = 0;
    bool pairs = kF32 && !HESS;
    auto flush = [&]() __attribute__((always_inline)) {
        wave_lds_fence();
        double s = 0.0;
        if (HESS || pairs) {
            const int row = lane >> 3, half = lane >> 2 & 1, part = lane & 3;
            const double *v = &buf[row][(HESS ? 16 + 16 * half : 16 + 32 * half) + part * 4];
#pragma unroll
            for (int x = 0; x < 4; ++x) s += v[x];
            s += dpp_add<0xb1>(s);  // lanes 1 and 2 apart
            s += dpp_add<0x4e>(s);
            const int e = HESS ? ids[2 * row] : ids[2 * row + half];
            if (row < n_buf && part == 0 && e >= 0) out[HESS ? half * E + e : e] = s;
        } else {
            const int row = lane >> 3, part = lane & 7;
#pragma unroll
            for (int x = 0; x < 8; ++x) s += buf[row][part * 8 + x];
            s += dpp_add<0xb1>(s);
            s += dpp_add<0x4e>(s);
            s += dpp_add<0x141>(s);  // the other half of eight
            if (row < n_buf && part == 0) out[ids[2 * row]] = s;
        }
        n_buf = 0;
        wave_lds_fence();
    };
    auto emit = [&](int e, int e2, double v) __attribute__((always_inline)) {
        buf[n_buf][lane] = v;
        if (lane < 2) ids[2 * n_buf + lane] = lane ? e2 : e;
        if (++n_buf == kBuf) flush();
    };

    // CB items at a time share a column's category lanes: lane c takes item
    // g * CB + c (weight 0 past the end).  Its L, dL and d2L are in rows 0, 1
    // and 2.
    double weight[NI / CB];
#pragma unroll
    for (int g = 0; g < NI / CB; ++g) {
        const int it = g * CB + blk % CB;
        weight[g] = it < left ? *(const __attribute__((address_space(1))) double *)(aln->w + p0 + col * NI + it) : 0.0;
    }
    // ... (of s2 in rows 2 and 3, when given)
    auto totals = [&](const double *s, const double *s2, int g) __attribute__((always_inline)) {
        double x = 0.0;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int it = g * CB + c;
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                v = __builtin_amdgcn_mfma_f64_4x4x4f64(mR[q], s[it * NQ + q], v, 0, 0, 0);
                if (s2) v = __builtin_amdgcn_mfma_f64_4x4x4f64(mS[q], s2[it * NQ + q], v, 0, 0, 0);
            }
            if constexpr (CB == 4) {
                v += row_ror<8>(v);
                v += row_ror<4>(v);
            }
            if constexpr (CB == 2) v += __shfl_xor(v, 4);
            if (c == 0 || blk % CB == c) x = v;
        }
        return x;
    };
    // The terms of an edge's derivatives by its own L: dL / L in row 1 and (HESS)
    // d2L / L - (dL / L)^2 in row 2, or dL / L of two edges in rows 1 and 3.
    auto ratio_terms = [&](const double *s, const double *s2) __attribute__((always_inline)) {
        double v = 0.0;
#pragma unroll
        for (int g = 0; g < NI / CB; ++g) {
            const double x = totals(s, s2, g);
            const double r = x * recip(HESS ? row0(x) : even_rows(x));
            double term = r;
            if constexpr (HESS) {
                const double r1 = row1(r);
                if (hi == 2) term = r - r1 * r1;
            }
            if (weight[g] > 0.0) v += weight[g] * term;  // (past the end L may be 0)
        }
        return hi == 1 || hi == (HESS ? 2 : 3) ? v : 0.0;
    };

    double acc[NR], wl[NR];
    int cnt[NI];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] = wl[r] = 0.0;
#pragma unroll
    for (int it = 0; it < NI; ++it) cnt[it] = 0;
    // FP64 partials and no second derivatives: L of a pattern is the same at
    // every edge (to rounding), so the root's serves all and an edge's terms
    // need no sum over a pattern's lanes -- unless a partial was scaled.
    bool ratio = kF32 || HESS;
    // The next op's sides and exponentials are loaded while this one runs.  (It
    // reads no slot that this one writes: a node's partial goes to the next op
    // in the accumulator.)
    const Op *prog = a.ops + td.op_first;
    Op op = load_op(prog, 0);
    Raw ra, rb;
    double x0[NQ], x1[NQ], x2[NQ];
    exps(op.tip_a, x0);
    exps(op.ea, x1);
    exps(op.eb, x2);
    fetch(op.a, ra);
    fetch(op.b, rb);
    for (int o = td.n_first; o > 0; --o) {
        const Op cur = op;
        double b1[NR], b2[NR], y0[NQ], y1[NQ];
        double u[NR];
        if (cur.code == OP_GDOWN) {
            // (loaded before the next op's sides, so as not to wait for those)
            Raw r0;
            if (cur.dst >= 0) fetch_tip(cur.dst, r0);
            else if (cur.dst != REF_ACC) fetch_slot(cur.dst, r0);
            side(cur.dst, r0, acc, u);
        }
        ++prog;
        op = load_op(prog, o > 1 ? 0 : -1);
        side(cur.a, ra, acc, b1);
        side(cur.b, rb, acc, b2);
#pragma unroll
        for (int r = 0; r < NR; ++r) b2[r] *= x2[r % NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            y0[q] = x0[q];
            y1[q] = x1[q];
        }
        exps(op.tip_a, x0);
        exps(op.ea, x1);
        exps(op.eb, x2);
        fetch(op.a, ra);
        fetch(op.b, rb);
        if (cur.code == OP_GUP) {
            double y[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) y[r] = mfma4(mU, y1[r % NQ] * b1[r]) * mfma4(mU, b2[r]);
            if (scale_joint<T, KP, NI>(y, cnt)) ratio = true;
            coeffs(y, acc, true);
            store(cur.dst, y, acc);
            continue;
        }
        if (cur.code == OP_GROOT) {
#pragma unroll
            for (int r = 0; r < NR; ++r) b1[r] *= b2[r];
            double lnl = 0.0, d = 0.0;
#pragma unroll
            for (int g = 0; g < NI / CB; ++g) {
                const double x = totals(b1, nullptr, g), wt_ = weight[g];
                const double Lp = row0(x), inv = recip(Lp);
                int c = 0;
#pragma unroll
                for (int k = 0; k < CB; ++k) c += (blk % CB == k ? 1 : 0) * cnt[g * CB + k];
                if (hi == 0 && wt_ > 0.0) lnl += wt_ * (log(Lp) - ((double)c * Round<T>::kExp * kLn2 + aln->log_k));
                const double r = x * inv;
                double term = r;
                if constexpr (HESS) {
                    const double r1 = row1(r);
                    if (hi == 2) term = r - r1 * r1;
                }
                if (wt_ > 0.0) d += wt_ * term;  // (past the end L may be 0)
                if constexpr (!kF32 && !HESS) {
                    // w / L of each item in all of the column's lanes
#pragma unroll
                    for (int k = 0; k < CB; ++k) {
                        double v = wt_ > 0.0 ? wt_ * inv : 0.0;
                        if constexpr (CB > 1) v = __shfl(v, (lane & ~((CB - 1) << 2)) | k << 2);
#pragma unroll
                        for (int q = 0; q < NQ; ++q) wl[(g * CB + k) * NQ + q] = lr[q] * v;
                    }
                }
            }
            pairs = !HESS && ratio;
            emit(cur.eb, -1, hi == 1 || (HESS && hi == 2) ? d : 0.0);
            lnl = wave_sum(lnl);
            if (lane == 0) out[stride - 1] = lnl;
            continue;
        }
        // OP_GDOWN
        double y[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            b1[r] *= y1[r % NQ];
            const double t = mfma4(mU, y0[r % NQ] * u[r]);
            y[r] = t * mfma4(mU, b2[r]);  // seen from child a
            u[r] = t * mfma4(mU, b1[r]);  // seen from child b
        }
        // In registers an outer partial keeps the range of FP64 (its derivatives
        // are ratios, which a pattern's scale does not change); stored as FP32
        // it is brought up to 2^-64 or more, as the stored pass's are.
        const bool sa = scale_joint<double, KP, NI>(y, nullptr), sb = scale_joint<double, KP, NI>(u, nullptr);
        if (sa || sb) ratio = true;
        double ub[NR];
        coeffs(y, acc, false);
        coeffs(u, ub, false);
        if (cur.b < 0) {
            if constexpr (kF32) {
                // (its largest entry is at least 2^-256 or zero)
                for (int k = 0; k < 4; ++k)
                    if (!scale_joint<float, KP, NI>(u, nullptr)) break;
            }
            store(REF_STACK0 - cur.b, u, ub);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            b1[r] *= acc[r];
            b2[r] *= ub[r];
        }
        if constexpr (HESS) {
            emit(cur.ea, 0, ratio_terms(b1, nullptr));
            emit(cur.eb, 0, ratio_terms(b2, nullptr));
        } else if (ratio) {
            if (!pairs) {
                if (n_buf) flush();
                pairs = true;
            }
            emit(cur.ea, cur.eb, ratio_terms(b1, b2));
        } else {
            double v1 = 0.0, v2 = 0.0;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                v1 += b1[r] * wl[r];
                v2 += b2[r] * wl[r];
            }
            emit(cur.ea, 0, v1);
            emit(cur.eb, 0, v2);
        }
    }
    if (n_buf) flush();
}

// Sums over a tree's waves: d1 (and d2) of every edge, lnL.  Four threads per
// edge take a quarter of the waves each, sixteen loads in flight, and the
// quarters are added in order (one thread per edge: 13.5 us for one tree of
// 27 taxa x 976 patterns, all latency).
constexpr int kSumEdges = 64;

__global__ void __launch_bounds__(4 * kSumEdges) k_grad_sums(const BatchArgs a, int stride, int wave_pats, double *lnl,
                                                            double *gout, double *hout) {
    __shared__ double part[3][4][kSumEdges];
    const int x = threadIdx.x % kSumEdges, seg = threadIdx.x / kSumEdges;
    const int64_t i = (int64_t)blockIdx.x * kSumEdges + x;
    if (i < a.n_edges) {
        const int b = a.edge_tree[i];
        const TreeDev &td = a.trees[b];
        const int e = (int)(i - td.edge_off), n = (a.alns[b].P + wave_pats - 1) / wave_pats, quarter = (n + 3) / 4;
        const int t0 = min(n, seg * quarter), t1 = min(n, t0 + quarter);
        const double *row = a.part + (size_t)td.tile_begin * kGradWaves * stride;
        auto sum = [&](int at) __attribute__((always_inline)) {
            const double *p = row + (size_t)t0 * stride + at;
            double s = 0.0;
            int t = t0;
            for (; t + 16 <= t1; t += 16, p += (size_t)16 * stride) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = p[(size_t)u * stride];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += v[u];
            }
            for (; t < t1; ++t, p += stride) s += *p;
            return s;
        };
        part[0][seg][x] = sum(e);
        if (hout) part[1][seg][x] = sum(td.n_edges + e);
        if (e == 0) part[2][seg][x] = sum(stride - 1);
    }
    __syncthreads();
    if (seg > 0 || i >= a.n_edges) return;
    auto total = [&](int f) __attribute__((always_inline)) {
        return ((part[f][0][x] + part[f][1][x]) + part[f][2][x]) + part[f][3][x];
    };
    gout[i] = total(0);
    if (hout) hout[i] = total(1);
    const int b = a.edge_tree[i];
    if (i == a.trees[b].edge_off && lnl) lnl[b] = total(2);
}

#define PT_KP_SWITCH(...)                                   \
    switch (kp) {                                           \
    case 1: { constexpr int KP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int KP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int KP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int KP = 8; __VA_ARGS__; } break;   \
    default: break;                                         \
    }

template <typename T, int KP>
void launch_grad_t(const BatchArgs &a, bool hess, int stride, hipStream_t s) {
    const dim3 grid(a.n_tiles), block(64 * kGradWaves);
    if (hess) hipLaunchKernelGGL((k_grad<T, KP, true>), grid, block, 0, s, a, stride);
    else hipLaunchKernelGGL((k_grad<T, KP, false>), grid, block, 0, s, a, stride);
}

}  // namespace

int grad_tile_patterns(int kp) {
    PT_KP_SWITCH(return kGradWaves * kGradItems * Lanes<KP>::kCols);
    return 0;
}

size_t grad_part_doubles(int tiles, int max_edges) { return (size_t)tiles * kGradWaves * (2 * (size_t)max_edges + 1); }

hipError_t launch_grad(int precision, const BatchArgs &a, const double *brlen, int max_edges, double *lnl,
                       double *grad, double *hess, hipStream_t s) {
    if (a.n_tiles <= 0) return hipSuccess;
    const int kp = a.kp, chunks = (max_edges * kp * 4 + kExpChunk - 1) / kExpChunk;
    const int stride = (hess ? 2 : 1) * max_edges + 1;
    hipError_t e = hipErrorInvalidValue;
    PT_KP_SWITCH({
        hipLaunchKernelGGL((k_exps<KP>), dim3((unsigned)a.n_trees * chunks), dim3(kExpChunk), 0, s, a, brlen, chunks);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (precision == PT_FP32) launch_grad_t<float, KP>(a, hess != nullptr, stride, s);
        else launch_grad_t<double, KP>(a, hess != nullptr, stride, s);
        e = hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_grad_sums, dim3((unsigned)((a.n_edges + kSumEdges - 1) / kSumEdges)), dim3(4 * kSumEdges), 0, s, a, stride,
                       grad_tile_patterns(kp) / kGradWaves, lnl, grad, hess);
    return hipGetLastError();
}

}  // namespace pt
