// partials.hpp -- device code of the kernels that store partials: updates,
// edge evaluations, eigenbasis tables and the Newton steps of one edge.
// (kernels.hip says how the work is laid out.)
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "kernels.hpp"
#include "lanes.hpp"
#include "pt.h"

namespace pt {
namespace {

constexpr double kLn2 = 0.69314718055994530942;

template <typename T>
struct Store;

template <>
struct Store<float> {
    static constexpr int kScaleExp = 64;
    // one category's four states as loaded, widened when used
    using Raw = float4;
    __device__ static inline Raw load_raw(const float *p) { return *reinterpret_cast<const float4 *>(p); }
    __device__ static inline void widen(const Raw &v, double x[4]) {
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    }
    __device__ static inline double as_stored(double x) { return (double)(float)x; }
    __device__ static inline Raw pack(const double x[4]) {
        return make_float4((float)x[0], (float)x[1], (float)x[2], (float)x[3]);
    }
    __device__ static inline void store_raw(float *p, const Raw &r) { *reinterpret_cast<float4 *>(p) = r; }
    __device__ static inline void store(float *p, const double x[4]) { store_raw(p, pack(x)); }
};

template <>
struct Store<double> {
    static constexpr int kScaleExp = 256;
    struct Raw {
        double2 a, b;
    };
    __device__ static inline Raw load_raw(const double *p) {
        Raw r;
        r.a = reinterpret_cast<const double2 *>(p)[0];
        r.b = reinterpret_cast<const double2 *>(p)[1];
        return r;
    }
    __device__ static inline void widen(const Raw &v, double x[4]) {
        x[0] = v.a.x; x[1] = v.a.y; x[2] = v.b.x; x[3] = v.b.y;
    }
    __device__ static inline double as_stored(double x) { return x; }
    __device__ static inline Raw pack(const double x[4]) {
        Raw r;
        r.a = make_double2(x[0], x[1]);
        r.b = make_double2(x[2], x[3]);
        return r;
    }
    __device__ static inline void store_raw(double *p, const Raw &r) {
        reinterpret_cast<double2 *>(p)[0] = r.a;
        reinterpret_cast<double2 *>(p)[1] = r.b;
    }
    __device__ static inline void store(double *p, const double x[4]) {
        reinterpret_cast<double2 *>(p)[0] = make_double2(x[0], x[1]);
        reinterpret_cast<double2 *>(p)[1] = make_double2(x[2], x[3]);
    }
};

// Model constants of the tree in flight, copied to LDS once per tree.
struct ModelS {
    double W[16];    // W_im = pi_i U_im = Uinv_mi
    double U[16];    // P(t) = U diag(exp(lam t)) Uinv
    double Uinv[16];
    double lam[4];
    double rate[kMaxCats];
    alignas(16) float WfT[16];   // W rounded to FP32 and transposed, W_im at 4 m + i (the FP32 tables of the optimisation loop)
    double log_k;    // ln K
};

__device__ inline void model_to_lds(const AlnDev *aln, ModelS *m) {
    for (int x = threadIdx.x; x < 16; x += blockDim.x) {
        m->W[x] = aln->W[x];
        m->WfT[(x & 3) * 4 + (x >> 2)] = (float)aln->W[x];
        m->U[x] = aln->U[x];
        m->Uinv[x] = aln->Uinv[x];
    }
    if (threadIdx.x == 0) m->log_k = aln->log_k;
    if (threadIdx.x < 4) m->lam[threadIdx.x] = aln->lam[threadIdx.x];
    if (threadIdx.x < kMaxCats) m->rate[threadIdx.x] = aln->rate[threadIdx.x];
}

// Load through a pointer known to address global memory (pointers read out
// of descriptors would otherwise be accessed with generic FLAT loads).
template <typename X>
__device__ inline X ldg(const X *p) {
    return *(const __attribute__((address_space(1))) X *)p;
}

// View of one tree's data for the device functions below.
template <typename T>
struct TreeView {
    const ModelS *m;     // LDS
    const double *pm;    // LDS: [E][Kp][16] (or global, see PmPtr)
    const float *pmf;    // optional FP32 copy of pm in LDS
    const uint8_t *tips; // [n][P]
    const double *w;     // [P]
    T *clv;              // slot 0 of this tree: [slot][Kp][P][4]
    uint16_t *cnt;       // slot 0 of this tree: [slot][P]
    int P, K;            // P: the pattern stride of the layouts
    int np;              // patterns this block works on (tips, w, clv, cnt start at its first)
};

template <typename T, int KP>
__device__ inline T *slot_ptr(const TreeView<T> &v, int ref, int k, int p) {
    return v.clv + (((size_t)ref * KP + k) * v.P + p) * 4;
}

__device__ inline void tip_vec(unsigned code, double x[4]) {
    x[0] = code & 1u; x[1] = (code >> 1) & 1u; x[2] = (code >> 2) & 1u; x[3] = (code >> 3) & 1u;
}

// Entry (i, j) of P(r_k t) = U diag(exp(lam r_k t)) Uinv, from the block's
// LDS copy of the model (the optimisation loop recomputes an edge's matrices
// after every length change, and global loads there cost a round trip).
__device__ inline double pm_entry(const ModelS *md, int k, int ij, double t) {
    const int i = ij >> 2, j = ij & 3;
    const double r = md->rate[k];
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) s += md->U[i * 4 + m] * exp(md->lam[m] * r * t) * md->Uinv[m * 4 + j];
    return s;
}

// The same entry from the exponentials ex[k*4 + m] = exp(lam_m r_k t), each
// computed once (by the same expression) instead of once per entry.
__device__ inline double pm_entry_ex(const ModelS *md, const double *ex, int k, int ij) {
    const int i = ij >> 2, j = ij & 3;
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) s += md->U[i * 4 + m] * ex[k * 4 + m] * md->Uinv[m * 4 + j];
    return s;
}

// Fixed-order block sum of three values; every thread receives the totals.
// `red` holds two buffers used alternately, so back-to-back sums need one
// barrier each.
template <int BS>
__device__ inline void block_sum3(double &a, double &b, double &c, double *red, int &parity) {
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    constexpr int W = BS / 64;
    double *r = red + parity * W * 3;
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        r[wave * 3 + 0] = a;
        r[wave * 3 + 1] = b;
        r[wave * 3 + 2] = c;
    }
    __syncthreads();
    a = b = c = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        a += r[w * 3 + 0];
        b += r[w * 3 + 1];
        c += r[w * 3 + 2];
    }
    parity ^= 1;
}

// A tree optimised by G > 1 blocks, each over its own share of the patterns
// (k_optimize): every block sum is combined across the blocks.  Lane 0 of
// each block's first wave publishes the block's triple in its own entry of
// one of two alternating slots, each value carrying the reduction's number
// (mod 4) in its two lowest mantissa bits; lanes 0..G-1 of that wave then
// poll the G entries in parallel, one entry per lane, until every value of
// every entry carries the number, and the G triples are summed in block
// order with the tag bits cleared.  Every block sums the same bits in the
// same order, so all hold identical totals and take identical decisions;
// clearing the two bits perturbs a value by at most 2^-51 relative.  One
// store and one load round trip per reduction, with no counter.  The
// accesses are device-scope atomics (coherent across the XCDs).  A slot is
// rewritten two reductions later, by when every block has read it (a block
// publishes reduction s + 1 only after reading all of s), and the previous
// content of a slot carries another number (or is zero, which no reduction
// uses as its tag).  A wait is bounded in time: when it runs out the tree is
// marked broken, its blocks stop waiting, and its status reports the failure.
// (The blocks' own partials are a different matter: see k_optimize.)
// per-tree words (kGroupSyncWords): broken, then slots [2][G][3]
static_assert(1 + 2 * kGroupBlocksMax * 3 <= kGroupSyncWords, "cross-block state does not fit");
constexpr long long kGroupWaitCycles = 1ll << 27;  // shader clocks before a wait gives up

// (a pointer read from LDS would otherwise be accessed with FLAT operations)
typedef __attribute__((address_space(1))) unsigned long long GlobalU64;

__device__ inline unsigned long long load_agent(GlobalU64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void store_agent(GlobalU64 *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline unsigned long long tag_bits(double v, unsigned long long tag) {
    return ((unsigned long long)__double_as_longlong(v) & ~3ull) | tag;
}

__device__ inline double untag(unsigned long long b) { return __longlong_as_double((long long)(b & ~3ull)); }

__device__ inline unsigned long long lane_u64(unsigned long long v, int lane) {
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)v, lane);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(v >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}

struct GroupS {  // in LDS; written by lane 0 of the block's first wave
    int G, g;
    int seq, is_broken;
    unsigned long long *broken, *slots;
    long long wait;  // shader clocks before a wait gives up
    double tot[3];
};

// Called by the block's first wave (all 64 lanes) with the block's totals.
__device__ inline void group_exchange(GroupS *gs, double a, double b, double c) {
    const int G = gs->G, g = gs->g, s = gs->seq;
    const int lane = threadIdx.x & 63;
    GlobalU64 *slot = (GlobalU64 *)gs->slots + (size_t)(s & 1) * G * 3;
    const unsigned long long want = (unsigned long long)((s + 1) & 3);
    const unsigned long long ta = tag_bits(a, want), tb = tag_bits(b, want), tc = tag_bits(c, want);
    if (lane == 0) {
        store_agent(slot + g * 3 + 0, ta);
        store_agent(slot + g * 3 + 1, tb);
        store_agent(slot + g * 3 + 2, tc);
    }
    unsigned long long va = ta, vb = tb, vc = tc;  // lane g keeps its own entry
    bool ok = lane >= G || lane == g;
    if (!gs->is_broken) {
        const long long t0 = clock64();
        for (;;) {
            if (!ok) {
                va = load_agent(slot + lane * 3 + 0);
                vb = load_agent(slot + lane * 3 + 1);
                vc = load_agent(slot + lane * 3 + 2);
                ok = (va & 3ull) == want && (vb & 3ull) == want && (vc & 3ull) == want;
            }
            if (__all(ok)) break;
            if (clock64() - t0 > gs->wait) {
                if (lane == 0) {
                    store_agent((GlobalU64 *)gs->broken, 1ull);
                    gs->is_broken = 1;
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
    for (int h = 0; h < G; ++h) {
        t0 += untag(lane_u64(va, h));
        t1 += untag(lane_u64(vb, h));
        t2 += untag(lane_u64(vc, h));
    }
    if (lane == 0) {
        gs->tot[0] = t0;
        gs->tot[1] = t1;
        gs->tot[2] = t2;
        gs->seq = s + 1;
    }
}

// Block sum of three values, then (gs set) the sum over the tree's blocks;
// every thread receives the totals.
template <int BS>
__device__ inline void group_sum3(double &a, double &b, double &c, double *red, int &parity, GroupS *gs) {
    block_sum3<BS>(a, b, c, red, parity);
    if (gs == nullptr) return;
    if (threadIdx.x < 64) group_exchange(gs, a, b, c);
    __syncthreads();
    a = gs->tot[0];
    b = gs->tot[1];
    c = gs->tot[2];
}

// Per-wave table of exp(lam_m r_k t) and its first two t-derivative factors:
// wx[km] = e, wx[32 + km] = lam_m r_k e, wx[64 + km] = (lam_m r_k)^2 e, with
// km = k*4 + m.  Lanes 0..4K-1 compute one entry each; LDS operations of a
// wave complete in order, so the wave's later reads see them.
constexpr int kWx = 3 * 4 * kMaxCats;  // doubles per wave

// R = float: the values rounded to FP32 (held widened, so that no reader
// converts them again).
template <typename R>
__device__ inline void wave_expo(double *wx, const ModelS *md, int K, double t) {
    const int lane = threadIdx.x & 63;
    if (lane < 4 * K) {
        const int k = lane >> 2, m = lane & 3;
        const double q = md->lam[m] * md->rate[k];
        const double e = exp(q * t);
        wx[lane] = (double)(R)e;
        wx[4 * kMaxCats + lane] = (double)(R)(e * q);
        wx[8 * kMaxCats + lane] = (double)(R)(e * q * q);
    }
    __builtin_amdgcn_wave_barrier();
}

// Up to four categories: an iteration's exponentials in registers, entry
// k*4 + m in lane k*4 + m of every row of 16 lanes, and a pattern's sums over
// them by row broadcast (as LDS broadcasts they were 24 reads of 8 clocks per
// row or pair of rows).  Every lane of a wave runs these.
struct LaneExpo {
    double e0, e1, e2;
    __device__ inline explicit LaneExpo(const double *wx) {
        const int l = threadIdx.x & 15;
        e0 = wx[l];
        e1 = wx[4 * kMaxCats + l];
        e2 = wx[8 * kMaxCats + l];
    }
};

// L, L1, L2 += the four coefficients of category KAT times its exponentials,
// in the order of m.
#define PT_DPP(Y, E, X, L) "v_fmac_f64_dpp %" #Y ", %" #E ", %" #X " row_newbcast:%" #L " row_mask:0xf bank_mask:0xf\n\t"
#define PT_DPP3(X, L) PT_DPP(0, 3, X, L) PT_DPP(1, 4, X, L) PT_DPP(2, 5, X, L)
template <int KAT>
__device__ inline void add_expo(const LaneExpo &e, const double s[4], double &L, double &L1, double &L2) {
    asm volatile("s_nop 1\n\t" PT_DPP3(6, 10) PT_DPP3(7, 11) PT_DPP3(8, 12) PT_DPP3(9, 13)
                 : "+&v"(L), "+&v"(L1), "+&v"(L2)
                 : "v"(e.e0), "v"(e.e1), "v"(e.e2), "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "n"(KAT * 4),
                   "n"(KAT * 4 + 1), "n"(KAT * 4 + 2), "n"(KAT * 4 + 3));
}
#undef PT_DPP3
#undef PT_DPP

// The same for category k < 4, known when unrolled.
__device__ inline void add_expo(int k, const LaneExpo &e, const double s[4], double &L, double &L1, double &L2) {
    if (k == 0) add_expo<0>(e, s, L, L1, L2);
    else if (k == 1) add_expo<1>(e, s, L, L1, L2);
    else if (k == 2) add_expo<2>(e, s, L, L1, L2);
    else add_expo<3>(e, s, L, L1, L2);
}

// One side of an update or edge evaluation for one pattern: a tip code, or
// the scaler count (CNT) and every category's partial of a slot.  TIP is a
// template parameter so that the code fetching a pattern's sides has no
// branch between its loads: they are all issued before the first is used,
// and their memory round trips overlap.
template <typename T, int KP, bool TIP, bool CNT = true>
struct Side {
    typename Store<T>::Raw r[KP];
    unsigned code;
    int c;
    __device__ inline void fetch(const TreeView<T> &v, int ref, int p) {
        if constexpr (TIP) {
            code = ldg(v.tips + (size_t)(-ref - 1) * v.P + p);
            c = 0;
        } else {
            c = CNT ? v.cnt[(size_t)ref * v.P + p] : 0;
            // the layout holds KP categories, so padded ones are in bounds
#pragma unroll
            for (int k = 0; k < KP; ++k) r[k] = Store<T>::load_raw(slot_ptr<T, KP>(v, ref, k, p));
        }
    }
    __device__ inline void get(int k, double x[4]) const {
        if constexpr (TIP) tip_vec(code, x);
        else Store<T>::widen(r[k], x);
    }
    // the same state vector in FP32 (FP32 partials only)
    __device__ inline void getf(int k, float x[4]) const {
        if constexpr (TIP) {
            x[0] = (float)(code & 1u); x[1] = (float)((code >> 1) & 1u);
            x[2] = (float)((code >> 2) & 1u); x[3] = (float)((code >> 3) & 1u);
        } else {
            static_assert(std::is_same<T, float>::value, "FP32 state vectors of FP32 partials only");
            x[0] = r[k].x; x[1] = r[k].y; x[2] = r[k].z; x[3] = r[k].w;
        }
    }
};

// Where an update reads its transition matrices (PM):
//   kPmLds    FP64 copy in LDS;
//   kPmConst  global memory the kernel never writes, through the constant
//             address space, so that the wave-uniform entries arrive by
//             scalar loads into scalar registers instead of being broadcast
//             to every lane;
//   kPmLds64  FP64 copy in LDS, an entry per lane of 16 (LaneMats);
//   kPmLds32  FP32 copy in LDS (half the broadcast bytes), for FP32 partials
//             in the optimisation loop, whose updates then compute in FP32
//             (update_pattern_f32).
enum : int { kPmLds = 0, kPmConst = 1, kPmLds32 = 2, kPmLds64 = 3 };

// The optimisation loop's: with eight categories in FP64 the registers of the
// per-lane form would spill.
template <typename T, int KP>
struct OptPm {
    static constexpr int value = std::is_same<T, float>::value ? kPmLds32 : KP <= 4 ? kPmLds64 : kPmLds;
};
template <int PM>
struct PmPtr {
    using type = const double *;
};
template <>
struct PmPtr<kPmConst> {
    using type = const __attribute__((address_space(4))) double *;
};
template <>
struct PmPtr<kPmLds32> {
    using type = const float *;
};
template <int PM, typename V>
__device__ inline typename PmPtr<PM>::type pm_base(const V &v) {
    if constexpr (PM == kPmLds32) return v.pmf;
    else return (typename PmPtr<PM>::type)v.pm;
}

// FP32 products in the optimisation loop, on the matrix cores:
// v_mfma_f32_4x4x1_16b takes, in each group of four lanes, lane i's matrix
// entry (row i) times every lane's vector entry, so with a pattern per lane
// and its states in registers, four of them multiply a 4x4 matrix with 64
// patterns' vectors, and a lane's operand is one row of the matrix (one
// 16-byte LDS read with four addresses in place of four broadcasts).  Each is
// a fused multiply-add, the chain of the scalar code bit for bit (checked on
// the device over 10^6 random results, subnormal ones among them).  A, B are
// the first two states summed: a matrix entry times a vector entry plus
// another is contracted with the later product rounded first, and lengths
// stay what they are only if both orders are kept.  The instruction ignores the execution mask, so every lane of a wave runs these
// functions, on a valid pattern.
typedef float F4 __attribute__((ext_vector_type(4)));

template <int A, int B>
__device__ inline F4 mat_vec(const float4 &row, const float x[4]) {
    F4 y = {0.0f, 0.0f, 0.0f, 0.0f};
    y = __builtin_amdgcn_mfma_f32_4x4x1f32(A ? row.y : row.x, x[A], y, 0, 0, 0);
    y = __builtin_amdgcn_mfma_f32_4x4x1f32(B ? row.y : row.x, x[B], y, 0, 0, 0);
    y = __builtin_amdgcn_mfma_f32_4x4x1f32(row.z, x[2], y, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_4x4x1f32(row.w, x[3], y, 0, 0, 0);
}

// This lane's row of every category's FP32 matrix of an edge.
template <int KP>
struct EdgeRows {
    float4 r[KP];
    __device__ inline EdgeRows(const float *pmf, int e) {
        const float4 *q = reinterpret_cast<const float4 *>(pmf + (size_t)e * KP * 16) + (threadIdx.x & 3);
#pragma unroll
        for (int k = 0; k < KP; ++k) r[k] = q[k * 4];
    }
};

// One pattern of an OP_UPDATE in FP32 arithmetic, for FP32 partials in the
// optimisation loop (matrices from the FP32 LDS copy): the same products and
// scaling rule as update_pattern, computed in the precision the partial is
// stored in, so no entry is widened to FP64 and narrowed back.  The new
// partial of every category goes to out[k] as stored.  No scaler count is
// kept: the loop's sums are ratios, which a pattern's scale does not change,
// and the lnL an optimisation reports comes from k_prune.
template <int KP, class SA, class SB>
__device__ inline void update_pattern_f32(int K, const EdgeRows<KP> &ma, const EdgeRows<KP> &mb, const SA &sa,
                                          const SB &sb, float4 out[KP]) {
    const float thr = 0x1p-64f, up = 0x1p64f;  // Store<float>::kScaleExp
    float o[KP][4];
    float mx = 0.0f;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        float xa[4], xb[4];
        sa.getf(k, xa);
        sb.getf(k, xb);
        const F4 ya = mat_vec<1, 0>(ma.r[k], xa), yb = mat_vec<1, 0>(mb.r[k], xb);
        const bool live = k < K;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[k][i] = live ? ya[i] * yb[i] : 0.0f;
            mx = fmaxf(mx, o[k][i]);
        }
    }
    const float f = mx < thr && mx > 0.0f ? up : 1.0f;
#pragma unroll
    for (int k = 0; k < KP; ++k) out[k] = make_float4(o[k][0] * f, o[k][1] * f, o[k][2] * f, o[k][3] * f);
}

// FP64 products in the optimisation loop: a matrix sits in one register pair,
// entry l of 16 in lane l of every row of 16 lanes, and each fused multiply-add
// takes its entry from there by a row broadcast, which 64-bit fused
// multiply-adds have.  Reading the entries from LDS as broadcasts instead took
// 64 lanes x 16 bytes per two of them: 100 such reads per update, 3k of its 8k
// clocks on a compute unit's four waves.  A, B are the first two states summed
// (the order of the scalar code, as in mat_vec).  Sources in lanes that the
// execution mask switches off are not read, so every lane of a wave runs this,
// and the block is volatile, so that it is not moved under a branch that its
// results alone are used in.  The wait at its start covers a matrix that was
// just moved by a vector instruction.
#define PT_DPP(Y, L, X) "v_fmac_f64_dpp %" #Y ", %4, %" #X " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
#define PT_DPP4(L0, L1, L2, L3, X) PT_DPP(0, L0, X) PT_DPP(1, L1, X) PT_DPP(2, L2, X) PT_DPP(3, L3, X)
template <int A, int B>
__device__ inline void mat_vec64(double mat, const double x[4], double y[4]) {
    static_assert((A == 0 && B == 1) || (A == 1 && B == 0), "the first two states");
    y[0] = y[1] = y[2] = y[3] = 0.0;
    if constexpr (A == 1)
        asm volatile("s_nop 1\n\t" PT_DPP4(1, 5, 9, 13, 6) PT_DPP4(0, 4, 8, 12, 5) PT_DPP4(2, 6, 10, 14, 7)
                PT_DPP4(3, 7, 11, 15, 8)
            : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3])
            : "v"(mat), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));
    else
        asm volatile("s_nop 1\n\t" PT_DPP4(0, 4, 8, 12, 5) PT_DPP4(1, 5, 9, 13, 6) PT_DPP4(2, 6, 10, 14, 7)
                PT_DPP4(3, 7, 11, 15, 8)
            : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3])
            : "v"(mat), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));
}
#undef PT_DPP4
#undef PT_DPP

// This lane's entry of every category's matrix of an edge.
template <int KP>
struct LaneMats {
    double r[KP];
    __device__ inline LaneMats(const double *pm, int e) {
        const double *q = pm + (size_t)e * KP * 16 + (threadIdx.x & 15);
#pragma unroll
        for (int k = 0; k < KP; ++k) r[k] = q[k * 16];
    }
};

// This lane's entry of W transposed.
__device__ inline double lane_model(const ModelS *md) {
    return md->W[(threadIdx.x & 3) * 4 + ((threadIdx.x >> 2) & 3)];
}

// update_pattern by mat_vec64 (every lane of the wave).
template <int KP, class SA, class SB>
__device__ inline int update_pattern_f64(int K, const LaneMats<KP> &ma, const LaneMats<KP> &mb, const SA &sa,
                                         const SB &sb, double o[KP][4]) {
    const double thr = 0x1p-256, up = 0x1p256;  // Store<double>::kScaleExp
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        double xa[4], xb[4], ya[4], yb[4];
        sa.get(k, xa);
        sb.get(k, xb);
        mat_vec64<1, 0>(ma.r[k], xa, ya);
        mat_vec64<1, 0>(mb.r[k], xb, yb);
        const bool live = k < K;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[k][i] = live ? ya[i] * yb[i] : 0.0;
            mx = fmax(mx, o[k][i]);
        }
    }
    int c = sa.c + sb.c;
    if (mx < thr && mx > 0.0) {
#pragma unroll
        for (int k = 0; k < KP; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[k][i] *= up;
        c += 1;
    }
    return c;
}

// The steps j < ni for which this lane's wave has any of the patterns
// base + j * BS + threadIdx.x.
template <int BS>
__device__ inline int wave_steps(int base, int ni, int np) {
    const int rest = np - base - (int)__builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    return rest > 0 ? min(ni, (rest + BS - 1) / BS) : 0;
}

// Steps taken at once by the FP32 loops below: the sides of all of them are
// fetched before the first is used, so their round trips to memory overlap
// (with eight categories the registers allow one).
template <int KP>
struct StepsAtOnce {
    static constexpr int value = KP <= 4 ? 2 : 1;
};

// N steps of an FP32 OP_UPDATE from pattern p0 (this lane's) on.
template <int BS, int KP, bool TA, bool TB, int N>
__device__ inline void update_steps(const TreeView<float> &v, const Op &op, const EdgeRows<KP> &ma,
                                    const EdgeRows<KP> &mb, int p0) {
    Side<float, KP, TA, false> sa[N];
    Side<float, KP, TB, false> sb[N];
    float4 out[N][KP];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int q = min(p0 + n * BS, v.np - 1);
        sa[n].fetch(v, op.a, q);
        sb[n].fetch(v, op.b, q);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) update_pattern_f32<KP>(v.K, ma, mb, sa[n], sb[n], out[n]);
#pragma unroll
    for (int n = 0; n < N; ++n)
        if (p0 + n * BS < v.np) {
#pragma unroll
            for (int k = 0; k < KP; ++k)
                if (k < v.K) Store<float>::store_raw(slot_ptr<float, KP>(v, op.dst, k, p0 + n * BS), out[n][k]);
        }
}

// One pattern of an OP_UPDATE from its two fetched sides, for the fused
// update and table build: o[k] and the returned scaler count are what
// update_sides computes, by the same expressions in the same order (so both
// paths give identical partials; update_sides keeps its own copy because
// sharing this one changed the register allocation of the FP32 kernels and
// slowed them).
template <typename T, int KP, int PM, class SA, class SB>
__device__ inline int update_pattern(const TreeView<T> &v, const Op &op, const SA &sa, const SB &sb,
                                     double o[KP][4]) {
    const auto pm = pm_base<PM>(v);
    const double thr = ldexp(1.0, -Store<T>::kScaleExp);
    const double up = ldexp(1.0, Store<T>::kScaleExp);
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        double xa[4], xb[4];
        sa.get(k, xa);
        sb.get(k, xb);
        const auto Pa = pm + ((size_t)op.ea * KP + k) * 16;
        const auto Pb = pm + ((size_t)op.eb * KP + k) * 16;
        const bool live = k < v.K;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double xsa = Pa[i * 4] * xa[0] + Pa[i * 4 + 1] * xa[1] + Pa[i * 4 + 2] * xa[2] +
                               Pa[i * 4 + 3] * xa[3];
            const double xsb = Pb[i * 4] * xb[0] + Pb[i * 4 + 1] * xb[1] + Pb[i * 4 + 2] * xb[2] +
                               Pb[i * 4 + 3] * xb[3];
            o[k][i] = live ? xsa * xsb : 0.0;
            mx = fmax(mx, o[k][i]);
        }
    }
    int c = sa.c + sb.c;
    if (mx < thr && mx > 0.0) {
#pragma unroll
        for (int k = 0; k < KP; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[k][i] *= up;
        c += 1;
    }
    return c;
}

// OP_UPDATE for this thread's patterns, sides of kinds TA / TB (tip or slot):
//   dst[k] = (P_k(t_ea) . side a[k]) * (P_k(t_eb) . side b[k]), elementwise over
// states, for every category k, then per-pattern scaling.
template <typename T, int BS, int KP, bool TA, bool TB, int PM>
__device__ inline void update_sides(const TreeView<T> &v, const Op &op, int base, int ni) {
    if constexpr (PM == kPmLds32) {
        const EdgeRows<KP> ma(v.pmf, op.ea), mb(v.pmf, op.eb);
        constexpr int kAtOnce = StepsAtOnce<KP>::value;
        const int nj = wave_steps<BS>(base, ni, v.np);
        int j = 0, p = base + threadIdx.x;
#pragma unroll 1
        for (; j + kAtOnce <= nj; j += kAtOnce, p += kAtOnce * BS)
            update_steps<BS, KP, TA, TB, kAtOnce>(v, op, ma, mb, p);
        if constexpr (kAtOnce == 2) {
            if (j < nj) update_steps<BS, KP, TA, TB, 1>(v, op, ma, mb, p);
        }
        return;
    }
    if constexpr (PM == kPmLds64) {
        const LaneMats<KP> ma(v.pm, op.ea), mb(v.pm, op.eb);
        const int nj = wave_steps<BS>(base, ni, v.np);
#pragma unroll 1
        for (int j = 0; j < nj; ++j) {
            const int p = base + j * BS + threadIdx.x, q = min(p, v.np - 1);
            Side<T, KP, TA> sa;
            Side<T, KP, TB> sb;
            sa.fetch(v, op.a, q);
            sb.fetch(v, op.b, q);
            double o[KP][4];
            const int c = update_pattern_f64<KP>(v.K, ma, mb, sa, sb, o);
            if (p < v.np) {
#pragma unroll
                for (int k = 0; k < KP; ++k)
                    if (k < v.K) Store<T>::store(slot_ptr<T, KP>(v, op.dst, k, p), o[k]);
                v.cnt[(size_t)op.dst * v.P + p] = (uint16_t)c;
            }
        }
        return;
    }
    const auto pm = pm_base<PM>(v);
    const double thr = ldexp(1.0, -Store<T>::kScaleExp);
    const double up = ldexp(1.0, Store<T>::kScaleExp);
#pragma unroll 1
    for (int j = 0; j < ni; ++j) {
        const int p = base + j * BS + threadIdx.x;
        if (p >= v.np) break;
        Side<T, KP, TA> sa;
        Side<T, KP, TB> sb;
        sa.fetch(v, op.a, p);
        sb.fetch(v, op.b, p);
        double o[KP][4];
        double mx = 0.0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            double xa[4], xb[4];
            sa.get(k, xa);
            sb.get(k, xb);
            const auto Pa = pm + ((size_t)op.ea * KP + k) * 16;
            const auto Pb = pm + ((size_t)op.eb * KP + k) * 16;
            const bool live = k < v.K;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double xsa = Pa[i * 4] * xa[0] + Pa[i * 4 + 1] * xa[1] + Pa[i * 4 + 2] * xa[2] +
                                   Pa[i * 4 + 3] * xa[3];
                const double xsb = Pb[i * 4] * xb[0] + Pb[i * 4 + 1] * xb[1] + Pb[i * 4 + 2] * xb[2] +
                                   Pb[i * 4 + 3] * xb[3];
                o[k][i] = live ? xsa * xsb : 0.0;
                mx = fmax(mx, o[k][i]);
            }
        }
        int c = sa.c + sb.c;
        if (mx < thr && mx > 0.0) {
#pragma unroll
            for (int k = 0; k < KP; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[k][i] *= up;
            c += 1;
        }
#pragma unroll
        for (int k = 0; k < KP; ++k)
            if (k < v.K) Store<T>::store(slot_ptr<T, KP>(v, op.dst, k, p), o[k]);
        v.cnt[(size_t)op.dst * v.P + p] = (uint16_t)c;
    }
}

// OP_UPDATE for this thread's patterns base + j*BS, j < ni.
template <typename T, int BS, int KP, int PM = kPmLds>
__device__ inline void do_update(const TreeView<T> &v, const Op &op, int base, int ni) {
    if (op.a < 0) {
        if (op.b < 0) update_sides<T, BS, KP, true, true, PM>(v, op, base, ni);
        else update_sides<T, BS, KP, true, false, PM>(v, op, base, ni);
    } else {
        if (op.b < 0) update_sides<T, BS, KP, false, true, PM>(v, op, base, ni);
        else update_sides<T, BS, KP, false, false, PM>(v, op, base, ni);
    }
}

// t-independent part of a pattern's lnL: scaler corrections and the 1/K
// category weight.
template <typename T>
__device__ inline double const_term(int c, double logK) {
    return -((double)c * Store<T>::kScaleExp * kLn2 + logK);
}

struct Sums3 {
    double l0, l1, l2;
    int parity;
};

// Eigenbasis coefficients from the two sides' state vectors of one category.
__device__ inline void coeffs_x(const ModelS *md, const double xa[4], const double xb[4], double s[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        double ua = 0.0, vb = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double wim = md->W[i * 4 + m];
            ua += wim * xa[i];
            vb += wim * xb[i];
        }
        s[m] = ua * vb;
    }
}

// One category's table coefficients for one pattern, in FP64, stored at dst
// and returned in sk.
template <class SA, class SB>
__device__ inline void table_coeffs(const ModelS *md, const SA &sa, const SB &sb, int k, double *dst, double sk[4]) {
    double xa[4], xb[4];
    sa.get(k, xa);
    sb.get(k, xb);
    coeffs_x(md, xa, xb, sk);
    Store<double>::store(dst, sk);
}

// The coefficients of every category in FP32, for tables stored in FP32 (the
// optimisation loop with FP32 partials): computed in the precision they are
// stored in, on the matrix cores (row: this lane's of W transposed).
template <int KP, class SA, class SB>
__device__ inline void coeffs_f32(const float4 &row, const SA &sa, const SB &sb, float4 s[KP]) {
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        float xa[4], xb[4];
        sa.getf(k, xa);
        sb.getf(k, xb);
        const F4 ua = mat_vec<0, 1>(row, xa), vb = mat_vec<0, 1>(row, xb);
        s[k] = make_float4(ua[0] * vb[0], ua[1] * vb[1], ua[2] * vb[2], ua[3] * vb[3]);
    }
}

__device__ inline float4 model_row(const ModelS *md) {
    return reinterpret_cast<const float4 *>(md->WfT)[threadIdx.x & 3];
}

// This thread's contributions to lnL, d1 and d2 across an edge whose sides
// are of kinds TA / TB, with the exponentials of its length in wx.
template <typename T, int BS, int KP, bool TA, bool TB>
__device__ inline void eval_sides(const TreeView<T> &v, int a, int b, int base, int ni, const double *wx,
                                  double logK, Sums3 &r) {
    const ModelS *md = v.m;
#pragma unroll 1
    for (int j = 0; j < ni; ++j) {
        const int p = base + j * BS + threadIdx.x;
        if (p >= v.np) break;
        Side<T, KP, TA> sa;
        Side<T, KP, TB> sb;
        sa.fetch(v, a, p);
        sb.fetch(v, b, p);
        const double w = ldg(v.w + p);
        double L = 0.0, L1 = 0.0, L2 = 0.0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (k < v.K) {
                double xa[4], xb[4], sk[4];
                sa.get(k, xa);
                sb.get(k, xb);
                coeffs_x(md, xa, xb, sk);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    L += sk[m] * wx[k * 4 + m];
                    L1 += sk[m] * wx[4 * kMaxCats + k * 4 + m];
                    L2 += sk[m] * wx[8 * kMaxCats + k * 4 + m];
                }
            }
        }
        const double inv = recip(L);
        const double r1 = L1 * inv;
        r.l0 += w * (log(L) + const_term<T>(sa.c + sb.c, logK));
        r.l1 += w * r1;
        r.l2 += w * (L2 * inv - r1 * r1);
    }
}

// OP_EVAL: block totals of lnL and its first two derivatives across an edge
// at length t, computed on the fly from the two sides.
template <typename T, int BS, int KP>
__device__ inline Sums3 eval_edge(const TreeView<T> &v, int a, int b, int base, int ni, double t, double *red,
                                  double *wx, int parity, GroupS *gs = nullptr) {
    wave_expo<double>(wx, v.m, v.K, t);
    const double logK = v.m->log_k;
    Sums3 r;
    r.l0 = r.l1 = r.l2 = 0.0;
    if (a < 0) {
        if (b < 0) eval_sides<T, BS, KP, true, true>(v, a, b, base, ni, wx, logK, r);
        else eval_sides<T, BS, KP, true, false>(v, a, b, base, ni, wx, logK, r);
    } else {
        if (b < 0) eval_sides<T, BS, KP, false, true>(v, a, b, base, ni, wx, logK, r);
        else eval_sides<T, BS, KP, false, false>(v, a, b, base, ni, wx, logK, r);
    }
    group_sum3<BS>(r.l0, r.l1, r.l2, red, parity, gs);
    r.parity = parity;
    return r;
}

// Whether the optimisation loop evaluates lnL at the end of a pass: with FP64
// partials the pass rule needs it; with FP32 partials the rule uses the
// steps' model values, and lnL is evaluated once, at the final lengths, by
// the register-resident pass (k_prune).  (A last pass of this kernel over FP64
// partials stored in the tree's buffer, and a pass lnL that nothing read, cost
// 16.3 against 8.6 ms a batch of 1024 radius-0 proposals of 64 taxa x 1711
// patterns, mostly that pass's 28 GB of traffic, 25.6 against 20.8 ms for 256
// trees over four alignments and 5.26 against 4.81 ms for 48 of 27 taxa.)
template <typename T>
constexpr bool kPassLnl = std::is_same<T, double>::value;

struct EdgeResult {
    double t, lnl;
    double gain;  // the objective's gain from the step by its quadratic model at the start, or +inf
    double rise;  // the same model's value for the step, whatever the sign of its second derivative
    int parity, iters;
    long long cyc_table, cyc_iters;
};

// One row of an edge's eigenbasis table from the pattern's two sides (the
// table is symmetric in them), for the fused update and table build: the
// row, weight and sums that table_sides gives for the pattern, by the same
// expressions in the same order (table_sides keeps its own copy for the same
// reason as update_sides).  Stores the row of every live category into tab
// ([k][row][4]) and the weight into wrow, adds the pattern's t-independent
// lnL term to cterm and, with FUSE, its terms of the first Newton iteration
// at the exponentials wxe to f1 and f2.
template <int KP, bool FUSE, class SA, class SB>
__device__ inline void table_row(const TreeView<double> &v, const SA &sa, const SB &sb, int p, size_t rows, double *tab,
                                 double *wrow, double w, double logK, const double *wxe, double &cterm, double &f1,
                                 double &f2) {
    const ModelS *md = v.m;
    cterm += w * const_term<double>(sa.c + sb.c, logK);
    wrow[p] = w;
    double L = 0.0, L1 = 0.0, L2 = 0.0;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        if (k < v.K) {
            double sk[4];
            table_coeffs(md, sa, sb, k, tab + ((size_t)k * rows + p) * 4, sk);
            if constexpr (FUSE) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    L += sk[m] * wxe[k * 4 + m];
                    L1 += sk[m] * wxe[4 * kMaxCats + k * 4 + m];
                    L2 += sk[m] * wxe[8 * kMaxCats + k * 4 + m];
                }
            }
        }
    }
    if constexpr (FUSE) {
        const double ia = recip(L);
        const double r1 = L1 * ia;
        f1 += w * r1;
        f2 += w * (L2 * ia - r1 * r1);
    }
}

// The same by mat_vec64 (mat: lane_model), by every lane of the wave; lanes
// with no pattern (valid false) fill rows that no one reads.
template <int KP, bool FUSE, class SA, class SB>
__device__ inline void table_row_f64(const TreeView<double> &v, double mat, const SA &sa, const SB &sb, int p,
                                     bool valid, size_t rows, double *tab, double *wrow, double w, double logK,
                                     const double *wxe, double &cterm, double &f1, double &f2) {
    wrow[p] = w;
    double L = 0.0, L1 = 0.0, L2 = 0.0;
    const LaneExpo e(wxe);
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        if (k < v.K) {
            double xa[4], xb[4], ua[4], vb[4], sk[4];
            sa.get(k, xa);
            sb.get(k, xb);
            mat_vec64<0, 1>(mat, xa, ua);
            mat_vec64<0, 1>(mat, xb, vb);
#pragma unroll
            for (int m = 0; m < 4; ++m) sk[m] = ua[m] * vb[m];
            Store<double>::store(tab + ((size_t)k * rows + p) * 4, sk);
            if constexpr (FUSE) add_expo(k, e, sk, L, L1, L2);
        }
    }
    if (!valid) return;
    cterm += w * const_term<double>(sa.c + sb.c, logK);
    if constexpr (FUSE) {
        const double ia = recip(L);
        const double r1 = L1 * ia;
        f1 += w * r1;
        f2 += w * (L2 * ia - r1 * r1);
    }
}

// The same for N rows from their FP32 coefficients s (this lane's patterns
// p0, p0 + BS, ... below np).
template <int BS, int KP, bool FUSE, int N>
__device__ inline void table_rows(int K, int np, const float4 (&s)[N][KP], int p0, size_t rows, float *tab, double *wrow,
                                  const double (&w)[N], const double *wxe, double &f1, double &f2) {
    double L[N] = {}, L1[N] = {}, L2[N] = {};
    if constexpr (FUSE) {
        const LaneExpo e(wxe);
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (k < K) {
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    double sk[4];
                    Store<float>::widen(s[n][k], sk);
                    add_expo(k, e, sk, L[n], L1[n], L2[n]);
                }
            }
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int p = p0 + n * BS;
        if (p >= np) break;
        wrow[p] = w[n];
#pragma unroll
        for (int k = 0; k < KP; ++k)
            if (k < K) *reinterpret_cast<float4 *>(tab + ((size_t)k * rows + p) * 4) = s[n][k];
        if constexpr (FUSE) {
            const double ia = recip(L[n]);
            const double r1 = L1[n] * ia;
            f1 += w[n] * r1;
            f2 += w[n] * (L2[n] * ia - r1 * r1);
        }
    }
}

// N steps of the FP32 eigenbasis table from pattern p0 (this lane's) on.
template <int BS, int KP, bool TA, bool TB, bool FUSE, int N>
__device__ inline void table_steps(const TreeView<float> &v, int a, int b, int p0, size_t rows, float *tab,
                                   double *wrow, const float4 &row, const double *wxe, double &f1, double &f2) {
    Side<float, KP, TA, false> sa[N];
    Side<float, KP, TB, false> sb[N];
    double w[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int q = min(p0 + n * BS, v.np - 1);
        sa[n].fetch(v, a, q);
        sb[n].fetch(v, b, q);
        w[n] = ldg(v.w + q);
    }
    float4 s[N][KP];
#pragma unroll
    for (int n = 0; n < N; ++n) coeffs_f32<KP>(row, sa[n], sb[n], s[n]);
    table_rows<BS, KP, FUSE, N>(v.K, v.np, s, p0, rows, tab, wrow, w, wxe, f1, f2);
}

// The eigenbasis table of an edge whose sides are of kinds TA / TB: this
// thread's rows of tab ([k][row][4]) and wrow; returns the sum of its rows'
// t-independent lnL terms.  FUSE: also adds the rows' terms of the first
// Newton iteration, at the exponentials wxe, to f1 and f2, from the values as
// stored and in the order of the row passes, so the sums are the ones a row
// pass over the finished table would give.
template <typename T, int BS, int KP, bool TA, bool TB, bool FUSE, bool PAIR>
__device__ inline double table_sides(const TreeView<T> &v, int a, int b, int ni, size_t rows, T *tab, double *wrow,
                                     double logK, const double *wxe, double &f1, double &f2) {
    double cterm = 0.0;
    if constexpr (std::is_same<T, float>::value) {
        // (the kernels with the fused update and table build leave PAIR off
        // to make room for it)
        constexpr int kAtOnce = PAIR ? StepsAtOnce<KP>::value : 1;
        const float4 row = model_row(v.m);
        const int nj = wave_steps<BS>(0, ni, v.np);
        int j = 0, p = threadIdx.x;
#pragma unroll 1
        for (; j + kAtOnce <= nj; j += kAtOnce, p += kAtOnce * BS)
            table_steps<BS, KP, TA, TB, FUSE, kAtOnce>(v, a, b, p, rows, tab, wrow, row, wxe, f1, f2);
        if constexpr (kAtOnce == 2) {
            if (j < nj) table_steps<BS, KP, TA, TB, FUSE, 1>(v, a, b, p, rows, tab, wrow, row, wxe, f1, f2);
        }
    } else if constexpr (OptPm<T, KP>::value == kPmLds64) {
        const double mat = lane_model(v.m);
        const int nj = wave_steps<BS>(0, ni, v.np);
#pragma unroll 1
        for (int j = 0; j < nj; ++j) {
            const int p = j * BS + threadIdx.x, q = min(p, v.np - 1);
            Side<T, KP, TA> sa;
            Side<T, KP, TB> sb;
            sa.fetch(v, a, q);
            sb.fetch(v, b, q);
            table_row_f64<KP, FUSE>(v, mat, sa, sb, p, p < v.np, rows, tab, wrow, ldg(v.w + q), logK, wxe, cterm, f1,
                                    f2);
        }
    } else {
#pragma unroll 1
        for (int j = 0; j < ni; ++j) {
            const int p = j * BS + threadIdx.x;
            if (p >= v.np) break;
            Side<T, KP, TA> sa;
            Side<T, KP, TB> sb;
            sa.fetch(v, a, p);
            sb.fetch(v, b, p);
            table_row<KP, FUSE>(v, sa, sb, p, rows, tab, wrow, ldg(v.w + p), logK, wxe, cterm, f1, f2);
        }
    }
    return cterm;
}

// An OP_UPDATE whose output is one side of the next OP_NEWTON, with one
// pattern per thread: the update's loads and those of the edge's other side
// (kind TO) issue together, and the edge's table row is built from the
// update's output, kept in registers and rounded as stored, instead of being
// read back.  The table is symmetric in the two sides, so which side the
// update made does not matter.  Returns the row's t-independent lnL term
// (see table_row).
template <typename T, int BS, int KP, bool TA, bool TB, bool TO, bool FUSE, int PM>
__device__ inline double update_table_sides(const TreeView<T> &v, const Op &op, int other, T *tab, double *wrow,
                                            double logK, double t, double *wxe, double &f1, double &f2) {
    double cterm = 0.0;
    const int p = threadIdx.x;
    if constexpr (std::is_same<T, float>::value) {
        if (wave_steps<BS>(0, 1, v.np) == 0) return 0.0;
        const int q = min(p, v.np - 1);
        Side<T, KP, TA, false> sa;
        Side<T, KP, TB, false> sb;
        Side<T, KP, TO, false> so;
        sa.fetch(v, op.a, q);
        sb.fetch(v, op.b, q);
        so.fetch(v, other, q);
        const double w = ldg(v.w + q);
        if constexpr (FUSE) wave_expo<T>(wxe, v.m, v.K, t);  // while the sides arrive
        const EdgeRows<KP> ma(v.pmf, op.ea), mb(v.pmf, op.eb);
        Side<T, KP, false, false> made;
        update_pattern_f32<KP>(v.K, ma, mb, sa, sb, made.r);
        float4 s[1][KP];
        coeffs_f32<KP>(model_row(v.m), made, so, s[0]);
        const double w1[1] = {w};
        table_rows<BS, KP, FUSE, 1>(v.K, v.np, s, p, (size_t)BS, tab, wrow, w1, wxe, f1, f2);
        if (p < v.np) {
#pragma unroll
            for (int k = 0; k < KP; ++k)
                if (k < v.K) Store<T>::store_raw(slot_ptr<T, KP>(v, op.dst, k, p), made.r[k]);
        }
    } else {
        static_assert(PM == kPmLds64, "the fused update and table build: FP32, or FP64 up to four categories");
        if (wave_steps<BS>(0, 1, v.np) == 0) return 0.0;
        const int q = min(p, v.np - 1);
        Side<T, KP, TA> sa;
        Side<T, KP, TB> sb;
        Side<T, KP, TO> so;
        sa.fetch(v, op.a, q);
        sb.fetch(v, op.b, q);
        so.fetch(v, other, q);
        const double w = ldg(v.w + q);
        if constexpr (FUSE) wave_expo<T>(wxe, v.m, v.K, t);  // while the sides arrive
        const LaneMats<KP> ma(v.pm, op.ea), mb(v.pm, op.eb);
        Side<T, KP, false> made;
        double o[KP][4];
        made.c = update_pattern_f64<KP>(v.K, ma, mb, sa, sb, o);
#pragma unroll
        for (int k = 0; k < KP; ++k) made.r[k] = Store<T>::pack(o[k]);
        table_row_f64<KP, FUSE>(v, lane_model(v.m), made, so, p, p < v.np, (size_t)BS, tab, wrow, w, logK, wxe, cterm,
                                f1, f2);
        if (p < v.np) {
#pragma unroll
            for (int k = 0; k < KP; ++k)
                if (k < v.K) Store<T>::store_raw(slot_ptr<T, KP>(v, op.dst, k, p), made.r[k]);
            v.cnt[(size_t)op.dst * v.P + p] = (uint16_t)made.c;
        }
    }
    return cterm;
}

// Newton pass over two table rows r0 and r1 (r1 < 0: only r0), so that
// each exponential read from the wave's LDS slice serves two patterns.  Adds
// the rows' d1 and d2 terms, or with lnl_only their weighted log L to d0; each
// row's sums run in the same order as for a single row.
template <typename T, int KP>
__device__ inline void newton_rows2(const T *tab, const double *wrow, size_t rows, int r0, int r1, const double *wx,
                                    int K, bool lnl_only, double &d0, double &d1, double &d2) {
    using Raw = typename Store<T>::Raw;
    constexpr int N = 2;
    const bool two = r1 >= 0;
    const int r[2] = {r0, two ? r1 : r0};
    Raw raw[N][KP];
    double w[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
#pragma unroll
        for (int k = 0; k < KP; ++k)
            if (k < K) raw[n][k] = Store<T>::load_raw(tab + ((size_t)k * rows + r[n]) * 4);
        w[n] = wrow[r[n]];
    }
    double L[N] = {}, L1[N] = {}, L2[N] = {};
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        if (k < K) {
            double s[N][4];
#pragma unroll
            for (int n = 0; n < N; ++n) Store<T>::widen(raw[n][k], s[n]);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double e0 = wx[k * 4 + m], e1 = wx[4 * kMaxCats + k * 4 + m],
                             e2 = wx[8 * kMaxCats + k * 4 + m];
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    L[n] += s[n][m] * e0;
                    L1[n] += s[n][m] * e1;
                    L2[n] += s[n][m] * e2;
                }
            }
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (n == 1 && !two) break;
        if (lnl_only) {
            d0 += w[n] * log(L[n]);
            continue;
        }
        const double ia = recip(L[n]);
        const double q = L1[n] * ia;
        d1 += w[n] * q;
        d2 += w[n] * (L2[n] * ia - q * q);
    }
}

// The same up to four categories, by every lane of a wave: rows r0 and (N = 2)
// r0 + step, of which those below np count.
template <typename T, int KP, int N>
__device__ inline void newton_rows_lanes(const T *tab, const double *wrow, size_t rows, int r0, int step, int np,
                                         const LaneExpo &e, int K, bool lnl_only, double &d0, double &d1, double &d2) {
    typename Store<T>::Raw raw[N][KP];
    double w[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
#pragma unroll
        for (int k = 0; k < KP; ++k)
            if (k < K) raw[n][k] = Store<T>::load_raw(tab + ((size_t)k * rows + r0 + n * step) * 4);
        w[n] = wrow[r0 + n * step];
    }
    double L[N] = {}, L1[N] = {}, L2[N] = {};
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        if (k < K) {
#pragma unroll
            for (int n = 0; n < N; ++n) {
                double s[4];
                Store<T>::widen(raw[n][k], s);
                add_expo(k, e, s, L[n], L1[n], L2[n]);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (r0 + n * step >= np) break;
        if (lnl_only) {
            d0 += w[n] * log(L[n]);
            continue;
        }
        const double ia = recip(L[n]);
        const double q = L1[n] * ia;
        d1 += w[n] * q;
        d2 += w[n] * (L2[n] * ia - q * q);
    }
}

// A Newton pass over this lane's rows (nj of them, nw the most of a lane of
// the wave) at the exponentials wx.
template <typename T, int BS, int KP>
__device__ inline void newton_pass(const T *tab, const double *wrow, size_t rows, int nj, int nw, int np,
                                   const double *wx, int K, bool lnl_only, double &d0, double &d1, double &d2) {
    if constexpr (KP <= 4) {
        const LaneExpo e(wx);
        int j = 0;
#pragma unroll 1
        for (; j + 2 <= nw; j += 2)
            newton_rows_lanes<T, KP, 2>(tab, wrow, rows, j * BS + threadIdx.x, BS, np, e, K, lnl_only, d0, d1, d2);
        if (j < nw)
            newton_rows_lanes<T, KP, 1>(tab, wrow, rows, j * BS + threadIdx.x, BS, np, e, K, lnl_only, d0, d1, d2);
    } else {
#pragma unroll 1
        for (int j = 0; j < nj; j += 2)
            newton_rows2<T, KP>(tab, wrow, rows, j * BS + threadIdx.x, j + 1 < nj ? (j + 1) * BS + threadIdx.x : -1, wx,
                                K, lnl_only, d0, d1, d2);
    }
}

// Relative Newton step below which an edge's iterations end without a
// confirming evaluation (see newton_edge).  Measured on the 48 C2
// neighbours: 1.46 -> 1.07 iterations per edge step (FP32 partials) and
// 1.70 -> 1.04 (FP64), for at most one more pass on a few trees.
constexpr double kNewtonAccept = 0.03;

// Over-relaxation of the edge steps from a tree's second pass on: an edge
// whose Newton step exceeds tol_t relative moves kRelax times that step
// (nonlinear successive over-relaxation of the coordinate-wise maximisation;
// Ortega and Rheinboldt, Iterative Solution of Nonlinear Equations in Several
// Variables, 1970).  The lengths are coupled, so plain coordinate steps
// converge linearly and slowly on some trees; the fixed point is the same
// maximum.  Steps below tol_t are not relaxed, so a tree's last pass (every
// step below tol_t) leaves plain Newton results.  Measured with the oracle's
// arithmetic: on the 48 C2 neighbours, passes mean 7.4 -> 6.6 and max 11 -> 8
// (FP32 tolerances) and mean 11.7 -> 9.4, max 18 -> 12 (FP64 tolerances); on
// 64-taxon trees mean 14.9 -> 9.3, max 18 -> 14; 1.3 and above took more
// passes.
constexpr double kRelax = 1.2;

// An edge's table built ahead of newton_edge (by update_table_sides): this
// thread's t-independent lnL term and first-iteration derivative terms.
struct EdgePre {
    double cterm, f1, f2;
};

// The first iteration's derivative terms are summed while the table is built
// (with the same rounding and order as the row passes of newton_edge), up to
// four padded categories: with eight the extra registers would spill.
template <int KP>
struct FuseFirst {
    static constexpr bool value = KP <= 4;
};

// OP_UPDATE of slot op.dst fused with the table build of the next OP_NEWTON,
// whose other side is `other`, at its current length t (one pattern per
// thread).
template <typename T, int BS, int KP, int PM>
__device__ inline EdgePre update_and_table(const TreeView<T> &v, const Op &op, int other, double t, T *tab,
                                           double *wrow, double *wx) {
    constexpr bool kFuse = FuseFirst<KP>::value;
    const double logK = v.m->log_k;
    EdgePre pre;
    pre.f1 = pre.f2 = 0.0;
#define PT_UT(TA, TB, TO)                                                                                        \
    pre.cterm = update_table_sides<T, BS, KP, TA, TB, TO, kFuse, PM>(v, op, other, tab, wrow, logK, t, wx, pre.f1, \
                                                                      pre.f2)
    if (op.a < 0) {
        if (op.b < 0) {
            if (other < 0) PT_UT(true, true, true); else PT_UT(true, true, false);
        } else {
            if (other < 0) PT_UT(true, false, true); else PT_UT(true, false, false);
        }
    } else {
        if (op.b < 0) {
            if (other < 0) PT_UT(false, true, true); else PT_UT(false, true, false);
        } else {
            if (other < 0) PT_UT(false, false, true); else PT_UT(false, false, false);
        }
    }
#undef PT_UT
    return pre;
}

// OP_NEWTON: safeguarded, projected Newton on the length of one edge, for
// lnL(t) - prior_rate * t (prior_rate 0: maximum likelihood).
//  - the eigenbasis coefficients of this thread's patterns are computed once
//    into `tab` (layout [k][row][4], rows = BS*ni pattern slots) and the
//    pattern weights into `wrow` (in LDS, or in a per-block global buffer),
//    then every iteration is a pass over them plus one block sum (up to four
//    padded categories, the first iteration's terms are summed while the
//    table is built);
//  - the bracket (lo, hi) starts as [t_min, t_max] and shrinks to t on the
//    side the first derivative points away from;
//  - a Newton step is taken when d2 < 0 and it stays in the bracket (the
//    original bounds count as inside), else the bracket is bisected
//    geometrically;
//  - a bound with the derivative pointing outwards is an optimum;
//  - a step of at most tol * max(t, 1e-6) is converged and not taken; a
//    Newton step of at most accept * max(t, 1e-6) (accept: the larger of
//    sqrt(tol) and kNewtonAccept, a square root taken once per tree) is
//    taken and ends the edge (quadratic convergence; the next pass revisits
//    the edge);
//  - the returned t is t_in + relax * (t_newton - t_in), kept in
//    [t_min, t_max], when that step exceeds tol_t * max(t_in, 1e-6), else
//    the Newton result;
//  - with want_lnl, lnL is evaluated at the returned t (FP64 partials).
// All threads hold identical block totals, so every thread takes the same
// decisions.
template <typename T, int BS, int KP, bool PAIR = true>
__device__ inline EdgeResult newton_edge(const TreeView<T> &v, int a, int b, double t, bool want_lnl,
                                         const OptParams &opt, T *tab, double *wrow, int ni, double *red,
                                         double *wx, int parity, GroupS *gs, double relax, double accept,
                                         const EdgePre *pre = nullptr) {
    const double t_in = t;
    const size_t rows = (size_t)BS * ni;
    const double logK = v.m->log_k;
    const long long c0 = clock64();
    constexpr bool kFuse = FuseFirst<KP>::value;
    double f1 = 0.0, f2 = 0.0;
    double cterm;
    if (pre) {  // the table is built (one pattern per thread)
        cterm = pre->cterm;
        f1 = pre->f1;
        f2 = pre->f2;
    } else {
        const double *wxe = wx;
        if constexpr (kFuse) wave_expo<T>(wx, v.m, v.K, t);
        if (a < 0) {
            if (b < 0) cterm = table_sides<T, BS, KP, true, true, kFuse, PAIR>(v, a, b, ni, rows, tab, wrow, logK, wxe, f1, f2);
            else cterm = table_sides<T, BS, KP, true, false, kFuse, PAIR>(v, a, b, ni, rows, tab, wrow, logK, wxe, f1, f2);
        } else {
            if (b < 0) cterm = table_sides<T, BS, KP, false, true, kFuse, PAIR>(v, a, b, ni, rows, tab, wrow, logK, wxe, f1, f2);
            else cterm = table_sides<T, BS, KP, false, false, kFuse, PAIR>(v, a, b, ni, rows, tab, wrow, logK, wxe, f1, f2);
        }
    }
    // rows this thread owns: tid + j*BS < P
    const int nj = v.np > (int)threadIdx.x ? min(ni, (v.np - (int)threadIdx.x + BS - 1) / BS) : 0;
    const int nw = wave_steps<BS>(0, ni, v.np);  // the most rows of a lane of this wave
    const long long c1 = clock64();
    double lo = opt.t_min, hi = opt.t_max;
    double d1_0 = 0.0, d2_0 = 0.0;  // derivatives at the starting length
    int iter = 1;
    for (;; ++iter) {
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        if (kFuse && iter == 1) {
            d1 = f1;
            d2 = f2;
        } else {
            // (FP32 partials: FP32 exponentials suffice for the derivatives,
            // they only steer Newton)
            wave_expo<T>(wx, v.m, v.K, t);
            newton_pass<T, BS, KP>(tab, wrow, rows, nj, nw, v.np, wx, v.K, false, d0, d1, d2);
        }
        group_sum3<BS>(d0, d1, d2, red, parity, gs);
        d1 -= opt.prior_rate;  // MAP: the exponential prior's log density is linear in t
        if (iter == 1) {
            d1_0 = d1;
            d2_0 = d2;
        }
        if (iter >= opt.max_newton) break;
        if (d1 > 0.0) lo = t;
        else if (d1 < 0.0) hi = t;
        else break;
        if ((t <= opt.t_min && d1 <= 0.0) || (t >= opt.t_max && d1 >= 0.0)) break;
        double tn = d2 < 0.0 ? t - d1 / d2 : NAN;
        if (tn < opt.t_min) tn = opt.t_min;
        if (tn > opt.t_max) tn = opt.t_max;
        const bool inside = !isnan(tn) && (tn > lo || (lo == opt.t_min && tn == opt.t_min)) &&
                            (tn < hi || (hi == opt.t_max && tn == opt.t_max));
        if (!inside) tn = sqrt(lo * hi);
        const double dt = fabs(tn - t), scale = fmax(t, 1e-6);
        if (dt <= opt.tol_newton * scale) break;
        t = tn;
        // Newton converges quadratically near the optimum: after a Newton
        // step of relative size d the remaining error is of order d^2, so a
        // step of at most kNewtonAccept (or sqrt(tol_newton)) relative is
        // taken without a confirming evaluation.  The next pass revisits the
        // edge, and the pass-level rule (no step above tol_t) bounds the
        // final accuracy.
        if (inside && dt <= accept * scale) break;
    }
    if (relax != 1.0 && fabs(t - t_in) > opt.tol_t * fmax(t_in, 1e-6))
        t = fmin(fmax(t_in + relax * (t - t_in), opt.t_min), opt.t_max);
    double lnl = 0.0;
    if (kPassLnl<T> && want_lnl) {
        wave_expo<double>(wx, v.m, v.K, t);
        double l0 = cterm, z1 = 0.0, z2 = 0.0;
        newton_pass<T, BS, KP>(tab, wrow, rows, nj, nw, v.np, wx, v.K, true, l0, z1, z2);
        group_sum3<BS>(l0, z1, z2, red, parity, gs);
        lnl = l0;
    }
    EdgeResult r;
    r.t = t;
    r.lnl = lnl;
    r.parity = parity;
    r.iters = iter;
    r.cyc_table = c1 - c0;
    r.cyc_iters = clock64() - c1;
    {
        const double dt = t - t_in;
        r.rise = d1_0 * dt + 0.5 * d2_0 * dt * dt;
        r.gain = d2_0 < 0.0 ? r.rise : INFINITY;
    }
    return r;
}

template <typename T>
__device__ inline TreeView<T> make_view(const TreeDev &td, const AlnDev *aln, const BatchArgs &a,
                                        const ModelS *m, const double *pm_lds) {
    TreeView<T> v;
    v.m = m;
    v.pm = pm_lds;
    v.pmf = nullptr;
    v.tips = aln->tips;
    v.w = aln->w;
    v.clv = reinterpret_cast<T *>(a.clv) + td.clv_off;
    v.cnt = a.cnt + td.cnt_off;
    v.P = aln->P;
    v.np = aln->P;
    v.K = aln->K;
    return v;
}

// Runs its argument with KP = the padded category count kp.
#define PT_KP_SWITCH(...)                                   \
    switch (kp) {                                           \
    case 1: { constexpr int KP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int KP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int KP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int KP = 8; __VA_ARGS__; } break;   \
    default: break;                                         \
    }

}  // namespace
}  // namespace pt
