// Fused graph-transformer attention forward over a CSR graph, for gfx950.
//
// Operation: paper Section 2.2, attention family (iii) with graph-transformer
// logits; single streaming pass with online softmax (Section 3.2, Appendix
// D.2).  For every destination row i and head h:
//     out[i,h,:] = sum_e softmax_e(scale * <Q[i,h,:], K[j_e,h,:]>) V[j_e,h,:]
// The same skeleton evaluates the GATv2 layer of the same family (Section 2.2;
// Appendix D.2, fused GATv2 forward), selected by the KIND template argument:
//     out[i,h,:] = sum_e softmax_e(<a[h,:], LeakyReLU(L[i,h,:] + R[j_e,h,:])>) R[j_e,h,:]
// where each CSR entry gathers one row (R serves as key and value).
//
// Mapping (designed for 64-wide wavefronts and eight XCDs with an L2 each, not
// taken from the paper's one-block-per-(node, head) CUDA layout):
//   * A call runs over slices of the node row: the heads of 256 bytes, or one
//     head of D elements where that is more.  A lane group of G lanes covers a
//     slice with one 16-byte load per lane, so every gathered K/V slice is one
//     coalesced request of whole cache lines, and a wave holds P = 64/G groups.
//   * A head's D elements occupy HL = D*sizeof(T)/16 consecutive lanes; the
//     score of a head is reduced across those lanes with DPP lane swaps.
//   * Degree-aware work split (Appendix B.1; Appendix D.1 for the chunked
//     heavy-node scheme): light rows get one group each; longer rows are cut
//     into pieces of one group each, the q-th eighth of a row's entries on XCD q
//     (see gt_rows.hpp), whose partial (max, sum, acc) states are merged in a
//     fixed order by a second kernel, so results are bitwise reproducible and
//     need no float atomics.
//   * Each group processes U entries per step: all U K-row and V-row loads
//     are issued before any is consumed, then one online-softmax update
//     covers the U entries (one rescale per step instead of one per entry).
//   * Neighbour indices are staged in LDS tiles loaded with one coalesced
//     4-byte load per lane.

#include <hip/hip_runtime.h>

#include <array>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <map>
#include <type_traits>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "gt_attn.h"

// Workspace of the allocation-free entry point (gt_attn_fwd_noalloc): one
// array per device, held from the library's load until the process ends.
// Host code never passes `scratch` itself to a kernel (in host code the name
// is a stand-in, not a device address): it takes the device address from
// hipGetSymbolAddress once per device (scratch_of below).
static __device__ __align__(256) char scratch[size_t(256) << 20];

namespace {

#include "gt_plan.hpp"

static_assert(sizeof(scratch) == kScratchBytes, "the plan bounds workspaces by the array's size");
constexpr int kBlock = kWave * kWavesPerBlock;

// Score kinds of the attention skeleton.
// KIND_GT_BF16W: the graph-transformer score with each softmax weight rounded
// to bf16 for P*V (bf16 rows pair two entries per dot2 instead of widening
// their value rows); an option for rows whose steps are arithmetic-bound.
enum { KIND_GT = 0, KIND_GATV2 = 1, KIND_GT_BF16W = 2 };

struct bf16_tag {};

template <typename T> struct Elt;
template <> struct Elt<float> { static constexpr int kBytes = 4; };
template <> struct Elt<bf16_tag> { static constexpr int kBytes = 2; };

template <typename T, int H, int D>
struct Geo {
    static constexpr int kEB = Elt<T>::kBytes;
    static constexpr int kEPV = 16 / kEB;                   // elements per 16-B vector
    static constexpr int kRowBytes = H * D * kEB;           // one node row, all heads
    static constexpr int kNVec = kRowBytes / 16;
    static constexpr int kG = kNVec < kWave ? kNVec : kWave;  // lanes per group
    static constexpr int kNV = kNVec / kG;                  // 16-B vectors per lane
    static constexpr int kP = kWave / kG;                   // groups per wave
    static constexpr int kHL = D * kEB / 16;                // lanes per head (per vector slot)
    static constexpr int kU0 = (8 / kNV) > 2 ? (8 / kNV) : 2;
    static constexpr int kU = kU0 < kG ? kU0 : kG;          // entries per step per group
    static constexpr int kHD = H * D;
    static_assert(kRowBytes % 16 == 0, "row must be a whole number of 16-B vectors");
    static_assert(kHL >= 1 && kG % kHL == 0, "heads must tile the lane group");
    static_assert(kG % kU == 0 && kP * kU <= kWave, "index tiles must cover whole steps");
};

// ------------------------------------------------------------ element codecs

template <typename T> __device__ __forceinline__ void widen(const uint4& r, float* f);

template <> __device__ __forceinline__ void widen<float>(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x);
    f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z);
    f[3] = __uint_as_float(r.w);
}

// bf16 element 2k sits in the low half of dword k (little endian); widening
// places the 16 bits in the upper half of an fp32 word, which is exact.
template <> __device__ __forceinline__ void widen<bf16_tag>(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16);
    f[1] = __uint_as_float(r.x & 0xFFFF0000u);
    f[2] = __uint_as_float(r.y << 16);
    f[3] = __uint_as_float(r.y & 0xFFFF0000u);
    f[4] = __uint_as_float(r.z << 16);
    f[5] = __uint_as_float(r.z & 0xFFFF0000u);
    f[6] = __uint_as_float(r.w << 16);
    f[7] = __uint_as_float(r.w & 0xFFFF0000u);
}

// fp32 -> bf16 bits, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint32_t bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

template <typename T> __device__ __forceinline__ uint4 narrow(const float* f);

template <> __device__ __forceinline__ uint4 narrow<float>(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
}

template <> __device__ __forceinline__ uint4 narrow<bf16_tag>(const float* f) {
    return make_uint4(bf16_rne(f[0]) | (bf16_rne(f[1]) << 16), bf16_rne(f[2]) | (bf16_rne(f[3]) << 16),
                      bf16_rne(f[4]) | (bf16_rne(f[5]) << 16), bf16_rne(f[6]) | (bf16_rne(f[7]) << 16));
}

// ---------------------------------------------------------- cross-lane sums

template <int CTRL> __device__ __forceinline__ float dpp(float x) {
    return __builtin_amdgcn_update_dpp(0.0f, x, CTRL, 0xF, 0xF, false);
}

// Sum over aligned groups of HL lanes; every lane of a group ends with the
// same bits (each step adds a pair of values in both orders, a+b == b+a).
template <int HL> __device__ __forceinline__ float head_sum(float x) {
    if constexpr (HL >= 2) x += dpp<0xB1>(x);    // quad_perm [1,0,3,2]: lane ^ 1
    if constexpr (HL >= 4) x += dpp<0x4E>(x);    // quad_perm [2,3,0,1]: lane ^ 2
    if constexpr (HL >= 8) x += dpp<0x141>(x);   // row_half_mirror: other quad of 8
    if constexpr (HL >= 16) x += dpp<0x140>(x);  // row_mirror: other half of 16
    if constexpr (HL >= 32) x += __shfl_xor(x, 16);
    if constexpr (HL >= 64) x += __shfl_xor(x, 32);
    return x;
}

// Sum of an int over the 64 lanes of a wavefront, in every lane (the head_sum
// pattern: DPP within rows of 16 lanes, then two cross-row swaps).
__device__ __forceinline__ int wave_sum_i32(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false);   // lane ^ 2
    x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false);  // other quad of 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false);  // other half of 16
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    return x;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Streaming 16-byte accesses for data touched once per call (the row vector,
// the output row): non-temporal, so they do not displace the gathered K/V rows
// that other rows reuse from L2 and the Infinity Cache.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once(const char* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store_once(char* p, const uint4& x) {
    const u32x4_t v = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(p));
}

// bf16 pair arithmetic (gfx950 v_dot2c_f32_bf16, v_cvt_pk_bf16_f32, v_perm_b32).
// A dword holds bf16 element 2k in its low half and 2k+1 in its high half.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// c + a.lo * b.lo + a.hi * b.hi, products of bf16 pairs accumulated in fp32
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c,
                                           false);
}

// two fp32 values rounded to nearest even bf16, x in the low half
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
    bf16x2_t r;
    r[0] = (__bf16)x;
    r[1] = (__bf16)y;
    return __builtin_bit_cast(uint32_t, r);
}

// (a.lo, b.lo) and (a.hi, b.hi): the same element of two rows as one pair
__device__ __forceinline__ uint32_t pair_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pair_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Exponent-all-ones test of the eight bf16 values of v, folded into acc: a
// half's masked exponent plus 0x80 reaches bit 15 only when all eight exponent
// bits are set (Inf or NaN); the halves cannot carry into each other.  Any
// such value made bit 15 or 31 of acc set.
__device__ __forceinline__ uint32_t fold_nonfinite_bf16(uint32_t acc, const uint4& v) {
    acc |= (v.x & 0x7F807F80u) + 0x00800080u;
    acc |= (v.y & 0x7F807F80u) + 0x00800080u;
    acc |= (v.z & 0x7F807F80u) + 0x00800080u;
    acc |= (v.w & 0x7F807F80u) + 0x00800080u;
    return acc;
}

// Orders LDS traffic of one wavefront around a tile hand-off (the hardware
// executes a wave's LDS operations in order; this stops compiler reordering).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ln(sum_e exp(s_e)) from the running state in base-2 units: the sum is
// 2^m * l, so the logarithm is (m + log2 l) * ln 2; -inf for an empty row.
__device__ __forceinline__ float lse_of(float m, float l) {
    return l > 0.0f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

#include "gt_rows.hpp"

// ------------------------------------------------------------ per-lane state

// Entries per step of a lane group: 8, or 4 where short rows dominate the work
// of a step: for the GATv2 score, whose steps are arithmetic-heavy, and for rows
// narrow enough that a wave holds four or more of them.  A shorter step spends
// less on the padding of short rows and holds fewer registers.
template <typename T, int HS, int D, int KIND>
struct StepOf {
    static constexpr int kU = Geo<T, HS, D>::kU;
    static constexpr int value = ((KIND == KIND_GATV2 || Geo<T, HS, D>::kP >= 4) && kU >= 8) ? kU / 2 : kU;
};

// What the lanes of a wavefront share while it works on one slice of HS heads:
// base pointers at the slice's first element (of node 0), the stride between
// nodes and the score's constants.  KIND_GATV2: each lane also keeps its part of
// the attention vector, in two forms, since
// a * LeakyReLU(x) = a(1+s)/2 * x + a(1-s)/2 * |x| (exact for any slope s): an
// element then costs one add and two FMAs (|x| is a free operand modifier)
// instead of a compare, a select and a multiply more.
template <typename T, int HS, int D, int KIND>
struct RowState;

template <typename T, int HS, int D, int KIND>
struct AttnOp {
    using Gm = Geo<T, HS, D>;
    using State = RowState<T, HS, D, KIND>;
    static constexpr bool kGat = KIND == KIND_GATV2;
    static constexpr int kG = Gm::kG;
    static constexpr int kU = StepOf<T, HS, D, KIND>::value;
    // Light rows in the partition's step order pay where a wave holds four or
    // more rows (its groups then wait on their longest row), and for the GATv2
    // score, whose steps are arithmetic-heavy, already at two.
    static constexpr bool kSorted = Gm::kP >= 4 || (kGat && Gm::kP >= 2);
    static constexpr int kSlotFloats = HS * D;
    const char* Q;
    const char* K;
    const char* V;
    char* out;
    float* lse;      // at the slice's first head, or nullptr
    float* part_acc;  // [slot][HS * D]
    float2* part_ml;  // [slot][HS]: (running max in log2 units, sum)
    int row_shift;    // log2 of the bytes of one node row (all heads)
    int heads;
    float c;  // scale * log2(e); log2(e) for GATv2
    float a[kGat ? Gm::kEPV : 1];   // a(1+s)/2
    float a2[kGat ? Gm::kEPV : 1];  // a(1-s)/2

    __device__ __forceinline__ uint64_t offset(int32_t row, int lig) const {
        return ((uint64_t)(uint32_t)row << row_shift) + (uint32_t)lig * 16u;
    }
};

// One lane's share of a row's running state.  KIND_GT: q holds Q[i] and each
// entry loads K[j] (score) and V[j] (value).  KIND_GATV2: q holds L[i] and each
// entry loads only R[j], which gives both the score and the value.
template <typename T, int HS, int D, int KIND = KIND_GT>
struct RowState {
    using Op = AttnOp<T, HS, D, KIND>;
    using Gm = Geo<T, HS, D>;
    static_assert(Gm::kNV == 1, "a slice is one 16-byte vector per lane");
    static constexpr int kU = StepOf<T, HS, D, KIND>::value;
    static constexpr bool kGat = KIND == KIND_GATV2;
    // bf16 graph-transformer rows: scores are bf16 dot2 on the raw Q and K
    // pairs, accumulated in fp32 (the products of bf16 pairs are exact).  P*V
    // widens the value rows exactly and multiplies them with the fp32 weights.
    // KIND_GT_BF16W pairs two entries instead: their weights are rounded to
    // one bf16 pair and a dot2 multiplies it with the same element of the two
    // entries' value rows (paired with v_perm), accumulating in fp32; that
    // halves the vector instructions of P*V, and each rounded weight is off by
    // at most the bf16 unit roundoff 2^-8, which bounds the extra error of out
    // by 2^-8 * sum_e p_e |v_e| / sum_e p_e.  Either way the normaliser (and
    // lse) sums the fp32 weights.  (GATv2 widens its gathered rows for the
    // score anyway.)
    static constexpr bool kDot2 = std::is_same<T, bf16_tag>::value && !kGat;
    static constexpr bool kPairPV = kDot2 && KIND == KIND_GT_BF16W;
    static_assert(!kPairPV || kU % 2 == 0, "dot2 pairs entries");
    float q[Gm::kEPV];
    float acc[Gm::kEPV];
    float m;     // running max of log2-scaled scores for this lane's head
    float l;     // running sum of 2^(s - m)
    uint4 qraw;  // the row vector as bf16 pairs (dot2 form)

    __device__ __forceinline__ void reset() {
        m = -INFINITY;
        l = 0.0f;
#pragma unroll
        for (int e = 0; e < Gm::kEPV; ++e) acc[e] = 0.0f;
    }

    __device__ __forceinline__ void begin(const Op& op, int32_t row, int lig) {
        begin_loaded(load_once(op.Q + op.offset(row, lig)));
    }

    // begin() with this lane's 16 bytes of the row vector already in registers.
    __device__ __forceinline__ void begin_loaded(const uint4& r) {
        if constexpr (kDot2)
            qraw = r;
        else
            widen<T>(r, q);
    }

    // Loads of one step: the K and V rows (GATv2: the R rows) of U entries,
    // 16 bytes per lane each.
    struct Batch {
        uint4 k[kU];
        uint4 v[kGat ? 1 : kU];
    };

    __device__ __forceinline__ void issue(const Op& op, const int32_t (&j)[kU], int lig, Batch& bt) const {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t off = op.offset(j[u], lig);
            bt.k[u] = *reinterpret_cast<const uint4*>(op.K + off);
            if constexpr (!kGat) bt.v[u] = *reinterpret_cast<const uint4*>(op.V + off);
        }
    }

    // Value row of entry u (GATv2: the gathered R row).
    __device__ __forceinline__ static const uint4& value(const Batch& bt, int u) {
        if constexpr (kGat)
            return bt.k[u];
        else
            return bt.v[u];
    }

    // Score of entry u (log2 units, before masking).
    __device__ __forceinline__ float score(const Op& op, const Batch& bt, int u) const {
#pragma clang fp contract(off)
        float d = 0.0f;
        if constexpr (kDot2) {
            const uint4 kr = bt.k[u];
            d = dot2_bf16(qraw.x, kr.x, d);
            d = dot2_bf16(qraw.y, kr.y, d);
            d = dot2_bf16(qraw.z, kr.z, d);
            d = dot2_bf16(qraw.w, kr.w, d);
        } else {
            float kf[Gm::kEPV];
            widen<T>(bt.k[u], kf);
            if constexpr (kGat) {
#pragma unroll
                for (int e = 0; e < Gm::kEPV; ++e) {
                    const float x = q[e] + kf[e];
                    d = fmaf(op.a[e], x, d);
                    d = fmaf(op.a2[e], fabsf(x), d);
                }
            } else {
#pragma unroll
                for (int e = 0; e < Gm::kEPV; ++e) d = fmaf(q[e], kf[e], d);
            }
        }
        return head_sum<Gm::kHL>(d) * op.c;
    }

    // Online-softmax update with the U entries of a batch; entries u >= nvalid
    // are copies of valid indices and contribute nothing (score -inf, weight 0).
    // The maximal entry gets weight exactly 1 (also in bf16), and an entry of
    // weight 0 adds exactly 0, so a single-entry row returns its value exactly;
    // dot2 steps with an odd number of valid entries pair the last one with a
    // weight-0 copy.
    __device__ __forceinline__ void consume(const Op& op, const Batch& bt, const int32_t (&)[kU], int nvalid) {
        // No implicit contraction: fusing the score product into the later
        // subtraction of the running max would give the maximal entry a weight
        // of 2^(rounding error) instead of exactly 1.
#pragma clang fp contract(off)
        constexpr int U = kU;
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float d = score(op, bt, u);  // unconditional: the head sum is cross-lane
            s[u] = (u < nvalid) ? d : -INFINITY;
        }
        float mb = m;
#pragma unroll
        for (int u = 0; u < U; ++u) mb = fmaxf(mb, s[u]);
        const float corr = fast_exp2(m - mb);  // 0 on the first step (m = -inf)
        l *= corr;
#pragma unroll
        for (int e = 0; e < Gm::kEPV; ++e) acc[e] *= corr;
        if constexpr (kPairPV) {
#pragma unroll
            for (int u = 0; u < U; u += 2) {
                const float p0 = fast_exp2(s[u] - mb), p1 = fast_exp2(s[u + 1] - mb);
                l += p0;  // the normaliser (and so lse) from the fp32 weights
                l += p1;
                const uint32_t pp = pack_bf16(p0, p1);
                const uint4 v0 = value(bt, u), v1 = value(bt, u + 1);
                const uint32_t a0[4] = {v0.x, v0.y, v0.z, v0.w}, a1[4] = {v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    acc[2 * x] = dot2_bf16(pp, pair_lo(a0[x], a1[x]), acc[2 * x]);
                    acc[2 * x + 1] = dot2_bf16(pp, pair_hi(a0[x], a1[x]), acc[2 * x + 1]);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float pu = fast_exp2(s[u] - mb);
                l += pu;
                float vf[Gm::kEPV];
                widen<T>(value(bt, u), vf);
#pragma unroll
                for (int e = 0; e < Gm::kEPV; ++e) acc[e] = fmaf(pu, vf[e], acc[e]);
            }
        }
        m = mb;
    }

    __device__ __forceinline__ void step(const Op& op, const int32_t (&j)[kU], int nvalid, int lig) {
        Batch bt;
        issue(op, j, lig, bt);
        consume(op, bt, j, nvalid);
    }

    // Merge a state (mo, lo, ao) of other entries of the same row.
    __device__ __forceinline__ void merge(float mo, float lo, const float (&ao)[Gm::kEPV]) {
#pragma clang fp contract(off)
        const float mn = fmaxf(m, mo);
        const float ca = (m == mn) ? 1.0f : fast_exp2(m - mn);
        const float cb = (mo == mn) ? 1.0f : fast_exp2(mo - mn);
        l = l * ca + lo * cb;
#pragma unroll
        for (int e = 0; e < Gm::kEPV; ++e) acc[e] = acc[e] * ca + ao[e] * cb;
        m = mn;
    }

    // Merge the state held by the lane `off` positions away (the same vector in
    // another group of the wave).
    __device__ __forceinline__ void merge_xor(int off) {
        const float mo = __shfl_xor(m, off);
        const float lo = __shfl_xor(l, off);
        float ao[Gm::kEPV];
#pragma unroll
        for (int e = 0; e < Gm::kEPV; ++e) ao[e] = __shfl_xor(acc[e], off);
        merge(mo, lo, ao);
    }

    __device__ __forceinline__ void store_out(const Op& op, int32_t row, int lig) const {
        const float inv = l > 0.0f ? 1.0f / l : 0.0f;
        float o[Gm::kEPV];
#pragma unroll
        for (int e = 0; e < Gm::kEPV; ++e) o[e] = acc[e] * inv;
        store_once(op.out + op.offset(row, lig), narrow<T>(o));
        if (op.lse && lig % Gm::kHL == 0) op.lse[(int64_t)row * op.heads + lig / Gm::kHL] = lse_of(m, l);
    }

    __device__ __forceinline__ void store_partial(const Op& op, int32_t slot, int lig) const {
        float* dst = op.part_acc + (int64_t)slot * Gm::kHD + lig * Gm::kEPV;
#pragma unroll
        for (int e = 0; e < Gm::kEPV; e += 4)
            *reinterpret_cast<float4*>(dst + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        if (lig % Gm::kHL == 0) op.part_ml[(int64_t)slot * HS + lig / Gm::kHL] = make_float2(m, l);
    }

    __device__ __forceinline__ void load_partial(const Op& op, int32_t slot, int lig, float& mo, float& lo,
                                                 float (&ao)[Gm::kEPV]) const {
        const float* src = op.part_acc + (int64_t)slot * Gm::kHD + lig * Gm::kEPV;
#pragma unroll
        for (int e = 0; e < Gm::kEPV; e += 4) {
            const float4 x = *reinterpret_cast<const float4*>(src + e);
            ao[e] = x.x;
            ao[e + 1] = x.y;
            ao[e + 2] = x.z;
            ao[e + 3] = x.w;
        }
        const float2 ml = op.part_ml[(int64_t)slot * HS + lig / Gm::kHL];
        mo = ml.x;
        lo = ml.y;
    }
};

struct AttnParams {
    RowWork w;
    const char* Q;
    const char* K;
    const char* V;
    char* out;
    float* lse;  // [N][H] natural-log logsumexp of the scaled scores, or nullptr
    const float* att;  // GATv2 attention vector [H][D]
    float slope;       // GATv2 LeakyReLU negative slope
    float c;           // scale * log2(e); log2(e) for GATv2
    int32_t row_shift;
    int32_t heads;
    int32_t slice0;    // slice of blockIdx.y == 0
    float* part_acc;   // [slice of this launch][slot][HS * D]
    float2* part_ml;   // [slice of this launch][slot][HS]
};

template <typename T, int HS, int D, int KIND>
__device__ __forceinline__ AttnOp<T, HS, D, KIND> slice_op(const AttnParams& p) {
    using Op = AttnOp<T, HS, D, KIND>;
    Op op;
    const int head = (p.slice0 + (int)blockIdx.y) * HS;
    const int64_t at = (int64_t)head * D * Elt<T>::kBytes;
    const int64_t slot = (int64_t)blockIdx.y * p.w.cap_slots;
    op.Q = p.Q + at;
    op.K = p.K + at;
    op.V = p.V + at;
    op.out = p.out + at;
    op.lse = p.lse ? p.lse + head : nullptr;
    op.part_acc = p.part_acc + slot * Op::kSlotFloats;
    op.part_ml = p.part_ml + slot * HS;
    op.row_shift = p.row_shift;
    op.heads = p.heads;
    op.c = p.c;
    if constexpr (Op::kGat) {
        // the attention vector is [H][D] fp32 in the row's element order
        const float* av = p.att + head * D + (threadIdx.x % Op::kG) * Op::Gm::kEPV;
        const float hs = 0.5f * p.slope;
#pragma unroll
        for (int e = 0; e < Op::Gm::kEPV; e += 4) {
            const float4 x4 = *reinterpret_cast<const float4*>(av + e);
            const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                op.a[e + t] = fmaf(hs, x[t], 0.5f * x[t]);
                op.a2[e + t] = fmaf(-hs, x[t], 0.5f * x[t]);
            }
        }
    }
    return op;
}

// Attention kernel: blockIdx.y is the slice (launched one after another), the
// blocks of a slice share its rows as row_loop says.
template <typename T, int HS, int D, int KIND>
__global__ void __launch_bounds__(kBlock) gt_attn_kernel(AttnParams p) {
    using Op = AttnOp<T, HS, D, KIND>;
    __shared__ __attribute__((aligned(16))) int32_t tiles[kWavesPerBlock][kWave / Op::kG * TileOf<Op::kG>::kEntries];
    const Op op = slice_op<T, HS, D, KIND>(p);
    row_loop(p.w, op, tiles[threadIdx.x / kWave]);
}

// Merge of the partial states of each cut row: one wavefront per row and slice.
// Lane group g merges pieces g, g + P, ..., kMergePieces of them in flight at a
// time, and the groups are merged across lanes: a fixed order, so the results
// are bitwise reproducible.
constexpr int kMergePieces = 4;

template <typename T, int HS, int D>
__global__ void __launch_bounds__(kBlock) gt_merge_kernel(AttnParams p) {
    using Op = AttnOp<T, HS, D, KIND_GT>;
    constexpr int G = Op::kG, P = kWave / G, EPV = Op::Gm::kEPV;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t g = lane / G;
    const int lig = lane % G;
    if (ROWS_CNT(p.w.counters, ROWS_PIECES) == 0) return;  // no long rows
    const CutRows cut(p.w, lane);
    const uint32_t n = cut.count(), waves = gridDim.x * kWavesPerBlock;
    const Op op = slice_op<T, HS, D, KIND_GT>(p);
    for (uint32_t i = blockIdx.x * kWavesPerBlock + wv; i < n; i += waves) {
        uint32_t slot, nq;
        const int32_t row = cut.row(p.w, i, lane, slot, nq);
        typename Op::State st;
        st.reset();
        for (uint32_t q0 = 0; q0 < nq; q0 += P * kMergePieces) {
            float mo[kMergePieces], lo[kMergePieces], ao[kMergePieces][EPV];
            // (a group without a piece reads the row's last and leaves it out)
#pragma unroll
            for (int u = 0; u < kMergePieces; ++u) {
                const uint32_t q = q0 + u * P + g;
                st.load_partial(op, (int32_t)(slot + (q < nq ? q : nq - 1)), lig, mo[u], lo[u], ao[u]);
            }
#pragma unroll
            for (int u = 0; u < kMergePieces; ++u) {
                if (q0 + u * P + g >= nq) mo[u] = -INFINITY, lo[u] = 0.0f;
#pragma unroll
                for (int e = 0; e < EPV; ++e) ao[u][e] = q0 + u * P + g < nq ? ao[u][e] : 0.0f;
                st.merge(mo[u], lo[u], ao[u]);
            }
        }
#pragma unroll
        for (int off = G; off < kWave; off <<= 1) st.merge_xor(off);
        if (g == 0) st.store_out(op, row, lig);
    }
}

// ------------------------------------------------------- dense-tile path
//
// Locally dense windows (Section 3.3 and Appendix D.3 of the paper pack local
// neighbourhoods into tiles for matrix cores; this is a gfx950 design of the
// same idea, not the paper's 16x8 TCB format).  Rows are grouped in aligned
// windows of 64; the window's own 64 ids are its tile columns.  The partition
// kernel flags the windows whose rows of at most tile_max entries it estimates
// to be dense (a sample of one entry in every 8th of them); this kernel takes
// these rows of a flagged window ("light rows" here; one workgroup per window),
// the row kernel every other row:
//   1. stage the window's rowptr, its K rows and its V rows (transposed) in
//      LDS with independent loads, and each light row's entries in registers;
//   2. per light row, a 64-bit mask of its in-window entries (a row with a
//      repeated in-window entry cannot be a mask and does not use the tile);
//   3. if the window holds at least `min_entries` masked entries and its V
//      tile only finite values, per head and per 16-row strip (one wave each):
//        S^T = K_w Q_strip^T  (bf16 MFMA 16x16x32, fp32 accumulate),
//      masked row-wise softmax statistics, and acc = P V_w (MFMA with P as
//      the sum of two bf16 terms, so the weights keep 16 significant bits;
//      with the bf16-weight option, one MFMA on P rounded to bf16); the
//      normaliser and lse sum the fp32 weights;
//   4. every light row then streams its remaining entries (all of them for a
//      row without a tile) with the CSR online-softmax step, continuing from
//      the tile's (m, l, acc), and writes its output.
//
// MFMA operand layout of v_mfma_f32_16x16x32_bf16 (64 lanes, l = lane):
//   A (16x32): lane l holds A[l%16][8*(l/16) + j], j = 0..7
//   B (32x16): lane l holds B[8*(l/16) + j][l%16]
//   C (16x16): lane l holds C[4*(l/16) + i][l%16], i = 0..3

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kWin = 64;          // window rows = tile columns
constexpr int kNoTile = -(1 << 28);  // a wave's window count that rules the tile out
// Padded row of the transposed V tile, in bf16 elements: 34 dwords, so that
// the 16 rows one P*V operand load reads (8 bytes per lane) start 2 banks
// apart and cover all 32 banks once (a 36-dword row put rows n and n + 8 on
// the same banks).
constexpr int kVtStride = 68;

struct TileParams {
    const int64_t* rowptr;
    const int32_t* colidx;
    const char* Q;
    const char* K;
    const char* V;
    char* out;
    float* lse;
    int64_t N;
    float c;  // scale * log2(e)
    int32_t tile_max;  // <= kWinMaxDeg
    int32_t min_entries;
    const uint8_t* win_flags;  // [ceil(N / 64)]: 1 for the dense windows the partition found
    const int32_t* counters;   // ROWS_WIN: any window dense (byte 0) / not dense (byte 1)
};

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

template <int H, int D>
struct TileLds {
    static constexpr int HD = H * D;
    static constexpr int KST = HD + 8;  // padded K row (bf16 elements)
    int64_t rp[kWin + 1];
    uint64_t masks[kWin];
    int32_t wave_cnt[kWavesPerBlock];
    // The K and V tiles are dead once the products are done; the strip results
    // and the index tiles of the remaining-entry stream then reuse their space.
    union alignas(16) {
        struct {
            uint16_t k[kWin][KST];
            uint16_t vt[HD][kVtStride];
        } kv;
        struct {
            float acc[kWavesPerBlock][16][HD + 4];  // padded: the MFMA-layout writes hit distinct banks
            int32_t ctile[kWavesPerBlock][kWave / (H * D / 8) * kWinMaxDeg];  // per lane group: one row's entries
        } rest;
    } big;
    float2 ml[kWavesPerBlock][16][H];
};

// Four workgroups per CU fit the LDS of a window (about 40 KB) when H*D <= 128
// and H <= 2; those shapes are held to 128 VGPRs so that registers allow it too.
// The stream stage of the tile kernel takes the row vectors of its rows from
// the strip's MFMA operand registers by cross-lane moves instead of reading Q
// a second time (on the SBM workload: 268 MB less fetched, about 10 us per
// call); for the 1x128 fp32-weight shape that holds 16 more registers across
// the products and spills, so it reads Q again.
template <int H, int D, int KIND>
struct QFromOperands {
    static constexpr bool value = !(H == 1 && D == 128 && KIND == KIND_GT);
};

template <int H, int D>
struct TileWaves {
    static constexpr int value = H <= 2 ? 4 : 1;
};

template <int H, int D, int KIND>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(TileWaves<H, D>::value)))
gt_tile_kernel(TileParams p) {
    using Gm = Geo<bf16_tag, H, D>;
    using L = TileLds<H, D>;
    using RS = RowState<bf16_tag, H, D, KIND>;  // (all heads: these rows are at most 256 bytes)
    constexpr int HD = H * D;
    constexpr int G = Gm::kG, P = Gm::kP, U = RS::kU;
    // fp32 weights (KIND_GT): P = hi + lo as two bf16 terms, two P*V
    // products, |P - hi - lo| <= 2^-17 P; KIND_GT_BF16W: P rounded to bf16
    constexpr bool kSplitP = KIND == KIND_GT;
    static_assert(HD <= 128 && D % 32 == 0, "tile path shapes");
    __shared__ __attribute__((aligned(16))) L lds;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int g16 = lane >> 4, n16 = lane & 15;  // MFMA lane coordinates
    // Workgroup b takes window b if the partition flagged it dense and returns
    // at once otherwise.  The word of window flags (one word every workgroup
    // reads, so a cached one) is loaded first: with no dense window, the
    // workgroup ends there; with no sparse one, the window's own flag is not
    // needed; otherwise it is read after the row-bound loads are issued.  (A
    // persistent loop over a list of the dense windows measured slower: it
    // raised the kernel's register pressure past its 128-VGPR budget and
    // spilled; a list also needs its entry before any other load.)
    const int64_t r0 = (int64_t)blockIdx.x * kWin;
    const int64_t wend = r0 + kWin;
    const int32_t win_state = ROWS_CNT(p.counters, ROWS_WIN);
    if ((win_state & 0xFF) == 0) return;
    const bool all_dense = (win_state & 0xFF00) == 0;

    // bounds of this lane's row in the mask stage (4 lanes per row), loaded
    // first so that its entries can be requested right after the staging loads
    const int srow = lane >> 2, sub = lane & 3;
    const int wrow = 16 * wv + srow;  // row within the window
    const int64_t r = r0 + wrow;
    // (rows past the end read rowptr[N] twice: an empty row.  The loads of
    // this stage are unconditional, with clamped addresses, so that the
    // compiler can wait for the row bounds alone while the later staging loads
    // are still in flight.)
    const int64_t mb = p.rowptr[r < p.N ? r : p.N];
    const int64_t me = p.rowptr[r + 1 < p.N ? r + 1 : p.N];
    if (!all_dense && !p.win_flags[blockIdx.x]) return;

    // ---- 1. staging.  Every load of the stage is issued before any LDS write,
    // with compile-time trip counts: the window's rowptr entries, its K and V
    // pieces and this lane's strip row of Q go out together, then the entries
    // of the mask stage (which wait only for the row bounds above), and only
    // then do the LDS writes wait for their data.  So staging a window costs
    // about two memory latencies (row bounds, then entries), not one per loop
    // trip.
    constexpr int kKPieces = kWin * (HD / 8);        // 16-byte pieces of the K tile
    constexpr int kVPieces = (kWin / 2) * (HD / 8);  // pieces of the row pairs of the V tile
    constexpr int kKIt = (kKPieces + kBlock - 1) / kBlock;
    constexpr int kVIt = (kVPieces + kBlock - 1) / kBlock;
    static_assert(kKPieces % kBlock == 0, "the K tile is a whole number of workgroup loads");
    // Rows past the end read the last row instead: their K columns and Q rows
    // are masked out of every score, and their V columns are zeroed when the
    // tile is written (a weight of 0 must not meet a non-finite value).  No
    // loaded register is overwritten before it arrives, which would make the
    // load wait at once.
    const int64_t last = p.N - 1;
    const int64_t rpv = p.rowptr[(r0 + tid < p.N) ? r0 + tid : p.N];
    uint4 kx[kKIt];
#pragma unroll
    for (int it = 0; it < kKIt; ++it) {
        // K rows as they are: 16 bytes of one row per lane
        const int v = tid + it * kBlock, cc = v % kWin, e0 = (v / kWin) * 8;
        const int64_t rk = r0 + cc;
        kx[it] = *reinterpret_cast<const uint4*>(p.K + ((rk < p.N ? rk : last) * HD + e0) * 2);
    }
    uint4 va[kVIt], vb[kVIt];
#pragma unroll
    for (int it = 0; it < kVIt; ++it) {
        // V transposed: a lane takes 8 elements of two consecutive rows (the
        // 1x32 shape has fewer pieces than lanes: the rest load piece 0)
        const int v0 = tid + it * kBlock;
        const int v = (kVPieces % kBlock == 0 || v0 < kVPieces) ? v0 : 0;
        const int pc = v % (kWin / 2), e0 = (v / (kWin / 2)) * 8;
        const int64_t ra = r0 + 2 * pc;
        va[it] = *reinterpret_cast<const uint4*>(p.V + ((ra < p.N ? ra : last) * HD + e0) * 2);
        vb[it] = *reinterpret_cast<const uint4*>(p.V + ((ra + 1 < p.N ? ra + 1 : last) * HD + e0) * 2);
    }
    // this lane's strip row of Q (all heads), as MFMA B operands
    const int64_t qrow = r0 + 16 * wv + n16;
    uint4 qreg[HD / 32];
#pragma unroll
    for (int t = 0; t < HD / 32; ++t) {
        qreg[t] = *reinterpret_cast<const uint4*>(p.Q + ((qrow < p.N ? qrow : last) * HD + 32 * t + 8 * g16) * 2);
    }

    // ---- 2. in-window masks: 4 lanes per row, 16 rows per wave.  The entries
    // come straight from colidx (one batch of independent loads, behind the
    // staging loads); the remaining-entry stream reads them again later, so
    // the window needs no LDS copy of its entries.
    const bool light = r < p.N && (me - mb) <= p.tile_max;
    constexpr int kMaskPer = kWinMaxDeg / 4;  // entries per lane (tile_max <= kWinMaxDeg)
    int32_t ent[kMaskPer] = {};
    if (light && me > mb) {
#pragma unroll
        for (int k = 0; k < kMaskPer; ++k) {
            const int64_t pos = mb + sub + 4 * k;
            ent[k] = p.colidx[pos < me ? pos : me - 1];
        }
    }
    // the staged tiles to LDS (read after the barrier below)
    if (tid <= kWin) lds.rp[tid] = rpv;
#pragma unroll
    for (int it = 0; it < kKIt; ++it) {
        const int v = tid + it * kBlock, cc = v % kWin, e0 = (v / kWin) * 8;
        *reinterpret_cast<uint4*>(&lds.big.kv.k[cc][e0]) = r0 + cc < p.N ? kx[it] : make_uint4(0, 0, 0, 0);
    }
    // Inf or NaN anywhere in the value tile: P*V sums over every column of
    // the window, and a weight of 0 times such a value is NaN, so one row's
    // value would leak into rows that do not reference it.  Such a window is
    // streamed instead (below).
    uint32_t vbits = 0;
#pragma unroll
    for (int it = 0; it < kVIt; ++it) {
        // each element pair as one dword, so the 32 lanes of a row pair write 32
        // consecutive dwords of one vt row
        const int v = tid + it * kBlock, pc = v % (kWin / 2), e0 = (v / (kWin / 2)) * 8;
        if (kVPieces % kBlock == 0 || v < kVPieces) {
            const int64_t ra = r0 + 2 * pc;
            const uint4 a = ra < p.N ? va[it] : make_uint4(0, 0, 0, 0);
            const uint4 b = ra + 1 < p.N ? vb[it] : make_uint4(0, 0, 0, 0);
            vbits = fold_nonfinite_bf16(fold_nonfinite_bf16(vbits, a), b);
            const uint32_t wa[4] = {a.x, a.y, a.z, a.w}, wb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                *reinterpret_cast<uint32_t*>(&lds.big.kv.vt[e0 + 2 * q][2 * pc]) = pair_lo(wa[q], wb[q]);
                *reinterpret_cast<uint32_t*>(&lds.big.kv.vt[e0 + 2 * q + 1][2 * pc]) = pair_hi(wa[q], wb[q]);
            }
        }
    }
    uint64_t mk = 0;
    int cnt = 0;
    if (light) {
#pragma unroll
        for (int k = 0; k < kMaskPer; ++k) {
            const int64_t j = ent[k];
            if (mb + sub + 4 * k < me && j >= r0 && j < wend) {
                mk |= 1ull << (j - r0);
                ++cnt;
            }
        }
    }
    mk |= shfl_xor_u64(mk, 1);
    mk |= shfl_xor_u64(mk, 2);
    cnt += __shfl_xor(cnt, 1);
    cnt += __shfl_xor(cnt, 2);
    const bool tile_ok = light && __popcll(mk) == cnt;  // no repeated in-window entry
    if (sub == 0) lds.masks[wrow] = tile_ok ? mk : 0;
    int wc = (sub == 0 && tile_ok) ? cnt : 0;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) wc += __shfl_xor(wc, o);
    // a wave that staged a non-finite value puts the window's count far below
    // any threshold
    const bool v_nonfinite = __ballot((vbits & 0x80008000u) != 0) != 0;
    if (lane == 0) lds.wave_cnt[wv] = v_nonfinite ? kNoTile : wc;
    const uint64_t ok_bits = __ballot(sub == 0 && tile_ok);     // bit 4*sr: strip row sr
    const uint64_t light_bits = __ballot(sub == 0 && light);
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) total += lds.wave_cnt[w];
    const bool dense = total >= p.min_entries;  // uniform over the workgroup

    // ---- 3. tiles
    float mx[H], lsum[H];
    f32x4_t oacc[H][D / 16];
    if (dense) {
        const uint64_t rmask = lds.masks[16 * wv + n16];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            f32x4_t sacc[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) sacc[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks) {
                const bf16x8_t bq = __builtin_bit_cast(bf16x8_t, qreg[(h * D) / 32 + ks]);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const bf16x8_t ak = __builtin_bit_cast(
                        bf16x8_t, *reinterpret_cast<const uint4*>(&lds.big.kv.k[16 * mt + n16][h * D + 32 * ks + 8 * g16]));
                    sacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, bq, sacc[mt], 0, 0, 0);
                }
            }
            // lane holds S[strip row n16][window column 16*mt + 4*g16 + i] = sacc[mt][i]
            float pr[16];
            float m = -INFINITY;
            {
#pragma clang fp contract(off)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int cc = 16 * mt + 4 * g16 + i;
                        const float sv = ((rmask >> cc) & 1ull) ? sacc[mt][i] * p.c : -INFINITY;
                        pr[4 * mt + i] = sv;
                        m = fmaxf(m, sv);
                    }
                m = fmaxf(m, __shfl_xor(m, 16));
                m = fmaxf(m, __shfl_xor(m, 32));
            }
            uint32_t pb[16], pl[kSplitP ? 16 : 1];
            float ls = 0.0f;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const float pv = (m == -INFINITY) ? 0.0f : fast_exp2(pr[t] - m);
                pb[t] = bf16_rne(pv);
                // pv - hi is exact in fp32; its bf16 rounding is the low term
                if constexpr (kSplitP) pl[t] = bf16_rne(pv - __uint_as_float(pb[t] << 16));
                ls += pv;  // the normaliser (and lse) from the fp32 weights
            }
            ls += __shfl_xor(ls, 16);
            ls += __shfl_xor(ls, 32);
            mx[h] = m;
            lsum[h] = ls;
            // acc = P V_w; K order of step ks, slot 8*g16 + j: window column
            // 16*(2ks + j/4) + 4*g16 + j%4, i.e. exactly the weights this lane holds
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) oacc[h][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const uint4 au = make_uint4(pb[8 * ks + 0] | (pb[8 * ks + 1] << 16), pb[8 * ks + 2] | (pb[8 * ks + 3] << 16),
                                            pb[8 * ks + 4] | (pb[8 * ks + 5] << 16), pb[8 * ks + 6] | (pb[8 * ks + 7] << 16));
                const bf16x8_t ap = __builtin_bit_cast(bf16x8_t, au);
                bf16x8_t apl = ap;
                if constexpr (kSplitP)
                    apl = __builtin_bit_cast(
                        bf16x8_t, make_uint4(pl[8 * ks + 0] | (pl[8 * ks + 1] << 16), pl[8 * ks + 2] | (pl[8 * ks + 3] << 16),
                                             pl[8 * ks + 4] | (pl[8 * ks + 5] << 16), pl[8 * ks + 6] | (pl[8 * ks + 7] << 16)));
#pragma unroll
                for (int dt = 0; dt < D / 16; ++dt) {
                    const int e = h * D + 16 * dt + n16;
                    const uint2 lo = *reinterpret_cast<const uint2*>(&lds.big.kv.vt[e][32 * ks + 4 * g16]);
                    const uint2 hi = *reinterpret_cast<const uint2*>(&lds.big.kv.vt[e][32 * ks + 16 + 4 * g16]);
                    const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
                    oacc[h][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap, bv, oacc[h][dt], 0, 0, 0);
                    if constexpr (kSplitP)
                        oacc[h][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(apl, bv, oacc[h][dt], 0, 0, 0);
                }
            }
        }
    }
    __syncthreads();  // K / V tiles no longer read: their LDS now holds the strip results
    if (dense) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) lds.big.rest.acc[wv][4 * g16 + i][h * D + 16 * dt + n16] = oacc[h][dt][i];
            if (g16 == 0) lds.ml[wv][n16][h] = make_float2(mx[h], lsum[h]);
        }
    }
    wave_lds_fence();

    // ---- 4. remaining entries of each light row, CSR online softmax, output.
    // Each lane group takes rows g, g + P, ... of the wave's strip; the entries
    // of a group's next row are requested before the current row's gathers.
    AttnOp<bf16_tag, H, D, KIND> op;
    op.Q = p.Q;
    op.K = p.K;
    op.V = p.V;
    op.out = p.out;
    op.lse = p.lse;
    op.row_shift = __builtin_ctz(HD * 2);
    op.heads = H;
    op.c = p.c;
    const int g = lane / G, lig = lane % G;
    int32_t* gtile = lds.big.rest.ctile[wv] + g * kWinMaxDeg;
    constexpr int kRowPer = (kWinMaxDeg + G - 1) / G;  // a light row: at most kWinMaxDeg entries
    constexpr int kPasses = 16 / P;
    // The row vector of the group's row of a pass, from the strip's MFMA
    // operands (lane 16*g16 + n16 of qreg[t] holds elements 32t + 8*g16 .. + 7
    // of strip row n16) by cross-lane moves, rather than a second read from
    // memory.  Taken at the top of each pass, where every lane is active (a
    // move reads zero from an inactive lane), with selects rather than
    // branches.
    constexpr bool kQRegs = QFromOperands<H, D, KIND>::value;
    auto row_vector = [&](int pass) -> uint4 {
        const int e0 = 8 * lig;  // first element of this lane's piece
        const int src = 16 * ((e0 % 32) / 8) + pass * P + g, tsel = e0 / 32;
        uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < HD / 32; ++t) {
            const uint32_t x[4] = {(uint32_t)__shfl((int)qreg[t].x, src), (uint32_t)__shfl((int)qreg[t].y, src),
                                   (uint32_t)__shfl((int)qreg[t].z, src), (uint32_t)__shfl((int)qreg[t].w, src)};
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = tsel == t ? x[c] : v[c];
        }
        return make_uint4(v[0], v[1], v[2], v[3]);
    };
    auto load_entries = [&](int pass, int32_t (&e)[kRowPer]) {
        const int sr = pass * P + g, wr = 16 * wv + sr;
        const int64_t eb = lds.rp[wr], ee = lds.rp[wr + 1];
        if (((light_bits >> (4 * sr)) & 1ull) && ee > eb) {
#pragma unroll
            for (int k = 0; k < kRowPer; ++k) {
                const int64_t pos = eb + lig + k * G;
                e[k] = p.colidx[pos < ee ? pos : ee - 1];
            }
        }
    };
    int32_t nxt[kRowPer] = {};
    load_entries(0, nxt);
    for (int pass = 0; pass < kPasses; ++pass) {
        int32_t re[kRowPer];
#pragma unroll
        for (int k = 0; k < kRowPer; ++k) re[k] = nxt[k];
        if (pass + 1 < kPasses) load_entries(pass + 1, nxt);
        uint4 qp = make_uint4(0, 0, 0, 0);
        if constexpr (kQRegs) qp = row_vector(pass);
        const int sr = pass * P + g;
        if (!((light_bits >> (4 * sr)) & 1ull)) continue;
        const bool use_tile = dense && ((ok_bits >> (4 * sr)) & 1ull);
        const int wr = 16 * wv + sr;
        const int64_t row = r0 + wr;
        RS st;
        st.reset();
        if constexpr (kQRegs)
            st.begin_loaded(qp);
        else
            st.begin(op, (int32_t)row, lig);
        if (use_tile) {
            const float2 ml = lds.ml[wv][sr][lig / Gm::kHL];
            st.m = ml.x;
            st.l = ml.y;
#pragma unroll
            for (int q = 0; q < Gm::kEPV; ++q) st.acc[q] = lds.big.rest.acc[wv][sr][lig * Gm::kEPV + q];
        }
        // the row's remaining entries (outside the tile) into gtile
        const int64_t eb = lds.rp[wr], ee = lds.rp[wr + 1];
        int n_take = 0;
#pragma unroll
        for (int k = 0; k < kRowPer; ++k) {
            const bool in = eb + lig + k * G < ee;
            const int32_t idx = re[k];
            const bool take = in && !(use_tile && idx >= r0 && idx < wend);
            const uint64_t bal = __ballot(take);
            const uint32_t gbits = (uint32_t)((bal >> (g * G)) & ((1ull << G) - 1));
            if (take) gtile[n_take + __popc(gbits & ((1u << lig) - 1u))] = idx;
            n_take += __popc(gbits);
        }
        wave_lds_fence();
        for (int t = 0; t < n_take; t += U) {
            const int nvalid = n_take - t < U ? n_take - t : U;
            int32_t j[U];
#pragma unroll
            for (int u = 0; u < U; ++u) j[u] = gtile[(t + u < n_take) ? t + u : n_take - 1];
            st.step(op, j, nvalid, lig);
        }
        wave_lds_fence();
        st.store_out(op, (int32_t)row, lig);
    }
}

// Clears n ints (the work-list counters at the start of a call).  A kernel
// rather than hipMemsetAsync, so that a call recorded into a HIP graph holds
// no memset node.
__global__ void __launch_bounds__(kBlock) gt_clear_kernel(int32_t* __restrict__ p, int32_t n) {
    for (int32_t i = threadIdx.x; i < n; i += kBlock) p[i] = 0;
}

__global__ void __launch_bounds__(kBlock) gt_csr_check_kernel(const int64_t* rowptr, const int32_t* colidx,
                                                            int64_t N, int64_t E, int32_t* bad) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (tid == 0 && (rowptr[0] != 0 || rowptr[N] != E)) atomicOr(bad, 1);
    for (int64_t i = tid; i < N; i += stride)
        if (rowptr[i + 1] < rowptr[i]) atomicOr(bad, 1);
    for (int64_t k = tid; k < E; k += stride)
        if (colidx[k] < 0 || colidx[k] >= N) atomicOr(bad, 1);
}

// ----------------------------------------------------------------- host side

thread_local std::string t_last_error;

gt_status fail(gt_status s, const std::string& msg) {
    t_last_error = msg;
    return s;
}

gt_status hip_fail(hipError_t e, const char* what) {
    return fail(GT_ERROR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

struct Profiler {
    std::mutex mu;
    bool on = false;
    std::vector<std::array<hipEvent_t, 4>> pending;
};
Profiler& profiler() {
    static Profiler* p = new Profiler();
    return *p;
}

// The four phase events of one profiled call (when profiling is enabled):
// created by start(), recorded by mark(), handed to the profiler by commit().
// A call that fails before commit() destroys them.
struct PhaseEvents {
    std::array<hipEvent_t, 4> ev{};
    bool on = false;
    hipError_t start(hipStream_t stream) {
        Profiler& pr = profiler();
        {
            std::lock_guard<std::mutex> lk(pr.mu);
            on = pr.on;
        }
        if (!on) return hipSuccess;
        for (auto& e : ev) {
            const hipError_t he = hipEventCreate(&e);
            if (he != hipSuccess) return he;
        }
        return hipEventRecord(ev[0], stream);
    }
    void mark(int k, hipStream_t stream) {
        if (on) (void)hipEventRecord(ev[k], stream);
    }
    void commit(hipStream_t stream) {
        if (!on) return;
        (void)hipEventRecord(ev[3], stream);
        Profiler& pr = profiler();
        std::lock_guard<std::mutex> lk(pr.mu);
        pr.pending.push_back(ev);
        on = false;
    }
    ~PhaseEvents() {
        if (on)
            for (auto e : ev)
                if (e) (void)hipEventDestroy(e);
    }
};

// Workspace.  Every call takes a workspace block (row lists, partial
// states of split rows, work-list counters) for its own use and hands it back
// once its kernels are enqueued; the block is then tagged with an event
// recorded on the call's stream after those kernels.  A later call, on any
// stream, takes a free block only if its event has completed, or if it was
// last used on the same stream, and then with a device-side wait on the event
// (hipStreamWaitEvent: stream order already implies it, and it keeps a
// recycled stream handle safe); the host never waits.  Otherwise the call
// gets a new block from the library's memory pool of the device
// (hipMallocFromPoolAsync on its stream).  Blocks are not tied to streams or
// pointers, and free blocks beyond kCacheBytes per device go back to the pool
// (stream-ordered after their last use); gt_workspace_release() returns every
// free block and trims the pools.  (Freeing each call's block with
// hipFreeAsync made the host wait in every call for the previous call's
// kernels, about 485 us per call behind a 0.5 ms kernel, so the host could
// never run ahead of the device.)  While the call's stream is being captured
// into a graph, the block is allocated and freed stream-ordered instead (both
// become graph nodes), since events recorded during a capture cannot be
// queried.
constexpr int kMaxDevices = 64;
constexpr uint64_t kPoolKeepBytes = uint64_t(256) << 20;
// free blocks kept per device: two large calls' at 256 MiB each (four streams with
// such calls: the host then waits in calls for blocks to come back, device time is
// the same; a single 357 MiB block given back after each backward of 9.2 ms and
// allocated again cost 5 %)
constexpr size_t kCacheBytes = size_t(512) << 20;
constexpr size_t kBlockGranule = size_t(1) << 20;

struct DevicePools {
    std::once_flag once[kMaxDevices];
    hipMemPool_t pool[kMaxDevices] = {};
    hipError_t err[kMaxDevices] = {};
    std::atomic<bool> ready[kMaxDevices] = {};  // pool[dev] / err[dev] are set
};
DevicePools& device_pools() {
    static DevicePools* p = new DevicePools();
    return *p;
}

hipError_t pool_of(int dev, hipMemPool_t* out) {
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    DevicePools& dp = device_pools();
    std::call_once(dp.once[dev], [&] {
        hipMemPoolProps props;
        std::memset(&props, 0, sizeof props);
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        hipMemPool_t pool = nullptr;
        hipError_t e = hipMemPoolCreate(&pool, &props);
        if (e == hipSuccess) {
            uint64_t keep = kPoolKeepBytes;
            e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
        }
        dp.pool[dev] = pool;
        dp.err[dev] = e;
        dp.ready[dev].store(true, std::memory_order_release);
    });
    *out = dp.pool[dev];
    return dp.err[dev];
}

struct WsBlock {
    char* ptr = nullptr;
    size_t bytes = 0;
    hipEvent_t ev = nullptr;       // recorded after the last user's kernels
    hipStream_t last = nullptr;    // the last user's stream
    // Forward calls keep two work-list counter sets at the start of the
    // block and use set gen % 2; each call's partition zeroes the other set
    // for the next call.  primed: set gen % 2 is zero (the last user was a
    // forward call whose partition was enqueued), so no clear is needed.
    uint32_t gen = 0;
    bool primed = false;
};

// Free blocks of one device, and the bytes of blocks that calls hold.
struct BlockCache {
    std::mutex mu;
    std::vector<WsBlock> free_blocks;
    size_t free_bytes = 0;
    size_t taken_bytes = 0;
};
BlockCache& block_cache(int dev) {
    static BlockCache* c = new BlockCache[kMaxDevices];
    return c[dev];
}

// Returns a block to the pool after its last use: ordered after the block's
// event on `stream` (the stream of the call that lets it go).
void free_block(const WsBlock& b, hipStream_t stream) {
    if (b.ev) {
        if (hipEventQuery(b.ev) != hipSuccess) (void)hipStreamWaitEvent(stream, b.ev, 0);
        (void)hipGetLastError();
        (void)hipEventDestroy(b.ev);
    }
    (void)hipFreeAsync(b.ptr, stream);
}

// One call's workspace; handed back (cached) or freed stream-ordered after
// the call's kernels when it goes out of scope (also on an error return
// after some launches).
struct CallWorkspace {
    enum Kind { NONE, CACHED, STREAM_ORDERED, SCRATCH };
    char* ptr = nullptr;
    hipStream_t stream = nullptr;
    int dev = -1;
    Kind kind = NONE;
    WsBlock block;
    bool keep_primed = false;  // set by a forward call once its partition is enqueued
    CallWorkspace() = default;
    CallWorkspace(const CallWorkspace&) = delete;
    CallWorkspace& operator=(const CallWorkspace&) = delete;
    ~CallWorkspace() {
        if (kind == STREAM_ORDERED) {
            (void)hipFreeAsync(ptr, stream);
        } else if (kind == CACHED) {
            BlockCache& c = block_cache(dev);
            if (hipEventRecord(block.ev, stream) != hipSuccess) {
                // no event, no safe reuse: free it in stream order
                (void)hipGetLastError();
                (void)hipEventDestroy(block.ev);
                block.ev = nullptr;
                (void)hipFreeAsync(block.ptr, stream);
                std::lock_guard<std::mutex> lk(c.mu);
                c.taken_bytes -= block.bytes;
                return;
            }
            block.last = stream;
            block.primed = keep_primed;
            std::vector<WsBlock> evict;
            {
                std::lock_guard<std::mutex> lk(c.mu);
                c.taken_bytes -= block.bytes;
                c.free_blocks.push_back(block);
                c.free_bytes += block.bytes;
                // over the cache bound: give back free blocks, completed ones
                // first, then the oldest
                while (c.free_bytes > kCacheBytes && !c.free_blocks.empty()) {
                    size_t k = 0;
                    for (size_t i = 0; i < c.free_blocks.size(); ++i)
                        if (hipEventQuery(c.free_blocks[i].ev) == hipSuccess) {
                            k = i;
                            break;
                        }
                    c.free_bytes -= c.free_blocks[k].bytes;
                    evict.push_back(c.free_blocks[k]);
                    c.free_blocks.erase(c.free_blocks.begin() + (std::ptrdiff_t)k);
                }
            }
            (void)hipGetLastError();
            for (const WsBlock& b : evict) free_block(b, stream);
        }
    }
};

gt_status acquire_workspace(int dev, size_t bytes, hipStream_t stream, CallWorkspace& ws) {
    hipMemPool_t pool = nullptr;
    hipError_t he = pool_of(dev, &pool);
    if (he != hipSuccess) return hip_fail(he, "workspace pool");
    ws.stream = stream;
    ws.dev = dev;
    const size_t need = (bytes + kBlockGranule - 1) / kBlockGranule * kBlockGranule;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if ((he = hipStreamIsCapturing(stream, &cap)) != hipSuccess) return hip_fail(he, "hipStreamIsCapturing");
    const bool capturing = cap != hipStreamCaptureStatusNone;
    if (!capturing) {
        // a free block that fits: completed first, then last used on this
        // stream; the smallest such
        BlockCache& c = block_cache(dev);
        bool found = false, done = false;
        {
            std::lock_guard<std::mutex> lk(c.mu);
            size_t best = 0;
            int best_rank = 2;
            for (size_t i = 0; i < c.free_blocks.size(); ++i) {
                const WsBlock& b = c.free_blocks[i];
                if (b.bytes < need) continue;
                const hipError_t q = hipEventQuery(b.ev);
                const int rank = q == hipSuccess ? 0 : (q == hipErrorNotReady && b.last == stream) ? 1 : 2;
                if (rank < best_rank || (rank == best_rank && rank < 2 && b.bytes < c.free_blocks[best].bytes)) {
                    best = i;
                    best_rank = rank;
                }
            }
            (void)hipGetLastError();  // a query's not-ready status
            if (best_rank < 2) {
                ws.block = c.free_blocks[best];
                c.free_blocks.erase(c.free_blocks.begin() + (std::ptrdiff_t)best);
                c.free_bytes -= ws.block.bytes;
                c.taken_bytes += ws.block.bytes;
                found = true;
                done = best_rank == 0;
            }
        }
        if (found) {
            ws.kind = CallWorkspace::CACHED;
            ws.ptr = ws.block.ptr;
            if (!done && (he = hipStreamWaitEvent(stream, ws.block.ev, 0)) != hipSuccess)
                return hip_fail(he, "workspace wait");
            return GT_SUCCESS;
        }
    }
    void* p = nullptr;
    he = hipMallocFromPoolAsync(&p, capturing ? bytes : need, pool, stream);
    if (he != hipSuccess || !p) {
        (void)hipGetLastError();
        return fail(GT_ERROR_OUT_OF_MEMORY, "workspace allocation of " + std::to_string(bytes) + " bytes failed");
    }
    ws.ptr = static_cast<char*>(p);
    if (capturing) {
        ws.kind = CallWorkspace::STREAM_ORDERED;
        return GT_SUCCESS;
    }
    hipEvent_t ev = nullptr;
    if ((he = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) {
        ws.kind = CallWorkspace::STREAM_ORDERED;  // freed in stream order on return
        return hip_fail(he, "workspace event");
    }
    ws.block = WsBlock{ws.ptr, need, ev, stream};
    ws.kind = CallWorkspace::CACHED;
    BlockCache& c = block_cache(dev);
    std::lock_guard<std::mutex> lk(c.mu);
    c.taken_bytes += need;
    return GT_SUCCESS;
}

// Device address of the scratch array on device `dev` (the current device),
// looked up once per device.
struct ScratchAddrs {
    std::once_flag once[kMaxDevices];
    char* ptr[kMaxDevices] = {};
    hipError_t err[kMaxDevices] = {};
};
ScratchAddrs& scratch_addrs() {
    static ScratchAddrs* s = new ScratchAddrs();
    return *s;
}

hipError_t scratch_of(int dev, char** out) {
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    ScratchAddrs& sa = scratch_addrs();
    std::call_once(sa.once[dev], [&] {
        void* p = nullptr;
        sa.err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        sa.ptr[dev] = sa.err[dev] == hipSuccess ? static_cast<char*>(p) : nullptr;
    });
    *out = sa.ptr[dev];
    if (sa.err[dev] == hipSuccess && !sa.ptr[dev]) return hipErrorInvalidSymbol;
    return sa.err[dev];
}

gt_status scratch_exceeded(size_t bytes) {
    return fail(GT_ERROR_INVALID_VALUE, "the call needs " + std::to_string(bytes) +
                                            " bytes of workspace, more than the " + std::to_string(kScratchBytes) +
                                            "-byte scratch array of gt_attn_fwd_noalloc");
}

// The workspace of one call: from the pool, or (allocation-free entry point)
// the device's scratch array, whose size bounds the accepted problems.
gt_status call_workspace(bool noalloc, int dev, size_t bytes, hipStream_t stream, CallWorkspace& ws) {
    if (!noalloc) return acquire_workspace(dev, bytes, stream, ws);
    if (bytes > kScratchBytes) return scratch_exceeded(bytes);
    char* p = nullptr;
    const hipError_t he = scratch_of(dev, &p);
    if (he != hipSuccess) return hip_fail(he, "hipGetSymbolAddress(scratch)");
    ws.ptr = p;
    ws.stream = stream;
    ws.kind = CallWorkspace::SCRATCH;
    return GT_SUCCESS;
}

// Zeroes `n` counter ints of a fresh workspace, in stream order.
hipError_t clear_counters(int32_t* p, int n, hipStream_t stream) {
    hipLaunchKernelGGL(gt_clear_kernel, dim3(1), dim3(kBlock), 0, stream, p, n);
    return hipGetLastError();
}

struct Args {
    const int64_t* rowptr;
    const int32_t* colidx;
    const void* Q;
    const void* K;
    const void* V;
    void* out;
    float* lse;
    int64_t N, E;
    int32_t H, D;
    float scale;
    int kind = KIND_GT;
    const float* att = nullptr;  // GATv2 attention vector
    float slope = 0.0f;          // GATv2 LeakyReLU slope
    bool noalloc = false;        // workspace from the scratch array, no allocation
};

// The device a call works on: the calling thread's current device.  The
// workspace, its events and the kernels' memory all belong to it, so a stream
// created on another device is refused rather than fed memory it may not be
// able to reach.  (A stream handle the runtime cannot resolve is left to the
// launch, which reports it.)
gt_status call_device(hipStream_t stream, int* dev) {
    hipError_t he = hipGetDevice(dev);
    if (he != hipSuccess) return hip_fail(he, "hipGetDevice");
    hipDevice_t sd = *dev;
    if (hipStreamGetDevice(stream, &sd) != hipSuccess) {
        (void)hipGetLastError();
        return GT_SUCCESS;
    }
    if (sd != *dev)
        return fail(GT_ERROR_INVALID_VALUE, "the stream belongs to device " + std::to_string(sd) +
                                                ", the current device is " + std::to_string(*dev));
    return GT_SUCCESS;
}

int device_cus(int dev) {
    static std::atomic<int> cache[64];
    if (dev < 0 || dev >= 64) return 256;
    if (cache[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

// Workgroups of the attention kernel that the device holds at once.
template <typename T, int HS, int D, int KIND>
int attn_resident(int dev) {
    static std::atomic<int> cache[64];
    if (dev < 0 || dev >= 64) return 4 * 256;
    if (cache[dev] == 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gt_attn_kernel<T, HS, D, KIND>, kBlock, 0) != hipSuccess ||
            nb <= 0)
            nb = 4;
        cache[dev] = nb * device_cus(dev);
    }
    return cache[dev];
}

template <int H, int D, int KIND>
hipError_t launch_tiles(const TileParams& tp, hipStream_t stream) {
    const int64_t n_windows = (tp.N + kWin - 1) / kWin;
    hipLaunchKernelGGL((gt_tile_kernel<H, D, KIND>), dim3((unsigned)n_windows), dim3(kBlock), 0, stream, tp);
    return hipGetLastError();
}

// The tile kernel of H heads, for bf16 rows of at most 256 bytes.
template <int D, int KIND>
hipError_t pick_tiles(int H, const TileParams& tp, hipStream_t stream) {
    if (H == 1) return launch_tiles<1, D, KIND>(tp, stream);
    if constexpr (D <= 64)
        if (H == 2) return launch_tiles<2, D, KIND>(tp, stream);
    if constexpr (D <= 32)
        if (H == 4) return launch_tiles<4, D, KIND>(tp, stream);
    return hipErrorInvalidValue;
}

template <typename T, int HS, int D, int KIND>
gt_status launch(const Args& a, const gt_tuning* tu, hipStream_t stream) {
    using Op = AttnOp<T, HS, D, KIND>;
    constexpr bool kTileShape = KIND != KIND_GATV2 && std::is_same<T, bf16_tag>::value && D <= 128;
    static_assert(!kTileShape || Op::kSorted, "the tile path leaves its rows out of the light-row order");
    const int slices = a.H / HS;
    const AttnPlan plan = plan_attn(AttnShape{a.N, a.E, a.H, a.D, Elt<T>::kBytes, HS, Op::Gm::kP, KIND == KIND_GATV2, Op::kSorted},
                                    tu, a.noalloc);
    if (a.noalloc && plan.need > kScratchBytes) return scratch_exceeded(plan.need);
    int dev = 0;
    if (const gt_status ds = call_device(stream, &dev); ds != GT_SUCCESS) return ds;
    hipError_t he = hipSuccess;
    const RowGrid rg = row_grid(a.N, a.E, Op::Gm::kP, plan.slots.slices, plan.tiles, attn_resident<T, HS, D, KIND>(dev), tu);

    RowWork w;
    w.rowptr = a.rowptr;
    w.colidx = a.colidx;
    w.N = a.N;
    w.E = (uint32_t)a.E;
    set_rule(w, plan.rule);
    w.cap_slots = plan.slots.cap;

    CallWorkspace cw;
    gt_status st = call_workspace(a.noalloc, dev, plan.bytes, stream, cw);
    if (st != GT_SUCCESS) return st;
    char* ws = cw.ptr;
    // Counter sets: a cached block alternates between its two (the partition
    // zeroes the other one for the block's next call), so a block whose last
    // user was a forward call needs no clear kernel; a new block, the
    // scratch array and a captured stream clear the one set they use.
    int32_t* cnt_base = reinterpret_cast<int32_t*>(ws);
    const bool alternate = cw.kind == CallWorkspace::CACHED;
    w.counters = cnt_base + (alternate ? (cw.block.gen & 1u) * kRowsSetWords : 0);
    w.long_list = reinterpret_cast<LongRow*>(ws + plan.o_long);
    w.light_list = plan.sorted ? reinterpret_cast<LightRow*>(ws + plan.o_light) : nullptr;
    w.light_deg = reinterpret_cast<uint8_t*>(ws + plan.o_deg);
    w.long_blocks = 0;
    w.light_first = false;
    w.maybe_no_light = plan.tiles;

    // (the allocation-free entry point records no profiling events: creating
    // them is a runtime allocation)
    PhaseEvents ph;
    if (!a.noalloc && (he = ph.start(stream)) != hipSuccess) return hip_fail(he, "profiling events");
    if (!(alternate && cw.block.primed) && (he = clear_counters(w.counters, kRowsSetWords, stream)) != hipSuccess)
        return hip_fail(he, "counter clear");

    SortParams pp;
    pp.w = w;
    pp.step = Op::kU;
    pp.groups = Op::Gm::kP;
    if (plan.tiles) {
        pp.win_flags = reinterpret_cast<uint8_t*>(ws + plan.o_win);
        pp.tile_min = plan.tile_min;
        pp.tile_max = plan.tile_max;
    }
    if (alternate) pp.zero_next = cnt_base + ((cw.block.gen + 1u) & 1u) * kRowsSetWords;
    if ((he = launch_sort_rows(pp, stream)) != hipSuccess) return hip_fail(he, "partition launch");
    if (alternate) {
        ++cw.block.gen;
        cw.keep_primed = true;
    }
    ph.mark(1, stream);  // the attention phase includes the tile kernel
    if constexpr (kTileShape) {
        if (plan.tiles) {
            TileParams tp;
            tp.rowptr = a.rowptr;
            tp.colidx = a.colidx;
            tp.Q = static_cast<const char*>(a.Q);
            tp.K = static_cast<const char*>(a.K);
            tp.V = static_cast<const char*>(a.V);
            tp.out = static_cast<char*>(a.out);
            tp.lse = a.lse;
            tp.N = a.N;
            tp.c = a.scale * 1.4426950408889634f;
            tp.tile_max = plan.tile_max;
            tp.min_entries = plan.tile_min;
            tp.win_flags = pp.win_flags;
            tp.counters = w.counters;
            if ((he = pick_tiles<D, KIND>(a.H, tp, stream)) != hipSuccess) return hip_fail(he, "tile launch");
        }
    }

    AttnParams ap;
    ap.w = w;
    ap.Q = static_cast<const char*>(a.Q);
    ap.K = static_cast<const char*>(a.K);
    ap.V = static_cast<const char*>(a.V);
    ap.out = static_cast<char*>(a.out);
    ap.lse = a.lse;
    ap.c = (KIND != KIND_GATV2 ? a.scale : 1.0f) * 1.4426950408889634f;
    ap.att = a.att;
    ap.slope = a.slope;
    ap.row_shift = floor_log2((uint64_t)a.H * D * Elt<T>::kBytes);
    ap.heads = a.H;
    ap.part_ml = reinterpret_cast<float2*>(ws + plan.o_ml);
    ap.part_acc = reinterpret_cast<float*>(ws + plan.o_acc);
    ap.w.long_blocks = rg.long_blocks;
    ap.w.light_first = rg.light_first;
    const int merge_grid = merge_blocks(plan.slots, plan.rule, device_cus(dev));
    for (int s = 0; s < slices; s += plan.slots.slices) {
        ap.slice0 = s;
        hipLaunchKernelGGL((gt_attn_kernel<T, HS, D, KIND>), dim3(rg.blocks, plan.slots.slices), dim3(kBlock), 0, stream, ap);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "attention launch");
        if (s + plan.slots.slices >= slices) ph.mark(2, stream);
        hipLaunchKernelGGL((gt_merge_kernel<T, HS, D>), dim3(merge_grid, plan.slots.slices), dim3(kBlock), 0, stream, ap);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "merge launch");
    }
    ph.commit(stream);
    return GT_SUCCESS;
}

using LaunchFn = gt_status (*)(const Args&, const gt_tuning*, hipStream_t);

// The kernels of one slice of a row of H heads of D elements: the heads of 256
// bytes, or one where a head has more.  (128-byte slices, the least that reads
// whole cache lines, let an L2 cover twice the sources but visit every row twice
// as often.  128 / 256 bytes, us per call: R-MAT scale 21 fp32 4x32 4666 / 4743,
// bf16 4x32 2530 / 2573, bf16 8x64 lognormal 9889 / 9159, fp32 4x32 power law of
// 169 K nodes 212 / 218, fp32 2x32 with 17 uniform sources for each of 1 M nodes
// 1363 / 1266; GATv2, one row per entry: R-MAT scale 20 fp32 1492 / 1250.)
constexpr int kSliceBytes = 256;

template <typename T, int KIND>
LaunchFn pick_hd(int32_t H, int32_t D, bool wide = false) {
    constexpr bool kBf16 = std::is_same<T, bf16_tag>::value;
    constexpr int kFit = kSliceBytes / Elt<T>::kBytes;  // elements
    if (H != 1 && H != 2 && H != 4 && H != 8) return nullptr;
    switch (D) {
        case 32:
            if constexpr (kFit >= 128)
                if (H >= 4) return &launch<T, 4, 32, KIND>;
            if constexpr (kFit >= 64)
                if (H >= 2) return &launch<T, 2, 32, KIND>;
            return &launch<T, 1, 32, KIND>;
        case 64:
            if constexpr (kFit >= 128)
                if (H >= 2) return &launch<T, 2, 64, KIND>;
            return &launch<T, 1, 64, KIND>;
        case 128:
            if constexpr (KIND == KIND_GATV2 && !kBf16)
                if (wide) return &launch<T, 2, 128, KIND>;
            return &launch<T, 1, 128, KIND>;
        case 256: return &launch<T, 1, 256, KIND>;
        case 512:  // a head must fit 64 lanes of 16 bytes
            if constexpr (kBf16)
                if (H <= 4) return &launch<T, 1, 512, KIND>;
            return nullptr;
        default: return nullptr;
    }
}

bool overlaps(const void* a, size_t an, const void* b, size_t bn) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + bn && y < x + an;
}

// Tuning fields are counts of entries, rows or workgroups: positive values
// beyond kTuningMax (about 2^31 - 2^16) would overflow the partition's
// rounding and comparisons, so they are refused.
constexpr int32_t kTuningMax = INT32_MAX - (1 << 16);

gt_status check_tuning(const gt_tuning* tu) {
    if (!tu) return GT_SUCCESS;
    const int32_t f[] = {tu->light_max_deg, tu->heavy_min_deg, tu->chunk_edges, tu->grid_blocks, tu->dense_tiles};
    for (int32_t v : f)
        if (v > kTuningMax)
            return fail(GT_ERROR_INVALID_VALUE, "a tuning field exceeds " + std::to_string(kTuningMax));
    return GT_SUCCESS;
}

gt_status run(gt_dtype dtype, const Args& a, const gt_tuning* tu, hipStream_t stream) {
    t_last_error.clear();
    if (check_tuning(tu) != GT_SUCCESS) return GT_ERROR_INVALID_VALUE;
    if (dtype != GT_DTYPE_F32 && dtype != GT_DTYPE_BF16) return fail(GT_ERROR_NOT_SUPPORTED, "unknown dtype");
    if (a.N < 0 || a.N >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "N must be in [0, 2^31)");
    if (a.E < 0 || a.E >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "E must be in [0, 2^31)");
    if (a.H < 1 || a.D < 1) return fail(GT_ERROR_INVALID_VALUE, "H and D must be positive");
    if (!std::isfinite(a.scale)) return fail(GT_ERROR_INVALID_VALUE, "scale must be finite");
    if (a.kind == KIND_GATV2 && !std::isfinite(a.slope)) return fail(GT_ERROR_INVALID_VALUE, "slope must be finite");
    LaunchFn fn;
    if (a.kind == KIND_GATV2)
        fn = dtype == GT_DTYPE_F32 ? pick_hd<float, KIND_GATV2>(a.H, a.D, wide_slices(a.N, a.E, (int64_t)a.H * a.D * 4))
                                   : pick_hd<bf16_tag, KIND_GATV2>(a.H, a.D);
    else
        fn = dtype == GT_DTYPE_F32 ? pick_hd<float, KIND_GT>(a.H, a.D)
             : (tu && tu->bf16_weights) ? pick_hd<bf16_tag, KIND_GT_BF16W>(a.H, a.D)
                                        : pick_hd<bf16_tag, KIND_GT>(a.H, a.D);
    if (!fn)
        return fail(GT_ERROR_NOT_SUPPORTED, "unsupported (H, D) = (" + std::to_string(a.H) + ", " +
                                                std::to_string(a.D) + "); H in {1,2,4,8} with D in {32,64,128,256}, or bf16 D = 512 with H in {1,2,4}");
    if (a.N == 0) return GT_SUCCESS;
    if (!a.rowptr) return fail(GT_ERROR_INVALID_VALUE, "rowptr is null");
    if (a.E > 0 && !a.colidx) return fail(GT_ERROR_INVALID_VALUE, "colidx is null");
    if (!a.Q || !a.K || !a.V || !a.out) return fail(GT_ERROR_INVALID_VALUE, "Q, K, V and out (L, R and out) must be non-null");
    for (const void* ptr : {a.Q, a.K, a.V, static_cast<const void*>(a.out)})
        if (reinterpret_cast<uintptr_t>(ptr) % 16 != 0)
            return fail(GT_ERROR_INVALID_VALUE, "Q, K, V and out (L, R and out) must be 16-byte aligned");
    const size_t bytes = (size_t)a.N * a.H * a.D * (dtype == GT_DTYPE_F32 ? 4 : 2);
    for (const void* in : {a.Q, a.K, a.V})
        if (overlaps(a.out, bytes, in, bytes)) return fail(GT_ERROR_INVALID_VALUE, "out overlaps Q, K or V (L or R)");
    if (a.lse) {
        const size_t lb = (size_t)a.N * a.H * sizeof(float);
        if (reinterpret_cast<uintptr_t>(a.lse) % 4 != 0) return fail(GT_ERROR_INVALID_VALUE, "lse must be 4-byte aligned");
        for (const void* o : {a.Q, a.K, a.V, static_cast<const void*>(a.out)})
            if (overlaps(a.lse, lb, o, bytes)) return fail(GT_ERROR_INVALID_VALUE, "lse overlaps Q, K, V or out");
    }
    if (a.kind == KIND_GATV2) {
        const size_t ab = (size_t)a.H * a.D * sizeof(float);
        if (!a.att || reinterpret_cast<uintptr_t>(a.att) % 16 != 0)
            return fail(GT_ERROR_INVALID_VALUE, "att must be non-null and 16-byte aligned");
        if (overlaps(a.out, bytes, a.att, ab) || (a.lse && overlaps(a.lse, (size_t)a.N * a.H * sizeof(float), a.att, ab)))
            return fail(GT_ERROR_INVALID_VALUE, "out or lse overlaps att");
    }
    return fn(a, tu, stream);
}

#include "gt_bwd.hpp"

gt_status run_bwd(gt_dtype dtype, const BwdArgs& a, hipStream_t stream) {
    t_last_error.clear();
    if (dtype != GT_DTYPE_F32 && dtype != GT_DTYPE_BF16) return fail(GT_ERROR_NOT_SUPPORTED, "unknown dtype");
    if (a.N < 0 || a.N >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "N must be in [0, 2^31)");
    if (a.E < 0 || a.E >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "E must be in [0, 2^31)");
    if (a.H < 1 || a.D < 1) return fail(GT_ERROR_INVALID_VALUE, "H and D must be positive");
    if (!std::isfinite(a.scale)) return fail(GT_ERROR_INVALID_VALUE, "scale must be finite");
    BwdFn fn = dtype == GT_DTYPE_F32 ? pick_bwd<float>(a.H, a.D) : pick_bwd<bf16_tag>(a.H, a.D);
    if (!fn)
        return fail(GT_ERROR_NOT_SUPPORTED, "unsupported (H, D) = (" + std::to_string(a.H) + ", " +
                                                std::to_string(a.D) + "); H in {1,2,4,8} with D in {32,64,128,256}, or bf16 D = 512 with H in {1,2,4}");
    if (a.N == 0) return GT_SUCCESS;
    if (!a.rowptr || !a.rowptr_t) return fail(GT_ERROR_INVALID_VALUE, "rowptr or rowptr_t is null");
    if (a.E > 0 && (!a.colidx || !a.colidx_t)) return fail(GT_ERROR_INVALID_VALUE, "colidx or colidx_t is null");
    const void* ins[] = {a.Q, a.K, a.V, a.O, a.dO};
    const void* outs[] = {a.dQ, a.dK, a.dV};
    for (const void* ptr : ins)
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 16 != 0)
            return fail(GT_ERROR_INVALID_VALUE, "Q, K, V, out and dout must be non-null and 16-byte aligned");
    for (const void* ptr : outs)
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 16 != 0)
            return fail(GT_ERROR_INVALID_VALUE, "dQ, dK and dV must be non-null and 16-byte aligned");
    if (!a.lse || reinterpret_cast<uintptr_t>(a.lse) % 4 != 0)
        return fail(GT_ERROR_INVALID_VALUE, "lse must be non-null and 4-byte aligned");
    const size_t bytes = (size_t)a.N * a.H * a.D * (dtype == GT_DTYPE_F32 ? 4 : 2);
    for (int g = 0; g < 3; ++g) {
        for (const void* in : ins)
            if (overlaps(outs[g], bytes, in, bytes)) return fail(GT_ERROR_INVALID_VALUE, "a gradient overlaps an input");
        if (overlaps(outs[g], bytes, a.lse, (size_t)a.N * a.H * sizeof(float)))
            return fail(GT_ERROR_INVALID_VALUE, "a gradient overlaps lse");
        // distinct gradients, also when two are the same pointer
        for (int g2 = g + 1; g2 < 3; ++g2)
            if (overlaps(outs[g], bytes, outs[g2], bytes)) return fail(GT_ERROR_INVALID_VALUE, "gradients overlap");
    }
    return fn(a, stream);
}

#include "gt_reduce.hpp"

gt_status run_reduce(gt_dtype dtype, int op, const ReduceArgs& a0, const gt_tuning* tu, hipStream_t stream) {
    t_last_error.clear();
    if (dtype != GT_DTYPE_F32 && dtype != GT_DTYPE_BF16) return fail(GT_ERROR_NOT_SUPPORTED, "unknown dtype");
    if (op != GT_REDUCE_MIN && op != GT_REDUCE_MAX) return fail(GT_ERROR_NOT_SUPPORTED, "unknown reduce op");
    if (check_tuning(tu) != GT_SUCCESS) return GT_ERROR_INVALID_VALUE;
    if (a0.N < 0 || a0.N >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "N must be in [0, 2^31)");
    if (a0.E < 0 || a0.E >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "E must be in [0, 2^31)");
    if (a0.F < 1) return fail(GT_ERROR_INVALID_VALUE, "F must be positive");
    const bool wide = wide_slices(a0.N, a0.E, (int64_t)a0.F * (dtype == GT_DTYPE_F32 ? 4 : 2));
    ReduceFn fn = dtype == GT_DTYPE_F32 ? pick_reduce<float>(a0.F, wide) : pick_reduce<bf16_tag>(a0.F, wide);
    if (!fn)
        return fail(GT_ERROR_NOT_SUPPORTED, "unsupported F = " + std::to_string(a0.F) +
                                                "; rows of 64 B to 4 KiB in powers of two (fp32 F in {16..1024}, "
                                                "bf16 F in {32..2048})");
    if (a0.N == 0) return GT_SUCCESS;
    if (!a0.rowptr) return fail(GT_ERROR_INVALID_VALUE, "rowptr is null");
    if (a0.E > 0 && !a0.colidx) return fail(GT_ERROR_INVALID_VALUE, "colidx is null");
    if (!a0.X || !a0.out) return fail(GT_ERROR_INVALID_VALUE, "X and out must be non-null");
    for (const void* ptr : {a0.X, static_cast<const void*>(a0.out), static_cast<const void*>(a0.arg)})
        if (reinterpret_cast<uintptr_t>(ptr) % 16 != 0)
            return fail(GT_ERROR_INVALID_VALUE, "X, out and arg must be 16-byte aligned");
    const size_t bytes = (size_t)a0.N * a0.F * (dtype == GT_DTYPE_F32 ? 4 : 2);
    const size_t abytes = (size_t)a0.N * a0.F * sizeof(int32_t);
    if (overlaps(a0.out, bytes, a0.X, bytes)) return fail(GT_ERROR_INVALID_VALUE, "out overlaps X");
    if (a0.arg && (overlaps(a0.arg, abytes, a0.X, bytes) || overlaps(a0.arg, abytes, a0.out, bytes)))
        return fail(GT_ERROR_INVALID_VALUE, "arg overlaps X or out");
    ReduceArgs a = a0;
    a.flip = op == GT_REDUCE_MAX ? 0xFFFFFFFFu : 0u;
    return fn(a, tu, stream);
}

#include "gt_study.hpp"

gt_status run_dot_aggr(const int64_t* rowptr, const int32_t* colidx, const float* X, float* out, int64_t N,
                       int64_t E, int32_t F, int32_t mapping, int32_t load_bytes, hipStream_t stream) {
    t_last_error.clear();
    if (N < 0 || N >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "N must be in [0, 2^31)");
    if (E < 0 || E >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "E must be in [0, 2^31)");
    DotFn fn = pick_dot(mapping, load_bytes, F);
    if (!fn)
        return fail(GT_ERROR_NOT_SUPPORTED, "unsupported dot-aggr variant: mapping in {0, 1}, load_bytes in "
                                            "{4, 16}, F in {32, 64, 128, 256, 512}");
    if (N == 0) return GT_SUCCESS;
    if (!rowptr || (E > 0 && !colidx) || !X || !out) return fail(GT_ERROR_INVALID_VALUE, "null pointer");
    if (reinterpret_cast<uintptr_t>(X) % 16 != 0 || reinterpret_cast<uintptr_t>(out) % 4 != 0)
        return fail(GT_ERROR_INVALID_VALUE, "X must be 16-byte and out 4-byte aligned");
    if (overlaps(out, (size_t)N * sizeof(float), X, (size_t)N * F * sizeof(float)))
        return fail(GT_ERROR_INVALID_VALUE, "out overlaps X");
    DotParams dp{rowptr, colidx, X, out, N};
    const int64_t blocks = (N + kWavesPerBlock - 1) / kWavesPerBlock;
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kBlock), 0, stream, dp);
    const hipError_t he = hipGetLastError();
    if (he != hipSuccess) return hip_fail(he, "dot-aggr launch");
    return GT_SUCCESS;
}

}  // namespace

extern "C" {

gt_status gt_attn_fwd(const int64_t* rowptr, const int32_t* colidx, const float* Q, const float* K,
                      const float* V, float* out, int64_t N, int64_t E, int32_t H, int32_t D, float scale,
                      hipStream_t stream) {
    return run(GT_DTYPE_F32, Args{rowptr, colidx, Q, K, V, out, nullptr, N, E, H, D, scale}, nullptr, stream);
}

gt_status gt_attn_fwd_bf16(const int64_t* rowptr, const int32_t* colidx, const uint16_t* Q, const uint16_t* K,
                           const uint16_t* V, uint16_t* out, int64_t N, int64_t E, int32_t H, int32_t D,
                           float scale, hipStream_t stream) {
    return run(GT_DTYPE_BF16, Args{rowptr, colidx, Q, K, V, out, nullptr, N, E, H, D, scale}, nullptr, stream);
}

gt_status gt_attn_fwd_ex(gt_dtype dtype, const int64_t* rowptr, const int32_t* colidx, const void* Q,
                         const void* K, const void* V, void* out, float* lse, int64_t N, int64_t E, int32_t H,
                         int32_t D, float scale, const gt_tuning* tuning, hipStream_t stream) {
    return run(dtype, Args{rowptr, colidx, Q, K, V, out, lse, N, E, H, D, scale}, tuning, stream);
}

gt_status gt_attn_fwd_noalloc(gt_dtype dtype, const int64_t* rowptr, const int32_t* colidx, const void* Q,
                              const void* K, const void* V, void* out, float* lse, int64_t N, int64_t E, int32_t H,
                              int32_t D, float scale, const gt_tuning* tuning, hipStream_t stream) {
    Args a{rowptr, colidx, Q, K, V, out, lse, N, E, H, D, scale};
    a.noalloc = true;
    return run(dtype, a, tuning, stream);
}

gt_status gt_gatv2_fwd(gt_dtype dtype, const int64_t* rowptr, const int32_t* colidx, const void* L, const void* R,
                       const float* att, float slope, void* out, float* lse, int64_t N, int64_t E, int32_t H,
                       int32_t D, const gt_tuning* tuning, hipStream_t stream) {
    Args a{rowptr, colidx, L, R, R, out, lse, N, E, H, D, 1.0f};
    a.kind = KIND_GATV2;
    a.att = att;
    a.slope = slope;
    return run(dtype, a, tuning, stream);
}

gt_status gt_attn_bwd(gt_dtype dtype, const int64_t* rowptr, const int32_t* colidx, const int64_t* rowptr_t,
                      const int32_t* colidx_t, const void* Q, const void* K, const void* V, const void* out,
                      const void* dout, const float* lse, void* dQ, void* dK, void* dV, int64_t N, int64_t E,
                      int32_t H, int32_t D, float scale, hipStream_t stream) {
    return run_bwd(dtype,
                   BwdArgs{rowptr, colidx, rowptr_t, colidx_t, Q, K, V, out, dout, lse, dQ, dK, dV, N, E, H, D, scale},
                   stream);
}

gt_status gt_segment_reduce(gt_dtype dtype, gt_reduce_op op, const int64_t* rowptr, const int32_t* colidx,
                            const void* X, void* out, int32_t* arg, int64_t N, int64_t E, int32_t F,
                            const gt_tuning* tuning, hipStream_t stream) {
    return run_reduce(dtype, (int)op, ReduceArgs{rowptr, colidx, X, out, arg, N, E, F, 0u}, tuning, stream);
}

gt_status gt_dot_aggr(const int64_t* rowptr, const int32_t* colidx, const float* X, float* out, int64_t N,
                      int64_t E, int32_t F, int32_t mapping, int32_t load_bytes, hipStream_t stream) {
    return run_dot_aggr(rowptr, colidx, X, out, N, E, F, mapping, load_bytes, stream);
}

gt_status gt_csr_validate(const int64_t* rowptr, const int32_t* colidx, int64_t N, int64_t E, int32_t* valid,
                          hipStream_t stream) {
    t_last_error.clear();
    if (!valid) return fail(GT_ERROR_INVALID_VALUE, "valid is null");
    *valid = 0;
    if (N < 0 || E < 0 || E >= (int64_t(1) << 31)) return fail(GT_ERROR_INVALID_VALUE, "bad N or E");
    if (!rowptr || (E > 0 && !colidx)) return fail(GT_ERROR_INVALID_VALUE, "null CSR pointer");
    int32_t* bad = nullptr;
    hipError_t he = hipMallocAsync(reinterpret_cast<void**>(&bad), sizeof(int32_t), stream);
    if (he != hipSuccess) return fail(GT_ERROR_OUT_OF_MEMORY, "flag allocation failed");
    // the flag is freed (stream-ordered) on every path once it was allocated
    auto failed = [&](hipError_t e, const char* what) {
        (void)hipFreeAsync(bad, stream);
        return hip_fail(e, what);
    };
    if ((he = hipMemsetAsync(bad, 0, sizeof(int32_t), stream)) != hipSuccess) return failed(he, "hipMemsetAsync");
    const int64_t work = N > E ? N : E;
    int grid = (int)((work + kBlock - 1) / kBlock);
    if (grid > 4096) grid = 4096;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(gt_csr_check_kernel, dim3(grid), dim3(kBlock), 0, stream, rowptr, colidx, N, E, bad);
    if ((he = hipGetLastError()) != hipSuccess) return failed(he, "validate launch");
    int32_t h_bad = 1;
    if ((he = hipMemcpyAsync(&h_bad, bad, sizeof(int32_t), hipMemcpyDeviceToHost, stream)) != hipSuccess)
        return failed(he, "hipMemcpyAsync");
    (void)hipFreeAsync(bad, stream);
    if ((he = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(he, "hipStreamSynchronize");
    *valid = h_bad == 0 ? 1 : 0;
    return GT_SUCCESS;
}

const char* gt_status_string(gt_status s) {
    switch (s) {
        case GT_SUCCESS: return "success";
        case GT_ERROR_INVALID_VALUE: return "invalid value";
        case GT_ERROR_NOT_SUPPORTED: return "not supported";
        case GT_ERROR_OUT_OF_MEMORY: return "out of memory";
        case GT_ERROR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

const char* gt_last_error_message(void) { return t_last_error.c_str(); }

gt_status gt_profile_enable(int32_t enable) {
    Profiler& pr = profiler();
    std::lock_guard<std::mutex> lk(pr.mu);
    for (auto& ev : pr.pending) {
        (void)hipEventSynchronize(ev[3]);
        for (auto e : ev) (void)hipEventDestroy(e);
    }
    pr.pending.clear();
    pr.on = enable != 0;
    return GT_SUCCESS;
}

gt_status gt_profile_collect(double ms[3], int64_t* calls) {
    t_last_error.clear();
    if (!ms || !calls) return fail(GT_ERROR_INVALID_VALUE, "null output");
    Profiler& pr = profiler();
    std::lock_guard<std::mutex> lk(pr.mu);
    ms[0] = ms[1] = ms[2] = 0.0;
    *calls = 0;
    gt_status st = GT_SUCCESS;
    for (auto& ev : pr.pending) {
        hipError_t he = hipEventSynchronize(ev[3]);
        if (he != hipSuccess) {
            st = hip_fail(he, "hipEventSynchronize");
        } else {
            for (int k = 0; k < 3; ++k) {
                float t = 0.0f;
                if (hipEventElapsedTime(&t, ev[k], ev[k + 1]) == hipSuccess) ms[k] += t;
            }
            ++*calls;
        }
        for (auto e : ev) (void)hipEventDestroy(e);
    }
    pr.pending.clear();
    return st;
}

gt_status gt_workspace_pool_stats(int32_t device, uint64_t* reserved_bytes, uint64_t* used_bytes) {
    t_last_error.clear();
    if (!reserved_bytes || !used_bytes) return fail(GT_ERROR_INVALID_VALUE, "null output");
    *reserved_bytes = 0;
    *used_bytes = 0;
    if (device < 0 || device >= kMaxDevices) return fail(GT_ERROR_INVALID_VALUE, "device out of range");
    DevicePools& dp = device_pools();
    if (!dp.ready[device].load(std::memory_order_acquire) || !dp.pool[device]) return GT_SUCCESS;
    uint64_t r = 0;
    const hipError_t he = hipMemPoolGetAttribute(dp.pool[device], hipMemPoolAttrReservedMemCurrent, &r);
    if (he != hipSuccess) return hip_fail(he, "hipMemPoolGetAttribute");
    BlockCache& c = block_cache(device);
    std::lock_guard<std::mutex> lk(c.mu);
    *reserved_bytes = r;
    *used_bytes = c.taken_bytes;
    return GT_SUCCESS;
}

gt_status gt_workspace_release(void) {
    t_last_error.clear();
    DevicePools& dp = device_pools();
    gt_status st = GT_SUCCESS;
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess) cur = -1;
    for (int dev = 0; dev < kMaxDevices; ++dev) {
        // a device's pool is created by its first call; devices without one
        // are skipped
        if (!dp.ready[dev].load(std::memory_order_acquire)) continue;
        hipMemPool_t pool = dp.pool[dev];
        if (!pool) continue;
        std::vector<WsBlock> blocks;
        {
            BlockCache& c = block_cache(dev);
            std::lock_guard<std::mutex> lk(c.mu);
            blocks.swap(c.free_blocks);
            c.free_bytes = 0;
        }
        hipError_t he = hipSetDevice(dev);
        // each free block after its last use, then the pool down to nothing
        for (const WsBlock& b : blocks) {
            if (he == hipSuccess) he = hipEventSynchronize(b.ev);
            (void)hipEventDestroy(b.ev);
            if (he == hipSuccess) he = hipFreeAsync(b.ptr, nullptr);
        }
        if (he == hipSuccess) he = hipStreamSynchronize(nullptr);
        if (he == hipSuccess) he = hipMemPoolTrimTo(pool, 0);
        if (he != hipSuccess) st = hip_fail(he, "returning workspace of a device");
    }
    if (cur >= 0) (void)hipSetDevice(cur);
    return st;
}

}  // extern "C"
