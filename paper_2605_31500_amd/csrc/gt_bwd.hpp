// Backward pass of the fused graph-transformer attention (included by
// gt_attn.hip inside its anonymous namespace; uses its device helpers, the row
// work order of gt_rows.hpp and the call workspace).
//
// Gradients for an upstream gradient dO (paper, Appendix D.2, backward pass of
// the graph transformer: the weights are recomputed from the stored per-row
// statistic L_i = ln sum_e exp(s_e), alpha_e = exp(s_e - L_i), and
// Delta_i = <O_i, dO_i>).  Per CSR entry e = (i, j) and head:
//     ds_e = alpha_e * (<dO_i, V_j> - Delta_i)
//     dQ_i += scale * ds_e * K_j          (pass 0, CSR rows i)
//     dK_j += scale * ds_e * Q_i          (pass 1, transposed rows j)
//     dV_j += alpha_e * dO_i              (pass 1)
// The paper's kernel walks the transposed graph and adds dK with atomics;
// here both passes are gathers over rows (the transposed structure is an
// input, as the paper's cached transposed adjacency), the pieces of cut rows are
// summed in a fixed order, and the results are bitwise reproducible.
//
// Both passes have the same per-entry shape, with (a, b) the row's own
// vectors and (x, y) the gathered ones:
//     pass 0: a = Q_i, b = dO_i, x = K_j, y = V_j, (L, Delta) of the row i
//     pass 1: a = K_j, b = V_j, x = Q_i, y = dO_i, (L, Delta) gathered at i
//     s = <a, x> scale, alpha = exp(s - L), ds = alpha (<b, y> - Delta)
//     acc1 += ds x;  pass 1 also: acc2 += alpha y
// Pass 0 leaves (L log2(e), Delta) of each row and head as one pair, so that an
// entry of pass 1 reads one line for both.  Like the forward, the passes gather
// two random rows per entry and are bound by the path from L2 to the fabric;
// us per call with whole rows in row order, and with slices and source ranges:
// R-MAT scale 20 bf16 4x32 3772 -> 2728, 300 K R-MAT nodes fp32 4x32 1794 -> 1373;
// lognormal 200 K nodes bf16 8x64 3798 -> 3631; power law fp32 4x32 of 169 K nodes
// 478 -> 442, of 16 K nodes 71 -> 66.

struct BwdParams {
    RowWork w;      // rows of this pass (CSR or transposed CSR)
    const char* A;  // row-own vectors a / b
    const char* B;
    const char* X;  // gathered vectors x / y
    const char* Y;
    const char* O;     // pass 0: forward output (for Delta)
    const float* lse;  // [N][H] natural log
    float2* stat;      // [N][H] (lse log2(e), Delta): written by pass 0, read by pass 1
    char* out1;        // dQ (pass 0) or dK (pass 1)
    char* out2;        // dV (pass 1)
    float c;      // scale * log2(e)
    float scale;
    int32_t row_shift;
    int32_t heads;
    int32_t slice0;  // slice of blockIdx.y == 0
    float* part;  // [slice of this launch][slot][NACC * HS * D]
};

// bf16 dot over the four pairs of two 16-byte vectors, accumulated in fp32
__device__ __forceinline__ float dot8_bf16(const uint4& a, const uint4& b) {
    float d = dot2_bf16(a.x, b.x, 0.0f);
    d = dot2_bf16(a.y, b.y, d);
    d = dot2_bf16(a.z, b.z, d);
    return dot2_bf16(a.w, b.w, d);
}

template <typename T, int HS, int D, int MODE>
struct BwdState;

template <typename T, int HS, int D, int MODE>
struct BwdOp {
    using Gm = Geo<T, HS, D>;
    using State = BwdState<T, HS, D, MODE>;
    static constexpr int kG = Gm::kG;
    static constexpr int kU = Gm::kP >= 4 && Gm::kU >= 8 ? Gm::kU / 2 : Gm::kU;
    static constexpr bool kSorted = Gm::kP >= 4;
    static constexpr int NACC = MODE ? 2 : 1;
    static constexpr int kSlotFloats = NACC * HS * D;
    const char* A;
    const char* B;
    const char* X;
    const char* Y;
    const char* O;
    const float* lse;  // at the slice's first head
    float2* stat;
    char* out1;
    char* out2;
    float* part;
    float c, scale;
    int row_shift, heads;

    __device__ __forceinline__ uint64_t offset(int32_t row, int lig) const {
        return ((uint64_t)(uint32_t)row << row_shift) + (uint32_t)lig * 16u;
    }
};

template <typename T, int HS, int D, int MODE>
__device__ __forceinline__ BwdOp<T, HS, D, MODE> bwd_op(const BwdParams& p) {
    using Op = BwdOp<T, HS, D, MODE>;
    const int head = (p.slice0 + (int)blockIdx.y) * HS;
    const int64_t at = (int64_t)head * D * Elt<T>::kBytes;
    Op op;
    op.A = p.A + at;
    op.B = p.B + at;
    op.X = p.X + at;
    op.Y = p.Y + at;
    op.O = p.O + at;
    op.lse = p.lse + head;
    op.stat = p.stat + head;
    op.out1 = p.out1 + at;
    op.out2 = p.out2 + at;
    op.part = p.part + (int64_t)blockIdx.y * p.w.cap_slots * Op::kSlotFloats;
    op.c = p.c;
    op.scale = p.scale;
    op.row_shift = p.row_shift;
    op.heads = p.heads;
    return op;
}

template <typename T, int HS, int D, int MODE>
struct BwdState {
    using Op = BwdOp<T, HS, D, MODE>;
    using Gm = Geo<T, HS, D>;
    static constexpr int EPV = Gm::kEPV, kU = Op::kU;
    // bf16 features: the two dots per entry are bf16 dot2 on raw pairs, and
    // the accumulations pair two entries: their coefficients (ds, alpha) are
    // rounded to one bf16 pair and dot2 multiplies it with the two entries'
    // elements, accumulating in fp32.
    static constexpr bool kDot2 = std::is_same<T, bf16_tag>::value;
    static_assert(!kDot2 || kU % 2 == 0, "dot2 pairs entries");
    uint4 a, b;  // the row's own vectors
    float acc1[EPV], acc2[EPV];
    float L2, Dl;  // pass 0: the row's statistics (of this lane's head)

    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc1[e] = acc2[e] = 0.0f;
    }

    __device__ __forceinline__ void begin(const Op& op, int32_t row, int lig) {
        const uint64_t off = op.offset(row, lig);
        a = load_once(op.A + off);
        b = load_once(op.B + off);
        if constexpr (MODE == 0) {
            const uint4 o = load_once(op.O + off);
            const int64_t at = (int64_t)row * op.heads + lig / Gm::kHL;
            L2 = op.lse[at] * 1.4426950408889634f;
            float d = 0.0f;
            if constexpr (kDot2) {
                d = dot8_bf16(o, b);
            } else {
                float of[EPV], bf[EPV];
                widen<T>(o, of);
                widen<T>(b, bf);
#pragma unroll
                for (int e = 0; e < EPV; ++e) d = fmaf(of[e], bf[e], d);
            }
            Dl = head_sum<Gm::kHL>(d);
            // (the pieces of a cut row all write the same pair)
            if (lig % Gm::kHL == 0) op.stat[at] = make_float2(L2, Dl);
        }
    }

    struct Batch {
        uint4 x[kU], y[kU];
        float2 st[MODE ? kU : 1];
    };

    __device__ __forceinline__ void issue(const Op& op, const int32_t (&j)[kU], int lig, Batch& bt) const {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t off = op.offset(j[u], lig);
            bt.x[u] = *reinterpret_cast<const uint4*>(op.X + off);
            bt.y[u] = *reinterpret_cast<const uint4*>(op.Y + off);
            if constexpr (MODE == 1) bt.st[u] = op.stat[(int64_t)j[u] * op.heads + lig / Gm::kHL];
        }
    }

    __device__ __forceinline__ void consume(const Op& op, const Batch& bt, const int32_t (&)[kU], int nvalid) {
#pragma clang fp contract(off)
        float al[kU], ds[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            float s = 0.0f, da = 0.0f;
            if constexpr (kDot2) {
                s = dot8_bf16(a, bt.x[u]);
                da = dot8_bf16(b, bt.y[u]);
            } else {
                float af[EPV], bf[EPV], x[EPV], y[EPV];
                widen<T>(a, af);
                widen<T>(b, bf);
                widen<T>(bt.x[u], x);
                widen<T>(bt.y[u], y);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    s = fmaf(af[e], x[e], s);
                    da = fmaf(bf[e], y[e], da);
                }
            }
            s = head_sum<Gm::kHL>(s) * op.c;
            da = head_sum<Gm::kHL>(da);
            const float l2 = MODE == 1 ? bt.st[MODE ? u : 0].x : L2;
            const float dl = MODE == 1 ? bt.st[MODE ? u : 0].y : Dl;
            al[u] = (u < nvalid) ? fast_exp2(s - l2) : 0.0f;
            ds[u] = al[u] * (da - dl);
        }
        if constexpr (kDot2) {
#pragma unroll
            for (int u = 0; u < kU; u += 2) {
                const uint32_t pds = pack_bf16(ds[u], ds[u + 1]);
                const uint32_t pal = pack_bf16(al[u], al[u + 1]);
                const uint4 x0 = bt.x[u], x1 = bt.x[u + 1], y0 = bt.y[u], y1 = bt.y[u + 1];
                const uint32_t xa[4] = {x0.x, x0.y, x0.z, x0.w}, xb[4] = {x1.x, x1.y, x1.z, x1.w};
                const uint32_t ya[4] = {y0.x, y0.y, y0.z, y0.w}, yb[4] = {y1.x, y1.y, y1.z, y1.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc1[2 * q] = dot2_bf16(pds, pair_lo(xa[q], xb[q]), acc1[2 * q]);
                    acc1[2 * q + 1] = dot2_bf16(pds, pair_hi(xa[q], xb[q]), acc1[2 * q + 1]);
                    if constexpr (MODE == 1) {
                        acc2[2 * q] = dot2_bf16(pal, pair_lo(ya[q], yb[q]), acc2[2 * q]);
                        acc2[2 * q + 1] = dot2_bf16(pal, pair_hi(ya[q], yb[q]), acc2[2 * q + 1]);
                    }
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                float x[EPV], y[EPV];
                widen<T>(bt.x[u], x);
                widen<T>(bt.y[u], y);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    acc1[e] = fmaf(ds[u], x[e], acc1[e]);
                    if constexpr (MODE == 1) acc2[e] = fmaf(al[u], y[e], acc2[e]);
                }
            }
        }
    }

    __device__ __forceinline__ void merge_xor(int off) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            acc1[e] += __shfl_xor(acc1[e], off);
            if constexpr (MODE == 1) acc2[e] += __shfl_xor(acc2[e], off);
        }
    }

    __device__ __forceinline__ void store_out(const Op& op, int32_t row, int lig) const {
        const uint64_t off = op.offset(row, lig);
        float o[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) o[e] = acc1[e] * op.scale;
        store_once(op.out1 + off, narrow<T>(o));
        if constexpr (MODE == 1) store_once(op.out2 + off, narrow<T>(acc2));
    }

    __device__ __forceinline__ void store_partial(const Op& op, int32_t slot, int lig) const {
        float* dst = op.part + (int64_t)slot * Op::kSlotFloats + lig * EPV;
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
            *reinterpret_cast<float4*>(dst + e) = make_float4(acc1[e], acc1[e + 1], acc1[e + 2], acc1[e + 3]);
            if constexpr (MODE == 1)
                *reinterpret_cast<float4*>(dst + HS * D + e) = make_float4(acc2[e], acc2[e + 1], acc2[e + 2], acc2[e + 3]);
        }
    }

    struct Partial {
        float a1[EPV], a2[MODE ? EPV : 1];
    };

    __device__ __forceinline__ static void load_partial(const Op& op, int32_t slot, int lig, Partial& pt) {
        const float* src = op.part + (int64_t)slot * Op::kSlotFloats + lig * EPV;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            pt.a1[e] = src[e];
            if constexpr (MODE == 1) pt.a2[e] = src[HS * D + e];
        }
    }

    __device__ __forceinline__ void add(const Partial& pt, bool valid) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float t1 = acc1[e] + pt.a1[e];
            acc1[e] = valid ? t1 : acc1[e];
            if constexpr (MODE == 1) {
                const float t2 = acc2[e] + pt.a2[e];
                acc2[e] = valid ? t2 : acc2[e];
            }
        }
    }
};

template <typename T, int HS, int D, int MODE>
__global__ void __launch_bounds__(kBlock) gt_bwd_kernel(BwdParams p) {
    using Op = BwdOp<T, HS, D, MODE>;
    __shared__ __attribute__((aligned(16))) int32_t tiles[kWavesPerBlock][kWave / Op::kG * TileOf<Op::kG>::kEntries];
    row_loop(p.w, bwd_op<T, HS, D, MODE>(p), tiles[threadIdx.x / kWave]);
}

// Sum of the partial states of each cut row in a fixed order (lane group g adds
// pieces g, g + P, ..., then the groups are summed across lanes), then scaling
// and storing: one wavefront per row and slice.
template <typename T, int HS, int D, int MODE>
__global__ void __launch_bounds__(kBlock) gt_bwd_merge_kernel(BwdParams p) {
    using Op = BwdOp<T, HS, D, MODE>;
    constexpr uint32_t G = Op::kG, P = kWave / G;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t g = lane / G;
    const int lig = lane % G;
    if (ROWS_CNT(p.w.counters, ROWS_PIECES) == 0) return;  // no long rows
    const CutRows cut(p.w, lane);
    const uint32_t n = cut.count(), waves = gridDim.x * kWavesPerBlock;
    const Op op = bwd_op<T, HS, D, MODE>(p);
    for (uint32_t i = blockIdx.x * kWavesPerBlock + wv; i < n; i += waves) {
        uint32_t slot, nq;
        const int32_t row = cut.row(p.w, i, lane, slot, nq);
        typename Op::State st;
        st.reset();
        for (uint32_t q0 = 0; q0 < nq; q0 += P * kMergePieces) {
            // (a group without a piece reads the row's last and leaves it out)
            typename Op::State::Partial pt[kMergePieces];
#pragma unroll
            for (uint32_t u = 0; u < kMergePieces; ++u) {
                const uint32_t q = q0 + u * P + g;
                st.load_partial(op, (int32_t)(slot + (q < nq ? q : nq - 1)), lig, pt[u]);
            }
#pragma unroll
            for (uint32_t u = 0; u < kMergePieces; ++u) st.add(pt[u], q0 + u * P + g < nq);
        }
#pragma unroll
        for (int off = G; off < kWave; off <<= 1) st.merge_xor(off);
        if (g == 0) st.store_out(op, row, lig);
    }
}

struct BwdArgs {
    const int64_t* rowptr;
    const int32_t* colidx;
    const int64_t* rowptr_t;
    const int32_t* colidx_t;
    const void* Q;
    const void* K;
    const void* V;
    const void* O;
    const void* dO;
    const float* lse;
    void* dQ;
    void* dK;
    void* dV;
    int64_t N, E;
    int32_t H, D;
    float scale;
};

template <typename T, int HS, int D, int MODE>
int bwd_resident(int dev) {
    static std::atomic<int> cache[64];
    if (dev < 0 || dev >= 64) return 4 * 256;
    if (cache[dev] == 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gt_bwd_kernel<T, HS, D, MODE>, kBlock, 0) != hipSuccess ||
            nb <= 0)
            nb = 4;
        cache[dev] = nb * device_cus(dev);
    }
    return cache[dev];
}

// One pass: the partition of its structure, then slice by slice its row kernel
// and the merge of the cut rows.
template <typename T, int HS, int D, int MODE>
gt_status launch_bwd_pass(BwdParams bp, const RowRule& rule, const SlotPlan& sp, int dev, hipStream_t stream) {
    using Op = BwdOp<T, HS, D, MODE>;
    hipError_t he = hipSuccess;
    const RowGrid rg = row_grid(bp.w.N, bp.w.E, Op::Gm::kP, sp.slices, false, bwd_resident<T, HS, D, MODE>(dev), nullptr);
    bp.w.long_blocks = rg.long_blocks;
    bp.w.light_first = rg.light_first;
    SortParams pp;
    pp.w = bp.w;
    pp.step = Op::kU;
    pp.groups = Op::Gm::kP;
    if ((he = launch_sort_rows(pp, stream)) != hipSuccess) return hip_fail(he, "partition launch");
    const int merge_grid = merge_blocks(sp, rule, device_cus(dev));
    for (int s = 0; s < bp.heads / HS; s += sp.slices) {
        bp.slice0 = s;
        hipLaunchKernelGGL((gt_bwd_kernel<T, HS, D, MODE>), dim3(rg.blocks, sp.slices), dim3(kBlock), 0, stream, bp);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "backward launch");
        hipLaunchKernelGGL((gt_bwd_merge_kernel<T, HS, D, MODE>), dim3(merge_grid, sp.slices), dim3(kBlock), 0, stream, bp);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "backward merge launch");
    }
    return GT_SUCCESS;
}

template <typename T, int HS, int D>
gt_status launch_bwd(const BwdArgs& a, hipStream_t stream) {
    using Op = BwdOp<T, HS, D, 1>;
    constexpr int kSlotBytes = Op::kSlotFloats * (int)sizeof(float);  // (pass 0: half of it)
    const int slices = a.H / HS;
    const RowRule rule = row_rule(a.N, a.E, slices, 2 * HS * D * Elt<T>::kBytes, 2 * kSlotBytes + 1024, Op::Gm::kP,
                                  nullptr);
    int dev = 0;
    if (const gt_status ds = call_device(stream, &dev); ds != GT_SUCCESS) return ds;
    hipError_t he = hipSuccess;

    // workspace: a counter set per pass | statistics | light rows | long rows | partial states
    RowWork w;
    w.N = a.N;
    w.E = (uint32_t)a.E;
    set_rule(w, rule);
    size_t off = 0;
    const size_t o_cnt = off;    off = align_up(off + 2 * kRowsSetWords * sizeof(int32_t), 256);
    const size_t o_stat = off;   off = align_up(off + (size_t)a.N * a.H * sizeof(float2), 256);
    const size_t o_light = off;  off = align_up(off + (Op::kSorted ? (size_t)a.N * sizeof(LightRow) : 0), 256);
    const size_t o_deg = off;    off = align_up(off + (Op::kSorted ? (size_t)a.N : 0), 256);
    const size_t o_long = off;
    off = align_up(off + (size_t)long_list_rows(a.N, a.E, w.light_max) * sizeof(LongRow), 256);
    const SlotPlan sp = slot_plan(rule, slices, kSlotBytes, off, false);
    w.cap_slots = sp.cap;
    const size_t o_part = off;   off = align_up(off + (size_t)sp.cap * sp.slices * kSlotBytes, 256);

    CallWorkspace cw;
    gt_status st = acquire_workspace(dev, off, stream, cw);
    if (st != GT_SUCCESS) return st;
    char* ws = cw.ptr;
    int32_t* cnt_sets = reinterpret_cast<int32_t*>(ws + o_cnt);
    if ((he = clear_counters(cnt_sets, 2 * kRowsSetWords, stream)) != hipSuccess) return hip_fail(he, "counter clear");
    w.light_list = Op::kSorted ? reinterpret_cast<LightRow*>(ws + o_light) : nullptr;
    w.light_deg = reinterpret_cast<uint8_t*>(ws + o_deg);
    w.long_list = reinterpret_cast<LongRow*>(ws + o_long);
    w.long_blocks = 0;
    w.light_first = false;
    w.maybe_no_light = false;

    for (int mode = 0; mode < 2; ++mode) {
        w.rowptr = mode == 0 ? a.rowptr : a.rowptr_t;
        w.colidx = mode == 0 ? a.colidx : a.colidx_t;
        w.counters = cnt_sets + mode * kRowsSetWords;
        BwdParams bp;
        bp.w = w;
        bp.A = static_cast<const char*>(mode == 0 ? a.Q : a.K);
        bp.B = static_cast<const char*>(mode == 0 ? a.dO : a.V);
        bp.X = static_cast<const char*>(mode == 0 ? a.K : a.Q);
        bp.Y = static_cast<const char*>(mode == 0 ? a.V : a.dO);
        bp.O = static_cast<const char*>(a.O);
        bp.lse = a.lse;
        bp.stat = reinterpret_cast<float2*>(ws + o_stat);
        bp.out1 = static_cast<char*>(mode == 0 ? a.dQ : a.dK);
        bp.out2 = static_cast<char*>(a.dV);
        bp.c = a.scale * 1.4426950408889634f;
        bp.scale = a.scale;
        bp.row_shift = floor_log2((uint64_t)a.H * D * Elt<T>::kBytes);
        bp.heads = a.H;
        bp.part = reinterpret_cast<float*>(ws + o_part);
        st = mode == 0 ? launch_bwd_pass<T, HS, D, 0>(bp, rule, sp, dev, stream)
                       : launch_bwd_pass<T, HS, D, 1>(bp, rule, sp, dev, stream);
        if (st != GT_SUCCESS) return st;
    }
    return GT_SUCCESS;
}

using BwdFn = gt_status (*)(const BwdArgs&, hipStream_t);

// Slices as in the forward: the heads of 256 bytes, or one.
template <typename T>
BwdFn pick_bwd(int32_t H, int32_t D) {
    constexpr bool kBf16 = std::is_same<T, bf16_tag>::value;
    if (H != 1 && H != 2 && H != 4 && H != 8) return nullptr;
    switch (D) {
        case 32:
            if constexpr (kBf16)
                if (H >= 4) return &launch_bwd<T, 4, 32>;
            if (H >= 2) return &launch_bwd<T, 2, 32>;
            return &launch_bwd<T, 1, 32>;
        case 64:
            if constexpr (kBf16)
                if (H >= 2) return &launch_bwd<T, 2, 64>;
            return &launch_bwd<T, 1, 64>;
        case 128: return &launch_bwd<T, 1, 128>;
        case 256: return &launch_bwd<T, 1, 256>;
        case 512:  // a head must fit 64 lanes of 16 bytes
            if constexpr (kBf16)
                if (H <= 4) return &launch_bwd<T, 1, 512>;
            return nullptr;
        default: return nullptr;
    }
}
