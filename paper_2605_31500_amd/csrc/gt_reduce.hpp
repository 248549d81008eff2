// Segment min/max aggregation over a CSR graph (the paper's reduction family,
// Section 2.2 family (ii); Appendix, degree-aware reduction-based
// aggregation).  For every destination row i and feature f:
//     out[i,f] = REDUCE over the CSR entries e of row i of X[j_e, f]
//     arg[i,f] = the source j_e that attains it (-1 for an empty row)
// with REDUCE = min or max under the order-preserving key of the paper's
// packed (value, index) merge: the fp32 bit pattern with all bits inverted
// when the sign bit is set and the sign bit set otherwise, compared as an
// unsigned integer, ties to the smallest source index.
//
// Design: each lane keeps, per feature it owns, one 64-bit word
// (key << 32 | source); the reduction is a plain unsigned 64-bit minimum
// (max uses the complemented key, so ties still go to the smallest source).
// The words are exactly the paper's packed atomics operands, but here they
// stay in registers: the rows are worked on as row_loop says (slices of 256
// bytes, one lane group per light row or piece of a longer one, the pieces' source
// ranges on their XCDs) and the partial words of cut rows are merged by a second
// kernel instead of 64-bit atomics.  Padding entries of a step repeat a valid
// entry, which a minimum absorbs, so they need no mask.
// Min with sources, whole rows in row order -> slices and source ranges (us per
// call): R-MAT scale 20, 128 fp32 features 1640 -> 1366; lognormal 500 K nodes, 512
// fp32 5316 -> 4486; power law 20 K nodes, 1024 bf16 138 -> 93, 169 K nodes, 512 fp32
// 502 -> 462.  Slices of 128 / 256 / 512 bytes (with rows cut from 65 entries on):
// 1518 / 1412 / 1376, 5095 / 4763 / 4705, 93 / 86 / 94 and 506 / 492 / 505.
// This file is included by gt_attn.hip inside its anonymous namespace.

constexpr uint64_t kRedEmpty = ~0ull;  // no entry yet: source 0xFFFFFFFF is never valid

// Key of one fp32 bit pattern, complemented for max: bits ^ 0x80000000 for a
// clear sign bit, ~bits for a set one (then ^ flip).
__device__ __forceinline__ uint32_t red_key(uint32_t bits, uint32_t flip) {
    const uint32_t neg = (uint32_t)((int32_t)bits >> 31);
    return bits ^ (neg & 0x7FFFFFFFu) ^ (0x80000000u ^ flip);
}

// Inverse of red_key for the stored word: the fp32 bit pattern.
__device__ __forceinline__ uint32_t red_value_bits(uint64_t w, uint32_t flip) {
    const uint32_t k = (uint32_t)(w >> 32) ^ flip;
    return (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
}

template <typename T> __device__ __forceinline__ uint32_t red_bits(const uint4& r, int e);
template <> __device__ __forceinline__ uint32_t red_bits<float>(const uint4& r, int e) {
    return e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w;
}
template <> __device__ __forceinline__ uint32_t red_bits<bf16_tag>(const uint4& r, int e) {
    const uint32_t w = (e >> 1) == 0 ? r.x : (e >> 1) == 1 ? r.y : (e >> 1) == 2 ? r.z : r.w;
    return (e & 1) ? (w & 0xFFFF0000u) : (w << 16);
}

template <typename T, int NVEC>
struct RedState;

// One slice of NVEC 16-byte vectors of the feature row.
template <typename T, int NVEC>
struct RedOp {
    using State = RedState<T, NVEC>;
    static constexpr int kEPV = 16 / Elt<T>::kBytes;  // elements per vector
    static constexpr int kG = NVEC;
    static constexpr int kU = 4;
    static constexpr bool kSorted = true;
    static constexpr int kSlotWords = NVEC * kEPV;
    const char* X;
    char* out;
    int32_t* arg;    // at the slice's first feature, or nullptr
    uint64_t* part;  // [slot][kSlotWords] packed (key, source)
    int row_shift;   // log2 of the bytes of one feature row
    int64_t features;
    uint32_t flip;   // 0 for min, 0xFFFFFFFF for max

    __device__ __forceinline__ uint64_t offset(int32_t row, int lig) const {
        return ((uint64_t)(uint32_t)row << row_shift) + (uint32_t)lig * 16u;
    }
};

template <typename T, int NVEC>
struct RedState {
    using Op = RedOp<T, NVEC>;
    static constexpr int kU = Op::kU, kEPV = Op::kEPV;
    uint64_t best[kEPV];

    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int e = 0; e < kEPV; ++e) best[e] = kRedEmpty;
    }

    __device__ __forceinline__ void begin(const Op&, int32_t, int) {}

    struct Batch {
        uint4 x[kU];
    };

    __device__ __forceinline__ void issue(const Op& op, const int32_t (&j)[kU], int lig, Batch& bt) const {
#pragma unroll
        for (int u = 0; u < kU; ++u) bt.x[u] = *reinterpret_cast<const uint4*>(op.X + op.offset(j[u], lig));
    }

    __device__ __forceinline__ void consume(const Op& op, const Batch& bt, const int32_t (&j)[kU], int) {
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int e = 0; e < kEPV; ++e) {
                const uint64_t w = ((uint64_t)red_key(red_bits<T>(bt.x[u], e), op.flip) << 32) | (uint32_t)j[u];
                best[e] = w < best[e] ? w : best[e];
            }
    }

    __device__ __forceinline__ void merge_xor(int off) {
#pragma unroll
        for (int e = 0; e < kEPV; ++e) {
            const uint32_t lo = __shfl_xor((uint32_t)best[e], off);
            const uint32_t hi = __shfl_xor((uint32_t)(best[e] >> 32), off);
            const uint64_t o = ((uint64_t)hi << 32) | lo;
            best[e] = o < best[e] ? o : best[e];
        }
    }

    __device__ __forceinline__ void store_out(const Op& op, int32_t row, int lig) const {
        uint32_t vb[kEPV];
        int32_t src[kEPV];
#pragma unroll
        for (int e = 0; e < kEPV; ++e) {
            const bool none = (uint32_t)best[e] == 0xFFFFFFFFu;
            vb[e] = none ? 0u : red_value_bits(best[e], op.flip);
            src[e] = none ? -1 : (int32_t)(uint32_t)best[e];
        }
        uint4 o;
        if constexpr (kEPV == 4) {
            o = make_uint4(vb[0], vb[1], vb[2], vb[3]);
        } else {
            // the selected value came from a bf16, so its low half is zero
            o = make_uint4((vb[0] >> 16) | (vb[1] & 0xFFFF0000u), (vb[2] >> 16) | (vb[3] & 0xFFFF0000u),
                           (vb[4] >> 16) | (vb[5] & 0xFFFF0000u), (vb[6] >> 16) | (vb[7] & 0xFFFF0000u));
        }
        store_once(op.out + op.offset(row, lig), o);
        if (op.arg) {
            char* arow = reinterpret_cast<char*>(op.arg + (int64_t)row * op.features + lig * kEPV);
#pragma unroll
            for (int e = 0; e < kEPV; e += 4)
                store_once(arow + e * 4, make_uint4((uint32_t)src[e], (uint32_t)src[e + 1], (uint32_t)src[e + 2], (uint32_t)src[e + 3]));
        }
    }

    __device__ __forceinline__ void store_partial(const Op& op, int32_t slot, int lig) const {
        uint64_t* dst = op.part + (int64_t)slot * Op::kSlotWords + lig * kEPV;
#pragma unroll
        for (int e = 0; e < kEPV; e += 2)
            *reinterpret_cast<uint4*>(dst + e) = make_uint4((uint32_t)best[e], (uint32_t)(best[e] >> 32),
                                                            (uint32_t)best[e + 1], (uint32_t)(best[e + 1] >> 32));
    }

    __device__ __forceinline__ void merge_partial(const Op& op, int32_t slot, int lig) {
        const uint64_t* src = op.part + (int64_t)slot * Op::kSlotWords + lig * kEPV;
#pragma unroll
        for (int e = 0; e < kEPV; ++e) best[e] = src[e] < best[e] ? src[e] : best[e];
    }
};

struct ReduceParams {
    RowWork w;
    const char* X;
    char* out;
    int32_t* arg;    // [N][F] or nullptr
    uint64_t* part;  // [slice of this launch][slot][kSlotWords]
    int32_t row_shift;
    int32_t features;
    int32_t slice0;  // slice of blockIdx.y == 0
    uint32_t flip;
};

template <typename T, int NVEC>
__device__ __forceinline__ RedOp<T, NVEC> reduce_op(const ReduceParams& p) {
    using Op = RedOp<T, NVEC>;
    const int slice = p.slice0 + (int)blockIdx.y;
    Op op;
    op.X = p.X + (int64_t)slice * NVEC * 16;
    op.out = p.out + (int64_t)slice * NVEC * 16;
    op.arg = p.arg ? p.arg + (int64_t)slice * Op::kSlotWords : nullptr;
    op.part = p.part + (int64_t)blockIdx.y * p.w.cap_slots * Op::kSlotWords;
    op.row_shift = p.row_shift;
    op.features = p.features;
    op.flip = p.flip;
    return op;
}

template <typename T, int NVEC>
__global__ void __launch_bounds__(kBlock) gt_reduce_kernel(ReduceParams p) {
    using Op = RedOp<T, NVEC>;
    __shared__ __attribute__((aligned(16))) int32_t tiles[kWavesPerBlock][kWave / Op::kG * TileOf<Op::kG>::kEntries];
    row_loop(p.w, reduce_op<T, NVEC>(p), tiles[threadIdx.x / kWave]);
}

// Merge of the partial words of each cut row, one wavefront per row and slice;
// a group without a piece reads the row's last again, which a minimum absorbs.
template <typename T, int NVEC>
__global__ void __launch_bounds__(kBlock) gt_reduce_merge_kernel(ReduceParams p) {
    using Op = RedOp<T, NVEC>;
    constexpr uint32_t G = Op::kG, P = kWave / G;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t g = lane / G;
    const int lig = lane % G;
    if (ROWS_CNT(p.w.counters, ROWS_PIECES) == 0) return;  // no long rows
    const CutRows cut(p.w, lane);
    const uint32_t n = cut.count(), waves = gridDim.x * kWavesPerBlock;
    const Op op = reduce_op<T, NVEC>(p);
    for (uint32_t i = blockIdx.x * kWavesPerBlock + wv; i < n; i += waves) {
        uint32_t slot, nq;
        const int32_t row = cut.row(p.w, i, lane, slot, nq);
        typename Op::State st;
        st.reset();
        for (uint32_t q0 = 0; q0 < nq; q0 += P * kMergePieces)
#pragma unroll
            for (uint32_t u = 0; u < kMergePieces; ++u) {
                const uint32_t q = q0 + u * P + g;
                st.merge_partial(op, (int32_t)(slot + (q < nq ? q : nq - 1)), lig);
            }
#pragma unroll
        for (int off = G; off < kWave; off <<= 1) st.merge_xor(off);
        if (g == 0) st.store_out(op, row, lig);
    }
}

struct ReduceArgs {
    const int64_t* rowptr;
    const int32_t* colidx;
    const void* X;
    void* out;
    int32_t* arg;
    int64_t N, E;
    int32_t F;
    uint32_t flip;
};

template <typename T, int NVEC>
int reduce_resident(int dev) {
    static std::atomic<int> cache[64];
    if (dev < 0 || dev >= 64) return 4 * 256;
    if (cache[dev] == 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gt_reduce_kernel<T, NVEC>, kBlock, 0) != hipSuccess ||
            nb <= 0)
            nb = 4;
        cache[dev] = nb * device_cus(dev);
    }
    return cache[dev];
}

template <typename T, int NVEC>
gt_status launch_reduce(const ReduceArgs& a, const gt_tuning* tu, hipStream_t stream) {
    using Op = RedOp<T, NVEC>;
    constexpr int kSlotBytes = Op::kSlotWords * (int)sizeof(uint64_t);
    const int slices = a.F / (NVEC * Op::kEPV);
    const RowRule rule = row_rule(a.N, a.E, slices, NVEC * 16, 3 * (2 * kSlotBytes + 256) / 4, kWave / NVEC, tu);
    int dev = 0;
    if (const gt_status ds = call_device(stream, &dev); ds != GT_SUCCESS) return ds;
    hipError_t he = hipSuccess;

    // workspace: counters | light rows | long rows | partial words
    RowWork w;
    w.rowptr = a.rowptr;
    w.colidx = a.colidx;
    w.N = a.N;
    w.E = (uint32_t)a.E;
    set_rule(w, rule);
    size_t off = 0;
    const size_t o_cnt = off;    off = align_up(off + kRowsSetWords * sizeof(int32_t), 256);
    const size_t o_light = off;  off = align_up(off + (size_t)a.N * sizeof(LightRow), 256);
    const size_t o_deg = off;    off = align_up(off + (size_t)a.N, 256);
    const size_t o_long = off;
    off = align_up(off + (size_t)long_list_rows(a.N, a.E, w.light_max) * sizeof(LongRow), 256);
    const SlotPlan sp = slot_plan(rule, slices, kSlotBytes, off, false);
    const RowGrid rg = row_grid(a.N, a.E, kWave / NVEC, sp.slices, false, reduce_resident<T, NVEC>(dev), tu);
    w.cap_slots = sp.cap;
    const size_t o_part = off;   off = align_up(off + (size_t)sp.cap * sp.slices * kSlotBytes, 256);

    CallWorkspace cw;
    gt_status st = acquire_workspace(dev, off, stream, cw);
    if (st != GT_SUCCESS) return st;
    char* ws = cw.ptr;
    w.counters = reinterpret_cast<int32_t*>(ws + o_cnt);
    w.light_list = reinterpret_cast<LightRow*>(ws + o_light);
    w.light_deg = reinterpret_cast<uint8_t*>(ws + o_deg);
    w.long_list = reinterpret_cast<LongRow*>(ws + o_long);
    w.long_blocks = rg.long_blocks;
    w.light_first = rg.light_first;
    w.maybe_no_light = false;

    PhaseEvents ph;
    if ((he = ph.start(stream)) != hipSuccess) return hip_fail(he, "profiling events");
    if ((he = clear_counters(w.counters, kRowsSetWords, stream)) != hipSuccess) return hip_fail(he, "counter clear");
    SortParams pp;
    pp.w = w;
    pp.step = Op::kU;
    pp.groups = kWave / NVEC;
    if ((he = launch_sort_rows(pp, stream)) != hipSuccess) return hip_fail(he, "partition launch");
    ph.mark(1, stream);

    ReduceParams rp;
    rp.w = w;
    rp.X = static_cast<const char*>(a.X);
    rp.out = static_cast<char*>(a.out);
    rp.arg = a.arg;
    rp.part = reinterpret_cast<uint64_t*>(ws + o_part);
    rp.row_shift = floor_log2((uint64_t)a.F * Elt<T>::kBytes);
    rp.features = a.F;
    rp.flip = a.flip;
    const int merge_grid = merge_blocks(sp, rule, device_cus(dev));
    for (int s = 0; s < slices; s += sp.slices) {
        rp.slice0 = s;
        hipLaunchKernelGGL((gt_reduce_kernel<T, NVEC>), dim3(rg.blocks, sp.slices), dim3(kBlock), 0, stream, rp);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "reduce launch");
        if (s + sp.slices >= slices) ph.mark(2, stream);
        hipLaunchKernelGGL((gt_reduce_merge_kernel<T, NVEC>), dim3(merge_grid, sp.slices), dim3(kBlock), 0, stream, rp);
        if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "reduce merge launch");
    }
    ph.commit(stream);
    return GT_SUCCESS;
}

using ReduceFn = gt_status (*)(const ReduceArgs&, const gt_tuning*, hipStream_t);

// Row sizes of 64 B .. 4 KiB: fp32 F in {16, ..., 1024}, bf16 F in {32, ..., 2048};
// slices of 256 bytes, or the row (1 KB where wide_slices says so).
template <typename T>
ReduceFn pick_reduce(int32_t F, bool wide) {
    constexpr int EPV = 16 / Elt<T>::kBytes;
    if (F <= 0 || F % EPV != 0) return nullptr;
    switch (F / EPV) {
        case 4: return &launch_reduce<T, 4>;
        case 8: return &launch_reduce<T, 8>;
        case 16:
        case 32:
        case 64:
        case 128: return &launch_reduce<T, 16>;
        case 256: return wide ? &launch_reduce<T, 64> : &launch_reduce<T, 16>;
        default: return nullptr;
    }
}
