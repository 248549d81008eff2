// Work order of the row kernels: which lane group reads which entries of which
// row, and on which XCD (included by gt_attn.hip inside its anonymous
// namespace).
//
// What bounds these kernels is the path from L2 to the fabric.  Gathers of random
// pieces read 24-27 TB/s where the table lies in an XCD's 4 MB L2, 7.0-7.3 TB/s
// from one of 128 MB (in the Infinity Cache) and 6.2-6.4 TB/s from one of 4 GB,
// pieces of 128 to 1024 bytes alike.  So the order of the work is built for L2
// hits:
//   * Feature slices.  A call runs over slices of the feature row (256 bytes, or
//     a head), one after another: an L2 then covers as many more sources as
//     there are slices.
//   * Source ranges per XCD.  The rows of a CSR are commonly sorted, so the q-th
//     of nq equal pieces of a row reads about the q-th nq-th of the sources.  A
//     long row is cut into nq = 8m pieces, and XCD x takes pieces xm .. xm+m-1
//     of every long row, all rows' first pieces first: at any time an L2 holds
//     an eighth of the sources or less, where it would otherwise see them all.
//     (Unsorted rows have no such locality and still pay for the pieces.  Listed
//     graphs with each row's entries shuffled, speed against whole rows in row
//     order: R-MAT scale 21 fp32 1.02, bf16 0.97, power law of 169 K nodes 0.98,
//     lognormal 1.16, backward of R-MAT scale 20 1.12.)
// Counted L2 hit rate and bytes beyond the L2 of a fp32 4x32 forward, whole rows
// in row order -> so: R-MAT scale 21 16.5 -> 42.8 %, 46.1 -> 32.1 GB, 6.13 -> 4.43
// ms; a power-law graph of 169 K nodes with uniform sources 8.6 -> 15.9 %, 1.45 ->
// 1.35 GB, 200 -> 189 us: 7.2 TB/s before and after.
//
// A row of degree d <= light_max is one segment.  Longer rows are listed by
// degree octave (class c: 2^c <= d < 2^(c+1)); all rows of a class are cut into
// the same number of pieces, so a piece is found from the row's place in its
// class list and its number, and no list of pieces is written.  A segment
// (a light row, a piece) is read by one lane group; pieces longer than
// group_len are spread over the P groups of a wavefront and merged there.

#define ROWS_CNT(c, i) ((c)[(i) * kRowsStride])

constexpr uint32_t kDegMany = 255;

struct RowWork : RowCut {
    const int64_t* rowptr;
    const int32_t* colidx;
    bool maybe_no_light;  // the tile path may have taken every light row
    uint32_t long_blocks;  // workgroups of a slice that take the long rows
    bool light_first;      // these are its last ones (else its first)
    int32_t* counters;
    LongRow* long_list;    // rows of degree > light_max, class after class, the longest first
    // [N] light rows in step order per partition block, row -1 elsewhere, and
    // their degrees (kDegMany: that many or more); nullptr: rows in id order
    LightRow* light_list;
    uint8_t* light_deg;
};

// Inclusive sum over lanes 0..31 (lanes 32..63 must hold 0; their result is
// not the sum).
__device__ __forceinline__ uint32_t scan32(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    return x;
}

__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}

// The classes' rows, pieces and places, one class per lane.
struct ClassPlan {
    uint32_t n;      // rows
    uint32_t nq;     // pieces of each row (1: not cut)
    uint32_t off;    // first row in long_list
    uint32_t slot0;  // first partial state (cut classes)
};

__device__ __forceinline__ ClassPlan class_plan(const RowWork& w, int lane) {
    const int c = kClasses - 1 - lane;
    ClassPlan pl;
    const uint32_t cap = lane < kClasses ? class_capacity(w, c) : 0u;
    pl.n = cap ? min((uint32_t)ROWS_CNT(w.counters, c), cap) : 0u;
    pl.off = scan32(cap) - cap;
    pl.nq = cap ? class_pieces(w, c) : 1u;
    uint32_t slots = pl.nq > 1 ? pl.n * pl.nq : 0u;
    uint32_t upto = scan32(slots);
    if (lane_value(upto, kClasses - 1) > w.cap_slots) {
        // Not enough room for the partial states: the longest rows keep their
        // pieces, then classes get half as many until they fit.
        uint32_t left = w.cap_slots;
        for (int i = 1; i < kClasses; ++i) {
            const uint32_t n = lane_value(pl.n, i);
            const uint32_t nq = fit_pieces(n, lane_value(pl.nq, i), left);
            if (nq > 1) left -= n * nq;
            if (lane == i) pl.nq = nq;
        }
        slots = pl.nq > 1 ? pl.n * pl.nq : 0u;
        upto = scan32(slots);
    }
    pl.slot0 = upto - slots;
    return pl;
}

// Index tile of a lane group: kR loads per lane.
template <int G> struct TileOf {
    static constexpr int kR = G >= 64 ? 1 : 2;
    static constexpr int kEntries = kR * G;
};

// One wavefront's share of a slice.  Op gives the arithmetic: kG lanes per
// group, kU entries per step, kSorted (light rows in the partition's step
// order), and a State with reset(), begin(op, row, lig), Batch, issue(op, j,
// lig, batch), consume(op, batch, j, nvalid), merge_xor(offset), store_out(op,
// row, lig) and store_partial(op, slot, lig).
//
// long_blocks workgroups of a slice take the long rows' pieces, the others the
// light rows.  An XCD's waves (blockIdx.x mod 8) take its batches (one
// segment per lane group each) in turn: the longest rows first, so that time
// runs with the source ranges, and the light rows of an eighth of the ids.  (In
// turn and not in equal consecutive shares, where waves of one workgroup get
// rows of one length and end far apart: R-MAT scale 21 fp32 5.30 against
// 5.05 ms; drawn one by one from an atomic counter by as many waves as the
// device holds: 5.29 ms, and the power-law graph of 169 K nodes 285 against
// 212 us.)  A light row's wave needs no counters, only its list entry.
// Segments are software-pipelined: list entries are requested two batches
// ahead, a segment's first index tile while its predecessor's first gathers are
// in flight and each further tile one tile ahead, so that a short row costs
// about one memory latency instead of three (list, colidx, features).
template <typename Op>
__device__ __forceinline__ void row_loop(const RowWork& w, const Op& op, int32_t* __restrict__ tile) {
    constexpr int G = Op::kG, P = kWave / G, U = Op::kU;
    constexpr int R = TileOf<G>::kR, TE = TileOf<G>::kEntries;
    static_assert(TE % U == 0, "index tiles hold whole steps");
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t g = lane / G, lig = lane % G;
    int32_t* gtile = tile + g * TE;

    // ---- this XCD's batches
    const uint32_t xcd = blockIdx.x % kXcds;
    const uint32_t rank = blockIdx.x / kXcds, ranks = gridDim.x / kXcds, long_ranks = w.long_blocks / kXcds;
    const uint32_t second = w.light_first ? ranks - long_ranks : long_ranks;  // the rest starts there
    const bool long_rows = (rank < second) != w.light_first;
    const uint32_t waves = (long_rows ? long_ranks : ranks - long_ranks) * kWavesPerBlock;
    uint32_t it = (rank < second ? rank : rank - second) * kWavesPerBlock +
                  __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t total, l0 = 0;
    ClassPlan pl{};
    uint32_t lo = 0, hi = 0, nb = 0, cum = 0;
    bool spread = false;
    if (long_rows) {
        if (it >= batch_bound((uint32_t)ROWS_CNT(w.counters, ROWS_PIECES), P)) return;
        pl = class_plan(w, lane);
        const uint64_t flat = (uint64_t)pl.n * pl.nq;  // pieces, piece number major
        lo = piece_share(flat, xcd);
        hi = piece_share(flat, xcd + 1);
        spread = lane < kClasses && class_spread(w, kClasses - 1 - lane, pl.nq);
        nb = piece_batches(hi - lo, spread, P);
        cum = scan32(nb);
        total = lane_value(cum, kClasses - 1);
    } else {
        const uint64_t n_light = ((uint64_t)w.N + P - 1) / P;
        l0 = (uint32_t)(n_light * xcd / kXcds);
        total = (uint32_t)(n_light * (xcd + 1) / kXcds) - l0;
        // (none left in the order: every light row lies in a dense window)
        if (w.maybe_no_light && ROWS_CNT(w.counters, ROWS_LIGHT) == 0) return;
    }
    if (it >= total) return;

    struct Seg {
        int32_t row;          // -1: none
        uint32_t begin, deg;  // its entries
        uint32_t q;           // piece q of nq
        uint32_t nq;          // (uniform)
        int32_t slot;         // partial state of a cut row's piece, or -1
        bool spread;          // (uniform) over the wavefront's groups
    };
    const bool sorted = Op::kSorted && w.light_list;
    auto fetch = [&](uint32_t i) -> Seg {
        Seg s{-1, 0u, 0u, 0u, 1u, -1, false};
        if (i >= total) return s;
        if (long_rows) {
            const int c = __builtin_ctzll(__ballot(i < cum && lane < kClasses));
            const uint32_t n = lane_value(pl.n, c), nq = lane_value(pl.nq, c), off = lane_value(pl.off, c);
            const uint32_t slot0 = lane_value(pl.slot0, c), first = lane_value(lo, c), last = lane_value(hi, c);
            const uint32_t at = i - (lane_value(cum, c) - lane_value(nb, c));
            s.spread = lane_value(spread ? 1u : 0u, c) != 0;
            const uint32_t f = first + (s.spread ? at : at * P + g);
            if (f < last) {
                const uint32_t q = f / n, k = f - q * n;
                const LongRow lr = w.long_list[(uint64_t)off + k];
                s.row = lr.row;
                s.begin = lr.begin;
                s.deg = lr.deg;
                if (nq > 1) s.slot = (int32_t)(slot0 + k * nq + q);
                s.q = s.spread ? q * P + g : q;
            }
            s.nq = s.spread ? nq * P : nq;
        } else {
            const int64_t pos = (int64_t)(l0 + i) * P + g;
            if (pos < w.N) {
                if (sorted) {
                    const LightRow lr = w.light_list[pos];
                    s.row = lr.row;
                    s.begin = lr.begin;
                    s.deg = w.light_deg[pos];
                } else {
                    s.row = (int32_t)pos;
                    const int64_t b = w.rowptr[pos];
                    s.begin = (uint32_t)b;
                    s.deg = (uint32_t)(w.rowptr[pos + 1] - b);
                }
            }
        }
        return s;
    };
    // the segment's entries, once its list entry is there: those of its piece
    auto settle = [&](Seg& s) {
        if (long_rows) {
            if (s.nq > 1) {
                const uint32_t len = s.deg / s.nq, more = s.deg - len * s.nq;
                s.begin += s.q * len + min(s.q, more);
                s.deg = len + (s.q < more ? 1u : 0u);
            }
        } else if (sorted) {
            if (s.row >= 0 && s.deg == kDegMany) s.deg = (uint32_t)(w.rowptr[(int64_t)s.row + 1] - s.begin);
        } else if (s.deg > (uint32_t)w.light_max) {
            s.row = -1;  // a long row
        }
        if (s.row < 0) s.deg = 0;
    };
    auto load_tile = [&](uint32_t tb, uint32_t te, int32_t (&v)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t pos = tb + r * G + lig;
            v[r] = w.colidx[pos < te ? pos : te - 1];
        }
    };

    Seg s = fetch(it), ahead = fetch(it + waves);
    settle(s);
    int32_t idx[R] = {};  // first tile of the segment
    if (s.deg) load_tile(s.begin, s.begin + s.deg, idx);
    while (it < total) {
        const Seg cs = s;
        int32_t tv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) tv[r] = idx[r];
        it += waves;
        s = ahead;
        ahead = fetch(it + waves);
        bool fetched = false;
        typename Op::State st;
        st.reset();
        if (cs.row >= 0) {
            st.begin(op, cs.row, lig);
            const uint32_t te = cs.begin + cs.deg;
            for (uint32_t tb = cs.begin; tb < te; tb += TE) {
                wave_lds_fence();
#pragma unroll
                for (int r = 0; r < R; ++r) gtile[r * G + lig] = tv[r];
                wave_lds_fence();
                if (tb + TE < te) load_tile(tb + TE, te, tv);
                const int nt = (int)(te - tb < TE ? te - tb : TE);
                for (int t = 0; t < nt; t += U) {
                    int32_t j[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) j[u] = gtile[t + u];
                    typename Op::State::Batch bt;
                    st.issue(op, j, lig, bt);
                    if (!fetched) {  // the next segment's first tile, behind this batch
                        settle(s);
                        if (s.deg) load_tile(s.begin, s.begin + s.deg, idx);
                        fetched = true;
                    }
                    st.consume(op, bt, j, nt - t < U ? nt - t : U);
                }
            }
        }
        if (!fetched) {
            settle(s);
            if (s.deg) load_tile(s.begin, s.begin + s.deg, idx);
        }
        bool write = cs.row >= 0;
        if (cs.spread) {
#pragma unroll
            for (int off = G; off < kWave; off <<= 1) st.merge_xor(off);
            write = write && g == 0;
        }
        if (write) {
            if (cs.slot < 0)
                st.store_out(op, cs.row, lig);
            else
                st.store_partial(op, cs.slot, lig);
        }
    }
}

// Rows that are cut, for the merge kernels: the i-th of them (in class order)
// and the place of its partial states.
struct CutRows {
    ClassPlan pl;
    uint32_t cum;  // cut rows up to and with this lane's class
    __device__ __forceinline__ CutRows(const RowWork& w, int lane) : pl(class_plan(w, lane)) {
        cum = scan32(pl.nq > 1 ? pl.n : 0u);
    }
    __device__ __forceinline__ uint32_t count() const { return lane_value(cum, kClasses - 1); }
    __device__ __forceinline__ int32_t row(const RowWork& w, uint32_t i, int lane, uint32_t& slot, uint32_t& nq) const {
        const int c = __builtin_ctzll(__ballot(i < cum && lane < kClasses));
        nq = lane_value(pl.nq, c);
        const uint32_t k = i - (lane_value(cum, c) - lane_value(pl.n, c));
        slot = lane_value(pl.slot0, c) + k * nq;
        return w.long_list[(uint64_t)lane_value(pl.off, c) + k].row;
    }
};

// ------------------------------------------------------------ the partition

struct SortParams {
    RowWork w;
    int32_t step = 1;      // entries per step of the light rows (their step classes)
    uint32_t groups = 1;  // lane groups per wavefront
    // Dense-tile windows (win_flags != nullptr): aligned 64-row windows whose
    // rows of at most tile_max entries are estimated to hold >= tile_min of them
    // inside the window are flagged for the tile kernel, and those rows left out
    // of the light-row order.  The estimate reads one entry of every 8th of them.
    uint8_t* win_flags = nullptr;  // [ceil(N / 64)]
    int32_t tile_min = 0;
    int32_t tile_max = 0;  // <= kWinMaxDeg and light_max
    // the workspace's other counter set, zeroed by block 0 for the next call
    // that takes this workspace (nullptr: none)
    int32_t* zero_next = nullptr;
};

// Degree binning.  A block owns RPT * 256 contiguous rows; thread t takes rows
// t, t+256, ... of the block, so every rowptr load is coalesced.  Long rows are
// counted by class and light rows by step count with LDS atomics (their return
// value is the row's place); one global atomic per class of a block reserves its
// part of the class list, from as many lanes at once.
//
// Light rows go out in descending step count (a counting sort in LDS), so the
// lane groups of a wave take rows of similar length and a wave does not wait on
// one long row among short ones: the degree bucketing of the degree-aware
// mapping (Appendix B.1), applied to the rows that share a wavefront.  The order
// within a class is arbitrary; every row is computed on its own, so the results
// do not depend on it.  Positions after the block's light rows hold -1.
template <int RPT>
__global__ void __launch_bounds__(kBlock) gt_sort_rows_kernel(SortParams p) {
    constexpr int kRows = kBlock * RPT;
    __shared__ uint32_t long_cnt[kClasses], long_base[kClasses];
    __shared__ uint32_t step_cnt[kClasses], step_base[kClasses];
    __shared__ int win_dense[RPT][kWavesPerBlock];  // dense-tile window flags of this block
    const RowWork& w = p.w;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    if (p.zero_next && blockIdx.x == 0)
        for (int i = threadIdx.x; i < kRowsSetWords; i += kBlock) p.zero_next[i] = 0;
    if (threadIdx.x < kClasses) {
        long_cnt[threadIdx.x] = 0;
        step_cnt[threadIdx.x] = 0;
    }
    int64_t rb[RPT], deg[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int64_t r = r0 + k * kBlock + threadIdx.x;
        rb[k] = 0;
        deg[k] = -1;  // past the last row
        if (r < w.N) {
            rb[k] = w.rowptr[r];
            deg[k] = w.rowptr[r + 1] - rb[k];
        }
    }
    // Dense-tile windows.  In iteration k, wave wv holds the 64 rows of one
    // aligned window (r0 is a multiple of 1024).  The window's rows of at most
    // tile_max entries hold ld of them; every 8th such row contributes its middle
    // entry as a sample, and the in-window share of the sampled rows' entries
    // (self-loops not counted) estimates the window's in-window entries (the tile
    // kernel counts them exactly and still streams a window that falls short).  A
    // dense window's rows of at most tile_max entries belong to the tile kernel
    // (tiled), all others stay on this path.
    bool tiled[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) tiled[k] = false;
    if (p.win_flags) {
        int32_t smp[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            smp[k] = -1;
            if (deg[k] > 0 && deg[k] <= p.tile_max && (lane & 7) == 0) smp[k] = w.colidx[rb[k] + deg[k] / 2];
        }
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int64_t r = r0 + k * kBlock + threadIdx.x;
            const bool lt = deg[k] >= 0 && deg[k] <= p.tile_max;
            // these degrees are <= 64, so a window's sums fit: ld <= 4096 and
            // the sampled sums (8 rows) <= 512, packed two to a word
            const int ld = wave_sum_i32(lt ? (int)deg[k] : 0);
            // a sampled self-loop does not count: every row has at most one,
            // and rows holding only their self-loop would make sparse windows
            // look dense
            const int sd = smp[k] >= 0 ? (int)deg[k] : 0;
            const int si = (smp[k] >= 0 && smp[k] != r && ((int64_t)smp[k] >> 6) == (r >> 6)) ? sd : 0;
            const int ss = wave_sum_i32(sd | (si << 16));
            const int sd_w = ss & 0xFFFF, si_w = ss >> 16;
            const bool dense = p.tile_min <= 1 ? ld > 0
                                               : (ld >= p.tile_min && si_w > 0 &&
                                                  (int64_t)si_w * ld >= (int64_t)p.tile_min * sd_w);
            tiled[k] = dense && lt;
            const int64_t win = (r0 + k * kBlock + wv * kWave) >> 6;
            if (lane == 0) {
                const bool exists = win * kWave < w.N;
                if (exists) p.win_flags[win] = dense ? 1 : 0;
                win_dense[k][wv] = !exists ? 2 : dense ? 1 : 0;  // 2: past the last row
            }
        }
    }
    __syncthreads();  // counts at zero
    int cls[RPT];       // class of a long row, -1 - step class of a light one, kClasses: neither
    uint32_t place[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        cls[k] = kClasses;
        if (deg[k] > w.light_max) {
            cls[k] = 63 - __builtin_clzll((uint64_t)deg[k]);
            cls[k] = cls[k] < kClasses - 1 ? cls[k] : kClasses - 1;
            place[k] = atomicAdd(&long_cnt[cls[k]], 1u);
        } else if (w.light_list && deg[k] >= 0 && !tiled[k]) {
            const int64_t st = (deg[k] + p.step - 1) / p.step;
            const int sc = (int)(st < kClasses - 1 ? st : kClasses - 1);
            cls[k] = -1 - sc;
            place[k] = atomicAdd(&step_cnt[sc], 1u);
        }
    }
    __syncthreads();
    // the block's reservations, and flags with plain stores
    if (wv == 0) {
        const int c = kClasses - 1 - lane;
        const uint32_t cap = lane < kClasses ? class_capacity(w, c) : 0u;
        const uint32_t off = scan32(cap) - cap;
        const uint32_t n = lane < kClasses ? long_cnt[c] : 0u;
        if (n) {
            const uint32_t base = (uint32_t)atomicAdd(&ROWS_CNT(w.counters, c), (int32_t)n);
            const bool fits = (uint64_t)base + n <= cap;
            if (!fits) atomicOr(&ROWS_CNT(w.counters, ROWS_OVERFLOW), 1);
            long_base[c] = fits ? off + base : ~0u;
        }
        const uint32_t groups = scan32(n ? (uint32_t)class_groups(w, c, n, p.groups) : 0u);
        if (lane == kClasses - 1 && groups) atomicAdd(&ROWS_CNT(w.counters, ROWS_PIECES), (int32_t)groups);
    } else if (wv == 1) {
        const int c = kClasses - 1 - lane;
        const uint32_t n = lane < kClasses ? step_cnt[c] : 0u;
        const uint32_t upto = scan32(n);
        if (lane < kClasses) step_base[c] = upto - n;
        // light rows left in the order: none lets the row kernel skip them
        // (every light row in dense windows)
        if (w.light_list && lane == kClasses - 1 && upto > 0) ROWS_CNT(w.counters, ROWS_LIGHT) = 1;
    } else if (wv == 2 && p.win_flags && lane < 2) {
        const int want = lane == 0 ? 1 : 0;  // lane 0: a dense window; lane 1: a sparse one
        bool seen = false;
        for (int k = 0; k < RPT; ++k)
            for (int v = 0; v < kWavesPerBlock; ++v) seen |= win_dense[k][v] == want;
        if (seen) reinterpret_cast<uint8_t*>(&ROWS_CNT(w.counters, ROWS_WIN))[lane] = 1;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int32_t r = (int32_t)(r0 + k * kBlock + threadIdx.x);
        if (cls[k] < 0) {
            const int64_t at = r0 + step_base[-1 - cls[k]] + place[k];
            w.light_list[at] = LightRow{r, (uint32_t)rb[k]};
            w.light_deg[at] = (uint8_t)(deg[k] < kDegMany ? deg[k] : kDegMany);
        } else if (cls[k] < kClasses && long_base[cls[k]] != ~0u)
            w.long_list[(uint64_t)long_base[cls[k]] + place[k]] = LongRow{r, (uint32_t)rb[k], (uint32_t)deg[k], 0u};
    }
    if (w.light_list) {
        // (class 0 is the last in the order)
        const int64_t n_light = (int64_t)step_base[0] + step_cnt[0];
        const int64_t rows_here = (w.N - r0 < kRows) ? w.N - r0 : kRows;
        for (int64_t j = n_light + threadIdx.x; j < rows_here; j += kBlock) w.light_list[r0 + j] = LightRow{-1, 0u};
    }
}

// Large graphs take 2048 rows per block, smaller ones 1024, giving more blocks
// in parallel.
hipError_t launch_sort_rows(const SortParams& sp, hipStream_t stream) {
    if (sp.w.N <= (int64_t(1) << 19)) {
        const int grid = (int)((sp.w.N + 4 * kBlock - 1) / (4 * kBlock));
        hipLaunchKernelGGL(gt_sort_rows_kernel<4>, dim3(grid), dim3(kBlock), 0, stream, sp);
    } else {
        const int grid = (int)((sp.w.N + 8 * kBlock - 1) / (8 * kBlock));
        hipLaunchKernelGGL(gt_sort_rows_kernel<8>, dim3(grid), dim3(kBlock), 0, stream, sp);
    }
    return hipGetLastError();
}
