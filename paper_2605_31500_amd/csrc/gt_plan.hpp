// How a call's rows are cut and how much of the device and of memory its row
// kernels take: arithmetic only, the same on the host and on the device (included
// by gt_attn.hip inside its anonymous namespace; a test compiles it for the CPU).
// gt_rows.hpp says why rows are cut.

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kXcds = 8;
constexpr int kWinMaxDeg = 64;  // the tile path's rows have at most this degree
constexpr int kDefaultTileMin = 256;
constexpr size_t kScratchBytes = size_t(256) << 20;  // array of the allocation-free entry point

constexpr int kClasses = 32;  // degree octaves

// How the rows of a call are cut.  A row of degree d <= light_max is one segment;
// longer rows are listed by degree octave (class c: 2^c <= d < 2^(c+1)), and all
// rows of a class are cut into the same number of pieces.
struct RowCut {
    int64_t N;
    uint32_t E;
    int32_t light_max;
    int32_t min_class;   // class of light_max + 1
    uint32_t split_min;  // classes whose shortest row has this many entries are cut
    uint32_t chunk;      // entries of a piece at most (unless nq_max or nq_floor says otherwise)
    uint32_t nq_floor, nq_max;
    uint32_t group_len;  // longest piece that one lane group reads
    uint32_t cap_slots;  // partial states there is room for
};

// Rows that class c can hold: their degrees are at least 2^c.
__host__ __device__ inline uint32_t class_capacity(const RowCut& w, int c) {
    if (c < w.min_class || c >= kClasses - 1) return 0;
    return (int64_t)(w.E >> c) < w.N ? w.E >> c : (uint32_t)w.N;
}

// Pieces of a row of class c, where there is room for their partial states.
__host__ __device__ inline uint32_t class_pieces(const RowCut& w, int c) {
    if ((1u << c) < w.split_min) return 1;
    const uint32_t nq = (2u << c) / w.chunk > w.nq_floor ? (2u << c) / w.chunk : w.nq_floor;
    return nq < w.nq_max ? nq : w.nq_max;
}

// Whether pieces of class c are too long for one lane group.
__host__ __device__ inline bool class_spread(const RowCut& w, int c, uint32_t nq) {
    return (uint32_t)((uint64_t(2) << c) / nq) > w.group_len;
}

// Pieces of each of n rows, nq of them or half as many until their partial states
// fit the `left` ones.
__host__ __device__ inline uint32_t fit_pieces(uint32_t n, uint32_t nq, uint32_t left) {
    while (nq > 1 && (uint64_t)n * nq > left) nq >>= 1;
    return nq;
}

// Pieces [lo, hi) of a class's n * nq that XCD xcd takes (piece number major).
__host__ __device__ inline uint32_t piece_share(uint64_t pieces, uint32_t xcd) {
    return (uint32_t)(pieces * xcd / kXcds);
}

// A wavefront's batches of `pieces` pieces: one each if they are spread over its P
// lane groups, else P at a time.
__host__ __device__ inline uint32_t piece_batches(uint32_t pieces, bool spread, uint32_t P) {
    return spread ? pieces : (pieces + P - 1) / P;
}

// Lane groups that n rows of class c ask for, P per wavefront, at most: fit_pieces
// may halve the pieces, and then they may get too long for one lane group.  (Over a
// graph fewer than 2^31: a lane group more than a row's first reads two entries or
// more.)
__host__ __device__ inline uint64_t class_groups(const RowCut& w, int c, uint32_t n, uint32_t P) {
    const uint32_t nq = class_pieces(w, c);
    uint32_t q = nq;
    while (q > 1 && !class_spread(w, c, q)) q >>= 1;
    const uint32_t most = class_spread(w, c, q) ? q * P : q;
    return (uint64_t)n * (most > nq ? most : nq);
}

// Batches of an XCD at most, if all classes together ask for `groups` lane groups
// (each class rounds up to a batch).
__host__ __device__ inline uint32_t batch_bound(uint32_t groups, uint32_t P) {
    return groups / (kXcds * P) + kClasses;
}

// A long row in its class list (entry positions fit 32 bits: E < 2^31).
struct LongRow {
    int32_t row;
    uint32_t begin;
    uint32_t deg;
    uint32_t pad;
};

struct LightRow {
    int32_t row;
    uint32_t begin;
};

// Work-list counters, cleared by a fill kernel or by an earlier call's
// partition.  Each sits on its own 128-byte line so that atomics on different
// counters do not serialise on one cache line.
//   0 .. 31: rows of each class;
//   ROWS_OVERFLOW: set if a list capacity was exceeded (the CSR precondition was
//     violated; the excess rows are dropped);
//   ROWS_LIGHT: nonzero if the light-row order holds any row;
//   ROWS_PIECES: lane groups that the long rows ask for, or more (a bound, by
//     which a wave without long work ends after one load);
//   ROWS_WIN: byte 0 nonzero if some window was found dense, byte 1 if some
//     window was not (byte flags written with plain stores, read as one word).
enum { ROWS_OVERFLOW = kClasses, ROWS_LIGHT, ROWS_WIN, ROWS_PIECES, ROWS_COUNT };
constexpr int kRowsStride = 32;                         // ints between counters
constexpr int kRowsSetWords = ROWS_COUNT * kRowsStride;  // one counter set

// RowCut, before the room for partial states is known.
struct RowRule {
    int32_t light_max;
    uint32_t split_min, chunk, nq_floor, nq_max, group_len;
    int64_t max_slots;     // partial states at most, over all graphs of this size
    int64_t likely_slots;  // enough for most of them
    bool forced;        // chunk length given by the caller
};

// Which rows are cut, and into how many pieces.  Rows of up to light_max entries
// are read by one lane group; longer ones by a wavefront, or, in classes from
// split_min on, in eight pieces: on eight XCDs at once, each of which reads its
// eighth of the sources.  Pieces are of about 64 entries from 512 on (1024 where
// the call's gathers take more than about 60 us), up to 32 of them; beyond that a
// wavefront reads a piece, since every piece has to be merged.  A piece costs
// `piece_bytes` of traffic (its partial state, written and read once, row vectors,
// list entry and index line) and a chain of its own, an entry `gather_bytes`.
//   * 64, cut from 128 where a piece is cheap beside two of its entries' gathers,
//     else from 256 (from 128 / 256 on, us per call: R-MAT scale 21 fp32 4x32 4605 /
//     4962; minimum of 64 bf16 features, lognormal 518 K nodes 398 / 376; GATv2
//     bf16 4x64, R-MAT 119 K nodes 179 / 168).  Light rows of up to 128 and 256
//     entries: 4605 and 4710 on the first.
//   * Wavefronts of one or two lane groups: no longer rows than 32 entries per
//     piece and group.
//   * Where the mean degree passes 32, a usual row may be above 64; the light
//     bound then goes up with it, so that not every row is cut or takes a
//     wavefront (light bound 64 and cut from 128 / as here: 12 K nodes of degree 71,
//     minimum of 256 fp32 features 74 / 64; 20 K of 150, fp32 4x32 198 / 173, GATv2
//     bf16 4x64 239 / 145.  Every row from 33 entries on in eight pieces, as was
//     done: 128, 205, 225).
//   * Mean degrees above 170: cut from 128, or from 512 where an L2 holds the
//     sources anyway and the rows fill the device (4000 nodes of degree 290, fp32
//     4x32, from 128 / 512: 72 / 57; 60 K of 201, from 128 / light to 256: 968 / 1250).
//   * The backward of vast graphs, whose pieces cost most: 128 (R-MAT scale 20 bf16
//     4x32, light bound 64 / 128: 2781 / 2720).
// At most 16 / 32 / 64 / 256 pieces: power law of 16 K nodes 41.1 / 37.9 / 39.4 /
// 41.7, R-MAT scale 21 4716 / 4683 / 4693 / 4793, backward of R-MAT scale 20 bf16
// 4x32 2720 / 2735 / 2736 / 3023.
RowRule row_rule(int64_t N, int64_t E, int slices, int gather_bytes, int piece_bytes, int groups, const gt_tuning* tu) {
    constexpr double kL2Bytes = 4.0 * 1024 * 1024, kGatherBytesPerSecond = 7.0e12;
    const double mean = (double)E / (double)N, sources = (double)N * gather_bytes;
    const bool cheap = piece_bytes <= 2 * gather_bytes, vast = sources > 64 * kL2Bytes;
    RowRule r;
    r.light_max = 64;
    r.split_min = cheap ? 128 : 256;
    if (groups <= 2) {
        r.light_max = groups == 2 ? 128 : 256;
        r.split_min = r.light_max;
    } else if (mean > 32 && mean <= 170) {
        while (r.light_max < 1.2 * mean) r.light_max *= 2;
        if (r.split_min < 2 * (uint32_t)r.light_max) r.split_min = 2 * r.light_max;
    } else if (mean > 170) {
        r.split_min = sources <= kL2Bytes && N * slices >= 4096 ? 512 : 128;
    } else if (!cheap && vast && piece_bytes > 1024) {
        r.light_max = 128;
    }
    // (eight pieces of two entries at the least)
    if (tu && tu->heavy_min_deg > 0) r.split_min = tu->heavy_min_deg > 16 ? tu->heavy_min_deg : 16;
    const bool large = (double)E * slices * gather_bytes / kGatherBytesPerSecond > 60e-6;
    r.chunk = large ? 128 : 64;
    r.nq_floor = kXcds;
    r.nq_max = 32;
    r.group_len = r.chunk;
    r.forced = false;
    const int64_t eights = kXcds * (E / r.split_min), more = 2 * (E / r.chunk);
    r.max_slots = (eights > more ? eights : more) + 1;
    r.likely_slots = mean >= r.split_min ? kXcds * N : r.max_slots / 8;
    if (tu && tu->light_max_deg > 0) r.light_max = tu->light_max_deg;
    if (tu && tu->chunk_edges > 0) {
        r.forced = true;
        r.chunk = ((uint32_t)tu->chunk_edges + kWave - 1) / kWave * kWave;
        r.split_min = r.chunk + 1;
        if (tu->heavy_min_deg > 0 && (uint32_t)tu->heavy_min_deg > r.split_min) r.split_min = (uint32_t)tu->heavy_min_deg;
        r.nq_floor = 1;
        r.nq_max = 32;
        r.max_slots = 2 * (E / r.chunk) + 1;
    }
    return r;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int floor_log2(uint64_t x) { return 63 - __builtin_clzll(x); }

// Entries of the class lists together: class_capacity over the classes.
uint64_t long_list_rows(int64_t N, int64_t E, int32_t light_max) {
    uint64_t n = 0;
    for (int c = floor_log2((uint64_t)light_max + 1); c < kClasses - 1; ++c) n += (uint64_t)((E >> c) < N ? (E >> c) : N);
    return n;
}

void set_rule(RowCut& w, const RowRule& r) {
    w.light_max = r.light_max;
    w.min_class = floor_log2((uint64_t)r.light_max + 1);
    w.split_min = r.split_min;
    w.chunk = r.chunk;
    w.nq_floor = r.nq_floor;
    w.nq_max = r.nq_max;
    w.group_len = r.group_len;
}

// Partial states and slices per launch.  Where the states of all slices fit
// kSlicesTogether bytes, the slices share a launch (and a merge); larger calls
// launch one slice at a time, which reuses the states' memory.
struct SlotPlan {
    uint32_t cap;
    int slices;  // per launch
};
constexpr size_t kSlicesTogether = size_t(192) << 20;
constexpr size_t kStatesLeast = size_t(128) << 20;    // of calls with a workspace of their own
constexpr size_t kBoundedStates = size_t(24) << 20;  // of calls that fit the allocation-free entry point

// `bounded`: the call's workspace has to fit the allocation-free entry point's
// array.  The states of the others may fill up a workspace of that size too, and
// get kStatesLeast however much its lists and statistics take: the longest rows
// come first, and so many of them keep the device busy (R-MAT scale 20 bf16 4x32
// backward, all classes in full: 224 MiB).
SlotPlan slot_plan(const RowRule& r, int slices, size_t slot_bytes, size_t other_bytes, bool bounded) {
    SlotPlan s;
    s.slices = slices;
    s.cap = (uint32_t)r.max_slots;
    const size_t left = other_bytes + 1024 < kScratchBytes ? kScratchBytes - other_bytes - 1024 : 0;
    const size_t room = (bounded || left > kStatesLeast ? left : kStatesLeast) / slot_bytes;
    const size_t all = kSlicesTogether / (slot_bytes * slices);
    if (!r.forced) {
        // (where they are not enough, rows are cut into fewer pieces)
        if (all >= (size_t)r.likely_slots)
            s.cap = (uint32_t)(all < (size_t)r.max_slots ? all : (size_t)r.max_slots);
        else
            s.slices = 1;
    }
    if ((!r.forced || bounded) && s.cap > room / s.slices) s.cap = (uint32_t)(room / s.slices);
    return s;
}

// Workgroups of a merge kernel for one slice: one wavefront per cut row if rows
// have eight pieces (two, where the caller gives their length), up to eight
// workgroups per CU.
int merge_blocks(const SlotPlan& sp, const RowRule& r, int cus) {
    const int64_t cut_rows = (int64_t)sp.cap / (r.forced ? 2 : kXcds) + 1;
    const int64_t g = (cut_rows + kWavesPerBlock - 1) / kWavesPerBlock;
    return (int)(g < cus * 8 ? g : cus * 8);
}

// Workgroups of a row kernel for one of the `slices` of a launch.  Light rows: one
// batch (a row per lane group) per wave while that is at most four times the
// workgroups that the device holds at once, two beyond (four where the tile path
// may take the rows): many more waves than it holds, so that the hardware scheduler
// evens out the per-wave work, but where they are few a second batch only makes
// the chain longer (one / two batches, us per call: 30 K nodes of degree 26 bf16
// 1x32 25 / 39, 12 K of degree 40 fp32 8x64 100 / 144; 286 K R-MAT nodes GATv2 fp32
// 8x32 498 / 469; 1, 2, 4 and 8 on R-MAT scale 21 fp32 4x32 5080, 5110, 5330, 5770).
// Long rows: a wave per 128 entries if three quarters of all lie in them, up to
// eight times what the device holds (a wave without a batch still costs its
// prologue; a wave per 64 entries of each lane group left rows of 65 to 255
// entries, a wavefront each, queueing up: 16 K nodes of a power law bf16 1x64 31.8
// -> 26.6, R-MAT of 16 K nodes fp32 4x32 37.4 -> 32.9).  They come first, since
// theirs is the longest chain; but on graphs of 16 entries per row or more whose
// workgroups all but fit the device they come last, where they cost next to
// nothing if no row is long (long rows first / last: 3000 nodes of degree 99, fp32
// 4x32 30.4 / 24.3, GATv2 bf16 4x64 40.5 / 32.4; power law of 15 K nodes bf16 8x32
// 34.9 / 36.8).
constexpr uint32_t kMostBlocks = 1u << 23;  // (a launch holds fewer than 2^32 threads)
struct RowGrid {
    uint32_t blocks, long_blocks;
    bool light_first;
};
RowGrid row_grid(int64_t N, int64_t E, int groups, int slices, bool tiles, int resident, const gt_tuning* tu) {
    auto blocks = [](int64_t batches, int64_t per_wave) {
        const int64_t g = (batches + per_wave * kWavesPerBlock - 1) / (per_wave * kWavesPerBlock);
        return (uint32_t)((g + kXcds - 1) / kXcds * kXcds);
    };
    RowGrid rg;
    const int64_t batches = (N + groups - 1) / groups;
    const bool few = (int64_t)blocks(batches, 1) * slices <= 4 * (int64_t)resident;
    rg.long_blocks = blocks(3 * (E / 4) / (groups < 2 ? 64 : 128) + 1, 1);
    const uint32_t most = (uint32_t)(tiles ? 2 : 8) * (uint32_t)resident / kXcds * kXcds;
    if (rg.long_blocks > most) rg.long_blocks = most;
    rg.blocks = rg.long_blocks + blocks(batches, few ? 1 : tiles ? 4 : 2);
    if (rg.blocks > kMostBlocks) rg.blocks = kMostBlocks;
    rg.light_first = E >= 16 * N && (int64_t)rg.blocks * slices <= 4 * (int64_t)resident;
    if (tu && tu->grid_blocks > 0) {
        rg.long_blocks = blocks(((int64_t)tu->grid_blocks + 1) / 2 * kWavesPerBlock, 1);
        rg.blocks = 2 * rg.long_blocks;
    }
    return rg;
}

// Whether rows that are gathered once per entry (GATv2, the reduction) are worked on
// in slices of 1 KB instead of 256 bytes.  Each slice reads the row's list entry and
// indices again, and rows of a few entries have nothing for a second XCD to find in
// its L2: four slices of a 4 KB row cost less than sixteen there (256 bytes / 1 KB, us
// per call: GATv2 fp32 8x128, 60 K nodes of degree 4 216 / 201, R-MAT of 500 K of
// degree 5 2215 / 1690; minimum of 1024 fp32 features 241 / 219 and 2414 / 1920), but
// not from 7 entries on (300 K lognormal nodes, minimum: 1574 / 1640), on small
// graphs (8 K R-MAT nodes: 51 / 60; 33 K of a power law, 2048 bf16 features: 169 /
// 217) or of shorter rows (1 KB, power law of 60 K nodes: 78 / 98).
bool wide_slices(int64_t N, int64_t E, int64_t row_bytes) {
    return row_bytes >= 4096 && N >= 48 * 1024 && 2 * E < 11 * N;
}

// One call of the attention forward: its sizes and its row kernel.
struct AttnShape {
    int64_t N, E;
    int32_t H, D;
    int32_t elt_bytes;
    int32_t slice_heads;  // heads of a slice
    int32_t groups;       // lane groups per wavefront
    bool gat;             // GATv2: one gathered row per entry, no tile path
    bool sorted;          // the row kernel takes light rows in step order
};

// What the allocation-free entry point counts as a call's workspace, for its
// documented limit: two counter sets, a list of all rows (two where a wavefront
// holds four rows or more), the lists and partial states of rows of `heavy` entries
// or more cut into chunks (of `chunk` entries, by default half the steps that the
// call's gathers take at 7 TB/s and a microsecond per step, up to 1024 entries, or
// an eighth of them up to 8192) for all heads at once, and the windows of the tile
// path.  Calls within the limit get a workspace within it; the others are refused.
size_t noalloc_need(const AttnShape& a, bool tiles, const gt_tuning* tu) {
    const int row = a.H * a.D * a.elt_bytes, vecs = row / 16, lanes = vecs < kWave ? vecs : kWave;
    const int rows = kWave / lanes, nv = vecs / lanes;
    int u = 8 / nv > 2 ? 8 / nv : 2;
    if (u > lanes) u = lanes;
    const int64_t light = tu && tu->light_max_deg > 0 ? tu->light_max_deg : 8 * u;
    const double steps = (double)a.E * (2.0 * row) / 7.0e12 / 1.0e-6;
    const double entries = 0.5 * steps * (rows * (rows >= 4 && u >= 8 ? u / 2 : u));
    auto whole = [](double x) { return ((int64_t)x + kWave - 1) / kWave * kWave; };
    int64_t chunk = 0.25 * entries > 8192.0   ? 8192
                    : 0.25 * entries > 1024.0 ? whole(0.25 * entries)
                    : entries >= 1024.0       ? 1024
                                              : whole(entries);
    if (chunk < kWave) chunk = kWave;
    int64_t heavy = rows >= 2 && chunk / 4 > 256 ? chunk / 4 : 256;
    if (tu && tu->heavy_min_deg > 0) heavy = tu->heavy_min_deg;
    if (tu && tu->chunk_edges > 0) chunk = whole(tu->chunk_edges);
    if (heavy <= light) heavy = light + 1;
    const size_t slots = 2 * (size_t)(a.E / chunk) + 1;
    const size_t parts[] = {3584,
                            (size_t)a.N * 4,
                            16 * ((size_t)(a.E / (chunk + 1)) + 1),
                            24 * ((size_t)(a.E / heavy) + slots),
                            slots * a.H * 8,
                            slots * a.H * a.D * 4,
                            rows >= 4 ? (size_t)a.N * 4 : 0,
                            tiles ? (size_t)(a.N + kWave - 1) / kWave : 0};
    size_t need = 0;
    for (const size_t bytes : parts) need = align_up(need + bytes, 256);
    return need;
}

// Rows, partial states and workspace of a call of the attention forward:
// counters | light rows | window flags | long rows | partial (m,l) | partial acc.
// The allocation-free entry point and the others get the same rows in the same
// pieces, and so the same bits, wherever the former takes the call.
struct AttnPlan {
    size_t need;  // noalloc_need
    RowRule rule;
    SlotPlan slots;
    bool tiles;   // the tile path takes light rows of dense windows
    bool sorted;  // light rows in step order
    int tile_min;
    int32_t tile_max;  // the tile path's rows have at most this degree; other light rows stay with the row kernel
    size_t o_light, o_deg, o_win, o_long, o_ml, o_acc, bytes;
};

AttnPlan plan_attn(const AttnShape& a, const gt_tuning* tu, bool noalloc) {
    const int slice_bytes = a.slice_heads * a.D * a.elt_bytes, slices = a.H / a.slice_heads;
    const int slot_bytes = a.slice_heads * (a.D * 4 + 8);
    AttnPlan p;
    p.rule = row_rule(a.N, a.E, slices, (a.gat ? 1 : 2) * slice_bytes, 3 * (2 * slot_bytes + 256) / 4, a.groups, tu);
    // Dense-tile windows (bf16 rows of at most 256 bytes): on by default, for
    // windows estimated to hold at least 256 in-window entries, which a 64-row
    // block at half density holds about eight times over (measured on the SBM
    // workload; on the R-MAT one no window qualifies and the tile kernel
    // finds an empty list).
    p.tile_min = tu && tu->dense_tiles != 0 ? tu->dense_tiles : kDefaultTileMin;  // < 0: off
    const bool tile_rows = !a.gat && a.elt_bytes == 2 && a.H * a.D <= 128, tile_call = tile_rows && p.tile_min > 0;
    // (the same light rows with the path off: a row that it streams has the same
    // bits then)
    if (tile_rows && !(tu && tu->light_max_deg > 0)) p.rule.light_max = kWinMaxDeg;

    p.need = noalloc_need(a, tile_call, tu);
    const bool bounded = !a.gat && p.need <= kScratchBytes;
    // Where the light rows' order would not fit the allocation-free entry point's
    // array (more than 26 million nodes), that entry point takes them in id order
    // (which changes no result) and neither has the tile path, which needs it.
    const bool fits = !bounded || (size_t)a.N * (sizeof(LightRow) + 1) <= kScratchBytes / 16 * 14;
    p.tiles = tile_call && fits;
    p.sorted = a.sorted && (!noalloc || fits);
    size_t off = align_up(2 * kRowsSetWords * sizeof(int32_t), 256);  // two counter sets
    auto place = [&off](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    if (p.sorted && fits) {
        p.o_light = place((size_t)a.N * sizeof(LightRow));
        p.o_deg = place((size_t)a.N);
    }
    p.o_win = place(p.tiles ? (size_t)(a.N + kWave - 1) / kWave : 0);
    // (a larger light bound makes the class lists shorter; the order above leaves
    // room for none and for kBoundedStates at the least)
    while (bounded && p.rule.light_max < INT32_MAX &&
           off + long_list_rows(a.N, a.E, p.rule.light_max) * sizeof(LongRow) + kBoundedStates > kScratchBytes)
        p.rule.light_max = p.rule.light_max < INT32_MAX / 2 ? 2 * p.rule.light_max + 1 : INT32_MAX;
    p.tile_max = p.rule.light_max < kWinMaxDeg ? p.rule.light_max : kWinMaxDeg;
    p.o_long = place((size_t)long_list_rows(a.N, a.E, p.rule.light_max) * sizeof(LongRow));
    p.slots = slot_plan(p.rule, slices, slot_bytes, off, bounded);
    const size_t slots = (size_t)p.slots.cap * p.slots.slices;
    p.o_ml = place(slots * a.slice_heads * 8);
    p.o_acc = place(slots * a.slice_heads * a.D * 4);
    if (!(p.sorted && fits)) {
        p.o_light = place(p.sorted ? (size_t)a.N * sizeof(LightRow) : 0);
        p.o_deg = place(p.sorted ? (size_t)a.N : 0);
    }
    p.bytes = off;
    return p;
}
