// Walk records and the walk kernel (Sections 2.1, 2.2.1 and 5.2).  Included by
// build.hip inside its anonymous namespace, after BLOCK and the schedule constants
// (NSLAB, NSEG) are defined.
#pragma once

// ----------------------------------------------------------------------- table
// Walk record of node v: 64-byte lines starting at line rline[v].  32-bit words of the
// first line: [0] rank, [1] degree | grounded flag, [2] node id, [3] the line of the
// record of the neighbour taken when the draw passes every threshold (the last one).
// Every off-diagonal entry m (CSR order) is a pair: the threshold floor(2^32 c_m / a_v)
// and the line of the neighbour's record.  Unused words of a record's lines are 0.
//   degree <= 6: the pairs sit in words 4 + 2m, 5 + 2m of the first line.  The record
//     is one line, so a walk step is one dependent 64-byte load: the next node's
//     record, whose header holds the rank for the home test and the node id to record
//     where the walk ends.
//   degree > 6: the pairs fill the following lines, eight per line (entry m at word
//     16 + 2m of the record); words 4 .. 15 of the first line hold the last threshold
//     of each of the first twelve of those lines.  Thresholds grow with m, so the
//     first line whose last threshold exceeds the draw holds the chosen entry: a step
//     loads that one line.
// Start record of v: the same layout, from line n_lines + rline[v], for the first step
// of v's walks, which moves to a higher-ranked neighbour only (the exact one-step part
// of Section 5.2): the thresholds are floor(2^32 cm_m / sum of the higher-ranked
// weights) over the cumulative higher-ranked weight cm_m, word 3 is the last
// higher-ranked neighbour's line and the grounded flag is clear.  The first step is
// then the same select-and-load as every other step.
//
// Bucket lines.  A node of degree 7..BUCKET_MAX_DEG whose draw range [0, 2^32) splits
// into B = 2^kb equal parts (kb = 3..6) that each meet at most six entries' threshold
// intervals also gets B bucket lines, placed before its first line: bucket line b
// holds the record's header and, in words 4..15 as in a narrow record, the entries
// (entry order, zero-width ones left out) whose intervals meet [b 2^(32-kb),
// (b+1) 2^(32-kb)).  The chosen entry of a draw in that range is among them, so the
// selection is the narrow one.  A walk that moves to such a node holds its next draw
// already (the walk kernel makes each block of eight draws one step ahead) and loads
// the bucket line of that draw: one dependent load per step instead of two.  The line
// words of entries (and word 3) carry the target's kb in their top bits when the
// records are bucketed (all walk lines below 2^LINE_KB_SHIFT; start records follow them, and
// a walk's start line is used as it is).  The first line and the
// continuation lines stay: a walk of the plain estimator starts from its row's own
// record.
//
// Near records.  Where every row has at most six neighbours and a matrix's entries lie
// on at most NEAR_DELTAS diagonals other than the main one (regular grids and stencils
// in their natural numbering, whatever their size), a record is half a line, 32 bytes:
// [0] rank | grounded << 31, [1..6] the thresholds (0xFFFFFFFF past the last entry), [7]
// codes: the neighbour's place in the matrix's list of diagonals, three of four bits
// for the entry 0, 1, ... (the last neighbour's from there on), the degree in bits 28..30.
// The chosen entry is the number of thresholds not above the draw; a record's index is
// its node.  Start records follow from index n on.  Half the bytes per step keep twice
// the nodes in the L2s (3D grid 128^3: walk kernel 136 -> 100 ms, L2 misses 3.9e9 ->
// 3.2e9).
constexpr int REC_WORDS = 16;
constexpr uint32_t LINE_KB_SHIFT = 27;
constexpr uint32_t LINE_MASK = (1u << LINE_KB_SHIFT) - 1u;
constexpr int64_t BUCKET_MAX_DEG = 64;
constexpr uint32_t DESC_INLINE = 0x40000000u;  // the line's pairs are in words 4..15

enum RecordFormat : int { REC_LINES = 0, REC_BUCKETS = 1, REC_NEAR = 2 };
constexpr int NEAR_WORDS = 8;
constexpr uint32_t NEAR_GROUNDED = 0x80000000u;
constexpr int NEAR_DELTAS = 8;         // diagonals of a matrix, at most
constexpr int NEAR_MATS = 256;         // matrices of a batch (their lists sit in LDS)
constexpr int32_t NO_DELTA = INT32_MIN;

// Adds d to a list of NEAR_DELTAS diagonals; false if it is full.
template <int SCOPE>
__device__ __forceinline__ bool near_insert(int32_t* list, int32_t d)
{
    for (int i = 0; i < NEAR_DELTAS; ++i) {
        int32_t have = __hip_atomic_load(list + i, __ATOMIC_RELAXED, SCOPE);
        if (have == NO_DELTA) have = (int32_t)atomicCAS((int*)list + i, NO_DELTA, d);
        if (have == d || have == NO_DELTA) return true;
    }
    return false;
}

// The diagonals j - v of every matrix's entries (delta [matrices][NEAR_DELTAS], NO_DELTA
// before the launch, in no particular order); *far |= 1 if a row has more than six
// neighbours or a matrix more than NEAR_DELTAS diagonals.  A workgroup (256 rows) first
// gathers the diagonals of its first row's matrix in LDS: a look at the one global list
// per entry took 5.9 ms of a build of the 128^3 grid, a look per workgroup takes it to
// 109.6 ms (115.9 before; 256 2D grids in a batch 76.3, 81.0 before).
__global__ __launch_bounds__(256) void k_near_deltas(int64_t n, const int64_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ col,
                                                     const int32_t* __restrict__ node_mat,
                                                     int32_t* delta, int32_t* far)
{
    __shared__ int32_t mine[NEAR_DELTAS];
    const int64_t v0 = (int64_t)blockIdx.x * blockDim.x, v = v0 + threadIdx.x;
    const int32_t mat0 = node_mat ? node_mat[v0] : 0;
    if (threadIdx.x < NEAR_DELTAS) mine[threadIdx.x] = NO_DELTA;
    __syncthreads();
    bool ok = true;
    if (v < n) {
        const int64_t r0 = rowptr[v], r1 = rowptr[v + 1];
        ok = r1 - r0 <= 7;
        const int32_t mat = node_mat ? node_mat[v] : 0;
        for (int64_t p = r0; ok && p < r1; ++p) {
            const int32_t d = col[p] - (int32_t)v;
            if (d == 0) continue;
            ok = mat == mat0 ? near_insert<__HIP_MEMORY_SCOPE_WORKGROUP>(mine, d)
                             : near_insert<__HIP_MEMORY_SCOPE_AGENT>(delta + (int64_t)mat * NEAR_DELTAS, d);
        }
    }
    __syncthreads();
    if (threadIdx.x < NEAR_DELTAS && mine[threadIdx.x] != NO_DELTA)
        ok = near_insert<__HIP_MEMORY_SCOPE_AGENT>(delta + (int64_t)mat0 * NEAR_DELTAS, mine[threadIdx.x]) && ok;
    if (!ok) atomicOr(far, 1);
}

// Most entries (of nonzero width) that meet one of the 2^kb draw ranges of node v.
__device__ uint32_t bucket_load(int64_t v, int64_t r0, int64_t r1, const int32_t* __restrict__ col,
                                const double* __restrict__ val, double a, uint32_t kb)
{
    const uint32_t sh = 32u - kb;
    uint32_t prev = 0u, cur = 0u, cnt = 0u, mx = 0u;
    double c = 0.0;
    for (int64_t p = r0; p < r1; ++p) {
        if (col[p] == v) continue;
        c = c + (-val[p]);
        const uint32_t thr = threshold32(c, a);
        if (thr > prev) {  // the entry's draws: [prev, thr)
            const uint32_t bl = prev >> sh, bh = (thr - 1u) >> sh;
            if (bl != cur) {
                mx = max(mx, cnt);
                cur = bl;
                cnt = 0u;
            }
            ++cnt;
            if (bh != bl) {
                mx = max(mx, cnt);
                cur = bh;
                cnt = 1u;
            }
        }
        prev = thr;
    }
    return max(mx, cnt);
}

// Lines per record and the bucket exponent kb of every node (0: no bucket lines);
// *any_bucket |= 1 if some node has bucket lines.
__global__ void k_rec_lines(int64_t n, const int64_t* __restrict__ rowptr,
                            const int32_t* __restrict__ col, const double* __restrict__ val,
                            int32_t bucketing, int32_t* __restrict__ lines, uint8_t* __restrict__ kbv,
                            int32_t* any_bucket)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int64_t r0 = rowptr[v], r1 = rowptr[v + 1];
    const int64_t deg = r1 - r0 - 1;
    uint32_t kb = 0u;
    if (bucketing && deg > 6 && deg <= BUCKET_MAX_DEG) {
        double a = 0.0;
        for (int64_t p = r0; p < r1; ++p)
            if (col[p] == v) a = val[p];
        for (uint32_t k = 3u; k <= 6u && kb == 0u; ++k)
            if (bucket_load(v, r0, r1, col, val, a, k) <= 6u) kb = k;
    }
    kbv[v] = (uint8_t)kb;
    if (kb) atomicOr(any_bucket, 1);
    lines[v] = (int32_t)((kb ? (1 << kb) : 0) + (deg <= 6 ? 1 : 1 + (deg + 7) / 8));
}

// a wide record's summary words: the last threshold of each of its first twelve
// continuation lines
__device__ __forceinline__ void wide_summary(uint32_t* rec, uint32_t m)
{
    const uint32_t L = (m + 7) / 8;
    for (uint32_t l = 1; l <= 12; ++l) {
        const uint32_t last = (l * 8 < m ? l * 8 : m) - 1;  // last entry of line l
        rec[3 + l] = l <= L ? rec[16 + 2 * last] : 0u;
    }
}

// the line word of an entry that moves to node j: its first record line, with its
// bucket exponent in the top bits when the records are bucketed
__device__ __forceinline__ uint32_t line_word(const int64_t* __restrict__ rline,
                                              const uint8_t* __restrict__ kbv, int32_t bucketing,
                                              int32_t j)
{
    return (uint32_t)rline[j] | (bucketing ? (uint32_t)kbv[j] << LINE_KB_SHIFT : 0u);
}

// Walks of row v: walking rows are those with a higher-ranked neighbour (the others are
// exact), or every row for the plain estimator.
__device__ __forceinline__ int32_t row_budget(bool walks, int64_t v, int32_t walks_per_row,
                                              const int32_t* __restrict__ budget_in,
                                              int32_t* max_budget)
{
    if (!walks || walks_per_row == NO_WALKS) return 0;
    const int32_t b = max(budget_in ? budget_in[v] : walks_per_row, 1);
    atomicMax(max_budget, b);
    return b;
}

__global__ void k_table(int64_t n, const int64_t* __restrict__ rowptr,
                        const int32_t* __restrict__ col, const double* __restrict__ val,
                        const int32_t* __restrict__ rank, const uint8_t* __restrict__ grounded,
                        int32_t walks_per_row, const int32_t* __restrict__ budget_in,
                        int32_t plain, const int64_t* __restrict__ rline,
                        const uint8_t* __restrict__ kbv, int32_t bucketing, int64_t n_lines,
                        uint32_t* __restrict__ recs, uint2* __restrict__ ent,
                        uint32_t* __restrict__ mthr, double* __restrict__ tau,
                        int32_t* __restrict__ budget, int32_t* max_budget)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int64_t r0 = rowptr[v], r1 = rowptr[v + 1];
    const int32_t rv = rank[v];
    double a = 0.0, motel = 0.0;
    for (int64_t p = r0; p < r1; ++p) {
        const int32_t j = col[p];
        if (j == v) a = val[p];
        else if (rank[j] > rv) motel = motel + (-val[p]);
    }
    const int64_t start = r0 - v;
    const uint32_t kb = kbv[v];
    const int64_t first = rline[v] + (kb ? (1 << kb) : 0);  // the first line, after the buckets
    uint32_t* rec = recs + (size_t)first * REC_WORDS;
    uint32_t* srec = recs + (size_t)(n_lines + first) * REC_WORDS;
    const uint32_t deg = (uint32_t)(r1 - r0 - 1);
    const bool wide = deg > 6;
    double c = 0.0, cm = 0.0;
    uint32_t m = 0, last_line = 0, last_motel_line = 0;
    for (int64_t p = r0; p < r1; ++p) {
        const int32_t j = col[p];
        if (j == v) continue;
        const double w = -val[p];
        c = c + w;
        const uint32_t line = line_word(rline, kbv, bucketing, j);
        if (rank[j] > rv) {
            cm = cm + w;
            last_motel_line = line;
        }
        const uint32_t thr = threshold32(c, a);
        const uint32_t mt = motel > 0.0 ? threshold32(cm, motel) : 0u;
        const uint32_t slot = wide ? 16 + 2 * m : 4 + 2 * m;
        rec[slot] = thr;
        rec[slot + 1] = line;
        srec[slot] = mt;
        srec[slot + 1] = line;
        if (ent) ent[start + m] = make_uint2((uint32_t)j, thr);
        if (mthr) mthr[start + m] = mt;
        last_line = line;
        ++m;
    }
    const uint32_t flags = grounded[v] ? DESC_GROUNDED : 0u;
    const uint32_t inl = wide ? 0u : DESC_INLINE;
    rec[0] = (uint32_t)rv;
    rec[1] = m | flags | inl;
    rec[2] = (uint32_t)v;
    rec[3] = last_line;
    srec[0] = (uint32_t)rv;
    srec[1] = m | inl;
    srec[2] = (uint32_t)v;
    srec[3] = last_motel_line;
    if (kb) {
        // bucket lines: the header, then the entries meeting each draw range in order
        const uint32_t B = 1u << kb, sh = 32u - kb;
        uint32_t* bl0 = recs + (size_t)rline[v] * REC_WORDS;
        for (uint32_t b = 0; b < B; ++b) {
            uint32_t* L = bl0 + (size_t)b * REC_WORDS;
            L[0] = (uint32_t)rv;
            L[1] = m | flags | DESC_INLINE;
            L[2] = (uint32_t)v;
            L[3] = last_line;
            for (int q = 4; q < REC_WORDS; ++q) L[q] = 0u;
        }
        uint32_t prev = 0u, cur = 0u, slot = 0u;
        double cc = 0.0;
        for (int64_t p = r0; p < r1; ++p) {
            const int32_t j = col[p];
            if (j == v) continue;
            cc = cc + (-val[p]);
            const uint32_t thr = threshold32(cc, a);
            if (thr > prev) {
                const uint32_t lw = line_word(rline, kbv, bucketing, j);
                for (uint32_t b = prev >> sh; b <= ((thr - 1u) >> sh); ++b) {
                    if (b != cur) {
                        cur = b;
                        slot = 0u;
                    }
                    uint32_t* L = bl0 + (size_t)b * REC_WORDS;
                    L[4 + 2 * slot] = thr;
                    L[5 + 2 * slot] = lw;
                    ++slot;
                }
            }
            prev = thr;
        }
    }
    if (wide) {
        wide_summary(rec, m);
        wide_summary(srec, m);
        for (uint32_t q = 16 + 2 * m; q % REC_WORDS != 0; ++q) {
            rec[q] = 0u;
            srec[q] = 0u;
        }
    } else {
        for (uint32_t q = 4 + 2 * m; q < REC_WORDS; ++q) {
            rec[q] = 0u;
            srec[q] = 0u;
        }
    }
    tau[v] = motel / a;
    budget[v] = row_budget(motel > 0.0 || plain, v, walks_per_row, budget_in, max_budget);
}

// The same for near records.
__global__ void k_table_near(int64_t n, const int64_t* __restrict__ rowptr,
                             const int32_t* __restrict__ col, const double* __restrict__ val,
                             const int32_t* __restrict__ rank, const uint8_t* __restrict__ grounded,
                             int32_t walks_per_row, const int32_t* __restrict__ budget_in,
                             int32_t plain, const int32_t* __restrict__ node_mat,
                             const int32_t* __restrict__ delta, uint4* __restrict__ recs,
                             uint2* __restrict__ ent, uint32_t* __restrict__ mthr,
                             double* __restrict__ tau, int32_t* __restrict__ budget,
                             int32_t* max_budget)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int64_t r0 = rowptr[v], r1 = rowptr[v + 1];
    const int32_t rv = rank[v];
    double a = 0.0, motel = 0.0;
    for (int64_t p = r0; p < r1; ++p) {
        const int32_t j = col[p];
        if (j == v) a = val[p];
        else if (rank[j] > rv) motel = motel + (-val[p]);
    }
    const int32_t* list = delta + (node_mat ? (int64_t)node_mat[v] * NEAR_DELTAS : 0);
    uint32_t t[6], mt[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) t[i] = mt[i] = 0xFFFFFFFFu;
    const int64_t start = r0 - v;
    double c = 0.0, cm = 0.0;
    uint32_t m = 0, codes = 0, last = 0, last_motel = 0;
    for (int64_t p = r0; p < r1; ++p) {
        const int32_t j = col[p];
        if (j == v) continue;
        const double w = -val[p];
        c = c + w;
        uint32_t code = 0;
        for (uint32_t i = 1; i < (uint32_t)NEAR_DELTAS; ++i)
            if (list[i] == j - (int32_t)v) code = i;
        if (rank[j] > rv) {
            cm = cm + w;
            last_motel = code;
        }
        const uint32_t thr = threshold32(c, a);
        const uint32_t mthr_m = motel > 0.0 ? threshold32(cm, motel) : 0u;
#pragma unroll
        for (uint32_t i = 0; i < 6; ++i)
            if (i == m) {
                t[i] = thr;
                mt[i] = mthr_m;
            }
        codes |= code << (4 * m);
        if (ent) ent[start + m] = make_uint2((uint32_t)j, thr);
        if (mthr) mthr[start + m] = mthr_m;
        last = code;
        ++m;
    }
    uint32_t mcodes = codes;
    for (uint32_t i = m; i < 7; ++i) {  // past every threshold: the last neighbour
        codes |= last << (4 * i);
        mcodes |= last_motel << (4 * i);
    }
    codes |= m << 28;
    mcodes |= m << 28;
    const uint32_t rw = (uint32_t)rv;
    uint4* rec = recs + (size_t)v * (NEAR_WORDS / 4);
    uint4* srec = recs + (size_t)(n + v) * (NEAR_WORDS / 4);
    rec[0] = make_uint4(rw | (grounded[v] ? NEAR_GROUNDED : 0u), t[0], t[1], t[2]);
    rec[1] = make_uint4(t[3], t[4], t[5], codes);
    srec[0] = make_uint4(rw, mt[0], mt[1], mt[2]);
    srec[1] = make_uint4(mt[3], mt[4], mt[5], mcodes);
    tau[v] = motel / a;
    budget[v] = row_budget(motel > 0.0 || plain, v, walks_per_row, budget_in, max_budget);
}

// ----------------------------------------------------------------------- walks
// Chunk: up to 64 walks of one row, everything a wave needs to start them.
struct ChunkDesc {
    uint32_t key;     // Philox key word of the row: its node id (in a batch, its id
                      // within its own matrix)
    uint32_t walks;   // first walk | count << 13 | matrix (near records of a batch) << 22
    uint32_t sline;   // the row's start record line
    uint32_t rank;    // the row's rank
    uint64_t rec;     // result index of the row's walk 0
    uint64_t seed;    // the seed of the row's matrix
};
static_assert(sizeof(ChunkDesc) == 32, "chunk descriptors are 32 bytes");
// a row has at most 8192 walks, a chunk at most CHUNK_WALKS <= 256 and a batch of near
// records at most NEAR_MATS matrices
constexpr int WALKS_FIRST_BITS = 13, WALKS_MAT_SHIFT = 22;
constexpr uint32_t WALKS_FIRST_MASK = (1u << WALKS_FIRST_BITS) - 1u, WALKS_COUNT_MASK = 0x1FFu;
static_assert(CHUNK_WALKS <= 256 && NEAR_MATS <= 1024, "chunk descriptor fields");

// chunk descriptors of the rows in schedule order: consecutive walks of a row, SRW_WAVE
// per chunk for the first nlong rows, CHUNK_WALKS for the others; a walk starts from
// the first line of the start record (sline_base: the start records) or, with
// sline_base 0, of the row's own record; near_n > 0: near records, n of them
__global__ void k_chunks(int64_t norder, int64_t nlong, const int32_t* __restrict__ order,
                         const int64_t* __restrict__ chunk_off, const int32_t* __restrict__ budget,
                         const int64_t* __restrict__ rline, const uint8_t* __restrict__ kbv,
                         int64_t sline_base, int64_t near_n,
                         const int32_t* __restrict__ rank, const int64_t* __restrict__ rec_off,
                         uint64_t seed, const int32_t* __restrict__ node_mat,
                         const int64_t* __restrict__ mat_off, const uint64_t* __restrict__ mat_seed,
                         ChunkDesc* __restrict__ cdesc)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= norder) return;
    const int32_t v = order[j];
    const int32_t b = budget[v];
    ChunkDesc d;
    d.key = (uint32_t)v;
    d.seed = seed;
    uint32_t mat = 0;
    if (node_mat) {
        const int32_t mi = node_mat[v];
        if (near_n > 0) mat = (uint32_t)mi;
        d.key = (uint32_t)(v - mat_off[mi]);
        d.seed = mat_seed[mi];
    }
    d.sline = near_n > 0 ? (uint32_t)(sline_base + v)
                         : (uint32_t)(sline_base + rline[v] + (kbv[v] ? (1 << kbv[v]) : 0));
    d.rank = (uint32_t)rank[v];
    d.rec = (uint64_t)rec_off[v];
    for (int64_t c = chunk_off[j]; c < chunk_off[j + 1]; ++c) {
        const uint32_t cs = j < nlong ? (uint32_t)SRW_WAVE : CHUNK_WALKS;
        const uint32_t w0 = (uint32_t)(c - chunk_off[j]) * cs;
        const uint32_t cnt = min(cs, (uint32_t)b - w0);
        d.walks = w0 | (cnt << WALKS_FIRST_BITS) | (mat << WALKS_MAT_SHIFT);
        cdesc[c] = d;
    }
}

struct WalkArgs {
    const uint4* recs;         // walk and start records, 4 x 16 bytes per line
    uint32_t lds_words;        // 16-byte words of recs (k_walk_lds copies them all to LDS)
    const int32_t* delta;      // near records: the matrices' diagonals
    uint32_t n_delta;          // their number, over all matrices
    uint32_t near_n;           // near records: nodes (start records follow)
    const ChunkDesc* chunks;
    const int64_t* bounds;     // NSEG + 1 segment starts
    uint64_t max_steps;
    uint32_t* rec_end;
    uint32_t* rec_vis;
    uint32_t* rec_len;
    unsigned long long* queue;  // chunks taken of every segment, QUEUE_STRIDE words apart
    uint32_t slab_claim;       // chunks a wave claims at once from a slab queue (>= 1)
    uint32_t n_first;          // bulk waves that start at once; the others once the long
                               // segment's rows are taken
    HandQueue hq;              // long walks handed over to single-walk waves
    unsigned long long* deg_sum;
    int* err;
    // walk reuse: per-lane stacks of stack_depth entries {rank, node, position,
    // stays}; counted walks go to out_key (start node << 32 | end node, END_GROUND for
    // ground) and out_vl (stays, steps).  A wave takes slots in blocks of REUSE_CHUNK
    // from *nrec and fills the slots it leaves unused with the key ~0 (sorts last);
    // slots at or beyond out_cap are only counted.  *steps_sum collects the simulated
    // steps.
    uint4* stack;
    uint32_t stack_depth;
    uint64_t* out_key;
    uint2* out_vl;
    unsigned long long* nrec;
    unsigned long long out_cap;
    unsigned long long* steps_sum;
};

constexpr uint32_t REUSE_CHUNK = 4096;

// The step cap of a walk whose steps are counted in 32 bits (by eights: the count stops short
// of wrapping round, or a walk that never ends would run for good).
__device__ __forceinline__ uint32_t step_limit(const WalkArgs& a)
{
    return (uint32_t)(a.max_steps < 0xFFFFFF00ull ? a.max_steps : 0xFFFFFF00ull);
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
    for (int d = 32; d > 0; d >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        v = o > v ? o : v;
    }
    return v;
}

// Emission of counted walks by the lanes currently executing (walk reuse).  The wave's
// slot block [*next, *end) is the same in every lane that runs this; a lane with
// `em` set writes one record.
__device__ __forceinline__ void emit_walks(const WalkArgs& a, bool em, uint32_t row, uint32_t end,
                                           uint32_t stays, uint32_t steps, uint64_t& next,
                                           uint64_t& bend)
{
    const int lane = __lane_id();
    const uint64_t lt = lanemask_lt();
    const uint64_t act = ballot(true);
    const uint64_t m = ballot(em);
    if (m == 0) return;
    const uint32_t cnt = (uint32_t)__popcll(m);
    if (next + cnt > bend) {
        // the rest of the block stays unused: mark it, then take a new block
        const uint32_t na = (uint32_t)__popcll(act), me = (uint32_t)__popcll(act & lt);
        for (uint64_t q = next + me; q < bend; q += na)
            if (q < a.out_cap) a.out_key[q] = ~0ull;
        const int leader = __ffsll((long long)act) - 1;
        unsigned long long c = 0;
        if (lane == leader) c = atomicAdd(a.nrec, (unsigned long long)REUSE_CHUNK);
        c = shfl_u64(c, leader);
        next = c;
        bend = c + REUSE_CHUNK;
    }
    if (em) {
        const uint64_t slot = next + (uint64_t)__popcll(m & lt);
        if (slot < a.out_cap) {
            a.out_key[slot] = ((uint64_t)row << 32) | end;
            a.out_vl[slot] = make_uint2(stays, steps);
        }
    }
    next += cnt;
}

// ------------------------------------------------------------- handed-over walks
// The lowest ranks' walks end only at ground and run up to 10^4 times the mean length,
// one dependent record load per step.  In a bulk wave such a step takes as long as the
// slowest of 64 random loads and a 64-lane step body: 0.93 us on the 3D grid 128^3 and
// 1.06 us on the 2M-node geometric graph with every wave busy, 0.56 and 0.84 us on an
// idle chip.  The load alone takes 0.09 us from L2, 0.27 us from the Infinity Cache and
// 0.36 us from HBM.  So a lane's walk that has grown old moves to a slot, and a wave that
// runs nothing else takes it: the walk's state and its records live in scalar registers
// (one scalar load of the record, compares and selects on the scalar unit), the lanes
// make the draws, 64 Philox blocks at a time.  A step then takes 0.2 us on the grid and
// 0.42 us on the graph (idle chip).  Walk kernel with walks handed over, on the same
// records: graph 780 -> 414 ms; grid 64^3 70 -> 34 ms; the grid 128^3 is bound by the
// bulk waves.
constexpr uint32_t HAND_MIN_AGE = 64;   // steps before a walk may move
constexpr uint32_t HAND_GROUPS = 8;     // groups of eight steps between a bulk wave's looks
constexpr int HAND_WAITING = 256;       // walks kept waiting for a free wave
constexpr int HAND_PER_LOOK = 2;        // walks a bulk wave hands over per look
constexpr int HAND_LAST = 4;            // a bulk wave without new work and with this few walks ends

__device__ __forceinline__ unsigned long long hand_load(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The hand-over queue's memory operations on the device.
struct HandMem {
    __device__ __forceinline__ uint64_t load(const unsigned long long* p) const
    {
        return readfirstlane64(hand_load(p));
    }
    __device__ __forceinline__ void store(unsigned long long* p, unsigned long long v) const
    {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint64_t add(unsigned long long* p, unsigned long long v) const
    {
        return wave_fetch_add(p, v);
    }
    __device__ __forceinline__ uint64_t cas(unsigned long long* p, unsigned long long from,
                                            unsigned long long to) const
    {
        return atomicCAS(p, from, to);
    }
    // lane 0's, the same in every lane
    __device__ __forceinline__ uint64_t cas_uniform(unsigned long long* p, unsigned long long from,
                                                    unsigned long long to) const
    {
        unsigned long long r = 0;
        if (__lane_id() == 0) r = atomicCAS(p, from, to);
        return lane0_u64(r);
    }
    __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(32); }
    __device__ __forceinline__ int64_t now() const { return wall_clock64(); }
    __device__ __forceinline__ uint32_t lane() const { return __lane_id(); }
    __device__ __forceinline__ uint32_t lanes() const { return 64u; }
};

// Wave-uniform data of an earlier launch, through the scalar cache.
template <typename V>
__device__ __forceinline__ V scalar_load(const void* p)
{
    typedef const V __attribute__((address_space(4)))* cptr;
    return *(cptr)readfirstlane64((uint64_t)p);
}
typedef uint32_t u32x8 __attribute__((ext_vector_type(8), aligned(32)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16), aligned(64)));

__device__ __forceinline__ void scalar_line(const uint4* recs, uint32_t line, uint32_t (&w)[16])
{
    const u32x16 v = scalar_load<u32x16>(recs + (size_t)line * 4);
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = v[i];
}

__device__ __forceinline__ ChunkDesc scalar_chunk(const ChunkDesc* chunks, uint64_t c)
{
    return __builtin_bit_cast(ChunkDesc, scalar_load<u32x8>(chunks + c));
}

// the record line that a line word and the draw made there select
template <int FMT>
__device__ __forceinline__ uint32_t word_line(uint32_t word, uint32_t u)
{
    if constexpr (FMT == REC_BUCKETS) {
        const uint32_t kb = word >> LINE_KB_SHIFT, base = word & LINE_MASK;
        return kb == 0u ? base : base + (u >> (32u - kb));
    }
    return word;
}

template <int FMT>
struct SingleRec {
    uint32_t w[FMT == REC_NEAR ? 8 : 16];
};

template <int FMT>
__device__ __forceinline__ SingleRec<FMT> load_single(const uint4* recs, uint32_t line)
{
    SingleRec<FMT> r;
    if constexpr (FMT == REC_NEAR) {
        const u32x8 v = scalar_load<u32x8>(recs + (size_t)line * (NEAR_WORDS / 4));
#pragma unroll
        for (int i = 0; i < 8; ++i) r.w[i] = v[i];
    } else {
        scalar_line(recs, line, r.w);
    }
    return r;
}

// Runs one walk of row cd to its end, the whole wave on it: t moves are made (a multiple
// of 8), `word` is the line word of the node reached.  Returns the sum of the degrees of
// the nodes left.
template <int FMT>
__device__ __forceinline__ uint64_t run_single(const WalkArgs& a, const ChunkDesc& cd, uint32_t w,
                                               uint32_t t, uint32_t word, uint32_t visits)
{
    const int lane = __lane_id();
    const uint32_t limit = step_limit(a);
    int32_t dl = 0;  // near records: lane i holds the matrix's diagonal i
    if (FMT == REC_NEAR && lane < NEAR_DELTAS)
        dl = a.delta[(cd.walks >> WALKS_MAT_SHIFT) * NEAR_DELTAS + lane];
    uint64_t degsum = 0;
    uint32_t endv = END_GROUND;
    uint32_t len = t;
    bool fin = false;
    while (!fin) {
        // lane i makes the eight draws of block len / 8 + i
        const u64x4 b = philox4x64_10((uint64_t)(len >> 3) + lane, w, cd.key, STREAM_WALK, cd.seed, 0);
        const uint32_t q[8] = {(uint32_t)b.x0, (uint32_t)(b.x0 >> 32), (uint32_t)b.x1, (uint32_t)(b.x1 >> 32),
                               (uint32_t)b.x2, (uint32_t)(b.x2 >> 32), (uint32_t)b.x3, (uint32_t)(b.x3 >> 32)};
        uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)q[0], 0);
        SingleRec<FMT> r = load_single<FMT>(a.recs, word_line<FMT>(word, u));
        for (int blk = 0; blk < 64 && !fin; ++blk) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // the next node, and its record's load, before anything else of this step
                uint32_t next;
                bool ground;
                if constexpr (FMT == REC_NEAR) {
                    uint32_t sh = 24;  // four times the number of thresholds not above u
#pragma unroll
                    for (int i = 6; i >= 1; --i) sh = u < r.w[i] ? 4u * (uint32_t)(i - 1) : sh;
                    next = word + (uint32_t)__builtin_amdgcn_readlane(dl, (int)((r.w[7] >> sh) & 7u));
                    ground = sh >= (r.w[7] >> 28) * 4u && (r.w[0] & NEAR_GROUNDED) != 0;
                } else {
                    next = ~0u;  // no line word: not found
                    if (r.w[1] & DESC_INLINE) {
#pragma unroll
                        for (int m = 5; m >= 0; --m) next = u < r.w[4 + 2 * m] ? r.w[5 + 2 * m] : next;
                    } else {
                        const uint32_t line = word_line<FMT>(word, u);
                        const uint32_t L = ((r.w[1] & DESC_DEG_MASK) + 7) / 8;
                        uint32_t l = L > 12 ? 13u : 0u;
#pragma unroll
                        for (int i = 11; i >= 0; --i) l = u < r.w[4 + i] ? (uint32_t)(i + 1) : l;
                        for (; l != 0 && l <= L && next == ~0u; ++l) {
                            uint32_t f[16];
                            scalar_line(a.recs, line + l, f);
#pragma unroll
                            for (int i = 7; i >= 0; --i) next = u < f[2 * i] ? f[2 * i + 1] : next;
                        }
                    }
                    ground = next == ~0u && (r.w[1] & DESC_GROUNDED) != 0;
                    next = next == ~0u ? r.w[3] : next;
                }
                // (after the last block of a batch: a load that is not used)
                const uint32_t un = (uint32_t)__builtin_amdgcn_readlane(
                    (int)q[(j + 1) & 7], j < 7 ? blk : (blk < 63 ? blk + 1 : 63));
                const SingleRec<FMT> rn = load_single<FMT>(a.recs, word_line<FMT>(next, un));
                const uint32_t rank = FMT == REC_NEAR ? r.w[0] & ~NEAR_GROUNDED : r.w[0];
                if (rank <= cd.rank) {
                    if (rank < cd.rank) {  // home
                        endv = FMT == REC_NEAR ? word : r.w[2];
                        fin = true;
                        break;
                    }
                    ++visits;
                }
                degsum += FMT == REC_NEAR ? r.w[7] >> 28 : r.w[1] & DESC_DEG_MASK;
                ++len;
                if (ground) {
                    fin = true;
                    break;
                }
                word = next;
                u = un;
                r = rn;
            }
            if (!fin && len > limit) fin = true;  // past the cap: the build fails
        }
    }
    if (len > limit) {
        endv = END_LIMIT;
        if (lane == 0) atomicOr(a.err, ERR_LIMIT);
    }
    if (lane == 0) {
        const uint64_t rec = cd.rec + w;
        a.rec_end[rec] = endv;
        a.rec_vis[rec] = visits;
        a.rec_len[rec] = len;
    }
    return degsum;
}

// A wave that has no other work: takes handed-over walks until none can come any more.
template <int FMT>
__device__ __forceinline__ void walk_handed_over(const WalkArgs& a)
{
    uint64_t degsum = 0;
    __builtin_amdgcn_s_setprio(3);  // few instructions per step, all of them on the chain
    HandedWalk w;
    while (hand_take(HandMem{}, a.hq, w)) {
        const ChunkDesc cd = scalar_chunk(a.chunks, (uint32_t)w.w0);
        degsum += run_single<FMT>(a, cd, (uint32_t)(w.w0 >> 32), (uint32_t)(w.w1 >> 32), (uint32_t)w.w1,
                                  (uint32_t)w.w2);
    }
    if (__lane_id() == 0 && degsum) atomicAdd(a.deg_sum, (unsigned long long)degsum);
}

// The wave's chunk: the next one of the range it has claimed, else a new claim from the
// segment it is at (one chunk of the long-walk segment, slab_claim of a slab), else from
// the next segment that has chunks left: the long-walk segment, the wave's own slab (by
// the XCD its workgroup runs on), the other slabs in turn.  False once all are taken.
struct ChunkCursor {
    uint64_t cur = 0, lim = 0;  // the chunk held and the end of the range claimed
    int seg = 0;
    uint32_t first = 0;  // the wave's first chunk of the long segment, not claimed (~0: none)
    bool begun = false;
};

__device__ __forceinline__ bool next_chunk(const WalkArgs& a, int home, ChunkCursor& k)
{
    if (k.cur + 1 < k.lim) {
        ++k.cur;
        return true;
    }
    const int lane = __lane_id();
    for (;;) {
        const uint64_t b0 = scalar_load<uint64_t>(a.bounds + k.seg);
        const uint64_t size = scalar_load<uint64_t>(a.bounds + k.seg + 1) - b0;
        const uint64_t n = k.seg == 0 ? 1ull : (uint64_t)a.slab_claim;
        const uint64_t c = !k.begun ? (uint64_t)k.first : size ? wave_fetch_add(&a.queue[k.seg * QUEUE_STRIDE], n) : 0ull;
        k.begun = true;
        if (c < size) {
            k.cur = b0 + c;
            k.lim = b0 + (c + n < size ? c + n : size);
            return true;
        }
        // one look at all the queues rather than one contended atomic at each
        const bool left = lane < NSEG && hand_load(&a.queue[lane * QUEUE_STRIDE]) <
                                             (unsigned long long)(a.bounds[lane + 1] - a.bounds[lane]);
        const uint32_t m = (uint32_t)ballot(left);
        if (m == 0) return false;
        if (m & 1u) {
            k.seg = 0;
        } else {
            const uint32_t s = m >> 1, h = (uint32_t)home;
            k.seg = 1 + (int)((h + (uint32_t)__ffs((int)((s >> h) | (s << (NSLAB - h)))) - 1u) % NSLAB);
        }
    }
}

// Bulk walk kernel body.  Every wave owns up to 64 walks at a time, one per lane, and
// runs in groups of eight steps, one Philox block per lane and group.  Before a group
// the idle lanes take the next walks of the current chunk.  A step loads the record of
// the node the lane is at (first the row's start record), tests it for home, and
// selects the next node from it: one dependent load per step.  Every lane runs every
// step; an idle lane sits at record 0 and keeps nothing.  A finished walk's results are
// stored just after the next record load is issued: stored at once, they would have to
// complete before that load could reuse their registers.
// recs: the records (a.recs, or the workgroup's copy of them in LDS); dict: the
// diagonals of near records, in LDS.
template <int FMT>
__device__ __forceinline__ void walk_bulk(const WalkArgs& a, const uint4* recs, const int32_t* dict,
                                          uint32_t first)
{
    const int lane = __lane_id();
    const uint64_t lt = lanemask_lt();
    const int home_slab = (int)(blockIdx.x % NSLAB);
    const uint32_t limit = step_limit(a);
    // wave-uniform chunk state
    ChunkCursor cur;
    cur.first = first;
    ChunkDesc cd{};
    uint32_t c_next = 0, c_end = 0;
    bool done = false, full = a.hq.cap == 0;  // full: no slot is left, or will be
    // per-lane walk state
    bool active = false, pend = false;
    uint32_t key = 0, w = 0, t = 0, visits = 0, rank_k = 0, cidx = 0, word = 0, dbase = 0;
    uint32_t endv = 0, len = 0;  // of the finished walk whose results wait
    uint64_t rec = 0, seedw = 0, degsum = 0;

    for (uint32_t g = 0;; ++g) {
        if (pend) {
            a.rec_end[rec] = endv;
            a.rec_vis[rec] = visits;
            a.rec_len[rec] = len;
            pend = false;
        }
        // Old walks move to single-walk waves.  While walks are still to be started: those
        // that have been running for at least half of this wave's time, if few are
        // waiting for a wave (the longest walks start first, so they are the oldest at any
        // time).  Afterwards: any walk, if a wave is idle; and the last few walks of a
        // wave all at once.
        if (!full && g != 0 && g % (done ? 2u : HAND_GROUPS) == 0) {
            const uint64_t act = ballot(active);
            const uint64_t cand = done ? act
                                       : ballot(active && t >= HAND_MIN_AGE && t >= 4 * g && t < 0x40000000u);
            if (cand != 0) {
                int room = HAND_LAST;
                if (!done || __popcll(act) > HAND_LAST) {
                    const uint64_t qs = readfirstlane64(hand_load(a.hq.hand + HAND_QUEUE));
                    const int waiting = (int)((uint32_t)qs - (uint32_t)(qs >> 32));
                    if (!done) room = waiting < HAND_WAITING ? HAND_PER_LOOK : 0;
                    else if (waiting >= 0) room = 0;
                    full = (uint32_t)qs >= a.hq.cap;
                    if (full) room = 0;
                }
                const int place = (int)__popcll(cand & lt);
                const bool go = ((cand >> lane) & 1ull) && place < room;
                const uint32_t cnt = (uint32_t)__popcll(ballot(go));
                if (cnt != 0) {
                    const uint32_t at = hand_reserve(HandMem{}, a.hq, cnt, full) + (uint32_t)place;
                    if (go && hand_put(HandMem{}, a.hq, at,
                                       {(uint64_t)cidx | (uint64_t)w << 32, (uint64_t)t << 32 | word,
                                        (uint64_t)visits})) {
                        active = false;
                        word = 0;
                    }
                }
            }
        }
        if (!done) {
            uint64_t idle = ballot(!active);
            while (idle != 0) {
                if (c_next >= c_end) {
                    if (!next_chunk(a, home_slab, cur)) {
                        done = true;
                        break;
                    }
                    cd = scalar_chunk(a.chunks, cur.cur);
                    c_next = cd.walks & WALKS_FIRST_MASK;
                    c_end = c_next + ((cd.walks >> WALKS_FIRST_BITS) & WALKS_COUNT_MASK);
                }
                const uint32_t avail = c_end - c_next;
                const uint32_t pos = (uint32_t)__popcll(idle & lt);
                const bool take = ((idle >> lane) & 1ull) && pos < avail;
                if (take) {
                    key = cd.key;
                    w = c_next + pos;
                    t = 0;
                    visits = 0;
                    active = true;
                    rank_k = cd.rank;
                    seedw = cd.seed;
                    rec = cd.rec + w;
                    word = cd.sline;
                    cidx = (uint32_t)cur.cur;
                    if (FMT == REC_NEAR) dbase = (cd.walks >> WALKS_MAT_SHIFT) * NEAR_DELTAS;
                }
                const uint64_t taken = ballot(take);
                c_next += (uint32_t)__popcll(taken);
                idle &= ~taken;
            }
        }
        if (ballot(active) == 0) {
            if (done) break;
            continue;
        }
        // draw t + j is the word j of the Philox block t / 8
        const u64x4 b = philox4x64_10((uint64_t)(t >> 3), w, key, STREAM_WALK, seedw, 0);
        const uint32_t q[8] = {(uint32_t)b.x0, (uint32_t)(b.x0 >> 32), (uint32_t)b.x1, (uint32_t)(b.x1 >> 32),
                               (uint32_t)b.x2, (uint32_t)(b.x2 >> 32), (uint32_t)b.x3, (uint32_t)(b.x3 >> 32)};
        uint32_t dacc = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t u = q[j];
            uint32_t rank, id, deg, next;
            bool ground;
            if constexpr (FMT == REC_NEAR) {
                const uint4* lp = recs + (size_t)word * (NEAR_WORDS / 4);
                const uint4 x0 = lp[0], x1 = lp[1];
                if (pend) {
                    a.rec_end[rec] = endv;
                    a.rec_vis[rec] = visits;
                    a.rec_len[rec] = len;
                    pend = false;
                }
                // only a group's first step can be at a start record
                id = j == 0 && word >= a.near_n ? word - a.near_n : word;
                rank = x0.x & ~NEAR_GROUNDED;
                deg = (x1.w >> 28) & 7u;
                uint32_t sh = 24;  // four times the number of thresholds not above u
                sh = u < x1.z ? 20u : sh;
                sh = u < x1.y ? 16u : sh;
                sh = u < x1.x ? 12u : sh;
                sh = u < x0.w ? 8u : sh;
                sh = u < x0.z ? 4u : sh;
                sh = u < x0.y ? 0u : sh;
                next = id + (uint32_t)dict[dbase + ((x1.w >> sh) & 7u)];
                ground = sh >= 4u * deg && (x0.x & NEAR_GROUNDED) != 0;
            } else {
                // a walk's first word is its start record's line itself, which may lie past
                // LINE_MASK (start records follow n_lines walk lines)
                const uint32_t line = j == 0 && t == 0 ? word : word_line<FMT>(word, u);
                const uint4* lp = recs + (size_t)line * 4;
                const uint4 r0 = lp[0], r1 = lp[1], r2 = lp[2], r3 = lp[3];
                if (pend) {
                    a.rec_end[rec] = endv;
                    a.rec_vis[rec] = visits;
                    a.rec_len[rec] = len;
                    pend = false;
                }
                const uint32_t e[16] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w,
                                        r2.x, r2.y, r2.z, r2.w, r3.x, r3.y, r3.z, r3.w};
                rank = e[0];
                id = e[2];
                deg = e[1] & DESC_DEG_MASK;
                next = ~0u;  // no line word: not found
                if (!active || (e[1] & DESC_INLINE) != 0u) {
                    // the first entry m with u < threshold_m, scanned from the top with
                    // selects; unused entries are zero words, and no u is below zero
#pragma unroll
                    for (int m = 5; m >= 0; --m) next = u < e[4 + 2 * m] ? e[5 + 2 * m] : next;
                } else {
                    // the first of the (up to twelve) summarised lines whose last threshold
                    // exceeds u holds the entry; beyond twelve lines, scan on from line 13
                    const uint32_t L = (deg + 7) / 8;
                    uint32_t l = L > 12 ? 13u : 0u;
#pragma unroll
                    for (int i = 11; i >= 0; --i)  // summaries past the last line are zero
                        l = u < e[4 + i] ? (uint32_t)(i + 1) : l;
                    for (; l != 0 && l <= L && next == ~0u; ++l) {
                        const uint4* fp = recs + (size_t)(line + l) * 4;
                        const uint4 f0 = fp[0], f1 = fp[1], f2 = fp[2], f3 = fp[3];
                        const uint32_t f[16] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w,
                                                f2.x, f2.y, f2.z, f2.w, f3.x, f3.y, f3.z, f3.w};
#pragma unroll
                        for (int i = 7; i >= 0; --i) next = u < f[2 * i] ? f[2 * i + 1] : next;
                    }
                }
                ground = next == ~0u && (e[1] & DESC_GROUNDED) != 0;
                next = next == ~0u ? e[3] : next;  // (rounding) past every threshold
            }
            const bool home = active && rank < rank_k;
            const bool move = active && !home;
            visits += rank == rank_k ? 1u : 0u;
            dacc += move ? deg : 0u;
            if (home || (move && ground)) {
                endv = home ? id : END_GROUND;
                len = t + (uint32_t)j + (home ? 0u : 1u);
                if (len > limit) atomicOr(a.err, ERR_LIMIT);
                pend = true;
                active = false;
            }
            word = active ? next : 0u;
        }
        degsum += dacc;
        t += 8;
        if (active && t > limit) {  // past the cap: the build fails
            atomicOr(a.err, ERR_LIMIT);
            endv = END_LIMIT;
            len = t;
            pend = true;
            active = false;
            word = 0;
        }
    }
    degsum = wave_sum(degsum);
    if (lane == 0 && degsum) atomicAdd(a.deg_sum, (unsigned long long)degsum);
}

// Persistent walk kernel.  Every wave owns up to 64 walks at a time, one per lane.
// Every R steps the idle lanes of a wave take the next walks of the current chunk;
// an exhausted chunk is replaced by the next one from the segment queues: the
// long-walk segment first, then the wave's own slab (by the XCD its workgroup runs
// on), then the other slabs in turn.  A lane's draws come from the Philox block of its
// (row, walk, step div 8), generated when step mod 8 = 0.  A lane holds the first
// line of its current record in registers (at the start of a walk, the row's start
// record); a step selects the entry from it (a wide record loads one more line),
// then loads the next node's record line: one dependent 64-byte load per step.
//
// REUSE (Section 5.3, Algorithm "reuse"): a lane also keeps the two stacks of the
// algorithm for its walk, as one stack of entries {rank, node, position, stays} whose
// top lives in registers and the rest in the lane's own region of a.stack.  The start
// is position 1 and the node reached by step t is position t + 2.  A node ranked
// below the top pops it, and a popped entry pushed more than one position earlier is
// a walk of at least two steps from its node: it is emitted as a record.  A node
// ranked above the top is pushed, one equal to it is a stay.  The walk ends exactly
// when the stack empties; the walk itself is the bottom entry's record.
#ifndef SRW_WALK_WAVES
#define SRW_WALK_WAVES 4  // waves per SIMD the register budget is cut for (the grid runs 2)
#endif
template <int R, bool REUSE, bool BUCKETS>
__device__ __forceinline__ void walk_body(const WalkArgs& a)
{
    const uint4* const recs = a.recs;
    const int lane = __lane_id();
    const uint64_t lt = lanemask_lt();
    // wave-uniform chunk state
    ChunkDesc cd{};
    uint32_t c_next = 0, c_end = 0;
    uint64_t c_cur = 0, c_lim = 0;  // the chunk held and the end of the range claimed
    bool done = false;
    const int home = 1 + (int)(blockIdx.x % NSLAB);
    int seg = 0, tried = 0;
    // per-lane walk state
    bool active = false;
    uint32_t key = 0, w = 0, visits = 0, rank_k = 0;
    uint32_t cline = 0;                        // current record's first line
    uint4 r0 = make_uint4(0, 0, 0, 0), r1 = r0, r2 = r0, r3 = r0;  // its words
    uint64_t t = 0, rec = 0, degsum = 0, seedw = 0;
    uint32_t q0 = 0, q1 = 0, q2 = 0, q3 = 0, q4 = 0, q5 = 0, q6 = 0, q7 = 0;
    // REUSE: stack top, depth below it, the lane's stack region, simulated steps
    uint32_t top_rank = 0, top_node = 0, top_pos = 0, top_vis = 0, depth = 0;
    uint4* const my_stack =
        REUSE ? a.stack + ((size_t)blockIdx.x * BLOCK + threadIdx.x) * a.stack_depth : nullptr;
    uint64_t steps_acc = 0;
    uint64_t blk_next = 0, blk_end = 0;  // the wave's block of record slots

    for (uint32_t iter = 0;; ++iter) {
        if ((iter % R) == 0 && !done) {
            uint64_t idle = ballot(!active);
            while (idle != 0) {
                if (c_next >= c_end) {
                    // next chunk: long segment, then home slab, then the other slabs
                    // the next chunk of the range already claimed, else a new claim:
                    // one chunk from the long segment, slab_claim from a slab
                    bool got = c_cur + 1 < c_lim;
                    unsigned long long cidx = got ? ++c_cur : 0ull;
                    while (!done && !got) {
                        const int sq = seg == 0 ? 0 : 1 + (home - 1 + tried) % NSLAB;
                        const unsigned long long size =
                            (unsigned long long)(a.bounds[sq + 1] - a.bounds[sq]);
                        const unsigned long long k = sq == 0 ? 1ull : (unsigned long long)a.slab_claim;
                        const unsigned long long c = wave_fetch_add(&a.queue[sq * QUEUE_STRIDE], k);
                        if (c < size) {
                            got = true;
                            cidx = (unsigned long long)a.bounds[sq] + c;
                            c_cur = cidx;
                            c_lim = (unsigned long long)a.bounds[sq] + (c + k < size ? c + k : size);
                        } else if (seg == 0) {
                            seg = 1;
                        } else if (++tried >= NSLAB) {
                            done = true;
                        }
                    }
                    if (done) break;
                    cd = a.chunks[cidx];
                    c_next = cd.walks & WALKS_FIRST_MASK;
                    c_end = c_next + ((cd.walks >> WALKS_FIRST_BITS) & WALKS_COUNT_MASK);
                }
                const uint32_t avail = c_end - c_next;
                const uint32_t pos = (uint32_t)__popcll(idle & lt);
                const bool take = ((idle >> lane) & 1ull) && pos < avail;
                if (take) {
                    key = cd.key;
                    w = c_next + pos;
                    t = 0;
                    visits = 1;
                    active = true;
                    rank_k = cd.rank;
                    seedw = cd.seed;
                    rec = cd.rec + w;
                    cline = cd.sline;
                    if constexpr (REUSE) {
                        top_rank = cd.rank;
                        top_node = cd.key;
                        top_pos = 1;
                        top_vis = 1;
                        depth = 0;
                    }
                    const uint4* lp = recs + (size_t)cline * 4;
                    r0 = lp[0];
                    r1 = lp[1];
                    r2 = lp[2];
                    r3 = lp[3];
                }
                const uint64_t taken = ballot(take);
                c_next += (uint32_t)__popcll(taken);
                idle &= ~taken;
            }
        }
        if (ballot(active) == 0) {
            if (done) break;
            continue;
        }
        if (active) {  // structured: the lanes rejoin before the next refill's ballots
        // draws: step t's is the word t mod 8 of the Philox block t div 8.  With bucket
        // lines a walk needs its next draw during a step, so the next block is made at
        // the block's last step and the first block when the walk starts.
        const uint32_t phase = (uint32_t)(t & 7);
        if (phase == 0 && (!BUCKETS || t == 0)) {
            const u64x4 b = philox4x64_10(t >> 3, w, key, STREAM_WALK, seedw, 0);
            q0 = (uint32_t)b.x0; q1 = (uint32_t)(b.x0 >> 32);
            q2 = (uint32_t)b.x1; q3 = (uint32_t)(b.x1 >> 32);
            q4 = (uint32_t)b.x2; q5 = (uint32_t)(b.x2 >> 32);
            q6 = (uint32_t)b.x3; q7 = (uint32_t)(b.x3 >> 32);
        }
        const uint32_t u = q0;
        q0 = q1; q1 = q2; q2 = q3; q3 = q4; q4 = q5; q5 = q6; q6 = q7;
        if constexpr (BUCKETS) {
            if (phase == 7) {  // q0 becomes the next step's draw
                const u64x4 b = philox4x64_10((t + 1) >> 3, w, key, STREAM_WALK, seedw, 0);
                q0 = (uint32_t)b.x0; q1 = (uint32_t)(b.x0 >> 32);
                q2 = (uint32_t)b.x1; q3 = (uint32_t)(b.x1 >> 32);
                q4 = (uint32_t)b.x2; q5 = (uint32_t)(b.x2 >> 32);
                q6 = (uint32_t)b.x3; q7 = (uint32_t)(b.x3 >> 32);
            }
        }

        const uint32_t deg = r0.y & DESC_DEG_MASK;
        degsum += deg;
        const bool inl = (r0.y & DESC_INLINE) != 0u;
        // The next node is the first entry m with u < threshold_m; the words of the
        // line held (a narrow record, a bucket line, or a wide record's first line)
        // are in registers.
        const uint32_t e[16] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w,
                                r2.x, r2.y, r2.z, r2.w, r3.x, r3.y, r3.z, r3.w};
        uint32_t next_line = 0;
        bool found = false;
        if (inl) {
            // entries 0..5 in words 4..15, scanned from the top with selects (the
            // lowest hit is taken last): no branches.  Unused entries are zero words,
            // and no u is below a zero threshold.
#pragma unroll
            for (int m = 5; m >= 0; --m) {
                const bool hit = u < e[4 + 2 * m];
                next_line = hit ? e[5 + 2 * m] : next_line;
                found = found || hit;
            }
        } else {
            // the first of the (up to twelve) summarised lines whose last threshold
            // exceeds u holds the entry; beyond twelve lines, scan on from line 13
            const uint32_t L = (deg + 7) / 8;
            uint32_t lh = 0;
#pragma unroll
            for (int i = 11; i >= 0; --i) {  // summaries past the last line are zero
                const bool h = u < e[4 + i];
                lh = h ? (uint32_t)(i + 1) : lh;
            }
            for (uint32_t l = lh ? lh : (L > 12 ? 13u : 0u); l != 0 && l <= L && !found; ++l) {
                const uint4* lp = recs + ((size_t)(cline + l) * 4);
                const uint4 x0 = lp[0], x1 = lp[1], x2 = lp[2], x3 = lp[3];
                const uint32_t f[16] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w,
                                        x2.x, x2.y, x2.z, x2.w, x3.x, x3.y, x3.z, x3.w};
                uint32_t nl = 0;
                bool hit_any = false;
#pragma unroll
                for (int i = 7; i >= 0; --i) {  // entries past the last are zero words
                    const bool hit = u < f[2 * i];
                    nl = hit ? f[2 * i + 1] : nl;
                    hit_any = hit_any || hit;
                }
                next_line = hit_any ? nl : next_line;
                found = hit_any;
            }
        }
        // past every threshold: to ground if v is grounded, else (rounding) to the
        // last neighbour; the grounded lane still loads that neighbour's line, which
        // keeps the load below unconditional
        const bool to_ground = !found && (r0.y & DESC_GROUNDED) != 0;
        if (!found) next_line = e[3];
        if constexpr (BUCKETS) {
            // the line word: a bucketed target's bucket line for the next draw (q0),
            // else its first line
            const uint32_t kb = next_line >> LINE_KB_SHIFT;
            const uint32_t base = next_line & LINE_MASK;
            next_line = kb == 0u ? base : base + (q0 >> (32u - kb));
        }
        const uint4* lp = recs + (size_t)next_line * 4;
        r0 = lp[0];
        r1 = lp[1];
        r2 = lp[2];
        r3 = lp[3];
        cline = next_line;
        // home: a node ranked below the row (the first step only reaches higher ranks)
        bool fin = to_ground || r0.x < rank_k;
        uint32_t endv = to_ground ? END_GROUND : r0.z;
        visits += (!fin && r0.x == rank_k);
        if constexpr (REUSE) {
            const uint32_t l = (uint32_t)t + 2;  // position of the node just reached
            bool below = to_ground || r0.x < top_rank;
            bool empty = false;
            while (below) {
                emit_walks(a, l > top_pos + 1, top_node, endv, top_vis, l - top_pos, blk_next,
                           blk_end);
                if (depth == 0) {
                    empty = true;
                    break;
                }
                --depth;
                const uint4 e = my_stack[depth];
                top_rank = e.x;
                top_node = e.y;
                top_pos = e.z;
                top_vis = e.w;
                below = to_ground || r0.x < top_rank;
            }
            if (!empty) {
                if (r0.x > top_rank) {
                    if (depth == a.stack_depth) {
                        atomicOr(a.err, ERR_STACK);
                        fin = true;
                    } else {
                        my_stack[depth] = make_uint4(top_rank, top_node, top_pos, top_vis);
                        ++depth;
                        top_rank = r0.x;
                        top_node = r0.z;
                        top_pos = l;
                        top_vis = 1;
                    }
                } else {
                    ++top_vis;
                }
            }
        }
        ++t;
        if (!fin && t >= a.max_steps) {
            fin = true;
            endv = END_LIMIT;
            atomicOr(a.err, ERR_LIMIT);
        }
        if (fin) {
            if constexpr (REUSE) {
                steps_acc += t;
            } else {
                a.rec_end[rec] = endv;
                a.rec_vis[rec] = visits;
                a.rec_len[rec] = (uint32_t)t;
            }
            active = false;
        }
        }  // active
        if constexpr (REUSE) {  // lanes that emitted moved the block on: agree again
            blk_next = wave_max_u64(blk_next);
            blk_end = wave_max_u64(blk_end);
        }
    }
    if constexpr (REUSE) {
        for (uint64_t q = blk_next + lane; q < blk_end; q += 64)
            if (q < a.out_cap) a.out_key[q] = ~0ull;
    }
    degsum = wave_sum(degsum);
    if (lane == 0 && degsum) atomicAdd(a.deg_sum, (unsigned long long)degsum);
    if constexpr (REUSE) {
        steps_acc = wave_sum(steps_acc);
        if (lane == 0 && steps_acc) atomicAdd(a.steps_sum, (unsigned long long)steps_acc);
    }
}

// refill periods other than 8
template <int R, bool BUCKETS>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(SRW_WALK_WAVES))) void k_walk_refill(WalkArgs a)
{
    walk_body<R, false, BUCKETS>(a);
}

// walk reuse keeps the stack top in registers as well: a larger register budget
template <bool BUCKETS>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_walk_reuse(WalkArgs a)
{
    walk_body<8, true, BUCKETS>(a);
}

// Each wave's part: a bulk wave, then (a.hq.cap) a single-walk wave.  A later workgroup
// looks for a while whether every bulk workgroup has started: if not, a late bulk wave
// starts at once, and a single-walk wave ends.
template <int FMT>
__device__ __forceinline__ void walk_wave(const WalkArgs& a, const uint4* recs, const int32_t* dict)
{
    __shared__ int all_here;
    const bool hand = a.hq.cap != 0;
    const HandMem mem;
    const uint32_t wave = blockIdx.x * (BLOCK / 64) + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool bulk = wave < a.hq.n_bulk;
    bool here = false;  // known that every bulk workgroup has started
    if (hand) {
        if (bulk && threadIdx.x == 0) atomicAdd(a.hq.hand + HAND_ARRIVED, 1ull);
        if (wave >= a.n_first) {
            if (threadIdx.x == 0) {
                int ok = 0;
                for (int i = 0; i < 64 && !ok; ++i) {
                    ok = hand_load(a.hq.hand + HAND_ARRIVED) >= a.hq.n_groups;
                    if (!ok) __builtin_amdgcn_s_sleep(64);
                }
                all_here = ok;
            }
            __syncthreads();  // n_first and n_bulk are whole workgroups
            here = all_here != 0;
        }
    }
    if (bulk) {
        if (here) {  // (a late wave)
            const unsigned long long size = (unsigned long long)(a.bounds[1] - a.bounds[0]);
            const int64_t t0 = mem.now();
            while (mem.load(a.queue) < size && mem.now() - t0 <= a.hq.wait_limit)
                __builtin_amdgcn_s_sleep(127);
        }
        walk_bulk<FMT>(a, recs, dict, wave < a.n_first ? wave : ~0u);
        here = hand && hand_finish(mem, a.hq);
    }
    if (here) walk_handed_over<FMT>(a);
}

template <int FMT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(SRW_WALK_WAVES))) void k_walk(WalkArgs a)
{
    __shared__ int32_t dict[FMT == REC_NEAR ? NEAR_MATS * NEAR_DELTAS : 1];
    if (FMT == REC_NEAR) {
        for (uint32_t i = threadIdx.x; i < a.n_delta; i += BLOCK) dict[i] = a.delta[i];
        __syncthreads();
    }
    walk_wave<FMT>(a, a.recs, dict);
}

// The same walks with the records staged in LDS: for a table of at most the LDS a
// workgroup can hold, every workgroup first copies it, and each step of a bulk wave then
// reads LDS instead of the caches.
template <int FMT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(SRW_WALK_WAVES))) void k_walk_lds(WalkArgs a)
{
    extern __shared__ uint4 table[];
    __shared__ int32_t dict[FMT == REC_NEAR ? NEAR_MATS * NEAR_DELTAS : 1];
    for (uint32_t i = threadIdx.x; i < a.lds_words; i += BLOCK) table[i] = a.recs[i];
    if (FMT == REC_NEAR)
        for (uint32_t i = threadIdx.x; i < a.n_delta; i += BLOCK) dict[i] = a.delta[i];
    __syncthreads();
    walk_wave<FMT>(a, table, dict);
}
