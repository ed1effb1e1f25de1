// Internal definitions shared by the HIP sources of libdv (device state,
// buffer table, kernel launchers).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dv.h"

#define DV_TILE 32                 // tile edge in sites (labelling, colouring)
#define DV_TILE_SITES (DV_TILE * DV_TILE)
#define DV_TILE_PIECES (DV_TILE_SITES / 2)   // most pieces, and most runs, of a tile
// Per-piece and per-run arrays hold the first DV_PIECES_LO pieces (DV_RUNS_LO
// runs) of every tile side by side, then the rest of every tile: a tile has a
// few pieces, so what the kernels touch is one line per tile in an array of 64
// or 128 bytes per tile, not a line in each of 1 to 4 KB.
#define DV_PIECES_LO 16
#define DV_RUNS_LO 64
#define DV_BORDER (4 * DV_TILE)    // border entries of a tile: top row, bottom row, left, right column
#define DV_BLOCK 256               // threads per tile workgroup
#define DV_EMPTY 0x77777777        // MAXLINK: empty row slot / no colour
#define DV_CAND_CAP 128            // candidate centre images held in LDS per chunk
#define DV_TILE_PAIRS 128          // couples a colouring tile lists for the row build
#define DV_LINE 32                 // words of a 128-byte line (a counter of its own line each:
                                   // atomics on one line take turns, about 5 ns each)
#define DV_ROW 16                  // slots of a row's table (a Delaunay row holds 6 on average)

// Lists of the tiles of a launch that need the general colouring, a lane of the wave
// that reads them each.  Atomics on one counter take turns, 11 ns each here: with a
// counter per frame the 16,384 tiles of an empty frame of 4096^2 spent 190 us on it.
#define GEN_LISTS 64

// error bits raised on the device during a frame
#define DV_E_KMAX 1u               // more components than K_max
#define DV_E_DEGREE 2u             // a Delaunay row overflowed max_degree
#define DV_E_ANY (DV_E_KMAX | DV_E_DEGREE)

#define DV_MAX_BATCH 64            // frames of one sequence processed by one launch
#define DV_MAX_ENTRIES 64          // frames (of one or several sequences) in one launch
#define DV_DEFAULT_BATCH 32        // what max_batch = 0 selects

// Flips of a results page that k_place also writes to pinned host memory (24
// bytes each), so that reading them takes no copy call: that call and its wait
// cost about 25 us, which is what 16,384 flips take over the bus.  A launch
// whose flips go beyond it leaves them to the copy.
#define DV_HOST_FLIPS 16384

// Per-frame header, one per batch slot (device memory).
struct FrameState {
    int32_t K_now;         // components found in the frame (raw, may exceed K_max)
    uint32_t err;          // DV_E_* bits of the frame
    int32_t rows_dirty;    // rows of the slot's adjacency that may hold entries
    int32_t n_amb;         // components crossing their own antipodal line
    int32_t K_past;        // K of the past frame it was compared with (0: none)
    int32_t pad;
    // breaking and arising couples found by the row comparison (one 64-bit sum)
    alignas(8) int32_t nb_acc;
    int32_t na_acc;
    int32_t spill;         // some row of the slot's adjacency has entries beyond its table
};

// Result record of one frame in a results page: written by the device into
// pinned host memory, read by the host once the launch has completed.
struct FrameOut {
    long long frame;       // accepted frames of the sequence up to and including this one
    int32_t status;        // 0 accepted, else DV_ERR_CAPACITY
    int32_t K, E;          // components (raw when rejected), undirected couples
    int32_t n_flips, n_break;
    int32_t excl_past, excl_now;
    int32_t amb;           // components crossing their own antipodal line
    int32_t trigger;       // global trigger
    int32_t flip_off;      // first flip of the frame in the page's flip array
    int32_t on_host;       // the frame's flips are in the page's host copy as well
    int32_t sel;           // past buffer that holds the frame after an accepted launch end
    int32_t K_past;        // K of the past frame it was compared with (0: none)
};

// Sequence header (device memory).  Two past buffers alternate: buffer `sel`
// holds the last accepted frame before the batch in flight; the batch's last
// accepted frame is copied into buffer 1 - sel, and the commit flips `sel`.
// There are two headers as well: a launch reads one (DV_PG_PAR) and its last
// kernel writes the other, so that the commit needs no launch of its own.
struct SeqState {
    int32_t sel;
    int32_t past_valid;
    int32_t K[2];          // components held by each past buffer
    int32_t pg_fill[2];    // flips held by each results page
    int64_t frame;         // accepted frames
};

// Component arrays of one buffer.
struct CompBuf {
    int32_t *qx, *qy;      // Q.8 centre
    double *fx, *fy;       // float64 centre
    int32_t *n;            // member count
    int32_t *root;         // smallest linear index of the component
    int32_t *amb;          // 1 when the component crosses its antipodal line
    // Rows of the adjacency: unordered sets.  The first `prim` = min(max_degree,
    // DV_ROW) slots of a row are a hash table (open addressing, empty slots hold
    // DV_EMPTY, any slot may be empty); a row whose table is full goes on in its
    // max_degree - prim slots of adjx, filled from the front.  Slots of adjx are
    // meaningful only when the table is full.
    int32_t *adj;          // [K_max][prim]
    int32_t *adjx;         // [K_max][max_degree - prim]
};

// Obstacle bits of a tile's window, one site wider than the tile on every side
// (periodic): words 0 .. 33 the rows -1 .. 32, bit x for column x of 0 .. 31;
// words 34, 35 the column left of the tile and 36, 37 the one right of it, bit r
// for row r - 1.  Zero beyond a ragged tile's window.
#define DV_OBITS 40

// Everything a kernel may touch: the buffers of one batch slot (one frame)
// and the past buffers shared by all slots.  The table of all slots lives in
// device memory; a kernel takes its frame's entry (found from a flat block index,
// or blockIdx.z) and, for the comparison, the entry of its past.
struct Bufs {
    int32_t seq;           // sequence of the entry within a launch (past and commit)
    int32_t lx, ly, ntx, nty;
    float thr;
    int32_t phase, conn;
    int32_t kmax, maxdeg;
    int32_t prim;          // table slots of a row: min(max_degree, DV_ROW)
    int32_t ncells;        // bucket grid = tile grid
    int32_t keep_maps;     // write the label / owner maps
    int32_t classify;      // fill the flips' event flags
    int32_t open_x, open_y;  // 1: walls across that axis instead of wrapping
    int32_t weighted;      // centres weighted by the quantised field (DV_WEIGHTED)
    const uint8_t *obst;   // [N] obstacle sites (nonzero), or null: none
    const uint32_t *obits; // [tiles][DV_OBITS] the same around each tile as bits (k_obits), or null
    int32_t *parent;       // [N] union-find over piece roots (linear site indices)
    uint16_t *bpc;         // [tiles][DV_BORDER] tile-local piece root of every tile-border
                           // site (0xffff outside): top row, bottom row, left column,
                           // right column, 32 entries each
    uint32_t *tedge;       // [tiles][4] inside bits of the same lines
    int32_t *labels;       // [N] output label map
    int32_t *owner;        // [N] output colour map
    // Per tile: the inside bits of its rows, the piece slot of each horizontal
    // run (raster order), and per piece its root site, size and coordinate sums
    // (PIECE_*; with weighted centres its weight sums, in no more memory).
    uint32_t *tmask;       // [tiles][32]
    uint16_t *trun;        // [tiles][DV_TILE_PIECES]
    unsigned long long *tpiece;  // [tiles][DV_TILE_PIECES]
    int32_t *prank;        // [tiles][DV_TILE_PIECES] canonical rank of each piece's component
                           // (before it is known, of weighted centres: the sum of w y)
    int32_t *npieces;      // [tiles]
    uint2 *seg;            // [ly][ntx] per (row, tile column): component-root bits, and the
                           // roots before the segment within its band
    int32_t *band_sum;     // [nty] roots per band of 32 rows
    // component accumulation (self-cleaning: finalize zeroes what it reads)
    long long *acc_x, *acc_y;   // sums of offsets from the root (weighted: of w * offset)
    long long *acc_w;           // [K_max] sums of the site weights (weighted centres only)
    int32_t *acc_n, *acc_amb, *acc_root;
    // bucket grid of the frame's centres
    int32_t *cell_count;   // [ncells]
    int32_t *cell_head;    // [ncells] last centre put into each cell (-1: none); comp_next
                           // leads to the one before (frames with many components)
    int32_t *cell_sum;     // [ncells / 256][DV_LINE] centres in each group of 256 cells
    int32_t *cell_start;   // [ncells + 1]
    int32_t *cell_items;   // [K_max] labels ordered by cell
    int2 *cell_q;          // [K_max] their Q.8 centres
    int32_t *comp_next;    // [K_max]
    int2 *tpairs;          // [tiles][DV_TILE_PAIRS] distinct couples found by each tile
                           // (before the colouring, of weighted centres: the low 16 bits of
                           // each piece's sum of w)
    int32_t *tpair_n;      // [tiles]
    int32_t *gen_list;     // [tiles + GEN_LISTS] part of the launch's lists of tiles that need the
                           // general colouring (flat tile indices; gen_place)
    int32_t *gen_n;        // [GEN_LISTS][DV_LINE] tiles on each list; word 1: there are some
                           // (shared by the slots; the launch's first entry's is used)
    int32_t *cnt;          // [K_max] preimages of each now label
    int32_t *inv;          // [K_max] now -> past (valid when cnt == 1)
    CompBuf cur;           // components and rows of the frame
    FrameState *fs;
    // comparison with the past
    int32_t *phi;          // [K_max] past -> now
    int32_t *nb, *na;      // [K_max] breaking / arising count per now row
    int4 *dpart;           // [chunks of rows] breaking, arising, row lengths, dropped
    int32_t *stage;        // [K_max][2 * max_degree][6] flips of each row, row order
    // event classification (when classify): per now label
    int32_t *act;          // [K_max] the row changed (an end of a flip)
    int32_t *ecnt;         // [K_max] active points connected in either graph
    int32_t *ebnd;         // [K_max] bit 0: boundary point of the now graph, bit 1: of the past
    CompBuf past[2];       // shared by the slots
    SeqState *st;          // [2] shared by the slots
    // results pages (shared by the slots): every frame's record and flips,
    // kept until the host has read them
    FrameOut *pg_info[2];  // [page frames] records, pinned host memory (device view)
    int32_t *pg_flips[2];  // [page frames * K_max * max_degree][6] flips, device memory
    int32_t *pg_host[2];   // [host_flips][6] the first flips of the page, pinned host memory
    int32_t host_flips;    // (0: no host copy)
    int32_t host_part;     // flips that do not all fit are copied as far as they do
    dv_frame_info *out_info;  // the frame's record as the caller's (device memory), or null
};

// A piece's record: member count, sums of its sites' tile-local x and y (a full
// tile: 1024, 15872, 15872) and its tile-local root site, in 16 bits each.
// With weighted centres the middle is the sum of w x (31 bits: weights are below
// 2^16), and the sum of w (26 bits) is in what the size and the root leave free and
// in 16 bits beside the record (PIECE_W): with the sum of w y in the rank's place
// the weights take no memory of their own (6 KB a tile as arrays of words, a fifth
// of a context of 4096^2 without maps).
#define PIECE_N(r) ((int)((r) & 0x7ffu))
#define PIECE_SX(r) ((int)(((r) >> 16) & 0xffffu))
#define PIECE_SY(r) ((int)(((r) >> 32) & 0xffffu))
#define PIECE_ROOT(r) ((int)(((r) >> 48) & 0x3ffu))
#define PIECE_WEIGHTED(r, w, wx)                                                                     \
    (((r) & 0x03ff0000000007ffull) | ((unsigned long long)(((w) >> 16) & 0x1fu) << 11) |             \
     ((unsigned long long)(wx) << 16) | ((unsigned long long)((w) >> 21) << 58))
#define PIECE_WX(r) ((unsigned)((r) >> 16))
#define PIECE_W(r, low) ((low) | (((unsigned)((r) >> 11) & 0x1fu) << 16) | ((unsigned)((r) >> 58) << 21))
static_assert(DV_TILE_PAIRS * sizeof(int2) == DV_TILE_PIECES * sizeof(uint16_t), "tpairs holds PIECE_W's low bits");

// Results-page position of a launch entry: bits 0-5 the frame's record, bit 6
// the page, bit 7 set when the page starts empty with this launch, bit 8 the
// sequence header that the launch reads.
#define DV_PG_POS(v) ((int)((v) & 63u))
#define DV_PG_PAGE(v) ((int)(((v) >> 6) & 1u))
#define DV_PG_FRESH(v) ((int)(((v) >> 7) & 1u))
#define DV_PG_PAR(v) ((int)(((v) >> 8) & 1u))

// Field pointers of the frames of one launch.
struct Fields {
    const float *p[DV_MAX_ENTRIES];
};

// One launch's work: entries 0 .. n-1 of the device slot table D (frames of
// one or several sequences, each with its own lattice), and the prefix sums
// of their tile and band counts, so that a flat block index finds its entry.
// Entry e of a launch is row idx[e] of a device slot table, which is a
// separate kernel argument (const, restrict: slot fields are loaded once,
// not after every store).  Everything else travels in the kernel arguments,
// so a launch over any subset of a table needs no upload.
struct Batch {
    const Bufs *D;         // the table (host side only; kernels take it separately)
    int n;
    int tiles, bands;      // totals over the entries
    int tpe, bpe;          // tiles / bands of every entry when all are alike, else 0
    int kmax, ntx;         // largest K_max and number of tile columns (launch shapes)
    int classify;          // some entry classifies events
    int geom;              // some entry has walls or obstacles (general kernels)
    int weighted;          // some entry has weighted centres
    int small;             // every entry fits k_mid
    int alone;             // every entry is the only one of its sequence (group launches)
    int past_known;        // every entry's past is known before the launch, or it has none
    int chunk;             // rows per chunk of k_diff
    int cpe;               // comparison blocks of every entry when all are alike, else 0
    int idx[DV_MAX_ENTRIES];        // table row of each entry
    uint32_t pslot[DV_MAX_ENTRIES]; // results-page position of each entry (DV_PG_*)
    int tbase[DV_MAX_ENTRIES + 1];  // first flat tile of each entry
    int bbase[DV_MAX_ENTRIES + 1];  // first flat band (32 rows) of each entry
    int cbase[DV_MAX_ENTRIES + 1];  // first block of each entry in the comparison kernels
};

// Rows that a block of k_diff takes at a time (a chunk), and leaves the counts
// of: 16 rows are one pass of its waves, which is the shortest chain where the
// chip is not full (1024^2 alone: 16 us with chunks of 64); with many frames
// chunks of 64 save block prologues and counts (20 frames of 4096^2).
#define DV_CHUNK_MIN 16
#define DV_CHUNK_MAX 64

// Blocks that the comparison (matching, k_diff, k_events) gives a frame:
// one per chunk of K_max rows, each block striding over the rest.  Each entry
// gets its own count: with the largest K_max of the launch for all of them, a
// group of 48 lattices of 256^2 .. 2048^2 launched 24,576 blocks per kernel,
// most of them empty.
// (an even number with chunks of 16 rows, so that the matching, whose blocks take 16
// points at a time, can have one for every two of them)
inline int compare_blocks(int kmax, int chunk) {
    const int b = (kmax + DV_CHUNK_MAX - 1) / DV_CHUNK_MAX * (DV_CHUNK_MAX / chunk);
    return b < 1024 ? b : 1024;
}

// Lattices whose labelling, from the finds on, and centres one block per frame
// does (k_mid): up to 512^2 sites.  There the four kernels it replaces are
// launches and latencies; a frame of 1024^2 would keep one block busy longer
// than they take.
#define CENTRES_MAX 4096     // most components whose centres one block makes
#define MID_TILES 256
#define MID_WORDS (MID_TILES * DV_TILE)
inline bool fits_mid(const Bufs &b) { return b.ncells <= MID_TILES && b.kmax <= CENTRES_MAX; }

// The comparison blocks of a launch of G.n entries with K_max kmax[i].
inline void set_compare_blocks(Batch &G, const int *kmax) {
    int total = 0;
    bool alike = true;
    for (int i = 0; i < G.n; ++i) {
        total += compare_blocks(kmax[i], DV_CHUNK_MAX);
        alike = alike && kmax[i] == kmax[0];
    }
    G.chunk = total <= 512 ? DV_CHUNK_MIN : DV_CHUNK_MAX;
    G.cbase[0] = 0;
    for (int i = 0; i < G.n; ++i) G.cbase[i + 1] = G.cbase[i] + compare_blocks(kmax[i], G.chunk);
    G.cpe = alike ? G.cbase[1] : 0;
}

// Comparison blocks per block of the matching: a block of 16 points for every 32
// rows of K_max with small chunks (one per 16 rows is too many empty blocks: 32
// frames of 256^2 with K_max 1024, 11 us against 7), for every 64 with large.
__host__ __device__ inline int match_blocks_div(int chunk) { return chunk == DV_CHUNK_MIN ? 2 : 1; }

// Entry holding flat index idx (base: prefix sums, n + 1 values; per: the
// common count when every entry has the same, else 0).
__device__ __forceinline__ int entry_of(const int *base, int per, int n, int idx) {
    if (per > 0) return idx / per;
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base[mid] <= idx) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Past of entry i of a launch, given the mask of accepted entries of its
// sequence: the last earlier one, else -1 for the sequence's past buffer.
__device__ __forceinline__ int past_slot(unsigned long long accepted, int i) {
    const unsigned long long m = accepted & ((1ull << i) - 1ull);
    return m ? 63 - __clzll(m) : -1;
}

// The same by a walk over the earlier entries with uniform (scalar) loads:
// cheaper where many waves each need it, since the entries' headers stay in
// the scalar cache.
// (In a launch whose entries all belong to different sequences there is
// nothing to walk: in a group of 48 the walk made k_diff 215 us, the matching 64 us.)
// Frames with one of the errors `bits` are passed over.
__device__ __forceinline__ int past_slot_walk(const Bufs *D, const Batch &G, int i, uint32_t bits) {
    if (G.alone) return -1;
    const int q = D[G.idx[i]].seq;
    for (int j = i - 1; j >= 0; --j)
        if (D[G.idx[j]].seq == q && (D[G.idx[j]].fs->err & bits) == 0) return j;
    return -1;
}

// Stage ids, in launch order (names in dv_api.hip).
enum {
    ST_TILE_CCL, ST_MERGE, ST_RESOLVE, ST_RELABEL, ST_FINALIZE, ST_OWNER_EDGES, ST_ROWS,
    ST_MATCH, ST_DIFF, ST_EVENTS, ST_PLACE, ST_COUNT
};

// Optional event bracketing of one stage (measurement only).
struct Prof {
    int stage = -1;          // stage to time, -1 none
    int cap = 0, used = 0;   // recorded launches
    hipEvent_t *ev = nullptr;  // [2 * cap]
    void begin(int id, hipStream_t s) {
        if (id == stage && used < cap) (void)hipEventRecord(ev[2 * used], s);
    }
    void end(int id, hipStream_t s) {
        if (id == stage && used < cap) {
            (void)hipEventRecord(ev[2 * used + 1], s);
            ++used;
        }
    }
};

// Bump placement of device buffers in one region, each piece 256-byte
// aligned; with a null base it only measures the region.
struct Carve {
    char *base = nullptr;
    size_t off = 0;
    template <class T>
    T *take(size_t count) {
        off = (off + 255) & ~(size_t)255;
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += (count ? count : 1) * sizeof(T);
        return p;
    }
};
// Buffers of one batch slot (one frame), and those shared by the slots of a
// sequence (past components, sequence header, results-page flips of
// page_frames frames each; the page records are placed by the caller).  B
// must hold the lattice, K_max, max_degree, the tile counts and keep_maps.
// (dv_api.hip)
void place_slot(Carve &cv, Bufs &b);
void place_shared(Carve &cv, Bufs &B, int page_frames);
// Checks of a configuration done before any device work, and the error text
// returned by dv_last_error(NULL) (dv_api.hip).
dv_status check_config(const dv_config *cfg);
dv_status fail_global(dv_status s, const char *msg);
// Slot-table fields of a configuration (lattice, tiles, threshold, flags):
// every pointer null (dv_api.hip).
Bufs table_base(const dv_config &cfg);

// Launchers (all on stream s).
// k_label.hip
void launch_label(const Batch &G, const Fields &F, hipStream_t s, Prof &P);
// k_voronoi.hip
void launch_voronoi(const Batch &G, hipStream_t s, Prof &P);
// k_diff.hip: comparison of every entry with its past, commit per sequence; the
// result of the launch that commits (k_place)
hipError_t launch_compare(const Batch &G, hipStream_t s, Prof &P);
// inspection helpers (k_diff.hip); slot: the most recent frame; par: the
// sequence header written last
void launch_obits(const Bufs &H, uint32_t *obits, hipStream_t s);   // obstacle bits from the mask
void launch_phi_out(const Bufs &H, const Bufs *D, int slot, int32_t *d_out, hipStream_t s);
void launch_edge_list(const Bufs &H, const Bufs *D, int par, int32_t *d_out_ab, int32_t *d_count,
                      int32_t *d_scratch, hipStream_t s);
