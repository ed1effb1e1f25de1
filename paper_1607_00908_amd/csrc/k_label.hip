// Cluster labelling and centre-of-mass sums (Sec. 3.1 of the paper).
//
// The lattice is cut into 32x32 tiles.  Per frame:
//   k_tile_ccl   threshold into row masks; union-find over the horizontal runs
//                of each tile in LDS; every tile-local root ("piece") gets an
//                entry in the global parent array (global linear site indices)
//                and a record with its size and coordinate sums.  What later
//                kernels need of the sites are the row masks (1 bit a site),
//                the piece slot of every run and the piece root of every
//                tile-border site (whole lines, read by k_merge);
//   k_merge      unions of pieces across tile borders and the periodic seams
//                (none across a wall);
//   k_resolve    per band of 32 rows: each piece finds its global root;
//                component roots (the smallest linear index of each component)
//                are marked in a bitmap of (row, tile column) segments, which
//                is scanned in raster order within the band;
//   k_rank       per piece: the canonical rank of its component (roots before
//                it in raster order), and its sums as exact integer offsets
//                from the component's root (signed minimum image), added to
//                the component's.
// The label map, when it is kept, is written with the colour map from the row
// masks and the runs' ranks.
// Union-find always links the larger index under the smaller one, so the root
// of every tree is its smallest index.
#include <algorithm>

#include "dv_device.h"

// v with lane `lane` replaced by the scalar s (v_writelane; the compiler has the
// operation as an intrinsic, not as a builtin)
extern "C" __device__ int dv_writelane(int s, int lane, int v) __asm("llvm.amdgcn.writelane.i32");

#define RES_TILES 1024   // tiles of a band handled per pass of k_resolve
#define RES_WORDS 8192   // segment words of a band held in LDS by k_resolve, at most
#define RES_BANDS 512    // bands from which k_resolve takes small blocks
#define MERGE_FEW 128    // tiles from which, and to which, a border has eight lanes in
#define MERGE_MANY 16384 // k_merge

// LDS of k_resolve for lattices of up to ntx tile columns (ints): segment words,
// and the prefix of the tiles' piece counts
__host__ __device__ inline int res_words(int ntx) {
    return ntx < RES_WORDS / DV_TILE ? ntx * DV_TILE : RES_WORDS;
}
__host__ __device__ inline int res_pre(int ntx) { return (ntx < RES_TILES ? ntx : RES_TILES) + 1; }

namespace {

// ---- union-find in LDS over tile-local indices -----------------------------
// Every parent is a smaller index than its child, so walks end at a root.
// Finds shorten the path they walk with plain stores (path splitting: a node
// gets its grandparent).  Such a store can replace a hook that another thread
// has just made on the same node; but that node had already stopped being a
// root, so the hooking thread's atomicMin returned its earlier parent and
// the thread retries with it: no union is lost.
__device__ __forceinline__ int lfind(int *L, int a) {
    int p = L[a];
    if (p == a) return a;
    int prev = a;
    for (;;) {
        const int next = L[p];
        if (next == p) return p;
        L[prev] = next;
        prev = p;
        p = next;
    }
}

__device__ void lunite(int *L, int a, int b) {
    bool done;
    do {
        a = lfind(L, a);
        b = lfind(L, b);
        if (a < b) {
            const int old = atomicMin(&L[b], a);
            done = (old == b);
            b = old;
        } else if (b < a) {
            const int old = atomicMin(&L[a], b);
            done = (old == a);
            a = old;
        } else {
            done = true;
        }
    } while (!done);
}

// ---- union-find in global memory over linear site indices -------------------
// gfind2 shortens paths as lfind does.  gfind_ro walks without writing: it is
// the find of a pass that also stores final roots, which a concurrent
// shortening store could otherwise replace with an intermediate ancestor.
__device__ __forceinline__ int gfind_ro(const gint *P, int a) {
    int p = P[a];
    while (p != a) {
        a = p;
        p = P[a];
    }
    return a;
}

// Finds of two nodes at once: the walks advance together, so the loads of a
// step are in flight together (a root's parent is itself, so both loads are
// always valid); each walk shortens its path (a node gets its grandparent, as
// in lfind), and each step moves to a smaller index, so both end.
__device__ __forceinline__ void gfind2(gint *P, int &a, int &b) {
    int pa = P[a], pb = P[b];
    int preva = a, prevb = b;
    bool da = pa == a, db = pb == b;
    while (!(da && db)) {
        const int na = P[pa], nb = P[pb];
        if (!da) {
            if (na == pa) {
                da = true;
            } else {
                P[preva] = na;
                preva = pa;
                pa = na;
            }
        }
        if (!db) {
            if (nb == pb) {
                db = true;
            } else {
                P[prevb] = nb;
                prevb = pb;
                pb = nb;
            }
        }
    }
    a = pa;
    b = pb;
}

// Hooks the larger of a, b under the smaller before any find: the pieces at a
// tile border are mostly still their own roots, and then that is the union (one
// exchange instead of two finds and one).  A larger one that was hooked already
// keeps the lower of its two parents, and the parents are united instead.
__device__ __forceinline__ void gunite(gint *P, int a, int b) {
    for (bool first = true; a != b; first = false) {
        if (!first) gfind2(P, a, b);
        const int lo = min(a, b), hi = max(a, b);
        if (lo == hi) return;
        const int old = __hip_atomic_fetch_min(P + hi, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == hi) return;
        a = lo;
        b = old;
    }
}

// Site weight of the density-weighted centres (centroid equation of Sec. 2):
// the field value quantised to 1/256, clamped to [1, 65535]: floor(256 rho + 1/2),
// exactly, by 32-bit floats: the product is exact, and in [1, 65535] the sum can
// only be rounded where it passes a power of two, by less than takes it to the
// next integer.  (The same weight as by 64-bit floats for all 2^32 values of rho;
// NaN and what lies below give 1.)
__device__ __forceinline__ int site_weight(float rho) {
    return (int)(fminf(fmaxf(256.0f * rho, 1.0f), 65535.0f) + 0.5f);
}

// bits 0 .. x (x <= 31)
__device__ __forceinline__ uint32_t bits_to(int x) { return (2u << x) - 1u; }

// length of the run that starts at column a of a row with inside mask m
__device__ __forceinline__ int run_length(uint32_t m, int a) {
    return __builtin_ctzll(~(unsigned long long)(m >> a));   // a full row is 32
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(unsigned v) { return __builtin_bit_cast(u16x2, v); }

// 32 x 32 bits, row y in lane y of each half of the wave: bit y of lane x becomes
// bit x of row y.  (Every lane must make the call.)
__device__ __forceinline__ uint32_t transpose32(uint32_t v, int lane) {
    auto step = [&](uint32_t x, int j, uint32_t m) {   // x: the value of lane ^ j
        const bool up = lane & j;
        const uint32_t keep = up ? ~m : m;
        const uint32_t r = __builtin_amdgcn_alignbit(x, x, up ? j : 32 - j);
        v = (v & keep) | (r & ~keep);
    };
    auto quad = [](uint32_t x) { return __builtin_amdgcn_update_dpp(0, (int)x, 0x1b, 0xf, 0xf, false); };
    step((uint32_t)__shfl_xor((int)v, 16, 64), 16, 0x0000ffffu);
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false), 8, 0x00ff00ffu);   // row_ror:8
    step((uint32_t)quad((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false)), 4,
         0x0f0f0f0fu);                                                                  // ^ 7 (half mirror), ^ 3
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, false), 2, 0x33333333u);
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false), 1, 0x55555555u);
    return v;
}

// The fields of a launch that exceed half the last-level cache (256 MiB), which
// what the launch writes goes through too, are read past it; smaller ones may be in
// it still.  (20 fields of 4096^2: 322 us through it, 304 past it; 48 fields of
// 200 MiB together, of which the next launch brings others: 88 and 67; one of
// 4096^2: 25 and 28; 32 of 1024^2: 38 and 40.)
#define STREAM_TILES 32768   // of 32 x 32 sites of 4 bytes
#define ACC_PIECES 64    // pieces whose sums are in LDS at a time

// One wave per tile, four tiles per block.  (GEOM: some entry of the launch has
// walls or obstacles; WT: some entry has weighted centres; NT: the fields are read
// past the cache; the other instances carry none of their code.)  The field is read with lane l on column l & 31 and
// the rows (l >> 5) + 2k, k = 0..15, so that every wave load covers two whole
// rows and its ballot is two row masks.  From there on nothing is done per
// site: lane y holds the mask of row y, and the union-find, the piece slots and
// the sums run over the horizontal runs (about 40 in a tile of droplets),
// numbered in raster order, so that the smallest run of a piece starts at its
// smallest site.  A wave waits for nothing but its own LDS accesses, so the
// tiles of a block overlap their latencies.  What is written per tile is 128
// bytes of masks, 256 of border roots, 2 bytes a run and 8 a piece.
template <bool GEOM, bool WT, bool NT>
__global__ __launch_bounds__(256, WT ? 4 : 8) void k_tile_ccl(const Bufs *__restrict__ D, Batch G, Fields F) {
    // (the same for every lane of the wave: read once, so that the slot's
    // fields are loaded into scalar registers)
    const int gt = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (gt >= G.tiles) return;   // a whole wave; there is no block barrier below
    const int e = entry_of(G.tbase, G.tpe, G.n, gt);
    const Bufs B = D[G.idx[e]];   // (a copy: the loads are not repeated after stores)
    // per wave: union-find over the runs (after the slots are assigned, a root's
    // entry also holds its slot in bits 16..), first site of each run, sums of
    // the pieces in their record's form
    __shared__ int Ls[4][DV_TILE_PIECES];
    __shared__ uint16_t Rs[4][DV_TILE_PIECES];
    __shared__ unsigned long long accs[4][ACC_PIECES];
    __shared__ unsigned accws[WT ? 4 : 1][3][ACC_PIECES];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int *L = Ls[w];
    uint16_t *R = Rs[w];
    unsigned long long *acc = accs[w];
    const int tile = gt - G.tbase[e];
    const int tx = tile % B.ntx, ty = tile / B.ntx;
    const int x0 = tx * DV_TILE, y0 = ty * DV_TILE;
    const int tw = min(DV_TILE, B.lx - x0), th = min(DV_TILE, B.ly - y0);
    FrameState *fs = B.fs;
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    const int cx = lane & 31, h = lane >> 5;
    // the field (and obstacle) values of the lane's sites, loads issued
    // together; beyond a ragged tile's edge a lane reads the nearest site of
    // the tile and ignores it
    const float *field = F.p[e];
    const size_t tbase = (size_t)y0 * B.lx + x0;
    const int xc = min(cx, tw - 1);
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const float *at = field + (tbase + (size_t)(min(h + 2 * k, th - 1) * B.lx + xc));
        v[k] = NT ? __builtin_nontemporal_load(at) : *at;
    }
    uint32_t ob = 0;   // lane y < 32: obstacle bits of row y
    if (GEOM && B.obits) ob = gmem(B.obits)[(size_t)tile * DV_OBITS + 1 + cx];
    // per-frame resets spread over the grid
    if (tile == 0 && lane == 0) {
        fs->K_now = 0;
        fs->err = 0;
        fs->n_amb = 0;
        fs->nb_acc = 0;
        fs->na_acc = 0;
    }
    if (gt == 0) {   // the launch's lists of tiles for the general colouring
        gmem(B.gen_n)[lane * DV_LINE] = 0;
        if (lane == 0) gmem(B.gen_n)[1] = 0;
    }
    if (lane == 0) {
        gmem(B.cell_count)[tile] = 0;
        gmem(B.cell_head)[tile] = -1;
        if ((tile & 255) == 0) gmem(B.cell_sum)[(tile >> 8) * DV_LINE] = 0;
    }
    {   // empty the rows this frame will fill
        const size_t rows = (size_t)fs->rows_dirty;
        const size_t stride = (size_t)B.ncells * 64;
        auto adj = gmem(B.cur.adj);
        for (size_t i = (size_t)tile * 64 + lane; i < rows * B.prim; i += stride) adj[i] = DV_EMPTY;
        if (fs->spill) {
            auto adjx = gmem(B.cur.adjx);
            const size_t total = rows * (B.maxdeg - B.prim);
            for (size_t i = (size_t)tile * 64 + lane; i < total; i += stride) adjx[i] = DV_EMPTY;
        }
    }
    int mi = 0;   // lane y < 32: inside mask of row y
    // (only the threshold is tested per site, and what lies beyond the tile is masked
    // out by rows: 20 frames of 4096^2 from 343 to 322 us)
    auto row_masks = [&](auto inside) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const unsigned long long bal = __ballot(inside(v[k]));
            mi = dv_writelane((int)(unsigned)bal, 2 * k, mi);
            mi = dv_writelane((int)(unsigned)(bal >> 32), 2 * k + 1, mi);
        }
    };
    if (B.phase == 0) row_masks([&](float x) { return x > B.thr; });
    else row_masks([&](float x) { return x < B.thr; });
    mi = lane < th ? mi & (int)(bits_to(tw - 1) & ~ob) : 0;
    const uint32_t m = (uint32_t)mi;
    if (lane < DV_TILE) gmem(B.tmask)[(size_t)tile * DV_TILE + lane] = m;
    // runs of the row and their numbers
    const uint32_t st = m & ~(m << 1);
    const int rc = __popc(st);
    const int rinc = wave_incl_sum(rc);
    const int rbase = rinc - rc, nruns = wave_last(rinc);
    for (int i = lane; i < nruns; i += 64) L[i] = i;
    wave_sync();
    // Unions of each run [a, b] with the runs of the row above that touch
    // it: columns a - 1 .. b + 1 (8-connectivity) or a .. b (4): the run
    // holding the lowest touching site of the row above, and every other
    // run of that row starting inside the span (their numbers follow).
    {
        const uint32_t up = (uint32_t)wave_prev(mi, 0);
        const uint32_t st_up = up & ~(up << 1);
        const int base_up = wave_prev(rbase, 0);
        uint32_t rst = st;
        for (int id = rbase; rst; ++id) {
            const int a = __ffs(rst) - 1;
            rst &= rst - 1;
            R[id] = (uint16_t)((lane << 5) | a);
            const int b = a + run_length(m, a) - 1;
            const int lo = (B.conn == 8 && a > 0) ? a - 1 : a;
            const int hi = (B.conn == 8 && b < 31) ? b + 1 : b;
            const uint32_t hit = up & bits_to(hi) & ~((1u << lo) - 1u);
            if (!hit) continue;
            const uint32_t first = bits_to(__ffs(hit) - 1);
            const int id0 = base_up + __popc(st_up & first) - 1;
            const int others = __popc(st_up & hit & ~first);
            for (int q = 0; q <= others; ++q) lunite(L, id, id0 + q);
        }
    }
    wave_sync();
    // roots by pointer jumping (a chain down the rows halves in every step)
    for (bool more = nruns > 0; more;) {
        bool ch = false;
        for (int i = lane; i < nruns; i += 64) {
            const int p = L[i], g = L[p];
            L[i] = g;
            ch |= p != g;
        }
        wave_sync();
        more = __ballot(ch) != 0ull;
    }
    // piece roots take consecutive slots in run order (a wave prefix); the slot
    // goes into bits 16.. of the root's entry
    int npc = 0;
    for (int i0 = 0; i0 < nruns; i0 += 64) {
        const int i = i0 + lane;
        const bool pr = i < nruns && L[i] == i;
        const unsigned long long bal = __ballot(pr);
        if (pr) {
            L[i] = i | ((npc + __popcll(bal & ((1ull << lane) - 1ull))) << 16);
            const int s = R[i];
            const int g = (y0 + (s >> 5)) * B.lx + x0 + (s & 31);
            gmem(B.parent)[g] = g;
        }
        npc += __popcll(bal);
    }
    wave_sync();
    // Sums of the pieces (a pass per ACC_PIECES of them: one in the usual case):
    // each run adds its length and the sums of its coordinates in closed form.
    for (int p0 = 0; p0 < npc; p0 += ACC_PIECES) {
        for (int i0 = 0; i0 < nruns; i0 += 64) {
            const int i = i0 + lane, en = i < nruns ? L[i] : 0;
            const int slot = (en >> 16) - p0;
            if (i < nruns && (en & 0xffff) == i && slot >= 0 && slot < ACC_PIECES)
                acc[slot] = (unsigned long long)R[i] << 48;
        }
        if (WT)
            for (int k = 0; k < 3; ++k) accws[w][k][lane] = 0u;
        wave_sync();
        for (int i0 = 0; i0 < nruns; i0 += 64) {
            const int i = i0 + lane;
            const bool on = i < nruns;
            const int s = on ? R[i] : 0;
            const uint32_t my = (uint32_t)__shfl(mi, s >> 5, 64);
            const int slot = on ? L[L[i] & 0xffff] >> 16 : 0;
            if (on && p0 == 0) {
                gmem(B.trun)[run_at(B, tile, i)] = (uint16_t)slot;
                if (WT) L[i] = (L[i] & 0xffff) | (slot << 16);   // (a root's is there)
            }
            if (on && slot >= p0 && slot < p0 + ACC_PIECES) {
                const int a = s & 31, len = run_length(my, a);
                const unsigned sx = (unsigned)((2 * a + len - 1) * len) >> 1;
                const unsigned sy = (unsigned)((s >> 5) * len);
                atomicAdd(&acc[slot - p0],
                          (unsigned long long)((unsigned)len | (sx << 16)) | ((unsigned long long)sy << 32));
            }
        }
        if (WT && B.weighted) {
            wave_sync();
            // weights: the sites of a vertical run of a column belong to one piece,
            // so each lane takes its column's runs in turn and adds up its rows'
            // sites of the run, two rows an instruction
            // (Prefix sums along the rows by lane moves, each end of a horizontal run
            // adding its sum, weights by 64-bit floats: 156 us per 16 frames of
            // 2048^2, 850 VALU and 690 SALU instructions a tile; this way 101 us,
            // 700 and 490.)
            unsigned wp[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                wp[k] = (unsigned)site_weight(v[k]) | ((unsigned)site_weight(v[k + 8]) << 16);
            uint32_t rem = transpose32((uint32_t)__shfl(mi, cx, 64), lane);
            while (__ballot(rem != 0u)) {
                const uint32_t low = rem & (0u - rem), sum = rem + low, run = rem & ~sum;
                rem &= sum;
                const int y = low ? __builtin_ctz(low) : 0;
                // (lane moves: every lane takes part)
                const uint32_t my = (uint32_t)__shfl(mi, y, 64);
                const int by = __shfl(rbase, y, 64);
                unsigned aw = 0, ay = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const u16x2 on = as_u16x2(((run >> h) >> (2 * k)) & 0x00010001u);
                    const u16x2 at = {(unsigned short)(2 * k), (unsigned short)(2 * k + 16)};
                    aw = __builtin_amdgcn_udot2(as_u16x2(wp[k]), on, aw, false);
                    ay = __builtin_amdgcn_udot2(as_u16x2(wp[k]), on * at, ay, false);
                }
                ay += h ? aw : 0u;
                if (aw) {
                    const int slot = (L[by + __popc(my & ~(my << 1) & bits_to(cx)) - 1] >> 16) - p0;
                    if (slot >= 0 && slot < ACC_PIECES) {
                        atomicAdd(&accws[w][0][slot], aw);
                        atomicAdd(&accws[w][1][slot], aw * (unsigned)cx);
                        atomicAdd(&accws[w][2][slot], ay);
                    }
                }
            }
        }
        wave_sync();
        if (p0 + lane < npc) {
            const size_t at = piece_at(B, tile, p0 + lane);
            unsigned long long rec = acc[lane];
            if (WT && B.weighted) {
                const unsigned sw = accws[w][0][lane];
                rec = PIECE_WEIGHTED(rec, sw, accws[w][1][lane]);
                gmem(B.prank)[at] = (int)accws[w][2][lane];
                gmem(reinterpret_cast<uint16_t *>(B.tpairs))[at] = (uint16_t)sw;
            }
            gmem(B.tpiece)[at] = rec;
        }
        wave_sync();
    }
    // the border array: piece root of each border site (0xffff outside, also
    // beyond a ragged tile's edge, so that merging needs no field), two whole
    // lines per lane: top and bottom row, left and right column
    {
        auto bp = gmem(B.bpc) + (size_t)tile * DV_BORDER;
        auto root_of = [&](bool in, int i) {
            return in ? (int)R[L[in ? i : 0] & 0xffff] : 0xffff;
        };
        const uint32_t mr = (uint32_t)(h ? __builtin_amdgcn_readlane(mi, th - 1) : __builtin_amdgcn_readlane(mi, 0));
        const int br = h ? __builtin_amdgcn_readlane(rbase, th - 1) : 0;
        const int a = root_of((mr >> cx) & 1u, br + __popc(mr & ~(mr << 1) & bits_to(cx)) - 1);
        const uint32_t mc = (uint32_t)__shfl(mi, cx, 64);
        const int bc = __shfl(rbase, cx, 64), nc = __popc(mc & ~(mc << 1));
        const int b = h == 0 ? root_of(mc & 1u, bc) : root_of((mc >> (tw - 1)) & 1u, bc + nc - 1);
        bp[lane] = (uint16_t)a;
        bp[2 * DV_TILE + lane] = (uint16_t)b;
        // inside bits of the four lines
        const uint32_t top = (uint32_t)__builtin_amdgcn_readlane(mi, 0);
        const uint32_t bottom = (uint32_t)__builtin_amdgcn_readlane(mi, th - 1);
        const unsigned long long sides = __ballot(((h ? mc >> (tw - 1) : mc) & 1u) != 0u);
        const uint32_t edge = lane == 0 ? top : lane == 1 ? bottom : lane == 2 ? (uint32_t)sides : (uint32_t)(sides >> 32);
        if (lane < 4) gmem(B.tedge)[(size_t)tile * 4 + lane] = edge;
    }
    if (lane == 0) gmem(B.npieces)[tile] = npc;
}

// Unions between inside sites of neighbouring tiles.  A lane per border: the
// lower half of a wave takes the last column of 32 tiles against the next
// column (periodic), the upper half their last row against the next row.
// Together they cover every adjacent pair that crosses a tile border, including
// the diagonal pairs at tile corners and the periodic seams; a pair across a
// wall is not formed.  The sites of a run along the border belong to one piece,
// so what is united is pairs of runs that touch, found from the lines' inside
// bits (the neighbour's with one site more at either end, which belongs to the
// diagonal neighbours), and a union is two piece roots read from the border
// arrays and usually one exchange.  (A lane per border site, with the pairs of
// neighbouring lanes compared to drop repeated ones: 243 us per 20 frames of
// 4096^2, 305 VALU instructions per tile; this way 42 us.)
// LANES: lanes of a border, each for the runs that start in its part.  Borders with
// many runs are the longest chains, so eight where the chip is not full: a frame of
// 512^2 of percolating noise 63 us with one lane, 23 with eight, one of 4096^2 of a
// random field 9.6 and 7.6; but 32 of 1024^2 4.8 and 6.1, 48 mixed fields 13.7 and
// 17.8, and one of 256^2, two blocks in place of one, 3.2 and 3.8.
template <bool GEOM, int LANES>
__global__ __launch_bounds__(256) void k_merge(const Bufs *__restrict__ D, Batch G) {
    const int t = threadIdx.x, side = (t >> 5) & 1;   // 0: last column, 1: last row
    const int gt = (blockIdx.x * 128 + (t >> 6) * 32 + (t & 31)) / LANES, part = t % LANES;
    if (gt >= G.tiles) return;
    const int e = entry_of(G.tbase, G.tpe, G.n, gt);
    const Bufs &B = D[G.idx[e]];
    const int tile = gt - G.tbase[e];
    const int ntx = B.ntx, nty = B.nty, lx = B.lx, ly = B.ly;
    const int tx = tile % ntx, ty = tile / ntx;
    const bool ox = GEOM && B.open_x, oy = GEOM && B.open_y;
    const bool right = tx + 1 == ntx, last = ty + 1 == nty;
    if (side ? oy && last : ox && right) return;
    const int xn = right ? 0 : tx + 1, yn = last ? 0 : ty + 1;
    const int xp = tx == 0 ? ntx - 1 : tx - 1, yp = ty == 0 ? nty - 1 : ty - 1;
    // the neighbour, and the diagonal ones before and after it along the line
    const int nx = side ? tx : xn, ny = side ? yn : ty;
    const int px = side ? xp : xn, py = side ? yn : yp;
    const int qx = xn, qy = yn;
    const bool pcut = side ? ox && tx == 0 : oy && ty == 0;
    const bool qcut = side ? ox && right : oy && last;
    const int tn = ny * ntx + nx, tp = py * ntx + px, tq = qy * ntx + qx;
    const int len = side ? min(DV_TILE, lx - tx * DV_TILE) : min(DV_TILE, ly - ty * DV_TILE);
    const int plen = side ? min(DV_TILE, lx - px * DV_TILE) : min(DV_TILE, ly - py * DV_TILE);
    const auto edge = gmem(B.tedge);
    const uint32_t own = edge[(size_t)tile * 4 + (side ? 1 : 3)];
    const int line = side ? 0 : 2;   // the neighbours' line: first row, first column
    const uint32_t mn = edge[(size_t)tn * 4 + line], mp = edge[(size_t)tp * 4 + line], mq = edge[(size_t)tq * 4 + line];
    if (!own) return;
    // bit k + 1: position k of the neighbour's line (-1 and len: the diagonal ones)
    const unsigned long long nb = ((unsigned long long)mn << 1) |
                                  (pcut ? 0ull : (unsigned long long)((mp >> (plen - 1)) & 1u)) |
                                  (qcut ? 0ull : (unsigned long long)(mq & 1u) << (len + 1));
    const auto bp = gmem(B.bpc);
    // piece root (linear index) at position k of a line of tile (cx, cy)
    auto piece = [&](int cx, int cy, int at) -> int {
        const int v = bp[(size_t)(cy * ntx + cx) * DV_BORDER + at];
        return (cy * DV_TILE + (v >> 5)) * lx + cx * DV_TILE + (v & 31);
    };
    gint *P = gmem(B.parent);
    const bool conn8 = B.conn == 8;
    // the starts of the lane's runs (one lane: what is left of the line)
    uint32_t rest = own;
    if (LANES > 1) rest &= ~(own << 1) & (bits_to(DV_TILE / LANES - 1) << (part * (DV_TILE / LANES)));
    while (rest) {
        const int a = __ffs(rest) - 1, b = a + run_length(own, a) - 1;
        rest &= LANES > 1 ? rest - 1u : ~(bits_to(b) & ~((1u << a) - 1u));
        // positions a - 1 .. b + 1 (4-connectivity: a .. b)
        const int lo = conn8 ? a : a + 1, hi = conn8 ? b + 2 : b + 1;
        unsigned long long hit = nb & ((2ull << hi) - 1ull) & ~((1ull << lo) - 1ull);
        // one site of each run, on the neighbour's own line where it has one there
        // (a diagonal neighbour's site next to it is united with it along the
        // other border)
        if (hit & 2ull) hit &= ~1ull;
        hit &= ~(hit << 1);
        if (!hit) continue;
        const int pa = piece(tx, ty, (side ? DV_TILE : 3 * DV_TILE) + a);
        for (; hit; hit &= hit - 1) {
            const int k = (int)__builtin_ctzll(hit) - 1;
            const int pb = k < 0 ? piece(px, py, line * DV_TILE + plen - 1)
                                 : k >= len ? piece(qx, qy, line * DV_TILE) : piece(nx, ny, line * DV_TILE + k);
            gunite(P, pa, pb);
        }
    }
}

// One block per band of 32 rows: every piece of the band's tiles finds its
// component root (the smallest linear index of the component); component
// roots set their bit in the band's (row, tile column) segment words, which
// are then scanned in raster order.  A segment's entry holds its bits and the
// number of roots before it within the band, band_sum the band's total.
// Segment (y, tile column c) covers sites y*lx + 32c .. 32c+31, so raster
// order of segments is the row-major order of the [ly][ntx] array.
// The words live in LDS while the band has at most RES_WORDS of them (lattices
// up to 8192 wide), else in the segments themselves.
// A band is a chain of dependent loads and barriers, so many bands take small
// blocks with no more LDS than the widest needs, of which eight fit a CU
// (launches of few bands: wide blocks, which take a band in fewer steps).
// (Blocks of 1024 threads with 36 KB for every band, a word a thread: 69 us per 20
// frames of 4096^2, 15 per 32 of 1024^2, 29 per 48 mixed ones; this way 42, 8 and
// 14; one frame of 4096^2 12 and 9.)
__global__ __launch_bounds__(1024) void k_resolve(const Bufs *__restrict__ D, Batch G) {
    const int e = entry_of(G.bbase, G.bpe, G.n, blockIdx.x);
    const Bufs B = D[G.idx[e]];
    extern __shared__ __align__(16) int lds[];
    __shared__ int wsum[16];
    const int nwords = res_words(G.ntx);
    uint32_t *words = reinterpret_cast<uint32_t *>(lds);
    int *pre = lds + nwords;   // res_pre(G.ntx)
    const int ty = blockIdx.x - G.bbase[e], t = threadIdx.x;
    const int y0 = ty * DV_TILE, th = min(DV_TILE, B.ly - y0);
    const int ntx = B.ntx;
    const int n = th * ntx, n4 = (n + 3) & ~3;
    uint2 *seg = B.seg + (size_t)y0 * ntx;
    const bool in_lds = n <= nwords;
    if (in_lds)
        for (int i = 4 * t; i < n4; i += 4 * blockDim.x) *reinterpret_cast<uint4 *>(words + i) = make_uint4(0, 0, 0, 0);
    else
        for (int i = t; i < n; i += blockDim.x) seg[i].x = 0u;
    __syncthreads();
    for (int c0 = 0; c0 < ntx; c0 += RES_TILES) {
        const int nt = min(RES_TILES, ntx - c0);
        const int tile0 = ty * ntx + c0;
        // pieces of tiles c0 .. c0 + nt - 1, numbered through a block scan
        const int total = block_exclusive_scan(B.npieces + tile0, pre, nt, wsum);
        __syncthreads();
        for (int f = t; f < total; f += blockDim.x) {
            int lo = 0, hi = nt - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= f) lo = mid; else hi = mid - 1;
            }
            const int tx = c0 + lo;
            const int r = PIECE_ROOT(gmem(B.tpiece)[piece_at(B, tile0 + lo, f - pre[lo])]);
            const int g = (y0 + (r >> 5)) * B.lx + tx * DV_TILE + (r & 31);
            const int root = gfind_ro(gmem(B.parent), g);
            const int word = (r >> 5) * ntx + tx;
            if (root != g) gmem(B.parent)[g] = root;
            else if (in_lds) atomicOr(&words[word], 1u << (r & 31));
            else atomicOr(&seg[word].x, 1u << (r & 31));
        }
        __syncthreads();
    }
    // raster-order prefix of the root bits within the band, four words a thread
    const int lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;
    int carry = 0;
    for (int c0 = 0; c0 < n; c0 += 4 * blockDim.x) {
        const int i = c0 + 4 * t;
        uint4 b = make_uint4(0, 0, 0, 0);
        if (in_lds && i < n) b = *reinterpret_cast<const uint4 *>(words + i);
        if (!in_lds) {
            b.x = i < n ? seg[i].x : 0u;
            b.y = i + 1 < n ? seg[i + 1].x : 0u;
            b.z = i + 2 < n ? seg[i + 2].x : 0u;
            b.w = i + 3 < n ? seg[i + 3].x : 0u;
        }
        const int p1 = __popc(b.x), p2 = p1 + __popc(b.y), p3 = p2 + __popc(b.z), v = p3 + __popc(b.w);
        const int x = wave_incl_sum(v);
        __syncthreads();
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        int before = carry + x - v;
        for (int w = 0; w < wid; ++w) before += wsum[w];
        // (a band starts at a multiple of 32 entries)
        if (i + 3 < n) {
            uint4 *to = reinterpret_cast<uint4 *>(seg + i);
            to[0] = make_uint4(b.x, before, b.y, before + p1);
            to[1] = make_uint4(b.z, before + p2, b.w, before + p3);
        } else {
            if (i < n) seg[i] = make_uint2(b.x, before);
            if (i + 1 < n) seg[i + 1] = make_uint2(b.y, before + p1);
            if (i + 2 < n) seg[i + 2] = make_uint2(b.z, before + p2);
        }
        int tot = 0;
        for (int w = 0; w < nw; ++w) tot += wsum[w];
        carry += tot;
    }
    if (t == 0) B.band_sum[ty] = carry;
}

__device__ __forceinline__ int wrap_off(int v, int L) {
    // v in (-L, L) -> signed minimum image in [-floor(L/2), L-1-floor(L/2)]
    const int h = L >> 1;
    if (v > L - 1 - h) v -= L;
    else if (v < -h) v += L;
    return v;
}

// Offsets of a component's sites from its root (gx, gy): minimum image on a
// periodic axis; on a walled axis plain differences (wrap_off over twice the
// length changes nothing), and no antipodal line to cross.
struct RootFrame {
    int gx, gy, wlx, wly, hix, hiy;
    __device__ RootFrame(const Bufs &B, int root) {
        gx = root % B.lx;
        gy = root / B.lx;
        wlx = B.open_x ? 2 * B.lx : B.lx;
        wly = B.open_y ? 2 * B.ly : B.ly;
        hix = B.open_x ? INT_MAX : B.lx - 1 - (B.lx >> 1);
        hiy = B.open_y ? INT_MAX : B.ly - 1 - (B.ly >> 1);
    }
    __device__ int dx(int x) const { return wrap_off(x - gx, wlx); }
    __device__ int dy(int y) const { return wrap_off(y - gy, wly); }
};

// The sums of the pieces of a tile that belong to one component (the bits `pieces`
// by slot - slot0) and meet its root's antipodal lines, run by run (site by site
// where the line cuts a run), by the whole wave: lane y takes the runs of row y.
// A site on the line with an adjacent inside site beyond it (a member: the unwrapped
// coordinates jump by L - 1 between them) makes the component ambiguous.
// (A pass over the tile for each of its pieces, with atomics by every lane: k_mid 208
// us for one frame of 512^2 of percolating noise and 132 for 256^2; this way 135 and
// 63.)
template <bool WT>
__device__ void piece_sums_by_run(const Bufs &B, const float *field, int tile, int slot0,
                                  unsigned long long pieces, int root, int rank, int lane) {
    const int x0 = (tile % B.ntx) * DV_TILE, y0 = (tile / B.ntx) * DV_TILE;
    const int lx = B.lx, ly = B.ly;
    const RootFrame O(B, root);
    const uint32_t m = lane < DV_TILE ? gmem(B.tmask)[(size_t)tile * DV_TILE + lane] : 0u;
    uint32_t st = m & ~(m << 1);
    const int rc = __popc(st);
    const int rbase = wave_incl_sum(rc) - rc;
    auto inside_at = [&](int xx, int yy) {
        const size_t tl = (size_t)(yy >> 5) * B.ntx + (xx >> 5);
        return (gmem(B.tmask)[tl * DV_TILE + (yy & 31)] >> (xx & 31)) & 1u;
    };
    const bool wt = WT && B.weighted;
    long long sx = 0, sy = 0, sw = 0;
    int n = 0;
    bool amb = false;
    for (int i = rbase; st; ++i) {
        const int a = __ffs(st) - 1;
        st &= st - 1;
        const int at = gmem(B.trun)[run_at(B, tile, i)] - slot0;
        if (at < 0 || at > 63 || !((pieces >> at) & 1ull)) continue;
        const int len = run_length(m, a), gy = y0 + lane;
        const int dy = O.dy(gy), dxa = O.dx(x0 + a), dxe = O.dx(x0 + a + len - 1);
        n += len;
        for (int k = 0; k < len; ++k) {
            const int w = wt ? site_weight(field[(size_t)gy * lx + x0 + a + k]) : 1;
            sx += (long long)w * O.dx(x0 + a + k);
            sy += (long long)w * dy;
            sw += w;
        }
        if (dy != O.hiy && dxe - dxa == len - 1 && !(dxa <= O.hix && O.hix <= dxe)) continue;
        const int yp = gy + 1 == ly ? 0 : gy + 1, ym = gy == 0 ? ly - 1 : gy - 1;
        for (int k = 0; k < len; ++k) {
            const int gx = x0 + a + k;
            const int dxk = O.dx(gx);
            if (dxk != O.hix && dy != O.hiy) continue;
            const int xp = gx + 1 == lx ? 0 : gx + 1, xm = gx == 0 ? lx - 1 : gx - 1;
            // (a diagonal neighbour around a seam that a wall closes is none)
            if (dxk == O.hix) {
                amb = amb || inside_at(xp, gy);
                if (B.conn == 8)
                    amb = amb || (inside_at(xp, ym) && !(B.open_y && gy == 0)) ||
                          (inside_at(xp, yp) && !(B.open_y && yp == 0));
            }
            if (dy == O.hiy) {
                amb = amb || inside_at(gx, yp);
                if (B.conn == 8)
                    amb = amb || (inside_at(xm, yp) && !(B.open_x && gx == 0)) ||
                          (inside_at(xp, yp) && !(B.open_x && xp == 0));
            }
        }
    }
    for (int o = 1; o < 64; o <<= 1) {
        sx += __shfl_xor(sx, o, 64);
        sy += __shfl_xor(sy, o, 64);
        if (wt) sw += __shfl_xor(sw, o, 64);
        n += __shfl_xor(n, o, 64);
    }
    const bool any = __ballot(amb) != 0ull;
    if (lane == 0) {
        atomicAdd(&B.acc_n[rank], n);
        atomicAdd((unsigned long long *)&B.acc_x[rank], (unsigned long long)sx);
        atomicAdd((unsigned long long *)&B.acc_y[rank], (unsigned long long)sy);
        if (wt) atomicAdd((unsigned long long *)&B.acc_w[rank], (unsigned long long)sw);
        if (any) atomicOr(&B.acc_amb[rank], 1);
    }
}

// Piece k of a tile: the canonical rank of its component (rank_of: of the
// component root's site), by piece slot, and its contribution to the
// component's sums: the sums of its tile-local coordinates moved by the offset
// of the tile's corner.  That holds when the tile meets neither antipodal line
// of the root (where the minimum image jumps, or the ambiguity of the component
// shows); other pieces, which are rare, are summed by run.  The component root's
// piece records the root for the centre.  Every lane of the wave makes the call;
// `have`: the lane has a piece.  The pieces of a tile in the wave are consecutive
// ones in consecutive lanes.
template <bool WT, class RankOf>
__device__ __forceinline__ void add_piece(const Bufs &B, const float *field, int tile, int k, bool have,
                                          RankOf rank_of) {
    const int lx = B.lx, lane = threadIdx.x & 63;
    const int x0 = (tile % B.ntx) * DV_TILE, y0 = (tile / B.ntx) * DV_TILE;
    const int tw = min(DV_TILE, lx - x0), th = min(DV_TILE, B.ly - y0);
    bool by_run = false;
    int Gr = 0, rank = 0;
    if (have) {
        const size_t at = piece_at(B, tile, k);
        const unsigned long long rec = gmem(B.tpiece)[at];
        unsigned wlow = 0, wy = 0;
        if (WT && B.weighted) {   // (the rank will take wy's place)
            wlow = gmem(reinterpret_cast<const uint16_t *>(B.tpairs))[at];
            wy = (unsigned)gmem(B.prank)[at];
        }
        const int r = PIECE_ROOT(rec), n = PIECE_N(rec);
        const int g = (y0 + (r >> 5)) * lx + x0 + (r & 31);
        Gr = gmem(B.parent)[g];    // component root (compressed)
        const RootFrame O(B, Gr);
        rank = rank_of(O.gx, O.gy);
        gmem(B.prank)[at] = rank;
        if (rank < B.kmax) {
            if (Gr == g) gmem(B.acc_root)[rank] = Gr;
            const int dx = O.dx(x0), dxe = O.dx(x0 + tw - 1), dy = O.dy(y0), dye = O.dy(y0 + th - 1);
            by_run = dxe - dx != tw - 1 || dye - dy != th - 1 || (dx <= O.hix && O.hix <= dxe) ||
                     (dy <= O.hiy && O.hiy <= dye);
            if (!by_run) {
                long long sx = PIECE_SX(rec) + n * dx, sy = PIECE_SY(rec) + n * dy;
                if (WT && B.weighted) {
                    const long long sw = PIECE_W(rec, wlow);
                    sx = PIECE_WX(rec) + sw * dx;
                    sy = wy + sw * dy;
                    atomicAdd((unsigned long long *)&B.acc_w[rank], (unsigned long long)sw);
                }
                atomicAdd((unsigned long long *)&B.acc_x[rank], (unsigned long long)sx);
                atomicAdd((unsigned long long *)&B.acc_y[rank], (unsigned long long)sy);
                atomicAdd(&B.acc_n[rank], n);
            }
        }
    }
    // (a tile's pieces of one component together)
    for (unsigned long long w = __ballot(by_run); w;) {
        const int l = __builtin_ctzll(w);
        const int t0 = __builtin_amdgcn_readlane(tile, l), root = __builtin_amdgcn_readlane(Gr, l);
        const unsigned long long same = __ballot(by_run && tile == t0 && Gr == root);
        piece_sums_by_run<WT>(B, field, t0, __builtin_amdgcn_readlane(k, l), same >> l, root,
                              __builtin_amdgcn_readlane(rank, l), lane);
        w &= ~same;
    }
}

// K of the frame, the capacity check, and the rows that the frame may fill.
__device__ __forceinline__ void publish_K(const Bufs &B, int K) {
    FrameState *fs = B.fs;
    fs->K_now = K;
    if (K > B.kmax) atomicOr(&fs->err, DV_E_KMAX);
    fs->rows_dirty = min(K, B.kmax);
    fs->spill = 0;   // (the rows beyond the tables were emptied by k_tile_ccl)
}

// RANK_LANES lanes per tile (a tile has few pieces in the usual case); each is a
// chain of three dependent loads (record, root, segment) and three atomics.
// Every block makes the prefix of the band totals for itself (one load per
// thread for up to 256 bands), which spares a launch in the chain (3 us and a
// gap); the frame's first block publishes K.
#define RANK_LANES 8
template <bool WT>
__global__ __launch_bounds__(256, 8) void k_rank(const Bufs *__restrict__ D, Batch G, Fields F) {
    __shared__ int band_pre[65536 / DV_TILE], wsum[16];
    const int e = blockIdx.z;
    const int tiles = G.tbase[e + 1] - G.tbase[e];
    if ((int)blockIdx.x * (256 / RANK_LANES) >= tiles) return;
    const Bufs &B = D[G.idx[e]];
    const int K = block_exclusive_scan(B.band_sum, band_pre, B.nty, wsum);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_K(B, K);
    __syncthreads();
    const int tile = blockIdx.x * (256 / RANK_LANES) + threadIdx.x / RANK_LANES;
    const int np = tile < tiles ? gmem(B.npieces)[tile] : 0;
    auto rank_of = [&](int gx, int gy) {
        const size_t seg = (size_t)gy * B.ntx + (gx >> 5);
        const uint32_t below = (1u << (gx & 31)) - 1u;
        const uint2 sg = ld_uint2(B.seg, seg);
        return band_pre[gy / DV_TILE] + (int)sg.y + __popc(sg.x & below);
    };
    for (int k0 = 0; __ballot(k0 < np); k0 += RANK_LANES) {
        const int k = k0 + threadIdx.x % RANK_LANES;
        add_piece<WT>(B, F.p[e], k < np ? tile : 0, k, k < np, rank_of);
    }
}

// The finds, the canonical numbering, the sums and the centres of a small frame
// by one block (fits_mid): k_resolve, k_rank and k_centres in one, with the
// segment words and their prefix in LDS.  (As launches of their own 6.1 + 5.0 +
// 5.4 us and two gaps for 256^2 alone.)
template <bool WT>
__global__ __launch_bounds__(1024) void k_mid(const Bufs *__restrict__ D, Batch G, Fields F) {
    __shared__ int pre[MID_TILES], wsum[16];
    __shared__ uint32_t words[MID_WORDS];
    __shared__ int prefix[MID_WORDS];
    const int e = blockIdx.z, t = threadIdx.x;
    const Bufs B = D[G.idx[e]];
    const int tiles = B.ncells, ntx = B.ntx;
    for (int i = t; i < MID_WORDS; i += 1024) words[i] = 0u;
    const int total = block_exclusive_scan(B.npieces, pre, tiles, wsum);
    __syncthreads();
    // piece f of the frame: its tile and slot
    auto locate = [&](int f, int &tile, int &slot) {
        int lo = 0, hi = tiles - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= f) lo = mid; else hi = mid - 1;
        }
        tile = lo;
        slot = f - pre[lo];
    };
    for (int f = t; f < total; f += 1024) {
        int tile, slot;
        locate(f, tile, slot);
        const int r = PIECE_ROOT(gmem(B.tpiece)[piece_at(B, tile, slot)]);
        const int y = (tile / ntx) * DV_TILE + (r >> 5), tx = tile % ntx;
        const int g = y * B.lx + tx * DV_TILE + (r & 31);
        const int root = gfind_ro(gmem(B.parent), g);
        if (root != g) gmem(B.parent)[g] = root;
        else atomicOr(&words[y * ntx + tx], 1u << (r & 31));
    }
    __syncthreads();
    // raster-order prefix of the root bits, a run of eight words per thread
    constexpr int PER = MID_WORDS / 1024;
    int v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        v[k] = __popc(words[t * PER + k]);   // (zero beyond the lattice)
        sum += v[k];
    }
    const int inc = wave_incl_sum(sum);
    if ((t & 63) == 63) wsum[t >> 6] = inc;
    __syncthreads();
    int before = inc - sum, K = 0;
    for (int w = 0; w < 16; ++w) {
        before += w < (t >> 6) ? wsum[w] : 0;
        K += wsum[w];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        prefix[t * PER + k] = before;
        before += v[k];
    }
    if (t == 0) publish_K(B, K);
    __syncthreads();
    auto rank_of = [&](int gx, int gy) {
        const int seg = gy * ntx + (gx >> 5);
        return prefix[seg] + __popc(words[seg] & ((1u << (gx & 31)) - 1u));
    };
    for (int f0 = 0; f0 < total; f0 += 1024) {
        const bool have = f0 + t < total;
        int tile = 0, slot = 0;
        if (have) locate(f0 + t, tile, slot);
        add_piece<WT>(B, F.p[e], tile, slot, have, rank_of);
    }
    __syncthreads();
    frame_centres(B, K, K > B.kmax, wsum);
}

}  // namespace

void launch_label(const Batch &G, const Fields &F, hipStream_t s, Prof &P) {
    const dim3 tiles4((G.tiles + 3) / 4), block(256);
    P.begin(ST_TILE_CCL, s);
    auto ccl = [&](auto kernel) { hipLaunchKernelGGL(kernel, tiles4, block, 0, s, G.D, G, F); };
    if (G.tiles > STREAM_TILES) {
        if (G.weighted) G.geom ? ccl(k_tile_ccl<true, true, true>) : ccl(k_tile_ccl<false, true, true>);
        else G.geom ? ccl(k_tile_ccl<true, false, true>) : ccl(k_tile_ccl<false, false, true>);
    } else {
        if (G.weighted) G.geom ? ccl(k_tile_ccl<true, true, false>) : ccl(k_tile_ccl<false, true, false>);
        else G.geom ? ccl(k_tile_ccl<true, false, false>) : ccl(k_tile_ccl<false, false, false>);
    }
    P.end(ST_TILE_CCL, s);
    P.begin(ST_MERGE, s);
    auto merge = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3((G.tiles * lanes + 127) / 128), block, 0, s, G.D, G);
    };
    if (G.tiles > MERGE_FEW && G.tiles <= MERGE_MANY) G.geom ? merge(k_merge<true, 8>, 8) : merge(k_merge<false, 8>, 8);
    else G.geom ? merge(k_merge<true, 1>, 1) : merge(k_merge<false, 1>, 1);
    P.end(ST_MERGE, s);
    P.begin(ST_RESOLVE, s);
    if (G.small) {
        const dim3 frames(1, 1, G.n);
        if (G.weighted) hipLaunchKernelGGL(k_mid<true>, frames, dim3(1024), 0, s, G.D, G, F);
        else hipLaunchKernelGGL(k_mid<false>, frames, dim3(1024), 0, s, G.D, G, F);
        P.end(ST_RESOLVE, s);
        return;
    }
    hipLaunchKernelGGL(k_resolve, dim3(G.bands), dim3(G.bands >= RES_BANDS ? 256 : 1024),
                       sizeof(int) * (res_words(G.ntx) + res_pre(G.ntx)), s, G.D, G);
    P.end(ST_RESOLVE, s);
    P.begin(ST_RELABEL, s);
    int most = 0;   // tiles of the largest entry
    for (int e = 0; e < G.n; ++e) most = std::max(most, G.tbase[e + 1] - G.tbase[e]);
    const dim3 rank_blocks((most + 256 / RANK_LANES - 1) / (256 / RANK_LANES), 1, G.n);
    if (G.weighted) hipLaunchKernelGGL(k_rank<true>, rank_blocks, block, 0, s, G.D, G, F);
    else hipLaunchKernelGGL(k_rank<false>, rank_blocks, block, 0, s, G.D, G, F);
    P.end(ST_RELABEL, s);
}
