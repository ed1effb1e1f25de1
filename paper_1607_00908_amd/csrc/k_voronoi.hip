// Centres, bucket grid, digital Voronoi colouring and Delaunay couples
// (Sec. 3.1 last step, Sec. 3.2.1 and Sec. 3.2.2 of the paper).
//
//   k_centres       exact Q.8 and float64 centres from the integer sums and
//                   the bucket grid (cell offsets, centres by cell), a block per
//                   frame; for large K_max as k_finalize and k_grid, over many
//   k_owner_edges   one wave per tile: candidate centres from the grid,
//                   nearest centre of every site of the tile and its one-site
//                   ring, owner and label maps, frame-gap vertex test and the
//                   first / second nearest-neighbour rules; the distinct couples
//                   of the tile go to the tile's couple list, tiles with too
//                   many or too far candidates to the launch's lists
//   k_rows          the couple lists into the adjacency rows with a lock-free
//                   set insert (rows are unordered sets, MAXLINK padded); the
//                   listed tiles by the general form of the colouring; beside
//                   them, in blocks of their own, the matching of Sec. 3.2.3
#include <algorithm>
#include <type_traits>

#include "dv_device.h"

namespace {

// Centres and bucket grid, a block per frame.
__global__ __launch_bounds__(1024) void k_centres(const Bufs *__restrict__ D, Batch G) {
    const Bufs B = D[G.idx[blockIdx.z]];
    __shared__ int wsum[16];
    frame_centres(B, B.fs->K_now, B.fs->err != 0, wsum);
}

// The same over many blocks: centres, each linked into its cell's list, and the
// sums of the groups of 256 cells (added up over the wave first: consecutive
// components lie in neighbouring cells, and atomics on one line take turns;
// with an atomic per centre for the group and one more for the cell's count 45
// us per 20 frames of 4096^2); then k_grid.
__global__ __launch_bounds__(1024) void k_finalize(const Bufs *__restrict__ D, Batch G) {
    const Bufs B = D[G.idx[blockIdx.z]];
    FrameState *fs = B.fs;
    const int K = fs->K_now;
    const int k0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    if (fs->err) {
        for (int k = k0; k < min(K, B.kmax); k += step) drop_sums(B, k);
        return;
    }
    int namb = 0;
    for (int k = k0; __ballot(k < K); k += step) {
        int group = -1;
        if (k < K) {
            const int cell = cell_of(B, centre_of(B, k, namb));
            gmem(B.comp_next)[k] = atomicExch(&B.cell_head[cell], k);
            group = cell >> 8;
        }
        for (unsigned long long m = __ballot(k < K); m;) {
            const int g = __builtin_amdgcn_readlane(group, (int)__builtin_ctzll(m));
            const unsigned long long same = __ballot(group == g);
            if (group == g && (same & ((1ull << (threadIdx.x & 63)) - 1ull)) == 0)
                atomicAdd(&B.cell_sum[g * DV_LINE], __popcll(same));
            m &= ~same;
        }
    }
    if (namb) atomicAdd(&fs->n_amb, namb);
}

// A block per 256 cells, a thread per cell: the cell's place follows from the
// sums of the groups before and a block scan of the lengths of the cells' lists
// (usually none to three centres), which the thread then writes out.  (One block
// per frame over all cells: 24 us for one frame of 4096^2.)
__global__ __launch_bounds__(256) void k_grid(const Bufs *__restrict__ D, Batch G) {
    const int e = blockIdx.z;
    if ((int)blockIdx.x * 256 >= G.tbase[e + 1] - G.tbase[e]) return;
    const Bufs B = D[G.idx[e]];
    __shared__ int wsum[2][4];
    if (B.fs->err) return;
    const int t = threadIdx.x, cell = blockIdx.x * 256 + t;
    const bool on = cell < B.ncells;
    const int head = on ? gmem(B.cell_head)[cell] : -1;
    int before = 0;
    for (int g = t; g < (int)blockIdx.x; g += 256) before += gmem(B.cell_sum)[g * DV_LINE];
    int c = 0;
    for (int k = head; k >= 0; k = gmem(B.comp_next)[k]) ++c;
    const int inc = wave_incl_sum(c);
    before = wave_last(wave_incl_sum(before));
    if ((t & 63) == 63) {
        wsum[0][t >> 6] = before;
        wsum[1][t >> 6] = inc;
    }
    __syncthreads();
    int pos = wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3] + inc - c;
    for (int w = 0; w < (t >> 6); ++w) pos += wsum[1][w];
    if (!on) return;
    gmem(B.cell_start)[cell] = pos;
    if (cell == B.ncells - 1) gmem(B.cell_start)[B.ncells] = pos + c;
    for (int k = head; k >= 0; ++pos) {
        const int next = gmem(B.comp_next)[k];
        gmem(B.cell_items)[pos] = k;
        st_int2(B.cell_q, pos, gmem(B.cur.qx)[k], gmem(B.cur.qy)[k]);
        k = next;
    }
}

// Frame of a site (Sec. 3.2.2), cyclic: spx, spxpy, spy, spymx, smx, smxmy,
// smy, smypx; inner-frame points a_k, b_k, c_k, d_k at (+-1/2, +-1/2) in Q.8.
// Written as expressions so that no table is read from memory.
__device__ __forceinline__ int frx(int k) { return (k == 0 || k == 1 || k == 7) ? 1 : (k == 2 || k == 6) ? 0 : -1; }
__device__ __forceinline__ int fry(int k) { return (k == 1 || k == 2 || k == 3) ? 1 : (k == 0 || k == 4) ? 0 : -1; }
__device__ __forceinline__ int inx(int r) { return (r == 1 || r == 2) ? -128 : 128; }
__device__ __forceinline__ int iny(int r) { return r >= 2 ? -128 : 128; }

// Lock-free set insert of v into row a.  The probe starts at a slot that
// depends on v, so that the couples of one centre, which several tiles find at
// the same time, meet in different slots: an insert is one read and at most one
// exchange in the usual case.  (With rows filled from the front every insert
// raced for the same first free slot: 15 us for a frame of 256^2 alone.)  A
// slot never goes back to empty within a frame, so every insert of v probes the
// same way up to the slot that holds it, and it is stored once.
__device__ __forceinline__ void row_insert(const Bufs &B, int a, int v, FrameState *fs) {
    const int prim = B.prim;
    gint *row = gmem(B.cur.adj) + (size_t)a * prim;
    int k = prim == DV_ROW ? v & (DV_ROW - 1) : v % prim;
    for (int i = 0; i < prim; ++i) {
        int old = row[k];
        if (old == DV_EMPTY)
            __hip_atomic_compare_exchange_strong(row + k, &old, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        if (old == DV_EMPTY || old == v) return;
        k = k + 1 == prim ? 0 : k + 1;
    }
    // the table is full: the row goes on in adjx, filled from the front
    const int rest = B.maxdeg - prim;
    if (rest) fs->spill = 1;
    gint *more = gmem(B.cur.adjx) + (size_t)a * rest;
    for (int i = 0; i < rest; ++i) {
        int old = DV_EMPTY;
        __hip_atomic_compare_exchange_strong(more + i, &old, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if (old == DV_EMPTY || old == v) return;
    }
    atomicOr(&fs->err, DV_E_DEGREE);
}

typedef short sh2 __attribute__((ext_vector_type(2)));   // packed 16-bit pair

// a.x b.x + a.y b.y + c on signed 16-bit pairs, exact in 32 bits.  Written
// as the three-operand instruction: the compiler's form of the builtin
// accumulates into its destination, which costs a copy of c for every use
// when c is shared by several products.
__device__ __forceinline__ int dot2_acc(sh2 a, sh2 b, int c) {
    int d;
    asm("v_dot2_i32_i16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

#define PAIR_CAP 256    // couples a tile can collect in LDS before writing through
#define TMP_CAP 128     // centres kept from the first pass

#define WSITES 5      // ceil(34*34 / 256) window sites per thread
#define RCAP 256      // item ranges held in LDS per batch
#define IMG_MAX 9     // periodic images one centre can contribute (tiny lattices)
#define CAND_BATCH 8  // centres appended per batch (room for IMG_MAX images each)

// Shared state of one colouring tile.
struct OwnerLds {
    int own[34 * 34];
    // candidate centres as appended: tile-relative Q.8 image positions, label
    int cx[DV_CAND_CAP], cy[DV_CAND_CAP];
    int lab[DV_CAND_CAP];
    // the kept ones, ordered by label for evaluation: x, y, |c|^2 as doubles,
    // or as 32-bit integers when every kept one is near the tile (imode)
    union {
        struct { double sx[DV_CAND_CAP], sy[DV_CAND_CAP], sk[DV_CAND_CAP]; };
        // (ixy: x in the low 16 bits, y in the high 16, for the packed dot product)
        struct { int ixy[DV_CAND_CAP], ik[DV_CAND_CAP]; };
    };
    int sl[DV_CAND_CAP];
    uint8_t keep[DV_CAND_CAP];   // the candidate is not beaten everywhere in the window
    int nkeep;                   // candidates kept (the ordered list's length)
    int fast;                    // the one-pass candidate list of the usual case was built
    int far;                     // some kept candidate is beyond the 32-bit range
    int imode;                   // the ordered list holds 32-bit integers
    int ncand;
    int nchunks;   // times the list was evaluated and emptied before the end
    // item ranges of the cell rectangle being visited
    int r_e0[RCAP], r_pre[RCAP + 1];
    int nranges;
    unsigned long long best;
    int wsum[16];
    // centres seen in the first pass: label, Q.8 centre, squared distance
    // to the tile centre
    int tmp[TMP_CAP];
    union {
        int2 tmpq[TMP_CAP];
        // (after the candidate list is built) inner-frame queries of each
        // thread's sites, bit 4i + r as in the thread's own mask
        unsigned pendw[DV_BLOCK];
    };
    long long tmpd[TMP_CAP];
    int ntmp;
    // couples found by the tile, (a << 32 | b) with a < b
    unsigned long long pair[PAIR_CAP];
    int npair;
};

// Visit every item (index into the cell-ordered centre arrays) of the cells
// in rows sy x column ranges sx.  fn(e) is called by the block's threads in
// parallel, in batches of at most `batch` items; before each batch every
// thread calls before(m) with the batch size m (uniform control flow; all
// earlier fn calls have completed).
template <class Fn, class Before>
__device__ void visit_items(const Bufs &B, OwnerLds &S, const Span &sx, const Span &sy, int batch,
                            Fn fn, Before before) {
    const int t = threadIdx.x;
    const auto cs = gmem(B.cell_start);
    // rows of the rectangle, enumerated in order
    int nrows = 0;
    for (int i = 0; i < sy.n; ++i) nrows += sy.hi(i) - sy.lo(i) + 1;
    const int per_row = sx.n;
    for (int rb = 0; rb < nrows; rb += RCAP / 2) {
        const int nr = min(RCAP / 2, nrows - rb);
        const int nrng = nr * per_row;
        // range j -> (row index rb + j / per_row, column range j % per_row)
        int cnt = 0;
        if (t < nrng) {
            int ri = rb + t / per_row;
            const int n0 = sy.hi0 - sy.lo0 + 1;
            const int row = (ri < n0) ? sy.lo0 + ri : sy.lo1 + (ri - n0);
            const int c = t % per_row;
            const int e0 = cs[row * B.ntx + sx.lo(c)], e1 = cs[row * B.ntx + sx.hi(c) + 1];
            S.r_e0[t] = e0;
            cnt = e1 - e0;
        }
        // exclusive scan of the counts (nrng <= RCAP / 2 * 2 <= blockDim)
        {
            const int lane = t & 63, wid = t >> 6;
            const int x = wave_incl_sum(cnt);
            if (lane == 63) S.wsum[wid] = x;
            __syncthreads();
            int before = 0;
            for (int w = 0; w < wid; ++w) before += S.wsum[w];
            if (t < RCAP) S.r_pre[t] = before + x - cnt;
            if (t == (int)blockDim.x - 1) S.r_pre[RCAP] = before + x;
            __syncthreads();
        }
        const int total = S.r_pre[RCAP];
        for (int f0 = 0; f0 < total; f0 += batch) {
            const int m = min(batch, total - f0);
            before(m);
            for (int j = t; j < m; j += blockDim.x) {
                const int f = f0 + j;
                // range holding flat index f: last j with pre[j] <= f
                int lo = 0, hi = nrng - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (S.r_pre[mid] <= f) lo = mid; else hi = mid - 1;
                }
                fn(S.r_e0[lo] + (f - S.r_pre[lo]));
            }
            __syncthreads();
        }
    }
}

// The general form of a tile's colouring, by a whole block: any number of
// candidates (evaluated in LDS-sized chunks), any distance, several periodic
// images of one centre (tiny lattices), no centre at all.
// GEOM: some entry of the launch has walls or obstacles; the periodic,
// unobstructed instance carries none of their tests.
template <bool GEOM>
__device__ __forceinline__ void owner_general(const Bufs &B, int tile, OwnerLds &S) {
    const int tx = tile % B.ntx, ty = tile / B.ntx;
    const bool ox = GEOM && B.open_x, oy = GEOM && B.open_y;
    // The usual candidate search reads the centres of the 7 x 7 cells around
    // the tile: first the bounds of their cell ranges (each row of cells of a
    // column span is one contiguous range of the cell-ordered arrays, at
    // most 7 x 2 ranges, a lane each in the first wave), then the centres.
    // The bounds are requested before anything else, so that their round
    // trip overlaps the frame header's.
    // (The frame's errors are not looked at: only frames without one list tiles,
    // and the inserts of this launch can still set DV_E_DEGREE, which the waves of a
    // block would see at different times, some leaving and some going on to the
    // block's barriers.  A frame that is rejected meanwhile is coloured to the end;
    // its inserts stay within its rows.)
    const int R0 = 3;
    const Span sx0 = span_cells(tx, R0, B.ntx, ox), sy0 = span_cells(ty, R0, B.nty, oy);
    const int n0y = sy0.hi0 - sy0.lo0 + 1, ncy = n0y + (sy0.n == 2 ? sy0.hi1 - sy0.lo1 + 1 : 0);
    const int nrng = ncy * sx0.n;
    int rb0 = 0, rb1 = 0;
    if ((int)threadIdx.x < nrng) {
        const int iy = threadIdx.x / sx0.n, c = threadIdx.x - iy * sx0.n;
        const int celly = iy < n0y ? sy0.lo0 + iy : sy0.lo1 + (iy - n0y);
        const auto cs = gmem(B.cell_start);
        rb0 = cs[celly * B.ntx + sx0.lo(c)];
        rb1 = cs[celly * B.ntx + sx0.hi(c) + 1];
    }
    FrameState *fs = B.fs;
    const int K = *gmem(&fs->K_now);
    const int x0 = tx * DV_TILE, y0 = ty * DV_TILE;
    const int tw = min(DV_TILE, B.lx - x0), th = min(DV_TILE, B.ly - y0);
    const int W = tw + 2, H = th + 2;
    const int t = threadIdx.x, lx = B.lx, ly = B.ly;
    // wrap periods (Q.8): the lattice period of a periodic axis; on a walled
    // axis a period that no distance reaches (images are not used there)
    const int MX = qperiod(lx, ox), MY = qperiod(ly, oy);
    const int OX = 256 * x0, OY = 256 * y0;   // tile origin (Q.8); coordinates below are relative

    // window sites of this thread: exact tile-relative Q.8 coordinates
    // (best value, owner) of the thread's window sites w = t + 256 i; the
    // site coordinates are rebuilt where needed (w / W by a multiply: w <
    // 1280 and W <= 34, so the 16-bit reciprocal is exact).  The float64
    // values are set by the first evaluation that uses them.
    double be[WSITES];
    int bl[WSITES];
    const int wmagic = (65536 + W - 1) / W;
#pragma unroll
    for (int i = 0; i < WSITES; ++i) bl[i] = DV_EMPTY;
    // the same sites as packed pairs wx | wy << 16: the first by the
    // reciprocal, each next one by adding 256 = wq W + wr (with a carry into
    // the row when wx reaches W)
    const int wq = DV_BLOCK / W, wr = DV_BLOCK - wq * W;
    auto site_pairs = [&](int P[WSITES]) {
        const int wy0 = (t * wmagic) >> 16;
        P[0] = (t - wy0 * W) | (wy0 << 16);
#pragma unroll
        for (int i = 1; i < WSITES; ++i) {
            const int q = P[i - 1] + (wr | (wq << 16));
            P[i] = (q & 0xffff) >= W ? q + (1 << 16) - W : q;
        }
    };
    // (the first wave reads these in program order, the others only after a
    // later barrier)
    if (t == 0) { S.ncand = 0; S.nchunks = 0; S.best = ~0ull; S.npair = 0; S.ntmp = 0; S.nkeep = 0; S.imode = 0; }

    // tile centre (absolute Q.8) and the window's relative x / y extent
    const int tcx = OX + 128 * (tw - 1), tcy = OY + 128 * (th - 1);
    const int wxlo = -256, wxhi = 256 * tw, wylo = -256, wyhi = 256 * th;

    // Nearest candidate of every window site.  Candidates that another
    // candidate beats everywhere in the window are dropped first: the
    // difference of the squared distances to two centres is affine in the
    // point, so when its minimum over the window rectangle (at the corner its
    // gradient picks) is positive, the other centre is strictly nearer at
    // every window site and inner-frame point, and the dropped one owns none
    // of them.  Some candidate always stays (strict domination has a minimal
    // element), and so does the owner of every point.  The test is exact in
    // float64: coordinates stay below 2^26 in magnitude (Q.8, images
    // included), so every square and sum is an integer below 2^53, and where
    // rounding could occur the value is far from zero.  The kept candidates
    // are ordered by label, so that a strict comparison already sends ties to
    // the lowest label; a later chunk (after an overflow) also compares
    // labels.
    // In the usual case every kept candidate lies within 23170 Q.8 units
    // (about 90 sites) of the tile origin on both axes: then |c|^2 < 2^30,
    // each product of a coordinate with a doubled point coordinate (at most
    // 16384 in magnitude) fits 24-bit operands, and every value below stays
    // inside 32-bit range, so the same exact comparison runs on integers.
    // That applies to the only evaluation of a tile (no overflow chunks);
    // otherwise the float64 form is used.
    auto eval_owners = [&](bool last, bool inited) {
        if (!inited) {
            if (t == 0) { S.nkeep = 0; S.far = 0; }
            __syncthreads();
        }
        const int nc = min(S.ncand, DV_CAND_CAP);
        if (nc <= 16) {   // the first wave: 4 lanes per candidate i, lane j of the group
                          // takes the rivals j, j + 4, ...
            if (t < 64) {
                const int i = t >> 2, gj = t & 3;
                bool beaten = false;
                if (i < nc) {
                    const double cx = (double)S.cx[i], cy = (double)S.cy[i];
                    const double cc = fma(cx, cx, cy * cy);
#pragma unroll 1
                    for (int j = gj; j < nc && !beaten; j += 4) {
                        if (j == i) continue;
                        const double jx = (double)S.cx[j], jy = (double)S.cy[j];
                        const double ax = 2.0 * (jx - cx), ay = 2.0 * (jy - cy);
                        const double f = fma(ax, ax >= 0.0 ? (double)wxlo : (double)wxhi,
                                             fma(ay, ay >= 0.0 ? (double)wylo : (double)wyhi,
                                                 cc - fma(jx, jx, jy * jy)));
                        beaten = f > 0.0;
                    }
                }
                const unsigned long long b = __ballot(beaten);
                const unsigned grp = (unsigned)(b >> (t & 60)) & 0xfu;
                const bool kept = gj == 0 && i < nc && !grp;
                if (gj == 0 && i < nc) S.keep[i] = grp ? 0 : 1;
                const bool farc = kept && (abs(S.cx[i]) > 23170 || abs(S.cy[i]) > 23170);
                const int nkept = __popcll(__ballot(kept));
                const bool anyfar = __ballot(farc) != 0ull;
                if (t == 0) {
                    S.nkeep = nkept;
                    S.far = anyfar ? 1 : 0;
                }
            }
        } else {   // 16 lanes per candidate i, lane j of the group takes the rivals j, j + 16, ...
            const int gi = t >> 4, gj = t & 15;
#pragma unroll 1
            for (int i0 = 0; i0 < nc; i0 += DV_BLOCK / 16) {
                const int i = i0 + gi;
                bool beaten = false;
                if (i < nc) {
                    const double cx = (double)S.cx[i], cy = (double)S.cy[i];
                    const double cc = fma(cx, cx, cy * cy);
#pragma unroll 1
                    for (int j = gj; j < nc && !beaten; j += 16) {
                        if (j == i) continue;
                        const double jx = (double)S.cx[j], jy = (double)S.cy[j];
                        // |w - c|^2 - |w - j|^2 = 2 w.(j - c) + |c|^2 - |j|^2
                        const double ax = 2.0 * (jx - cx), ay = 2.0 * (jy - cy);
                        const double f = fma(ax, ax >= 0.0 ? (double)wxlo : (double)wxhi,
                                             fma(ay, ay >= 0.0 ? (double)wylo : (double)wyhi,
                                                 cc - fma(jx, jx, jy * jy)));
                        beaten = f > 0.0;
                    }
                }
                const unsigned long long b = __ballot(beaten);
                const unsigned grp = (unsigned)(b >> (t & 48)) & 0xffffu;
                if (gj == 0 && i < nc) {
                    S.keep[i] = grp ? 0 : 1;
                    if (!grp) {
                        atomicAdd(&S.nkeep, 1);
                        if (abs(S.cx[i]) > 23170 || abs(S.cy[i]) > 23170) S.far = 1;
                    }
                }
            }
        }
        __syncthreads();
        const bool im = last && S.nchunks == 0 && !S.far;
        // kept candidate c with label lab goes to position r of the ordered list
        auto place = [&](int c, int r, int lab) {
            const int ix = S.cx[c], iy = S.cy[c];
            if (im) {
                S.ixy[r] = (int)(((unsigned)iy << 16) | ((unsigned)ix & 0xffffu));
                S.ik[r] = ix * ix + iy * iy;
            } else {
                const double x = (double)ix, y = (double)iy;
                S.sx[r] = x;
                S.sy[r] = y;
                S.sk[r] = x * x + y * y;
            }
            S.sl[r] = lab;
        };
        if (nc <= 64) {
            // the first wave, lane c holding candidate c: its position counts
            // the kept candidates before it by (label, index), visited one
            // kept candidate at a time
            if (t < 64) {
                const bool kc = t < nc && S.keep[t];
                const int lab = t < nc ? S.lab[t] : 0;
                int r = 0;
                for (unsigned long long m = __ballot(kc); m; m &= m - 1) {
                    const int j = (int)__builtin_ctzll(m);
                    const int l2 = __builtin_amdgcn_readlane(lab, j);
                    r += (l2 < lab || (l2 == lab && j < t)) ? 1 : 0;
                }
                if (kc) place(t, r, lab);
            }
        } else {
            for (int c = t; c < nc; c += DV_BLOCK) {
                if (!S.keep[c]) continue;
                const int lab = S.lab[c];
                int r = 0;
                for (int j = 0; j < nc; ++j) {
                    const int l2 = S.lab[j];
                    r += (S.keep[j] && (l2 < lab || (l2 == lab && j < c))) ? 1 : 0;
                }
                place(c, r, lab);
            }
        }
        if (t == 0) S.imode = im ? 1 : 0;
        __syncthreads();
        const int nk = S.nkeep;
        if (im) {
            // the only evaluation: strict comparison, ties to the first (lowest
            // label).  -2 w and the candidate are 16-bit pairs (|2 w| <= 16384,
            // |c| <= 23170), so e = -2 w . c + |c|^2 is one packed dot product
            // with exact 32-bit accumulation
            sh2 m2[WSITES];
            int bi[WSITES];
            {
                int P[WSITES];
                site_pairs(P);
#pragma unroll
                for (int i = 0; i < WSITES; ++i) {
                    // (-512 (wx - 1), -512 (wy - 1)) = ((1, 1) - (wx, wy)) * 512
                    m2[i] = (sh2{1, 1} - __builtin_bit_cast(sh2, P[i])) * (short)512;
                    bi[i] = INT_MAX;
                }
            }
            // candidates in order, two per step (the compiler does not unroll
            // a loop around inline assembly)
            auto cand = [&](int c) {
                const sh2 cq = __builtin_bit_cast(sh2, S.ixy[c]);
                const int kk = S.ik[c];
                const int lab = S.sl[c];
#pragma unroll
                for (int i = 0; i < WSITES; ++i) {
                    const int e = dot2_acc(m2[i], cq, kk);
                    const bool lt = e < bi[i];
                    bi[i] = lt ? e : bi[i];
                    bl[i] = lt ? lab : bl[i];
                }
            };
            int c = 0;
            for (; c + 1 < nk; c += 2) {
                cand(c);
                cand(c + 1);
            }
            if (c < nk) cand(c);
            return;
        }
        double m2x[WSITES], m2y[WSITES];
#pragma unroll
        for (int i = 0; i < WSITES; ++i) {
            const int w = t + i * DV_BLOCK;
            const int wy = (w * wmagic) >> 16, wx = w - wy * W;
            m2x[i] = -512.0 * (wx - 1);
            m2y[i] = -512.0 * (wy - 1);
        }
        if (S.nchunks == 0) {
#pragma unroll
            for (int i = 0; i < WSITES; ++i) be[i] = 1.0e300;
            for (int c = 0; c < nk; ++c) {
                const double cx = S.sx[c], cy = S.sy[c], kk = S.sk[c];
                const int lab = S.sl[c];
#pragma unroll
                for (int i = 0; i < WSITES; ++i) {
                    const double e = fma(m2x[i], cx, fma(m2y[i], cy, kk));
                    const bool lt = e < be[i];
                    be[i] = lt ? e : be[i];
                    bl[i] = lt ? lab : bl[i];
                }
            }
        } else {
            for (int c = 0; c < nk; ++c) {
                const double cx = S.sx[c], cy = S.sy[c], kk = S.sk[c];
                const int lab = S.sl[c];
#pragma unroll
                for (int i = 0; i < WSITES; ++i) {
                    const double e = fma(m2x[i], cx, fma(m2y[i], cy, kk));
                    if (e < be[i] || (e == be[i] && lab < bl[i])) { be[i] = e; bl[i] = lab; }
                }
            }
        }
    };

    // candidate list entry for centre e: every image of the centre that is the
    // minimum image of some window point (relative offset within [-M/2, M/2]).
    // The offset rx lies in (-MX, MX) and the window is at most one lattice
    // wide, so only the images k = -1 .. 2 can qualify.  On a walled axis
    // (M = 512 L) the centre itself always qualifies and a shifted copy only
    // for a centre on the first or last site line, seen from the tile at the
    // other wall: that copy is farther than the centre from every point inside
    // the domain (the only points whose colour is used), so it owns none.
    auto image_masks = [&](int rx, int ry, unsigned &mxk, unsigned &myk) {
        mxk = 0;
        myk = 0;
#pragma unroll
        for (int k = -1; k <= 2; ++k) {
            const int vx = rx + k * MX, vy = ry + k * MY;
            if (vx >= wxlo - MX / 2 && vx <= wxhi + MX / 2) mxk |= 1u << (k + 1);
            if (vy >= wylo - MY / 2 && vy <= wyhi + MY / 2) myk |= 1u << (k + 1);
        }
    };
    auto add_images = [&](int lab, int2 q) {
        const int rx = q.x - OX, ry = q.y - OY;
        unsigned mxk, myk;
        image_masks(rx, ry, mxk, myk);
        for (unsigned a = mxk; a; a &= a - 1) {
            const int cx = rx + (__ffs(a) - 2) * MX;
            for (unsigned b = myk; b; b &= b - 1) {
                const int cy = ry + (__ffs(b) - 2) * MY;
                const int slot = atomicAdd(&S.ncand, 1);
                if (slot >= DV_CAND_CAP) continue;   // overflow: caller falls back
                S.cx[slot] = cx;
                S.cy[slot] = cy;
                S.lab[slot] = lab;
            }
        }
    };
    // radius around the tile centre that holds every centre able to own a
    // window site or inner-frame point: bound + twice the window's half diagonal
    auto hdiag2 = [&]() {
        const double hx = 0.5 * (tw + 1), hy = 0.5 * (th + 1);
        return 2.0 * sqrt(hx * hx + hy * hy) + 2.0;
    };

    if (K > 0) {
        // --- usual case, one pass by the first wave: the 7x7 cells around the
        // tile give a bound (nearest centre seen) and, when they cover the
        // radius it implies, every candidate as well; the other waves wait at
        // the barrier
        if (t < 64) {
            // the centres of the square's cells, lane-parallel: one centre per
            // lane over the concatenated ranges whose bounds were requested
            // at the start; the bound is one wave minimum
            const int e0 = rb0, cnt = rb1 - rb0;
            const int inc = wave_incl_sum(cnt);
            const int total = wave_last(inc);
            const int pre = inc - cnt;
            unsigned long long dmin = ~0ull;
            // the lane's item of the first 64 stays in registers; later ones
            // (more than 64 centres in the square) go to LDS
            int2 q0 = make_int2(0, 0);
            int lab0 = 0;
            long long d0 = 0;
            for (int f0 = 0; f0 < total; f0 += 64) {
                const int f = f0 + t;
                // range of item f: the last one whose exclusive prefix is <= f
                int r = 0;
                for (int k = 1; k < nrng; ++k) r = __builtin_amdgcn_readlane(pre, k) <= f ? k : r;
                const int e = __shfl(e0, r, 64) + f - __shfl(pre, r, 64);
                if (f < total) {
                    const int2 q = ld_int2(B.cell_q, e);
                    const int lab = gmem(B.cell_items)[e];
                    const long long d = d2q(tcx, tcy, q.x, q.y, MX, MY);
                    dmin = min(dmin, (unsigned long long)d);
                    if (f0 == 0) {
                        q0 = q;
                        lab0 = lab;
                        d0 = d;
                    } else if (f < TMP_CAP) {
                        S.tmp[f] = lab;
                        S.tmpq[f] = q;
                        S.tmpd[f] = d;
                    }
                }
            }
            dmin = wave_min_u64(dmin);
            // the bound covers the candidates' radius: the list is built here
            bool fast = dmin != ~0ull && total <= TMP_CAP;
            double rq2 = 0.0;
            if (fast) {
                const double rho = sqrt((double)dmin) / 256.0 + hdiag2();
                const int wlx = lx - DV_TILE * (B.ntx - 1), wly = ly - DV_TILE * (B.nty - 1);
                const double cov_x = span_full(sx0, B.ntx) ? 1e30 : (double)(DV_TILE * (R0 - 1) + wlx);
                const double cov_y = span_full(sy0, B.nty) ? 1e30 : (double)(DV_TILE * (R0 - 1) + wly);
                fast = rho <= cov_x && rho <= cov_y;
                rq2 = (256.0 * rho) * (256.0 * rho);
            }
            if (fast) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                int nc = 0;   // list slots taken so far (every lane the same)
                for (int f0 = 0; f0 < total; f0 += 64) {
                    const int f = f0 + t;
                    int2 q = q0;
                    int lab = lab0;
                    long long d = d0;
                    if (f0 > 0 && f < total) {
                        q = S.tmpq[f];
                        lab = S.tmp[f];
                        d = S.tmpd[f];
                    }
                    unsigned mxk = 0, myk = 0;
                    int rx = 0, ry = 0;
                    if (f < total && (double)d <= rq2) {
                        rx = q.x - OX;
                        ry = q.y - OY;
                        image_masks(rx, ry, mxk, myk);
                    }
                    const int c = __popc(mxk) * __popc(myk);
                    const int x = wave_incl_sum(c);
                    int slot = nc + x - c;
                    for (unsigned a = mxk; a; a &= a - 1) {
                        const int cx = rx + (__ffs(a) - 2) * MX;
                        for (unsigned b = myk; b; b &= b - 1) {
                            if (slot < DV_CAND_CAP) {
                                S.cx[slot] = cx;
                                S.cy[slot] = ry + (__ffs(b) - 2) * MY;
                                S.lab[slot] = lab;
                            }
                            ++slot;
                        }
                    }
                    nc += wave_last(x);
                }
                if (t == 0) S.ncand = nc;
            }
            if (t == 0) {
                S.best = dmin;
                S.ntmp = total;
                S.fast = fast ? 1 : 0;
                S.nkeep = 0;
                S.far = 0;
            }
        }
        __syncthreads();
        const bool done = S.fast && S.ncand <= DV_CAND_CAP;
        if (!done) {
            // --- general case (from an empty list): a growing square of cells
            // for the bound, then every cell meeting the disc, evaluated in
            // LDS-sized chunks
            if (t == 0) S.ncand = 0;
            __syncthreads();
            for (int R = R0;; R *= 2) {
                if (S.best != ~0ull) break;
                const Span sx = span_cells(tx, 2 * R, B.ntx, ox), sy = span_cells(ty, 2 * R, B.nty, oy);
                visit_items(B, S, sx, sy, 1 << 30,
                            [&](int e) {
                                const int2 q = ld_int2(B.cell_q, e);
                                atomicMin(&S.best, (unsigned long long)d2q(tcx, tcy, q.x, q.y, MX, MY));
                            },
                            [](int) {});
                if (span_full(sx, B.ntx) && span_full(sy, B.nty)) break;
            }
            const double rho = sqrt((double)S.best) / 256.0 + hdiag2();
            const double rq2 = (256.0 * rho) * (256.0 * rho);
            const double px = tcx / 256.0, py = tcy / 256.0;
            const Span sx = span_sites((int)floor(px - rho), (int)floor(px + rho), lx, ox);
            const Span sy = span_sites((int)floor(py - rho), (int)floor(py + rho), ly, oy);
            visit_items(
                B, S, sx, sy, CAND_BATCH,
                [&](int e) {
                    const int2 q = ld_int2(B.cell_q, e);
                    if ((double)d2q(tcx, tcy, q.x, q.y, MX, MY) <= rq2) add_images(gmem(B.cell_items)[e], q);
                },
                [&](int m) {
                    // evaluate and empty the list when this batch could overflow it
                    if (S.ncand + m * IMG_MAX > DV_CAND_CAP) {
                        eval_owners(false, false);
                        __syncthreads();
                        if (t == 0) { S.ncand = 0; S.nchunks += 1; }
                        __syncthreads();
                    }
                });
        }
        eval_owners(true, done);
    }
    // window sites with no colour: beyond a wall, and obstacles.  (Without
    // either, a window 34 sites wide is stored as it is numbered.)
    if (!GEOM && W == 34) {
#pragma unroll
        for (int i = 0; i < WSITES; ++i)
            if (t + i * DV_BLOCK < W * H) S.own[t + i * DV_BLOCK] = bl[i];
    } else
#pragma unroll
    for (int i = 0; i < WSITES; ++i) {
        const int w = t + i * DV_BLOCK;
        const int wy = (w * wmagic) >> 16, wx = w - wy * W;
        if (w >= W * H) continue;
        int ax = x0 + wx - 1, ay = y0 + wy - 1;
        bool none = (ox && (ax < 0 || ax >= lx)) || (oy && (ay < 0 || ay >= ly));
        if (GEOM && B.obst && !none) {
            ax = ax < 0 ? ax + lx : (ax >= lx ? ax - lx : ax);
            ay = ay < 0 ? ay + ly : (ay >= ly ? ay - ly : ay);
            none = gmem(B.obst)[(size_t)ay * lx + ax] != 0;
        }
        S.own[wy * 34 + wx] = none ? DV_EMPTY : bl[i];
    }
    __syncthreads();

    // --- frame gaps and the neighbour rules.  The inner-frame points whose
    // colour decides a second-neighbour link are collected, then coloured
    // against the candidate list (or, after a candidate-list overflow, by the
    // exact grid search).
    const bool in_lds = S.nchunks == 0;
    const bool imode = S.imode;
    const int ncl = S.nkeep;   // the ordered list of the single chunk
    auto emit = [&](int a, int b) {
        const int slot = atomicAdd(&S.npair, 1);
        if (slot < PAIR_CAP) {
            S.pair[slot] = ((unsigned long long)(unsigned)a << 32) | (unsigned)b;
        } else {
            row_insert(B, a, b, fs);
            row_insert(B, b, a, fs);
        }
    };
    // thread t takes column t & 31 and the four rows 4 (t >> 5) .. + 3, so the
    // colours around its sites are one 6 x 3 block of the window
    const int cx = t & 31, ry = t >> 5, lane = t & 63;
    const int ys = 4 * ry;
    int g[6][3];
#pragma unroll
    for (int a = 0; a < 6; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) g[a][b] = S.own[(ys + a) * 34 + cx + b];
    // vertex sites of the thread (frame gaps >= 3): bit i for row ys + i.
    // (The map pointer and flag are read once: the stores could alias the
    // slot table as far as the compiler knows.)
    const bool keep_maps = B.keep_maps;
    const auto orow = gmem(B.owner) + ((size_t)(y0 + ys) * lx + x0 + cx);
    unsigned vmask = 0;
    if (!GEOM) {
        // The frame of the site in row ys + i is the border of rows i .. i + 2
        // of the block: its gaps are the changes along rows i and i + 2 and
        // down columns 0 and 2 (rows i to i + 1 and i + 1 to i + 2), each
        // change counted once for the thread's four sites.  (Without walls
        // and obstacles no frame point is MAXLINK once the site has a colour:
        // there is a centre, so every point has one.)
        int hr[6], vc[5];
#pragma unroll
        for (int a = 0; a < 6; ++a) hr[a] = (g[a][0] != g[a][1] ? 1 : 0) + (g[a][1] != g[a][2] ? 1 : 0);
#pragma unroll
        for (int a = 0; a < 5; ++a) vc[a] = (g[a][0] != g[a + 1][0] ? 1 : 0) + (g[a][2] != g[a + 1][2] ? 1 : 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int y = ys + i;
            if (cx >= tw || y >= th) continue;
            const int ckk = g[i + 1][1];
            if (keep_maps) orow[(size_t)i * lx] = ckk;
            // (with no centre every colour is MAXLINK and there are no gaps)
            const int gaps = hr[i] + hr[i + 2] + vc[i] + vc[i + 1];
            vmask |= gaps >= 3 ? 1u << i : 0u;
        }
    } else
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int y = ys + i;
        if (cx >= tw || y >= th) continue;
        const int ckk = g[i + 1][1];
        if (keep_maps) orow[(size_t)i * lx] = ckk;
        if (ckk == DV_EMPTY) continue;
        int f[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) f[k] = g[i + 1 + fry(k)][1 + frx(k)];
        // (a change next to a point without colour is no gap)
        int gaps = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int a = f[k], b = f[(k + 1) & 7];
            gaps += (a != b && a != DV_EMPTY && b != DV_EMPTY) ? 1 : 0;
        }
        vmask |= gaps >= 3 ? 1u << i : 0u;
    }
    // The neighbour rules at the wave's vertex sites, which are few: the
    // sites are listed in lane order (a wave prefix of the per-lane counts)
    // and each takes four lanes, lane r applying the first- and
    // second-neighbour rules of frame direction r (spx, spy, smx, smy rotated
    // by quarter turns).  A second-neighbour candidate goes to the mask of
    // the thread owning the site (bit 4i + r), read back below.
    // (a wave without vertex sites, the usual case, skips both steps)
    const int vcnt = __popc(vmask);
    const int vinc = wave_incl_sum(vcnt);
    const int vtotal = wave_last(vinc);
    if (vtotal > 0) {
        S.pendw[t] = 0u;
        const int cnt = vcnt, inc = vinc, total = vtotal;
        for (int p0 = 0; p0 < total; p0 += 16) {
            const int item = min(p0 + (lane >> 2), total - 1), r = lane & 3;
            // lane holding the item: the first one whose inclusive count exceeds it
            int L = 0;
            for (int step = 32; step > 0; step >>= 1)
                L += __shfl(inc, L + step - 1, 64) <= item ? step : 0;
            unsigned m = (unsigned)__shfl((int)vmask, L, 64);
            for (int k = item - (__shfl(inc, L, 64) - __shfl(cnt, L, 64)); k > 0; --k) m &= m - 1;
            const int i = __ffs(m) - 1;
            const int tl = (t & ~63) | L;
            const int c = (4 * (tl >> 5) + i + 1) * 34 + (tl & 31) + 1;
            const int k0 = 2 * r, k1 = (2 * r + 2) & 7, k7 = (2 * r + 7) & 7;
            const int ckk = S.own[c];
            const int tg = S.own[c + fry(k0) * 34 + frx(k0)];
            const int pa = S.own[c + fry(k1) * 34 + frx(k1)], pb = S.own[c + fry(k7) * 34 + frx(k7)];
            const int dg = S.own[c + fry(k0 + 1) * 34 + frx(k0 + 1)];
            if (p0 + (lane >> 2) < total) {
                if ((!GEOM || tg != DV_EMPTY) && pa != pb && tg != ckk) emit(min(ckk, tg), max(ckk, tg));
                if ((!GEOM || dg != DV_EMPTY) && dg != ckk && pa != pb && pa != tg)
                    atomicOr(&S.pendw[tl], 1u << (4 * i + r));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const unsigned pend = S.pendw[t];   // bit 4i + r: site i needs the colour of inner-frame point r
        // Inner-frame queries, which are few: numbered within the wave (a wave
        // prefix of the per-lane counts) and answered one per lane, 64 at a time.
        const int qcnt = __popc(pend);
        const int qinc = wave_incl_sum(qcnt);
        const int qtotal = wave_last(qinc);
        for (int p0 = 0; p0 < qtotal; p0 += 64) {
            const int cnt = qcnt, inc = qinc, total = qtotal;
            const int item = min(p0 + lane, total - 1);
            // lane holding the item: the first one whose inclusive count exceeds it
            int L = 0;
            for (int step = 32; step > 0; step >>= 1)
                L += __shfl(inc, L + step - 1, 64) <= item ? step : 0;
            unsigned m = (unsigned)__shfl((int)pend, L, 64);
            for (int k = item - (__shfl(inc, L, 64) - __shfl(cnt, L, 64)); k > 0; --k) m &= m - 1;
            if (p0 + lane >= total) continue;
            const int bit = __ffs(m) - 1, r = bit & 3;
            const int tl = (t & ~63) | L;
            const int qsx = tl & 31, qsy = 4 * (tl >> 5) + (bit >> 2);
            int mq;
            if (in_lds && imode) {
                // (the packed form of the evaluation; |2 q| <= 16128 as for the sites)
                const sh2 q2 = sh2{(short)(-2 * (256 * qsx + inx(r))), (short)(-2 * (256 * qsy + iny(r)))};
                int bee = INT_MAX;
                mq = DV_EMPTY;
                // the single chunk is ordered by label: ties keep the first
                for (int k = 0; k < ncl; ++k) {
                    const int e = dot2_acc(q2, __builtin_bit_cast(sh2, S.ixy[k]), S.ik[k]);
                    const bool lt = e < bee;
                    bee = lt ? e : bee;
                    mq = lt ? S.sl[k] : mq;
                }
            } else if (in_lds) {
                const double qx = -2.0 * (256.0 * qsx + inx(r)), qy = -2.0 * (256.0 * qsy + iny(r));
                double bee = 1.0e300;
                mq = DV_EMPTY;
                // the single chunk is ordered by label: ties keep the first
                for (int k = 0; k < ncl; ++k) {
                    const double e = fma(qx, S.sx[k], fma(qy, S.sy[k], S.sk[k]));
                    const bool lt = e < bee;
                    bee = lt ? e : bee;
                    mq = lt ? S.sl[k] : mq;
                }
            } else {
                // (on a walled axis the point is inside: its diagonal
                // partner has a colour)
                int X = OX + 256 * qsx + inx(r), Y = OY + 256 * qsy + iny(r);
                if (X < 0) X += MX;
                if (Y < 0) Y += MY;
                mq = point_nearest(B, X, Y);
            }
            const int c = (qsy + 1) * 34 + qsx + 1;
            const int ckk = S.own[c];
            const int dg = S.own[c + fry(2 * r + 1) * 34 + frx(2 * r + 1)];
            if (mq == dg || mq == ckk) emit(min(ckk, dg), max(ckk, dg));
        }
    }
    __syncthreads();
    // --- distinct couples of the tile into the rows
    // (a group of GL lanes per couple looks for an earlier copy; one wave holds
    // whole groups, and a ballot ORs the group's answers)
    const int np = min(S.npair, PAIR_CAP);
    int GL = 64;
    while (GL > 1 && np * GL > DV_BLOCK) GL >>= 1;
    const int sub = t & (GL - 1);
    const unsigned long long gmask = (GL == 64 ? ~0ull : ((1ull << GL) - 1ull)) << ((t & 63) & ~(GL - 1));
    for (int i0 = 0; i0 < np; i0 += DV_BLOCK / GL) {
        const int i = i0 + t / GL;
        unsigned long long key = 0;
        bool dup = false;
        if (i < np) {
            key = S.pair[i];
            for (int j = sub; j < i; j += GL)
                if (S.pair[j] == key) { dup = true; break; }
        }
        const bool first = i < np && !(__ballot(dup) & gmask);
        if (!first || sub != 0) continue;
        const int a = (int)(key >> 32), b = (int)(key & 0xffffffffu);
        row_insert(B, a, b, fs);
        row_insert(B, b, a, fs);
    }
}

// ---- the usual case of a tile, by one wave ---------------------------------
#define OWNER_WAVES 4     // tiles, a wave each, of a block of k_owner_edges
#define FAST_CAND 64      // candidates (a lane each)
#define FAST_ITEMS 512    // centres in the cells around a tile
#define FAR_CELLS 12      // cells on either side looked at around a tile in a wide void
enum { TILE_DONE, TILE_FAR, TILE_GENERAL };
#define RANK_NONE 0x7f    // colour code of a site without colour
struct FastLds {
    union {
        struct {
            int lab[128];                      // label of each colour code
            unsigned long long adj[FAST_CAND]; // couples of the tile: bit b of adj[a], a < b
            uint16_t list[DV_TILE_SITES];      // vertex sites, y << 5 | x
            // candidates gathered in passes; the code that stands for a code's
            // label (several images of one centre have codes of their own)
            int cx[FAST_CAND], cy[FAST_CAND], cl[FAST_CAND];
            int canon[FAST_CAND];
        };
        // (label map, after the colouring)
        struct {
            int2 runlab[DV_TILE_PIECES + 1];   // -1 and the label of each run
            uint2 rows[DV_TILE];               // changes along each row, twice the runs before it
        };
    };
};

// What a tile's label map is made from, loaded ahead of its use: the row masks,
// and the piece slots and labels of the first 64 runs.
struct LabelLoads {
    uint32_t m = 0;
    int slot0 = 0, lab0 = 0;
    bool have = false;
    __device__ __forceinline__ void first(const Bufs &B, int tile) {
        const int lane = threadIdx.x & 63;
        m = lane < DV_TILE ? gmem(B.tmask)[(size_t)tile * DV_TILE + lane] : 0u;
        slot0 = gmem(B.trun)[run_at(B, tile, lane)];   // (in use or not)
    }
    __device__ __forceinline__ void second(const Bufs &B, int tile) {
        const int lane = threadIdx.x & 63;
        const int nruns = wave_last(wave_incl_sum(__popc(m & ~(m << 1))));
        if (lane < nruns) lab0 = gmem(B.prank)[piece_at(B, tile, slot0)];
        have = true;
    }
};

// The tile's part of the label map, by the wave that coloured it: the table
// holds -1 and the run's label for every run, and a site's entry is the number
// of changes in its row up to it (even outside) after twice the runs of the rows
// above.  It rides along because its stores overlap the colouring's VALU work
// (a kernel of its own: 329 us per 20 frames of 4096^2).
__device__ __forceinline__ void label_tile(const Bufs &B, int tile, LabelLoads &Q, FastLds &S) {
    const int lane = threadIdx.x & 63;
    const int x0 = (tile % B.ntx) * DV_TILE, y0 = (tile / B.ntx) * DV_TILE;
    const int lx = B.lx, tw = min(DV_TILE, lx - x0), th = min(DV_TILE, B.ly - y0);
    if (!Q.have) Q.second(B, tile);
    const uint32_t m = Q.m;
    const int rc = __popc(m & ~(m << 1));
    const int rinc = wave_incl_sum(rc), nruns = wave_last(rinc);
    if (lane < DV_TILE) S.rows[lane] = make_uint2(m ^ (m << 1), 2u * (unsigned)(rinc - rc));
    for (int i = lane; i <= nruns; i += 64) {
        int lab = Q.lab0;
        if (i >= 64 && i < nruns) {
            const int slot = gmem(B.trun)[run_at(B, tile, i)];
            lab = gmem(B.prank)[piece_at(B, tile, slot)];
        }
        S.runlab[i] = make_int2(-1, lab);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int col = lane & 31, h = lane >> 5;
    const uint32_t upto = (2u << col) - 1u;
    const int nrow = min(max(th - 16 * h, 0), 16);
    const int *tab = &S.runlab[0].x;
    // (uniform row address, 32-bit lane offset)
    auto row = reinterpret_cast<__attribute__((address_space(1))) char *>(gmem(B.labels) + (size_t)y0 * lx + x0);
    const unsigned off = 4u * (unsigned)(16 * h * lx + col);
    if ((lx & 31) == 0 && th == DV_TILE) {
#pragma unroll
        for (int a = 0; a < 16; ++a, row += (size_t)lx * 4) {
            const uint2 r = S.rows[16 * h + a];
            st_map<true>(row, off, tab[r.y + __popc(r.x & upto)]);
        }
    } else if (col < tw) {
#pragma unroll
        for (int a = 0; a < 16; ++a, row += (size_t)lx * 4) {
            const uint2 r = S.rows[16 * h + a];
            if (a < nrow) st_map<false>(row, off, tab[r.y + __popc(r.x & upto)]);
        }
    }
}

// Bit 7 of every byte of x that is not zero (bytes below 0x80), over the eight
// registers of a lane's column: register i holds the rows i, i + 8, i + 16, so
// shifting the bits of one register down while the next is added leaves row a
// at bit a.
__device__ __forceinline__ uint32_t add_rows(uint32_t acc, uint32_t x) {
    return (acc >> 1) | ((x + 0x7f7f7fu) & 0x808080u);
}

// Colouring, vertex test and neighbour rules of one tile by one wave.  Nothing is
// written when the tile is left to others: TILE_FAR in a void wider than its keys
// reach, TILE_GENERAL.  Q: the loads of the tile's label map, issued here behind
// those the colouring waits for.
//
// What bounds it is VALU issue, so nothing is done per site that can be done
// per row, per column or per candidate:
//  - candidates: the centres of the 7 x 7 cells around the tile, a lane each;
//    those within the radius that the nearest one implies are tested against
//    each other (a centre that another one beats everywhere in the window owns
//    nothing) by their distances to the window's four corners, in exact 32-bit
//    integers;
//  - colours: |c|^2 - 2 w.c of a window point w (in half sites, p) is 256 (q -
//    p.c) + r with |c|^2 = 256 q + r, so with the kept centres ranked by (r,
//    label) the key (q - p.c) << 8 | rank orders them by distance, then label,
//    exactly; a step down a column subtracts a constant, and the nearest centre
//    of a site is the least key: two additions and a three-way minimum for two
//    candidates (all within 112 sites of the tile, so keys fit 32 bits);
//  - lane l holds column l & 31, rows 16 (l >> 5) - 1 .. + 16; the columns left
//    and right of the tile are a point per lane;
//  - changes along and across the rows: four colours per register, compared
//    with the next lane's (or the next row's) at once, one bit per row; the
//    eight terms of the frame-gap count of all rows are added bit-sliced;
//  - the few vertex sites take eight lanes each, a frame point per lane, whose
//    colour is evaluated again (no colour goes through memory but the map's).
// With maps it is 980 VALU and 660 SALU instructions per tile and 3.9 TB/s of
// map writes (678 us per 20 frames of 4096^2; 102 us per 16 frames of 2048^2
// without maps, 84 % of the VALU issue rate).  (The radius by float square roots
// and float bounds, and keys with subtracted products: 1057, 683 and 106 us, and
// 162 instead of 152 us for the channel.)  A block per tile with the window
// in LDS took 522 VALU instructions per wave of 256 sites, 1440 us without the
// label map.
template <bool GEOM>
__device__ __forceinline__ int owner_fast(const Bufs &B, int tile, FastLds &S, LabelLoads &Q) {
    const int lane = threadIdx.x & 63;
    const int tx = tile % B.ntx, ty = tile / B.ntx;
    const bool ox = GEOM && B.open_x, oy = GEOM && B.open_y;
    FrameState *fs = B.fs;
    int ob = 0;   // obstacle bits of the window
    if (GEOM && B.obits) ob = (int)gmem(B.obits)[(size_t)tile * DV_OBITS + min(lane, DV_OBITS - 1)];
    const int lx = B.lx, ly = B.ly;
    const int x0 = tx * DV_TILE, y0 = ty * DV_TILE;
    const int tw = min(DV_TILE, lx - x0), th = min(DV_TILE, ly - y0);
    const int MX = qperiod(lx, ox), MY = qperiod(ly, oy);
    // tile centre (Q.8), and its position relative to site (16, 16) of the tile,
    // the origin of the coordinates below
    const int tcx = 256 * x0 + 128 * (tw - 1), tcy = 256 * y0 + 128 * (th - 1);
    const int ocx = 128 * (tw - 1) - 4096, ocy = 128 * (th - 1) - 4096;
    auto dist2 = [](int dx, int dy) { return (float)dx * (float)dx + (float)dy * (float)dy; };
    int cx = 0, cy = 0, cl = 0;       // the lane's centre, image nearest to the tile centre, relative to it
    int rb0 = 0, pre = 0, nrng = 0, total = 0;
    // centre of item f of the cells around the tile
    auto item = [&](int f, int &dx, int &dy, int &lab) {
        int r = 0;
        for (int k = 1; k < nrng; ++k) r = __builtin_amdgcn_readlane(pre, k) <= f ? k : r;
        const int e = __shfl(rb0, r, 64) + f - __shfl(pre, r, 64);
        if (f < total) {
            const int2 q = ld_int2(B.cell_q, e);
            lab = gmem(B.cell_items)[e];
            dx = wrap_q(q.x - tcx, MX);
            dy = wrap_q(q.y - tcy, MY);
        }
    };
    // Centres of the 7 x 7 cells around the tile, and where these do not hold
    // every candidate (the nearest centre more than 45 sites from the tile
    // centre: 3 % of the tiles of a random field), of the 9 x 9.  Each row of cells
    // of a column span is one contiguous range of the cell-ordered arrays (at
    // most 9 x 2, a lane each).  The radius around the tile centre that holds
    // every centre able to own a window site or inner-frame point is the
    // nearest one's distance + twice the window's half diagonal (rounded down to
    // whole sites from two sites more, which covers the float rounding too).
    int rho = 0;
#pragma unroll 1
    for (int R0 = 3;; ++R0) {
        const Span sx = span_cells(tx, R0, B.ntx, ox), sy = span_cells(ty, R0, B.nty, oy);
        const int n0y = sy.hi0 - sy.lo0 + 1, ncy = n0y + (sy.n == 2 ? sy.hi1 - sy.lo1 + 1 : 0);
        nrng = ncy * sx.n;
        rb0 = 0;
        int rb1 = 0;
        if (lane < nrng) {
            const int iy = sx.n == 2 ? lane >> 1 : lane, c = sx.n == 2 ? lane & 1 : 0;
            const int celly = iy < n0y ? sy.lo0 + iy : sy.lo1 + (iy - n0y);
            const auto cs = gmem(B.cell_start);
            rb0 = cs[celly * B.ntx + sx.lo(c)];
            rb1 = cs[celly * B.ntx + sx.hi(c) + 1];
        }
        if (R0 == 3) {
            if (B.keep_maps) Q.first(B, tile);
            if (*gmem(&fs->err)) return TILE_DONE;
        }
        const int inc = wave_incl_sum(rb1 - rb0);
        total = wave_last(inc);
        pre = inc - (rb1 - rb0);
        if (total > FAST_ITEMS) return TILE_GENERAL;
        item(lane, cx, cy, cl);
        if (R0 == 3 && B.keep_maps) Q.second(B, tile);
        // (distances are not negative: as integers their bits have the same order)
        int dmin = lane < total ? __float_as_int(dist2(cx, cy)) : __float_as_int(3.0e38f);
        for (int f0 = 64; f0 < total; f0 += 64) {
            int dx = 0, dy = 0, lab;
            item(f0 + lane, dx, dy, lab);
            if (f0 + lane < total) dmin = min(dmin, __float_as_int(dist2(dx, dy)));
        }
        const float near = __builtin_amdgcn_sqrtf(__int_as_float(wave_min_bits(dmin)));
        const float diag = __builtin_amdgcn_sqrtf((float)((tw + 1) * (tw + 1) + (th + 1) * (th + 1)));
        rho = __builtin_amdgcn_readfirstlane((int)fminf(near * (1.0f / 256.0f) + diag + 2.0f, 1.0e6f));
        const int wlx = lx - DV_TILE * (B.ntx - 1), wly = ly - DV_TILE * (B.nty - 1);
        const int cov_x = span_full(sx, B.ntx) ? 112 : min(112, DV_TILE * (R0 - 1) + wlx);
        const int cov_y = span_full(sy, B.nty) ? 112 : min(112, DV_TILE * (R0 - 1) + wly);
        if (rho <= cov_x && rho <= cov_y) break;
        if (R0 == 4 || (total > 0 && rho > 112)) return TILE_FAR;
    }
    const float rq2 = (float)(65536 * rho * rho);   // (rho <= 112: below 2^30)
    // on a small lattice another image of a centre can be the nearest one of some
    // points of the window: each image within the radius is a candidate then
    const bool img = (!ox && 2 * (rho + 18) > lx) || (!oy && 2 * (rho + 18) > ly);
    unsigned long long sel;
    if (total <= 64 && !img) {
        sel = __ballot(lane < total && dist2(cx, cy) <= rq2);
    } else {
        // (images one period away are all there are within the radius)
        if (img && ((!ox && 2 * rho > 3 * lx) || (!oy && 2 * rho > 3 * ly))) return TILE_GENERAL;
        const int ix = img && !ox ? 1 : 0, iy = img && !oy ? 1 : 0;
        int nc = 0;
        for (int f0 = 0; f0 < total; f0 += 64) {
            int dx = 0, dy = 0, lab = 0;
            item(f0 + lane, dx, dy, lab);
            for (int k = -iy; k <= iy; ++k)
                for (int j = -ix; j <= ix; ++j) {
                    const int ax = dx + j * MX, ay = dy + k * MY;
                    const bool in = f0 + lane < total && dist2(ax, ay) <= rq2;
                    const unsigned long long b = __ballot(in);
                    const int slot = nc + __popcll(b & ((1ull << lane) - 1ull));
                    if (in && slot < FAST_CAND) {
                        S.cx[slot] = ax;
                        S.cy[slot] = ay;
                        S.cl[slot] = lab;
                    }
                    nc += __popcll(b);
                }
        }
        if (nc > FAST_CAND) return TILE_GENERAL;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        sel = nc == 64 ? ~0ull : (1ull << nc) - 1ull;
        const bool use = (sel >> lane) & 1ull;
        cx = use ? S.cx[lane] : 0;
        cy = use ? S.cy[lane] : 0;
        cl = use ? S.cl[lane] : 0;
    }
    cx += ocx;
    cy += ocy;
    // (|c| <= 112 sites + 16 for a ragged tile's centre: 256 c within 2^23, squares
    // and corner values within 2^31)
    const int kc = __mul24(cx, cx) + __mul24(cy, cy);
    // |w|^2 less than the squared distance at the window's corners w = 256 s: the
    // difference of two centres' is affine in w, so a centre farther than another
    // one at all four is farther everywhere in the window
    int d00, d01, d10, d11;
    {
        const int x0c = __mul24(cx, -17), x1c = __mul24(cx, tw - 16);
        const int y0c = __mul24(cy, -17), y1c = __mul24(cy, th - 16);
        d00 = kc - 512 * (x0c + y0c);
        d01 = kc - 512 * (x1c + y0c);
        d10 = kc - 512 * (x0c + y1c);
        d11 = kc - 512 * (x1c + y1c);
    }
    bool beaten = false;
    for (unsigned long long m = sel; m; m &= m - 1) {
        const int j = (int)__builtin_ctzll(m);
        beaten |= (d00 > __builtin_amdgcn_readlane(d00, j)) & (d01 > __builtin_amdgcn_readlane(d01, j)) &
                  (d10 > __builtin_amdgcn_readlane(d10, j)) & (d11 > __builtin_amdgcn_readlane(d11, j));
    }
    const bool kept = ((sel >> lane) & 1ull) && !beaten;
    const unsigned long long mk = __ballot(kept);
    const int nk = __popcll(mk);
    // rank by (|c|^2 mod 256, label); labels are below 2^24.  (Images of one centre
    // at the same remainder: by lane, so that every candidate has its own.)
    const unsigned ord = ((unsigned)kc << 24) | (unsigned)cl;
    int rank = 0;
    for (unsigned long long m = mk; m; m &= m - 1)
        rank += (unsigned)__builtin_amdgcn_readlane((int)ord, (int)__builtin_ctzll(m)) < ord ? 1 : 0;
    if (img) {
        for (unsigned long long m = mk; m; m &= m - 1) {
            const int j = (int)__builtin_ctzll(m);
            rank += (unsigned)__builtin_amdgcn_readlane((int)ord, j) == ord && j < lane ? 1 : 0;
        }
        int canon = rank;
        for (unsigned long long m = mk; m; m &= m - 1) {
            const int j = (int)__builtin_ctzll(m);
            const int rj = __builtin_amdgcn_readlane(rank, j);
            canon = __builtin_amdgcn_readlane(cl, j) == cl ? min(canon, rj) : canon;
        }
        if (kept) S.canon[rank] = canon;
    }
    const int kbase = (int)(((unsigned)kc >> 8) << 8) | rank;
    const int kx = -256 * cx, ky = -256 * cy;
    if (kept) S.lab[rank] = cl;
    if (lane == 0) S.lab[RANK_NONE] = DV_EMPTY;
    S.adj[lane] = 0ull;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();

    // key of candidate j at the point p (half sites)
    auto key = [&](int j, int px, int py) {
        return __mul24(py, __builtin_amdgcn_readlane(ky, j)) +
               (__mul24(px, __builtin_amdgcn_readlane(kx, j)) + __builtin_amdgcn_readlane(kbase, j));
    };
    const int col = lane & 31, h = lane >> 5;
    int best[18];   // rows 16 h - 1 + a
    // the columns beside the tile (x = -1 and 32), row `col`, and the tile's
    // column next to them (one inwards); the same at the window's corners
    const int ex = h ? 32 : -34, ey = 2 * (col - 16), ei = h ? -2 : 2;
    const int fx = (lane & 1) ? 32 : -34, fy = (lane & 2) ? 32 : -34, fi = (lane & 1) ? -2 : 2;
    int bp, bq, cp, cq;
    {
        const int px = 2 * (col - 16), py = 2 * (16 * h - 17);
        // candidates j and i into the least keys (FIRST: which start with them)
        auto two = [&](auto first, int j, int i) {
            constexpr bool FIRST = decltype(first)::value;
            auto least = [&](int &b, int u, int v) { b = FIRST ? min(u, v) : min(min(b, u), v); };
            const int kyj = __builtin_amdgcn_readlane(ky, j), kyi = __builtin_amdgcn_readlane(ky, i);
            const int kxj = __builtin_amdgcn_readlane(kx, j), kxi = __builtin_amdgcn_readlane(kx, i);
            int k1 = key(j, px, py), k2 = key(i, px, py);
#pragma unroll
            for (int a = 0; a < 18; ++a) {
                least(best[a], k1, k2);
                k1 += 2 * kyj;
                k2 += 2 * kyi;
            }
            k1 = key(j, ex, ey);
            k2 = key(i, ex, ey);
            least(bp, k1, k2);
            least(bq, k1 + __mul24(ei, kxj), k2 + __mul24(ei, kxi));
            k1 = key(j, fx, fy);
            k2 = key(i, fx, fy);
            least(cp, k1, k2);
            least(cq, k1 + __mul24(fi, kxj), k2 + __mul24(fi, kxi));
        };
        // (the last of an odd number: paired with itself)
        auto next = [](unsigned long long &m) {
            const int j = (int)__builtin_ctzll(m);
            m &= m - 1;
            return j;
        };
        unsigned long long m = mk;
        int j = next(m), i = m ? next(m) : j;
        two(std::true_type{}, j, i);
        while (m) {
            j = next(m);
            i = m ? next(m) : j;
            two(std::false_type{}, j, i);
        }
    }
    bp &= 0xff;
    bq &= 0xff;
    cp &= 0xff;
    cq &= 0xff;
    if (img) {   // one code per label
#pragma unroll
        for (int a = 0; a < 18; ++a) best[a] = S.canon[best[a] & 0xff];
        bp = S.canon[bp];
        bq = S.canon[bq];
        cp = S.canon[cp];
        cq = S.canon[cq];
    }
    // sites without colour: beyond a wall, and obstacles.  Lane r holds row r - 1
    // of the window, `row_none` the columns 0 .. 31, `side_none` the columns left
    // (bit 0) and right (bit 1) of the tile; most tiles have none.  (A byte of the
    // mask loaded per site, and the vertex test in tiles of one colour too: 215 us
    // for 32 frames of a 2048 x 1024 channel with posts, this way 162; reading the
    // bits also took the labelling of those from 148 to 89 us.)
    uint32_t row_none = 0, side_none = 0;
    bool any_none = false;
    if (GEOM) {
        if (B.obits) {
            const int left = h ? __builtin_amdgcn_readlane(ob, 35) : __builtin_amdgcn_readlane(ob, 34);
            const int right = h ? __builtin_amdgcn_readlane(ob, 37) : __builtin_amdgcn_readlane(ob, 36);
            row_none = lane < 34 ? (uint32_t)ob : 0u;
            side_none = (((uint32_t)left >> col) & 1u) | ((((uint32_t)right >> col) & 1u) << 1);
        }
        if (ox && x0 == 0) side_none |= 1u;
        if (ox && x0 + tw == lx) {
            side_none |= 2u;
            if (tw < 32) row_none |= 1u << tw;
        }
        if (oy && ((y0 == 0 && lane == 0) || (y0 + th == ly && lane == th + 1))) {
            row_none = ~0u;
            side_none = 3u;
        }
        any_none = __ballot(lane < th + 2 && (row_none | side_none) != 0u) != 0ull;
    }
    if (GEOM && any_none) {
        // (lanes and rows beyond a ragged tile's ring read its last one)
        const int xc = min(col, tw);
#pragma unroll
        for (int a = 0; a < 18; ++a) {
            const int up = __builtin_amdgcn_readlane((int)row_none, min(a, th + 1));
            const int dn = __builtin_amdgcn_readlane((int)row_none, min(16 + a, th + 1));
            if (((uint32_t)(h ? dn : up) >> xc) & 1u) best[a] = RANK_NONE;
        }
        // (lane moves: every lane takes part)
        const int yc = min(col, th) + 1, yr = (lane & 2) ? th + 1 : 0;
        const uint32_t rc = (uint32_t)__shfl((int)row_none, yc, 64), sc = (uint32_t)__shfl((int)side_none, yc, 64);
        const uint32_t rr = (uint32_t)__shfl((int)row_none, yr, 64), sr = (uint32_t)__shfl((int)side_none, yr, 64);
        if ((sc >> h) & 1u) bp = RANK_NONE;
        if ((rc >> (h ? tw - 1 : 0)) & 1u) bq = RANK_NONE;
        if ((sr >> (lane & 1)) & 1u) cp = RANK_NONE;
        if ((rr >> ((lane & 1) ? tw - 1 : 0)) & 1u) cq = RANK_NONE;
    }
    const int nrow = min(max(th - 16 * h, 0), 16);   // the lane's rows inside the tile
    if (B.keep_maps) {
        // (uniform row address, 32-bit lane offset)
        auto row = reinterpret_cast<__attribute__((address_space(1))) char *>(gmem(B.owner) + (size_t)y0 * lx + x0);
        const unsigned off = 4u * (unsigned)(16 * h * lx + col);
        if ((lx & 31) == 0 && th == DV_TILE) {
#pragma unroll
            for (int a = 0; a < 16; ++a, row += (size_t)lx * 4)
                st_map<true>(row, off, S.lab[best[a + 1] & 0xff]);
        } else if (col < tw) {
#pragma unroll
            for (int a = 0; a < 16; ++a, row += (size_t)lx * 4)
                if (a < nrow) st_map<false>(row, off, S.lab[best[a + 1] & 0xff]);
        }
    }
    if (!any_none && nk == 1) {   // one colour: no vertex
        if (lane == 0) gmem(B.tpair_n)[tile] = 0;
        return TILE_DONE;
    }
    // register i: colour codes of the rows i, i + 8, i + 16 of the column
    uint32_t rw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        rw[i] = __builtin_amdgcn_perm((unsigned)best[i + 8], (unsigned)best[i], 0x0c0c0400u);
        if (i < 2) rw[i] = __builtin_amdgcn_perm((unsigned)best[i + 16], rw[i], 0x0c040100u);
    }
    // bit a: the colours of row a change towards the next column, towards the next row
    uint32_t H = 0, V = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        H = add_rows(H, rw[i] ^ (uint32_t)wave_next((int)rw[i], 0));
        V = add_rows(V, rw[i] ^ (i < 7 ? rw[i + 1] : rw[0] >> 8));
    }
    uint32_t E = 0;   // rows without colour
    // (a change next to a point without colour is no gap)
    bool okp = true, okq = true, okc = true, okd = true;
    if (GEOM && any_none) {
#pragma unroll
        for (int i = 0; i < 8; ++i) E = add_rows(E, rw[i] ^ 0x7f7f7fu);
        E = ~E;
        H &= ~(E | (uint32_t)wave_next((int)E, 0));
        V &= ~(E | (E >> 1));
        okp = bp != RANK_NONE;
        okq = bq != RANK_NONE;
        okc = cp != RANK_NONE;
        okd = cq != RANK_NONE;
    }
    // the same for the columns beside the tile: bit r + 1 for row r (left column in
    // the lower lanes, right in the upper)
    const int bn = wave_next(bp, 0);
    const unsigned long long hs = __ballot(bp != bq && okp && okq);
    const unsigned long long vs = __ballot(bp != bn && okp && (!GEOM || bn != RANK_NONE));
    const unsigned hc = (unsigned)__ballot(cp != cq && okc && okd);
    auto side_v = [&](int corner, int edge) -> unsigned long long {
        const int a = __builtin_amdgcn_readlane(cp, corner), b = __builtin_amdgcn_readlane(bp, edge);
        return a != b && (!GEOM || (a != RANK_NONE && b != RANK_NONE)) ? 1ull : 0ull;
    };
    auto side_mask = [&](unsigned long long rows, unsigned long long top, unsigned long long bottom, int n) {
        return (rows << 1) | top | (bottom << n);
    };
    const unsigned long long hl = side_mask(hs & 0xffffffffull, hc & 1u, (hc >> 2) & 1u, 33);
    const unsigned long long hr = side_mask(hs >> 32, (hc >> 1) & 1u, (hc >> 3) & 1u, 33);
    const unsigned long long vl = side_mask(vs & 0x7fffffffull, side_v(0, 0), side_v(2, 31), 32);
    const unsigned long long vr = side_mask((vs >> 32) & 0x7fffffffull, side_v(1, 32), side_v(3, 63), 32);
    auto half = [&](unsigned long long m) { return h ? (uint32_t)(m >> 16) : (uint32_t)m; };
    const bool lft = col == 0, rgt = col == 31;
    // (lane moves: every lane takes part)
    const uint32_t hp = (uint32_t)wave_prev((int)H, 0), vp = (uint32_t)wave_prev((int)V, 0);
    const uint32_t vn = (uint32_t)wave_next((int)V, 0);
    const uint32_t HR = rgt ? half(hr) : H;
    const uint32_t HL = lft ? half(hl) : hp;
    const uint32_t VL = lft ? half(vl) : vp;
    const uint32_t VR = rgt ? half(vr) : vn;
    // frame of row a: the changes along rows a - 1 and a + 1 and down the columns on
    // both sides, rows a - 1 to a and a to a + 1; three or more of the eight
    uint32_t vm;
    {
        const uint32_t i0 = HL << 1, i1 = HR << 1, i2 = HL >> 1, i3 = HR >> 1;
        const uint32_t i4 = VL << 1, i5 = VR << 1, i6 = VL, i7 = VR;
        auto maj = [](uint32_t a, uint32_t b, uint32_t c) { return (a & b) | (c & (a | b)); };
        const uint32_t s1 = i0 ^ i1 ^ i2, c1 = maj(i0, i1, i2);
        const uint32_t s2 = i3 ^ i4 ^ i5, c2 = maj(i3, i4, i5);
        const uint32_t s3 = i6 ^ i7, c3 = i6 & i7;
        const uint32_t s4 = s1 ^ s2 ^ s3, c4 = maj(s1, s2, s3);
        // s4 + 2 (c1 + c2 + c3 + c4) >= 3
        const uint32_t two = maj(c1, c2, c3) | (c4 & (c1 | c2 | c3));
        vm = two | (s4 & (c1 | c2 | c3 | c4));
    }
    vm = ((vm & ~E) >> 1) & ((1u << nrow) - 1u);
    if (col >= tw) vm = 0;
    const int vinc = wave_incl_sum(__popc(vm)), nv = wave_last(vinc);
    for (int slot = vinc - __popc(vm); vm; vm &= vm - 1)
        S.list[slot++] = (uint16_t)(((16 * h + __ffs(vm) - 1) << 5) | col);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // The neighbour rules, eight lanes per vertex site: lane k colours frame point
    // k; the even lanes (k = 2 r: spx, spy, smx, smy) also the inner-frame point of
    // their quarter and apply the first- and second-neighbour rules of direction r,
    // the odd ones also the site itself.
    for (int i0 = 0; i0 < nv; i0 += 8) {
        const int k = lane & 7, i = i0 + (lane >> 3);
        const int sxy = S.list[min(i, nv - 1)];
        const int x = sxy & 31, y = sxy >> 5;
        const int qx = 2 * (x + frx(k) - 16), qy = 2 * (y + fry(k) - 16);
        const int ux = 2 * (x - 16) + ((k & 1) ? 0 : inx(k >> 1) / 128);
        const int uy = 2 * (y - 16) + ((k & 1) ? 0 : iny(k >> 1) / 128);
        int f = INT_MAX, u = INT_MAX;
        for (unsigned long long m = mk; m; m &= m - 1) {
            const int j = (int)__builtin_ctzll(m);
            f = min(f, key(j, qx, qy));
            u = min(u, key(j, ux, uy));
        }
        f &= 0xff;
        u &= 0xff;
        if (img) {
            f = S.canon[f];
            u = S.canon[u];
        }
        if (GEOM && any_none) {
            const int nx = x + frx(k), ny = y + fry(k) + 1;
            const uint32_t rn = (uint32_t)__shfl((int)row_none, ny, 64), sn = (uint32_t)__shfl((int)side_none, ny, 64);
            if (nx < 0 ? sn & 1u : nx >= tw ? sn & 2u : (rn >> nx) & 1u) f = RANK_NONE;
        }
        const int g = lane & 56;
        const int ckk = __shfl(u, g | 1, 64), dg = __shfl(f, g | ((k + 1) & 7), 64);
        const int pa = __shfl(f, g | ((k + 2) & 7), 64), pb = __shfl(f, g | ((k + 7) & 7), 64);
        if (!(k & 1) && i < nv) {
            auto couple = [&](int a, int b) { atomicOr(&S.adj[min(a, b)], 1ull << max(a, b)); };
            if ((!GEOM || f != RANK_NONE) && pa != pb && f != ckk) couple(ckk, f);
            if ((!GEOM || dg != RANK_NONE) && dg != ckk && pa != pb && pa != f && (u == dg || u == ckk))
                couple(ckk, dg);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // the tile's distinct couples to its list (k_rows fills the rows); beyond the
    // list's capacity into the rows directly
    unsigned long long am = S.adj[lane];
    const int ainc = wave_incl_sum(__popcll(am));
    const int la = am ? S.lab[lane] : 0;
    for (int slot = ainc - __popcll(am); am; am &= am - 1, ++slot) {
        const int lb = S.lab[__builtin_ctzll(am)];
        if (slot < DV_TILE_PAIRS) {
            st_int2(B.tpairs, (size_t)tile * DV_TILE_PAIRS + slot, la, lb);
        } else {
            row_insert(B, la, lb, fs);
            row_insert(B, lb, la, fs);
        }
    }
    if (lane == 0) gmem(B.tpair_n)[tile] = min(wave_last(ainc), DV_TILE_PAIRS);
    return TILE_DONE;
}

// A tile in a void wider than the keys of owner_fast reach: most have one colour,
// which takes no keys to find.  The nearest centre to the tile centre owns the
// whole window if it beats every other one (and their images, one period away,
// where the radius reaches them) at the window's four corners: exactly, in 64 bits.
// The others are all centres of the frame where these are few, else those of the 25
// x 25 cells around the tile, if these hold every one within the radius.  Returns
// false (nothing written) when the tile may have several colours.  Such a tile has
// no vertex.  (Every tile of a void by the general form: 20 frames of 4096^2 with
// 10 droplets 5500 us, with 500 3550; this way 1310 and 2320.)
template <bool GEOM>
__device__ __forceinline__ bool far_tile(const Bufs &B, int tile) {
    const int lane = threadIdx.x & 63;
    const int tx = tile % B.ntx, ty = tile / B.ntx;
    const bool ox = GEOM && B.open_x, oy = GEOM && B.open_y;
    const int lx = B.lx, ly = B.ly;
    // (then one period away is all there is)
    if (min(lx, ly) < 2 * DV_TILE) return false;
    const int x0 = tx * DV_TILE, y0 = ty * DV_TILE;
    const int tw = min(DV_TILE, lx - x0), th = min(DV_TILE, ly - y0);
    const int MX = qperiod(lx, ox), MY = qperiod(ly, oy);
    const int tcx = 256 * x0 + 128 * (tw - 1), tcy = 256 * y0 + 128 * (th - 1);   // tile centre (Q.8)
    int ob = 0;   // obstacle bits of the tile's rows
    if (GEOM && B.obits) ob = (int)gmem(B.obits)[(size_t)tile * DV_OBITS + 1 + (lane & 31)];
    // every centre as one range, or a range per row of cells of a column span
    int rb0 = 0, pre = 0, nrng = 1, total = *gmem(&B.fs->K_now);
    const bool every = total <= FAST_ITEMS;
    const Span sx = span_cells(tx, FAR_CELLS, B.ntx, ox), sy = span_cells(ty, FAR_CELLS, B.nty, oy);
    if (!every) {
        const int n0y = sy.hi0 - sy.lo0 + 1, ncy = n0y + (sy.n == 2 ? sy.hi1 - sy.lo1 + 1 : 0);
        nrng = ncy * sx.n;
        int rb1 = 0;
        if (lane < nrng) {
            const int iy = sx.n == 2 ? lane >> 1 : lane, c = sx.n == 2 ? lane & 1 : 0;
            const int celly = iy < n0y ? sy.lo0 + iy : sy.lo1 + (iy - n0y);
            rb0 = gmem(B.cell_start)[celly * B.ntx + sx.lo(c)];
            rb1 = gmem(B.cell_start)[celly * B.ntx + sx.hi(c) + 1];
        }
        const int inc = wave_incl_sum(rb1 - rb0);
        total = wave_last(inc);
        pre = inc - (rb1 - rb0);
        if (total == 0 || total > FAST_ITEMS) return false;
    }
    // centre of item f, its image nearest to the tile centre relative to that
    auto item = [&](int f, int &dx, int &dy, int &lab) {
        int r = 0;
        for (int k = 1; k < nrng; ++k) r = __builtin_amdgcn_readlane(pre, k) <= f ? k : r;
        const int e = __shfl(rb0, r, 64) + f - __shfl(pre, r, 64);
        if (f < total) {
            const int2 q = ld_int2(B.cell_q, e);
            lab = gmem(B.cell_items)[e];
            dx = wrap_q(q.x - tcx, MX);
            dy = wrap_q(q.y - tcy, MY);
        }
    };
    unsigned long long dn = ~0ull;
    int nx = 0, ny = 0, nl = DV_EMPTY;   // (without a centre: MAXLINK)
    for (int f0 = 0; f0 < total; f0 += 64) {
        int dx = 0, dy = 0, lab = 0;
        item(f0 + lane, dx, dy, lab);
        const unsigned long long d = (unsigned long long)((long long)dx * dx + (long long)dy * dy);
        if (f0 + lane < total && d < dn) {
            dn = d;
            nx = dx;
            ny = dy;
            nl = lab;
        }
    }
    const unsigned long long d0 = wave_min_u64(dn);
    const int at = (int)__builtin_ctzll(__ballot(dn == d0));
    nx = __builtin_amdgcn_readlane(nx, at);
    ny = __builtin_amdgcn_readlane(ny, at);
    nl = __builtin_amdgcn_readlane(nl, at);
    if (total > 0) {
        // the radius of owner_fast
        const float diag = __builtin_amdgcn_sqrtf((float)((tw + 1) * (tw + 1) + (th + 1) * (th + 1)));
        const int rho = (int)(__builtin_amdgcn_sqrtf((float)d0) * (1.0f / 256.0f) + diag + 2.0f);
        const int wlx = lx - DV_TILE * (B.ntx - 1), wly = ly - DV_TILE * (B.nty - 1);
        if (!every && ((!span_full(sx, B.ntx) && rho > DV_TILE * (FAR_CELLS - 1) + wlx) ||
                       (!span_full(sy, B.nty) && rho > DV_TILE * (FAR_CELLS - 1) + wly)))
            return false;
        const int ix = !ox && 2 * (rho + 18) > lx ? 1 : 0, iy = !oy && 2 * (rho + 18) > ly ? 1 : 0;
        bool beats = true;
        for (int f0 = 0; f0 < total; f0 += 64) {
            int dx = 0, dy = 0, lab = nl;   // (the centre itself, and lanes without one, pass)
            item(f0 + lane, dx, dy, lab);
            for (int k = -iy; k <= iy; ++k)
                for (int j = -ix; j <= ix; ++j) {
                    const int ax = dx + j * MX, ay = dy + k * MY;
                    const long long least = (long long)ax * ax + (long long)ay * ay - (long long)d0 -
                                            256ll * (tw + 1) * abs(ax - nx) - 256ll * (th + 1) * abs(ay - ny);
                    beats = beats && (least > 0 || lab == nl);
                }
        }
        if (__ballot(!beats)) return false;
    }
    if (lane == 0) gmem(B.tpair_n)[tile] = 0;
    if (B.keep_maps) {
        // two rows at a time
        const int col = lane & 31, h = lane >> 5;
        auto at = gmem(B.owner) + (size_t)y0 * lx + x0;
        for (int y = 0; y < th; y += 2) {
            const int none = h ? __builtin_amdgcn_readlane(ob, y + 1) : __builtin_amdgcn_readlane(ob, y);
            if (y + h < th && col < tw)
                at[(size_t)(y + h) * lx + col] = ((unsigned)none >> col) & 1u ? DV_EMPTY : nl;
        }
    }
    return true;
}

// Where entry v of the launch's lists is: the lists' places, taken in turn, fill the
// arrays of the launch's entries one after another.
__device__ __forceinline__ int *gen_place(const Bufs *D, const Batch &G, int v) {
    const int e = entry_of(G.tbase, G.tpe, G.n, min(v, G.tiles - 1));
    return D[G.idx[e]].gen_list + (v - G.tbase[e]);
}

// A wave per tile; no wave waits for another.  Four neighbouring tiles make a
// block, so that their rows of the maps are written from one place at about one
// time (20 frames of 4096^2: blocks of 1, 2, 4, 8, 16 tiles 836, 799, 754, 781,
// 819 us; with a barrier at the block's end 979).  Tiles that need the general
// form go to the launch's lists (k_rows colours them).
template <bool GEOM>
__global__ __launch_bounds__(64 * OWNER_WAVES, 8) void k_owner_edges(const Bufs *__restrict__ D, Batch G) {
    __shared__ FastLds S[OWNER_WAVES];
    const int w = threadIdx.x >> 6;
    const int gt = __builtin_amdgcn_readfirstlane(blockIdx.x * OWNER_WAVES + w);
    if (gt >= G.tiles) return;
    const int e = entry_of(G.tbase, G.tpe, G.n, gt);
    const Bufs &B = D[G.idx[e]];
    const int tile = gt - G.tbase[e];
    LabelLoads Q;
    int left = owner_fast<GEOM>(B, tile, S[w], Q);
    if (left == TILE_FAR) left = far_tile<GEOM>(B, tile) ? TILE_DONE : TILE_GENERAL;
    if (left == TILE_GENERAL && (threadIdx.x & 63) == 0) {
        gmem(B.tpair_n)[tile] = 0;
        // (turned by one list from each GEN_LISTS tiles to the next, so that the tiles
        // of a column spread over them too)
        int *const counts = D[G.idx[0]].gen_n;
        const int l = (gt + gt / GEN_LISTS) % GEN_LISTS, n = atomicAdd(&counts[l * DV_LINE], 1);
        *gen_place(D, G, n * GEN_LISTS + l) = gt;
        if (n == 0) counts[1] = 1;
    }
    if (B.keep_maps) {
        __builtin_amdgcn_wave_barrier();
        label_tile(B, tile, Q, S[w]);
    }
}

// Rows from the tiles' couple lists: LANES lanes per tile (a tile lists a few
// couples), one lane per couple end.  Rows are sets: a couple found by
// several tiles is stored once.  The first `gen` blocks colour the tiles that
// k_owner_edges left to the general form (usually none: they find the frames'
// lists empty), whose couples go into the rows directly.  The next `match`
// blocks make Phi, which needs the centres alone: beside the rows, for the past
// that a frame has if the rows reject none (k_rematch sees to the rest).
template <int LANES, bool GEOM>
__global__ __launch_bounds__(DV_BLOCK, 8) void k_rows(const Bufs *__restrict__ D, Batch G, int gen, int match) {
    if ((int)blockIdx.x < gen) {
        __shared__ OwnerLds S;
        const int *counts = D[G.idx[0]].gen_n;
        if (!counts[1]) return;
        // lane l holds the number of tiles on list l
        const int n = gmem(counts)[(threadIdx.x & (GEN_LISTS - 1)) * DV_LINE];
        const int inc = wave_incl_sum(n), total = wave_last(inc);
        for (int i = blockIdx.x; i < total; i += gen) {
            const int l = (int)__builtin_ctzll(__ballot(inc > i));
            const int gt = __builtin_amdgcn_readfirstlane(
                *gen_place(D, G, (i - __builtin_amdgcn_readlane(inc - n, l)) * GEN_LISTS + l));
            const int e = entry_of(G.tbase, G.tpe, G.n, gt);
            owner_general<GEOM>(D[G.idx[e]], gt - G.tbase[e], S);
            __syncthreads();
        }
        return;
    }
    if ((int)blockIdx.x < gen + match) {
        match_block(D, G, blockIdx.x - gen);
        return;
    }
    const int gt = (blockIdx.x - gen - match) * (256 / LANES) + (threadIdx.x / LANES);
    const int lane = threadIdx.x % LANES;
    if (gt >= G.tiles) return;
    const int e = entry_of(G.tbase, G.tpe, G.n, gt);
    const Bufs &B = D[G.idx[e]];
    const int tile = gt - G.tbase[e];
    FrameState *fs = B.fs;
    if (fs->err) return;
    const int n = gmem(B.tpair_n)[tile];
    for (int j = lane; j < 2 * n; j += LANES) {
        const int2 p = ld_int2(B.tpairs, (size_t)tile * DV_TILE_PAIRS + (j >> 1));
        if (j & 1) row_insert(B, p.y, p.x, fs);
        else row_insert(B, p.x, p.y, fs);
    }
}

// The obstacle bits of every tile's window from the mask (once per
// dv_set_obstacles), a wave per tile: a load and a ballot for two rows, a lane per
// site, and for each side column, a lane per row.  (A thread per word, its bytes one
// after another, added 18 us to a call for 256^2 and 69 for 4096^2; this way 8 and
// 25, where a frame of a 2048 x 1024 channel then takes 4 us less.)
__global__ __launch_bounds__(256) void k_obits(Bufs B, uint32_t *out) {
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (tile >= B.ncells) return;
    const int x0 = (tile % B.ntx) * DV_TILE, y0 = (tile / B.ntx) * DV_TILE;
    const int tw = min(DV_TILE, B.lx - x0), th = min(DV_TILE, B.ly - y0);
    auto at = [&](int x, int y) -> bool {   // a site of the window
        int ax = x0 + x, ay = y0 + y;
        ax = ax < 0 ? ax + B.lx : (ax >= B.lx ? ax - B.lx : ax);
        ay = ay < 0 ? ay + B.ly : (ay >= B.ly ? ay - B.ly : ay);
        return gmem(B.obst)[(size_t)ay * B.lx + ax] != 0;
    };
    uint32_t v = 0;   // lane i: word i
    const int x = lane & 31;
#pragma unroll
    for (int i = 0; i < 34; i += 2) {
        const int y = i - 1 + (lane >> 5);
        const unsigned long long rows = __ballot(y <= th && x <= tw && at(x, y));
        v = lane == i ? (uint32_t)rows : lane == i + 1 ? (uint32_t)(rows >> 32) : v;
    }
    const bool on = lane <= th + 1;
    const unsigned long long left = __ballot(on && at(-1, lane - 1)), right = __ballot(on && at(tw, lane - 1));
    v = lane == 34 ? (uint32_t)left : lane == 35 ? (uint32_t)(left >> 32) : v;
    v = lane == 36 ? (uint32_t)right : lane == 37 ? (uint32_t)(right >> 32) : v;
    if (lane < DV_OBITS) out[(size_t)tile * DV_OBITS + lane] = v;
}

}  // namespace

void launch_obits(const Bufs &H, uint32_t *obits, hipStream_t s) {
    hipLaunchKernelGGL(k_obits, dim3((H.ncells + 3) / 4), dim3(256), 0, s, H, obits);
}

void launch_voronoi(const Batch &G, hipStream_t s, Prof &P) {
    const int fgrid = (int)std::min<long long>((G.kmax + 1023) / 1024, 256);
    P.begin(ST_FINALIZE, s);
    if (G.small) {
        // (done by k_mid)
    } else if (G.kmax <= CENTRES_MAX) {
        hipLaunchKernelGGL(k_centres, dim3(1, 1, G.n), dim3(1024), 0, s, G.D, G);
    } else {
        int most = 0;   // cells of the largest entry
        for (int e = 0; e < G.n; ++e) most = std::max(most, G.tbase[e + 1] - G.tbase[e]);
        hipLaunchKernelGGL(k_finalize, dim3(fgrid, 1, G.n), dim3(1024), 0, s, G.D, G);
        hipLaunchKernelGGL(k_grid, dim3((most + 255) / 256, 1, G.n), dim3(256), 0, s, G.D, G);
    }
    P.end(ST_FINALIZE, s);
    P.begin(ST_OWNER_EDGES, s);
    const dim3 oblocks((G.tiles + OWNER_WAVES - 1) / OWNER_WAVES), othreads(64 * OWNER_WAVES);
    if (G.geom) hipLaunchKernelGGL(k_owner_edges<true>, oblocks, othreads, 0, s, G.D, G);
    else hipLaunchKernelGGL(k_owner_edges<false>, oblocks, othreads, 0, s, G.D, G);
    P.end(ST_OWNER_EDGES, s);
    P.begin(ST_ROWS, s);
    // An insert is a chain of dependent reads and an exchange.  With the tiles of
    // a few frames the chip is not full and the longest list decides: 16 lanes
    // per tile (256^2 alone: 15 us with 4 lanes, 5.7 with 16; 32 frames of 1024^2,
    // 32,768 tiles: 28 and 22).  With many tiles the lanes without a couple cost
    // more than the chains (20 frames of 4096^2, 327,680 tiles: 91 and 140 us).
    // General-form blocks: enough to fill the chip when every tile needs it.
    const int gen = std::min(G.tiles, 2048);
    const int match = G.cbase[G.n] / match_blocks_div(G.chunk);
    auto rows = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3(gen + match + (G.tiles * lanes + 255) / 256), dim3(256), 0, s, G.D, G, gen,
                           match);
    };
    if (G.tiles <= 65536) G.geom ? rows(k_rows<16, true>, 16) : rows(k_rows<16, false>, 16);
    else G.geom ? rows(k_rows<4, true>, 4) : rows(k_rows<4, false>, 4);
    P.end(ST_ROWS, s);
}
