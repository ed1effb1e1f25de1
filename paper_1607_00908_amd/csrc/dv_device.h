// Device helpers shared by the HIP sources of libdv: exact Q.8 distances
// (minimum image on periodic axes, plain on walled ones) and the bucket grid
// of centres (one cell per 32x32 tile).
#pragma once

#include "dv_internal.h"

// Global-memory view of a buffer pointer read from the slot table.  The table
// lives in device memory, so the compiler cannot tell that its pointers are
// global and would emit flat accesses, which also count against the LDS wait
// counter; accesses through this view are global instructions.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gmem(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}
using gint = __attribute__((address_space(1))) int;

// Index of a tile's piece (run) in the per-piece (per-run) arrays.
__device__ __forceinline__ size_t piece_at(const Bufs &B, int tile, int slot) {
    return slot < DV_PIECES_LO
               ? (size_t)tile * DV_PIECES_LO + slot
               : (size_t)B.ncells * DV_PIECES_LO + (size_t)tile * (DV_TILE_PIECES - DV_PIECES_LO) + (slot - DV_PIECES_LO);
}
__device__ __forceinline__ size_t run_at(const Bufs &B, int tile, int i) {
    return i < DV_RUNS_LO
               ? (size_t)tile * DV_RUNS_LO + i
               : (size_t)B.ncells * DV_RUNS_LO + (size_t)tile * (DV_TILE_PIECES - DV_RUNS_LO) + (i - DV_RUNS_LO);
}

// int2 element i of a buffer, through a global 64-bit access
__device__ __forceinline__ int2 ld_int2(const int2 *p, size_t i) {
    const unsigned long long v = gmem(reinterpret_cast<const unsigned long long *>(p))[i];
    return make_int2((int)(unsigned)v, (int)(unsigned)(v >> 32));
}
__device__ __forceinline__ uint2 ld_uint2(const uint2 *p, size_t i) {
    const unsigned long long v = gmem(reinterpret_cast<const unsigned long long *>(p))[i];
    return make_uint2((unsigned)v, (unsigned)(v >> 32));
}
__device__ __forceinline__ void st_int2(int2 *p, size_t i, int a, int b) {
    gmem(reinterpret_cast<unsigned long long *>(p))[i] =
        (unsigned long long)(unsigned)a | ((unsigned long long)(unsigned)b << 32);
}

// v to a map in device memory at a uniform row address and a 32-bit byte offset
// of the lane.  The maps are written once and not read by any kernel, so where a
// tile's rows are whole lines (WHOLE: the lattice's width is a multiple of 32)
// the stores are marked as streaming: they leave the caches to the tables that
// the kernels share (20 frames of 4096^2 with maps: k_owner_edges 746 -> 699 us,
// all kernels 2067 -> 1962).  Elsewhere a line gets its parts from two tiles and
// the caches have to put them together.
template <bool WHOLE>
__device__ __forceinline__ void st_map(__attribute__((address_space(1))) char *row, unsigned off, int v) {
    if (WHOLE) __builtin_nontemporal_store(v, reinterpret_cast<gint *>(row + off));
    else *reinterpret_cast<gint *>(row + off) = v;
}

// ---- wave-wide operations through DPP lane moves --------------------------
// (every lane of the wave must be active).  Lane moves within rows of 16
// lanes (row_shr), then the last lane of a row broadcast into the rows above
// it (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3); lanes
// without a source take the identity.  The control codes are those of the
// GFX9 data-parallel primitives.
#define DPP_ROW_SHR(n) (0x110 + (n))
#define DPP_WAVE_SHL1 0x130
#define DPP_WAVE_SHR1 0x138
#define DPP_ROW_BCAST15 0x142
#define DPP_ROW_BCAST31 0x143

// inclusive prefix sum over the lanes of the wave
__device__ __forceinline__ int wave_incl_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_SHR(1), 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_SHR(2), 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_SHR(4), 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_SHR(8), 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_BCAST15, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, DPP_ROW_BCAST31, 0xc, 0xf, false);
    return x;
}

// value of the last lane (a scalar)
__device__ __forceinline__ int wave_last(int x) { return __builtin_amdgcn_readlane(x, 63); }

// one step of wave_min_u64: the minimum with the value CTRL moves in
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long min_step_u64(unsigned long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)(unsigned)v, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xf, false);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    return o < v ? o : v;
}

// minimum over the lanes of the wave, in every lane (unsigned 64-bit)
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    v = min_step_u64<DPP_ROW_SHR(1), 0xf>(v);
    v = min_step_u64<DPP_ROW_SHR(2), 0xf>(v);
    v = min_step_u64<DPP_ROW_SHR(4), 0xf>(v);
    v = min_step_u64<DPP_ROW_SHR(8), 0xf>(v);
    v = min_step_u64<DPP_ROW_BCAST15, 0xa>(v);
    v = min_step_u64<DPP_ROW_BCAST31, 0xc>(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}

// value of the previous lane of the wave (lane 0: `first`)
__device__ __forceinline__ int wave_prev(int x, int first) {
    return __builtin_amdgcn_update_dpp(first, x, DPP_WAVE_SHR1, 0xf, 0xf, false);
}

// value of the next lane of the wave (lane 63: `last`)
__device__ __forceinline__ int wave_next(int x, int last) {
    return __builtin_amdgcn_update_dpp(last, x, DPP_WAVE_SHL1, 0xf, 0xf, false);
}

// minimum over the lanes of the wave (a scalar; lanes without a source take INT_MAX)
__device__ __forceinline__ int wave_min_bits(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_SHR(1), 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_SHR(2), 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_SHR(4), 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_SHR(8), 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_BCAST15, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, DPP_ROW_BCAST31, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// value of the lane R places on within the row of 16 lanes (rotated; every
// lane of the row active)
template <int R>
__device__ __forceinline__ int row16(int x) {
    if (R == 0) return x;
    return __builtin_amdgcn_update_dpp(x, x, 0x120 + (R ? R : 1), 0xf, 0xf, false);
}

// For each lane, over the values v of the 16 lanes of its row: any equal to x,
// the number below x.  (Every lane of the wave must make the call.)
template <int R = 0>
__device__ __forceinline__ bool row16_has(int v, int x) {
    if constexpr (R == 16) return false;
    else return (row16<R>(v) == x) | row16_has<R + 1>(v, x);
}
template <int R = 0>
__device__ __forceinline__ int row16_below(int v, int x) {
    if constexpr (R == 16) return 0;
    else return (row16<R>(v) < x ? 1 : 0) + row16_below<R + 1>(v, x);
}

// v in (-M, M) -> signed minimum image in [-M/2, M/2 - 1]  (M = 256 L, even)
__device__ __forceinline__ int wrap_q(int v, int M) {
    const int h = M >> 1;
    if (v >= h) v -= M;
    else if (v < -h) v += M;
    return v;
}

// Wrap period (Q.8) of an axis for distances: 256 L on a periodic axis.  On
// a walled axis 512 L: no difference of two in-domain points (|v| < 256 L)
// reaches half of it, so wrap_q leaves every difference as it is.
__device__ __forceinline__ int qperiod(int L, int open) { return open ? 512 * L : 256 * L; }

// squared distance between Q.8 points; X, Y, cx, cy in [0, 256 L); MX, MY
// wrap periods (qperiod)
__device__ __forceinline__ long long d2q(int X, int Y, int cx, int cy, int MX, int MY) {
    const int dx = wrap_q(X - cx, MX), dy = wrap_q(Y - cy, MY);
    return (long long)dx * dx + (long long)dy * dy;
}

__device__ __forceinline__ int pmod(int v, int m) {
    const int r = v % m;
    return r < 0 ? r + m : r;
}

// Up to two ranges of cell indices along one axis (accessors select between
// two scalars, so a Span never lives in scratch memory).
struct Span {
    int lo0, hi0, lo1, hi1;
    int n;
    __device__ __forceinline__ int lo(int i) const { return i ? lo1 : lo0; }
    __device__ __forceinline__ int hi(int i) const { return i ? hi1 : hi0; }
};

// Cells whose sites meet the site interval [a, b] (integers, a <= b): wrapped
// on a periodic axis, cut at the walls on an open one.
__device__ __forceinline__ Span span_sites(int a, int b, int L, int open) {
    Span s;
    const int ncell = (L + DV_TILE - 1) / DV_TILE;
    if (open) {
        a = max(a, 0);
        b = min(b, L - 1);
        s.lo1 = 0; s.hi1 = -1;
        if (a > b) { s.n = 0; s.lo0 = 0; s.hi0 = -1; }
        else { s.n = 1; s.lo0 = a / DV_TILE; s.hi0 = b / DV_TILE; }
        return s;
    }
    if (b - a >= L - 1) {
        s.n = 1; s.lo0 = 0; s.hi0 = ncell - 1; s.lo1 = 0; s.hi1 = -1;
        return s;
    }
    a = pmod(a, L);
    b = pmod(b, L);
    if (a <= b) {
        s.n = 1; s.lo0 = a / DV_TILE; s.hi0 = b / DV_TILE; s.lo1 = 0; s.hi1 = -1;
    } else {
        s.n = 2; s.lo0 = a / DV_TILE; s.hi0 = ncell - 1; s.lo1 = 0; s.hi1 = b / DV_TILE;
    }
    return s;
}

// Cells within Chebyshev cell distance R of cell c (no repeats; wrapped on a
// periodic axis, cut at the walls on an open one).
__device__ __forceinline__ Span span_cells(int c, int R, int ncell, int open) {
    Span s;
    if (open) {
        s.n = 1; s.lo0 = max(c - R, 0); s.hi0 = min(c + R, ncell - 1); s.lo1 = 0; s.hi1 = -1;
        return s;
    }
    if (2 * R + 1 >= ncell) {
        s.n = 1; s.lo0 = 0; s.hi0 = ncell - 1; s.lo1 = 0; s.hi1 = -1;
        return s;
    }
    const int a = c - R, b = c + R;
    if (a < 0) {
        s.n = 2; s.lo0 = a + ncell; s.hi0 = ncell - 1; s.lo1 = 0; s.hi1 = b;
    } else if (b >= ncell) {
        s.n = 2; s.lo0 = a; s.hi0 = ncell - 1; s.lo1 = 0; s.hi1 = b - ncell;
    } else {
        s.n = 1; s.lo0 = a; s.hi0 = b; s.lo1 = 0; s.hi1 = -1;
    }
    return s;
}

__device__ __forceinline__ bool span_full(const Span &s, int ncell) {
    return s.n == 1 && s.lo0 == 0 && s.hi0 == ncell - 1;
}

// Nearest now centre of the Q.8 point (X, Y) in [0, 256 lx) x [0, 256 ly),
// exact, ties to the lowest label, by the bucket grid.  K >= 1.  First a growing square of
// cells around the point's cell until a centre is seen; its distance bounds
// the answer, so every cell meeting the disc of that radius (+1 site) around
// the point is then scanned.
__device__ int point_nearest(const Bufs &B, int X, int Y) {
    const int MX = qperiod(B.lx, B.open_x), MY = qperiod(B.ly, B.open_y);
    const int cx = X >> 13, cy = Y >> 13;
    const auto cs = gmem(B.cell_start);
    long long bd = LLONG_MAX;
    for (int R = 1;; R *= 2) {
        const Span sx = span_cells(cx, R, B.ntx, B.open_x), sy = span_cells(cy, R, B.nty, B.open_y);
        for (int ry = 0; ry < sy.n; ++ry)
            for (int row = sy.lo(ry); row <= sy.hi(ry); ++row)
                for (int rx = 0; rx < sx.n; ++rx) {
                    const int e0 = cs[row * B.ntx + sx.lo(rx)], e1 = cs[row * B.ntx + sx.hi(rx) + 1];
                    for (int e = e0; e < e1; ++e) {
                        const int2 q = ld_int2(B.cell_q, e);
                        const long long d = d2q(X, Y, q.x, q.y, MX, MY);
                        if (d < bd) bd = d;
                    }
                }
        if (bd != LLONG_MAX || (span_full(sx, B.ntx) && span_full(sy, B.nty))) break;
    }
    // disc of radius sqrt(bd) + 1 site around the point
    const double rho = sqrt((double)bd) / 256.0 + 1.0;
    const double px = X / 256.0, py = Y / 256.0;
    const Span sx = span_sites((int)floor(px - rho), (int)floor(px + rho), B.lx, B.open_x);
    const Span sy = span_sites((int)floor(py - rho), (int)floor(py + rho), B.ly, B.open_y);
    long long best = LLONG_MAX;
    int bl = DV_EMPTY;
    for (int ry = 0; ry < sy.n; ++ry)
        for (int row = sy.lo(ry); row <= sy.hi(ry); ++row)
            for (int rx = 0; rx < sx.n; ++rx) {
                const int e0 = cs[row * B.ntx + sx.lo(rx)], e1 = cs[row * B.ntx + sx.hi(rx) + 1];
                for (int e = e0; e < e1; ++e) {
                    const int2 q = ld_int2(B.cell_q, e);
                    const long long d = d2q(X, Y, q.x, q.y, MX, MY);
                    const int lab = gmem(B.cell_items)[e];
                    if (d < best || (d == best && lab < bl)) { best = d; bl = lab; }
                }
            }
    return bl;
}

// Lexicographic (distance, label) minimum across a group of GL lanes (an
// aligned part of a wave).
template <int GL>
__device__ __forceinline__ void group_min_dl(long long &d, int &lab) {
    for (int o = GL / 2; o > 0; o >>= 1) {
        const long long d2 = __shfl_xor(d, o, 64);
        const int l2 = __shfl_xor(lab, o, 64);
        if (d2 < d || (d2 == d && l2 < lab)) { d = d2; lab = l2; }
    }
}

// Same search as point_nearest with a group of GL lanes (an aligned part of
// a wave) sharing the cells: lane j of the group takes the (row, column
// range) pairs j, j + GL, ...  Every lane of the group must call it with the
// same point; every lane of the group gets the answer.
template <int GL>
__device__ int group_nearest(const Bufs &B, int X, int Y) {
    const int MX = qperiod(B.lx, B.open_x), MY = qperiod(B.ly, B.open_y);
    const int cx = X >> 13, cy = Y >> 13;
    const int lane = threadIdx.x & (GL - 1);
    const auto cs = gmem(B.cell_start);
    long long bd = LLONG_MAX;
    int dummy = 0;
    for (int R = 1;; R *= 2) {
        const Span sx = span_cells(cx, R, B.ntx, B.open_x), sy = span_cells(cy, R, B.nty, B.open_y);
        const int n0 = sy.hi0 - sy.lo0 + 1, nrows = n0 + (sy.n == 2 ? sy.hi1 - sy.lo1 + 1 : 0);
        for (int j = lane; j < nrows * sx.n; j += GL) {
            const int ri = j / sx.n, c = j % sx.n;
            const int row = ri < n0 ? sy.lo0 + ri : sy.lo1 + (ri - n0);
            const int e0 = cs[row * B.ntx + sx.lo(c)], e1 = cs[row * B.ntx + sx.hi(c) + 1];
            for (int e = e0; e < e1; ++e) {
                const int2 q = ld_int2(B.cell_q, e);
                const long long d = d2q(X, Y, q.x, q.y, MX, MY);
                if (d < bd) bd = d;
            }
        }
        group_min_dl<GL>(bd, dummy);
        if (bd != LLONG_MAX || (span_full(sx, B.ntx) && span_full(sy, B.nty))) break;
    }
    const double rho = sqrt((double)bd) / 256.0 + 1.0;
    const double px = X / 256.0, py = Y / 256.0;
    const Span sx = span_sites((int)floor(px - rho), (int)floor(px + rho), B.lx, B.open_x);
    const Span sy = span_sites((int)floor(py - rho), (int)floor(py + rho), B.ly, B.open_y);
    const int n0 = sy.hi0 - sy.lo0 + 1, nrows = n0 + (sy.n == 2 ? sy.hi1 - sy.lo1 + 1 : 0);
    long long best = LLONG_MAX;
    int bl = DV_EMPTY;
    for (int j = lane; j < nrows * sx.n; j += GL) {
        const int ri = j / sx.n, c = j % sx.n;
        const int row = ri < n0 ? sy.lo0 + ri : sy.lo1 + (ri - n0);
        const int e0 = cs[row * B.ntx + sx.lo(c)], e1 = cs[row * B.ntx + sx.hi(c) + 1];
        for (int e = e0; e < e1; ++e) {
            const int2 q = ld_int2(B.cell_q, e);
            const long long d = d2q(X, Y, q.x, q.y, MX, MY);
            const int lab = gmem(B.cell_items)[e];
            if (d < best || (d == best && lab < bl)) { best = d; bl = lab; }
        }
    }
    group_min_dl<GL>(best, bl);
    return bl;
}

// past components of frame i: slot j's frame, or the shared buffer
struct PastOf {
    CompBuf C;
    int K;
    bool valid;
};

__device__ __forceinline__ PastOf past_of_slot(const Bufs *D, const Batch &G, int i, int j) {
    PastOf r;
    if (j >= 0) {
        r.C = D[G.idx[j]].cur;
        r.K = D[G.idx[j]].fs->K_now;
        r.valid = true;
    } else {
        const SeqState *st = D[G.idx[i]].st + DV_PG_PAR(G.pslot[i]);
        r.C = D[G.idx[i]].past[st->sel];
        r.K = st->past_valid ? st->K[st->sel] : 0;
        r.valid = st->past_valid != 0;
    }
    return r;
}

// Past of frame i (every lane of the calling wave must make the call: lane j
// loads entry j); for one-block-per-frame kernels.
__device__ __forceinline__ PastOf past_of(const Bufs *D, const Batch &G, int i,
                                          unsigned long long accepted) {
    return past_of_slot(D, G, i, past_slot(accepted, i));
}

// (by the scalar walk: the per-row kernels run many waves per frame)
__device__ __forceinline__ PastOf past_of(const Bufs *D, const Batch &G, int i) {
    return past_of_slot(D, G, i, past_slot_walk(D, G, i, DV_E_ANY));
}

#define MATCH_LANES 16
// Phi of the past points blk * (groups of a block), + nblk of those, ... of P for
// the frame of B.
__device__ __forceinline__ void match_points(const Bufs &B, const PastOf &P, int blk, int nblk) {
    const int KP = P.K, KN = B.fs->K_now;
    // a group of MATCH_LANES lanes per past centre (the search of one point
    // rarely visits more cells than that)
    const int lane = threadIdx.x & (MATCH_LANES - 1);
    const int ng = blockDim.x / MATCH_LANES;
    for (int p = blk * ng + (threadIdx.x / MATCH_LANES); p < KP; p += nblk * ng) {
        int n = -1;
        if (KN > 0) n = group_nearest<MATCH_LANES>(B, gmem(P.C.qx)[p], gmem(P.C.qy)[p]);
        if (lane == 0) {
            gmem(B.phi)[p] = n;
            if (n >= 0) {
                atomicAdd(&B.cnt[n], 1);
                gmem(B.inv)[n] = p;
            }
        }
    }
}

// Block b of the matching of a launch (256 threads), before the rows' lengths are
// checked: with the past that an entry has if no row is too long.
__device__ __forceinline__ void match_block(const Bufs *D, const Batch &G, int b) {
    const int per = match_blocks_div(G.chunk);   // comparison blocks of the launch per block of the matching
    const int i = entry_of(G.cbase, G.cpe, G.n, b * per);
    const int blk = b - G.cbase[i] / per, nblk = (G.cbase[i + 1] - G.cbase[i]) / per;
    const Bufs B = D[G.idx[i]];
    if (B.fs->err & DV_E_KMAX) return;
    const PastOf P = past_of_slot(D, G, i, past_slot_walk(D, G, i, DV_E_KMAX));
    if (P.valid) match_points(B, P, blk, nblk);
}

// Block-wide exclusive scan of in[0, n) into out[0, n); returns the total.
// Every thread of the block must call it.  blockDim.x is a multiple of 64.
__device__ int block_exclusive_scan(const int *in, int *out, int n, int *wsum /* LDS [16] */) {
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;
    int carry = 0;
    for (int c0 = 0; c0 < n; c0 += blockDim.x) {
        const int i = c0 + t;
        const int v = i < n ? in[i] : 0;
        const int x = wave_incl_sum(v);
        __syncthreads();
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        int before = carry;
        for (int w = 0; w < wid; ++w) before += wsum[w];
        if (i < n) out[i] = before + x - v;
        int tot = 0;
        for (int w = 0; w < nw; ++w) tot += wsum[w];
        carry += tot;
    }
    return carry;
}

// The same, each thread taking a contiguous run of up to PER elements per
// pass (PER * blockDim.x elements a pass: one pass for the usual sizes), the
// loads of a run issued together.
template <int PER>
__device__ int block_exclusive_scan_wide(const int *in, int *out, int n, int *wsum /* LDS [16] */) {
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;
    const int nthr = (int)blockDim.x;
    int carry = 0;
    for (int c0 = 0; c0 < n; c0 += nthr * PER) {
        const int m = min(n - c0, nthr * PER);
        const int per = (m + nthr - 1) / nthr;
        const int b = c0 + t * per;
        const int e = min(b + per, c0 + m);
        int v[PER];
        int sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v[k] = b + k < e ? in[b + k] : 0;
            sum += v[k];
        }
        const int x = wave_incl_sum(sum);
        __syncthreads();
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        int before = carry + x - sum;
        for (int w = 0; w < wid; ++w) before += wsum[w];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (b + k < e) out[b + k] = before;
            before += v[k];
        }
        int tot = 0;
        for (int w = 0; w < nw; ++w) tot += wsum[w];
        carry += tot;
    }
    return carry;
}

// ---- centres: a component's position from its sums -------------------------
__device__ __forceinline__ long long floor_div(long long a, long long b) {
    long long q = a / b;
    if ((a % b) != 0 && a < 0) q -= 1;
    return q;
}

__device__ __forceinline__ long long pmod64(long long v, long long m) {
    const long long r = v % m;
    return r < 0 ? r + m : r;
}

// floor(256 S / W + 1/2) for W > 0 without forming 512 S (a weighted sum can
// use most of the 64 bits): with S = q W + r, 0 <= r < W, it is
// 256 q + floor((512 r + W) / (2 W)), and 512 r stays far below 2^63.
__device__ __forceinline__ long long q8_round(long long S, long long W) {
    const long long q = floor_div(S, W), r = S - q * W;
    return 256 * q + (512 * r + W) / (2 * W);
}

// Centre k of the frame from its sums (which are left empty for the next
// frame).  Returns its Q.8 position; namb counts ambiguous components.
__device__ __forceinline__ int2 centre_of(const Bufs &B, int k, int &namb) {
    const CompBuf &C = B.cur;
    const long long n = gmem(B.acc_n)[k], sx = gmem(B.acc_x)[k], sy = gmem(B.acc_y)[k];
    const int root = gmem(B.acc_root)[k], amb = gmem(B.acc_amb)[k];
    gmem(B.acc_n)[k] = 0;
    gmem(B.acc_x)[k] = 0;
    gmem(B.acc_y)[k] = 0;
    gmem(B.acc_amb)[k] = 0;
    const int rx = root % B.lx, ry = root / B.lx;
    // weighted centres divide by the total weight, the others by n
    long long W = n;
    if (B.weighted) {
        W = gmem(B.acc_w)[k];
        gmem(B.acc_w)[k] = 0;
    }
    const int qx = (int)pmod64(256LL * rx + q8_round(sx, W), 256LL * B.lx);
    const int qy = (int)pmod64(256LL * ry + q8_round(sy, W), 256LL * B.ly);
    double fx = (double)rx + (double)sx / (double)W;
    double fy = (double)ry + (double)sy / (double)W;
    if (fx < 0) fx += B.lx; else if (fx >= B.lx) fx -= B.lx;
    if (fy < 0) fy += B.ly; else if (fy >= B.ly) fy -= B.ly;
    gmem(C.qx)[k] = qx;
    gmem(C.qy)[k] = qy;
    gmem(C.fx)[k] = fx;
    gmem(C.fy)[k] = fy;
    gmem(C.n)[k] = (int)n;
    gmem(C.root)[k] = root;
    gmem(C.amb)[k] = amb;
    gmem(B.cnt)[k] = 0;
    gmem(B.inv)[k] = -1;
    namb += amb;
    return make_int2(qx, qy);
}

// a rejected frame still leaves the sums it accumulated (ranks below K_max)
// empty for the next frame
__device__ __forceinline__ void drop_sums(const Bufs &B, int k) {
    gmem(B.acc_n)[k] = 0;
    gmem(B.acc_x)[k] = 0;
    gmem(B.acc_y)[k] = 0;
    gmem(B.acc_amb)[k] = 0;
    if (B.weighted) gmem(B.acc_w)[k] = 0;
}

__device__ __forceinline__ int cell_of(const Bufs &B, int2 q) { return (q.y >> 13) * B.ntx + (q.x >> 13); }

// Centres and bucket grid of a frame by one block of 1024 threads, where K_max is
// at most CENTRES_MAX: a thread keeps its centres in registers from the division to the
// scatter.  (As two launches: 3.6 + 4.2 us and a gap for one small frame.)
__device__ __forceinline__ void frame_centres(const Bufs &B, int K, bool rejected, int *wsum /* LDS [16] */) {
    FrameState *fs = B.fs;
    const int t = threadIdx.x;
    if (rejected) {
        for (int k = t; k < min(K, B.kmax); k += 1024) drop_sums(B, k);
        return;
    }
    constexpr int PER = CENTRES_MAX / 1024;
    int2 q[PER];
    int slot[PER], namb = 0;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int k = t + 1024 * p;
        if (k >= K) continue;
        q[p] = centre_of(B, k, namb);
        slot[p] = atomicAdd(&B.cell_count[cell_of(B, q[p])], 1);
    }
    if (namb) atomicAdd(&fs->n_amb, namb);
    __syncthreads();
    // (contiguous runs of up to 16 counts per thread: one pass for up to
    // 16384 cells)
    const int total = block_exclusive_scan_wide<16>(B.cell_count, B.cell_start, B.ncells, wsum);
    if (t == 0) B.cell_start[B.ncells] = total;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int k = t + 1024 * p;
        if (k >= K) continue;
        const int pos = B.cell_start[cell_of(B, q[p])] + slot[p];
        B.cell_items[pos] = k;
        B.cell_q[pos] = q[p];
    }
}
