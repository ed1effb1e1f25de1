// Comparison of every frame of a launch with its past (Sec. 3.2.3 and 3.2.4),
// one launch per step for all of them (k_diff and k_events: the entry of a flat
// block index; k_rematch: blockIdx.x; k_place: blockIdx.z).  The past of
// a frame is the last earlier frame of the batch that passed its stage checks
// (known on the device from the frame headers), else the shared past buffer,
// so the comparisons of a batch are independent of each other.
//
//   match     Phi(p) = nearest now centre of every past centre p, a group
//             of 16 lanes per point through the frame's bucket grid, exact,
//             ties to the lowest label; preimage counts of the now points.
//             Blocks of k_rows do this (match_block); k_rematch repeats it where
//             a past was rejected by its rows.
//   k_diff    16 lanes per now label n (a whole wave for a row beyond its
//             table).  The batch's last accepted frame copies its components
//             and rows into the spare past buffer (the past of the next
//             batch).  When n has exactly one preimage p, lane j holds slot j
//             of the now row of n and slot j of the past row of p translated
//             through Phi (kept entries only).  Rows are sets, so membership
//             is tested by rotating the rows' lanes.  A couple of
//             T(p) missing from R(n) is breaking, one of R(n) missing from
//             T(p) is arising; each is reported once, from the row of its
//             smaller now label, and staged in increasing order of the other
//             end.
//   k_events  (event classification only) one wave per changed row: active
//             neighbours in either graph, boundary points of either graph.
//   k_place   a block per 256 rows: places the staged flips in canonical order
//             (breaking first, then arising, each by (a, b)) in the results
//             page from the chunks' counts; the frame's first block writes its
//             record, that of a sequence's last accepted frame the sequence's
//             next header (the commit).  Kept past and now points correspond
//             one to one, so the number of dropped past points is K_past -
//             (K_now - dropped now points).
#include <algorithm>

#include "dv_device.h"

namespace {

// The matching again for entries whose past has turned out to be another one: a frame
// was rejected by the length of a row (rare; else every block sees in one look at all
// headers that there is none).  An entry's blocks need no order: a past point takes
// its image with the wrong past off the counts and adds the one with the right past;
// inv is written for every point that is counted now.  (The matching as a launch of
// its own behind the rows: 12 us for 32 frames of 1024^2, 8 for 32 of 256^2, 51 for
// 20 of 4096^2; as blocks of k_rows it adds 7, 2 and 43, and this launch takes 2 to
// 5.  With one block per entry, 16 frames of 2048^2 of which two are rejected took
// 695 us here.)
#define REMATCH_BLOCKS 32   // blocks of an entry, at most; one per 256 rows of K_max
__global__ __launch_bounds__(256) void k_rematch(const Bufs *__restrict__ D, Batch G) {
    const int i = blockIdx.x, lane = threadIdx.x & 63;
    const bool late = lane < G.n && D[G.idx[lane]].fs->err == DV_E_DEGREE;
    if (!__ballot(late)) return;
    const Bufs B = D[G.idx[i]];
    if (B.fs->err) return;
    const int j = past_slot_walk(D, G, i, DV_E_ANY), was = past_slot_walk(D, G, i, DV_E_KMAX);
    if (j == was) return;
    const PastOf P = past_of_slot(D, G, i, j);
    if (!P.valid) return;
    const int KP = P.K, KO = past_of_slot(D, G, i, was).K, KN = B.fs->K_now;
    const int ng = blockDim.x / MATCH_LANES;
    for (int p = blockIdx.y * ng + threadIdx.x / MATCH_LANES; p < max(KP, KO); p += gridDim.y * ng) {
        int n = -1;
        if (KN > 0 && p < KP) n = group_nearest<MATCH_LANES>(B, gmem(P.C.qx)[p], gmem(P.C.qy)[p]);
        if ((lane & (MATCH_LANES - 1)) == 0) {
            const int o = p < KO ? gmem(B.phi)[p] : -1;
            if (o >= 0) atomicAdd(&B.cnt[o], -1);
            if (p < KP) gmem(B.phi)[p] = n;
            if (n >= 0) {
                atomicAdd(&B.cnt[n], 1);
                gmem(B.inv)[n] = p;
            }
        }
    }
}

// The row of point n of C, slot `lane` (a row has at most 64): the table, and
// the rest when the table is full.  Every lane of the wave must make the call.
__device__ __forceinline__ int row_slot(const CompBuf &C, int prim, int maxdeg, int n, int lane) {
    int v = lane < prim ? gmem(C.adj)[(size_t)n * prim + lane] : DV_EMPTY;
    const bool full = __popcll(__ballot(v != DV_EMPTY)) == prim;
    if (full && lane >= prim && lane < maxdeg) v = gmem(C.adjx)[(size_t)n * (maxdeg - prim) + lane - prim];
    return v;
}

// Whether x is among the values of v in the lanes of `mask` (wave-uniform).
__device__ __forceinline__ bool wave_has(int v, unsigned long long mask, int x) {
    bool in = false;
    for (; mask; mask &= mask - 1) in |= __builtin_amdgcn_readlane(v, __builtin_ctzll(mask)) == x;
    return in;
}
__device__ __forceinline__ int wave_below(int v, unsigned long long mask, int x) {
    int c = 0;
    for (; mask; mask &= mask - 1) c += __builtin_amdgcn_readlane(v, __builtin_ctzll(mask)) < x ? 1 : 0;
    return c;
}

// A flip into row n's staging area: breaking ones from slot 0, arising ones
// from slot D.
__device__ __forceinline__ void stage_flip(const Bufs &B, int n, int slot, int b, int pa, int pb, int kind) {
    gint *r = gmem(B.stage) + ((size_t)n * (2 * B.maxdeg) + slot) * 6;
    r[0] = n; r[1] = b; r[2] = pa; r[3] = pb; r[4] = kind; r[5] = 0;
}

// Kept now point that slot value q of a past row goes to, else DV_EMPTY.
__device__ __forceinline__ int translated(const Bufs &B, int q) {
    if (q == DV_EMPTY) return DV_EMPTY;
    const int n = gmem(B.phi)[q];
    return n >= 0 && gmem(B.cnt)[n] == 1 ? n : DV_EMPTY;
}

// Row n against the translated past row of its only preimage p, by the whole
// wave (rows of any length).  cb, ca: breaking and arising couples staged.
__device__ __forceinline__ void diff_row_wide(const Bufs &B, const CompBuf &P, int n, int p, int lane, int &cb, int &ca,
                              int &act) {
    const int m = row_slot(B.cur, B.prim, B.maxdeg, n, lane), q = row_slot(P, B.prim, B.maxdeg, p, lane);
    const int mv = (m != DV_EMPTY && gmem(B.cnt)[m] == 1) ? m : DV_EMPTY;
    const int tv = translated(B, q);
    const unsigned long long mm = __ballot(mv != DV_EMPTY), mt = __ballot(tv != DV_EMPTY);
    const bool brk = tv != DV_EMPTY && !wave_has(mv, mm, tv);
    const bool ari = mv != DV_EMPTY && !wave_has(tv, mt, mv);
    const unsigned long long dmask = __ballot(brk || ari);
    act = dmask ? 1 : 0;
    const bool bo = brk && tv > n, ao = ari && mv > n;
    const unsigned long long mb = __ballot(bo), ma = __ballot(ao);
    cb = __popcll(mb);
    ca = __popcll(ma);
    if (bo) stage_flip(B, n, wave_below(tv, mb, tv), tv, p, q, -1);
    if (ao) stage_flip(B, n, B.maxdeg + wave_below(mv, ma, mv), mv, p, gmem(B.inv)[mv], 1);
}

// A row is 64 bytes (its table), so 16 lanes hold it and a wave takes four rows
// at once: the kernel is a chain of dependent loads (now row and preimage, past
// row, its images, their preimage counts), which four rows share.  Rows beyond
// their table are rare and take the whole wave.  A block takes a chunk of
// consecutive rows and stores their counts; only the flip totals, which the
// other frames of the launch need, are summed with an atomic.  (A wave per row
// with 48 slots, and four atomics per block of four rows on one line of the
// frame header: 165 us per 20 frames of 4096^2, 9,000 rows each, 55 us per 32
// frames of 1024^2.  Four rows per wave alone, with a block per 16 rows: 358 us,
// all of it the atomics.)
template <int CHUNK>
__global__ __launch_bounds__(256) void k_diff(const Bufs *__restrict__ Dt, Batch G) {
    __shared__ int4 s_red[4];
    const int i = entry_of(G.cbase, G.cpe, G.n, blockIdx.x);
    const int blk = blockIdx.x - G.cbase[i], nblk = G.cbase[i + 1] - G.cbase[i];
    const Bufs B = Dt[G.idx[i]];
    FrameState *fs = B.fs;
    if (fs->err) return;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int KN = fs->K_now;
    if (blk * CHUNK >= KN) return;
    const PastOf PO = past_of(Dt, G, i);
    const bool pv = PO.valid;
    const CompBuf P = PO.C, N = B.cur, Q = Dt[G.idx[i]].past[1 - B.st[DV_PG_PAR(G.pslot[i])].sel];
    // the sequence's last accepted frame of the launch leaves its copy for the
    // next launch
    bool keep = true;
    for (int q = i + 1; q < G.n && keep && !G.alone; ++q)
        if (Dt[G.idx[q]].seq == B.seq && Dt[G.idx[q]].fs->err == 0) keep = false;
    const int D = B.maxdeg, prim = B.prim;
    const int j = lane & 15, gsh = lane & 48;   // slot of the lane, first lane of its row
    for (int chunk = blk; chunk * CHUNK < KN; chunk += nblk) {
        int e2 = 0, exn = 0, tb = 0, ta = 0;
#pragma unroll 1
        for (int it = 0; it < CHUNK / 16; ++it) {
            const int n = chunk * CHUNK + it * 16 + (t >> 4);
            const bool on = n < KN;
            if (!__ballot(on)) break;
            const int m = on && j < prim ? gmem(N.adj)[(size_t)n * prim + j] : DV_EMPTY;
            const int cn = on ? gmem(B.cnt)[n] : 0;
            const int p = on ? gmem(B.inv)[n] : -1;
            const int dR = __popc((unsigned)(__ballot(m != DV_EMPTY) >> gsh) & 0xffffu);
            const bool longR = dR == prim && prim < D;   // (the row may go on)
            if (keep && on) {
                if (j < prim) gmem(Q.adj)[(size_t)n * prim + j] = m;
                if (longR)
                    for (int k = j; k < D - prim; k += 16)
                        gmem(Q.adjx)[(size_t)n * (D - prim) + k] = gmem(N.adjx)[(size_t)n * (D - prim) + k];
                switch (j) {
                    case 0: gmem(Q.qx)[n] = gmem(N.qx)[n]; break;
                    case 1: gmem(Q.qy)[n] = gmem(N.qy)[n]; break;
                    case 2: gmem(Q.fx)[n] = gmem(N.fx)[n]; break;
                    case 3: gmem(Q.fy)[n] = gmem(N.fy)[n]; break;
                    case 4: gmem(Q.n)[n] = gmem(N.n)[n]; break;
                    case 5: gmem(Q.root)[n] = gmem(N.root)[n]; break;
                    case 6: gmem(Q.amb)[n] = gmem(N.amb)[n]; break;
                    default: break;
                }
            }
            const bool cmp = pv && cn == 1;
            if (pv && on && cn != 1 && j == 0) ++exn;
            const int q = cmp && j < prim ? gmem(P.adj)[(size_t)p * prim + j] : DV_EMPTY;
            const int dT = __popc((unsigned)(__ballot(q != DV_EMPTY) >> gsh) & 0xffffu);
            const bool wide = longR || (dT == prim && prim < D);
            const bool use = cmp && !wide;
            const int mv = (use && m != DV_EMPTY && gmem(B.cnt)[m] == 1) ? m : DV_EMPTY;
            const int tv = use ? translated(B, q) : DV_EMPTY;
            // (lane moves: every lane takes part)
            const bool tin = row16_has(mv, tv), min_ = row16_has(tv, mv);
            const bool brk = tv != DV_EMPTY && !tin;
            const bool ari = mv != DV_EMPTY && !min_;
            const unsigned long long dall = __ballot(brk || ari);
            const unsigned dmask = (unsigned)(dall >> gsh) & 0xffffu;
            int actv = dmask ? 1 : 0, cb = 0, ca = 0, deg = dR;
            if (dall) {
                // each couple once, from the row of its smaller now label
                const bool bo = brk && tv > n, ao = ari && mv > n;
                cb = __popc((unsigned)(__ballot(bo) >> gsh) & 0xffffu);
                ca = __popc((unsigned)(__ballot(ao) >> gsh) & 0xffffu);
                const int bv = bo ? tv : DV_EMPTY, av = ao ? mv : DV_EMPTY;
                const int rb = row16_below(bv, bv), ra = row16_below(av, av);
                if (bo) stage_flip(B, n, rb, tv, p, q, -1);
                if (ao) stage_flip(B, n, D + ra, mv, p, gmem(B.inv)[mv], 1);
            }
            for (unsigned long long w = __ballot(wide && on && j == 0); w; w &= w - 1) {
                const int l = __builtin_ctzll(w);
                const int nw = __builtin_amdgcn_readlane(n, l), pw = __builtin_amdgcn_readlane(p, l);
                const int dw = __popcll(__ballot(row_slot(N, prim, D, nw, lane) != DV_EMPTY));
                int b = 0, a = 0, ac = 0;
                if (__builtin_amdgcn_readlane((int)cmp, l)) diff_row_wide(B, P, nw, pw, lane, b, a, ac);
                if (lane == l) {
                    cb = b;
                    ca = a;
                    actv = ac;
                    deg = dw;
                }
            }
            if (on && j == 0) {
                gmem(B.nb)[n] = cb;
                gmem(B.na)[n] = ca;
                e2 += deg;
                tb += cb;
                ta += ca;
                if (B.classify) gmem(B.act)[n] = actv;
            }
        }
        // the chunk's counts: nonzero only in the lanes j == 0
        for (int o = 16; o < 64; o <<= 1) {
            e2 += __shfl_xor(e2, o, 64);
            exn += __shfl_xor(exn, o, 64);
            tb += __shfl_xor(tb, o, 64);
            ta += __shfl_xor(ta, o, 64);
        }
        if (lane == 0) s_red[wid] = make_int4(tb, ta, e2, exn);
        __syncthreads();
        if (t == 0) {
            int4 a = s_red[0];
            for (int w = 1; w < 4; ++w) {
                a.x += s_red[w].x;
                a.y += s_red[w].y;
                a.z += s_red[w].z;
                a.w += s_red[w].w;
            }
            B.dpart[chunk] = a;
            // flip totals of the frame: k_place puts every frame's flips after
            // those of the frames before it in the results page
            if (a.x | a.y)
                atomicAdd(reinterpret_cast<unsigned long long *>(&fs->nb_acc),
                          (unsigned long long)(unsigned)a.x | ((unsigned long long)(unsigned)a.y << 32));
        }
        __syncthreads();
    }
}

// Event classification (Sec. 3.2.4), for every active now label n (an end of a
// flip): the active points connected to n in either graph, and whether n is a
// boundary point of the now graph and of the translated past graph (one of its
// couples has ends sharing fewer than two neighbours).  Both graphs keep only
// points with exactly one preimage, as in k_diff.

// The same for one row by the whole wave, neighbours' rows one after another
// (rows of any length).
__device__ __forceinline__ void events_row_wide(const Bufs &B, const CompBuf &P, int n, int lane) {
    const int D = B.maxdeg, prim = B.prim;
    const auto cnt = gmem(B.cnt), inv = gmem(B.inv), act = gmem(B.act);
    const int m = row_slot(B.cur, prim, D, n, lane), q = row_slot(P, prim, D, inv[n], lane);
    const int mv = (m != DV_EMPTY && cnt[m] == 1) ? m : DV_EMPTY;
    const int tv = translated(B, q);
    const unsigned long long mm = __ballot(mv != DV_EMPTY), mt = __ballot(tv != DV_EMPTY);
    const bool aR = mv != DV_EMPTY && act[mv];
    const bool aT = tv != DV_EMPTY && !wave_has(mv, mm, tv) && act[tv];
    const int count = __popcll(__ballot(aR)) + __popcll(__ballot(aT));
    bool anyN = false, anyP = false;
    for (unsigned long long k = mm; k; k &= k - 1) {
        const int x = __builtin_amdgcn_readlane(mv, __builtin_ctzll(k));
        const int y = row_slot(B.cur, prim, D, x, lane);
        anyN |= __popcll(__ballot(y != DV_EMPTY && wave_has(mv, mm, y))) < 2;
    }
    for (unsigned long long k = mt; k; k &= k - 1) {
        const int x = inv[__builtin_amdgcn_readlane(tv, __builtin_ctzll(k))];
        const int y = translated(B, row_slot(P, prim, D, x, lane));
        anyP |= __popcll(__ballot(y != DV_EMPTY && wave_has(tv, mt, y))) < 2;
    }
    if (lane == 0) {
        gmem(B.ecnt)[n] = count;
        gmem(B.ebnd)[n] = (anyN ? 1 : 0) | (anyP ? 2 : 0);
    }
}

// Per lane, over the values v of its row of 16 lanes: how many of e[0..16) are
// among them (e's values are distinct, DV_EMPTY never counts).
template <int R = 0>
__device__ __forceinline__ int row16_shared(int v, const int e[16]) {
    if constexpr (R == 16) return 0;
    else {
        const int x = row16<R>(v);
        int c = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) c += e[k] == x ? 1 : 0;
        return (x != DV_EMPTY ? c : 0) + row16_shared<R + 1>(v, e);
    }
}

// 16 lanes per row as in k_diff; lane j reads the whole row (table) of its
// neighbour with loads that do not wait for each other.  (A wave per row with
// the neighbours' entries read one after another: 175 us of 560 us per 12
// frames of 1531 x 877; the chain of dependent loads is what costs.)
__global__ __launch_bounds__(256) void k_events(const Bufs *__restrict__ Dt, Batch G) {
    const int i = entry_of(G.cbase, G.cpe, G.n, blockIdx.x);
    const int blk = blockIdx.x - G.cbase[i], nblk = G.cbase[i + 1] - G.cbase[i];
    const Bufs B = Dt[G.idx[i]];
    const FrameState *fs = B.fs;
    if (!B.classify || fs->err) return;
    const PastOf PO = past_of(Dt, G, i);
    if (!PO.valid) return;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int KN = fs->K_now, D = B.maxdeg, prim = B.prim;
    const int j = lane & 15, gsh = lane & 48;
    const CompBuf P = PO.C, N = B.cur;
    const auto cnt = gmem(B.cnt), inv = gmem(B.inv), act = gmem(B.act);
    for (int n0 = (blk * 4 + wid) * 4; n0 < KN; n0 += nblk * 16) {
        const int n = n0 + (lane >> 4);
        const bool on = n < KN && act[n];
        if (!__ballot(on)) continue;
        const int m = on && j < prim ? gmem(N.adj)[(size_t)n * prim + j] : DV_EMPTY;
        const int p = on ? inv[n] : 0;
        const int q = on && j < prim ? gmem(P.adj)[(size_t)p * prim + j] : DV_EMPTY;
        const int mv = (m != DV_EMPTY && cnt[m] == 1) ? m : DV_EMPTY;
        const int tv = translated(B, q);
        const bool aR = mv != DV_EMPTY && act[mv];
        const bool tin = row16_has(mv, tv);   // (lane moves: every lane takes part)
        const bool aT = tv != DV_EMPTY && !tin && act[tv];
        const int pt = tv != DV_EMPTY ? inv[tv] : 0;
        int e[16];
        bool full = true;   // the neighbour's table is full
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            e[k] = mv != DV_EMPTY && k < prim ? gmem(N.adj)[(size_t)mv * prim + k] : DV_EMPTY;
            if (k < prim) full = full && e[k] != DV_EMPTY;
        }
        const int shN = row16_shared(mv, e);
        const bool bN = mv != DV_EMPTY && shN < 2;
        bool wide = full && mv != DV_EMPTY;
        full = true;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            e[k] = tv != DV_EMPTY && k < prim ? gmem(P.adj)[(size_t)pt * prim + k] : DV_EMPTY;
            if (k < prim) full = full && e[k] != DV_EMPTY;
        }
        // (images of the neighbour's neighbours; only kept points are in tv's row,
        // and two past points never share a kept image)
#pragma unroll
        for (int k = 0; k < 16; ++k) e[k] = e[k] != DV_EMPTY ? gmem(B.phi)[e[k]] : DV_EMPTY;
        const int shP = row16_shared(tv, e);
        const bool bP = tv != DV_EMPTY && shP < 2;
        wide = prim < D && (wide || (full && tv != DV_EMPTY));
        const unsigned nfull = (unsigned)(__ballot(m != DV_EMPTY) >> gsh) & 0xffffu;
        const unsigned pfull = (unsigned)(__ballot(q != DV_EMPTY) >> gsh) & 0xffffu;
        wide = wide || (prim < D && (__popc(nfull) == prim || __popc(pfull) == prim));
        const unsigned gw = (unsigned)(__ballot(wide) >> gsh) & 0xffffu;
        const int count = __popc((unsigned)(__ballot(aR) >> gsh) & 0xffffu) +
                          __popc((unsigned)(__ballot(aT) >> gsh) & 0xffffu);
        const bool anyN = ((unsigned)(__ballot(bN) >> gsh) & 0xffffu) != 0;
        const bool anyP = ((unsigned)(__ballot(bP) >> gsh) & 0xffffu) != 0;
        if (on && j == 0 && !gw) {
            gmem(B.ecnt)[n] = count;
            gmem(B.ebnd)[n] = (anyN ? 1 : 0) | (anyP ? 2 : 0);
        }
        for (unsigned long long w = __ballot(on && j == 0 && gw); w; w &= w - 1)
            events_row_wide(B, P, __builtin_amdgcn_readlane(n, __builtin_ctzll(w)), lane);
    }
}

// flags of a placed flip record (a, b, pa, pb, kind, flags)
__device__ __forceinline__ int event_flags(const Bufs &B, int a, int b, int kind) {
    const auto ecnt = gmem(B.ecnt), ebnd = gmem(B.ebnd);
    int f = (ecnt[a] >= 3 && ecnt[b] >= 3) ? 1 : 0;
    const int bit = kind < 0 ? 2 : 1;
    if ((ebnd[a] & bit) && (ebnd[b] & bit)) f |= 2;
    return f;
}

// n 8-byte words from src to dst (distinct buffers), four loads in flight
__device__ __forceinline__ void copy_words(const int2 *__restrict__ src, int2 *__restrict__ dst, int n) {
    const auto s = gmem(reinterpret_cast<const unsigned long long *>(src));
    const auto d = gmem(reinterpret_cast<unsigned long long *>(dst));
    int j = 0;
    for (; j + 4 <= n; j += 4) {
        const unsigned long long a0 = s[j], a1 = s[j + 1], a2 = s[j + 2], a3 = s[j + 3];
        d[j] = a0;
        d[j + 1] = a1;
        d[j + 2] = a2;
        d[j + 3] = a3;
    }
    for (; j < n; ++j) d[j] = s[j];
}

// Where a row's flips go is the sum of the counts before it.  A block takes 256
// rows, a thread each: the counts of the chunks of k_diff give the sums before
// the block (a few loads per thread, all in flight), a block scan the rest.
// Every block reads the frames' headers for the flips of the earlier frames.
// (That grows with K^2, but from little: 0.28 ms for 2^20 rows and 4.1 for 2^22, where
// one block per frame took 2.2 and 9.6; beyond 9 million rows that would be shorter.)
// (One block per frame over all rows, and a launch for the commit: 43 + 5 us for
// one frame of 4096^2, 9,000 rows.)
#define PLACE_ROWS 256
// 8 bytes at a caller's array of dv_flip, which is 4-byte aligned
struct __attribute__((packed, aligned(4))) Word8 {
    unsigned long long v;
};
__global__ __launch_bounds__(PLACE_ROWS) void k_place(const Bufs *__restrict__ Dt, Batch G) {
    __shared__ int red[8][4];
    const int i = blockIdx.z;
    const Bufs &B = Dt[G.idx[i]];
    FrameState *fs = B.fs;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const bool ok = fs->err == 0;
    const int KN = fs->K_now;
    if (blockIdx.x > 0 && (!ok || (int)blockIdx.x * PLACE_ROWS >= KN)) return;
    // lane j of each wave holds entry j of the launch: which belong to the
    // sequence, which of those were accepted, and their flips
    bool mine = false, good = false;
    int nfl = 0;
    if (G.alone ? lane == i : lane < G.n) {
        const Bufs &Bj = Dt[G.idx[lane]];
        const FrameState *fj = Bj.fs;
        mine = Bj.seq == B.seq;
        good = mine && fj->err == 0;
        if (good) nfl = fj->nb_acc + fj->na_acc;
    }
    const unsigned long long seqm = __ballot(mine), acc = __ballot(good);
    const unsigned long long below = (1ull << i) - 1ull;
    const int ninc = wave_incl_sum(nfl), all_flips = wave_last(ninc);
    const int before = __builtin_amdgcn_readlane(ninc - nfl, i);
    // results page of the frame: the flips of the page before it are those
    // the page held before the launch and those of the earlier accepted frames
    // of the same sequence in the launch (all of one sequence share one page)
    const uint32_t ps = G.pslot[i];
    const int pg = DV_PG_PAGE(ps), par = DV_PG_PAR(ps);
    const SeqState *sq = B.st + par;
    const int fill = DV_PG_FRESH(ps) ? 0 : sq->pg_fill[pg];
    const int base = fill + before;
    int *const flips = B.pg_flips[pg] + (size_t)6 * base;
    // the host copy of the flips, when those of the whole launch fit
    const bool on_host = fill + all_flips <= B.host_flips;
    int *const hflips = B.pg_host[pg] + (size_t)6 * base;
    const int hroom = on_host || B.host_part ? max(B.host_flips - base, 0) : 0;   // of the frame's
    int nbk = 0, nar = 0, e2 = 0, excl = 0;
    if (ok) {
        const int D = B.maxdeg;
        // row n's staged flips to their places in the frame's list; records
        // are 24 bytes, copied as 8-byte words with the loads issued together
        auto place_row = [&](int n, int cb, int ca, int offb, int offa) {
            const int *stg = B.stage + (size_t)n * (2 * D) * 6;
            int *fb = flips + (size_t)6 * offb;
            int *fa = flips + (size_t)6 * offa;
            copy_words(reinterpret_cast<const int2 *>(stg), reinterpret_cast<int2 *>(fb), 3 * cb);
            copy_words(reinterpret_cast<const int2 *>(stg + 6 * D), reinterpret_cast<int2 *>(fa), 3 * ca);
            if (B.classify) {
                for (int j = 0; j < cb; ++j) fb[6 * j + 5] = event_flags(B, fb[6 * j], fb[6 * j + 1], -1);
                for (int j = 0; j < ca; ++j) fa[6 * j + 5] = event_flags(B, fa[6 * j], fa[6 * j + 1], 1);
            }
        };
        for (int g = blockIdx.x; g == 0 || g * PLACE_ROWS < KN; g += gridDim.x) {
            const int n = g * PLACE_ROWS + t, c0 = g * (PLACE_ROWS / G.chunk);
            const int cb = n < KN ? gmem(B.nb)[n] : 0, ca = n < KN ? gmem(B.na)[n] : 0;
            // breaking and arising before the block's rows, in the frame; row
            // lengths and dropped now points of the frame (at most 2 K_max D and
            // K_max: below 2^31)
            int v[6] = {0, 0, 0, 0, 0, 0};
            for (int c = t; c * G.chunk < KN; c += PLACE_ROWS) {
                const int4 d = B.dpart[c];
                v[0] += c < c0 ? d.x : 0;
                v[1] += c < c0 ? d.y : 0;
                v[2] += d.x;
                v[3] += d.y;
                v[4] += d.z;
                v[5] += d.w;
            }
            const int ib = wave_incl_sum(cb), ia = wave_incl_sum(ca);
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = wave_last(wave_incl_sum(v[k]));
            __syncthreads();
            if (lane == 63) {
#pragma unroll
                for (int k = 0; k < 6; ++k) red[k][wid] = v[k];
                red[6][wid] = ib;
                red[7][wid] = ia;
            }
            __syncthreads();
            auto total = [&](int k) { return red[k][0] + red[k][1] + red[k][2] + red[k][3]; };
            nbk = total(2);
            nar = total(3);
            e2 = total(4);
            excl = total(5);
            int offb = total(0) + ib - cb, offa = nbk + total(1) + ia - ca;
            for (int w = 0; w < wid; ++w) {
                offb += red[6][w];
                offa += red[7][w];
            }
            if (cb | ca) place_row(n, cb, ca, offb, offa);
            const int gb = total(6), ga = total(7);
            if (hroom > 0 && gb + ga > 0) {
                // the block's two runs of flips to the host, in whole words
                __syncthreads();
                const int b0 = total(0), a0 = nbk + total(1);
                const int nb = min(gb, hroom - b0), na = min(ga, hroom - a0);
                const auto src = gmem(reinterpret_cast<const unsigned long long *>(flips));
                const auto dst = gmem(reinterpret_cast<Word8 *>(hflips));
                for (int w = t; w < 3 * nb; w += PLACE_ROWS) dst[3 * b0 + w].v = src[3 * b0 + w];
                for (int w = t; w < 3 * na; w += PLACE_ROWS) dst[3 * a0 + w].v = src[3 * a0 + w];
            }
        }
    }
    if (blockIdx.x > 0) return;
    const PastOf PO = past_of(Dt, G, i, acc);   // (every lane)
    if (t != 0) return;
    const int KP = ok && PO.valid ? PO.K : 0;
    fs->K_past = KP;
    // the frame's result record (host memory, read after the launch)
    FrameOut r;
    r.frame = sq->frame + __popcll(acc & (below | (1ull << i)));
    r.status = ok ? 0 : 2;   // DV_ERR_CAPACITY: the frame is not a past
    r.K = KN;
    r.E = e2 / 2;
    r.n_flips = nbk + nar;
    r.n_break = nbk;
    r.excl_past = ok && PO.valid ? KP - (KN - excl) : 0;
    r.excl_now = excl;
    r.amb = fs->n_amb;
    r.trigger = (nbk + nar) > 0 ? 1 : 0;
    r.flip_off = base;
    r.on_host = on_host ? 1 : 0;
    r.sel = 1 - sq->sel;
    r.K_past = KP;
    B.pg_info[pg][DV_PG_POS(ps)] = r;
    if (B.out_info) {
        dv_frame_info fi;
        fi.frame = r.frame;
        fi.status = r.status;
        fi.n_components = r.K;
        fi.n_edges = r.status == 0 ? r.E : 0;
        fi.n_flips = r.n_flips;
        fi.n_breaking = r.n_break;
        fi.n_excluded_past = r.excl_past;
        fi.n_excluded_now = r.excl_now;
        fi.n_ambiguous_centroids = r.amb;
        fi.global_trigger = (uint32_t)r.trigger;
        *B.out_info = fi;
    }
    // commit, by the sequence's last accepted entry (or its last one, when none
    // was accepted): the next launch's header, with the spare past buffer as the
    // past when any frame was accepted
    const unsigned long long own = acc ? acc : seqm;
    if (63 - __clzll(own) == i) {
        SeqState o = *sq;
        // (by selects: an indexed local would live in memory)
        o.pg_fill[0] = pg == 0 ? fill + all_flips : o.pg_fill[0];
        o.pg_fill[1] = pg == 1 ? fill + all_flips : o.pg_fill[1];
        if (acc) {
            const int nxt = 1 - sq->sel;
            o.sel = nxt;
            o.K[0] = nxt == 0 ? KN : o.K[0];
            o.K[1] = nxt == 1 ? KN : o.K[1];
            o.past_valid = 1;
            o.frame = sq->frame + __popcll(acc);
        }
        B.st[1 - par] = o;
    }
}

// Phi of the most recent comparison with dropped past points as -1 (inspection).
__global__ __launch_bounds__(256) void k_phi_out(const Bufs *__restrict__ D, int slot, int *out) {
    const Bufs &B = D[slot];
    const int KP = B.fs->K_past;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < KP; p += gridDim.x * blockDim.x) {
        const int n = B.phi[p];
        out[p] = (n >= 0 && B.cnt[n] == 1) ? n : -1;
    }
}

// ---- inspection: sorted couple list (a < b) of the past buffer -------------
// 16 lanes per row, lane j holding slot j of the table, so that a row is one
// load; a row beyond its table is rare and taken by the whole wave.
__global__ __launch_bounds__(256) void k_edge_count(const Bufs *__restrict__ D, int par, int *cntv) {
    const Bufs B = D[0];
    const int sel = B.st[par].sel, K = B.st[par].K[sel];
    const CompBuf C = D[0].past[sel];
    const int prim = B.prim, maxdeg = B.maxdeg;
    const int lane = threadIdx.x & 63, j = lane & 15, gsh = lane & 48;
    for (int a0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4; a0 < K; a0 += gridDim.x * 16) {
        const int a = a0 + (lane >> 4);
        const int v = a < K && j < prim ? gmem(C.adj)[(size_t)a * prim + j] : DV_EMPTY;
        const bool full = prim < maxdeg && __popc((unsigned)(__ballot(v != DV_EMPTY) >> gsh) & 0xffffu) == prim;
        int c = __popc((unsigned)(__ballot(v != DV_EMPTY && v > a) >> gsh) & 0xffffu);
        for (unsigned long long w = __ballot(full && j == 0); w; w &= w - 1) {
            const int l = __builtin_ctzll(w), aw = __builtin_amdgcn_readlane(a, l);
            const int u = row_slot(C, prim, maxdeg, aw, lane);
            const int cw = __popcll(__ballot(u != DV_EMPTY && u > aw));
            if (lane == l) c = cw;
        }
        if (a < K && j == 0) cntv[a] = c;
    }
}

__global__ __launch_bounds__(1024) void k_edge_scan(const Bufs *__restrict__ D, int par, const int *cntv,
                                                    int *offv, int *total) {
    __shared__ int wsum[16];
    const SeqState *st = D[0].st + par;
    const int K = st->K[st->sel];
    const int tot = block_exclusive_scan(cntv, offv, K, wsum);
    if (threadIdx.x == 0) *total = tot;
}

// entries above a, written in increasing order (rows are unordered sets)
__global__ __launch_bounds__(256) void k_edge_write(const Bufs *__restrict__ D, int par, const int *offv,
                                                     int *ab) {
    const Bufs B = D[0];
    const int sel = B.st[par].sel, K = B.st[par].K[sel];
    const CompBuf C = D[0].past[sel];
    const int prim = B.prim, maxdeg = B.maxdeg;
    const int lane = threadIdx.x & 63, j = lane & 15, gsh = lane & 48;
    auto put = [&](int a, int at, int v) { st_int2(reinterpret_cast<int2 *>(ab), at, a, v); };
    for (int a0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4; a0 < K; a0 += gridDim.x * 16) {
        const int a = a0 + (lane >> 4);
        const int v = a < K && j < prim ? gmem(C.adj)[(size_t)a * prim + j] : DV_EMPTY;
        const bool full = prim < maxdeg && __popc((unsigned)(__ballot(v != DV_EMPTY) >> gsh) & 0xffffu) == prim;
        const int x = v > a && !full ? v : DV_EMPTY;
        const int rank = row16_below(x, x);
        if (x != DV_EMPTY) put(a, offv[a] + rank, x);
        for (unsigned long long w = __ballot(full && j == 0); w; w &= w - 1) {
            const int aw = __builtin_amdgcn_readlane(a, __builtin_ctzll(w));
            const int u = row_slot(C, prim, maxdeg, aw, lane);
            const bool in = u != DV_EMPTY && u > aw;
            const unsigned long long mk = __ballot(in);
            const int r = wave_below(u, mk, u);
            if (in) put(aw, offv[aw] + r, u);
        }
    }
}

}  // namespace

hipError_t launch_compare(const Batch &G, hipStream_t s, Prof &P) {
    const int grid = G.cbase[G.n];
    P.begin(ST_MATCH, s);
    // (Phi is made by blocks of k_rows)
    if (!G.past_known) {
        const int blocks = std::min((G.kmax + 255) / 256, REMATCH_BLOCKS);
        hipLaunchKernelGGL(k_rematch, dim3(G.n, blocks), dim3(256), 0, s, G.D, G);
    }
    P.end(ST_MATCH, s);
    P.begin(ST_DIFF, s);
    if (G.chunk == DV_CHUNK_MIN) hipLaunchKernelGGL(k_diff<DV_CHUNK_MIN>, dim3(grid), dim3(256), 0, s, G.D, G);
    else hipLaunchKernelGGL(k_diff<DV_CHUNK_MAX>, dim3(grid), dim3(256), 0, s, G.D, G);
    P.end(ST_DIFF, s);
    if (G.classify) {
        P.begin(ST_EVENTS, s);
        hipLaunchKernelGGL(k_events, dim3(grid), dim3(256), 0, s, G.D, G);
        P.end(ST_EVENTS, s);
    }
    P.begin(ST_PLACE, s);
    const int pblocks = std::min((G.kmax + PLACE_ROWS - 1) / PLACE_ROWS, 128);
    const Bufs *D = G.D;
    Batch arg = G;
    void *args[] = {&D, &arg};
    const hipError_t e =
        hipLaunchKernel(reinterpret_cast<const void *>(k_place), dim3(pblocks, 1, G.n), dim3(PLACE_ROWS), args, 0, s);
    P.end(ST_PLACE, s);
    return e;
}

void launch_phi_out(const Bufs &H, const Bufs *D, int slot, int32_t *d_out, hipStream_t s) {
    const int grid = (int)std::min<long long>((H.kmax + 255) / 256, 1024);
    hipLaunchKernelGGL(k_phi_out, dim3(grid), dim3(256), 0, s, D, slot, d_out);
}

void launch_edge_list(const Bufs &H, const Bufs *D, int par, int32_t *d_out_ab, int32_t *d_count,
                      int32_t *d_scratch, hipStream_t s) {
    const int kgrid = (int)std::min<long long>((H.kmax + 15) / 16, 1024);
    int *cntv = d_scratch, *offv = d_scratch + H.kmax;
    hipLaunchKernelGGL(k_edge_count, dim3(kgrid), dim3(256), 0, s, D, par, cntv);
    hipLaunchKernelGGL(k_edge_scan, dim3(1), dim3(1024), 0, s, D, par, (const int *)cntv, offv, d_count);
    hipLaunchKernelGGL(k_edge_write, dim3(kgrid), dim3(256), 0, s, D, par, (const int *)offv, d_out_ab);
}
