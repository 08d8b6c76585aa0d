// region.hpp -- the register-resident revisit kernel of the reconstruction, for
// AMD MI355X (gfx950).
//
// A region is R * NW rows x 256 columns of a tile, owned by one workgroup of NW
// waves while it works on it.  Each wave holds a strip of R rows in registers,
// 4 columns per lane: the marker and the mask as pairs of 16-bit lanes (the even
// and the odd columns), on which the packed 16-bit minimum and maximum work
// directly.  A wave sweeps its strip down and up: each row takes the maximum of
// itself, the row before it in the sweep and the neighbours of both along the
// row, under its mask -- about 11 instructions for the 256 pixels of a row,
// where a row closed along its whole length through prefix scans of clamp maps
// (kernels.hpp's sweep) takes about 180 and every row waits for the one before
// it.  A cheap sweep moves a value any distance along the sweep but one column
// (four inside a lane for 4-connectivity) along the row, so more of them are
// needed, on nuclei tiles about 30 pairs in all against 8; the work per pixel
// still falls several times, and so does the length of a visit.
//
// The strips of a region exchange their first and last rows through LDS after
// every pair of sweeps (a value read while its neighbour writes it is the older
// or the newer one, both valid lower bounds), and a wave sits the next pair
// out when neither its own strip nor the rows next to it changed in the last one.  After
// at most REGION_PAIRS pairs a visit stores its changed strips and checks its
// border, converged or not: regions that trade borders often follow a path
// across them together instead of one after the other (nuclei tile: the longest
// visits of all generations add up to 64 pairs instead of 189).  A region that
// is not converged yet goes on with a fresh halo; from the sixth such pass on,
// or from the second where a single strip is still changing (a flood that runs
// along a few rows), each starts with a full row closure of the rows of the strips
// that changed last, so that long horizontal runs (wide flat areas, corridors)
// move whole rows at a time.  (A flood along 3 x 300000 pixels, 4-connected, 4.8
// ms, 14.3 with five passes before every closure and 20.7 on the queue kernel; 200 x
// 60000 35.2, 43.6, 41.5.  In regions of 64 rows the sixth pass stays the line for
// images of more than STRIP_ROWS rows, whose floods seldom keep to a strip: the
// sooner closure cost the 512 x 512 tile 2 %.)
//
// A launch with at most a region per workgroup waits on chains of visits: there
// each workgroup keeps its region in registers after a visit and waits for the
// next request itself (wait_own).  With more regions than that a workgroup takes
// the next one from the ring, as the queue kernel does.
//
// What bounds it, on a 4096 x 4096 tile (512 regions): for the first ~110 us the
// sweeps' vector instructions (2.9 us per pair with all strips at work, 2.4 by
// count of instructions); after that the passes' fixed part, 5 us of loads,
// stores and atomics that complete at the memory side, in chains of up to 17
// passes.  Memory traffic is far from a limit.  Whole calls, against the queue
// kernel: 4096 x 4096 tile, 8-connected 1.40 -> 0.35 ms; 512 x 512 0.67 -> 0.14
// ms; 1531 x 2053, 4-connected, odd pitch 0.45 -> 0.13 ms; 24 uneven tasks in a
// batch 3.1 -> 1.2 ms.  (Without the waiting workgroups: 0.39, 0.16, 0.18 ms.)
// Small launches run on regions of 64 rows with strips of 8: 0.12 and 0.11 ms for
// the second and the third of these.
//
// Scheduling (block states, ring, tickets, counts of outstanding work) is that
// of kernels.hpp with regions as its blocks; wave 0 runs it for the workgroup.
#pragma once
#include "kernels.hpp"

// A value the compiler must not see through (wave-uniform, or one per lane), so
// that what derives from it is computed at its use instead of being kept in
// registers across a loop.  (The host emulation needs nothing of it.)
#ifndef RK_OPAQUE_S
#define RK_OPAQUE_S(v) asm volatile("" : "+s"(v))
#define RK_OPAQUE_V(v) asm volatile("" : "+v"(v))
#endif

namespace rk {

constexpr int REGION_PAIRS = 8;        // sweep pairs of a visit before its borders are traded
constexpr int REGION_CLOSURE_PASS = 5; // passes without convergence before rows are closed (see above for the single strip)
constexpr int STRIP_ROWS = 192;        // images of at most this many rows are strips (see the launch's choice of regions)

// LDS of a region's workgroup, in 32-bit words
template <int R, int NW>
struct RegionLds {
    static constexpr int RH = R * NW;
    static constexpr int EX = 0;                        // [NW][2][64] first and last row of each strip, packed
    static constexpr int FLAG = EX + NW * 2 * LANES;    // [2][NW] what the pair of that parity changed (below)
    static constexpr int CTL = FLAG + 2 * NW;           // control words (below)
    static constexpr int COL = CTL + 8;                 // bytes [2][RH]: the first and the last column
    static constexpr int WORDS = COL + 2 * RH / 4;
    RK_LDS uint32_t *w;
    __device__ __forceinline__ RK_LDS uint32_t *ex(int strip, int last) const { return w + EX + (2 * strip + last) * LANES; }
    __device__ __forceinline__ RK_LDS uint32_t *flag(int parity) const { return w + FLAG + parity * NW; }
    __device__ __forceinline__ RK_LDS uint8_t *col(int side) const { return (RK_LDS uint8_t *)(w + COL) + side * RH; }
};
// what a pair of sweeps changed in a strip: anything, its first row, its last row
enum { SC_ANY = 1, SC_FIRST = 2, SC_LAST = 4 };
// control words: the region to visit (or < 0: leave), whether it is its first
// visit, something stored, neighbours wanted, run again, give up, its strips are
// still in registers
enum { RC_REGION = 0, RC_FIRST = 1, RC_STORED = 2, RC_WANT = 3, RC_AGAIN = 4, RC_FAIL = 5, RC_KEPT = 6 };

template <int R, int NW>
__host__ __device__ constexpr size_t region_lds_bytes() { return (size_t)RegionLds<R, NW>::WORDS * 4; }

// ---- pixel pairs: word x holds columns 4l + {0,1,2,3}; even = columns 0 and 2, odd = 1 and 3
__device__ __forceinline__ uint32_t pmax(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pmin(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t evens(uint32_t v) { return v & 0x00ff00ffu; }
__device__ __forceinline__ uint32_t odds(uint32_t v) { return (v >> 8) & 0x00ff00ffu; }
__device__ __forceinline__ uint32_t joined(uint32_t e, uint32_t o) { return e | (o << 8); }

// maximum of every pixel of a row with its left and right neighbour (0 past the block)
__device__ __forceinline__ void row_max3(uint32_t e, uint32_t o, uint32_t &me, uint32_t &mo) {
    const uint32_t left = (o << 16) | (from_lower(o) >> 16);    // left neighbours of the even columns
    const uint32_t right = (from_upper(e) << 16) | (e >> 16);   // right neighbours of the odd ones
    const uint32_t m = pmax(e, o);
    me = pmax(m, left);
    mo = pmax(m, right);
}

template <int R>
struct Strip {
    uint32_t e[R], o[R];     // marker
    uint32_t ie[R], io[R];   // mask
};

// one row of a sweep: pe, po the row before it (swept already)
template <int CONN>
__device__ __forceinline__ void sweep_row(uint32_t &e, uint32_t &o, uint32_t ie, uint32_t io, uint32_t pe, uint32_t po) {
    uint32_t me, mo;
    if (CONN == 8) {
        row_max3(pmax(e, pe), pmax(o, po), me, mo);
        e = pmin(me, ie);
        o = pmin(mo, io);
    } else {
        row_max3(e, o, me, mo);
        e = pmin(pmax(me, pe), ie);
        o = pmin(pmax(mo, po), io);
        // (without diagonal steps a path turns along the row more often: two
        // more steps inside the lane's 4 columns, a third fewer pairs)
        o = pmax(o, pmin(e, io));
        e = pmax(e, pmin(o, ie));
    }
}

// One step of an inclusive scan of lane maps v -> max(a, min(v, b)) within 16-lane
// rows: this lane's map after the one of the lane CTRL selects (identity where
// there is none).
template <int CTRL>
__device__ __forceinline__ void lane_map_step(uint32_t &a, uint32_t &b) {
    const uint32_t pa = dpp_or<CTRL>(0u, a), pb = dpp_or<CTRL>(255u, b);
    a = max(a, min(pa, b));
    b = min(pb, b);
}

// Close a row along its whole length (every value carried as far as the mask
// lets it, from both ends): the 4 columns of a lane, a prefix scan of the lanes'
// maps, the 4 columns again with what enters the lane.  About 95 instructions,
// against 180 of row_closure, whose maps are per pixel and start from given values.
__device__ __forceinline__ void close_row(uint32_t &e, uint32_t &o, uint32_t ie, uint32_t io) {
    const int row = lane_id() >> 4;
    const uint32_t t = pmin(ie, io), bound = min(t & 0xffffu, t >> 16);   // what passes a lane
    {   // left to right
        o = pmax(o, pmin(e, io));
        e = pmax(e, pmin(o << 16, ie));
        o = pmax(o, pmin(e, io));
        uint32_t a = o >> 16, b = bound;
        lane_map_step<DPP_ROW_SHR + 1>(a, b);
        lane_map_step<DPP_ROW_SHR + 2>(a, b);
        lane_map_step<DPP_ROW_SHR + 4>(a, b);
        lane_map_step<DPP_ROW_SHR + 8>(a, b);
        const uint32_t e1 = (uint32_t)__builtin_amdgcn_readlane((int)a, 15);
        const uint32_t e2 = max((uint32_t)__builtin_amdgcn_readlane((int)a, 31),
                                min(e1, (uint32_t)__builtin_amdgcn_readlane((int)b, 31)));
        const uint32_t e3 = max((uint32_t)__builtin_amdgcn_readlane((int)a, 47),
                                min(e2, (uint32_t)__builtin_amdgcn_readlane((int)b, 47)));
        const uint32_t x = max(dpp_or<DPP_ROW_SHR + 1>(0u, a),
                               min(sel_row(row, 0u, e1, e2, e3), dpp_or<DPP_ROW_SHR + 1>(255u, b)));
        e = pmax(e, pmin(x, ie));
        o = pmax(o, pmin(e, io));
        e = pmax(e, pmin(o << 16, ie));
        o = pmax(o, pmin(e, io));
    }
    {   // right to left
        e = pmax(e, pmin(o, ie));
        o = pmax(o, pmin(e >> 16, io));
        e = pmax(e, pmin(o, ie));
        uint32_t a = e & 0xffffu, b = bound;
        lane_map_step<DPP_ROW_SHL + 1>(a, b);
        lane_map_step<DPP_ROW_SHL + 2>(a, b);
        lane_map_step<DPP_ROW_SHL + 4>(a, b);
        lane_map_step<DPP_ROW_SHL + 8>(a, b);
        const uint32_t e2 = (uint32_t)__builtin_amdgcn_readlane((int)a, 48);
        const uint32_t e1 = max((uint32_t)__builtin_amdgcn_readlane((int)a, 32),
                                min(e2, (uint32_t)__builtin_amdgcn_readlane((int)b, 32)));
        const uint32_t e0 = max((uint32_t)__builtin_amdgcn_readlane((int)a, 16),
                                min(e1, (uint32_t)__builtin_amdgcn_readlane((int)b, 16)));
        const uint32_t x = max(dpp_or<DPP_ROW_SHL + 1>(0u, a),
                               min(sel_row(row, e0, e1, e2, 0u), dpp_or<DPP_ROW_SHL + 1>(255u, b)));
        o = pmax(o, pmin(x << 16, io));
        e = pmax(e, pmin(o, ie));
        o = pmax(o, pmin(e >> 16, io));
        e = pmax(e, pmin(o, ie));
    }
}

template <int R, int CONN>
__device__ __forceinline__ void sweep_strip(Strip<R> &s, uint32_t above, uint32_t below) {
    uint32_t pe = evens(above), po = odds(above);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        sweep_row<CONN>(s.e[r], s.o[r], s.ie[r], s.io[r], pe, po);
        pe = s.e[r];
        po = s.o[r];
        __builtin_amdgcn_sched_barrier(0);   // (rows interleaved further ahead take registers the strip needs)
    }
    pe = evens(below);
    po = odds(below);
#pragma unroll
    for (int r = R - 1; r >= 0; --r) {
        sweep_row<CONN>(s.e[r], s.o[r], s.ie[r], s.io[r], pe, po);
        pe = s.e[r];
        po = s.o[r];
        __builtin_amdgcn_sched_barrier(0);   // (rows interleaved further ahead take registers the strip needs)
    }
}

// Sum of a lane's marker values.  Sweeps only raise, so an unchanged sum is an
// unchanged strip (each 16-bit half adds at most 2 * 64 * 255 and never carries).
template <int R>
__device__ __forceinline__ uint32_t strip_sum(const Strip<R> &s) {
    static_assert(R <= 64, "16-bit halves");
    uint32_t t = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) t += s.e[r] + s.o[r];
    return t;
}

// The halo of a strip: lane k (0..R+1) the marker (clipped) and mask of the pixel
// left of row k - 1, lane 32 + k of the one right of it; `north` / `south` the
// packed rows above and below the region (first and last strip).
struct RegionHalo {
    uint32_t cj, ci;
    uint32_t nj, ni, sj, si;
};

template <int R, int NW>
__device__ __forceinline__ void region_halo(const TaskDev &t, const BlockGeom &g, int wv, RegionHalo &h) {
    static_assert(R + 2 <= 32, "one lane per halo row and side");
    constexpr int RH = R * NW;
    int ln = lane_id();
    RK_OPAQUE_V(ln);   // (the halo's addresses are not kept across the region's passes)
    const int valid = min(4, g.bw - 4 * ln);
    h.cj = h.ci = h.nj = h.ni = h.sj = h.si = 0u;
    const int k = ln & 31, y = wv * R + k - 1;   // row of the region
    const bool east = ln >= 32;
    const bool row_in = k < R + 2 && ((y >= 0 && y < g.bh) || (y == -1 && g.has_n) || (y == RH && g.has_s));
    if (row_in && (east ? g.has_e : g.has_w)) {
        const int gx = east ? g.x0 + BW : g.x0 - 1;
        h.ci = mask1(t, g.y0 + y, gx);
        h.cj = cload8(t.j + (int64_t)(g.y0 + y) * t.pitch_j + gx);
    }
    if (wv == 0 && g.has_n && valid > 0) {
        h.ni = mask4(t, g.y0 - 1, g.x0 + 4 * ln, valid);
        h.nj = cload4(t.j + (int64_t)(g.y0 - 1) * t.pitch_j, g.x0 + 4 * ln, valid, t.aligned);
    }
    if (wv == NW - 1 && g.has_s && valid > 0) {
        h.si = mask4(t, g.y0 + RH, g.x0 + 4 * ln, valid);
        h.sj = cload4(t.j + (int64_t)(g.y0 + RH) * t.pitch_j, g.x0 + 4 * ln, valid, t.aligned);
    }
    h.cj = min(h.cj, h.ci);
    h.nj = bmin4(h.nj, h.ni);
    h.sj = bmin4(h.sj, h.si);
}

// Raise the strip's border pixels from the halo.  (The halo does not change
// while a pass sweeps, so this once per pass is all it takes.)  `seen`: the
// column halo of the pass before, whose values the strip has already.
template <int R>
__device__ __forceinline__ void seed_from_halo(Strip<R> &s, const RegionHalo &h, uint32_t &seen, int conn) {
    const int ln = lane_id();
    if (__ballot(h.cj != seen)) {
        seen = h.cj;
        const uint32_t near = max(from_lower(h.cj), from_upper(h.cj));
        const uint32_t c = conn == 8 ? max(h.cj, near) : h.cj;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t west = (uint32_t)__builtin_amdgcn_readlane((int)c, r + 1);
            const uint32_t east = (uint32_t)__builtin_amdgcn_readlane((int)c, r + 33);
            s.e[r] = pmax(s.e[r], pmin(s.ie[r], ln == 0 ? west : 0u));
            s.o[r] = pmax(s.o[r], pmin(s.io[r], ln == LANES - 1 ? east << 16 : 0u));
        }
    }
    uint32_t ne = evens(h.nj), no = odds(h.nj), se = evens(h.sj), so = odds(h.sj);
    if (conn == 8) {
        row_max3(ne, no, ne, no);
        row_max3(se, so, se, so);
    }
    s.e[0] = pmax(s.e[0], pmin(s.ie[0], ne));
    s.o[0] = pmax(s.o[0], pmin(s.io[0], no));
    s.e[R - 1] = pmax(s.e[R - 1], pmin(s.ie[R - 1], se));
    s.o[R - 1] = pmax(s.o[R - 1], pmin(s.io[R - 1], so));
}

// accesses at a wave-uniform address plus a lane's offset (the offset opaque: its
// widening stays beside the access, which then takes it as a 32-bit offset)
__device__ __forceinline__ uint32_t ld32(const uint8_t *p, uint32_t off) {
    RK_OPAQUE_V(off);
    return *(const RK_GLOBAL uint32_t *)(gp(p) + off);
}
__device__ __forceinline__ uint32_t ld8(const uint8_t *p, uint32_t off) {
    RK_OPAQUE_V(off);
    return gp(p)[off];
}
__device__ __forceinline__ uint32_t cld32(const uint8_t *p, uint32_t off) {
    RK_OPAQUE_V(off);
    return cload32(p + off);
}
__device__ __forceinline__ uint32_t cld8(const uint8_t *p, uint32_t off) {
    RK_OPAQUE_V(off);
    return cload8(p + off);
}
__device__ __forceinline__ void cst32(uint8_t *p, uint32_t off, uint32_t v) {
    RK_OPAQUE_V(off);
    cstore32(p + off, v);
}
__device__ __forceinline__ void cst8(uint8_t *p, uint32_t off, uint32_t v) {
    RK_OPAQUE_V(off);
    cstore8(p + off, v);
}

// Load the strip's rows (0 outside the image).  Row addresses are wave-uniform
// (scalar), the lane adds its columns; rows past the image re-read the strip's
// last row and are zeroed, so that every load is issued without a branch per row.
// A lane with all its 4 columns in a dword-aligned image loads dwords, any other
// bytes, column by column.
template <int R>
__device__ __forceinline__ void load_strip(const TaskDev &t, const BlockGeom &g, int y0, int rows, Strip<R> &s) {
    const uint32_t x = 4u * (uint32_t)lane_id();
    const int valid = min(4, g.bw - (int)x);
    uint32_t iv[R], jv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) iv[r] = jv[r] = 0u;
    if (rows > 0) {
        const uint8_t *i0 = t.i + (int64_t)y0 * t.pitch_i + g.x0, *j0 = t.j + (int64_t)y0 * t.pitch_j + g.x0;
        const bool dwords = t.aligned && valid == 4;
        if (dwords) {
            const uint8_t *pi = i0, *pj = j0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                iv[r] = ld32(pi, x);
                jv[r] = cld32(pj, x);
                pi += r + 1 < rows ? t.pitch_i : 0;
                pj += r + 1 < rows ? t.pitch_j : 0;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (valid > k) {
                    const uint8_t *pi = i0 + k, *pj = j0 + k;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        iv[r] |= ld8(pi, x) << (8 * k);
                        jv[r] |= cld8(pj, x) << (8 * k);
                        pi += r + 1 < rows ? t.pitch_i : 0;
                        pj += r + 1 < rows ? t.pitch_j : 0;
                    }
                }
        }
    }
    const uint32_t keep = valid >= 4 ? 0xffffffffu : (valid <= 0 ? 0u : ((1u << (8 * valid)) - 1u));
    const uint32_t flip = t.minv ? keep : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t m = r < rows ? iv[r] ^ flip : 0u;
        s.ie[r] = evens(m);
        s.io[r] = odds(m);
        s.e[r] = pmin(evens(jv[r]), s.ie[r]);
        s.o[r] = pmin(odds(jv[r]), s.io[r]);
    }
}

template <int R>
__device__ __forceinline__ void store_strip(const TaskDev &t, const BlockGeom &g, int y0, int rows, const Strip<R> &s) {
    const uint32_t x = 4u * (uint32_t)lane_id();
    const int valid = min(4, g.bw - (int)x);
    y0 = uniform(y0);
    rows = uniform(rows);
    RK_OPAQUE_S(y0);   // (neither the row addresses nor the rows' tests are kept across the region's passes)
    RK_OPAQUE_S(rows);
    uint8_t *j0 = t.j + (int64_t)y0 * t.pitch_j + g.x0;
    if (t.aligned && valid == 4) {
        uint8_t *p = j0;
#pragma unroll
        for (int r = 0; r < R; ++r, p += t.pitch_j)
            if (r < rows) cst32(p, x, joined(s.e[r], s.o[r]));
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (valid > k) {
                uint8_t *p = j0 + k;
#pragma unroll
                for (int r = 0; r < R; ++r, p += t.pitch_j)
                    if (r < rows) cst8(p, x, (k & 1 ? s.o[r] : s.e[r]) >> (k & 2 ? 16 : 0));
            }
    }
}

// The strips changed according to the flags of one parity; *run: whether strip wv
// has to sweep (its own change, or one of the row next to it).
template <int R, int NW>
__device__ __forceinline__ uint32_t changed_strips(const RegionLds<R, NW> &L, int parity, int wv, bool *run) {
    const int ln = lane_id();
    const uint32_t f = ln < NW ? L.flag(parity)[ln] : 0u;
    const uint32_t any = (uint32_t)__ballot((f & SC_ANY) != 0u);
    const uint32_t next = (any >> wv) | ((uint32_t)__ballot((f & SC_LAST) != 0u) << 1 >> wv) |
                          ((uint32_t)__ballot((f & SC_FIRST) != 0u) >> 1 >> wv);
    *run = (next & 1u) != 0u;
    return any;
}

// Sweep pairs until no strip of the region changes, at most REGION_PAIRS, from
// the flags of parity 1 (set before the barrier that precedes the call).  Returns
// the strips changed in the last pair (0: the region is converged).  All waves
// of the workgroup.
template <int R, int NW, int CONN>
__device__ __forceinline__ uint32_t sweep_region(const RegionLds<R, NW> &L, int wv, Strip<R> &s, uint32_t &sum,
                                                 uint32_t *own, uint32_t &requested) {
    const int ln = lane_id();
    bool run;
    uint32_t active = changed_strips<R, NW>(L, 1, wv, &run);
    for (int it = 0; it < REGION_PAIRS && active; ++it) {
        // (a region still changing at the end reads its halo anew, which answers the requests up to here)
        if (it == REGION_PAIRS - 2 && wv == 0 && ln == 0)
            requested = __hip_atomic_fetch_and(own, ~ST_D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t changed = 0;
        if (run) {
            const uint32_t above = wv > 0 ? ((volatile RK_LDS uint32_t *)L.ex(wv - 1, 1))[ln] : 0u;
            const uint32_t below = wv < NW - 1 ? ((volatile RK_LDS uint32_t *)L.ex(wv + 1, 0))[ln] : 0u;
            const uint32_t fe = s.e[0], fo = s.o[0], le = s.e[R - 1], lo = s.o[R - 1];
            sweep_strip<R, CONN>(s, above, below);
            const uint32_t now = strip_sum(s);
            if (__ballot(now != sum)) {
                changed = SC_ANY;
                if (__ballot((s.e[0] ^ fe) | (s.o[0] ^ fo))) {
                    ((volatile RK_LDS uint32_t *)L.ex(wv, 0))[ln] = joined(s.e[0], s.o[0]);
                    changed |= SC_FIRST;
                }
                if (__ballot((s.e[R - 1] ^ le) | (s.o[R - 1] ^ lo))) {
                    ((volatile RK_LDS uint32_t *)L.ex(wv, 1))[ln] = joined(s.e[R - 1], s.o[R - 1]);
                    changed |= SC_LAST;
                }
            }
            sum = now;
        }
        if (ln == 0) L.flag(it & 1)[wv] = changed;
        if (it == REGION_PAIRS - 1 && wv == 0) vm_sync();   // (the request bit is taken before any halo is read)
        __syncthreads();
        active = changed_strips<R, NW>(L, it & 1, wv, &run);
    }
    return active;
}

// Neighbouring regions (bits as request_neighbours takes them) that this
// strip's border pixels can still raise, judged against the halo.
template <int R, int NW>
__device__ __forceinline__ uint32_t wanted_neighbours(const RegionLds<R, NW> &L, const BlockGeom &g, int wv,
                                                      const Strip<R> &s, const RegionHalo &h, int conn) {
    constexpr int RH = R * NW;
    int ln = lane_id();
    RK_OPAQUE_V(ln);
    uint32_t want = 0;
    {   // west and east columns, and the corner regions
        const int k = ln & 31, side = ln >> 5, y = wv * R + k - 1;
        const RK_LDS uint8_t *c = L.col(side);
        const bool here = k >= 1 && k <= R && y < g.bh;
        bool viol = false, corner = false;
        if (here) {
            uint32_t out = c[y];
            if (conn == 8) {
                if (y > 0) out = max(out, (uint32_t)c[y - 1]);
                if (y + 1 < g.bh) out = max(out, (uint32_t)c[y + 1]);
            }
            viol = h.cj < min(out, h.ci);
        } else if (conn == 8 && ((k == 0 && y == -1) || (k == R + 1 && y == RH && g.bh == RH))) {
            corner = h.cj < min((uint32_t)c[y < 0 ? 0 : RH - 1], h.ci);
        }
        const unsigned long long v = __ballot(viol), d = __ballot(corner);
        if (v & 0xffffffffull) want |= 4u;
        if (v >> 32) want |= 8u;
        if (wv == 0) want |= ((uint32_t)(d & 1ull) << 4) | ((uint32_t)((d >> 32) & 1ull) << 5);
        if (wv == NW - 1)
            want |= ((uint32_t)((d >> (R + 1)) & 1ull) << 6) | ((uint32_t)((d >> (R + 33)) & 1ull) << 7);
    }
    if (wv == 0) {
        uint32_t e = s.e[0], o = s.o[0];
        if (conn == 8) row_max3(e, o, e, o);
        if (__ballot(pmax(pmin(e, evens(h.ni)), evens(h.nj)) != evens(h.nj)) ||
            __ballot(pmax(pmin(o, odds(h.ni)), odds(h.nj)) != odds(h.nj)))
            want |= 1u;
    }
    if (wv == NW - 1) {
        uint32_t e = s.e[R - 1], o = s.o[R - 1];
        if (conn == 8) row_max3(e, o, e, o);
        if (__ballot(pmax(pmin(e, evens(h.si)), evens(h.sj)) != evens(h.sj)) ||
            __ballot(pmax(pmin(o, odds(h.si)), odds(h.sj)) != odds(h.sj)))
            want |= 2u;
    }
    return want;
}

// One pass over the loaded region and its halo: seeds, sweeps, changed strips
// stored, border pixels left in LDS.  `carry`: this strip changed in the last
// pair of the pass before (or the region is new); `loaded`: the strip's sum when
// it was last stored or loaded.  Returns the strips still changing; if any, the
// halo is read anew while the stores complete, for the next pass; else (wave 0,
// lane 0) `requested` receives the region's state, its request bit taken.
template <int R, int NW>
__device__ __forceinline__ uint32_t region_pass(const RegionLds<R, NW> &L, const TaskDev &t, const BlockGeom &g, int wv,
                                                int y0, int rows, Strip<R> &s, RegionHalo &h, uint32_t &seen, bool first,
                                                uint32_t carry, uint32_t loaded, uint32_t *own,
                                                uint32_t &requested) {
    const int ln = lane_id();
    seed_from_halo<R>(s, h, seen, t.conn);
    uint32_t sum = strip_sum(s);
    ((volatile RK_LDS uint32_t *)L.ex(wv, 0))[ln] = joined(s.e[0], s.o[0]);
    ((volatile RK_LDS uint32_t *)L.ex(wv, 1))[ln] = joined(s.e[R - 1], s.o[R - 1]);
    const bool moved = __ballot(sum != loaded) != 0ull;
    if (ln == 0) L.flag(1)[wv] = (carry || moved) ? (uint32_t)(SC_ANY | SC_FIRST | SC_LAST) : 0u;
    __syncthreads();
    const uint32_t active = t.conn == 8 ? sweep_region<R, NW, 8>(L, wv, s, sum, own, requested)
                                        : sweep_region<R, NW, 4>(L, wv, s, sum, own, requested);
    const bool dirty = first || __ballot(sum != loaded) != 0ull;
    if (dirty && rows > 0) {
        store_strip<R>(t, g, y0, rows, s);
        if (ln == 0) __hip_atomic_fetch_or(L.w + L.CTL + RC_STORED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (active)
        region_halo<R, NW>(t, g, wv, h);
    else if (wv == 0 && ln == 0)   // take a request that came meanwhile (answered with the stores)
        requested |= __hip_atomic_fetch_and(own, ~ST_D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ln == 0 || ln == LANES - 1) {
        RK_LDS uint8_t *c = L.col(ln == 0 ? 0 : 1) + wv * R;
        // (a region with an eastern neighbour is 256 columns wide)
#pragma unroll
        for (int r = 0; r < R; ++r) c[r] = (uint8_t)(ln == 0 ? s.e[r] : s.o[r] >> 16);
    }
    vm_sync();   // the stores are complete before any request
    __syncthreads();
    return active;
}

// ---- scheduling of regions

// A region whose workgroup waits for its next request itself (state bit L, in
// place of R): a request then only sets D and counts, no ring slot.
constexpr uint32_t ST_L = 16u;
constexpr uint32_t ST_X = 32u;   // all work is done: set in every state word of a launch that has waiting workgroups
// How long it waits (wall-clock ticks of 10 ns) before it gives the region up and
// takes a ticket like any other.  Bounded, so that regions still in the ring
// are never left to workgroups that have not started (the GPU may be shared).
constexpr uint64_t REGION_LINGER = 10000;

// Wait for a request of the region `own`, left in state V | L.  Returns own
// (claimed), -1 when all work is done, or -3 when it was given up.  (wave 0)
__device__ __forceinline__ int wait_own(const KArgs &a, int own) {
    int res = 0;
    if (lane_id() == 0) {
        uint32_t *word = state_word(a, (uint32_t)own);
        const uint64_t t0 = wall_clock64();
        res = -3;
        while (true) {
            uint32_t s = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (s & ST_D) {
                if (__hip_atomic_compare_exchange_strong(word, &s, ST_V | ST_R, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)) {
                    res = own;
                    break;
                }
                continue;
            }
            if (s & ST_X) {
                res = -1;
                break;
            }
            if (wall_clock64() - t0 > REGION_LINGER &&
                __hip_atomic_compare_exchange_strong(word, &s, ST_V, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                break;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return uniform(res);
}

// Neighbour k (N, S, W, E, NW, NE, SW, SE) of a region, as an offset of its id.
__device__ __forceinline__ int region_step(int k, int nbx) {
    return k == 0 ? -nbx : k == 1 ? nbx : k == 2 ? -1 : k == 3 ? 1 : k == 4 ? -nbx - 1 : k == 5 ? -nbx + 1
         : k == 6 ? nbx - 1 : nbx + 1;
}

// Requests sent and not yet accounted for: lane k (< 8) the neighbour's state
// before its request (all bits set: none sent).
constexpr uint32_t REQ_NONE = 0xffffffffu;

// Counts of outstanding work are taken ahead of the requests they are for: a
// visit holds REGION_CREDIT counts besides its own, topped up after each pass
// (so that the additions are complete, past the next pass's wait for its stores,
// before any request uses them) and given back at its end.  A workgroup that
// takes a request up at once may therefore finish and count down before the
// request is accounted for.
constexpr uint32_t REGION_CREDIT = 16;   // twice the most requests of one pass: those of the pass before may not be
                                         // accounted for yet

__device__ __forceinline__ void take_credit(const KArgs &a, int ti, uint32_t &credit) {
    if (lane_id() == 0 && credit < REGION_CREDIT) {
        __hip_atomic_fetch_add(a.tile_pending + ti, REGION_CREDIT - credit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&a.work->pending, REGION_CREDIT - credit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    credit = REGION_CREDIT;
}

// Account for answered requests (wave 0): those that made an idle region pending
// use up credit, and are written to the ring unless its workgroup waits for
// them.  False: gave up waiting for a ring slot.
__device__ __forceinline__ bool account_requests(const KArgs &a, uint32_t ring_cap, uint32_t gb, int nbx, uint32_t &old,
                                                 uint32_t &credit, WaveStats &st) {
    const int ln = lane_id();
    const uint32_t nb = (uint32_t)((int)gb + region_step(ln & 7, nbx));
    const bool counted = ln < 8 && old != REQ_NONE && !(old & (ST_R | ST_D));
    const bool queue = counted && !(old & ST_L);
    old = REQ_NONE;
    const unsigned long long cm = __ballot(counted), qm = __ballot(queue);
    if (!cm) return true;
    const uint32_t nc = (uint32_t)__popcll(cm), nq = (uint32_t)__popcll(qm);
    credit -= nc;
    if (ln == 0) st.request += nc;
    if (!nq) return true;
    uint32_t base = 0;
    if (ln == 0) base = __hip_atomic_fetch_add(&a.work->ring_tail, nq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    base = uniform(base);
    uint32_t *slot = a.ring + (size_t)((base + prefix_count(qm)) % ring_cap) * RING_STRIDE;
    const uint64_t t0 = wall_clock64();   // a slot is free unless its previous occupant has not been taken out yet
    while (true) {
        const bool busy = queue && __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        if (!__ballot(busy)) break;
        if (expired(a, t0)) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    if (queue) __hip_atomic_store(slot, nb + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Requests of the neighbours in `want`, one lane each; nothing waits for the answers.
__device__ __forceinline__ void send_requests(const KArgs &a, uint32_t gb, int nbx, uint32_t want, uint32_t &old) {
    const int ln = lane_id();
    if (ln < 8 && ((want >> ln) & 1u))
        old = __hip_atomic_fetch_or(state_word(a, (uint32_t)((int)gb + region_step(ln, nbx))), ST_D, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
}

// The end of a converged region's pass (wave 0): its requests and its release,
// all atomics in flight together (lane 8: the region's own state word, `held`
// if nobody requested it meanwhile; then it is not released but run again).
// `keep` as in request_neighbours (null: never).  *again: run again.  Returns
// false if the launch has to give up.
__device__ __forceinline__ bool release_region(const KArgs &a, uint32_t ring_cap, uint32_t gb, int nbx, uint32_t want,
                                               bool linger, uint32_t held, int *keep, int *again, uint32_t &credit,
                                               WaveStats &st) {
    const int ln = lane_id();
    const bool mine = ln < 8 && ((want >> ln) & 1u);
    const int cand = (keep != nullptr && *keep < 0 && want != 0u) ? (int)__builtin_ctz(want) : -1;
    uint32_t *own = state_word(a, gb), *nb = state_word(a, (uint32_t)((int)gb + region_step(ln & 7, nbx)));
    const uint32_t idle = linger ? (ST_V | ST_L) : ST_V;
    uint32_t old = REQ_NONE, seen = held;
    bool kept = false, released = false;
    if (mine && ln != cand) old = __hip_atomic_fetch_or(nb, ST_D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ln == 8)
        released = __hip_atomic_compare_exchange_strong(own, &seen, idle, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
    if (mine && ln == cand) {
        uint32_t expected = ST_V;   // idle: visited, not owned, not requested
        kept = __hip_atomic_compare_exchange_strong(nb, &expected, ST_V | ST_R, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        if (!kept) old = __hip_atomic_fetch_or(nb, ST_D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool stuck = false;
    if (ln == 8 && !released) {   // requested meanwhile: keep the region, take the request
        stuck = true;
        for (int q = 0; q < CAS_TRIES && stuck; ++q) {
            const bool more = (seen & ST_D) != 0u;
            stuck = !__hip_atomic_compare_exchange_strong(own, &seen, more ? (ST_V | ST_R) : idle, __ATOMIC_RELAXED,
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!stuck) released = !more;
        }
    }
    *again = __ballot(ln == 8 && !released) ? 1 : 0;
    if (__ballot(kept)) {
        *keep = (int)gb + region_step(cand, nbx);
        if (ln == 0) st.request += 1;
    }
    return account_requests(a, ring_cap, gb, nbx, old, credit, st) && __ballot(stuck) == 0ull;
}

template <typename T>
__device__ __forceinline__ T *uniform_ptr(T *p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    return (T *)(uintptr_t)(((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v));
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    return (int64_t)(((uint64_t)uniform((uint32_t)((uint64_t)v >> 32)) << 32) | uniform((uint32_t)v));
}

// The fields of task k that a region's visit uses, in scalar registers.
__device__ __forceinline__ TaskDev region_task(const TaskTable &tt, int k) {
    const TaskDev q = task_of(tt, k);
    TaskDev t{};
    t.j = uniform_ptr(q.j);
    t.i = uniform_ptr(q.i);
    t.pitch_j = uniform64(q.pitch_j);
    t.pitch_i = uniform64(q.pitch_i);
    t.h = uniform(q.h);
    t.w = uniform(q.w);
    t.conn = uniform(q.conn);
    t.minv = uniform(q.minv);
    t.nby = uniform(q.nby);
    t.nbx = uniform(q.nbx);
    t.block0 = uniform(q.block0);
    t.aligned = uniform(q.aligned);
    t.stat_rows = uniform(q.stat_rows);
    return t;
}

template <int R, int NW>
__global__ __launch_bounds__(64 * NW, 4) void region_drain(TaskTable tt, KArgs a) {
    constexpr int RH = R * NW;
    RegionLds<R, NW> L;
    L.w = (RK_LDS uint32_t *)dyn_lds();
    volatile RK_LDS uint32_t *ctl = L.w + L.CTL;
    const int ln = lane_id();
    const int wv = uniform((int)(threadIdx.x >> 6));
    Work *w = a.work;
    const uint32_t ring_cap = ring_cap_of(tt);
    WaveStats st;
    // (the line lies where every region has a workgroup; with more of them a
    // waiting workgroup would hold up the regions in the ring)
    const bool linger = total_blocks_of(tt) <= gridDim.x;
    int keep = -1;        // (wave 0) region this workgroup requested and keeps for its next visit
    uint32_t credit = 0;  // (wave 0) counts of outstanding work held for requests
    int held = -1;        // region whose strips are in registers
    int cur_ti = -1;      // task of the last visit (most visits stay in one task) and its regions
    uint32_t t_first = 0, t_end = 0;
    Strip<R> s;
    uint32_t seen = 0u;   // column halo the strip has been seeded with
    for (bool start = true;; start = false) {
        if (wv == 0) {   // the next region, claimed (revisit_drain's protocol)
            int gsel = keep, first = 0, lost = 0;
            bool claimed = keep >= 0;
            keep = -1;
            if (start) {   // nothing was requested at all: no visit will ever complete
                uint32_t pend = 0;
                if (ln == 0) pend = __hip_atomic_load(&w->pending, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                if (uniform(pend) == 0u) gsel = -2;
            } else if (linger) {
                gsel = wait_own(a, held);
                claimed = gsel >= 0;
                if (gsel == -1) gsel = -2;
                if (gsel == -3) gsel = -1;
            }
            if (gsel == -1) {
                uint32_t ticket = 0;
                if (ln == 0)
                    ticket = __hip_atomic_fetch_add(&w->ring_head, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
                gsel = wait_ticket(a, ring_cap, uniform(ticket));
            }
            if (gsel >= 0 && !claimed) {
                if (ln == 0) {
                    uint32_t q = __hip_atomic_load(state_word(a, (uint32_t)gsel), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const uint32_t skew = a.test_fault == 1 ? 0x80000000u : 0u;   // (test hook, as in revisit_drain)
                    lost = 1;
                    for (int k = 0; k < CAS_TRIES; ++k) {
                        uint32_t e = q ^ skew;
                        if (__hip_atomic_compare_exchange_strong(state_word(a, (uint32_t)gsel), &e, (q & ~ST_D) | ST_R,
                                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT)) {
                            lost = 0;
                            break;
                        }
                        q = e;
                    }
                    first = (q & ST_V) ? 0 : 1;
                    if (lost) __hip_atomic_store(&w->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (uniform(lost)) gsel = -2;   // never work on a region this workgroup does not own
            }
            if (ln == 0) {
                ctl[RC_REGION] = (uint32_t)gsel;
                ctl[RC_FIRST] = (uint32_t)first;
                ctl[RC_KEPT] = claimed && linger ? 1u : 0u;
                ctl[RC_STORED] = 0u;
                ctl[RC_WANT] = 0u;
                ctl[RC_FAIL] = 0u;
            }
        }
        __syncthreads();
        const int gsel = uniform((int)ctl[RC_REGION]);
        const bool first = uniform(ctl[RC_FIRST]) != 0u, in_registers = uniform(ctl[RC_KEPT]) != 0u;
        if (gsel < 0) break;
        const uint32_t gb = (uint32_t)gsel;
        held = gsel;
        if (cur_ti < 0 || gb < t_first || gb >= t_end) cur_ti = uniform(find_task(tt, gb));
        const TaskDev t = region_task(tt, cur_ti);
        t_first = t.block0;
        t_end = t.block0 + (uint32_t)(t.nby * t.nbx);
        const int lb = (int)(gb - t.block0);
        const int by = uniform(lb / t.nbx), bx = lb - by * t.nbx;
        const BlockGeom g = geom<RH>(t, by, bx);
        const int y0 = g.y0 + wv * R, rows = max(0, min(R, g.bh - wv * R));
        if (wv == 0) take_credit(a, cur_ti, credit);   // (a kept region's task is the one before's)
        if (wv == 0 && ln == 0) {   // statistics count the caller's work blocks
            if (first) st.dense += (unsigned)((g.bh + t.stat_rows - 1) / t.stat_rows);
            else st.revisit += 1;
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);

        RegionHalo h;
        region_halo<R, NW>(t, g, wv, h);
        if (!in_registers) {
            load_strip<R>(t, g, y0, rows, s);
            seen = 0u;
        }
        bool fail = false;
        int stuck_passes = 0;
        const bool soon = R >= 16 || t.h <= STRIP_ROWS;   // a single strip's change closes its rows in the next pass
        uint32_t carry = first ? 1u : 0u, held_state = first ? ST_R : (ST_V | ST_R), sent = REQ_NONE;
        uint32_t *own = state_word(a, gb);
        for (int pass = 0;; ++pass) {
            const uint32_t loaded = strip_sum(s);
            if (carry && stuck_passes >= REGION_CLOSURE_PASS) {   // (a strip at rest has nothing to close)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r < rows) {
                        uint32_t ie = s.ie[r];
                        RK_OPAQUE_V(ie);   // (what derives from the mask is not kept across the region's passes)
                        close_row(s.e[r], s.o[r], ie, s.io[r]);
                    }
                    __builtin_amdgcn_sched_barrier(0);   // one row at a time: its temporaries would spill
                }
            }
            const bool dense = first && pass == 0;
            uint32_t want = 0, requested = 0;
            const uint32_t active =
                region_pass<R, NW>(L, t, g, wv, y0, rows, s, h, seen, dense, carry, loaded, own, requested);
            carry = (active >> wv) & 1u;
            stuck_passes = !active ? 0 : stuck_passes + (soon && (active & (active - 1u)) == 0u ? REGION_CLOSURE_PASS : 1);
            if (ctl[RC_STORED]) {
                want = wanted_neighbours<R, NW>(L, g, wv, s, h, t.conn);
                if (want && ln == 0)
                    __hip_atomic_fetch_or(L.w + L.CTL + RC_WANT, want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
            if (wv == 0) {
                int again = 1;
                want = uniform(ctl[RC_WANT]);
                bool ok = account_requests(a, ring_cap, gb, t.nbx, sent, credit, st);
                if (active || uniform(requested & ST_D)) {   // go on: the answers are looked at after the next pass
                    send_requests(a, gb, t.nbx, want, sent);
                } else {
                    ok &= release_region(a, ring_cap, gb, t.nbx, want, linger, held_state, linger ? nullptr : &keep,
                                         &again, credit, st);
                    held_state = ST_V | ST_R;
                }
                if (again) take_credit(a, cur_ti, credit);
                if (ln == 0) {
                    if (again) st.rerun += 1;
                    ctl[RC_AGAIN] = (uint32_t)again;
                    if (!ok) ctl[RC_FAIL] = 1u;
                    ctl[RC_STORED] = 0u;
                    ctl[RC_WANT] = 0u;
                }
            }
            if (active) continue;   // (a failure is seen at the end of the next pass; the control words are
                                    // written again only past that pass's first barrier)
            __syncthreads();
            fail = uniform(ctl[RC_FAIL]) != 0u;
            if (!uniform(ctl[RC_AGAIN]) || fail) break;
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            region_halo<R, NW>(t, g, wv, h);   // (while a region keeps changing it is read with the stores)
        }
        // ---- the visit is complete (counts as in revisit_drain)
        if (wv == 0) {
            int last = 0;
            if (ln == 0) {
                if (((st.revisit + st.dense) & 7u) == 0u || first)
                    __hip_atomic_fetch_add(&w->progress, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (fail) __hip_atomic_store(&w->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (keep < 0) {
                    const uint32_t left = __hip_atomic_fetch_sub(a.tile_pending + cur_ti, 1u + credit, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT) - credit;
                    const uint32_t all = __hip_atomic_fetch_sub(&w->pending, 1u + credit, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT) - credit;
                    if (left == 1u) {
                        __hip_atomic_store(a.tile_done + cur_ti, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (a.host_done)   // every visit waited for its stores: the host may take the result
                            __hip_atomic_store(a.host_done + cur_ti, a.launch_seq, __ATOMIC_RELEASE,
                                               __HIP_MEMORY_SCOPE_SYSTEM);
                    }
                    last = all == 1u;
                }
            }
            if (keep < 0) credit = 0;
            if (uniform(last)) {
                if (linger)
                    for (uint32_t i = (uint32_t)ln; i < total_blocks_of(tt); i += LANES)
                        __hip_atomic_fetch_or(state_word(a, i), ST_X, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                release_waiters(a, ring_cap);
            }
        }
        if (fail) break;
    }
    if (wv == 0) flush_stats(w, st);
}

}  // namespace rk
