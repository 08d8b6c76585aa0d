// label.hpp -- device code of connected-component labelling (BWLabel) and the
// area filter (AreaThreshold) of binary uint8 images, for AMD MI355X (gfx950).
//
// Both are listed in Table 1 of the paper (Sec. V-A) among the segmentation
// operations.  Definitions: the foreground is the set of nonzero pixels; two
// foreground pixels are connected through foreground paths of 4- or
// 8-neighbour steps (pixels outside the image do not exist); each component
// gets one label 1..n, numbered in raster order of its first pixel; the
// background gets 0.  The area filter keeps (255) the pixels of components
// whose pixel count lies in [min_area, max_area] and clears the rest.
//
// Method (union-find on the label plane itself, then a rank relabelling):
//   label_local     one workgroup per 16 x 256 tile, 4 rows a wave: each row's runs of
//                   foreground pixels become depth-one trees, then one
//                   union-find link (LDS atomic min: the larger root under
//                   the smaller) per pair of touching runs of adjacent rows,
//                   path compression, then every foreground pixel's node id
//                   is written: the pitched index + 1 of its tile root (0 on
//                   the background);
//   label_merge     one wave per tile: the tile's top row and left column
//                   against the neighbouring tiles' pixels, as a global
//                   union-find with agent-scope atomic min on the label plane
//                   (lock-free: a link only ever lowers a root's parent);
//   label_flatten   every pixel's node id becomes its root's; a root (the
//                   component's smallest pitched index, i.e. its raster-first
//                   pixel) sets its bit in a bitmap over pitched indices;
//   rank_*          exclusive prefix count of the bitmap words (per-segment
//                   sums, one wave scanning the segments, per-word offsets);
//   label_final     label = (roots before the pixel's root) + 1.
// Node ids are pitched indices (y * pitch + x) + 1, so the order of ids is the
// raster order and the parent of id a is stored at element a - 1.
#pragma once
#include "kernels.hpp"

namespace rk {

constexpr int LT_H = 16;     // rows of a labelling tile
constexpr int LT_ROWS = 4;   // rows of a wave of the tile's workgroup
constexpr int LT_WAVES = LT_H / LT_ROWS;
constexpr int LT_W = 256;    // columns (64 lanes x 4 pixels)
constexpr uint32_t LT_BG = 0xffffffffu;
constexpr int RANK_SEG = 1024;   // bitmap words per scan segment (64 lanes x 16)

struct LabelArgs {
    const uint8_t *img;     // input image (nonzero = foreground)
    int64_t pitch_img;      // bytes
    int32_t *lab;           // label plane (int32), written in place
    int64_t pitch_lab;      // elements
    int32_t h, w;
    int32_t conn;
    int32_t tiles_x;        // tiles per row of tiles
    uint32_t *bits;         // root bitmap over pitched indices (null: no ranks wanted)
    uint32_t *word_off;     // roots before each bitmap word
    uint32_t *seg_sum;      // roots per segment of RANK_SEG words
    uint32_t n_words;
    uint32_t n_segs;
    int32_t *count;         // receives the number of components (may be null)
    int32_t fg_inv;         // 1: the foreground is the pixels below 255 (the complement's nonzero pixels)
};

typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // (element-aligned: all that an access needs)

// 4 label elements at columns x..x+3 of a row (x a multiple of 4); elements
// at or past w read 0 and are not written.
__device__ __forceinline__ void lab_load4(const int32_t *row, int x, int w, int32_t v[4]) {
    if (x + 4 <= w) {
        const i32x4_any q = *(const RK_GLOBAL i32x4_any *)(row + x);
        v[0] = q.x;
        v[1] = q.y;
        v[2] = q.z;
        v[3] = q.w;
        return;
    }
    for (int k = 0; k < 4; ++k) v[k] = x + k < w ? ((const RK_GLOBAL int32_t *)row)[x + k] : 0;
}

__device__ __forceinline__ void lab_store4(int32_t *row, int x, int w, const int32_t v[4]) {
    if (x + 4 <= w) {
        i32x4_any q;
        q.x = v[0];
        q.y = v[1];
        q.z = v[2];
        q.w = v[3];
        *(RK_GLOBAL i32x4_any *)(row + x) = q;
        return;
    }
    for (int k = 0; k < 4; ++k)
        if (x + k < w) ((RK_GLOBAL int32_t *)row)[x + k] = v[k];
}

// ---- tile-local union-find in LDS (indices within the tile)

__device__ __forceinline__ uint32_t lds_find(RK_LDS uint32_t *par, uint32_t a) {
    while (true) {
        const uint32_t p = __hip_atomic_load(par + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (p == a) return a;
        a = p;
    }
}

__device__ __forceinline__ void lds_union(RK_LDS uint32_t *par, uint32_t a, uint32_t b) {
    while (true) {
        a = lds_find(par, a);
        b = lds_find(par, b);
        if (a == b) return;
        if (a < b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        // a is (or was) a root above b: hang it under b unless someone linked it meanwhile
        const uint32_t old = __hip_atomic_fetch_min(par + a, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old == a) return;
        a = old;
    }
}

// ---- global union-find on the label plane (node ids: pitched index + 1)

// Find with path halving: every other node on the path is pointed at its
// grandparent (an atomic minimum: a parent always has the smaller id, so the
// entry only moves up its own tree, whatever other waves write meanwhile).
// Without it, a component spanning many tiles (a background, a corridor)
// builds chains as long as the tiles it crosses.  The loads are at the
// device-coherent level, a trip to memory each: over copies that a cache holds from
// before other waves linked or shortened a chain, a walk ends far below the root, and
// goes on from there by one g_union minimum per entry (labels of a 2995 x 1846
// serpentine, a leg every 3 rows: 325 us with ordinary loads, 110 so; of a 5000 x 64
// spiral 285 us with ordinary loads in the first step alone, 155 so; hole filling
// of a 2048 x 2048 nuclei mask 96 and 97.5).
__device__ __forceinline__ int32_t g_find(int32_t *lab, int32_t a) {
    while (true) {
        const int32_t p = __hip_atomic_load((RK_GLOBAL int32_t *)(lab + (a - 1)), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
        if (p == a) return a;
        const int32_t gp = __hip_atomic_load((RK_GLOBAL int32_t *)(lab + (p - 1)), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if (gp == p) return p;
        __hip_atomic_fetch_min((RK_GLOBAL int32_t *)(lab + (a - 1)), gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a = gp;
    }
}

// The same without the halving, once no tree changes any more but by entries
// moving up to their root.
__device__ __forceinline__ int32_t g_root(const int32_t *lab, int32_t a) {
    while (true) {
        const int32_t p = ((const RK_GLOBAL int32_t *)lab)[a - 1];
        if (p == a) return a;
        a = p;
    }
}

__device__ __forceinline__ void g_union(int32_t *lab, int32_t a, int32_t b) {
    while (true) {
        a = g_find(lab, a);
        b = g_find(lab, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = __hip_atomic_fetch_min((RK_GLOBAL int32_t *)(lab + (a - 1)), b, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        if (old == a) return;   // a was a root
        a = old;                // (smaller than a: the walk ends)
    }
}

// inclusive prefix maximum over the 64 lanes of a wave (unsigned values; 0
// is the identity): DPP row shifts inside each 16-lane row, then the totals of
// the rows before through readlane
__device__ __forceinline__ uint32_t wave_prefix_max(uint32_t v) {
    v = max(v, dpp_or<DPP_ROW_SHR + 1>(0u, v));
    v = max(v, dpp_or<DPP_ROW_SHR + 2>(0u, v));
    v = max(v, dpp_or<DPP_ROW_SHR + 4>(0u, v));
    v = max(v, dpp_or<DPP_ROW_SHR + 8>(0u, v));
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
    const uint32_t r1 = max(r0, (uint32_t)__builtin_amdgcn_readlane((int)v, 31));
    const uint32_t r2 = max(r1, (uint32_t)__builtin_amdgcn_readlane((int)v, 47));
    return max(v, sel_row(lane_id() >> 4, 0u, r0, r1, r2));
}

// The 4 pixels at columns x..x+3 of row y as foreground bytes: nonzero where
// the pixel is foreground (fg_inv: below 255), 0 elsewhere and past the image.
__device__ __forceinline__ uint32_t fg_load4(const LabelArgs &a, int y, int x, int valid) {
    uint32_t v = gload4(a.img + (int64_t)y * a.pitch_img, x, valid);
    if (a.fg_inv) {
        const uint32_t keep = valid >= 4 ? 0xffffffffu : (valid <= 0 ? 0u : ((1u << (8 * valid)) - 1u));
        v = (~v) & keep;
    }
    return v;
}

// Phase 1: tile-local labelling.  Grid: one workgroup of LT_WAVES waves per tile
// (grid-stride); dynamic LDS: LT_H * LT_W * 4 bytes.  Wave v holds rows
// LT_ROWS * v.. of the tile, lane l columns 4l..4l+3 of each.
//   a. runs: every foreground pixel's parent is the first pixel of its run of
//      foreground pixels in the row (one prefix maximum over the lanes of the
//      last background column), so a run is a tree of depth one;
//   b. unions between each run and every run of the row above that touches
//      it, issued once per pair of runs: by the pixel under (4-conn) or
//      diagonally under (8-conn) the upper run's first pixel inside the
//      window the run can reach;
//   c. path compression; d. node ids out.
// label_tile is one tile (all waves of the workgroup; `par` holds LT_H * LT_W
// words of LDS); label_local runs it over the tiles of one image.
// Bound by chains of LDS accesses, so a tile's rows are spread over LT_WAVES
// waves (a tile of one wave ran 4 times as long a chain, at the 10 waves a
// compute unit's LDS then holds), and the links and the compression go through
// each lane's own list of bits (a step of the wave serves every lane that has
// something left).  The 4096 x 4096 binary tile takes 23 us (16 MB read, 64 MB
// written: 3.5 TB/s; 42 with a tile to a wave), a 2048 x 2048 mask, whose 1024
// tiles leave most of the chip idle, 17 (29).  2 rows a wave: the same.
__device__ void label_tile(const LabelArgs &a, RK_LDS uint32_t *par, int y0, int x0) {
    const int ln = lane_id();
    const int r0 = uniform((int)(threadIdx.x >> 6)) * LT_ROWS;   // the wave's first row of the tile
    const int c = 4 * ln;
    const int th = min(LT_H, a.h - y0), tw = min(LT_W, a.w - x0);
    const int valid = min(4, tw - c);
    uint32_t fg = 0;   // bit 4(r+1)+k: pixel (r0+r, c+k) is foreground; bits 0..3: the row above the wave's rows
    uint32_t rows[LT_ROWS];   // all loads in flight together
#pragma unroll
    for (int r = 0; r < LT_ROWS; ++r)
        rows[r] = r0 + r < th ? fg_load4(a, y0 + r0 + r, x0 + c, valid) : 0u;
#pragma unroll
    for (int r = 0; r < LT_ROWS; ++r) {
        const uint32_t v = rows[r];
        int lb = -1;          // last background column so far in this lane
        int lbk[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool f = ((v >> (8 * k)) & 0xffu) != 0u;
            fg |= (f ? 1u : 0u) << (4 * r + 4 + k);
            if (!f) lb = c + k;
            lbk[k] = lb;
        }
        // last background column before this lane (-1: none), through
        // values shifted by one so that 0 is the identity
        const int excl = (int)from_lower(wave_prefix_max((uint32_t)(lb + 1))) - 1;
        u32x4 start;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool f = (fg >> (4 * r + 4 + k)) & 1u;
            start[k] = f ? (uint32_t)((r0 + r) * LT_W + max(excl, lbk[k]) + 1) : LT_BG;
        }
        *(RK_LDS u32x4 *)(par + (r0 + r) * LT_W + c) = start;
    }
    __syncthreads();
    if (r0 > 0) {   // (links move entries meanwhile, but none to or from LT_BG)
        const u32x4 above = *(const RK_LDS u32x4 *)(par + (r0 - 1) * LT_W + c);
#pragma unroll
        for (int k = 0; k < 4; ++k) fg |= (above[k] != LT_BG ? 1u : 0u) << k;
    }
    // every pixel's neighbours as bits at its own position (no neighbour
    // inside the tile: background; the tile borders are joined by label_merge)
    const uint32_t left = ((fg & 0x77777777u) << 1) | ((from_lower(fg) >> 3) & 0x11111111u);
    const uint32_t right = ((fg >> 1) & 0x77777777u) | ((from_upper(fg) & 0x11111111u) << 3);
    const uint32_t up = fg << 4, up_left = left << 4, up_right = right << 4;
    const uint32_t own = fg & ~0xfu;
    const uint32_t base = (uint32_t)((r0 - 1) * LT_W + c);   // of bit 0
    // links, each once per pair of runs (see above); a lane walks through its
    // own, so that the wave takes as many steps as its busiest lane has links
    // instead of one per pixel position
    uint32_t links = a.conn == 8 ? own & ~left & (up_left | up) : own & up & ~(left & up_left);
    for (; links; links &= links - 1) {
        const int q = __builtin_ctz(links);
        const uint32_t i = base + (uint32_t)((q >> 2) * LT_W + (q & 3));
        lds_union(par, i, i - LT_W - (a.conn == 8 ? (up_left >> q) & 1u : 0u));
    }
    if (a.conn == 8)
        for (links = own & ~up & up_right; links; links &= links - 1) {
            const int q = __builtin_ctz(links);
            const uint32_t i = base + (uint32_t)((q >> 2) * LT_W + (q & 3));
            lds_union(par, i, i - LT_W + 1u);
        }
    __syncthreads();
    // path compression of the run starts (every other pixel's parent is its
    // run's start, so afterwards its root is two steps away)
    for (uint32_t starts = own & ~left; starts; starts &= starts - 1) {
        const int q = __builtin_ctz(starts);
        const uint32_t i = base + (uint32_t)((q >> 2) * LT_W + (q & 3));
        par[i] = lds_find(par, i);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < LT_ROWS; ++r) {
        const u32x4 start = *(const RK_LDS u32x4 *)(par + (r0 + r) * LT_W + c);
        int32_t ids[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool f = (fg >> (4 * r + 4 + k)) & 1u;
            const uint32_t root = par[f ? start[k] : 0u];
            const int ry = (int)(root / LT_W), rx = (int)(root % LT_W);
            ids[k] = f ? (int32_t)((int64_t)(y0 + ry) * a.pitch_lab + x0 + rx + 1) : 0;
        }
        if (r0 + r < th) lab_store4(a.lab + (int64_t)(y0 + r0 + r) * a.pitch_lab, x0 + c, a.w, ids);
    }
    __syncthreads();
}

__global__ __launch_bounds__(64 * LT_WAVES) void label_local(LabelArgs a) {
    RK_LDS uint32_t *par = (RK_LDS uint32_t *)dyn_lds();
    const int n_tiles = a.tiles_x * ((a.h + LT_H - 1) / LT_H);
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
        label_tile(a, par, (tile / a.tiles_x) * LT_H, (tile % a.tiles_x) * LT_W);
}

// Phase 2: unions across tile borders.  One 64-lane workgroup per tile
// (grid-stride).  The top row meets the row above (the tiles above), the left
// column meets the column to the left; with 8-connectivity the diagonal
// neighbours too.  Every pair of adjacent pixels in different tiles is met at
// least once.
// Unions across the tile's top row and left column, issued once per pair of
// touching runs (the rule label_tile uses inside a tile): along the top row,
// pixel x of the tile's row (c) and the row above (a); a pixel whose left
// neighbour c[x-1] is foreground joins a[x-1] and a[x] through it, and a[x+1]
// through a[x] when that is foreground; so with 8-connectivity c[x] links
// a[x-1] (or else a[x]) only if it starts a run, and a[x+1] only if a[x] is
// background; with 4-connectivity a[x] only if c[x-1] and a[x-1] are not both
// foreground.  The left column is the same along the rows (a: column x0 - 1).
// A skip relies on c[x-1] joined to c[x] and a[x-1] to a[x], so it is taken
// only where c[x-1] lies inside this tile (label_tile joined the run); the
// first pixel of the row (or column) always links explicitly.  Then every
// implied link rests on links inside one tile, and a pair of diagonal or
// cross-corner neighbours in other tiles is always linked explicitly.  A
// component spanning many tiles (a background) costs a few unions per tile
// instead of one per border pixel.
// Bound by the walks to the roots (a trip to the L2 for every step): all entries
// that decide the links are loaded at once, a lane then goes through its own
// links, and those between the pair of nodes that the first lane joins (along a
// border mostly two large components) are left to that lane.  9.0 us for the
// 4096 x 4096 binary tile, 16.5 for the background of a 2048 x 2048 mask (10.5 and
// 18.3 with the neighbours loaded pixel by pixel).
__device__ void merge_tile(const LabelArgs &a, int y0, int x0) {
    const int ln = lane_id();
    const int th = min(LT_H, a.h - y0), tw = min(LT_W, a.w - x0);
    auto at = [&](int y, int x) -> int32_t {
        return y >= 0 && y < a.h && x >= 0 && x < a.w ? ((const RK_GLOBAL int32_t *)a.lab)[(int64_t)y * a.pitch_lab + x] : 0;
    };
    const int x = x0 + 4 * ln;
    int32_t c[4] = {0, 0, 0, 0}, u[4] = {0, 0, 0, 0};   // the tile's top row, the row above it
    int32_t ul = 0, ur = 0;                             // u[-1], u[4]
    if (y0 > 0) {
        if (x < x0 + tw) {
            lab_load4(a.lab + (int64_t)y0 * a.pitch_lab, x, a.w, c);
            lab_load4(a.lab + (int64_t)(y0 - 1) * a.pitch_lab, x, a.w, u);
        }
        if (ln == 0) ul = at(y0 - 1, x0 - 1);
        if (ln == LANES - 1) ur = at(y0 - 1, x0 + LT_W);
    }
    // lane l: rows y0 - 1 + l of the tile's left column and the column left of it
    int32_t cc = 0, cu = 0;
    if (x0 > 0 && ln <= th + 1) {
        cc = ln >= 1 && ln <= th ? at(y0 - 1 + ln, x0) : 0;
        cu = at(y0 - 1 + ln, x0 - 1);
    }
    const int32_t cl0 = (int32_t)from_lower((uint32_t)c[3]);   // c[-1]: 0 for the first lane (outside this tile)
    const int32_t u_lo = (int32_t)from_lower((uint32_t)u[3]), u_up = (int32_t)from_upper((uint32_t)u[0]);
    if (ln != 0) ul = u_lo;
    if (ln != LANES - 1) ur = u_up;
    const int32_t cc_lo = (int32_t)from_lower((uint32_t)cc), cu_lo = (int32_t)from_lower((uint32_t)cu);
    const int32_t cu_up = (int32_t)from_upper((uint32_t)cu);
    // links: bit k, the top row's pixel k with o[k]; bit 4 + k, with the pixel
    // above right of it; bits 8 and 9, the left column's pixel likewise
    uint32_t links = 0;
    int32_t o[5];
    auto link = [&](int bit, int32_t self, bool in, int32_t before, int32_t al, int32_t au, int32_t ar, int32_t &other) {
        const bool cl = in && before != 0;   // the pixel before it inside this tile
        other = au;
        if (self == 0) return;
        if (a.conn == 8) {
            if (al != 0) other = al;
            if (!cl && (al != 0 || au != 0)) links |= 1u << bit;
            if (au == 0 && ar != 0) links |= 1u << (bit == 8 ? 9 : bit + 4);
        } else if (au != 0 && (!cl || !(in && al != 0))) {
            links |= 1u << bit;
        }
    };
#pragma unroll
    for (int k = 0; k < 4; ++k)
        link(k, c[k], k > 0 || ln > 0, k > 0 ? c[k - 1] : cl0, k > 0 ? u[k - 1] : ul, u[k], k < 3 ? u[k + 1] : ur, o[k]);
    link(8, cc, ln >= 2, cc_lo, cu_lo, cu, cu_up, o[4]);
    int32_t done_s = 0, done_o = 0;
    for (uint64_t live = __ballot(links != 0u); live != 0ull; live = __ballot(links != 0u)) {
        const uint32_t bit = links & (0u - links);
        links ^= bit;
        int32_t self = cc, other = bit == 1u << 9 ? cu_up : o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (bit & (0x11u << k)) self = c[k];
            if (bit == 1u << k) other = o[k];
            if (bit == 0x10u << k) other = k < 3 ? u[k + 1] : ur;
        }
        const int first = __builtin_ctzll(live);
        const int32_t fs = __builtin_amdgcn_readlane(self, first), fo = __builtin_amdgcn_readlane(other, first);
        const bool again = (self == done_s && other == done_o) || (ln != first && self == fs && other == fo);
        if (bit != 0u && !again) {
            g_union(a.lab, self, other);
            done_s = self;
            done_o = other;
        }
    }
}

__global__ __launch_bounds__(64) void label_merge(LabelArgs a) {
    const int n_tiles = a.tiles_x * ((a.h + LT_H - 1) / LT_H);
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
        merge_tile(a, (tile / a.tiles_x) * LT_H, (tile % a.tiles_x) * LT_W);
}

// Clear a word array (a fill kernel rather than a memset node).
__global__ void clear_words(uint32_t *p, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// The kernels below go over the label plane in units of LF_ROWS rows of 256
// columns, a wave per unit (64 lanes x 4 pixels a row, the rows' loads out
// together; a row per wave took 81 us against 76 for the labelling of the
// 4096 x 4096 binary tile, each of its last passes moving 128 MB).
constexpr int LF_ROWS = 4;

__device__ __forceinline__ int64_t lf_units(int h, int w) {
    return (int64_t)((h + LF_ROWS - 1) / LF_ROWS) * ((w + LT_W - 1) / LT_W);
}

struct LfUnit {
    int y0, rows, x;   // first row, rows inside the image, the lane's first column
    __device__ __forceinline__ LfUnit(int64_t q, int h, int w) {
        const int chunks = (w + LT_W - 1) / LT_W;
        y0 = (int)(q / chunks) * LF_ROWS;
        rows = min(LF_ROWS, h - y0);
        x = (int)(q % chunks) * LT_W + 4 * lane_id();
    }
    __device__ __forceinline__ void load(const int32_t *lab, int64_t pitch, int w, int32_t v[LF_ROWS][4]) const {
#pragma unroll
        for (int r = 0; r < LF_ROWS; ++r) {
            v[r][0] = v[r][1] = v[r][2] = v[r][3] = 0;
            if (r < rows) lab_load4(lab + (int64_t)(y0 + r) * pitch, x, w, v[r]);
        }
    }
};

// Phase 3: every foreground pixel takes its root's id; roots set their bit.
// Grid-stride over the units.
__global__ __launch_bounds__(64) void label_flatten(LabelArgs a) {
    const int64_t n = lf_units(a.h, a.w);
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const LfUnit u(q, a.h, a.w);
        int32_t v[LF_ROWS][4];
        u.load(a.lab, a.pitch_lab, a.w, v);
        int32_t last_v = 0, last_r = 0;   // (a lane's pixels mostly share a tile root)
#pragma unroll
        for (int r = 0; r < LF_ROWS; ++r) {
            int32_t *row = a.lab + (int64_t)(u.y0 + r) * a.pitch_lab;
            bool any = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (v[r][k] == 0) continue;
                if (v[r][k] != last_v) {
                    last_v = v[r][k];
                    last_r = g_root(a.lab, last_v);
                }
                any |= last_r != v[r][k];
                v[r][k] = last_r;
                const int32_t self = (int32_t)((int64_t)(u.y0 + r) * a.pitch_lab + u.x + k + 1);
                if (last_r == self && a.bits) {
                    const uint32_t bit = (uint32_t)(self - 1);
                    __hip_atomic_fetch_or(a.bits + (bit >> 5), 1u << (bit & 31u), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (any) lab_store4(row, u.x, a.w, v[r]);
        }
    }
}

// inclusive prefix sum over the 64 lanes of a wave
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
    const int ln = lane_id();
#pragma unroll
    for (int d = 1; d < LANES; d <<= 1) {
        const uint32_t o = __shfl_up(v, (unsigned)d);
        if (ln >= d) v += o;
    }
    return v;
}

// Phase 4a: roots per segment of RANK_SEG bitmap words.
__global__ __launch_bounds__(64) void rank_segments(LabelArgs a) {
    const int ln = lane_id();
    for (uint32_t s = blockIdx.x; s < a.n_segs; s += gridDim.x) {
        uint32_t sum = 0;
        const uint32_t w0 = s * RANK_SEG + (uint32_t)ln * 16u;
        for (uint32_t j = 0; j < 16u; ++j)
            if (w0 + j < a.n_words) sum += (uint32_t)__popc(a.bits[w0 + j]);
        const uint32_t tot = __shfl(wave_prefix(sum), LANES - 1);
        if (ln == 0) a.seg_sum[s] = tot;
    }
}

// Phase 4b: one wave turns the segment sums into exclusive offsets (in place)
// and writes the number of components.
__global__ __launch_bounds__(64) void rank_scan(LabelArgs a) {
    const int ln = lane_id();
    uint32_t carry = 0;
    for (uint32_t s0 = 0; s0 < a.n_segs; s0 += LANES) {
        const uint32_t s = s0 + (uint32_t)ln;
        const uint32_t v = s < a.n_segs ? a.seg_sum[s] : 0u;
        const uint32_t inc = wave_prefix(v);
        if (s < a.n_segs) a.seg_sum[s] = carry + inc - v;
        carry += __shfl(inc, LANES - 1);
    }
    if (ln == 0 && a.count) *a.count = (int32_t)carry;
}

// Phase 4c: roots before every bitmap word.
__global__ __launch_bounds__(64) void rank_words(LabelArgs a) {
    const int ln = lane_id();
    for (uint32_t s = blockIdx.x; s < a.n_segs; s += gridDim.x) {
        const uint32_t w0 = s * RANK_SEG + (uint32_t)ln * 16u;
        uint32_t cnt[16];
        uint32_t sum = 0;
        for (uint32_t j = 0; j < 16u; ++j) {
            cnt[j] = w0 + j < a.n_words ? (uint32_t)__popc(a.bits[w0 + j]) : 0u;
            sum += cnt[j];
        }
        uint32_t run = a.seg_sum[s] + wave_prefix(sum) - sum;
        for (uint32_t j = 0; j < 16u; ++j) {
            if (w0 + j < a.n_words) a.word_off[w0 + j] = run;
            run += cnt[j];
        }
    }
}

// Phase 5: final labels 1..n in raster order of the roots.  Grid-stride over
// the units.
__global__ __launch_bounds__(64) void label_final(LabelArgs a) {
    const int64_t n = lf_units(a.h, a.w);
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const LfUnit u(q, a.h, a.w);
        int32_t v[LF_ROWS][4];
        u.load(a.lab, a.pitch_lab, a.w, v);
        int32_t last_v = 0, last_l = 0;
#pragma unroll
        for (int r = 0; r < LF_ROWS; ++r) {
            if ((v[r][0] | v[r][1] | v[r][2] | v[r][3]) == 0) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (v[r][k] == 0) continue;
                if (v[r][k] != last_v) {
                    last_v = v[r][k];
                    const uint32_t root = (uint32_t)(last_v - 1);
                    const uint32_t below = a.bits[root >> 5] & ((1u << (root & 31u)) - 1u);
                    last_l = (int32_t)(a.word_off[root >> 5] + (uint32_t)__popc(below) + 1u);
                }
                v[r][k] = last_l;
            }
            lab_store4(a.lab + (int64_t)(u.y0 + r) * a.pitch_lab, u.x, a.w, v[r]);
        }
    }
}

// ---- area filter (on a flattened label plane: every foreground pixel holds
// its component's root id, so no rank relabelling is needed)

struct AreaArgs {
    const int32_t *lab;
    int64_t pitch_lab;
    uint32_t *area;         // pixel count per root id (index 0 unused)
    uint8_t *out;           // the image, overwritten with 255 / 0
    int64_t pitch_out;
    int32_t h, w;
    int64_t min_area, max_area;
};

// Pixel counts per root id: equal ids that follow one another in a lane's pixels
// are added with one atomic.  Grid-stride over the units.
__global__ __launch_bounds__(64) void area_count(AreaArgs a) {
    const int64_t n = lf_units(a.h, a.w);
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const LfUnit u(q, a.h, a.w);
        int32_t v[LF_ROWS][4];
        u.load(a.lab, a.pitch_lab, a.w, v);
        int32_t cur = 0;
        uint32_t run = 0;
#pragma unroll
        for (int r = 0; r < LF_ROWS; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (v[r][k] == 0) continue;
                if (v[r][k] != cur) {
                    if (cur != 0) __hip_atomic_fetch_add(a.area + cur, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    cur = v[r][k];
                    run = 0;
                }
                run += 1;
            }
        if (cur != 0) __hip_atomic_fetch_add(a.area + cur, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ __launch_bounds__(64) void area_apply(AreaArgs a) {
    const int64_t n = lf_units(a.h, a.w);
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const LfUnit u(q, a.h, a.w);
        int32_t v[LF_ROWS][4];
        u.load(a.lab, a.pitch_lab, a.w, v);
        int32_t last_v = 0;
        uint32_t keep = 0;
#pragma unroll
        for (int r = 0; r < LF_ROWS; ++r) {
            uint32_t out = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (v[r][k] == 0) continue;
                if (v[r][k] != last_v) {
                    last_v = v[r][k];
                    const int64_t ar = (int64_t)a.area[last_v];
                    keep = ar >= a.min_area && ar <= a.max_area ? 0xffu : 0u;
                }
                out |= keep << (8 * k);
            }
            if (r < u.rows) gstore4(a.out + (int64_t)(u.y0 + r) * a.pitch_out, u.x, min(4, a.w - u.x), out);
        }
    }
}

}  // namespace rk
