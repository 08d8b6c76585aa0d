// component.hpp -- the component route of the reconstruction kernels: tasks
// whose mask takes at most two values, 0 and one c > 0, reconstructed through
// connected-component labelling instead of block visits.
//
// For such a mask the reconstruction has a closed form.  By its bottleneck-
// path characterisation (rho(p) is the largest, over sources q and paths from
// q to p, of min(J(q), the smallest mask value on the path)), a path through a
// pixel of mask 0 contributes 0, and a path inside one connected component C
// of {I = c} contributes min(J(q), c).  A path from outside C into C must pass
// a pixel of mask 0, so
//     rho(p) = 0                                    where I(p) = 0,
//     rho(p) = max over q in C(p) of min(J(q), c)   where I(p) = c.
// That is a labelling of {I != 0} followed by a maximum per component: work
// proportional to the pixels, with no chain of dependent block visits.  A
// 1-pixel corridor winding across a 4096 x 4096 tile, which the block
// scheduler can only follow one block at a time (hundreds of thousands of
// visits in sequence), takes a few labelling passes here.  The bytes are the
// same as the block route's (the reconstruction is unique); the route is only
// faster.
//
// Kernels (workgroups of four waves for the first two, of one for the others,
// grid-stride over the blocks of all tasks of the launch, in the scheduler's
// block numbering: a block of BH x 256 pixels is BH / 16 labelling tiles of
// 16 x 256, or units of 4 rows or one of 256 pixels), after reset_work has
// sampled every task's mask (sample_route):
//   comp_classify     OR and AND of the nonzero (transformed) mask values of
//                     every task, into two words per task: the mask is
//                     two-valued when they are equal (one nonzero value) or the
//                     OR is 0 (an all-zero mask).  A wave skips the rows of a
//                     task already known to hold two different nonzero values,
//                     or that cannot take the route whatever its values.
//                     The last workgroup decides every task's route
//                     (decide_tasks), and prepare then fills the ring with the
//                     blocks of the others.  The whole kernel returns at once
//                     when the samples already decided every route;
//   comp_label_local  tile-local labelling of {I != 0} (label.hpp's label_tile)
//                     into the task's int32 label plane;
//   comp_label_merge  unions across tile borders (merge_tile);
//   comp_offer        each pixel whose min(J, I) is positive offers it to its
//                     root: an atomic maximum on the root's own entry of the
//                     label plane, encoded as ENC + value (ENC is above every
//                     node id, so a root entry at or above ENC marks a root
//                     that has an offer);
//   comp_write        the reconstruction: 0 on mask 0, else the value its
//                     root's entry holds (0 for a root without any offer),
//                     written as the task's result (into the caller's marker
//                     for a dilation, mapped as finish_result would otherwise).
// These tasks need no marker plane (the offers derive their initial marker
// as init_marker would), and none of their blocks is ever queued: init_marker,
// the ring and finish_result skip them.
#pragma once
#include "kernels.hpp"
#include "label.hpp"

namespace rk {

constexpr int32_t COMP_ENC = 0x40000000;   // above every node id (pitched index + 1 < 2^30)

// Labelling arguments of a task's (transformed) mask and label plane.
__device__ __forceinline__ LabelArgs comp_label_args(const TaskDev &t) {
    LabelArgs la{};
    la.img = t.i;
    la.pitch_img = t.pitch_i;
    la.lab = t.lab;
    la.pitch_lab = t.pitch_lab;
    la.h = t.h;
    la.w = t.w;
    la.conn = t.conn;
    la.tiles_x = t.nbx;     // LT_W == BW: a block column is a tile column
    la.bits = nullptr;
    la.fg_inv = t.minv;
    return la;
}

// Walks the global index space of the launch's blocks: unit u of `per` units
// per block -> task, block row / column.  cur caches the last task.
struct UnitWalk {
    int cur = -1;
    TaskDev t{};
    uint32_t t_end = 0;
    __device__ __forceinline__ void at(const TaskTable &tt, uint32_t gb) {
        if (cur < 0 || gb < t.block0 || gb >= t_end) {
            cur = uniform(find_task(tt, gb));
            t = task_of(tt, cur);
            t_end = t.block0 + (uint32_t)(t.nby * t.nbx);
        }
    }
};

// Classification: one workgroup of CLASS_WAVES waves per block of up to 32 rows, or
// 32 rows of a higher one (grid-stride), a wave's rows loaded together; each lane
// keeps the OR and AND of its nonzero mask bytes, a wave combines them once per
// task it leaves, and only a combination that changes a task's words is written
// (the words are read with plain loads first: a stale copy holds no bit that the
// current one lacks, so what it already shows need not be written).  A wave skips
// the blocks of a task whose words already show two different nonzero values (it
// can never take the route).
// Bound by its chain: table, words, rows, then one count per workgroup on a
// single word; so a workgroup covers many rows and a wave few: 15 us for one
// 2048 x 2048 mask, 21 with 32 rows to a wave and a wave to a workgroup.
constexpr int CLASS_WAVES = 4;

// Whether a task's words, read while waves add to them, show two different nonzero
// values.  The words change one after the other: an OR beside the AND's identity is
// one wave's on its way, of a mask that may hold a single value.  (The AND of two
// different values is never the identity.)
__device__ __forceinline__ bool shows_grey(uint32_t o, uint32_t n) { return o != 0u && n != 0xffu && o != n; }

template <int BH>
__global__ __launch_bounds__(64 * CLASS_WAVES) void comp_classify(TaskTable tt, KArgs a) {
    if (a.work->classify_skip == seq_of(tt)) return;   // the samples decided every route
    const int ln = lane_id(), wv = uniform((int)(threadIdx.x >> 6));
    constexpr int UH = BH < 32 ? BH : 32;         // rows of a unit
    constexpr int CH = UH / CLASS_WAVES;          // rows of a wave, their loads in flight together
    constexpr int PER = BH / UH;
    const uint32_t n = total_blocks_of(tt) * PER;
    UnitWalk wk;
    int acc_k = -1;                 // task whose partial OR / AND this wave holds
    uint32_t acc_or = 0, acc_and = 0xffffffffu;   // four bytes side by side
    uint32_t seen_or = 0, seen_and = 0;           // its words as read last
    const uint32_t seq = seq_of(tt);
    auto flush = [&]() {
        if (acc_k < 0) return;
        acc_or |= acc_or >> 16;
        acc_and &= acc_and >> 16;
        acc_or = (acc_or | acc_or >> 8) & 0xffu;
        acc_and = (acc_and & acc_and >> 8) & 0xffu;
        for (int d = 1; d < LANES; d <<= 1) {
            acc_or |= (uint32_t)__shfl_xor((int)acc_or, d);
            acc_and &= (uint32_t)__shfl_xor((int)acc_and, d);
        }
        uint32_t *wo = a.route + ROUTE_WORDS * acc_k, *wa = wo + 1;
        if (ln == 0 && ((acc_or & ~seen_or) | (seen_and & ~acc_and)) != 0u) {
            // looked up again: where the samples met no foreground, every wave's copies
            // still say so, and one word would take as many atomics as there are waves
            // (hole filling of a 4096 x 4096 checkerboard 240 us, 142 so)
            seen_or = __hip_atomic_load(wo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            seen_and = __hip_atomic_load(wa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (ln == 0 && ((acc_or & ~seen_or) | (seen_and & ~acc_and)) != 0u) {
            if ((acc_or & ~seen_or) != 0u) __hip_atomic_fetch_or(wo, acc_or, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((seen_and & ~acc_and) != 0u) __hip_atomic_fetch_and(wa, acc_and, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // (read back after both: of the waves that make a task grey together, the last one sees it)
            const uint32_t no = __hip_atomic_load(wo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t na = __hip_atomic_load(wa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // this task is grey (any writer, same value; a plain load first so
            // that a line already holding it is not written again by every wave)
            if (shows_grey(no, na) && a.work->has_grey != seq)
                __hip_atomic_store(&a.work->has_grey, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        acc_or = 0;
        acc_and = 0xffffffffu;
    };
    for (uint32_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t gb = u / PER;
        wk.at(tt, gb);
        const TaskDev &t = wk.t;
        if (!t.lab) continue;
        if (wk.cur != acc_k) {
            flush();
            acc_k = wk.cur;
        }
        const uint32_t *rw = a.route + ROUTE_WORDS * wk.cur;
        seen_or = rw[0];
        seen_and = rw[1];
        if (uniform(shows_grey(seen_or, seen_and) ? 1 : 0)) continue;
        // a thick mask beside grey work keeps the block route whatever its
        // values (decide_tasks), so it is not read either
        if (uniform(a.route_policy != 1 && rw[4] == 0u && a.work->has_grey == seq ? 1 : 0)) continue;
        const int lb = (int)(gb - t.block0);
        const BlockGeom g = geom<BH>(t, lb / t.nbx, lb % t.nbx);
        const int x = g.x0 + 4 * ln;
        const int valid = min(4, g.bw - 4 * ln);
        const int r0 = (int)(u % PER) * UH + wv * CH;
        uint32_t m[CH];
#pragma unroll
        for (int r = 0; r < CH; ++r) m[r] = (r0 + r < g.bh && valid > 0) ? mask4(t, g.y0 + r0 + r, x, valid) : 0u;
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const uint32_t zero = ~(m[r] | ((m[r] & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u;   // of the bytes that are 0
            acc_or |= m[r];
            acc_and &= m[r] | (zero >> 7) * 0xffu;
        }
    }
    flush();
    // the last workgroup to finish decides every task's route (decide_tasks).
    // All writes above are at the device-coherent level, and every wave waits
    // for its own before its workgroup counts (a barrier alone waits for LDS
    // only), so the count needs no release of this XCD's L2
    vm_sync();
    __syncthreads();
    if (wv != 0) return;
    uint32_t prior = 0;
    if (ln == 0)
        prior = __hip_atomic_fetch_add(&a.work->classify_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (uniform(prior) + 1u == gridDim.x) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        decide_tasks(tt, a);
    }
}

template <int BH>
__global__ __launch_bounds__(64 * LT_WAVES) void comp_label_local(TaskTable tt, KArgs a) {
    if (a.work->route_any != seq_of(tt)) return;   // no task of the launch takes the route
    RK_LDS uint32_t *par = (RK_LDS uint32_t *)dyn_lds();
    constexpr int PER = BH / LT_H;
    const uint64_t n = (uint64_t)total_blocks_of(tt) * PER;
    UnitWalk wk;
    for (uint64_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t gb = (uint32_t)(u / PER);
        wk.at(tt, gb);
        if (!on_component_route(a, wk.t, wk.cur)) continue;
        const int lb = (int)(gb - wk.t.block0);
        const int y0 = (lb / wk.t.nbx) * BH + (int)(u % PER) * LT_H, x0 = (lb % wk.t.nbx) * BW;
        if (y0 >= wk.t.h) continue;
        const LabelArgs la = comp_label_args(wk.t);
        label_tile(la, par, y0, x0);
    }
}

template <int BH>
__global__ __launch_bounds__(64) void comp_label_merge(TaskTable tt, KArgs a) {
    if (a.work->route_any != seq_of(tt)) return;   // no task of the launch takes the route
    constexpr int PER = BH / LT_H;
    const uint64_t n = (uint64_t)total_blocks_of(tt) * PER;
    UnitWalk wk;
    for (uint64_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t gb = (uint32_t)(u / PER);
        wk.at(tt, gb);
        if (!on_component_route(a, wk.t, wk.cur)) continue;
        const int lb = (int)(gb - wk.t.block0);
        const int y0 = (lb / wk.t.nbx) * BH + (int)(u % PER) * LT_H, x0 = (lb % wk.t.nbx) * BW;
        if (y0 >= wk.t.h) continue;
        merge_tile(comp_label_args(wk.t), y0, x0);
    }
}

// The root of node id a, *entry receiving what the root's own entry held: its id,
// or COMP_ENC + offer (which only a root's entry becomes).  Plain loads: while
// the route's last two kernels run, entries only change to an ancestor or, at
// roots, to COMP_ENC + offer, so a stale value still leads to the root.  A node
// that is further than one step away is pointed straight at its root, so the
// other pixels of its tile take one step.
__device__ __forceinline__ int32_t comp_root(int32_t *lab, int32_t a, int32_t *entry) {
    const RK_GLOBAL int32_t *l = (const RK_GLOBAL int32_t *)lab;
    int32_t p = l[a - 1];
    if (p == a || p >= COMP_ENC) {
        *entry = p;
        return a;
    }
    int32_t r = p;
    for (p = l[r - 1]; p != r && p < COMP_ENC; p = l[r - 1]) {
        __hip_atomic_store((RK_GLOBAL int32_t *)(lab + (a - 1)), p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r = p;
    }
    *entry = p;
    return r;
}

// Rows of a unit of the last two kernels: their loads go out together.  Both are
// bound by the latency of the walks from a pixel to its root: one row at a time,
// with every entry rewritten as its root's, they took 32-40 us and 14 us for the
// hole filling of a 2048 x 2048 mask, now 11 and 11.  Up to COMP_FEW such units (one
// per compute unit) a wave takes one row instead: the chip is idle either way, and
// a lane's walks follow one another (offers of a 3 x 2817 mask 14.7 us, 7.9 with
// a row to a wave; 300 x 300 81 us per call, 66).
constexpr int COMP_ROWS = 4;
constexpr uint64_t COMP_FEW = 256;

// The offers.  Only a positive min(J, I) can raise anything, so a pixel without
// one reads no label: hole filling, whose marker is the image frame, leaves
// almost all of the label plane alone here.  A lane sums up neighbouring pixels
// of one component, and the wave the lanes that share the first one's root (one
// component mostly fills the row), before they reach the root's entry.
template <int BH, int ROWS>
__device__ __forceinline__ void offer_units(const TaskTable &tt, const KArgs &a) {
    const int ln = lane_id();
    constexpr int PER = BH / ROWS;
    const uint64_t n = (uint64_t)total_blocks_of(tt) * PER;
    UnitWalk wk;
    for (uint64_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t gb = (uint32_t)(u / PER);
        wk.at(tt, gb);
        const TaskDev &t = wk.t;
        if (!on_component_route(a, t, wk.cur)) continue;
        const int lb = (int)(gb - t.block0);
        const int y0 = (lb / t.nbx) * BH + (int)(u % PER) * ROWS, x0 = (lb % t.nbx) * BW;
        if (y0 >= t.h) continue;
        const int x = x0 + 4 * ln;
        const int valid = min(4, t.w - x);
        // min(J, I), J the task's initial marker (the caller's for a dilation,
        // else derived here: no marker plane is prepared for a task on this route)
        uint32_t jm[ROWS], some = 0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int y = y0 + r;
            jm[r] = 0;
            if (y < t.h && valid > 0) {
                const uint8_t *jrow = t.j + (int64_t)y * t.pitch_j;
                const uint32_t j0 = t.op == OP_DILATE ? gload4(jrow, x, valid) : initial_marker4(t, jrow, y, x, valid);
                if (j0 != 0u) jm[r] = bmin4(j0, mask4(t, y, x, valid));
            }
            some |= jm[r];
        }
        int32_t root = 0;       // the lane's current root and the largest offer made to it
        uint32_t best = 0;
        auto offer = [&](int32_t r, uint32_t v) {   // (only when above what the entry shows already)
            int32_t *slot = t.lab + (r - 1);
            const int32_t seen = __hip_atomic_load((RK_GLOBAL int32_t *)slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (seen < COMP_ENC + (int32_t)v)
                __hip_atomic_fetch_max((RK_GLOBAL int32_t *)slot, COMP_ENC + (int32_t)v, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        };
        if (some != 0u) {
            int32_t v[ROWS][4];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                v[r][0] = v[r][1] = v[r][2] = v[r][3] = 0;
                if (jm[r] != 0u) lab_load4(t.lab + (int64_t)(y0 + r) * t.pitch_lab, x, t.w, v[r]);
            }
            int32_t last_v = 0, last_r = 0;   // the lane's pixels mostly share one tile root: one find for them
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t off = byte_of(jm[r], k);
                    if (off == 0u) continue;
                    int32_t e = v[r][k];
                    if (e >= COMP_ENC) {          // this pixel is a root that already has an offer
                        e = (int32_t)((int64_t)(y0 + r) * t.pitch_lab + x + k + 1);
                    } else {
                        if (e != last_v) {
                            int32_t entry;
                            last_v = e;
                            last_r = comp_root(t.lab, e, &entry);
                        }
                        e = last_r;
                    }
                    if (e != root) {
                        if (best != 0u) offer(root, best);
                        root = e;
                        best = 0;
                    }
                    best = max(best, off);
                }
        }
        const uint64_t lanes = __ballot(best != 0u);
        if (lanes == 0ull) continue;
        const int first = __builtin_ctzll(lanes);
        const int32_t shared = __builtin_amdgcn_readlane(root, first);
        const bool with = best != 0u && root == shared;
        const uint32_t top = (uint32_t)__builtin_amdgcn_readlane((int)wave_prefix_max(with ? best : 0u), LANES - 1);
        if (ln == first) offer(shared, top);
        else if (best != 0u && !with) offer(root, best);
    }
}

template <int BH>
__global__ __launch_bounds__(64) void comp_offer(TaskTable tt, KArgs a) {
    if (a.work->route_any != seq_of(tt)) return;   // no task of the launch takes the route
    if ((uint64_t)total_blocks_of(tt) * (BH / COMP_ROWS) <= COMP_FEW) offer_units<BH, 1>(tt, a);
    else offer_units<BH, COMP_ROWS>(tt, a);
}

// The result: every pixel's root is looked up here (a pixel points at its tile's
// root, and that one, from the merge or from an earlier look-up, at or near the
// component's).
template <int BH, int ROWS>
__device__ __forceinline__ void write_units(const TaskTable &tt, const KArgs &a) {
    const int ln = lane_id();
    constexpr int PER = BH / ROWS;
    const uint64_t n = (uint64_t)total_blocks_of(tt) * PER;
    UnitWalk wk;
    for (uint64_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t gb = (uint32_t)(u / PER);
        wk.at(tt, gb);
        const TaskDev &t = wk.t;
        if (!on_component_route(a, t, wk.cur)) continue;
        const int lb = (int)(gb - t.block0);
        const int y0 = (lb / t.nbx) * BH + (int)(u % PER) * ROWS, x0 = (lb % t.nbx) * BW;
        if (y0 >= t.h) continue;
        if (lb == 0 && u % PER == 0 && ln == 0)   // one count per task that took the route
            __hip_atomic_fetch_add(&a.work->stat_route, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int x = x0 + 4 * ln;
        const int valid = min(4, t.w - x);
        if (valid <= 0) continue;
        int32_t e[ROWS][4];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            e[r][0] = e[r][1] = e[r][2] = e[r][3] = 0;
            if (y0 + r < t.h) lab_load4(t.lab + (int64_t)(y0 + r) * t.pitch_lab, x, t.w, e[r]);
        }
        int32_t last_e = 0;
        uint32_t last_val = 0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int y = y0 + r;
            if (y >= t.h) break;
            uint32_t out = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                int32_t ent = e[r][k];
                if (ent == 0) continue;                   // mask 0
                if (ent != last_e) {
                    last_e = ent;
                    if (ent < COMP_ENC) (void)comp_root(t.lab, ent, &ent);
                    last_val = ent >= COMP_ENC ? (uint32_t)(ent - COMP_ENC) : 0u;
                }
                out |= last_val << (8 * k);
            }
            // the result itself: the reconstruction into the caller's marker for a
            // dilation, else mapped into the task's result plane
            if (t.op == OP_DILATE)
                gstore4(t.j + (int64_t)y * t.pitch_j, x, valid, out);
            else
                gstore4(t.img + (int64_t)y * t.pitch_img, x, valid, mapped_result4(t, out, y, x, valid));
        }
    }
}

template <int BH>
__global__ __launch_bounds__(64) void comp_write(TaskTable tt, KArgs a) {
    if (a.work->route_any != seq_of(tt)) return;   // no task of the launch takes the route
    if ((uint64_t)total_blocks_of(tt) * (BH / COMP_ROWS) <= COMP_FEW) write_units<BH, 1>(tt, a);
    else write_units<BH, COMP_ROWS>(tt, a);
}

}  // namespace rk
