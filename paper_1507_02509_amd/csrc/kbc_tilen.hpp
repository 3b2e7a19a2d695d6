// kbc_tilen.hpp -- T >= 3 fused time steps on one workgroup tile.
//
// A workgroup owns an output tile of 64 x TH nodes.  Step s (1 .. T) runs on
// the tile extended by T - s nodes on every side (periodic), so that the next
// step finds every population it pulls; step 1 gathers from the state buffer
// exactly as the single step does and step T writes the tile to the
// destination buffer, so T steps read and write the state once.
//
// Between the steps the populations live in one LDS window, updated in place.
// Each step alternates between two conventions so that a node reads and
// writes the same nine slots and no other node's (P. Bailey, J. Myre,
// S. D. C. Walsh, D. J. Lilja, M. O. Saar, "Accelerating lattice Boltzmann
// fluid flow simulations using graphics processors", 2009, the A-A pattern):
//   * step 1, and every odd step s < T, leaves its result pushed: population
//     i of node x in slot (i, x + v_i);
//   * an even step reads its node's own slots (i, x) and leaves its result
//     turned: population i in slot (opp(i), x);
//   * an odd step s >= 3 pulls population i from slot (opp(i), x - v_i).  As i
//     runs over the velocities these are the slots (j, x + v_j) that it pushes
//     to.
// So one barrier per step orders everything and the window needs no second
// copy: 9 x (TH + 2 (T - 2)) x (64 + 2 (T - 2)) values.  Values in the window
// are in the storage form, rounded as the single step rounds them on the way
// to memory, and every step runs the same collision code: T fused steps are
// bitwise identical to T single steps.
//
// Work split: the 64 interior columns of an extended row are one wave task
// (uniform row, scalar bases, as in the single step); the 2 (T - s) columns
// beside them are packed, 64 nodes of several rows to a task.  A step's tasks
// go round-robin to the NW waves, the packed ones first.  A ragged last tile
// takes only the rows its own output needs.
#pragma once

#include "kbc_tile2.hpp"

namespace kbc {

__host__ __device__ constexpr int opp(int i) { return i == 0 ? 0 : (i < 5 ? (i + 1) % 4 + 1 : (i - 5 + 2) % 4 + 5); }

template <int FORM, int T, int TH>
constexpr size_t stepn_lds() {
    return size_t{9} * (TH + 2 * (T - 2)) * (64 + 2 * (T - 2)) * sizeof(typename Form<FORM>::S);
}

// Steps S .. T of stepn_tile on the LDS window (S >= 2).
template <int FORM, int COLL, int VAR, int GM, int T, int TH, int NW, bool NT, int S>
__device__ __forceinline__ void stepn_rest(typename Form<FORM>::S* __restrict__ win,
                                           typename Form<FORM>::S* __restrict__ dst, int nx, int ny, int64_t pitch,
                                           int x0, int y0, int th, int lane, int w,
                                           const Coef<typename Form<FORM>::R>& K) {
    using E = typename Form<FORM>::S;
    constexpr int M = T - 2;                              // window margin around the tile
    constexpr int WH = TH + 2 * M, WW = 64 + 2 * M;
    constexpr int H = T - S;                              // this step's margin
    constexpr int packed = (2 * H * (TH + 2 * H) + 63) / 64;
    const int rows = th + 2 * H, side = 2 * H * rows;
    constexpr bool even = S % 2 == 0;
    __syncthreads();
    // the node at window offset o (row * WW + column)
    auto node = [&](int o, E (&v)[9]) {
        const E* p = win + o;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if constexpr (even)
                v[i] = p[i * WH * WW];
            else
                v[i] = p[opp(i) * WH * WW - kCy[i] * WW - kCx[i]];
        }
        collide_stored<FORM, COLL, VAR, GM>(v, K);
    };
    for (int t = w; t < packed + rows; t += NW) {
        E v[9];
        if constexpr (S < T) {
            int o = (t - packed + M - H) * WW + lane + M;
            bool on = true;
            if (t < packed) {
                const int k = t * 64 + lane;
                const int r = k / (2 * H), q = k - r * 2 * H;
                o = (r + M - H) * WW + (q < H ? q : q + 64) + M - H;
                on = k < side;
            }
            if (on) {
                node(o, v);
                E* p = win + o;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    if constexpr (even)
                        p[opp(i) * WH * WW] = v[i];
                    else
                        p[i * WH * WW + kCy[i] * WW + kCx[i]] = v[i];
                }
            }
        } else if (x0 + lane < nx) {
            node((t + M) * WW + lane + M, v);
            const uint32_t c0 = static_cast<uint32_t>(x0 + lane) * sizeof(E);
#pragma unroll
            for (int i = 0; i < 9; ++i) st_at<NT>(row_ptr(dst, y0 + t, i, pitch), c0, v[i]);
        }
    }
    if constexpr (S < T)
        stepn_rest<FORM, COLL, VAR, GM, T, TH, NW, NT, S + 1>(win, dst, nx, ny, pitch, x0, y0, th, lane, w, K);
}

// T fused steps on the output tile with corner (x0, y0), for the 64 NW
// threads of the calling workgroup (all of which must call it).
template <int FORM, int COLL, int VAR, int GM, int T, int TH, int NW, bool NT>
__device__ __forceinline__ void stepn_tile(const typename Form<FORM>::S* __restrict__ src,
                                           typename Form<FORM>::S* __restrict__ dst, int nx, int ny, int64_t pitch,
                                           int x0, int y0, const Coef<typename Form<FORM>::R>& K) {
    using E = typename Form<FORM>::S;
    static_assert(T >= 3, "two steps have a tile of their own (step2_tile)");
    constexpr int M = T - 2, H = T - 1;
    constexpr int WH = TH + 2 * M, WW = 64 + 2 * M;
    constexpr int packed = (2 * H * (TH + 2 * H) + 63) / 64;
    const int th = ny - y0 < TH ? ny - y0 : TH;           // rows of a ragged last tile
    const int rows = th + 2 * H, side = 2 * H * rows;
    __shared__ E win[9 * WH * WW];
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));

    const int gx = pmod(x0 + lane, nx);
    const uint32_t c0 = static_cast<uint32_t>(gx) * sizeof(E);
    const uint32_t cm = static_cast<uint32_t>(gx == 0 ? nx - 1 : gx - 1) * sizeof(E);
    const uint32_t cp = static_cast<uint32_t>(gx == nx - 1 ? 0 : gx + 1) * sizeof(E);
    auto load_row = [&](int r, E (&v)[9]) {
        const int y = wrap_uniform(y0 + r - H, ny), ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
        v[0] = ld_at(row_ptr(src, y, 0, pitch), c0);
        v[1] = ld_at(row_ptr(src, y, 1, pitch), cm);
        v[2] = ld_at(row_ptr(src, ym, 2, pitch), c0);
        v[3] = ld_at(row_ptr(src, y, 3, pitch), cp);
        v[4] = ld_at(row_ptr(src, yp, 4, pitch), c0);
        v[5] = ld_at(row_ptr(src, ym, 5, pitch), cm);
        v[6] = ld_at(row_ptr(src, ym, 6, pitch), cp);
        v[7] = ld_at(row_ptr(src, yp, 7, pitch), cp);
        v[8] = ld_at(row_ptr(src, yp, 8, pitch), cm);
    };
    auto row = [&](int r, E (&v)[9]) {
        collide_stored<FORM, COLL, VAR, GM>(v, K);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int a = r - 1 + kCy[i];
            if (a >= 0 && a < WH) win[(i * WH + a) * WW + lane + M + kCx[i]] = v[i];
        }
    };
    // the wave's rows: the first one's loads are in flight during the packed
    // nodes, the next one's while a row collides (two register sets, as in
    // step2_tile)
    int r = (w - packed % NW + NW) % NW;
    E va[9], vb[9];
    if (r < rows) load_row(r, va);
    for (int t = w; t < packed; t += NW) {
        const int k = t * 64 + lane;
        if (k >= side) continue;
        const int q = k / (2 * H), m = k - q * 2 * H;
        const int c = m < H ? m : m + 64;                  // extended column, 0 .. 64 + 2 H - 1
        const int x = pmod(x0 + c - H, nx), y = pmod(y0 + q - H, ny);
        const int xm = wrap1(x - 1, nx), xp = wrap1(x + 1, nx);
        const E* p0 = src + static_cast<int64_t>(y) * 9 * pitch;
        const E* pm = src + static_cast<int64_t>(wrap1(y - 1, ny)) * 9 * pitch;
        const E* pp = src + static_cast<int64_t>(wrap1(y + 1, ny)) * 9 * pitch;
        E v[9];
        v[0] = p0[x];
        v[1] = p0[pitch + xm];
        v[2] = pm[2 * pitch + x];
        v[3] = p0[3 * pitch + xp];
        v[4] = pp[4 * pitch + x];
        v[5] = pm[5 * pitch + xm];
        v[6] = pm[6 * pitch + xp];
        v[7] = pp[7 * pitch + xp];
        v[8] = pp[8 * pitch + xm];
        collide_stored<FORM, COLL, VAR, GM>(v, K);
        // window column c - 1 (+ v_x), window row q - 1 (+ v_y): the outer
        // ring's outward populations have no slot
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int a = q - 1 + kCy[i], b = c - 1 + kCx[i];
            if (a >= 0 && a < WH && b >= 0 && b < WW) win[(i * WH + a) * WW + b] = v[i];
        }
    }
    for (; r + 2 * NW < rows; r += 2 * NW) {
        load_row(r + NW, vb);
        row(r, va);
        load_row(r + 2 * NW, va);
        row(r + NW, vb);
    }
    if (r + NW < rows) {
        load_row(r + NW, vb);
        row(r, va);
        row(r + NW, vb);
    } else if (r < rows) {
        row(r, va);
    }
    stepn_rest<FORM, COLL, VAR, GM, T, TH, NW, NT, 2>(win, dst, nx, ny, pitch, x0, y0, th, lane, w, K);
}

// Waves per SIMD a four-step kernel is compiled for: what one workgroup needs,
// and for FP64's tile of eight waves what two workgroups per CU need: left
// alone KBC-B takes 132 registers, which leaves one (1024^2 18.5 us per step, 14.1
// with 128; KBC-A spills two registers for it).
template <int FORM, int GM, int NW>
constexpr int stepn_waves() {
    return FORM == F64 && NW == 8 && GM != GEXACT ? 4 : (NW + 3) / 4;
}

// Launch shapes of four steps: tile rows, waves per workgroup and store kind
// as one code, and the call of a launcher's at<TH, NW, NT>() for a code.
constexpr int step4_code(int rows, int waves, bool nt = true) { return rows | waves << 8 | (nt ? 1 << 16 : 0); }

// The shapes of many tiles per CU: the ones step4_shape (kbc_step4.hip)
// chooses for a collision.
template <int FORM, int COLL, int VAR, int GM, typename Launch>
int step4_many(int code, const Launch& l) {
    constexpr bool kFix = COLL == KBCC && GM == GFIX, kEst = COLL == KBCC && GM == GEST;
    constexpr bool kLight = COLL == LBGK || kFix;
    if constexpr (FORM == F32 && (kLight || kEst)) {
        switch (code) {
            case step4_code(12, 8): return l.template at<12, 8, true>();
            case step4_code(16, 8): return l.template at<16, 8, true>();
            case step4_code(20, 8): return l.template at<20, 8, true>();
            case step4_code(24, 8): return l.template at<24, 8, true>();
            case step4_code(28, 12): return l.template at<28, 12, true>();
            default: break;
        }
    }
    if constexpr (FORM == F32 && kLight)
        if (code == step4_code(12, 8, false)) return l.template at<12, 8, false>();
    if constexpr (FORM == F16 && kLight) {
        if (code == step4_code(24, 8)) return l.template at<24, 8, true>();
        if (code == step4_code(24, 8, false)) return l.template at<24, 8, false>();
    }
    if constexpr (FORM == F16 && kEst)
        if (code == step4_code(40, 12)) return l.template at<40, 12, true>();
    if constexpr (FORM == F64 && COLL == LBGK) {
        if (code == step4_code(12, 12)) return l.template at<12, 12, true>();
        if (code == step4_code(12, 12, false)) return l.template at<12, 12, false>();
    }
    if constexpr (FORM == F64 && (kFix || kEst))
        if (code == step4_code(12, 8)) return l.template at<12, 8, true>();
    if constexpr (FORM == F64 && kFix)
        if (code == step4_code(12, 8, false)) return l.template at<12, 8, false>();
    return -1;
}

// The shapes of at most one tile per CU, for every collision (FP64's exact
// stabiliser: the lowest only).
template <int FORM, int COLL, int VAR, int GM, typename Launch>
int step4_one(int code, const Launch& l) {
    if (code == step4_code(2, 10)) return l.template at<2, 10, true>();
    if constexpr (FORM != F64 || COLL != KBCC || GM != GEXACT) {
        constexpr int w = FORM == F64 ? 12 : 16;
        switch (code) {
            case step4_code(4, 12): return l.template at<4, 12, true>();
            case step4_code(8, 16): return l.template at<8, 16, true>();
            case step4_code(12, w): return l.template at<12, w, true>();
            case step4_code(16, w): return l.template at<16, w, true>();
            default: break;
        }
        if constexpr (FORM != F64)
            if (code == step4_code(28, 12)) return l.template at<28, 12, true>();
    }
    return -1;
}

}  // namespace kbc
