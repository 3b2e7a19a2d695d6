// kbc_adjoint2.hip -- two adjoint steps per launch.
//
// A workgroup owns a 64 x TH tile of lambda^n.  Step n + 1 runs on the tile
// extended by one node on every side: each node y gathers f^{n+1} and
// lambda^{n+2} as the single adjoint step does and pushes population i of
// lambda^{n+1}(y) to where step n reads it, slot (i, y - v_i) of an LDS window
// over the tile (mu_i(x) = lambda_i(x + v_i)).  Step n then reads its nine mu
// from its own slots, gathers f^n and writes lambda^n.  lambda^{n+1} never goes
// to memory: 72 instead of 108 bytes per node and step in FP32, and one launch
// instead of two, for 9 (TH = 16) to 19 % (TH = 8) more derivatives in the
// ring.  The two bound the single step: memory on large lattices (0.93 of what
// a copy-like kernel reaches), launch and load latency on small ones.
// The per-node code and the values it reads are the single step's, so
// lambda^n is bitwise the same; dL/dbeta is summed per 64-node piece of a row,
// as the single step does for the same callers.
//
// On small lattices the launch also recomputes two (or one) of the next
// segment's states in further workgroups: two fused forward steps (step2_in)
// that write the state between them too.
//
// us per adjoint step of a rollout, recomputation included, single / paired:
// FP32 KBC-D 64^2 6.3 / 4.2, 256^2 5.6 / 4.8, 512^2 10.5 / 9.0, 2048^2 128 / 116,
// 4096^2 492 / 422; FP64 512^2 18.3 / 15.3, 2048^2 249 / 207; FP32 LBGK 4096^2 502 /
// 422.  On the large ones the states' traffic binds now: 126 bytes per node and
// step with the recomputation, at 5.0 TB/s.
#include "kbc_adjoint.hpp"
#include "kbc_launch.hpp"
#include "kbc_tile2.hpp"

namespace kbc {

namespace {

template <int FORM, int COLL, int VAR, int GM, bool FROZEN, int TH>
__device__ __forceinline__ void adj2_tile(typename Form<FORM>::R* __restrict__ winp,
                                          const typename Form<FORM>::S* __restrict__ state_b,
                                          const typename Form<FORM>::S* __restrict__ state_a,
                                          const typename Form<FORM>::R* __restrict__ lin,
                                          typename Form<FORM>::R* __restrict__ lout, int nx, int ny, int64_t pitch,
                                          int tx, int ty, int pieces, const Coef<typename Form<FORM>::R>& K,
                                          double* __restrict__ part_b, double* __restrict__ part_a) {
    using F = Form<FORM>;
    using R = typename F::R;
    using S = typename F::S;
    constexpr int TW = 64, EW = TW + 2;
    auto& win = *reinterpret_cast<R (*)[9][TH][EW]>(winp);   // slot (row r, column c): mu of output node (c - 1, r)
    const int x0 = tx * TW, y0 = ty * TH;
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int th = ny - y0 < TH ? ny - y0 : TH;               // rows of a ragged last tile

    const uint32_t gx = static_cast<uint32_t>(pmod(x0 + lane, nx));
    const uint32_t gm = gx == 0 ? static_cast<uint32_t>(nx - 1) : gx - 1;
    const uint32_t gp = gx == static_cast<uint32_t>(nx - 1) ? 0u : gx + 1;
    auto load_state = [&](const S* __restrict__ st, int y, R (&g)[9]) {
        const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
        const uint32_t s = sizeof(S);
        g[0] = F::dec(ld_at(row_ptr(st, y, 0, pitch), gx * s), 0);
        g[1] = F::dec(ld_at(row_ptr(st, y, 1, pitch), gm * s), 1);
        g[2] = F::dec(ld_at(row_ptr(st, ym, 2, pitch), gx * s), 2);
        g[3] = F::dec(ld_at(row_ptr(st, y, 3, pitch), gp * s), 3);
        g[4] = F::dec(ld_at(row_ptr(st, yp, 4, pitch), gx * s), 4);
        g[5] = F::dec(ld_at(row_ptr(st, ym, 5, pitch), gm * s), 5);
        g[6] = F::dec(ld_at(row_ptr(st, ym, 6, pitch), gp * s), 6);
        g[7] = F::dec(ld_at(row_ptr(st, yp, 7, pitch), gp * s), 7);
        g[8] = F::dec(ld_at(row_ptr(st, yp, 8, pitch), gm * s), 8);
    };
    auto piece_sum = [&](double* part, int y, R dbn) {
        const double s = wave_sum_d(x0 + lane < nx ? static_cast<double>(dbn) : 0.0);
        if (lane == 0) part[static_cast<int64_t>(y) * pieces + tx] = s;
    };

    // ---- step n + 1, the 64 interior columns of every extended row; the next
    // row's loads are in flight while a row is differentiated (held there: the
    // scheduler would sink them)
    auto load_both = [&](int ey, R (&g)[9], R (&mu)[9]) {
        const int y = wrap_uniform(y0 - 1 + ey, ny), ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
        load_state(state_b, y, g);
        const uint32_t r = sizeof(R);
        mu[0] = ld_at(row_ptr(lin, y, 0, pitch), gx * r);
        mu[1] = ld_at(row_ptr(lin, y, 1, pitch), gp * r);
        mu[2] = ld_at(row_ptr(lin, yp, 2, pitch), gx * r);
        mu[3] = ld_at(row_ptr(lin, y, 3, pitch), gm * r);
        mu[4] = ld_at(row_ptr(lin, ym, 4, pitch), gx * r);
        mu[5] = ld_at(row_ptr(lin, yp, 5, pitch), gp * r);
        mu[6] = ld_at(row_ptr(lin, yp, 6, pitch), gm * r);
        mu[7] = ld_at(row_ptr(lin, ym, 7, pitch), gm * r);
        mu[8] = ld_at(row_ptr(lin, ym, 8, pitch), gp * r);
    };
    auto row_b = [&](int ey, const R (&g)[9], const R (&mu)[9]) {
        R lam[9], dbn;
        collide_vjp<R, COLL, VAR, GM, FROZEN>(g, mu, K, lam, dbn);
        // node (lane, ey - 1) -> slot (lane - v_x + 1, ey - 1 - v_y)
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int q = ey - 1 - kCy[i];
            if (q >= 0 && q < TH) win[i][q][lane + 1 - kCx[i]] = lam[i];
        }
        if (ey >= 1 && ey <= th) piece_sum(part_b, y0 + ey - 1, dbn);
    };
    // FP64 has no registers for a second row (170 against 128, two waves per
    // SIMD instead of four)
    constexpr bool kAhead = FORM != F64;
    R ga[9], ma[9], gb[9], mb[9];
    if constexpr (!kAhead) {
        for (int ey = w; ey < th + 2; ey += 4) {
            load_both(ey, ga, ma);
            row_b(ey, ga, ma);
        }
    } else {
        int ey = w;
        const int end = th + 2;
        if (ey < end) load_both(ey, ga, ma);
        for (; ey + 4 < end; ey += 4) {
            load_both(ey + 4, gb, mb);
            __builtin_amdgcn_sched_barrier(0);
            row_b(ey, ga, ma);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                ga[i] = gb[i];
                ma[i] = mb[i];
            }
        }
        if (ey < end) row_b(ey, ga, ma);
    }
    // ---- and the two columns beside them
    if (w == 3) {
        for (int k = lane; k < 2 * (th + 2); k += 64) {
            const int side = k >= th + 2 ? 1 : 0, ey = k - side * (th + 2);
            const int x = pmod(side ? x0 + TW : x0 - 1, nx), y = pmod(y0 - 1 + ey, ny);
            R g[9], mu[9], lam[9], dbn;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int xm = wrap1(x - kCx[i], nx), ym = wrap1(y - kCy[i], ny);
                const int xp = wrap1(x + kCx[i], nx), yp = wrap1(y + kCy[i], ny);
                g[i] = F::dec(state_b[(static_cast<int64_t>(ym) * 9 + i) * pitch + xm], i);
                mu[i] = lin[(static_cast<int64_t>(yp) * 9 + i) * pitch + xp];
            }
            collide_vjp<R, COLL, VAR, GM, FROZEN>(g, mu, K, lam, dbn);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                if (kCx[i] != (side ? 1 : -1)) continue;      // the others leave the tile
                const int q = ey - 1 - kCy[i];
                if (q >= 0 && q < TH) win[i][q][side ? TW : 1] = lam[i];
            }
        }
    }
    // ---- step n on the tile, its state loaded a row ahead (the first row's
    // before the barrier)
    if (kAhead && w < th) load_state(state_a, y0 + w, ga);
    __syncthreads();
    for (int oy = w; oy < th; oy += 4) {
        const int y = y0 + oy;
        R lam[9], dbn;
        if constexpr (kAhead) {
            if (oy + 4 < th) load_state(state_a, y + 4, gb);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            load_state(state_a, y, ga);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) ma[i] = win[i][oy][lane + 1];
        collide_vjp<R, COLL, VAR, GM, FROZEN>(ga, ma, K, lam, dbn);
        if (x0 + lane < nx) {
            const uint32_t o = static_cast<uint32_t>(x0 + lane) * sizeof(R);
#pragma unroll
            for (int i = 0; i < 9; ++i) st_at<false>(row_ptr(lout, y, i, pitch), o, lam[i]);
        }
        piece_sum(part_a, y, dbn);
        if constexpr (kAhead) {
#pragma unroll
            for (int i = 0; i < 9; ++i) ga[i] = gb[i];
        }
    }
}

template <int FORM, int COLL, int VAR, int GM, bool FROZEN, int TH>
__global__ __launch_bounds__(256) void k_adj2(const typename Form<FORM>::S* __restrict__ state_b,
                                              const typename Form<FORM>::S* __restrict__ state_a,
                                              const typename Form<FORM>::R* __restrict__ lin,
                                              typename Form<FORM>::R* __restrict__ lout, int nx, int ny, int64_t pitch,
                                              int ntx, int nty, int per_xcd, Coef<typename Form<FORM>::R> K,
                                              double* __restrict__ part_b, double* __restrict__ part_a,
                                              const typename Form<FORM>::S* __restrict__ fsrc,
                                              typename Form<FORM>::S* __restrict__ fmid,
                                              typename Form<FORM>::S* __restrict__ fdst) {
    using S = typename Form<FORM>::S;
    using R = typename Form<FORM>::R;
    __shared__ R win[step2_values<TH>()];   // of either part: a workgroup runs one
    const unsigned nadj = 8u * static_cast<unsigned>(per_xcd);
    const unsigned b = blockIdx.x < nadj ? blockIdx.x : blockIdx.x - nadj;
    const int u = static_cast<int>(b & 7u) * per_xcd + static_cast<int>(b >> 3);
    if (u >= ntx * nty) return;   // the whole workgroup leaves together
    int tx, ty;
    panel_tile(u, ntx, nty, tx, ty);
    if (blockIdx.x < nadj) {
        adj2_tile<FORM, COLL, VAR, GM, FROZEN, TH>(win, state_b, state_a, lin, lout, nx, ny, pitch, tx, ty, ntx, K,
                                                   part_b, part_a);
    } else if (fmid) {
        step2_in<FORM, COLL, VAR, GM, TH, false, false, true>(reinterpret_cast<S*>(win), fsrc, fmid, fdst, nx, ny,
                                                              pitch, tx * 64, ty * TH, K, SlabHalo<S>{});
    } else {
        step_tile<FORM, COLL, VAR, GM, 1, TH / 4, false>(fsrc, fdst, nx, ny, pitch, tx, ty, K);
    }
}

template <int FORM, int COLL, int VAR, int GM>
struct AdjPairOp {
    template <bool FROZEN, int TH>
    static int launch(const Lattice& L, const void* state_b, const void* state_a, const void* lin, void* lout,
                      double* part_b, double* part_a, const void* fsrc, void* fmid, void* fdst) {
        using S = typename Form<FORM>::S;
        using R = typename Form<FORM>::R;
        const int ntx = adjoint_pieces(L), nty = (L.ny + TH - 1) / TH;
        const int64_t per_xcd = (static_cast<int64_t>(ntx) * nty + 7) / 8;
        const int64_t grid = 8 * per_xcd * (fsrc ? 2 : 1);
        if (!grid_fits(grid, 256)) return kTooLarge;
        k_adj2<FORM, COLL, VAR, GM, FROZEN, TH><<<dim3(static_cast<unsigned>(grid)), dim3(256), 0, L.stream>>>(
            static_cast<const S*>(state_b), static_cast<const S*>(state_a), static_cast<const R*>(lin),
            static_cast<R*>(lout), L.nx, L.ny, L.pitch, ntx, nty, static_cast<int>(per_xcd), make_coef<R>(L), part_b,
            part_a, static_cast<const S*>(fsrc), static_cast<S*>(fmid), static_cast<S*>(fdst));
        return hipGetLastError() == hipSuccess ? 0 : -2;
    }
    static int run(const Lattice& L, const void* state_b, const void* state_a, const void* lin, void* lout,
                   double* part_b, double* part_a, const void* fsrc, void* fmid, void* fdst) {
        if constexpr (COLL == KBCC && GM == GEXACT) {
            return -5;
        } else {
            // a held stabiliser differs for the estimate only
            if constexpr (COLL == KBCC && GM == GEST)
                if (L.adj_frozen) return rows<true>(L, state_b, state_a, lin, lout, part_b, part_a, fsrc, fmid, fdst);
            return rows<false>(L, state_b, state_a, lin, lout, part_b, part_a, fsrc, fmid, fdst);
        }
    }
    // 16-row tiles where there are enough of them (as the fused step; FP64 has
    // no room), 4-row tiles while they leave CUs idle: a wave's chain of rows
    // is the launch's time there
    template <bool FROZEN, typename... A>
    static int rows(const Lattice& L, A... a) {
        const int64_t cols = adjoint_pieces(L);
        if (cols * ((L.ny + 3) / 4) <= 256) return launch<FROZEN, 4>(L, a...);
        if constexpr (FORM != F64)
            if (cols * ((L.ny + 15) / 16) >= 1792) return launch<FROZEN, 16>(L, a...);
        return launch<FROZEN, 8>(L, a...);
    }
};

}  // namespace

// The exact stabiliser keeps single steps: its iteration makes the ring
// dearer than what the second launch costs.
bool adjoint_pairs(const Lattice& L) { return L.collision == LBGK || L.gamma_mode != GEXACT; }

int launch_adjoint_pair(const Lattice& L, const void* state_b, const void* state_a, const void* lin, void* lout,
                        double* partials, double* slice_b, double* slice_a, const void* fsrc, void* fmid, void* fdst) {
    const int64_t np = static_cast<int64_t>(adjoint_pieces(L)) * L.ny;
    const bool direct = adjoint_piece_partials(L) == 0;
    double* const pb = direct ? slice_b : partials;
    double* const pa = direct ? slice_a : partials + np;
    int rc = dispatch<AdjPairOp>(L, state_b, state_a, lin, lout, pb, pa, fsrc, fmid, fdst);
    if (rc || direct) return rc;
    rc = launch_fold_pieces(L, pb, slice_b);
    return rc ? rc : launch_fold_pieces(L, pa, slice_a);
}

}  // namespace kbc
