// kbc_step4.hip -- four fused time steps per launch on a single lattice; the
// tile body is stepn_tile (kbc_tilen.hpp).
//
// Where four steps pay against two (step4_shape), us per step with two / four
// steps per launch (of calls that are whole groups of eight; a call's other steps
// run as pairs):
//
//   * Small lattices, at most one tile per CU.  There a launch is a chain of
//     latencies (about 2.4 us for the launch itself, then the loads, then one
//     collision after another), and the arithmetic repeated in the tiles'
//     margins costs nothing while CUs are idle.  The smallest tile height that
//     still gives every CU at most one tile is taken, with enough waves that
//     each has one row or two per step.  FP32 KBC-B 64^2 2.59 / 1.32, 256^2 2.73 /
//     1.52, 320^2 2.82 / 1.85, 384^2 3.46 / 2.15, 512^2 3.58 / 2.61, 640^2 4.52 /
//     3.78; FP64 64^2 3.13 / 1.69, 512^2 5.00 / 4.19; FP16 512^2 3.61 / 2.61;
//     FP32 LBGK 512^2 2.77 / 1.70; exact stabiliser FP32 128^2 12.0 / 5.4.
//   * Larger ones that memory binds at two steps: LBGK and the fixed
//     stabiliser in every form, FP32 and FP64 KBC, FP16 KBC beyond the
//     last-level cache.  Four steps halve the traffic for a quarter more
//     collisions in the margins.  FP32 LBGK 4096^2 117 / 62, FP64 LBGK 2048^2
//     55.4 / 34.3, FP16 LBGK 3072^2 41.9 / 28.9; FP32 KBC-B 8192^2 450 / 364,
//     4096^2 115 / 92, 1280^2 12.0 / 11.3, 1024^2 8.2 / 7.7; FP64 KBC-B 3072^2 134 /
//     110, 1024^2 14.9 / 13.4; FP16 KBC-B 4096^2 91 / 86.
//
// Two steps stay where arithmetic binds: FP16 KBC inside the last-level cache
// (1536^2 16.1 / 16.2), the exact stabiliser beyond one tile per CU (1024^2
// 15.0 / 16.7) and in FP64 beyond the two-row tiles (64^2 19 / 13, 300 x 217
// 18 / 23, 512^2 29 / 33).  FP64's exact two-row kernel is held to the 168
// registers of its ten waves and spills 65 (KBC-D) to 165 (KBC-A) more.
#include "kbc_launch.hpp"
#include "kbc_tilen.hpp"

namespace kbc {

namespace {

constexpr int64_t kCus = 256;

// Wave tasks of one tile: its rows and packed margin nodes over four steps.
constexpr int tasks_of(int rows) {
    int n = rows;
    for (int h = 1; h <= 3; ++h) n += rows + 2 * h + (2 * h * (rows + 2 * h) + 63) / 64;
    return n;
}

template <int FORM, int COLL, int VAR, int GM, int TH, int NW, bool NT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(stepn_waves<FORM, GM, NW>())))
void k_step4(const typename Form<FORM>::S* __restrict__ src,
             typename Form<FORM>::S* __restrict__ dst, int nx, int ny,
             int64_t pitch, int ntx, int nty, int per_xcd,
             Coef<typename Form<FORM>::R> K) {
    const int b = blockIdx.x;
    const int u = (b & 7) * per_xcd + (b >> 3);
    if (u >= ntx * nty) return;   // the whole workgroup leaves together
    int tx, ty;
    panel_tile(u, ntx, nty, tx, ty);
    stepn_tile<FORM, COLL, VAR, GM, 4, TH, NW, NT>(src, dst, nx, ny, pitch, tx * 64, ty * TH, K);
}

template <int FORM, int COLL, int VAR, int GM>
struct Step4Op {
    template <int TH, int NW, bool NT>
    static int go(const Lattice& L, const void* src, void* dst) {
        using F = Form<FORM>;
        using S = typename F::S;
        static_assert(stepn_lds<FORM, 4, TH>() <= 160u * 1024u, "the window must fit the LDS of a CU");
        const int ntx = (L.nx + 63) / 64;
        const int nty = (L.ny + TH - 1) / TH;
        const int64_t per_xcd64 = (static_cast<int64_t>(ntx) * nty + 7) / 8;
        if (!grid_fits(8 * per_xcd64, 64 * NW)) return kTooLarge;
        const int per_xcd = static_cast<int>(per_xcd64);
        k_step4<FORM, COLL, VAR, GM, TH, NW, NT><<<dim3(8u * per_xcd), dim3(64 * NW), 0, L.stream>>>(
            static_cast<const S*>(src), static_cast<S*>(dst), L.nx, L.ny, L.pitch, ntx, nty, per_xcd,
            make_coef<typename F::R>(L));
        return hipGetLastError() == hipSuccess ? 0 : -2;
    }
    // called by step4_one / step4_many for the launch's shape
    struct Launch {
        const Lattice& L;
        const void* src;
        void* dst;
        template <int TH, int NW, bool NT>
        int at() const {
            return go<TH, NW, NT>(L, src, dst);
        }
    };
    static int run(const Lattice& L, const void* src, void* dst, int sh) {
        const int rc = step4_one<FORM, COLL, VAR, GM>(sh, Launch{L, src, dst});
        return rc == -1 ? step4_many<FORM, COLL, VAR, GM>(sh, Launch{L, src, dst}) : rc;
    }
};

}  // namespace

int step4_shape(const Lattice& L, const int32_t* sizes, int count, double state_bytes, int nt, bool one_per_cu) {
    if (L.halo_lo) return 0;   // a slab's halo holds the rows for two steps
    auto tiles = [&](int rows) {
        int64_t n = 0;
        for (int k = 0; k < count; ++k)
            n += static_cast<int64_t>((sizes[2 * k] + 63) / 64) * ((sizes[2 * k + 1] + rows - 1) / rows);
        return n;
    };
    // a very wide, flat lattice can need more work-items than a dispatch holds
    // where tiles of two steps (four waves) do not: 2^28 x 25 FP16 LBGK
    auto shape = [&](int rows, int waves, bool store_nt = true) {
        return grid_fits(8 * ((tiles(rows) + 7) / 8), 64 * waves) ? step4_code(rows, waves, store_nt) : 0;
    };
    // one tile per CU (an ensemble's launches are built for many).  Two rows only up to half of that: a tile's six margin
    // rows weigh most there (192^2 with 288 such tiles 1.82, with four rows
    // 1.44).  FP64 has room for fewer waves' registers, and not for 28 rows.
    const bool f64 = L.form == F64, exact = L.collision != LBGK && L.gamma_mode == GEXACT;
    if (one_per_cu) {
        if (tiles(2) <= kCus / 2) return shape(2, 10);
        if (f64 && exact) return 0;
        if (tiles(4) <= kCus) return shape(4, 12);
        if (tiles(8) <= kCus) return shape(8, 16);
        if (tiles(12) <= kCus) return shape(12, f64 ? 12 : 16);
        if (tiles(16) <= kCus) return shape(16, f64 ? 12 : 16);
        if (!f64 && tiles(28) <= kCus) return shape(28, 12);
    } else if (tiles(16) <= kCus) {
        return 0;
    }
    // many tiles per CU.  Plain stores matter to the light collisions only,
    // which the last-level cache feeds (FP32 LBGK 1280^2: plain 7.1, others
    // 8.6); KBC measures the same or 1 % better with non-temporal ones.
    if (exact) return 0;
    const bool light = L.collision == LBGK || L.gamma_mode == GFIX;
    if (f64) return L.collision == LBGK ? shape(12, 12, nt != 0) : shape(12, 8, !light || nt != 0);
    if (L.form == F16) {
        if (light) return shape(24, 8, nt != 0);
        // (40 rows 93, 32 rows 95, 24 rows 97 us per step at 4096^2)
        return state_bytes > 256.0 * 1024.0 * 1024.0 ? shape(40, 12) : 0;
    }
    if (light && !nt) return shape(12, 8, false);
    // FP32: the height whose busiest CU has the least to do.  The order this
    // gives is the measured one on 1200^2, 900 x 1500, 800^2, 1024^2, 1536^2,
    // 1921 x 1083, 2600 x 700, 640 x 1500, 2048^2 and 4096^2 (1200^2: 24, 16, 20,
    // 28 rows 11.6, 11.8, 12.0, 12.1)
    int best_rows = 0;
    int64_t best_cost = 0;
    for (int rows : {28, 24, 20, 16, 12}) {
        const int64_t cost = ((tiles(rows) + kCus - 1) / kCus) * tasks_of(rows);
        if (!best_rows || cost < best_cost) {
            best_cost = cost;
            best_rows = rows;
        }
    }
    return best_rows == 28 ? shape(28, 12) : shape(best_rows, 8);
}

int launch_step4(const Lattice& L, const void* src, void* dst, int shape) {
    return dispatch<Step4Op>(L, src, dst, shape);
}

}  // namespace kbc
