// kbc_step4.hip -- four fused time steps per launch on a single lattice; the
// tile body is stepn_tile (kbc_tilen.hpp).
//
// Where four steps pay against two (step4_shape):
//
//   * Small lattices, at most one tile per CU.  There a launch is a chain of
//     latencies (about 2.4 us for the launch itself, then the loads, then one
//     collision after another), and the arithmetic repeated in the tiles'
//     margins costs nothing while CUs are idle.  The smallest tile height that
//     still gives every CU at most one tile is taken, with enough waves that
//     each has one row or two per step.  us per step, two / four steps per
//     launch: FP32 KBC-B 64^2 2.55 / 1.27, 256^2 2.74 / 1.51, 320^2 2.86 / 1.85,
//     384^2 3.48 / 2.23, 512^2 3.64 / 2.67, 640^2 4.60 / 4.12; FP64 64^2 3.14 /
//     1.70, 512^2 5.31 / 4.44; FP16 512^2 3.80 / 3.03; exact stabiliser FP32
//     512^2 9.03 / 6.94.
//   * Lattices bound by memory at two steps per launch: LBGK and the fixed
//     stabiliser in every form, and FP32 KBC beyond the last-level cache.  Four
//     steps halve the traffic for a quarter more collisions in the margins.
//     FP32 LBGK 4096^2 118 / 71.5 us, 1024^2 (plain stores) 7.15 / 5.57; FP64
//     LBGK 2048^2 58.5 / 43.0; FP16 LBGK 3072^2 46.0 / 40.4; FP32 KBC-B
//     4096^2 123 / 109.5.
//
// Two steps stay where arithmetic binds: FP16 and FP64 KBC and the exact
// stabiliser beyond one tile per CU (FP16 KBC-B 3072^2 61.1 / 67.9 us, FP64
// 138 / 140, exact 150 / 168), and FP32 KBC inside the last-level cache (1536^2
// 17.5 / 17.7).
#include "kbc_launch.hpp"
#include "kbc_tilen.hpp"

namespace kbc {

namespace {

// at most one tile per CU: 256 CUs
constexpr int64_t kCus = 256;
// Shapes of many tiles per CU are numbered apart from the heights of one
constexpr int kManyTiles = 64;

int64_t tiles_of(const Lattice& L, int rows) {
    return static_cast<int64_t>((L.nx + 63) / 64) * ((L.ny + rows - 1) / rows);
}

template <int FORM, int COLL, int VAR, int GM, int TH, int NW, bool NT>
__global__ __launch_bounds__(64 * NW) void k_step4(const typename Form<FORM>::S* __restrict__ src,
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
    static int run(const Lattice& L, const void* src, void* dst, int shape, int nt) {
        constexpr bool kWide = FORM == F64;   // FP64: taller windows leave room for fewer waves' registers
        constexpr bool kLight = COLL == LBGK || GM == GFIX;
        switch (shape) {
            case 2: return go<2, 10, true>(L, src, dst);
            case 4: return go<4, 12, true>(L, src, dst);
            case 8: return go<8, 16, true>(L, src, dst);
            case 12: return go<12, kWide ? 12 : 16, true>(L, src, dst);
            case 16: return go<16, kWide ? 12 : 16, true>(L, src, dst);
            case 28:
                if constexpr (FORM != F64) return go<28, 12, true>(L, src, dst);
                return -1;
            case kManyTiles + 12:
                if constexpr (kLight && FORM == F64)
                    return nt ? go<12, 8, true>(L, src, dst) : go<12, 8, false>(L, src, dst);
                if constexpr (kLight && FORM == F32) return go<12, 8, false>(L, src, dst);
                return -1;
            case kManyTiles + 24:
                if constexpr (FORM == F32 && kLight) return go<24, 12, true>(L, src, dst);
                if constexpr (FORM == F32 && COLL == KBCC && GM == GEST) return go<24, 8, true>(L, src, dst);
                if constexpr (FORM == F16 && kLight)
                    return nt ? go<24, 8, true>(L, src, dst) : go<24, 8, false>(L, src, dst);
                return -1;
            default: return -1;
        }
    }
};

}  // namespace

int step4_shape(const Lattice& L, int nt) {
    if (L.halo_lo) return 0;   // a slab's halo holds the rows for two steps
    // small lattices (their default store kind is non-temporal: the other,
    // set by the caller, keeps two steps)
    if (nt) {
        for (int rows : {2, 4, 8, 12, 16, 28})
            if (tiles_of(L, rows) <= kCus && (rows != 28 || L.form != F64) && (rows != 2 || tiles_of(L, 2) <= kCus / 2))
                return rows;
    }
    const bool light = L.collision == LBGK || L.gamma_mode == GFIX;
    if (light) {
        if (L.form == F64) return kManyTiles + 12;
        if (L.form == F16) return kManyTiles + 24;
        return kManyTiles + (nt ? 24 : 12);
    }
    // FP32 KBC: where both state buffers outgrow the 256 MiB last-level cache
    const double state_bytes = 2.0 * 9.0 * 4.0 * static_cast<double>(L.pitch) * L.ny;
    if (L.form == F32 && L.gamma_mode == GEST && nt && state_bytes > 256.0 * 1024.0 * 1024.0) return kManyTiles + 24;
    return 0;
}

int launch_step4(const Lattice& L, const void* src, void* dst, int shape, int nt) {
    return dispatch<Step4Op>(L, src, dst, shape, nt);
}

}  // namespace kbc
