// kbc_ensemble4.hip -- an ensemble's members advanced by four fused steps per
// launch (tile body of the single lattice's four-step launch, kbc_tilen.hpp),
// where the shapes of many tiles per CU are faster than pairs of steps
// (step4_shape, over all members' tiles).  Tables, tile numbering and XCD bands
// as in kbc_ensemble.hip.  32 FP32 members of 128 .. 1024 nodes a side, 20
// steps: 1522 us in pairs, 1298 with four steps per launch.
#include "kbc_launch.hpp"
#include "kbc_tilen.hpp"

namespace kbc {

namespace {

// one workgroup per 64 x TH output tile
template <int FORM, int COLL, int VAR, int GM, int TH, int NW, bool NT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(stepn_waves<FORM, GM, NW>())))
void k_ens4(const EnsEntry* __restrict__ tab,
            const int32_t* __restrict__ tile_member, int ntiles, int per_xcd,
            int parity) {
    using F = Form<FORM>;
    using S = typename F::S;
    using R = typename F::R;
    const int b = blockIdx.x;
    const int t = (b & 7) * per_xcd + (b >> 3);
    if (t >= ntiles) return;   // the whole workgroup leaves together
    const EnsEntry& e = tab[tile_member[t]];
    const int lt = t - e.tile_start;
    stepn_tile<FORM, COLL, VAR, GM, 4, TH, NW, NT>(static_cast<const S*>(e.buf[parity]),
                                                   static_cast<S*>(e.buf[parity ^ 1]), e.nx, e.ny, e.pitch,
                                                   (lt % e.ntx) * 64, (lt / e.ntx) * TH, coef_of<R>(e));
}

// a.nsteps launches of four fused steps
template <int FORM, int COLL, int VAR, int GM>
struct Ens4Op {
    struct Launch {
        const EnsLaunch& a;
        template <int TH, int NW, bool NT>
        int at() const {
            const int per_xcd = (a.ntiles + 7) / 8;
            if (!grid_fits(8 * static_cast<int64_t>(per_xcd), 64 * NW)) return kTooLarge;
            for (int s = 0; s < a.nsteps; ++s) {
                k_ens4<FORM, COLL, VAR, GM, TH, NW, NT>
                    <<<dim3(8u * static_cast<unsigned>(per_xcd)), dim3(64 * NW), 0, a.stream>>>(
                        a.table, a.tile_member, a.ntiles, per_xcd, (a.parity + s) & 1);
                if (hipGetLastError() != hipSuccess) return -2;
            }
            return 0;
        }
    };
    static int run(const Lattice& L, const EnsLaunch& a) {
        (void)L;
        if (!a.tile_member) return -1;
        return step4_many<FORM, COLL, VAR, GM>(a.rows, Launch{a});
    }
};

}  // namespace

int launch_ensemble4(const Lattice& L, const EnsLaunch& a) { return dispatch<Ens4Op>(L, a); }

}  // namespace kbc
