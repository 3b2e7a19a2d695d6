// kbc_aux.hip -- kernels around the step: initial state, moments, population
// import/export, diagnostics reductions and the bandwidth reference copy.
//
// All of them address the state the way the step does: the pre-collision
// population f_i(x, t = n) sits in population row i of lattice row y - v_iy,
// at column x - v_ix ([ny][9][pitch] layout).
#include "kbc_launch.hpp"
#include "kbc_tile2.hpp"

namespace kbc {

namespace {

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// element offset of f_i(x, y) in a state buffer
__device__ __forceinline__ int64_t src_off(int i, int x, int y, int nx, int ny, int64_t pitch) {
    const int xs = wrap(x - kCx[i], nx), ys = wrap(y - kCy[i], ny);
    return (static_cast<int64_t>(ys) * 9 + i) * pitch + xs;
}

// ------------------------------------------------------------ initial state
// Grad's approximation eq. (Grad) in deviation form:
//   f*_i - W_i rho0 = W_i [ (rho - rho0) + 3 rho (v.u)
//                           + 4.5 ( rho (v.u)^2 - rho |u|^2 / 3 + Pi1 : v v - tr(Pi1) / 3 ) ]
// with Pi1 = -(rho / (6 beta)) (grad u + grad u^T) (eq. P1AC, cs2 = 1/3); the
// equilibrium eq. (Eq) is the case Pi1 = 0.
template <int FORM>
__global__ __launch_bounds__(256) void k_init(typename Form<FORM>::S* __restrict__ dst, int nx, int ny,
                                              int64_t pitch, double rho0, double beta,
                                              const double* __restrict__ rho,
                                              const double* __restrict__ ux,
                                              const double* __restrict__ uy,
                                              const double* __restrict__ grad, int mode) {
    using F = Form<FORM>;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const int64_t N = static_cast<int64_t>(nx) * ny;
    const int64_t n = static_cast<int64_t>(y) * nx + x;
    const double r = rho ? rho[n] : rho0;
    const double u = ux[n], v = uy[n];
    double Pxx = 0.0, Pyy = 0.0, Pxy = 0.0;
    if (mode != 0) {
        double dxux, dyux, dxuy, dyuy;
        if (mode == 2) {
            dxux = grad[n];
            dyux = grad[N + n];
            dxuy = grad[2 * N + n];
            dyuy = grad[3 * N + n];
        } else {
            const int64_t xp = static_cast<int64_t>(y) * nx + wrap(x + 1, nx);
            const int64_t xm = static_cast<int64_t>(y) * nx + wrap(x - 1, nx);
            const int64_t yp = static_cast<int64_t>(wrap(y + 1, ny)) * nx + x;
            const int64_t ym = static_cast<int64_t>(wrap(y - 1, ny)) * nx + x;
            dxux = 0.5 * (ux[xp] - ux[xm]);
            dyux = 0.5 * (ux[yp] - ux[ym]);
            dxuy = 0.5 * (uy[xp] - uy[xm]);
            dyuy = 0.5 * (uy[yp] - uy[ym]);
        }
        const double k = -r / (6.0 * beta);
        Pxx = 2.0 * k * dxux;
        Pyy = 2.0 * k * dyuy;
        Pxy = k * (dyux + dxuy);
    }
    const double dr = r - rho0;
    const double u2 = u * u + v * v;
    const double tr3 = (Pxx + Pyy) / 3.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double cx = kCx[i], cy = kCy[i];
        const double cu = cx * u + cy * v;
        const double pvv = Pxx * cx * cx + 2.0 * Pxy * cx * cy + Pyy * cy * cy;
        const double dev = weight(i) * (dr + 3.0 * r * cu + 4.5 * (r * cu * cu - r * u2 / 3.0 + pvv - tr3));
        const int xs = wrap(x - kCx[i], nx), ys = wrap(y - kCy[i], ny);
        dst[(static_cast<int64_t>(ys) * 9 + i) * pitch + xs] = F::enc64(dev, i);
    }
}

// --------------------------------------------------------------- moments
template <int FORM, int COLL, int VAR, int GM>
__global__ __launch_bounds__(256) void k_moments(const typename Form<FORM>::S* __restrict__ src, int nx,
                                                 int ny, int64_t pitch,
                                                 Coef<typename Form<FORM>::R> K, double rho0,
                                                 double* __restrict__ rho, double* __restrict__ ux,
                                                 double* __restrict__ uy, double* __restrict__ gam) {
    using F = Form<FORM>;
    using R = typename F::R;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    typename F::S s[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) s[i] = src[src_off(i, x, y, nx, ny, pitch)];
    double dr = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double g = F::dec64(s[i], i);
        dr += g;
        jx += kCx[i] * g;
        jy += kCy[i] * g;
    }
    const int64_t n = static_cast<int64_t>(y) * nx + x;
    const double r = rho0 + dr;
    if (rho) rho[n] = r;
    if (ux) ux[n] = jx / r;
    if (uy) uy[n] = jy / r;
    if (gam) {
        R g[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = F::dec(s[i], i);
        gam[n] = static_cast<double>(collide<R, COLL, VAR, GM>(g, K));
    }
}

// ------------------------------------------------------- population import/export
template <int FORM>
__global__ __launch_bounds__(256) void k_get_pop(const typename Form<FORM>::S* __restrict__ src, int nx,
                                                 int ny, int64_t pitch, double rho0,
                                                 double* __restrict__ f) {
    using F = Form<FORM>;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const int64_t N = static_cast<int64_t>(nx) * ny;
    const int64_t n = static_cast<int64_t>(y) * nx + x;
#pragma unroll
    for (int i = 0; i < 9; ++i)
        f[i * N + n] = F::dec64(src[src_off(i, x, y, nx, ny, pitch)], i) + weight(i) * rho0;
}

template <int FORM>
__global__ __launch_bounds__(256) void k_set_pop(typename Form<FORM>::S* __restrict__ dst, int nx, int ny,
                                                 int64_t pitch, double rho0,
                                                 const double* __restrict__ f) {
    using F = Form<FORM>;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const int64_t N = static_cast<int64_t>(nx) * ny;
    const int64_t n = static_cast<int64_t>(y) * nx + x;
#pragma unroll
    for (int i = 0; i < 9; ++i)
        dst[src_off(i, x, y, nx, ny, pitch)] = F::enc64(f[i * N + n] - weight(i) * rho0, i);
}

// ----------------------------------------------------------- diagnostics
// Slots of the per-block partials.
enum {
    D_RHO = 0, D_JX, D_JY, D_E, D_E2, D_S, D_G, D_G2, D_NONFIN, D_FEQNEG, D_RHO2,
    D_Z, D_Z2, D_P, D_P2, D_UNUSED
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum `cnt` per-thread values across the 256-thread block and store them at
// partials[blockIdx.x * kDiagSlots + first + k].
template <int CNT>
__device__ __forceinline__ void block_store(double (&acc)[CNT], double* partials, int first) {
    __shared__ double red[4][CNT];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
        const double s = wave_sum(acc[k]);
        if (lane == 0) red[wv][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < CNT) {
        const int k = threadIdx.x;
        partials[static_cast<int64_t>(blockIdx.x) * kDiagSlots + first + k] =
            (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    }
}

// u = j / r to within an ulp: one refined reciprocal of the density and a
// correction step per component (11 instructions); the library division, 11
// instructions each, where the density is too small or large for that (or not
// finite).
__device__ __forceinline__ void velocity(double jx, double jy, double r, double& u, double& v) {
    const double ar = fabs(r);
    if (ar > 1e-150 && ar < 1e150) {
        const double ir = rcpR(r), a = jx * ir, b = jy * ir;
        u = fmaR(fmaR(-r, a, jx), ir, a);
        v = fmaR(fmaR(-r, b, jy), ir, b);
    } else {
        u = jx / r;
        v = jy / r;
    }
}

// All statistics of the state in one pass.  Bound by FP64 vector issue (about
// 600 instructions per node, 200 of them the nine logarithms); the state is
// read once (1.3 times through L2) and nothing but the sums is written.
//
// A workgroup takes 64 x TH tiles of its XCD's band in turn.  The
// vorticity at a node needs the velocity one node away and the palinstrophy
// the vorticity one node away, so the velocity is formed on the tile extended
// by two nodes on every side and the vorticity on one, both kept in LDS; the
// previous three passes instead wrote and re-read both fields in memory
// (2048^2 FP32 KBC-D: 228 us for the call, 99 with one pass).  Rows of 64 nodes
// are one wave each (uniform row, scalar bases); the four columns beside the
// tile are lanes of their own.
template <int FORM, int COLL, int VAR, int GM, int TH>
__global__ __launch_bounds__(256) void k_diag(const typename Form<FORM>::S* __restrict__ src, int nx, int ny,
                                              int64_t pitch, Coef<typename Form<FORM>::R> K, double rho0, int ntx,
                                              int ntiles, double* __restrict__ partials) {
    using F = Form<FORM>;
    using R = typename F::R;
    using S = typename F::S;
    constexpr int TW = 64, EW = TW + 4, EH = TH + 4;
    __shared__ double su[EH][EW], sv[EH][EW], sw[TH + 2][TW + 2];
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    double acc[15] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    const int per_xcd = (ntiles + 7) >> 3, nwg = static_cast<int>(gridDim.x >> 3);
    const int band0 = static_cast<int>(blockIdx.x & 7u) * per_xcd;
    const int band1 = (band0 + per_xcd < ntiles) ? band0 + per_xcd : ntiles;
    for (int t = band0 + static_cast<int>(blockIdx.x >> 3); t < band1; t += nwg) {
        const int ty = t / ntx;
        const int x0 = (t - ty * ntx) * TW, y0 = ty * TH;
        // velocity on the extended tile; the other sums on the tile's own nodes
        const int gx = pmod(x0 + lane, nx);
        const int gxm = gx == 0 ? nx - 1 : gx - 1, gxp = gx == nx - 1 ? 0 : gx + 1;
        for (int ey = w; ey < EH; ey += 4) {
            const int yy = y0 - 2 + ey;
            const int y = wrap_uniform(yy, ny), ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
            const uint32_t c0 = static_cast<uint32_t>(gx) * sizeof(S), cm = static_cast<uint32_t>(gxm) * sizeof(S),
                           cp = static_cast<uint32_t>(gxp) * sizeof(S);
            S s[9];
            s[0] = ld_at(row_ptr(src, y, 0, pitch), c0);
            s[1] = ld_at(row_ptr(src, y, 1, pitch), cm);
            s[2] = ld_at(row_ptr(src, ym, 2, pitch), c0);
            s[3] = ld_at(row_ptr(src, y, 3, pitch), cp);
            s[4] = ld_at(row_ptr(src, yp, 4, pitch), c0);
            s[5] = ld_at(row_ptr(src, ym, 5, pitch), cm);
            s[6] = ld_at(row_ptr(src, ym, 6, pitch), cp);
            s[7] = ld_at(row_ptr(src, yp, 7, pitch), cp);
            s[8] = ld_at(row_ptr(src, yp, 8, pitch), cm);
            double q[9], dr = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                q[i] = F::dec64(s[i], i);
                dr += q[i];
                if (kCx[i]) jx += kCx[i] * q[i];
                if (kCy[i]) jy += kCy[i] * q[i];
            }
            const double r = rho0 + dr;
            double u, v;
            velocity(jx, jy, r, u, v);
            su[ey][lane + 2] = u;
            sv[ey][lane + 2] = v;
            if (ey < 2 || ey >= TH + 2 || yy >= ny || x0 + lane >= nx) continue;
            const double u2 = u * u + v * v;
            // entropy -sum f ln(f / W), with ln(f / W) = 2 atanh of (f - W) / (f + W)
            // (17 FP64 instructions, against about 100 for the library logarithm
            // and 11 for the division f / W; and as f - W is formed from the
            // stored deviation, no digits of a small one are lost): the general form where a population is
            // beyond a factor two of its weight (or not finite: then dr is not)
            double Sn = 0.0, zmax = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const double num = q[i] + weight(i) * (rho0 - 1.0), den = q[i] + weight(i) * (rho0 + 1.0);
                const double a = num * rcpR(den), z = a * a;
                zmax = fmax(zmax, z);
                Sn = fmaR(q[i] + weight(i) * rho0, -2.0 * a * atanh_poly(z), Sn);
            }
            const bool sum_finite = isfinite(dr);
            bool finite = true;
            if (!(sum_finite && zmax <= 1.0 / 9.0)) {
                Sn = 0.0;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const double f = q[i] + weight(i) * rho0;
                    finite = finite && isfinite(f);
                    Sn -= f * log(f / weight(i));
                }
            }
            // some feq_i <= 0 (or NaN): none where rho > 0 and |u|^2 < 1/6,
            // as 1 + e_i >= 1/2 - 1.5 |u|^2
            bool neg = false;
            if (!(r > 0.0 && u2 < 1.0 / 6.0)) {
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const double cu = kCx[i] * u + kCy[i] * v;
                    const double feq = weight(i) * r * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * u2);
                    neg = neg || !(feq > 0.0);
                }
            }
            R g[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) g[i] = F::dec(s[i], i);
            const double gm = static_cast<double>(collide<R, COLL, VAR, GM>(g, K));
            const double e = 0.5 * u2;
            acc[0] += r;
            acc[1] += jx;
            acc[2] += jy;
            acc[3] += e;
            acc[4] = fmaR(e, e, acc[4]);
            acc[5] += Sn;
            acc[6] += gm;
            acc[7] = fmaR(gm, gm, acc[7]);
            acc[8] += finite ? 0.0 : 1.0;
            acc[9] += neg ? 1.0 : 0.0;
            acc[10] = fmaR(r, r, acc[10]);
        }
        // the two columns on each side
        for (int k = static_cast<int>(threadIdx.x); k < 4 * EH; k += 256) {
            const int ey = k >> 2, c = k & 3;
            const int ex = c < 2 ? c : TW + c;
            const int x = pmod(x0 - 2 + ex, nx), y = pmod(y0 - 2 + ey, ny);
            double dr = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const double q = F::dec64(src[src_off(i, x, y, nx, ny, pitch)], i);
                dr += q;
                if (kCx[i]) jx += kCx[i] * q;
                if (kCy[i]) jy += kCy[i] * q;
            }
            velocity(jx, jy, rho0 + dr, su[ey][ex], sv[ey][ex]);
        }
        __syncthreads();
        // vorticity on the tile and one node around it
        for (int k = static_cast<int>(threadIdx.x); k < (TH + 2) * (TW + 2); k += 256) {
            const int r = k / (TW + 2), c = k - r * (TW + 2);
            sw[r][c] = 0.5 * (sv[r + 1][c + 2] - sv[r + 1][c]) - 0.5 * (su[r + 2][c + 1] - su[r][c + 1]);
        }
        __syncthreads();
        for (int oy = w; oy < TH; oy += 4) {
            if (y0 + oy >= ny || x0 + lane >= nx) continue;
            const double om = sw[oy + 1][lane + 1];
            const double z = 0.5 * om * om;
            const double hx = 0.5 * (sw[oy + 1][lane + 2] - sw[oy + 1][lane]);
            const double hy = 0.5 * (sw[oy + 2][lane + 1] - sw[oy][lane + 1]);
            const double p = 0.5 * (hx * hx + hy * hy);
            acc[11] += z;
            acc[12] = fmaR(z, z, acc[12]);
            acc[13] += p;
            acc[14] = fmaR(p, p, acc[14]);
        }
        // the next tile writes su, sv after every wave is past the vorticity
        // (the barrier above) and sw after the next tile's first barrier
    }
    block_store<15>(acc, partials, 0);
}

// out[k] = sum over the kDiagBlocks partials of slot k, in a fixed order: one
// workgroup of kDiagSlots threads per group of blocks, then across the groups
__global__ __launch_bounds__(1024) void k_diag_sum(const double* __restrict__ partials, double* __restrict__ out) {
    constexpr int kGroups = 1024 / kDiagSlots;
    __shared__ double red[kGroups][kDiagSlots];
    const int k = static_cast<int>(threadIdx.x) % kDiagSlots, g = static_cast<int>(threadIdx.x) / kDiagSlots;
    double s = 0.0;
    for (int b = g; k != D_UNUSED && b < kDiagBlocks; b += kGroups) s += partials[static_cast<int64_t>(b) * kDiagSlots + k];
    red[g][k] = s;
    __syncthreads();
    if (g == 0) {
        double t = 0.0;
        for (int j = 0; j < kGroups; ++j) t += red[j][k];
        out[k] = t;
    }
}

// ------------------------------------------------------------ copy reference
// The plainest streaming copy: one 4-byte word per lane, one pass, the same
// access granularity as the step kernel's loads and stores.  It is the
// reference both for achievable bandwidth and for scaling the HBM byte
// counters of the profiler.
__global__ __launch_bounds__(256) void k_copy(float* __restrict__ dst, const float* __restrict__ src, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

dim3 node_grid(const Lattice& L) {
    return dim3(static_cast<unsigned>((L.nx + 63) / 64), static_cast<unsigned>((L.ny + 3) / 4));
}

int ok_launch() { return hipGetLastError() == hipSuccess ? 0 : -2; }

template <int FORM, int COLL, int VAR, int GM>
struct MomOp {
    static int run(const Lattice& L, const void* src, double* rho, double* ux, double* uy, double* g) {
        using F = Form<FORM>;
        k_moments<FORM, COLL, VAR, GM><<<node_grid(L), dim3(64, 4), 0, L.stream>>>(
            static_cast<const typename F::S*>(src), L.nx, L.ny, L.pitch, make_coef<typename F::R>(L),
            L.rho0, rho, ux, uy, g);
        return ok_launch();
    }
};

template <int FORM, int COLL, int VAR, int GM>
struct DiagOp {
    template <int TH>
    static int go(const Lattice& L, const void* src, double* partials) {
        using F = Form<FORM>;
        const int ntx = (L.nx + 63) / 64;
        const int64_t ntiles = static_cast<int64_t>(ntx) * ((L.ny + TH - 1) / TH);
        if (ntiles > kMaxDiagTiles) return kTooLarge;
        k_diag<FORM, COLL, VAR, GM, TH><<<kDiagBlocks, 256, 0, L.stream>>>(
            static_cast<const typename F::S*>(src), L.nx, L.ny, L.pitch, make_coef<typename F::R>(L), L.rho0, ntx,
            static_cast<int>(ntiles), partials);
        return ok_launch();
    }
    // 16-row tiles (a quarter more velocities than nodes) where they give
    // every workgroup of the grid one; 8-row tiles below that, where the
    // length of a workgroup's row loop is the time
    static int run(const Lattice& L, const void* src, double* partials, double* out) {
        const int64_t tiles16 = static_cast<int64_t>((L.nx + 63) / 64) * ((L.ny + 15) / 16);
        const int rc = tiles16 >= kDiagBlocks ? go<16>(L, src, partials) : go<8>(L, src, partials);
        if (rc) return rc;
        k_diag_sum<<<1, 1024, 0, L.stream>>>(partials, out);
        return ok_launch();
    }
};

}  // namespace

int launch_init(const Lattice& L, void* dst, const double* rho, const double* ux, const double* uy,
                const double* grad, int mode) {
    const dim3 g = node_grid(L), b(64, 4);
    switch (L.form) {
        case F16: k_init<F16><<<g, b, 0, L.stream>>>(static_cast<_Float16*>(dst), L.nx, L.ny, L.pitch, L.rho0, L.beta, rho, ux, uy, grad, mode); break;
        case F32: k_init<F32><<<g, b, 0, L.stream>>>(static_cast<float*>(dst), L.nx, L.ny, L.pitch, L.rho0, L.beta, rho, ux, uy, grad, mode); break;
        case F64: k_init<F64><<<g, b, 0, L.stream>>>(static_cast<double*>(dst), L.nx, L.ny, L.pitch, L.rho0, L.beta, rho, ux, uy, grad, mode); break;
        default: return -1;
    }
    return ok_launch();
}

int launch_moments(const Lattice& L, const void* src, double* rho, double* ux, double* uy, double* gamma) {
    return dispatch<MomOp>(L, src, rho, ux, uy, gamma);
}

int launch_get_pop(const Lattice& L, const void* src, double* f) {
    const dim3 g = node_grid(L), b(64, 4);
    switch (L.form) {
        case F16: k_get_pop<F16><<<g, b, 0, L.stream>>>(static_cast<const _Float16*>(src), L.nx, L.ny, L.pitch, L.rho0, f); break;
        case F32: k_get_pop<F32><<<g, b, 0, L.stream>>>(static_cast<const float*>(src), L.nx, L.ny, L.pitch, L.rho0, f); break;
        case F64: k_get_pop<F64><<<g, b, 0, L.stream>>>(static_cast<const double*>(src), L.nx, L.ny, L.pitch, L.rho0, f); break;
        default: return -1;
    }
    return ok_launch();
}

int launch_set_pop(const Lattice& L, void* dst, const double* f) {
    const dim3 g = node_grid(L), b(64, 4);
    switch (L.form) {
        case F16: k_set_pop<F16><<<g, b, 0, L.stream>>>(static_cast<_Float16*>(dst), L.nx, L.ny, L.pitch, L.rho0, f); break;
        case F32: k_set_pop<F32><<<g, b, 0, L.stream>>>(static_cast<float*>(dst), L.nx, L.ny, L.pitch, L.rho0, f); break;
        case F64: k_set_pop<F64><<<g, b, 0, L.stream>>>(static_cast<double*>(dst), L.nx, L.ny, L.pitch, L.rho0, f); break;
        default: return -1;
    }
    return ok_launch();
}

int launch_diag(const Lattice& L, const void* src, double* partials, double* out) {
    return dispatch<DiagOp>(L, src, partials, out);
}

int launch_copy(void* dst, const void* src, size_t n_words, hipStream_t stream) {
    const int64_t n = static_cast<int64_t>(n_words);
    if (n == 0) return 0;
    const int64_t blocks = (n + 255) / 256;
    if (!grid_fits(blocks, 256)) return kTooLarge;
    k_copy<<<static_cast<unsigned>(blocks), 256, 0, stream>>>(static_cast<float*>(dst), static_cast<const float*>(src), n);
    return ok_launch();
}

}  // namespace kbc
