// kbc_spectra.hip -- shell-summed kinetic-energy and enstrophy spectra of a
// square periodic lattice (turbulence statistics of section "Decaying
// Two-Dimensional Turbulence").
//
// With u_hat the unnormalised discrete Fourier transform of a velocity
// component on N x N nodes, Parseval gives <|u|^2> = sum_k |u_hat(k)|^2 / N^4,
// so E = (1/2) <|u|^2> splits over wavevectors k (integers, |k_a| <= N/2) as
// e(k) = (|ux_hat|^2 + |uy_hat|^2) / (2 N^4).  E(k) sums e over the shell
// round(|k|) = k; Z(k) sums e(k) (2 pi |k| / N)^2, the spectral enstrophy
// (1/2) <omega^2> with the exact derivative.  Shells above kmax are dropped.
//
// The transform is real-to-complex, so the stored half plane 0 <= k_x <= N/2
// counts twice except the columns k_x = 0 and k_x = N/2 (N even).  Both
// components go through one batched plan, in place on padded rows: half the
// launches and half the scratch of two separate out-of-place transforms.  (One
// complex transform of ux + i uy takes the same time, but its plan takes twice
// as long to make and three times as long to destroy.)
//
// The shell sums are bound by reading the transforms once.  A workgroup takes
// 256 values of k_x by kRows of |k_y|, adds the two modes (k_x, +-k_y) of a
// point in registers and collects shells in LDS; a tile spans few shells, so
// it writes its short window of sums to memory, and a second kernel adds, for
// each shell, the windows that hold it in a fixed order.  (Adding every mode
// to the shell's word in memory with atomics was bound by the atomics: 265 of
// the call's 433 us at 2048^2; the call now takes 162.)  The order of the LDS
// additions is not fixed: results repeat to rounding.
#include <hipfft/hipfft.h>

#include <cmath>

#include "kbc_launch.hpp"
#include "kbc_tile.hpp"

namespace kbc {

namespace {

// ux and uy of the state, [n][stride] each
template <int FORM>
__global__ __launch_bounds__(256) void k_velocity(const typename Form<FORM>::S* __restrict__ src, int n,
                                                  int64_t pitch, double rho0, int64_t stride,
                                                  double* __restrict__ ux, double* __restrict__ uy) {
    using F = Form<FORM>;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= n || y >= n) return;
    double dr = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        int xs = x - kCx[i], ys = y - kCy[i];
        xs = xs < 0 ? xs + n : (xs >= n ? xs - n : xs);
        ys = ys < 0 ? ys + n : (ys >= n ? ys - n : ys);
        const double g = F::dec64(src[(static_cast<int64_t>(ys) * 9 + i) * pitch + xs], i);
        dr += g;
        jx += kCx[i] * g;
        jy += kCy[i] * g;
    }
    const double r = rho0 + dr;
    ux[y * stride + x] = jx / r;
    uy[y * stride + x] = jy / r;
}

constexpr int kCols = 256;                   // k_x values of a tile, one per thread
constexpr int kRows = 8;                     // |k_y| values of a tile
// shells a tile can touch: |k| changes by less than kCols + kRows across it
constexpr int kWindow = kCols + kRows + 2;

// round(|k|) for |k_x| = a, |k_y| = b
__device__ __forceinline__ int shell_of(double k2) { return static_cast<int>(floor(sqrt(k2) + 0.5)); }
__device__ __forceinline__ double norm2(int a, int b) {
    return static_cast<double>(a) * a + static_cast<double>(b) * b;
}

__global__ __launch_bounds__(256) void k_shells(const double2* __restrict__ fx, const double2* __restrict__ fy, int n,
                                                double scale, double kunit2, double2* __restrict__ windows) {
    __shared__ double se[kWindow], sz[kWindow];
    for (int i = static_cast<int>(threadIdx.x); i < kWindow; i += 256) se[i] = sz[i] = 0.0;
    __syncthreads();
    const int half = n / 2;
    const int a0 = static_cast<int>(blockIdx.y) * kCols, b0 = static_cast<int>(blockIdx.x) * kRows;
    const int base = shell_of(norm2(a0, b0));
    const int a = a0 + static_cast<int>(threadIdx.x);
    if (a <= half) {
        // -k_x is another mode, the conjugate of a stored one
        const double w = (a != 0 && 2 * a != n) ? 2.0 * scale : scale;
        auto mode = [&](int ky) {
            const int64_t m = static_cast<int64_t>(ky) * (half + 1) + a;
            const double2 u = fx[m], v = fy[m];
            return u.x * u.x + u.y * u.y + (v.x * v.x + v.y * v.y);
        };
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int b = b0 + r;
            if (b > half) break;
            double e = mode(b);
            if (b != 0 && 2 * b != n) e += mode(n - b);
            e *= w;
            const double k2 = norm2(a, b);
            const int s = shell_of(k2) - base;
            __hip_atomic_fetch_add(&se[s], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_add(&sz[s], e * k2 * kunit2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
    double2* out = windows + static_cast<int64_t>(blockIdx.y * gridDim.x + blockIdx.x) * kWindow;
    for (int i = static_cast<int>(threadIdx.x); i < kWindow; i += 256) out[i] = make_double2(se[i], sz[i]);
}

// one wave per shell: the windows of the na x nb tiles that hold it (none
// beyond the corner |k_x| = |k_y| = half)
__global__ __launch_bounds__(256) void k_shell_sums(const double2* __restrict__ windows, int na, int nb, int half,
                                                    int kmax, double* __restrict__ ek, double* __restrict__ zk) {
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const int last = shell_of(norm2(half, half));
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 4;
    for (int64_t sl = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6); sl <= kmax; sl += stride) {
        const int s = static_cast<int>(sl);
        double e = 0.0, q = 0.0;
        if (s <= last) {
            for (int ia = 0; ia < na && ia * kCols <= s + 1; ++ia)
                for (int ib = lane; ib < nb && ib * kRows <= s + 1; ib += 64) {
                    const int at = s - shell_of(norm2(ia * kCols, ib * kRows));
                    if (at < 0 || at >= kWindow) continue;
                    const double2 v = windows[(static_cast<int64_t>(ia) * nb + ib) * kWindow + at];
                    e += v.x;
                    q += v.y;
                }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                e += __shfl_xor(e, o, 64);
                q += __shfl_xor(q, o, 64);
            }
        }
        if (lane == 0) {
            if (ek) ek[s] = e;
            if (zk) zk[s] = q;
        }
    }
}

int fft_fail(hipfftResult r) { return r == HIPFFT_SUCCESS ? 0 : -2; }

int64_t tiles_a(int n) { return (n / 2) / kCols + 1; }
int64_t tiles_b(int n) { return (n / 2) / kRows + 1; }

template <int FORM>
void velocity(const Lattice& L, const void* state, int64_t stride, double* ux, double* uy) {
    const dim3 g(static_cast<unsigned>((L.nx + 63) / 64), static_cast<unsigned>((L.ny + 3) / 4));
    k_velocity<FORM><<<g, dim3(64, 4), 0, L.stream>>>(static_cast<const typename Form<FORM>::S*>(state), L.nx, L.pitch,
                                                      L.rho0, stride, ux, uy);
}

}  // namespace

// both components on rows of n / 2 + 1 complex values, then the tiles' windows
int64_t spectra_work(int n) {
    return 4 * static_cast<int64_t>(n) * (n / 2 + 1) + 2 * kWindow * tiles_a(n) * tiles_b(n);
}

int launch_spectra(const Lattice& L, const void* state, void** plan_slot, double* work, int kmax, double* ek,
                   double* zk) {
    const int n = L.nx;
    if (L.nx != L.ny || kmax < 0) return -1;
    const int nh = n / 2 + 1;
    const int64_t nn = static_cast<int64_t>(n) * n, plane = static_cast<int64_t>(n) * nh;
    double2* fx = reinterpret_cast<double2*>(work);
    double2* fy = fx + plane;
    double2* windows = fy + plane;
    const int64_t stride = 2 * nh;
    double* uy = work + 2 * plane;
    switch (L.form) {
        case F16: velocity<F16>(L, state, stride, work, uy); break;
        case F32: velocity<F32>(L, state, stride, work, uy); break;
        case F64: velocity<F64>(L, state, stride, work, uy); break;
        default: return -1;
    }
    if (hipGetLastError() != hipSuccess) return -2;
    hipfftHandle plan = reinterpret_cast<hipfftHandle>(*plan_slot);
    if (!plan) {
        long long dims[2] = {n, n}, real_rows[2] = {n, 2 * nh}, complex_rows[2] = {n, nh};
        size_t size = 0;
        if (hipfftCreate(&plan) != HIPFFT_SUCCESS) return -2;
        if (hipfftMakePlanMany64(plan, 2, dims, real_rows, 1, 2 * plane, complex_rows, 1, plane, HIPFFT_D2Z, 2, &size) !=
            HIPFFT_SUCCESS) {
            (void)hipfftDestroy(plan);
            return -2;
        }
        *plan_slot = reinterpret_cast<void*>(plan);
    }
    if (fft_fail(hipfftSetStream(plan, L.stream))) return -2;
    if (fft_fail(hipfftExecD2Z(plan, work, reinterpret_cast<hipfftDoubleComplex*>(fx)))) return -2;
    const double scale = 0.5 / (static_cast<double>(nn) * static_cast<double>(nn));
    const double ku = 2.0 * M_PI / n;
    const int na = static_cast<int>(tiles_a(n)), nb = static_cast<int>(tiles_b(n));
    k_shells<<<dim3(static_cast<unsigned>(nb), static_cast<unsigned>(na)), dim3(256), 0, L.stream>>>(
        fx, fy, n, scale, ku * ku, windows);
    if (hipGetLastError() != hipSuccess) return -2;
    const int groups = kmax / 4 + 1;
    k_shell_sums<<<dim3(static_cast<unsigned>(groups < 65536 ? groups : 65536)), dim3(256), 0, L.stream>>>(
        windows, na, nb, n / 2, kmax, ek, zk);
    return hipGetLastError() == hipSuccess ? 0 : -2;
}

void destroy_spectra_plan(void* plan) {
    if (plan) (void)hipfftDestroy(reinterpret_cast<hipfftHandle>(plan));
}

}  // namespace kbc
