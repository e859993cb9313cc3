// Depth p = 1: <Z_u Z_v> and its derivatives in closed form (Sec. 2.3 cone of radius 1).
//
// With one layer the mixer matters on u and v only; every other qubit of the cone stays in
// |+> up to phases, so its trace leaves a cosine per neighbour.  With theta = gamma delta,
// c = cos, N the neighbours x of u or v (w_ux, w_vx: their couplings, 0 if absent)
//   A = prod_N c(theta w_ux),  B = prod_N c(theta w_vx),
//   D = prod_N c(theta (w_ux - w_vx)),  S = prod_N c(theta (w_ux + w_vx)):
//   <ZZ> = -1/2 sin(4 beta) sin(theta w_uv) (A + B) + 1/2 sin^2(2 beta) (D - S)
// (couplings between neighbours drop out).  The products carry their theta derivative along,
// all in FP64.  A term costs a few operations per neighbour where a statevector of the cone
// costs 2^k, so a call is bound by its launches.
#include "depth1.hpp"

namespace qaoa {
namespace {

struct D1Val {
    double zz, dg, db;
};

template <bool GRAD>
__device__ D1Val d1_term(const ConeD1& c, const double2* __restrict__ nb, double th, double beta) {
    double A = 1.0, B = 1.0, D = 1.0, S = 1.0;
    double dA = 0.0, dB = 0.0, dD = 0.0, dS = 0.0;
    // couplings repeat (unit and integer weights): one sine and cosine per change of |w|
    double wl = 0.0, cl = 1.0, sl = 0.0;
    auto sc = [&](double w, double& cw, double& sw) {
        const double a = fabs(w);
        if (a == 0.0) {   // an angle that is no number stays one
            sw = th * 0.0;
            cw = 1.0 + sw;
            return;
        }
        if (a != wl) {
            wl = a;
            sincos(th * a, &sl, &cl);
        }
        cw = cl;
        sw = w < 0.0 ? -sl : sl;
    };
    for (int j = 0; j < c.n; ++j) {
        const double2 w = nb[c.off + j];
        double ca, sa, cb, sb;
        sc(w.x, ca, sa);
        sc(w.y, cb, sb);
        const double cd = ca * cb + sa * sb, cs = ca * cb - sa * sb;
        if constexpr (GRAD) {
            const double sd = sa * cb - ca * sb, ss = sa * cb + ca * sb;
            dA = dA * ca - A * (w.x * sa);
            dB = dB * cb - B * (w.y * sb);
            dD = dD * cd - D * ((w.x - w.y) * sd);
            dS = dS * cs - S * ((w.x + w.y) * ss);
        }
        A *= ca;
        B *= cb;
        D *= cd;
        S *= cs;
    }
    double cw, sw, s2, c2;
    sc(c.wuv, cw, sw);
    sincos(2.0 * beta, &s2, &c2);
    const double s4 = 2.0 * s2 * c2;
    D1Val v;
    v.zz = -0.5 * s4 * sw * (A + B) + 0.5 * s2 * s2 * (D - S);
    if constexpr (GRAD) {
        v.dg = -0.5 * s4 * (c.wuv * cw * (A + B) + sw * (dA + dB)) + 0.5 * s2 * s2 * (dD - dS);
        v.db = -2.0 * (c2 * c2 - s2 * s2) * sw * (A + B) + s4 * (D - S);
    } else {
        v.dg = v.db = 0.0;
    }
    return v;
}

// One thread per (cone, point), cones fastest (the term rows are written in orbit order).
template <bool GRAD>
__global__ void __launch_bounds__(256) k_depth1_terms(D1Args a, int64_t item0, int64_t n_items) {
    for (int64_t t = item0 + blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n_items;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t point = t / a.n_cones;
        const ConeD1 c = a.cones[t - point * a.n_cones];
        const size_t ip = static_cast<size_t>(c.inst) * a.gamma_P + point;
        const D1Val v = d1_term<GRAD>(c, a.nb, a.gamma[ip] * a.deltas[c.inst], a.beta[ip]);
        a.zz[static_cast<size_t>(point) * a.M + c.orbit] = v.zz;
        if constexpr (GRAD) {
            double* g = a.g + static_cast<size_t>(point) * 2 * a.M + c.orbit;
            g[0] = v.dg;
            g[a.M] = v.db;
        }
    }
}

// Terms and their orbit-weighted sums in one launch (one instance, cones in orbit order): 2^lb
// lanes per point, each summing orbits lane, lane + 2^lb, ..., then a tree: the order of
// k_combine, whose 256 threads hold zeros beyond the last orbit.  zz and g are written where
// the caller reads them.
template <bool GRAD>
__global__ void __launch_bounds__(256)
k_depth1_point(D1Args a, int lb, const double* __restrict__ W, double* __restrict__ energy,
               double* __restrict__ dgamma, double* __restrict__ dbeta) {
    constexpr int NV = GRAD ? 3 : 1;
    __shared__ double sh[NV][256];
    const int lanes = 1 << lb;
    const int lane = threadIdx.x & (lanes - 1);
    const int64_t point = blockIdx.x * static_cast<int64_t>(256 >> lb) + (threadIdx.x >> lb);
    const double delta = a.deltas[0];
    double acc[3] = {0.0, 0.0, 0.0};
    if (point < a.P) {
        const double th = a.gamma[point] * delta, be = a.beta[point];
        for (int64_t m = lane; m < a.n_cones; m += lanes) {
            const D1Val v = d1_term<GRAD>(a.cones[m], a.nb, th, be);
            if (a.zz) a.zz[static_cast<size_t>(point) * a.M + m] = v.zz;
            acc[0] += W[m] * (1.0 - v.zz) * 0.5;
            if constexpr (GRAD) {
                if (a.g) {
                    double* g = a.g + static_cast<size_t>(point) * 2 * a.M + m;
                    g[0] = a.g_scale * v.dg;
                    g[a.M] = v.db;
                }
                acc[1] += -0.5 * W[m] * v.dg;
                acc[2] += -0.5 * W[m] * v.db;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) sh[i][threadIdx.x] = acc[i];
    for (int s = lanes >> 1; s > 0; s >>= 1) {
        __syncthreads();
        if (lane < s) {
#pragma unroll
            for (int i = 0; i < NV; ++i) sh[i][threadIdx.x] += sh[i][threadIdx.x + s];
        }
    }
    if (lane == 0 && point < a.P) {
        energy[point] = sh[0][threadIdx.x];
        if constexpr (GRAD) {
            dgamma[point] = delta * sh[1][threadIdx.x];
            dbeta[point] = sh[2][threadIdx.x];
        }
    }
}

// The same where points leave compute units idle: 1024 threads per point, whose four waves a SIMD hide
// each other's chains of FP64 sines, put the weighted terms into LDS, and the sums follow in the same
// order (thread t of 256 the orbits t, t + 256, ...: the same bits).
template <bool GRAD>
__global__ void __launch_bounds__(1024)
k_depth1_wide(D1Args a, const double* __restrict__ W, double* __restrict__ energy, double* __restrict__ dgamma,
              double* __restrict__ dbeta) {
    constexpr int NV = GRAD ? 3 : 1;
    __shared__ double sh[NV][D1_POINT];
    const int tid = threadIdx.x, n = static_cast<int>(a.n_cones);
    const int64_t point = blockIdx.x;
    const double delta = a.deltas[0], th = a.gamma[point] * delta, be = a.beta[point];
    for (int m = tid; m < n; m += 1024) {
        const D1Val v = d1_term<GRAD>(a.cones[m], a.nb, th, be);
        if (a.zz) a.zz[static_cast<size_t>(point) * a.M + m] = v.zz;
        sh[0][m] = W[m] * (1.0 - v.zz) * 0.5;
        if constexpr (GRAD) {
            if (a.g) {
                double* g = a.g + static_cast<size_t>(point) * 2 * a.M + m;
                g[0] = a.g_scale * v.dg;
                g[a.M] = v.db;
            }
            sh[1][m] = -0.5 * W[m] * v.dg;
            sh[2][m] = -0.5 * W[m] * v.db;
        }
    }
    __syncthreads();
    if (tid < 256) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            double x = 0.0;
            for (int m = tid; m < n; m += 256) x += sh[i][m];
            sh[i][tid] = x;   // no other thread reads this place
        }
    }
    for (int s = 128; s > 0; s >>= 1) {
        __syncthreads();
        if (tid < s) {
#pragma unroll
            for (int i = 0; i < NV; ++i) sh[i][tid] += sh[i][tid + s];
        }
    }
    if (tid == 0) {
        energy[point] = sh[0][0];
        if constexpr (GRAD) {
            dgamma[point] = delta * sh[1][0];
            dbeta[point] = sh[2][0];
        }
    }
}

}  // namespace

hipError_t launch_depth1_terms(const D1Args& a, int64_t item0, int64_t n_items, bool grad, hipStream_t st) {
    const int64_t n = n_items - item0;
    if (n <= 0) return hipSuccess;
    const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, int64_t{1} << 20));
    if (grad) hipLaunchKernelGGL(k_depth1_terms<true>, dim3(blocks), dim3(256), 0, st, a, item0, n_items);
    else hipLaunchKernelGGL(k_depth1_terms<false>, dim3(blocks), dim3(256), 0, st, a, item0, n_items);
    return hipGetLastError();
}

hipError_t launch_depth1_point(const D1Args& a, const double* W, double* energy, double* dgamma, double* dbeta,
                               hipStream_t st) {
    // One workgroup per point and compute unit (256 of them) at most: 1002 orbits with Gaussian couplings
    // and the gradient, 1, 33, 256 points: 18.9, 19.2, 20.1 us in 256 threads, 13.8, 14.3, 16.8 in 1024; 257
    // points, with one compute unit taking a second point: 25.3 and 27.4; 1000 points: 43.4 and 54.6.
    if (a.n_cones > 256 && a.P <= 256) {
        if (a.n_cones > D1_POINT) return hipErrorInvalidValue;
        if (a.P <= 0) return hipSuccess;
        const dim3 grid(static_cast<unsigned>(a.P));
        if (dgamma) hipLaunchKernelGGL(k_depth1_wide<true>, grid, dim3(1024), 0, st, a, W, energy, dgamma, dbeta);
        else hipLaunchKernelGGL(k_depth1_wide<false>, grid, dim3(1024), 0, st, a, W, energy, nullptr, nullptr);
        return hipGetLastError();
    }
    int lb = 0;
    while (lb < 8 && (int64_t{1} << lb) < a.n_cones) ++lb;
    const int64_t per = 256 >> lb;
    // a grid holds fewer than 2^32 threads
    constexpr int64_t CH = static_cast<int64_t>(UINT32_MAX) / 256;
    const int64_t blocks = (a.P + per - 1) / per;
    for (int64_t b0 = 0; b0 < blocks; b0 += CH) {
        D1Args c = a;
        const int64_t p0 = b0 * per;
        c.P = a.P - p0;
        c.gamma = a.gamma + p0;
        c.beta = a.beta + p0;
        c.zz = a.zz ? a.zz + static_cast<size_t>(p0) * a.M : nullptr;
        c.g = a.g ? a.g + static_cast<size_t>(p0) * 2 * a.M : nullptr;
        const dim3 grid(static_cast<unsigned>(std::min<int64_t>(CH, blocks - b0)));
        if (dgamma)
            hipLaunchKernelGGL(k_depth1_point<true>, grid, dim3(256), 0, st, c, lb, W, energy + p0, dgamma + p0,
                               dbeta + p0);
        else
            hipLaunchKernelGGL(k_depth1_point<false>, grid, dim3(256), 0, st, c, lb, W, energy + p0, nullptr, nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qaoa
