// Device kernels of the fast spectral collision operator (Sec. 4 of the paper) for
// gfx950, and the host-side launch sequence.
//
// Pipeline for a slice of nb nodes (all fields complex, index space, z fastest):
//   1. forward_zy, fft_pass  f_hat = DFT(f) / N^3                  (per node, species)
//   2. gain_kernel     per (node, gain class, rho_q, x-chunk c):
//                        S_q = sum_p w_p A_p B_p in physical space, where
//                        A_p = IDFT(f_hat^i e^{+i pi rho a l.sigma_p / L})  (= f^i(v + a rho sigma_p))
//                        B_p = IDFT(f_hat^j e^{-i pi rho b m.sigma_p / L})  (= f^j(v - b rho sigma_p)),
//                      then the partial forward DFT of S_q over the chunk  -> P
//   3. radial_kernel   Q_hat+ = sum_terms sum_q w_q F(|k|, rho_q) / N^3 * DFT(S_q)
//                      L_hat  = sum_j G-_ij(|k|) f_hat^j          -> Gt, Lt (k_z <= N/2 half)
//   4. half_xpass      inverse DFT of Gt and Lt along x, on the stored half
//   5. inverse_yz      inverse DFT along y and z (Hermitian rows, real result) fused with
//                      Q = IDFT(Gt) - f^i IDFT(Lt)
//
// The sigma-sum is taken before the forward transform of the gain because, for the
// VHS family, F(k, rho, sigma) does not depend on sigma; with an antipodal design the
// two orderings of an unlike pair share S_q and a like pair needs half the directions
// (see the host set-up).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gain.hpp"

namespace dgfs {

// ========================================================= FP64 conservation
// The s+4 invariants A Q of a node in FP64, lambda = (A A^T)^{-1} A Q, then
// Q_out = Q - A^T lambda.  Rows of A: h_i^3 on species i (s rows), m_i h_i^3 v_d
// (3 rows), m_i h_i^3 |v|^2 (1 row), on species i's own grid (half-width Ls[i]).
// With UPDATE, the projected value is not stored but added to the state:
// f <- f + dt * Q_projected (forward-Euler step of a homogeneous relaxation).
// The grid size is a template argument for the compiled N (NC > 0), so the index
// arithmetic of the velocity coordinates uses constant divisors; NC = 0 reads it from Nrt.
//
// G workgroups share a node: each reduces the whole node (from L2; the same order
// whatever G, so a node's result does not depend on the batch) and updates every G-th part.
// One workgroup per node was bound by its one CU's FP64 issue and load latency when there
// were few nodes.  A thread takes V consecutive z values (one 16-byte access when the
// pointers allow it), so the velocity terms that belong to the row are formed once per V
// values.  One FP64 node at N = 16: 16.1 -> 7.2 us, at N = 64: 327 -> 106 us; three FP32 nodes
// of three species at N = 24 (with the update): 37.6 -> 11.2 us; 256 FP32 nodes at N = 32:
// 69 -> 49 us for 201 MB (4.1 TB/s; a copy reaches 5.15).
template <typename TIN, int V, bool VEC>
__device__ __forceinline__ void load_v(const TIN* p, double* v) {
    if constexpr (VEC) {
        typedef TIN vec __attribute__((ext_vector_type(V)));
        const vec t = *reinterpret_cast<const vec*>(p);
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = double(t[j]);
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = double(p[j]);
    }
}

template <typename TIN, bool UPDATE, int NC, bool VEC>
__global__ __launch_bounds__(1024) void conserve_kernel(const TIN* Q, double* out, TIN* fstate, double dt,
                                                        const double* __restrict__ Minv,
                                                        const double* __restrict__ mass,
                                                        const double* __restrict__ Ls, int s, int Nrt, int G) {
    constexpr int R = 12;  // s + 4 <= 12
    constexpr int V = int(16 / sizeof(TIN));   // divides N (every supported N is a multiple of 8)
    __shared__ double red[16][R];
    __shared__ double aq[R];
    __shared__ double lam[R];
    const int N = NC > 0 ? NC : Nrt;
    const int b = int(blockIdx.x) / G, g = int(blockIdx.x) % G;
    const int n3 = N * N * N, nv = n3 / V;
    const int64_t tot = int64_t(s) * n3;
    const TIN* q = Q + int64_t(b) * tot;
    const int nr = s + 4;
    const int tid = threadIdx.x;
    double minv[R];   // row tid of the inverse Gram matrix, read ahead of its use
    if (tid < nr) {
#pragma unroll
        for (int c = 0; c < R; ++c) minv[c] = c < nr ? Minv[tid * nr + c] : 0.0;
    }
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
    for (int i = 0; i < s; ++i) {
        const double L = Ls[i], h = 2.0 * L / N;
        const TIN* qi = q + int64_t(i) * n3;
        double a0 = 0.0, ax = 0.0, ay = 0.0, az = 0.0, ae = 0.0;
#pragma unroll 4
        for (int n = tid; n < nv; n += 1024) {
            const int e = n * V;
            const double vx = fma(double(e / (N * N)), h, -L), vy = fma(double((e / N) % N), h, -L),
                         vz = fma(double(e % N), h, -L);
            double v[V];
            load_v<TIN, V, VEC>(qi + e, v);
            // sums of q, q j and q j^2 over the V values z = z0 + j
            double s0 = v[0], s1 = 0.0, s2 = 0.0;
#pragma unroll
            for (int j = 1; j < V; ++j) {
                s0 += v[j];
                s1 = fma(double(j), v[j], s1);
                s2 = fma(double(j * j), v[j], s2);
            }
            const double hs1 = h * s1, r1 = fma(vz, s0, hs1);
            a0 += s0;
            ax = fma(s0, vx, ax);
            ay = fma(s0, vy, ay);
            az += r1;
            // sum q |v|^2 = (vx^2 + vy^2) s0 + vz (r1 + h s1) + h^2 s2
            ae = fma(fma(vx, vx, vy * vy), s0, fma(vz, r1 + hs1, fma(h * h, s2, ae)));
        }
        const double h3 = h * h * h, mh = mass[i] * h3;
#pragma unroll
        for (int r = 0; r < R - 4; ++r)
            if (r == i) acc[r] = h3 * a0;
        acc[R - 4] = fma(mh, ax, acc[R - 4]);
        acc[R - 3] = fma(mh, ay, acc[R - 3]);
        acc[R - 2] = fma(mh, az, acc[R - 2]);
        acc[R - 1] = fma(mh, ae, acc[R - 1]);
    }
    // block reduction of the rows in use
    const int wave = tid / 64, lane = tid % 64;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= s && r < R - 4) continue;
        double v = acc[r];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) red[wave][r] = v;
    }
    __syncthreads();
    // invariant vector in the order (species 0..s-1, px, py, pz, energy)
    if (tid < nr) {
        const int r = tid < s ? tid : tid - s + R - 4;
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) v += red[w][r];
        aq[tid] = v;
    }
    __syncthreads();
    if (tid < nr) {
        double v = 0.0;
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (c < nr) v = fma(minv[c], aq[c], v);
        lam[tid] = v;
    }
    __syncthreads();
    for (int i = 0; i < s; ++i) {
        const double L = Ls[i], h = 2.0 * L / N, h3 = h * h * h, mh = mass[i] * h3;
        const double c0 = lam[i] * h3, cx_ = mh * lam[s], cy = mh * lam[s + 1], cz = mh * lam[s + 2],
                     ce = mh * lam[s + 3];
        const int64_t off = int64_t(b) * tot + int64_t(i) * n3;
#pragma unroll 2
        for (int n = tid + 1024 * g; n < nv; n += 1024 * G) {
            const int e = n * V;
            const double vx = fma(double(e / (N * N)), h, -L), vy = fma(double((e / N) % N), h, -L);
            const double row = c0 + cx_ * vx + cy * vy + ce * fma(vx, vx, vy * vy);
            double v[V];
            load_v<TIN, V, VEC>(Q + off + e, v);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const double vz = fma(double(e % N + j), h, -L);
                v[j] -= fma(fma(ce, vz, cz), vz, row);
            }
            if constexpr (UPDATE) {
                double f[V];
                load_v<TIN, V, VEC>(fstate + off + e, f);
                if constexpr (VEC) {
                    typedef TIN vec __attribute__((ext_vector_type(V)));
                    vec t;
#pragma unroll
                    for (int j = 0; j < V; ++j) t[j] = TIN(f[j] + dt * v[j]);
                    *reinterpret_cast<vec*>(fstate + off + e) = t;
                } else {
#pragma unroll
                    for (int j = 0; j < V; ++j) fstate[off + e + j] = TIN(f[j] + dt * v[j]);
                }
            } else {
                if constexpr (VEC) {
                    typedef double vec __attribute__((ext_vector_type(2)));
#pragma unroll
                    for (int j = 0; j < V; j += 2) *reinterpret_cast<vec*>(out + off + e + j) = vec{v[j], v[j + 1]};
                } else {
#pragma unroll
                    for (int j = 0; j < V; ++j) out[off + e + j] = v[j];
                }
            }
        }
    }
}

// ======================================================= elementwise (stepping)
// out = a x + b y over n values (x, y, out may coincide elementwise).
template <typename T>
__global__ __launch_bounds__(256) void axpby_kernel(const T* x, const T* y, T* out, T a, T b, int64_t n) {
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t < n) out[t] = a * x[t] + b * y[t];
}

// ================================================================== launches
namespace {

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Compiled gain-kernel geometries (CH, CZ) per N and precision; the first is the default
// (the fastest measured on MI355X for that N; autotune.py re-measures on the device).
// (32, 2, 0): the matrix-core gain (FP32 VHS plans of the circular form; the others get
// the first geometry with CZ > 0).
// N = 36 and 72 are the padded grids of the dealiased form at N = 24 and 48 only.
constexpr int kTilesF32[][3] = {{16, 1, 1}, {16, 2, 1}, {16, 1, 2}, {24, 3, 1}, {24, 3, 2}, {24, 3, 4}, {24, 3, 3},
                                {24, 1, 1}, {32, 2, 0}, {32, 2, 1}, {32, 4, 1}, {32, 4, 2}, {48, 6, 2}, {48, 12, 4},
                                {48, 12, 2}, {48, 12, 1}, {48, 12, 3}, {64, 16, 4}, {36, 3, 2}, {72, 24, 4}};
constexpr int kTilesF64[][3] = {{16, 1, 1}, {24, 3, 2}, {32, 4, 2}, {48, 12, 4}, {64, 32, 8}, {36, 6, 4},
                                {72, 72, 8}};

}  // namespace

int tile_candidates(int N, int precision, GainGeometry* out, int max) {
    int n = 0;
    auto scan = [&](const auto& tab) {
        for (const auto& t : tab)
            if (t[0] == N && n < max) out[n++] = GainGeometry{t[1], t[2]};
    };
    if (precision == DGFS_FP64) scan(kTilesF64);
    else scan(kTilesF32);
    return n;
}

bool gain_geometry(int N, int precision, GainGeometry* g, bool matrix_ok) {
    GainGeometry cand[16];
    const int n = tile_candidates(N, precision, cand, 16);
    for (int k = 0; k < n; ++k)
        if (cand[k].CZ != 0 || matrix_ok) {
            *g = cand[k];
            return true;
        }
    return false;
}

hipError_t launch_collide(const dgfs_plan& p, const void* f, void* Q, int64_t nb, Scratch ws, bool pairs,
                          hipStream_t st, hipEvent_t* ev) {
    if (p.inner) {
        switch (p.N) {
            case 16: return run_dealias_16(p, *p.inner, f, Q, int(nb), ws.p, pairs, st, ev);
            case 24: return run_dealias_24(p, *p.inner, f, Q, int(nb), ws.p, pairs, st, ev);
            case 32: return run_dealias_32(p, *p.inner, f, Q, int(nb), ws.p, pairs, st, ev);
            case 48: return run_dealias_48(p, *p.inner, f, Q, int(nb), ws.p, pairs, st, ev);
            default: return hipErrorInvalidValue;
        }
    }
    if (p.vss) {
        switch (p.N) {
            case 16: return run_vss_16(p, f, Q, int(nb), ws, pairs, st, ev);
            case 24: return run_vss_24(p, f, Q, int(nb), ws, pairs, st, ev);
            case 32: return run_vss_32(p, f, Q, int(nb), ws, pairs, st, ev);
            case 48: return run_vss_48(p, f, Q, int(nb), ws, pairs, st, ev);
            default: return hipErrorInvalidValue;
        }
    }
    switch (p.N) {
        case 16: return run_tiles_16(p, f, Q, int(nb), ws, pairs, st, ev);
        case 24: return run_tiles_24(p, f, Q, int(nb), ws, pairs, st, ev);
        case 32: return run_tiles_32(p, f, Q, int(nb), ws, pairs, st, ev);
        case 48: return run_tiles_48(p, f, Q, int(nb), ws, pairs, st, ev);
        case 64: return run_tiles_64(p, f, Q, int(nb), ws, pairs, st, ev);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conserve(const dgfs_plan& p, const void* Q, double* out, void* fstate, double dt, int64_t nb,
                           hipStream_t st) {
    const char* dev = static_cast<const char*>(p.dev);
    const double* minv = reinterpret_cast<const double*>(dev + p.off_minv);
    const double* mass = minv + (p.s + 4) * (p.s + 4);
    const double* Ls = mass + p.s;
    // 16-byte accesses where every pointer allows them (a species' field is a whole multiple
    // of 16 bytes)
    auto al16 = [](const void* x) { return reinterpret_cast<uintptr_t>(x) % 16 == 0; };
    const bool vec = al16(Q) && al16(out) && al16(fstate);
    // Workgroups per node: up to one per CU (a CU holds one of this size), at most 8 (beyond that the repeated
    // reduction is most of the work).  A result written over its own input needs one: the
    // others would still be reading it.
    const size_t qb = size_t(nb) * p.s * p.n3() * p.elem(), ob = size_t(nb) * p.s * p.n3() * sizeof(double);
    const uintptr_t qa = reinterpret_cast<uintptr_t>(Q), oa = reinterpret_cast<uintptr_t>(out),
                    fa = reinterpret_cast<uintptr_t>(fstate);
    const bool overlap = (out && oa < qa + qb && qa < oa + ob) || (fstate && fa < qa + qb && qa < fa + qb);
    const int G = overlap ? 1 : int(std::max<int64_t>(1, std::min<int64_t>(8, 256 / nb)));
    const dim3 grid(static_cast<unsigned>(nb * G)), block(1024);
    auto go = [&](auto tin, auto nc, auto upd, auto vc) {
        using TIN = decltype(tin);
        conserve_kernel<TIN, decltype(upd)::value, decltype(nc)::value, decltype(vc)::value><<<grid, block, 0, st>>>(
            static_cast<const TIN*>(Q), out, static_cast<TIN*>(fstate), dt, minv, mass, Ls, p.s, p.N, G);
    };
    auto run = [&](auto tin, auto nc) {
        if (fstate && vec) go(tin, nc, std::true_type{}, std::true_type{});
        else if (fstate) go(tin, nc, std::true_type{}, std::false_type{});
        else if (vec) go(tin, nc, std::false_type{}, std::true_type{});
        else go(tin, nc, std::false_type{}, std::false_type{});
    };
    auto by_n = [&](auto tin) {
        switch (p.N) {
            case 16: run(tin, std::integral_constant<int, 16>{}); break;
            case 24: run(tin, std::integral_constant<int, 24>{}); break;
            case 32: run(tin, std::integral_constant<int, 32>{}); break;
            case 48: run(tin, std::integral_constant<int, 48>{}); break;
            case 64: run(tin, std::integral_constant<int, 64>{}); break;
            default: run(tin, std::integral_constant<int, 0>{}); break;
        }
    };
    if (p.precision == DGFS_FP64) by_n(double{});
    else by_n(float{});
    return hipGetLastError();
}

hipError_t launch_axpby(const dgfs_plan& p, const void* x, const void* y, void* out, double a, double b, int64_t n,
                        hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>((n + 255) / 256)), block(256);
    if (p.precision == DGFS_FP64)
        axpby_kernel<double><<<grid, block, 0, st>>>(static_cast<const double*>(x), static_cast<const double*>(y),
                                                      static_cast<double*>(out), a, b, n);
    else
        axpby_kernel<float><<<grid, block, 0, st>>>(static_cast<const float*>(x), static_cast<const float*>(y),
                                                     static_cast<float*>(out), float(a), float(b), n);
    return hipGetLastError();
}

}  // namespace dgfs
