// The fused gain kernel, the radial-sum/loss kernel, the combination kernel and the
// launch sequence of one batch slice, as templates over (precision, N, tile).  Each
// tiles_<N>.hip instantiates them for one N.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fft.hpp"
#include "passes.hpp"
#include "plan.hpp"

namespace dgfs {

// ================================================================ gain kernel
// What a gain work item accumulates and stores:
// GAIN_REAL     Re S summed over the class's directions (VHS: F real and even in k);
//               the Hermitian half of the partial is stored.
// GAIN_COMPLEX  the complex S summed over the class's directions, whole spectrum stored
//               (the dealiased form, whose inputs are not spectra of real fields: the
//               shifted fields come from unpaired transforms).
// GAIN_VSS      VSS (F depends on sigma): a class holds at most two directions; their
//               real parts are transformed together as Re S_0 + i Re S_1 (whole spectrum
//               stored), and their imaginary parts, which reach the result only on the
//               planes k_x, k_y or k_z = N/2 (the literal Nyquist reading), are reduced
//               to those planes (sums with (-1)^x, (-1)^y, (-1)^z) and stored.
// GAIN_TERMS    one direction of a GAIN_REAL item: its Re(A B) alone, stored unweighted in
//               physical space for gain_sum_kernel (split_rule in plan.hpp).
enum { GAIN_REAL = 0, GAIN_COMPLEX = 1, GAIN_VSS = 2, GAIN_TERMS = 3 };

// How the x-pass issues the loads of the next sub-sequence while it combines the current
// one, chosen per geometry by measurement (tiles_<N>.hip, vss_<N>.hip): not at all, in a
// buffer that is copied at every step, or in two buffers in turn (no copies, more registers
// alive).  The packed form takes any value but PIPE_OFF as two buffers.  FP64 gains, ms
// off / rotating / two: N = 16 (200 nodes) 0.527 / 0.442 / 0.427, N = 24 (60) 2.03 / 2.28 /
// 2.14, N = 32 (32) 3.91 / 3.15 / 3.33, N = 48 (4) 3.62 / 3.02 / 2.93, N = 64 (1) 6.49 / 5.65
// / 5.59 (4.77 / 5.32 since it keeps x-transforms, below): the 16-byte loads leave few in
// flight otherwise; at N = 24 the registers cost a wavefront.
enum { PIPE_OFF = 0, PIPE_ROTATE = 1, PIPE_TWO = 2 };

// Geometry of one work item: the x-chunk c (x-indices = c mod CH, NP = N/CH of them)
// of one S_q field.  Each y/z pencil of the chunk is shared by CZ thread groups: group
// cz keeps the outputs with index = cz mod CZ (decimation in frequency), so a thread
// holds NS = N/CZ values per field.  The group index is uniform per wavefront when
// NTC = NP*N is a multiple of 64, so every twiddle is a compile-time constant; the padded
// grids of the dealiased form (36, 72) have no such split, and there the one wavefront
// that straddles two groups runs both groups' code under its lane masks.
template <typename T, int N, int CH, int CZ>
struct GainK {
    static constexpr int NP = N / CH;
    static constexpr int NS = N / CZ;
    static constexpr int NTC = NP * N;
    static constexpr int NT = NTC * CZ;
    static constexpr int KZH = N / 2 + 1;               // stored k_z of a partial (Hermitian half)
    static constexpr int NPEN = N * KZH;                // stored (k_y, k_z) pencils of a partial
    static constexpr int PX = (NPEN + NT - 1) / NT;     // stored pencils per thread (guarded)
    static constexpr int NPENF = N * N;                 // every (k_y, k_z) pencil (VSS: complex field)
    static constexpr int PXF = (NPENF + NT - 1) / NT;
    static constexpr int ROW = N + 1;                  // padded LDS row (bank spread)
    static constexpr int LDS = NP * N * ROW;
    // packed form: line-data regions [2][NP][N+1], the correction array [N][ROWC] (in
    // the main buffer) and the thread groups GC of its transforms (one wavefront each)
    static constexpr int LINES = 2 * NP * (N + 1);
    static constexpr int ROWC = N + 2 * NP + 1;
    static constexpr int GC = (N % 4 == 0 && 256 <= NT) ? 4 : (N % 3 == 0 && 192 <= NT) ? 3 : (128 <= NT) ? 2 : 1;
    static_assert(NP * CH == N && NS * CZ == N, "CH and CZ must divide N");
    static_assert(NTC % 64 == 0 || N % 9 == 0, "a CZ group must be whole wavefronts (except the 36, 72 grids)");
};

// Workgroups are dealt to the 8 XCDs round-robin.  Of every eight nodes each XCD takes one
// whole, so that a node's spectra are read through one L2; with NG > 1 the items of up to NG
// of its nodes (b, b + 8, ...) run interleaved, same item next to each other.  The items of
// the last nb % 8 nodes are dealt to all XCDs instead: with one XCD per node a call of one
// node ran on 32 of the 256 CUs (N = 64, FP64, one node: 52.1 ms in the gain, 6.5 ms dealt),
// and a ragged batch left XCDs idle for a whole node's time at its end.  Each XCD then reads
// these nodes' spectra for itself, which are at most a few MB at a time: the workgroups in
// flight cover a class of a few nodes.  They go class by class, in the order `ord` (most
// directions first), so that the short items fill the end: five FP64 nodes at N = 32, one
// SSP-RK2 step, node by node 1.27 ms, class by class 1.13; 63 FP32 nodes at N = 24, two steps,
// 3.40 and 3.21 ms; five FP32 nodes at N = 32 0.274 and 0.228 ms.
// A node has ncls classes of ipc items; returns the node and item of workgroup g, false past
// the last one.  ord may be null (classes of equal length).
template <int NG>
__device__ __forceinline__ bool gain_item(int g, int nb, int ncls, int ipc, const int* ord, int& b, int& item) {
    const int xcd = g & 7, local = g >> 3;
    const int octets = nb >> 3, ipn = ncls * ipc;
    if (local < octets * ipn) {
        const int grp = local / (ipn * NG), rem = local % (ipn * NG);
        const int w = NG == 1 ? 1 : min(NG, octets - grp * NG);
        b = (grp * NG + rem % w) * 8 + xcd;
        item = rem / w;
        return true;
    }
    const int t = (local - octets * ipn) * 8 + xcd, r = nb & 7;
    if (t >= r * ipn) return false;
    const int rank = t / (r * ipc), rem = t % (r * ipc);
    b = octets * 8 + rem / ipc;
    item = (ord ? ord[rank] : rank) * ipc + rem % ipc;
    return true;
}
// Workgroups to launch for gain_item.
inline unsigned gain_groups(int nb, int64_t ipn) {
    return unsigned(8 * ((nb / 8) * ipn + ((nb % 8) * ipn + 7) / 8));
}

template <typename T>
struct GainArgs {
    const cx<T>* fhat;  // [nb][s][N^3], DFT / N^3
    cx<T>* P;           // [nb][ncls][nrho][CH][N/CH][N][N/2+1]  (k_z <= N/2 of each partial);
                        // GAIN_COMPLEX, GAIN_VSS: [nb][ncls][nrho][CH][N/CH][N][N]  (whole spectrum)
    T* PL;              // GAIN_VSS: [nb][ncls][nrho][2][(2 + CH) N^2]  Nyquist-plane sums of Im S_d:
                        //   [x][y] over z, [x][z] over y, then per chunk [y][z] over its x
    const cx<T>* kx;    // [dirs][nrho][2][CH][N]  x-phase merged with the chunk split
    const cx<T>* yz;    // [dirs][nrho][2][2][N]   y- and z-phases
    const T* nyq;       // [dirs][nrho][2]         2 sin(theta_x N / 2) of the x-phase
    const int* cls;     // [ncls][4] = i, j, ndir, dir_offset
    const T* wdir;      // [ncls]
    const int* ord;     // [ncls] classes, most directions first
    const int* xs;      // [dirs]  1: the direction before it in its class has the same sigma_x
    T* D;               // GAIN_TERMS: [nb][dirs][nq][CH][N/CZ][threads]  Re(A B) of one direction
    int s, ncls, nrho, nb, tdirs;
    int q0 = 0, nq = 0; // GAIN_TERMS and gain_sum_kernel: the radial points q0 .. q0 + nq - 1
};

// out[j] = X[CZ j + CZI] of the length-N DFT (sign SIGN) of the sequence
// x[n] = src[n * stride]: the CZ strided input sub-sequences are combined with the
// split factors e^{SIGN 2 pi i t CZI / CZ}, twiddled by e^{SIGN 2 pi i l CZI / N},
// then transformed with an N/CZ-point FFT.  With PAD the middle third of the sequence is
// zero and not read (a spectrum padded by 3/2); a sum that misses terms then starts from a
// zero that the compiler does not see, so that it neither moves signs through the twiddle
// products nor folds them, and every output keeps the rounding of the full sum.
template <int N, int CZ, int CZI, int SIGN, int STRIDE, bool PAD = false, typename T>
__device__ __forceinline__ void split_fft(const cx<T>* src, cx<T>* out) {
    constexpr int NS = N / CZ;
    T zero = T(0);
    if constexpr (PAD) asm("" : "+v"(zero));
    static_for<0, NS>([&](auto l) {
        auto kept = [](int n) { return n < N / 3 || n >= N - N / 3; };
        int terms = 0;       // terms and first are resolved at compile time (constant indices)
        for (int t = 0; t < CZ; ++t) terms += !PAD || kept(l + t * NS);
        cx<T> acc = cx<T>{zero, zero};
        bool first = terms == CZ || (CZI == 0 && terms > 0);
        static_for<0, CZ>([&](auto t) {
            constexpr int n = decltype(l)::value + decltype(t)::value * NS;
            if constexpr (!PAD || n < N / 3 || n >= N - N / 3) {
                constexpr long k = long(decltype(t)::value) * CZI;
                const cx<T> v = rot<SIGN, k, CZ>(src[n * STRIDE]);
                acc = first ? v : acc + v;
                first = false;
            }
        });
        out[l] = rot<SIGN, long(decltype(l)::value) * CZI, long(N)>(acc);
        // keep at most a few loads in flight: the pencil's inputs are combined as they
        // arrive instead of all being held in registers at once
        if constexpr (decltype(l)::value % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
    fft<NS, SIGN>(out);
}

// Call f(integral_constant<int, cz>) for the runtime (wave-uniform) group index cz.
template <int CZ, typename F>
__device__ __forceinline__ void with_group(int cz, F&& f) {
    if constexpr (CZ == 1) {
        f(std::integral_constant<int, 0>{});
    } else {
        static_for<0, CZ>([&](auto g) {
            if (cz == decltype(g)::value) f(g);
        });
    }
}

// y-pass (through LDS, in place on columns) and z-pass (rows, result kept) of one
// field whose x-pass output is in buf; out[j] = value at z-index CZ j + cz of the
// thread's pencil (m, r).  With PAD the middle thirds of the y- and z-modes are zero: their
// rows and columns are neither read nor written, and the y-pass's columns are dealt to the
// first 2/3 of each group's threads.
template <typename T, int N, int CH, int CZ, int SIGN, bool PAD = false>
__device__ __forceinline__ void yz_passes(cx<T>* buf, int cz, int m, int r, cx<T>* out) {
    using K = GainK<T, N, CH, CZ>;
    cx<T> v[K::NS];
    int my = m, ry = r;
    bool act = true;
    if constexpr (PAD) {
        constexpr int NK = N - N / 3;
        const int u = m * N + r;
        act = u < K::NP * NK;
        my = u / NK;
        ry = u % NK;
        if (ry >= N / 3) ry += N / 3;
    }
    if (act)
        with_group<CZ>(cz, [&](auto g) {
            split_fft<N, CZ, decltype(g)::value, SIGN, K::ROW, PAD>(buf + (my * N) * K::ROW + ry, v);
        });
    __syncthreads();
    if (act) {
#pragma unroll
        for (int j = 0; j < K::NS; ++j) buf[(my * N + CZ * j + cz) * K::ROW + ry] = v[j];
    }
    __syncthreads();
    with_group<CZ>(cz, [&](auto g) {
        split_fft<N, CZ, decltype(g)::value, SIGN, 1, PAD>(buf + (m * N + r) * K::ROW, out);
    });
}

// Buffer loads: a wave-uniform base in the resource descriptor, the lane's byte offset
// in a VGPR and a uniform byte offset in an SGPR, so the strided x-pass loads need no
// per-lane 64-bit address arithmetic.  Offsets beyond the descriptor's range read 0.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t field_rsrc(const cx<T>* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<cx<T>*>(base), 0, bytes, 0x00020000);
}

template <typename T>
__device__ __forceinline__ cx<T> bload(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    } else {
        return __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    }
}

// Work slots of the x-pass.  The Hermitian pairs P = (l_y, l_z) <-> -P (mod N) by a
// representative: rows 1..N/2-1 with all l_z, then rows 0 and N/2 with l_z in
// 1..N/2-1.  The four self-paired pencils (P = -P) follow: with SELF, as two slots that
// each take (l_y, 0) and (l_y, N/2) for l_y = 0 and l_y = N/2 (N^2/2 slots in all);
// otherwise one slot each (N^2/2 + 2 slots).  Returns false for a self-paired slot.
template <int N, bool SELF>
__device__ __forceinline__ bool pencil_slot(int slot, int& ly, int& lz) {
    constexpr int H = N / 2;
    constexpr int RA = (H - 1) * N;
    if (slot < RA) {
        ly = 1 + slot / N;
        lz = slot % N;
        return true;
    }
    const int t = slot - RA;
    if (t < 2 * (H - 1)) {
        ly = t < H - 1 ? 0 : H;
        lz = 1 + t % (H - 1);
        return true;
    }
    const int u = t - 2 * (H - 1);
    if constexpr (SELF) {
        ly = u * H;
        lz = 0;
    } else {
        ly = (u >> 1) * H;
        lz = (u & 1) * H;
    }
    return false;
}

// sum_t of the chunk terms in[l + t NP] * kx[l + t NP] for one pencil, with two load
// buffers in turn: the next batch of NP loads is in flight while the other is consumed,
// and no register copies between batches.  U tables (one per output) share the loads.
// (In FP32 at N = 32 the one-field x-pass keeps its rotating buffer, which compiles without
// spills there.)
template <typename T, int NP, int CH, int U>
__device__ __forceinline__ void x_sum_pipe(__amdgpu_buffer_rsrc_t rs, int vo, int rs_stride,
                                           const cx<T>* const (&kx)[U], cx<T>* const (&y)[U]) {
    cx<T> b0[NP], b1[NP];
    auto load = [&](cx<T>* b, int t) {
#pragma unroll
        for (int l = 0; l < NP; ++l) b[l] = bload<T>(rs, vo, (l + t * NP) * rs_stride);
    };
    auto use = [&](const cx<T>* b, int t) {
#pragma unroll
        for (int l = 0; l < NP; ++l)
#pragma unroll
            for (int u = 0; u < U; ++u) cmac(y[u][l], b[l], kx[u][l + t * NP]);
    };
    load(b0, 0);
    int t = 0;
#pragma unroll 1
    for (; t + 2 < CH; t += 2) {
        load(b1, t + 1);
        use(b0, t);
        load(b0, t + 2);
        use(b1, t + 1);
    }
    if constexpr (CH % 2 == 0) {
        load(b1, CH - 1);
        use(b0, CH - 2);
        use(b1, CH - 1);
    } else {
        use(b0, CH - 1);
    }
}

// The x-transformed pencils of a direction, kept by their threads for the next direction of
// its class.  The x-pass depends on a direction through its sigma_x alone, and the design's
// points are sorted by it, so a class's directions come in runs of one sigma_x: of 12
// directions (icosahedron) 5 are fresh, of 6 (half of them) 3, of 24 6, of the octahedron's 6
// 3.  The others take the kept values back (the same values: nothing is rounded again)
// instead of reading the spectrum and combining it anew.  It pays where the values find room in
// registers or where the x-pass is most of the kernel.  Calls in us, without / with:
//   VSS, M = 12: FP32 N = 32 (96 nodes) 8550 / 7790, but N = 24 (40) 1227 / 1220 with M = 6 691 /
//     751, N = 16 (100) 486 / 492 and N = 48 (5) 2401 / 2476; FP64 N = 32 (8) 2030 / 1863, N = 24
//     (20) 1575 / 1400, N = 16 (60) 771 / 749; M = 6: FP32 N = 32 (96) 4635 / 4595, FP64 N = 32
//     1161 / 1150, N = 24 857 / 827, but N = 16 428 / 449;
//   VHS, N = 64: FP32 (2 nodes) 3370 / 2966, FP64 (1) 4357 / 3790, M = 24 3575 / 2703, but M = 6
//     FP32 487 / 516, FP64 589 / 667;
//   VHS, FP64: N = 32 (16) 1672 / 1663, M = 24 (20) 1948 / 1680, M = 6 (16) 941 / 971; N = 24 (60)
//     2018 / 1991, M = 24 1884 / 1640, M = 6 1121 / 1165; but
//     N = 16 (200) 844 / 1140 and N = 48 (4) 3327 / 3662;
//   VHS, FP32: N = 24 (63, DG) 3208 / 3641 and N = 16 (300) 583 / 722 (a wavefront per SIMD
//     less); dealiased N = 32 (10) 1998 / 2460; the packed N = 48 form (7) 2296 / 3022 (two
//     fields' values in private memory; in a place of the workspace per workgroup, 8 nodes
//     of three species, 5.7 / 7.1 ms in the gain).
// So some geometries keep them always, and some unless more than half of a plan's directions are
// fresh (the octahedron's are: 2 of 3 and 3 of 6; the VSS classes of two directions, 5 of 6).
enum { KEEP_NEVER = 0, KEEP_ALWAYS = 1, KEEP_BY_REUSE = 2 };
template <typename T, int N, int MODE>
constexpr int keep_rule() {
    constexpr bool dbl = sizeof(T) == 8;
    if (MODE == GAIN_VSS) return N == 32 || (N == 24 && dbl) ? KEEP_ALWAYS : N == 16 && dbl ? KEEP_BY_REUSE : KEEP_NEVER;
    return MODE == GAIN_REAL && (N == 64 || (dbl && (N == 24 || N == 32))) ? KEEP_BY_REUSE : KEEP_NEVER;
}
template <int NP, typename T>
__device__ __forceinline__ void keep_x(cx<T>* to, const cx<T>* from) {
#pragma unroll
    for (int l = 0; l < NP; ++l) to[l] = from[l];
}

// Chunk c of IDFT(f_hat * phase) for one shifted field: out[j] at (x = CH m + c,
// y = r, z = CZ j + cz).  The x-pass reads the spectrum from global memory (coalesced
// over (l_y, l_z)) and keeps only the chunk's x-outputs: the CH strided input
// sub-sequences are combined with kxt, which carries the x-phase, the split factor
// e^{2 pi i t c / CH} and the twiddle e^{2 pi i l c / N}.  The y- and z-phases are
// constant along an x-pencil and multiply its outputs.  With PIPE != PIPE_OFF the loads of
// the next sub-sequence are issued before the current one is combined.
//
// f is real, so f_hat(l_x, -P) = conj(f_hat(-l_x, P)); with the linear x-phase this
// gives, for every output x-index n, G(-P)[n] = conj(G(P)[n] + delta_P (-1)^n) where
// delta_P = f_hat(N/2, P) (e^{i theta N/2} - e^{-i theta N/2}) accounts for the DFT
// index N/2 standing for the mode -N/2 on both sides.  So only one pencil of each pair
// is transformed; its partner costs a conjugate, one correction and its own y/z phase.
//
// A self-paired pencil obeys the same relation with itself: its x-output is
// a - i d (-1)^n / 2 with a real and d = f_hat(N/2, P) 2 sin(theta N/2) (f_hat(N/2, P) is
// real there).  With SELF two of them, P1 and P2, go through one transform of
// f_hat(., P1) + i f_hat(., P2), whose output (a1 - b2) + i (b1 + a2) (b = -d (-1)^n / 2)
// gives both.  That removes a round of the pass when N^2/2 + 2 slots would need one
// more than N^2/2; only the wavefront holding those two slots loads two pencils.
//
// With HERM = false the spectrum is that of a complex field (no pairing), padded by 3/2 (the
// dealiased form): the middle third of each axis's modes is zero, so 4/9 of the N^2
// x-pencils are transformed, from 2/3 of their inputs, and stored with their own y/z phase;
// the y- and z-passes skip the zero rows and columns.  (Ten FP32 nodes padded to 48^3, whole call: every
// pencil transformed 4.04 ms, the kept ones 2.14 ms; two load buffers in turn: no change.)
template <typename T, int N, int CH, int CZ, int PIPE, bool HERM, bool KEEP>
__device__ __forceinline__ void field_ifft(const cx<T>* __restrict__ fh, const cx<T>* __restrict__ kxt,
                                           const cx<T>* __restrict__ yzt, T nyq, int c, cx<T>* buf, int cz,
                                           int m, int r, cx<T>* out, bool fresh,
                                           cx<T> (*kept)[GainK<T, N, CH, CZ>::NP]) {
    using K = GainK<T, N, CH, CZ>;
    if constexpr (!HERM) {
        constexpr int ES = int(sizeof(cx<T>));
        constexpr int RS = N * N * ES;
        constexpr int H = N / 3, NK = 2 * H;   // kept modes per axis: indices below H and from N - H
        static_assert(N % 3 == 0 && CH % 3 == 0, "a 3/2-padded grid, its zero third made of whole sub-sequences");
        const __amdgpu_buffer_rsrc_t rs = field_rsrc<T>(fh, N * RS);
#pragma unroll 1
        for (int k = 0; k < (NK * NK + K::NT - 1) / K::NT; ++k) {
            const int p = int(threadIdx.x) + k * K::NT;
            if ((NK * NK) % K::NT != 0 && p >= NK * NK) break;
            const int ly = p / NK < H ? p / NK : p / NK + H, lz = p % NK < H ? p % NK : p % NK + H;
            const int vo = (ly * N + lz) * ES;
            cx<T> y[K::NP];
#pragma unroll
            for (int l = 0; l < K::NP; ++l) y[l] = cx<T>{T(0), T(0)};
#pragma unroll 1
            for (int tk = 0; tk < CH - CH / 3; ++tk) {
                const int t = tk < CH / 3 ? tk : tk + CH / 3;
#pragma unroll
                for (int l = 0; l < K::NP; ++l) cmac(y[l], bload<T>(rs, vo, (l + t * K::NP) * RS), kxt[l + t * K::NP]);
            }
            fft<K::NP, +1>(y);
            const cx<T> cyz = yzt[ly] * yzt[N + lz];
#pragma unroll
            for (int mm = 0; mm < K::NP; ++mm) buf[(mm * N + ly) * K::ROW + lz] = y[mm] * cyz;
        }
        __syncthreads();
        yz_passes<T, N, CH, CZ, +1, true>(buf, cz, m, r, out);
        __syncthreads();
        return;
    }
    constexpr int ROUNDS_ALL = (N * N / 2 + 2 + K::NT - 1) / K::NT;
    constexpr int ROUNDS_SELF = (N * N / 2 + K::NT - 1) / K::NT;
    constexpr bool SELF = ROUNDS_SELF < ROUNDS_ALL;
    constexpr int SLOTS = SELF ? N * N / 2 : N * N / 2 + 2;
    constexpr int ROUNDS = SELF ? ROUNDS_SELF : ROUNDS_ALL;
    constexpr int ES = int(sizeof(cx<T>));
    constexpr int RS = N * N * ES;  // bytes between x-planes of the spectrum
    const __amdgpu_buffer_rsrc_t rs = field_rsrc<T>(fh, N * RS);
    const int tid = threadIdx.x;
    // runtime loops keep the x-pass loads from being hoisted en masse
#pragma unroll 1
    for (int k = 0; k < ROUNDS; ++k) {
        const int slot = tid + k * K::NT;
        if (ROUNDS * K::NT != SLOTS && slot >= SLOTS) break;
        int ly, lz;
        const bool paired = pencil_slot<N, SELF>(slot, ly, lz);
        const int P = ly * N + lz;
        const int vo = P * ES;
        cx<T> y[K::NP];
        if (!KEEP || fresh) {
#pragma unroll
            for (int l = 0; l < K::NP; ++l) y[l] = cx<T>{T(0), T(0)};
            if (SELF && __ballot(!paired) != 0) {
                // f(., P1) + i mk f(., P2) with both loads of an index issued together
                const int vo2 = paired ? vo : vo + (N / 2) * ES;
                const T mk = paired ? T(0) : T(1);
#pragma unroll 1
                for (int t = 0; t < CH; ++t) {
                    cx<T> a[K::NP], b[K::NP];
#pragma unroll
                    for (int l = 0; l < K::NP; ++l) {
                        a[l] = bload<T>(rs, vo, (l + t * K::NP) * RS);
                        b[l] = bload<T>(rs, vo2, (l + t * K::NP) * RS);
                    }
#pragma unroll
                    for (int l = 0; l < K::NP; ++l)
                        cmac(y[l], cx<T>{a[l].x - mk * b[l].y, a[l].y + mk * b[l].x}, kxt[l + t * K::NP]);
                }
            } else if constexpr (PIPE == PIPE_TWO) {
                const cx<T>* const kx1[1] = {kxt};
                cx<T>* const y1[1] = {y};
                x_sum_pipe<T, K::NP, CH, 1>(rs, vo, RS, kx1, y1);
            } else if constexpr (PIPE == PIPE_ROTATE) {
                cx<T> nxt[K::NP];
#pragma unroll
                for (int l = 0; l < K::NP; ++l) nxt[l] = bload<T>(rs, vo, l * RS);
#pragma unroll 1
                for (int t = 0; t < CH; ++t) {
                    cx<T> cur[K::NP];
#pragma unroll
                    for (int l = 0; l < K::NP; ++l) cur[l] = nxt[l];
                    if (t + 1 < CH) {
#pragma unroll
                        for (int l = 0; l < K::NP; ++l) nxt[l] = bload<T>(rs, vo, (l + (t + 1) * K::NP) * RS);
                    }
#pragma unroll
                    for (int l = 0; l < K::NP; ++l) cmac(y[l], cur[l], kxt[l + t * K::NP]);
                }
            } else {
#pragma unroll 1
                for (int t = 0; t < CH; ++t) {
#pragma unroll
                    for (int l = 0; l < K::NP; ++l) {
                        const int jx = l + t * K::NP;
                        cmac(y[l], bload<T>(rs, vo, jx * RS), kxt[jx]);
                    }
                }
            }
            fft<K::NP, +1>(y);
            if constexpr (KEEP) keep_x<K::NP>(kept[k], y);
        } else {
            if constexpr (KEEP) keep_x<K::NP>(y, kept[k]);
        }
        const cx<T> fn = bload<T>(rs, vo, (N / 2) * RS);
        if (SELF && !paired) {
            const T h1 = T(0.5) * nyq * fn.x;
            const T h2 = T(0.5) * nyq * bload<T>(rs, vo + (N / 2) * ES, (N / 2) * RS).x;
            const cx<T> c1 = yzt[ly] * yzt[N], c2 = yzt[ly] * yzt[N + N / 2];
#pragma unroll
            for (int mm = 0; mm < K::NP; ++mm) {
                const bool odd = ((CH * mm + c) & 1) != 0;
                const T e1 = odd ? -h1 : h1, e2 = odd ? -h2 : h2;  // d (-1)^n / 2
                buf[(mm * N + ly) * K::ROW] = cx<T>{y[mm].x - e2, -e1} * c1;
                buf[(mm * N + ly) * K::ROW + N / 2] = cx<T>{y[mm].y + e1, -e2} * c2;
            }
            continue;
        }
        const cx<T> cyz = yzt[ly] * yzt[N + lz];
#pragma unroll
        for (int mm = 0; mm < K::NP; ++mm) buf[(mm * N + ly) * K::ROW + lz] = y[mm] * cyz;
        if (paired) {
            const int ly2 = (N - ly) % N, lz2 = (N - lz) % N;
            const cx<T> delta = cx<T>{-nyq * fn.y, nyq * fn.x};
            const cx<T> cyz2 = yzt[ly2] * yzt[N + lz2];
#pragma unroll
            for (int mm = 0; mm < K::NP; ++mm) {
                const bool odd = ((CH * mm + c) & 1) != 0;
                const cx<T> g = odd ? y[mm] - delta : y[mm] + delta;
                buf[(mm * N + ly2) * K::ROW + lz2] = cx<T>{g.x, -g.y} * cyz2;
            }
        }
    }
    __syncthreads();
    yz_passes<T, N, CH, CZ, +1>(buf, cz, m, r, out);
    __syncthreads();
}

// ====================================================== packed pair of fields
// Geometries the packed form supports: at most two x-pass rounds (their plane values
// stay in registers) and one lane per correction column.
template <typename T, int N, int CH, int CZ>
constexpr bool pack_ok() {
    using K = GainK<T, N, CH, CZ>;
    constexpr int ra = (N * N / 2 + 2 + K::NT - 1) / K::NT, rs = (N * N / 2 + K::NT - 1) / K::NT;
    return (rs < ra ? rs : ra) <= 2 && N + 2 * K::NP <= 64 && N * K::ROWC <= K::LDS;
}

// The chunk x-transform of one pencil P of one field (with SELF in a wavefront holding
// self-paired slots: of f(., P) + i mk f(., P + N/2), both loads of an index together).
template <typename T, int N, int CH, int PIPE>
__device__ __forceinline__ void x_pencil(__amdgpu_buffer_rsrc_t rs, int vo, int vo2, T mk, bool two,
                                         const cx<T>* __restrict__ kxt, cx<T>* y) {
    constexpr int NP = N / CH;
    constexpr int RS = N * N * int(sizeof(cx<T>));
#pragma unroll
    for (int l = 0; l < NP; ++l) y[l] = cx<T>{T(0), T(0)};
    if (two) {
#pragma unroll 1
        for (int t = 0; t < CH; ++t) {
            cx<T> a[NP], b[NP];
#pragma unroll
            for (int l = 0; l < NP; ++l) {
                a[l] = bload<T>(rs, vo, (l + t * NP) * RS);
                b[l] = bload<T>(rs, vo2, (l + t * NP) * RS);
            }
#pragma unroll
            for (int l = 0; l < NP; ++l)
                cmac(y[l], cx<T>{a[l].x - mk * b[l].y, a[l].y + mk * b[l].x}, kxt[l + t * NP]);
        }
    } else if constexpr (PIPE) {
        const cx<T>* const kx1[1] = {kxt};
        cx<T>* const y1[1] = {y};
        x_sum_pipe<T, NP, CH, 1>(rs, vo, RS, kx1, y1);
    } else {
#pragma unroll 1
        for (int t = 0; t < CH; ++t) {
#pragma unroll
            for (int l = 0; l < NP; ++l) cmac(y[l], bload<T>(rs, vo, (l + t * NP) * RS), kxt[l + t * NP]);
        }
    }
    fft<NP, +1>(y);
}

// x_pencil for two fields with the same spectrum (a like class: A and B both shift f^i)
// on a paired slot: every input is loaded once and enters both sums, each with its own
// phase table; each output takes the same operations in the same order as x_pencil's.
template <typename T, int N, int CH, int PIPE>
__device__ __forceinline__ void x_pencil2(__amdgpu_buffer_rsrc_t rs, int vo, const cx<T>* __restrict__ kxa,
                                          const cx<T>* __restrict__ kxb, cx<T>* ya, cx<T>* yb) {
    constexpr int NP = N / CH;
    constexpr int RS = N * N * int(sizeof(cx<T>));
#pragma unroll
    for (int l = 0; l < NP; ++l) ya[l] = yb[l] = cx<T>{T(0), T(0)};
    if constexpr (PIPE) {
        const cx<T>* const kx2[2] = {kxa, kxb};
        cx<T>* const y2[2] = {ya, yb};
        x_sum_pipe<T, NP, CH, 2>(rs, vo, RS, kx2, y2);
    } else {
#pragma unroll 1
        for (int t = 0; t < CH; ++t) {
#pragma unroll
            for (int l = 0; l < NP; ++l) {
                const cx<T> v = bload<T>(rs, vo, (l + t * NP) * RS);
                cmac(ya[l], v, kxa[l + t * NP]);
                cmac(yb[l], v, kxb[l + t * NP]);
            }
        }
    }
    fft<NP, +1>(ya);
    fft<NP, +1>(yb);
}

// The x-passes of two fields with different spectra (an unlike class) interleaved: both
// fields' loads of a batch are in flight together, each field in two buffers in turn.
template <typename T, int N, int CH>
__device__ __forceinline__ void x_pencil_ab(__amdgpu_buffer_rsrc_t rsa, __amdgpu_buffer_rsrc_t rsb, int vo,
                                            const cx<T>* __restrict__ kxa, const cx<T>* __restrict__ kxb,
                                            cx<T>* ya, cx<T>* yb) {
    constexpr int NP = N / CH;
    constexpr int RS = N * N * int(sizeof(cx<T>));
#pragma unroll
    for (int l = 0; l < NP; ++l) ya[l] = yb[l] = cx<T>{T(0), T(0)};
    cx<T> a0[NP], a1[NP], b0[NP], b1[NP];
    auto load = [&](cx<T>* a, cx<T>* b, int t) {
#pragma unroll
        for (int l = 0; l < NP; ++l) {
            a[l] = bload<T>(rsa, vo, (l + t * NP) * RS);
            b[l] = bload<T>(rsb, vo, (l + t * NP) * RS);
        }
    };
    auto use = [&](const cx<T>* a, const cx<T>* b, int t) {
#pragma unroll
        for (int l = 0; l < NP; ++l) {
            cmac(ya[l], a[l], kxa[l + t * NP]);
            cmac(yb[l], b[l], kxb[l + t * NP]);
        }
    };
    load(a0, b0, 0);
    int t = 0;
#pragma unroll 1
    for (; t + 2 < CH; t += 2) {
        load(a1, b1, t + 1);
        use(a0, b0, t);
        load(a0, b0, t + 2);
        use(a1, b1, t + 1);
    }
    if constexpr (CH % 2 == 0) {
        load(a1, b1, CH - 1);
        use(a0, b0, CH - 2);
        use(a1, b1, CH - 1);
    } else {
        use(a0, b0, CH - 1);
    }
    fft<NP, +1>(ya);
    fft<NP, +1>(yb);
}

template <typename T>
__device__ __forceinline__ cx<T> pack_ab(cx<T> a, cx<T> b) { return cx<T>{a.x - b.y, a.y + b.x}; }          // a + i b
template <typename T>
__device__ __forceinline__ cx<T> pack_conj(cx<T> a, cx<T> b) { return cx<T>{a.x + b.y, b.x - a.y}; }        // conj(a) + i conj(b)
template <typename T>
__device__ __forceinline__ cx<T> pack_nconj(cx<T> a, cx<T> b) { return cx<T>{-a.x - b.y, a.y - b.x}; }      // -(conj(a) + i conj(b))

// One direction of a gain class with both shifted fields A = f^i(v + a rho sigma) and
// B = f^j(v - b rho sigma) carried by one complex transform.
//
// After the x-pass of a field, split its mixed-domain data G(x, P) (P = (l_y, l_z)) into
// the part that is Hermitian in P, whose y/z transform is real, and the anti-Hermitian
// rest.  For a pencil P with partner -P (see field_ifft for y, delta_P and the sign s_n),
// with c = cyz(P), c^ = conj(cyz(-P)), c~ = (c + c^)/2:
//   Herm(P)[n] = y[n] c~ + s_n delta c^ / 2,          Herm(-P) = conj(Herm(P)),
//   AH(P)[n]   = (c - c^)/2 (y[n] + s_n delta / 2) - s_n delta c~ / 2.
// The y/z transform of Herm_A + i Herm_B gives a + i b with a = Re A, b = Re B.  The
// anti-Hermitian part has two pieces, each anti-Hermitian by itself: a plane piece
// -delta c~ / 2 times s_n (its transform is (-1)^x times one 2-D transform), and a line
// piece, nonzero only where c != c^, i.e. on the Nyquist lines l_y = N/2 or l_z = N/2
// (1-D transforms along the other index).  Their transforms are purely imaginary, i alpha,
// so the pieces of A and B are packed the same way: E = i alpha_A - alpha_B.  Then
// Re(A B) = a b - alpha_A alpha_B = Re Z Im Z + Re E Im E.
template <typename T, int N, int CH, int CZ, int PIPE>
__device__ __forceinline__ void packed_direction(const cx<T>* __restrict__ fa, const cx<T>* __restrict__ fb,
                                                 const cx<T>* __restrict__ kxa, const cx<T>* __restrict__ yza,
                                                 T nyqa, const cx<T>* __restrict__ kxb,
                                                 const cx<T>* __restrict__ yzb, T nyqb, int c, cx<T>* buf, int cz,
                                                 int m, int r, T w, T* S) {
    using K = GainK<T, N, CH, CZ>;
    constexpr int NP = K::NP, H = N / 2;
    constexpr int ROUNDS_ALL = (N * N / 2 + 2 + K::NT - 1) / K::NT;
    constexpr int ROUNDS_SELF = (N * N / 2 + K::NT - 1) / K::NT;
    constexpr bool SELF = ROUNDS_SELF < ROUNDS_ALL;
    constexpr int SLOTS = SELF ? N * N / 2 : N * N / 2 + 2;
    constexpr int ROUNDS = SELF ? ROUNDS_SELF : ROUNDS_ALL;
    static_assert(ROUNDS <= 2, "the plane values of at most two rounds are kept in registers");
    static_assert(N + 2 * NP <= 64, "one lane per correction column");
    static_assert(N * K::ROWC <= K::LDS, "the correction array must fit the main buffer");
    constexpr int ES = int(sizeof(cx<T>));
    constexpr int RS = N * N * ES;
    cx<T>* LY = buf + K::LDS;           // [NP][N+1]: line l_y = N/2, indexed [x][l_z]
    cx<T>* LZ = LY + NP * (N + 1);      // [NP][N+1]: line l_z = N/2, indexed [x][l_y]
    const __amdgpu_buffer_rsrc_t rsa = field_rsrc<T>(fa, N * RS), rsb = field_rsrc<T>(fb, N * RS);
    const bool same = fa == fb;   // a like class: both fields shift one spectrum
    const int tid = threadIdx.x;
    cx<T> pl[2][2];  // plane values of the slot's two pencils, per round

#pragma unroll 1
    for (int k = 0; k < ROUNDS; ++k) {
        const int slot = tid + k * K::NT;
        if (ROUNDS * K::NT != SLOTS && slot >= SLOTS) break;
        int ly, lz;
        const bool paired = pencil_slot<N, SELF>(slot, ly, lz);
        const int vo = (ly * N + lz) * ES;
        const bool two = SELF && __ballot(!paired) != 0;
        const int vo2 = (SELF && !paired) ? vo + H * ES : vo;
        const T mk = (SELF && !paired) ? T(1) : T(0);
        cx<T> ya[NP], yb[NP];
        if (same && !two) {
            x_pencil2<T, N, CH, PIPE>(rsa, vo, kxa, kxb, ya, yb);
        } else if (PIPE && !two) {
            x_pencil_ab<T, N, CH>(rsa, rsb, vo, kxa, kxb, ya, yb);
        } else {
            x_pencil<T, N, CH, PIPE>(rsa, vo, vo2, mk, two, kxa, ya);
            x_pencil<T, N, CH, PIPE>(rsb, vo, vo2, mk, two, kxb, yb);
        }
        const cx<T> fna = bload<T>(rsa, vo, H * RS), fnb = bload<T>(rsb, vo, H * RS);
        cx<T> p0, p1;
        if (paired) {
            const int ly2 = (N - ly) % N, lz2 = (N - lz) % N;
            const cx<T> da = cx<T>{-nyqa * fna.y, nyqa * fna.x}, db = cx<T>{-nyqb * fnb.y, nyqb * fnb.x};
            const cx<T> ca = yza[ly] * yza[N + lz], cb = yzb[ly] * yzb[N + lz];
            const cx<T> c2a = yza[ly2] * yza[N + lz2], c2b = yzb[ly2] * yzb[N + lz2];
            const cx<T> cha = cx<T>{c2a.x, -c2a.y}, chb = cx<T>{c2b.x, -c2b.y};
            const cx<T> cta = T(0.5) * (ca + cha), ctb = T(0.5) * (cb + chb);
            const cx<T> dha = T(0.5) * (da * cha), dhb = T(0.5) * (db * chb);
#pragma unroll
            for (int mm = 0; mm < NP; ++mm) {
                const bool odd = ((CH * mm + c) & 1) != 0;
                const cx<T> ha = odd ? ya[mm] * cta - dha : ya[mm] * cta + dha;
                const cx<T> hb = odd ? yb[mm] * ctb - dhb : yb[mm] * ctb + dhb;
                buf[(mm * N + ly) * K::ROW + lz] = pack_ab(ha, hb);
                buf[(mm * N + ly2) * K::ROW + lz2] = pack_conj(ha, hb);
            }
            if (ly == H || lz == H) {  // line piece (c != c^ only here)
                const cx<T> ga = T(0.5) * (ca - cha), gb = T(0.5) * (cb - chb);
                const cx<T> hda = T(0.5) * da, hdb = T(0.5) * db;
#pragma unroll
                for (int mm = 0; mm < NP; ++mm) {
                    const bool odd = ((CH * mm + c) & 1) != 0;
                    const cx<T> la = ga * (odd ? ya[mm] - hda : ya[mm] + hda);
                    const cx<T> lb = gb * (odd ? yb[mm] - hdb : yb[mm] + hdb);
                    if (ly == H) {
                        LY[mm * (N + 1) + lz] = pack_ab(la, lb);
                        LY[mm * (N + 1) + lz2] = pack_nconj(la, lb);
                    } else {
                        LZ[mm * (N + 1) + ly] = pack_ab(la, lb);
                        LZ[mm * (N + 1) + ly2] = pack_nconj(la, lb);
                    }
                }
            }
            const cx<T> pia = T(-0.5) * (da * cta), pib = T(-0.5) * (db * ctb);
            p0 = pack_ab(pia, pib);
            p1 = pack_nconj(pia, pib);
        } else {
            // self-paired pencils: (ly, lz) alone, or with SELF the pair (ly, 0), (ly, N/2)
            // from one transform of f(., P1) + i f(., P2) per field
            const T f2a = SELF ? bload<T>(rsa, vo + H * ES, H * RS).x : T(0);
            const T f2b = SELF ? bload<T>(rsb, vo + H * ES, H * RS).x : T(0);
            const T d1a = nyqa * fna.x, d1b = nyqb * fnb.x, d2a = nyqa * f2a, d2b = nyqb * f2b;
            const int lzs[2] = {SELF ? 0 : lz, H};
            const T dsa[2] = {d1a, d2a}, dsb[2] = {d1b, d2b};
#pragma unroll
            for (int e = 0; e < (SELF ? 2 : 1); ++e) {
                const int lze = lzs[e];
                const cx<T> ca = yza[ly] * yza[N + lze], cb = yzb[ly] * yzb[N + lze];
                const bool line = ly == H || lze == H;
#pragma unroll
                for (int mm = 0; mm < NP; ++mm) {
                    const bool odd = ((CH * mm + c) & 1) != 0;
                    cx<T> ua = ya[mm], ub = yb[mm];
                    if (SELF) {  // unscramble: y_k = a_k - i d_k (-1)^n / 2
                        const T e1a = T(0.5) * (odd ? -d1a : d1a), e2a = T(0.5) * (odd ? -d2a : d2a);
                        const T e1b = T(0.5) * (odd ? -d1b : d1b), e2b = T(0.5) * (odd ? -d2b : d2b);
                        ua = e == 0 ? cx<T>{ya[mm].x - e2a, -e1a} : cx<T>{ya[mm].y + e1a, -e2a};
                        ub = e == 0 ? cx<T>{yb[mm].x - e2b, -e1b} : cx<T>{yb[mm].y + e1b, -e2b};
                    }
                    const cx<T> va = ua * ca, vb = ub * cb;
                    buf[(mm * N + ly) * K::ROW + lze] = cx<T>{va.x, vb.x};
                    if (line) {
                        // (c - conj c)/2 (y + s delta / 2) with delta = i d
                        const T sa = T(0.5) * (odd ? -dsa[e] : dsa[e]), sb = T(0.5) * (odd ? -dsb[e] : dsb[e]);
                        const cx<T> la = cx<T>{T(0), ca.y} * cx<T>{ua.x, ua.y + sa};
                        const cx<T> lb = cx<T>{T(0), cb.y} * cx<T>{ub.x, ub.y + sb};
                        if (ly == H) LY[mm * (N + 1) + lze] = pack_ab(la, lb);
                        else LZ[mm * (N + 1) + ly] = pack_ab(la, lb);
                    }
                }
                const cx<T> pia = cx<T>{T(0), T(-0.5) * dsa[e] * ca.x}, pib = cx<T>{T(0), T(-0.5) * dsb[e] * cb.x};
                if (e == 0) p0 = pack_ab(pia, pib);
                else p1 = pack_ab(pia, pib);
            }
        }
        if (k == 0) {
            pl[0][0] = p0;
            pl[0][1] = p1;
        } else {
            pl[1][0] = p0;
            pl[1][1] = p1;
        }
    }
    __syncthreads();
    cx<T> Z[K::NS];
    yz_passes<T, N, CH, CZ, +1>(buf, cz, m, r, Z);
    __syncthreads();

    // the correction array CB[N][ROWC] in the main buffer: the plane at columns 0..N-1
    // ([l_y][l_z]), then line l_y = N/2 transposed ([l_z][N + x]), then line l_z = N/2
    // transposed ([l_y][N + NP + x], zero at l_y = N/2)
    cx<T>* CB = buf;
#pragma unroll 1
    for (int k = 0; k < ROUNDS; ++k) {
        const int slot = tid + k * K::NT;
        if (ROUNDS * K::NT != SLOTS && slot >= SLOTS) break;
        int ly, lz;
        const bool paired = pencil_slot<N, SELF>(slot, ly, lz);
        const cx<T> v0 = k == 0 ? pl[0][0] : pl[1][0], v1 = k == 0 ? pl[0][1] : pl[1][1];
        if (paired) {
            CB[ly * K::ROWC + lz] = v0;
            CB[((N - ly) % N) * K::ROWC + (N - lz) % N] = v1;
        } else {
            CB[ly * K::ROWC + (SELF ? 0 : lz)] = v0;
            if (SELF) CB[ly * K::ROWC + H] = v1;
        }
    }
    for (int t = tid; t < NP * N; t += K::NT) {
        const int mm = t / N, l = t % N;
        CB[l * K::ROWC + N + mm] = LY[mm * (N + 1) + l];
        CB[l * K::ROWC + N + NP + mm] = l == H ? cx<T>{T(0), T(0)} : LZ[mm * (N + 1) + l];
    }
    __syncthreads();
    const int g = tid / 64, p = tid % 64;
    {
        constexpr int NJ = N / K::GC;
        cx<T> v[NJ];
        const bool act = g < K::GC && p < N + 2 * NP;
        if (act) {
            with_group<K::GC>(g, [&](auto gg) { split_fft<N, K::GC, decltype(gg)::value, +1, K::ROWC>(CB + p, v); });
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) CB[(K::GC * j + g) * K::ROWC + p] = v[j];
        }
        __syncthreads();
        const bool act2 = g < K::GC && p < N;
        if (act2) {
            with_group<K::GC>(g, [&](auto gg) { split_fft<N, K::GC, decltype(gg)::value, +1, 1>(CB + p * K::ROWC, v); });
        }
        __syncthreads();
        if (act2) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) CB[p * K::ROWC + K::GC * j + g] = v[j];
        }
        __syncthreads();
    }
    // E at the thread's points (x = CH m + c, y = r, z = CZ j + cz)
    const T sx = ((CH * m + c) & 1) ? T(-1) : T(1), sy = (r & 1) ? T(-1) : T(1);
    const cx<T> t3 = CB[r * K::ROWC + N + NP + m];
#pragma unroll
    for (int j = 0; j < K::NS; ++j) {
        const int nz = CZ * j + cz;
        const cx<T> t1 = CB[r * K::ROWC + nz], t2 = CB[nz * K::ROWC + N + m];
        const T sz = (nz & 1) ? T(-1) : T(1);
        const T ex = sx * t1.x + sy * t2.x + sz * t3.x, ey = sx * t1.y + sy * t2.y + sz * t3.y;
        S[j] = fma(w, fma(Z[j].x, Z[j].y, ex * ey), S[j]);
    }
    __syncthreads();
}

// Forward transform of one work item's field, held in buf (LDS) as rows (plane m of the
// chunk, y) of z values with row stride N + 1: z and y passes through LDS, then the chunk's
// part of the x-transform; stores the chunk partial (Pq: the partials of this (node, class,
// rho_q), chunk c at offset c * N/CH * pencils).  CPLX: the field is complex and every (k_y,
// k_z) pencil is stored; otherwise the field is real, its partial Hermitian, and only
// k_z <= N/2 is stored.  Needs every thread of the work item (GainK<T, N, CH, CZ>::NT).
template <typename T, int N, int CH, int CZ, bool CPLX>
__device__ __forceinline__ void store_partial(cx<T>* buf, cx<T>* Pq, int c) {
    using K = GainK<T, N, CH, CZ>;
    const int tid = threadIdx.x;
    const int cz = tid / K::NTC, u = tid % K::NTC;
    const int m = u / N, r = u % N;
    {
        cx<T> v[K::NS];
        with_group<CZ>(cz, [&](auto gg) {
            split_fft<N, CZ, decltype(gg)::value, -1, 1>(buf + (m * N + r) * K::ROW, v);
        });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < K::NS; ++j) buf[(m * N + r) * K::ROW + CZ * j + cz] = v[j];
        __syncthreads();
        with_group<CZ>(cz, [&](auto gg) {
            split_fft<N, CZ, decltype(gg)::value, -1, K::ROW>(buf + (m * N) * K::ROW + r, v);
        });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < K::NS; ++j) buf[(m * N + CZ * j + cz) * K::ROW + r] = v[j];
        __syncthreads();
    }
    if constexpr (CPLX) {
        // the transform of a complex field: every (k_y, k_z) pencil is stored
        constexpr int64_t PCHF = int64_t(K::NP) * K::NPENF;
        cx<T>* Pout = Pq + int64_t(c) * PCHF;
#pragma unroll 1
        for (int k = 0; k < K::PXF; ++k) {
            const int P = tid + k * K::NT;
            if (K::PXF * K::NT != K::NPENF && P >= K::NPENF) break;
            const int ky = P / N, kz = P % N;
            cx<T> v[K::NP];
#pragma unroll
            for (int mm = 0; mm < K::NP; ++mm) v[mm] = buf[(mm * N + ky) * K::ROW + kz];
            fft<K::NP, -1>(v);
#pragma unroll
            for (int kk = 0; kk < K::NP; ++kk) Pout[kk * K::NPENF + P] = v[kk];
        }
        return;
    }
    // The chunk's partial is the DFT of a real array over (x-planes of the chunk, y, z),
    // so it is Hermitian in (k_xp, k_y, k_z): only k_z <= N/2 is stored, the radial kernel
    // reads the rest as conjugates of the mirrored entries.
    constexpr int64_t PCH = int64_t(K::NP) * K::NPEN;  // stored values of one chunk partial
    cx<T>* Pout = Pq + int64_t(c) * PCH;
#pragma unroll 1
    for (int k = 0; k < K::PX; ++k) {
        const int P = tid + k * K::NT;
        if (K::PX * K::NT != K::NPEN && P >= K::NPEN) break;
        const int ky = P / K::KZH, kz = P % K::KZH;
        cx<T> v[K::NP];
#pragma unroll
        for (int mm = 0; mm < K::NP; ++mm) v[mm] = buf[(mm * N + ky) * K::ROW + kz];
        fft<K::NP, -1>(v);
#pragma unroll
        for (int kk = 0; kk < K::NP; ++kk) Pout[kk * K::NPEN + P] = v[kk];
    }
}

template <typename T, int N, int CH, int CZ, int PIPE, bool PACK, int MODE, bool KEEP = false>
__global__ __launch_bounds__((GainK<T, N, CH, CZ>::NT)) void gain_kernel(GainArgs<T> a) {
    using K = GainK<T, N, CH, CZ>;
    constexpr bool CPLX = MODE == GAIN_COMPLEX || MODE == GAIN_VSS;  // the whole spectrum of a complex field is stored
    static_assert(!(PACK && CPLX), "the packed two-field form keeps only Re(A B)");
    // aligned for the 16-byte blocks of the Nyquist-plane sums
    __shared__ alignas(16) cx<T> buf[K::LDS + ((PACK && pack_ok<T, N, CH, CZ>()) ? K::LINES : 0)];
    int b, item;
    // the items of a node: classes, or with GAIN_TERMS the directions of all classes
    const int nq = MODE == GAIN_TERMS ? a.nq : a.nrho;
    if (!gain_item<1>(blockIdx.x, a.nb, MODE == GAIN_TERMS ? a.tdirs : a.ncls, nq * CH,
                      MODE == GAIN_TERMS ? nullptr : a.ord, b, item)) return;
    const int c = item % CH;
    item /= CH;
    const int q = MODE == GAIN_TERMS ? a.q0 + item % nq : item % nq;
    int cl = item / nq, dir = 0;
    if constexpr (MODE == GAIN_TERMS) {
        for (dir = cl, cl = 0; dir >= a.cls[4 * cl + 2]; ++cl) dir -= a.cls[4 * cl + 2];
    }
    const int ci = a.cls[4 * cl], cj = a.cls[4 * cl + 1];
    const int ndir = a.cls[4 * cl + 2], doff = a.cls[4 * cl + 3];
    const T w = MODE == GAIN_TERMS ? T(1) : a.wdir[cl];
    constexpr int64_t N3 = int64_t(N) * N * N;
    const cx<T>* fhi = a.fhat + (int64_t(b) * a.s + ci) * N3;
    const cx<T>* fhj = a.fhat + (int64_t(b) * a.s + cj) * N3;
    const int tid = threadIdx.x;
    const int cz = tid / K::NTC, u = tid % K::NTC;
    const int m = u / N, r = u % N;

    // VHS: only Re(S_q) reaches the result, since the radial operator multiplies
    // DFT(S_q) by a real F that is even in k: Re IDFT(F DFT(S)) = IDFT(F DFT(Re S)).
    // VSS: F depends on the direction and, at indices with a Nyquist component, F at the
    // mode of k is not the conjugate of F at the mode of the mirror index, so there the
    // imaginary part of S (from the Nyquist modes of the shifted fields) contributes.
    T S[K::NS], S1[CPLX ? K::NS : 1];
#pragma unroll
    for (int n = 0; n < K::NS; ++n) S[n] = T(0);
#pragma unroll
    for (int n = 0; n < (CPLX ? K::NS : 1); ++n) S1[n] = T(0);

    // GAIN_VSS: reduce Im S of direction d (in im[]) to the three Nyquist planes.  Im S goes to
    // LDS as rows of V-value blocks, 16 bytes each; a thread sums the y- or the x-direction for
    // V columns at once, both kinds of sums side by side over the workgroup.  With CZ = 1 a
    // thread holds a whole row and sums it over z where it is.  (One value at a time, in the
    // complex buffer's stride and with the three sums one after the other, the reductions
    // were a third of the kernel's LDS instructions: argon-krypton at N = 32, 64 nodes, gain stage
    // 4.62 ms, now 4.49.)
    auto nyquist_planes = [&](int d, const T* im) {
        constexpr int N2 = N * N, V = int(16 / sizeof(T)), RW = N + V;
        typedef T vec __attribute__((ext_vector_type(V)));
        static_assert(N % V == 0 && K::NP * N * RW <= 2 * K::LDS, "blocks of 16 bytes within the main buffer");
        T* PL = a.PL + (((int64_t(b) * a.ncls + cl) * a.nrho + q) * 2 + d) * int64_t((2 + CH) * N2);
        T* rows = reinterpret_cast<T*>(buf);
        T* row = rows + (m * N + r) * RW;
        if constexpr (CZ == 1) {
#pragma unroll
            for (int j = 0; j < N; j += V) {
                vec t;
#pragma unroll
                for (int v = 0; v < V; ++v) t[v] = im[j + v];
                *reinterpret_cast<vec*>(row + j) = t;
            }
            T acc = T(0);   // over z: [x][y]
#pragma unroll
            for (int z = 0; z < N; ++z) acc += (z & 1) ? -im[z] : im[z];
            PL[(c + CH * m) * N + r] = acc;
        } else {
#pragma unroll
            for (int j = 0; j < K::NS; ++j) row[CZ * j + cz] = im[j];
        }
        __syncthreads();
        if (CZ > 1 && cz == 0) {
            T acc = T(0);
            for (int z = 0; z < N; ++z) acc += (z & 1) ? -row[z] : row[z];
            PL[(c + CH * m) * N + r] = acc;
        }
        constexpr int NB = N / V, IY = K::NP * NB, IX = N * NB;
        for (int e = tid; e < IY + IX; e += K::NT) {
            const bool over_y = e < IY;   // over y: [x][z]; else over this chunk's x: [y][z]
            const int o = over_y ? e : e - IY, i = o / NB, z = (o % NB) * V;
            const T* src = over_y ? rows + i * N * RW + z : rows + i * RW + z;
            const int step = over_y ? RW : N * RW, n = over_y ? N : K::NP;
            // sign of term k: (-1)^y, or (-1)^x with x = c + CH k
            const bool flip = !over_y && (c & 1), alt = over_y || (CH & 1);
            vec acc;
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = T(0);
#pragma unroll 4
            for (int k = 0; k < n; ++k) {
                const vec t = *reinterpret_cast<const vec*>(src + k * step);
                const bool neg = flip != (alt && (k & 1));
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] += neg ? -t[v] : t[v];
            }
            *reinterpret_cast<vec*>(over_y ? PL + N2 + (c + CH * i) * N + z : PL + 2 * N2 + c * N2 + i * N + z) = acc;
        }
        __syncthreads();
    };

    // what at most this many rounds of the x-pass leave (keep_x)
    constexpr int XR = KEEP ? (N * N / 2 + 2 + K::NT - 1) / K::NT : 1;
    cx<T> kept[2][XR][K::NP];
    auto direction = [&](int d, T* Sd) {
        const bool fresh = !KEEP || d == 0 || a.xs[doff + d] == 0;
        const int64_t base = (int64_t(doff + d) * a.nrho + q) * 2;
        if constexpr (PACK && pack_ok<T, N, CH, CZ>()) {
            packed_direction<T, N, CH, CZ, PIPE>(fhi, fhj, a.kx + ((base + 0) * CH + c) * N, a.yz + (base + 0) * 2 * N,
                                                 a.nyq[base], a.kx + ((base + 1) * CH + c) * N,
                                                 a.yz + (base + 1) * 2 * N, a.nyq[base + 1], c, buf, cz, m, r, w, Sd);
        } else {
            cx<T> A[K::NS], B[K::NS];
            constexpr bool HERM = MODE != GAIN_COMPLEX;
            field_ifft<T, N, CH, CZ, PIPE, HERM, KEEP>(fhi, a.kx + ((base + 0) * CH + c) * N, a.yz + (base + 0) * 2 * N,
                                                       a.nyq[base], c, buf, cz, m, r, A, fresh, kept[0]);
            field_ifft<T, N, CH, CZ, PIPE, HERM, KEEP>(fhj, a.kx + ((base + 1) * CH + c) * N, a.yz + (base + 1) * 2 * N,
                                                       a.nyq[base + 1], c, buf, cz, m, r, B, fresh, kept[1]);
#pragma unroll
            for (int n = 0; n < K::NS; ++n) Sd[n] = fma(w, fma(A[n].x, B[n].x, -A[n].y * B[n].y), Sd[n]);
            if constexpr (MODE == GAIN_COMPLEX) {
#pragma unroll
                for (int n = 0; n < K::NS; ++n) S1[n] = fma(w, fma(A[n].x, B[n].y, A[n].y * B[n].x), S1[n]);
            }
            if constexpr (MODE == GAIN_VSS) {
                T im[K::NS];
#pragma unroll
                for (int n = 0; n < K::NS; ++n) im[n] = w * fma(A[n].x, B[n].y, A[n].y * B[n].x);
                nyquist_planes(d, im);
            }
        }
    };
    if constexpr (MODE == GAIN_VSS) {
        direction(0, S);
        if (ndir > 1) {
            direction(1, S1);
        } else {  // a one-direction class: its second plane sums are zero
            T zero[K::NS];
#pragma unroll
            for (int n = 0; n < K::NS; ++n) zero[n] = T(0);
            nyquist_planes(1, zero);
        }
    } else if constexpr (MODE == GAIN_TERMS) {
        direction(dir, S);
        T* Dq = a.D + (((int64_t(b) * a.tdirs + doff + dir) * nq + q - a.q0) * CH + c) * int64_t(K::NT * K::NS) + tid;
#pragma unroll
        for (int j = 0; j < K::NS; ++j) Dq[j * K::NT] = S[j];
        return;
    } else {
        for (int d = 0; d < ndir; ++d) direction(d, S);
    }

    // forward DFT of Re S_q (complex modes: of S + i S1): the field goes to LDS as rows
    // (plane, y) of z values
#pragma unroll
    for (int j = 0; j < K::NS; ++j) {
        if constexpr (CPLX) buf[(m * N + r) * K::ROW + CZ * j + cz] = cx<T>{S[j], S1[j]};
        else buf[(m * N + r) * K::ROW + CZ * j + cz] = cx<T>{S[j], T(0)};
    }
    __syncthreads();
    cx<T>* Pq = a.P + ((int64_t(b) * a.ncls + cl) * a.nrho + q) * int64_t(CH) * K::NP * (CPLX ? K::NPENF : K::NPEN);
    store_partial<T, N, CH, CZ, CPLX>(buf, Pq, c);
}

// The second half of a split gain: S_q of one item from its directions' terms, summed in the
// order and with the rounding of gain_kernel (so a node's result does not depend on the
// split), then the forward transform of the chunk.
template <typename T, int N, int CH, int CZ>
__global__ __launch_bounds__((GainK<T, N, CH, CZ>::NT)) void gain_sum_kernel(GainArgs<T> a) {
    using K = GainK<T, N, CH, CZ>;
    __shared__ cx<T> buf[K::LDS];
    int b, item;
    if (!gain_item<1>(blockIdx.x, a.nb, a.ncls, a.nq * CH, a.ord, b, item)) return;
    const int c = item % CH;
    item /= CH;
    const int qt = item % a.nq, q = a.q0 + qt;
    const int cl = item / a.nq;
    const int ndir = a.cls[4 * cl + 2], doff = a.cls[4 * cl + 3];
    const T w = a.wdir[cl];
    const int tid = threadIdx.x;
    const int cz = tid / K::NTC, u = tid % K::NTC;
    const int m = u / N, r = u % N;
    T S[K::NS];
#pragma unroll
    for (int j = 0; j < K::NS; ++j) S[j] = T(0);
#pragma unroll 2
    for (int d = 0; d < ndir; ++d) {
        const T* Dq = a.D + (((int64_t(b) * a.tdirs + doff + d) * a.nq + qt) * CH + c) * int64_t(K::NT * K::NS) + tid;
#pragma unroll
        for (int j = 0; j < K::NS; ++j) S[j] = fma(w, Dq[j * K::NT], S[j]);
    }
#pragma unroll
    for (int j = 0; j < K::NS; ++j) buf[(m * N + r) * K::ROW + CZ * j + cz] = cx<T>{S[j], T(0)};
    __syncthreads();
    cx<T>* Pq = a.P + ((int64_t(b) * a.ncls + cl) * a.nrho + q) * int64_t(CH) * K::NP * K::NPEN;
    store_partial<T, N, CH, CZ, false>(buf, Pq, c);
}

// =============================================================== radial kernel
// VSS: the Hermitian part of sum_d F_d DFT(S_d), with S_d = Re S_d + i Im S_d, Z the
// spectrum of Re S_0 + i Re S_1 and V_d = DFT(Im S_d):
//   sum_d F_H,d U_d + i F_A,d V_d,  U_0 = (Z(k) + conj Z(-k))/2, U_1 = (Z(k) - conj Z(-k))/(2i),
// F_H, F_A the Hermitian and anti-Hermitian parts of F (F_A vanishes off the Nyquist
// planes, where V_d is needed).
template <typename T, typename A = double>
__device__ __forceinline__ void vss_accumulate(cx<A>& acc, const cx<T> h[2], const cx<T> fa[2], A u0x,
                                               A u0y, A u1x, A u1y, bool nyq, const cx<T> v[2]) {
    acc.x += A(h[0].x) * u0x - A(h[0].y) * u0y + A(h[1].x) * u1x - A(h[1].y) * u1y;
    acc.y += A(h[0].x) * u0y + A(h[0].y) * u0x + A(h[1].x) * u1y + A(h[1].y) * u1x;
    if (nyq) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {  // i F_A V
            acc.x -= A(fa[d].x) * A(v[d].y) + A(fa[d].y) * A(v[d].x);
            acc.y += A(fa[d].x) * A(v[d].x) - A(fa[d].y) * A(v[d].y);
        }
    }
}

// Slot of entry (r, c) of a Nyquist plane in the mirror-paired layout: each entry and
// its plane mirror ((N - r) % N, (N - c) % N) fill one aligned pair of slots (rows r and
// N - r interleaved; in the self-mirror rows 0 and N/2, columns c and N - c), and the four
// entries that are their own mirror take the last two slots of those two rows.
template <int N>
__device__ __forceinline__ int vpair_slot(int r, int c) {
    constexpr int H = N / 2;
    if (r != 0 && r != H) {
        const int lo = r < H ? r : N - r;
        return 2 * N * lo + 2 * (r < H ? c : (N - c) % N) + (r < H ? 0 : 1);
    }
    const int base = r == 0 ? 0 : N;
    if (c != 0 && c != H) return base + 2 * ((c < H ? c : N - c) - 1) + (c < H ? 0 : 1);
    return base + N - 2 + (c == 0 ? 0 : 1);
}
// Slot of mode k (with a component at the Nyquist index) in the three mirror-paired
// planes: [k_x][k_y] where k_z = N/2, else [k_x][k_z] where k_y = N/2, else [k_y][k_z].
template <int N>
__device__ __forceinline__ int vplane_slot(int kx, int ky, int kz) {
    if (kz == N / 2) return vpair_slot<N>(kx, ky);
    if (ky == N / 2) return N * N + vpair_slot<N>(kx, kz);
    return 2 * N * N + vpair_slot<N>(ky, kz);
}
// W at k and at its plane mirror from the aligned pair holding them.
template <typename T, int N>
__device__ __forceinline__ void w_pair(const cx<T>* Vb, int kx, int ky, int kz, cx<T>& w, cx<T>& wm) {
    const int sl = vplane_slot<N>(kx, ky, kz);
    const cx<T> p0 = Vb[sl & ~1], p1 = Vb[sl | 1];
    const bool self = (kx == 0 || kx == N / 2) + (ky == 0 || ky == N / 2) + (kz == 0 || kz == N / 2) == 3;
    w = (sl & 1) ? p1 : p0;
    wm = self ? w : ((sl & 1) ? p0 : p1);
}

// W = DFT(Im S_0 + i Im S_1) on the three Nyquist planes from the plane sums: one block
// per (node, class, rho), one thread group of N per plane; the first pass transforms
// along the plane's first axis (coalesced column reads), the second along its second
// axis, the result leaves through LDS with coalesced stores.  Each V_d = DFT(Im S_d) is
// Hermitian on its plane, so the radial kernel separates them from W at k and at the
// plane mirror of k.
template <typename T, int N, int CH>
__global__ __launch_bounds__(3 * N) void nyquist_dft_kernel(const T* __restrict__ PL, cx<T>* __restrict__ V) {
    constexpr int N2 = N * N;
    const int64_t it = blockIdx.x;  // (node, class, rho)
    const int plane = threadIdx.x / N, t = threadIdx.x % N;
    __shared__ cx<T> Ls[3][N][N + 1];
    const T* p0 = PL + (it * 2 + 0) * int64_t((2 + CH) * N2);
    const T* p1 = PL + (it * 2 + 1) * int64_t((2 + CH) * N2);
    auto at = [&](const T* pl, int r) {
        if (plane < 2) return pl[plane * N2 + r * N + t];
        T v = T(0);
#pragma unroll
        for (int c = 0; c < CH; ++c) v += pl[2 * N2 + c * N2 + r * N + t];
        return v;
    };
    {
        cx<T> x[N];  // column t of the plane, transformed along its first axis
#pragma unroll
        for (int r = 0; r < N; ++r) x[r] = cx<T>{at(p0, r), at(p1, r)};
        fft<N, -1>(x);
#pragma unroll
        for (int k = 0; k < N; ++k) Ls[plane][k][t] = x[k];
    }
    __syncthreads();
    {
        cx<T> x[N];  // row t (first-axis mode t), transformed along the second axis
#pragma unroll
        for (int c2 = 0; c2 < N; ++c2) x[c2] = Ls[plane][t][c2];
        fft<N, -1>(x);
#pragma unroll
        for (int k = 0; k < N; ++k) Ls[plane][t][k] = x[k];
    }
    __syncthreads();
    cx<T>* out = V + it * int64_t(3 * N2) + plane * N2;   // mirror-paired slots (vpair_slot)
    for (int row = 0; row < N; ++row) out[vpair_slot<N>(row, t)] = Ls[plane][row][t];
}


// V_0 and V_1 at k from W at k and at its plane mirror.
template <typename T>
__device__ __forceinline__ void split_w(const cx<T>& W, const cx<T>& Wm, cx<T> v[2]) {
    v[0] = cx<T>{T(0.5) * (W.x + Wm.x), T(0.5) * (W.y - Wm.y)};
    v[1] = cx<T>{T(0.5) * (W.y + Wm.y), T(0.5) * (Wm.x - W.x)};
}

template <typename T>
struct RadialArgs {
    const cx<T>* P;
    const cx<T>* fhat;
    cx<T>* Gt;          // [nb][nslots][N][N][N/2+1]  gain spectrum, the k_z <= N/2 half
    cx<T>* Lt;          // [nb][nslots][N][N][N/2+1]  loss spectrum, the same half
    const T* F;         // [nftab][nrho][K2]  w_q F(|k|, rho_q) / N^3
    const cx<T>* Fv;    // VSS: [nftab][nrho][2 directions][2][N][N][N/2+1]  F_H, F_A: the Hermitian and
                        //      anti-Hermitian parts (in the index sense) of w_q w_sigma F / N^3
    const cx<T>* V;     // VSS: [nb][ncls][nrho][3][N^2]  DFT(Im S_0 + i Im S_1) on the planes k_z, k_y, k_x = N/2,
                        //      each plane in the mirror-paired slots of vpair_slot
    const T* G;         // [ngtab][K2]        G-(|k|)
    const cx<T>* tw;    // [N][CH]  e^{-2 pi i kx c / N}
    const int* slots;   // [nslots][5]
    const int* gterms;  // [..][2]
    const int* lterms;  // [..][2]
    const int* cuses;   // [ncls][4]  (slot, F table) x 2 per class, -1 if unused
    int s, ncls, nrho, nb, nslots, K2;
};

// One thread per Hermitian pair {k, -k} of the output spectrum: it takes the
// representative with k_z <= N/2 (the stored half of the partials), forms
// Q_hat+(k) = sum_terms sum_q w_q F(|k|, rho_q)/N^3 DFT(S_q)(k) and the loss spectrum
// L(k) = sum_j G-(|k|) f_hat^j(k) for the CH x-modes k_x = k_xp + j N/CH, and writes
// both to the k_z <= N/2 half of the output spectra: the spectra are Hermitian (S_q and
// f are real, F and G- are real and even in k), and the inverse transform takes them as
// such.
// VSS: each class (up to two directions) partial is the whole spectrum Z of
// Re S_0 + i Re S_1; the thread reads Z at k and -k and adds the Nyquist-plane terms
// (vss_accumulate).
//
// QS threads share an element: thread group g of the workgroup sums the radial points
// q = g mod QS, the partial sums meet in LDS, and each group finishes the x-modes
// j = g mod QS.  A small call has few elements (one FP64 node at N = 64: 8448 threads for
// QS = 1, 1.15 ms in the latency of 64 dependent rounds of 32 loads each, 0.28 ms for
// QS = 8; three N = 24 nodes 20 -> 10 us, one FP64 node at N = 16 8.3 -> 4.9 us, both with
// QS = 4).  At large batches the kernel is bound by memory either way, and the shorter runs of
// consecutive elements cost it a little (256 nodes at N = 32: 0.562 ms for QS = 1, 0.598 for
// 4; 63 nodes at N = 24: 39 and 40 us; 50 heavy/light nodes at N = 48: 0.603 and 0.606 ms),
// so N = 32, with two or four chunks and the largest batches, keeps QS = 1.
// QS depends on N alone, so that a node's sums do not depend on the batch.
template <int N>
constexpr int radial_qs() { return N == 64 ? 8 : N == 32 ? 1 : 4; }

template <typename T, int N, int CH, bool VSS, int QS>
__global__ __launch_bounds__(256) void radial_kernel(RadialArgs<T> a) {
    static_assert(!VSS || QS == 1, "the shared form covers the VHS sum");
    constexpr int NP = N / CH;
    constexpr int KZH = N / 2 + 1;
    constexpr int EL = 256 / QS;   // elements of a workgroup
    constexpr int64_t N2 = int64_t(N) * N, N3 = N2 * N, PCH = int64_t(NP) * N * KZH;
    __shared__ cx<double> part[QS > 1 ? QS : 1][QS > 1 ? CH : 1][QS > 1 ? EL : 1];
    const int g = int(threadIdx.x) / EL, el = int(threadIdx.x) % EL;
    int64_t t = int64_t(blockIdx.x) * EL + el;
    const bool act = t < int64_t(a.nb) * a.nslots * PCH;
    if (QS == 1 && !act) return;
    if (!act) t = 0;   // shares the barrier and stores nothing
    const int e = int(t % PCH);
    const int64_t bs = t / PCH;
    const int slot = int(bs % a.nslots);
    const int b = int(bs / a.nslots);
    const int kz = e % KZH, ky = (e / KZH) % N, kxp = e / (N * KZH);
    auto sq = [](int k) {
        const int mk = k < N / 2 ? k : k - N;
        return mk * mk;
    };
    const int kyz2 = sq(ky) + sq(kz);
    int k2[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) k2[j] = sq(kxp + j * NP) + kyz2;
    const int* sd = a.slots + 5 * slot;
    const int g0 = sd[1], ng = sd[2], l0 = sd[3], nl = sd[4];

    // the sum over radial points and classes is kept in FP64 (free here: the kernel is
    // bound by its reads of the partials)
    cx<double> acc[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) acc[j] = cx<double>{0.0, 0.0};
    if constexpr (VSS) {
        constexpr int64_t PCHF = int64_t(NP) * N2, NREP = N2 * KZH;
        const int kxpm = (NP - kxp) % NP, kym = (N - ky) % N, kzm = (N - kz) % N;
        const int64_t eP = (int64_t(kxp) * N + ky) * N + kz, ePm = (int64_t(kxpm) * N + kym) * N + kzm;
        for (int gi = 0; gi < ng; ++gi) {
            const int cl = a.gterms[2 * (g0 + gi)], ft = a.gterms[2 * (g0 + gi) + 1];
            const cx<T>* Pb = a.P + (int64_t(b) * a.ncls + cl) * a.nrho * (CH * PCHF);
            const cx<T>* Fb = a.Fv + int64_t(ft) * a.nrho * 4 * NREP + (int64_t(kxp) * N + ky) * KZH + kz;
            const cx<T>* Vb = a.V + (int64_t(b) * a.ncls + cl) * a.nrho * (3 * N2);
            for (int q = 0; q < a.nrho; ++q) {
                cx<T> pc[CH], pm[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    pc[c] = Pb[int64_t(q) * (CH * PCHF) + c * PCHF + eP];
                    pm[c] = Pb[int64_t(q) * (CH * PCHF) + c * PCHF + ePm];
                }
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int kx = kxp + j * NP, kxm = (N - kx) % N;
                    cx<T> Z = pc[0], Zm = pm[0];
#pragma unroll
                    for (int c = 1; c < CH; ++c) {
                        cmac(Z, a.tw[kx * CH + c], pc[c]);
                        cmac(Zm, a.tw[kxm * CH + c], pm[c]);
                    }
                    cx<T> h[2], fa[2], v[2];
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        h[d] = Fb[((int64_t(q) * 2 + d) * 2 + 0) * NREP + int64_t(j) * NP * N * KZH];
                        fa[d] = Fb[((int64_t(q) * 2 + d) * 2 + 1) * NREP + int64_t(j) * NP * N * KZH];
                    }
                    const bool nyq = kx == N / 2 || ky == N / 2 || kz == N / 2;
                    if (nyq)
                    {
                        cx<T> w, wm;
                        w_pair<T, N>(Vb + int64_t(q) * (3 * N2), kx, ky, kz, w, wm);
                        split_w<T>(w, wm, v);
                    }
                    vss_accumulate<T>(acc[j], h, fa, 0.5 * (double(Z.x) + double(Zm.x)),
                                      0.5 * (double(Z.y) - double(Zm.y)), 0.5 * (double(Z.y) + double(Zm.y)),
                                      0.5 * (double(Zm.x) - double(Z.x)), nyq, v);
                }
            }
        }
    }
    // the chunk twiddles e^{-2 pi i kxp c / N} of this thread's k_xp, loaded once
    cx<T> twc[CH];
#pragma unroll
    for (int c = 1; c < CH; ++c) twc[c] = a.tw[kxp * CH + c];
    for (int gi = 0; gi < (VSS ? 0 : ng); ++gi) {
        const int cl = a.gterms[2 * (g0 + gi)], ft = a.gterms[2 * (g0 + gi) + 1];
        const cx<T>* Pb = a.P + (int64_t(b) * a.ncls + cl) * a.nrho * (CH * PCH) + e;
        const T* Ft = a.F + int64_t(ft) * a.nrho * a.K2;
        for (int q = g; q < a.nrho; q += QS) {
            // the last radix-CH step of the x-transform (decimation in time): with
            // k_x = k_xp + j N/CH, DFT(S)(k_x) = sum_c (e^{-2 pi i kxp c / N} P_c) e^{-2 pi i j c / CH}
            cx<T> y[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const cx<T> pc = Pb[int64_t(q) * (CH * PCH) + c * PCH];
                y[c] = c == 0 ? pc : pc * twc[c];
            }
            fft<CH, -1>(y);
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const double fq = double(Ft[q * a.K2 + k2[j]]);
                acc[j].x = fma(fq, double(y[j].x), acc[j].x);
                acc[j].y = fma(fq, double(y[j].y), acc[j].y);
            }
        }
    }
    const int64_t ob = (int64_t(b) * a.nslots + slot) * (N2 * KZH);
    auto store = [&](int j, cx<double> sum) {
        const int kx = kxp + j * NP;
        cx<T> lac{T(0), T(0)};
        for (int li = 0; li < nl; ++li) {
            const int sj = a.lterms[2 * (l0 + li)], gt = a.lterms[2 * (l0 + li) + 1];
            const T gm = a.G[int64_t(gt) * a.K2 + sq(kx) + kyz2];
            const cx<T> v = a.fhat[(int64_t(b) * a.s + sj) * N3 + kx * N2 + ky * N + kz];
            lac.x = fma(gm, v.x, lac.x);
            lac.y = fma(gm, v.y, lac.y);
        }
        const int64_t o = ob + (int64_t(kx) * N + ky) * KZH + kz;
        a.Gt[o] = cx<T>{T(sum.x), T(sum.y)};
        a.Lt[o] = lac;
    };
    if constexpr (QS == 1) {
#pragma unroll
        for (int j = 0; j < CH; ++j) store(j, acc[j]);
    } else {
#pragma unroll
        for (int j = 0; j < CH; ++j) part[g][j][el] = acc[j];
        __syncthreads();
        if (!act) return;
        for (int j = g; j < CH; j += QS) {
            cx<double> sum = part[0][j][el];
#pragma unroll
            for (int u = 1; u < QS; ++u) sum = sum + part[u][j][el];
            store(j, sum);
        }
    }
}

// Row r (0 <= r < NP N) of the radial thread order, as the (k_xp, k_y) row of a chunk
// partial, enumerated in mirror pairs: the groups k_xp = 0 and k_xp = NP/2 (each its own
// mirror in k_xp; rows k_y and -k_y adjacent, 0 and N/2 first), then the rows of k_xp
// and NP - k_xp for k_xp = 1 .. NP/2 - 1, each beside its mirror.  A thread reads the
// partials at k and -k, so with this order a workgroup's reads of a row and of its
// mirror row fall in the same cache lines at the same time.
template <int N, int NP>
__device__ __forceinline__ void mirror_paired_row(int r, int& kxp, int& ky) {
    static_assert(NP % 2 == 0, "row pairing needs an even number of x-planes per chunk");
    if (r < 2 * N) {
        kxp = r < N ? 0 : NP / 2;
        const int rr = r < N ? r : r - N, i = rr >> 1;
        ky = (rr & 1) ? (i == 0 ? N / 2 : N - i) : i;
        return;
    }
    const int g = (r - 2 * N) / (2 * N), rr = (r - 2 * N) % (2 * N), i = rr >> 1;
    kxp = (rr & 1) ? NP - 1 - g : 1 + g;
    ky = (rr & 1) ? (N - i) % N : i;
}

// VSS radial sum with every slot of NB nodes in one thread: per class (up to two
// directions), use and radial point the table values are loaded once and applied to the
// NB nodes' partials (read at k and -k; the second use of an unlike class finds them in
// L2).  The per-slot accumulators are indexed with compile-time slots (SMAX >= nslots) under
// uniform compares, so they stay in registers.  They are of the plan precision (FP32 plans
// sum in FP32): that halves their registers.  Loss terms and outputs as in radial_kernel.
// A node's arithmetic is the same for every NB.
//
// Large calls are bound by memory and want the tables shared by as many nodes as three
// wavefronts per SIMD allow; small ones are bound by the latency of ncls nrho dependent
// rounds of loads and want threads (vss_nodes).  At N = 32, FP32 (two chunks), ms for NB =
// 1 / 2 / 3 / 4: 3 nodes 0.32 / 0.48 / 0.64 / 0.64, 10 nodes 0.44 / 0.53 / 0.70 / 0.88, 32
// nodes 1.03 / 0.87 / 0.83 / 1.00, 96 nodes 2.56 / 1.97 / 1.84 / 2.09 (816 workgroups of NB
// = 4 are 1.06 rounds), 256 nodes 6.7 / 4.8 / 4.3 / 3.95.  With three chunks (N = 24) one
// node a thread is the fastest (40 nodes 0.46 / 0.52 / - / 0.87).
// WPE, the wavefronts per SIMD asked of the compiler: three where the registers allow it
// (up to two chunks in FP32), else what they do: N = 24 spilled for three (40 nodes, NB = 4,
// 1.82 ms, for two 0.87), and so did FP64 (20 nodes at N = 32 10.6 ms; for one, NB = 2, 1.17).
template <typename T, int CH>
constexpr int vss_wpe() { return sizeof(T) == 8 ? 1 : CH <= 2 ? 3 : 2; }
// Nodes per thread: one while that does not fill the chip's 1024 SIMDs with three wavefronts each
// (3072; FP64: 1536), four where a quarter of the one-node wavefronts are twice that many (6144)
// or, with one chunk, whose registers are fewer, 2048 (N = 16, 300 nodes of three species, 2700:
// 2.87 ms a call for two, 2.79 for four; 100 nodes of two, 900: 0.18 and 0.30 ms in the kernel),
// between them three, or two with one chunk; fewer where the accumulators (NB x SMAX x CH) would
// not fit.
template <typename T, int CH, int SMAX>
constexpr int vss_nb_max() { return sizeof(T) == 8 ? (CH <= 4 && SMAX == 2 ? 2 : 1) : CH >= 3 ? 1 : 8 / (CH * SMAX) >= 2 ? 4 : 2; }
template <typename T, int CH, int SMAX>
int vss_nodes(int64_t nb, int64_t blocks_per_node) {
    constexpr int most = vss_nb_max<T, CH, SMAX>();
    const int64_t waves = nb * blocks_per_node * 4;
    if (most == 1 || waves <= (sizeof(T) == 8 ? 1536 : 3072)) return 1;
    if (most == 2) return 2;
    return waves / 4 >= (CH == 1 ? 2048 : 2 * 3072) ? 4 : CH == 1 ? 2 : 3;
}

template <typename T, int N, int CH, int NB, int SMAX>
__global__ __launch_bounds__(256, (vss_wpe<T, CH>())) void radial_vss_kernel(RadialArgs<T> a) {
    constexpr int NP = N / CH;
    constexpr int KZH = N / 2 + 1;
    constexpr int64_t N2 = int64_t(N) * N, N3 = N2 * N, PCH = int64_t(NP) * N * KZH;
    constexpr int64_t PCHF = int64_t(NP) * N2, NREP = N2 * KZH;
    // Blocks with consecutive indices take the same 256 stored entries for consecutive
    // node groups, so a block's slice of the kernel-mode tables is read from its XCD's L2
    // by the node groups that follow, not from memory per group.
    const int64_t ngroups = (a.nb + NB - 1) / NB;
    const int64_t ng = int64_t(blockIdx.x) % ngroups;
    const int64_t eblk = int64_t(blockIdx.x) / ngroups;
    if (eblk * 256 + threadIdx.x >= PCH) return;
    const int e = int(eblk * 256 + threadIdx.x);
    const int b0 = int(ng) * NB;
    const int kz = e % KZH;
    int kxp, ky;
    mirror_paired_row<N, NP>(e / KZH, kxp, ky);
    const int kxpm = (NP - kxp) % NP, kym = (N - ky) % N, kzm = (N - kz) % N;
    const int64_t eP = (int64_t(kxp) * N + ky) * N + kz, ePm = (int64_t(kxpm) * N + kym) * N + kzm;
    const int64_t fo = (int64_t(kxp) * N + ky) * KZH + kz;

    cx<T> acc[NB][SMAX][CH];
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int sl = 0; sl < SMAX; ++sl)
#pragma unroll
            for (int j = 0; j < CH; ++j) acc[u][sl][j] = cx<T>{T(0), T(0)};

    constexpr int N2I = N * N;
    bool nyq[CH];
    int wi[CH];   // the aligned pair holding W at k and at its plane mirror (pair 0 off the planes)
    bool wodd[CH], wself[CH];
    bool nyq_any = false;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        const int kx = kxp + j * NP;
        nyq[j] = kx == N / 2 || ky == N / 2 || kz == N / 2;
        const int sl = nyq[j] ? vplane_slot<N>(kx, ky, kz) : 0;
        wi[j] = sl & ~1;
        wodd[j] = (sl & 1) != 0;
        wself[j] = (kx == 0 || kx == N / 2) + (ky == 0 || ky == N / 2) + (kz == 0 || kz == N / 2) == 3;
        nyq_any = nyq_any || nyq[j];
    }
    for (int cl = 0; cl < a.ncls; ++cl) {
        const int s0 = a.cuses[4 * cl], s1 = a.cuses[4 * cl + 2];
        if (s0 < 0) continue;
        const cx<T>* F0 = a.Fv + int64_t(a.cuses[4 * cl + 1]) * a.nrho * 4 * NREP + fo;
        const cx<T>* F1 = a.Fv + int64_t(s1 >= 0 ? a.cuses[4 * cl + 3] : a.cuses[4 * cl + 1]) * a.nrho * 4 * NREP + fo;
        for (int q = 0; q < a.nrho; ++q) {
            // F_H of both uses and both directions; F_A only where some lane has a Nyquist mode
            cx<T> h0[CH][2], h1[CH][2], a0[CH][2], a1[CH][2];
#pragma unroll
            for (int j = 0; j < CH; ++j)
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const int64_t o = ((int64_t(q) * 2 + d) * 2) * NREP + int64_t(j) * NP * N * KZH;
                    h0[j][d] = F0[o];
                    h1[j][d] = F1[o];
                    a0[j][d] = cx<T>{T(0), T(0)};
                    a1[j][d] = cx<T>{T(0), T(0)};
                }
            if (nyq_any) {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const int64_t o = ((int64_t(q) * 2 + d) * 2 + 1) * NREP + int64_t(j) * NP * N * KZH;
                        a0[j][d] = F0[o];
                        a1[j][d] = F1[o];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int b = b0 + u;
                if (b >= a.nb) break;
                const cx<T>* Pb = a.P + ((int64_t(b) * a.ncls + cl) * a.nrho + q) * (CH * PCHF);
                const cx<T>* Vb = a.V + ((int64_t(b) * a.ncls + cl) * a.nrho + q) * (3 * N2I);
                cx<T> pc[CH], pm[CH], w0[CH], w1[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    pc[c] = Pb[c * PCHF + eP];
                    pm[c] = Pb[c * PCHF + ePm];
                }
                // the Nyquist-plane values, read with the partials (every lane, the
                // lanes off the planes all at one address) rather than after them
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    w0[j] = Vb[wi[j]];
                    w1[j] = Vb[wi[j] + 1];
                }
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int kx = kxp + j * NP, kxm = (N - kx) % N;
                    cx<T> Z = pc[0], Zm = pm[0];
#pragma unroll
                    for (int c = 1; c < CH; ++c) {
                        cmac(Z, a.tw[kx * CH + c], pc[c]);
                        cmac(Zm, a.tw[kxm * CH + c], pm[c]);
                    }
                    cx<T> v[2];
                    if (nyq[j]) {
                        const cx<T> w = wodd[j] ? w1[j] : w0[j];
                        split_w<T>(w, wself[j] ? w : (wodd[j] ? w0[j] : w1[j]), v);
                    }
                    const T u0x = T(0.5) * (Z.x + Zm.x), u0y = T(0.5) * (Z.y - Zm.y);
                    const T u1x = T(0.5) * (Z.y + Zm.y), u1y = T(0.5) * (Zm.x - Z.x);
#pragma unroll
                    for (int sl = 0; sl < SMAX; ++sl) {
                        if (sl == s0) vss_accumulate<T, T>(acc[u][sl][j], h0[j], a0[j], u0x, u0y, u1x, u1y, nyq[j], v);
                        if (sl == s1) vss_accumulate<T, T>(acc[u][sl][j], h1[j], a1[j], u0x, u0y, u1x, u1y, nyq[j], v);
                    }
                }
            }
        }
    }

    int k2[CH];
    auto sq = [](int k) {
        const int mk = k < N / 2 ? k : k - N;
        return mk * mk;
    };
#pragma unroll
    for (int j = 0; j < CH; ++j) k2[j] = sq(kxp + j * NP) + sq(ky) + sq(kz);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int b = b0 + u;
        if (b >= a.nb) break;
#pragma unroll
        for (int sl = 0; sl < SMAX; ++sl) {
            if (sl >= a.nslots) break;
            const int* sd = a.slots + 5 * sl;
            const int l0 = sd[3], nl = sd[4];
            cx<T> lac[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) lac[j] = cx<T>{T(0), T(0)};
            for (int li = 0; li < nl; ++li) {
                const int sj = a.lterms[2 * (l0 + li)], gt = a.lterms[2 * (l0 + li) + 1];
                const cx<T>* fj = a.fhat + (int64_t(b) * a.s + sj) * N3 + ky * N + kz;
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int kx = kxp + j * NP;
                    const T gm = a.G[int64_t(gt) * a.K2 + k2[j]];
                    const cx<T> v = fj[kx * N2];
                    lac[j].x = fma(gm, v.x, lac[j].x);
                    lac[j].y = fma(gm, v.y, lac[j].y);
                }
            }
            const int64_t ob = (int64_t(b) * a.nslots + sl) * (N2 * KZH);
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int64_t o = ob + (int64_t(kxp + j * NP) * N + ky) * KZH + kz;
                a.Gt[o] = cx<T>{T(acc[u][sl][j].x), T(acc[u][sl][j].y)};
                a.Lt[o] = lac[j];
            }
        }
    }
}

// ====================================================== inverse transform + combine
// The inverse transform of the gain and loss spectra (Hermitian, the k_z <= N/2 half
// stored): the x-pass runs on the half in place (half_xpass_kernel); the y-pass and the
// z-pass, which restores each row's conjugate half and keeps the real part, run on one
// x-plane after the other through LDS, fused with the combination Q = g - f_i l of the
// slot's species i (inverse_yz_kernel).
template <typename T, int N>
__global__ __launch_bounds__(256) void half_xpass_kernel(cx<T>* data, int64_t npencils) {
    constexpr int KZH = N / 2 + 1;
    constexpr int64_t NH = int64_t(N) * N * KZH, stride = int64_t(N) * KZH;
    const int64_t pid = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (pid >= npencils) return;
    const int64_t field = pid / (N * KZH);
    const int64_t base = field * NH + (pid - field * (N * KZH));
    cx<T> v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = data[base + k * stride];
    fft<N, +1>(v);
#pragma unroll
    for (int k = 0; k < N; ++k) data[base + k * stride] = v[k];
}

// PL x-planes of a slot to a workgroup: 2 PL KZH columns of both spectra, then PL N rows,
// on about as many threads, a few workgroups to a CU.  With the y- and z-passes as two launches 512 FP32
// slots at N = 32 took 50 + 57 us, together 59; one FP64 node at N = 16 10.0 us, now 4.7.
template <int N>
struct InverseTile {
    static constexpr int PL = N <= 16 ? 3 : N == 24 ? 2 : N == 32 ? 3 : 1;
    static constexpr int KZH = N / 2 + 1;   // odd for every N here: rows of KZH values spread over the banks
    static constexpr int NT = (2 * PL * KZH + 63) / 64 * 64;
};

template <typename T, int N>
__global__ __launch_bounds__(InverseTile<N>::NT) void inverse_yz_kernel(const cx<T>* __restrict__ Gh,
                                                                        const cx<T>* __restrict__ Lh,
                                                                        const T* __restrict__ f, T* __restrict__ Q,
                                                                        const int* __restrict__ slots, int nslots,
                                                                        int s, int64_t nplanes) {
    using K = InverseTile<N>;
    constexpr int KZH = K::KZH;
    constexpr int64_t N2 = int64_t(N) * N, N3 = N2 * N;
    __shared__ cx<T> buf[2][K::PL][N * KZH];
    const int t = threadIdx.x;
    const int64_t p0 = int64_t(blockIdx.x) * K::PL;
    if (t < 2 * K::PL * KZH) {
        const int fld = t / (K::PL * KZH), pl = t / KZH % K::PL, kz = t % KZH;
        if (p0 + pl < nplanes) {
            const cx<T>* src = (fld == 0 ? Gh : Lh) + (p0 + pl) * (N * KZH) + kz;
            cx<T> v[N];
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] = src[k * KZH];
            fft<N, +1>(v);
#pragma unroll
            for (int k = 0; k < N; ++k) buf[fld][pl][k * KZH + kz] = v[k];
        }
    }
    __syncthreads();
    const int pl = t / N, y = t % N;
    const int64_t plane = p0 + pl;       // (node, slot, x)
    if (pl >= K::PL || plane >= nplanes) return;
    const int64_t bs = plane / N;
    const int64_t xy = (plane - bs * N) * N + y;
    const int sp = slots[5 * int(bs % nslots)];
    const int64_t b = bs / nslots;
    const cx<T>* g = &buf[0][pl][y * KZH];
    const cx<T>* l = &buf[1][pl][y * KZH];
    cx<T> vg[N], vl[N];
#pragma unroll
    for (int k = 0; k < KZH; ++k) {
        vg[k] = g[k];
        vl[k] = l[k];
    }
#pragma unroll
    for (int k = KZH; k < N; ++k) {
        vg[k] = cx<T>{vg[N - k].x, -vg[N - k].y};
        vl[k] = cx<T>{vl[N - k].x, -vl[N - k].y};
    }
    fft<N, +1>(vg);
    fft<N, +1>(vl);
    const T* fr = f + (b * s + sp) * N3 + xy * N;
    T* q = Q + bs * N3 + xy * N;
#pragma unroll
    for (int z = 0; z < N; ++z) q[z] = vg[z].x - fr[z] * vl[z].x;
}

// The gain stage of FP32 VHS plans at N = 32 on the matrix cores (gain_mfma.hip, geometry
// (2, 0)): prepares each (node, species) input in `prep` (mfma_prep_bytes per pair) and
// writes the chunk partials P exactly as gain_kernel<float, 32, 2, 1> lays them out.
hipError_t launch_gain_mfma32(const dgfs_plan& p, const float* f, cx<float>* P, void* prep, int nb, hipStream_t st);

namespace detail {

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// ev (optional): 6 events recorded at the stage boundaries (start, after forward FFT,
// after gain, after radial, after the inverse x/y passes, after the z-pass + combine).
// MF: the gain stage runs on the matrix cores (FP32, N = 32, VHS only).
template <typename T, int N, int CH, int CZ, int PIPE, bool PACK, bool VSS, bool MF = false>
hipError_t run_slice(const dgfs_plan& p, const T* f, T* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                     hipEvent_t* ev) {
    static_assert(!MF || (std::is_same_v<T, float> && N == 32 && CH == 2 && !VSS), "matrix-core gain: FP32 VHS N = 32");
    constexpr int MODE = VSS ? GAIN_VSS : GAIN_REAL;
    auto mark = [&](int k) {
        if (ev) hipEventRecord(ev[k], st);
    };
    const SlotSet& ss = pairs ? p.pair_slots : p.sum_slots;
    constexpr int64_t N3 = int64_t(N) * N * N;
    const int ncls = int(p.classes.size());
    char* w = static_cast<char*>(ws.p);
    cx<T>* fhat = reinterpret_cast<cx<T>*>(w);
    w += align256(sizeof(cx<T>) * nb * p.s * N3);
    cx<T>* P = reinterpret_cast<cx<T>*>(w);
    w += align256(sizeof(cx<T>) * int64_t(nb) * ncls * p.nrho * (VSS ? N3 : (N3 / N) * (N / 2 + 1)));
    T* PL = nullptr;
    cx<T>* Vn = nullptr;
    if constexpr (VSS) {
        PL = reinterpret_cast<T*>(w);
        w += align256(sizeof(T) * int64_t(nb) * ncls * p.nrho * 2 * (2 + CH) * N * N);
        Vn = reinterpret_cast<cx<T>*>(w);
        w += align256(sizeof(cx<T>) * int64_t(nb) * ncls * p.nrho * 3 * N * N);
    }
    constexpr int64_t NH = int64_t(N) * N * (N / 2 + 1);  // stored half of a spectrum
    cx<T>* Gt = reinterpret_cast<cx<T>*>(w);
    cx<T>* Lt = Gt + int64_t(nb) * ss.nslots * NH;  // contiguous with Gt

    const char* dev = static_cast<const char*>(p.dev);
    mark(0);
    hipError_t e = fft3d_forward<T, N>(fhat, f, int64_t(nb) * p.s, T(1.0 / double(N3)), st);
    if (e != hipSuccess) return e;
    mark(1);

    GainArgs<T> ga;
    ga.fhat = fhat;
    ga.P = P;
    ga.PL = PL;
    ga.kx = reinterpret_cast<const cx<T>*>(dev + p.off_kx);
    ga.yz = reinterpret_cast<const cx<T>*>(dev + p.off_yz);
    ga.nyq = reinterpret_cast<const T*>(dev + p.off_nyq);
    ga.cls = reinterpret_cast<const int*>(dev + p.off_cls);
    ga.wdir = reinterpret_cast<const T*>(dev + p.off_wdir);
    ga.s = p.s;
    ga.ncls = ncls;
    ga.nrho = p.nrho;
    ga.nb = nb;
    ga.ord = reinterpret_cast<const int*>(dev + p.off_ord);
    ga.xs = reinterpret_cast<const int*>(dev + p.off_xs);
    ga.D = nullptr;
    ga.tdirs = p.total_dirs;
    if constexpr (MF) {
        // the prepared inputs follow the loss spectra
        char* prep = reinterpret_cast<char*>(Lt + int64_t(nb) * ss.nslots * NH);
        prep += (256 - reinterpret_cast<uintptr_t>(prep) % 256) % 256;
        if ((e = launch_gain_mfma32(p, f, P, prep, nb, st)) != hipSuccess) return e;
    } else {
        const int64_t ipn = int64_t(ncls) * p.nrho * CH;
        const dim3 block(GainK<T, N, CH, CZ>::NT);
        bool split = false;
        if constexpr (!VSS && N <= 32) {
            // the terms follow the loss spectra, where the caller's workspace reaches so far
            char* terms = reinterpret_cast<char*>(Lt + int64_t(nb) * ss.nslots * NH);
            terms += (256 - reinterpret_cast<uintptr_t>(terms) % 256) % 256;
            const size_t bytes = p.ws_split(nb), used = size_t(terms - static_cast<char*>(ws.p));
            if (bytes != 0 && used <= ws.bytes && bytes <= ws.bytes - used) {
                split = true;
                ga.D = reinterpret_cast<T*>(terms);
                // as many radial points at a time as the memory holds, in equal groups
                const int fit = int(std::min<size_t>(p.nrho, bytes / (sizeof(T) * N3 * nb * p.total_dirs)));
                const int groups = (p.nrho + fit - 1) / fit, per = (p.nrho + groups - 1) / groups;
                for (ga.q0 = 0; ga.q0 < p.nrho; ga.q0 += per) {
                    ga.nq = std::min(per, p.nrho - ga.q0);
                    gain_kernel<T, N, CH, CZ, PIPE, PACK, GAIN_TERMS>
                        <<<dim3(gain_groups(nb, int64_t(p.total_dirs) * ga.nq * CH)), block, 0, st>>>(ga);
                    gain_sum_kernel<T, N, CH, CZ>
                        <<<dim3(gain_groups(nb, int64_t(ncls) * ga.nq * CH)), block, 0, st>>>(ga);
                }
            }
        }
        constexpr int rule = keep_rule<T, N, MODE>();
        const dim3 grid(gain_groups(nb, ipn));
        const bool keep = rule == KEEP_ALWAYS || (rule == KEEP_BY_REUSE && 2 * p.fresh_dirs <= p.total_dirs);
        if constexpr (rule != KEEP_NEVER)
            if (!split && keep) gain_kernel<T, N, CH, CZ, PIPE, PACK, MODE, true><<<grid, block, 0, st>>>(ga);
        if constexpr (rule != KEEP_ALWAYS)
            if (!split && !keep) gain_kernel<T, N, CH, CZ, PIPE, PACK, MODE><<<grid, block, 0, st>>>(ga);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if constexpr (VSS) {
        nyquist_dft_kernel<T, N, CH><<<dim3(unsigned(int64_t(nb) * ncls * p.nrho)), dim3(3 * N), 0, st>>>(PL, Vn);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    mark(2);

    RadialArgs<T> ra;
    ra.P = P;
    ra.fhat = fhat;
    ra.Gt = Gt;
    ra.Lt = Lt;
    ra.F = reinterpret_cast<const T*>(dev + p.off_F);
    ra.Fv = reinterpret_cast<const cx<T>*>(dev + p.off_F);
    ra.V = Vn;
    ra.G = reinterpret_cast<const T*>(dev + p.off_G);
    ra.tw = reinterpret_cast<const cx<T>*>(dev + p.off_tw);
    ra.slots = reinterpret_cast<const int*>(dev + ss.off_slots);
    ra.gterms = reinterpret_cast<const int*>(dev + ss.off_gterms);
    ra.lterms = reinterpret_cast<const int*>(dev + ss.off_lterms);
    ra.cuses = reinterpret_cast<const int*>(dev + ss.off_cuses);
    ra.s = p.s;
    ra.ncls = ncls;
    ra.nrho = p.nrho;
    ra.nb = nb;
    ra.nslots = ss.nslots;
    ra.K2 = p.K2;
    const int64_t pch = int64_t(N / CH) * N * (N / 2 + 1);
    const int64_t rthreads = int64_t(nb) * ss.nslots * pch;
    if constexpr (VSS) {
        // few slots: every slot of vss_nodes nodes in one thread
        const int64_t eblocks = (pch + 255) / 256;
        auto fused = [&](auto smax) {
            constexpr int SMAX = decltype(smax)::value, MOST = vss_nb_max<T, CH, SMAX>();
            const int NB = vss_nodes<T, CH, SMAX>(nb, eblocks);
            const dim3 grid(unsigned(((nb + NB - 1) / NB) * eblocks)), block(256);
            if (NB == 1) radial_vss_kernel<T, N, CH, 1, SMAX><<<grid, block, 0, st>>>(ra);
            if constexpr (MOST >= 2)
                if (NB == 2) radial_vss_kernel<T, N, CH, 2, SMAX><<<grid, block, 0, st>>>(ra);
            if constexpr (MOST >= 4) {
                if (NB == 3) radial_vss_kernel<T, N, CH, 3, SMAX><<<grid, block, 0, st>>>(ra);
                if (NB == 4) radial_vss_kernel<T, N, CH, 4, SMAX><<<grid, block, 0, st>>>(ra);
            }
        };
        if (ss.nslots <= 2) {
            fused(std::integral_constant<int, 2>{});
        } else if (ss.nslots <= 4) {
            fused(std::integral_constant<int, 4>{});
        } else {
            radial_kernel<T, N, CH, true, 1><<<dim3(unsigned((rthreads + 255) / 256)), dim3(256), 0, st>>>(ra);
        }
    } else {
        constexpr int QS = radial_qs<N>();
        constexpr int64_t EL = 256 / QS;
        radial_kernel<T, N, CH, false, QS><<<dim3(unsigned((rthreads + EL - 1) / EL)), dim3(256), 0, st>>>(ra);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    mark(3);

    {
        const int64_t np = 2 * int64_t(nb) * ss.nslots * N * (N / 2 + 1);
        half_xpass_kernel<T, N><<<dim3(unsigned((np + 255) / 256)), dim3(256), 0, st>>>(Gt, np);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    mark(4);

    const int64_t planes = int64_t(nb) * ss.nslots * N;
    constexpr int IPL = InverseTile<N>::PL;
    inverse_yz_kernel<T, N><<<dim3(unsigned((planes + IPL - 1) / IPL)), dim3(InverseTile<N>::NT), 0, st>>>(
        Gt, Lt, f, Q, ra.slots, ss.nslots, p.s, planes);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    mark(5);
    return hipSuccess;
}

}  // namespace detail

// Per-N entry points (tiles_<N>.hip): run one slice with the plan's tile geometry.
hipError_t run_tiles_16(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                        hipEvent_t* ev);
hipError_t run_tiles_24(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                        hipEvent_t* ev);
hipError_t run_tiles_32(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                        hipEvent_t* ev);
hipError_t run_tiles_48(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                        hipEvent_t* ev);
hipError_t run_tiles_64(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                        hipEvent_t* ev);
// The same for plans with a VSS kernel (vss_<N>.hip).
hipError_t run_vss_16(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                      hipEvent_t* ev);
hipError_t run_vss_24(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                      hipEvent_t* ev);
hipError_t run_vss_32(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                      hipEvent_t* ev);
hipError_t run_vss_48(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                      hipEvent_t* ev);

}  // namespace dgfs
