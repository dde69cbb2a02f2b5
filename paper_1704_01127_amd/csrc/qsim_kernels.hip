// GPU kernels of the state-vector simulator (gfx950 / MI355X).
//
// State: 2^n interleaved complex amplitudes (float2 or double2), amplitude
// index i = sum_q b_q 2^q (Haener & Steiger, Sec. 2).
//
// Cluster kernels apply one dense k-qubit gate in place (Sec. 3.2): with the
// targets sorted (t_0 < ... < t_{k-1}), a "column" c is an assignment of the
// n-k other bits, deposited into the non-target positions; the 2^k amplitudes
// of a column are gathered, multiplied by the 2^k x 2^k matrix and scattered
// back. Consecutive columns differ in the lowest non-target bits, so a wave's
// columns are contiguous runs of memory.
//
// For k >= 4 (float) / k >= 3 (double) the product is a real GEMM on the
// matrix cores: with the state's (re, im) interleaving the complex matrix
// becomes the real 2^(k+1) x 2^(k+1) matrix [[Re m, -Im m], [Im m, Re m]] per
// entry - the (m_R, m_R) / (-m_I, m_I) pairing of Sec. 3.2, Eqs. (1)-(3) -
// and one MFMA block multiplies it by 32 (float) or 16 (double) columns. The
// rows and inner index of that matrix are permuted once, when it is built,
// so that every lane's MFMA operands and results are exactly the amplitudes
// it loads and stores: lane (p, h) of a float wave owns the amplitudes whose
// highest target bit is h in column p, with no LDS round trip for the state.
//
// How the kernels walk the state. A pass is bound by HBM, and what DRAM gives
// depends on how compact the stretch of the state in flight is. Most kernels
// therefore do one tile per wave, work-groups in memory order: the hardware
// hands the next tiles to whichever compute unit is free, so the tiles in
// flight stay next to each other. Waves of a persistent grid drift apart (an
// in-place linear pass over 8 GiB: 3.0 ms against 3.4 ms, a 64-row gather of
// 256-byte runs 3.2-3.3 against 3.5-3.8), also when each takes its own
// contiguous share (3.3 ms for 2 MiB per work-group). The matrix is then read
// from L2 once per work-group, which costs less than it gains. A state beyond
// the 256 MiB last-level cache is moved with non-temporal accesses, another
// 5-10 % (linear: 2.65 ms = 6.5 TB/s); a smaller one is not, since the next
// pass finds it in the cache (25 qubits complex64: 90 us against 101 us with
// them), and neither are accesses that cover a 128-byte line only in part
// (a 6-qubit cluster on qubits 0-5 gathered directly: 24 ms against 4.6 ms).
#include "qsim_internal.h"

#include <cmath>
#include <cstring>
#include <type_traits>

namespace qsim {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename T> struct Cplx;
template <> struct Cplx<float> { using type = float2; };
template <> struct Cplx<double> { using type = double2; };

// Insert a zero bit at position t.
__device__ __forceinline__ uint64_t insert_zero(uint64_t c, int t) {
    const uint64_t low = (uint64_t(1) << t) - 1;
    return ((c & ~low) << 1) | (c & low);
}

// Deposit column index c into the non-target bit positions.
template <int K>
__device__ __forceinline__ uint64_t deposit_cols(uint64_t c, const ClusterGeom& g) {
#pragma unroll
    for (int j = 0; j < K; ++j) c = insert_zero(c, g.t[j]);
    return c;
}

// Offset of target index x: bit j of x at state bit t[j], j < NB.
template <int NB>
__device__ __forceinline__ uint64_t target_off(int x, const ClusterGeom& g) {
    uint64_t o = 0;
#pragma unroll
    for (int j = 0; j < NB; ++j)
        if ((x >> j) & 1) o |= uint64_t(1) << g.t[j];
    return o;
}

// ------------------------------------------------------------ diagonal factors
// Factor of the diagonal gates that depends on the non-target bits of a
// column (sign parity, sign mask over target bits, complex phase).
template <typename T>
struct ColFactor {
    uint32_t sgn, w;
    T cr, ci;
};

template <typename T, typename E>
__device__ __forceinline__ ColFactor<T> col_factor(E* __restrict__ e, uint64_t base) {
    ColFactor<T> f{0u, 0u, T(1), T(0)};
    const int ncc = e->n_cc;
    for (int i = 0; i < ncc; ++i)
        f.sgn ^= (uint32_t)((base >> e->cc[i][0]) & (base >> e->cc[i][1]) & 1);
    const int nm = e->n_mix;
    for (int i = 0; i < nm; ++i) f.w ^= (uint32_t)((base >> e->mix[i][1]) & 1) << e->mix[i][0];
    const int np = e->n_ph;
    if (np) {
        double cr = 1.0, ci = 0.0;
        for (int i = 0; i < np; ++i) {
            if ((base >> e->ph_q[i]) & 1) {
                const double a = e->ph[i][0], b = e->ph[i][1];
                const double t = cr * a - ci * b;
                ci = cr * b + ci * a;
                cr = t;
            }
        }
        f.cr = (T)cr;
        f.ci = (T)ci;
    }
    return f;
}

template <typename T>
__device__ __forceinline__ void apply_factor(T& re, T& im, const ColFactor<T>& f, uint32_t y, bool ph) {
    if (ph) {
        const T r = re * f.cr - im * f.ci;
        const T i = re * f.ci + im * f.cr;
        re = r;
        im = i;
    }
    const bool neg = ((f.sgn ^ (uint32_t)__popc(y & f.w)) & 1u) != 0;
    re = neg ? -re : re;
    im = neg ? -im : im;
}

// Work-groups of a launch are dealt to the 8 XCDs round-robin (work-group b
// runs on XCD b % 8). Renumbered so that the work-groups of one XCD are
// consecutive, the tiles a persistent grid has in flight form one contiguous
// stretch per XCD (each XCD has its own L2). A bijection of the work-group
// numbers when the grid is a multiple of 8, else the identity.
__device__ __forceinline__ uint32_t xcd_block() {
    const uint32_t b = blockIdx.x, g = gridDim.x;
    return (g & 7) == 0 ? (b & 7) * (g >> 3) + (b >> 3) : b;
}

// Work-group number of a launch that covers a state with one work-group per
// kWgBytes of it: in memory order beyond the caches (see beyond_caches), else
// by stretches, one per XCD. Passes that follow each other then find what fits
// in an XCD's L2 (4 MiB) where the last one left it: 363 gates one by one on a
// 20-qubit complex128 state (16 MiB) 1.91 ms, in memory order 2.38.
template <uint32_t kWgBytes>
__device__ __forceinline__ uint32_t tile_block() {
    return gridDim.x < (uint32_t(512) << 20) / kWgBytes ? xcd_block() : blockIdx.x;
}

// Float64 sums of p = |a|^2 (slot 0), p^2 (slot 1) and -p ln p (slot 2) over
// float amplitudes. ln p = e ln 2 + ln m with p = m 2^e split exactly and
// ln m (m in [1/2, 1)) in float, within ~1.4e-7 absolute - far below what a
// float state resolves; a double log costs as much ALU time as reading the
// state.
__device__ __forceinline__ void stats_acc_f(double (&v)[8], float x, float y) {
    const double pr = (double)x * (double)x + (double)y * (double)y;
    v[0] += pr;
    v[1] += pr * pr;
    if (pr > 0.0) {
        int e;
        const double m = frexp(pr, &e);
        v[2] -= pr * ((double)e * 0.6931471805599453 + (double)logf((float)m));
    }
}

// Block reduction of up to 8 values into out (defined with the reductions).
__device__ void block_reduce_store(double (&vals)[8], int nv, unsigned maxmask, double* out);

// Lane l's value of x, in every lane (l uniform).
__device__ __forceinline__ double readlane_f64(double x, int l) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Row sums of a plain complex128 d x d matrix, times amp, into LDS: eight
// threads per row, each summing every eighth entry (so all loads are in
// flight at once), combined by shuffles within the eight. Every thread of the
// block takes part (the shuffles); the caller synchronises afterwards.
template <typename V2>
__device__ __forceinline__ void row_sums(const double2* __restrict__ M, int d, double amp, V2* out) {
    const int sub = (int)threadIdx.x & 7;
    for (int r0 = 0; r0 < d; r0 += (int)blockDim.x / 8) {
        const int r = r0 + (int)threadIdx.x / 8;
        double re = 0.0, im = 0.0;
        if (r < d)
            for (int x = sub; x < d; x += 8) {
                const double2 m = M[r * d + x];
                re += m.x;
                im += m.y;
            }
#pragma unroll
        for (int o = 4; o > 0; o >>= 1) {
            re += __shfl_xor(re, o);
            im += __shfl_xor(im, o);
        }
        if (r < d && sub == 0) {
            out[r].x = (decltype(out[r].x))(re * amp);
            out[r].y = (decltype(out[r].y))(im * amp);
        }
    }
}

typedef float vf4 __attribute__((ext_vector_type(4)));
typedef double vd2 __attribute__((ext_vector_type(2)));
// Explicitly global pointers for code that also runs on pointers read from a
// descriptor (the compiler would otherwise use flat memory instructions,
// whose outstanding loads also hold up every LDS wait).
#define QSIM_GLOBAL __attribute__((address_space(1)))
typedef QSIM_GLOBAL float2 g_float2;
typedef QSIM_GLOBAL vf4 g_vf4;
typedef const QSIM_GLOBAL EpiDesc g_epi;
// Diagonal descriptors read through the constant address space: uniform,
// read-only data the compiler then loads with scalar instructions. (Vector
// loads of them would share the vector-memory counter with a tile's prefetch,
// and waiting for them would wait for the whole prefetch.)
typedef const __attribute__((address_space(4))) EpiDesc c_epi;

// 16-byte accesses of the state; NT: past the caches (non-temporal).
template <bool NT, typename V>
__device__ __forceinline__ V load16(const V* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT, typename V>
__device__ __forceinline__ void store16(V* p, V v) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Copy a cluster matrix of N elements into LDS: 16-byte loads, all in flight
// before the first LDS store (a loop of single loads would wait for each).
template <int N, int THREADS, typename T, typename V4>
__device__ __forceinline__ void load_matrix(T* __restrict__ dst, const V4* __restrict__ src) {
    typedef vf4 v4;
    constexpr int CHUNKS = N * (int)sizeof(T) / 16;
    static_assert(N * sizeof(T) % 16 == 0, "matrix is a whole number of 16-byte chunks");
    constexpr int PER = CHUNKS / THREADS;
    constexpr int REST = CHUNKS % THREADS;
    v4 r[PER > 0 ? PER : 1];
#pragma unroll
    for (int i = 0; i < PER; ++i) r[i] = src[threadIdx.x + i * THREADS];
    v4 t{0.0f, 0.0f, 0.0f, 0.0f};
    if (REST && threadIdx.x < REST) t = src[PER * THREADS + threadIdx.x];
#pragma unroll
    for (int i = 0; i < PER; ++i) reinterpret_cast<v4*>(dst)[threadIdx.x + i * THREADS] = r[i];
    if (REST && threadIdx.x < REST) reinterpret_cast<v4*>(dst)[PER * THREADS + threadIdx.x] = t;
}

// The same in two steps, for a kernel that has other loads to issue in
// between: the loads of BYTES of matrix at construction, the LDS stores later.
template <int BYTES, int THREADS>
struct MatrixRegs {
    static constexpr int CHUNKS = BYTES / 16, PER = CHUNKS / THREADS, REST = CHUNKS % THREADS;
    static_assert(BYTES % 16 == 0, "matrix is a whole number of 16-byte chunks");
    vf4 r[PER > 0 ? PER : 1], t;
    __device__ __forceinline__ explicit MatrixRegs(const void* src) {
        const vf4* m = reinterpret_cast<const vf4*>(src);
#pragma unroll
        for (int i = 0; i < PER; ++i) r[i] = m[i * THREADS + threadIdx.x];
        if (REST && threadIdx.x < REST) t = m[PER * THREADS + threadIdx.x];
    }
    __device__ __forceinline__ void store(void* dst) const {
        vf4* m = reinterpret_cast<vf4*>(dst);
#pragma unroll
        for (int i = 0; i < PER; ++i) m[i * THREADS + threadIdx.x] = r[i];
        if (REST && threadIdx.x < REST) m[PER * THREADS + threadIdx.x] = t;
    }
};

// The value of x in the lane whose index differs in bit B.
template <int B>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    if constexpr (B == 0) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true);  // quad [1,0,3,2]
    if constexpr (B == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true);  // quad [2,3,0,1]
    if constexpr (B == 2) {  // mirrored within 8 lanes (index ^ 7), then within 4 (^ 3)
        const int m = __builtin_amdgcn_mov_dpp((int)x, 0x141, 0xf, 0xf, true);
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xf, 0xf, true);
    }
    if constexpr (B == 3) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);  // row rotated by 8
    const int lane = (int)(threadIdx.x & 63);
    if constexpr (B == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (lane & 32) ? r[0] : r[1];
    }
}
template <int B>
__device__ __forceinline__ double lane_xor(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = lane_xor<B>((uint32_t)b), hi = lane_xor<B>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// ------------------------------------------------------------ cluster: MFMA, float
// Wave tile: all 2^K target combinations x 32*NB columns. Lane l: p = l%32,
// h = l/32 owns target indices x = j | h << (K-1), j < 2^(K-1), of its
// column(s). Without a target at bit 0 (LOWT = false) and NB = 2 a lane's two
// columns are adjacent in memory (one 16-byte load per amplitude pair); with
// t_0 = 0 (LOWT) the amplitudes j, j+1 of one column are adjacent instead.
template <int K, int NB, bool LOWT>
struct TileF32 {
    static constexpr int HX = (1 << K) / 2;
    static constexpr int COLS = 32 * NB;

    __device__ __forceinline__ static void bases(uint64_t tile, int p, const ClusterGeom& g, uint64_t (&base)[NB]) {
        if (LOWT || NB == 1) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) base[nb] = deposit_cols<K>(tile * COLS + p + 32 * nb, g);
        } else {
            base[0] = deposit_cols<K>(tile * COLS + 2 * p, g);
            base[NB - 1] = base[0] | 1;
        }
    }
    __device__ __forceinline__ static void load(const float2* __restrict__ psi, const uint64_t (&base)[NB],
                                                uint64_t hoff, const ClusterGeom& g, float (&B)[NB][2 * HX]) {
        if (!LOWT && NB == 2) {
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const float4 v = *reinterpret_cast<const float4*>(psi + (base[0] | hoff | target_off<K - 1>(j, g)));
                B[0][2 * j] = v.x; B[0][2 * j + 1] = v.y;
                B[NB - 1][2 * j] = v.z; B[NB - 1][2 * j + 1] = v.w;
            }
        } else if (LOWT) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < HX; j += 2) {
                    const float4 v =
                        *reinterpret_cast<const float4*>(psi + (base[nb] | hoff | target_off<K - 1>(j, g)));
                    B[nb][2 * j] = v.x; B[nb][2 * j + 1] = v.y;
                    B[nb][2 * j + 2] = v.z; B[nb][2 * j + 3] = v.w;
                }
        } else {
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const float2 v = psi[base[0] | hoff | target_off<K - 1>(j, g)];
                B[0][2 * j] = v.x; B[0][2 * j + 1] = v.y;
            }
        }
    }
    __device__ __forceinline__ static void store(float2* __restrict__ psi, const uint64_t (&base)[NB], uint64_t hoff,
                                                 const ClusterGeom& g, const float (&O)[NB][2 * HX]) {
        if (!LOWT && NB == 2) {
#pragma unroll
            for (int j = 0; j < HX; ++j)
                *reinterpret_cast<float4*>(psi + (base[0] | hoff | target_off<K - 1>(j, g))) =
                    make_float4(O[0][2 * j], O[0][2 * j + 1], O[NB - 1][2 * j], O[NB - 1][2 * j + 1]);
        } else if (LOWT) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < HX; j += 2)
                    *reinterpret_cast<float4*>(psi + (base[nb] | hoff | target_off<K - 1>(j, g))) =
                        make_float4(O[nb][2 * j], O[nb][2 * j + 1], O[nb][2 * j + 2], O[nb][2 * j + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < HX; ++j)
                psi[base[0] | hoff | target_off<K - 1>(j, g)] = make_float2(O[0][2 * j], O[0][2 * j + 1]);
        }
    }
};

// Persistent: each wave walks tiles with a stride of the whole grid and
// prefetches the next tile's amplitudes into registers before it runs the
// current tile's MFMA chain, so loads stay in flight under the matrix work.
//
// STATS: the launch is the last op of a run; the kernel also sums p = |a|^2,
// p^2 and -p ln p of the amplitudes it stores (float64, per work-group into
// part[blockIdx.x * 8 + 0..2]), so the state need not be read again for them.
template <int K, int NB, bool LOWT, bool STATS = false>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_mfma(float2* __restrict__ psi,
                                                             const float* __restrict__ Ap,
                                                             const EpiDesc* __restrict__ epi,
                                                             ClusterGeom g, double* __restrict__ part) {
    using T = TileF32<K, NB, LOWT>;
    constexpr int D = 1 << K;
    constexpr int HX = D / 2;       // amplitudes per lane and column
    constexpr int RB = 2 * D / 32;  // 32-row blocks of the real-split matrix
    constexpr int S = D;            // MFMA steps (inner dimension 2^(K+1), 2 per step)
    __shared__ float As[RB * S * 64];
    load_matrix<RB * S * 64, 256>(As, reinterpret_cast<const vf4*>(Ap));
    __syncthreads();

    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const uint64_t hoff = h ? (uint64_t(1) << g.t[K - 1]) : 0;
    const uint64_t ntiles = g.ncols / T::COLS;
    const uint64_t stride = (uint64_t)gridDim.x * 4;
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;

    // The prefetch is unconditional (the last tile is re-read instead of
    // reading past the end) so the load count per iteration is fixed and the
    // waits the compiler places for the amplitudes cover only their own loads.
    uint64_t tile = (uint64_t)xcd_block() * 4 + (threadIdx.x >> 6);
    double sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (tile >= ntiles) {  // uniform in the wave: every wave reaches one reduction
        if constexpr (STATS) block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
        return;
    }
    const uint64_t last = ntiles - 1;
    float B[NB][2 * HX];
    uint64_t base[NB];
    T::bases(tile, p, g, base);
    T::load(psi, base, hoff, g, B);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    do {
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        float Bn[NB][2 * HX];
        uint64_t basen[NB];
        T::bases(nxt, p, g, basen);
        T::load(psi, basen, hoff, g, Bn);
        __builtin_amdgcn_sched_barrier(0);

        floatx16 acc[NB][RB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[nb][rb][i] = 0.0f;
        int aoff = lane;
        asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float a = As[(rb * S + s) * 64 + aoff];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb][rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, B[nb][s], acc[nb][rb], 0, 0, 0);
            }
        }
        // acc[nb][j / 8][2 (j % 8) + {0, 1}] is output amplitude j of the lane
        float O[NB][2 * HX];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < 2 * HX; ++j) O[nb][j] = acc[nb][j / 16][j % 16];
        if (has_epi) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const ColFactor<float> f = col_factor<float>(epi, base[nb]);
#pragma unroll
                for (int j = 0; j < HX; ++j)
                    apply_factor(O[nb][2 * j], O[nb][2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
            }
        }
        if constexpr (STATS) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < HX; ++j) stats_acc_f(sv, O[nb][2 * j], O[nb][2 * j + 1]);
        }
        T::store(psi, base, hoff, g, O);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            base[nb] = basen[nb];
#pragma unroll
            for (int j = 0; j < 2 * HX; ++j) B[nb][j] = Bn[nb][j];
        }
        tile += stride;
    } while (tile < ntiles);
    if constexpr (STATS) block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
}

// ------------------------------------------------------------ cluster: MFMA, float, k = 6
// Three-multiplication complex product: with M = Mr + i Mi and x = xr + i xi,
//   Re(M x) = Mr xr - Mi xi,   Im(M x) = (Mr + Mi)(xr + xi) - Mr xr - Mi xi,
// three real 64 x 64 products instead of the four blocks of the real-split
// matrix: 25% fewer matrix-core operations, which is what bounds k = 6.
// v_mfma_f32_16x16x4_f32: operand lane l holds row / column l % 16 at inner
// index l / 16; result register r of lane l holds row 4 (l / 16) + r. Wave
// tile: 16 columns; lane (p, q) = (l % 16, l / 16) owns amplitudes j | q << 4,
// j < 16, of column p. At step s the lane supplies inner index s | q << 4,
// its own amplitude j = s; result register r of row block rb lands on its
// amplitude (4 rb + r) | q << 4 (the builder permutes the matrix rows so).
template <bool LOWT>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_gauss6(float2* __restrict__ psi,
                                                               const float* __restrict__ Ap,
                                                               const EpiDesc* __restrict__ epi,
                                                               ClusterGeom g) {
    constexpr int K = 6, HX = 16;
    __shared__ float As[3 * 4 * 16 * 64];
    load_matrix<3 * 4 * 16 * 64, 256>(As, reinterpret_cast<const vf4*>(Ap));
    __syncthreads();

    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
    const uint64_t qoff = ((q & 1) ? uint64_t(1) << g.t[4] : 0) | ((q >> 1) ? uint64_t(1) << g.t[5] : 0);
    const uint64_t ntiles = g.ncols / 16;
    const uint64_t stride = (uint64_t)gridDim.x * 4;
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;

    uint64_t tile = (uint64_t)xcd_block() * 4 + (threadIdx.x >> 6);
    if (tile >= ntiles) return;
    const uint64_t last = ntiles - 1;
    auto load = [&](uint64_t b, float (&X)[2 * HX]) {
        if (LOWT) {
#pragma unroll
            for (int j = 0; j < HX; j += 2) {
                const float4 v = *reinterpret_cast<const float4*>(psi + (b | target_off<4>(j, g)));
                X[2 * j] = v.x; X[2 * j + 1] = v.y; X[2 * j + 2] = v.z; X[2 * j + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const float2 v = psi[b | target_off<4>(j, g)];
                X[2 * j] = v.x; X[2 * j + 1] = v.y;
            }
        }
    };
    uint64_t base = deposit_cols<K>(tile * 16 + p, g);
    float B[2 * HX];
    load(base | qoff, B);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    do {
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        const uint64_t basen = deposit_cols<K>(nxt * 16 + p, g);
        float Bn[2 * HX];
        load(basen | qoff, Bn);
        __builtin_amdgcn_sched_barrier(0);

        ColFactor<float> f{0u, 0u, 1.0f, 0.0f};
        if (has_epi) f = col_factor<float>(epi, base);
        vf4 a1[4], a2[4], a3[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) a1[rb][i] = a2[rb][i] = a3[rb][i] = 0.0f;
        int aoff = lane;
        asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
        for (int st = 0; st < 16; ++st) {
            const float xr = B[2 * st], xi = B[2 * st + 1], xs = xr + xi;
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                a1[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(As[((0 * 4 + rb) * 16 + st) * 64 + aoff], xr, a1[rb], 0,
                                                             0, 0);
                a2[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(As[((1 * 4 + rb) * 16 + st) * 64 + aoff], xi, a2[rb], 0,
                                                             0, 0);
                a3[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(As[((2 * 4 + rb) * 16 + st) * 64 + aoff], xs, a3[rb], 0,
                                                             0, 0);
            }
        }
        // amplitude j = 4 rb + r of the lane
        float O[2 * HX];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                O[2 * (4 * rb + r)] = a1[rb][r] - a2[rb][r];
                O[2 * (4 * rb + r) + 1] = a3[rb][r] - a1[rb][r] - a2[rb][r];
            }
        if (has_epi) {
#pragma unroll
            for (int j = 0; j < HX; ++j)
                apply_factor(O[2 * j], O[2 * j + 1], f, (uint32_t)(j | (q << 4)), has_ph);
        }
        const uint64_t b0 = base | qoff;
        if (LOWT) {
#pragma unroll
            for (int j = 0; j < HX; j += 2)
                *reinterpret_cast<float4*>(psi + (b0 | target_off<4>(j, g))) =
                    make_float4(O[2 * j], O[2 * j + 1], O[2 * j + 2], O[2 * j + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < HX; ++j) psi[b0 | target_off<4>(j, g)] = make_float2(O[2 * j], O[2 * j + 1]);
        }
        base = basen;
#pragma unroll
        for (int j = 0; j < 2 * HX; ++j) B[j] = Bn[j];
        tile += stride;
    } while (tile < ntiles);
}

// ------------------------------------------------------------ cluster: float state, k = 6, fp16 matrix cores
// The real-split product of a 6-qubit cluster needs 32 flop per byte of state,
// beyond what the fp32 matrix cores sustain at HBM speed. The fp16 matrix
// cores are 16 times faster, so the product runs on them with each operand
// split into two halves, v = hi + lo (hi = fp16(v), lo = fp16(v - hi)):
//   A x ~= A_hi x_hi + A_hi x_lo + A_lo x_hi,
// accumulated in fp32 (the dropped A_lo x_lo and the split residuals are
// ~2^-22 relative, the size of fp32 rounding). The matrix is stored as
// 16 M, split by the builder. Each column of the state tile is scaled by a
// power of two that puts its largest magnitude just below 2^14 (exact, and no
// fp16 overflow for any input), and its results are scaled back.
// v_mfma_f32_32x32x16_f16: operand lane l, element i holds row / column l % 32
// at inner index 8 (l / 32) + i; result register r of lane l holds row
// 8 (r / 4) + 4 (l / 32) + r % 4 (as for the fp32 32x32 instruction). Lane
// (p, h) owns amplitudes j | h << 5 of column p; at step s it supplies its
// floats 8 s .. 8 s + 7 (amplitudes 4 s .. 4 s + 3, re / im interleaved).
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// fp16 halves of two scaled floats, packed: H = (f16(x0 sc), f16(x1 sc)),
// L = (f16(x0 sc - H.lo), f16(x1 sc - H.hi)), rounded to nearest even - the
// arithmetic of (_Float16)(x * sc) and (_Float16)(x * sc - hi), four
// mixed-precision FMAs per pair (checked bit for bit against that form; the
// compiler's own code computed the high halves twice to pack them).
__device__ __forceinline__ void split_pair_f16(float x0, float x1, float sc, uint32_t& H, uint32_t& L) {
    __asm__("v_fma_mixlo_f16 %0, %2, %4, 0\n\t"
            "v_fma_mixhi_f16 %0, %3, %4, 0\n\t"
            "v_fma_mixlo_f16 %1, %2, %4, -%0 op_sel_hi:[0,0,1]\n\t"
            "v_fma_mixhi_f16 %1, %3, %4, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
            : "=&v"(H), "=&v"(L)
            : "v"(x0), "v"(x1), "v"(sc));
}

// The fp16 halves (hi, lo) of a lane's N floats of one column, scaled by the
// power of two that puts the column's largest magnitude (over this lane and
// its partner lane, lane ^ 32) just below 2^14: exact scaling, no fp16
// overflow for any input, zero columns stay zero. Returns the exponent se
// of that scale (the results are scaled back by 2^(-se) times the matrix's
// own 2^-4). Float i of the lane is element i % 8 of xh / xl[i / 8].
template <int N>
__device__ __forceinline__ int split_halves(const float (&X)[N], half8 (&xh)[N / 8], half8 (&xl)[N / 8]) {
    float mx = 0.0f;  // |x| is a free operand modifier of the max
#pragma unroll
    for (int i = 0; i < N; ++i) mx = fmaxf(mx, fabsf(X[i]));
    const uint32_t mb = max(__float_as_uint(mx), (uint32_t)__shfl_xor((int)__float_as_uint(mx), 32));
    const int e = (int)(mb >> 23) - 126;  // largest magnitude < 2^e
    const int se = min(max(14 - e, -100), 100);
    const float sc = __builtin_ldexpf(1.0f, se);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int st = 0; st < N / 8; ++st) {
        u32x4 h, l;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t a, b;
            split_pair_f16(X[8 * st + 2 * q], X[8 * st + 2 * q + 1], sc, a, b);
            h[q] = a;
            l[q] = b;
        }
        xh[st] = __builtin_bit_cast(half8, h);
        xl[st] = __builtin_bit_cast(half8, l);
    }
    return se;
}


// Swap a (in the odd 16-lane rows of the wave) with b (in the even rows):
// afterwards lane l of an even row holds in b what lane l + 16 held in a, and
// lane l + 16 holds in a what lane l held in b.
__device__ __forceinline__ void lane_swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// One wave tile per wave, work-groups in memory order; NT: a state beyond the
// caches. Bound by HBM (the product takes about half of the pass). 30 qubits,
// 23 target sets: 3.0 ms per pass (5.7 TB/s) where accesses cover whole lines,
// 3.45 ms as a persistent grid with 8-byte accesses.
template <bool LOWT, bool NT>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_split6(float2* __restrict__ psi,
                                                               const half8* __restrict__ Ap,
                                                               const EpiDesc* __restrict__ epi,
                                                               ClusterGeom g) {
    constexpr int K = 6, HX = 32, RB = 4, S = 8, NP = RB * S * 64;
    __shared__ half8 L[2 * NP];  // hi, lo
    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    // without a target on qubit 0, lanes p and p + 16 hold neighbouring
    // columns and access both as 16 bytes, even rows in the lower lane, odd
    // rows in the upper (as in k_cluster_f32_split7)
    constexpr bool PAIR = !LOWT;
    const int cpair = PAIR ? 2 * (p & 15) : p;
    const uint64_t cown = PAIR ? (uint64_t)((p >> 4) & 1) : 0;
    const uint64_t tile = (uint64_t)tile_block<4 * 2048 * 8>() * 4 + (threadIdx.x >> 6);
    const uint64_t base = deposit_cols<K>(tile * 32 + cpair, g);
    const uint64_t b0 = base | (h ? uint64_t(1) << g.t[K - 1] : 0) | (cown ? uint64_t(1) << g.t[0] : 0);
    float X[2 * HX];
    MatrixRegs<2 * NP * 16, 256> mr(Ap);
    const bool act = tile < g.ncols / 32;
    if (act) {
#pragma unroll
        for (int j = 0; j < HX; j += 2) {
            const vf4* q = reinterpret_cast<const vf4*>(psi + (b0 | target_off<K - 1>(j, g)));
            const vf4 v = load16<NT>(q);
            X[2 * j] = v.x; X[2 * j + 1] = v.y; X[2 * j + 2] = v.z; X[2 * j + 3] = v.w;
        }
    }
    mr.store(L);
    __syncthreads();
    if (!act) return;
    if constexpr (PAIR) {  // rows j, j + 1 of the lane's own column
#pragma unroll
        for (int j = 0; j < HX; j += 2) {
            lane_swap16(X[2 * j], X[2 * j + 2]);
            lane_swap16(X[2 * j + 1], X[2 * j + 3]);
        }
    }
    half8 xh[S], xl[S];
    const float unscale = __builtin_ldexpf(1.0f, -split_halves<2 * HX>(X, xh, xl) - 4);
    floatx16 acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
#pragma unroll
    for (int st = 0; st < S; ++st) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const half8 ah = L[(rb * S + st) * 64 + lane];
            const half8 al = L[NP + (rb * S + st) * 64 + lane];
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
        }
    }
    float O[2 * HX];
#pragma unroll
    for (int j = 0; j < 2 * HX; ++j) O[j] = acc[j / 16][j % 16] * unscale;
    if (epi != nullptr) {
        const ColFactor<float> f = col_factor<float>((c_epi*)epi, base | cown);
        const bool has_ph = epi->n_ph > 0;
#pragma unroll
        for (int j = 0; j < HX; ++j)
            apply_factor(O[2 * j], O[2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
    }
#pragma unroll
    for (int j = 0; j < HX; j += 2) {
        if constexpr (PAIR) {  // row j of both columns (lower lane), row j + 1 (upper)
            lane_swap16(O[2 * j], O[2 * j + 2]);
            lane_swap16(O[2 * j + 1], O[2 * j + 3]);
        }
        vf4* q = reinterpret_cast<vf4*>(psi + (b0 | target_off<K - 1>(j, g)));
        const vf4 v{O[2 * j], O[2 * j + 1], O[2 * j + 2], O[2 * j + 3]};
        store16<NT>(q, v);
    }
}

// The last op of a run whose sums are wanted: as the STATS form of
// k_cluster_f32_mfma, it also sums the stored amplitudes' p, p^2 and -p ln p
// into part, per work-group. Persistent, since the partials of one work-group
// per tile would not fit their area; the next tile is prefetched.
template <bool LOWT>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_split6_sum(float2* __restrict__ psi,
                                                               const half8* __restrict__ Ap,
                                                               const EpiDesc* __restrict__ epi,
                                                               ClusterGeom g, double* __restrict__ part) {
    constexpr int K = 6, HX = 32, RB = 4, S = 8;
    using T = TileF32<K, 1, LOWT>;
    __shared__ half8 Ah[RB * S * 64];
    __shared__ half8 Al[RB * S * 64];
    load_matrix<RB * S * 64 * 8, 256>(reinterpret_cast<_Float16*>(Ah), reinterpret_cast<const vf4*>(Ap));
    load_matrix<RB * S * 64 * 8, 256>(reinterpret_cast<_Float16*>(Al),
                                      reinterpret_cast<const vf4*>(Ap + RB * S * 64));
    __syncthreads();

    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const uint64_t hoff = h ? (uint64_t(1) << g.t[K - 1]) : 0;
    const uint64_t ntiles = g.ncols / 32;
    const uint64_t stride = (uint64_t)gridDim.x * 4;
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;

    uint64_t tile = (uint64_t)xcd_block() * 4 + (threadIdx.x >> 6);
    double sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (tile >= ntiles) {  // uniform in the wave: every wave reaches one reduction
        block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
        return;
    }
    const uint64_t last = ntiles - 1;

    // split the column's amplitudes (scaled) into fp16 halves; returns the
    // factor that undoes the column and matrix scaling
    auto split = [&](const float (&X)[2 * HX], half8 (&xh)[S], half8 (&xl)[S]) -> float {
        return __builtin_ldexpf(1.0f, -split_halves<2 * HX>(X, xh, xl) - 4);
    };

    float B[1][2 * HX];
    uint64_t base[1];
    T::bases(tile, p, g, base);
    T::load(psi, base, hoff, g, B);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    half8 xh[S], xl[S];
    float unscale = split(B[0], xh, xl);
    do {
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        float Bn[1][2 * HX];
        uint64_t basen[1];
        T::bases(nxt, p, g, basen);
        T::load(psi, basen, hoff, g, Bn);
        __builtin_amdgcn_sched_barrier(0);

        floatx16 acc[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
        int aoff = lane;
        asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
        for (int st = 0; st < S; ++st) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const half8 ah = Ah[(rb * S + st) * 64 + aoff];
                const half8 al = Al[(rb * S + st) * 64 + aoff];
                acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
                acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
                acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
            }
        }
        float O[1][2 * HX];
#pragma unroll
        for (int j = 0; j < 2 * HX; ++j) O[0][j] = acc[j / 16][j % 16] * unscale;
        if (has_epi) {
            const ColFactor<float> f = col_factor<float>(epi, base[0]);
#pragma unroll
            for (int j = 0; j < HX; ++j)
                apply_factor(O[0][2 * j], O[0][2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
        }
#pragma unroll
        for (int j = 0; j < HX; ++j) stats_acc_f(sv, O[0][2 * j], O[0][2 * j + 1]);
        T::store(psi, base, hoff, g, O);
        base[0] = basen[0];
        unscale = split(Bn[0], xh, xl);
        tile += stride;
    } while (tile < ntiles);
    block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
}

// A column's diagonal-epilogue factor (col_factor), split for a wave that
// walks many tiles: terms on the state bits above the tile (uniform in the
// wave, new each tile) and terms on the column bits (fixed per lane) are
// separate, and a CZ pair with one qubit of each kind is a mask over the
// column index, set per tile. Target bits take no part (the host moved such
// terms into the matrix or the mask over rows).
// Tile part of base (tile bits zero) for a K-qubit cluster: bit 0 the sign,
// bits 1..K the mask over rows, the 5 bits above them the mask over the
// column index; the phase in (cr, ci).
template <int K = 6>
__device__ __forceinline__ uint32_t epi_tile_part(c_epi* __restrict__ e, uint64_t base, uint64_t colmask,
                                                  double& cr, double& ci) {
    uint32_t sgn = 0, w = 0, cross = 0;
    const int ncc = e->n_cc;
    for (int i = 0; i < ncc; ++i) {
        const int a = e->cc[i][0], b = e->cc[i][1];
        const bool ca = (colmask >> a) & 1, cb = (colmask >> b) & 1;
        if (!ca && !cb)
            sgn ^= (uint32_t)((base >> a) & (base >> b) & 1);
        else if (ca && !cb)
            cross ^= (uint32_t)((base >> b) & 1) << __popcll(colmask & ((uint64_t(1) << a) - 1));
        else if (!ca && cb)
            cross ^= (uint32_t)((base >> a) & 1) << __popcll(colmask & ((uint64_t(1) << b) - 1));
    }
    const int nm = e->n_mix;
    for (int i = 0; i < nm; ++i) {
        const int b = e->mix[i][1];
        if (!((colmask >> b) & 1)) w ^= (uint32_t)((base >> b) & 1) << e->mix[i][0];
    }
    cr = 1.0;
    ci = 0.0;
    const int np = e->n_ph;
    for (int i = 0; i < np; ++i) {
        const int q = e->ph_q[i];
        if (!((colmask >> q) & 1) && ((base >> q) & 1)) {
            const double a = e->ph[i][0], b = e->ph[i][1];
            const double t = cr * a - ci * b;
            ci = cr * b + ci * a;
            cr = t;
        }
    }
    return sgn | (w << 1) | (cross << (K + 1));
}

// Column part of the same factor (cbits: the column's state bits).
__device__ __forceinline__ void epi_lane_part(c_epi* __restrict__ e, uint64_t cbits, uint64_t colmask, uint32_t& sgn,
                                              uint32_t& w, double& cr, double& ci) {
    sgn = 0;
    w = 0;
    const int ncc = e->n_cc;
    for (int i = 0; i < ncc; ++i) {
        const int a = e->cc[i][0], b = e->cc[i][1];
        if (((colmask >> a) & 1) && ((colmask >> b) & 1)) sgn ^= (uint32_t)((cbits >> a) & (cbits >> b) & 1);
    }
    const int nm = e->n_mix;
    for (int i = 0; i < nm; ++i) {
        const int b = e->mix[i][1];
        if ((colmask >> b) & 1) w ^= (uint32_t)((cbits >> b) & 1) << e->mix[i][0];
    }
    cr = 1.0;
    ci = 0.0;
    const int np = e->n_ph;
    for (int i = 0; i < np; ++i) {
        const int q = e->ph_q[i];
        if (((colmask >> q) & 1) && ((cbits >> q) & 1)) {
            const double a = e->ph[i][0], b = e->ph[i][1];
            const double t = cr * a - ci * b;
            ci = cr * b + ci * a;
            cr = t;
        }
    }
}

// Combine the two parts for column index p (tile part read from its lane).
template <int K = 6>
__device__ __forceinline__ ColFactor<float> epi_combine(uint32_t tb, double tr, double ti, uint32_t ls, uint32_t lw,
                                                        double lr, double li, int p) {
    ColFactor<float> f;
    f.sgn = ls ^ (tb & 1u) ^ ((uint32_t)__popc((uint32_t)p & (tb >> (K + 1)) & 31u) & 1u);
    f.w = lw ^ ((tb >> 1) & ((1u << K) - 1u));
    f.cr = (float)(tr * lr - ti * li);
    f.ci = (float)(tr * li + ti * lr);
    return f;
}

// ------------------------------------------------------------ cluster: float state, k = 7, fp16 matrix cores
// A 7-qubit cluster doubles the matrix work per byte of state of a 6-qubit
// one and still stays below the HBM time on the fp16 matrix cores, so it
// takes the same operand halves (A x ~= A_hi x_hi + A_hi x_lo + A_lo x_hi,
// fp32 accumulation). Its real-split matrix (2^8 x 2^8 entries) would not fit
// in LDS, so the complex product is written with the real and imaginary
// parts of M instead (Sec. 3.2, Eqs. (1)-(3)):
//   Re y = Re M Re x - Im M Im x,   Im y = Im M Re x + Re M Im x,
// four real products on two matrices (their halves: 128 KiB of LDS; the
// minus sign goes onto the halves of Im x, an exact sign flip). One
// work-group of 4 waves per compute unit.
// Wave tile: 32 columns x 2^7 targets. Lane l: p = l % 32 (column), h = l / 32
// owns the amplitudes j | h << 6 (j < 64) of its column, for its loads and
// its stores. v_mfma_f32_32x32x16_f16: at step s the lane supplies the halves
// of its amplitudes j = 8 s .. 8 s + 7 (inner index 16 s + 8 h + i <->
// amplitude (8 s + i) | h << 6); result register r of row block rb holds its
// amplitude j = 16 rb + r (physical row 8 (r / 4) + 4 h + r % 4). The builder
// permutes M once to match (LAYOUT_SPLIT7).
template <bool LOWT, bool STATS = false, bool NT = false>
__global__ __launch_bounds__(256, 1) void k_cluster_f32_split7(float2* __restrict__ psi,
                                                               const half8* __restrict__ Ap,
                                                               const EpiDesc* __restrict__ epi,
                                                               ClusterGeom g, double* __restrict__ part,
                                                               uint32_t* __restrict__ tickets) {
    constexpr int K = 7, HX = 64, RB = 4, S = 8, NP = RB * S * 64;
    // parts: 16 Re M hi, lo, 16 Im M hi, lo; entry (rb, s, lane) of each
    __shared__ half8 L[4 * NP];
    load_matrix<4 * NP * 8, 256>(reinterpret_cast<_Float16*>(L), reinterpret_cast<const vf4*>(Ap));
    __syncthreads();

    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const uint64_t hoff = h ? (uint64_t(1) << g.t[K - 1]) : 0;
    // Without a target on qubit 0 the tile's columns are neighbouring
    // amplitudes. Lanes p and p + 16 (p < 16 within each half-wave) then hold
    // columns 2 p and 2 p + 1: each accesses both columns of every other row
    // (even rows in the lower lane, odd ones in the upper) as one 16 byte
    // access, and one lane swap per 32-bit value (v_permlane16_swap, between
    // the two 16-lane rows) gives each lane its own column after a load and
    // the pair of columns before a store. Half the memory instructions of
    // 8-byte accesses, for the same 256-byte runs: 2 % off the pass. Not in
    // the STATS form, whose store phase is bound by its float64 sums (the
    // swaps made it 3 % slower). With a target on qubit 0 the 16 byte
    // accesses are two rows of the lane's own column.
    constexpr bool PAIR = !LOWT && !STATS;
    const int cpair = PAIR ? 2 * (p & 15) : p;                  // first column of the lane's accesses
    const uint64_t cown = PAIR ? (uint64_t)((p >> 4) & 1) : 0;  // the lane's own column: cpair + cown
    const uint64_t roff = cown ? (uint64_t(1) << g.t[0]) : 0;   // odd rows
    const uint64_t ntiles = g.ncols / 32;
    // Beyond the caches tiles are handed out in order, by one counter per XCD for
    // its own eighth of the state, so that the waves, which drift apart, still
    // work on one compact stretch per XCD (30 qubits, 23 target sets: 3.45 ms per
    // pass against 3.55 ms with a fixed stride, 3.74 ms without non-temporal
    // accesses as well); smaller states take a fixed stride (20 qubits: the
    // counters cost 0.7 us), and so do passes that take the sums, which come out
    // the same bit for bit only if a wave's tiles are.
    const bool dealt = tickets != nullptr;
    const uint32_t mine = dealt ? blockIdx.x & 7 : 0u;
    const uint32_t nmine = (uint32_t)(dealt ? ntiles / 8 : ntiles);
    const uint64_t tile0 = (uint64_t)mine * nmine;
    const uint32_t stride = gridDim.x * 4;
    auto take = [&](uint32_t fixed) -> uint32_t {  // the next tile's number (dealt: in lane 0)
        return dealt ? (lane == 0 ? atomicAdd(tickets + mine * 32, 1u) : 0u) : fixed;
    };
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;
    // state offset of the lane's amplitude j = 8 a + i: olo[i] | ohi[a] (bits of
    // j on targets 0..2 and 3..5; target 6 is h)
    uint64_t olo[8], ohi[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        olo[i] = target_off<3>(i, g);
        ohi[i] = ((i & 1) ? uint64_t(1) << g.t[3] : 0) | ((i & 2) ? uint64_t(1) << g.t[4] : 0) |
                 ((i & 4) ? uint64_t(1) << g.t[5] : 0);
    }

    uint32_t cur = __builtin_amdgcn_readfirstlane(take(xcd_block() * 4 + (threadIdx.x >> 6)));
    double sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (cur >= nmine) {  // uniform in the wave: every wave reaches one reduction
        if constexpr (STATS) block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
        return;
    }
    uint32_t ahead = take(cur + stride);
    // amplitudes 8 a .. 8 a + 7 of the lane for a in [A0, A1)
    // (the bits are disjoint, so the OR is a sum: one pointer per group a,
    // then the low offsets added to it)
    // (b: the lane's access base, odd-row offset included)
    auto load = [&](uint64_t b, float (&X)[2 * HX], int a0, int a1) {
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            if (a < a0 || a >= a1) continue;
            const float2* pa = psi + (b | ohi[a]);
            if (LOWT || PAIR) {
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    const vf4 v = load16<NT>(reinterpret_cast<const vf4*>(pa + olo[i]));
                    const int j = 8 * a + i;
                    X[2 * j] = v.x; X[2 * j + 1] = v.y; X[2 * j + 2] = v.z; X[2 * j + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float2 v = pa[olo[i]];
                    const int j = 8 * a + i;
                    X[2 * j] = v.x; X[2 * j + 1] = v.y;
                }
            }
        }
    };
    // real and imaginary parts of amplitudes 8 s + i, scaled, into fp16
    // halves; returns the factor that undoes the column and matrix scaling
    half8 rh[S], rl[S], ih[S], il[S];
    auto split = [&](float (&X)[2 * HX]) -> float {
        if constexpr (PAIR) {  // rows j, j + 1 of the lane's own column
#pragma unroll
            for (int j = 0; j < HX; j += 2) {
                lane_swap16(X[2 * j], X[2 * j + 2]);
                lane_swap16(X[2 * j + 1], X[2 * j + 3]);
            }
        }
        float mx = 0.0f;  // largest magnitude (|x| is a free operand modifier of the max)
#pragma unroll
        for (int i = 0; i < 2 * HX; ++i) mx = fmaxf(mx, fabsf(X[i]));
        uint32_t mb = __float_as_uint(mx);
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 32));  // the other half of the column
        const int e = (int)(mb >> 23) - 126;               // largest magnitude < 2^e
        const int se = min(max(14 - e, -100), 100);
        const float sc = __builtin_ldexpf(1.0f, se);
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            u32x4 hr, lr, hi4, li4;
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // amplitudes j, j + 1: halves q of the registers
                const int j = 8 * s + 2 * q;
                uint32_t a, b, c, d;
                split_pair_f16(X[2 * j], X[2 * j + 2], sc, a, b);
                split_pair_f16(X[2 * j + 1], X[2 * j + 3], sc, c, d);
                hr[q] = a;
                lr[q] = b;
                hi4[q] = c;
                li4[q] = d;
            }
            rh[s] = __builtin_bit_cast(half8, hr);
            rl[s] = __builtin_bit_cast(half8, lr);
            ih[s] = __builtin_bit_cast(half8, hi4);
            il[s] = __builtin_bit_cast(half8, li4);
        }
        return __builtin_ldexpf(1.0f, -se - 4);
    };
    floatx16 ar[RB], ai[RB];
    // the products of steps s0 .. s1 - 1
    auto mma = [&](int s0, int s1) {
        int aoff = lane;
        asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (s < s0 || s >= s1) continue;
            // -Im x: the sign bits of both packed halves flipped by one XOR per register
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 sbit = {0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
            const half8 nh = __builtin_bit_cast(half8, __builtin_bit_cast(u32x4, ih[s]) ^ sbit);
            const half8 nl = __builtin_bit_cast(half8, __builtin_bit_cast(u32x4, il[s]) ^ sbit);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int at = (rb * S + s) * 64 + aoff;
                const half8 Rh = L[at], Rl = L[NP + at], Ih = L[2 * NP + at], Il = L[3 * NP + at];
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rh, rl[s], ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ih, rl[s], ai[rb], 0, 0, 0);
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rl, rh[s], ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Il, rh[s], ai[rb], 0, 0, 0);
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rh, rh[s], ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ih, rh[s], ai[rb], 0, 0, 0);
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ih, nl, ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rh, il[s], ai[rb], 0, 0, 0);
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Il, nh, ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rl, ih[s], ai[rb], 0, 0, 0);
                ar[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ih, nh, ar[rb], 0, 0, 0);
                ai[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Rh, ih[s], ai[rb], 0, 0, 0);
            }
        }
    };

    uint64_t base = deposit_cols<K>((tile0 + cur) * 32 + cpair, g);
    float unscale;
    {
        float B[2 * HX];
        load(base | hoff | roff, B, 0, 8);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_sched_barrier(0);
        unscale = split(B);
    }
    do {
        // past the end the last tile is read again, so that every round has the
        // same loads; the number after it is on its way meanwhile
        const uint32_t nxt = __builtin_amdgcn_readfirstlane(ahead);
        const uint64_t basen = deposit_cols<K>((tile0 + min(nxt, nmine - 1)) * 32 + cpair, g);
        ahead = take(nxt + stride);
        // the next tile's loads go out in two halves: the second once the
        // first four steps have freed their operand registers
        float Bn[2 * HX];
        load(basen | hoff | roff, Bn, 0, 4);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) ar[rb][i] = ai[rb][i] = 0.0f;
        mma(0, 4);
        __builtin_amdgcn_sched_barrier(0);
        load(basen | hoff | roff, Bn, 4, 8);
        __builtin_amdgcn_sched_barrier(0);
        mma(4, 8);
        // Diagonal epilogue: the column's sign parity and phase are one complex
        // factor for all its amplitudes, so they join the scale (ucr, uci);
        // the sign mask over the target index becomes bit j of msk for the
        // lane's amplitude j (target 6 is the lane's h: its term is the
        // column's). The store loop is specialised on which parts are present.
        float ucr = unscale, uci = 0.0f;
        uint32_t mlo = 0, mhi = 0;  // bit j of mhi:mlo: amplitude j changes sign
        bool ph = false, sg = false;
        if (has_epi) {
            const ColFactor<float> f = col_factor<float>(epi, base | cown);
            if ((f.sgn ^ ((uint32_t)h & (f.w >> (K - 1)))) & 1u) ucr = -ucr;
            if (has_ph) {
                uci = ucr * f.ci;
                ucr = ucr * f.cr;
                ph = true;
            }
            const uint32_t pat[5] = {0xaaaaaaaau, 0xccccccccu, 0xf0f0f0f0u, 0xff00ff00u, 0xffff0000u};
#pragma unroll
            for (int b = 0; b < 5; ++b)
                if ((f.w >> b) & 1u) {
                    mlo ^= pat[b];
                    mhi ^= pat[b];
                }
            if ((f.w >> 5) & 1u) mhi = ~mhi;
            sg = epi->n_mix > 0;  // uniform: the descriptor has sign-mask terms
        }
        const uint64_t b0 = base | hoff | roff;
        auto store_all = [&](auto PH, auto SG) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const int j = 16 * rb + r;
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const float xr = ar[rb][r + u], xi = ai[rb][r + u];
                        if constexpr (decltype(PH)::value) {  // one fixed contraction in every variant
                            v[2 * u] = fmaf(xr, ucr, -(xi * uci));
                            v[2 * u + 1] = fmaf(xr, uci, xi * ucr);
                        } else {
                            v[2 * u] = xr * ucr;
                            v[2 * u + 1] = xi * ucr;
                        }
                        if constexpr (decltype(SG)::value) {
                            const int jj = j + u;
                            const uint32_t m = jj < 32 ? mlo : mhi;
                            const uint32_t sb = (m << (31 - (jj & 31))) & 0x80000000u;
                            v[2 * u] = __uint_as_float(__float_as_uint(v[2 * u]) ^ sb);
                            v[2 * u + 1] = __uint_as_float(__float_as_uint(v[2 * u + 1]) ^ sb);
                        }
                    }
                    if constexpr (STATS) {
                        stats_acc_f(sv, v[0], v[1]);
                        stats_acc_f(sv, v[2], v[3]);
                    }
                    if constexpr (PAIR) {  // row j of both columns (lower lane), row j + 1 (upper)
                        lane_swap16(v[0], v[2]);
                        lane_swap16(v[1], v[3]);
                    }
                    float2* pa = psi + (b0 | ohi[j >> 3]);
                    if (LOWT || PAIR) {
                        store16<NT>(reinterpret_cast<vf4*>(pa + olo[j & 7]), vf4{v[0], v[1], v[2], v[3]});
                    } else {
                        pa[olo[j & 7]] = make_float2(v[0], v[1]);
                        pa[olo[(j + 1) & 7]] = make_float2(v[2], v[3]);
                    }
                }
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        if constexpr (STATS) {  // once per run: one general path (uci = 0, no mask bits when absent)
            store_all(T_(), T_());
        } else if (ph) {
            if (sg) store_all(T_(), T_()); else store_all(T_(), F_());
        } else {
            if (sg) store_all(F_(), T_()); else store_all(F_(), F_());
        }
        base = basen;
        unscale = split(Bn);
        cur = nxt;
    } while (cur < nmine);
    if constexpr (STATS) block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);
}

// ------------------------------------------------------------ cluster: MFMA, double
// v_mfma_f64_16x16x4_f64: lane l: p = l%16 (column), q = l/16 owns target
// indices x = j | q << (K-2), j < 2^(K-2), of its column(s). Operand A/B: lane
// l holds row / column l%16 at inner index l/16; result register r of lane l
// holds row 4 r + l/16, column l%16.
//
// k = 3..5: one wave tile of 16 NB columns per wave, work-groups in memory order.
// k = 5 keeps the fp64 matrix cores busy for two thirds of the pass, so its
// tiles are narrow (NB = 1) and four waves share a SIMD.
template <int K, int NB, bool NT>
__global__ __launch_bounds__(256, NB == 1 ? 4 : 2) void k_cluster_f64_mfma(vd2* __restrict__ psi, const double* __restrict__ Ap,
                                                             const EpiDesc* __restrict__ epi, ClusterGeom g) {
    constexpr int D = 1 << K, HX = D / 4, RB = 2 * D / 16, S = 2 * D / 4, COLS = 16 * NB;
    __shared__ double As[RB * S * 64];
    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
    const uint64_t qoff = ((q & 1) ? (uint64_t(1) << g.t[K - 2]) : 0) | ((q & 2) ? (uint64_t(1) << g.t[K - 1]) : 0);
    const uint64_t tile = (uint64_t)tile_block<4 * D * COLS * 16>() * 4 + (threadIdx.x >> 6);
    const bool act = tile < g.ncols / COLS;
    uint64_t base[NB];
    double B[NB][2 * HX];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) base[nb] = deposit_cols<K>(tile * COLS + p + 16 * nb, g);
    MatrixRegs<RB * S * 64 * 8, 256> mr(Ap);
    if (act) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const vd2 v = load16<NT>(psi + (base[nb] | qoff | target_off<K - 2>(j, g)));
                B[nb][2 * j] = v.x;
                B[nb][2 * j + 1] = v.y;
            }
    }
    mr.store(As);
    __syncthreads();
    if (!act) return;
    doublex4 acc[NB][RB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[nb][rb][i] = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const double a = As[(rb * S + s) * 64 + lane];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[nb][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[nb][s], acc[nb][rb], 0, 0, 0);
        }
    }
    // acc[nb][j / 2][2 (j % 2) + {0, 1}] is output amplitude j of the lane
    const bool has_epi = epi != nullptr, has_ph = has_epi && epi->n_ph > 0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        ColFactor<double> f{0u, 0u, 1.0, 0.0};
        if (has_epi) f = col_factor<double>((c_epi*)epi, base[nb]);
#pragma unroll
        for (int j = 0; j < HX; ++j) {
            double re = acc[nb][j / 2][2 * (j % 2)], im = acc[nb][j / 2][2 * (j % 2) + 1];
            if (has_epi) apply_factor(re, im, f, (uint32_t)(j | (q << (K - 2))), has_ph);
            store16<NT>(psi + (base[nb] | qoff | target_off<K - 2>(j, g)), vd2{re, im});
        }
    }
}

// k = 6 (bound by the fp64 matrix cores; its matrix fills the LDS):
// persistent, each wave prefetches its next tile of 16 columns before the
// current tile's MFMA chain.
template <int K, int NB, int THREADS>
__global__ __launch_bounds__(THREADS, 512 / THREADS) void k_cluster_f64_mfma_loop(double2* __restrict__ psi,
                                                                           const double* __restrict__ Ap,
                                                                           const EpiDesc* __restrict__ epi,
                                                                           ClusterGeom g) {
    constexpr int D = 1 << K;
    constexpr int HX = D / 4;
    constexpr int RB = 2 * D / 16;
    constexpr int S = 2 * D / 4;
    constexpr int COLS = 16 * NB;
    constexpr int WAVES = THREADS / 64;
    __shared__ double As[RB * S * 64];
    load_matrix<RB * S * 64, THREADS>(As, reinterpret_cast<const vf4*>(Ap));
    __syncthreads();

    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
    const uint64_t qoff = ((q & 1) ? (uint64_t(1) << g.t[K - 2]) : 0) | ((q & 2) ? (uint64_t(1) << g.t[K - 1]) : 0);
    const uint64_t ntiles = g.ncols / COLS;
    const uint64_t stride = (uint64_t)gridDim.x * WAVES;
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;

    auto load = [&](uint64_t t, uint64_t (&bs)[NB], double (&B)[NB][2 * HX]) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bs[nb] = deposit_cols<K>(t * COLS + p + 16 * nb, g);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const double2 v = psi[bs[nb] | qoff | target_off<K - 2>(j, g)];
                B[nb][2 * j] = v.x;
                B[nb][2 * j + 1] = v.y;
            }
    };

    uint64_t tile = (uint64_t)xcd_block() * WAVES + (threadIdx.x >> 6);
    if (tile >= ntiles) return;
    const uint64_t last = ntiles - 1;
    double B[NB][2 * HX];
    uint64_t base[NB];
    load(tile, base, B);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    do {
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        double Bn[NB][2 * HX];
        uint64_t basen[NB];
        load(nxt, basen, Bn);
        __builtin_amdgcn_sched_barrier(0);

        doublex4 acc[NB][RB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[nb][rb][i] = 0.0;
        int aoff = lane;
        asm volatile("" : "+v"(aoff));
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const double a = As[(rb * S + s) * 64 + aoff];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[nb][s], acc[nb][rb], 0, 0, 0);
            }
        }
        // acc[nb][j / 2][2 (j % 2) + {0, 1}] is output amplitude j of the lane
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            ColFactor<double> f{0u, 0u, 1.0, 0.0};
            if (has_epi) f = col_factor<double>(epi, base[nb]);
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                double re = acc[nb][j / 2][2 * (j % 2)], im = acc[nb][j / 2][2 * (j % 2) + 1];
                if (has_epi) apply_factor(re, im, f, (uint32_t)(j | (q << (K - 2))), has_ph);
                psi[base[nb] | qoff | target_off<K - 2>(j, g)] = make_double2(re, im);
            }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            base[nb] = basen[nb];
#pragma unroll
            for (int j = 0; j < 2 * HX; ++j) B[nb][j] = Bn[nb][j];
        }
        tile += stride;
    } while (tile < ntiles);
}

// ------------------------------------------------------------ cluster: MFMA, LDS-staged
// The same MFMA products, but the wave tile (targets x 2^C columns) is moved
// between HBM and registers as linear runs of its tile index tau: lane l reads
// and writes 16 consecutive bytes, so each load / store instruction covers
// runs of at least 2^C amplitudes whatever the target bits are (targets on
// the lowest bits scatter a direct register gather across many cache lines).
// The re-ordering into the MFMA operand layout goes through a private LDS
// buffer of the wave; the next tile's linear loads are in flight while the
// current tile's MFMA chain runs.



// LDS exchange between lanes of one wave: LDS operations of a wave execute in
// order, so only the compiler must be kept from reordering them.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// State offset of tile t: t deposited into the non-tile bit positions.
template <int NT>
__device__ __forceinline__ uint64_t tile_base(uint64_t t, const StageGeom& sg) {
#pragma unroll
    for (int i = 0; i < NT; ++i) t = insert_zero(t, sg.tb[i]);
    return t;
}

// tau of target index x (bits m0 <= m < m1 of x).
template <int M0, int M1>
__device__ __forceinline__ int tau_of_targets(int x, const StageGeom& sg) {
    int t = 0;
#pragma unroll
    for (int m = M0; m < M1; ++m)
        if ((x >> m) & 1) t |= 1 << sg.tpos[m];
    return t;
}

template <int C>
__device__ __forceinline__ int tau_of_column(int c, const StageGeom& sg) {
    int t = 0;
#pragma unroll
    for (int b = 0; b < C; ++b)
        if ((c >> b) & 1) t |= 1 << sg.cpos[b];
    return t;
}

template <int C>
__device__ __forceinline__ uint64_t state_bits_of_column(int c, const StageGeom& sg) {
    uint64_t o = 0;
#pragma unroll
    for (int b = 0; b < C; ++b)
        if ((c >> b) & 1) o |= uint64_t(1) << sg.tb[sg.cpos[b]];
    return o;
}

// Linear loads and the LDS re-ordering of the float staged kernel.
template <int K, int C, bool LOWT>
struct StageF32 {
    static constexpr int HX = (1 << K) / 2;
    static constexpr int NB = (1 << C) / 32;
    static constexpr int NL = (1 << (K + C)) / 128;
    // t0: the tile's base (uniform in the wave); lane_off: the lane's bits
    __device__ __forceinline__ static void load_lin(const g_float2* __restrict__ psi, uint64_t t0,
                                                    uint64_t lane_off, const StageGeom& sg, vf4 (&R)[NL]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = *reinterpret_cast<const g_vf4*>(psi + ((t0 | sg.ioff[i]) | lane_off));
    }
    __device__ __forceinline__ static void stage_in(vf4* L4, int lane, const int (&tc)[NB], int th,
                                                    const StageGeom& sg, const vf4 (&R)[NL],
                                                    float (&B)[NB][2 * HX]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) L4[i * 64 + lane] = R[i];
        wave_lds_fence();
        if (!LOWT) {
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const vf4 v = L4[(tc[0] | th | tau_of_targets<0, K - 1>(j, sg)) >> 1];
                B[0][2 * j] = v.x; B[0][2 * j + 1] = v.y;
                B[1][2 * j] = v.z; B[1][2 * j + 1] = v.w;
            }
        } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < HX; j += 2) {
                    const vf4 v = L4[(tc[nb] | th | tau_of_targets<0, K - 1>(j, sg)) >> 1];
                    B[nb][2 * j] = v.x; B[nb][2 * j + 1] = v.y;
                    B[nb][2 * j + 2] = v.z; B[nb][2 * j + 3] = v.w;
                }
        }
        wave_lds_fence();
    }
};

// float: lane l covers tau = 2 (i * 64 + l) + {0, 1} in linear order. In MFMA
// order lane (p, h) owns target indices j | h << (K-1) of columns 2p, 2p+1
// (tau bit 0 is a column bit) or p, p+32 (tau bit 0 is target 0, LOWT).
//
// One wave applies the cluster whose matrix is in LDS (As) to tiles
// tile, tile + stride, ... < tile_end, staging through its LDS buffer L4.
template <int K, int C, bool LOWT>
__device__ __forceinline__ void staged_f32_tiles(g_float2* __restrict__ psi, const float* As, vf4* L4,
                                                 c_epi* __restrict__ epi, const StageGeom& sg,
                                                 uint64_t tile, uint64_t tile_end, uint64_t stride) {
    constexpr int D = 1 << K;
    constexpr int HX = D / 2;
    constexpr int RB = 2 * D / 32;
    constexpr int S = D;
    constexpr int NB = (1 << C) / 32;
    constexpr int NT = K + C;
    constexpr int TILE = 1 << NT;
    constexpr int NL = TILE / 128;
    static_assert(NB == 2, "two column blocks per lane");
    // an opaque lane: what is derived from it is computed per call, not hoisted
    // into a caller's loop (the batch kernel's item loop) and kept live there
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int p = lane & 31, h = lane >> 5;
    uint64_t lane_off = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b + 1];
    int tc[NB];
    uint64_t cbits[NB];
    if (!LOWT) {
        tc[0] = tau_of_column<C>(2 * p, sg);
        tc[1] = tc[0] | 1;
        cbits[0] = state_bits_of_column<C>(2 * p, sg);
        cbits[1] = state_bits_of_column<C>(2 * p + 1, sg);
    } else {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            tc[nb] = tau_of_column<C>(p + 32 * nb, sg);
            cbits[nb] = state_bits_of_column<C>(p + 32 * nb, sg);
        }
    }
    const int th = h << sg.tpos[K - 1];
    const uint64_t ntiles = tile_end;
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;

    if (tile >= ntiles) return;
    const uint64_t last = ntiles - 1;
    vf4 R[NL];
    StageF32<K, C, LOWT>::load_lin(psi, tile_base<NT>(tile, sg), lane_off, sg, R);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    float B[NB][2 * HX];
    StageF32<K, C, LOWT>::stage_in(L4, lane, tc, th, sg, R, B);
    do {
        // the lane offset stays one value: the 16 chunk addresses built from it
        // are recomputed (an OR each) instead of held across the loop
        asm volatile("" : "+v"(lane_off));
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        StageF32<K, C, LOWT>::load_lin(psi, tile_base<NT>(nxt, sg), lane_off, sg, R);
        __builtin_amdgcn_sched_barrier(0);

        floatx16 acc[NB][RB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[nb][rb][i] = 0.0f;
        int aoff = lane;
        asm volatile("" : "+v"(aoff));
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float a = As[(rb * S + s) * 64 + aoff];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb][rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, B[nb][s], acc[nb][rb], 0, 0, 0);
            }
        }
        float O[NB][2 * HX];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < 2 * HX; ++j) O[nb][j] = acc[nb][j / 16][j % 16];
        const uint64_t tb0 = tile_base<NT>(tile, sg);
        if (has_epi) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const ColFactor<float> f = col_factor<float>(epi, tb0 | cbits[nb]);
#pragma unroll
                for (int j = 0; j < HX; ++j)
                    apply_factor(O[nb][2 * j], O[nb][2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
            }
        }
        // MFMA order -> LDS -> linear order -> HBM
        if (!LOWT) {
#pragma unroll
            for (int j = 0; j < HX; ++j)
                L4[(tc[0] | th | tau_of_targets<0, K - 1>(j, sg)) >> 1] =
                    vf4{O[0][2 * j], O[0][2 * j + 1], O[1][2 * j], O[1][2 * j + 1]};
        } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < HX; j += 2)
                    L4[(tc[nb] | th | tau_of_targets<0, K - 1>(j, sg)) >> 1] =
                        vf4{O[nb][2 * j], O[nb][2 * j + 1], O[nb][2 * j + 2], O[nb][2 * j + 3]};
        }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const vf4 v = L4[i * 64 + lane];
            *reinterpret_cast<g_vf4*>(psi + ((tb0 | sg.ioff[i]) | lane_off)) = v;
        }
        wave_lds_fence();
        StageF32<K, C, LOWT>::stage_in(L4, lane, tc, th, sg, R, B);
        tile += stride;
    } while (tile < ntiles);
}



template <int K, int C, bool LOWT>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_stage(float2* __restrict__ psi,
                                                              const float* __restrict__ Ap,
                                                              const EpiDesc* __restrict__ epi, ClusterGeom g,
                                                              StageGeom sg) {
    constexpr int D = 1 << K;
    constexpr int RB = 2 * D / 32;
    constexpr int S = D;
    constexpr int TILE = 1 << (K + C);
    __shared__ float As[RB * S * 64];
    __shared__ vf4 Ls[4][TILE / 2];
    load_matrix<RB * S * 64, 256>(As, reinterpret_cast<const vf4*>(Ap));
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: tile bases are scalar
    staged_f32_tiles<K, C, LOWT>((g_float2*)psi, As, Ls[w], (c_epi*)epi, sg, (uint64_t)xcd_block() * 4 + w,
                                 g.ncols >> C, (uint64_t)gridDim.x * 4);
}

// double: lane l covers tau = i * 64 + l in linear order; in MFMA order lane
// (p, q) owns target indices j | q << (K-2) of columns p and p + 16. One wave
// tile per wave, work-groups in memory order. The 32 KiB matrix of k = 5 takes
// the place of the four tiles in LDS once they are in registers (as in
// k_cluster_f32_split6s); its tiles have 16 columns (C = 4), so four
// work-groups share a compute unit and the fp64 products (two thirds of the
// pass) run under the others' accesses. k = 5, 28 qubits, 23 target sets: 1.60
// ms against 1.68 ms as a persistent grid of 8-wave work-groups and 1.78 ms for
// the direct kernel; 24 qubits 98 us against 143 us. k = 3 / 4: 1.52 / 1.60
// against 1.68 / 1.70 ms.
template <int K, int C, bool NT>
__global__ __launch_bounds__(256, C == 4 ? 4 : 2) void k_cluster_f64_stage(vd2* __restrict__ psi, const double* __restrict__ Ap,
                                                              const EpiDesc* __restrict__ epi, ClusterGeom g,
                                                              StageGeom sg) {
    constexpr int D = 1 << K, HX = D / 4, RB = 2 * D / 16, S = 2 * D / 4, NB = (1 << C) / 16, TB = K + C,
                  TILE = 1 << TB, NL = TILE / 64, AN = RB * S * 64;
    constexpr bool SHARE = K == 5;
    __shared__ vd2 Ls[4 * TILE + (SHARE ? 0 : AN / 2)];
    static_assert(!SHARE || AN / 2 <= 4 * TILE, "the matrix fits the tiles' place");
    double* As = reinterpret_cast<double*>(SHARE ? Ls : Ls + 4 * TILE);
    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4,
              w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: the tile base is scalar
    vd2* L = Ls + w * TILE;
    uint64_t lane_off = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b];
    const uint64_t tile = (uint64_t)tile_block<4 * (1 << TB) * 16>() * 4 + w;
    const bool act = tile < (g.ncols >> C);
    const uint64_t tb0 = tile_base<TB>(tile, sg);
    vd2 R[NL];
    if (act) {
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = load16<NT>(psi + ((tb0 | sg.ioff[i]) | lane_off));
    }
    MatrixRegs<AN * 8, 256> mr(Ap);
    int tc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) tc[nb] = tau_of_column<C>(p + 16 * nb, sg);
    const int tq = ((q & 1) << sg.tpos[K - 2]) | ((q >> 1) << sg.tpos[K - 1]);
    double B[NB][2 * HX];
    if (act) {
#pragma unroll
        for (int i = 0; i < NL; ++i) L[i * 64 + lane] = R[i];
        wave_lds_fence();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const vd2 v = L[tc[nb] | tq | tau_of_targets<0, K - 2>(j, sg)];
                B[nb][2 * j] = v.x;
                B[nb][2 * j + 1] = v.y;
            }
    }
    if constexpr (SHARE) __syncthreads();
    mr.store(As);
    __syncthreads();
    doublex4 acc[NB][RB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[nb][rb][i] = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const double a = As[(rb * S + s) * 64 + lane];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[nb][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[nb][s], acc[nb][rb], 0, 0, 0);
        }
    }
    if constexpr (SHARE) __syncthreads();  // every wave is done with the matrix
    if (!act) return;
    const bool has_epi = epi != nullptr, has_ph = has_epi && epi->n_ph > 0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        ColFactor<double> f{0u, 0u, 1.0, 0.0};
        if (has_epi) f = col_factor<double>((c_epi*)epi, tb0 | state_bits_of_column<C>(p + 16 * nb, sg));
#pragma unroll
        for (int j = 0; j < HX; ++j) {
            double re = acc[nb][j / 2][2 * (j % 2)], im = acc[nb][j / 2][2 * (j % 2) + 1];
            if (has_epi) apply_factor(re, im, f, (uint32_t)(j | (q << (K - 2))), has_ph);
            L[tc[nb] | tq | tau_of_targets<0, K - 2>(j, sg)] = vd2{re, im};
        }
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < NL; ++i) store16<NT>(psi + ((tb0 | sg.ioff[i]) | lane_off), (vd2)L[i * 64 + lane]);
}

// ------------------------------------------------------------ several 5-qubit clusters per pass
// Any two 5-qubit clusters touch at most 10 qubits, so both fit in one tile of
// 2^11 amplitudes (their qubits plus the lowest other ones): the tile is read
// from HBM once, each cluster is applied to it in LDS, and it is written back
// once - one pass for M clusters (the GPU form of applying several gates while
// a block sits in fast memory, Fig. 2). Each cluster's product runs on the fp16
// matrix cores with operand halves (as for k = 6), which keeps M = 2 within the
// matrix-core time of one pass. The tile is kept in LDS in tile order tau; for
// cluster m the lanes read their two columns (the tile bits that are not m's
// targets) in MFMA order, and write the results back to the same places.
// sg[m]: the common tile bits (tb, ioff) and cluster m's target / column
// positions (tpos, cpos); tile bit 0 is either a column bit of m (lane (p, h)
// owns columns 2p, 2p + 1) or m's target 0 (columns p, p + 32).
struct MultiArgs {
    StageGeom sg[2];
    const half8* A[2];        // fp16-halves matrices (LAYOUT_SPLIT16F, k = 5)
    const EpiDesc* epi[2];
    int32_t lowt[2];
};

// LDS slot of amplitude v (tile order) in the multi-cluster kernel. With SWZ
// the higher index bits are folded into bits 1..3 by XOR, so lanes whose
// amplitudes differ only in high bits - a cluster's columns can sit on any
// tile bits - use different banks. The map is linear over XOR, hence
// slot(a | b) = slot(a) ^ slot(b) for disjoint a, b: column and target parts
// of an address are mapped once, outside the tile loop.
template <bool SWZ>
__device__ __forceinline__ int lds_slot(int v) {
    return SWZ ? v ^ ((((v >> 4) ^ (v >> 7) ^ (v >> 10)) & 7) << 1) : v;
}

template <int M, int WAVES, bool SWZ>
__global__ __launch_bounds__(WAVES * 64, 8 / WAVES) void k_cluster_f32_multi(float2* __restrict__ psi, MultiArgs a,
                                                                           uint64_t ntiles) {
    constexpr int K = 5, C = 6, HX = 16, RB = 2, S = 4, NL = 16;
    __shared__ half8 As[M][2][RB * S * 64];  // [cluster][hi, lo]
    __shared__ float2 Ls[WAVES][1 << (K + C)];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(As[m][0]),
                                                reinterpret_cast<const vf4*>(a.A[m]));
        load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(As[m][1]),
                                                reinterpret_cast<const vf4*>(a.A[m] + RB * S * 64));
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    float2* L = Ls[w];
    g_float2* gpsi = (g_float2*)psi;
    const StageGeom& sg0 = a.sg[0];
    uint64_t lane_off = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg0.tb[b + 1];
    // Uniform state kept small (scalar registers are scarce here, and a
    // scalar reload waits on the LDS counter too): the tile chunks' state
    // offsets and each cluster's target offsets are linear in the index bits,
    // so four masks each stand for the sixteen values.
    uint64_t imask[4];  // state bit of tile bit 7 + b
#pragma unroll
    for (int b = 0; b < 4; ++b) imask[b] = uint64_t(1) << sg0.tb[7 + b];
    int tmask[M][4];    // mapped LDS offset of target b (b < 4) of cluster m
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int b = 0; b < 4; ++b) tmask[m][b] = lds_slot<SWZ>(1 << a.sg[m].tpos[b]);
    auto chunk_off = [&](int i) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((i >> b) & 1) o |= imask[b];
        return o;
    };
    auto load_tile = [&](uint64_t b0, vf4 (&R)[NL]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = *reinterpret_cast<const g_vf4*>(gpsi + (b0 | chunk_off(i)));
    };

    uint64_t tile = (uint64_t)xcd_block() * WAVES + w;
    if (tile >= ntiles) return;
    const uint64_t stride = (uint64_t)gridDim.x * WAVES;
    const uint64_t last = ntiles - 1;
    vf4 R[NL];
    load_tile(tile_base<K + C>(tile, sg0) | lane_off, R);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    do {
        // the tile to LDS (tile order: lane l holds amplitudes 2 (i 64 + l) + {0, 1}),
        // then prefetch the next one
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int v = lds_slot<SWZ>(2 * (i * 64 + lane));  // bit 0 is 0 and not swizzled
            L[v] = make_float2(R[i].x, R[i].y);
            L[v | 1] = make_float2(R[i].z, R[i].w);
        }
        wave_lds_fence();
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        load_tile(tile_base<K + C>(nxt, sg0) | lane_off, R);
        __builtin_amdgcn_sched_barrier(0);
        const uint64_t tb0 = tile_base<K + C>(tile, sg0);

#pragma unroll
        for (int m = 0; m < M; ++m) {
            const StageGeom& sg = a.sg[m];
            c_epi* epi = (c_epi*)a.epi[m];
            const bool has_ph = epi != nullptr && epi->n_ph > 0;
            // the lane's two columns one after the other: amplitudes j | h << 4
#pragma unroll 1
            for (int nb = 0; nb < 2; ++nb) {
                const int col = a.lowt[m] ? p + 32 * nb : 2 * p + nb;
                const int coff = lds_slot<SWZ>(tau_of_column<C>(col, sg) | (h << sg.tpos[K - 1]));
                float X[2 * HX];
                auto toff = [&](int j) {
                    int o = 0;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if ((j >> b) & 1) o ^= tmask[m][b];
                    return o;
                };
#pragma unroll
                for (int j = 0; j < HX; ++j) {
                    const float2 v = L[coff ^ toff(j)];
                    X[2 * j] = v.x;
                    X[2 * j + 1] = v.y;
                }
                // fp16 halves, the column scaled by a power of two (shared by lanes p, p + 32)
                half8 xh[S], xl[S];
                const float unscale = __builtin_ldexpf(1.0f, -split_halves<2 * HX>(X, xh, xl) - 4);
                floatx16 acc[RB];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
                int aoff = lane;
                asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
                for (int st = 0; st < S; ++st)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const half8 ah = As[m][0][(rb * S + st) * 64 + aoff];
                        const half8 al = As[m][1][(rb * S + st) * 64 + aoff];
                        acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
                        acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
                        acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
                    }
#pragma unroll
                for (int j = 0; j < 2 * HX; ++j) X[j] = acc[j / 16][j % 16] * unscale;
                if (epi != nullptr) {
                    const ColFactor<float> f = col_factor<float>(epi, tb0 | state_bits_of_column<C>(col, sg));
#pragma unroll
                    for (int j = 0; j < HX; ++j)
                        apply_factor(X[2 * j], X[2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
                }
                // every lane reads its column before any writes it (the lanes of a
                // column pair, p and p + 32, read disjoint amplitudes)
#pragma unroll
                for (int j = 0; j < HX; ++j) L[coff ^ toff(j)] = make_float2(X[2 * j], X[2 * j + 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            wave_lds_fence();
        }
        // tile order -> HBM
        {
            const uint64_t b0 = tb0 | lane_off;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int v = lds_slot<SWZ>(2 * (i * 64 + lane));
                const float2 u = L[v], x = L[v | 1];
                *reinterpret_cast<g_vf4*>(gpsi + (b0 | chunk_off(i))) = vf4{u.x, u.y, x.x, x.y};
            }
        }
        wave_lds_fence();
        tile += stride;
    } while (tile < ntiles);
}

// Two 5-qubit clusters per pass on a tile of 2^10 amplitudes: the 10 tile bits
// hold both clusters' targets; each cluster's columns are the other 5 tile
// bits, one per lane pair (lane (p, h): column p, amplitudes j | h << 4). The
// smaller tile (8 KiB per wave) and the smaller register set let 12 waves
// share a CU, which hides more of each wave's serial chain (LDS, split,
// matrix cores, epilogue) under the other waves.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void k_cluster_f32_pair10(float2* __restrict__ psi, MultiArgs a,
                                                                   uint64_t ntiles) {
    constexpr int K = 5, NT = 10, HX = 16, RB = 2, S = 4, NL = 8;
    __shared__ half8 As[2][2][RB * S * 64];  // [cluster][hi, lo]
    __shared__ float2 Ls[WAVES][1 << NT];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(As[m][0]),
                                                reinterpret_cast<const vf4*>(a.A[m]));
        load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(As[m][1]),
                                                reinterpret_cast<const vf4*>(a.A[m] + RB * S * 64));
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    float2* L = Ls[w];
    g_float2* gpsi = (g_float2*)psi;
    const StageGeom& sg0 = a.sg[0];
    uint64_t lane_off = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg0.tb[b + 1];
    uint64_t imask[3];  // state bit of tile bit 7 + b
#pragma unroll
    for (int b = 0; b < 3; ++b) imask[b] = uint64_t(1) << sg0.tb[7 + b];
    auto chunk_off = [&](int i) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < 3; ++b)
            if ((i >> b) & 1) o |= imask[b];
        return o;
    };
    // per cluster: mapped target offsets (linear in j) and the lane's column
    int tmask[2][4], coff[2];
    uint64_t cbits[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const StageGeom& sg = a.sg[m];
#pragma unroll
        for (int b = 0; b < 4; ++b) tmask[m][b] = lds_slot<true>(1 << sg.tpos[b]);
        coff[m] = lds_slot<true>(tau_of_column<5>(p, sg) | (h << sg.tpos[K - 1]));
        cbits[m] = state_bits_of_column<5>(p, sg);
    }

    uint64_t tile = (uint64_t)xcd_block() * WAVES + w;
    if (tile >= ntiles) return;
    const uint64_t stride = (uint64_t)gridDim.x * WAVES;
    const uint64_t last = ntiles - 1;
    vf4 R[NL];
    auto load_tile = [&](uint64_t b0) {
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = *reinterpret_cast<const g_vf4*>(gpsi + (b0 | chunk_off(i)));
    };
    load_tile(tile_base<NT>(tile, sg0) | lane_off);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);
    do {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int v = lds_slot<true>(2 * (i * 64 + lane));
            L[v] = make_float2(R[i].x, R[i].y);
            L[v | 1] = make_float2(R[i].z, R[i].w);
        }
        wave_lds_fence();
        const uint64_t nxt = tile + stride < last ? tile + stride : last;
        load_tile(tile_base<NT>(nxt, sg0) | lane_off);
        __builtin_amdgcn_sched_barrier(0);
        const uint64_t tb0 = tile_base<NT>(tile, sg0);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            auto toff = [&](int j) {
                int o = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if ((j >> b) & 1) o ^= tmask[m][b];
                return o;
            };
            float X[2 * HX];
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const float2 v = L[coff[m] ^ toff(j)];
                X[2 * j] = v.x;
                X[2 * j + 1] = v.y;
            }
            half8 xh[S], xl[S];
            const int se = split_halves<2 * HX>(X, xh, xl);
            floatx16 acc[RB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
            int aoff = lane;
            asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
            for (int st = 0; st < S; ++st)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const half8 ah = As[m][0][(rb * S + st) * 64 + aoff];
                    const half8 al = As[m][1][(rb * S + st) * 64 + aoff];
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
                }
            // undo the scaling, with the column's diagonal phase folded in
            float ur = __builtin_ldexpf(1.0f, -se - 4), ui = 0.0f;
            uint32_t sgn = 0, wm = 0;
            c_epi* epi = (c_epi*)a.epi[m];
            if (epi != nullptr) {
                const ColFactor<float> f = col_factor<float>(epi, tb0 | cbits[m]);
                sgn = f.sgn;
                wm = f.w;
                ui = ur * f.ci;
                ur = ur * f.cr;
            }
#pragma unroll
            for (int j = 0; j < HX; ++j) {
                const float re = acc[j / 8][2 * (j % 8)], im = acc[j / 8][2 * (j % 8) + 1];
                float orr = re * ur - im * ui, oi = re * ui + im * ur;
                const bool neg = ((sgn ^ (uint32_t)__popc((uint32_t)(j | (h << (K - 1))) & wm)) & 1u) != 0;
                orr = neg ? -orr : orr;
                oi = neg ? -oi : oi;
                L[coff[m] ^ toff(j)] = make_float2(orr, oi);
            }
            wave_lds_fence();
        }
        {
            const uint64_t b0 = tb0 | lane_off;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int v = lds_slot<true>(2 * (i * 64 + lane));
                const float2 u = L[v], x = L[v | 1];
                *reinterpret_cast<g_vf4*>(gpsi + (b0 | chunk_off(i))) = vf4{u.x, u.y, x.x, x.y};
            }
        }
        wave_lds_fence();
        tile += stride;
    } while (tile < ntiles);
}

// ------------------------------------------------------------ cluster: float state, k = 6, LDS-staged
// The direct kernel above reads lane p's column with one load per amplitude;
// when several targets sit on the lowest state bits the 32 columns of a load
// are spread over up to 64 cache lines (8 - 16 bytes used of each), and the
// vector L1 becomes the bottleneck. This variant reads a tile of 2^11
// amplitudes (the 6 targets and the 5 lowest other bits) with linear 16-byte
// loads - 1 KiB runs - and re-orders it through LDS. Per wave the LDS holds
// half a tile (8 KiB): tile bit 10 is either target 5 (h) or column bit 4,
// so each lane's whole column lies in one half and the halves are staged one
// after the other. Eight waves and the matrix halves (64 KiB) fill 128 KiB.
// Core (fp16 halves on matrix cores, column scaling, epilogue) as above.
// Addresses: slot(tau) = swizzle(tau) & 1023 (StageGeom::swz, chosen per
// geometry so that the columns of a read pass fall on distinct banks), linear
// over XOR, so the lane's column part and the row part are mapped separately.
//
// One wave applies the cluster whose fp16 matrix halves are in LDS (Ah, Al)
// to tiles tile, tile + stride, ... < tile_end (tile numbers uniform in the
// wave), staging through its 8 KiB LDS buffer L.
//
// FOLD: the input is not loaded but computed - the state after the uniform
// start, a first cluster and its diagonal epilogue (see k_fold2_f32).
struct FoldIn {
    const float2* W;  // LDS: w over the first cluster's qubits (bit m of the index: its qubit m)
    int ymask[6];     // per row bit (this cluster's target m): the w-index bit it sets, 0 if none
    int t1[6];        // the first cluster's qubits
    int k1;
    c_epi* epi1;      // the first epilogue relative to this cluster's targets, or null
    // table form (FOLD 2): the second cluster's outputs split by the row bits
    // it shares with the first cluster (sigma: their pattern) and by the
    // first epilogue's row signs w. Row sigma + Wc[w] of Y (kFoldRow float2
    // each, in LDS) holds M2 applied to the sign vector of w restricted to
    // the rows of pattern sigma; a column's outputs are the sum over sigma of
    // W[ic | iys[sigma]] times that row.
    const float2* Y;
    const int* Wc;  // per row-sign mask w: its compressed index << (shared bits)
    int no;         // patterns sigma: 2^(shared row bits), at most 4
    int iys[4];     // w index of each pattern's shared rows
};
// LDS row of one table pattern: 64 outputs and a 16-byte pad, so that the
// rows of different patterns start on different banks
constexpr int kFoldRow = 66;

// FOLD: 0 the tile is loaded; 1 the column's inputs are computed from the
// first cluster's closed form and multiplied on the matrix cores; 2 the
// column's outputs are combined from the table of FoldIn::Y.
template <bool LOWT, int FOLD = 0>
__device__ __forceinline__ void split6s_tiles(g_float2* __restrict__ gpsi, const half8* Ah, const half8* Al, float2* L,
                                              c_epi* __restrict__ epi, const StageGeom& sg, uint64_t tile,
                                              uint64_t tile_end, uint64_t stride, const FoldIn* fin = nullptr) {
    constexpr int K = 6, C = 5, TB = K + C, HX = 32, RB = 4, S = 8, NL = 16;
    // an opaque lane: what is derived from it is computed per call, not hoisted
    // into a caller's loop (the batch kernel's item loop) and kept live there
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int p = lane & 31, h = lane >> 5;
    vf4* L4 = reinterpret_cast<vf4*>(L);
    bool has_epi = epi != nullptr;
    bool has_ph = has_epi && epi->n_ph > 0;
    if constexpr (FOLD != 0) {
        has_epi = has_epi || fin->epi1 != nullptr;
        has_ph = has_ph || (fin->epi1 != nullptr && fin->epi1->n_ph > 0);
    }
    uint64_t lane_off = 0;  // state offset of tile bits 1..6 (the lane of a linear load)
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b + 1];
    // LDS slot of tau (the geometry's swizzle; linear over XOR)
    auto sslot = [&](int v) {
        int o = v;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            if ((v >> (5 + i)) & 1) o ^= sg.swz[i];
        return o;
    };
    // the lane's column (tile order, then LDS slot), its half of the targets
    const int ctau = tau_of_column<C>(p, sg) | (h << sg.tpos[K - 1]);
    int lslot = sslot(ctau);
    uint32_t h5 = (uint32_t)h << (K - 1);
    const uint64_t cbits = state_bits_of_column<C>(p, sg);
    const int lph = (ctau >> 10) & 1;  // the half of the tile holding the column
    int lin = sslot(2 * lane);  // slot of linear chunk 0; chunk i adds slot(128 i) by XOR
    // row j's slot and linear chunk i's state offset, rebuilt from 5 and 4
    // uniform masks at each use (cheap scalar work) rather than 32 + 16 values
    // held across the loop
    int rmask[K - 1];
#pragma unroll
    for (int m = 0; m < K - 1; ++m) rmask[m] = sslot(1 << sg.tpos[m]);
    int cmask[4];  // slots of the linear chunks' bits (tau bits 7..10)
#pragma unroll
    for (int b = 0; b < 4; ++b) cmask[b] = sslot(128 << b);
    uint64_t imask[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) imask[b] = uint64_t(1) << sg.tb[7 + b];
    auto rslot = [&](int j) {
        int o = 0;
#pragma unroll
        for (int m = 0; m < K - 1; ++m)
            if ((j >> m) & 1) o ^= rmask[m];
        return o;
    };
    auto ioff = [&](int i) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((i >> b) & 1) o |= imask[b];
        return o;
    };
    auto cslot = [&](int i) {  // slot offset of linear chunk i (tau = 128 i)
        int o = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((i >> b) & 1) o ^= cmask[b];
        return o;
    };

    if (tile >= tile_end) return;
    const uint64_t last = tile_end - 1;
    // FOLD: the epilogue factors of both clusters and the w index, split into
    // column parts (here, once) and tile parts (lane j forms those of the
    // wave's tile it + j once per 64 tiles; each tile reads them from its lane)
    uint64_t colmask = 0;
    uint32_t l1s = 0, l1w = 0, l2s = 0, l2w = 0, t1b = 0, t2b = 0;
    double l1r = 1.0, l1i = 0.0, l2r = 1.0, l2i = 0.0, t1r = 1.0, t1i = 0.0, t2r = 1.0, t2i = 0.0;
    int icl = 0, it = 0;
    if constexpr (FOLD != 0) {
#pragma unroll
        for (int b = 0; b < C; ++b) colmask |= uint64_t(1) << sg.tb[sg.cpos[b]];
        if (fin->epi1 != nullptr) epi_lane_part(fin->epi1, cbits, colmask, l1s, l1w, l1r, l1i);
        if (epi != nullptr) epi_lane_part(epi, cbits, colmask, l2s, l2w, l2r, l2i);
#pragma unroll
        for (int m = 0; m < 6; ++m)
            if (m < fin->k1) icl |= (int)((cbits >> fin->t1[m]) & 1) << m;
    }
    vf4 R[NL];
    auto load_tile = [&](uint64_t t0) {  // t0: the tile's base (uniform)
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = *reinterpret_cast<const g_vf4*>(gpsi + ((t0 | ioff(i)) | lane_off));
    };
    if constexpr (FOLD == 0) {
        load_tile(tile_base<TB>(tile, sg));
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_sched_barrier(0);
    }
    do {
        // per-lane bases stay in place: the 16 chunk addresses derived from them
        // are recomputed (one OR / XOR each) instead of held across the loop
        asm volatile("" : "+v"(lane_off), "+v"(lin), "+v"(lslot), "+v"(h5));
        asm volatile("" : "+s"(rmask[0]), "+s"(rmask[1]), "+s"(rmask[2]), "+s"(rmask[3]), "+s"(rmask[4]));
        asm volatile("" : "+s"(imask[0]), "+s"(imask[1]), "+s"(imask[2]), "+s"(imask[3]));
        asm volatile("" : "+s"(cmask[0]), "+s"(cmask[1]), "+s"(cmask[2]), "+s"(cmask[3]));
        float X[2 * HX];
        ColFactor<float> f1{0u, 0u, 1.0f, 0.0f}, f2{0u, 0u, 1.0f, 0.0f};
        if constexpr (FOLD != 0) {
            // the column's inputs from the closed form: w at the first cluster's
            // index (its qubits among the column bits, then among the row bits),
            // negated where a gate of the first epilogue couples a row bit with
            // a column bit; the column-only factor of that epilogue joins the
            // output factor
            if ((it & 63) == 0) {
                const uint64_t bj = tile_base<TB>(tile + (uint64_t)lane * stride, sg);  // past the end: unused
                t1b = 0;
                t2b = 0;
                if (fin->epi1 != nullptr) t1b = epi_tile_part(fin->epi1, bj, colmask, t1r, t1i);
                if (epi != nullptr) t2b = epi_tile_part(epi, bj, colmask, t2r, t2i);
                int ict = 0;
#pragma unroll
                for (int m = 0; m < 6; ++m)
                    if (m < fin->k1) ict |= (int)((bj >> fin->t1[m]) & 1) << m;
                t1b |= (uint32_t)ict << 12;
            }
            const int sl = it & 63;
            const uint32_t b1 = (uint32_t)__builtin_amdgcn_readlane((int)t1b, sl);
            const int ic = icl | (int)((b1 >> 12) & 63u);
            if (fin->epi1 != nullptr)
                f1 = epi_combine(b1, readlane_f64(t1r, sl), readlane_f64(t1i, sl), l1s, l1w, l1r, l1i, p);
            if (epi != nullptr)
                f2 = epi_combine((uint32_t)__builtin_amdgcn_readlane((int)t2b, sl), readlane_f64(t2r, sl),
                                 readlane_f64(t2i, sl), l2s, l2w, l2r, l2i, p);
            ++it;
            if constexpr (FOLD == 1) {
                const int yh = h ? fin->ymask[K - 1] : 0;
#pragma unroll
                for (int j = 0; j < HX; ++j) {
                    int iy = yh;
#pragma unroll
                    for (int b = 0; b < K - 1; ++b)
                        if ((j >> b) & 1) iy |= fin->ymask[b];
                    const float2 v = fin->W[ic | iy];
                    const bool neg = (__popc(((uint32_t)j | h5) & f1.w) & 1u) != 0;
                    X[2 * j] = neg ? -v.x : v.x;
                    X[2 * j + 1] = neg ? -v.y : v.y;
                }
            } else {
                // its half of the outputs (rows j | h << 5): the table rows of
                // its row-sign mask, weighted by w at its shared-row patterns
                const int pb = fin->Wc[f1.w & 63u];
#pragma unroll
                for (int j = 0; j < 2 * HX; ++j) X[j] = 0.0f;
#pragma unroll
                for (int sp = 0; sp < 4; ++sp) {
                    if (sp < fin->no) {
                        const float2 a = fin->W[ic | fin->iys[sp]];
                        const vf4* row = reinterpret_cast<const vf4*>(fin->Y + (pb + sp) * kFoldRow + h * HX);
#pragma unroll
                        for (int q = 0; q < HX / 2; ++q) {
                            const vf4 v = row[q];
                            X[4 * q] = fmaf(a.x, v.x, fmaf(-a.y, v.y, X[4 * q]));
                            X[4 * q + 1] = fmaf(a.x, v.y, fmaf(a.y, v.x, X[4 * q + 1]));
                            X[4 * q + 2] = fmaf(a.x, v.z, fmaf(-a.y, v.w, X[4 * q + 2]));
                            X[4 * q + 3] = fmaf(a.x, v.w, fmaf(a.y, v.z, X[4 * q + 3]));
                        }
                    }
                }
            }
        } else {
        // tile -> LDS, half by half; each lane reads its column in its half
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
#pragma unroll
            for (int ii = 0; ii < NL / 2; ++ii) {
                const int i = ph * (NL / 2) + ii;
                L4[((lin ^ cslot(i)) & 1023) >> 1] = R[i];
            }
            wave_lds_fence();
            if (lph == ph) {
                if (LOWT) {
#pragma unroll
                    for (int j = 0; j < HX; j += 2) {
                        const vf4 v = L4[((lslot ^ rslot(j)) & 1023) >> 1];
                        X[2 * j] = v.x; X[2 * j + 1] = v.y; X[2 * j + 2] = v.z; X[2 * j + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < HX; ++j) {
                        const float2 v = L[(lslot ^ rslot(j)) & 1023];
                        X[2 * j] = v.x; X[2 * j + 1] = v.y;
                    }
                }
            }
            wave_lds_fence();
        }
        }
        if constexpr (FOLD != 2) {
            // fp16 halves of the scaled column (shared scale with lane p + 32)
            half8 xh[S], xl[S];
            const int se = split_halves<2 * HX>(X, xh, xl);
            // the column is in registers: prefetch the next tile (issued here, the
            // peak register use is the halves + accumulators + the tile in flight)
            if constexpr (FOLD == 0) {
                const uint64_t nxt = tile + stride < last ? tile + stride : last;
                __builtin_amdgcn_sched_barrier(0);
                load_tile(tile_base<TB>(nxt, sg));
                __builtin_amdgcn_sched_barrier(0);
            }
            floatx16 acc[RB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
            int aoff = lane;
            asm volatile("" : "+v"(aoff));  // keep the matrix reads inside the loop (not in registers)
#pragma unroll
            for (int st = 0; st < S; ++st)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const half8 ah = Ah[(rb * S + st) * 64 + aoff];
                    const half8 al = Al[(rb * S + st) * 64 + aoff];
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
                    acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
                }
            const float unscale = __builtin_ldexpf(1.0f, -se - 4);
#pragma unroll
            for (int j = 0; j < 2 * HX; ++j) X[j] = acc[j / 16][j % 16] * unscale;
        }
        const uint64_t tb0 = tile_base<TB>(tile, sg);
        if (has_epi) {
            ColFactor<float> f{0u, 0u, 1.0f, 0.0f};
            if constexpr (FOLD != 0) {
                f = f2;
            } else {
                if (epi != nullptr) f = col_factor<float>(epi, tb0 | cbits);
            }
            if constexpr (FOLD != 0) {  // the first epilogue's column-only sign and phase
                f.sgn ^= f1.sgn;
                const float r = f.cr * f1.cr - f.ci * f1.ci;
                f.ci = f.cr * f1.ci + f.ci * f1.cr;
                f.cr = r;
            }
#pragma unroll
            for (int j = 0; j < HX; ++j)
                apply_factor(X[2 * j], X[2 * j + 1], f, (uint32_t)j | h5, has_ph);
        }
        // results -> LDS -> HBM, half by half
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
            if (lph == ph) {
                if (LOWT) {
#pragma unroll
                    for (int j = 0; j < HX; j += 2)
                        L4[((lslot ^ rslot(j)) & 1023) >> 1] = vf4{X[2 * j], X[2 * j + 1], X[2 * j + 2], X[2 * j + 3]};
                } else {
#pragma unroll
                    for (int j = 0; j < HX; ++j) L[(lslot ^ rslot(j)) & 1023] = make_float2(X[2 * j], X[2 * j + 1]);
                }
            }
            wave_lds_fence();
#pragma unroll
            for (int ii = 0; ii < NL / 2; ++ii) {
                const int i = ph * (NL / 2) + ii;
                *reinterpret_cast<g_vf4*>(gpsi + ((tb0 | ioff(i)) | lane_off)) =
                    L4[((lin ^ cslot(i)) & 1023) >> 1];
            }
            wave_lds_fence();
        }
        tile += stride;
    } while (tile < tile_end);
}

// Staged 6-qubit kernel: one wave tile per wave, work-groups in memory order
// (see k_cluster_f32_split6). The work-group's 64 KiB of LDS hold its four
// tiles first (linear loads, each lane reads its column), then the matrix,
// then the results on their way to linear stores: two work-groups per compute
// unit, so one's loads and stores run under the other's product. Its tile is
// read in whole lines whatever the targets are: 30 qubits, 23 target sets, mean
// 3.08 ms (worst 3.7) against 3.52 ms as a persistent grid that held the matrix
// and half tiles side by side.
template <bool LOWT, bool NT>
__global__ __launch_bounds__(256, 2) void k_cluster_f32_split6s(float2* __restrict__ psi,
                                                                const half8* __restrict__ Ap,
                                                                const EpiDesc* __restrict__ epi, StageGeom sg,
                                                                uint64_t ntiles) {
    constexpr int K = 6, C = 5, TB = K + C, HX = 32, RB = 4, S = 8, NL = 16, NP = RB * S * 64;
    __shared__ half8 L[2 * NP];
    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t tile = (uint64_t)tile_block<4 * 2048 * 8>() * 4 + w;
    const bool act = tile < ntiles;
    vf4* T4 = reinterpret_cast<vf4*>(L) + w * 1024;  // this wave's tile
    constexpr bool PAIR = !LOWT;
    const int cpair = PAIR ? 2 * (p & 15) : p, cown = PAIR ? (p >> 4) & 1 : 0;
    auto sslot = [&](int v) {  // LDS slot of tau (the geometry's swizzle; linear over XOR)
        int o = v;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            if ((v >> (5 + i)) & 1) o ^= sg.swz[i];
        return o;
    };
    const int lin = sslot(2 * lane);
    const int lslot = sslot(tau_of_column<C>(cpair, sg) | (h << sg.tpos[K - 1]) | (cown << sg.tpos[0]));
    int cmask[4], rmask[K - 1];
    uint64_t imask[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        cmask[b] = sslot(128 << b);
        imask[b] = uint64_t(1) << sg.tb[7 + b];
    }
#pragma unroll
    for (int m = 0; m < K - 1; ++m) rmask[m] = sslot(1 << sg.tpos[m]);
    auto sel = [](int i, auto& m, auto o, int nb) {
#pragma unroll
        for (int b = 0; b < 5; ++b)
            if (b < nb && ((i >> b) & 1)) o ^= m[b];
        return o;
    };
    uint64_t lane_off = 0;  // state offset of tile bits 1..6 (the lane of a linear access)
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b + 1];
    const uint64_t tb0 = tile_base<TB>(tile, sg);
    vf4* mem = reinterpret_cast<vf4*>(psi + (tb0 | lane_off));
    vf4 R[NL];
    if (act) {
#pragma unroll
        for (int i = 0; i < NL; ++i) R[i] = load16<NT>(mem + (sel(i, imask, uint64_t(0), 4) >> 1));
    }
    MatrixRegs<2 * NP * 16, 256> mr(Ap);
    float X[2 * HX];
    if (act) {
#pragma unroll
        for (int i = 0; i < NL; ++i) T4[sel(i, cmask, lin, 4) >> 1] = R[i];
        wave_lds_fence();
#pragma unroll
        for (int j = 0; j < HX; j += 2) {
            const vf4 v = T4[sel(PAIR ? j & ~1 : j, rmask, lslot, 5) >> 1];
            X[2 * j] = v.x; X[2 * j + 1] = v.y; X[2 * j + 2] = v.z; X[2 * j + 3] = v.w;
        }
    }
    __syncthreads();
    mr.store(L);
    if constexpr (PAIR) {  // rows j, j + 1 of the lane's own column
#pragma unroll
        for (int j = 0; j < HX; j += 2) {
            lane_swap16(X[2 * j], X[2 * j + 2]);
            lane_swap16(X[2 * j + 1], X[2 * j + 3]);
        }
    }
    half8 xh[S], xl[S];
    const float unscale = __builtin_ldexpf(1.0f, -split_halves<2 * HX>(X, xh, xl) - 4);
    __syncthreads();
    floatx16 acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][i] = 0.0f;
#pragma unroll
    for (int st = 0; st < S; ++st) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const half8 ah = L[(rb * S + st) * 64 + lane];
            const half8 al = L[NP + (rb * S + st) * 64 + lane];
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xl[st], acc[rb], 0, 0, 0);
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, xh[st], acc[rb], 0, 0, 0);
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, xh[st], acc[rb], 0, 0, 0);
        }
    }
    __syncthreads();  // every wave is done with the matrix
    if (!act) return;
#pragma unroll
    for (int j = 0; j < 2 * HX; ++j) X[j] = acc[j / 16][j % 16] * unscale;
    if (epi != nullptr) {
        const ColFactor<float> f = col_factor<float>((c_epi*)epi, tb0 | state_bits_of_column<C>(cpair | cown, sg));
        const bool has_ph = epi->n_ph > 0;
#pragma unroll
        for (int j = 0; j < HX; ++j)
            apply_factor(X[2 * j], X[2 * j + 1], f, (uint32_t)(j | (h << (K - 1))), has_ph);
    }
#pragma unroll
    for (int j = 0; j < HX; j += 2) {
        if constexpr (PAIR) {
            lane_swap16(X[2 * j], X[2 * j + 2]);
            lane_swap16(X[2 * j + 1], X[2 * j + 3]);
        }
        T4[sel(j, rmask, lslot, 5) >> 1] = vf4{X[2 * j], X[2 * j + 1], X[2 * j + 2], X[2 * j + 3]};
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < NL; ++i)
        store16<NT>(mem + (sel(i, imask, uint64_t(0), 4) >> 1), (vf4)T4[sel(i, cmask, lin, 4) >> 1]);
}

// ------------------------------------------------------------ uniform start + two clusters, one write-only pass
// From the uniform start, after a first cluster (qubits T1, matrix M1) and its
// diagonal epilogue E1 the state is a closed form: psi(x) = w[x on T1] E1(x),
// w = 2^(-n/2) times the row sums of M1. Relative to the second cluster's
// targets T2, E1 splits into terms on T2 alone (folded into the second matrix,
// before its gates, when it is built), terms coupling one T2 qubit with one
// column bit (a sign mask over the row index, per column) and terms on column
// bits alone (a sign and a phase per column, which commute with the product
// and join the second epilogue). The second cluster is then applied to inputs
// computed from w instead of loaded: one write-only pass stands for the
// initialisation and two cluster passes. The second cluster has 6 qubits; its
// core and write-back are those of the staged 6-qubit kernel.
struct Fold2Args {
    const double2* M1;  // first cluster: plain complex128 2^k1 x 2^k1, row-major
    double amp;         // 2^(-n/2)
    int32_t k1;
    int32_t t1[7];      // its qubits (sorted)
};

template <bool LOWT>
__global__ __launch_bounds__(512, 1) void k_fold2_f32(float2* __restrict__ psi, const half8* __restrict__ Ap,
                                                      const EpiDesc* __restrict__ epi2, const EpiDesc* __restrict__ epi1,
                                                      StageGeom sg, Fold2Args f, uint64_t ntiles) {
    constexpr int RB = 4, S = 8, WAVES = 8;
    __shared__ half8 Ah[RB * S * 64];
    __shared__ half8 Al[RB * S * 64];
    __shared__ float2 Ls[WAVES][1024];
    __shared__ float2 W[64];
    load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(Ah), reinterpret_cast<const vf4*>(Ap));
    load_matrix<RB * S * 64 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(Al),
                                            reinterpret_cast<const vf4*>(Ap + RB * S * 64));
    const int d1 = 1 << f.k1;
    if ((int)threadIdx.x < 64) W[threadIdx.x] = make_float2(0.0f, 0.0f);
    __syncthreads();
    row_sums(f.M1, d1, f.amp, W);  // w: the first cluster applied to the uniform vector
    __syncthreads();
    FoldIn fin;
    fin.W = W;
    fin.k1 = f.k1;
    fin.epi1 = (c_epi*)epi1;
#pragma unroll
    for (int m = 0; m < 6; ++m) fin.t1[m] = f.t1[m];
#pragma unroll
    for (int m2 = 0; m2 < 6; ++m2) {
        const int q = sg.tb[sg.tpos[m2]];
        int b = 0;
#pragma unroll
        for (int m1 = 0; m1 < 6; ++m1)
            if (m1 < f.k1 && f.t1[m1] == q) b = 1 << m1;
        fin.ymask[m2] = b;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    split6s_tiles<LOWT, 1>((g_float2*)psi, Ah, Al, Ls[w], (c_epi*)epi2, sg, (uint64_t)xcd_block() * WAVES + w,
                              ntiles, (uint64_t)gridDim.x * WAVES, &fin);
}

// Table form: the second cluster's inputs are x[r] = w[ic | iy(r)] s(r) -
// w at the first cluster's index (ic from the column bits, iy from the rows
// the two clusters share), s the first epilogue's row signs. Split by the
// pattern sigma of the shared rows, M2 x = sum over sigma of
// w[ic | iy(sigma)] M2 (s restricted to the rows of pattern sigma), and s is
// fixed by the mask of its sign-flipped rows. One work-group per (sigma,
// compressed mask) forms M2 times that signed indicator in float64; the pass
// below weights and sums its rows per column.
struct FoldTabArgs {
    const double2* M2;  // second cluster: plain complex128 2^k2 x 2^k2, row-major
    int32_t omask;      // rows (second cluster's target bits) shared with the first cluster
    int32_t rmask;      // rows the first epilogue's mixed terms sign-flip
};

// bits of v at the set bits of mask (B bits), packed low; and back
template <int B>
__device__ __forceinline__ int pext_bits(int v, int mask) {
    int o = 0, k = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
        if ((mask >> b) & 1) o |= ((v >> b) & 1) << k++;
    return o;
}
template <int B>
__device__ __forceinline__ int pdep_bits(int v, int mask) {
    int o = 0, k = 0;
#pragma unroll
    for (int b = 0; b < B; ++b)
        if ((mask >> b) & 1) o |= ((v >> k++) & 1) << b;
    return o;
}

// one work-group of 2^K2 threads (one per output row) per table row
template <int K2>
__global__ __launch_bounds__(1 << K2) void k_fold2_table(float2* __restrict__ Y, FoldTabArgs a) {
    constexpr int D2 = 1 << K2;
    __shared__ double x[D2];
    const int t = threadIdx.x;
    const int no = __popc(a.omask);
    const int P = blockIdx.x;
    const int sigma = P & ((1 << no) - 1);
    const int w = pdep_bits<K2>(P >> no, a.rmask);
    x[t] = pext_bits<K2>(t, a.omask) != sigma ? 0.0 : ((__popc(t & w) & 1) ? -1.0 : 1.0);
    __syncthreads();
    double re = 0.0, im = 0.0;
    for (int s = 0; s < D2; ++s) {
        const double2 m = a.M2[t * D2 + s];
        re = fma(m.x, x[s], re);
        im = fma(m.y, x[s], im);
    }
    Y[P * D2 + t] = make_float2((float)re, (float)im);
}

template <bool LOWT>
__global__ __launch_bounds__(512, 1) void k_fold2t_f32(float2* __restrict__ psi, const float2* __restrict__ Yg,
                                                       const EpiDesc* __restrict__ epi2,
                                                       const EpiDesc* __restrict__ epi1, StageGeom sg, Fold2Args f,
                                                       FoldTabArgs a, uint64_t ntiles) {
    constexpr int WAVES = 8;
    __shared__ float2 Y[kFoldTabRows * kFoldRow];
    __shared__ float2 Ls[WAVES][1024];
    __shared__ float2 W[64];
    __shared__ int Wc[64];
    const int no = __popc(a.omask);
    // the table into LDS, rows padded to kFoldRow
    const int nq = 32 << (no + __popc(a.rmask));  // 16-byte pieces
    for (int i = (int)threadIdx.x; i < nq; i += (int)blockDim.x)
        reinterpret_cast<vf4*>(Y + (i >> 5) * kFoldRow)[i & 31] = reinterpret_cast<const vf4*>(Yg)[i];
    if ((int)threadIdx.x < 64) {
        W[threadIdx.x] = make_float2(0.0f, 0.0f);
        Wc[threadIdx.x] = pext_bits<6>((int)threadIdx.x, a.rmask) << no;
    }
    __syncthreads();
    row_sums(f.M1, 1 << f.k1, f.amp, W);  // w: the first cluster applied to the uniform vector
    __syncthreads();
    FoldIn fin;
    fin.W = W;
    fin.k1 = f.k1;
    fin.epi1 = (c_epi*)epi1;
#pragma unroll
    for (int m = 0; m < 6; ++m) fin.t1[m] = f.t1[m];
    int ymask[6];
#pragma unroll
    for (int m2 = 0; m2 < 6; ++m2) {
        const int q = sg.tb[sg.tpos[m2]];
        int b = 0;
#pragma unroll
        for (int m1 = 0; m1 < 6; ++m1)
            if (m1 < f.k1 && f.t1[m1] == q) b = 1 << m1;
        ymask[m2] = b;
        fin.ymask[m2] = b;
    }
    fin.Y = Y;
    fin.Wc = Wc;
    fin.no = 1 << no;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int rows = pdep_bits<6>(s, a.omask);
        int iy = 0;
#pragma unroll
        for (int m = 0; m < 6; ++m)
            if ((rows >> m) & 1) iy |= ymask[m];
        fin.iys[s] = iy;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    split6s_tiles<LOWT, 2>((g_float2*)psi, nullptr, nullptr, Ls[w], (c_epi*)epi2, sg, (uint64_t)xcd_block() * WAVES + w,
                           ntiles, (uint64_t)gridDim.x * WAVES, &fin);
}

// Table form with a 7-qubit second cluster (the first has at most 7 qubits):
// the write-only pass has no matrix in LDS, only the table (rows of 128
// outputs). The lanes own the amplitudes the 7-qubit cluster kernel's lanes do
// - lane (p, h) the amplitudes j | h << 6 of column p; each output is summed
// from at most 4 table rows, weighted by w at the first cluster's index, then
// takes both epilogues' column factors and the second one's row signs.
//
// The pass is bound by its stores. Those of the lanes' own order scatter over
// partial 128-byte lines when the targets are low bits (at 30 qubits 2.71 ms
// with targets 0-3 and 7-9, 1.70 ms with 0, 1, 6, 7, 12, 13, 19). So each wave
// turns its tile round in LDS, a quarter at a time (the tile less targets 4
// and 5: 8 KiB; a whole tile a wave would leave room for only 4 waves), and
// stores 16 bytes a lane in state order: 1.62 and 1.58 ms (a plain
// fill takes 1.25). Non-temporal stores gained nothing here (1.72 and 1.65).
constexpr int kFold7Row = 130;  // LDS row: 128 outputs and a 16-byte pad

__global__ __launch_bounds__(512, 1) void k_fold2t7_f32(float2* __restrict__ psi, const float2* __restrict__ Yg,
                                                        const EpiDesc* __restrict__ epi2,
                                                        const EpiDesc* __restrict__ epi1, ClusterGeom g, Fold2Args f,
                                                        FoldTabArgs a, StageGeom sg) {
    constexpr int K = 7, HX = 64, WAVES = 8;
    __shared__ float2 Y[kFoldTab7Rows * kFold7Row];
    __shared__ float2 W[128];
    __shared__ int Wc[128];
    __shared__ vf4 Ls[WAVES][512];
    const int no = __popc(a.omask);
    const int nq = 64 << (no + __popc(a.rmask));  // 16-byte pieces of the table
    for (int i = (int)threadIdx.x; i < nq; i += (int)blockDim.x)
        reinterpret_cast<vf4*>(Y + (i >> 6) * kFold7Row)[i & 63] = reinterpret_cast<const vf4*>(Yg)[i];
    if ((int)threadIdx.x < 128) {
        W[threadIdx.x] = make_float2(0.0f, 0.0f);
        Wc[threadIdx.x] = pext_bits<7>((int)threadIdx.x, a.rmask) << no;
    }
    __syncthreads();
    row_sums(f.M1, 1 << f.k1, f.amp, W);  // w: the first cluster applied to the uniform vector
    __syncthreads();
    // w-index bits of the rows both clusters hold, per shared-row pattern
    int iys[4];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
        const int rows = pdep_bits<7>(sp, a.omask);
        int iy = 0;
#pragma unroll
        for (int m = 0; m < K; ++m)
            if ((rows >> m) & 1)
#pragma unroll
                for (int m1 = 0; m1 < 7; ++m1)
                    if (m1 < f.k1 && f.t1[m1] == g.t[m]) iy |= 1 << m1;
        iys[sp] = iy;
    }
    const int nsp = 1 << no;

    const int lane = threadIdx.x & 63, p = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t ntiles = g.ncols / 32;
    const uint64_t stride = (uint64_t)gridDim.x * WAVES;
    // the quarter in LDS: the tile without the bits of targets 4 and 5
    vf4* L4 = Ls[w];
    float2* L2 = reinterpret_cast<float2*>(L4);
    auto slot = [](int v) { return v ^ (((v >> 5) & 15) << 1); };  // upper bits folded into the bank bits
    const int x4 = sg.tpos[4], x5 = sg.tpos[5];
    auto sub = [&](int b) { return b - (b > x4) - (b > x5); };  // position of tile bit b in it
    int ct = h << sub(sg.tpos[6]);
#pragma unroll
    for (int b = 0; b < 5; ++b)
        if ((p >> b) & 1) ct |= 1 << sub(sg.cpos[b]);
    const int lslot = slot(ct), lin = slot(2 * lane);
    int rmask[4], cmask[3];
#pragma unroll
    for (int m = 0; m < 4; ++m) rmask[m] = slot(1 << sub(sg.tpos[m]));
#pragma unroll
    for (int b = 0; b < 3; ++b) cmask[b] = slot(128 << b);
    uint64_t lane_off = 0, imask[3] = {0, 0, 0};  // state offsets of its linear order
#pragma unroll
    for (int b = 0; b < 12; ++b) {
        if (b == x4 || b == x5) continue;
        const int at = sub(b);
        const uint64_t bit = uint64_t(1) << sg.tb[b];
        if (at >= 1 && at <= 6 && ((lane >> (at - 1)) & 1)) lane_off |= bit;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (at == 7 + c) imask[c] = bit;
    }
    for (uint64_t tile = (uint64_t)xcd_block() * WAVES + w; tile < ntiles; tile += stride) {
        const uint64_t tb0 = deposit_cols<K>(tile * 32, g);
        const uint64_t base = deposit_cols<K>(tile * 32 + p, g);
        // the first cluster's index from the column's bits (its qubits among
        // the second's targets are rows: zero in base)
        int ic = 0;
#pragma unroll
        for (int m = 0; m < 7; ++m)
            if (m < f.k1) ic |= (int)((base >> f.t1[m]) & 1) << m;
        ColFactor<float> f1{0u, 0u, 1.0f, 0.0f}, f2{0u, 0u, 1.0f, 0.0f};
        if (epi1 != nullptr) f1 = col_factor<float>((c_epi*)epi1, base);
        if (epi2 != nullptr) f2 = col_factor<float>((c_epi*)epi2, base);
        const int pb = Wc[f1.w & 127u];
        float X[2 * HX];
#pragma unroll
        for (int j = 0; j < 2 * HX; ++j) X[j] = 0.0f;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
            if (sp < nsp) {
                const float2 wv = W[ic | iys[sp]];
                const vf4* row = reinterpret_cast<const vf4*>(Y + (pb + sp) * kFold7Row + h * HX);
#pragma unroll
                for (int q = 0; q < HX / 2; ++q) {
                    const vf4 v = row[q];
                    X[4 * q] = fmaf(wv.x, v.x, fmaf(-wv.y, v.y, X[4 * q]));
                    X[4 * q + 1] = fmaf(wv.x, v.y, fmaf(wv.y, v.x, X[4 * q + 1]));
                    X[4 * q + 2] = fmaf(wv.x, v.z, fmaf(-wv.y, v.w, X[4 * q + 2]));
                    X[4 * q + 3] = fmaf(wv.x, v.w, fmaf(wv.y, v.z, X[4 * q + 3]));
                }
            }
        }
        // the column factor of both epilogues (the first one's row signs are
        // in the table; the second one's sign mask over the lane's rows j and
        // its term on target 6, the lane's h)
        const uint32_t sgn = f1.sgn ^ f2.sgn ^ ((uint32_t)h & (f2.w >> (K - 1)));
        float ucr = f1.cr * f2.cr - f1.ci * f2.ci, uci = f1.cr * f2.ci + f1.ci * f2.cr;
        if (sgn & 1u) {
            ucr = -ucr;
            uci = -uci;
        }
        const uint32_t wl = f2.w & 63u;
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = 16 * qt + r;
                const float xr = X[2 * j], xi = X[2 * j + 1];
                const float neg = (__popc((uint32_t)j & wl) & 1) ? -1.0f : 1.0f;
                int at = lslot;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if ((r >> m) & 1) at ^= rmask[m];
                L2[at] = make_float2(neg * fmaf(xr, ucr, -(xi * uci)), neg * fmaf(xr, uci, xi * ucr));
            }
            wave_lds_fence();
            vf4* out = reinterpret_cast<vf4*>(psi + (tb0 | ((qt & 1) ? uint64_t(1) << g.t[4] : 0) |
                                                     ((qt & 2) ? uint64_t(1) << g.t[5] : 0) | lane_off));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                int at = lin;
                uint64_t o = 0;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if ((i >> c) & 1) {
                        at ^= cmask[c];
                        o |= imask[c];
                    }
                out[o >> 1] = L4[at >> 1];
            }
            wave_lds_fence();
        }
    }
}

// ------------------------------------------------------------ batched persistent launch
// Many independent circuits in one launch. Work items (an op and a run of its
// tiles) are handed out by an atomic ticket in dependency order -
// the j-th op of every circuit before any (j+1)-th op - so an item only ever
// waits for items with smaller tickets, which running work-groups hold. Before
// starting, a work-group waits until all earlier items of its circuit are
// complete (per-circuit counter, release / acquire at device scope); the wait
// is bounded by the device's wall clock and sets an error flag instead of
// hanging. counters: [0] ticket, [1] error flag, [2 + c] completed items of
// circuit c.
//
// Loop shape: the loop body ends with a work-group barrier, and the single
// thread-0 block (publish the previous item, take a ticket) opens it, so the
// loop has one latch that every thread passes. A thread-0 block just before
// the back edge would give the header two back edges; the compiler may then
// split the loop into an inner loop that every other thread keeps running -
// through the barriers, re-reading a stale ticket - while thread 0 waits
// outside it. The ticket goes through readfirstlane so that the exit test is
// uniform, too.
__global__ __launch_bounds__(512, 1) void k_batch_f32(const BatchOp* __restrict__ ops,
                                                      const BatchItem* __restrict__ items, uint32_t n_items,
                                                      uint32_t* counters, uint32_t item_tiles, uint64_t wait_ticks) {
    constexpr int K = 5, C = 6, WAVES = 8;
    // One LDS buffer, two layouts. 5-qubit ops: the real-split matrix (16 KiB)
    // and a 16 KiB tile per wave; 6-qubit ops: the fp16 matrix halves (64 KiB)
    // and an 8 KiB half tile per wave. 144 KiB: one work-group per CU.
    __shared__ vf4 Lraw[1024 + WAVES * 1024];
    // the ticket is broadcast through the matrix region (read before the
    // barrier that precedes every matrix load)
    uint32_t* s_it = reinterpret_cast<uint32_t*>(Lraw);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint32_t* done = counters + 2;
    int prev = -1;  // circuit of the item just finished (uniform)
    for (;;) {
        if (threadIdx.x == 0) {
            // the previous item's stores are complete and released (fence + barrier below)
            if (prev >= 0) __hip_atomic_fetch_add(done + prev, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            *s_it = atomicAdd(counters, 1u);
        }
        __syncthreads();
        const uint32_t it = __builtin_amdgcn_readfirstlane(*s_it);
        if (it >= n_items) break;
        const BatchItem item = items[it];
        const BatchOp* op = ops + item.op;
        const uint32_t dep = op->dep;
        const int circ = op->circuit;
        if (threadIdx.x == 0 && dep > 0) {
            const uint64_t t0 = wall_clock64();
            while (__hip_atomic_load(done + circ, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < dep) {
                if (wall_clock64() - t0 > wait_ticks) {
                    atomicOr(counters + 1, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(4);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const uint64_t tiles = op->tiles;
        const uint64_t t_end = item.tile0 + item_tiles < tiles ? item.tile0 + item_tiles : tiles;
        g_float2* psi = (g_float2*)op->psi;
        if (op->kind == 0) {
            const g_vf4* A = (const g_vf4*)op->A;
            c_epi* epi = (c_epi*)op->epi;
            float* As = reinterpret_cast<float*>(Lraw);
            load_matrix<2 * 32 * 64, WAVES * 64>(As, A);
            __syncthreads();
            vf4* L4 = Lraw + 1024 + w * 1024;
            if (op->lowt)
                staged_f32_tiles<K, C, true>(psi, As, L4, epi, op->sg, item.tile0 + w, t_end, WAVES);
            else
                staged_f32_tiles<K, C, false>(psi, As, L4, epi, op->sg, item.tile0 + w, t_end, WAVES);
        } else if (op->kind == 3) {
            // a 6-qubit cluster: fp16 matrix halves, staged half tiles
            const g_vf4* A = (const g_vf4*)op->A;
            c_epi* epi = (c_epi*)op->epi;
            half8* Ah = reinterpret_cast<half8*>(Lraw);
            half8* Al = Ah + 2048;
            load_matrix<2048 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(Ah), A);
            load_matrix<2048 * 8, WAVES * 64>(reinterpret_cast<_Float16*>(Al), A + 2048);
            __syncthreads();
            float2* L = reinterpret_cast<float2*>(Lraw + 4096 + w * 512);
            if (op->lowt)
                split6s_tiles<true>(psi, Ah, Al, L, epi, op->sg, item.tile0 + w, t_end, WAVES);
            else
                split6s_tiles<false>(psi, Ah, Al, L, epi, op->sg, item.tile0 + w, t_end, WAVES);
        } else if (op->kind == 4) {
            // the uniform start with the circuit's first cluster, written in one
            // pass: amplitude (column, target index y) = w[y] times the column's
            // epilogue factor, w = 2^(-n/2) times the row sums of the cluster
            // an opaque copy of the lane: what this branch derives from it is not
            // hoisted out of the item loop, where it would be live in every branch
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int k = (int)op->k, d = 1 << k, cb = 11 - k;
            const double2* M = reinterpret_cast<const double2*>(op->A);
            c_epi* epi = (c_epi*)op->epi;
            const bool has_ph = epi != nullptr && epi->n_ph > 0;
            float2* Wl = reinterpret_cast<float2*>(Lraw);  // 64 entries
            ColFactor<float>* Fl = reinterpret_cast<ColFactor<float>*>(Lraw + 32 + w * 64);  // per wave, 64
            row_sums(M, d, std::sqrt(__builtin_ldexp(1.0, -op->n)), Wl);
            __syncthreads();
            const StageGeom& sg = op->sg;
            // tile index tau -> (y over the targets, column index): linear over
            // OR, so the lane's, the chunk's and bit 0's parts are taken apart
            auto y_of = [&](int tau) {
                int y = 0;
                for (int m = 0; m < k; ++m) y |= ((tau >> sg.tpos[m]) & 1) << m;
                return y;
            };
            auto c_of = [&](int tau) {
                int c = 0;
                for (int b = 0; b < cb; ++b) c |= ((tau >> sg.cpos[b]) & 1) << b;
                return c;
            };
            const int yl = y_of(ln << 1), cl = c_of(ln << 1), y1 = y_of(1), c1 = c_of(1);
            // per chunk bit (tile bits 7..10): its row / column index bit and state offset
            int ych[4], cch[4];
            uint64_t och[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                ych[b] = y_of(128 << b);
                cch[b] = c_of(128 << b);
                och[b] = uint64_t(1) << sg.tb[7 + b];
            }
            uint64_t lane_off = 0;
#pragma unroll
            for (int b = 0; b < 6; ++b)
                if ((ln >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b + 1];
            uint64_t cstate = 0;  // state bits of column `lane` (its factor is this lane's to compute)
            for (int b = 0; b < cb; ++b)
                if ((ln >> b) & 1) cstate |= uint64_t(1) << sg.tb[sg.cpos[b]];
            g_vf4* p4 = reinterpret_cast<g_vf4*>(psi);
            for (uint64_t t = item.tile0 + w; t < t_end; t += WAVES) {
                const uint64_t tb0 = tile_base<11>(t, sg);
                if (ln < (1 << cb)) {
                    ColFactor<float> f{0u, 0u, 1.0f, 0.0f};
                    if (epi != nullptr) f = col_factor<float>(epi, tb0 | cstate);
                    Fl[ln] = f;
                }
                wave_lds_fence();
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    int yi = 0, ci = 0;  // uniform
                    uint64_t o = tb0 | lane_off;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if ((i >> b) & 1) {
                            yi |= ych[b];
                            ci |= cch[b];
                            o |= och[b];
                        }
                    vf4 v;
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int y = yl | yi | (b ? y1 : 0), c = cl | ci | (b ? c1 : 0);
                        const float2 a = Wl[y];
                        const ColFactor<float> f = Fl[c];
                        float re = a.x, im = a.y;
                        apply_factor(re, im, f, (uint32_t)y, has_ph);
                        v[2 * b] = re;
                        v[2 * b + 1] = im;
                    }
                    p4[o >> 1] = v;  // linear chunk i of the tile
                }
                wave_lds_fence();
            }
        } else {
            // initialisation: tile t is amplitudes [t 2^11, (t + 1) 2^11)
            // 2^(-n/2): a power of two, times 1/sqrt(2) for odd n (both exact scalings of a rounded constant)
            const float val = op->kind == 1 ? 0.0f
                                            : __builtin_ldexpf((op->n & 1) ? 0.70710678118654752440f : 1.0f,
                                                               -(op->n >> 1));
            g_vf4* p4 = reinterpret_cast<g_vf4*>(psi);
            for (uint64_t t = item.tile0 + w; t < t_end; t += WAVES) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint64_t q = (t << 10) + (uint64_t)(i * 64 + lane);  // index of an amplitude pair
                    vf4 v = {val, 0.0f, val, 0.0f};
                    if (op->kind == 1 && q == 0) v.x = 1.0f;
                    p4[q] = v;
                }
            }
        }
        // every wave waits until its stores are complete in L2; after the
        // barrier, thread 0's device-scope release (an L2 write-back, then the
        // counter) publishes them all. A release fence in every wave would
        // write the L2 back once per wave, which costs more than the tiles.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        prev = circ;
    }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t n, uint32_t v) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------ cluster: vector ALU
// One column per thread; the matrix M[y][x] (complex) sits in LDS and is read
// as a broadcast. Used for small k and for states too small for a wave tile.
template <typename T, int K>
__global__ __launch_bounds__(256) void k_cluster_valu(typename Cplx<T>::type* __restrict__ psi,
                                                      const typename Cplx<T>::type* __restrict__ M,
                                                      const EpiDesc* __restrict__ epi, ClusterGeom g) {
    using V = typename Cplx<T>::type;
    constexpr int D = 1 << K;
    __shared__ V Ms[D * D];
    for (int i = threadIdx.x; i < D * D; i += 256) Ms[i] = M[i];
    __syncthreads();
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t c = (uint64_t)blockIdx.x * 256 + threadIdx.x; c < g.ncols; c += stride) {
        const uint64_t base = deposit_cols<K>(c, g);
        V v[D];
#pragma unroll
        for (int x = 0; x < D; ++x) v[x] = psi[base | target_off<K>(x, g)];
        ColFactor<T> f{0u, 0u, T(1), T(0)};
        if (has_epi) f = col_factor<T>(epi, base);
#pragma unroll
        for (int y = 0; y < D; ++y) {
            T ar = 0, ai = 0;
#pragma unroll
            for (int x = 0; x < D; ++x) {
                const V m = Ms[y * D + x];
                ar += m.x * v[x].x - m.y * v[x].y;
                ai += m.x * v[x].y + m.y * v[x].x;
            }
            if (has_epi) apply_factor(ar, ai, f, (uint32_t)y, has_ph);
            V o;
            o.x = ar;
            o.y = ai;
            psi[base | target_off<K>(y, g)] = o;
        }
    }
}

// (ar, ai) += m v, in one fixed contraction: the forms of a cluster kernel
// with and without the sums store the same bits.
template <typename T, typename M, typename V>
__device__ __forceinline__ void cmac(T& ar, T& ai, const M& m, const V& v) {
    ar += __builtin_elementwise_fma(m.x, v.x, -(m.y * v.y));
    ai += __builtin_elementwise_fma(m.x, v.y, m.y * v.x);
}

// Two- and three-qubit clusters on states that fit the caches, and (STATS) a last
// one whose sums are wanted. With one column per thread, targets among
// the lowest state bits put lanes 2^k amplitudes apart, so each load
// instruction spreads over 2^k times the cache lines it uses, and a thread
// that holds its column and the matrix limits occupancy. Here a wave tile is
// 64 columns: the k targets and the 6 lowest non-target bits, whose lowest 6
// positions are always state bits 0..5. Chunk x of the tile (tau = 64 x +
// lane) is one contiguous run of 64 amplitudes; LDS hands each thread its
// column, then takes the results back for contiguous stores. STATS (float
// only): also sum p, p^2 and -p ln p of the stored amplitudes into part (per
// work-group), as the matrix-core kernels' STATS forms do.
template <typename T, int K, bool STATS>
__device__ __forceinline__ void valu_columns(typename Cplx<T>::type* __restrict__ psi,
                                             const typename Cplx<T>::type* __restrict__ M,
                                             const EpiDesc* __restrict__ epi, const StageGeom& sg, uint64_t tiles,
                                             double* __restrict__ part) {
    static_assert(!STATS || std::is_same<T, float>::value, "sums of float states only");
    using V = typename Cplx<T>::type;
    constexpr int D = 1 << K, RS = D + 1;  // LDS row of a column, padded
    __shared__ V Ms[D * D];
    __shared__ V Ls[4][64 * RS];
    for (int i = threadIdx.x; i < D * D; i += 256) Ms[i] = M[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    V* L = Ls[threadIdx.x >> 6];
    // element tau = 64 x + lane: its column (bits cpos) and target index (bits tpos)
    int yl = 0, cl = 0, yx[D], cx[D];
#pragma unroll
    for (int m = 0; m < K; ++m)
        if (sg.tpos[m] < 6) yl |= ((lane >> sg.tpos[m]) & 1) << m;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if (sg.cpos[b] < 6) cl |= ((lane >> sg.cpos[b]) & 1) << b;
#pragma unroll
    for (int x = 0; x < D; ++x) {
        yx[x] = 0;
        cx[x] = 0;
#pragma unroll
        for (int m = 0; m < K; ++m)
            if (sg.tpos[m] >= 6) yx[x] |= ((x >> (sg.tpos[m] - 6)) & 1) << m;
#pragma unroll
        for (int b = 0; b < 6; ++b)
            if (sg.cpos[b] >= 6) cx[x] |= ((x >> (sg.cpos[b] - 6)) & 1) << b;
    }
    // state offset of this thread's column (lane = column inside the tile)
    uint64_t coff = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) coff |= uint64_t(1) << sg.tb[sg.cpos[b]];
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;
    double sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (uint64_t tile = (uint64_t)xcd_block() * 4 + (threadIdx.x >> 6); tile < tiles;
         tile += (uint64_t)gridDim.x * 4) {
        const uint64_t tb0 = tile_base<K + 6>(tile, sg);
        V v[D];
#pragma unroll
        for (int x = 0; x < D; ++x) v[x] = psi[tb0 | sg.ioff[x] | (uint64_t)lane];
#pragma unroll
        for (int x = 0; x < D; ++x) L[(cl | cx[x]) * RS + (yl | yx[x])] = v[x];
        wave_lds_fence();
#pragma unroll
        for (int x = 0; x < D; ++x) v[x] = L[lane * RS + x];
        ColFactor<T> f{0u, 0u, T(1), T(0)};
        if (has_epi) f = col_factor<T>(epi, tb0 | coff);
#pragma unroll
        for (int y = 0; y < D; ++y) {
            T ar = 0, ai = 0;
#pragma unroll
            for (int x = 0; x < D; ++x) {
                cmac(ar, ai, Ms[y * D + x], v[x]);
            }
            if (has_epi) apply_factor(ar, ai, f, (uint32_t)y, has_ph);
            if constexpr (STATS) stats_acc_f(sv, ar, ai);
            V o;
            o.x = ar;
            o.y = ai;
            L[lane * RS + y] = o;  // a thread reads and writes only its own row here
        }
        wave_lds_fence();
#pragma unroll
        for (int x = 0; x < D; ++x) psi[tb0 | sg.ioff[x] | (uint64_t)lane] = L[(cl | cx[x]) * RS + (yl | yx[x])];
        wave_lds_fence();  // the next tile's writes come after these reads
    }
    if constexpr (STATS) block_reduce_store(sv, 3, 0u, part + blockIdx.x * 8);  // every thread gets here
}

template <typename T, int K>
__global__ __launch_bounds__(256) void k_cluster_valu_cached(typename Cplx<T>::type* __restrict__ psi,
                                                             const typename Cplx<T>::type* __restrict__ M,
                                                             const EpiDesc* __restrict__ epi, StageGeom sg,
                                                             uint64_t tiles) {
    valu_columns<T, K, false>(psi, M, epi, sg, tiles, nullptr);
}

// Clusters of one to three qubits on states beyond the caches: 8 KiB
// of state per wave (the targets and the lowest other bits), one tile per
// wave, work-groups in memory order. The tile moves as linear 16-byte accesses
// of whole runs whatever the targets are, all in flight at once; LDS hands
// each lane its columns and takes the results back. 28 qubits complex64, k = 1 /
// 2 / 3: 755 / 768 / 747 us against 862 / 845 / 832 us for the kernels above,
// which win inside the caches (18 qubits: 6.2 against 9.2 us for k = 1: more
// waves, each with less to do).
template <typename T, int K>
__device__ __forceinline__ void valu_tile(typename Cplx<T>::type* __restrict__ psi,
                                          const typename Cplx<T>::type* __restrict__ M,
                                          const EpiDesc* __restrict__ epi, const StageGeom& sg, uint64_t tiles) {
    using V = typename Cplx<T>::type;
    constexpr bool F = sizeof(T) == 4;
    constexpr int D = 1 << K, TB = F ? 10 : 9, C = TB - K, NC = (1 << C) / 64;  // columns of a lane: lane + 64 i
    constexpr int AB = F ? 1 : 0;  // tau bits of one 16-byte access
    typedef T vt2 __attribute__((ext_vector_type(2)));
    __shared__ V Ms[D * D];
    __shared__ vf4 Ls[4][512];
    if ((int)threadIdx.x < D * D) Ms[threadIdx.x] = M[threadIdx.x];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    vf4* L4 = Ls[w];
    vt2* L = reinterpret_cast<vt2*>(L4);
    const uint64_t tile = (uint64_t)blockIdx.x * 4 + w;
    const bool act = tile < tiles;
    const uint64_t tb0 = tile_base<TB>(tile, sg);
    // slot of tau: its upper bits folded into the bank bits (linear over XOR)
    auto slot = [](int t) { return F ? t ^ (((t >> 5) & 15) << 1) : t ^ ((t >> 4) & 15); };
    uint64_t lane_off = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) lane_off |= uint64_t(1) << sg.tb[b + AB];
    auto at = [&](int i) -> vf4* {  // linear access i of the tile
        return reinterpret_cast<vf4*>(psi + ((tb0 | sg.ioff[i]) | lane_off));
    };
    if (act) {
        vf4 R[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) R[i] = load16<true>((const vf4*)at(i));
#pragma unroll
        for (int i = 0; i < 8; ++i) L4[slot((i * 64 + lane) << AB) >> AB] = R[i];
    }
    __syncthreads();
    if (!act) return;
    const bool has_epi = epi != nullptr, has_ph = has_epi && epi->n_ph > 0;
    int rs[D];
#pragma unroll
    for (int x = 0; x < D; ++x) rs[x] = slot(tau_of_targets<0, K>(x, sg));
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        int tc = 0;
        uint64_t cb = 0;
#pragma unroll
        for (int b = 0; b < C; ++b)
            if (((lane + 64 * i) >> b) & 1) {
                tc |= 1 << sg.cpos[b];
                cb |= uint64_t(1) << sg.tb[sg.cpos[b]];
            }
        const int ts = slot(tc);
        vt2 v[D];
#pragma unroll
        for (int x = 0; x < D; ++x) v[x] = L[ts ^ rs[x]];
        ColFactor<T> f{0u, 0u, T(1), T(0)};
        if (has_epi) f = col_factor<T>((c_epi*)epi, tb0 | cb);
#pragma unroll
        for (int y = 0; y < D; ++y) {
            T ar = 0, ai = 0;
#pragma unroll
            for (int x = 0; x < D; ++x) {
                cmac(ar, ai, Ms[y * D + x], v[x]);
            }
            if (has_epi) apply_factor(ar, ai, f, (uint32_t)y, has_ph);
            L[ts ^ rs[y]] = vt2{ar, ai};  // the column's own slots
        }
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 8; ++i) store16<true>(at(i), (vf4)L4[slot((i * 64 + lane) << AB) >> AB]);
}

// STATS: the persistent form, since the partials of one work-group per tile
// would outgrow their area.
template <typename T, int K, bool STATS = false>
__global__ __launch_bounds__(256, sizeof(T) == 4 && K == 3 ? 3 : 4) void k_cluster_valu_staged(
    typename Cplx<T>::type* __restrict__ psi, const typename Cplx<T>::type* __restrict__ M,
    const EpiDesc* __restrict__ epi, StageGeom sg, uint64_t tiles, double* __restrict__ part) {
    if constexpr (STATS)
        valu_columns<T, K, true>(psi, M, epi, sg, tiles, part);
    else
        valu_tile<T, K>(psi, M, epi, sg, tiles);
}

// ------------------------------------------------------------ diagonal pass
// Every amplitude times the diagonal factor of its index (Sec. 3.5: diagonal
// gates need no gather). A work-group covers a run of 64 windows of 128
// consecutive amplitudes, 16 per wave, loaded up to 16 at a time before any
// factor is applied. The index splits into lo (bits 0..6, fixed per lane) and
// hi (the window, uniform per wave): terms of lo bits only are per-lane
// constants; CZ pairs with one bit in each half give a sign mask over lo. Both
// parts cost a loop over every gate of the pass, so the work-group forms them
// once: wave w takes every fourth gate, lane j the lo part of its own two
// indices and the hi part of window j of the run, and LDS combines the four
// waves' parts. 28 qubits complex64, 14 pairs and 10 phases: 690 us (6.2 TB/s)
// against 835 us for a wave that walked runs of its own; 20 qubits: 18 against
// 35 us, where those loops are most of it. Each XCD takes its own stretch here
// (linear accesses: 690 us against 734 us in plain order). The descriptor lists the pairs in `cc` and the phases in `ph`.
template <typename T, bool NT>
__global__ __launch_bounds__(256) void k_diag(typename Cplx<T>::type* __restrict__ psi, int n,
                                              const EpiDesc* __restrict__ desc) {
    constexpr bool F = sizeof(T) == 4;
    constexpr int LO = 7;                 // amplitude index bits inside a window
    constexpr int RB = 6;                 // a work-group's run: 2^RB windows
    constexpr int W = (1 << RB) / 4;      // windows of a wave
    constexpr int U = F ? 16 : 8;         // of them in flight at a time
    c_epi* e = (c_epi*)desc;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t run = xcd_block();
    const uint64_t N = uint64_t(1) << n;
    const uint64_t nwin = n >= LO ? uint64_t(1) << (n - LO) : 1;
    // this wave's share of the gates: signs of the lane's two lo indices (bits
    // 0, 1), sign mask over lo (bits 2..8) and sign (bit 9) of window `lane`,
    // phases of the two lo indices and of the window
    __shared__ uint32_t Ps[4][64];
    __shared__ double Pr[4][3][64], Pi[4][3][64];
    const uint64_t hi = ((run << RB) | (uint64_t)lane) << LO;
    {
        uint32_t sg = 0u, wm = 0u, sh = 0u;
        double r[3] = {1.0, 1.0, 1.0}, q[3] = {0.0, 0.0, 0.0};
        const int np = e->n_cc, nph = e->n_ph;
        for (int i = w; i < np; i += 4) {
            const int a = e->cc[i][0], b = e->cc[i][1];
            if (a < LO && b < LO) {
                const uint32_t l0 = 2 * lane, l1 = l0 + 1;
                sg ^= ((l0 >> a) & (l0 >> b) & 1u) | (((l1 >> a) & (l1 >> b) & 1u) << 1);
            } else if (a >= LO && b >= LO) {
                sh ^= (uint32_t)((hi >> a) & (hi >> b) & 1);
            } else if (a < LO) {
                wm ^= (uint32_t)((hi >> b) & 1) << a;
            } else {
                wm ^= (uint32_t)((hi >> a) & 1) << b;
            }
        }
        for (int i = w; i < nph; i += 4) {
            const int b = e->ph_q[i];
            const double c = e->ph[i][0], sn = e->ph[i][1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const bool on = k == 2 ? b >= LO && ((hi >> b) & 1) : b < LO && (((2 * lane + k) >> b) & 1);
                if (on) {
                    const double t = r[k] * c - q[k] * sn;
                    q[k] = r[k] * sn + q[k] * c;
                    r[k] = t;
                }
            }
        }
        Ps[w][lane] = sg | wm << 2 | sh << 9;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Pr[w][k][lane] = r[k];
            Pi[w][k][lane] = q[k];
        }
    }
    __syncthreads();
    uint32_t ps = 0u;
    double r[3] = {1.0, 1.0, 1.0}, q[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        ps ^= Ps[v][lane];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double c = Pr[v][k][lane], sn = Pi[v][k][lane];
            const double t = r[k] * c - q[k] * sn;
            q[k] = r[k] * sn + q[k] * c;
            r[k] = t;
        }
    }
    typedef T vt2 __attribute__((ext_vector_type(2)));
    constexpr int PER = F ? 1 : 2;  // 16-byte accesses of a lane per window
#pragma unroll
    for (int w0 = 0; w0 < W; w0 += U) {
        vf4 v[U * PER];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t win = (run << RB) | (uint64_t)(w * W + w0 + u);
            const uint64_t i0 = (win << LO) | (uint64_t)(2 * lane);
            // windows past the end, and lanes past the end of states of fewer than 7 qubits
            if (win < nwin && i0 < N)
#pragma unroll
                for (int k = 0; k < PER; ++k) v[u * PER + k] = load16<NT>(reinterpret_cast<const vf4*>(psi + i0) + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int wl = w * W + w0 + u;
            const uint64_t win = (run << RB) | (uint64_t)wl;
            const uint64_t i0 = (win << LO) | (uint64_t)(2 * lane);
            const uint32_t pw = (uint32_t)__builtin_amdgcn_readlane((int)ps, wl) >> 2;
            const double hr = readlane_f64(r[2], wl), hq = readlane_f64(q[2], wl);
            if (win >= nwin || i0 >= N) continue;
            T z[4];
            if constexpr (F) {
#pragma unroll
                for (int k = 0; k < 4; ++k) z[k] = v[u][k];
            } else {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const vt2 d = __builtin_bit_cast(vt2, v[u * PER + k]);
                    z[2 * k] = d.x;
                    z[2 * k + 1] = d.y;
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t lo = 2 * lane + h;
                const bool neg = ((ps >> h ^ pw >> 7 ^ (uint32_t)__popc(lo & pw & 0x7fu)) & 1u) != 0;
                const T fr = (T)(hr * r[h] - hq * q[h]);
                const T fi = (T)(hr * q[h] + hq * r[h]);
                const T re = z[2 * h] * fr - z[2 * h + 1] * fi;
                const T im = z[2 * h] * fi + z[2 * h + 1] * fr;
                z[2 * h] = neg ? -re : re;
                z[2 * h + 1] = neg ? -im : im;
            }
            vf4* out = reinterpret_cast<vf4*>(psi + i0);
            if constexpr (F) {
                store16<NT>(out, vf4{z[0], z[1], z[2], z[3]});
            } else {
                store16<NT>(out, __builtin_bit_cast(vf4, vt2{z[0], z[1]}));
                store16<NT>(out + 1, __builtin_bit_cast(vf4, vt2{z[2], z[3]}));
            }
        }
    }
}

// ------------------------------------------------------------ per-gate kernels
// The plain method's kernels stream the state in 16-byte units (one complex128
// or two complex64 amplitudes), several per thread in flight, work-groups in
// memory order. A qubit whose bit lies inside a 128-byte line (unit bits 0..2)
// is handled on whole lines: as single accesses of every second unit the
// lines would be moved half used, and non-temporal stores of part of a line
// are several times slower. 28 qubits complex64: H 710 us (6.0 TB/s) against
// 850-905 us one pair per thread, T 350-740 against 412-885 us, CZ 172-735
// against 206-870 us by the qubits.
template <typename T>
struct Unit;
template <>
struct Unit<float> {
    typedef vf4 type;
    static constexpr int AMPS = 2, BITS = 1;
};
template <>
struct Unit<double> {
    typedef vd2 type;
    static constexpr int AMPS = 1, BITS = 0;
};

// A single-qubit gate on the pairs (i, i + 2^q) with bit q of i clear (Sec. 2).
// MODE 0: unit bit ub >= 3, a thread takes both units of four pairs;
// 1..3: unit bit 0..2, a lane owns a unit and takes its partner's from the lane
// that differs in that bit; 4: the pair lies in one (complex64) unit.
template <typename T>
struct Gate2x2 {
    T m[8];
};
// Units of a thread: 8 in flight. In the caches (not NT) MODE 0 takes 4, for
// more wavefronts: 23 / 24 qubits complex128, H on the highest qubit 38.4 /
// 71.7 us against 41.1 / 73.5; on whole lines 8 are as fast or faster.
constexpr int gate1q_units(int mode, bool nt) { return mode == 0 && !nt ? 4 : 8; }

template <typename T, int MODE, bool NT>
__global__ __launch_bounds__(256, 6) void k_gate1q(typename Unit<T>::type* __restrict__ psi, int ub, Gate2x2<T> g,
                                                uint64_t units) {
    using V = typename Unit<T>::type;
    constexpr int A = Unit<T>::AMPS;
    const T* m = g.m;
    constexpr int PER = gate1q_units(MODE, NT);
    const uint32_t wg = tile_block<256 * PER * 16>();
    // row of the 2x2: c0 a + c1 b
    auto row = [](T c0r, T c0i, T c1r, T c1i, T ar, T ai, T br, T bi, T& re, T& im) {
        re = (c0r * ar - c0i * ai) + (c1r * br - c1i * bi);
        im = (c0r * ai + c0i * ar) + (c1r * bi + c1i * br);
    };
    if constexpr (MODE == 0) {
        constexpr int P = PER / 2;
        V a[P], b[P];
        uint64_t at[P];
        const uint64_t bit = uint64_t(1) << ub, pairs = units / 2;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const uint64_t p = ((uint64_t)wg * P + u) * 256 + threadIdx.x;
            at[u] = insert_zero(min(p, pairs - 1), ub);
            a[u] = load16<NT>(psi + at[u]);
            b[u] = load16<NT>(psi + (at[u] | bit));
        }
#pragma unroll
        for (int u = 0; u < P; ++u) {
            if (((uint64_t)wg * P + u) * 256 + threadIdx.x >= pairs) break;
            V x, y;
#pragma unroll
            for (int k = 0; k < A; ++k) {
                T r, i;
                row(m[0], m[1], m[2], m[3], a[u][2 * k], a[u][2 * k + 1], b[u][2 * k], b[u][2 * k + 1], r, i);
                x[2 * k] = r;
                x[2 * k + 1] = i;
                row(m[4], m[5], m[6], m[7], a[u][2 * k], a[u][2 * k + 1], b[u][2 * k], b[u][2 * k + 1], r, i);
                y[2 * k] = r;
                y[2 * k + 1] = i;
            }
            store16<NT>(psi + at[u], x);
            store16<NT>(psi + (at[u] | bit), y);
        }
    } else {
        constexpr int P = PER;
        V a[P];
        const uint64_t u0 = (uint64_t)wg * P * 256 + threadIdx.x;
#pragma unroll
        for (int u = 0; u < P; ++u) a[u] = load16<NT>(psi + min(u0 + u * 256, units - 1));
#pragma unroll
        for (int u = 0; u < P; ++u) {
            V o = a[u];
            if constexpr (MODE == 4) {
                T r, i;
                row(m[0], m[1], m[2], m[3], a[u][0], a[u][1], a[u][2], a[u][3], r, i);
                o[0] = r;
                o[1] = i;
                row(m[4], m[5], m[6], m[7], a[u][0], a[u][1], a[u][2], a[u][3], r, i);
                o[2] = r;
                o[3] = i;
            } else {
                const vf4 own = __builtin_bit_cast(vf4, a[u]);
                vf4 oth;
#pragma unroll
                for (int k = 0; k < 4; ++k) oth[k] = __uint_as_float(lane_xor<MODE - 1>(__float_as_uint(own[k])));
                const V b = __builtin_bit_cast(V, oth);
                const bool hi = (threadIdx.x >> (MODE - 1)) & 1;
#pragma unroll
                for (int k = 0; k < A; ++k) {
                    const T lr = hi ? b[2 * k] : a[u][2 * k], li = hi ? b[2 * k + 1] : a[u][2 * k + 1];
                    const T hr = hi ? a[u][2 * k] : b[2 * k], hh = hi ? a[u][2 * k + 1] : b[2 * k + 1];
                    T r, i;
                    row(hi ? m[4] : m[0], hi ? m[5] : m[1], hi ? m[6] : m[2], hi ? m[7] : m[3], lr, li, hr, hh, r, i);
                    o[2 * k] = r;
                    o[2 * k + 1] = i;
                }
            }
            if (u0 + u * 256 < units) store16<NT>(psi + (u0 + u * 256), o);
        }
    }
}

// Diagonal gates of the plain method: diag(1, e^{i phi}) on one qubit (only
// amplitudes with its bit set change) or CZ (NEG: amplitudes with both bits
// set are negated). hb0 < hb1: the set unit bits that select the units (-1:
// none), all from 3 up, from 2 in the caches; lomask: set bits among the lower
// ones, and odd: the second amplitude of a complex64 unit only - these select
// among the units that are moved.
// spread: each XCD takes its own stretch of the state, in the caches (see
// tile_block) and, beyond them, for unit bit 7. Selecting every other
// 2 KiB (unit bit 7) leaves half of the memory channels idle in one compact
// stretch: 28 qubits complex64, T on qubit 8, 354 us spread over eight against
// 546 us; any other bit is as fast or faster in memory order (T on qubit 27:
// 350 against 374 us). P: units of a thread (24 qubits complex128, T on qubit 0:
// 73 us with 2, 78 with 8).
template <typename T, bool NEG, bool NT, int P>
__global__ __launch_bounds__(256, 6) void k_phase(typename Unit<T>::type* __restrict__ psi, int hb0, int hb1, int lomask,
                                               int odd, int spread, T cr, T ci, uint64_t count) {
    using V = typename Unit<T>::type;
    constexpr int A = Unit<T>::AMPS;
    V a[P];
    uint64_t at[P];
    const uint64_t u0 = (uint64_t)(spread ? xcd_block() : blockIdx.x) * P * 256 + threadIdx.x;
#pragma unroll
    for (int u = 0; u < P; ++u) {
        uint64_t i = min(u0 + u * 256, count - 1);
        if (hb0 >= 0) i = insert_zero(i, hb0) | uint64_t(1) << hb0;
        if (hb1 >= 0) i = insert_zero(i, hb1) | uint64_t(1) << hb1;
        at[u] = i;
        a[u] = load16<NT>(psi + i);
    }
    const bool sel = ((int)threadIdx.x & lomask) == lomask;  // unit bits 0..2 are lane bits
#pragma unroll
    for (int u = 0; u < P; ++u) {
        V o = a[u];
#pragma unroll
        for (int k = 0; k < A; ++k) {
            if (!sel || (A == 2 && k == 0 && odd)) continue;
            if constexpr (NEG) {
                o[2 * k] = -a[u][2 * k];
                o[2 * k + 1] = -a[u][2 * k + 1];
            } else {
                o[2 * k] = a[u][2 * k] * cr - a[u][2 * k + 1] * ci;
                o[2 * k + 1] = a[u][2 * k] * ci + a[u][2 * k + 1] * cr;
            }
        }
        if (u0 + u * 256 < count) store16<NT>(psi + at[u], o);
    }
}

// ------------------------------------------------------------ initialisation
template <typename T>
__global__ __launch_bounds__(256) void k_init(typename Cplx<T>::type* __restrict__ psi, uint64_t count,
                                              int mode, T val) {
    using V = typename Cplx<T>::type;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += stride) {
        V v;
        v.x = (mode == 0) ? (i == 0 ? T(1) : T(0)) : val;
        v.y = T(0);
        psi[i] = v;
    }
}

// ------------------------------------------------------------ initialisation folded into the first cluster
// The uniform state (the skipped leading H layer, Sec. 3.6) is a product state,
// and so is the first cluster's result on it: amplitude i is
// w[y(i)] = 2^(-n/2) sum_x M[y(i)][x], y(i) the target bits of i, times the
// cluster's diagonal epilogue factor. One write-only pass replaces the
// initialisation and the first cluster's read-and-write pass. M is the plain
// complex128 matrix; w is summed in float64 and rounded once.
template <typename T, int K>
__global__ __launch_bounds__(256) void k_init_cluster(typename Cplx<T>::type* __restrict__ psi, ClusterGeom g,
                                                      const double2* __restrict__ M,
                                                      const EpiDesc* __restrict__ epi, double amp) {
    using V = typename Cplx<T>::type;
    constexpr int D = 1 << K;
    __shared__ double2 w[D];
    __shared__ uint64_t toff[D];
    row_sums(M, D, amp, w);
    if ((int)threadIdx.x < D) {
        uint64_t o = 0;
        for (int m = 0; m < K; ++m)
            if ((threadIdx.x >> m) & 1) o |= uint64_t(1) << g.t[m];
        toff[threadIdx.x] = o;
    }
    __syncthreads();
    const bool has_epi = epi != nullptr;
    const bool has_ph = has_epi && epi->n_ph > 0;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    if constexpr (sizeof(T) == 4) {
        // float: 16-byte stores. With qubit 0 a target, amplitudes y, y + 1 of a
        // column are neighbours; otherwise columns 2c, 2c + 1 differ in bit 0 only
        // and a thread writes both, side by side.
        if (g.t[0] == 0) {
            for (uint64_t c = (uint64_t)xcd_block() * 256 + threadIdx.x; c < g.ncols; c += stride) {
                const uint64_t base = deposit_cols<K>(c, g);
                ColFactor<T> f{0u, 0u, T(1), T(0)};
                if (has_epi) f = col_factor<T>(epi, base);
#pragma unroll 8
                for (int y = 0; y < D; y += 2) {
                    const double2 v0 = w[y], v1 = w[y + 1];
                    T r0 = (T)v0.x, i0 = (T)v0.y, r1 = (T)v1.x, i1 = (T)v1.y;
                    if (has_epi) {
                        apply_factor(r0, i0, f, (uint32_t)y, has_ph);
                        apply_factor(r1, i1, f, (uint32_t)(y + 1), has_ph);
                    }
                    *reinterpret_cast<vf4*>(psi + (base | toff[y])) = vf4{r0, i0, r1, i1};
                }
            }
            return;
        }
        if (g.ncols >= 2) {
            for (uint64_t c = (uint64_t)xcd_block() * 256 + threadIdx.x; c < g.ncols / 2; c += stride) {
                const uint64_t base = deposit_cols<K>(2 * c, g);  // bit 0 clear; column 2c + 1 is base | 1
                ColFactor<T> f0{0u, 0u, T(1), T(0)}, f1 = f0;
                if (has_epi) {
                    f0 = col_factor<T>(epi, base);
                    f1 = col_factor<T>(epi, base | 1);
                }
#pragma unroll 8
                for (int y = 0; y < D; ++y) {
                    const double2 v = w[y];
                    T r0 = (T)v.x, i0 = (T)v.y, r1 = r0, i1 = i0;
                    if (has_epi) {
                        apply_factor(r0, i0, f0, (uint32_t)y, has_ph);
                        apply_factor(r1, i1, f1, (uint32_t)y, has_ph);
                    }
                    *reinterpret_cast<vf4*>(psi + (base | toff[y])) = vf4{r0, i0, r1, i1};
                }
            }
            return;
        }
    }
    // one thread per column (assignment of the non-target bits): its diagonal
    // factor once, then the column's 2^k amplitudes
    for (uint64_t c = (uint64_t)xcd_block() * 256 + threadIdx.x; c < g.ncols; c += stride) {
        const uint64_t base = deposit_cols<K>(c, g);
        ColFactor<T> f{0u, 0u, T(1), T(0)};
        if (has_epi) f = col_factor<T>(epi, base);
#pragma unroll
        for (int y = 0; y < D; ++y) {
            const double2 v = w[y];
            T re = (T)v.x, im = (T)v.y;
            if (has_epi) apply_factor(re, im, f, (uint32_t)y, has_ph);
            V o;
            o.x = re;
            o.y = im;
            psi[base | toff[y]] = o;
        }
    }
}

// ------------------------------------------------------------ cluster-matrix builder
// A cluster's matrix is built column by column in float64: column x starts as
// the basis vector e_x of the 2^k space and takes the cluster's gates in
// order (it is reused for all 2^(n-k) columns of the state, Sec. 3.2). The
// result is written in the layout of the kernel that will apply it.
//
// A wave holds its columns in registers, one entry per lane: row bits 0..5
// are lane bits (row bit 6 of a 7-qubit matrix is a second register; below 6
// qubits the lanes above the rows hold further columns), and each lane has
// kBuildCols consecutive columns. A one-qubit gate is then one exchange with
// the lane whose index differs in one bit (a DPP move, or a permlane swap for
// bits 4 and 5) and a complex 2x2 product, a diagonal gate touches the lane's
// own entry only, and no gate needs a barrier. What bounds the launch is this
// chain over the gates, so the columns are spread over as many waves as keep
// kBuildCols of them per lane (4: the entries a lane then holds are
// neighbours in the fp16-halves layouts, which are written 16 bytes at a
// time): 16 waves for a 6-qubit matrix, 32 for a 7-qubit one. Measured
// against one work-group per matrix that held it in LDS with a barrier per
// gate: 17 us instead of 62 for the 11 matrices of a 20-qubit depth-25
// circuit, 26 instead of 85 for the 14 of the 30-qubit one, 53 instead of 155
// for the 634 of a batch of 64 circuits, and 4 / 6 / 9 us instead of 36 / 92 /
// 190 for a single dense gate of 4 / 5 / 6 qubits.
constexpr int kBuildThreads = 256;
constexpr int kBuildCols = 4;        // columns per lane
constexpr int kBuildGateChunk = 64;  // gates staged in LDS at a time

// build_parts(k) work-groups per matrix of k qubits hold kBuildThreads / 64
// waves of kBuildCols * 2^(6-k) columns each; kBuildCols for k = 7.

struct BuildLds {
    // gates of the current chunk; op: 0 CZ, 1 diagonal one-qubit (phase m[6..7]
    // on |1>), 2 one-qubit, 3 dense
    double m[kBuildGateChunk][8];
    int32_t op[kBuildGateChunk], nq[kBuildGateChunk], off[kBuildGateChunk], pos[kBuildGateChunk][6];
    // a dense gate's input: entry (row, column of the lane) of each wave
    double2 v[kBuildThreads / 64][128 * kBuildCols];
};

// R registers per column: 2 for k = 7 (row bit 6), else 1.
template <int R>
__device__ __forceinline__ void build_matrix(const BuildOp& op, int part, const BuildGate* __restrict__ gates,
                                             const BuildTail& tail, const double* __restrict__ dense,
                                             char* __restrict__ out, BuildLds& L) {
    constexpr int C = kBuildCols;
    const int k = R == 2 ? 7 : op.k, D = 1 << k;
    const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const int rows = R == 2 ? 64 : D;              // rows on lanes
    const int yl = lane & (rows - 1);              // row bits held by the lane index
    const int grp = R == 2 ? 0 : lane >> k;        // which of the slot's columns
    const int x0 = ((part * (kBuildThreads / 64) + wv) * (R == 2 ? 1 : 64 >> k) + grp) * C;  // the lane's first column
    double vr[R][C], vi[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            vr[r][c] = (yl | r << 6) == x0 + c ? 1.0 : 0.0;
            vi[r][c] = 0.0;
        }
    for (int g0 = 0; g0 < op.n_gates; g0 += kBuildGateChunk) {
        const int ng = min(kBuildGateChunk, op.n_gates - g0);
        if (g0) __syncthreads();  // the previous chunk has been read
        if ((int)threadIdx.x < ng) {
            const int t = (int)threadIdx.x;
            BuildGate bg = tail.gate;
            if (!tail.one) bg = gates[op.gate0 + g0 + t];
            L.op[t] = bg.kind == G_CZ ? 0 : (bg.kind == G_DENSE ? 3 : (gate_is_diagonal(bg.kind) ? 1 : 2));
            L.nq[t] = bg.nq;
            L.off[t] = bg.dense_off;
#pragma unroll
            for (int j = 0; j < 6; ++j) L.pos[t][j] = bg.pos[j];
            double m[8];
            gate2x2(bg.kind, bg.theta, m);  // zeros for CZ and dense gates
#pragma unroll
            for (int j = 0; j < 8; ++j) L.m[t][j] = m[j];
        }
        __syncthreads();
        // the next gate's record is read while the current one is applied
        int nop = L.op[0], np0 = L.pos[0][0], np1 = L.pos[0][1];
        double nm[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) nm[j] = L.m[0][j];
        for (int gi = 0; gi < ng; ++gi) {
            const int kind = __builtin_amdgcn_readfirstlane(nop);
            const int a = __builtin_amdgcn_readfirstlane(np0), b = __builtin_amdgcn_readfirstlane(np1);
            double m[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) m[j] = nm[j];
            const int ni = min(gi + 1, ng - 1);
            nop = L.op[ni];
            np0 = L.pos[ni][0];
            np1 = L.pos[ni][1];
#pragma unroll
            for (int j = 0; j < 8; ++j) nm[j] = L.m[ni][j];
            if (kind == 0) {
                const int mask = (1 << a) | (1 << b);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool neg = ((yl | r << 6) & mask) == mask;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        vr[r][c] = neg ? -vr[r][c] : vr[r][c];
                        vi[r][c] = neg ? -vi[r][c] : vi[r][c];
                    }
                }
            } else if (kind == 1) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (((yl | r << 6) >> a) & 1) {
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const double x = vr[r][c], y = vi[r][c];
                            vr[r][c] = m[6] * x - m[7] * y;
                            vi[r][c] = m[6] * y + m[7] * x;
                        }
                    }
            } else if (kind == 2) {
                if (R == 2 && a == 6) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const double ar = vr[0][c], ai = vi[0][c], br = vr[R - 1][c], bi = vi[R - 1][c];
                        vr[0][c] = (m[0] * ar - m[1] * ai) + (m[2] * br - m[3] * bi);
                        vi[0][c] = (m[0] * ai + m[1] * ar) + (m[2] * bi + m[3] * br);
                        vr[R - 1][c] = (m[4] * ar - m[5] * ai) + (m[6] * br - m[7] * bi);
                        vi[R - 1][c] = (m[4] * ai + m[5] * ar) + (m[6] * bi + m[7] * br);
                    }
                } else {
                    // own and partner coefficients: this row's of the 2x2
                    const bool hi = (yl >> a) & 1;
                    const double sr = hi ? m[6] : m[0], si = hi ? m[7] : m[1];
                    const double pr = hi ? m[4] : m[2], pi = hi ? m[5] : m[3];
                    auto mix = [&](auto BIT) {
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const double x = vr[r][c], y = vi[r][c];
                                const double u = lane_xor<decltype(BIT)::value>(x), w = lane_xor<decltype(BIT)::value>(y);
                                vr[r][c] = (sr * x - si * y) + (pr * u - pi * w);
                                vi[r][c] = (sr * y + si * x) + (pr * w + pi * u);
                            }
                    };
                    switch (a) {
                        case 0: mix(std::integral_constant<int, 0>()); break;
                        case 1: mix(std::integral_constant<int, 1>()); break;
                        case 2: mix(std::integral_constant<int, 2>()); break;
                        case 3: mix(std::integral_constant<int, 3>()); break;
                        case 4: mix(std::integral_constant<int, 4>()); break;
                        default: mix(std::integral_constant<int, 5>()); break;
                    }
                }
            } else {
                // dense: bit j of the gate's index is row bit pos[j]
                const int dq = __builtin_amdgcn_readfirstlane(L.nq[gi]), dd = 1 << dq;
                const double2* u = reinterpret_cast<const double2*>(dense + __builtin_amdgcn_readfirstlane(L.off[gi]));
                int pm = 0;
                for (int j = 0; j < dq; ++j) pm |= 1 << __builtin_amdgcn_readfirstlane(L.pos[gi][j]);
                auto ext = [&](int y) {  // the gate's index of row y
                    int o = 0;
                    for (int j = 0; j < dq; ++j) o |= ((y >> __builtin_amdgcn_readfirstlane(L.pos[gi][j])) & 1) << j;
                    return o;
                };
                auto dep = [&](int xl) {
                    int o = 0;
                    for (int j = 0; j < dq; ++j) o |= ((xl >> j) & 1) << __builtin_amdgcn_readfirstlane(L.pos[gi][j]);
                    return o;
                };
                if (g0 == 0 && gi == 0) {  // on the basis vectors: the gate's own entries
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int y = yl | r << 6;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const int x = x0 + c;
                            double2 e = make_double2(0.0, 0.0);
                            if (x < D && ((x ^ y) & ~pm) == 0) e = u[ext(y) * dd + ext(x)];
                            vr[r][c] = e.x;
                            vi[r][c] = e.y;
                        }
                    }
                } else {
                    // every lane reads the inputs of its row from LDS, the same
                    // address for all rows that agree outside the gate
                    double2* V = L.v[wv];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) V[(lane | r << 6) * C + c] = make_double2(vr[r][c], vi[r][c]);
                    __syncthreads();
                    const double2* row[R];
                    int src[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        row[r] = u + ext(yl | r << 6) * dd;
                        src[r] = (lane | r << 6) & ~pm;
#pragma unroll
                        for (int c = 0; c < C; ++c) vr[r][c] = vi[r][c] = 0.0;
                    }
#pragma unroll 4
                    for (int xl = 0; xl < dd; ++xl) {
                        const int o = dep(xl);
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const double2 e = row[r][xl];
                            const double2* in = V + (src[r] | o) * C;
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const double2 z = in[c];
                                vr[r][c] += e.x * z.x - e.y * z.y;
                                vi[r][c] += e.x * z.y + e.y * z.x;
                            }
                        }
                    }
                    __syncthreads();  // a following dense gate rewrites the inputs
                }
            }
        }
    }
    if (x0 >= D) return;  // columns beyond the matrix (k < 5); x0 + C <= D otherwise, or D < C
    const int h = 1 << (k - 1), jm = h - 1;
    if (op.layout == LAYOUT_PLAIN) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (x0 + c >= D) continue;  // k = 1: two columns
                const int at = (yl | r << 6) * D + x0 + c;
                if (op.is_double)
                    reinterpret_cast<double2*>(out)[at] = make_double2(vr[r][c], vi[r][c]);
                else
                    reinterpret_cast<float2*>(out)[at] = make_float2((float)vr[r][c], (float)vi[r][c]);
            }
    } else if (op.layout == LAYOUT_SPLIT7) {
        // k = 7: fp16 halves of 16 Re M and 16 Im M for v_mfma_f32_32x32x16_f16
        // (k_cluster_f32_split7). Entry (rb, s, lane l, i) of each part:
        // physical row rho = l % 32 of row block rb is amplitude
        // (16 rb + 4 (rho / 8) + rho % 4) | ((rho / 4) % 2) << 6; inner element
        // i of the lanes with l / 32 = hin is amplitude (8 s + i) | hin << 6.
        // The lane's columns are four neighbouring i.
        if constexpr (R == 2) {
            typedef _Float16 half4v __attribute__((ext_vector_type(4)));
            constexpr int S7 = 8, NP7 = 4 * S7 * 64 * 8;  // halves per part
            _Float16* A = reinterpret_cast<_Float16*>(out);
            const int s = (x0 & 63) >> 3, i = x0 & 7, hin = x0 >> 6;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int rb = lane >> 4, q = lane & 15, rho = ((q >> 2) << 3) | (r << 2) | (q & 3);
                half4v p[4];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float fr = (float)(16.0 * vr[r][c]), fi = (float)(16.0 * vi[r][c]);
                    p[0][c] = (_Float16)fr;
                    p[1][c] = (_Float16)(fr - (float)p[0][c]);
                    p[2][c] = (_Float16)fi;
                    p[3][c] = (_Float16)(fi - (float)p[2][c]);
                }
                const int at = ((rb * S7 + s) * 64 + (rho | hin << 5)) * 8 + i;
#pragma unroll
                for (int w = 0; w < 4; ++w) *reinterpret_cast<half4v*>(A + w * NP7 + at) = p[w];
            }
            // the kernel's tile counters
            if (part == 0 && threadIdx.x < 256) reinterpret_cast<uint32_t*>(out + kTicketOff7)[threadIdx.x] = 0u;
        }
    } else if (op.layout == LAYOUT_SPLIT16F) {
        // k = 5 or 6, fp16 halves of 16 x the real-split matrix for
        // v_mfma_f32_32x32x16_f16: RB = 2^(k-4) row blocks, S = 2^(k-3) steps
        // of 16 inner indices. Entry (rb, s, lane l, i): physical row rho =
        // l % 32 of row block rb (result rows as in LAYOUT_MFMA32F), inner index
        // float 8 s + i of the lanes with l / 32 = hin, i.e. component i % 2 of
        // amplitude (4 s + i / 2) | hin << (k - 1). hi block, then lo block.
        // The lane's four columns are the eight i of one entry.
        typedef _Float16 half8v __attribute__((ext_vector_type(8)));
        const int RB = 1 << (k - 4), S = 1 << (k - 3);
        const int y = yl, hout = y >> (k - 1), j = y & jm, rb = j >> 3;
        const int rho0 = (((j >> 1) & 3) << 3) | (hout << 2) | ((j & 1) << 1);
        const int hin = x0 >> (k - 1), s = (x0 & jm) >> 2;
        half8v* Ahi = reinterpret_cast<half8v*>(out);
        half8v* Alo = Ahi + RB * S * 64;
#pragma unroll
        for (int a = 0; a < 2; ++a) {  // row [Re, -Im] or [Im, Re] of the entry
            half8v hi, lo;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const float f = (float)(16.0 * (a == b ? vr[0][c] : (a == 0 ? -vi[0][c] : vi[0][c])));
                    hi[2 * c + b] = (_Float16)f;
                    lo[2 * c + b] = (_Float16)(f - (float)hi[2 * c + b]);
                }
            const int at = (rb * S + s) * 64 + (rho0 | a | hin << 5);
            Ahi[at] = hi;
            Alo[at] = lo;
        }
    } else if (op.layout == LAYOUT_MFMA32F) {
        // entry (rb, s, lane l): physical row rho = l % 32 of row block rb is
        // component rho % 2 of amplitude (8 rb + 2 (rho / 8) + (rho / 2) % 2) |
        // ((rho / 4) % 2) << (k - 1); inner index s of the lanes with l / 32 =
        // hin is component s % 2 of amplitude (s / 2) | hin << (k - 1)
        const int S = D, y = yl, hout = y >> (k - 1), j = y & jm, rb = j >> 3;
        const int rho0 = (((j >> 1) & 3) << 3) | (hout << 2) | ((j & 1) << 1);
        float* A = reinterpret_cast<float*>(out);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int x = x0 + c, hin = x >> (k - 1), s = 2 * (x & jm);
            float* e = A + (rb * S + s) * 64 + (rho0 | hin << 5);
            e[0] = (float)vr[0][c];
            e[64] = (float)-vi[0][c];
            e[1] = (float)vi[0][c];
            e[65] = (float)vr[0][c];
        }
    } else if (op.layout == LAYOUT_GAUSS32F) {
        // k = 6: three 64 x 64 real matrices P = 0: Re M, 1: Im M, 2: Re M + Im M,
        // for v_mfma_f32_16x16x4_f32. Entry (P, rb, s, lane l): physical row
        // i = l % 16 of row block rb, inner index s | (l / 16) << 4. The result
        // of physical row i lands in register i % 4 of the lanes with l / 16 =
        // i / 4, which own amplitude (4 rb + i % 4) | (i / 4) << 4.
        const int i = (yl & 3) | ((yl >> 4) << 2), rb = (yl >> 2) & 3;
        float* A = reinterpret_cast<float*>(out);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int x = x0 + c, s = x & 15, l = i | ((x >> 4) << 4);
            A[((0 * 4 + rb) * 16 + s) * 64 + l] = (float)vr[0][c];
            A[((1 * 4 + rb) * 16 + s) * 64 + l] = (float)vi[0][c];
            A[((2 * 4 + rb) * 16 + s) * 64 + l] = (float)(vr[0][c] + vi[0][c]);
        }
    } else {  // LAYOUT_MFMA16D
        // entry (rb, s, lane l): physical row rho = l % 16 of row block rb, inner
        // index 4 s + l / 16: component (rho / 4) % 2 of amplitude
        // (2 rb + rho / 8) | (rho % 4) << (k - 2) (result row rho lands in register
        // rho / 4 of the lanes with l / 16 = rho % 4), and component s % 2 of
        // amplitude (s / 2) | (l / 16) << (k - 2)
        const int S = 2 * D / 4, qm = (1 << (k - 2)) - 1;
        const int y = yl, qout = y >> (k - 2), j = y & qm, rb = j >> 1;
        double* A = reinterpret_cast<double*>(out);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int x = x0 + c, qin = x >> (k - 2), s = 2 * (x & qm);
            const int rho = ((j & 1) << 3) | qout;  // component 0 of the row; component 1: rho | 4
            double* e = A + (rb * S + s) * 64 + (rho | qin << 4);
            e[0] = vr[0][c];
            e[64] = -vi[0][c];
            e[4] = vi[0][c];
            e[68] = vr[0][c];
        }
    }
}

// With a tail (see BuildTail), ops, gates and dense lie in pinned host memory:
// a work-group reads its gates into LDS in one round and a dense gate's
// entries once each, so they come over the link as fast as a copy would bring
// them, without the copy's launch and the host's wait for it. The launch itself
// takes longer (11 matrices of a 20-qubit circuit 17.8 us instead of 16.3, one
// dense 3-qubit gate 4.5 instead of 3.9); the 20-qubit depth-25 circuit went
// from 343 to 293 us with its sums also written to pinned memory, the 12-qubit
// one of depth 16 from 124 to 87. The work-groups
// behind the last matrix copy the tail; each one stores its flag when its
// reads have been consumed.
__global__ __launch_bounds__(kBuildThreads) void k_build(const BuildOp* __restrict__ ops, int n_ops,
                                                         const BuildGate* __restrict__ gates,
                                                         const double* __restrict__ dense, char* __restrict__ mat_base,
                                                         BuildTail tail) {
    __shared__ BuildLds L;
    const int part = (int)blockIdx.y;
    if ((int)blockIdx.x < n_ops) {
        BuildOp op = tail.op;
        if (!tail.one) op = ops[blockIdx.x];
        char* out = mat_base + op.out_off;
        if (part < build_parts(op.k)) {  // the grid is sized for the widest matrix
            if (op.k == 7)
                build_matrix<2>(op, part, gates, tail, dense, out, L);
            else
                build_matrix<1>(op, part, gates, tail, dense, out, L);
        }
    } else {
        const uint4* src = reinterpret_cast<const uint4*>(tail.src);
        uint4* dst = reinterpret_cast<uint4*>(tail.dst);
        for (size_t i = (size_t)part * kBuildThreads + threadIdx.x; i < tail.bytes / 16;
             i += (size_t)gridDim.y * kBuildThreads)
            dst[i] = src[i];
    }
    if (tail.flags) {
        __builtin_amdgcn_s_waitcnt(0);  // this wave's reads, also those nothing used
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(tail.flags + blockIdx.y * gridDim.x + blockIdx.x, tail.seq, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ------------------------------------------------------------ float64 reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Block reduction of up to 8 values; slot i is summed unless bit i of maxmask is set.
__device__ void block_reduce_store(double (&vals)[8], int nv, unsigned maxmask, double* out) {
    __shared__ double sh[4][8];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = 0; i < nv; ++i) vals[i] = ((maxmask >> i) & 1) ? wave_max(vals[i]) : wave_sum(vals[i]);
    if (lane == 0)
        for (int i = 0; i < nv; ++i) sh[w][i] = vals[i];
    __syncthreads();
    if (threadIdx.x < nv) {
        const int i = threadIdx.x;
        double r = sh[0][i];
        for (int ww = 1; ww < 4; ++ww) r = ((maxmask >> i) & 1) ? fmax(r, sh[ww][i]) : r + sh[ww][i];
        out[i] = r;
    }
}

// The streaming reductions are bound by HBM. A work-group takes runs of U * 256
// consecutive units (W amplitudes: 16 bytes a lane, where the pointers are so
// aligned) and issues all of a run's loads before any arithmetic: a run is one
// stretch of pages and channels, where a grid-wide stride between a lane's
// loads touched U windows 4 MiB apart. Beyond the caches the accesses are
// non-temporal. At 27 qubits, fp32: k_stats with probabilities 318 -> 275 us
// (5.9 TB/s), k_compare 440 -> 306 us (7.0 TB/s).
template <typename T, int W>
struct AmpUnit {
    typedef T type __attribute__((ext_vector_type(2 * W)));
};
template <typename P, int W>
struct ProbUnit {
    typedef P type __attribute__((ext_vector_type(W)));
};
template <typename P>
struct ProbUnit<P, 1> {
    typedef P type;
};

template <typename T, typename P, int W, int U, bool NT>
__global__ __launch_bounds__(256) void k_stats(const void* __restrict__ psi, uint64_t units, void* __restrict__ probs,
                                               double* __restrict__ part) {
    using V = typename AmpUnit<T, W>::type;
    using Q = typename ProbUnit<P, W>::type;
    const V* in = reinterpret_cast<const V*>(psi);
    Q* out = reinterpret_cast<Q*>(probs);
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    auto acc = [&](const V& a, uint64_t i) {
        Q q;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const T x = a[2 * w], y = a[2 * w + 1];
            const double pr = (double)x * (double)x + (double)y * (double)y;
            if constexpr (sizeof(T) == 4) {
                stats_acc_f(v, x, y);
            } else {
                v[0] += pr;
                v[1] += pr * pr;
                if (pr > 0.0) v[2] -= pr * log(pr);
            }
            if constexpr (W == 1)
                q = (P)pr;
            else
                q[w] = (P)pr;
        }
        if (out) store16<NT>(out + i, q);
    };
    const uint64_t step = (uint64_t)gridDim.x * U * 256;
    for (uint64_t i0 = (uint64_t)blockIdx.x * U * 256 + threadIdx.x; i0 < units; i0 += step) {
        V a[U];  // units is a multiple of U * 256, or U is 1
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = load16<NT>(in + i0 + u * 256);
#pragma unroll
        for (int u = 0; u < U; ++u) acc(a[u], i0 + u * 256);
    }
    block_reduce_store(v, 3, 0u, part + blockIdx.x * 8);
}

template <typename T, typename R, int W, int U, bool NT>
__global__ __launch_bounds__(256) void k_compare(const void* __restrict__ psi, const void* __restrict__ ref,
                                                 uint64_t units, double* __restrict__ part) {
    using V = typename AmpUnit<T, W>::type;
    using X = typename AmpUnit<R, W>::type;
    const V* pa = reinterpret_cast<const V*>(psi);
    const X* pr = reinterpret_cast<const X*>(ref);
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const uint64_t step = (uint64_t)gridDim.x * U * 256;
    for (uint64_t i0 = (uint64_t)blockIdx.x * U * 256 + threadIdx.x; i0 < units; i0 += step) {
        V a[U];
        X r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = load16<NT>(pa + i0 + u * 256);
            r[u] = load16<NT>(pr + i0 + u * 256);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const double ar = a[u][2 * w], ai = a[u][2 * w + 1], rr = r[u][2 * w], ri = r[u][2 * w + 1];
                v[0] += rr * ar + ri * ai;  // Re <ref|psi>
                v[1] += rr * ai - ri * ar;  // Im <ref|psi>
                v[2] += rr * rr + ri * ri;
                v[3] += ar * ar + ai * ai;
                const double dr = ar - rr, di = ai - ri;
                v[4] = fmax(v[4], dr * dr + di * di);
            }
    }
    v[4] = sqrt(v[4]);  // the root is monotone: the same value as the largest root
    block_reduce_store(v, 5, 1u << 4, part + blockIdx.x * 8);
}

// Sum (or max) the per-block partials in a fixed order: deterministic. One
// work-group, bound by latency: eight rows of partials a thread in flight.
template <int NV, unsigned MAXMASK>
__global__ __launch_bounds__(256) void k_reduce_final(const double* __restrict__ part, int nblocks,
                                                      double* __restrict__ res) {
    constexpr int R = kReduceBlocks / 256;
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b0 = threadIdx.x; b0 < nblocks; b0 += R * 256) {
        double x[R][NV];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int b = b0 + 256 * r;
#pragma unroll
            for (int i = 0; i < NV; ++i) x[r][i] = b < nblocks ? part[b * 8 + i] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = ((MAXMASK >> i) & 1) ? fmax(v[i], x[r][i]) : v[i] + x[r][i];
    }
    block_reduce_store(v, NV, MAXMASK, res);
}

// ------------------------------------------------------------ launchers
namespace {
inline unsigned grid_for(uint64_t work, unsigned per_block, unsigned cap) {
    const uint64_t b = (work + per_block - 1) / per_block;
    return (unsigned)(b < 1 ? 1 : (b > cap ? cap : b));
}
// Work-groups of four one-tile waves.
inline unsigned tile_grid(uint64_t tiles) { return (unsigned)((tiles + 3) / 4); }
// Does every access instruction of a direct kernel cover whole 128-byte lines?
// Its rows from target `first` up are separate instructions, the rest of the
// tile is on the lanes, so no such target may be among the line's `bits` bits.
inline bool whole_lines(const ClusterGeom& g, int first, int bits) { return g.t[first] >= bits; }
constexpr unsigned kStreamGrid = 8192;  // blocks of 256 threads for grid-stride streaming kernels
// Streaming reductions: runs of rounds from this many work-groups up, single
// rounds below (one fp32 call at 20 qubits, 256 work-groups of runs or 2048 of
// single rounds: 27.7 or 31.0 us; at 18 qubits, 64 or 512: 27.0 both ways).
constexpr unsigned kDeepBlocks = 64;
constexpr unsigned kPersistGrid = 2048; // work-groups of the persistent cluster kernels
constexpr unsigned kPairGrid = 256;     // one 12-wave work-group per compute unit (LDS-limited)
constexpr unsigned kStagedGrid = 256;   // one 8-wave work-group per compute unit (LDS-limited)
constexpr unsigned kSplit7Grid = 256;   // one 4-wave work-group per compute unit (LDS-limited)
}  // namespace

hipError_t launch_init(void* psi, int n, bool dbl, int mode, hipStream_t st) {
    const uint64_t cnt = uint64_t(1) << n;
    const unsigned grid = grid_for(cnt, 256, kStreamGrid);
    const double val = std::ldexp(1.0, -n) > 0 ? std::sqrt(std::ldexp(1.0, -n)) : 0.0;
    if (dbl)
        hipLaunchKernelGGL(k_init<double>, dim3(grid), dim3(256), 0, st, (double2*)psi, cnt, mode, val);
    else
        hipLaunchKernelGGL(k_init<float>, dim3(grid), dim3(256), 0, st, (float2*)psi, cnt, mode, (float)val);
    return hipGetLastError();
}

// Tile of 11 bits holding the targets of every cluster (their union plus the
// lowest other bits); sg[j] gets the tile bits and cluster j's positions.
constexpr bool kMultiSwz = true;

static void make_multi_geom(int n, int m, const int32_t (*t)[5], StageGeom* sg, int nt_want = 11) {
    uint64_t tile = 0;
    for (int j = 0; j < m; ++j)
        for (int q = 0; q < 5; ++q) tile |= uint64_t(1) << t[j][q];
    for (int b = 0; b < n && __builtin_popcountll(tile) < nt_want; ++b) tile |= uint64_t(1) << b;
    int tb[16], nt = 0;
    for (int b = 0; b < n; ++b)
        if (tile >> b & 1) tb[nt++] = b;
    for (int j = 0; j < m; ++j) {
        StageGeom& g = sg[j];
        std::memset(&g, 0, sizeof(g));
        g.nt = nt;
        for (int r = 0; r < nt; ++r) g.tb[r] = tb[r];
        int nc = 0;
        for (int r = 0; r < nt; ++r) {
            bool is_t = false;
            for (int q = 0; q < 5; ++q)
                if (tb[r] == t[j][q]) {
                    g.tpos[q] = r;
                    is_t = true;
                }
            if (!is_t) g.cpos[nc++] = r;
        }
        for (int i = 0; i < 16; ++i) {
            const uint64_t tau = uint64_t(i) << 7;
            uint64_t off = 0;
            for (int r = 0; r < nt; ++r)
                if (tau >> r & 1) off |= uint64_t(1) << tb[r];
            g.ioff[i] = off;
        }
    }
}

hipError_t launch_multi(void* psi, int n, int m, const int32_t (*targets)[5], const void* const* mats,
                        const EpiDesc* const* epis, hipStream_t st) {
    if (m < 1 || m > 2 || n < 11) return hipErrorInvalidValue;
    MultiArgs a;
    std::memset(&a, 0, sizeof(a));
    make_multi_geom(n, m, targets, a.sg);
    if (a.sg[0].nt != 11) return hipErrorInvalidValue;
    for (int j = 0; j < m; ++j) {
        a.A[j] = reinterpret_cast<const half8*>(mats[j]);
        a.epi[j] = epis[j];
        a.lowt[j] = a.sg[j].tpos[0] == 0;
    }
    const uint64_t ntiles = uint64_t(1) << (n - 11);
    MultiArgs a10 = a;
    if (m == 2 && g_pair_tile == 10) make_multi_geom(n, m, targets, a10.sg, 10);
    // the 10-bit tile needs state bit 0 (16-byte accesses of amplitude pairs)
    if (m == 2 && g_pair_tile == 10 && a10.sg[0].nt == 10 && a10.sg[0].tb[0] == 0) {
        const uint64_t nt10 = uint64_t(1) << (n - 10);
        const unsigned grid = grid_for(nt10, 12, kPairGrid);
        hipLaunchKernelGGL((k_cluster_f32_pair10<12>), dim3(grid), dim3(768), 0, st, (float2*)psi, a10, nt10);
    } else if (m == 2) {
        const unsigned grid = grid_for(ntiles, 8, kPersistGrid / 2);
        hipLaunchKernelGGL((k_cluster_f32_multi<2, 8, kMultiSwz>), dim3(grid), dim3(512), 0, st, (float2*)psi, a,
                           ntiles);
    } else {
        const unsigned grid = grid_for(ntiles, 4, kPersistGrid);
        hipLaunchKernelGGL((k_cluster_f32_multi<1, 4, kMultiSwz>), dim3(grid), dim3(256), 0, st, (float2*)psi, a,
                           ntiles);
    }
    return hipGetLastError();
}

hipError_t launch_fold2(void* psi, const ClusterGeom& g2, const void* mat2, const EpiDesc* epi2, const EpiDesc* epi1,
                        const ClusterGeom& g1, const void* mat1, int omask, int rmask, void* table,
                        hipStream_t st) {
    if (g2.k < 6 || g2.k > 7 || g2.n < 12 - (7 - g2.k) || g1.k < 1 || g1.k > g2.k) return hipErrorInvalidValue;
    if (g2.k == 7 && omask < 0) return hipErrorInvalidValue;  // a 7-qubit second cluster: the table form only
    Fold2Args f;
    std::memset(&f, 0, sizeof(f));
    f.M1 = reinterpret_cast<const double2*>(mat1);
    f.amp = std::sqrt(std::ldexp(1.0, -g2.n));
    f.k1 = g1.k;
    for (int m = 0; m < g1.k; ++m) f.t1[m] = g1.t[m];
    const StageGeom sg = make_stage_geom(g2, 5, 7);
    const uint64_t tiles = g2.ncols >> 5;
    const unsigned grid = grid_for(tiles, 8, kStagedGrid);
    if (omask >= 0) {
        const int no = __builtin_popcount((unsigned)omask), nr = __builtin_popcount((unsigned)rmask);
        const int rmax = g2.k == 7 ? kFoldTab7Rows : kFoldTabRows, mmax = (1 << g2.k) - 1;
        if (table == nullptr || omask > mmax || rmask < 0 || rmask > mmax || no > 2 || (1 << (no + nr)) > rmax)
            return hipErrorInvalidValue;
        FoldTabArgs a;
        a.M2 = reinterpret_cast<const double2*>(mat2);
        a.omask = omask;
        a.rmask = rmask;
        if (g2.k == 7) {
            hipLaunchKernelGGL(k_fold2_table<7>, dim3(1u << (no + nr)), dim3(128), 0, st, (float2*)table, a);
            const unsigned grid7 = grid_for(g2.ncols / 32, 8, kSplit7Grid);
            hipLaunchKernelGGL(k_fold2t7_f32, dim3(grid7), dim3(512), 0, st, (float2*)psi, (const float2*)table, epi2,
                               epi1, g2, f, a, sg);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(k_fold2_table<6>, dim3(1u << (no + nr)), dim3(64), 0, st, (float2*)table, a);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, st, (float2*)psi, (const float2*)table, epi2, epi1, sg,
                               f, a, tiles);
        };
        g2.t[0] == 0 ? go(k_fold2t_f32<true>) : go(k_fold2t_f32<false>);
        return hipGetLastError();
    }
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, st, (float2*)psi, (const half8*)mat2, epi2, epi1, sg, f,
                           tiles);
    };
    g2.t[0] == 0 ? go(k_fold2_f32<true>) : go(k_fold2_f32<false>);
    return hipGetLastError();
}

hipError_t launch_init_cluster(void* psi, bool dbl, const ClusterGeom& g, const void* mat, const EpiDesc* epi,
                               hipStream_t st) {
    const unsigned grid = grid_for(g.ncols, 256, kStreamGrid);
    const double amp = std::sqrt(std::ldexp(1.0, -g.n));
    auto go = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if (dbl)
            hipLaunchKernelGGL((k_init_cluster<double, K>), dim3(grid), dim3(256), 0, st, (double2*)psi, g,
                               (const double2*)mat, epi, amp);
        else
            hipLaunchKernelGGL((k_init_cluster<float, K>), dim3(grid), dim3(256), 0, st, (float2*)psi, g,
                               (const double2*)mat, epi, amp);
    };
    switch (g.k) {
        case 1: go(std::integral_constant<int, 1>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        case 3: go(std::integral_constant<int, 3>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        case 5: go(std::integral_constant<int, 5>()); break;
        case 6: go(std::integral_constant<int, 6>()); break;
        case 7: go(std::integral_constant<int, 7>()); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_build(const BuildOp* ops, int n_ops, int kmax, const BuildGate* gates, const double* dense,
                        char* mat_base, const BuildTail& tail, int* groups, hipStream_t st) {
    const int nx = n_ops + (tail.bytes > 0), ny = build_parts(kmax);
    *groups = nx * ny;
    if (nx <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_build, dim3(nx, ny), dim3(kBuildThreads), 0, st, ops, n_ops, gates, dense, mat_base, tail);
    return hipGetLastError();
}

// Tile geometry of the staged kernels: the C lowest non-target bits are the
// columns; chunk i of the linear order starts at tau = i << unit.
StageGeom make_stage_geom(const ClusterGeom& g, int C, int unit) {
    StageGeom sg;
    std::memset(&sg, 0, sizeof(sg));
    uint64_t tmask = 0;
    for (int m = 0; m < g.k; ++m) tmask |= uint64_t(1) << g.t[m];
    int cols[16], nc = 0;
    for (int b = 0; b < g.n && nc < C; ++b)
        if (!(tmask >> b & 1)) cols[nc++] = b;
    uint64_t tilemask = tmask;
    for (int b = 0; b < nc; ++b) tilemask |= uint64_t(1) << cols[b];
    sg.nt = 0;
    for (int b = 0; b < g.n; ++b)
        if (tilemask >> b & 1) sg.tb[sg.nt++] = b;
    for (int r = 0; r < sg.nt; ++r) {
        for (int m = 0; m < g.k; ++m) if (sg.tb[r] == g.t[m]) sg.tpos[m] = r;
        for (int c = 0; c < nc; ++c) if (sg.tb[r] == cols[c]) sg.cpos[c] = r;
    }
    // LDS slots of the 6-qubit staged loop (11-bit tiles, half a tile per
    // wave): each column bit above tau bit 4 folds, by XOR, into a slot bit
    // among 1..4 that no lower column bit holds, so the 32 columns of an
    // 8-byte read have distinct slot bits 0..4 (no bank conflicts counted)
    // whatever bits the targets take; with target 0 on tau bit 0 (16-byte
    // reads) it is faster than a fixed fold as well, although conflicts are
    // still counted there. Bit 0 is never folded: it pairs amplitudes for
    // 16-byte accesses. The map is a bijection and linear over XOR.
    if (g.k == 6 && C == 5) {
        const bool lowt = g.t[0] == 0;
        int used = 1;
        for (int c = 0; c < nc; ++c)
            if (sg.cpos[c] < 5) used |= 1 << sg.cpos[c];
        for (int c = 0; c < (lowt ? 4 : 5) && c < nc; ++c) {
            if (sg.cpos[c] < 5) continue;
            int t = 1;
            while (t < 5 && ((used >> t) & 1)) ++t;
            if (t == 5) break;
            sg.swz[sg.cpos[c] - 5] = 1 << t;
            used |= 1 << t;
        }
    }
    const int chunks = 1 << (sg.nt - unit);
    for (int i = 0; i < chunks && i < 32; ++i) {
        const uint64_t tau = uint64_t(i) << unit;
        uint64_t off = 0;
        for (int r = 0; r < sg.nt; ++r)
            if (tau >> r & 1) off |= uint64_t(1) << sg.tb[r];
        sg.ioff[i] = off;
    }
    return sg;
}

int cluster_layout(bool dbl, int k, int n) {
    if (k == 7) return (!dbl && k <= max_cluster_k(dbl, n)) ? LAYOUT_SPLIT7 : -1;  // no other 7-qubit kernel
    if (!dbl) {
        if (k == 6) {
            if (n - k < 5) return LAYOUT_PLAIN;
            return g_k6_kernel == 2 ? LAYOUT_SPLIT16F : (g_k6_kernel == 1 ? LAYOUT_GAUSS32F : LAYOUT_MFMA32F);
        }
        // 4 and 5 qubits: the fp32 matrix cores at every size. The 6-qubit fp16-halves
        // kernel, the cluster padded with identity qubits, took 3.03 against 3.49 ms
        // for 5 qubits at 30 (24 qubits: 52 against 65-73 us), but a matrix entry above
        // 4094 overflows its halves, a matrix scaled by 1e-6 comes out wrong by 9e-3,
        // and columns that differ in a padding qubit share one scale.
        return (k >= 4 && n - k >= 6) ? LAYOUT_MFMA32F : LAYOUT_PLAIN;
    }
    const int nb = (k == 6) ? 1 : 2;
    return (k >= 3 && n - k >= 4 + (nb == 2)) ? LAYOUT_MFMA16D : LAYOUT_PLAIN;
}

namespace {
template <int K>
hipError_t launch_valu_k(void* psi, bool dbl, const ClusterGeom& g, const void* mat, const EpiDesc* epi,
                         hipStream_t st, double* stats_part = nullptr, unsigned* stats_blocks = nullptr) {
    if constexpr (K <= 3) {
        if (!stats_part && beyond_caches(g.n, dbl)) {
            const int tb = dbl ? 9 : 10;  // 8 KiB wave tiles
            const StageGeom sg = make_stage_geom(g, tb - K, dbl ? 6 : 7);
            const uint64_t tiles = uint64_t(1) << (g.n - tb);
            auto go = [&](auto kern, auto* p) {
                hipLaunchKernelGGL(kern, dim3(tile_grid(tiles)), dim3(256), 0, st, p, (decltype(p))mat, epi, sg,
                                   tiles, nullptr);
            };
            dbl ? go(k_cluster_valu_staged<double, K>, (double2*)psi)
                : go(k_cluster_valu_staged<float, K>, (float2*)psi);
            return hipGetLastError();
        }
    }
    if (K >= 2 && K <= 3 && g.n - K >= 6) {
        constexpr int KS = K >= 2 && K <= 3 ? K : 2;
        const StageGeom sg = make_stage_geom(g, 6, 6);  // tile: the targets and 6 column bits
        for (int i = 0; i < 6; ++i)
            if (sg.tb[i] != i) return hipErrorInvalidValue;  // cannot happen: bits 0..5 are tile bits
        const uint64_t tiles = g.ncols >> 6;
        if (stats_part) {  // float (checked by the caller); the partials area holds kReduceBlocks work-groups
            if (dbl) return hipErrorInvalidValue;
            const unsigned grid = grid_for(tiles, 4, kReduceBlocks);
            *stats_blocks = grid;
            hipLaunchKernelGGL((k_cluster_valu_staged<float, KS, true>), dim3(grid), dim3(256), 0, st,
                               (float2*)psi, (const float2*)mat, epi, sg, tiles, stats_part);
            return hipGetLastError();
        }
        const unsigned grid = grid_for(tiles, 4, kStreamGrid);
        if (dbl)
            hipLaunchKernelGGL((k_cluster_valu_cached<double, KS>), dim3(grid), dim3(256), 0, st, (double2*)psi,
                               (const double2*)mat, epi, sg, tiles);
        else
            hipLaunchKernelGGL((k_cluster_valu_cached<float, KS>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float2*)mat, epi, sg, tiles);
        return hipGetLastError();
    }
    if (stats_part) return hipErrorInvalidValue;  // no sums in the plain form
    const unsigned grid = grid_for(g.ncols, 256, kStreamGrid);
    if (dbl)
        hipLaunchKernelGGL((k_cluster_valu<double, K>), dim3(grid), dim3(256), 0, st, (double2*)psi,
                           (const double2*)mat, epi, g);
    else
        hipLaunchKernelGGL((k_cluster_valu<float, K>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                           (const float2*)mat, epi, g);
    return hipGetLastError();
}

template <int K>
hipError_t launch_mfma32_k(void* psi, const ClusterGeom& g, const void* mat, const EpiDesc* epi, int variant,
                           hipStream_t st, double* stats_part, unsigned* stats_blocks) {
    if (stats_part && variant == 1) return hipErrorInvalidValue;  // sums come from the direct kernel only
    if (K <= 5 && variant == 1) {
        constexpr int KS = K <= 5 ? K : 5;
        const StageGeom sg = make_stage_geom(g, 6, 7);
        const uint64_t tiles = g.ncols >> 6;
        const unsigned grid = grid_for(tiles, 4, kPersistGrid);
        if (g.t[0] == 0)
            hipLaunchKernelGGL((k_cluster_f32_stage<KS, 6, true>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float*)mat, epi, g, sg);
        else
            hipLaunchKernelGGL((k_cluster_f32_stage<KS, 6, false>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float*)mat, epi, g, sg);
        return hipGetLastError();
    }
    constexpr int NB = (K == 6) ? 1 : 2;
    const uint64_t tiles = g.ncols / (32 * NB);
    const unsigned grid = grid_for(tiles, 4, kPersistGrid);
    if (stats_part) {
        *stats_blocks = grid;
        if (g.t[0] == 0)
            hipLaunchKernelGGL((k_cluster_f32_mfma<K, NB, true, true>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float*)mat, epi, g, stats_part);
        else
            hipLaunchKernelGGL((k_cluster_f32_mfma<K, NB, false, true>), dim3(grid), dim3(256), 0, st,
                               (float2*)psi, (const float*)mat, epi, g, stats_part);
        return hipGetLastError();
    }
    if (g.t[0] == 0)
        hipLaunchKernelGGL((k_cluster_f32_mfma<K, NB, true>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                           (const float*)mat, epi, g, nullptr);
    else
        hipLaunchKernelGGL((k_cluster_f32_mfma<K, NB, false>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                           (const float*)mat, epi, g, nullptr);
    return hipGetLastError();
}

template <int K>
hipError_t launch_mfma64_k(void* psi, const ClusterGeom& g, const void* mat, const EpiDesc* epi, int variant,
                           hipStream_t st) {
    if (K <= 5 && variant == 1) {
        constexpr int KS = K <= 5 ? K : 5;
        constexpr int C = KS == 5 ? 4 : 5;
        const StageGeom sg = make_stage_geom(g, C, 6);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(tile_grid(g.ncols >> C)), dim3(256), 0, st, (vd2*)psi, (const double*)mat,
                               epi, g, sg);
        };
        beyond_caches(g.n, true) ? go(k_cluster_f64_stage<KS, C, true>) : go(k_cluster_f64_stage<KS, C, false>);
        return hipGetLastError();
    }
    if constexpr (K == 6) {
        const unsigned grid = grid_for(g.ncols / 16, 8, kPersistGrid);
        hipLaunchKernelGGL((k_cluster_f64_mfma_loop<6, 1, 512>), dim3(grid), dim3(512), 0, st, (double2*)psi,
                           (const double*)mat, epi, g);
    } else {
        constexpr int NB = K == 5 ? 1 : 2;
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(tile_grid(g.ncols / (16 * NB))), dim3(256), 0, st, (vd2*)psi,
                               (const double*)mat, epi, g);
        };
        beyond_caches(g.n, true) && whole_lines(g, 0, 3) ? go(k_cluster_f64_mfma<K, NB, true>)
                                                       : go(k_cluster_f64_mfma<K, NB, false>);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_cluster(void* psi, bool dbl, const ClusterGeom& g, const void* mat, int layout,
                          const EpiDesc* epi, int variant, hipStream_t st, double* stats_part,
                          unsigned* stats_blocks) {
    // the sums of the stored amplitudes come from the direct float matrix-core kernels only
    if (stats_part && (!cluster_stats_supported(dbl, g.n, g.k, layout, variant) || !stats_blocks))
        return hipErrorInvalidValue;
    if (layout == LAYOUT_PLAIN) {
        switch (g.k) {
            case 1: return launch_valu_k<1>(psi, dbl, g, mat, epi, st);
            case 2: return launch_valu_k<2>(psi, dbl, g, mat, epi, st, stats_part, stats_blocks);
            case 3: return launch_valu_k<3>(psi, dbl, g, mat, epi, st, stats_part, stats_blocks);
            case 4: return launch_valu_k<4>(psi, dbl, g, mat, epi, st);
            case 5: return launch_valu_k<5>(psi, dbl, g, mat, epi, st);
            case 6: return launch_valu_k<6>(psi, dbl, g, mat, epi, st);
            default: return hipErrorInvalidValue;
        }
    }
    if (layout == LAYOUT_SPLIT7 && !dbl && g.k == 7 && g.n >= 12) {
        const uint64_t tiles = g.ncols / 32;
        const unsigned grid = grid_for(tiles, 4, kSplit7Grid);
        // the tile counters behind the matrix, which its builder zeroes (a pass
        // over a state this large has a full grid and a multiple of 8 tiles). A
        // pass that takes the sums has none: which tiles a wave adds up would
        // depend on the order in which the waves ask, and so the sums' last bits.
        uint32_t* tickets = beyond_caches(g.n, false) && !stats_part
                                ? reinterpret_cast<uint32_t*>(static_cast<char*>(const_cast<void*>(mat)) + kTicketOff7)
                                : nullptr;
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, (float2*)psi, (const half8*)mat, epi, g, stats_part,
                               tickets);
        };
        if (stats_part) {
            *stats_blocks = grid;
            g.t[0] == 0 ? go(k_cluster_f32_split7<true, true>) : go(k_cluster_f32_split7<false, true>);
            return hipGetLastError();
        }
        const bool nt = beyond_caches(g.n, false) && whole_lines(g, 1, 4);
        if (g.t[0] == 0)
            nt ? go(k_cluster_f32_split7<true, false, true>) : go(k_cluster_f32_split7<true>);
        else
            nt ? go(k_cluster_f32_split7<false, false, true>) : go(k_cluster_f32_split7<false>);
        return hipGetLastError();
    }
    if (layout == LAYOUT_SPLIT16F && !dbl && g.k == 6 && variant == 1) {
        const StageGeom sg = make_stage_geom(g, 5, 7);  // 11 tile bits; chunks of 2^7 amplitudes
        const uint64_t tiles = g.ncols >> 5;
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(tile_grid(tiles)), dim3(256), 0, st, (float2*)psi, (const half8*)mat, epi,
                               sg, tiles);
        };
        const bool nt = beyond_caches(g.n, false);
        if (g.t[0] == 0)
            nt ? go(k_cluster_f32_split6s<true, true>) : go(k_cluster_f32_split6s<true, false>);
        else
            nt ? go(k_cluster_f32_split6s<false, true>) : go(k_cluster_f32_split6s<false, false>);
        return hipGetLastError();
    }
    if (layout == LAYOUT_SPLIT16F && !dbl && g.k == 6) {
        const uint64_t tiles = g.ncols / 32;
        const unsigned grid = grid_for(tiles, 4, kPersistGrid);
        if (stats_part) {
            *stats_blocks = grid;
            if (g.t[0] == 0)
                hipLaunchKernelGGL((k_cluster_f32_split6_sum<true>), dim3(grid), dim3(256), 0, st, (float2*)psi,
                                   (const half8*)mat, epi, g, stats_part);
            else
                hipLaunchKernelGGL((k_cluster_f32_split6_sum<false>), dim3(grid), dim3(256), 0, st,
                                   (float2*)psi, (const half8*)mat, epi, g, stats_part);
            return hipGetLastError();
        }
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(tile_grid(tiles)), dim3(256), 0, st, (float2*)psi, (const half8*)mat, epi, g);
        };
        const bool nt = beyond_caches(g.n, false) && whole_lines(g, 1, 4);
        if (g.t[0] == 0)
            nt ? go(k_cluster_f32_split6<true, true>) : go(k_cluster_f32_split6<true, false>);
        else
            nt ? go(k_cluster_f32_split6<false, true>) : go(k_cluster_f32_split6<false, false>);
        return hipGetLastError();
    }
    if (layout == LAYOUT_GAUSS32F && !dbl && g.k == 6) {
        const uint64_t tiles = g.ncols / 16;
        const unsigned grid = grid_for(tiles, 4, kPersistGrid);
        if (g.t[0] == 0)
            hipLaunchKernelGGL(k_cluster_f32_gauss6<true>, dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float*)mat, epi, g);
        else
            hipLaunchKernelGGL(k_cluster_f32_gauss6<false>, dim3(grid), dim3(256), 0, st, (float2*)psi,
                               (const float*)mat, epi, g);
        return hipGetLastError();
    }
    if (layout == LAYOUT_MFMA32F && !dbl) {
        switch (g.k) {
            case 4: return launch_mfma32_k<4>(psi, g, mat, epi, variant, st, stats_part, stats_blocks);
            case 5: return launch_mfma32_k<5>(psi, g, mat, epi, variant, st, stats_part, stats_blocks);
            case 6: return launch_mfma32_k<6>(psi, g, mat, epi, variant, st, stats_part, stats_blocks);
            default: return hipErrorInvalidValue;
        }
    }
    if (layout == LAYOUT_MFMA16D && dbl) {
        switch (g.k) {
            case 3: return launch_mfma64_k<3>(psi, g, mat, epi, variant, st);
            case 4: return launch_mfma64_k<4>(psi, g, mat, epi, variant, st);
            case 5: return launch_mfma64_k<5>(psi, g, mat, epi, variant, st);
            case 6: return launch_mfma64_k<6>(psi, g, mat, epi, variant, st);
            default: return hipErrorInvalidValue;
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_diag(void* psi, bool dbl, int n, const EpiDesc* epi, hipStream_t st) {
    const uint64_t nwin = n >= 7 ? (uint64_t(1) << (n - 7)) : 1;
    const unsigned grid = (unsigned)((nwin + 63) >> 6);  // runs of 64 windows, one per work-group
    auto go = [&](auto kern, auto* p) { hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, p, n, epi); };
    const bool nt = beyond_caches(n, dbl);
    if (dbl)
        nt ? go(k_diag<double, true>, (double2*)psi) : go(k_diag<double, false>, (double2*)psi);
    else
        nt ? go(k_diag<float, true>, (float2*)psi) : go(k_diag<float, false>, (float2*)psi);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchOp* ops, const BatchItem* items, uint32_t n_items, uint32_t* counters,
                        uint32_t n_circuits, uint32_t item_tiles, uint64_t wait_ticks, unsigned grid,
                        hipStream_t st) {
    const uint32_t nc = n_circuits + 2;
    hipLaunchKernelGGL(k_fill_u32, dim3((nc + 255) / 256), dim3(256), 0, st, counters, nc, 0u);
    hipLaunchKernelGGL(k_batch_f32, dim3(grid), dim3(512), 0, st, ops, items, n_items, counters, item_tiles,
                       wait_ticks);
    return hipGetLastError();
}

namespace {
template <typename T, bool NT>
hipError_t launch_gate1q_t(void* psi, int n, int q, const double m[8], hipStream_t st) {
    using U = Unit<T>;
    auto* p = (typename U::type*)psi;
    const uint64_t units = uint64_t(1) << (n - U::BITS);
    const int ub = q - U::BITS;
    Gate2x2<T> g;
    for (int i = 0; i < 8; ++i) g.m[i] = (T)m[i];
    auto go = [&](auto kern, uint64_t per_group) {
        hipLaunchKernelGGL(kern, dim3((unsigned)((units + per_group - 1) / per_group)), dim3(256), 0, st, p, ub, g,
                           units);
    };
    if (ub >= 3) go(k_gate1q<T, 0, NT>, 256 * gate1q_units(0, NT));
    else if (ub == 2) go(k_gate1q<T, 3, NT>, 256 * gate1q_units(3, NT));
    else if (ub == 1) go(k_gate1q<T, 2, NT>, 256 * gate1q_units(2, NT));
    else if (ub == 0) go(k_gate1q<T, 1, NT>, 256 * gate1q_units(1, NT));
    else if constexpr (U::BITS == 1) go(k_gate1q<T, 4, NT>, 256 * gate1q_units(4, NT));
    return hipGetLastError();
}

// A phase (or, NEG, a sign) on the amplitudes whose bits q0 (and q1 >= 0) are set.
// Where the selected units fit the caches, unit bit 2 selects too: half lines are
// enough there (T on qubit 3, complex64: 24 qubits 30 us, whole lines 39; 26 qubits
// 162 and 174), while HBM moves whole lines anyway (27 qubits: 404 us half lines,
// 357 whole). Units of a thread: 8 from HBM and on half lines, else 2 for more
// wavefronts, and 1 for a selection of a larger state (26 qubits, T on the highest:
// 74 us; 8 units in memory order 79).
template <typename T, bool NEG>
hipError_t launch_phase_t(void* psi, int n, int q0, int q1, double cs, double sn, hipStream_t st) {
    using U = Unit<T>;
    constexpr bool dbl = sizeof(T) == 8;
    int hb[2], nh, lomask, odd;
    auto select = [&](int lowest) {  // unit bits from `lowest` up select units, lower ones inside them
        hb[0] = hb[1] = -1;
        nh = lomask = odd = 0;
        for (int q : {std::min(q0, q1), std::max(q0, q1)}) {
            const int ub = q - U::BITS;
            if (q < 0) continue;
            if (ub < 0) odd = 1;
            else if (ub < lowest) lomask |= 1 << ub;
            else hb[nh++] = ub;
        }
    };
    select(2);
    const bool nt = beyond_caches(n - nh, dbl);
    if (nt) select(3);
    const uint64_t count = uint64_t(1) << (n - U::BITS - nh);
    const int spread = !nt || hb[0] == 7 || hb[1] == 7;
    auto go = [&](auto kern, int per_thread) {
        const unsigned per_group = 256 * per_thread;
        hipLaunchKernelGGL(kern, dim3((unsigned)((count + per_group - 1) / per_group)), dim3(256), 0, st,
                           (typename U::type*)psi, hb[0], hb[1], lomask, odd, spread, (T)cs, (T)sn, count);
    };
    if (nt) go(k_phase<T, NEG, true, 8>, 8);
    else if (beyond_caches(n, dbl)) go(k_phase<T, NEG, false, 1>, 1);
    else if (hb[0] == 2) go(k_phase<T, NEG, false, 8>, 8);
    else go(k_phase<T, NEG, false, 2>, 2);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_gate1q(void* psi, bool dbl, int n, int q, const double m[8], hipStream_t st) {
    if (beyond_caches(n, dbl))
        return dbl ? launch_gate1q_t<double, true>(psi, n, q, m, st) : launch_gate1q_t<float, true>(psi, n, q, m, st);
    return dbl ? launch_gate1q_t<double, false>(psi, n, q, m, st) : launch_gate1q_t<float, false>(psi, n, q, m, st);
}

hipError_t launch_phase1q(void* psi, bool dbl, int n, int q, double cs, double sn, hipStream_t st) {
    return dbl ? launch_phase_t<double, false>(psi, n, q, -1, cs, sn, st)
               : launch_phase_t<float, false>(psi, n, q, -1, cs, sn, st);
}

hipError_t launch_cz(void* psi, bool dbl, int n, int a, int b, hipStream_t st) {
    return dbl ? launch_phase_t<double, true>(psi, n, a, b, 0, 0, st)
               : launch_phase_t<float, true>(psi, n, a, b, 0, 0, st);
}

namespace {
// Launch of a streaming reduction over `units` (a power of two): runs of U
// rounds where they still fill the chip, else single rounds.
template <typename F>
unsigned launch_stream(uint64_t units, bool nt, F&& go) {
    constexpr int U = 8;
    const bool deep = units >= uint64_t(U) * 256 * kDeepBlocks;
    const unsigned grid = grid_for(units, deep ? U * 256 : 256, kReduceBlocks);
    if (!deep)
        go(grid, std::integral_constant<int, 1>{}, std::false_type{});
    else if (nt)
        go(grid, std::integral_constant<int, U>{}, std::true_type{});
    else
        go(grid, std::integral_constant<int, U>{}, std::false_type{});
    return grid;
}
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Up to this many units one work-group takes the sums of a state alone, with
// no second launch (two rounds of 8 accesses a lane).
constexpr uint64_t kAloneUnits = 4096;

template <typename T, typename P, int W>
void launch_stats_t(const void* psi, int n, void* probs, double* part, double* res, hipStream_t st) {
    const uint64_t units = (uint64_t(1) << n) / W;
    if (units <= kAloneUnits) {
        if (units >= 8 * 256)
            hipLaunchKernelGGL((k_stats<T, P, W, 8, false>), dim3(1), dim3(256), 0, st, psi, units, probs, res);
        else
            hipLaunchKernelGGL((k_stats<T, P, W, 1, false>), dim3(1), dim3(256), 0, st, psi, units, probs, res);
        return;
    }
    const unsigned grid = launch_stream(units, beyond_caches(n, sizeof(T) == 8), [&](unsigned g, auto u, auto nt) {
        hipLaunchKernelGGL((k_stats<T, P, W, decltype(u)::value, decltype(nt)::value>), dim3(g), dim3(256), 0, st, psi,
                           units, probs, part);
    });
    hipLaunchKernelGGL((k_reduce_final<3, 0u>), dim3(1), dim3(256), 0, st, part, (int)grid, res);
}

template <typename T, typename R, int W>
void launch_compare_t(const void* psi, int n, const void* ref, double* part, double* res, hipStream_t st) {
    const uint64_t units = (uint64_t(1) << n) / W;
    if (units <= kAloneUnits) {
        if (units >= 8 * 256)
            hipLaunchKernelGGL((k_compare<T, R, W, 8, false>), dim3(1), dim3(256), 0, st, psi, ref, units, res);
        else
            hipLaunchKernelGGL((k_compare<T, R, W, 1, false>), dim3(1), dim3(256), 0, st, psi, ref, units, res);
        return;
    }
    const unsigned grid = launch_stream(units, beyond_caches(n, sizeof(T) == 8), [&](unsigned g, auto u, auto nt) {
        hipLaunchKernelGGL((k_compare<T, R, W, decltype(u)::value, decltype(nt)::value>), dim3(g), dim3(256), 0, st,
                           psi, ref, units, part);
    });
    hipLaunchKernelGGL((k_reduce_final<5, 1u << 4>), dim3(1), dim3(256), 0, st, part, (int)grid, res);
}
}  // namespace

// Two complex64 amplitudes a lane where every pointer allows 16-byte accesses
// (8 bytes for the fp32 probabilities): a state may be a caller's view.
hipError_t launch_stats(const void* psi, bool dbl, int n, void* probs, bool probs_dbl, double* part,
                        double* res, hipStream_t st) {
    const bool wide = aligned(psi, 16) && aligned(probs, probs_dbl ? 16 : 8);
    if (dbl)
        probs_dbl ? launch_stats_t<double, double, 1>(psi, n, probs, part, res, st)
                  : launch_stats_t<double, float, 1>(psi, n, probs, part, res, st);
    else if (wide)
        probs_dbl ? launch_stats_t<float, double, 2>(psi, n, probs, part, res, st)
                  : launch_stats_t<float, float, 2>(psi, n, probs, part, res, st);
    else
        probs_dbl ? launch_stats_t<float, double, 1>(psi, n, probs, part, res, st)
                  : launch_stats_t<float, float, 1>(psi, n, probs, part, res, st);
    return hipGetLastError();
}

// ------------------------------------------------------------ bit permutation
// One work-group per tile, in memory order: the whole tile is loaded into
// registers (every load in flight), written to LDS at its permuted index, and
// stored back in the original order of addresses, so loads and stores are
// both 16-byte accesses of runs over the tile's lowest bits (the host puts the
// lowest non-moving state bits into the tile for that; bit 0 is always one of
// its bits for complex64). In place: a tile is read completely before any of it is written,
// and tiles are disjoint.
template <typename T, int NB, bool NT>
__global__ __launch_bounds__(256) void k_permute(typename Cplx<T>::type* __restrict__ psi, PermGeom pg, int share) {
    constexpr bool F = sizeof(T) == 4;
    constexpr int AB = F ? 1 : 0;  // tau bits of one 16-byte access
    constexpr int N = 1 << (NB - AB), PER = (N + 255) / 256;  // accesses of the tile, of a thread
    typedef T vt2 __attribute__((ext_vector_type(2)));
    __shared__ vf4 buf4[N];
    vt2* buf = reinterpret_cast<vt2*>(buf4);
    // tiles that share cache lines stay on one XCD (its L2 joins their accesses)
    uint64_t base = share ? xcd_block() : blockIdx.x;
#pragma unroll
    for (int i = 0; i < NB; ++i) base = insert_zero(base, pg.tb[i]);
    // slot of tau: its upper bits folded into the bank bits (linear over XOR)
    auto slot = [](int t) { return F ? t ^ (((t >> 5) & 15) << 1) : t ^ ((t >> 4) & 15); };
    // state offset and permuted slot of access t (both linear over its bits)
    auto off = [&](int t) {
        uint64_t o = 0;
#pragma unroll
        for (int j = AB; j < NB; ++j) o |= uint64_t((t >> (j - AB)) & 1) << pg.tb[j];
        return o;
    };
    auto dst = [&](int t) {
        int d = 0;
#pragma unroll
        for (int j = AB; j < NB; ++j) d |= ((t >> (j - AB)) & 1) << pg.to[j];
        return slot(d);
    };
    const int t = (int)threadIdx.x;
    const bool on = N >= 256 || t < N;
    typename Cplx<T>::type* mine = psi + (base | off(t));
    const int d0 = dst(t), d1 = F ? slot(1 << pg.to[0]) : 0;
    vf4 v[PER];
    if (on) {
#pragma unroll
        for (int r = 0; r < PER; ++r) v[r] = load16<NT>(reinterpret_cast<const vf4*>(mine + off(r * 256)));
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int d = d0 ^ dst(r * 256);
            if constexpr (F) {
                buf[d] = vt2{v[r].x, v[r].y};
                buf[d ^ d1] = vt2{v[r].z, v[r].w};
            } else {
                buf[d] = __builtin_bit_cast(vt2, v[r]);
            }
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int r = 0; r < PER; ++r)
            store16<NT>(reinterpret_cast<vf4*>(mine + off(r * 256)), (vf4)buf4[slot((r * 256 + t) << AB) >> AB]);
    }
}

namespace {
template <int NB>
hipError_t launch_permute_nt(void* psi, bool dbl, int n, const PermGeom& pg, hipStream_t st) {
    const unsigned grid = (unsigned)(uint64_t(1) << (n - NB));
    // a tile holds whole 128-byte lines when the lowest bits are tile bits
    const bool lines = NB < 4 || pg.tb[dbl ? 2 : 3] == (dbl ? 2 : 3);
    auto go = [&](auto kern, auto* p) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, p, pg, lines ? 0 : 1);
    };
    const bool nt = beyond_caches(n, dbl) && lines;
    if constexpr (NB <= 12)
        if (dbl) {
            nt ? go(k_permute<double, NB, true>, (double2*)psi) : go(k_permute<double, NB, false>, (double2*)psi);
            return hipGetLastError();
        }
    nt ? go(k_permute<float, NB, true>, (float2*)psi) : go(k_permute<float, NB, false>, (float2*)psi);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_permute(void* psi, bool dbl, int n, const PermGeom& pg, hipStream_t st) {
    if (pg.nt < 1 || pg.nt > (dbl ? 12 : kPermTileBits) || pg.nt > n || (!dbl && pg.tb[0] != 0)) return hipErrorInvalidValue;
    switch (pg.nt) {
        case 1: return launch_permute_nt<1>(psi, dbl, n, pg, st);
        case 2: return launch_permute_nt<2>(psi, dbl, n, pg, st);
        case 3: return launch_permute_nt<3>(psi, dbl, n, pg, st);
        case 4: return launch_permute_nt<4>(psi, dbl, n, pg, st);
        case 5: return launch_permute_nt<5>(psi, dbl, n, pg, st);
        case 6: return launch_permute_nt<6>(psi, dbl, n, pg, st);
        case 7: return launch_permute_nt<7>(psi, dbl, n, pg, st);
        case 8: return launch_permute_nt<8>(psi, dbl, n, pg, st);
        case 9: return launch_permute_nt<9>(psi, dbl, n, pg, st);
        case 10: return launch_permute_nt<10>(psi, dbl, n, pg, st);
        case 11: return launch_permute_nt<11>(psi, dbl, n, pg, st);
        case 12: return launch_permute_nt<12>(psi, dbl, n, pg, st);
        default: return launch_permute_nt<13>(psi, dbl, n, pg, st);
    }
}

hipError_t launch_reduce_stats(const double* part, unsigned nblocks, double* res, hipStream_t st) {
    hipLaunchKernelGGL((k_reduce_final<3, 0u>), dim3(1), dim3(256), 0, st, part, (int)nblocks, res);
    return hipGetLastError();
}

hipError_t launch_compare(const void* psi, bool dbl, int n, const void* ref, bool ref_dbl, double* part,
                          double* res, hipStream_t st) {
    const bool wide = aligned(psi, 16) && aligned(ref, 16);
    if (dbl)
        ref_dbl ? launch_compare_t<double, double, 1>(psi, n, ref, part, res, st)
                : launch_compare_t<double, float, 1>(psi, n, ref, part, res, st);
    else if (ref_dbl)
        launch_compare_t<float, double, 1>(psi, n, ref, part, res, st);
    else if (wide)
        launch_compare_t<float, float, 2>(psi, n, ref, part, res, st);
    else
        launch_compare_t<float, float, 1>(psi, n, ref, part, res, st);
    return hipGetLastError();
}

}  // namespace qsim
