// modal.hip -- the solve in the discrete sine modes of the cross-section.
//
// On a mesh whose nodes fill the pipe's lattice (X_i = (i+1) a/N, i + 1 < N, the
// same in y) the four-term operator of Eq. 8 is diagonal in x and y: the four
// cosines of each mode (m, n) combine to
//   4 sin(m pi X/a) sin(m pi X'/a) sin(n pi Y/b) sin(n pi Y'/b),
// and on the lattice the modes m, 2N - m, 2N + m, ... have the same sines up to
// sign, so they fold onto m' = 1 .. N - 1.  A solve is then
//   M1 x sine transform  (nx, ny, nz)   -> (nmx, ny, nzp)      [sine]
//   M2 y sine transform  (nmx, ny, nzp) -> (nmx, nmy, nzp)     [sine]
//   M3 z sum of every mode line with its folded z factor, in place: a recursion
//      while few modes fold onto a line [zexp], else a convolution (real lines
//      zero-padded, one real spectrum per line) [zconv]; banded plans a filter [zband]
//   M4 y sine transform back, M5 x sine transform back to (nx, ny, nz);
// where the planes of one axis fit LDS, M2 to M4 are one launch [plane] and the
// longer axis goes first and last.  Nothing is padded in x and y: 10 n values move instead of the 35 n of the
// padded transform (n = nx ny nz, the spectra included).  nzp is nz rounded up
// to a 16-byte vector.  A node on a wall carries no mode: its charge is not read and its
// potential is zero.  Whole solves, padded transform -> sine modes: 128x128x512
// FP32 234 -> 103 us, FP64 455 -> 164 us; 256x256x1024 FP32 1854 -> 772 us;
// 64x64x256 FP64 74 -> 37 us; 32x32x32 FP64 27 -> 22 us; errors against 64 bits no larger (FP32 1.4e-7
// against 2.1e-7 at 128x128x512).
#include <algorithm>

#include "pass_common.h"

#if !defined(PIPE_TU) || PIPE_TU == 1
#define PIPE_TU_FP32 1
#endif
#if !defined(PIPE_TU) || PIPE_TU == 2
#define PIPE_TU_FP64 1
#endif

namespace pipe {

// ---------------------------------------------------------------- sine transform
//
// The sine matrix of odd m is even about the middle of the lattice, that of even
// m odd, so each transform is two half-size products (folded: half the
// multiplications): with s_i = x_i + x_{na-1-i}, d_i = x_i - x_{na-1-i}, i < na/2,
//   y_m = sum_i sin(m pi (i+1)/N) s_i (m odd),  sum_i sin(..) d_i (m even);
// back, x_i = E_i + O_i and x_{na-1-i} = E_i - O_i from the two sums over m.
// N = na + 1 has large prime factors on the usual meshes (129 = 3 43, 257), so
// the products run on the matrix cores, in the working precision.

template <typename real, int V> struct vec_t { typedef real type __attribute__((ext_vector_type(V))); };
template <typename real> struct vec_t<real, 1> { typedef real type; };
template <typename real, int V> using vecv = typename vec_t<real, V>::type;

// 16 x 16 x 4 matrix instruction: A[lane % 16][lane / 16], B[lane / 16][lane % 16];
// register r of the result holds row(lane, r), column lane % 16.
template <typename real> struct Mfma16;
template <> struct Mfma16<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mac(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static constexpr int STEP = 1;   // rows between the registers of a lane
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <> struct Mfma16<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mac(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static constexpr int STEP = 4;
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

template <typename real, int V> __device__ __forceinline__ real velem(const vecv<real, V>& v, int e) {
    if constexpr (V == 1) return v;
    else return v[e];
}
template <typename real, int V> __device__ __forceinline__ void vset(vecv<real, V>& v, int e, real x) {
    if constexpr (V == 1) v = x;
    else v[e] = x;
}

// What both kernels below share: the operand access and the block's arithmetic.
// UV: the user's array (input of the forward, output of the inverse transform) is
// accessed as vectors; else value by value, bounded by nz.  Arrays are addressed as
// a uniform base and a 32-bit byte offset (the launcher checks that they fit).
template <typename real, bool INV, int V, bool UV> struct Sine {
    using vec = vecv<real, V>;
    using M = Mfma16<real>;
    using acc_t = typename M::acc;
    static constexpr int VA = 16 / sizeof(real), NA = 4 / VA;   // A values per load, loads per 16-deep block
    using veca = vecv<real, VA>;

    // Vector column cg = slab wv + g of the z rows.
    struct Column {
        unsigned slab, g;
        __device__ __forceinline__ Column(unsigned cg, unsigned wv) : slab(cg / wv), g(cg % wv) {}
        __device__ __forceinline__ void advance(unsigned dslab, unsigned dg, unsigned wv) {
            slab += dslab;
            g += dg;
            if (g >= wv) {
                g -= wv;
                ++slab;
            }
        }
        __device__ __forceinline__ unsigned offset(unsigned ss_bytes) const {
            return slab * ss_bytes + g * (unsigned)(V * sizeof(real));
        }
    };
    static __device__ __forceinline__ vec load(const SineArgs& a, gptr<const char> base, unsigned off, unsigned g, bool ok) {
        if constexpr (INV || UV) {
            return *reinterpret_cast<gptr<const vec>>(base + off);
        } else {
            const gptr<const real> p = reinterpret_cast<gptr<const real>>(base + off);
            vec v{};
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (ok && (int)g * V + e < a.nz) vset<real, V>(v, e, p[e]);
            return v;
        }
    }
    static __device__ __forceinline__ void store(const SineArgs& a, gptr<char> base, unsigned off, unsigned g, const vec& v) {
        if constexpr (!INV || UV) {
            *reinterpret_cast<gptr<vec>>(base + off) = v;
        } else {
            const gptr<real> p = reinterpret_cast<gptr<real>>(base + off);
#pragma unroll
            for (int e = 0; e < V; ++e)
                if ((int)g * V + e < a.nz) p[e] = velem<real, V>(v, e);
        }
    }
    // Sums of a product over the 16-deep blocks: each block is two 8-deep chains from
    // zero (one rounding per product, on partial sums of 8 terms) and the chains are
    // added pairwise.  One plain chain over the whole depth left FP32 solves 1.2x
    // (depth 64) to 2x (depth 128) further off than the padded transform.
    //
    // part[l] holds the sum of 2^l blocks; merge<KB> takes in block kb (compile-time after
    // unrolling) like a binary counter, the last block everything into part[0].
    static constexpr int LEVELS = 4;
    template <int KB> static __device__ __forceinline__ void merge(int kb, acc_t t, acc_t (&part)[LEVELS][V], int c) {
        int l = 0;
#pragma unroll
        for (int q = 0; q < LEVELS; ++q) {
            if (q == l && ((kb >> q) & 1)) {
                t = part[q][c] + t;
                l = q + 1;
            }
        }
        const bool last = kb + 1 == KB;
        // what is left of the counter above level l
#pragma unroll
        for (int q = 0; q < LEVELS; ++q)
            if (last && q >= l && ((kb >> q) & 1)) t = part[q][c] + t;
#if defined(__HIP_DEVICE_COMPILE__)
        // the additions are done here: left alone, the compiler moves those of all
        // blocks past the last product and holds every chain's result until then
        asm volatile("" : "+v"(t));
#endif
#pragma unroll
        for (int q = 0; q < LEVELS; ++q)
            if (q == (last ? 0 : l)) part[q][c] = t;
    }
    // forward: a 16-row tile of one parity's modes (i0 the lane's first row in it)
    static __device__ __forceinline__ void put_modes(const SineArgs& a, int i0, int par, const acc_t* sum, gptr<char> out,
                                                     unsigned col, unsigned g) {
        const unsigned es = (unsigned)(a.out_es * sizeof(real)), o0 = col + (par ? a.no + i0 : i0) * es;
        const int n = par ? a.ne : a.no;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            vec v;
#pragma unroll
            for (int c = 0; c < V; ++c) vset<real, V>(v, c, sum[c][r]);
            if (i0 + r * M::STEP < n) store(a, out, o0 + r * M::STEP * es, g, v);
        }
    }
    // inverse: a 16-row tile of nodes and its mirror image from the two parities' sums
    static __device__ __forceinline__ void put_nodes(const SineArgs& a, int i0, const acc_t* so, const acc_t* se,
                                                     gptr<char> out, unsigned col, unsigned g) {
        const unsigned es = (unsigned)(a.out_es * sizeof(real)), o0 = col + i0 * es, m0 = col + (a.na - 1 - i0) * es;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + r * M::STEP;
            vec o, e;
#pragma unroll
            for (int c = 0; c < V; ++c) {
                vset<real, V>(o, c, so[c][r]);
                vset<real, V>(e, c, se[c][r]);
            }
            if (i < a.he) {
                store(a, out, o0 + r * M::STEP * es, g, o + e);
                store(a, out, m0 - r * M::STEP * es, g, o - e);
            } else if (i < a.h) {
                store(a, out, o0 + r * M::STEP * es, g, o);
            }
        }
        // a node row on the wall (na = n - 1) carries no mode
        if (i0 == 0 && a.na < a.n) store(a, out, col + a.na * es, g, vec{});
    }
};

// Persistent: block b takes tiles b, b + grid, ... of g 16-lane column groups (V
// columns a lane) and all rows.  Wave w < rt g owns row tile w % rt of column
// group w / rt and keeps that tile's matrix rows (both parities, KB 16-deep
// blocks) in registers.  Rows come two tiles ahead: loaded into registers during
// the products of one tile, written to the free LDS buffer, folded (forward),
// during those of the next (its first half of waves after the odd modes, the other
// half, which shares the SIMDs, before them, so that the matrix cores are not left
// idle), used in the one after.  Column tile c of a group is the columns V j + c
// (j = lane % 16), so the B operands of all V tiles come with one LDS vector read
// and a row of the result leaves as one vector a lane, 16 lanes contiguous.
//
// Measured per pass: 256 rows x 262144 columns FP32 170 us (536 MB: 3.2 TB/s; the
// matrix cores' bound is 109 us, a pass without the products takes 108 us; one tile
// per block with the matrix streamed 195-240 us); 128 x 65536 FP32 20 us, FP64 38 us
// (memory alone 13 and 26).  Half-width columns at 128 rows, or registers for four
// waves per SIMD, were no faster.
template <typename real, bool INV, int V, int KB, bool UV>
__global__ __launch_bounds__(512) void sine_kernel(SineArgs a, const GroupArgs* __restrict__ group) {
    using S = Sine<real, INV, V, UV>;
    using M = typename S::M;
    using vec = typename S::vec;
    using veca = typename S::veca;
    using acc_t = typename S::acc_t;
    const void* in = a.in;
    void* out = a.out;
    if (group) {
        in = group[blockIdx.z].in;
        out = group[blockIdx.z].out;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    vec* lds = reinterpret_cast<vec*>(smem);           // [buffer][column group][parity][16 KB rows][16]
    constexpr int KP = 16 * KB;
    const gptr<const char> gin = to_global((const char*)in);
    const gptr<char> gout = to_global((char*)out);
    const int gw = a.g * 16, buf = a.g * 2 * KP * 16;
    const int cl = threadIdx.x % gw, r0 = threadIdx.x / gw, rs = blockDim.x / gw;   // 4 rs >= KP
    // rows of the two halves: forward i and its mirror image (folded here),
    // backward mode 2i + 1 and mode 2i + 2; zero beyond the half sizes
    const int na_ = INV ? a.no : a.h, nb_ = INV ? a.ne : a.he;
    const unsigned ies = (unsigned)(a.in_es * sizeof(real)), iss = (unsigned)(a.in_ss * sizeof(real));
    const unsigned xo = r0 * ies, yo = (INV ? a.no + r0 : a.na - 1 - r0) * ies;
    const unsigned tiles = (unsigned)((a.ngroups + gw - 1) / gw), wv = (unsigned)a.wv;
    const unsigned dslab = gridDim.x * gw / wv, dg = gridDim.x * gw % wv;
    vec x[4], y[4];
    typename S::Column cin(blockIdx.x * gw + cl, wv);
    unsigned fetched = blockIdx.x;      // the tile the next fetch takes
    auto fetch = [&] {
        // column 0 stands in for one past the end, row 0 for an absent row: no branch,
        // and nothing here uses the values, so the loads stay in flight
        const bool act = fetched * gw + cl < (unsigned)a.ngroups;
        const unsigned g = act ? cin.g : 0, col = act ? cin.offset(iss) : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = r0 + u * rs;
            x[u] = S::load(a, gin, col + (i < na_ ? xo + u * rs * ies : 0), g, act && i < na_);
            y[u] = S::load(a, gin, col + (i < nb_ ? (INV ? yo + u * rs * ies : yo - u * rs * ies) : 0), g, act && i < nb_);
        }
        cin.advance(dslab, dg, wv);
        fetched += gridDim.x;
    };
    auto stage = [&](vec* l) {
        l += (cl / 16) * 2 * KP * 16 + cl % 16;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = r0 + u * rs;
            if (i < nb_) {
                l[i * 16] = INV ? x[u] : x[u] + y[u];
                l[(KP + i) * 16] = INV ? y[u] : x[u] - y[u];
            } else if (i < na_) {
                l[i * 16] = x[u];
            }
        }
    };
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const bool works = wave < a.rt * a.g;
    const int rt = wave % a.rt, gi = works ? wave / a.rt : 0;
    const int i0 = rt * 16 + M::row(lane, 0);
    fetch();
    veca A[2][KB][S::NA];
    const gptr<const veca> frag = reinterpret_cast<gptr<const veca>>(to_global((const real*)a.frag));
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int q = 0; q < S::NA; ++q) A[p][kb][q] = frag[(((long)p * a.rt + rt) * KB + kb) * S::NA * 64 + q * 64 + lane];
    // the rows past the half sizes, zero in both buffers from here on
    for (int i = na_ + r0; i < KP; i += rs)
        for (int q = 0; q < 2; ++q) lds[q * buf + ((cl / 16) * 2 * KP + i) * 16 + cl % 16] = vec{};
    for (int i = nb_ + r0; i < KP; i += rs)
        for (int q = 0; q < 2; ++q) lds[q * buf + ((cl / 16) * 2 * KP + KP + i) * 16 + cl % 16] = vec{};
    stage(lds);
    if (fetched < tiles) fetch();
#if defined(__HIP_DEVICE_COMPILE__)
    // wait for the matrix rows here: a wait inside the loop would also wait for the
    // loads issued ahead there
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int q = 0; q < S::NA; ++q) asm volatile("" : "+v"(A[p][kb][q]));
#endif
    typename S::Column cout(blockIdx.x * gw + gi * 16 + (lane & 15), wv);
    const unsigned oss = (unsigned)(a.out_ss * sizeof(real));
    const int turn = (wave / 4) & 1 ? 0 : 1;
    int cur = 0;
    for (unsigned tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        __syncthreads();
        const vec* b = lds + cur * buf + gi * 2 * KP * 16 + (lane >> 4) * 16 + (lane & 15);
        const bool act = works && tile * gw + gi * 16 + (lane & 15) < (unsigned)a.ngroups;
        const unsigned col = cout.offset(oss);
        acc_t odd[V];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (p == turn && tile + gridDim.x < tiles) {
                stage(lds + (cur ^ 1) * buf);
                if (fetched < tiles) fetch();
            }
            if (!works) continue;
            // MFMAs of one column tile, then the additions of the one before (done by
            // then, and in the shadow of these): the order is fixed by the barriers
            acc_t part[S::LEVELS][V], c0, c1, d0, d1;
            vec bc[4], bn[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) bc[s] = b[(p * KP + 4 * s) * 16];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const veca* af = A[p][kb];
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    c0 = M::mac(af[0][0], velem<real, V>(bc[0], c), acc_t{});
                    c1 = M::mac(af[2 / S::VA][2 % S::VA], velem<real, V>(bc[2], c), acc_t{});
                    c0 = M::mac(af[1 / S::VA][1 % S::VA], velem<real, V>(bc[1], c), c0);
                    c1 = M::mac(af[3 / S::VA][3 % S::VA], velem<real, V>(bc[3], c), c1);
                    if (c == 0 && kb + 1 < KB) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) bn[s] = b[(p * KP + (kb + 1) * 16 + 4 * s) * 16];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (kb + c > 0) S::template merge<KB>(c ? kb : kb - 1, d0 + d1, part, c ? c - 1 : V - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    d0 = c0;
                    d1 = c1;
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) bc[s] = bn[s];
            }
            S::template merge<KB>(KB - 1, d0 + d1, part, V - 1);
            if constexpr (INV) {
                if (p == 0) {
#pragma unroll
                    for (int c = 0; c < V; ++c) odd[c] = part[0][c];
                } else if (act) {
                    S::put_nodes(a, i0, odd, part[0], gout, col, cout.g);
                }
            } else if (act) {
                S::put_modes(a, i0, p, part[0], gout, col, cout.g);
            }
        }
        cout.advance(dslab, dg, wv);
        cur ^= 1;
    }
}

// The same with the matrix read from L2 one 16-deep block ahead, for depths whose
// rows do not fit the registers: one tile per block, waves over its row tiles.
template <typename real, bool INV, int V, bool UV>
__global__ __launch_bounds__(512) void sine_stream_kernel(SineArgs a, const GroupArgs* __restrict__ group) {
    using S = Sine<real, INV, V, UV>;
    using M = typename S::M;
    using vec = typename S::vec;
    using veca = typename S::veca;
    using acc_t = typename S::acc_t;
    const void* in = a.in;
    void* out = a.out;
    if (group) {
        in = group[blockIdx.z].in;
        out = group[blockIdx.z].out;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    vec* lds = reinterpret_cast<vec*>(smem);           // [parity][16 kb rows][16]
    const int kp = a.kb * 16;
    const unsigned wv = (unsigned)a.wv;
    const gptr<const char> gin = to_global((const char*)in);
    const gptr<char> gout = to_global((char*)out);
    {
        const int cl = threadIdx.x % 16, r0 = threadIdx.x / 16, rs = blockDim.x / 16;
        const unsigned cg = blockIdx.x * 16 + cl;
        const bool act = cg < (unsigned)a.ngroups;
        const typename S::Column c(act ? cg : 0, wv);
        const unsigned es = (unsigned)(a.in_es * sizeof(real)), col = c.offset((unsigned)(a.in_ss * sizeof(real)));
        const int na_ = INV ? a.no : a.h, nb_ = INV ? a.ne : a.he;
        constexpr int U = 4;
        for (int ib = r0; ib < kp; ib += U * rs) {
            vec x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = ib + u * rs;
                x[u] = S::load(a, gin, col + (i < na_ ? i * es : 0), c.g, act && i < na_);
                y[u] = S::load(a, gin, col + (i < nb_ ? (INV ? a.no + i : a.na - 1 - i) * es : 0), c.g, act && i < nb_);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = ib + u * rs;
                if (i < kp) {
                    const vec xv = i < na_ ? x[u] : vec{}, yv = i < nb_ ? y[u] : vec{};
                    lds[i * 16 + cl] = INV ? xv : xv + yv;
                    lds[(kp + i) * 16 + cl] = INV ? yv : (i < nb_ ? xv - yv : vec{});
                }
            }
        }
    }
    __syncthreads();
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, nw = blockDim.x / 64;
    const gptr<const veca> frag = reinterpret_cast<gptr<const veca>>(to_global((const real*)a.frag));
    const unsigned cg = blockIdx.x * 16 + (lane & 15);
    const bool act = cg < (unsigned)a.ngroups;
    const typename S::Column c(act ? cg : 0, wv);
    const unsigned col = c.offset((unsigned)(a.out_ss * sizeof(real)));
    for (int rt = wave; rt < a.rt; rt += nw) {
        const int i0 = rt * 16 + M::row(lane, 0);
        acc_t odd[V];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const gptr<const veca> f = frag + ((long)p * a.rt + rt) * a.kb * S::NA * 64 + lane;
            const vec* b = lds + p * kp * 16 + (lane >> 4) * 16 + (lane & 15);
            // 8-deep chains added up over 64, then those sums over the depth
            acc_t sum[V], four[V];
#pragma unroll
            for (int c = 0; c < V; ++c) sum[c] = four[c] = acc_t{};
            veca af[S::NA], an[S::NA];
#pragma unroll
            for (int q = 0; q < S::NA; ++q) af[q] = f[q * 64];
            for (int kb = 0; kb < a.kb; ++kb) {
                const int kn = kb + 1 < a.kb ? kb + 1 : kb;
#pragma unroll
                for (int q = 0; q < S::NA; ++q) an[q] = f[(kn * S::NA + q) * 64];
                vec v[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) v[s] = b[(kb * 16 + 4 * s) * 16];
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    acc_t c0 = M::mac(af[0][0], velem<real, V>(v[0], c), acc_t{});
                    acc_t c1 = M::mac(af[2 / S::VA][2 % S::VA], velem<real, V>(v[2], c), acc_t{});
                    c0 = M::mac(af[1 / S::VA][1 % S::VA], velem<real, V>(v[1], c), c0);
                    c1 = M::mac(af[3 / S::VA][3 % S::VA], velem<real, V>(v[3], c), c1);
                    four[c] += c0 + c1;
                }
                if (kb % 4 == 3 || kb + 1 == a.kb) {
#pragma unroll
                    for (int c = 0; c < V; ++c) {
                        sum[c] += four[c];
                        four[c] = acc_t{};
                    }
                }
#pragma unroll
                for (int q = 0; q < S::NA; ++q) af[q] = an[q];
            }
            if constexpr (INV) {
                if (p == 0) {
#pragma unroll
                    for (int c = 0; c < V; ++c) odd[c] = sum[c];
                } else if (act) {
                    S::put_nodes(a, i0, odd, sum, gout, col, c.g);
                }
            } else if (act) {
                S::put_modes(a, i0, p, sum, gout, col, c.g);
            }
        }
    }
}

// ---------------------------------------------------------------- z convolution
//
// In place on lines of n values (pitch apart): forward transform of the line
// zero-padded to 2 NH, product with the line's real spectrum, inverse, first n
// values kept.  The line is read as NH packed pairs Z; with e = Z_k + conj
// Z_{NH-k}, o = -i W^k (Z_k - conj Z_{NH-k}) (twice the spectra of the even and
// odd samples) the two bins k and NH - k of the half spectrum are (e +- o)/2,
// their product with the spectra t_k, t_{NH-k} and the packing of the inverse
// give
//   A = p e + m o,  B = m e + p o,  p, m = (t_k +- t_{NH-k})/2,
//   Z'_k = A + i W^{-k} B,  Z'_{NH-k} = conj(A - i W^{-k} B),
// so one thread takes both bins, and the table holds the pairs (p, m) for
// k <= NH/2 (scale factors included).  k = 0 is the pair (0, NH) by the same
// formula, and Z'_{NH/2} = 2 p Z_{NH/2}.
//
// A line lies inside one wavefront (P = NH/E lanes, P divides 64), and after the
// last stage lane t holds the bins t + q P, q < E, which are also the inputs of
// the inverse transform's first stage.  The partner of bin t + q P is bin
// E - 1 - q of lane P - t (lane 0: bin E - q of its own), so the product needs one
// lane exchange each way and no pass through LDS.  Only the first half of the
// packed pairs is ever non-zero (n <= NH) or kept.
//
// Bound by its vector and LDS instructions as much as by memory: 16384 lines of 512
// FP32 27 us (100 MB: 3.7 TB/s), FP64 59 us; 65536 lines of 1024 FP32 236 us (805
// MB).  With the product through LDS, twiddles read there and no pruning: 35, 63 and
// 280 us.  More waves per SIMD by a register cap spill and run slower.

// Length plan: at most 12 values per thread, 16 at NH = 1024, which keeps the line
// in one wavefront.
template <typename real, int NH> constexpr int zc_V() { return NH == 1024 ? 0 : narrow_variant<NH>(sizeof(real) == 8 ? 8 : 12); }

// Lines per block: 256 threads, fewer while their LDS exceeds 64 KB (FP64, NH = 1024).
template <typename real, int NH> constexpr int zc_lines() {
    int l = 256 / (NH / Plan<NH, zc_V<real, NH>()>::E);
    while (l * lpad_len<z_pad<NH>()>(NH) * 2 * (int)sizeof(real) > 65536) l /= 2;
    return l;
}

// Stage twiddles from LDS.
template <class PL, typename TW> struct TwLds {
    const TW* tw;
    template <int s> __device__ __forceinline__ TW get(int t, int b, int r) const {
        constexpr int NS = plan_ns<PL>(s), P = PL::LEN / PL::E;
        return tw[stage_tw_offset<PL>(NS) + (r - 1) * NS + (t + b * P) % NS];
    }
};
// The same held in registers: they do not change from line to line.
template <class PL> constexpr int tw_slot(int s) {
    int n = 0;
    for (int i = 1; i < s; ++i) n += PL::E / PL::radix(i) * (PL::radix(i) - 1);
    return n;
}
template <class PL, typename TW> struct TwRegs {
    TW w[tw_slot<PL>(PL::S) > 0 ? tw_slot<PL>(PL::S) : 1];
    template <int s> __device__ __forceinline__ TW get(int, int b, int r) const {
        return w[tw_slot<PL>(s) + b * (PL::radix(s) - 1) + r - 1];
    }
    template <int s = 1> __device__ __forceinline__ void load(const TwLds<PL, TW>& from, int t) {
        if constexpr (s < PL::S) {
#pragma unroll
            for (int b = 0; b < PL::E / PL::radix(s); ++b)
#pragma unroll
                for (int r = 1; r < PL::radix(s); ++r)
                    w[tw_slot<PL>(s) + b * (PL::radix(s) - 1) + r - 1] = from.template get<s>(t, b, r);
            load<s + 1>(from, t);
        }
    }
};

// DFT of R values of which only the first half is non-zero: the even outputs are
// the half-size DFT of it, the odd ones that of the half times W_R^r.
template <int R, typename C> __device__ __forceinline__ void dft_half_zero(C* v) {
    using real = decltype(C::x);
    if constexpr (R == 4 || R == 8 || R == 16) {
        constexpr int H = R / 2;
        C e[H], o[H];
#pragma unroll
        for (int r = 0; r < H; ++r) {
            e[r] = v[r];
            const real c[8] = {1, (real)0.92387953251128675612818318939679, (real)0.70710678118654752440084436210485,
                               (real)0.38268343236508977172845998403040, 0, (real)-0.38268343236508977172845998403040,
                               (real)-0.70710678118654752440084436210485, (real)-0.92387953251128675612818318939679};
            const int q = r * (16 / R);   // W_16^q = cos(2 pi q/16) - i sin(2 pi q/16)
            if (q == 0) o[r] = v[r];
            else if (q == 4) o[r] = cmake<C>(v[r].y, -v[r].x);
            else o[r] = cmul(v[r], cmake<C>(c[q], -(q < 4 ? c[4 - q] : c[q - 4])));
        }
        dft<H, false>(e);
        dft<H, false>(o);
#pragma unroll
        for (int r = 0; r < H; ++r) {
            v[2 * r] = e[r];
            v[2 * r + 1] = o[r];
        }
    } else {
        dft<R, false>(v);
    }
}

// Stages s.. of a transform inside a wavefront, results left in v: value b R + r of
// the last stage is bin t + (b + r E/R) P.  HALF: stage 0's inputs e >= N/2 are zero.
template <class PL, int s, bool INV, bool HALF, typename C, typename Tw, typename Lds>
__device__ __forceinline__ void wave_stages(C* v, int t, const Tw& tw, Lds lds) {
    constexpr int R = PL::radix(s), NS = plan_ns<PL>(s), NB = PL::E / R;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if constexpr (s > 0) {
#pragma unroll
            for (int r = 1; r < R; ++r) v[b * R + r] = ctw<INV>(v[b * R + r], tw.template get<s>(t, b, r));
        }
        if constexpr (s == 0 && HALF) dft_half_zero<R>(&v[b * R]);
        else dft<R, INV>(&v[b * R]);
    }
    if constexpr (s + 1 < PL::S) {
        stage_store<PL, R, NS>(v, t, [&](int e, C x) { lds.set(e, x); });
        line_sync<Sync::WAVE>();
        stage_load<PL, PL::radix(s + 1)>(v, t, [&](int e) { return lds.get(e); });
        line_sync<Sync::WAVE>();
        wave_stages<PL, s + 1, INV, HALF>(v, t, tw, lds);
    }
}

// The value of another lane (byte index 4 * lane).
__device__ __forceinline__ float from_lane(float x, int idx) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(idx, __float_as_int(x)));
}
__device__ __forceinline__ double from_lane(double x, int idx) {
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(idx, __double2hiint(x)),
                            __builtin_amdgcn_ds_bpermute(idx, __double2loint(x)));
}

template <typename real, int NH>
__global__ __launch_bounds__((zc_lines<real, NH>() * (NH / Plan<NH, zc_V<real, NH>()>::E)))
void zconv_kernel(real* data, long pitch, int n, long nlines, const cplx<real>* table, const twid<real>* __restrict__ tw,
                  const twid<real>* __restrict__ tw2, const GroupArgs* __restrict__ group) {
    using C = cplx<real>;
    using TW = twid<real>;
    if (group) {
        data = (real*)group[blockIdx.z].out;
        table = (const C*)group[blockIdx.z].table;
    }
    using PL = Plan<NH, zc_V<real, NH>()>;
    constexpr int E = PL::E, P = NH / E, LPW = zc_lines<real, NH>(), H = E / 2;
    static_assert(64 % P == 0 && E % 2 == 0 && NH % 2 == 0, "a line per wavefront, bins paired");
    constexpr int R0 = PL::radix(0), NB0 = E / R0, RL = PL::radix(PL::S - 1), NBL = E / RL;
    constexpr int LR = (R0 + 1) / 2, NL = NB0 * LR;          // inputs of stage 0 that may be non-zero
    constexpr int PADN = lpad_len<z_pad<NH>()>(NH);
    constexpr int NP = NH / 2 + 1;
    constexpr bool TWR = sizeof(real) == 4 && tw_slot<PL>(PL::S) <= 16;   // stage twiddles in registers
    __shared__ C lds[PL::S > 1 ? LPW * PADN : 1];
    __shared__ TW s_tw[stage_tw_size<PL>() > 0 ? stage_tw_size<PL>() : 1];
    stage_twiddles(s_tw, tw, stage_tw_size<PL>());
    __syncthreads();
    const int t = threadIdx.x % P, l = threadIdx.x / P;
    const int peer = ((threadIdx.x & 63) - t + (P - t) % P) * 4;
    LdsLine<C, z_pad<NH>()> view{lds + (PL::S > 1 ? l * PADN : 0)};
    const TwLds<PL, TW> twl{s_tw};
    TwRegs<PL, TW> twr;
    if constexpr (TWR) twr.load(twl, t);
    TW w2[H];
#pragma unroll
    for (int q = 0; q < H; ++q) w2[q] = tw2[t + q * P];
    const long ngroups = (nlines + LPW - 1) / LPW;
    const gptr<real> gd = to_global(data);
    const gptr<const C> gt = to_global(table);
    // packed pairs of stage 0 (first half), spectra pairs of the bins t + q P, q < E/2,
    // and of bin NH/2
    auto load = [&](C* v, C* pm, real& mid, long line) {
        const bool active = line < nlines;
        const gptr<const C> src = reinterpret_cast<gptr<const C>>(gd + (active ? line : 0) * pitch);
#pragma unroll
        for (int b = 0; b < NB0; ++b)
#pragma unroll
            for (int r = 0; r < LR; ++r) {
                const int m = t + b * P + r * (NH / R0);
                C x = cmake<C>(0, 0);
                if (active && 2 * m < n) {
                    x = src[m];                       // pitch is even, rows 16-byte aligned
                    if (2 * m + 1 >= n) x.y = 0;
                }
                v[b * LR + r] = x;
            }
        const gptr<const C> tl = gt + (active ? line : 0) * NP;
#pragma unroll
        for (int q = 0; q < H; ++q) pm[q] = tl[t + q * P];
        mid = tl[NH / 2].x;
    };
    C nxt[NL], pn[H];
    real mn = 0;
    long g = blockIdx.x;
    if (g < ngroups) load(nxt, pn, mn, g * LPW + l);
    for (; g < ngroups; g += gridDim.x) {
        C v[E], pm[H];
        const real mid = mn;
#pragma unroll
        for (int b = 0; b < NB0; ++b)
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                if (r < LR) v[b * R0 + r] = nxt[b * LR + r];
                else v[b * R0 + r] = cmake<C>(0, 0);
            }
#pragma unroll
        for (int q = 0; q < H; ++q) pm[q] = pn[q];
        const long gn = g + gridDim.x;
        if (gn < ngroups) load(nxt, pn, mn, gn * LPW + l);
        if constexpr (TWR) wave_stages<PL, 0, false, true>(v, t, twr, view);
        else wave_stages<PL, 0, false, true>(v, t, twl, view);
        // bin q of this lane after the forward / before the inverse transform
        auto out = [&](int q) -> C& { return v[(q % NBL) * RL + q / NBL]; };
        C u[E];
        auto inp = [&](int q) -> C& { return u[(q % NB0) * R0 + q / NB0]; };
        C back[H];
#pragma unroll
        for (int q = 0; q < H; ++q) {
            const C zk = out(q);
            C zn;
            if constexpr (P > 1) {
                const C mine = out(E - 1 - q), own = out((E - q) % E);
                zn.x = from_lane(mine.x, peer);
                zn.y = from_lane(mine.y, peer);
                if (t == 0) zn = own;
            } else {
                zn = out((E - q) % E);
            }
            zn = cconj(zn);
            const C ev = cadd(zk, zn);
            const C d = ctw<false>(csub(zk, zn), w2[q]);
            const C od = cmake<C>(d.y, -d.x);                        // -i W^k (Z_k - conj Z_{NH-k})
            const real p = pm[q].x, m = pm[q].y;
            const C A = cmake<C>(fma(p, ev.x, m * od.x), fma(p, ev.y, m * od.y));
            const C B = ctw<true>(cmake<C>(fma(m, ev.x, p * od.x), fma(m, ev.y, p * od.y)), w2[q]);
            inp(q) = cmake<C>(A.x - B.y, A.y + B.x);                 // A + i W^{-k} B
            back[q] = cmake<C>(A.x + B.y, B.x - A.y);                // conj(A - i W^{-k} B)
        }
        const C half = cscale(out(H), 2 * mid);                      // lane 0: bin NH/2
#pragma unroll
        for (int i = H; i < E; ++i) {
            C own = half;
            if (i > H) own = back[E - i];
            if constexpr (P > 1) {
                C z;
                z.x = from_lane(back[E - 1 - i].x, peer);
                z.y = from_lane(back[E - 1 - i].y, peer);
                if (t == 0) z = own;
                inp(i) = z;
            } else {
                inp(i) = own;
            }
        }
        if constexpr (TWR) wave_stages<PL, 0, true, false>(u, t, twr, view);
        else wave_stages<PL, 0, true, false>(u, t, twl, view);
        const long line = g * LPW + l;
        const bool active = line < nlines;
        const gptr<C> dst = reinterpret_cast<gptr<C>>(gd + (active ? line : 0) * pitch);
#pragma unroll
        for (int b = 0; b < NBL; ++b)
#pragma unroll
            for (int r = 0; r < (RL + 1) / 2; ++r) {
                const int m = t + b * P + r * (NH / RL);
                if (active && 2 * m < n) dst[m] = u[b * RL + r];
            }
    }
}

// ---------------------------------------------------------------- z recursion
//
// The z factor of every mode is an exponential beyond the first plane, W(d) = C
// r^{d-1} for d >= 1 with r = e^{-kappa hz} (Eq. 9 as it stands, Eq. 15 with its
// constant factor), and a mode line folds at most 2 x 2 of them while no more than
// 2N modes are kept per axis (beyond, in steps of four).  The z convolution is then
//   out_k = W(0) x_k + sum_e C_e (F_k + G_k),
//   F_{k+1} = r F_k + x_k,  G_{k-1} = r G_k + x_k:
// no transform, no padding and no spectra to read (2 n values move instead of 3 n).
// Lane t of the P lanes of a line holds values t V .. t V + V - 1: it runs the two
// recursions over its own values, the lanes' results are combined by log2(P) shifts
// with weights r^{V 2^s}, and it runs them again from what comes in.  r is applied as
// an unevaluated sum hi + lo: a single rounding of r is raised to the distance it
// carries (FP32 errors up to 4x the transform's at kappa hz = 0.05; with it at most
// 0.94x over kappa hz = 1e-4 .. 2).
//
// Measured: 16384 lines of 512, four exponentials, FP32 21 us (the z convolution 27),
// FP64 40 us (60); 65536 lines of 1024, one exponential, FP32 123 us (236; a copy of
// the lines takes 110).  16 values a lane instead of 8 up to 512: 22 and 54 us.  The
// entries of a step's exponentials lie side by side, one vector load each: 27 x 9216
// lines of 192 FP32 191 -> 163 us.
template <typename real> __device__ __forceinline__ real lane_shift(real x, int idx, bool in) {
    const real v = from_lane(x, idx);
    return in ? v : (real)0;
}
// The recursion sum of one line from a lane's values x; tl: the line's table row with
// ng groups of NE exponentials; t: lane of the line, lane: of the wave.
template <typename real, int V, int NE>
__device__ __forceinline__ void zexp_line(const real* x, real* o, gptr<const real> tl, int ng, int logp, int t, int lane) {
    using ent = vecv<real, NE>;
    const int P = 1 << logp;
    const real c0 = tl[0];
#pragma unroll
    for (int j = 0; j < V; ++j) o[j] = c0 * x[j];
    for (int q = 0; q < ng; ++q) {
        const auto te = reinterpret_cast<gptr<const ent>>(tl + kZexpLead + q * NE * kZexpEntries);
        const ent vh = te[0], vl = te[1], vc = te[2];
        real rh[NE], rl[NE], f[NE], g[NE];
        auto step = [&](int e, real y, real xv) { return fma(rh[e], y, fma(rl[e], y, xv)); };
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            rh[e] = velem<real, NE>(vh, e);
            rl[e] = velem<real, NE>(vl, e);
            real s = 0, b = 0;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                s = step(e, s, x[j]);
                b = step(e, b, x[V - 1 - j]);
            }
            f[e] = lane_shift(s, (lane - 1) * 4, t >= 1);
            g[e] = lane_shift(b, (lane + 1) * 4, t + 1 < P);
        }
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            if (s >= logp) break;
            const int d = 1 << s;
            const ent vw = te[3 + s];
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const real w = velem<real, NE>(vw, e);
                f[e] = fma(w, lane_shift(f[e], (lane - d) * 4, t >= d), f[e]);
                g[e] = fma(w, lane_shift(g[e], (lane + d) * 4, t + d < P), g[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const real c = velem<real, NE>(vc, e);
            real y = f[e], z = g[e];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                o[j] = fma(c, y, o[j]);
                y = step(e, y, x[j]);
                o[V - 1 - j] = fma(c, z, o[V - 1 - j]);
                z = step(e, z, x[V - 1 - j]);
            }
        }
    }
}
// A lane's V values of a row of n (rows hold whole 16-byte vectors), zero beyond, and back.
template <typename real, int V, typename P> __device__ __forceinline__ void zexp_load(real* x, P row, int k0, int n) {
    constexpr int VW = 16 / sizeof(real);
    using vec = vecv<real, VW>;
#pragma unroll
    for (int q = 0; q < V / VW; ++q) {
        vec v{};
        if (k0 + q * VW < n) v = *reinterpret_cast<gptr<const vec>>(row + k0 + q * VW);
#pragma unroll
        for (int e = 0; e < VW; ++e) x[q * VW + e] = k0 + q * VW + e < n ? v[e] : (real)0;
    }
}

// WAVE: a line per wavefront (P = 64); its table row is then the same for every lane
// and comes by scalar loads.
template <typename real, int V, int NE, bool WAVE>
__global__ __launch_bounds__(256) void zexp_kernel(real* data, long pitch, int n, long nlines, const real* table, int logp,
                                                   int ng, const GroupArgs* __restrict__ group) {
    constexpr int VW = 16 / sizeof(real), NV = V / VW;
    using vec = vecv<real, VW>;
    if (group) {
        data = (real*)group[blockIdx.z].out;
        table = (const real*)group[blockIdx.z].table;
    }
    if constexpr (WAVE) logp = 6;
    if constexpr (sizeof(real) == 4) ng = 1;
    const int P = 1 << logp, t = threadIdx.x & (P - 1), lane = threadIdx.x & 63;
    const long line = (long)blockIdx.x * (256 >> logp) + (threadIdx.x >> logp);
    const bool active = line < nlines;
    const long at = WAVE ? __builtin_amdgcn_readfirstlane((int)(active ? line : 0)) : (active ? line : 0);
    const gptr<real> row = to_global(data) + at * pitch;
    real x[V], o[V];
    zexp_load<real, V>(x, row, t * V, n);
    zexp_line<real, V, NE>(x, o, to_global(table) + at * zexp_row(ng * NE), ng, logp, t, lane);
    if (!active) return;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        vec v;
#pragma unroll
        for (int e = 0; e < VW; ++e) v[e] = o[q * VW + e];
        if (t * V + q * VW < n) reinterpret_cast<gptr<vec>>(row + t * V)[q] = v;
    }
}

// ---------------------------------------------------------------- sines, z, sines of a plane
//
// M2 to M4 in one block for one mode of the outer axis, where a plane (rows of the
// other axis, nz) fits LDS: its sines, the z sum of its mode lines and its sines back,
// with the plane read and written once (6 n values less traffic) and three launches a
// solve instead of five.  Bound by the serial work of one block per plane: one product,
// the z sum, one product (32x32x32 FP64 6.7 us, 70x40x75 FP64 17).  A wave's job is 16
// rows of both parities in 16 V columns; with a wave taking all rows of its columns,
// lines of 32 left three of four waves idle (a 128x128x32 FP32 solve 40 us, now 26; in
// five launches 34).  The forward product is in place, so its sums (kPlaneJobs a wave at
// most) stay in registers until all waves have read.  KC: 16-deep blocks of matrix rows
// in flight.  NE: exponentials of a recursion step, 0: the z sum directly, by a window
// of 8 values a lane and 8 distances a step, where a recursion over many folded modes
// costs more (9x96x57 FP32, 40 exponentials a line: 47 us, 31 by the padded transforms).
constexpr int kPlaneJobs = 3;      // 160 KB hold 40 jobs of 4 KB
template <typename real, int KC, int NE>
__global__ __launch_bounds__(1024) void plane_kernel(PlaneArgs a, const GroupArgs* __restrict__ group) {
    constexpr int V = 8 / sizeof(real);
    using S = Sine<real, true, V, true>;
    using M = typename S::M;
    using vec = typename S::vec;
    using veca = typename S::veca;
    using acc_t = typename S::acc_t;
    constexpr int VW = 16 / sizeof(real);
    using wide = vecv<real, VW>;
    const real* in = (const real*)a.in;
    real* out = (real*)a.out;
    const real* table = (const real*)a.table;
    if (group) {
        in = out = (real*)group[blockIdx.z].out;
        table = (const real*)group[blockIdx.z].table;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    real* lds = reinterpret_cast<real*>(smem);         // [parity][KP rows][pitch]
    const int T = a.t, KP = 16 * T;
    // this block's columns: wl from z0, of which w from hp are its own
    const int z0 = (int)blockIdx.y * a.w - a.hp, wl = a.wl, klo = z0 < 0 ? -z0 : 0;
    const int khi = min(wl, a.nz - z0), kend = min(a.hp + a.w, a.nzp - z0);
    const gptr<const real> src = to_global(in) + blockIdx.x * a.ps + z0;
    const gptr<real> dst = to_global(out) + blockIdx.x * a.ps + z0;
    const int lane = threadIdx.x % 64, nw = blockDim.x / 64, pitch = a.pitch;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // rows in, folded
    const int wv = wl / VW;
#pragma unroll 2
    for (int i = threadIdx.x; i < KP * wv; i += blockDim.x) {
        const int r = i / wv, k = (i % wv) * VW;
        wide x{}, y{};
        const bool in_line = k >= klo && z0 + k < a.nzp;
        if (in_line && r < a.h) x = *reinterpret_cast<gptr<const wide>>(src + r * a.rs + k);
        if (in_line && r < a.he) y = *reinterpret_cast<gptr<const wide>>(src + (a.na - 1 - r) * a.rs + k);
        *reinterpret_cast<wide*>(lds + r * pitch + k) = x + y;
        *reinterpret_cast<wide*>(lds + (KP + r) * pitch + k) = r < a.he ? x - y : wide{};
    }
    __syncthreads();
    const int groups = (wl + 16 * V - 1) / (16 * V);
    // a lane's column of group cg from k0 on; past the last column another of the group
    auto column = [&](int k0, int cg) {
        const int own = k0 + (cg * 16 + (lane & 15)) * V;
        return own < wl ? own : k0 + cg * 16 * V;
    };
    // sum[parity] of row tile rt (of nrt) over kbn 16-deep blocks
    auto product = [&](const void* frag_, int nrt, int kbn, int rt, int col, acc_t (&sum)[2][V]) {
        const gptr<const veca> frag = reinterpret_cast<gptr<const veca>>(to_global((const real*)frag_)) + lane;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int c = 0; c < V; ++c) sum[p][c] = acc_t{};
#pragma unroll 1
            for (int k0 = 0; k0 < (KC == 4 ? kbn : 1); k0 += KC) {
                veca af[KC][S::NA];
                acc_t part[V];
                __builtin_amdgcn_sched_barrier(0);       // no loads of the next parity before this
                const gptr<const veca> fk = frag + ((p * nrt + rt) * kbn + k0) * S::NA * 64;
                if (k0 + KC <= kbn) {
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int q = 0; q < S::NA; ++q) af[k][q] = fk[(k * S::NA + q) * 64];
                } else {            // few modes, or the last blocks
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int q = 0; q < S::NA; ++q)
                            if (k0 + k < kbn) af[k][q] = fk[(k * S::NA + q) * 64];
                }
#pragma unroll
                for (int c = 0; c < V; ++c) part[c] = acc_t{};
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    if (k0 + k >= kbn) break;
                    vec b[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        b[s] = *reinterpret_cast<const vec*>(lds + (p * KP + (k0 + k) * 16 + 4 * s + (lane >> 4)) * pitch +
                                                             col);
#pragma unroll
                    for (int c = 0; c < V; ++c) {
                        acc_t c0 = M::mac(af[k][0][0], velem<real, V>(b[0], c), acc_t{});
                        acc_t c1 = M::mac(af[k][2 / S::VA][2 % S::VA], velem<real, V>(b[2], c), acc_t{});
                        c0 = M::mac(af[k][1 / S::VA][1 % S::VA], velem<real, V>(b[1], c), c0);
                        c1 = M::mac(af[k][3 / S::VA][3 % S::VA], velem<real, V>(b[3], c), c1);
                        part[c] += c0 + c1;
                    }
                }
#pragma unroll
                for (int c = 0; c < V; ++c) sum[p][c] += part[c];
            }
        }
    };
    {
        acc_t sum[kPlaneJobs][2][V];
#pragma unroll
        for (int j = 0; j < kPlaneJobs; ++j) {
            const int job = wave + j * nw, cg = job % groups, rt = job / groups;
            if (rt >= a.tm) break;
            product(a.fwd, a.tm, T, rt, column(0, cg), sum[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPlaneJobs; ++j) {
            const int job = wave + j * nw, cg = job % groups, rt = job / groups;
            if (rt >= a.tm) break;
            const int col = (cg * 16 + (lane & 15)) * V;
            if (col < wl)
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        vec v;
#pragma unroll
                        for (int c = 0; c < V; ++c) vset<real, V>(v, c, sum[j][p][c][r]);
                        *reinterpret_cast<vec*>(lds + (p * KP + rt * 16 + M::row(lane, r)) * pitch + col) = v;
                    }
        }
    }
    __syncthreads();
    {
        constexpr int VZ = 8;
        const int P = 1 << a.logp, t = lane & (P - 1), per = 64 >> a.logp, lines = a.no + a.ne;
        for (int l0 = wave * per; l0 < lines; l0 += nw * per) {      // the wave's lanes stay together
            const int l = l0 + (lane >> a.logp);
            const bool active = l < lines;
            const int at = active ? l : l0;
            real* row = lds + (at < a.no ? at : KP + at - a.no) * pitch;
            auto get = [&](real* x, int k0) {      // 8 values from k0 (a multiple of 8), zero outside the line
#pragma unroll
                for (int q = 0; q < VZ / VW; ++q) {
                    const int k = k0 + q * VW;
                    wide v{};
                    if (k >= klo && k < khi) v = *reinterpret_cast<const wide*>(row + k);
#pragma unroll
                    for (int e = 0; e < VW; ++e) x[q * VW + e] = k + e < khi ? v[e] : (real)0;
                }
            };
            real x[VZ], o[VZ];
            get(x, t * VZ);
            const gptr<const real> tl = to_global(table) + blockIdx.x * a.tp + at * a.tl;
            if constexpr (NE > 0) {
                zexp_line<real, VZ, NE>(x, o, tl, a.ng, a.logp, t, lane);
            } else {
                const real c0 = tl[0];
                real lo[VZ], hi[VZ];
#pragma unroll
                for (int i = 0; i < VZ; ++i) {
                    o[i] = c0 * x[i];
                    lo[i] = hi[i] = x[i];
                }
#pragma unroll(sizeof(real) == 4 ? 2 : 1)
                for (int jb = 1; jb <= a.ng; ++jb) {
                    real c[VZ], u[VZ], w[VZ];
#pragma unroll
                    for (int q = 0; q < VZ / VW; ++q) {
                        const wide v = reinterpret_cast<gptr<const wide>>(tl + jb * VZ)[q];
#pragma unroll
                        for (int e = 0; e < VW; ++e) c[q * VW + e] = v[e];
                    }
                    get(u, (t - jb) * VZ);
                    get(w, (t + jb) * VZ);
#pragma unroll
                    for (int j = 1; j <= VZ; ++j)
#pragma unroll
                        for (int i = 0; i < VZ; ++i)
                            o[i] = fma(c[j - 1], (i >= j ? lo[i - j] : u[VZ + i - j]) + (i + j < VZ ? hi[i + j] : w[i + j - VZ]),
                                       o[i]);
#pragma unroll
                    for (int i = 0; i < VZ; ++i) {
                        lo[i] = u[i];
                        hi[i] = w[i];
                    }
                }
            }
            if (active) {
#pragma unroll
                for (int q = 0; q < VZ / VW; ++q) {
                    wide v;
#pragma unroll
                    for (int e = 0; e < VW; ++e) v[e] = o[q * VW + e];
                    if (t * VZ + q * VW < khi) *reinterpret_cast<wide*>(row + t * VZ + q * VW) = v;
                }
            }
        }
    }
    __syncthreads();
    const int own = (a.w + 16 * V - 1) / (16 * V);
    for (int job = wave; job < own * T; job += nw) {
        const int cg = job % own, rt = job / own;
        acc_t sum[2][V];
        product(a.inv, T, a.tm, rt, column(a.hp, cg), sum);
        const int col = a.hp + (cg * 16 + (lane & 15)) * V;
        if (col >= kend) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = rt * 16 + M::row(lane, r);
            vec o, e;
#pragma unroll
            for (int c = 0; c < V; ++c) {
                vset<real, V>(o, c, sum[0][c][r]);
                vset<real, V>(e, c, sum[1][c][r]);
            }
            auto put = [&](int row, const vec& v) {
                *reinterpret_cast<gptr<vec>>(dst + row * a.rs + col) = v;
            };
            if (i < a.he) {
                put(i, o + e);
                put(a.na - 1 - i, o - e);
            } else if (i < a.h) {
                put(i, o);
            }
            if (i == 0 && a.na < a.n) put(a.na, vec{});      // a node row on the wall
        }
    }
}

// ---------------------------------------------------------------- neighbouring planes
//
// The z sum of a banded plan (Eq. 18) on the mode lines: a symmetric filter of 2 NB
// + 1 values, one 16-byte vector of outputs a thread.  The window's vectors come from
// L1 after the first thread; memory bound (one read and one write of the lines).
// Whole banded solves at 128x128x256 FP32, N = 2, 20 x 20 modes: 76 us by the padded
// transform's coefficient product, 32 us here; with 256 x 256 modes 57 us, 66 us with
// the z convolution cut at N in place of the filter.
template <typename real, int NB>
__global__ __launch_bounds__(256) void zband_kernel(const real* in, real* out, unsigned wv, unsigned total,
                                                    const real* table) {
    constexpr int V = 16 / sizeof(real), Q = (NB + V - 1) / V;   // window: Q vectors each side
    using vec = vecv<real, V>;
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const unsigned line = i / wv, g = i % wv;
    const gptr<const vec> src = reinterpret_cast<gptr<const vec>>(to_global(in)) + i;
    const gptr<const real> t = to_global(table) + (size_t)line * (NB + 1);
    real w[V * (2 * Q + 1)], c[NB + 1];
#pragma unroll
    for (int d = 0; d <= NB; ++d) c[d] = t[d];
#pragma unroll
    for (int q = -Q; q <= Q; ++q) {
        vec v{};
        if ((int)g + q >= 0 && (int)g + q < (int)wv) v = src[q];
#pragma unroll
        for (int e = 0; e < V; ++e) w[(q + Q) * V + e] = v[e];
    }
    vec o;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        real acc = c[0] * w[Q * V + e];
#pragma unroll
        for (int d = 1; d <= NB; ++d) acc = fma(c[d], w[Q * V + e - d] + w[Q * V + e + d], acc);
        o[e] = acc;
    }
    reinterpret_cast<gptr<vec>>(to_global(out))[i] = o;
}

// ---------------------------------------------------------------- launchers

// Depth (16-deep blocks) up to which the matrix rows stay in registers, and the
// columns a lane then holds: one 16-byte vector, half of it where FP64 rows take
// 128 registers.
constexpr int kSineBlocks = 8;
template <typename real> constexpr int sine_V(int kb) {
    return sizeof(real) == 4 ? (kb <= kSineBlocks ? 4 : 2) : (kb <= 4 ? 2 : 1);
}

template <typename real, bool INV, bool UV, int KB, int V>
static hipError_t launch_sine_kb(SineArgs a, hipStream_t s, const GroupArgs* group, int ngroup) {
    const int row_waves = a.rt > KB ? a.rt : KB;      // 4 row loads a thread and half
    // column groups per block: at least four waves while the tiles cover the chip
    a.g = 1;
    while (a.g < 4 && row_waves * a.g < 4 && a.ngroups * ngroup / (32 * a.g) >= 512) a.g *= 2;
    const int waves = row_waves * a.g;
    const long lds = 2l * 2 * 16 * KB * a.g * 16 * V * sizeof(real);
    // blocks that fit a CU: 160 KB of LDS, 8 waves (2 per SIMD) where the matrix
    // rows fill the registers, 16 where they do not
    const int fit = (int)std::max(1l, std::min(163840 / lds, (long)(KB * (int)sizeof(real) > 16 ? 8 : 16) / waves));
    const long ntile = (a.ngroups + a.g * 16 - 1) / (a.g * 16);
    const long cap = std::max(1l, 256l * fit / ngroup);
    const dim3 grid((unsigned)std::min(ntile, cap), 1, (unsigned)ngroup);
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute((const void*)sine_kernel<real, INV, V, KB, UV>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sine_kernel<real, INV, V, KB, UV>), grid, dim3(64 * waves), lds, s, a, group);
    return hipGetLastError();
}

template <typename real, bool INV, bool UV, bool NARROW>
static hipError_t launch_sine_depth(SineArgs a, hipStream_t s, const GroupArgs* group, int ngroup) {
    switch (a.kb) {
#define X(KB_)                                                                                                \
    case KB_: return launch_sine_kb<real, INV, UV, KB_, NARROW ? 1 : sine_V<real>(KB_)>(a, s, group, ngroup);
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
#undef X
    }
    return hipErrorInvalidValue;
}
template <typename real, bool INV, bool UV>
static hipError_t launch_sine_dir(SineArgs a, hipStream_t s, const GroupArgs* group, int ngroup) {
    if (a.rt <= 8 && a.kb <= kSineBlocks) {
        // one column a lane where that makes few tiles: the products of a tile are one wave's
        // serial work, a block's matrix rows the price.  Tiles up to which it pays, by depth in
        // blocks (whole solves in us, wide -> narrow; in brackets the tiles of a pass): one block
        // FP32 32x32x250 (500) 23.3 -> 21.9, 30x31x500 (969) 25.6 -> 28.5, FP64 32x32x128 (256)
        // 20.5 -> 20.1, 32x32x250 26.6 -> 27.2 (few modes, more rows: within 3 % either way, FP64
        // 20 modes 128x128x100 (800) 32.4 -> 33.0, 200x200x60 (750) 41.6 -> 40.1); two FP32 64x64x256 (1024) 31.0 -> 28.2, 64x64x640
        // (2560) 46.2 -> 42.1, 64x64x1000 (4000) 54.5 -> 57.2, FP64 64x64x384 (1536) 47.6 -> 45.1,
        // 40x40x720 (1800) 46.8 -> 48.2, 64x64x500 (2000) 54.3 -> 53.1; more FP32 250x100x60
        // (375, 938) 50.9 -> 45.0, 160x160x64 (640) 47.0 -> 50.4, FP64 120x120x60 (450) 44.7 -> 46.1.
        const bool fp32 = sizeof(real) == 4;
        const int v = sine_V<real>(a.kb), few = a.kb == 2 ? (fp32 ? 2560 : 1536) : fp32 ? 512 : 256;
        if (v > 1 && (a.ngroups * v + 15) / 16 * ngroup <= few) {
            a.wv *= v;
            a.ngroups *= v;
            return launch_sine_depth<real, INV, false, true>(a, s, group, ngroup);
        }
        return launch_sine_depth<real, INV, UV, false>(a, s, group, ngroup);
    }
    // more than 256 rows on either side: half-width columns keep 2 x 16 kb rows in 64 KB
    constexpr int V = 8 / sizeof(real);
    a.g = 1;
    a.wv = a.wv * sine_V<real>(a.kb) / V;
    a.ngroups = a.ngroups * sine_V<real>(a.kb) / V;
    const dim3 grid((unsigned)((a.ngroups + 15) / 16), 1, (unsigned)ngroup);
    hipLaunchKernelGGL((sine_stream_kernel<real, INV, V, UV>), grid, dim3(512), 2u * 16 * a.kb * 16 * V * sizeof(real), s, a,
                       group);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_sine(const SineAxis& ax, bool inverse, const void* in, void* out, int nz, int nzp, long in_ss,
                       long in_es, long out_ss, long out_es, long nslabs, bool user_vec, hipStream_t s,
                       const GroupArgs* group, int ngroup) {
    if (nslabs <= 0 || nz <= 0 || nzp < nz || ax.na < 1 || ax.na > kSineMaxRows || ax.nm < 1 || ax.nm > ax.na ||
        nzp % (16 / (int)sizeof(real)))
        return hipErrorInvalidValue;
    // the kernels' 32-bit byte offsets
    const long in_rows = inverse ? ax.nm : ax.na, out_rows = inverse ? ax.n : ax.nm;
    if (((in_rows - 1) * in_es + (nslabs - 1) * in_ss + nzp) * (long)sizeof(real) >= (1l << 32) ||
        ((out_rows - 1) * out_es + (nslabs - 1) * out_ss + nzp) * (long)sizeof(real) >= (1l << 32))
        return hipErrorInvalidValue;
    SineArgs a{};
    a.in = in;
    a.out = out;
    a.in_ss = in_ss; a.in_es = in_es; a.out_ss = out_ss; a.out_es = out_es;
    a.nz = nz;
    a.n = ax.n; a.na = ax.na;
    a.h = (ax.na + 1) / 2; a.he = ax.na / 2;
    a.no = (ax.nm + 1) / 2; a.ne = ax.nm / 2;
    const int rows = inverse ? a.h : a.no, depth = inverse ? a.no : a.h;
    a.rt = (rows + 15) / 16;
    a.kb = (depth + 15) / 16;
    a.frag = (const char*)ax.frag + (inverse ? sine_frag_elems(ax.na, ax.nm, false) * sizeof(real) : 0);
    const int v = sine_V<real>(a.kb);
    a.wv = nzp / v;
    a.ngroups = nslabs * a.wv;
    if (inverse)
        return user_vec ? launch_sine_dir<real, true, true>(a, s, group, ngroup)
                        : launch_sine_dir<real, true, false>(a, s, group, ngroup);
    return user_vec ? launch_sine_dir<real, false, true>(a, s, group, ngroup)
                    : launch_sine_dir<real, false, false>(a, s, group, ngroup);
}

// Transform lengths of the z convolution (kZconvLengths).
#define PIPE_FOR_EACH_ZCONV_N(X) \
    X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384) X(512) X(768) X(1024)

// Blocks of a kernel that run on one CU at once.  The persistent z convolution gets
// exactly as many as run (a second, partly filled wave of blocks costs more than the
// uneven shares: 256x256x1024 FP32 236 us at 768 = 3 a CU, 260 at 2048, 305 at 1024).
static int resident_blocks(const void* kernel, int threads) {
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel, threads, 0) != hipSuccess || b < 1) b = 4;
    return b;
}

template <typename real>
hipError_t launch_zconv(int nh, void* data, long pitch, int n, long nlines, const void* table, const TwiddleBank& twb,
                        hipStream_t s, const GroupArgs* group, int ngroup) {
    using C = cplx<real>;
    const twid<real>* tw2 = twb.get<twid<real>>(2 * nh);
    if (!tw2 || nlines <= 0 || n < 1 || n > nh || pitch < n || pitch % 2) return hipErrorInvalidValue;
    switch (nh) {
#define X(N_)                                                                                            \
    case N_: {                                                                                           \
        constexpr int V = zc_V<real, N_>(), LPW = zc_lines<real, N_>();                                  \
        const twid<real>* tw = twb.stage<twid<real>>(N_, V);                                             \
        if (!tw) return hipErrorInvalidValue;                                                            \
        static const int fit = resident_blocks((const void*)zconv_kernel<real, N_>, LPW * (N_ / Plan<N_, V>::E)); \
        const long ng = (nlines + LPW - 1) / LPW, cap = std::max(1l, 256l * fit / ngroup);               \
        dim3 grid((unsigned)(ng < cap ? ng : cap), 1, (unsigned)ngroup);                                 \
        hipLaunchKernelGGL((zconv_kernel<real, N_>), grid, dim3(LPW * (N_ / Plan<N_, V>::E)), 0, s,       \
                           (real*)data, pitch, n, nlines,                                                \
                           (const C*)table, tw, tw2, group);                                             \
        return hipGetLastError();                                                                        \
    }
        PIPE_FOR_EACH_ZCONV_N(X)
#undef X
    }
    return hipErrorInvalidValue;
}

template <typename real, int V>
static hipError_t launch_zexp_v(void* data, long pitch, int n, long nlines, int ne, const void* table, hipStream_t s,
                                const GroupArgs* group, int ngroup) {
    int logp = 0;
    while ((V << logp) < n) ++logp;
    if (logp > 6) return hipErrorInvalidValue;
    const long per = 256 >> logp;
    const dim3 grid((unsigned)((nlines + per - 1) / per), 1, (unsigned)ngroup), block(256);
    const int ng = ne > 4 ? ne / 4 : 1;
    switch (ne > 4 ? 4 : ne) {
#define X(N_)                                                                                              \
    case N_:                                                                                               \
        if (logp == 6)                                                                                     \
            hipLaunchKernelGGL((zexp_kernel<real, V, N_, true>), grid, block, 0, s, (real*)data, pitch, n, nlines, \
                               (const real*)table, logp, ng, group);                                       \
        else                                                                                               \
            hipLaunchKernelGGL((zexp_kernel<real, V, N_, false>), grid, block, 0, s, (real*)data, pitch, n, nlines, \
                               (const real*)table, logp, ng, group);                                       \
        return hipGetLastError();
        X(1) X(2) X(4)
#undef X
    }
    return hipErrorInvalidValue;
}
template <typename real>
hipError_t launch_zexp(void* data, long pitch, int n, long nlines, int ne, const void* table, hipStream_t s,
                       const GroupArgs* group, int ngroup) {
    if (nlines <= 0 || n < 1 || n > 1024 || pitch < n || pitch % (16 / (int)sizeof(real))) return hipErrorInvalidValue;
    const int v = zexp_values(n, (int)sizeof(real));
    return v == 16   ? launch_zexp_v<real, 16>(data, pitch, n, nlines, ne, table, s, group, ngroup)
           : v == 12 ? launch_zexp_v<real, 12>(data, pitch, n, nlines, ne, table, s, group, ngroup)
                     : launch_zexp_v<real, 8>(data, pitch, n, nlines, ne, table, s, group, ngroup);
}

template <typename real>
hipError_t launch_plane(const SineAxis& ax, const PlaneSplit& split, long rs, long ps, int nplanes, const void* in,
                        void* out, int nz, int nzp, int ne, int nb, const void* table, long line_stride,
                        long plane_stride, hipStream_t s, const GroupArgs* group, int ngroup) {
    constexpr int VW = 16 / sizeof(real);
    const bool whole = split.w >= nz;
    const int wl = whole ? nzp : split.w + 2 * split.hp;
    const size_t lds = plane_lds_bytes(ax, wl, (int)sizeof(real));
    if (nplanes <= 0 || nz < 1 || nzp < nz || nzp % VW || !lds || ne < 0 || nb < 0) return hipErrorInvalidValue;
    // a part of the lines: whole lane windows, and the neighbours' planes that its sums reach
    if (!whole && (split.w < 8 || split.w % 8 || split.hp < 8 * nb || split.hp % 8 || ne || in == out || group))
        return hipErrorInvalidValue;
    PlaneArgs a{};
    a.in = in;
    a.out = out;
    a.table = table;
    a.fwd = ax.frag;
    a.inv = (const char*)ax.frag + sine_frag_elems(ax.na, ax.nm, false) * sizeof(real);
    a.rs = rs; a.ps = ps;
    a.n = ax.n; a.na = ax.na;
    a.h = (ax.na + 1) / 2; a.he = ax.na / 2;
    a.no = (ax.nm + 1) / 2; a.ne = ax.nm / 2;
    a.tm = (a.no + 15) / 16;
    a.t = (a.h + 15) / 16;
    a.nz = nz; a.nzp = nzp;
    a.w = whole ? nzp : split.w;
    a.hp = whole ? 0 : split.hp;
    a.wl = wl;
    a.pitch = (int)(lds / (2 * 16 * a.t) / sizeof(real));
    a.logp = 0;
    while ((8 << a.logp) < (whole ? nz : wl)) ++a.logp;
    const int per = ne < 4 ? ne : 4;
    a.ng = per ? ne / per : nb;
    const long row = plane_table_row(ne, nb);
    a.tl = line_stride * row;
    a.tp = plane_stride * row;
    // a wave per job: at least four (row loads, z lines), at most sixteen
    const int jobs = (wl + 16 * 8 / (int)sizeof(real) - 1) / (16 * 8 / (int)sizeof(real)) * a.t;
    if (jobs > 16 * kPlaneJobs) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nplanes, (unsigned)((nz + a.w - 1) / a.w), (unsigned)ngroup), block(64 * (jobs < 4 ? 4 : jobs > 16 ? 16 : jobs));
    switch (per + 8 * (a.t < 4 ? a.t : 4)) {
#define X(K_, N_)                                                                                            \
    case N_ + 8 * K_: {                                                                                      \
        if (lds > 65536) {                                                                                   \
            const hipError_t e = hipFuncSetAttribute((const void*)plane_kernel<real, K_, N_>,                \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);  \
            if (e != hipSuccess) return e;                                                                   \
        }                                                                                                    \
        hipLaunchKernelGGL((plane_kernel<real, K_, N_>), grid, block, lds, s, a, group);                     \
        return hipGetLastError();                                                                            \
    }
#define Y(K_) X(K_, 0) X(K_, 1) X(K_, 2) X(K_, 4)
        Y(1) Y(2) Y(3) Y(4)
#undef Y
#undef X
    }
    return hipErrorInvalidValue;
}

template <typename real>
hipError_t launch_zband(const void* in, void* out, long pitch, long nlines, int nb, const void* table, hipStream_t s) {
    const int v = 16 / (int)sizeof(real);
    if (nlines <= 0 || pitch <= 0 || pitch % v || nlines * pitch / v >= (1l << 32)) return hipErrorInvalidValue;
    const unsigned wv = (unsigned)(pitch / v), total = (unsigned)(nlines * pitch / v);
    const dim3 grid((total + 255) / 256), block(256);
    switch (nb) {
#define X(N_)                                                                                                 \
    case N_:                                                                                                  \
        hipLaunchKernelGGL((zband_kernel<real, N_>), grid, block, 0, s, (const real*)in, (real*)out, wv, total, \
                           (const real*)table);                                                               \
        return hipGetLastError();
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#undef X
    }
    return hipErrorInvalidValue;
}

#define PIPE_INST(real)                                                                                        \
    template hipError_t launch_sine<real>(const SineAxis&, bool, const void*, void*, int, int, long, long, long, \
                                          long, long, bool, hipStream_t, const GroupArgs*, int);          \
    template hipError_t launch_zconv<real>(int, void*, long, int, long, const void*, const TwiddleBank&,         \
                                           hipStream_t, const GroupArgs*, int);                                \
    template hipError_t launch_zexp<real>(void*, long, int, long, int, const void*, hipStream_t,                \
                                          const GroupArgs*, int);                                              \
    template hipError_t launch_plane<real>(const SineAxis&, const PlaneSplit&, long, long, int, const void*, void*, int, \
                                           int, int, int, const void*, long, long, hipStream_t, const GroupArgs*, int); \
    template hipError_t launch_zband<real>(const void*, void*, long, long, int, const void*, hipStream_t);
#if PIPE_TU_FP32
PIPE_INST(float)
#endif
#if PIPE_TU_FP64
PIPE_INST(double)
#endif
#undef PIPE_INST

}  // namespace pipe
