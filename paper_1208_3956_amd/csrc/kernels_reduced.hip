// Strip operators of the reduced form (Algorithm 3, Sec. 2.3) as explicit dense blocks.
//
// A reduced sweep feeds a strip solve values at 3 columns of every row and reads 5 columns of
// every row back: upward psi on beta_s, beta_s + 1 and the transmission source on beta_s - 1,
// beta_s in, the interface columns of v and the next strip's source out; downward the mirror
// image.  The block substitutions of kernels_solve.hip carry all 64 columns of every row
// through a chain of 2 (m - 1) dependent products per chunk to get there.  Here the strip is
// cut into chunks of M rows (the fine chunks of the factorisation joined in groups of
// kappa), and per direction the factorisation stores, for a chunk c with separators above
// and below,
//   Rm_c   (64 x 6M)        right-hand side of the separator closing chunk c from the inputs of
//                          chunks c, c + 1
//   Sm     (64 ns x 64 ns)  inverse of the separators' Schur complement, all ns of them
//   Tm_c   (5M x (3M + 128)) outputs of the chunk's rows (its closing separator's included) from
//                          its inputs and the two separators
// so that a strip solve is three independent dense products (one when ns = 0) with no chain
// inside.  At 2032 rows, M = 64: 1984 matrix values per row and direction against 3 x 4096
// of the block factors, and 4.1 instead of 15 GFLOP for 64 right-hand sides.
//
// All panels and matrices are held in the matrix cores' operand order: element (row or
// right-hand side n, k) of a 16-wide tile at k-group k / 8, lane 16 (k % 4) + n, half
// (k / 4) % 2, so that a lane's loads are 16 bytes wide and a wave's consecutive, and the
// products need no staging.
#include "gj_register.hpp"
#include "helm_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace helm {

namespace {

using namespace gjr;
constexpr int NT = 256;
constexpr int TI = 6;            // target columns / input columns per row of the build's blocks
typedef float mf4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- products of a strip solve
// A product's tiles: 16 rows by W right-hand sides; element j of a lane's accumulator lies in
// row row(lane, j), column lane % W.
template <typename T> struct Wide;
template <> struct Wide<float> {
    using acc = mf4;
    static constexpr int W = 16, REGS = 4;
    static __device__ inline acc mul(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int lane, int j) { return 4 * (lane >> 4) + j; }
    static __device__ inline float get(const acc& c, int j) { return c[j]; }
};
template <> struct Wide<double> {
    using acc = md4;
    static constexpr int W = 16, REGS = 4;
    static __device__ inline acc mul(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int lane, int j) { return (lane >> 4) + 4 * j; }
    static __device__ inline double get(const acc& c, int j) { return c[j]; }
};
// four right-hand sides: the blocks of 4x4x4 are the tile's four groups of rows, so that the left
// operand's layout is that of 16x16x4; sums over k in the same order (FP64 only: the FP32
// form keeps a sum per k, so that a column's bits would depend on the panel's width)
template <typename T> struct Quad;
template <> struct Quad<double> {
    using acc = double;
    static constexpr int W = 4, REGS = 1;
    static __device__ inline acc mul(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int lane, int) { return (lane & 12) + (lane >> 4); }
    static __device__ inline double get(const acc& c, int) { return c; }
};

// the two k-steps of group gi in this lane
__device__ inline void load_group(const float2* p, int gi, int lane, float2 (&v)[2]) {
    const float4 x = reinterpret_cast<const float4*>(p)[(size_t)gi * 64 + lane];
    v[0] = make_float2(x.x, x.y);
    v[1] = make_float2(x.z, x.w);
}
__device__ inline void load_group(const double2* p, int gi, int lane, double2 (&v)[2]) {
    v[0] = p[((size_t)gi * 2) * 64 + lane];
    v[1] = p[((size_t)gi * 2 + 1) * 64 + lane];
}

// One 16-row tile of a product for NC column tiles of TL::W right-hand sides: the four waves
// take a quarter of the k range each and add their tiles through LDS in a fixed order, so a
// right-hand side's result does not depend on its neighbours.  Four real products per complex
// one.  Operands come straight from memory, U k-groups (8 U values of k) ahead of their products.
//   MODE 0  r^ = Rm p           tile = 4 separator + quarter
//   MODE 1  x_s = Sm r^         tile = 4 separator + quarter
//   MODE 2  outputs = Tm [p; x_s]   tile = (chunk, active output, 16-row group)
// The column tiles of a row tile follow each other on one XCD (blocks 8 apart), which reads
// the matrix from memory once.  Bound by the launch (4 to 5 us of any dependent one) and, at
// 2032 rows, by reading Tm (42 MB in FP32, 8.6 us; 13.5 us a launch with 16 right-hand sides)
// or by the products (64: 2.7 GFLOP, 32 us).  Not faster: eight waves with 2 x 2 tiles each
// (64 -> 90 us a strip solve), registers for five workgroups a CU instead of three (56 -> 56).
template <typename T, typename TL, int NC, int MODE>
__global__ void __launch_bounds__(NT) k_red_mul(RedArgs<T> a, int tiles, int nc) {
    using V = cplx<T>;
    constexpr int U = std::is_same<T, float>::value || (TL::W == 4 && NC == 1) ? 4 : 2, W = TL::W;
    constexpr int CPG = 16 / W;                     // column tiles per group of right-hand sides
    __shared__ V red[4][NC][16][W];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int tile = blockIdx.z * 8 + blockIdx.x, c0 = blockIdx.y * NC;
    // all arguments at once: each is otherwise read where it is used, one scalar load's latency
    // after the other (0.3 of 6 to 14 us a launch)
    asm volatile("" ::"s"(a.A), "s"(a.p), "s"(a.pn), "s"(a.rh), "s"(a.xs), "s"(a.dst), "s"(a.dst_rs), "s"(a.dst_ls), "s"(a.base),
                 "s"(a.trA), "s"(a.trB), "s"(a.omap), "s"(a.M), "s"(a.nrhs), "s"(tiles));
    if (tile >= tiles) return;
    const int per = a.Mp / 16, KP = 3 * a.Mp;
    int c, o = 0, lg = 0, ng, nga;
    const V* A;
    if (MODE == 0) {
        c = tile >> 2;
        nga = ng = 2 * KP / 8;
        A = a.A + (size_t)tile * 16 * 2 * KP;
    } else if (MODE == 1) {
        c = 0;
        nga = ng = 8 * a.ns;
        A = a.A + (size_t)tile * 16 * 64 * a.ns;
    } else {
        c = tile / (a.nout * per);
        const int rem = tile - c * a.nout * per;
        o = a.omap >> 4 * (rem / per) & 7;
        lg = rem % per;
        const int K = KP + (a.ns ? 2 * WP : 0);
        nga = KP / 8;
        ng = K / 8;
        A = a.A + ((size_t)(c * 5 + o) * per + lg) * 16 * K;
    }
    const V* Bp[NC];
    const V* Bx[NC];
    int bl[NC];                                     // this lane's place in the panel's groups
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        const int ct = min(c0 + u, nc - 1), g = ct / CPG;
        bl[u] = W == 16 ? lane : (lane & 48) + (ct % CPG) * W + lane % W;
        Bp[u] = MODE == 1 ? a.rh + (size_t)g * a.ns * WP * 16 : a.p + ((size_t)g * a.P + c) * KP * 16;
        Bx[u] = MODE == 2 ? a.xs + ((size_t)g * (a.ns + 2) + c) * WP * 16 - (size_t)nga * 128 : nullptr;
    }
    const int k0 = ng * w / 4, k1 = ng * (w + 1) / 4;
    typename TL::acc cr[NC], ci[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) { cr[u] = typename TL::acc{}; ci[u] = cr[u]; }
    struct Stage { V a[U][2], b[U][NC][2]; };
    auto load = [&](Stage& s, int k) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int gi = min(k + i, k1 - 1);
            load_group(A, gi, lane, s.a[i]);
#pragma unroll
            for (int u = 0; u < NC; ++u) load_group(MODE == 2 && gi >= nga ? Bx[u] : Bp[u], gi, bl[u], s.b[i][u]);
        }
    };
    auto mul = [&](const Stage& s, int k) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (k + i >= k1) break;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const V x = s.a[i][h];
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    const V y = s.b[i][u][h];
                    cr[u] = TL::mul(x.x, y.x, cr[u]);
                    ci[u] = TL::mul(x.x, y.y, ci[u]);
                }
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    const V y = s.b[i][u][h];
                    cr[u] = TL::mul(-x.y, y.y, cr[u]);
                    ci[u] = TL::mul(x.y, y.x, ci[u]);
                }
            }
        }
    };
    if (k0 < k1) {
        Stage s0, s1;
        load(s0, k0);
        for (int k = k0; k < k1; k += 2 * U) {
            load(s1, k + U);
            mul(s0, k);
            load(s0, k + 2 * U);
            mul(s1, k + U);
        }
    }
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
        for (int j = 0; j < TL::REGS; ++j)
            red[w][u][TL::row(lane, j)][lane % W] = cmk<V>(TL::get(cr[u], j), TL::get(ci[u], j));
    __syncthreads();
#pragma unroll
    for (int q = t; q < 16 * W * NC; q += NT) {
        const int u = q / (16 * W), row = q / W % 16, ct = c0 + u, g = ct / CPG, rn = (ct % CPG) * W + q % W;
        if (ct >= nc) break;
        const V v = cadd(cadd(red[0][u][row][q % W], red[1][u][row][q % W]), cadd(red[2][u][row][q % W], red[3][u][row][q % W]));
        if (MODE == 0) {
            a.rh[(size_t)g * a.ns * WP * 16 + red_pos<T>(tile * 16 + row, rn)] = v;
        } else if (MODE == 1) {
            a.xs[(size_t)g * (a.ns + 2) * WP * 16 + red_pos<T>(WP + tile * 16 + row, rn)] = v;
        } else {
            const int lr = 16 * lg + row, l = c * a.M + lr, r = 16 * g + rn;
            if (lr < a.M && l < a.Ny) {
                double2 x = ccast<double2>(v);
                if (o == 4) {
                    if (a.trA && r < a.nrhs) {
                        const double2 ta = a.trA[(size_t)r * a.Ny + l], tb = a.trB[(size_t)r * a.Ny + l];
                        x.x += a.tc * (tb.x - ta.x);
                        x.y += a.tc * (tb.y - ta.y);
                    }
                    a.pn[((size_t)g * a.P + c) * KP * 16 + red_pos<T>(lr, rn)] = ccast<V>(x);
                } else if (r < a.nrhs) {
                    const size_t at = (size_t)r * a.dst_rs + (size_t)l * a.dst_ls + a.oat[o];
                    if (a.base) x = cadd(x, a.base[at]);
                    a.dst[at] = x;
                }
            }
        }
    }
}

// Inputs of a sweep's strips in operand order: entries 1, 2 of every row from psi (upward) or
// the residual windows (downward); entry 0, the transmission source, is the previous strip's
// output (zero for the sweep's first strip).  Lanes of a wave take 16 right-hand sides x 4 rows
// of one strip, the four waves neighbouring strips (they share the cache lines of a row).
template <typename T>
__global__ void __launch_bounds__(NT) k_red_inputs(RedIn<T> a) {
    using V = cplx<T>;
    const int lane = threadIdx.x & 63, n = lane & 15, q4 = lane >> 4;
    const int s = a.s0 + 4 * blockIdx.z + (threadIdx.x >> 6), g = blockIdx.y;
    const int c = blockIdx.x / (a.Mp / 8), i8 = blockIdx.x % (a.Mp / 8);
    const int r = 16 * g + n;
    if (s >= a.s1 || r >= a.nrhs) return;
    V* p = a.p + (((size_t)s * a.G + g) * a.P + c) * 3 * a.Mp * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int lr = 8 * i8 + 4 * h + q4, l = c * a.M + lr;
        if (lr >= a.M || l >= a.Ny) continue;
        double2 x = cmk<double2>(0.0, 0.0), y = x;
        if (a.src) {
            const double2* src = a.src + ((size_t)r * a.Ny + l) * a.ls + (size_t)(s - a.s0) * a.cs + a.c0;
            x = src[0];
            y = src[1];
        }
        p[red_pos<T>(a.Mp + lr, n)] = ccast<V>(x);
        p[red_pos<T>(2 * a.Mp + lr, n)] = ccast<V>(y);
        if (s == a.sfirst) {
            double2 t = cmk<double2>(0.0, 0.0);
            if (a.trA) {
                const double2 ta = a.trA[(size_t)r * a.Ny + l], tb = a.trB[(size_t)r * a.Ny + l];
                t = cmk<double2>(a.tc * (tb.x - ta.x), a.tc * (tb.y - ta.y));
            }
            p[red_pos<T>(lr, n)] = ccast<V>(t);
        }
    }
}

__global__ void k_copy_win_cols(const double2* __restrict__ src, double2* __restrict__ dst, long nrows, long wrow, int c0,
                                int n) {
    const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (p >= nrows * n) return;
    const size_t at = (size_t)(p / n) * wrow + c0 + p % n;
    dst[at] = src[at];
}
__global__ void k_gather_win(const double2* __restrict__ field, const int* __restrict__ bw, int NI, long nrows, int Nx,
                             double2* __restrict__ win) {
    const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (p >= nrows * NI * 4) return;
    const long row = p / (4 * NI);
    const int j = (int)(p % (4 * NI)) >> 2, c = (int)(p & 3);
    win[((size_t)row * NI + j) * IWIN + c] = field[(size_t)row * Nx + bw[j] + c];
}
__global__ void k_iface_sum(const double2* __restrict__ vw, const double2* __restrict__ ww, const int* __restrict__ bw, int NI,
                            long nrows, int Nx, double2* __restrict__ out) {
    const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (p >= nrows * NI) return;
    const long row = p / NI;
    const int j = (int)(p % NI);
    const size_t at = (size_t)row * NI * IWIN + j * IWIN + 2;
    out[(size_t)row * Nx + bw[j] + 2] = cadd(vw[at], ww[at]);
}

// ---------------------------------------------------------------- build (FP64)
// A node is a run of fine chunks with the separators inside it eliminated; its block K holds
// the node's inverse from inputs (rows x TI input columns, then the couplings to the
// separators above and below, 64 columns each, scaled as the spikes X~, Y~) to outputs (rows
// x TI target columns, then all 64 columns of its first and of its last row).  Index of
// (column i, row lr) is i n + lr with n row slots, D = 6 n + 128; element (out, in) at in D + out.
struct RedBuild {
    const double2* F;        // factors of the batch's first slot, [slot][Ny][NSLOT][BLK]
    const double2* cy; const double2* by; const double2* ay; const double2* ayh;
    const double2* sax; const double2* saxh; const int* scol; const int* sW; const int* tcol;   // from that slot on
    const double* k2;
    int* err;
    double cond_max;         // of the separators eliminated in a join
    int Nx, Ny, m, P;        // fine chunks
    double ih2;
    __device__ const double2* slot(int u, int l, int sl) const { return F + (((size_t)u * Ny + l) * NSLOT + sl) * BLK; }
    // targets 0..2: beta_s .. beta_s + 2, 3..5: beta_{s+1} - 2 .. beta_{s+1}
    __device__ int tgt(int u, int o) const { return tcol[u * 8 + o]; }
    // inputs 0..2: beta_s - 1 .. beta_s + 1, 3..5: beta_{s+1} - 1 .. beta_{s+1} + 1
    __device__ int inp(int u, int i) const {
        const int q = tcol[u * 8 + (i < 3 ? 0 : 3)];
        return q < 0 ? -1 : i < 3 ? q - 1 + i : q + 1 + (i - 3);
    }
};

// Largest 1-norm condition estimate of a separator's Schur complement in a join; above it the strips
// stay with the block substitutions, which do not eliminate separators node by node.  Measured
// against extended precision on strips without PML near a resonance (162 rows): from chunks of 8
// rows, three levels of joins, the error of the reduced operator is 1.6 to 10 times the
// substitutions' at 3e3, 5 at 4e5, 25 at 4e7; from chunks of 48 (no join) it is theirs at any
// condition, so that leaves and the factorisation's own separators need no limit of their own.
// With PML the estimate stays below 4e4 (178 problems of 48 to 2000 points a side) and P below
// 1.03 times their error.  In complex64 the joins are in FP64 all the same, and the dense operator
// is the more accurate one at any condition at which either has a digit.
template <typename T> struct RedCond { static constexpr double max = 1e5; };
template <> struct RedCond<float> { static constexpr double max = 1e9; };

// 64 x 64 by 64 x 16 products of a chain: the block's A operands of this lane in registers
struct Chain {
    double2 g[16];
    const int n, q4, w;
    __device__ Chain(int lane, int w_) : n(lane & 15), q4(lane >> 4), w(w_) {}
    __device__ void load(const double2* G) {
        G += (size_t)q4 * WP + 16 * w + n;
#pragma unroll
        for (int s = 0; s < 16; ++s) g[s] = G[4 * s * WP];
    }
    // out = block x V, the block of the next product loaded between the products
    __device__ void mul(const double2 (*Vb)[16], const double2* next, double2 (&out)[4]) {
        const double2* Gn = next + (size_t)q4 * WP + 16 * w + n;
        md4 cr = {0, 0, 0, 0}, ci = cr;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const double2 x = g[s], v = Vb[4 * s + q4][n];
            cr = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v.x, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v.y, ci, 0, 0, 0);
            cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, v.y, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, v.x, ci, 0, 0, 0);
            g[s] = Gn[4 * s * WP];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = cmk<double2>(cr[j], ci[j]);
    }
};

// Leaf blocks: the fine chunk's inverse applied to unit vectors at its input columns, 16 rows'
// unit vectors of one input column per workgroup (forward from the first of those rows),
// block substitution with the chunk's G_l.  z holds the forward results until the backward
// pass.  Grid (fine chunks, TI x row groups, slots).
__global__ void __launch_bounds__(NT) k_red_leaf(RedBuild b, double2* __restrict__ K, double2* __restrict__ z) {
    __shared__ double2 Vs[2][WP][16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, q4 = lane >> 4;
    const int c = blockIdx.x, u = blockIdx.z, m = b.m, mg = (m + 15) / 16;
    const int in = blockIdx.y / mg, lg = blockIdx.y % mg;
    const int q = b.inp(u, in);
    const int r0 = c * m, r1 = c < b.P - 1 ? r0 + m - 1 : b.Ny;
    const int rs = r0 + 16 * lg;                          // first unit row
    if (q < 0 || rs >= r1) return;
    const int D = TI * m + 2 * WP;
    K += ((size_t)u * b.P + c) * D * D;
    z += ((((size_t)u * b.P + c) * gridDim.y + blockIdx.y) * m) * WP * 16;
    const int row0 = 16 * w + q4;                         // this lane's rows row0 + 4 j, column n
    int tmask[4] = {0, 0, 0, 0};
    for (int o = 0; o < TI; ++o)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (b.tgt(u, o) == row0 + 4 * j) tmask[j] |= 1 << o;
    const int ur = rs + n;                                // row of this column's unit vector
    const bool valid = ur < r1;
    double2* col = K + (size_t)(in * m + (valid ? ur - r0 : 0)) * D;
    auto emit = [&](int l, const double2 (&y)[4]) {
        if (!valid) return;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            for (int o = 0; o < TI; ++o)
                if (tmask[j] >> o & 1) col[o * m + (l - r0)] = y[j];
            if (l == r0) col[TI * m + row0 + 4 * j] = y[j];
            if (l == r1 - 1) col[TI * m + WP + row0 + 4 * j] = y[j];
        }
    };
    Chain ch(lane, w);
    ch.load(b.slot(u, rs, 0));
    double2 y[4];
    int buf = 0;
    for (int l = rs; l < r1; ++l, buf ^= 1) {
        const double2 cl = b.cy[l];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double2 e = cmk<double2>(l == ur && row0 + 4 * j == q ? 1.0 : 0.0, 0.0);
            Vs[buf][row0 + 4 * j][n] = l > rs ? csub(e, cmul(cl, y[j])) : e;
        }
        __syncthreads();
        // after the last forward row the backward pass starts with G_{r1-2}
        ch.mul(Vs[buf], b.slot(u, l + 1 < r1 ? l + 1 : max(r1 - 2, r0), 0), y);
#pragma unroll
        for (int j = 0; j < 4; ++j) z[((size_t)(l - r0) * WP + row0 + 4 * j) * 16 + n] = y[j];
    }
    emit(r1 - 1, y);
    for (int l = r1 - 2; l >= r0; --l, buf ^= 1) {
        const double2 bl = b.by[l];
        double2 zl[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            zl[j] = cmk<double2>(0.0, 0.0);
            if (l >= rs) zl[j] = z[((size_t)(l - r0) * WP + row0 + 4 * j) * 16 + n];
            Vs[buf][row0 + 4 * j][n] = y[j];
        }
        __syncthreads();
        double2 p[4];
        ch.mul(Vs[buf], b.slot(u, max(l - 1, r0), 0), p);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = csub(zl[j], cmul(bl, p[j]));
        emit(l, y);
    }
}

// The leaf blocks' coupling columns from the stored spikes.  Grid (fine chunks, 2 sides, slots).
__global__ void __launch_bounds__(NT) k_red_leaf_spikes(RedBuild b, double2* __restrict__ K) {
    const int c = blockIdx.x, side = blockIdx.y, u = blockIdx.z, m = b.m;
    const int r0 = c * m, r1 = c < b.P - 1 ? r0 + m - 1 : b.Ny;
    const int D = TI * m + 2 * WP;
    if (side == 0 ? c == 0 : c == b.P - 1) return;        // no separator there: zero columns
    K += ((size_t)u * b.P + c) * D * D + (size_t)(TI * m + side * WP) * D;
    for (int idx = threadIdx.x; idx < (r1 - r0) * TI * WP; idx += NT) {
        const int lr = idx % (r1 - r0), o = idx / (r1 - r0) % TI, k = idx / (r1 - r0) / TI;
        const int q = b.tgt(u, o);
        if (q >= 0) K[(size_t)k * D + o * m + lr] = b.slot(u, r0 + lr, 1 + side)[k * WP + q];
    }
    for (int idx = threadIdx.x; idx < BLK; idx += NT) {
        const int i = idx & (WP - 1), k = idx / WP;
        K[(size_t)k * D + TI * m + i] = b.slot(u, r0, 1 + side)[idx];
        K[(size_t)k * D + TI * m + WP + i] = b.slot(u, r1 - 1, 1 + side)[idx];
    }
}

// Joining two neighbouring nodes A, B (n row slots each) over the separator s between them:
//   S = T_s - c_s Y~A_{s-1} - b_s X~B_{s+1},  g = S^{-1}
// Grid (joined nodes, slots).
__global__ void __launch_bounds__(NT) k_red_schur(RedBuild b, const double2* __restrict__ K, int n, int nch,
                                                  double2* __restrict__ gout) {
    __shared__ GJShared sh;
    const int j2 = blockIdx.x, u = blockIdx.y;
    if (2 * j2 + 1 >= nch) return;
    const int D = TI * n + 2 * WP, s = (2 * j2 + 1) * n - 1, W = b.sW[u];
    const double2* KA = K + ((size_t)u * nch + 2 * j2) * D * D;
    const double2* KB = KA + (size_t)D * D;
    const int i = threadIdx.x & (WP - 1), g = threadIdx.x >> 6;
    double2 d = cmk<double2>(0.0, 0.0), xup = d, xlo = d;
    if (i < W) {
        const double2 axq = b.sax[(size_t)u * WP + i];
        const double2 e = b.saxh[(size_t)u * (WP + 1) + i + 1], wv = b.saxh[(size_t)u * (WP + 1) + i];
        d = cadd(cmul(axq, cadd(e, wv)), cmul(b.ay[s], cadd(b.ayh[s + 1], b.ayh[s])));
        d.x *= b.ih2; d.y *= b.ih2;
        d.x -= b.k2[(size_t)s * b.Nx + b.scol[(size_t)u * WP + i]];
        const double2 o = cmul(axq, e), q = cmul(axq, wv);
        xup = cmk<double2>(-o.x * b.ih2, -o.y * b.ih2);
        xlo = cmk<double2>(-q.x * b.ih2, -q.y * b.ih2);
    }
    const double2 cs = b.cy[s], bs = b.by[s];
    double2 M[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = g + 4 * r;
        double2 v = cmk<double2>(0.0, 0.0);
        if (i < W && j < W) {
            v = sel(j == i, d, sel(j == i + 1, xup, sel(j == i - 1, xlo, v)));
            v = csub(v, cmul(cs, KA[(size_t)(TI * n + WP + j) * D + TI * n + WP + i]));
            v = csub(v, cmul(bs, KB[(size_t)(TI * n + j) * D + TI * n + i]));
        }
        M[r] = v;
    }
    gj_invert_store(M, W, sh, gout + ((size_t)u * gridDim.x + j2) * BLK, nullptr, b.err, b.cond_max);
}

// Products of 64 x 64 tiles from LDS (leading dimension LDT, element (r, k) of X at k LDT + r,
// (k, c) of Y at c LDT + k): wave w rows 16 w .., four 16-column tiles.
constexpr int LDT = WP + 1;
__device__ inline void tile64(const double2* X, const double2* Y, md4 (&cr)[4], md4 (&ci)[4]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, q4 = lane >> 4;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) { cr[tt] = md4{0, 0, 0, 0}; ci[tt] = cr[tt]; }
#pragma unroll 4
    for (int s = 0; s < 16; ++s) {
        const double2 x = X[(4 * s + q4) * LDT + 16 * w + n];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const double2 y = Y[(16 * tt + n) * LDT + 4 * s + q4];
            cr[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, cr[tt], 0, 0, 0);
            ci[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.y, ci[tt], 0, 0, 0);
            cr[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, y.y, cr[tt], 0, 0, 0);
            ci[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, ci[tt], 0, 0, 0);
        }
    }
}

// x_s of the joined node for each of its inputs: Xs = g [-c_s A_last | E | -b_s B_first], 64 x D2.
// Grid (64-column tiles of D2, joined nodes, slots).
__global__ void __launch_bounds__(NT) k_red_xs(RedBuild b, const double2* __restrict__ K, int n, int nch,
                                               const double2* __restrict__ gin, double2* __restrict__ Xs) {
    __shared__ double2 G[WP * LDT];
    __shared__ double2 Y[WP * LDT];
    const int j2 = blockIdx.y, u = blockIdx.z;
    if (2 * j2 + 1 >= nch) return;
    const int D = TI * n + 2 * WP, n2 = 2 * n, D2 = TI * n2 + 2 * WP, s = (2 * j2 + 1) * n - 1;
    const double2* KA = K + ((size_t)u * nch + 2 * j2) * D * D;
    const double2* KB = KA + (size_t)D * D;
    const double2* g = gin + ((size_t)u * gridDim.y + j2) * BLK;
    const double2 cs = b.cy[s], bs = b.by[s];
    for (int idx = threadIdx.x; idx < BLK; idx += NT) {
        const int i = idx & (WP - 1), k = idx / WP, x = blockIdx.x * WP + k;
        G[k * LDT + i] = g[idx];
        double2 v = cmk<double2>(0.0, 0.0);
        if (x < D2) {
            const int e = x < TI * n2 ? x / n2 : x < TI * n2 + WP ? TI : TI + 1;
            const int lr = e < TI ? x % n2 : 0;
            if (e < TI && lr == n - 1) {
                v = cmk<double2>(i == b.inp(u, e) ? 1.0 : 0.0, 0.0);
            } else {
                const bool A = e < TI ? lr < n : e == TI;
                const size_t xc = e < TI ? (size_t)e * n + (A ? lr : lr - n) : (size_t)TI * n + (x - TI * n2);
                const double2 t = A ? KA[xc * D + TI * n + WP + i] : KB[xc * D + TI * n + i];
                const double2 f = A ? cs : bs;
                v = cmul(cmk<double2>(-f.x, -f.y), t);
            }
        }
        Y[k * LDT + i] = v;
    }
    __syncthreads();
    md4 cr[4], ci[4];
    tile64(G, Y, cr, ci);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nn = lane & 15, q4 = lane >> 4;
    Xs += ((size_t)u * gridDim.y + j2) * (size_t)D2 * WP;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
        const int x = blockIdx.x * WP + 16 * tt + nn;
        if (x < D2)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                Xs[(size_t)x * WP + 16 * w + q4 + 4 * j] = cmk<double2>(cr[tt][j], ci[tt][j]);
    }
}

// The joined node's block: A's and B's own entries minus their couplings to s times x_s, and
// x_s itself on row s (a last node without a partner is copied).  Grid (64-wide tiles of
// inputs, of outputs, joined nodes x slots).
__global__ void __launch_bounds__(NT) k_red_join(RedBuild b, const double2* __restrict__ K, int n, int nch, int nj,
                                                 const double2* __restrict__ Xs, double2* __restrict__ K2) {
    __shared__ double2 Um[WP * LDT];
    __shared__ double2 Y[WP * LDT];
    const int j2 = blockIdx.z % nj, u = blockIdx.z / nj;
    const bool two = 2 * j2 + 1 < nch;
    const int D = TI * n + 2 * WP, n2 = 2 * n, D2 = TI * n2 + 2 * WP;
    const double2* KA = K + ((size_t)u * nch + 2 * j2) * D * D;
    const double2* KB = KA + (size_t)D * D;
    K2 += ((size_t)u * nj + j2) * (size_t)D2 * D2;
    Xs += ((size_t)u * nj + j2) * (size_t)D2 * WP;
    // place of index x (input or output) of the joined node: child 0 (A), 1 (B), 2 (row s), 3 (none)
    auto place = [&](int x, int& at, int& e) {
        if (x >= D2) return 3;
        if (x < TI * n2) {
            e = x / n2;
            const int lr = x - e * n2;
            if (two && lr == n - 1) return 2;
            if (lr < n) { at = e * n + lr; return 0; }
            at = e * n + lr - n;
            return two ? 1 : 3;
        }
        const int k = x - TI * n2;
        at = TI * n + k;
        return two && k >= WP ? 1 : 0;
    };
    const int x0 = blockIdx.x * WP, y0 = blockIdx.y * WP;
    if (two) {
        for (int idx = threadIdx.x; idx < BLK; idx += NT) {
            const int i = idx & (WP - 1), k = idx / WP;
            int at = 0, e = 0;
            const int pl = place(y0 + i, at, e);
            double2 v = cmk<double2>(0.0, 0.0);
            if (pl == 0) v = KA[(size_t)(TI * n + WP + k) * D + at];
            if (pl == 1) v = KB[(size_t)(TI * n + k) * D + at];
            Um[k * LDT + i] = v;
            Y[k * LDT + i] = x0 + k < D2 ? Xs[(size_t)(x0 + k) * WP + i] : cmk<double2>(0.0, 0.0);
        }
        __syncthreads();
    }
    md4 cr[4], ci[4];
    if (two) tile64(Um, Y, cr, ci);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nn = lane & 15, q4 = lane >> 4;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
        const int x = x0 + 16 * tt + nn;
        int xat = 0, xe = 0;
        const int xp = place(x, xat, xe);
        if (x >= D2) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int y = y0 + 16 * w + q4 + 4 * j;
            int yat = 0, ye = 0;
            const int yp = place(y, yat, ye);
            if (y >= D2) continue;
            double2 v = cmk<double2>(0.0, 0.0);
            if (yp == 2) {
                const int q = b.tgt(u, ye);
                if (q >= 0) v = Xs[(size_t)x * WP + q];
            } else {
                if (xp == yp && xp < 2) v = (xp == 0 ? KA : KB)[(size_t)xat * D + yat];
                if (two && yp < 2) v = csub(v, cmk<double2>(cr[tt][j], ci[tt][j]));
            }
            K2[(size_t)x * D2 + y] = v;
        }
    }
}

// Sm, the inverse of the separators' Schur complement restricted to the coarse separators:
// the recurrences of the factored fine separators (z'_c = G'_c r_c - K_c z'_{c-1},
// x_c = z'_c - U'_c x_{c+1}) on 16 unit vectors of one coarse separator per workgroup.
// Grid (4 ns, slots).
template <typename T>
__global__ void __launch_bounds__(NT) k_red_sinv(RedBuild b, int kappa, int ns, double2* __restrict__ z,
                                                 cplx<T>* __restrict__ Sm) {
    using V = cplx<T>;
    __shared__ double2 Vs[2][WP][16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, q4 = lane >> 4;
    const int cc = blockIdx.x >> 2, u = blockIdx.y, col = 16 * (blockIdx.x & 3) + n;
    const int nsf = b.P - 1, c0 = kappa * (cc + 1) - 1;
    auto sep = [&](int c) { return c * b.m + b.m - 1; };
    z += ((size_t)u * gridDim.x + blockIdx.x) * nsf * WP * 16;
    Sm += (size_t)u * (64 * ns) * (size_t)(64 * ns);
    const int row0 = 16 * w + q4, kcol = 64 * cc + col;
    double2 y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        y[j] = b.slot(u, sep(c0), 0)[(size_t)col * WP + row0 + 4 * j];
        z[((size_t)c0 * WP + row0 + 4 * j) * 16 + n] = y[j];
    }
    Chain ch(lane, w);
    int buf = 0;
    // block of forward step c (slot 1 of separator c), then of the backward steps (slot 2)
    auto blk = [&](int c) { return c < nsf ? b.slot(u, sep(c), 1) : b.slot(u, sep(max(2 * nsf - 2 - c, 0)), 2); };
    ch.load(blk(c0 + 1));
    for (int c = c0 + 1; c < nsf; ++c, buf ^= 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) Vs[buf][row0 + 4 * j][n] = y[j];
        __syncthreads();
        ch.mul(Vs[buf], blk(c + 1), y);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            y[j] = cmk<double2>(-y[j].x, -y[j].y);
            z[((size_t)c * WP + row0 + 4 * j) * 16 + n] = y[j];
        }
    }
    auto emit = [&](int c) {
        if ((c + 1) % kappa) return;
        const int rc = (c + 1) / kappa - 1;               // coarse separator
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = row0 + 4 * j, tile = 4 * rc + (row >> 4);
            Sm[(size_t)tile * 16 * 64 * ns + red_pos<T>(kcol, row & 15)] = ccast<V>(y[j]);
        }
    };
    if ((nsf % kappa) == 0) emit(nsf - 1);
    for (int c = nsf - 2; c >= 0; --c, buf ^= 1) {
        double2 zl[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            zl[j] = cmk<double2>(0.0, 0.0);
            if (c >= c0) zl[j] = z[((size_t)c * WP + row0 + 4 * j) * 16 + n];
            Vs[buf][row0 + 4 * j][n] = y[j];
        }
        __syncthreads();
        double2 p[4];
        ch.mul(Vs[buf], blk(2 * nsf - 2 - max(c - 1, 0)), p);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = csub(zl[j], p[j]);
        emit(c);
    }
}

// combined inputs of a direction: the transmission source feeds two columns of a row
struct InCols { int a, b; };
__device__ inline InCols dir_in(int dir, int e) {
    if (dir == 0) return e == 0 ? InCols{0, 1} : e == 1 ? InCols{1, -1} : InCols{2, -1};
    return e == 0 ? InCols{4, 5} : e == 1 ? InCols{3, -1} : InCols{4, -1};
}
// outputs of a direction: plain target columns, and (o = 4) the next strip's transmission
// source, coefficient x (x[target t1] - x[target t0])
struct OutCols { int t, t0, t1; };
__device__ inline OutCols dir_out(int dir, int o) {
    if (dir == 0) {
        const int t[4] = {0, 1, 3, 4};
        return o < 4 ? OutCols{t[o], -1, -1} : OutCols{-1, 4, 5};
    }
    const int t[4] = {4, 5, 1, 2};
    return o < 4 ? OutCols{t[o], -1, -1} : OutCols{-1, 0, 1};
}

// Tm in operand order, from the coarse nodes' blocks.  Grid (chunk x 5 outputs x row groups,
// direction, slots).
template <typename T>
__global__ void __launch_bounds__(NT) k_red_pack_t(RedBuild b, const double2* __restrict__ K, int n, int M, int Mp,
                                                   int P, int ns, cplx<T>* __restrict__ Tm, size_t tsz) {
    using V = cplx<T>;
    const int per = Mp / 16, dir = blockIdx.y, u = blockIdx.z;
    const int lg = blockIdx.x % per, o = blockIdx.x / per % 5, c = blockIdx.x / per / 5;
    const int D = TI * n + 2 * WP, KP = 3 * Mp, Kt = KP + (ns ? 2 * WP : 0);
    K += ((size_t)u * P + c) * (size_t)D * D;
    Tm += ((size_t)u * 2 + dir) * tsz + (size_t)blockIdx.x * 16 * Kt;
    const OutCols oc = dir_out(dir, o);
    const double cf = dir == 0 ? -b.ih2 : b.ih2;
    const int row = threadIdx.x & 15, lr = 16 * lg + row;
    const bool closing = c < P - 1 && lr == M - 1;        // the separator closing the chunk
    const bool ok = lr < M && c * M + lr < b.Ny;
    const int qt = oc.t >= 0 ? b.tgt(u, oc.t) : -1, q0 = oc.t0 >= 0 ? b.tgt(u, oc.t0) : -1,
              q1 = oc.t1 >= 0 ? b.tgt(u, oc.t1) : -1;
    // entry of target t (its strip column q) on row lr from input x of the node
    for (int k = threadIdx.x >> 4; k < Kt; k += NT / 16) {
        double2 v = cmk<double2>(0.0, 0.0);
        if (ok && k < KP) {
            const int e = k / Mp, lk = k - e * Mp;
            if (!closing && lk < M) {
                const InCols ic = dir_in(dir, e);
                auto ent = [&](int t) {
                    double2 x = K[(size_t)(ic.a * n + lk) * D + t * n + lr];
                    if (ic.b >= 0) x = cadd(x, K[(size_t)(ic.b * n + lk) * D + t * n + lr]);
                    return x;
                };
                if (qt >= 0) v = ent(oc.t);
                else if (q0 >= 0) {
                    v = csub(ent(oc.t1), ent(oc.t0));
                    v.x *= cf; v.y *= cf;
                }
            }
        } else if (ok) {
            const int side = (k - KP) / WP, q = (k - KP) % WP;
            if (closing) {
                if (side == 1) {
                    if (qt >= 0) v.x = q == qt ? 1.0 : 0.0;
                    else if (q0 >= 0) v.x = q == q1 ? cf : q == q0 ? -cf : 0.0;
                }
            } else {
                auto ent = [&](int t) { return K[(size_t)(TI * n + side * WP + q) * D + t * n + lr]; };
                if (qt >= 0) { const double2 x = ent(oc.t); v = cmk<double2>(-x.x, -x.y); }
                else if (q0 >= 0) {
                    v = csub(ent(oc.t0), ent(oc.t1));
                    v.x *= cf; v.y *= cf;
                }
            }
        }
        Tm[red_pos<T>(k, row)] = ccast<V>(v);
    }
}

// Rm in operand order.  Grid (4 ns, direction, slots).
template <typename T>
__global__ void __launch_bounds__(NT) k_red_pack_r(RedBuild b, const double2* __restrict__ K, int n, int M, int Mp,
                                                   int P, int ns, cplx<T>* __restrict__ Rm, size_t rsz) {
    using V = cplx<T>;
    const int c = blockIdx.x >> 2, dir = blockIdx.y, u = blockIdx.z;
    const int D = TI * n + 2 * WP, KP = 3 * Mp, s = c * M + M - 1;
    const double2* KA = K + ((size_t)u * P + c) * (size_t)D * D;
    const double2* KB = KA + (size_t)D * D;
    Rm += ((size_t)u * 2 + dir) * rsz + (size_t)blockIdx.x * 16 * 2 * KP;
    const int row = threadIdx.x & 15, q = 16 * (blockIdx.x & 3) + row;
    const double2 cs = b.cy[s], bs = b.by[s];
    for (int k = threadIdx.x >> 4; k < 2 * KP; k += NT / 16) {
        const int half = k / KP, e = k % KP / Mp, lk = k % KP % Mp;
        const InCols ic = dir_in(dir, e);
        double2 v = cmk<double2>(0.0, 0.0);
        if (lk < M) {
            if (half == 0 && lk == M - 1) {
                v.x = q == b.inp(u, ic.a) || (ic.b >= 0 && q == b.inp(u, ic.b)) ? 1.0 : 0.0;
            } else {
                const double2* N = half ? KB : KA;
                const int at = half ? TI * n + q : TI * n + WP + q;
                double2 x = N[(size_t)(ic.a * n + lk) * D + at];
                if (ic.b >= 0) x = cadd(x, N[(size_t)(ic.b * n + lk) * D + at]);
                const double2 f = half ? bs : cs;
                v = cmul(cmk<double2>(-f.x, -f.y), x);
            }
        }
        Rm[red_pos<T>(k, row)] = ccast<V>(v);
    }
}

template <typename T, typename TL, int NC, int MODE>
void launch_mul_as(const RedArgs<T>& a, int tiles, int nc, hipStream_t st) {
    hipLaunchKernelGGL((k_red_mul<T, TL, NC, MODE>), dim3(8, (nc + NC - 1) / NC, (tiles + 7) / 8), dim3(NT), 0, st, a, tiles,
                       nc);
}
// Which tiles.  Up to 16 right-hand sides the 4 ns row tiles of Rm and Sm are fewer than the CUs
// and bound by their waves' FP64 products (64 cycles each): tiles of four right-hand sides
// make them 1/4 as long (1 right-hand side) or spread them over four times the CUs (16).  Sm
// at 2032 rows, one right-hand side: 10.3 -> 7.4 us, Rm 8.9 -> 6.9; 1032 rows, 16: 12.1 -> 9.6 and
// 6.4 -> 5.6.  Tm has tiles enough: four at a time only where there are no more (2032 rows: 19.7 ->
// 15.9 us; with 8 right-hand sides at 532 rows 7.4 -> 10.8, with 16 at 1032 13.0 -> 22).  Beyond 16,
// two groups of right-hand sides per workgroup read the matrix half as often, but not where the
// groups are needed to fill the chip: Sm, Rm at 2032 rows and 64 right-hand sides 11.0, 10.1 us
// with two, 7.2, 7.2 with one.  At 150 to 2032 rows and 2 to 128 right-hand sides, both precisions,
// a strip solve by these rules is within 4% of the fastest of their alternatives.
template <typename T, int MODE>
void launch_mul(const RedArgs<T>& a, int tiles, hipStream_t st) {
    if (a.G > 1 && (MODE == 2 || tiles * a.G > 512)) launch_mul_as<T, Wide<T>, 2, MODE>(a, tiles, a.G, st);
    else if (a.G > 1) launch_mul_as<T, Wide<T>, 1, MODE>(a, tiles, a.G, st);
    else if constexpr (std::is_same<T, double>::value) {
        if (MODE != 2 || a.nrhs <= 4) launch_mul_as<T, Quad<T>, 1, MODE>(a, tiles, (a.nrhs + 3) / 4, st);
        else launch_mul_as<T, Wide<T>, 1, MODE>(a, tiles, 1, st);
    } else launch_mul_as<T, Wide<T>, 1, MODE>(a, tiles, 1, st);
}

}  // namespace

template <typename T>
hipError_t launch_red_strip(const RedArgs<T>& a0, const cplx<T>* Tm, const cplx<T>* Rm, const cplx<T>* Sm,
                            hipStream_t st) {
    RedArgs<T> a = a0;
    if (a.ns) {
        a.A = Rm;
        launch_mul<T, 0>(a, 4 * a.ns, st);
        a.A = Sm;
        launch_mul<T, 1>(a, 4 * a.ns, st);
    }
    a.A = Tm;
    launch_mul<T, 2>(a, a.P * a.nout * (a.Mp / 16), st);
    return hipGetLastError();
}
template hipError_t launch_red_strip<float>(const RedArgs<float>&, const float2*, const float2*, const float2*, hipStream_t);
template hipError_t launch_red_strip<double>(const RedArgs<double>&, const double2*, const double2*, const double2*,
                                             hipStream_t);

template <typename T>
hipError_t launch_red_inputs(const RedIn<T>& a, hipStream_t st) {
    hipLaunchKernelGGL((k_red_inputs<T>), dim3(a.P * (a.Mp / 8), a.G, (a.s1 - a.s0 + 3) / 4), dim3(NT), 0, st, a);
    return hipGetLastError();
}
template hipError_t launch_red_inputs<float>(const RedIn<float>&, hipStream_t);
template hipError_t launch_red_inputs<double>(const RedIn<double>&, hipStream_t);

hipError_t launch_copy_win_cols(const double2* src, double2* dst, long nrows, long wrow, int c0, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_copy_win_cols, dim3((unsigned)((nrows * n + NT - 1) / NT)), dim3(NT), 0, st, src, dst, nrows, wrow,
                       c0, n);
    return hipGetLastError();
}
hipError_t launch_gather_win(const double2* field, const int* bw, int J, long nrows, int Nx, double2* win, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_win, dim3((unsigned)((nrows * (J - 1) * 4 + NT - 1) / NT)), dim3(NT), 0, st, field, bw, J - 1,
                       nrows, Nx, win);
    return hipGetLastError();
}
hipError_t launch_iface_sum(const double2* vw, const double2* ww, const int* bw, int J, long nrows, int Nx,
                            double2* out, hipStream_t st) {
    hipLaunchKernelGGL(k_iface_sum, dim3((unsigned)((nrows * (J - 1) + NT - 1) / NT)), dim3(NT), 0, st, vw, ww, bw, J - 1,
                       nrows, Nx, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- plan and build (host side)
RedPlan red_plan(const Chunks& ch, int Ny) {
    // kappa: the power of two that leaves the fewest matrix values per strip and direction
    // (chunks of at most 128 rows, so that the build's blocks stay small): larger chunks
    // cost 15 M values per row in Tm, smaller ones (64 ns)^2 in Sm.  2032 rows: M = 32 21 M
    // values, 64 7.9 M, 128 7.5 M; 1032: 5.0, 3.0, 3.1; a launch weighs as much as the
    // 1.5 M values read in its 3 us.
    RedPlan best;
    double bc = 0.0;
    if (ch.m > 128) return best;
    for (int lev = 0, kap = 1; lev < 8; ++lev, kap *= 2) {
        RedPlan p;
        p.kappa = kap;
        p.levels = lev;
        p.M = kap * ch.m;
        if (lev > 0 && p.M > 128) break;
        p.P = (ch.P + kap - 1) / kap;
        p.ns = p.P - 1;
        if (p.P == 1) p.M = std::min(p.M, Ny);
        p.Mp = (p.M + 15) / 16 * 16;
        p.n = kap * ch.m;
        const int K = 3 * p.Mp + (p.ns ? 2 * WP : 0);
        p.tsz = (size_t)p.P * 5 * p.Mp * K;
        p.rsz = (size_t)p.ns * 64 * 6 * p.Mp;
        p.ssz = (size_t)64 * p.ns * 64 * p.ns;
        const double cost = (double)p.tsz + p.rsz + p.ssz + (p.ns ? 3e6 : 0.0);
        if (lev == 0 || cost < bc) { best = p; bc = cost; }
        if (p.P == 1) break;
    }
    return best;
}

namespace {
size_t leaf_z_elems(const Chunks& ch) { return (size_t)ch.P * TI * ((ch.m + 15) / 16) * ch.m * WP * 16; }
}  // namespace

RedBuildSize red_build_size(const RedPlan& p, const Chunks& ch, int nfac) {
    // per slot: the two largest levels' blocks, x_s and inverses of a join, the chains' results
    RedBuildSize s;
    size_t kmax = 0, xmax = 0, gmax = 0;
    for (int lev = 0, n = ch.m, P = ch.P; lev <= p.levels; ++lev, n *= 2, P = (P + 1) / 2) {
        const size_t D = (size_t)TI * n + 2 * WP;
        kmax = std::max(kmax, (size_t)P * D * D);
        if (lev) { xmax = std::max(xmax, (size_t)P * D * WP); gmax = std::max(gmax, (size_t)P * BLK); }
    }
    s.K = kmax;
    s.X = xmax;
    s.g = gmax;
    s.z = std::max(leaf_z_elems(ch), (size_t)4 * p.ns * std::max(ch.P - 1, 0) * WP * 16);
    const size_t per = (2 * s.K + s.X + s.g + s.z) * sizeof(double2);
    // slots per batch: about 2 GB of workspace (enough workgroups to fill the chip)
    s.batch = (int)std::max<size_t>(1, std::min<size_t>((size_t)nfac, ((size_t)2 << 30) / per));
    s.bytes = per * s.batch;
    return s;
}

template <typename T>
hipError_t launch_red_build(const RedPlan& p, const RedBuildSize& sz, const DevTables& t, const Geom& g,
                            const Chunks& ch, int nfac, const double2* F64, double2* ws, int* err, cplx<T>* Tm,
                            cplx<T>* Rm, cplx<T>* Sm, hipStream_t st) {
    for (int u0 = 0; u0 < nfac; u0 += sz.batch) {
        const int nu = std::min(sz.batch, nfac - u0);
        RedBuild b;
        b.F = F64 + (size_t)u0 * g.Ny * NSLOT * BLK;
        b.cy = t.cy; b.by = t.by; b.ay = t.ay; b.ayh = t.ayh; b.k2 = t.k2;
        b.sax = t.sax + (size_t)u0 * WP; b.saxh = t.saxh + (size_t)u0 * (WP + 1);
        b.scol = t.scol + (size_t)u0 * WP; b.sW = t.sW + u0; b.tcol = t.tcol + (size_t)u0 * 8;
        b.err = err;
        b.cond_max = RedCond<T>::max;
        b.Nx = g.Nx; b.Ny = g.Ny; b.m = ch.m; b.P = ch.P; b.ih2 = 1.0 / (g.h * g.h);
        double2* K = ws;
        double2* K2 = K + sz.K * sz.batch;
        double2* X = K2 + sz.K * sz.batch;
        double2* gi = X + sz.X * sz.batch;
        double2* z = gi + sz.g * sz.batch;
        int n = ch.m, P = ch.P;
        const size_t D0 = (size_t)TI * n + 2 * WP;
        hipError_t e = hipMemsetAsync(K, 0, (size_t)nu * P * D0 * D0 * sizeof(double2), st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_red_leaf, dim3(P, TI * ((n + 15) / 16), nu), dim3(NT), 0, st, b, K, z);
        hipLaunchKernelGGL(k_red_leaf_spikes, dim3(P, 2, nu), dim3(NT), 0, st, b, K);
        for (int lev = 0; lev < p.levels; ++lev) {
            const int nj = (P + 1) / 2, D2 = TI * 2 * n + 2 * WP, nt = (D2 + WP - 1) / WP;
            hipLaunchKernelGGL(k_red_schur, dim3(nj, nu), dim3(NT), 0, st, b, K, n, P, gi);
            hipLaunchKernelGGL(k_red_xs, dim3(nt, nj, nu), dim3(NT), 0, st, b, K, n, P, gi, X);
            hipLaunchKernelGGL(k_red_join, dim3(nt, nt, nj * nu), dim3(NT), 0, st, b, K, n, P, nj, X, K2);
            std::swap(K, K2);
            n *= 2;
            P = nj;
        }
        hipLaunchKernelGGL((k_red_pack_t<T>), dim3(P * 5 * (p.Mp / 16), 2, nu), dim3(NT), 0, st, b, K, n, p.M, p.Mp,
                           P, p.ns, Tm + (size_t)u0 * 2 * p.tsz, p.tsz);
        if (p.ns) {
            hipLaunchKernelGGL((k_red_pack_r<T>), dim3(4 * p.ns, 2, nu), dim3(NT), 0, st, b, K, n, p.M, p.Mp, P,
                               p.ns, Rm + (size_t)u0 * 2 * p.rsz, p.rsz);
            hipLaunchKernelGGL((k_red_sinv<T>), dim3(4 * p.ns, nu), dim3(NT), 0, st, b, p.kappa, p.ns, z,
                               Sm + (size_t)u0 * p.ssz);
        }
    }
    return hipGetLastError();
}
template hipError_t launch_red_build<float>(const RedPlan&, const RedBuildSize&, const DevTables&, const Geom&,
                                            const Chunks&, int, const double2*, double2*, int*, float2*, float2*,
                                            float2*, hipStream_t);
template hipError_t launch_red_build<double>(const RedPlan&, const RedBuildSize&, const DevTables&, const Geom&,
                                             const Chunks&, int, const double2*, double2*, int*, double2*, double2*,
                                             double2*, hipStream_t);

}  // namespace helm
