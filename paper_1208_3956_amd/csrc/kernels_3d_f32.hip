// Complex64 slab factorisation of the mixed-precision 3-D path (the same block recursion
// along y as the FP64 one, Sec. 2.2 with the 7-point stencil):
//     S_l = T_l - c_l b_{l-1} G_{l-1} - b_l c_{l+1} G_{l+1},  G_l = S_l^{-1},
// with one of the two terms on the planes below and above the middle one, both on it.
// Each S_l is built over its own slot of the stored factor and inverted in place by
// blocked Gauss-Jordan elimination with pivoting only inside the 64 x 64 diagonal blocks:
// for the column block K,
//     P = A_KK^{-1}                                   (register Gauss-Jordan, FP64)
//     C = A(:, K) - E_K,   R = P [A(K, :) with A_KK := I]
//     A := A_mod - C R,    A_mod = A with the column block K replaced by E_K,
// which leaves A_KK = P, A(K, J) = P A(K, J), A(I, K) = -A(I, K) P and
// A(I, J) -= A(I, K) P A(K, J): one step of block Gauss-Jordan.  After the last block A
// holds S^{-1} with no permutation to undo.  The rows of block K are written as R
// directly rather than through the product (in FP32 that form would cancel to an error of
// order eps cond(A_KK)).  The update is a rank-128 (64) complex GEMM on
// v_mfma_f32_16x16x4f32 with three real products per complex one (Gauss's form),
// accumulated in FP32.
// Without a search over the whole column the elimination relies on well-conditioned
// diagonal blocks: every inverted block's 1-norm condition number is checked, and the
// factorisation reports it (err bit 2) so that the caller can redo the slab factor with
// the FP64 Gauss-Jordan with partial pivoting over the whole column.
#include "helm_internal.hpp"
#include "gj_register.hpp"

namespace helm {

namespace {

using namespace gjr;

typedef float mf4 __attribute__((ext_vector_type(4)));

constexpr double COND_MAX = 1e6;   // largest accepted 1-norm condition of a diagonal block
// strides of the work arrays, one set per matrix of a call (the same for 64- and 128-wide blocks)
constexpr size_t WSTR = 8 * (size_t)BLK;   // FP64 scratch blocks
constexpr size_t PSTR = 128 * 128;         // P
__host__ __device__ inline size_t cstr(int Bp) { return (size_t)128 * Bp; }   // C and R

// The matrices of a call: plane l0 of the ns slabs, then plane l1 of the ns slabs (the
// elimination's two ends), slabs `stride` entries apart
struct Planes {
    float2* F;
    size_t stride;
    int ns, l0, l1;
    __device__ int slab(int u) const { return u < ns ? u : u - ns; }
    __device__ int plane(int u) const { return u < ns ? l0 : l1; }
    __device__ float2* at(int u, int Bp) const { return F + slab(u) * stride + (size_t)plane(u) * Bp * Bp; }
};

// S_l = T_l - c_l b_{l-1} G_{l-1} (low) - b_l c_{l+1} G_{l+1} (up) into the plane-l slot of
// every slab (below, above: bit 0 for plane l0, bit 1 for l1) (identity on the padding); the neighbour planes' slots are already inverted.  T
// in FP64, rounded.
__global__ void __launch_bounds__(256) k3f_build_S(Fac3Args a, Planes F, int below, int above) {
    const int u = blockIdx.y, s = F.slab(u), l = F.plane(u);
    const bool low = below >> (u >= F.ns) & 1, up = above >> (u >= F.ns) & 1;
    const size_t BB = (size_t)a.Bp * a.Bp;
    const int W = a.sW[s], B = W * a.Nz;
    float2* S = F.at(u, a.Bp);
    double2 cb = make_double2(0.0, 0.0), bc = cb;
    if (low) cb = cmul(a.cy[l], a.by[l - 1]);
    if (up) bc = cmul(a.by[l], a.cy[l + 1]);
    const double2 ydiag = cmul(a.ay[l], cadd(a.ayh[l + 1], a.ayh[l]));
    const double2* sax = a.sax + (size_t)s * WP;
    const double2* saxh = a.saxh + (size_t)s * (WP + 1);
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < BB; e += (size_t)gridDim.x * blockDim.x) {
        const int col = (int)(e / a.Bp), row = (int)(e % a.Bp);
        double2 v = make_double2(0.0, 0.0);
        if (row < B && col < B) {
            if (low) v = csub(v, cmul(cb, ccast<double2>((S - BB)[e])));
            if (up) v = csub(v, cmul(bc, ccast<double2>((S + BB)[e])));
            const int xr = row % W, zr = row / W, xc = col % W, zc = col / W;
            double2 t = make_double2(0.0, 0.0);
            if (row == col) {
                const double2 xd = cmul(sax[xr], cadd(saxh[xr + 1], saxh[xr]));
                const double2 zd = cmul(a.az[zr], cadd(a.azh[zr + 1], a.azh[zr]));
                t = cadd(cadd(xd, ydiag), zd);
                t.x *= a.ih2; t.y *= a.ih2;
                const int gx = a.scol[(size_t)s * WP + xr];
                t.x -= a.k2[((size_t)zr * a.Ny + l) * a.Nx + gx];
            } else if (zr == zc && (xc == xr + 1 || xc == xr - 1)) {
                t = cmul(sax[xr], xc == xr + 1 ? saxh[xr + 1] : saxh[xr]);
                t.x *= -a.ih2; t.y *= -a.ih2;
            } else if (xr == xc && (zc == zr + 1 || zc == zr - 1)) {
                t = cmul(a.az[zr], zc == zr + 1 ? a.azh[zr + 1] : a.azh[zr]);
                t.x *= -a.ih2; t.y *= -a.ih2;
            }
            v = cadd(v, t);
        } else if (row == col) {
            v = make_double2(1.0, 0.0);
        }
        S[e] = make_float2((float)v.x, (float)v.y);
    }
}

// The 32 x 32 quadrant at (I0, J0) of A - C R (the block column K, kcol: I - C R) by one wave, the
// even and the odd rows and columns as MFMA tiles.
template <int NB>
__device__ __attribute__((always_inline)) inline void update_quadrant(float2* A, const float2* cb, const float2* rb, int Bp, int I0,
                                                                      int J0, bool kcol) {
    const int lane = threadIdx.x & 63, n = lane & 15, q4 = lane >> 4;
    const float2* cp = cb + (size_t)q4 * Bp + I0 + 2 * n;
    const float2* rp = rb + (size_t)q4 * Bp + J0 + 2 * n;
    // complex products by three real ones (x1 = -sum Cr Rr, x2 = sum Ci Ri,
    // x3 = -sum (Cr + Ci)(Rr + Ri)):  Re = A.r + x1 + x2,  Im = A.i + x3 - x1 + x2
    mf4 x1[2][2], x2[2][2], x3[2][2];
#pragma unroll
    for (int ia = 0; ia < 2; ++ia)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            x1[ia][jb] = mf4{0.f, 0.f, 0.f, 0.f};
            x2[ia][jb] = x1[ia][jb];
            x3[ia][jb] = x1[ia][jb];
        }
    constexpr int D = 4, NK = NB / 4;                   // ring of k-steps, D - 1 ahead
    float2 c[D][2], r[D][2];
    auto load = [&](int d, int kb) {
        const size_t o = (size_t)(kb < NK ? kb : NK - 1) * 4 * Bp;
        const float4 x = *reinterpret_cast<const float4*>(cp + o), y = *reinterpret_cast<const float4*>(rp + o);
        c[d][0] = make_float2(x.x, x.y);
        c[d][1] = make_float2(x.z, x.w);
        r[d][0] = make_float2(y.x, y.y);
        r[d][1] = make_float2(y.z, y.w);
    };
    auto steps = [&](int from, int to) {
        for (int kb = from; kb < to; kb += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load((d + D - 1) % D, kb + d + D - 1);
                float cs[2], rs[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) { cs[u] = c[d][u].x + c[d][u].y; rs[u] = r[d][u].x + r[d][u].y; }
#pragma unroll
                for (int ia = 0; ia < 2; ++ia)
#pragma unroll
                    for (int jb = 0; jb < 2; ++jb) {
                        x1[ia][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(c[d][ia].x, r[d][jb].x, x1[ia][jb], 0, 0, 0);
                        x2[ia][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(c[d][ia].y, r[d][jb].y, x2[ia][jb], 0, 0, 0);
                        x3[ia][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[ia], rs[jb], x3[ia][jb], 0, 0, 0);
                    }
            }
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, d);
    steps(0, NK - 8);
    // A's entries are read eight steps before they are needed: earlier, the first steps wait for memory
    float4 av[2][4];                                    // column J0 + 2 n + jb, rows I0 + 8 q4 + 2 j, + 1
    float4* at[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        at[jb] = reinterpret_cast<float4*>(A + (size_t)(J0 + 2 * n + jb) * Bp + I0 + 8 * q4);
#pragma unroll
        for (int j = 0; j < 4; ++j) av[jb][j] = at[jb][j];
    }
    steps(NK - 8, NK);
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float4 a0 = av[jb][j];
            if (kcol) {
                const int d = J0 + 2 * n + jb - (I0 + 8 * q4 + 2 * j);
                a0 = make_float4(d == 0 ? 1.f : 0.f, 0.f, d == 1 ? 1.f : 0.f, 0.f);
            }
            at[jb][j] = make_float4(a0.x - x1[0][jb][j] + x2[0][jb][j], a0.y - x3[0][jb][j] + x1[0][jb][j] + x2[0][jb][j],
                                    a0.z - x1[1][jb][j] + x2[1][jb][j], a0.w - x3[1][jb][j] + x1[1][jb][j] + x2[1][jb][j]);
        }
}

// The diagonal block at k0 (NB wide) of slab s brought up to date with the elimination of the 128
// columns before it: its tiles of that update (Cb null: nothing to do)
template <int NB>
__device__ __attribute__((always_inline)) inline void update_diag(float2* A, const float2* Cb, const float2* Rb, int Bp, int k0,
                                                                  int s) {
    if (!Cb) return;
    const int w = threadIdx.x >> 6;
    for (int q = 0; q < (NB / 64) * (NB / 64); ++q)
        update_quadrant<128>(A, Cb + (size_t)s * cstr(Bp), Rb + (size_t)s * cstr(Bp), Bp, k0 + 64 * (q & 1) + 32 * (w & 1),
                             k0 + 64 * (q >> 1) + 32 * (w >> 1), false);
    __syncthreads();
}

// P = A_KK^{-1} for the diagonal block at k0 of every slab (one workgroup per slab, the
// block in registers, FP64), stored column-major (leading dimension 64) in FP64 and
// complex64.  err bit 1: zero or non-finite pivot; bit 2: 1-norm condition above COND_MAX.
__global__ void __launch_bounds__(256) k3f_diag_inv(Planes F, int Bp, int k0,
                                                   const float2* __restrict__ Cb, const float2* __restrict__ Rb,
                                                   double2* __restrict__ Pd, float2* __restrict__ Pf,
                                                   int* __restrict__ err) {
    __shared__ GJShared sh;
    __shared__ double na[4][64], np[4][64];
    __builtin_amdgcn_s_setprio(3);
    const int s = blockIdx.x;
    float2* A = F.at(s, Bp);
    update_diag<64>(A, Cb, Rb, Bp, k0, s);
    const int i = threadIdx.x & 63, g = threadIdx.x >> 6;
    double2 M[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float2 v = A[(size_t)(k0 + g + 4 * r) * Bp + k0 + i];
        M[r] = make_double2(v.x, v.y);
    }
    double2* pd = Pd + (size_t)s * WSTR;
    gj_invert_store(M, WP, sh, pd, Pf + (size_t)s * PSTR, err);
    {
        // column sums of |A_KK| and |P|: thread (column c, quarter h) sums 16 rows
        const int c = threadIdx.x & 63, h = threadIdx.x >> 6;
        double sa = 0.0, sp = 0.0;
#pragma unroll 4
        for (int r = 16 * h; r < 16 * h + 16; ++r) {
            const float2 v = A[(size_t)(k0 + c) * Bp + k0 + r];
            sa += sqrt((double)v.x * v.x + (double)v.y * v.y);
            const double2 p = pd[(size_t)c * WP + r];
            sp += sqrt(p.x * p.x + p.y * p.y);
        }
        na[h][c] = sa;
        np[h][c] = sp;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        // the maxima over the columns by one wave
        const int c = threadIdx.x;
        double ma = na[0][c] + na[1][c] + na[2][c] + na[3][c];
        double mp = np[0][c] + np[1][c] + np[2][c] + np[3][c];
        for (int off = 32; off > 0; off >>= 1) {
            ma = fmax(ma, __shfl_xor(ma, off));
            mp = fmax(mp, __shfl_xor(mp, off));
        }
        if (c == 0 && !(ma * mp <= COND_MAX)) atomicOr(err, 2);
    }
}

// P = A_KK^{-1} for a 128 x 128 diagonal block from its 64 x 64 blocks [A11 A12; A21 A22]:
//     P11 = A11^{-1},  S = A22 - A21 P11 A12,  P22 = S^{-1},
//     P12 = -P11 A12 P22,  P21 = -P22 A21 P11,  P11 <- P11 - P12 A21 P11
// (pivoting inside the two 64 x 64 inverses), in FP64, one workgroup per slab, with eight
// 64 x 64 scratch blocks per slab in global memory; P is stored complex64, column-major
// (leading dimension 128).  err bits as in the 64-wide kernel.
__global__ void __launch_bounds__(256) k3f_diag_inv128(Planes F, int Bp, int k0,
                                                      const float2* __restrict__ Cb, const float2* __restrict__ Rb,
                                                      double2* __restrict__ Wd, float2* __restrict__ Pf,
                                                      int* __restrict__ err) {
    __shared__ GJShared sh;
    __shared__ double na[4], np[4];
    __builtin_amdgcn_s_setprio(3);                       // beside the update's waves
    const int s = blockIdx.x, t = threadIdx.x;
    float2* A = F.at(s, Bp);
    update_diag<128>(A, Cb, Rb, Bp, k0, s);
    double2* W = Wd + (size_t)s * WSTR;
    double2 *A12 = W, *A21 = W + BLK, *A22 = W + 2 * BLK, *P11 = W + 3 * BLK;
    double2 *T1 = W + 4 * BLK, *P22 = W + 5 * BLK, *T2 = W + 6 * BLK, *P12 = W + 7 * BLK;
    auto at = [&](int r, int c) {
        const float2 v = A[(size_t)(k0 + c) * Bp + k0 + r];
        return make_double2(v.x, v.y);
    };
#pragma unroll 8
    for (int e = t; e < BLK; e += 256) {
        const int r = e % WP, c = e / WP;
        A12[e] = at(r, 64 + c);
        A21[e] = at(64 + r, c);
        A22[e] = at(64 + r, 64 + c);
    }
    const int i = t & 63, g = t >> 6;
    const double2 one = make_double2(1.0, 0.0), mone = make_double2(-1.0, 0.0);
    double2 M[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) M[r] = at(i, g + 4 * r);
    gj_invert_store(M, WP, sh, P11, nullptr, err);                 // ends with a barrier
    gemm64_mfma(T1, WP, P11, WP, A12, WP, one, nullptr, 0);        // T1 = P11 A12
    gemm64_mfma(A22, WP, A21, WP, T1, WP, mone, A22, WP);          // S = A22 - A21 T1
#pragma unroll
    for (int r = 0; r < 16; ++r) M[r] = A22[(size_t)(g + 4 * r) * WP + i];
    gj_invert_store(M, WP, sh, P22, nullptr, err);
    gemm64_mfma(P12, WP, T1, WP, P22, WP, mone, nullptr, 0);       // P12 = -T1 P22
    gemm64_mfma(T2, WP, A21, WP, P11, WP, one, nullptr, 0);        // T2 = A21 P11
    gemm64_mfma(A21, WP, P22, WP, T2, WP, mone, nullptr, 0);       // P21 = -P22 T2 (over A21)
    gemm64_mfma(P11, WP, P12, WP, T2, WP, mone, P11, WP);          // P11 = P11 - P12 T2
    float2* P = Pf + (size_t)s * PSTR;
#pragma unroll 8
    for (int e = t; e < 128 * 128; e += 256) {
        const int r = e % 128, c = e / 128;
        const double2* src = r < 64 ? (c < 64 ? P11 : P12) : (c < 64 ? A21 : P22);
        const double2 v = src[(size_t)(c & 63) * WP + (r & 63)];
        P[e] = make_float2((float)v.x, (float)v.y);
    }
    __syncthreads();
    // column 1-norms of A_KK and P, a column per wave at a time (a thread per column reads 128 lines
    // at once: 30 us)
    double ma = 0.0, mp = 0.0;
#pragma unroll 4
    for (int c = 32 * g; c < 32 * g + 32; ++c) {
        double sa = 0.0, sp = 0.0;
#pragma unroll
        for (int r = i; r < 128; r += 64) {
            const double2 v = at(r, c);
            const float2 q = P[(size_t)c * 128 + r];
            sa += sqrt(v.x * v.x + v.y * v.y);
            sp += sqrt((double)q.x * q.x + (double)q.y * q.y);
        }
        ma = fmax(ma, wave_sum(sa));
        mp = fmax(mp, wave_sum(sp));
    }
    if (i == 0) { na[g] = ma; np[g] = mp; }
    __syncthreads();
    if (t == 0) {
        for (int q = 1; q < 4; ++q) { ma = fmax(ma, na[q]); mp = fmax(mp, np[q]); }
        if (!(ma * mp <= COND_MAX)) atomicOr(err, 2);
    }
}

// The operands of the update for the column block K = k0 .. k0 + NB - 1 (grid: RCW-column
// tiles x slabs):
//   C(i, k) = A(i, k0 + k) - [i = k0 + k]     rows of tile jt,  stored Cb[s][k][Bp]
//   R(k, j) = sum_m P(k, m) A(k0 + m, j)      columns of tile jt, R(:, K) = P, Rb[s][k][Bp]
// P is NB x NB, column-major (leading dimension NB).  The NB x RCW x NB product runs on
// v_mfma_f32_16x16x4f32: wave w computes NB/4 rows of R from NB/4 w on, P read in lane layout from
// global memory eight k-steps ahead, the A block from LDS.  The two tiles of a pair hold the
// even and the odd rows (columns), so that a lane's two operands (results) are one 16-byte access.
// Bound by latency, one short round of workgroups: 32 columns, 2 to 3 workgroups a CU (15 slabs of
// 1344 unknowns, 128 columns eliminated: 61 us with 64 columns and loads where they are
// used, 38 us).
constexpr int RCW = 32;                // columns of a workgroup of k3f_rc
template <int NB>
__global__ void __launch_bounds__(256) k3f_rc(Planes F, int Bp, int k0, const float2* __restrict__ Pf,
                                             float2* __restrict__ Cb, float2* __restrict__ Rb) {
    constexpr int NK = NB / 4, D = 8, CL = NB / 16, AL = RCW * NB / 512;
    __shared__ float2 As[RCW][NB + 1];  // As[j][m] = A(k0 + m, J0 + j)
    const int s = blockIdx.y, J0 = blockIdx.x * RCW, t = threadIdx.x;
    const float2* A = F.at(s, Bp);
    float2* cb = Cb + (size_t)s * cstr(Bp);
    float2* rb = Rb + (size_t)s * cstr(Bp);
    const float2* P = Pf + (size_t)s * PSTR;
    const bool own = J0 >= k0 && J0 < k0 + NB;
    // C rows of this tile and the A block, two values a load, all loads before the first use
    const int ci = J0 + 2 * (t & 15), ck = t >> 4, am = 2 * (t % (NB / 2)), aj = t / (NB / 2);
    float4 cv[CL], xv[AL];
#pragma unroll
    for (int q = 0; q < AL; ++q)
        xv[q] = *reinterpret_cast<const float4*>(A + (size_t)(J0 + aj + q * (512 / NB)) * Bp + k0 + am);
#pragma unroll
    for (int q = 0; q < CL; ++q) cv[q] = *reinterpret_cast<const float4*>(A + (size_t)(k0 + ck + 16 * q) * Bp + ci);
#pragma unroll
    for (int q = 0; q < AL; ++q) {
        As[aj + q * (512 / NB)][am] = make_float2(xv[q].x, xv[q].y);
        As[aj + q * (512 / NB)][am + 1] = make_float2(xv[q].z, xv[q].w);
    }
#pragma unroll
    for (int q = 0; q < CL; ++q) {
        const int k = ck + 16 * q;
        if (ci == k0 + k) cv[q].x -= 1.0f;
        if (ci + 1 == k0 + k) cv[q].z -= 1.0f;
        *reinterpret_cast<float4*>(cb + (size_t)k * Bp + ci) = cv[q];
    }
    if (own) {
        for (int e = t; e < NB * RCW; e += 256) {
            const int k = e / RCW, jj = e % RCW;
            rb[(size_t)k * Bp + J0 + jj] = P[(size_t)(J0 - k0 + jj) * NB + k];
        }
        return;
    }
    __syncthreads();
    // wave w: NB / 4 rows, as pairs of 16-row tiles of even and odd rows where there are two
    constexpr int RW = NB / 64;
    const int lane = t & 63, w = t >> 6, n = lane & 15, q4 = lane >> 4;
    mf4 re[RW][2], im[RW][2];
#pragma unroll
    for (int ra = 0; ra < RW; ++ra)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) { re[ra][jb] = mf4{0.f, 0.f, 0.f, 0.f}; im[ra][jb] = re[ra][jb]; }
    const float2* pp = P + (size_t)q4 * NB + 16 * RW * w + RW * n;     // P(RW (16 w + n) + ra, 4 ks + q4)
    float2 a[D][RW];
    auto load = [&](int d, int ks) {
        const float2* q = pp + (size_t)4 * (ks < NK ? ks : NK - 1) * NB;
        if constexpr (RW == 2) {
            const float4 x = *reinterpret_cast<const float4*>(q);
            a[d][0] = make_float2(x.x, x.y);
            a[d][1] = make_float2(x.z, x.w);
        } else {
            a[d][0] = *q;
        }
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, d);
    for (int kb = 0; kb < NK; kb += D)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            load((d + D - 1) % D, kb + d + D - 1);
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const float2 b = As[2 * n + jb][4 * (kb + d) + q4];
#pragma unroll
                for (int ra = 0; ra < RW; ++ra) {
                    re[ra][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][ra].x, b.x, re[ra][jb], 0, 0, 0);
                    im[ra][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][ra].x, b.y, im[ra][jb], 0, 0, 0);
                    re[ra][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a[d][ra].y, b.y, re[ra][jb], 0, 0, 0);
                    im[ra][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][ra].y, b.x, im[ra][jb], 0, 0, 0);
                }
            }
        }
#pragma unroll
    for (int ra = 0; ra < RW; ++ra)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<float4*>(rb + (size_t)(16 * RW * w + RW * (4 * q4 + j) + ra) * Bp + J0 + 2 * n) =
                make_float4(re[ra][0][j], im[ra][0][j], re[ra][1][j], im[ra][1][j]);
}

// A := A_mod - C R on every 64 x 64 tile of every slab.  The tiles are spread over the
// eight XCDs in contiguous runs of the slab-major, column-major tile order (a run covers
// whole columns of one or two slabs, so the C panel and the R columns a run reads stay in
// that XCD's L2).  Wave w computes the 32 x 32 quadrant (w & 1, w >> 1) as 2 x 2 MFMA
// tiles, the even and the odd rows and columns: a lane's operands of both tiles are one
// 16-byte load straight from global memory, its results four rows of a column each way.
// Bound by the CU's loads of operands beside the matrix cores (15 slabs of 1344 unknowns, 128
// columns: 242 us with 8-byte loads and A read first behind eight waits, 195 us; 153 us without
// any operand loads, 91 us the memory traffic alone).  128 registers, so that four
// waves share a SIMD (with three: 205 us); 64 x 32 per wave: 204 us.
template <int NB>
__global__ void __launch_bounds__(256, 4) k3f_update(Planes F, int Bp, int k0, int ns, const float2* __restrict__ Cb,
                                                 const float2* __restrict__ Rb, int kn, int nbn) {
    const int nb = Bp / 64, nt = nb * nb;
    const int total = ns * nt, per = (total + 7) / 8;
    const int gi = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (gi >= total) return;
    const int s = gi / nt, tt = gi % nt, it = tt % nb, jt = tt / nb;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, q4 = lane >> 4;
    const int I0 = it * 64 + 32 * (w & 1), J0 = jt * 64 + 32 * (w >> 1);
    float2* A = F.at(s, Bp);
    auto next = [&](int x) { return x * 64 >= kn && x * 64 < kn + nbn; };
    if (next(it) && next(jt)) return;                   // the next diagonal block's own
    const bool kcol = jt * 64 >= k0 && jt * 64 < k0 + NB;
    if (it * 64 >= k0 && it * 64 < k0 + NB) {
        // the rows of block K become R(:, J) = P A(K, J): written directly, since forming
        // them as A(K, J) - (A_KK - I) R(:, J) would cancel A(K, J) against A_KK P A(K, J)
        // and leave an FP32 error of order eps cond(A_KK)
        const float2* rr = Rb + (size_t)s * cstr(Bp);
#pragma unroll
        for (int ia = 0; ia < 2; ++ia)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                const int col = J0 + 16 * jb + n;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = I0 + 16 * ia + 4 * q4 + j;
                    A[(size_t)col * Bp + row] = rr[(size_t)(row - k0) * Bp + col];
                }
            }
        return;
    }
    update_quadrant<NB>(A, Cb + (size_t)s * cstr(Bp), Rb + (size_t)s * cstr(Bp), Bp, I0, J0, kcol);
}

}  // namespace

size_t factor3_f32_work_bytes(int J, int Bp) {
    // per slab: eight FP64 64 x 64 scratch blocks (the 64-wide inverse uses the first),
    // P (complex64, up to 128 x 128), C and R (up to 128 x Bp each)
    return (size_t)J * (WSTR * sizeof(double2) + PSTR * sizeof(float2) + 2 * cstr(Bp) * sizeof(float2));
}

// Plane l0 and (l1 >= 0) plane l1 of every slab: column blocks of 128 (a last block of 64 when
// Bp is an odd multiple of 64).  A 128-wide block halves the passes of the update over the
// matrices (the update is bound by HBM and MFMA about equally at 64).  The inverse of a
// diagonal block, one workgroup per matrix, needs no more of the update before it than the
// block's own tiles: it makes these itself, on st, beside the update of the rest on st2 (ev: two
// events).  It is launched first: its workgroups find no room on a CU that the update has
// filled, and would wait for the update's end.  Both ends in one launch, so that the update
// of 30 matrices of 1344 (408 us alone) covers the inverse (192 alone, 366 beside it): 75 planes
// of 15 slabs in 271 ms; 273 to 298 with the ends' chains on a stream each, 360 with the update
// launched first.
hipError_t launch_factor3_plane_f32(const Fac3Args& a, int l0, int l1, float2* Ff, size_t stride, void* work, int* err,
                                    int below, int above, hipStream_t st, hipStream_t st2, const hipEvent_t* ev) {
    const Planes F{Ff, stride, a.J, l0, l1};
    const int ns = l1 < 0 ? a.J : 2 * a.J;
    const size_t BB = (size_t)a.Bp * a.Bp;
    double2* Wd = static_cast<double2*>(work);
    float2* Pf = reinterpret_cast<float2*>(Wd + (size_t)ns * WSTR);
    float2* Cb = Pf + (size_t)ns * PSTR;
    float2* Rb = Cb + (size_t)ns * cstr(a.Bp);
    const unsigned nbs = (unsigned)std::min<size_t>((BB + 255) / 256, 4096);
    hipLaunchKernelGGL(k3f_build_S, dim3(nbs, ns), dim3(256), 0, st, a, F, below, above);
    const int nb = a.Bp / 64;
    const int total = ns * nb * nb, per = (total + 7) / 8;
    auto width = [&](int k0) { return k0 + 128 <= a.Bp ? 128 : a.Bp - k0; };
    auto diag = [&](int k0, const float2* C, hipStream_t q) {
        if (width(k0) == 128)
            hipLaunchKernelGGL(k3f_diag_inv128, dim3(ns), dim3(256), 0, q, F, a.Bp, k0, C, Rb, Wd, Pf, err);
        else hipLaunchKernelGGL(k3f_diag_inv, dim3(ns), dim3(256), 0, q, F, a.Bp, k0, C, Rb, Wd, Pf, err);
    };
    auto after = [&](hipStream_t from, hipStream_t to, hipEvent_t e) {
        const hipError_t r = hipEventRecord(e, from);
        return r == hipSuccess ? hipStreamWaitEvent(to, e, 0) : r;
    };
    diag(0, nullptr, st);
    for (int k0 = 0; k0 < a.Bp;) {
        const int w = width(k0), kn = k0 + w, nbn = width(kn);
        const dim3 grc(a.Bp / RCW, ns), gup(8 * per);
        hipError_t r;
        if (w == 128) hipLaunchKernelGGL(k3f_rc<128>, grc, dim3(256), 0, st, F, a.Bp, k0, Pf, Cb, Rb);
        else hipLaunchKernelGGL(k3f_rc<64>, grc, dim3(256), 0, st, F, a.Bp, k0, Pf, Cb, Rb);
        const hipStream_t q = nbn > 0 ? st2 : st;
        if (nbn > 0) {
            if ((r = after(st, st2, ev[0])) != hipSuccess) return r;
            diag(kn, Cb, st);
        }
        if (w == 128) hipLaunchKernelGGL(k3f_update<128>, gup, dim3(256), 0, q, F, a.Bp, k0, ns, Cb, Rb, kn, nbn);
        else hipLaunchKernelGGL(k3f_update<64>, gup, dim3(256), 0, q, F, a.Bp, k0, ns, Cb, Rb, kn, nbn);
        if (nbn > 0 && (r = after(st2, st, ev[1])) != hipSuccess) return r;
        k0 = kn;
    }
    return hipGetLastError();
}

}  // namespace helm
