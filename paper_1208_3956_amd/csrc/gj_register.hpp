// Gauss-Jordan inversion of a 64 x 64 complex block held in registers (FP64) and a
// 64 x 64 complex block product on FP64 MFMA, shared by the strip factorisation (2-D) and
// the complex64 slab factorisation (3-D), where they invert the diagonal blocks.
#pragma once
#include "helm_internal.hpp"

namespace helm {
namespace gjr {

// ---------------------------------------------------------------- register Gauss-Jordan
// Layout: lane i holds row i; wave g holds columns j = g + 4 r, r = 0..15, in M[r].  A step k
// pivots on column k (wave k % 4) at the unused row p of largest modulus and eliminates
// column k from every other row.  No rows are swapped and the pivot row is not scaled at
// its step: row p keeps its values (its column-k entry becomes 1) and is multiplied by its
// reciprocal pivot after the last step, which leaves every elimination unchanged because the
// updates are linear in the pivot row.  The finished array holds the inverse with row i at
// position step(i) (the step that pivoted on row i) and column j at position perm(j) (the row
// pivoted at step j).  The columns cycle through the registers: after every four steps the
// array is rotated by one register, so the column of the current step is always M[0].
//
// One workgroup and 64 dependent steps: a step is bound by its chain of the pivot row's lane reads
// and products (about 750 clocks for 64 + 64 instructions), the search (270) and a barrier
// with its round through LDS (280).  The wave that owns column k + 1 finds the pivot and forms
// the multipliers for all waves after its update of step k, so there is one such round a step.
// 53 -> 49 us for a 64 x 64 block (before: every wave's own multipliers with two divisions from a
// second read of LDS, a 64-bit search, products waiting for the lane reads).  Deferring the
// owner's update past the barrier took 56: the waves wait for it one step later.
struct GJShared {
    double2 f[2][WP];        // multipliers of the step (double-buffered: one barrier per step)
    double2 inv[2];          // reciprocal pivot
    int piv[2];
    int perm[WP];
    double nrm[2][4];        // per wave: largest column 1-norm of the block, of its inverse
};

// A block whose 1-norm condition estimate ||S||_1 ||S^-1||_1 exceeds this is numerically
// singular in FP64 (its inverse has no correct digit): the factorisation reports it
constexpr double GJ_COND_MAX = 1e13;

// sum over the 64 lanes of a wavefront (butterfly, every lane gets the sum)
__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// largest column 1-norm over this wave's 16 register columns (rows i >= W are zero)
__device__ inline double wave_colnorm_max(const double2 (&M)[16]) {
    double best = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) best = fmax(best, wave_sum(sqrt(M[r].x * M[r].x + M[r].y * M[r].y)));
    return best;
}

// wavefront maximum of 32-bit keys (row shifts, then broadcasts: lane 63 holds it)
__device__ inline unsigned wave_max_u32(unsigned v) {
#define HELM_DPP_MAX(ctrl) v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false))
    HELM_DPP_MAX(0x111);
    HELM_DPP_MAX(0x112);
    HELM_DPP_MAX(0x114);
    HELM_DPP_MAX(0x118);
    HELM_DPP_MAX(0x142);
    HELM_DPP_MAX(0x143);
#undef HELM_DPP_MAX
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// conj(z) / d of d = |z|^2 (0 for d = 0): each quotient by the hardware's estimate of 1 / d, two Newton
// steps and a correction of the quotient itself
__device__ inline double2 cinv(double2 z, double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    r = d > 0.0 ? r : 0.0;
    const double x = z.x * r, y = -z.y * r;
    return make_double2(fma(fma(-d, x, z.x), r, x), fma(fma(-d, y, -z.y), r, y));
}

// component-wise select (a select of whole double2 values goes through scratch memory)
__device__ inline double2 sel(bool c, double2 a, double2 b) {
    return cmk<double2>(c ? a.x : b.x, c ? a.y : b.y);
}

__device__ inline double readlane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Inverse of the leading W x W block of the matrix in M (zero elsewhere), written column-major
// with leading dimension WP to dst (zero outside the leading block); ends with a barrier so
// that dst can be read back by the workgroup.  Sets bit 1 of err when a pivot is zero or not
// finite, bit 2 when the 1-norm condition estimate exceeds cond_max.
__device__ inline void gj_invert_store(double2 (&M)[16], int W, GJShared& sh, double2* __restrict__ dst,
                                float2* __restrict__ dst32, int* err, double cond_max = GJ_COND_MAX) {
    const int i = threadIdx.x & (WP - 1), g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool used = i >= W;
    int my_step = i;                               // rows beyond W keep their position
    double2 my_inv = cmk<double2>(1.0, 0.0);
    int rot = 0;                                   // rotations done: M[r] holds column g + 4 (r + rot)
    {
        const double cn = wave_colnorm_max(M);
        if (i == 0) sh.nrm[0][g] = cn;
    }
    // pivot of column k (v: this lane's entry) among the unused rows and the step's multipliers.
    // |v|^2 is compared by its upper half and, where several rows share the largest, by its lower
    // half without the last 6 bits (ties go to the lower row).  14 bits of it alone, and products
    // with 1 / d in cinv without the correction, save 2% of a factorisation's inversions (32 strips
    // of 1032 rows: 9.2 -> 9.05 ms) and cost up to 45 times the error where a block is close to
    // singular.
    auto publish = [&](int k, double2 v) {
        const int buf = k & 1;
        const double mag = v.x * v.x + v.y * v.y;
        const unsigned hi = used ? 0u : (unsigned)__double2hiint(mag);
        const unsigned top = wave_max_u32(hi);
        unsigned long long rows = __ballot(!used && hi == top);
        if (rows & (rows - 1)) {
            const unsigned lo = used || hi != top ? 0u : (unsigned)__double2loint(mag) & ~63u;
            const unsigned low = wave_max_u32(lo);
            rows = __ballot(!used && hi == top && lo == low);
        }
        const int p = __ffsll(rows) - 1;           // of at least one unused row
        const double2 pv = cmk<double2>(readlane_f64(v.x, p), readlane_f64(v.y, p));
        const double den = pv.x * pv.x + pv.y * pv.y;
        const double2 inv = cinv(pv, den);
        sh.f[buf][i] = sel(i == p, cmk<double2>(0.0, 0.0), cmul(v, inv));
        if (i == 0) {
            sh.piv[buf] = p;
            sh.inv[buf] = inv;
            sh.perm[k] = p;
            if (!(den > 0.0 && isfinite(den))) atomicOr(err, 1);
        }
    };
    if (g == 0) publish(0, M[0]);
    __syncthreads();
    for (int kk = 0; 4 * kk < W; ++kk) {
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
            const int k = 4 * kk + gg;
            if (k < W) {
                constexpr int next_reg[4] = {0, 0, 0, 1};
                const int nr = next_reg[gg], buf = k & 1;     // column k + 1: wave (gg + 1) % 4, M[nr]
                const int p = __builtin_amdgcn_readfirstlane(sh.piv[buf]);
                const double2 f = sh.f[buf][i], inv = sh.inv[buf];
                if (i == p) {
                    used = true;
                    my_step = k;
                    my_inv = inv;
                }
                // a column's lane reads two columns ahead of its last products, in this order
                // (left to itself each product waits for the lane read before it)
                double Rx[3], Ry[3], u[2][2];
                auto column = [&](int r) {
                    if (r < 16) {
                        Rx[r % 3] = readlane_f64(M[r].x, p);
                        Ry[r % 3] = readlane_f64(M[r].y, p);
                    }
                    if (r > 0 && r < 17) {
                        u[r & 1][0] = fma(f.y, Ry[(r + 2) % 3], M[r - 1].x);
                        u[r & 1][1] = fma(-f.y, Rx[(r + 2) % 3], M[r - 1].y);
                    }
                    if (r > 1) {
                        M[r - 2].x = fma(-f.x, Rx[(r + 1) % 3], u[(r + 1) & 1][0]);
                        M[r - 2].y = fma(-f.x, Ry[(r + 1) % 3], u[(r + 1) & 1][1]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
#pragma unroll
                for (int r = 0; r < 18; ++r) column(r);
                if (g == gg) M[0] = sel(i == p, cmk<double2>(1.0, 0.0), cmk<double2>(-f.x, -f.y));
                if (g == ((gg + 1) & 3) && k + 1 < W) publish(k + 1, M[nr]);
                __syncthreads();
            }
        }
        // rotate: the next four columns come to M[0]
        const double2 m0 = M[0];
#pragma unroll
        for (int r = 0; r < 15; ++r) M[r] = M[r + 1];
        M[15] = m0;
        ++rot;
    }
    double2 out[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = g + 4 * ((r + rot) & 15);
        const int pj = j < W ? sh.perm[j] : j;
        const double2 v = cmul(M[r], my_inv);
        out[r] = j < W ? v : cmk<double2>(0.0, 0.0);
        dst[(size_t)pj * WP + my_step] = v;
        if (dst32) dst32[(size_t)pj * WP + my_step] = make_float2((float)v.x, (float)v.y);
    }
    // permuting rows and columns leaves the set of column 1-norms unchanged: the largest
    // over the stored array is ||S^-1||_1 (the identity outside the leading block excluded)
    {
        const double cn = wave_colnorm_max(out);
        if ((threadIdx.x & 63) == 0) sh.nrm[1][g] = cn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int q = 0; q < 4; ++q) { a = fmax(a, sh.nrm[0][q]); b = fmax(b, sh.nrm[1][q]); }
        if (!(a * b <= cond_max)) atomicOr(err, 2);
    }
}


// C = alpha * A * B (+ D) on v_mfma_f64_16x16x4f64: full WP x WP, column-major with leading
// dimensions, operands in LDS or global memory, C may alias A, B or D.  Wave w computes rows
// 16 w .. 16 w + 15 in four 16-column tiles; a complex product is four real ones.  Lane
// layout (one 16x16x4 block of doubles): A[l % 16][l / 16], B[l / 16][l % 16] and
// C[l / 16 + 4 j][l % 16] in component j (rows interleaved by 4, unlike the FP32 block).
typedef double md4 __attribute__((ext_vector_type(4)));

__device__ __attribute__((always_inline)) inline void gemm64_mfma(double2* C, int ldc, const double2* A, int lda, const double2* B, int ldb,
                            double2 alpha, const double2* D, int ldd) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, q4 = lane >> 4;
    double2 av[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) av[s] = A[(16 * w + n) + (size_t)(4 * s + q4) * lda];
    md4 cr[4], ci[4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) { cr[tt] = md4{0.0, 0.0, 0.0, 0.0}; ci[tt] = cr[tt]; }
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        double2 bv[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) bv[tt] = B[(4 * s + q4) + (size_t)(16 * tt + n) * ldb];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            cr[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].x, bv[tt].x, cr[tt], 0, 0, 0);
            ci[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].x, bv[tt].y, ci[tt], 0, 0, 0);
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            cr[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[s].y, bv[tt].y, cr[tt], 0, 0, 0);
            ci[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].y, bv[tt].x, ci[tt], 0, 0, 0);
        }
    }
    double2 v[4][4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double2 x = cmul(alpha, cmk<double2>(cr[tt][j], ci[tt][j]));
            if (D) x = cadd(x, D[(16 * w + q4 + 4 * j) + (size_t)(16 * tt + n) * ldd]);
            v[tt][j] = x;
        }
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int j = 0; j < 4; ++j) C[(16 * w + q4 + 4 * j) + (size_t)(16 * tt + n) * ldc] = v[tt][j];
    __syncthreads();
}

}  // namespace gjr
}  // namespace helm
