// Strip solves x = A^(j)^{-1} r with the chunked block-LU factors (the subdomain solves of
// eqs. solve_upward / solve_downward, Sec. 2.1-2.2), for a panel of right-hand sides.
//
// With chunks I_c (interior rows) and separators s_c (see kernels_factor.hip):
//   phase A   (chunks x rhs groups)  y_I = A_I^{-1} r_I by forward / backward block
//             substitution  z_l = G_l (r_l - c_l z_{l-1}),  y_l = z_l - b_l G_l y_{l+1}
//   phase B0  (separators x rhs)     a_c = G'_c r^_c,  r^_c = r_s - c_s y_{s-1} - b_s y_{s+1}
//   phase B   (one workgroup per rhs) z'_c = a_c - K_c z'_{c-1};  x_s = z'_c - U'_c x_{s'}
//   phase C   (rows x rhs groups)    x_l = y_l - X~_l x_{s above} - Y~_l x_{s below}
// Phase A (and B0) gather the right-hand side (a field restricted to the strip plus the
// two-column transmission source of Sec. 2.2); phase C scatters the requested columns of x
// and the two trace columns the next strip needs.  When only a few columns are requested
// (the reduced form), phase C computes just those from compact copies of the spike rows.
//
// The chains of phases A and B read the factor blocks of the next steps from global memory
// into rings of registers: the latency of the block loads stays off the dependency chain.
//
// Arithmetic is in T (float or double complex); gathered and scattered fields are FP64.
#include "helm_internal.hpp"

#include <type_traits>

namespace helm {

namespace {

constexpr int NT = 256;

template <typename T>
struct SolveArgs {
    const cplx<T>* F;     // factors of the strip: [Ny][NSLOT][WP*WP]
    const cplx<T>* Fc;    // compact spike rows of the strip: [Ny][2][8][WP] (reduced phase C)
    const int* tcol;      // 8 strip-local columns of the compact rows (-1 = unused)
    const cplx<T>* Fs;    // separator propagators of the strip: [P-1][2][WP*WP] (two-level solve)
    const cplx<T>* Fa;    // complex64: G_l in phase-A operand order, [Ny][WP*WP] (see helm_internal.hpp)
    const cplx<T>* Fw;    // complex64: chain blocks in operand order, [P-1][4][WP*WP]
    cplx<T>* Yw;          // workspace [nrhs][Ny][WP]
    const double2* cy;
    const double2* by;
    IOSpec io;
    int Ny, W, m, P, nrhs;
    int q, G;             // separator groups (two-level separator solve when G >= 2)
};

// Block coordinates of a workgroup: the launch's own (one problem), or its place inside one
// problem of a multi-problem launch (nz: the number of z blocks that problem uses).
struct Blk {
    int x, y, z, nz;
};
__device__ inline Blk own_blk() { return Blk{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, (int)gridDim.z}; }

// Several problems' strip solves in one launch (one strip of each): their arguments by value
// in the kernel-argument block, x blocks [xs[k], xs[k+1]) belonging to problem k, which uses
// ny[k] y blocks and nz[k] z blocks of the launch's maximum (the others return at once).
template <typename T>
struct MultiArgs {
    SolveArgs<T> a[MULTI_MAX];
    int xs[MULTI_MAX + 1];
    int ny[MULTI_MAX], nz[MULTI_MAX];
    int n;
};
static_assert(sizeof(MultiArgs<float>) <= 4096, "multi-problem arguments exceed the kernel-argument block");

// problem of this workgroup and its block coordinates inside it; false: idle workgroup
template <typename T>
__device__ inline bool multi_blk(const MultiArgs<T>& m, int& k, Blk& b) {
    const int bx = (int)blockIdx.x;
    k = 0;
    while (k + 1 < m.n && bx >= m.xs[k + 1]) ++k;
    b = Blk{bx - m.xs[k], (int)blockIdx.y, (int)blockIdx.z, m.nz[k]};
    return b.y < m.ny[k] && b.z < m.nz[k];
}

// Several strips of one problem in one launch: the grid's z is the strip (times nz where the
// kernel uses z blocks of its own); what differs from strip to strip comes from a table.
// One group of right-hand sides and more than a round of workgroups: the strips' workgroups of
// one x (a chunk, a row) run one after the other on one XCD (`near`), so that strips that
// share a factorisation read each block from memory once, not once per strip: 64 layered
// strips of 2032 rows, one right-hand side, complex128, 39.6 -> 37.9 ms a solve; P at 532 rows,
// 8 right-hand sides, 2.14 -> 2.02 ms; strips with factors of their own the same.  With four
// groups (64 right-hand sides, the products bind) 289 -> 291 ms, and where all workgroups run at
// once there is nothing to order (4 strips of 122 rows: 1.74 -> 1.77 ms): both left as they are.
template <typename T>
struct BatchArgs {
    SolveArgs<T> a;               // factors of slot 0, workspace of the first strip
    const StripIO* io;            // first strip of the launch
    const int* tcol;
    long F_st, Fc_st, Fs_st, Fa_st, Fw_st, Yw_st;
    long tr_st;                   // elements of one trace (two per strip)
};
// block coordinates in that order: blocks 8 apart share an XCD; 8 values of x at a time, the last
// gridDim.x % 8 of them on all
__device__ inline int3 near_block() {
    const unsigned X = gridDim.x, Z = gridDim.z, in = gridDim.y * Z, X8 = X & ~7u;
    const unsigned L = blockIdx.x + X * (blockIdx.y + gridDim.y * blockIdx.z);
    const bool tail = L >= X8 * in;
    const unsigned i = tail ? L - X8 * in : L >> 3, q = i / in, r = i - q * in;
    return make_int3((int)(tail ? X8 + q : 8 * q + (L & 7)), (int)(r / Z), (int)(r % Z));
}
template <typename T>
__device__ inline SolveArgs<T> batch_strip(const BatchArgs<T>& b, int nz, Blk& B, bool near = false) {
    near = near && gridDim.y == 1 && gridDim.x * gridDim.z > 256;
    const int3 id = near ? near_block() : make_int3((int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z);
    const int k = id.z / nz;
    B = Blk{id.x, id.y, id.z - k * nz, nz};
    const StripIO x = b.io[k];
    SolveArgs<T> a = b.a;
    a.F += x.fs * b.F_st;
    a.Fc += x.fs * b.Fc_st;
    a.Fs += x.fs * b.Fs_st;
    a.Fa += x.fs * b.Fa_st;
    a.Fw += x.fs * b.Fw_st;
    a.Yw += k * b.Yw_st;
    a.tcol = b.tcol + 8 * k;
    a.W = x.W;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a.io.o_lo[i] = x.o_lo[i];
        a.io.o_hi[i] = x.o_hi[i];
        a.io.dst_off[i] = x.o_off[i];
    }
    a.io.qo0 = x.qo0;
    a.io.qo1 = x.qo1;
    if (a.io.tro0) {
        a.io.tro0 += 2 * k * b.tr_st;
        a.io.tro1 += 2 * k * b.tr_st;
    }
    return a;
}

template <typename T>
__device__ inline cplx<T> gather(const IOSpec& io, int r, int l, int q, int Ny) {
    double2 v = cmk<double2>(0.0, 0.0);
    if (q >= io.src_lo && q < io.src_hi)
        v = io.src[(size_t)r * io.src_rs + (size_t)l * io.src_ls + (q + io.src_off)];
    if (tr_col(io, q)) {
        const double2 ta = io.trA[(size_t)r * Ny + l], tb = io.trB[(size_t)r * Ny + l];
        v.x += io.coef * (tb.x - ta.x);
        v.y += io.coef * (tb.y - ta.y);
    }
    return ccast<cplx<T>>(v);
}

// Branch-free gather in two halves: load_raw issues the loads (clamped addresses; lanes
// outside the source or transmission columns read element 0 and discard it), combine
// forms the right-hand-side value.  Keeping the uses apart from the loads lets the loads
// of the next step overlap the current one.  io.src, io.trA and io.trB must be valid
// pointers (the host points unused transmission traces at the source).
struct RawRhs {
    double2 v, ta, tb;
};
__device__ inline RawRhs load_raw(const IOSpec& io, int r, int l, int q, int Ny, int nrhs, int W) {
    const bool ok = r < nrhs && q < W;
    const bool in_src = ok && q >= io.src_lo && q < io.src_hi;
    const bool in_tr = ok && tr_col(io, q);
    const size_t ps = in_src ? (size_t)r * io.src_rs + (size_t)l * io.src_ls + (q + io.src_off) : 0;
    const size_t pt = in_tr ? (size_t)r * Ny + l : 0;
    RawRhs x;
    x.v = io.src[ps];
    x.ta = io.trA[pt];
    x.tb = io.trB[pt];
    if (!in_src) x.v = cmk<double2>(0.0, 0.0);
    if (!in_tr) { x.ta = cmk<double2>(0.0, 0.0); x.tb = x.ta; }
    return x;
}
// The same for the four consecutive columns q0 .. q0 + 3 of one row: the transmission term
// is the same for both of its columns, so the two trace values are loaded once.
struct RawRhs4 {
    double2 v[4];
    double2 ta, tb;
};
__device__ inline void load_raw4(RawRhs4& x, const IOSpec& io, int r, int l, int q0, int Ny, int nrhs, int W) {
    const bool rok = r < nrhs;
    const bool tr = rok && io.q_t >= 0 && io.q_t + 1 >= q0 && io.q_t <= q0 + 3;
    const size_t pt = tr ? (size_t)r * Ny + l : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int q = q0 + j;
        const bool in_src = rok && q < W && q >= io.src_lo && q < io.src_hi;
        const size_t ps = in_src ? (size_t)r * io.src_rs + (size_t)l * io.src_ls + (q + io.src_off) : 0;
        x.v[j] = io.src[ps];
        if (!in_src) x.v[j] = cmk<double2>(0.0, 0.0);
    }
    x.ta = io.trA[pt];
    x.tb = io.trB[pt];
    if (!tr) { x.ta = cmk<double2>(0.0, 0.0); x.tb = x.ta; }
}
__device__ inline float2 combine4(const IOSpec& io, const RawRhs4& x, int j, int q) {
    double2 v = x.v[j];
    if (tr_col(io, q)) {
        v.x += io.coef * (x.tb.x - x.ta.x);
        v.y += io.coef * (x.tb.y - x.ta.y);
    }
    return make_float2((float)v.x, (float)v.y);
}

template <typename T>
__device__ inline cplx<T> combine(const IOSpec& io, const RawRhs& x) {
    double2 v = x.v;
    v.x += io.coef * (x.tb.x - x.ta.x);
    v.y += io.coef * (x.tb.y - x.ta.y);
    return ccast<cplx<T>>(v);
}

template <typename T>
__device__ inline const cplx<T>* fslot(const SolveArgs<T>& a, int l, int sl) {
    return a.F + ((size_t)l * NSLOT + sl) * BLK;
}

template <typename T>
__device__ inline void scatter(const SolveArgs<T>& a, int r, int l, int i, cplx<T> x) {
    const IOSpec& io = a.io;
    const double2 xv = ccast<double2>(x);
    const bool o0 = i >= io.o_lo[0] && i < io.o_hi[0];
    const bool o = o0 || (i >= io.o_lo[1] && i < io.o_hi[1]);
    if (o && io.dst) {
        double2* p = io.dst + (size_t)r * io.dst_rs + (size_t)l * io.dst_ls + (i + io.dst_off[o0 ? 0 : 1]);
        *p = io.accumulate ? cadd(*p, xv) : xv;
    }
    if (i == io.qo0 && io.tro0) io.tro0[(size_t)r * a.Ny + l] = xv;
    if (i == io.qo1 && io.tro1) io.tro1[(size_t)r * a.Ny + l] = xv;
}

// acc[u] += sum_{k<W} M(i,k) vin[k][g + G*u]   (M column-major WP x WP)
template <typename T, int R, int G>
__device__ inline void matvec(cplx<T> (&acc)[R / G], const cplx<T>* M, const cplx<T> (*vin)[R],
                              int W, int i, int g) {
    constexpr int U = R / G;
#pragma unroll 4
    for (int k = 0; k < W; ++k) {
        const cplx<T> mk = M[k * WP + i];
#pragma unroll
        for (int u = 0; u < U; ++u) cfma(acc[u], mk, vin[k][g + G * u]);
    }
}

// ---------------------------------------------------------------- phase A, few right-hand sides
// Panels of at most 4 right-hand sides (R = 1, 2 or 4 per workgroup): a chain of matrix-vector
// products, bound by the latency of a step and by the 64 x 64 block each step reads (64 KB in
// complex128, about 0.43 us through one CU's load path).  Thread (i, w) multiplies row i of the
// block with the 16 columns 16 w .. 16 w + 15 straight from registers (a ring of D blocks, D
// steps ahead); the four waves' partial sums meet in LDS behind the step's only barrier.  Wave w
// then needs the result only at its own 16 columns: lane (row 16 w + lane % 16, right-hand side
// lane / 16) adds the four partial sums, forms the next step's operand there and keeps it in a
// part of LDS that only its wave reads.
// PRE (here and below): the right-hand side is in the workspace rows already, in T, and is
// overwritten by the result (a lane reads a row's entries before it stores the same ones).
template <typename T, int R, bool PRE>
__device__ __forceinline__ void phase_a_few(const SolveArgs<T>& a, const Blk& B) {
    using V = cplx<T>;
    constexpr int D = std::is_same<T, double>::value && R > 1 ? 3 : 4;   // 3: no spills
    __shared__ V vecw[4][R][16];
    __shared__ V part[2][4][R][WP];
    const int t = threadIdx.x, i = t & (WP - 1), w = t >> 6, k0 = 16 * w;
    const int c = B.x;
    const int r0 = c * a.m;
    const int r1 = (c < a.P - 1) ? c * a.m + a.m - 1 : a.Ny;
    const int n = r1 - r0;
    const int steps = 2 * n - 1;                 // forward r0..r1-1, backward r1-2..r0
    auto row_of = [&](int k) {
        k = k < steps ? k : steps - 1;
        return k < n ? r0 + k : r1 - 2 - (k - n);
    };
    // this lane's element of the vectors
    const int q = k0 + (i & 15), bl = i >> 4, b = bl < R ? bl : R - 1;
    const int r = B.y * R + b;
    const bool own = bl < R && r < a.nrhs;
    V* Yr = a.Yw + (size_t)(own ? r : 0) * a.Ny * WP + q;
    V breg[D][16];
    auto load_blk = [&](int k, V (&g)[16]) {
        const V* G = fslot(a, row_of(k), 0) + (size_t)k0 * WP + i;
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) g[kk] = G[kk * WP];
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load_blk(d, breg[d]);
    V z = cmk<V>(0, 0);
    // loads of the next row, issued a step ahead: its right-hand side and coupling (forward),
    // z_l and coupling (backward)
    RawRhs raw;
    V pre = z;
    auto load_rhs = [&](int l) {
        if constexpr (PRE) pre = Yr[(size_t)l * WP];
        else raw = load_raw(a.io, own ? r : a.nrhs, l, q, a.Ny, a.nrhs, a.W);
    };
    load_rhs(r0);
    double2 cn = a.cy[r0];
    V zn = z;
    // v: the step's operand (this lane's element); returns (G v) there
    auto product = [&](int k, V (&g)[16], V v) {
        const int buf = k & 1;
        if (bl < R) vecw[w][bl][i & 15] = v;
        __builtin_amdgcn_wave_barrier();         // only this wave's lanes read the entries
        V acc[R];
#pragma unroll
        for (int u = 0; u < R; ++u) acc[u] = cmk<V>(0, 0);
#pragma unroll
        for (int kk = 0; kk < 16; ++kk)
#pragma unroll
            for (int u = 0; u < R; ++u) cfma(acc[u], g[kk], vecw[w][u][kk]);
        load_blk(k + D, g);
#pragma unroll
        for (int u = 0; u < R; ++u) part[buf][w][u][i] = acc[u];
        __syncthreads();
        return cadd(cadd(part[buf][0][b][q], part[buf][1][b][q]), cadd(part[buf][2][b][q], part[buf][3][b][q]));
    };
    auto step = [&](int k, int j) {
        const int l = row_of(k);
        if (k < n) {
            V v = pre;
            if constexpr (!PRE) v = combine<T>(a.io, raw);
            if (k > 0) v = csub(v, cmul(ccast<V>(cn), z));
            const int ln = l + 1 < r1 ? l + 1 : l;
            load_rhs(ln);
            cn = a.cy[ln];
            z = product(k, breg[j], v);
            if (own) Yr[(size_t)l * WP] = z;
            if (k == n - 1 && n > 1) { cn = a.by[r1 - 2]; zn = Yr[(size_t)(r1 - 2) * WP]; }
        } else {
            const V zl = zn, bk = ccast<V>(cn);
            const int lb = l - 1 >= r0 ? l - 1 : l;
            cn = a.by[lb];
            zn = Yr[(size_t)lb * WP];
            z = csub(zl, cmul(bk, product(k, breg[j], z)));
            if (own) Yr[(size_t)l * WP] = z;
        }
    };
    int k = 0;
    for (; k + D <= steps; k += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) step(k + j, j);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (k + j < steps) step(k + j, j);
}
template <typename T, int R>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1))) k_phase_a_few(SolveArgs<T> a) {
    phase_a_few<T, R, false>(a, own_blk());
}
template <typename T, int R>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1))) k_phase_a_few_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B, true);
    phase_a_few<T, R, true>(a, B);
}

// ---------------------------------------------------------------- phase A, MFMA
// complex64, 16 right-hand sides per workgroup.  The block product Z = G V (64 x 64 times
// 64 x 16, complex) runs on v_mfma_f32_16x16x4f32 as three real products (Gauss's form:
// M1 = Gr Vr, M2 = Gi Vi, M3 = (Gr + Gi)(Vr + Vi), Zr = M1 - M2, Zi = M3 - M1 - M2; 48
// instead of 64 MFMAs per step, 126 instead of 133 us per launch at 2000^2, iteration
// counts unchanged); wave w owns output rows 16w..16w+15.
// MFMA lane layout (16x16x4, one block): A[l % 16][l / 16], B[l / 16][l % 16],
// C[4 (l / 16) + j][l % 16] in component j.
typedef float mf4 __attribute__((ext_vector_type(4)));

// The blocks G_l are not staged through LDS: each lane loads exactly its MFMA A operands
// (16 values per block, A[16w + n][4s + q4] for k-step s) straight from global memory into
// a ring of D register blocks, D steps ahead.  Only the right-hand-side panel of a step
// (64 x 16) goes through LDS, double-buffered, so a step has a single barrier.  Each lane
// gathers the right-hand-side values of its own four output positions.  The ring slot a
// step's products read is refilled inside the product loop, one 16-byte load after the six
// products that read its pair: the four waves of a workgroup reach their products together
// after the barrier, and loads issued after the products kept the CU's load path busy
// while the matrix cores idled (and the stores and right-hand-side loads queued behind).
template <int D, bool PRE = false>
__device__ __forceinline__ void phase_a_mfma(const SolveArgs<float>& a, const Blk& B) {
    using V = float2;
    constexpr int R = 16;
    __shared__ V Vs[2][WP][R];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int n = lane & 15, q4 = lane >> 4;            // MFMA column (rhs), row quad
    const int c = B.x, rbase = B.y * R;
    const int r0 = c * a.m;
    const int r1 = (c < a.P - 1) ? c * a.m + a.m - 1 : a.Ny;
    const int nr = r1 - r0;
    const int nsteps = 2 * nr - 1;                       // forward nr rows, backward nr - 1
    const V zero = make_float2(0.f, 0.f);
    const int rn = rbase + n;                            // rhs of this lane's MFMA column
    const bool rn_ok = rn < a.nrhs;
    const int qrow = 16 * w + 4 * q4;                    // first of this lane's 4 output rows
    const size_t ybase = (size_t)(rn_ok ? rn : 0) * a.Ny * WP + qrow;
    // targets-only solves read y at the compact target columns (phase C) and on the first
    // and last interior row (the separators' right-hand sides); full solves read it all
    bool tm[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bool on = false;
        for (int k = 0; k < 8; ++k) on = on || (a.tcol[k] == qrow + j);
        tm[j] = on;
    }
    auto row_of = [&](int k) {
        k = k < nsteps ? k : nsteps - 1;
        return k < nr ? r0 + k : r1 - 2 - (k - nr);
    };
    // the A operands of k-steps 2i and 2i + 1 come in one 16-byte load (operand-order copy)
    auto g_ptr = [&](int k) {
        return reinterpret_cast<const float4*>(a.Fa + (size_t)row_of(k) * BLK) + w * 8 * 64 + lane;
    };
    auto load_g = [&](int k, V (&g)[16]) {
        const float4* G = g_ptr(k);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 v = G[i * 64];
            g[2 * i] = make_float2(v.x, v.y);
            g[2 * i + 1] = make_float2(v.z, v.w);
        }
    };
    RawRhs4 raw;
    V pre[4];
    auto load_rhs = [&](int l) {
        if constexpr (PRE) {
            const float4* y = reinterpret_cast<const float4*>(a.Yw + ybase + (size_t)l * WP);
            const float4 y0 = y[0], y1 = y[1];
            pre[0] = make_float2(y0.x, y0.y);
            pre[1] = make_float2(y0.z, y0.w);
            pre[2] = make_float2(y1.x, y1.y);
            pre[3] = make_float2(y1.z, y1.w);
        } else {
            load_raw4(raw, a.io, rn, l, qrow, a.Ny, a.nrhs, a.W);
        }
    };
    V greg[D][16];
    V z[4], zn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { z[j] = zero; zn[j] = zero; }
    double2 cnext = a.cy[r0], bnext = a.by[r0];
    load_rhs(r0);
#pragma unroll
    for (int d = 0; d < D; ++d) load_g(d, greg[d]);

    // products of block g with the staged panel; g is refilled with block knext meanwhile
    auto mfma_block = [&](V (&g)[16], const V (*Vb)[R], V (&out)[4], int knext) {
        const float4* Gn = g_ptr(knext);
        // three real products per complex one: M1 = Gr Vr, M2 = Gi Vi, M3 = (Gr + Gi)(Vr + Vi);
        // Zr = M1 - M2, Zi = M3 - M1 - M2
        mf4 m1 = {0.f, 0.f, 0.f, 0.f}, m2 = m1, m3 = m1, n1 = m1, n2 = m1, n3 = m1;
        V vb[16];
#pragma unroll
        for (int s4 = 0; s4 < 16; ++s4) vb[s4] = Vb[4 * s4 + q4][n];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s4 = 0; s4 < 16; s4 += 2) {
            const V g0 = g[s4], g1 = g[s4 + 1];
            const V v0 = vb[s4], v1 = vb[s4 + 1];
            m1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x, v0.x, m1, 0, 0, 0);
            m2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.y, v0.y, m2, 0, 0, 0);
            m3 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x + g0.y, v0.x + v0.y, m3, 0, 0, 0);
            n1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.x, v1.x, n1, 0, 0, 0);
            n2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.y, v1.y, n2, 0, 0, 0);
            n3 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.x + g1.y, v1.x + v1.y, n3, 0, 0, 0);
            const float4 nv = Gn[(s4 >> 1) * 64];
            g[s4] = make_float2(nv.x, nv.y);
            g[s4 + 1] = make_float2(nv.z, nv.w);
            __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);   // six MFMAs,
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // then the pair's load
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float p1 = m1[j] + n1[j], p2 = m2[j] + n2[j], p3 = m3[j] + n3[j];
            out[j] = make_float2(p1 - p2, p3 - p1 - p2);
        }
    };

    // component-wise select (a select of whole float2 values goes through scratch memory)
    auto keep = [](bool on, V x) { return make_float2(on ? x.x : 0.f, on ? x.y : 0.f); };
    // ---- forward row l = r0 + k:  z_l = G_l (r_l - c_l z_{l-1})
    auto fwd_step = [&](int k, int j) {
        const int buf = k & 1;
        const int l = r0 + k;
        // the first row of a chunk has no coupling inside phase A (scalar selects: no
        // aggregate select that would go through memory)
        const float clx = k > 0 ? (float)cnext.x : 0.f, cly = k > 0 ? (float)cnext.y : 0.f;
        const V cl = make_float2(clx, cly);
        V v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            V r;
            if constexpr (PRE) r = pre[u];
            else r = combine4(a.io, raw, u, qrow + u);
            v[u] = csub(r, cmul(cl, z[u]));
        }
        // next step's small loads first (vmcnt retires in issue order); clamped, branch-free
        const int ln = l + 1 < r1 ? l + 1 : l;
        cnext = a.cy[ln];
        load_rhs(ln);
#pragma unroll
        for (int u = 0; u < 4; ++u) Vs[buf][qrow + u][n] = v[u];
        __syncthreads();
        V acc[4];
        mfma_block(greg[j], Vs[buf], acc, k + D);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            z[u] = keep(rn_ok, acc[u]);
            if (rn_ok) a.Yw[ybase + (size_t)l * WP + u] = acc[u];
        }
    };
    // ---- backward row l = r1 - 2 - (k - nr):  y_l = z_l - b_l G_l y_{l+1}
    auto bwd_step = [&](int k, int j) {
        const int buf = k & 1;
        const int l = r1 - 2 - (k - nr);
        V zl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) zl[u] = zn[u];
        const V bl = ccast<V>(bnext);
        const int lb = l - 1 >= r0 ? l - 1 : l;
        bnext = a.by[lb];
#pragma unroll
        for (int u = 0; u < 4; ++u) zn[u] = a.Yw[ybase + (size_t)lb * WP + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) Vs[buf][qrow + u][n] = z[u];
        __syncthreads();
        V acc[4];
        mfma_block(greg[j], Vs[buf], acc, k + D);
        const bool store_y = !a.io.targets_only || l == r0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const V y = csub(zl[u], cmul(bl, acc[u]));
            z[u] = keep(rn_ok, y);
            if (rn_ok && (store_y || tm[u])) a.Yw[ybase + (size_t)l * WP + u] = y;
        }
    };
    int k = 0;
    for (; k + D <= nr; k += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) fwd_step(k + j, j);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (k + j < nr) fwd_step(k + j, j);
    if (nr < 2) return;
    // z_{r1-2} and b_{r1-2} of the first backward row (ybase is valid for every lane: lanes
    // beyond nrhs read rows of right-hand side 0 and discard them)
    bnext = a.by[r1 - 2];
#pragma unroll
    for (int u = 0; u < 4; ++u) zn[u] = a.Yw[ybase + (size_t)(r1 - 2) * WP + u];
    // backward steps k = nr .. 2 nr - 2 use ring slot k % D: the loop is unrolled for the
    // slot of its first step
    auto bwd_loop = [&](auto off_tag) {
        constexpr int OFF = decltype(off_tag)::value;
        int kb = nr;
        for (; kb + D <= nsteps; kb += D) {
#pragma unroll
            for (int j = 0; j < D; ++j) bwd_step(kb + j, (j + OFF) % D);
        }
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (kb + j < nsteps) bwd_step(kb + j, (j + OFF) % D);
    };
    static_assert(D >= 1 && D <= 4, "ring alignment dispatch below covers D <= 4");
    const int off = nr % D;
    if (off == 0) bwd_loop(std::integral_constant<int, 0>{});
    if constexpr (D > 1) { if (off == 1) bwd_loop(std::integral_constant<int, 1 % D>{}); }
    if constexpr (D > 2) { if (off == 2) bwd_loop(std::integral_constant<int, 2 % D>{}); }
    if constexpr (D > 3) { if (off == 3) bwd_loop(std::integral_constant<int, 3 % D>{}); }
}
template <int D>
__global__ void __launch_bounds__(NT) k_phase_a_mfma(SolveArgs<float> a) { phase_a_mfma<D>(a, own_blk()); }
template <int D>
__global__ void __launch_bounds__(NT) k_phase_a_mfma_b(BatchArgs<float> b) {
    Blk B;
    const SolveArgs<float> a = batch_strip(b, 1, B, true);
    phase_a_mfma<D, true>(a, B);
}
template <int D>
__global__ void __launch_bounds__(NT) k_phase_a_mfma_multi(MultiArgs<float> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) phase_a_mfma<D>(m.a[k], b);
}

// ---------------------------------------------------------------- phase A, FP64 MFMA
// complex128, 16 right-hand sides per workgroup: the block product of a step (64 x 64 times
// 64 x 16, complex) as four real products on v_mfma_f64_16x16x4f64, wave w owning output rows
// 16 w .. 16 w + 15.  The FP64 matrix and vector peaks are equal on MI355X; what the VALU form
// lost was everything else: every block went through registers into LDS and back (64 KB each
// way per step) behind two barriers.  Here each lane loads its 16 A operands of a block
// straight into a ring of two register blocks and refills them between the products, as in
// the complex64 form, and a step has one barrier.  Bound by its 64 MFMAs per wave and step
// (64 cycles each, 1.7 us a step at 2.4 GHz).
// FP64 lane layout: A[l % 16][l / 16], B[l / 16][l % 16], C[l / 16 + 4 j][l % 16].
typedef double md4 __attribute__((ext_vector_type(4)));

template <bool PRE>
__device__ __forceinline__ void phase_a_mfma64(const SolveArgs<double>& a, const Blk& B) {
    using V = double2;
    constexpr int R = 16;
    __shared__ V Vs[2][WP][R];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int n = lane & 15, q4 = lane >> 4;
    const int c = B.x, rbase = B.y * R;
    const int r0 = c * a.m;
    const int r1 = (c < a.P - 1) ? c * a.m + a.m - 1 : a.Ny;
    const int nr = r1 - r0;
    const int nsteps = 2 * nr - 1;
    const int rn = rbase + n;
    const bool rn_ok = rn < a.nrhs;
    const int qrow = 16 * w + q4;                        // this lane's output rows: qrow + 4 j
    const size_t ybase = (size_t)(rn_ok ? rn : 0) * a.Ny * WP + qrow;
    bool tm[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bool on = false;
        for (int k = 0; k < 8; ++k) on = on || (a.tcol[k] == qrow + 4 * j);
        tm[j] = on;
    }
    auto row_of = [&](int k) {
        k = k < nsteps ? k : nsteps - 1;
        return k < nr ? r0 + k : r1 - 2 - (k - nr);
    };
    auto g_ptr = [&](int k) { return fslot(a, row_of(k), 0) + (size_t)q4 * WP + 16 * w + n; };
    V greg[2][16];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const V* G = g_ptr(d);
#pragma unroll
        for (int s = 0; s < 16; ++s) greg[d][s] = G[4 * s * WP];
    }
    // right-hand-side values of the lane's four rows (clamped, branch-free loads)
    V rv[4], ta, tb;
    auto load_rhs = [&](int l) {
        if constexpr (PRE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) rv[j] = a.Yw[ybase + (size_t)l * WP + 4 * j];
            return;
        }
        const bool tr = rn_ok && a.io.q_t >= 0;
        const size_t pt = tr ? (size_t)rn * a.Ny + l : 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = qrow + 4 * j;
            const bool in = rn_ok && q < a.W && q >= a.io.src_lo && q < a.io.src_hi;
            const size_t ps = in ? (size_t)rn * a.io.src_rs + (size_t)l * a.io.src_ls + (q + a.io.src_off) : 0;
            const V v = a.io.src[ps];
            rv[j] = cmk<V>(in ? v.x : 0.0, in ? v.y : 0.0);
        }
        const V va = a.io.trA[pt], vb = a.io.trB[pt];
        ta = cmk<V>(tr ? va.x : 0.0, tr ? va.y : 0.0);
        tb = cmk<V>(tr ? vb.x : 0.0, tr ? vb.y : 0.0);
    };
    V z[4], zn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { z[j] = cmk<V>(0.0, 0.0); zn[j] = z[j]; }
    V cnext = a.cy[r0], bnext = a.by[r0];
    load_rhs(r0);

    auto mfma_block = [&](V (&g)[16], const V (*Vb)[R], V (&out)[4], int knext) {
        const V* Gn = g_ptr(knext);
        md4 cr = {0.0, 0.0, 0.0, 0.0}, ci = cr;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const V gs = g[s], v = Vb[4 * s + q4][n];
            cr = __builtin_amdgcn_mfma_f64_16x16x4f64(gs.x, v.x, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f64_16x16x4f64(gs.x, v.y, ci, 0, 0, 0);
            cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-gs.y, v.y, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f64_16x16x4f64(gs.y, v.x, ci, 0, 0, 0);
            g[s] = Gn[4 * s * WP];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = cmk<V>(cr[j], ci[j]);
    };
    // ---- forward row l = r0 + k:  z_l = G_l (r_l - c_l z_{l-1})
    auto fwd_step = [&](int k, int j) {
        const int buf = k & 1, l = r0 + k;
        const V cl = cmk<V>(k > 0 ? cnext.x : 0.0, k > 0 ? cnext.y : 0.0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            V v = rv[u];
            if (!PRE && tr_col(a.io, qrow + 4 * u)) {
                v.x += a.io.coef * (tb.x - ta.x);
                v.y += a.io.coef * (tb.y - ta.y);
            }
            Vs[buf][qrow + 4 * u][n] = csub(v, cmul(cl, z[u]));
        }
        const int ln = l + 1 < r1 ? l + 1 : l;
        cnext = a.cy[ln];
        load_rhs(ln);
        __syncthreads();
        V acc[4];
        mfma_block(greg[j], Vs[buf], acc, k + 2);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            z[u] = cmk<V>(rn_ok ? acc[u].x : 0.0, rn_ok ? acc[u].y : 0.0);
            if (rn_ok) a.Yw[ybase + (size_t)l * WP + 4 * u] = acc[u];
        }
    };
    // ---- backward row l = r1 - 2 - (k - nr):  y_l = z_l - b_l G_l y_{l+1}
    auto bwd_step = [&](int k, int j) {
        const int buf = k & 1, l = r1 - 2 - (k - nr);
        V zl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) zl[u] = zn[u];
        const V bl = bnext;
        const int lb = l - 1 >= r0 ? l - 1 : l;
        bnext = a.by[lb];
#pragma unroll
        for (int u = 0; u < 4; ++u) zn[u] = a.Yw[ybase + (size_t)lb * WP + 4 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u) Vs[buf][qrow + 4 * u][n] = z[u];
        __syncthreads();
        V acc[4];
        mfma_block(greg[j], Vs[buf], acc, k + 2);
        const bool store_y = !a.io.targets_only || l == r0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const V y = csub(zl[u], cmul(bl, acc[u]));
            z[u] = cmk<V>(rn_ok ? y.x : 0.0, rn_ok ? y.y : 0.0);
            if (rn_ok && (store_y || tm[u])) a.Yw[ybase + (size_t)l * WP + 4 * u] = y;
        }
    };
    int k = 0;
    for (; k + 2 <= nr; k += 2) { fwd_step(k, 0); fwd_step(k + 1, 1); }
    if (k < nr) fwd_step(k, 0);
    if (nr < 2) return;
    bnext = a.by[r1 - 2];
#pragma unroll
    for (int u = 0; u < 4; ++u) zn[u] = a.Yw[ybase + (size_t)(r1 - 2) * WP + 4 * u];
    // the first backward step uses ring slot nr % 2
    auto bwd_loop = [&](auto off_tag) {
        constexpr int OFF = decltype(off_tag)::value;
        int kb = nr;
        for (; kb + 2 <= nsteps; kb += 2) { bwd_step(kb, OFF); bwd_step(kb + 1, OFF ^ 1); }
        if (kb < nsteps) bwd_step(kb, OFF);
    };
    if (nr & 1) bwd_loop(std::integral_constant<int, 1>{});
    else bwd_loop(std::integral_constant<int, 0>{});
}
__global__ void __launch_bounds__(NT) k_phase_a_mfma64(SolveArgs<double> a) { phase_a_mfma64<false>(a, own_blk()); }
__global__ void __launch_bounds__(NT) k_phase_a_mfma64_b(BatchArgs<double> b) {
    Blk B;
    const SolveArgs<double> a = batch_strip(b, 1, B, true);
    phase_a_mfma64<true>(a, B);
}

// ---------------------------------------------------------------- phase B0
// a_c = G'_c r^_c for every separator (grid: separators x rhs groups), stored at row s_c.
template <typename T, int R>
__device__ __forceinline__ void phase_b0(const SolveArgs<T>& a, const Blk& B) {
    using V = cplx<T>;
    constexpr int G = 4, U = R / G;
    __shared__ V vin[WP][R];
    const int t = threadIdx.x, i = t & (WP - 1), g = t >> 6;
    const int c = B.x, rbase = B.y * R;
    const int s = c * a.m + a.m - 1;
    const V cs = ccast<V>(a.cy[s]), bs = ccast<V>(a.by[s]);
    const V zero = cmk<V>(0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = rbase + g + G * u;
        V v = zero;
        if (r < a.nrhs && i < a.W) {
            if (a.io.pre) v = a.Yw[((size_t)r * a.Ny + s) * WP + i];
            else v = gather<T>(a.io, r, s, i, a.Ny);
            v = csub(v, cmul(cs, a.Yw[((size_t)r * a.Ny + (s - 1)) * WP + i]));
            v = csub(v, cmul(bs, a.Yw[((size_t)r * a.Ny + (s + 1)) * WP + i]));
        }
        vin[i][g + G * u] = v;
    }
    __syncthreads();
    V acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = zero;
    matvec<T, R, G>(acc, fslot(a, s, 0), vin, a.W, i, g);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = rbase + g + G * u;
        if (r < a.nrhs) a.Yw[((size_t)r * a.Ny + s) * WP + i] = acc[u];
    }
}

template <typename T, int R>
__global__ void __launch_bounds__(NT) k_phase_b0(SolveArgs<T> a) { phase_b0<T, R>(a, own_blk()); }
template <typename T, int R>
__global__ void __launch_bounds__(NT) k_phase_b0_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    phase_b0<T, R>(a, B);
}

// ---------------------------------------------------------------- phase B
// One right-hand side per workgroup; the k-sum of every matvec is split over the 4 waves
// and combined through LDS.  Forward z'_0 = a_0, z'_c = a_c - K_c z'_{c-1}; backward
// x_{P-2} = z'_{P-2}, x_c = z'_c - U'_c x_{c+1}.  The blocks of the next D steps are in
// flight in registers while a step runs (ring of D+1 LDS buffers).
constexpr int ZMAX = 64;   // separators whose z' the chain keeps in LDS

// Thread (i, w) owns row i of the matvec and the 16 columns 16w..16w+15 of every block:
// the blocks of the next D steps are loaded straight into registers in that layout (no
// LDS staging), so a step is 16 multiply-adds from registers, one partial-sum exchange
// and two barriers.  ZB: the forward results z'_c stay in LDS (zb) for the backward pass
// and the forward inputs a_c are loaded D steps ahead into a register ring (requires
// P - 1 <= ZMAX); otherwise the next input is loaded one step ahead from global memory.
template <typename T, int D, bool ZB>
__device__ __forceinline__ void phase_b(const SolveArgs<T>& a, const Blk& B) {
    using V = cplx<T>;
    __shared__ V vec[WP];
    __shared__ V part[4][WP];
    __shared__ V zb[ZB ? ZMAX + 1 : 1][WP];     // row ZMAX: discard row for backward steps
    const int t = threadIdx.x, i = t & (WP - 1), w = t >> 6;
    const int r = B.x;
    const int ns = a.P - 1;                  // separators
    const int nf = ns - 1;                   // forward steps (c = 1..ns-1)
    const int steps = nf + (ns - 1);         // + backward steps (c = ns-2..0)
    if (steps <= 0) return;
    const int k0 = w * 16;
    auto sep = [&](int c) { return c * a.m + a.m - 1; };
    // separator row and factor block of step k (clamped to the last step: loads past the
    // end re-read the last block and are never used)
    auto sep_of = [&](int k) {
        k = k < steps ? k : steps - 1;
        return sep(k < nf ? k + 1 : ns - 2 - (k - nf));
    };
    auto blk = [&](int k) {
        k = k < steps ? k : steps - 1;
        return k < nf ? fslot(a, sep(k + 1), 1) : fslot(a, sep(ns - 2 - (k - nf)), 2);
    };
    auto load_blk = [&](int k, V (&b)[16]) {
        const V* g = blk(k) + (size_t)k0 * WP + i;
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) b[kk] = g[kk * WP];
    };
    // forward input of step k: a_{k+1} (clamped to the last forward step)
    auto fwd_in = [&](int k) { return sep((k < nf ? k : nf - 1) + 1); };
    V* Yr = a.Yw + (size_t)r * a.Ny * WP;
    // every thread keeps the value of its row i; the four waves hold identical copies
    const V a0 = Yr[(size_t)sep(0) * WP + i];    // z'_0 = a_0
    vec[i] = a0;
    V nextv = cmk<V>(0, 0);
    V av[D];
    if (ZB) {
        zb[0][i] = a0;
#pragma unroll
        for (int d = 0; d < D; ++d) av[d] = Yr[(size_t)fwd_in(d) * WP + i];
    } else {
        nextv = Yr[(size_t)sep_of(0) * WP + i];
    }
    V breg[D][16];
#pragma unroll
    for (int d = 0; d < D; ++d) load_blk(d, breg[d]);
    __syncthreads();
    auto step = [&](int k, int j) {
        const int s = sep_of(k);
        const bool fwd = k < nf;
        V curv;                                  // a_c (forward) or z'_c (backward)
        if (ZB) {
            const int cb = fwd ? ZMAX : ns - 2 - (k - nf);
            const V zr = zb[cb][i];
            curv = fwd ? av[j] : zr;
            av[j] = Yr[(size_t)fwd_in(k + D) * WP + i];
        } else {
            curv = nextv;
            nextv = Yr[(size_t)sep_of(k + 1) * WP + i];
        }
        V acc0 = cmk<V>(0, 0), acc1 = acc0;
#pragma unroll
        for (int kk = 0; kk < 16; kk += 2) {
            cfma(acc0, breg[j][kk], vec[k0 + kk]);
            cfma(acc1, breg[j][kk + 1], vec[k0 + kk + 1]);
        }
        part[w][i] = cadd(acc0, acc1);
        load_blk(k + D, breg[j]);               // block of step k + D into the freed slot
        __syncthreads();
        const V sum = cadd(cadd(part[0][i], part[1][i]), cadd(part[2][i], part[3][i]));
        const V v = csub(curv, sum);            // a_c - K_c z'  or  z'_c - U'_c x
        Yr[(size_t)s * WP + i] = v;
        vec[i] = v;
        if (ZB) zb[fwd ? k + 1 : ZMAX][i] = v;
        __syncthreads();
    };
    int k = 0;
    for (; k + D <= steps; k += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) step(k + j, j);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (k + j < steps) step(k + j, j);
}

template <typename T, int D, bool ZB>
__global__ void __launch_bounds__(NT) k_phase_b(SolveArgs<T> a) { phase_b<T, D, ZB>(a, own_blk()); }
template <typename T, int D, bool ZB>
__global__ void __launch_bounds__(NT) k_phase_b_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    phase_b<T, D, ZB>(a, B);
}

// ---------------------------------------------------------------- phase B, two levels
// The separator recurrences are cut into G groups of q separators.  With zeta / xi the
// recurrences of a group started from zero and the propagators Phi / Psi of the factor,
//   forward   z'_c = zeta_c + Phi_c z'_{first-1},   backward  x_c = xi_c + Psi_c x_{last+1},
// so the solve is: local forward chains (all groups in parallel), a chain over the groups'
// last separators, fix-up + local backward chains (parallel), a chain over the groups'
// first separators, fix-up (parallel): about 2q + 2G dependent steps instead of 2(P-1).
// A workgroup takes RB right-hand sides (every block it loads serves all of them); entries
// of right-hand sides beyond nrhs (a ragged last group) are computed from clamped loads and
// never stored.  The chains are latency bound: at 64 right-hand sides one per workgroup was
// the fastest (separator solve per strip 77 us; two per workgroup 84, four 105, eight 237).
//
// sep_chain: thread (i, w) owns row i and the 16 columns 16w..16w+15 of every block; wave
// w keeps its own copy of the vectors (their 16 entries it reads are produced by its own
// lanes), so a step needs one barrier (for the 4-wave partial sums).  Step k:
//   v_k = in_k + sgn (M_k vec),  out_k = v_k,  vec = v_k if chain (else vec stays v0).
// Blocks and inputs of the next D steps are in flight in registers.
template <typename T> struct SepRB { static constexpr int RB = 1; };

// SW: blk(k) is an operand-order block of Fw (complex64): the lane's columns 16 w + 2 j,
// 16 w + 2 j + 1 come in one 16-byte load; otherwise a factor block in its own layout.
template <typename T, int D, int RB, bool SW = false, typename BF, typename RF>
__device__ void sep_chain(int n, bool chain, const cplx<T> (&v0)[RB], T sgn, BF blk, RF row,
                          const bool (&okb)[RB], cplx<T> (*vecw)[RB][WP], cplx<T> (*part)[4][RB][WP]) {
    using V = cplx<T>;
    if (n <= 0) return;
    const int t = threadIdx.x, i = t & (WP - 1), w = t >> 6, k0 = 16 * w;
#pragma unroll
    for (int b = 0; b < RB; ++b) vecw[w][b][i] = v0[b];
    __builtin_amdgcn_wave_barrier();   // the wave's own lanes produced the entries it reads
    V breg[D][16], ireg[D][RB];
    auto load = [&](int k, V (&bl)[16], V (&x)[RB]) {
        const int kc = k < n ? k : n - 1;
        if constexpr (SW) {
            const float4* M = reinterpret_cast<const float4*>(blk(kc)) + w * 8 * 64 + i;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float4 v = M[j * 64];
                bl[2 * j] = make_float2(v.x, v.y);
                bl[2 * j + 1] = make_float2(v.z, v.w);
            }
        } else {
            const V* M = blk(kc) + (size_t)k0 * WP + i;
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) bl[kk] = M[kk * WP];
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) x[b] = row(kc, b)[i];
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, breg[d], ireg[d]);
    auto step = [&](int k, int j) {
        V acc[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[b] = cmk<V>(0, 0);
#pragma unroll
        for (int kk = 0; kk < 16; ++kk)
#pragma unroll
            for (int b = 0; b < RB; ++b) cfma(acc[b], breg[j][kk], vecw[w][b][k0 + kk]);
        V xin[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) xin[b] = ireg[j][b];
        load(k + D, breg[j], ireg[j]);
#pragma unroll
        for (int b = 0; b < RB; ++b) part[k & 1][w][b][i] = acc[b];
        __syncthreads();
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const V sum = cadd(cadd(part[k & 1][0][b][i], part[k & 1][1][b][i]),
                               cadd(part[k & 1][2][b][i], part[k & 1][3][b][i]));
            const V v = cmk<V>(xin[b].x + sgn * sum.x, xin[b].y + sgn * sum.y);
            if (okb[b]) row(k, b)[i] = v;
            if (chain) vecw[w][b][i] = v;
        }
        __builtin_amdgcn_wave_barrier();
    };
    int k = 0;
    for (; k + D <= n; k += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) step(k + j, j);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (k + j < n) step(k + j, j);
    __syncthreads();
}

// Independent updates v_k = in_k + M_k v (k < n, the same vectors v for every k): wave w
// takes k = w, w + 4, ..., each lane one row of the full 64-column products, so the waves
// need no barrier between updates.  v0 holds this lane's entries of the vectors.
template <typename T, int RB, typename BF, typename RF>
__device__ void sep_fix(int n, const cplx<T> (&v0)[RB], BF blk, RF row, const bool (&okb)[RB],
                        cplx<T> (*vecw)[RB][WP]) {
    using V = cplx<T>;
    const int i = threadIdx.x & (WP - 1), w = threadIdx.x >> 6;
#pragma unroll
    for (int b = 0; b < RB; ++b) vecw[w][b][i] = v0[b];
    __builtin_amdgcn_wave_barrier();
    for (int k = w; k < n; k += 4) {
        const V* M = blk(k) + i;
        V acc[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[b] = cmk<V>(0, 0);
#pragma unroll 16
        for (int kk = 0; kk < WP; ++kk) {
            const V m = M[(size_t)kk * WP];
#pragma unroll
            for (int b = 0; b < RB; ++b) cfma(acc[b], m, vecw[w][b][kk]);
        }
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (okb[b]) {
                V* dst = row(k, b) + i;
                *dst = cadd(*dst, acc[b]);
            }
    }
    __syncthreads();
}

template <typename T>
struct SepCtx {
    const SolveArgs<T>& a;
    int ns, rbase;
    __device__ int sep(int c) const { return c * a.m + a.m - 1; }
    __device__ int first(int g) const { return g * a.q; }
    __device__ int last(int g) const { return min(g * a.q + a.q, ns) - 1; }
    __device__ const cplx<T>* prop(int c, int dir) const { return a.Fs + ((size_t)c * 2 + dir) * BLK; }
    __device__ bool ok(int b) const { return rbase + b < a.nrhs; }
    __device__ int rhs(int b) const { return rbase + b < a.nrhs ? rbase + b : a.nrhs - 1; }   // clamped
    __device__ cplx<T>* yrow(int b, int c) const { return a.Yw + ((size_t)rhs(b) * a.Ny + sep(c)) * WP; }
};

#define SEPK_PROLOGUE_N(RBN)                                              \
    using V = cplx<T>;                                                    \
    constexpr int RB = (RBN);                                             \
    __shared__ V vecw[4][RB][WP];                                         \
    __shared__ V part[2][4][RB][WP];                                      \
    const int i = threadIdx.x & (WP - 1);                                 \
    SepCtx<T> X{a, a.P - 1, B.x * RB};                                    \
    bool okb[RB];                                                         \
    for (int b = 0; b < RB; ++b) okb[b] = X.ok(b);                        \
    auto vecs_at = [&](int c, V (&v)[RB]) {                               \
        for (int b = 0; b < RB; ++b) v[b] = X.yrow(b, c)[i];              \
    };                                                                    \
    (void)i;
#define SEPK_PROLOGUE SEPK_PROLOGUE_N(SepRB<T>::RB)
// The local chains without their independent products run 8 groups x the right-hand sides
// as workgroups: two right-hand sides per workgroup (every block load serves both) keep
// one workgroup per CU, which measured faster than two workgroups of one.
template <typename T> struct SepLocalRB { static constexpr int RB = 2; };

// local forward chains: zeta_c = a_c - K_c zeta_{c-1} inside group g = blockIdx.y.  First
// the group's right-hand sides a_c = G'_c r^_c, r^_c = r_s - c_s y_{s-1} - b_s y_{s+1}
// (s = sep(c)), independent per separator: wave w takes c0 + w, c0 + w + 4, ...
template <typename T, int D, bool SETUP>
__device__ __forceinline__ void sep_fwd_local(const SolveArgs<T>& a, const Blk& B) {
    SEPK_PROLOGUE_N(SETUP ? SepRB<T>::RB : SepLocalRB<T>::RB)
    const int g = B.y, c0 = X.first(g), c1 = X.last(g);
    if constexpr (SETUP) {
        const int w = threadIdx.x >> 6;
        for (int c = c0 + w; c <= c1; c += 4) {
            const int sr = X.sep(c);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int r = X.rhs(b);
                const V* Yr = a.Yw + (size_t)r * a.Ny * WP;
                V v = cmk<V>(0, 0);
                if (i < a.W) {
                    if (a.io.pre) v = Yr[(size_t)sr * WP + i];
                    else v = gather<T>(a.io, r, sr, i, a.Ny);
                    v = csub(v, cmul(ccast<V>(a.cy[sr]), Yr[(size_t)(sr - 1) * WP + i]));
                    v = csub(v, cmul(ccast<V>(a.by[sr]), Yr[(size_t)(sr + 1) * WP + i]));
                }
                vecw[w][b][i] = v;
            }
            __builtin_amdgcn_wave_barrier();
            const V* M = fslot(a, sr, 0) + i;
            V acc[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) acc[b] = cmk<V>(0, 0);
#pragma unroll 16
            for (int kk = 0; kk < WP; ++kk) {
                const V m = M[(size_t)kk * WP];
#pragma unroll
                for (int b = 0; b < RB; ++b) cfma(acc[b], m, vecw[w][b][kk]);
            }
#pragma unroll
            for (int b = 0; b < RB; ++b)
                if (okb[b]) a.Yw[((size_t)X.rhs(b) * a.Ny + sr) * WP + i] = acc[b];
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
    }
    V v0[RB];
    vecs_at(c0, v0);
    if constexpr (!SETUP && std::is_same<T, float>::value)
        sep_chain<T, D, RB, true>(c1 - c0, true, v0, T(-1),
                                  [&](int k) { return a.Fw + ((size_t)(c0 + 1 + k) * 4 + 0) * BLK; },
                                  [&](int k, int b) { return X.yrow(b, c0 + 1 + k); }, okb, vecw, part);
    else
        sep_chain<T, D, RB>(c1 - c0, true, v0, T(-1),
                            [&](int k) { return fslot(a, X.sep(c0 + 1 + k), 1); },
                            [&](int k, int b) { return X.yrow(b, c0 + 1 + k); }, okb, vecw, part);
}

// chain over the groups' last separators: z'_{last g} = zeta_{last g} + Phi_{last g} z'_{last g-1}
template <typename T, int D>
__device__ __forceinline__ void sep_fwd_top(const SolveArgs<T>& a, const Blk& B) {
    SEPK_PROLOGUE
    V v0[RB];
    vecs_at(X.last(0), v0);
    if constexpr (std::is_same<T, float>::value)
        sep_chain<T, D, RB, true>(a.G - 1, true, v0, T(1),
                                  [&](int k) { return a.Fw + ((size_t)X.last(k + 1) * 4 + 2) * BLK; },
                                  [&](int k, int b) { return X.yrow(b, X.last(k + 1)); }, okb, vecw, part);
    else
        sep_chain<T, D, RB>(a.G - 1, true, v0, T(1),
                            [&](int k) { return X.prop(X.last(k + 1), 0); },
                            [&](int k, int b) { return X.yrow(b, X.last(k + 1)); }, okb, vecw, part);
}

// fix-up of the group's other separators (unless FIX is false: done before, on MFMA), then
// its local backward chain xi_c = z'_c - U'_c xi_{c+1} (the group's last separator starts it)
template <typename T, int D, bool FIX>
__device__ __forceinline__ void sep_fix_bwd_local(const SolveArgs<T>& a, const Blk& B) {
    SEPK_PROLOGUE_N(FIX ? SepRB<T>::RB : SepLocalRB<T>::RB)
    const int g = B.y, c0 = X.first(g), c1 = X.last(g);
    if (FIX && g >= 1) {
        V vf[RB];
        vecs_at(X.last(g - 1), vf);
        sep_fix<T, RB>(c1 - c0, vf,
                       [&](int k) { return X.prop(c0 + k, 0); },
                       [&](int k, int b) { return X.yrow(b, c0 + k); }, okb, vecw);
    }
    V v0[RB];
    vecs_at(c1, v0);
    if constexpr (!FIX && std::is_same<T, float>::value)
        sep_chain<T, D, RB, true>(c1 - c0, true, v0, T(-1),
                                  [&](int k) { return a.Fw + ((size_t)(c1 - 1 - k) * 4 + 1) * BLK; },
                                  [&](int k, int b) { return X.yrow(b, c1 - 1 - k); }, okb, vecw, part);
    else
        sep_chain<T, D, RB>(c1 - c0, true, v0, T(-1),
                            [&](int k) { return fslot(a, X.sep(c1 - 1 - k), 2); },
                            [&](int k, int b) { return X.yrow(b, c1 - 1 - k); }, okb, vecw, part);
}

// chain over the groups' first separators: x_{first g} = xi_{first g} + Psi_{first g} x_{first g+1}
template <typename T, int D>
__device__ __forceinline__ void sep_bwd_top(const SolveArgs<T>& a, const Blk& B) {
    SEPK_PROLOGUE
    V v0[RB];
    vecs_at(X.first(a.G - 1), v0);
    if constexpr (std::is_same<T, float>::value)
        sep_chain<T, D, RB, true>(a.G - 1, true, v0, T(1),
                                  [&](int k) { return a.Fw + ((size_t)X.first(a.G - 2 - k) * 4 + 3) * BLK; },
                                  [&](int k, int b) { return X.yrow(b, X.first(a.G - 2 - k)); }, okb, vecw, part);
    else
        sep_chain<T, D, RB>(a.G - 1, true, v0, T(1),
                            [&](int k) { return X.prop(X.first(a.G - 2 - k), 1); },
                            [&](int k, int b) { return X.yrow(b, X.first(a.G - 2 - k)); }, okb, vecw, part);
}

// fix-up of the group's other separators: x_c = xi_c + Psi_c x_{first g+1}
template <typename T, int D>
__device__ __forceinline__ void sep_bwd_fix(const SolveArgs<T>& a, const Blk& B) {
    SEPK_PROLOGUE
    const int g = B.y, c0 = X.first(g), c1 = X.last(g);
    V vf[RB];
    vecs_at(X.first(g + 1), vf);
    sep_fix<T, RB>(c1 - c0, vf,
                   [&](int k) { return X.prop(c0 + 1 + k, 1); },
                   [&](int k, int b) { return X.yrow(b, c0 + 1 + k); }, okb, vecw);
}
#undef SEPK_PROLOGUE
#undef SEPK_PROLOGUE_N
// The separators' independent products for 16 right-hand sides at a time on MFMA (complex64):
//   MODE 0  a_c = G'_c r^_c for every separator c (the local forward chains' right-hand sides)
//   MODE 1  z'_c += Phi_c z'_{last g-1} for the separators of group g >= 1 but its last
//   MODE 2  x_c += Psi_c x_{first g+1} for the separators of group g < G - 1 but its first
// Grid (separators, right-hand-side groups).  Each workgroup stages its 64 x 16 operand in
// LDS and forms one (64 x 64) by (64 x 16) product in four real products (three lose
// accuracy that the iteration counts of the complex64 solves feel), so a block is read
// once per 16 right-hand sides (the per-right-hand-side workgroups of the chains read it once
// each, which makes these products bound by the CU's load bandwidth).  A workgroup writes only
// its own separator and reads only separators that no workgroup of the launch writes.
template <int MODE>
__device__ __forceinline__ void sep_par_mfma(const SolveArgs<float>& a, const Blk& B) {
    using V = float2;
    __shared__ V X[WP][17];
    const int ns = a.P - 1, c = B.x, g = c / a.q;
    const int c0 = g * a.q, c1 = min(c0 + a.q, ns) - 1;
    if (MODE == 1 && (g < 1 || c == c1)) return;
    if (MODE == 2 && (g >= a.G - 1 || c == c0)) return;
    const int sr = c * a.m + a.m - 1;                                   // the separator's row
    const int so = MODE == 1 ? (c0 - 1) * a.m + a.m - 1 : (c1 + 1) * a.m + a.m - 1;   // operand's
    const V* M = MODE == 0 ? fslot(a, sr, 0) : a.Fs + ((size_t)c * 2 + (MODE == 1 ? 0 : 1)) * BLK;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = lane & 15, q4 = lane >> 4;
    const int rbase = B.y * 16;
    // every load of the workgroup is issued before the first use: the A operands, then the
    // operand tile (four passes of 256 threads; branch-free, clamped addresses)
    V gA[16];
    const V* F = M + 16 * w + n;
#pragma unroll
    for (int s = 0; s < 16; ++s) gA[s] = F[(4 * s + q4) * WP];
    constexpr int NP = 16 * WP / NT;
    RawRhs raw[NP];
    V ym[NP], yp[NP], own[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int idx = threadIdx.x + p * NT, q = idx >> 6, k = idx & (WP - 1), r = rbase + q;
        const V* Yr = a.Yw + (size_t)(r < a.nrhs ? r : a.nrhs - 1) * a.Ny * WP + k;
        if (MODE == 0) {
            if (a.io.pre) own[p] = Yr[(size_t)sr * WP];
            else raw[p] = load_raw(a.io, r, sr, k, a.Ny, a.nrhs, a.W);
            ym[p] = Yr[(size_t)(sr - 1) * WP];
            yp[p] = Yr[(size_t)(sr + 1) * WP];
        } else {
            ym[p] = Yr[(size_t)so * WP];
        }
    }
    // the fix-ups add to this lane's four entries of the separator
    const int rn = rbase + n;
    V* y = a.Yw + ((size_t)(rn < a.nrhs ? rn : a.nrhs - 1) * a.Ny + sr) * WP + 16 * w + 4 * q4;
    V yold[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) yold[u] = MODE == 0 ? make_float2(0.f, 0.f) : y[u];
    const double2 cys = a.cy[sr], bys = a.by[sr];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int idx = threadIdx.x + p * NT, q = idx >> 6, k = idx & (WP - 1);
        V v = make_float2(0.f, 0.f);
        if (rbase + q < a.nrhs && k < a.W) {
            if (MODE == 0) {
                if (a.io.pre) v = own[p];
                else v = combine<float>(a.io, raw[p]);
                v = csub(v, cmul(ccast<V>(cys), ym[p]));
                v = csub(v, cmul(ccast<V>(bys), yp[p]));
            } else {
                v = ym[p];
            }
        }
        X[k][q] = v;
    }
    __syncthreads();
    V xb[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) xb[s] = X[4 * s + q4][n];
    __builtin_amdgcn_sched_barrier(0);
    mf4 aR = {0.f, 0.f, 0.f, 0.f}, aI = aR;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const V g4 = gA[s];
        const V x = xb[s];
        aR = __builtin_amdgcn_mfma_f32_16x16x4f32(g4.x, x.x, aR, 0, 0, 0);
        aI = __builtin_amdgcn_mfma_f32_16x16x4f32(g4.x, x.y, aI, 0, 0, 0);
        aR = __builtin_amdgcn_mfma_f32_16x16x4f32(-g4.y, x.y, aR, 0, 0, 0);
        aI = __builtin_amdgcn_mfma_f32_16x16x4f32(g4.y, x.x, aI, 0, 0, 0);
    }
    if (rn >= a.nrhs) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const V v = make_float2(aR[u], aI[u]);
        y[u] = MODE == 0 ? v : cadd(yold[u], v);
    }
}

template <int MODE>
__global__ void __launch_bounds__(NT) k_sep_par_mfma(SolveArgs<float> a) { sep_par_mfma<MODE>(a, own_blk()); }
template <int MODE>
__global__ void __launch_bounds__(NT) k_sep_par_mfma_multi(MultiArgs<float> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_par_mfma<MODE>(m.a[k], b);
}

template <typename T, int D, bool SETUP = true>
__global__ void __launch_bounds__(NT) k_sep_fwd_local(SolveArgs<T> a) { sep_fwd_local<T, D, SETUP>(a, own_blk()); }
template <typename T, int D, bool SETUP = true>
__global__ void __launch_bounds__(NT) k_sep_fwd_local_multi(MultiArgs<T> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_fwd_local<T, D, SETUP>(m.a[k], b);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_fwd_top(SolveArgs<T> a) { sep_fwd_top<T, D>(a, own_blk()); }
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_fwd_top_multi(MultiArgs<T> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_fwd_top<T, D>(m.a[k], b);
}
template <typename T, int D, bool FIX = true>
__global__ void __launch_bounds__(NT) k_sep_fix_bwd_local(SolveArgs<T> a) { sep_fix_bwd_local<T, D, FIX>(a, own_blk()); }
template <typename T, int D, bool FIX = true>
__global__ void __launch_bounds__(NT) k_sep_fix_bwd_local_multi(MultiArgs<T> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_fix_bwd_local<T, D, FIX>(m.a[k], b);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_top(SolveArgs<T> a) { sep_bwd_top<T, D>(a, own_blk()); }
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_top_multi(MultiArgs<T> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_bwd_top<T, D>(m.a[k], b);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_fix(SolveArgs<T> a) { sep_bwd_fix<T, D>(a, own_blk()); }
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_fix_multi(MultiArgs<T> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) sep_bwd_fix<T, D>(m.a[k], b);
}

// the same for the strips of a batch
template <int MODE>
__global__ void __launch_bounds__(NT) k_sep_par_mfma_b(BatchArgs<float> b) {
    Blk B;
    const SolveArgs<float> a = batch_strip(b, 1, B);
    sep_par_mfma<MODE>(a, B);
}
template <typename T, int D, bool SETUP = true>
__global__ void __launch_bounds__(NT) k_sep_fwd_local_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    sep_fwd_local<T, D, SETUP>(a, B);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_fwd_top_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    sep_fwd_top<T, D>(a, B);
}
template <typename T, int D, bool FIX = true>
__global__ void __launch_bounds__(NT) k_sep_fix_bwd_local_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    sep_fix_bwd_local<T, D, FIX>(a, B);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_top_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    sep_bwd_top<T, D>(a, B);
}
template <typename T, int D>
__global__ void __launch_bounds__(NT) k_sep_bwd_fix_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B);
    sep_bwd_fix<T, D>(a, B);
}

// ---------------------------------------------------------------- phase C (all columns)
template <typename T, int R>
__device__ __forceinline__ void phase_c(const SolveArgs<T>& a, const Blk& B) {
    using V = cplx<T>;
    constexpr int G = 4, U = R / G;
    __shared__ V va[WP][R];
    __shared__ V vb[WP][R];
    const int t = threadIdx.x, i = t & (WP - 1), g = t >> 6;
    const int l = B.x, rbase = B.y * R;
    const int c = l / a.m;
    const bool is_sep = (c < a.P - 1) && (l == c * a.m + a.m - 1);
    const bool top = !is_sep && c > 0;
    const bool bot = !is_sep && c < a.P - 1;
    const V zero = cmk<V>(0, 0);
    V x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = rbase + g + G * u;
        // clamped load, component-wise select (a select of whole values goes through scratch)
        const bool rok = r < a.nrhs;
        const V xl = a.Yw[((size_t)(rok ? r : 0) * a.Ny + l) * WP + i];
        x[u] = cmk<V>(rok ? xl.x : T(0), rok ? xl.y : T(0));
        V xa = zero, xb = zero;
        if (r < a.nrhs) {
            if (top) xa = a.Yw[((size_t)r * a.Ny + (c * a.m - 1)) * WP + i];
            if (bot) xb = a.Yw[((size_t)r * a.Ny + (c * a.m + a.m - 1)) * WP + i];
        }
        va[i][g + G * u] = xa;
        vb[i][g + G * u] = xb;
    }
    __syncthreads();
    if (top || bot) {
        V acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = zero;
        if (top) matvec<T, R, G>(acc, fslot(a, l, 1), va, a.W, i, g);
        if (bot) matvec<T, R, G>(acc, fslot(a, l, 2), vb, a.W, i, g);
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = csub(x[u], acc[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = rbase + g + G * u;
        if (r < a.nrhs && i < a.W) scatter<T>(a, r, l, i, x[u]);
    }
}

template <typename T, int R>
__global__ void __launch_bounds__(NT) k_phase_c(SolveArgs<T> a) { phase_c<T, R>(a, own_blk()); }
template <typename T, int R>
__global__ void __launch_bounds__(NT) k_phase_c_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B, true);
    phase_c<T, R>(a, B);
}

// ---------------------------------------------------------------- phase C (all columns), MFMA
// complex64: per chunk and group of 16 right-hand sides, x_l = y_l - [X~_l Y~_l] [x_a; x_b]
// for every row l of the chunk (the separator closing it is final after phase B and only
// copied), one (64 x 128) by (128 x 16) product per row on v_mfma_f32_16x16x4f32 in three
// real products.  The chunk's two separator vectors are the B operands of every row and stay
// in registers; each lane loads its A operands (A[16w + n][4s + q4] of X~_l, then of Y~_l)
// straight from global memory.  The 64 x 16 result is transposed through LDS so that the
// scatter writes whole rows of one right-hand side (consecutive x positions) instead of
// four-element pieces of sixteen right-hand sides.  Grid (chunks, right-hand-side groups,
// row groups): row group z takes the chunk's rows z, z + gridDim.z, ...
__device__ __forceinline__ void phase_c_mfma(const SolveArgs<float>& a, const Blk& B) {
    using V = float2;
    __shared__ V X[2 * WP][16];
    __shared__ V O[16][WP + 1];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = lane & 15, q4 = lane >> 4;
    const int c = B.x, rbase = B.y * 16;
    const int r0 = c * a.m;
    const bool has_a = c > 0, has_b = c < a.P - 1;
    const int r1 = has_b ? c * a.m + a.m - 1 : a.Ny;     // separator closing the chunk, or Ny
    const int nrow = r1 - r0 + (has_b ? 1 : 0);
    const V zero = make_float2(0.f, 0.f);
    for (int idx = t; idx < 2 * WP * 16; idx += NT) {
        const int k = idx >> 4, q = idx & 15, r = rbase + q, kk = k & (WP - 1);
        V v = zero;
        if (r < a.nrhs && kk < a.W) {
            if (k < WP) {
                if (has_a) v = a.Yw[((size_t)r * a.Ny + (r0 - 1)) * WP + kk];
            } else if (has_b) {
                v = a.Yw[((size_t)r * a.Ny + r1) * WP + kk];
            }
        }
        X[k][q] = v;
    }
    __syncthreads();
    float xr[32], xi[32], xs[32];
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        const V v = X[4 * s + q4][n];
        xr[s] = v.x; xi[s] = v.y; xs[s] = v.x + v.y;
    }
    const int rn = rbase + n;
    const int qrow = 16 * w + 4 * q4;
    const size_t ybase = (size_t)(rn < a.nrhs ? rn : 0) * a.Ny * WP + qrow;
    for (int j = B.z; j < nrow; j += B.nz) {
        const int l = r0 + j;
        mf4 m1 = {0.f, 0.f, 0.f, 0.f}, m2 = m1, m3 = m1;
        if (!(has_b && l == r1)) {
            if (has_a) {
                const V* F = fslot(a, l, 1) + 16 * w + n;
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const V g = F[(4 * s + q4) * WP];
                    m1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, xr[s], m1, 0, 0, 0);
                    m2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, xi[s], m2, 0, 0, 0);
                    m3 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x + g.y, xs[s], m3, 0, 0, 0);
                }
            }
            if (has_b) {
                const V* F = fslot(a, l, 2) + 16 * w + n;
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const V g = F[(4 * s + q4) * WP];
                    m1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, xr[16 + s], m1, 0, 0, 0);
                    m2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, xi[16 + s], m2, 0, 0, 0);
                    m3 = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x + g.y, xs[16 + s], m3, 0, 0, 0);
                }
            }
        }
        V y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) y[u] = a.Yw[ybase + (size_t)l * WP + u];
        __syncthreads();                                  // the previous row's scatter has read O
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float p1 = m1[u], p2 = m2[u], p3 = m3[u];
            O[n][qrow + u] = make_float2(y[u].x - (p1 - p2), y[u].y - (p3 - p1 - p2));
        }
        __syncthreads();
        for (int idx = t; idx < 16 * WP; idx += NT) {
            const int q = idx >> 6, i = idx & (WP - 1), r = rbase + q;
            if (r < a.nrhs && i < a.W) scatter<float>(a, r, l, i, O[q][i]);
        }
    }
}
__global__ void __launch_bounds__(NT) k_phase_c_mfma(SolveArgs<float> a) { phase_c_mfma(a, own_blk()); }
__global__ void __launch_bounds__(NT) k_phase_c_mfma_b(BatchArgs<float> b, int nz) {
    Blk B;
    const SolveArgs<float> a = batch_strip(b, nz, B, true);
    phase_c_mfma(a, B);
}
__global__ void __launch_bounds__(NT) k_phase_c_mfma_multi(MultiArgs<float> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) phase_c_mfma(m.a[k], b);
}

// ---------------------------------------------------------------- phase C (target columns)
// Only the 8 compact columns tcol[] of the strip; thread = (slot = t / 32, rhs = t % 32);
// ROWS consecutive rows per workgroup share the separator vectors of their chunk.
constexpr int CT_ROWS = 8;

template <typename T>
__device__ __forceinline__ void phase_c_targets(const SolveArgs<T>& a, const Blk& B) {
    using V = cplx<T>;
    constexpr int RC = 32;
    __shared__ V va[WP][RC];
    __shared__ V vb[WP][RC];
    __shared__ V fr[16][WP];
    const int t = threadIdx.x, rbase = B.y * RC;
    const int sl = t / RC, rr = t % RC, r = rbase + rr;
    const int q = a.tcol[sl];
    const V zero = cmk<V>(0, 0);
    const int l0 = B.x * CT_ROWS, l1 = min(a.Ny, l0 + CT_ROWS);
    int loaded = -1;
    for (int l = l0; l < l1; ++l) {
        const int c = l / a.m;
        if (c != loaded) {                       // uniform over the workgroup
            __syncthreads();
            for (int idx = t; idx < WP * RC; idx += NT) {
                const int k = idx / RC, q2 = idx % RC, r2 = rbase + q2;
                V xa = zero, xb = zero;
                if (r2 < a.nrhs && k < a.W) {
                    if (c > 0) xa = a.Yw[((size_t)r2 * a.Ny + (c * a.m - 1)) * WP + k];
                    if (c < a.P - 1) xb = a.Yw[((size_t)r2 * a.Ny + (c * a.m + a.m - 1)) * WP + k];
                }
                va[k][q2] = xa;
                vb[k][q2] = xb;
            }
            __syncthreads();
            loaded = c;
        }
        const bool is_sep = (c < a.P - 1) && (l == c * a.m + a.m - 1);
        // the 2 x 8 compact spike rows of row l (zero outside the strip width)
        const V* src = a.Fc + (size_t)l * 2 * 8 * WP;
        for (int idx = t; idx < 2 * 8 * WP; idx += NT) fr[idx / WP][idx % WP] = src[idx];
        __syncthreads();
        if (q >= 0 && r < a.nrhs) {
            V x = a.Yw[((size_t)r * a.Ny + l) * WP + q];
            if (!is_sep) {
                V acc = zero;
#pragma unroll 16
                for (int k = 0; k < WP; ++k) {
                    cfma(acc, fr[sl][k], va[k][rr]);
                    cfma(acc, fr[8 + sl][k], vb[k][rr]);
                }
                x = csub(x, acc);
            }
            scatter<T>(a, r, l, q, x);
        }
        __syncthreads();
    }
}

template <typename T>
__global__ void __launch_bounds__(NT) k_phase_c_targets(SolveArgs<T> a) { phase_c_targets<T>(a, own_blk()); }
template <typename T>
__global__ void __launch_bounds__(NT) k_phase_c_targets_b(BatchArgs<T> b) {
    Blk B;
    const SolveArgs<T> a = batch_strip(b, 1, B, true);
    phase_c_targets<T>(a, B);
}

// complex64 target columns per chunk as one small product on v_mfma_f32_16x16x4f32:
// rows (l, t) of the chunk's interior rows l and the 8 target columns t, columns 16
// right-hand sides, k over [x_above; x_below] (128): out = Fc(l, t, :) [xa; xb], x = y - out.
// Grid (chunks, right-hand-side groups of 16, tile groups); wave w of tile group z takes row
// tiles w + 4 z, w + 4 z + 4 gridDim.z, ...  Every workgroup stages the chunk's two separator
// vectors; the separator row that closes the chunk is copied (its x is final after phase B)
// by tile group 0.
__device__ __forceinline__ void phase_c_targets_mfma(const SolveArgs<float>& a, const Blk& B) {
    using V = float2;
    __shared__ V X[2 * WP][17];
    __shared__ V XF[2][WP][17];
    __shared__ int tcs[8];                 // the target columns (the tiles' output addresses)
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = lane & 15, q4 = lane >> 4;
    const int c = B.x, rbase = B.y * 16;
    const int r0 = c * a.m;
    const int r1 = (c < a.P - 1) ? c * a.m + a.m - 1 : a.Ny;
    const int nr = r1 - r0;
    const bool has_a = c > 0, has_b = c < a.P - 1;
    // The two-level separator solve leaves the fix-up x_s = xi_s + Psi_s x_{first(g+1)} of the
    // separators that are not the first of their group g < G-1 to this kernel: each chunk
    // applies it to its own two separators (side 0 above, side 1 below).
    bool fix[2];
    int sfirst[2], sidx[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int cs = side ? c : c - 1;
        const int g = cs >= 0 && a.q > 0 ? cs / a.q : 0;
        sidx[side] = cs;
        fix[side] = a.io.targets_only && a.G >= 2 && a.Fs && a.P > 2 && (side ? has_b : has_a) &&
                    g < a.G - 1 && cs != g * a.q;
        sfirst[side] = (g + 1) * a.q;
    }
    // branch-free staging: every lane loads (a clamped address) and keeps or drops the value
    {
        V xv[8], fv[8];
        bool keepv[8], keepf[8];
        // element e: right-hand side j = e / 128, k = e % 128 (consecutive lanes read
        // consecutive columns of one right-hand side's row)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = t + NT * u;
            const int k = e & (2 * WP - 1), j = e >> 7, r = rbase + j, kk = k & (WP - 1);
            const bool above = k < WP;
            keepv[u] = r < a.nrhs && kk < a.W && (above ? has_a : has_b);
            const int row = above ? (has_a ? r0 - 1 : r0) : (has_b ? r1 : r0);
            const size_t rr = (size_t)(r < a.nrhs ? r : 0) * a.Ny;
            xv[u] = a.Yw[(rr + row) * WP + kk];
            const int side = above ? 0 : 1;
            keepf[u] = keepv[u] && fix[side];
            // a dropped value reads row 0: an address the compiler cannot equate with xv's,
            // which would make it reuse xv behind a wait for every element
            const int frow = fix[side] ? sfirst[side] * a.m + a.m - 1 : 0;
            fv[u] = a.Yw[(rr + frow) * WP + kk];
        }
        const int tc = a.tcol[t & 7];          // waited for with the loads above
        if (t < 8) tcs[t] = tc;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = t + NT * u;
            const int k = e & (2 * WP - 1), j = e >> 7;
            X[k][j] = make_float2(keepv[u] ? xv[u].x : 0.f, keepv[u] ? xv[u].y : 0.f);
            XF[k >> 6][k & (WP - 1)][j] = make_float2(keepf[u] ? fv[u].x : 0.f, keepf[u] ? fv[u].y : 0.f);
        }
    }
    __syncthreads();
    if (fix[0] || fix[1]) {
        // X[side] += Psi_s XF[side] (64 x 64 by 64 x 16 on MFMA in four real products;
        // wave w: rows 16 w ..); both sides' blocks are loaded before either product
        V g[2][16];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const V* Ps = a.Fs + ((size_t)(fix[side] ? sidx[side] : 0) * 2 + 1) * BLK + 16 * w + n;
#pragma unroll
            for (int s4 = 0; s4 < 16; ++s4) g[side][s4] = Ps[(size_t)(4 * s4 + q4) * WP];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (!fix[side]) continue;
            mf4 aR = {0.f, 0.f, 0.f, 0.f}, aI = aR;
#pragma unroll
            for (int s4 = 0; s4 < 16; ++s4) {
                const V g0 = g[side][s4];
                const V v0 = XF[side][4 * s4 + q4][n];
                aR = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x, v0.x, aR, 0, 0, 0);
                aI = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x, v0.y, aI, 0, 0, 0);
                aR = __builtin_amdgcn_mfma_f32_16x16x4f32(-g0.y, v0.y, aR, 0, 0, 0);
                aI = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.y, v0.x, aI, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                V& xr = X[WP * side + 16 * w + 4 * q4 + j][n];
                xr = make_float2(xr.x + aR[j], xr.y + aI[j]);
            }
        }
        __syncthreads();
    }
    const int rn = rbase + n;
    const int nrows = nr * 8, ntile = (nrows + 15) / 16;
    // k-step s of a side takes the column kc(s) = 8 (s / 2) + 2 q4 + s % 2 in this lane, so
    // that the lane's two columns of k-steps 2i, 2i + 1 are adjacent and come in one 16-byte
    // load (each load instruction reads 64 contiguous bytes of 16 compact rows).  The B panel
    // of every tile, [x_above; x_below], in the same order:
    V vb[32];
#pragma unroll
    for (int s4 = 0; s4 < 32; ++s4) vb[s4] = X[WP * (s4 >> 4) + 8 * ((s4 & 15) >> 1) + 2 * q4 + (s4 & 1)][n];
    for (int tile = w + 4 * B.z; tile < ntile; tile += 4 * B.nz) {
        // A operands: row rho = 16 tile + n (clamped), columns kc(s) of both sides
        const int rho = min(16 * tile + n, nrows - 1);
        const int l = r0 + (rho >> 3), tt = rho & 7;
        const float4* fa = reinterpret_cast<const float4*>(a.Fc + ((size_t)(l * 2 + 0) * 8 + tt) * WP) + q4;
        const float4* fb = reinterpret_cast<const float4*>(a.Fc + ((size_t)(l * 2 + 1) * 8 + tt) * WP) + q4;
        V g[32];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 va = fa[4 * i], vb4 = fb[4 * i];
            g[2 * i] = make_float2(va.x, va.y);
            g[2 * i + 1] = make_float2(va.z, va.w);
            g[16 + 2 * i] = make_float2(vb4.x, vb4.y);
            g[16 + 2 * i + 1] = make_float2(vb4.z, vb4.w);
        }
        // the y values of this lane's four outputs, loaded before the products (the
        // stores of the outputs below could alias them, so they cannot move up by themselves)
        V y[4];
        int qo[4], lo4[4];
        bool ok[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ro = 16 * tile + 4 * q4 + j;
            const int roc = ro < nrows ? ro : nrows - 1;
            lo4[j] = r0 + (roc >> 3);
            qo[j] = tcs[roc & 7];
            ok[j] = ro < nrows && qo[j] >= 0 && rn < a.nrhs;
            const size_t yi = ((size_t)(rn < a.nrhs ? rn : 0) * a.Ny + lo4[j]) * WP + (qo[j] >= 0 ? qo[j] : 0);
            y[j] = a.Yw[yi];
        }
        __builtin_amdgcn_sched_barrier(0);       // every operand of the tile in flight first
        // four real products per complex one (the three-product form costs accuracy here)
        mf4 aR0 = {0.f, 0.f, 0.f, 0.f}, aI0 = aR0, aR1 = aR0, aI1 = aR0;
#pragma unroll
        for (int s4 = 0; s4 < 32; s4 += 2) {
            const V g0 = g[s4], g1 = g[s4 + 1];
            const V v0 = vb[s4], v1 = vb[s4 + 1];
            aR0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x, v0.x, aR0, 0, 0, 0);
            aI0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.x, v0.y, aI0, 0, 0, 0);
            aR1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.x, v1.x, aR1, 0, 0, 0);
            aI1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.x, v1.y, aI1, 0, 0, 0);
            aR0 = __builtin_amdgcn_mfma_f32_16x16x4f32(-g0.y, v0.y, aR0, 0, 0, 0);
            aI0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0.y, v0.x, aI0, 0, 0, 0);
            aR1 = __builtin_amdgcn_mfma_f32_16x16x4f32(-g1.y, v1.y, aR1, 0, 0, 0);
            aI1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1.y, v1.x, aI1, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (ok[j]) {
                const V x = make_float2(y[j].x - (aR0[j] + aR1[j]), y[j].y - (aI0[j] + aI1[j]));
                scatter<float>(a, rn, lo4[j], qo[j], x);
            }
        }
    }
    // the separator row closing this chunk (its x, fixed up above if needed, is in X)
    if (has_b && B.z == 0 && t < 8 * 16) {
        const int tt = t >> 4, r = rbase + (t & 15), q = tcs[tt];
        if (q >= 0 && r < a.nrhs) scatter<float>(a, r, r1, q, X[WP + q][t & 15]);
    }
}
__global__ void __launch_bounds__(NT) k_phase_c_targets_mfma(SolveArgs<float> a) {
    phase_c_targets_mfma(a, own_blk());
}
__global__ void __launch_bounds__(NT) k_phase_c_targets_mfma_b(BatchArgs<float> b, int nz) {
    Blk B;
    const SolveArgs<float> a = batch_strip(b, nz, B, true);
    phase_c_targets_mfma(a, B);
}
__global__ void __launch_bounds__(NT) k_phase_c_targets_mfma_multi(MultiArgs<float> m) {
    int k;
    Blk b;
    if (multi_blk(m, k, b)) phase_c_targets_mfma(m.a[k], b);
}

template <typename T> struct Depth { static constexpr int D = 2; };
template <> struct Depth<float> { static constexpr int D = 4; };

// R = 4: panels of at most 4 right-hand sides, one workgroup per chunk takes all of them
template <typename T, int R>
void launch_phase_a(const SolveArgs<T>& a, int, hipStream_t st) {
    const dim3 g(a.P), b(NT);
    if (a.nrhs == 1) hipLaunchKernelGGL((k_phase_a_few<T, 1>), g, b, 0, st, a);
    else if (a.nrhs == 2) hipLaunchKernelGGL((k_phase_a_few<T, 2>), g, b, 0, st, a);
    else hipLaunchKernelGGL((k_phase_a_few<T, 4>), g, b, 0, st, a);
}
template <>
void launch_phase_a<float, 16>(const SolveArgs<float>& a, int RG, hipStream_t st) {
    hipLaunchKernelGGL(k_phase_a_mfma<2>, dim3(a.P, RG), dim3(NT), 0, st, a);
}

template <>
void launch_phase_a<double, 16>(const SolveArgs<double>& a, int RG, hipStream_t st) {
    hipLaunchKernelGGL(k_phase_a_mfma64, dim3(a.P, RG), dim3(NT), 0, st, a);
}

template <typename T, int R>
hipError_t run(const SolveArgs<T>& a, bool targets, hipStream_t st, KTimer* kt) {
    const int RG = (a.nrhs + R - 1) / R;
    if (kt) kt->begin(K_PHASE_A, st);
    launch_phase_a<T, R>(a, RG, st);
    if (kt) kt->end(K_PHASE_A, st);
    if (a.P > 1) {
        if (kt) kt->begin(K_PHASE_B, st);
        if (a.P > 2 && a.G >= 2 && a.Fs) {
            constexpr int DS = Depth<T>::D;
            const unsigned nr = (unsigned)((a.nrhs + SepRB<T>::RB - 1) / SepRB<T>::RB);
            if constexpr (std::is_same<T, float>::value) {
                // the independent products on MFMA, the chains one right-hand side per
                // workgroup; targets-only solves fix the separators up inside phase C
                const dim3 gp(a.P - 1, (a.nrhs + 15) / 16);
                const unsigned nl = (unsigned)((a.nrhs + SepLocalRB<T>::RB - 1) / SepLocalRB<T>::RB);
                hipLaunchKernelGGL(k_sep_par_mfma<0>, gp, dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_fwd_local<T, DS, false>), dim3(nl, a.G), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_fwd_top<T, DS>), dim3(nr), dim3(NT), 0, st, a);
                hipLaunchKernelGGL(k_sep_par_mfma<1>, gp, dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_fix_bwd_local<T, DS, false>), dim3(nl, a.G), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_bwd_top<T, DS>), dim3(nr), dim3(NT), 0, st, a);
                if (!targets) hipLaunchKernelGGL(k_sep_par_mfma<2>, gp, dim3(NT), 0, st, a);
            } else {
                // the local forward chains form their own right-hand sides a_c
                hipLaunchKernelGGL((k_sep_fwd_local<T, DS>), dim3(nr, a.G), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_fwd_top<T, DS>), dim3(nr), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_fix_bwd_local<T, DS>), dim3(nr, a.G), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_bwd_top<T, DS>), dim3(nr), dim3(NT), 0, st, a);
                hipLaunchKernelGGL((k_sep_bwd_fix<T, DS>), dim3(nr, a.G - 1), dim3(NT), 0, st, a);
            }
        } else {
            hipLaunchKernelGGL((k_phase_b0<T, R>), dim3(a.P - 1, RG), dim3(NT), 0, st, a);
        }
        if (a.P > 2 && !(a.G >= 2 && a.Fs)) {
            if (a.P - 1 <= ZMAX)
                hipLaunchKernelGGL((k_phase_b<T, Depth<T>::D, true>), dim3(a.nrhs), dim3(NT), 0, st, a);
            else
                hipLaunchKernelGGL((k_phase_b<T, Depth<T>::D, false>), dim3(a.nrhs), dim3(NT), 0, st, a);
        }
        if (kt) kt->end(K_PHASE_B, st);
    }
    if (kt) kt->begin(K_PHASE_C, st);
    if (targets) {
        if constexpr (std::is_same<T, float>::value) {
            // the 16-row tiles of a chunk are spread over TS workgroups (two tiles per wave
            // at m = 32: measured faster than one or four)
            const int tiles = ((a.m - 1) * 8 + 15) / 16;
            const int TS = std::min(8, std::max(1, (tiles + 7) / 8));      // targets_groups
            hipLaunchKernelGGL(k_phase_c_targets_mfma, dim3(a.P, (a.nrhs + 15) / 16, TS), dim3(NT), 0, st, a);
        }
        else
            hipLaunchKernelGGL((k_phase_c_targets<T>), dim3((a.Ny + CT_ROWS - 1) / CT_ROWS, (a.nrhs + 31) / 32),
                               dim3(NT), 0, st, a);
    }
    else if constexpr (std::is_same<T, float>::value) {
        // about four workgroups per CU: row groups split each chunk's rows (phase_c_groups)
        const int per = a.P * ((a.nrhs + 15) / 16);
        const int TS = std::max(1, std::min(std::min(8, a.m), (1024 + per - 1) / per));
        hipLaunchKernelGGL(k_phase_c_mfma, dim3(a.P, (a.nrhs + 15) / 16, TS), dim3(NT), 0, st, a);
    } else
        hipLaunchKernelGGL((k_phase_c<T, R>), dim3(a.Ny, RG), dim3(NT), 0, st, a);
    if (kt) kt->end(K_PHASE_C, st);
    return hipGetLastError();
}

template <typename T>
SolveArgs<T> solve_args(const DevTables& t, const Geom& g, const Chunks& ch, int s, int fs,
                        const cplx<T>* F, const cplx<T>* Fc, const cplx<T>* Fs, const cplx<T>* Fa,
                        const cplx<T>* Fw, cplx<T>* Yw, int nrhs, const IOSpec& io) {
    SolveArgs<T> a;
    a.F = F + (size_t)fs * g.Ny * NSLOT * BLK;
    a.Fs = Fs ? Fs + (size_t)fs * (ch.P - 1) * 2 * BLK : nullptr;
    a.Fa = Fa ? Fa + (size_t)fs * g.Ny * BLK : nullptr;
    a.Fw = Fw ? Fw + (size_t)fs * (ch.P - 1) * 4 * BLK : nullptr;
    a.q = ch.q;
    a.G = ch.G;
    a.Fc = Fc ? Fc + (size_t)fs * g.Ny * 2 * 8 * WP : nullptr;
    a.tcol = t.tcol + s * 8;
    a.Yw = Yw;
    a.cy = t.cy;
    a.by = t.by;
    a.io = io;
    if (!Fc) a.io.targets_only = 0;     // without compact rows phase C reads every column
    if (!a.io.trA || !a.io.trB || a.io.q_t < 0) {   // the gather always dereferences them
        a.io.trA = a.io.trB = a.io.src;
        a.io.q_t = -1;
        a.io.coef = 0.0;
    }
    a.Ny = g.Ny;
    a.W = g.strips[s].W;
    a.m = ch.m;
    a.P = ch.P;
    a.nrhs = nrhs;
    return a;
}

}  // namespace

template <typename T>
hipError_t launch_strip_solve(const DevTables& t, const Geom& g, const Chunks& ch, int s, int fs,
                              const cplx<T>* F, const cplx<T>* Fc, const cplx<T>* Fs, const cplx<T>* Fa,
                              const cplx<T>* Fw, cplx<T>* Yw, int nrhs, const IOSpec& io, hipStream_t st,
                              KTimer* kt) {
    const SolveArgs<T> a = solve_args<T>(t, g, ch, s, fs, F, Fc, Fs, Fa, Fw, Yw, nrhs, io);
    // complex64 reads the operand-order copies: phase A on MFMA (more than 4 right-hand
    // sides) and the separator chains of the two-level solve
    if (std::is_same<T, float>::value &&
        ((nrhs > 4 && !Fa) || (ch.P > 2 && ch.G >= 2 && Fs && !Fw)))
        return hipErrorInvalidValue;
    const bool targets = a.io.targets_only != 0;
    if (nrhs <= 4) return run<T, 4>(a, targets, st, kt);
    return run<T, 16>(a, targets, st, kt);
}

namespace {
SolveArgs<float> job_args(const StripJob& j) {
    return solve_args<float>(*j.t, *j.g, *j.ch, j.s, j.fs, static_cast<const float2*>(j.F),
                             static_cast<const float2*>(j.Fc), static_cast<const float2*>(j.Fs),
                             static_cast<const float2*>(j.Fa), static_cast<const float2*>(j.Fw),
                             static_cast<float2*>(j.Yw), j.nrhs, j.io);
}
// Right-hand sides of a batch of strips, in the workspace rows: the strip's source columns of
// the field, and (inputs pu, pd given) what the sweeps feed the strip at its interfaces: the
// transmission sources of both sweeps and the residual at the right interface.  One wave per
// row, lanes along x.  Grid (rows / 4, right-hand sides, strips).
template <typename T>
__global__ void __launch_bounds__(NT) k_batch_rhs(BatchRhs<T> a) {
    using V = cplx<T>;
    const int q = threadIdx.x & (WP - 1), l = 4 * blockIdx.x + (threadIdx.x >> 6), r = blockIdx.y, k = blockIdx.z;
    if (l >= a.Ny) return;
    const StripIO x = a.io[k];
    double2 v = cmk<double2>(0.0, 0.0);
    if (a.f && q >= x.s_lo && q < x.s_hi) v = a.f[((size_t)r * a.Ny + l) * a.Nx + x.a + q];
    if (a.pu || a.pd) {
        // inputs of row l: operand order (red_pos), entries t | psi, g | psi, g per chunk
        const int c = l / a.M, lr = l - c * a.M, n = r & 15;
        const size_t base = (((size_t)(a.s0 + k) * a.G + (r >> 4)) * a.P + c) * 3 * a.Mp * 16;
        if (a.pu && x.eL >= 0 && (q == x.eL - 1 || q == x.eL)) v = cadd(v, ccast<double2>(a.pu[base + red_pos<T>(lr, n)]));
        if (a.pd && x.eR >= 0 && q >= x.eR - 1 && q <= x.eR + 1) {
            if (q < x.eR + 1)
                v = cadd(v, ccast<double2>(a.pd[base + red_pos<T>((q - x.eR + 2) * a.Mp + lr, n)]));
            if (q > x.eR - 1) v = cadd(v, ccast<double2>(a.pd[base + red_pos<T>(lr, n)]));
        }
    }
    a.Yw[(((size_t)k * gridDim.y + r) * a.Ny + l) * WP + q] = ccast<V>(v);
}

template <typename T, int R>
hipError_t run_batch(const BatchArgs<T>& b, int ns, bool targets, hipStream_t st, KTimer* kt) {
    const SolveArgs<T>& a = b.a;
    const unsigned RG = (a.nrhs + R - 1) / R, z = ns;
    const unsigned nr1 = a.nrhs, RG16 = (a.nrhs + 15) / 16;
    if (kt) kt->begin(K_PHASE_A, st, ns);
    if constexpr (R == 4) {
        const dim3 g(a.P, 1, z);
        if (a.nrhs == 1) hipLaunchKernelGGL((k_phase_a_few_b<T, 1>), g, dim3(NT), 0, st, b);
        else if (a.nrhs == 2) hipLaunchKernelGGL((k_phase_a_few_b<T, 2>), g, dim3(NT), 0, st, b);
        else hipLaunchKernelGGL((k_phase_a_few_b<T, 4>), g, dim3(NT), 0, st, b);
    } else if constexpr (std::is_same<T, float>::value) {
        hipLaunchKernelGGL(k_phase_a_mfma_b<2>, dim3(a.P, RG, z), dim3(NT), 0, st, b);
    } else {
        hipLaunchKernelGGL(k_phase_a_mfma64_b, dim3(a.P, RG, z), dim3(NT), 0, st, b);
    }
    if (kt) kt->end(K_PHASE_A, st);
    if (a.P > 1) {
        if (kt) kt->begin(K_PHASE_B, st, ns);
        constexpr int DS = Depth<T>::D;
        if (a.P > 2 && a.G >= 2 && a.Fs) {
            if constexpr (std::is_same<T, float>::value) {
                const dim3 gp(a.P - 1, RG16, z);
                const unsigned nl = (a.nrhs + SepLocalRB<T>::RB - 1) / SepLocalRB<T>::RB;
                hipLaunchKernelGGL(k_sep_par_mfma_b<0>, gp, dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_fwd_local_b<T, DS, false>), dim3(nl, a.G, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_fwd_top_b<T, DS>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL(k_sep_par_mfma_b<1>, gp, dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_fix_bwd_local_b<T, DS, false>), dim3(nl, a.G, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_bwd_top_b<T, DS>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
                if (!targets) hipLaunchKernelGGL(k_sep_par_mfma_b<2>, gp, dim3(NT), 0, st, b);
            } else {
                hipLaunchKernelGGL((k_sep_fwd_local_b<T, DS>), dim3(nr1, a.G, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_fwd_top_b<T, DS>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_fix_bwd_local_b<T, DS>), dim3(nr1, a.G, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_bwd_top_b<T, DS>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
                hipLaunchKernelGGL((k_sep_bwd_fix_b<T, DS>), dim3(nr1, a.G - 1, z), dim3(NT), 0, st, b);
            }
        } else {
            hipLaunchKernelGGL((k_phase_b0_b<T, R>), dim3(a.P - 1, RG, z), dim3(NT), 0, st, b);
            if (a.P > 2) {
                if (a.P - 1 <= ZMAX) hipLaunchKernelGGL((k_phase_b_b<T, DS, true>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
                else hipLaunchKernelGGL((k_phase_b_b<T, DS, false>), dim3(nr1, 1, z), dim3(NT), 0, st, b);
            }
        }
        if (kt) kt->end(K_PHASE_B, st);
    }
    if (kt) kt->begin(K_PHASE_C, st, ns);
    if constexpr (std::is_same<T, float>::value) {
        // tiles and rows spread as in the launches of one strip; a batch fills the chip with fewer
        const int tiles = ((a.m - 1) * 8 + 15) / 16, per = a.P * (int)RG16 * ns;
        const int tz = std::min(8, std::max(1, (tiles + 7) / 8));
        const int cz = std::max(1, std::min(std::min(8, a.m), (1024 + per - 1) / per));
        if (targets) hipLaunchKernelGGL(k_phase_c_targets_mfma_b, dim3(a.P, RG16, z * tz), dim3(NT), 0, st, b, tz);
        else hipLaunchKernelGGL(k_phase_c_mfma_b, dim3(a.P, RG16, z * cz), dim3(NT), 0, st, b, cz);
    } else {
        if (targets)
            hipLaunchKernelGGL((k_phase_c_targets_b<T>), dim3((a.Ny + CT_ROWS - 1) / CT_ROWS, (a.nrhs + 31) / 32, z),
                               dim3(NT), 0, st, b);
        else hipLaunchKernelGGL((k_phase_c_b<T, R>), dim3(a.Ny, RG, z), dim3(NT), 0, st, b);
    }
    if (kt) kt->end(K_PHASE_C, st);
    return hipGetLastError();
}

// rows of the full-column phase C per workgroup: about four workgroups per CU
int phase_c_groups(const SolveArgs<float>& a) {
    const int per = a.P * ((a.nrhs + 15) / 16);
    return std::max(1, std::min(std::min(8, a.m), (1024 + per - 1) / per));
}
int targets_groups(const SolveArgs<float>& a) {
    const int tiles = ((a.m - 1) * 8 + 15) / 16;
    return std::min(8, std::max(1, (tiles + 7) / 8));
}
}  // namespace

template <typename T>
hipError_t launch_strip_batch(const DevTables& t, const Geom& g, const Chunks& ch, const BatchRhs<T>& rhs,
                              int ns, const cplx<T>* F, const cplx<T>* Fc,
                              const cplx<T>* Fs, const cplx<T>* Fa, const cplx<T>* Fw, const IOSpec& io,
                              hipStream_t st, KTimer* kt) {
    const int nrhs = rhs.nrhs;
    if (std::is_same<T, float>::value && ((nrhs > 4 && !Fa) || (ch.P > 2 && ch.G >= 2 && Fs && !Fw)))
        return hipErrorInvalidValue;
    if (kt) kt->begin(K_OTHER, st, 1);
    hipLaunchKernelGGL((k_batch_rhs<T>), dim3((g.Ny + 3) / 4, nrhs, ns), dim3(NT), 0, st, rhs);
    if (kt) kt->end(K_OTHER, st);
    BatchArgs<T> b;
    b.a = solve_args<T>(t, g, ch, rhs.s0, 0, F, Fc, Fs, Fa, Fw, rhs.Yw, nrhs, io);
    b.a.io.pre = 1;
    b.io = rhs.io;
    b.tcol = t.tcol + 8 * rhs.s0;
    b.F_st = (long)g.Ny * NSLOT * BLK;
    b.Fc_st = (long)g.Ny * 2 * 8 * WP;
    b.Fs_st = (long)(ch.P - 1) * 2 * BLK;
    b.Fa_st = Fa ? (long)g.Ny * BLK : 0;
    b.Fw_st = Fw ? (long)(ch.P - 1) * 4 * BLK : 0;
    if (!Fs) b.Fs_st = 0;
    b.Yw_st = (long)nrhs * g.Ny * WP;
    b.tr_st = (long)nrhs * g.Ny;
    const bool targets = b.a.io.targets_only != 0;
    if (nrhs <= 4) return run_batch<T, 4>(b, ns, targets, st, kt);
    return run_batch<T, 16>(b, ns, targets, st, kt);
}
template hipError_t launch_strip_batch<float>(const DevTables&, const Geom&, const Chunks&, const BatchRhs<float>&,
                                              int, const float2*, const float2*, const float2*,
                                              const float2*, const float2*, const IOSpec&, hipStream_t, KTimer*);
template hipError_t launch_strip_batch<double>(const DevTables&, const Geom&, const Chunks&, const BatchRhs<double>&,
                                               int, const double2*, const double2*, const double2*,
                                               const double2*, const double2*, const IOSpec&, hipStream_t, KTimer*);

bool strip_jobs_fusable(const StripJob* jobs, int n) {
    if (n < 2 || n > MULTI_MAX) return false;
    int targets = -1;
    for (int k = 0; k < n; ++k) {
        const StripJob& j = jobs[k];
        if (!j.f32 || j.g->dim != 2 || j.nrhs <= 4) return false;
        if (!(j.ch->P > 2 && j.ch->G >= 2 && j.Fs)) return false;        // two-level separators
        if (!j.Fa || !j.Fw) return false;                                // operand-order copies
        const int tk = (j.io.targets_only && j.Fc) ? 1 : 0;
        if (targets >= 0 && tk != targets) return false;
        targets = tk;
    }
    return true;
}

hipError_t launch_strip_solve_multi(const StripJob* jobs, int n, hipStream_t st, KTimer* kt) {
    if (!strip_jobs_fusable(jobs, n)) return hipErrorInvalidValue;
    MultiArgs<float> m{};
    m.n = n;
    for (int k = 0; k < n; ++k) m.a[k] = job_args(jobs[k]);
    const bool targets = m.a[0].io.targets_only != 0;
    // x blocks per problem, and per-problem y / z extents (the launch takes the largest)
    auto shape = [&](auto xper, auto yper, auto zper, dim3& grid) {
        m.xs[0] = 0;
        int my = 1, mz = 1;
        for (int k = 0; k < n; ++k) {
            m.xs[k + 1] = m.xs[k] + xper(m.a[k]);
            m.ny[k] = yper(m.a[k]);
            m.nz[k] = zper(m.a[k]);
            my = std::max(my, m.ny[k]);
            mz = std::max(mz, m.nz[k]);
        }
        grid = dim3(m.xs[n], my, mz);
    };
    auto P = [](const SolveArgs<float>& a) { return a.P; };
    auto RG = [](const SolveArgs<float>& a) { return (a.nrhs + 15) / 16; };
    auto NR = [](const SolveArgs<float>& a) { return a.nrhs; };     // one right-hand side per block
    auto NL = [](const SolveArgs<float>& a) {                       // the local chains' blocks
        return (a.nrhs + SepLocalRB<float>::RB - 1) / SepLocalRB<float>::RB;
    };
    auto G = [](const SolveArgs<float>& a) { return a.G; };
    auto NS = [](const SolveArgs<float>& a) { return a.P - 1; };      // separators
    auto one = [](const SolveArgs<float>&) { return 1; };
    constexpr int DS = Depth<float>::D;
    dim3 grid;
    if (kt) kt->begin(K_PHASE_A, st);
    shape(P, RG, one, grid);
    hipLaunchKernelGGL(k_phase_a_mfma_multi<2>, grid, dim3(NT), 0, st, m);
    if (kt) kt->end(K_PHASE_A, st);
    if (kt) kt->begin(K_PHASE_B, st);
    shape(NS, RG, one, grid);
    hipLaunchKernelGGL(k_sep_par_mfma_multi<0>, grid, dim3(NT), 0, st, m);
    shape(NL, G, one, grid);
    hipLaunchKernelGGL((k_sep_fwd_local_multi<float, DS, false>), grid, dim3(NT), 0, st, m);
    shape(NR, one, one, grid);
    hipLaunchKernelGGL((k_sep_fwd_top_multi<float, DS>), grid, dim3(NT), 0, st, m);
    shape(NS, RG, one, grid);
    hipLaunchKernelGGL(k_sep_par_mfma_multi<1>, grid, dim3(NT), 0, st, m);
    shape(NL, G, one, grid);
    hipLaunchKernelGGL((k_sep_fix_bwd_local_multi<float, DS, false>), grid, dim3(NT), 0, st, m);
    shape(NR, one, one, grid);
    hipLaunchKernelGGL((k_sep_bwd_top_multi<float, DS>), grid, dim3(NT), 0, st, m);
    if (!targets) {
        shape(NS, RG, one, grid);
        hipLaunchKernelGGL(k_sep_par_mfma_multi<2>, grid, dim3(NT), 0, st, m);
    }
    if (kt) kt->end(K_PHASE_B, st);
    if (kt) kt->begin(K_PHASE_C, st);
    if (targets) {
        shape(P, RG, targets_groups, grid);
        hipLaunchKernelGGL(k_phase_c_targets_mfma_multi, grid, dim3(NT), 0, st, m);
    } else {
        shape(P, RG, phase_c_groups, grid);
        hipLaunchKernelGGL(k_phase_c_mfma_multi, grid, dim3(NT), 0, st, m);
    }
    if (kt) kt->end(K_PHASE_C, st);
    return hipGetLastError();
}

template hipError_t launch_strip_solve<float>(const DevTables&, const Geom&, const Chunks&, int, int,
                                              const float2*, const float2*, const float2*, const float2*,
                                              const float2*, float2*, int, const IOSpec&, hipStream_t, KTimer*);
template hipError_t launch_strip_solve<double>(const DevTables&, const Geom&, const Chunks&, int, int,
                                               const double2*, const double2*, const double2*,
                                               const double2*, const double2*, double2*, int, const IOSpec&,
                                               hipStream_t, KTimer*);

namespace {
// Fa[slot][row]: out[((w * 8 + i) * 64 + 16 q4 + n) * 2 + h] = G[16 w + n][8 i + 4 h + q4] of
// F[slot][row][0] (column-major: element (r, c) at c * WP + r)
__global__ void __launch_bounds__(NT) k_swizzle_a(const float2* __restrict__ F, float2* __restrict__ Fa) {
    const size_t blk = blockIdx.x;                       // slot * Ny + row
    const float2* src = F + blk * NSLOT * BLK;
    float2* dst = Fa + blk * BLK;
    for (int o = threadIdx.x; o < BLK; o += NT) {
        const int h = o & 1, lane = (o >> 1) & 63, i = (o >> 7) & 7, w = o >> 10;
        const int q4 = lane >> 4, n = lane & 15;
        dst[o] = src[(8 * i + 4 * h + q4) * WP + 16 * w + n];
    }
}
// Fw[slot][c][kind]: out[((w * 8 + j) * 64 + i) * 2 + h] = M[i][16 w + 2 j + h] for M = the
// slot-1 / slot-2 block at separator row c m + m - 1 (kind 0 / 1) or the propagator Fs[c][0 / 1]
// (kind 2 / 3)
__global__ void __launch_bounds__(NT) k_swizzle_w(const float2* __restrict__ F, const float2* __restrict__ Fs,
                                                  float2* __restrict__ Fw, int Ny, int m, int ns) {
    const int kind = blockIdx.x & 3, c = (blockIdx.x >> 2) % ns, slot = (blockIdx.x >> 2) / ns;
    const int row = c * m + m - 1;
    const float2* src = kind < 2 ? F + (((size_t)slot * Ny + row) * NSLOT + 1 + kind) * BLK
                                 : Fs + (((size_t)slot * ns + c) * 2 + (kind - 2)) * BLK;
    float2* dst = Fw + (size_t)blockIdx.x * BLK;
    for (int o = threadIdx.x; o < BLK; o += NT) {
        const int h = o & 1, i = (o >> 1) & 63, j = (o >> 7) & 7, w = o >> 10;
        dst[o] = src[(16 * w + 2 * j + h) * WP + i];
    }
}
}  // namespace

hipError_t launch_swizzle_factors(const float2* F, const float2* Fs, float2* Fa, float2* Fw,
                                  const Geom& g, const Chunks& ch, int nfac, hipStream_t st) {
    if (nfac <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_swizzle_a, dim3((unsigned)(nfac * g.Ny)), dim3(NT), 0, st, F, Fa);
    const int ns = ch.P - 1;
    if (Fw && Fs && ns > 0)
        hipLaunchKernelGGL(k_swizzle_w, dim3((unsigned)(nfac * ns * 4)), dim3(NT), 0, st, F, Fs, Fw, g.Ny,
                           ch.m, ns);
    return hipGetLastError();
}

}  // namespace helm
