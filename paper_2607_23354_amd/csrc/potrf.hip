// potrf.hip -- Cholesky factor and inverse of the 128 x 128 diagonal blocks, and the
// panels of the single FP32 factor around them.
//
// The blocked right-looking Cholesky (factor of Z, which is symmetric
// positive definite for distinct Euclidean points, Section 3.2) needs at each
// panel step the factor L11 of the diagonal block and its explicit inverse (for the
// substitutions, and for the batched panel solve).  Eight waves do both (factor128),
// in eight steps of 16 columns, with every 16 x 16 block in the registers of one wave:
//   * row layout: lane 16 g + i, register r of a block hold entry (i, 4 g + r), so a
//     block is four registers, the accumulator of v_mfma_f32_16x16x4 (of the
//     transposed block) and, register by register, either of its operands;
//   * wave I owns row block I of A (until step I) and then row block I of the
//     identity, which the same column operations turn into L^{-T};
//   * step j: wave j has factored and inverted its diagonal block (eliminate16);
//     every other wave multiplies its block of column j by that inverse, X =
//     L_Ij of a row block of A, (L^{-T})_Ij of one of the identity.  Then wave j + 1
//     brings its diagonal block up to date from its own registers and goes
//     straight on to factor it, while the others take the update R_K -= X L_Kj^T of
//     their blocks right of column j.
//
// What bounds it: the chain of 128 pivots, and in it the instructions (about 60 per
// four columns; a lone wave issues one about every seven cycles), not their
// arithmetic.  14.5 us per block (4 us of it the load and the first instruction
// fetches), against 26.6 us for 32-column sweeps on 32 x 32 matrix instructions with
// the block in LDS, whose chain waits for two 64-cycle instructions per pivot pair.
// Products are summed from zero and then subtracted: with the minuend as the matrix
// instruction's accumulator the diagonal's backward error was twice as large, and
// biased (rms 2.1e-7 against 1.0e-7; 1.4e-7 with the 32-column sweeps; m = 8, n = 5000).
//
// k_panel factors a panel of up to 512 columns in one launch, a workgroup per 128 rows:
// the top block's workgroups factor the diagonal blocks one after another, and
// every 16-column step of theirs goes to all workgroups below through a small exchange
// in memory the moment it is done, where it is applied to their rows at once.  The
// chain is then four diagonal blocks and the hand-offs between them, instead of
// those and seven launches that each wait for the last workgroup of the one before
// (a panel of 512 columns: 88 us instead of 112 us at n = 3001 and 8192, 105 us instead of
// 160 us at n = 32768).  Clock stamps at n = 3072: the diagonal blocks
// take 13 us each; before the last three of them stand the steps of their row blocks, 1.9 us
// for 16 columns with one later tile and 2.9 us with three, which never wait for data.
// Every workgroup keeps its rows of the sub-panel and the sums for
// the later ones in registers, so each entry is loaded, updated by a subtraction
// per 128 columns' sum, and stored once; the backward error went down by up to 40 %
// (2.0e-7 instead of 3.4e-7, m = 8, n = 5000).
//
// A pivot that is not positive (or not finite) marks status[0] with the
// global pivot index + 1 (its column turns into NaNs; the kernel still finishes);
// the host then refactors with a diagonal shift.
#include "internal.hpp"

#include <algorithm>

namespace mag {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NB = 128;
constexpr int SB = 16;            // block edge
constexpr int NBLK = NB / SB;     // blocks per row = waves
constexpr int NTP = 64 * NBLK;    // threads
constexpr int kPanelSteps = 32;   // 16-column steps of the widest panel (512 columns)

__device__ inline float bcast(float v, int src_lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src_lane));
}

// Lane 16 k + i of the result: v[k] of lane 16 T + i (the four registers of one
// 16-lane group spread over the four groups: the operand of one MFMA).
template <int T>
__device__ __forceinline__ float gather4(const float (&v)[4])
{
    const auto u = [](float x) { return (unsigned)__float_as_int(x); };
    // (a, b) -> rows (a0, b0, a2, b2) and (a1, b1, a3, b3)
    const auto p = __builtin_amdgcn_permlane16_swap(u(v[0]), u(v[1]), false, false);
    const auto q = __builtin_amdgcn_permlane16_swap(u(v[2]), u(v[3]), false, false);
    const auto w = __builtin_amdgcn_permlane32_swap(p[T & 1], q[T & 1], false, false);
    return __int_as_float((int)w[T >> 1]);
}

// Columns 4 T .. 4 T + 3 of the pivot block P (held by lane group T) and of X.
// TRACK: pivot k into lane k of piv.
template <int T, bool TRACK>
__device__ __forceinline__ void eliminate4(v4f &P, v4f &X, int lane, int &piv)
{
    float l[4], x[4], s[4][4], inv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) l[c] = P[c];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float p = bcast(l[c], 20 * T + c);
        if (TRACK) piv = (lane == 4 * T + c) ? __float_as_int(p) : piv;
        inv[c] = __builtin_amdgcn_rsqf(p);
        l[c] *= inv[c];
#pragma unroll
        for (int k = c + 1; k < 4; ++k) {
            s[k][c] = bcast(l[c], 20 * T + k);  // L(4 T + k, 4 T + c)
            l[k] = fmaf(-l[c], s[k][c], l[k]);
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        x[c] = X[c];
#pragma unroll
        for (int k = 0; k < c; ++k) x[c] = fmaf(-x[k], s[c][k], x[c]);
        x[c] *= inv[c];
    }
    const bool mine = (lane >> 4) == T;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        P[c] = mine ? l[c] : P[c];
        X[c] = mine ? x[c] : X[c];
    }
    if (T < 3) {
        // the columns right of these (rows of the transposed blocks): -= L (L or X)^T
        const float lg = gather4<T>(l), xg = gather4<T>(x);
        const float la = (lane & 15) >= 4 * T + 4 ? -lg : 0.0f;
        P = __builtin_amdgcn_mfma_f32_16x16x4f32(la, lg, P, 0, 0, 0);
        X = __builtin_amdgcn_mfma_f32_16x16x4f32(la, xg, X, 0, 0, 0);
    }
}

// Factor the pivot block P (row layout, symmetric) into L and apply the same
// column operations to the identity: X(i, k) = L^{-1}(k, i).
template <bool TRACK>
__device__ __forceinline__ void eliminate16(v4f &P, v4f &X, int lane, int &piv)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) X[r] = ((lane & 15) == 4 * (lane >> 4) + r) ? 1.0f : 0.0f;
    eliminate4<0, TRACK>(P, X, lane, piv);
    eliminate4<1, TRACK>(P, X, lane, piv);
    eliminate4<2, TRACK>(P, X, lane, piv);
    eliminate4<3, TRACK>(P, X, lane, piv);
}

// The first pivot of the 16-column block P that is not positive and finite: the
// elimination taken again with its pivots kept (only after a breakdown).
__device__ __noinline__ int first_bad_pivot(v4f P, int lane)
{
    v4f X;
    int piv = __float_as_int(1.0f);
    eliminate16<true>(P, X, lane, piv);
    const float p = __int_as_float(piv);
    return __ffsll((long long)__ballot(!(p > 0.0f && p < INFINITY))) - 1;
}

// Q[m] = Q[m + 1] - X L_K^T, K = j + 1 + m, for M0 <= m < M1 (L: the blocks L_K in
// LDS), summed from zero, one matrix instruction of every block in turn (the four of a block
// wait for one another)
template <int M0, int M1>
__device__ __forceinline__ void block_updates(v4f (&Q)[NBLK], const v4f &x, const v4f (*L)[64], int j, int lane)
{
    v4f y[M1 - M0], acc[M1 - M0];
#pragma unroll
    for (int m = M0; m < M1; ++m) {
        y[m - M0] = L[(j + 1 + m) & (NBLK - 1)][lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m - M0][r] = 0.0f;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < M1 - M0; ++m)
            acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[m][r], x[r], acc[m], 0, 0, 0);
#pragma unroll
    for (int m = M0; m < M1; ++m) Q[m] = Q[m + 1] - acc[m - M0];
}

// Below the diagonal block the products run on the BF16 matrix cores, each FP32 operand
// as the exact sum of three BF16 components h, m, l (8 bits of the significand each)
// and all products but m l, l m and l l, below FP32's own rounding: per 16 x 16 x 16 block
// three instructions of 16 cycles (two products each) in place of four of 32.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v8u __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

// A block's rows in components: words 0, 1: columns 4 g .. 4 g + 3 of l; 2, 3: of h; 4, 5: of
// m.  Words 0-3 and 2-5 are the two K = 32 operands.
struct Split {
    v2u c[3];
};

__device__ __forceinline__ Split split_rows(const v4f &x)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    const auto pack = [](const v2f &v) { return __builtin_bit_cast(unsigned, __builtin_convertvector(v, v2b)); };
    const auto rest = [](const v2f &v, unsigned u) {
        v2f d;
        d[0] = v[0] - __int_as_float((int)(u << 16));
        d[1] = v[1] - __int_as_float((int)(u & 0xffff0000u));
        return d;
    };
    Split s;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        v2f v;
        v[0] = x[2 * p];
        v[1] = x[2 * p + 1];
        s.c[1][p] = pack(v);
        v = rest(v, s.c[1][p]);
        s.c[2][p] = pack(v);
        s.c[0][p] = pack(rest(v, s.c[2][p]));
    }
    return s;
}

struct SplitX {  // the operand every block of a row is multiplied by: (h, h), (m, m), (h, l)
    v4u hh, mm, hl;
};

__device__ __forceinline__ v4u join(const v2u &a, const v2u &b)
{
    return __builtin_shufflevector(a, b, 0, 1, 2, 3);
}

__device__ __forceinline__ SplitX widen(const Split &s)
{
    SplitX x;
    x.hh = join(s.c[1], s.c[1]);
    x.mm = join(s.c[2], s.c[2]);
    x.hl = join(s.c[1], s.c[0]);
    return x;
}

__device__ __forceinline__ v4f mfma_b(const v4u &y, const v4u &x, const v4f &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, y), __builtin_bit_cast(v8b, x), c, 0, 0, 0);
}

// A block of a step in LDS, lane by lane.
struct SplitBlock {
    v2u l[64];
    v4u hm[64];
    __device__ __forceinline__ void put(int lane, const Split &s)
    {
        l[lane] = s.c[0];
        hm[lane] = join(s.c[1], s.c[2]);
    }
};

// acc[m] += X L_K^T, K = (K0 + m) mod 8, for four blocks of L in LDS.
__device__ __forceinline__ void four_blocks(v4f *acc, const SplitX &x, const SplitBlock *L, int K0, int lane)
{
    v4u hm[4], lh[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const SplitBlock &b = L[(K0 + m) & (NBLK - 1)];
        const v2u l = b.l[lane];
        const v4u h = b.hm[lane];
        const v8u w = __builtin_shufflevector(join(l, l), h, 0, 1, 4, 5, 6, 7, -1, -1);
        lh[m] = __builtin_shufflevector(w, w, 0, 1, 2, 3);
        hm[m] = __builtin_shufflevector(w, w, 2, 3, 4, 5);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = mfma_b(lh[m], x.hl, acc[m]);
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = mfma_b(hm[m], x.mm, acc[m]);
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = mfma_b(hm[m], x.hh, acc[m]);
}

// ---- hand-off of a panel's top block between workgroups ---------------------------
// A block passes in its components, a plane of 512 bytes each (an inverse in FP32: two),
// by relaxed atomics of 8 bytes past the L2s; kUnset in a word marks what is not
// there yet.
constexpr uint32_t kUnset = 0x7fa5f00du;  // a signalling NaN, in BF16 too (arithmetic yields quiet ones)
constexpr int kBlockWords = 192;          // 8-byte words

// Block of 16-row block row R >= g at 16-column step g of the top block of a panel of
// 16 `steps` columns (a step's blocks stand together).
__device__ __forceinline__ uint64_t *xblock(uint64_t *xch, int steps, int g, int R)
{
    return xch + (g * steps - g * (g + 1) / 2 + R) * kBlockWords;
}

// Bytes of the exchange of a panel of `cols` columns.
__host__ __device__ constexpr int64_t exchange_bytes(int64_t cols)
{
    const int64_t R = cols / SB;
    return R * (R + 1) / 2 * kBlockWords * 8;
}
static_assert(exchange_bytes(256) % 4096 == 0 && exchange_bytes(512) % 4096 == 0, "whole workgroups of k_unset");

__device__ __forceinline__ v2u ld_plane(const uint64_t *p, int c, int lane)
{
    return __builtin_bit_cast(v2u, __hip_atomic_load(p + 64 * c + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ __forceinline__ void st_plane(uint64_t *p, int c, int lane, v2u v)
{
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (v[r] == kUnset) v[r] = 0x7fc07fc0u;
    __hip_atomic_store(p + 64 * c + lane, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_split(uint64_t *p, int lane, const Split &s)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) st_plane(p, c, lane, s.c[c]);
}

// Factor of the 128 x 128 block at Ab (global pivot index k0) whose row block I is in
// the wave's registers: Q[m], block (I, m) for m <= I and zero beyond, and dg = Q[I].
// PUB: the blocks L_Kj and the inverses of the 16 x 16 diagonal blocks go to the exchange,
// steps g0 .. g0 + 7.
template <bool PUB>
__device__ __forceinline__ void factor128(v4f (&Q)[NBLK], const v4f &dg, float *__restrict__ Ab, int64_t ld, int64_t k0,
                                          float *__restrict__ Linv, int *__restrict__ status, v4f (*Lx)[64], float *Yd,
                                          int &bad, int I, int lane, uint64_t *xch, int steps, int g0)
{
    const int g = lane >> 4, i = lane & 15;
    v4f P = dg, P0, X;
    // wave j: factor its diagonal block P and put the inverse in LDS
    auto diagonal = [&]() {
        int none = 0;
        P0 = P;
        __builtin_amdgcn_s_setprio(3);
        eliminate16<false>(P, X, lane, none);
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) Yd[(4 * g + r) * SB + i] = X[r];
    };
    if (I == 0) diagonal();
    __syncthreads();
    // one copy of the step's code (unrolled over j the kernel spends its time on
    // instruction fetches)
#pragma unroll 1
    for (int j = 0; j < NBLK; ++j) {
        if (I != j) {
            const v4f y = *reinterpret_cast<const v4f *>(Yd + i * SB + 4 * g);
            if (PUB && I == ((j + 2) & (NBLK - 1))) {
                uint64_t *p = xblock(xch, steps, g0 + j, g0 + j);
                st_plane(p, 0, lane, __builtin_bit_cast(v4u, y).xy);
                st_plane(p, 1, lane, __builtin_bit_cast(v4u, y).zw);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) X[r] = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) X = __builtin_amdgcn_mfma_f32_16x16x4f32(y[r], Q[0][r], X, 0, 0, 0);
        }
        if (I > j) {
            Lx[I][lane] = X;
            if (PUB && I != j + 1) st_split(xblock(xch, steps, g0 + j, g0 + I), lane, split_rows(X));
        }
        __syncthreads();
        // for wave j + 1, which goes on with the pivots
        if (PUB && j + 1 < NBLK && I == ((j + 3) & (NBLK - 1)))
            st_split(xblock(xch, steps, g0 + j, g0 + j + 1), lane, split_rows(Lx[j + 1][lane]));
        // out: L and L^T of this block column, rows of the inverse
        if (I == j) {
            float d = 1.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 4 * g + r;
                d = (k == i) ? P[r] : d;
                if (k <= i) {
                    Ab[(SB * j + k) * ld + SB * j + i] = P[r];
                    Ab[(SB * j + i) * ld + SB * j + k] = P[r];
                }
            }
            // a pivot that is not positive and finite leaves a NaN on the diagonal
            if (bad == 0 && __ballot(!(d > 0.0f && d < INFINITY)) != 0) {
                const int c = first_bad_pivot(P0, lane);
                if (lane == 0) bad = (int)(k0 + SB * j + c + 1);
            }
        }
        if (I > j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) Ab[(SB * j + 4 * g + r) * ld + SB * I + i] = X[r];
            *reinterpret_cast<v4f *>(Ab + (SB * I + i) * ld + SB * j + 4 * g) = X;
        } else {
            *reinterpret_cast<v4f *>(Linv + (SB * I + i) * NB + SB * j + 4 * g) = X;
            if (I != j) {
                v4f z;
#pragma unroll
                for (int r = 0; r < 4; ++r) z[r] = 0.0f;
                *reinterpret_cast<v4f *>(Linv + (SB * j + i) * NB + SB * I + 4 * g) = z;
            }
        }
        if (I == j + 1) {
            // summed from zero (rounded below the diagonal's own magnitude)
            v4f acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[r], X[r], acc, 0, 0, 0);
            P = Q[1] - acc;
            diagonal();
#pragma unroll
            for (int m = 0; m < NBLK; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) Q[m][r] = 0.0f;
        } else {
            // row blocks of A stop at their diagonal
            const int last = I <= j ? NBLK - 1 : I;
            if (j + 1 <= last) block_updates<0, 4>(Q, X, Lx, j, lane);
            if (j + 5 <= last) block_updates<4, 7>(Q, X, Lx, j, lane);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && bad != 0) atomicCAS(&status[kStBreakdown], 0, bad);
}

// A diagonal block of the identity padding: its diagonal entries alone.
__device__ __forceinline__ void factor_padding(float *__restrict__ Ab, int64_t ld, float *__restrict__ Linv)
{
    for (int e = threadIdx.x; e < NB * NB; e += NTP) {
        const int c = e >> 7, r = e & (NB - 1);
        float l = 0.0f, v = 0.0f;
        if (r == c) {
            const float d = Ab[(int64_t)c * ld + r];
            v = __builtin_amdgcn_rsqf(d);
            l = d * v;
        }
        Ab[(int64_t)c * ld + r] = l;
        Linv[e] = v;
    }
}

// The row block of a wave: waves w and w + 4 share a SIMD, and a long row block goes
// with a short one.
__device__ __forceinline__ int row_block()
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return wave < NBLK / 2 ? wave : 3 * NBLK / 2 - 1 - wave;
}

// Row block I of the 128 x 128 tile at At.
__device__ __forceinline__ void load_rows(v4f (&Q)[NBLK], const float *__restrict__ At, int64_t ld, int I, int lane)
{
    const unsigned off = 4 * (lane >> 4) * (unsigned)ld + SB * I + (lane & 15);
#pragma unroll
    for (int K = 0; K < NBLK; ++K)
#pragma unroll
        for (int r = 0; r < 4; ++r) Q[K][r] = (At + (SB * K + r) * ld)[off];
}

// Diagonal block I of the 128 x 128 block at Ab, from its lower triangle.
__device__ __forceinline__ v4f load_diagonal(const float *__restrict__ Ab, int64_t ld, int I, int lane)
{
    const int g = lane >> 4, i = lane & 15;
    v4f d;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int k = 4 * g + r, lo = k < i ? k : i, hi = k < i ? i : k;
        d[r] = Ab[(SB * I + lo) * ld + SB * I + hi];
    }
    return d;
}

// Batched: one workgroup per problem whose padded size exceeds k0.
__global__ void __launch_bounds__(NTP)
k_potrf128_b(const BProb *__restrict__ P, BWork w, int64_t k0)
{
    const BProb &q = P[w.plist[blockIdx.x]];
    if (!q.active || k0 >= q.npad) return;
    __shared__ v4f Lx[NBLK][64];   // the blocks L_Kj of a step, row layout
    __shared__ float Yd[SB * SB];  // the inverse of its diagonal block, Yd[k * SB + c]
    __shared__ int bad;
    const int lane = threadIdx.x & 63, I = row_block();
    float *Ab = q.A + k0 * q.npad + k0, *Linv = q.dinv + (k0 / NB) * NB * NB;
    if (k0 >= q.n) {
        factor_padding(Ab, q.npad, Linv);
        return;
    }
    // Q[m] at step j: block (I, j + m) of A while j + m <= I; from step I on, of the
    // eliminated identity
    v4f Q[NBLK];
    load_rows(Q, Ab, q.npad, I, lane);
    const v4f dg = load_diagonal(Ab, q.npad, I, lane);
#pragma unroll
    for (int K = 0; K < NBLK; ++K)
#pragma unroll
        for (int r = 0; r < 4; ++r) Q[K][r] = K < I ? Q[K][r] : (K == I ? dg[r] : 0.0f);
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    factor128<false>(Q, dg, Ab, q.npad, k0, Linv, q.ints, Lx, Yd, bad, I, lane, nullptr, 0, 0);
}

// ---- one panel in one launch -------------------------------------------------------
struct PanelArgs {
    float *A;         // the matrix
    int64_t ld, k, n;
    int nsub;         // 128-column sub-panels
    float *dinv;      // inverse of the panel's first diagonal block, the others behind it
    int *status, *ticket;
    uint64_t *xch, *xnext;  // this launch's exchange and the next one's
    int unset;              // 16-byte words that the next one takes
    long spin_limit;
};

constexpr int MT = kPanelSteps / NBLK;  // most tiles (128-column sub-panels) of a panel

struct PanelShared {
    SplitBlock B[2][MT][NBLK];  // a step's blocks: of the sub-panel's own rows, of the later tiles'
    SplitBlock O[2][NBLK];      // and of the workgroup's own rows
    v4f Y[2][64];               // the inverse of the step's diagonal block
    float Yd[SB * SB];
    int bad, ib;
};

// Sub-panel S of the rows below its diagonal block: tile Q (updated by the earlier
// sub-panels) into L, acc[t - 1] += L L_t^T for the panel's later tiles t.
template <int S>
__device__ __forceinline__ void below(const PanelArgs &a, PanelShared &sh, v4f (&Q)[NBLK], v4f (&acc)[MT - 1][NBLK],
                                      Split (&pf)[MT], int ib, int I, int lane, long &limit)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, i = lane & 15;
    const bool top = ib < a.nsub;
    const int lim = top ? ib : a.nsub;  // tiles whose blocks come from other workgroups
    // block `wave` of tile S + q at step g: the wave's share of a step's blocks
    auto need = [&](int g, int q) {
        return q == 0 ? wave >= (g & (NBLK - 1)) : (g >> 3) + q < lim;
    };
    auto fetch = [&](int g) {
#pragma unroll
        for (int q = 0; q < MT; ++q)
            if (need(g, q)) {
                const uint64_t *p = xblock(a.xch, NBLK * a.nsub, g, NBLK * ((g >> 3) + q) + wave);
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (c < 2 || q > 0 || wave != (g & (NBLK - 1))) pf[q].c[c] = ld_plane(p, c, lane);
            }
    };
    auto missing = [&](int g) {
        bool u = false;
#pragma unroll
        for (int q = 0; q < MT; ++q)
            if (need(g, q)) {
                // (the two words of an atomic come together)
                u = u || pf[q].c[0][0] == kUnset || pf[q].c[1][0] == kUnset;
                if (q > 0 || wave != (g & (NBLK - 1))) u = u || pf[q].c[2][0] == kUnset;
            }
        return __ballot(u) != 0;
    };
    // until the step's blocks are there: the top block's workgroups poll the data, the
    // others one entry of each block, now and then
    auto wait = [&](int g) {
        long spins = 0;
        while (missing(g)) {
            if (++spins > limit) {
                if (lane == 0) a.status[kStSpinTimeout] = 1;
                limit = 0;
                return;
            }
            if (!top) {
                const int s = g >> 3;
                bool mine = false;
                if (lane == 0) mine = need(g, 0);
#pragma unroll
                for (int q = 1; q < MT; ++q)
                    if (lane == q) mine = need(g, q);
                const uint64_t *e = xblock(a.xch, NBLK * a.nsub, g, NBLK * (s + (lane & (MT - 1))) + wave) + 127;
                for (;;) {
                    uint64_t v = 0;
                    if (mine) v = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (__ballot(mine && (uint32_t)(v >> 32) == kUnset) == 0 || ++spins > limit) break;
                    __builtin_amdgcn_s_sleep(8);
                }
            }
            fetch(g);
        }
    };
    float *low = a.A + (a.k + NB * S + 4 * g4) * a.ld + a.k + NB * ib + SB * I + i;
    float *up = a.A + (a.k + NB * ib + SB * I + i) * a.ld + a.k + NB * S + 4 * g4;
    if (S == 0) fetch(0);
#pragma unroll 1
    for (int j = 0; j < NBLK + (top ? 1 : 0); ++j) {
        const int g = NBLK * S + j, cur = j & 1;
        SplitX x;
        if (j < NBLK) {
            wait(g);
#pragma unroll
            for (int q = 0; q < MT - S; ++q)
                if (need(g, q)) {
                    if (q == 0 && wave == j)
                        sh.Y[cur][lane] = __builtin_bit_cast(v4f, join(pf[0].c[0], pf[0].c[1]));
                    else
                        sh.B[cur][q][wave].put(lane, pf[q]);
                }
            if (g + 1 < NBLK * lim) fetch(g + 1);
            __syncthreads();
            v4f X;
            {
                const v4f y = sh.Y[cur][lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) X[r] = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) X = __builtin_amdgcn_mfma_f32_16x16x4f32(y[r], Q[0][r], X, 0, 0, 0);
            }
            const Split xs = split_rows(X);
            if (top) {
                st_split(xblock(a.xch, NBLK * a.nsub, g, NBLK * ib + I), lane, xs);
                sh.O[cur][I].put(lane, xs);
            }
            x = widen(xs);
#pragma unroll
            for (int r = 0; r < 4; ++r) low[r * a.ld] = X[r];
            *reinterpret_cast<v4f *>(up) = X;
            low += SB * a.ld;
            up += SB;
            // the blocks right of this one in the sub-panel
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (j < NBLK - 1 - 4 * h) {
                    v4f u[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r) u[m][r] = 0.0f;
                    four_blocks(u, x, sh.B[cur][0], j + 1 + 4 * h, lane);
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        if (4 * h + m < NBLK - 1) Q[4 * h + m] = Q[4 * h + m + 1] - u[m];
                }
        } else {
            __syncthreads();
        }
        // the later tiles; the workgroup's own (its diagonal block's) one step behind, when
        // every wave's block is in LDS
#pragma unroll
        for (int t = S + 1; t < MT; ++t) {
            const bool own = top && t == ib;
            if ((j < NBLK && t < lim) || (own && j > 0)) {
                const SplitBlock *L = sh.B[cur][t - S];
                if (own) {
                    L = sh.O[cur ^ 1];
                    Split xs;
                    xs.c[0] = L[I].l[lane];
                    const v4u hm = L[I].hm[lane];
                    xs.c[1] = hm.xy;
                    xs.c[2] = hm.zw;
                    x = widen(xs);
                }
                __builtin_amdgcn_sched_barrier(0);  // keeps the tiles' operands from being live together
#pragma unroll
                for (int h = 0; h < 2; ++h) four_blocks(acc[t - 1] + 4 * h, x, L, 4 * h, lane);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// The workgroup's part in sub-panel S: its tile below the diagonal block, or (true) that
// block's rows into Q and dg for the factorisation.
template <int S>
__device__ __forceinline__ bool panel_step(const PanelArgs &a, PanelShared &sh, v4f (&Q)[NBLK], v4f &dg,
                                           v4f (&acc)[MT - 1][NBLK], Split (&pf)[MT], int ib, int I, int lane, long &limit)
{
    const int64_t k0 = a.k + NB * S;
    float *At = a.A + k0 * a.ld + a.k + NB * ib;  // tile (ib, S)
    if (k0 >= a.n) {
        // the identity padding (uniform)
        if (ib == S) return true;
        float *Up = a.A + (a.k + NB * ib) * a.ld + k0;
        for (int e = threadIdx.x; e < NB * NB; e += NTP) {
            At[(int64_t)(e >> 7) * a.ld + (e & (NB - 1))] = 0.0f;
            Up[(int64_t)(e >> 7) * a.ld + (e & (NB - 1))] = 0.0f;
        }
        return false;
    }
    load_rows(Q, At, a.ld, I, lane);
    if (ib == S) dg = load_diagonal(At, a.ld, I, lane);
    if (S > 0) {
#pragma unroll
        for (int K = 0; K < NBLK; ++K) {
            const v4f u = acc[S > 0 ? S - 1 : 0][K];
            Q[K] -= u;
            if (K == I) dg -= u;
        }
    }
    if (ib == S) return true;
    below<S>(a, sh, Q, acc, pf, ib, I, lane, limit);
    return false;
}

// blk, count: this workgroup's index among the panel's
__device__ __forceinline__ void panel_body(const PanelArgs &a, int blk, int count)
{
    __shared__ PanelShared sh;
    const int lane = threadIdx.x & 63, I = row_block();
    // the panel's rows of (most likely) this workgroup on their way to the L2 meanwhile, a
    // line per thread and tile
    float warm = 0.0f;
    for (int t = 0; t < a.nsub; ++t)
        warm += a.A[(a.k + NB * t + (threadIdx.x >> 2)) * a.ld + a.k + NB * (int64_t)blk + 32 * (threadIdx.x & 3)];
    if (threadIdx.x == 0) {
        // tickets: a workgroup waits only for earlier ones, which are running
        sh.ib = atomicAdd(a.ticket, 1);
        if (sh.ib == count - 1) *a.ticket = 0;
        sh.bad = 0;
    }
    __syncthreads();
    const int ib = __builtin_amdgcn_readfirstlane(sh.ib);
    asm volatile("" ::"v"(warm));
    v4f Q[NBLK], dg, acc[MT - 1][NBLK];
    Split pf[MT];
#pragma unroll
    for (int r = 0; r < 4; ++r) dg[r] = 0.0f;
#pragma unroll
    for (int t = 0; t < MT - 1; ++t)
#pragma unroll
        for (int K = 0; K < NBLK; ++K)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t][K][r] = 0.0f;
#pragma unroll
    for (int q = 0; q < MT; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) pf[q].c[c][0] = pf[q].c[c][1] = 0;
    long limit = a.spin_limit;
    if (!panel_step<0>(a, sh, Q, dg, acc, pf, ib, I, lane, limit) &&
        !panel_step<1>(a, sh, Q, dg, acc, pf, ib, I, lane, limit)) {
        if (a.nsub == 2) return;
        if (!panel_step<2>(a, sh, Q, dg, acc, pf, ib, I, lane, limit) &&
            !panel_step<3>(a, sh, Q, dg, acc, pf, ib, I, lane, limit))
            return;
    }
    // block ib of the diagonal
    {
        const int64_t k0 = a.k + NB * ib;
        float *Ab = a.A + k0 * a.ld + k0, *Linv = a.dinv + ib * NB * NB;
        if (k0 >= a.n) {
            factor_padding(Ab, a.ld, Linv);
        } else {
#pragma unroll
            for (int K = 0; K < NBLK; ++K)
#pragma unroll
                for (int r = 0; r < 4; ++r) Q[K][r] = K < I ? Q[K][r] : (K == I ? dg[r] : 0.0f);
            factor128<true>(Q, dg, Ab, a.ld, k0, Linv, a.status, reinterpret_cast<v4f (*)[64]>(sh.B), sh.Yd, sh.bad, I, lane, a.xch,
                            NBLK * a.nsub, NBLK * ib);
        }
    }
    if (ib == 0) {
        // done early: unset the next launch's exchange
        v4u u;
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] = kUnset;
        for (int e = threadIdx.x; e < a.unset; e += NTP) reinterpret_cast<v4u *>(a.xnext)[e] = u;
    }
}

__global__ void __launch_bounds__(NTP)
k_panel(PanelArgs a)
{
    panel_body(a, blockIdx.x, gridDim.x);
}

// The exchange buffer: the ticket, then two banks that the panels take in turn, the second
// behind the widest panel's (a matrix of one panel has no second one).
constexpr int64_t kHeaderBytes = 256;  // the banks' planes on whole lines (off them a panel takes 1.5 us more)
constexpr int64_t kBankBytes = exchange_bytes(NB * MT);

__device__ __host__ inline PanelArgs panel_args(float *A, int64_t ld, int64_t k, int64_t nb, int64_t n, float *dinv,
                                                int *status, void *work, int index, long spin_limit)
{
    char *w = (char *)work;
    const int64_t left = ld - k - nb;
    PanelArgs a;
    a.A = A;
    a.ld = ld;
    a.k = k;
    a.n = n;
    a.nsub = (int)(nb / NB);
    a.dinv = dinv + (k / NB) * NB * NB;
    a.status = status;
    a.ticket = (int *)w;
    a.xch = (uint64_t *)(w + kHeaderBytes + (index & 1) * kBankBytes);
    a.xnext = (uint64_t *)(w + kHeaderBytes + (~index & 1) * kBankBytes);
    a.unset = (int)(exchange_bytes(left < nb ? left : nb) / 16);
    a.spin_limit = spin_limit;
    return a;
}

// Batched: the panel at k of every active problem, each with its own exchange and tickets;
// a problem's workgroups are consecutive, so its first ones, which the others wait
// for, are dispatched first.
__global__ void __launch_bounds__(NTP)
k_panel_b(const BProb *__restrict__ P, BWork w, int64_t k, long spin_limit)
{
    const int i = bfind(w.pref, w.na, blockIdx.x);
    const BProb &q = P[w.plist[i]];
    if (!q.active) return;
    const int64_t left = q.npad - k;
    panel_body(panel_args(q.A, q.npad, k, left < NB * MT ? left : NB * MT, q.n, q.dinv, q.ints, q.panel,
                          (int)(k / (NB * MT)), spin_limit),
               (int)(blockIdx.x - w.pref[i]), (int)(left / NB));
}

__device__ __forceinline__ void unset(v4u *x, int64_t i)
{
    v4u u;
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = kUnset;
    x[i] = u;
}

// Ticket zero and the first bank unset, 4096 bytes of it per workgroup.
__device__ __forceinline__ void panel_begin(void *work)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *(int *)work = 0;
    unset((v4u *)((char *)work + kHeaderBytes), blockIdx.x * 256 + threadIdx.x);
}

__global__ void __launch_bounds__(256)
k_panel_begin(void *__restrict__ work)
{
    panel_begin(work);
}

__global__ void __launch_bounds__(256)
k_panel_begin_b(const BProb *__restrict__ P)
{
    const BProb &q = P[blockIdx.y];
    if (q.active && 4096 * (int64_t)blockIdx.x < exchange_bytes(q.npad < NB * MT ? q.npad : NB * MT)) panel_begin(q.panel);
}

}  // namespace

void launch_potrf128_b(hipStream_t s, const BProb *P, const BWork &w, int64_t k0)
{
    if (w.na > 0) hipLaunchKernelGGL(k_potrf128_b, dim3(w.na), dim3(NTP), 0, s, P, w, k0);
}

size_t panel_work_bytes() { return kHeaderBytes + 2 * kBankBytes; }

size_t panel_b_work_bytes(int64_t npad)
{
    const int64_t w = NB * MT;
    return kHeaderBytes + exchange_bytes(std::min(npad, w)) + exchange_bytes(std::min(std::max<int64_t>(npad - w, 0), w));
}

void launch_panel_begin(hipStream_t s, void *work, int64_t nb)
{
    hipLaunchKernelGGL(k_panel_begin, dim3((unsigned)(exchange_bytes(nb) / 4096)), dim3(256), 0, s, work);
}

void launch_panel(hipStream_t s, float *A, int64_t ld, int64_t k, int64_t nb, int64_t n, float *dinv, int *status,
                  void *work, int index, long spin_limit)
{
    hipLaunchKernelGGL(k_panel, dim3((unsigned)((ld - k) / NB)), dim3(NTP), 0, s,
                       panel_args(A, ld, k, nb, n, dinv, status, work, index, spin_limit));
}

int64_t panel_b_units(int64_t npad, int64_t k) { return k < npad ? (npad - k) / NB : 0; }

void launch_panel_begin_b(hipStream_t s, const BProb *P, int B, int64_t maxpad)
{
    const int64_t bytes = exchange_bytes(std::min<int64_t>(maxpad, NB * MT));
    hipLaunchKernelGGL(k_panel_begin_b, dim3((unsigned)(bytes / 4096), (unsigned)B), dim3(256), 0, s, P);
}

void launch_panel_b(hipStream_t s, const BProb *P, const BWork &w, int64_t k, long spin_limit)
{
    if (w.total > 0) hipLaunchKernelGGL(k_panel_b, dim3((unsigned)w.total), dim3(NTP), 0, s, P, w, k, spin_limit);
}

}  // namespace mag
