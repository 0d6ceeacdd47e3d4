// potrf.hip -- Cholesky factor and inverse of one 128 x 128 diagonal block.
//
// The blocked right-looking Cholesky (factor of Z, which is symmetric
// positive definite for distinct Euclidean points, Section 3.2) needs at each
// panel step the factor L11 of the diagonal block and, to turn the panel's
// triangular solve into an MFMA contraction, the explicit inverse L11^{-1}.
// One workgroup of eight waves does both, in eight steps of 16 columns, with
// every 16 x 16 block in the registers of one wave:
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
// A pivot that is not positive (or not finite) marks status[0] with the
// global pivot index + 1 (its column turns into NaNs; the kernel still finishes);
// the host then refactors with a diagonal shift.
#include "internal.hpp"

namespace mag {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NB = 128;
constexpr int SB = 16;            // block edge
constexpr int NBLK = NB / SB;     // blocks per row = waves
constexpr int NTP = 64 * NBLK;    // threads

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

// FUSED: the block is first updated by the 128 columns of the sub-panel left of it
// (its rows of that sub-panel's L21), A -= L21 L21^T; Us holds the row blocks of 64
// of those columns at a time.
template <bool FUSED>
__device__ __forceinline__ void potrf128_body(float *__restrict__ A, int64_t ld, int64_t k0, int64_t n,
                                              float *__restrict__ Linv, int *__restrict__ status, v4f (*Us)[NBLK][64])
{
    __shared__ v4f Lx[NBLK][64];   // the blocks L_Kj of a step, row layout
    __shared__ float Yd[SB * SB];  // the inverse of its diagonal block, Yd[k * SB + c]
    __shared__ int bad;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // the row block of a wave: waves w and w + 4 share a SIMD, and a long row block goes
    // with a short one
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = wave < NBLK / 2 ? wave : 3 * NBLK / 2 - 1 - wave;
    const int g = lane >> 4, i = lane & 15;
    float *Ab = A + k0 * ld + k0;

    if (k0 >= n) {
        // a block of the identity padding (uniform): its diagonal entries alone
        for (int e = tid; e < NB * NB; e += NTP) {
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
        return;
    }

    // Q[m] at step j: block (I, j + m) of A while j + m <= I; from step I on, of the
    // eliminated identity.  All loads first; the diagonal block from its lower
    // triangle, mirrored.
    v4f Q[NBLK], dg;
    {
        const unsigned off = 4 * g * (unsigned)ld + SB * I + i;
#pragma unroll
        for (int K = 0; K < NBLK; ++K)
#pragma unroll
            for (int r = 0; r < 4; ++r) Q[K][r] = (Ab + (SB * K + r) * ld)[off];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = 4 * g + r, lo = k < i ? k : i, hi = k < i ? i : k;
            dg[r] = Ab[(SB * I + lo) * ld + SB * I + hi];
        }
#pragma unroll
        for (int K = 0; K < NBLK; ++K)
#pragma unroll
            for (int r = 0; r < 4; ++r) Q[K][r] = K < I ? Q[K][r] : (K == I ? dg[r] : 0.0f);
    }
    if (tid == 0) bad = 0;
    if (FUSED) {
        const unsigned off = 4 * g * (unsigned)ld + SB * I + i;
        v4f x[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) x[h][c][r] = (Ab - (NB - 64 * h - SB * c - r) * ld)[off];
        v4f acc[NBLK];
#pragma unroll
        for (int K = 0; K < NBLK; ++K)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[K][r] = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h > 0) __syncthreads();
#pragma unroll
            for (int c = 0; c < 4; ++c) Us[c][I][lane] = x[h][c];
            __syncthreads();
#pragma unroll
            for (int K = 0; K < NBLK; ++K) {
                if (K > I) continue;  // uniform per wave
                v4f y[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) y[c] = Us[c][K][lane];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[K] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[c][r], x[h][c][r], acc[K], 0, 0, 0);
            }
        }
#pragma unroll
        for (int K = 0; K < NBLK; ++K) {
            Q[K] -= acc[K];
            if (K == I) dg = Q[K];
        }
    }
    __syncthreads();

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
#pragma unroll
            for (int r = 0; r < 4; ++r) X[r] = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) X = __builtin_amdgcn_mfma_f32_16x16x4f32(y[r], Q[0][r], X, 0, 0, 0);
        }
        if (I > j) Lx[I][lane] = X;
        __syncthreads();
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
    if (tid == 0 && bad != 0) atomicCAS(&status[kStBreakdown], 0, bad);
}

__global__ void __launch_bounds__(NTP)
k_potrf128(float *__restrict__ A, int64_t ld, int64_t k0, int64_t n, float *__restrict__ Linv,
           int *__restrict__ status)
{
    potrf128_body<false>(A, ld, k0, n, Linv, status, nullptr);
}

// Batched: one workgroup per problem whose padded size exceeds k0.
__global__ void __launch_bounds__(NTP)
k_potrf128_b(const BProb *__restrict__ P, BWork w, int64_t k0)
{
    const BProb &q = P[w.plist[blockIdx.x]];
    if (!q.active || k0 >= q.npad) return;
    potrf128_body<false>(q.A, q.npad, k0, q.n, q.dinv + (k0 / NB) * NB * NB, q.ints, nullptr);
}

// ---- sub-panel update and the next diagonal block in one launch ------------------
// C (i, j) -= P P^T for one 128 x 128 tile (rows i0.., columns j0..) by the 128
// columns at P, on eight waves of 32 x 64 each; K staged through LDS in
// double-buffered chunks of 16 by direct loads (see gemm_mfma.hip).
typedef float v16f __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(1))) void *gptr;
typedef __attribute__((address_space(3))) void *lptr;
constexpr int KC = 16;

__device__ __forceinline__ void update_tile(float *__restrict__ C, int64_t ldc, const float *__restrict__ P,
                                            int64_t ldp, int64_t i0, int64_t j0, float *lds)
{
    float (*Ps)[KC][NB] = reinterpret_cast<float (*)[KC][NB]>(lds);
    float (*Qs)[KC][NB] = reinterpret_cast<float (*)[KC][NB]>(lds + 2 * KC * NB);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = (wave & 3) * 32, wj = (wave >> 2) * 64;
    const int l32 = lane & 31, hi = lane >> 5;
    v16f acc[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[jb][r] = 0.0f;
    // wave w stages k-rows 2 w and 2 w + 1 of P and of Q
    const int64_t off = (int64_t)(threadIdx.x >> 5) * ldp + 4 * (threadIdx.x & 31);
    const float *pg = P + off + i0, *qg = P + off + j0;
    auto stage_in = [&](int b) {
        __builtin_amdgcn_global_load_lds((gptr)pg, (lptr)&Ps[b][2 * wave][0], 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gptr)qg, (lptr)&Qs[b][2 * wave][0], 16, 0, 0);
        pg += KC * ldp;
        qg += KC * ldp;
    };
    stage_in(0);
    __syncthreads();
    constexpr int nst = NB / KC;
    for (int st = 0; st < nst; ++st) {
        const int buf = st & 1;
        if (st + 1 < nst) stage_in(buf ^ 1);
#pragma unroll
        for (int kp = 0; kp < KC / 2; ++kp) {
            const int p = 2 * kp + hi;
            const float pv = Ps[buf][p][wi + l32];
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(Qs[buf][p][wj + l32], pv, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(Qs[buf][p][wj + 32 + l32], pv, acc[1], 0, 0, 0);
        }
        __syncthreads();  // waits for the direct loads of the next stage too
    }
    float cv[2][16];
    float *c0 = C + (j0 + wj) * ldc + i0 + wi + l32;
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) cv[jb][r] = c0[(jb * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * ldc];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            c0[(jb * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * ldc] = cv[jb][r] - acc[jb][r];
}

// The columns kk + 128 .. kk + 128 (1 + ncol) of the trailing rows (from kk + 128) updated
// by the sub-panel at kk, lower 128-tiles only; workgroup 0 takes the first tile,
// the next diagonal block, and goes on to factor it while the others update
// theirs: its 12 us of pivots run beside the update instead of after it, and it
// needs no load of its own.
constexpr int kUpdateLds = 4 * KC * NB * 4;  // bytes: two buffers of P and Q stages
static_assert(kUpdateLds >= (int)(4 * NBLK * 64 * sizeof(v4f)), "the row blocks of the fused update fit the stages");

__global__ void __launch_bounds__(NTP, 4)
k_update_potrf(float *__restrict__ A, int64_t ld, int64_t kk, int64_t n, int ncol, float *__restrict__ Linv,
               int *__restrict__ status)
{
    __shared__ v4f lds[kUpdateLds / sizeof(v4f)];
    if (blockIdx.x == 0) {
        potrf128_body<true>(A, ld, kk + NB, n, Linv, status, reinterpret_cast<v4f (*)[NBLK][64]>(lds));
        return;
    }
    const int64_t T = (ld - kk - NB) / NB;  // tile rows
    int64_t u = blockIdx.x, tj = 0;
    while (u >= T - tj) {  // column tj has T - tj tiles
        u -= T - tj;
        ++tj;
    }
    update_tile(A + (kk + NB) * ld + kk + NB, ld, A + kk * ld + kk + NB, ld, (tj + u) * NB, tj * NB,
                reinterpret_cast<float *>(lds));
}

}  // namespace

void launch_potrf128_b(hipStream_t s, const BProb *P, const BWork &w, int64_t k0)
{
    if (w.na > 0) hipLaunchKernelGGL(k_potrf128_b, dim3(w.na), dim3(NTP), 0, s, P, w, k0);
}

void launch_potrf128(hipStream_t s, float *A, int64_t ld, int64_t k0, int64_t n, float *Linv, int *status)
{
    hipLaunchKernelGGL(k_potrf128, dim3(1), dim3(NTP), 0, s, A, ld, k0, n, Linv, status);
}

void launch_update_potrf(hipStream_t s, float *A, int64_t ld, int64_t kk, int64_t n, int ncol, float *Linv, int *status)
{
    const int64_t T = (ld - kk - NB) / NB;
    if (T <= 0 || ncol <= 0) return;
    const int64_t nc = ncol < T ? ncol : T;
    const int64_t tiles = nc * T - nc * (nc - 1) / 2;
    hipLaunchKernelGGL(k_update_potrf, dim3((unsigned)tiles), dim3(NTP), 0, s, A, ld, kk, n, (int)nc, Linv, status);
}

}  // namespace mag
