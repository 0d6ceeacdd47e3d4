// gemm_split.hip -- the FP32 factor's trailing update on the BF16 matrix cores.
//
//   C (N x N, lower 128-tiles)  <-  C - P P^T,   P an N x K panel of L in FP32
//
// An FP32 number is exactly the sum of three BF16 numbers (8 significand bits
// each, 24 in all): x = h + m + l with h = bf16(x), m = bf16(x - h),
// l = x - h - m.  A product of two split numbers is the sum of nine BF16
// products, every one exact in FP32; six of them
//   h h' + h m' + m h' + m m' + h l' + l h'
// leave out only m l', l m' and l l', which are below 2^-24 |x x'| each (the
// rounding of one FP32 product).  Sums are FP32 accumulators: the five small
// products on one of their own, added to that of h h' at the end, so the sum is
// rounded at most four times per 16 columns where the FP32 matrix
// instruction (v_mfma_f32_32x32x2) rounds it 16 times.  Backward error of the
// factor, ||L L^T - Z||_F / ||Z||_F against 64 bits, with the FP32 instruction and
// with the split: 3.5e-7 and 2.2e-7 (Gaussian cloud, n = 3001, half the cutoff
// scale), 5.4e-7 and 2.9e-7 (n = 8192, a quarter of it), 1.42e-7 and 1.26e-7 (n =
// 8192 at it), 9.8e-8 both where the rounding of Z itself dominates.
//
// What bounds it: the matrix cores at the clock the power limit leaves (1.6 GHz of
// 2.4 under this load; registers-only BF16 MFMA sustains 1.83 PFLOP/s, a sixth
// of which is 304 TF/s of update).  At rows = 20480, K = 1024: 195 TF/s (2.22 ms)
// against 128 TF/s of the FP32 instruction, itself at 81 % of its peak.  128 x 128
// tiles throughout, whose two accumulators (128 registers) leave room for two
// workgroups on a CU: on 256 x 128 tiles the small products have to be added to the
// sum every 16 columns (192 TF/s; a third of the vector issue) or one workgroup is
// alone on its CU (172 TF/s), and on 128 x 128 ones that addition cost 53 us
// instead of 45 at 1024 rows, 59 instead of 50 at 2048 and 442 instead of 403 at 8192.
// A third stage buffer, 32 columns per stage and other orders of the products change
// nothing or lose.
#include "internal.hpp"

namespace mag {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(1))) void *gptr;  // global operand of a direct LDS load
typedef __attribute__((address_space(3))) void *lptr;        // its LDS destination

constexpr int NS = 3;     // BF16 components of an FP32 entry
constexpr int KC = 16;    // columns of P per LDS stage (one MFMA k-step)
constexpr int TM = 128;   // tile edge
constexpr int NT = 256;   // threads per workgroup
constexpr int kXcds = 8;
constexpr int kSup = 512; // edge of a super-tile (k_syrk_split)

// ---- the split image ---------------------------------------------------------
// Unit: 16 bytes, one component of 8 consecutive columns of one row.  Plane
// q = NS (column group) + component holds `stride` rows, so 64 rows of a plane
// are 1 KB in a row: one direct-to-LDS instruction of a wave, and one half of an
// MFMA operand read from LDS without bank conflicts.

__device__ __forceinline__ void split8(const float (&x)[8], v8bf (&c)[NS])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const __bf16 h = (__bf16)x[j];
        const float r = x[j] - (float)h;
        const __bf16 m = (__bf16)r;
        c[0][j] = h;
        c[1][j] = m;
        c[2][j] = (__bf16)(r - (float)m);
    }
}

// row r of column group g of the columns at P (column-major) into img
__device__ __forceinline__ void split_unit(const float *__restrict__ P, int64_t ldp, int64_t r, int64_t g,
                                           v8bf *__restrict__ img, int64_t stride)
{
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = P[(8 * g + j) * ldp + r];
    v8bf c[NS];
    split8(x, c);
#pragma unroll
    for (int s = 0; s < NS; ++s) img[(g * NS + s) * stride + r] = c[s];
}

// rows [0, rows) of the columns at P into img
__global__ void __launch_bounds__(NT)
k_split(const float *__restrict__ P, int64_t ldp, int64_t rows, v8bf *__restrict__ img, int64_t stride)
{
    const int64_t r = blockIdx.x * (int64_t)NT + threadIdx.x;
    if (r < rows) split_unit(P, ldp, r, blockIdx.y, img, stride);
}

// ---- the update ---------------------------------------------------------------
// Workgroup tile 128 x 128, four waves in 2 x 2, each 64 x 64 as four 32 x 32
// MFMA blocks (A from the column rows Q, B from the rows P: a lane holds one
// row of C, its registers the columns).
constexpr int IB = TM / 64;           // 32-row blocks of a wave
constexpr int PU = 2 * NS * TM;       // 16-byte units of a P stage
constexpr int ST = 2 * PU;            // of a stage (P and Q)
constexpr int CH = ST / 64;           // 64-unit chunks of a stage
static_assert(CH % 4 == 0, "chunks divide over the waves");

__device__ __forceinline__ void split_tile_body(float *__restrict__ C, int64_t ldc, const v8bf *__restrict__ img,
                                                int64_t stride, int64_t i0, int64_t j0, int64_t rows, int64_t K)
{
    __shared__ v8bf lds[2 * ST];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = (wave & 1) * (TM / 2), wj = (wave >> 1) * 64;
    const int l32 = lane & 31, hi = lane >> 5;

    // the five small products (roundings 2^-8 below those of the sum) on accumulators of
    // their own, added to the sum at the end
    v16f acc[2][IB], low[2][IB];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int ib = 0; ib < IB; ++ib)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[jb][ib][r] = low[jb][ib][r] = 0.0f;

    // chunk u of this wave: 64 rows of one plane of P or Q
    const char *src[CH / 4];
#pragma unroll
    for (int u = 0; u < CH / 4; ++u) {
        const int c = wave + 4 * u;
        const bool isP = c < PU / 64;
        const int cc = isP ? c : c - PU / 64;
        const int64_t row = (isP ? i0 : j0) + 64 * (cc % IB);
        src[u] = reinterpret_cast<const char *>(img + (int64_t)(cc / IB) * stride + row) + 16 * lane;
    }
    const int64_t step = (int64_t)2 * NS * stride * 16;
    auto stage_in = [&](int b) {
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) {
            __builtin_amdgcn_global_load_lds((gptr)src[u], (lptr)&lds[b * ST + 64 * (wave + 4 * u)], 16, 0, 0);
            src[u] += step;
        }
    };
    stage_in(0);
    __syncthreads();
    const int nst = (int)(K / KC);
    for (int st = 0; st < nst; ++st) {
        const int buf = st & 1;
        if (st + 1 < nst) stage_in(buf ^ 1);  // that buffer was last read before the previous barrier
        const v8bf *Ps = lds + buf * ST, *Qs = Ps + PU;
        __builtin_amdgcn_s_setprio(1);  // over a co-resident workgroup's epilogue (2 %)
        v8bf q[2][NS];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) q[jb][s] = Qs[(hi * NS + s) * TM + wj + 32 * jb + l32];
        constexpr int qa[5] = {2, 0, 1, 1, 0}, pa[5] = {0, 2, 1, 0, 1};
#pragma unroll
        for (int ib = 0; ib < IB; ++ib) {
            v8bf p[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) p[s] = Ps[(hi * NS + s) * TM + wi + 32 * ib + l32];
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb)
                    low[jb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[jb][qa[t]], p[pa[t]], low[jb][ib], 0, 0, 0);
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
                acc[jb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[jb][0], p[0], acc[jb][ib], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();  // waits for the direct loads of the next stage too
    }

#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int ib = 0; ib < IB; ++ib)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[jb][ib][r] += low[jb][ib][r];

    // C -= acc, 16 columns of the wave's rows at a time through LDS (free after the
    // last barrier), so C moves in float4 accesses; column stride 72 keeps both
    // halves of the wave on distinct banks
    float *Tw = reinterpret_cast<float *>(lds) + wave * (16 * 72);
    const int64_t ri = i0 + wi;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int jb = q >> 1, rq = q & 1;
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) {
            const int r = 8 * rq + rr;
            const int c16 = 8 * (rr >> 2) + 4 * hi + (r & 3);
#pragma unroll
            for (int ib = 0; ib < 2; ++ib) Tw[c16 * 72 + 32 * ib + l32] = acc[jb][ib][r];
        }
#pragma unroll
        for (int rd = 0; rd < 4; ++rd) {
            const int c16 = 4 * rd + (lane >> 4);
            const float4 a = *reinterpret_cast<const float4 *>(&Tw[c16 * 72 + 4 * (lane & 15)]);
            float4 *cp = reinterpret_cast<float4 *>(C + (j0 + wj + 32 * jb + 16 * rq + c16) * ldc + ri +
                                                    4 * (lane & 15));
            float4 c = *cp;
            c.x -= a.x;
            c.y -= a.y;
            c.z -= a.z;
            c.w -= a.w;
            *cp = c;
        }
    }
}

__device__ inline void tri_index(int64_t idx, int64_t &ti, int64_t &tj)
{
    int64_t r = (int64_t)((sqrt(8.0 * (double)idx + 1.0) - 1.0) * 0.5);
    while (r * (r + 1) / 2 > idx) --r;
    while ((r + 1) * (r + 2) / 2 <= idx) ++r;
    ti = r;
    tj = idx - r * (r + 1) / 2;
}

// Workgroups are dealt to the 8 XCDs round-robin by id; consecutive ids of one
// XCD walk the tiles of one 512 x 512 super-tile of the lower triangle, so the
// workgroups that share operand rows run on one L2 at about the same time (edges
// of 1024 and 2048 measured 1 % and 3 % slower at 20480 rows).
__global__ void __launch_bounds__(NT, 2)
k_syrk_split(float *__restrict__ C, int64_t ldc, const v8bf *__restrict__ img, int64_t stride, int64_t rows,
             int64_t K)
{
    constexpr int SE = kSup / TM;
    const int64_t b = blockIdx.x;
    const int64_t xcd = b % kXcds, slot = b / kXcds;
    const int64_t sidx = (slot / (SE * SE)) * kXcds + xcd, within = slot % (SE * SE);
    int64_t si, sj;
    tri_index(sidx, si, sj);
    const int64_t i0 = si * kSup + (within / SE) * TM;
    const int64_t j0 = sj * kSup + (within % SE) * TM;
    if (i0 >= rows || j0 > i0) return;  // padding slot (uniform per workgroup)
    split_tile_body(C, ldc, img, stride, i0, j0, rows, K);
}

// The first tilesN columns of tiles of C alone (lower tiles): the strip of a panel pair.  The
// tiles of a row share its operand, so they go to one XCD.
__global__ void __launch_bounds__(NT, 2)
k_strip_split(float *__restrict__ C, int64_t ldc, const v8bf *__restrict__ img, int64_t stride, int64_t rows, int64_t K,
              int tilesN)
{
    const int64_t b = blockIdx.x;
    const int64_t xcd = b % kXcds, slot = b / kXcds;
    const int64_t i0 = ((slot / tilesN) * kXcds + xcd) * TM, j0 = (slot % tilesN) * TM;
    if (i0 >= rows || j0 > i0) return;
    split_tile_body(C, ldc, img, stride, i0, j0, rows, K);
}

// Batched: the trailing rows of every active problem after the K columns at kk.
// Units of the split: (rows / 256) x (K / 8); of the update, tiles by rows of
// tiles.
__global__ void __launch_bounds__(NT)
k_split_b(const BProb *__restrict__ Pr, BWork w, int64_t kk, int64_t K)
{
    const int i = bfind(w.pref, w.na, blockIdx.x);
    const BProb &q = Pr[w.plist[i]];
    if (!q.active) return;
    const int64_t u = blockIdx.x - w.pref[i], rows = q.npad - kk - K, rb = rows / NT;
    split_unit(q.A + kk * q.npad + kk + K, q.npad, (u % rb) * NT + threadIdx.x, u / rb, (v8bf *)q.img, rows);
}

__global__ void __launch_bounds__(NT, 2)
k_syrk_split_b(const BProb *__restrict__ Pr, BWork w, int64_t kk, int64_t K)
{
    const int i = bfind(w.pref, w.na, blockIdx.x);
    const BProb &q = Pr[w.plist[i]];
    if (!q.active) return;
    const int64_t u = blockIdx.x - w.pref[i], rows = q.npad - kk - K;
    int64_t ti, tj;
    tri_index(u, ti, tj);
    split_tile_body(q.A + (kk + K) * q.npad + kk + K, q.npad, (const v8bf *)q.img, rows, ti * TM, tj * TM, rows, K);
}

}  // namespace

size_t split_image_bytes(int64_t rows, int64_t K) { return (size_t)round_up(rows, 256) * (size_t)(K / 8) * NS * 16; }

void launch_split(hipStream_t s, const float *P, int64_t ldp, int64_t rows, int64_t K, void *img, int64_t img_rows,
                  int64_t row0, int64_t col0)
{
    if (rows <= 0 || K <= 0) return;
    const int64_t stride = round_up(img_rows, 256);
    hipLaunchKernelGGL(k_split, dim3((unsigned)((rows + NT - 1) / NT), (unsigned)(K / 8)), dim3(NT), 0, s, P, ldp, rows,
                       (v8bf *)img + (col0 / 8) * NS * stride + row0, stride);
}

// Units of one problem of the batched split and update (rows: a multiple of 256).
int64_t split_b_units(int64_t rows, int64_t K) { return rows > 0 ? rows / NT * (K / 8) : 0; }
int64_t syrk_split_b_units(int64_t rows)
{
    const int64_t T = rows > 0 ? rows / TM : 0;
    return T * (T + 1) / 2;
}

void launch_split_b(hipStream_t s, const BProb *P, const BWork &w, int64_t kk, int64_t K)
{
    if (w.total > 0) hipLaunchKernelGGL(k_split_b, dim3((unsigned)w.total), dim3(NT), 0, s, P, w, kk, K);
}

void launch_syrk_split_b(hipStream_t s, const BProb *P, const BWork &w, int64_t kk, int64_t K)
{
    if (w.total > 0) hipLaunchKernelGGL(k_syrk_split_b, dim3((unsigned)w.total), dim3(NT), 0, s, P, w, kk, K);
}

void launch_syrk_split(hipStream_t s, float *C, int64_t ldc, const void *img, int64_t img_rows, int64_t row0,
                       int64_t rows, int64_t K)
{
    if (rows <= 0 || K <= 0) return;
    const int64_t st = (rows + kSup - 1) / kSup;
    const int64_t nsup = st * (st + 1) / 2;
    const int64_t blocks = (nsup + kXcds - 1) / kXcds * kXcds * (kSup / TM) * (kSup / TM);
    hipLaunchKernelGGL(k_syrk_split, dim3((unsigned)blocks), dim3(NT), 0, s, C, ldc, (const v8bf *)img + row0,
                       round_up(img_rows, 256), rows, K);
}

void launch_strip_split(hipStream_t s, float *C, int64_t ldc, const void *img, int64_t rows, int64_t N, int64_t K)
{
    const int64_t tm = rows / TM, tn = N / TM;
    if (tm <= 0 || tn <= 0 || K <= 0) return;
    const int64_t blocks = (tm + kXcds - 1) / kXcds * kXcds * tn;
    hipLaunchKernelGGL(k_strip_split, dim3((unsigned)blocks), dim3(NT), 0, s, C, ldc, (const v8bf *)img,
                       round_up(rows, 256), rows, K, (int)tn);
}

}  // namespace mag
