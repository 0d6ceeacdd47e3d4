// trsv.hip -- preconditioner apply z = L^{-T} L^{-1} r of the refinement, and
// the substitution of the FP64 dense factor.
//
// L is a Cholesky factor (column-major, leading dimension npad, L in the lower
// triangle and L^T in the upper one), FP32 or FP64; r and z are FP64 and all
// arithmetic is FP64.  The diagonal blocks (128 x 128 of the FP32 factor, 64 x 64 of
// the FP64 one) are applied through their explicit inverses (in the factor's type,
// from the factorisation), so a block step is a small matrix-vector product.  Two
// kernels share the hand-off protocol below:
//   * trsv1_body (one workgroup per block, further down) serves the FP32 factors, with a
//     composite near step in single solves: 0.52 ms per direction at n = 32768; batched
//     (k_trsv_b, whose near step is not composite) 0.47 ms for 64 clouds of 1000 to
//     6000 points and 11 us for 32 of 50 to 400;
//   * the band kernel (trsv_body, one workgroup per two blocks) serves the FP64 factor,
//     whose inverses of both blocks just fit LDS: 1.1 ms per direction at n = 32768,
//     4.3 GB at 3.9 TB/s.
//
// Each triangular solve is ONE launch and no host round trips ("sync-free"
// substitution):
//   * a workgroup takes a ticket from an atomic counter; ticket order is the
//     order of the substitution, so every block a workgroup waits for belongs to a
//     workgroup that is already running -- forward progress does not depend
//     on how many workgroups fit on the device;
//   * block b streams its off-diagonal tiles in order (forward: L(b, j) from
//     the lower triangle; backward: L^T(b, j) from the upper triangle, where
//     the factorisation keeps the transpose); the tiles of a pair of blocks
//     are loaded into registers a whole pair-step ahead of the wait
//     for the solution blocks they multiply, and the workgroup's own right-hand
//     side and resident tiles before the first wait, so the HBM stream stays off
//     the dependency chain;
//   * the solution vector is the flag: before a solve every entry holds an
//     "unset" bit pattern (a signalling NaN no arithmetic produces); a workgroup
//     writes its solution entries with relaxed agent-scope atomic stores, and
//     a waiting wave reads the entries it needs with relaxed
//     agent-scope atomic loads until none is unset.  Each entry is written
//     once, so a value that is not the pattern is final: no counter, no
//     release or acquire fence (each fence a wave executes costs microseconds
//     of L2 write-back or invalidation) and no second read of the data;
//   * spin-waits are bounded: on exhaustion the kernel sets a status word and
//     finishes, and the host reports an error.
// HBM traffic per direction: one triangle of the factor, read once.
#include "internal.hpp"

namespace mag {
namespace {

constexpr int kSlot = 64;  // ints between the two tickets (256 bytes)

// counter layout (ints): fwd ticket @0, bwd ticket @kSlot
constexpr int kFwdTicket = 0;
constexpr int kBwdTicket = kSlot;
constexpr int kCounterInts = 2 * kSlot;

// the "unset" entry: a signalling NaN payload (arithmetic yields quiet NaNs)
constexpr uint64_t kUnset = 0x7ff4dead0badf00dull;

__device__ inline uint64_t ld_entry(const double *x, int64_t i)
{
    return __hip_atomic_load(reinterpret_cast<const uint64_t *>(x) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void st_entry(double *x, int64_t i, double v)
{
    __hip_atomic_store(reinterpret_cast<uint64_t *>(x) + i, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// The next ticket of this direction.  Its first workgroup zeroes the other
// direction's tickets (that solve is over or not begun), so a pair of solves
// leaves the counters as it found them but for the backward ticket, which the
// next forward solve zeroes.
template <bool BWD>
__device__ inline int take_ticket(int *counters)
{
    const int ticket = atomicAdd(&counters[BWD ? kBwdTicket : kFwdTicket], 1);
    if (ticket == 0) counters[BWD ? kFwdTicket : kBwdTicket] = 0;
    return ticket;
}

// The vectors' "unset" state is kept up by the solves themselves: the forward one
// unsets the entries of z, which the backward one will write, and the backward
// one those of its right-hand side y, each once it has read it, for the next
// forward solve.
template <bool BWD>
__device__ inline void unset_after_read(double *rhs, double *z, int64_t i)
{
    reinterpret_cast<uint64_t *>(BWD ? rhs : z)[i] = kUnset;
}

// Wave 0 (lanes 0..63): wait until the 64 entries of block j0 (and j1 if two)
// of x are set, and copy them to xs[0] (xs[1]).  Bounded: after spin_limit
// polls the status word is set and whatever was read is used.
__device__ inline void wait_blocks(const double *x, int64_t j0, int64_t j1, bool two, double (&xs)[2][64],
                                   int *status, long spin_limit)
{
    const int lane = threadIdx.x;
    uint64_t a, c = 0;
    long spins = 0;
    for (;;) {
        a = ld_entry(x, j0 * 64 + lane);
        if (two) c = ld_entry(x, j1 * 64 + lane);
        if (__ballot(a == kUnset || (two && c == kUnset)) == 0) break;
        if (++spins > spin_limit) {
            if (lane == 0) status[kStSpinTimeout] = 1;
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    xs[0][lane] = __builtin_bit_cast(double, a);
    if (two) xs[1][lane] = __builtin_bit_cast(double, c);
}

// Four consecutive factor entries (one row group of a tile column).
template <typename T>
struct Quad {
    T v[4];
};
__device__ inline void load_quad(const float *p, Quad<float> &q)
{
    const float4 f = *reinterpret_cast<const float4 *>(p);
    q.v[0] = f.x;
    q.v[1] = f.y;
    q.v[2] = f.z;
    q.v[3] = f.w;
}
__device__ inline void load_quad(const double *p, Quad<double> &q)
{
    const double2 a = *reinterpret_cast<const double2 *>(p);
    const double2 b = *reinterpret_cast<const double2 *>(p + 2);
    q.v[0] = a.x;
    q.v[1] = a.y;
    q.v[2] = b.x;
    q.v[3] = b.y;
}

// One triangular solve with the FP64 factor.  Forward (BWD = false): y = L^{-1} r, block b
// pulls tiles L(b, j), j < b, from the lower triangle.  Backward (BWD = true):
// z = L^{-T} y, block b pulls tiles L^T(b, j), j > b, from the upper
// triangle, where the factorisation stored L^T.  Both read a 64-row band of
// column segments per step, the same HBM access pattern.
//
// A workgroup owns two consecutive blocks (a 128-row band): it streams both
// blocks' tiles against every finished block outside the band, then solves
// the first block, applies the band's inner tile and solves the second, so
// the dependency chain crosses workgroups once per 128 rows.
template <bool BWD>
__device__ __forceinline__ void trsv_body(const double *__restrict__ L, int64_t ld,
                                          const double *__restrict__ dinv,
                                          double *__restrict__ rhs, double *__restrict__ x, double *__restrict__ z,
                                          int *counters, int nblk, int *status, long spin_limit)
{
    constexpr int BS = 64;
    constexpr int RG = BS / 4;      // row groups of a tile (4 rows each)
    constexpr int CG = 256 / RG;    // column groups
    constexpr int CPG = BS / CG;    // columns per group
    constexpr int H = 256 / BS;     // parts of a diagonal-block row's product
    constexpr int HC = BS / H;      // columns per part
    __shared__ double Dl[2][BS * (BS + 1)];  // Dinv of the two blocks, row-major, padded stride
    __shared__ double xs[2][BS];
    __shared__ double part[CG][BS];     // per column group partial sums of a block's rows
    __shared__ int s_band;
    const int tid = threadIdx.x;
    const int nband = nblk / 2;
    if (tid == 0) {
        const int ticket = take_ticket<BWD>(counters);
        s_band = BWD ? nband - 1 - ticket : ticket;
    }
    __syncthreads();
    const int band = s_band;
    // blocks in solve order: forward (2 band, 2 band + 1), backward (2 band + 1, 2 band)
    const int b0 = BWD ? 2 * band + 1 : 2 * band;
    const int b1 = BWD ? 2 * band : 2 * band + 1;
    // tile products: thread (rg, cg) owns rows 4 rg .. 4 rg + 3 and columns
    // CPG cg .. CPG cg + CPG - 1 of a BS x BS tile (four entries per column)
    const int rg = tid % RG, cg = tid / RG;
    // block solves: thread (h, row) takes part h of row's dot product
    const int row = tid % BS;
    const int h = tid / BS;

    // tile (b, j): element (r, c) at L[(j BS + c) ld + b BS + r] -- forward L(b, j)
    // from the lower triangle, backward L^T(b, j) from the upper triangle
    using Tile = Quad<double>[CPG];
    auto load = [&](int b, int j, Tile &t) {
        const double *p = L + ((int64_t)j * BS + CPG * cg) * ld + (int64_t)b * BS + 4 * rg;
#pragma unroll
        for (int c = 0; c < CPG; ++c) load_quad(p + (int64_t)c * ld, t[c]);
    };
    auto gemv = [&](const Tile &t, const double *xv, double (&acc)[4]) {
#pragma unroll
        for (int c = 0; c < CPG; ++c) {
            const double v = xv[CPG * cg + c];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += t[c].v[i] * v;
        }
    };

    // the right-hand side of both blocks and the band's inner tile (b1, b0) do not
    // depend on other bands: fetch them first, off the dependency chain
    double rhs0 = 0.0, rhs1 = 0.0;
    if (tid < BS) {
        rhs0 = rhs[(int64_t)b0 * BS + tid];
        rhs1 = rhs[(int64_t)b1 * BS + tid];
        unset_after_read<BWD>(rhs, z, (int64_t)b0 * BS + tid);
        unset_after_read<BWD>(rhs, z, (int64_t)b1 * BS + tid);
    }
    Tile ti;
    load(b1, b0, ti);

    // Dinv (column-major in memory) into row-major padded LDS
    for (int q = 0; q < 2; ++q) {
        const double *src = dinv + (int64_t)(q == 0 ? b0 : b1) * BS * BS;
        for (int e = tid; e < BS * BS; e += 256) {
            const int rr = e % BS, cc = e / BS;
            Dl[q][rr * (BS + 1) + cc] = src[e];
        }
    }
    double acc0[4] = {0.0, 0.0, 0.0, 0.0}, acc1[4] = {0.0, 0.0, 0.0, 0.0};
    // blocks outside the band, in the order they finish, two at a time.  A
    // pair's tiles are fetched before its wait, the next pair's right after it.
    const int nsteps = BWD ? (nblk - 2 - 2 * band) : 2 * band;
    Tile ta0, ta1, tb0, tb1;
    auto jof = [&](int st) { return BWD ? (nblk - 1 - st) : st; };
    // steps st and st + 1 (if any): wave 0 waits for both solution blocks (a
    // band writes its two blocks moments apart) and copies them to LDS
    auto consume2 = [&](int st, bool two) {
        if (tid < 64) wait_blocks(x, jof(st), two ? jof(st + 1) : 0, two, xs, status, spin_limit);
        __syncthreads();
        gemv(ta0, xs[0], acc0);
        gemv(ta1, xs[0], acc1);
        if (two) {
            gemv(tb0, xs[1], acc0);
            gemv(tb1, xs[1], acc1);
        }
        // xs is rewritten by the next step; after the last one, only once the
        // partial sums have passed the next barrier
        if (st + 2 < nsteps) __syncthreads();
    };
    if (nsteps > 0) {
        load(b0, jof(0), ta0);
        load(b1, jof(0), ta1);
    }
    if (nsteps > 1) {
        load(b0, jof(1), tb0);
        load(b1, jof(1), tb1);
    }
    for (int st = 0; st < nsteps; st += 2) {
        const bool two = st + 1 < nsteps;
        consume2(st, two);
        // both tiles of the next pair, a whole step ahead of their wait
        if (st + 2 < nsteps) {
            load(b0, jof(st + 2), ta0);
            load(b1, jof(st + 2), ta1);
        }
        if (st + 3 < nsteps) {
            load(b0, jof(st + 3), tb0);
            load(b1, jof(st + 3), tb1);
        }
    }

    // first block: x_b0 = Dinv_b0 (rhs_b0 - acc0)   (backward: Dinv^T)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[cg][4 * rg + i] = acc0[i];
    __syncthreads();
    if (tid < BS) {
        double sacc = 0.0;
#pragma unroll
        for (int g = 0; g < CG; ++g) sacc += part[g][tid];
        xs[0][tid] = rhs0 - sacc;
    }
    __syncthreads();
    double v = 0.0;
#pragma unroll 16
    for (int c = 0; c < HC; ++c) {
        const int cc = h * HC + c;
        v += (BWD ? Dl[0][cc * (BS + 1) + row] : Dl[0][row * (BS + 1) + cc]) * xs[0][cc];
    }
    part[h][row] = v;
    __syncthreads();
    if (tid < BS) {
        double sv = part[0][tid];
#pragma unroll
        for (int g = 1; g < H; ++g) sv += part[g][tid];
        xs[1][tid] = sv;
    }
    __syncthreads();
    // wave 0 writes the band's solution entries (each write releases that entry)
    if (tid < 64) st_entry(x, (int64_t)b0 * BS + tid, xs[1][tid]);
    // second block: acc1 += L(b1, b0) x_b0, then x_b1 = Dinv_b1 (rhs_b1 - acc1)
    gemv(ti, xs[1], acc1);
#pragma unroll
    for (int i = 0; i < 4; ++i) part[cg][4 * rg + i] = acc1[i];
    __syncthreads();
    if (tid < BS) {
        double sacc = 0.0;
#pragma unroll
        for (int g = 0; g < CG; ++g) sacc += part[g][tid];
        xs[0][tid] = rhs1 - sacc;
    }
    __syncthreads();
    v = 0.0;
#pragma unroll 16
    for (int c = 0; c < HC; ++c) {
        const int cc = h * HC + c;
        v += (BWD ? Dl[1][cc * (BS + 1) + row] : Dl[1][row * (BS + 1) + cc]) * xs[0][cc];
    }
    part[h][row] = v;
    __syncthreads();
    if (tid < 64) {
        double sv = part[0][tid];
#pragma unroll
        for (int g = 1; g < H; ++g) sv += part[g][tid];
        st_entry(x, (int64_t)b1 * BS + tid, sv);
    }
}

template <bool BWD>
__global__ void __launch_bounds__(256)
k_trsv(const double *__restrict__ L, int64_t ld, const double *__restrict__ dinv,
       double *__restrict__ rhs, double *__restrict__ x, double *__restrict__ z, int *counters, int nblk,
       int *status, long spin_limit)
{
    trsv_body<BWD>(L, ld, dinv, rhs, x, z, counters, nblk, status, spin_limit);
}

// One triangular solve of the FP32 factor with one 128-row block per
// workgroup and a composite near step.  With the solve's block b, its
// predecessor n (b - 1 forward, b + 1 backward) and the blocks before that
// ("far", streamed two at a time as in trsv_body):
//   x_b = y - Q_b x_n,   y = D_b (rhs_b - sum_far T(b, j) x_j),   Q_b = D_b T(b, n),
// with D_b the block's inverse (transposed backward) and T the streamed tile
// (forward L(b, j) from the lower triangle, backward L^T(b, j) from the upper
// one).  Q_b (k_near_q) and D_b stay resident from the workgroup's start, y is
// formed once the far blocks are in, so after its predecessor's block arrives
// a workgroup applies one resident tile and one reduction: the dependency
// chain costs one hand-off and one 128 x 128 product per block.
//
// Bound by that chain: the hand-off (a store becoming visible to a poll, about
// 1 us) and the product after it, 1.6 us a block together.  Hence eight waves that
// own 16 columns of every tile each: a wave polls its own 16 entries of a block
// and multiplies by them with no workgroup barrier between, Q_b is converted to
// FP64 before the wait, and one barrier is left, at the sum over the waves.  With
// one polling wave, two barriers and 256 threads a direction took 55 us at
// n = 3001 and 0.58 ms at n = 32768, now 40 us and 0.52 ms.
// COMPOSITE false (the batched solves): x_b = D_b (rhs_b - sum T(b, j) x_j), T(b, n)
// resident in the place of Q_b and D_b applied after the wait, so nothing but the factor's
// own FP32 entries is multiplied by, and no near tiles are formed with every factor (0.36 ms
// for 64 clouds of 1000 to 6000 points) for the two applications of its solve.
template <bool BWD, bool COMPOSITE>
__device__ __forceinline__ void trsv1_body(const float *__restrict__ L, int64_t ld, const float *__restrict__ dinv,
                                           const float *__restrict__ Qb, double *__restrict__ rhs,
                                           double *__restrict__ x, double *__restrict__ z, int *counters, int nblk,
                                           int *status, long spin_limit, const Gate &gate)
{
    constexpr int BS = 128, NW = 8, NT = 64 * NW;
    constexpr int WC = BS / NW;          // columns of a wave
    constexpr int TC = WC / 2;           // and of a thread (half waves take half each)
    constexpr int NP = NT / BS, PC = BS / NP;  // parts of the block product's sums
    __shared__ float Dl[BS * (BS + 1)];  // D_b, row-major, padded stride
    __shared__ double xs[NW][2][WC];
    __shared__ double part[NW][BS];
    __shared__ double rb[BS];
    __shared__ int s_blk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        // (the tickets are taken, and left for the next solve, behind a closed gate too)
        const double g = gate.value();  // on its way beside the ticket
        const int ticket = take_ticket<BWD>(counters);
        s_blk = !(g > gate.tol) ? -1 : BWD ? nblk - 1 - ticket : ticket;
    }
    __syncthreads();
    const int b = s_blk;
    if (b < 0) return;
    const int rg = lane & 31, ch = lane >> 5;     // tile products: rows 4 rg .., columns TC ch .. of the wave's
    const int row = tid & (BS - 1), h = tid >> 7;  // block product: part h of row's sum
    using Tile = Quad<float>[TC];
    auto load = [&](const float *base, int64_t ldb, Tile &t) {
        const float *p = base + (int64_t)(WC * wave + TC * ch) * ldb + 4 * rg;
#pragma unroll
        for (int c = 0; c < TC; ++c) load_quad(p + (int64_t)c * ldb, t[c]);
    };
    auto tile = [&](int j) { return L + (int64_t)j * BS * ld + (int64_t)b * BS; };
    auto gemv = [&](const Tile &t, const double *xv, double (&acc)[4]) {
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            const double v = xv[TC * ch + c];
            acc[0] += (double)t[c].v[0] * v;
            acc[1] += (double)t[c].v[1] * v;
            acc[2] += (double)t[c].v[2] * v;
            acc[3] += (double)t[c].v[3] * v;
        }
    };
    // the wave's entries of block j0 (lanes 0..15) and j1 (16..31) into xs[wave]
    auto wait = [&](int j0, int j1, bool two, bool nap) {
        const int e = lane & (WC - 1);
        const bool mine = lane < WC || (two && lane < 2 * WC);
        const int64_t at = (int64_t)(lane < WC ? j0 : j1) * BS + WC * wave + e;
        uint64_t a = 0;
        long spins = 0;
        for (;;) {
            if (mine) a = ld_entry(x, at);
            if (__ballot(mine && a == kUnset) == 0) break;
            if (++spins > spin_limit) {
                if (lane == 0) status[kStSpinTimeout] = 1;
                break;
            }
            if (nap) __builtin_amdgcn_s_sleep(1);
        }
        if (mine) xs[wave][lane < WC ? 0 : 1][e] = __builtin_bit_cast(double, a);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // read back by this wave only
        __builtin_amdgcn_wave_barrier();
    };
    // sums of the wave's two half-wave column groups, then of the waves (part)
    auto to_part = [&](double (&acc)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += __shfl_xor(acc[i], 32);
        if (ch == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) part[wave][4 * rg + i] = acc[i];
        }
    };
    auto jof = [&](int st) { return BWD ? (nblk - 1 - st) : st; };
    const int nsteps = BWD ? (nblk - 1 - b) : b;  // blocks solved before this one
    const bool has_near = nsteps >= 1;
    const int nfar = has_near ? nsteps - 1 : 0;

    // resident from the start: the right-hand side, D_b and the near tile Q_b
    double r0 = 0.0;
    if (tid < BS) {
        r0 = rhs[(int64_t)b * BS + tid];
        unset_after_read<BWD>(rhs, z, (int64_t)b * BS + tid);
    }
    Tile tq;
    if (has_near) load(COMPOSITE ? Qb + (int64_t)b * BS * BS : tile(jof(nsteps - 1)), COMPOSITE ? BS : ld, tq);
    Tile ta, tb;
    if (nfar > 0) load(tile(jof(0)), ld, ta);
    if (nfar > 1) load(tile(jof(1)), ld, tb);
    {
        const float *src = dinv + (int64_t)b * BS * BS;
        float d[BS * BS / NT];
#pragma unroll
        for (int e = 0; e < BS * BS / NT; ++e) d[e] = src[tid + NT * e];
#pragma unroll
        for (int e = 0; e < BS * BS / NT; ++e) Dl[row * (BS + 1) + h + NP * e] = d[e];
    }
    double q[TC][4];
#pragma unroll
    for (int c = 0; c < TC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) q[c][i] = has_near ? (double)tq[c].v[i] : 0.0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int st = 0; st < nfar; st += 2) {
        const bool two = st + 1 < nfar;
        wait(jof(st), two ? jof(st + 1) : 0, two, true);
        gemv(ta, xs[wave][0], acc);
        if (two) gemv(tb, xs[wave][1], acc);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // xs is rewritten by the next wait
        __builtin_amdgcn_wave_barrier();
        if (st + 2 < nfar) load(tile(jof(st + 2)), ld, ta);
        if (st + 3 < nfar) load(tile(jof(st + 3)), ld, tb);
    }
    // the predecessor's block through tq
    auto near = [&](double (&a)[4]) {
        wait(jof(nsteps - 1), 0, false, false);
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            const double xv = xs[wave][0][TC * ch + c];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] += q[c][i] * xv;
        }
    };
    if (!COMPOSITE && has_near) near(acc);
    // y = D_b (rhs_b - acc)
    to_part(acc);
    __syncthreads();
    if (tid < BS) {
        double sacc = 0.0;
#pragma unroll
        for (int g = 0; g < NW; ++g) sacc += part[g][tid];
        rb[tid] = r0 - sacc;
    }
    __syncthreads();
    double v = 0.0;
#pragma unroll 16
    for (int c = 0; c < PC; ++c) {
        const int cc = h * PC + c;
        const float d = BWD ? Dl[cc * (BS + 1) + row] : Dl[row * (BS + 1) + cc];
        v += (double)d * rb[cc];
    }
    part[h][row] = v;
    __syncthreads();
    double y = 0.0;
    if (tid < BS) {
#pragma unroll
        for (int g = 0; g < NP; ++g) y += part[g][tid];
    }
    if (!COMPOSITE || !has_near) {
        if (tid < BS) st_entry(x, (int64_t)b * BS + tid, y);
        return;
    }
    __syncthreads();  // part is rewritten below
    // x_b = y - Q_b x_n
    double aq[4] = {0.0, 0.0, 0.0, 0.0};
    near(aq);
    to_part(aq);
    __syncthreads();
    if (tid < BS) {
        double sq = 0.0;
#pragma unroll
        for (int g = 0; g < NW; ++g) sq += part[g][tid];
        st_entry(x, (int64_t)b * BS + tid, y - sq);
    }
}

template <bool BWD>
__global__ void __launch_bounds__(512)
k_trsv1(const float *__restrict__ L, int64_t ld, const float *__restrict__ dinv, const float *__restrict__ Qb,
        double *__restrict__ rhs, double *__restrict__ x, double *__restrict__ z, int *counters, int nblk, int *status,
        long spin_limit, Gate gate)
{
    trsv1_body<BWD, true>(L, ld, dinv, Qb, rhs, x, z, counters, nblk, status, spin_limit, gate);
}

// The near tiles of k_trsv1 for every 128-block of the FP32 factor, both
// directions: Q = D_b T(b, n) (forward: D_b L(b, b - 1); backward: D_b^T L^T(b, b + 1))
// with FP64 accumulation of the FP32 entries, stored in FP32, column-major, at
// Q + (d nblk + b) 128^2.  The first block in solve order has none.
// A workgroup forms one 64 x 64 quadrant on the FP64 matrix cores (at small sizes the
// launch is one block's latency: 44 us for a whole block per workgroup on the
// vector unit); K in two stages of 64, of which the triangular D leaves one empty
// for half of the quadrants.  v_mfma_f64_16x16x4: lane 16 kq + q supplies A(q, kq) and
// B(kq, q) and holds D(kq + 4 v, q); A from the tile's columns and B from D's rows,
// so sixteen lanes store sixteen consecutive rows.
__global__ void __launch_bounds__(256)
k_near_q(const float *__restrict__ A, int64_t npad, const float *__restrict__ dinv, float *__restrict__ Q, int nblk)
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int B = 128, H = 64, SL = 80;  // stage stride: the four k-rows of a read on disjoint banks
    __shared__ float Xs[H * SL];  // X(i, k) at Xs[k SL + i]
    __shared__ float Ys[H * SL];  // Y(k, j) at Ys[k SL + j]
    const int b = blockIdx.x, d = blockIdx.y;
    const bool bwd = d == 1;
    if (bwd ? (b >= nblk - 1) : (b == 0)) return;  // uniform per workgroup
    const int jn = bwd ? b + 1 : b - 1;
    const int i0 = H * (blockIdx.z & 1), j0 = H * (blockIdx.z >> 1);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane & 15, kq = lane >> 4;
    const float *D = dinv + (int64_t)b * B * B;  // column-major inverse
    v4d acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[t][v] = 0.0;
    for (int k0 = 0; k0 < B; k0 += H) {
        if (bwd ? (k0 < i0) : (k0 > i0)) continue;  // D(i, k) = 0 for k > i, D(k, i) for k < i
        // every load in flight before the first LDS store
        float xv[H * H / 256], yv[H * H / 256];
        const int u = tid & (H - 1), v0 = tid >> 6;
#pragma unroll
        for (int e = 0; e < H * H / 256; ++e) {
            const int v = v0 + 4 * e;
            xv[e] = bwd ? D[(i0 + v) * B + k0 + u] : D[(k0 + v) * B + i0 + u];
            // tile T(b, jn): element (r, c) at A[(jn B + c) npad + b B + r], as Y(k = r, j = c)
            yv[e] = A[((int64_t)jn * B + j0 + v) * npad + (int64_t)b * B + k0 + u];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < H * H / 256; ++e) {
            const int v = v0 + 4 * e;
            Xs[bwd ? u * SL + v : v * SL + u] = xv[e];
            Ys[u * SL + v] = yv[e];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < H; k += 4) {
            const double x = (double)Xs[(k + kq) * SL + 16 * wave + q];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Ys[(k + kq) * SL + 16 * t + q], x, acc[t], 0, 0, 0);
        }
    }
    float *dst = Q + ((int64_t)d * nblk + b) * B * B;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[(j0 + 16 * t + kq + 4 * v) * B + i0 + 16 * wave + q] = (float)acc[t][v];
}

// Batched: workgroups of problem p take tickets from p's own counters, so the
// forward-progress argument holds per problem; problems never wait on each other.
template <bool BWD>
__global__ void __launch_bounds__(512)
k_trsv_b(const BProb *__restrict__ P, BWork w, int rhs_slot, int x_slot, int z_slot, long spin_limit)
{
    const int i = bfind(w.pref, w.na, blockIdx.x);
    const BProb &q = P[w.plist[i]];
    if (!q.active) return;
    trsv1_body<BWD, false>(q.A, q.npad, q.dinv, nullptr, q.vec + (int64_t)rhs_slot * q.npad,
                          q.vec + (int64_t)x_slot * q.npad, q.vec + (int64_t)z_slot * q.npad, q.ints + 64,
                          (int)(q.npad / 128), q.ints, spin_limit, Gate());
}

// Tickets zero and the vector in `slot` unset, one workgroup per problem.
__global__ void k_prec_begin_b(const BProb *__restrict__ P, int slot)
{
    const BProb &q = P[blockIdx.x];
    for (int e = threadIdx.x; e < kCounterInts; e += blockDim.x) q.ints[64 + e] = 0;
    uint64_t *a = reinterpret_cast<uint64_t *>(q.vec + (int64_t)slot * q.npad);
    for (int64_t e = threadIdx.x; e < q.npad; e += blockDim.x) a[e] = kUnset;
}

// Start of a refinement: status words (optional) and tickets zero, y unset, ones
// on [0, n) and zero on [n, npad) into rhs (optional).
__global__ void k_refine_begin(double *__restrict__ y, double *__restrict__ rhs, int64_t n, int64_t npad,
                               int *counters, int *status)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e < kCounterInts) counters[e] = 0;
    if (status && e < kStCount) status[e] = 0;
    if (e < npad) {
        reinterpret_cast<uint64_t *>(y)[e] = kUnset;
        if (rhs) rhs[e] = e < n ? 1.0 : 0.0;
    }
}

}  // namespace

size_t prec_counter_ints() { return kCounterInts; }

int64_t prec_b_units(int64_t npad) { return npad / 128; }

void launch_prec_begin_b(hipStream_t s, const BProb *P, int B, int tmp_slot)
{
    if (B > 0) hipLaunchKernelGGL(k_prec_begin_b, dim3(B), dim3(256), 0, s, P, tmp_slot);
}

// x_slot = (L L^T)^{-1} rhs_slot for every problem of the work list (units = npad/128 each)
void launch_prec_apply_b(hipStream_t s, const BProb *P, const BWork &w, int rhs_slot, int tmp_slot,
                         int x_slot, long spin_limit)
{
    if (w.na <= 0) return;
    hipLaunchKernelGGL(k_trsv_b<false>, dim3((unsigned)w.total), dim3(512), 0, s, P, w, rhs_slot, tmp_slot, x_slot,
                       spin_limit);
    hipLaunchKernelGGL(k_trsv_b<true>, dim3((unsigned)w.total), dim3(512), 0, s, P, w, tmp_slot, x_slot, tmp_slot,
                       spin_limit);
}

void launch_refine_begin(hipStream_t s, double *y_tmp, double *rhs, int64_t n, int64_t npad, int *counters,
                         int *status)
{
    hipLaunchKernelGGL(k_refine_begin, dim3((unsigned)((npad + 255) / 256)), dim3(256), 0, s, y_tmp, rhs, n, npad,
                       counters, status);
}

void launch_prec_apply(hipStream_t s, const float *L, int64_t npad, const float *dinv,
                       const double *r, double *y_tmp, double *z, int *counters, int *status, const float *Q,
                       long spin_limit, Gate gate)
{
    const int nblk = (int)(npad / 128);
    const float *Qb = Q + (int64_t)nblk * 128 * 128;  // the backward direction's tiles
    double *rhs = const_cast<double *>(r);  // the forward solve only reads it
    hipLaunchKernelGGL(k_trsv1<false>, dim3(nblk), dim3(512), 0, s, L, npad, dinv, Q, rhs, y_tmp, z, counters, nblk,
                       status, spin_limit, gate);
    hipLaunchKernelGGL(k_trsv1<true>, dim3(nblk), dim3(512), 0, s, L, npad, dinv, Qb, y_tmp, z, (double *)nullptr,
                       counters, nblk, status, spin_limit, gate);
}

size_t near_q_floats(int64_t npad) { return (size_t)npad * 256; }

void launch_near_q(hipStream_t s, const float *A, int64_t npad, const float *dinv, float *Q)
{
    const int nblk = (int)(npad / 128);
    if (nblk < 2) return;
    hipLaunchKernelGGL(k_near_q, dim3((unsigned)nblk, 2, 4), dim3(256), 0, s, A, npad, dinv, Q, nblk);
}

void launch_chol64_solve(hipStream_t s, const double *L, int64_t npad, const double *dinv, const double *r,
                         double *y_tmp, double *z, int *counters, int *status,
                        long spin_limit)
{
    const int nblk = (int)(npad / 64);  // even: npad is a multiple of 256
    double *rhs = const_cast<double *>(r);  // the forward solve only reads it
    hipLaunchKernelGGL(k_trsv<false>, dim3(nblk / 2), dim3(256), 0, s, L, npad, dinv, rhs, y_tmp, z, counters, nblk,
                       status, spin_limit);
    hipLaunchKernelGGL(k_trsv<true>, dim3(nblk / 2), dim3(256), 0, s, L, npad, dinv, y_tmp, z, (double *)nullptr,
                       counters, nblk, status, spin_limit);
}

}  // namespace mag
