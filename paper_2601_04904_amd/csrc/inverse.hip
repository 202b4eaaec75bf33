// Batched inverse of the diagonal Schur blocks, S = Atil_kk^-1 (the
// inverse-instead-of-trsm formulation of Sec. II-B), by blocked Gauss-Jordan
// elimination with partial pivoting inside the block.
//
// The elimination runs on M = A^T: a row-major d x d block read as a
// column-major matrix is its transpose, so the caller's block is the working
// matrix's starting value without a copy, and A^-1 = (M^-1)^T.
//
// Pivoting is implicit: no rows are swapped.  For column j the pivot is the
// not-yet-used row of M of largest |re| + |im| (lowest row index among
// magnitudes equal to 11 mantissa bits); that row is scaled and column j is
// eliminated from every other row.  In place, the slot of column j then
// holds column p_j of the accumulated transform T (T M = Q, Q the
// permutation with Q e_j = e_{p_j}), so at the end, with W the working matrix,
//     M^-1[j][c] = W[p_j][pinv(c)],   A^-1[c][j] = W[p_j][pinv(c)].
//
// Blocks up to 112 are inverted by one workgroup in one launch (gauss.h).  For
// larger ones the working matrix lives in memory and is eliminated in panels of
// kInvNB columns, a launch each:
//
// Layout: W (d x d) is column-major, element (r, c) at c * d + r, so a load of 16
// rows of a column by 16 lanes covers 256 consecutive bytes.
//
// Blocking: panel p is eliminated by one workgroup that holds it in registers.
// With F the eliminated panel (d x NB) and G the NB pivot rows as they were before
// it, its effect on every other column block is W <- W' + F G, W' the block with
// the pivot rows cleared: applied in the next panel's launch, by the panel
// workgroup to its own block (look-ahead) and by the other workgroups to the rest.
//
// What bounds it: the column chain of the panel workgroup, one CU while the others
// wait.  Measured alone, us per inverse (FP64 FMAs with every column of the panel
// updated at every pivot -> this form): d = 32 41 -> 19, 64 81 -> 43, 100 133 ->
// 112, 128 162 -> 138, 256 377 -> 289, 512 974 -> 843, 1024 3030 -> 2822.
//
// One launch per panel p = 0 .. np (np = ceil(d / NB)):
//   p < np : the panel workgroup applies T_{p-1} to block p and eliminates it;
//            every other column block except p - 1 takes T_{p-1}.
//   p = np : every column block except np - 1 takes T_{np-1}, and all of them
//            are written to the result, transposed and unscrambled.
// Column blocks are read from the caller's block until they are first
// written (block 0 and 1 by the panel workgroup, the others in launch 1).
#include "gauss.h"

namespace btsq {

// Where column block `blk` of the working matrix lives at the start of launch
// p: the caller's block (read as column-major M) until its first write.
__device__ inline const double2* block_source(const InvJob& J, int blk, int p) {
    const bool written = blk <= 1 ? p > blk : p > 1;
    return written ? J.W : J.src;
}

// The transform of panel p - 1 on a block: W <- W' + F G with F the panel's final
// columns (d x pnc, read from the working matrix), G the block's entries in the
// panel's pivot rows, W' the block with those rows cleared.  col[b]: 1 + the
// column within the panel that row m of row block b is the pivot row of, or 0.
// (W += (F - E) G would be the same with one subtraction, but loses digits in the
// pivot rows where the pivot is large.)  All of the workgroup calls it.
template <int NRB>
__device__ inline void apply_panel(PanelBlock<NRB>& W, const double2* F, int d, int pnc, int row0, int m, int i,
                                   const int* col, double2 (*G)[kInvNB]) {
    // F is read four row blocks at a time, one such chunk ahead of its MFMAs
    constexpr int CH = NRB / 4, NCH = kInvNB / 4 * CH;
    double2 f[2][4];
    auto load = [&](int t) {
        const int c = 4 * (t / CH) + i;
        const double2* column = F + (size_t)min(c, pnc - 1) * d;
#pragma unroll
        for (int b = 0; b < 4; ++b) f[t & 1][b] = column[min(row0 + (4 * (t % CH) + b) * 16 + m, d - 1)];
    };
    load(0);
#pragma unroll
    for (int b = 0; b < NRB; ++b) W.take_row(b, col[b] > 0, i, G[(col[b] - 1) & (kInvNB - 1)]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NCH; ++t) {
        const int kk = t / CH;
        if (t + 1 < NCH) load(t + 1);
        double2 g = G[4 * kk + i][m];
        if (pnc < kInvNB) g = sel2(4 * kk + i < pnc, g, make_double2(0.0, 0.0));
#pragma unroll
        for (int b = 0; b < 4; ++b) W.update(4 * (t % CH) + b, f[t & 1][b], g);
    }
}

// Column block blk of a matrix, rows past d repeating row d - 1 and columns past
// nc zero.
template <int NRB>
__device__ inline void load_block(PanelBlock<NRB>& W, const double2* src, int d, int j0, int nc, int row0, int m, int i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + i;
        const double2* column = src + (size_t)(j0 + min(c, nc - 1)) * d;
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            const double2 v = column[min(row0 + b * 16 + m, d - 1)];
            W.re[b][r] = v.x;
            W.im[b][r] = v.y;
        }
        // two row block sets: half the loads at a time, or their destinations and
        // the block together do not fit the registers
        if (NRB > 4 && r == 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (nc < kInvNB) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + i >= nc) {
#pragma unroll
                for (int b = 0; b < NRB; ++b) W.re[b][r] = W.im[b][r] = 0.0;
            }
    }
}

template <int NRB>
__device__ inline void store_block(const PanelBlock<NRB>& W, double2* dst, int d, int j0, int nc, int row0, int m, int i) {
    // opaque, so that the addresses are worked out here instead of being kept in
    // registers since load_block
    asm volatile("" : "+s"(j0), "+s"(row0));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + i;
        double2* column = dst + (size_t)(j0 + c) * d;
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            const int row = row0 + b * 16 + m;
            if (row < d && c < nc) column[row] = make_double2(W.re[b][r], W.im[b][r]);
        }
    }
}

// Update workgroup of launch p for column block blk: the block takes T_{p-1}; in
// the last launch it is also written to the result.  It reads the pivot rows of
// panel p-1 in its own columns only, so no workgroup reads what another writes
// in the same launch.  One operand read per 16 MFMAs: the same product on FP64
// FMAs read G from LDS once per wave and FMA group, which kept LDS busy twice as
// long as the arithmetic took.
template <int NW, int Q>
__device__ void step_update(const InvJob& J, int p, int blk, int tid) {
    constexpr int NB = kInvNB;
    constexpr int NRB = 4 * Q;
    constexpr int WR = 64 * Q;
    __shared__ double2 G[NB][NB];
    __shared__ int place[NW * WR];      // first: 1 + panel column of the rows; last launch: inverse permutation
    const int d = J.d;
    const int np = (d + NB - 1) / NB;
    const int c0 = blk * NB;
    if (c0 >= d || p == 0 || p > np) return;          // no such columns / nothing to apply
    const bool last = p == np;
    if (blk == p) return;                              // the panel workgroup's block
    const bool apply = blk != p - 1;                   // block p-1 is final after launch p-1
    if (!apply && !last) return;                       // nothing to do until the write-out
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = wave * WR, m = lane & 15, i = lane >> 4;
    const int q0 = (p - 1) * NB;                       // first column of panel p-1
    const int pnc = min(NB, d - q0);
    const int nc = min(NB, d - c0);
    PanelBlock<NRB> W;
    load_block(W, block_source(J, blk, p), d, c0, nc, row0, m, i);
    if (apply) {
        for (int e = tid; e < NW * WR; e += 64 * NW) place[e] = 0;
        __syncthreads();
        if (tid < pnc) place[J.perm[q0 + tid]] = tid + 1;
        __syncthreads();
        int col[NRB];
#pragma unroll
        for (int b = 0; b < NRB; ++b) col[b] = place[row0 + b * 16 + m];
        apply_panel(W, J.W + (size_t)q0 * d, d, pnc, row0, m, i, col, G);
    }
    if (!last) {
        store_block(W, J.W, d, c0, nc, row0, m, i);
        return;
    }
    // inverse permutation (cleared first: after a singular pivot the pivot rows
    // need not be a permutation, and every index stays in range)
    __syncthreads();
    for (int e = tid; e < d; e += 64 * NW) place[e] = 0;
    __syncthreads();
    for (int e = tid; e < d; e += 64 * NW) place[J.perm[e]] = e;
    __syncthreads();
    // A^-1[perm[col]][pinv(r)] = W[r][col]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + i;
        double2* out = J.dst + (size_t)J.perm[c0 + min(c, nc - 1)] * d;
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            const int row = row0 + b * 16 + m;
            if (row < d && c < nc) out[place[row]] = make_double2(W.re[b][r], W.im[b][r]);
        }
    }
}

// ---------------------------------------------------------------------------
// Panel workgroup of launch p: applies T_{p-1} to block p (look-ahead) and
// eliminates its kInvNB = 16 columns, four at a time.
//
// The block is held transposed in the accumulator layout of
// v_mfma_f64_16x16x4: wave w owns the 64 Q rows from 64 Q w on, as 4 Q row
// blocks of 16; lane l of block rb holds columns l/16 + 4r (r = 0..3) of row
// l%16, real and imaginary part apart.  Register r of the four blocks of 64
// rows is then a 4 x 4 grid (column 4r + l/16, block) that two stages of lane
// swaps turn into one row per lane with the four columns 4r .. 4r + 3 in
// registers, and the same swaps turn it back, into the layout the MFMA reads
// its second operand in.  In the row-per-lane form the group is eliminated:
// pivot search over the lanes, the winner's four entries handed to every wave
// through one LDS record, one barrier per column.  With F the eliminated group
// (d x 4) and G the group's four pivot rows as they were before it, the block
// becomes
//     W <- W' + F G,
// W' the block with the pivot rows cleared, G zero in the group's columns and
// F in their place: the same transform as W += (F - E) G, and one K = 4 step
// of complex MFMAs per row block.
//
// Per group of four at d = 512: four exchanges through LDS of about 1500 cycles and
// 2048 cycles of MFMAs (the FP64 rate of the CU), plus about 2500 of transposes,
// pivot rows and the barrier.
template <int NW, int Q>
__device__ void step_panel(const InvJob& J, int p, int tid, DevStatus* status) {
    constexpr int NB = kInvNB;
    constexpr int NRB = 4 * Q;                 // row blocks per wave
    constexpr int WR = 64 * Q;                 // rows per wave
    __shared__ double2 G[NB][NB];
    __shared__ GroupRec<NW, Q> rec;

    const int d = J.d;
    const int j0 = p * NB;
    if (j0 >= d) return;
    // The panel's column chain is the critical path of the whole inverse and
    // is latency-bound; where product workgroups of the other stream share
    // this CU, their waves would otherwise take most of the issue slots.
    __builtin_amdgcn_s_setprio(3);
    const int nc = min(NB, d - j0);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = wave * WR;
    const int m = lane & 15, i = lane >> 4;
    const double2* src = block_source(J, p, p);

    // (rows past d are marked used, so never chosen, and are not stored)
    // the places past NW that a read of four keys covers (no wave writes them, and
    // every wave passes a barrier before its first read)
    if (NW % 4 != 0 && tid < 2)
        for (int w = NW; w < (NW + 3) / 4 * 4; ++w) reinterpret_cast<unsigned*>(rec.key[tid])[w] = 0;
    PanelBlock<NRB> W;
    int used[Q];
    unsigned kmask[Q], krow[Q];       // key bits and row bits of a row's key, both 0 once it is used
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int r = row0 + q * 64 + lane;
        used[q] = p > 0 ? J.used[min(r, d - 1)] : 0;
        const bool free = r < d && used[q] == 0;
        kmask[q] = free ? kKeyBits : 0u;
        krow[q] = free ? key_row_bits(r) : 0u;
    }
    load_block(W, src, d, j0, nc, row0, m, i);
    if (p > 0) {
        // look-ahead
        int col[NRB];
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            const int row = row0 + b * 16 + m;
            const int c = row < d ? J.used[row] - (j0 - NB) : 0;
            col[b] = max(c, 0);
        }
        apply_panel(W, J.W + (size_t)(j0 - NB) * d, d, NB, row0, m, i, col, G);
        __syncthreads();      // G is reused below
    }

    bool bad = false;
    auto group = [&](auto gc) {
        constexpr int grp = decltype(gc)::value;      // its registers: component grp of the blocks
        const int g0 = grp * kGrp;
        if (g0 >= nc) return;
        const int count = min(kGrp, nc - g0);
        double2 u[Q][kGrp];
        int piv[kGrp];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int b = 0; b < 4; ++b) u[q][b] = make_double2(W.re[4 * q + b][grp], W.im[4 * q + b][grp]);
            transpose4(u[q]);
        }
        eliminate_group<NW, Q>(u, kmask, krow, count, row0, wave, lane, &rec, piv, bad);
#pragma unroll
        for (int s = 0; s < kGrp; ++s) {
            if (s >= count) {
                if (wave == 0 && lane < NB) G[s][lane] = make_double2(0.0, 0.0);
            } else {
                if (tid == 0) J.perm[j0 + g0 + s] = piv[s];
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (row0 + q * 64 + lane == piv[s]) used[q] = j0 + g0 + s + 1;
            }
        }
        // the group's pivot rows to G, F to its place in the block
        take_group_rows(W, row0, m, i, piv, G);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            transpose4(u[q]);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                W.re[4 * q + b][grp] = u[q][b].x;
                W.im[4 * q + b][grp] = u[q][b].y;
            }
        }
        __syncthreads();
        const double2 g = sel2((m >> 2) == grp, make_double2(0.0, 0.0), G[i][m]);
#pragma unroll
        for (int b = 0; b < NRB; ++b) W.update(b, u[b / 4][b % 4], g);
    };
    [&]<int... S>(std::integer_sequence<int, S...>) {
        (group(std::integral_constant<int, S>{}), ...);
    }(std::make_integer_sequence<int, NB / kGrp>{});
    if (bad && tid == 0 && atomicCAS(&status->code, 0, 3) == 0) status->tag = J.tag;

    // write back block p and the used flags
    store_block(W, J.W, d, j0, nc, row0, m, i);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int r = row0 + q * 64 + lane;
        if (r < d) J.used[r] = used[q];
    }
}

// grid.x = njobs * wg_per_job; workgroup 0 of a job is the panel workgroup.
template <int NW, int Q>
// At most 256 registers (two waves per SIMD): with 128 the column loop of 8 x 64 rows
// spills, 30.6 against 26.9 us per launch at d = 512.  At 256 only 8 x 128 rows spill, 12
// registers (36 bytes of scratch a lane).
__global__ __launch_bounds__(64 * NW, 2)
void inv_step(const InvJob* __restrict__ jobs, int p, int wg_per_job, DevStatus* status) {
    const int job = blockIdx.x / wg_per_job;
    const int w = blockIdx.x - job * wg_per_job;
    const InvJob J = jobs[job];
    if (w == 0) step_panel<NW, Q>(J, p, threadIdx.x, status);
    else {
        // The next panel's block goes to the update workgroup 8 of the job, whose
        // id is congruent to the panel workgroup's mod 8 (same XCD, same L2), so
        // the next launch's panel workgroup reads it where it was written.  A
        // bijection of the block indices: one transposition.
        int u = w - 1;
        const int next = p + 1;
        if (wg_per_job > 8 && next < wg_per_job - 1) u = u == 7 ? next : u == next ? 7 : u;
        step_update<NW, Q>(J, p, u, threadIdx.x);
    }
}

// Small blocks: one workgroup per matrix, one launch.
template <int NW, int Q>
__global__ __launch_bounds__(64 * NW, 2)
void inv_small(const InvJob* __restrict__ jobs, DevStatus* status) {
    __shared__ SmallInvLds<NW, Q> L;
    const InvJob J = jobs[blockIdx.x];
    __builtin_amdgcn_s_setprio(3);       // as in the panel workgroup
    small_inverse<NW, Q>(J.src, J.dst, J.d, J.tag, L, threadIdx.x, status);
}

// Kernel shape for dimension d.  Up to 112 one workgroup inverts the block in one
// launch (0, 1), above it is a launch per panel (2 .. 5).  Measured, us for one
// inverse, one workgroup against panels: d = 64 43 / 72, 100 112 / 114, 112 127 /
// 123 (in nine launches), 128 157 / 138.
int inv_variant(int d) { return d <= 64 ? 0 : d <= 112 ? 1 : d <= 128 ? 2 : d <= 256 ? 3 : d <= 512 ? 4 : 5; }

// Launches of one inverse of dimension d: panel steps p = 0 .. inv_steps(d) - 1.
int inv_steps(int d) { return inv_variant(d) < kFirstPanelVariant ? 1 : (d + kInvNB - 1) / kInvNB + 1; }

template <int NW, int Q>
static void launch_step(const InvJob* d_jobs, int njobs, int wg, int panel, DevStatus* status, hipStream_t s) {
    hipLaunchKernelGGL((inv_step<NW, Q>), dim3(njobs * wg), dim3(64 * NW), 0, s, d_jobs, panel, wg, status);
}

hipError_t launch_inv_step(const InvJob* d_jobs, int njobs, int variant, int panel, int maxd,
                           DevStatus* status, hipStream_t s) {
    if (njobs <= 0) return hipSuccess;
    const int wg = 1 + (maxd + kInvNB - 1) / kInvNB;
    switch (variant) {
        case 0: hipLaunchKernelGGL((inv_small<4, 1>), dim3(njobs), dim3(256), 0, s, d_jobs, status); break;
        case 1: hipLaunchKernelGGL((inv_small<8, 2>), dim3(njobs), dim3(512), 0, s, d_jobs, status); break;
        case 2: launch_step<2, 1>(d_jobs, njobs, wg, panel, status, s); break;
        case 3: launch_step<4, 1>(d_jobs, njobs, wg, panel, status, s); break;
        case 4: launch_step<8, 1>(d_jobs, njobs, wg, panel, status, s); break;
        default: launch_step<8, 2>(d_jobs, njobs, wg, panel, status, s); break;
    }
    return hipGetLastError();
}

// The whole inverse of njobs matrices that all use the panel kernel shape of
// dimension maxd: one launch per panel plus the final one.
hipError_t launch_inverse_sequence(const InvJob* d_jobs, int njobs, int maxd, DevStatus* status,
                                   hipStream_t s) {
    hipError_t e = hipSuccess;
    for (int p = 0; p < inv_steps(maxd) && e == hipSuccess; ++p)
        e = launch_inv_step(d_jobs, njobs, inv_variant(maxd), p, maxd, status, s);
    return e;
}

}  // namespace btsq
