// Whole solves of small instances: one workgroup per instance, one launch
// for a batch.
//
// With diagonal blocks and tip of at most kFusedMaxDim, every operation of
// the sweeps is a product of small blocks, and one grouped launch per
// dependency level leaves the GPU waiting on launches most of the time.
// Here one workgroup executes its instance's whole operation list -- the
// products, diagonal-block inverses and block sums of the forward and
// backward sweeps (Alg. 1 and 2, with the arrowhead terms of Sec. III-A and
// the partition and reduced-system steps of Sec. III-B when asked for) -- in
// dependency order.  Instances are independent, so no workgroup ever waits on
// another one.
//
// A step is all the products of one dependency level, or one inverse, or one
// sum, with a workgroup barrier between steps.  The products of a step are
// cut into 16 x 16 complex tiles and the waves take the tiles in turn: a wave
// reads its rows of A and columns of B from memory straight into the layout of
// v_mfma_f64_16x16x4 (nothing is shared between waves at 16 x 16, so LDS and
// its barriers would only add latency).  Inverses are gauss.h's one-workgroup
// form.
//
// What bounds it: the chain of an instance's steps on one CU (memory latency
// and a barrier per step, and the column chain of each inverse).  512 instances
// of n = 16, b = 32 in one launch: 2.9 -> 1.9 ms (LDS-staged 32 x 32 tiles by the
// whole workgroup, one product at a time, an inverse with three barriers per
// column -> this form); one instance 2.15 -> 1.12 ms.
#include "tile16.h"
#include <climits>

namespace btsq {

// Values every lane holds alike, moved to scalar registers so that branches and
// addresses on them stay uniform.
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline double uni(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)uni((int)(unsigned)b), hi = (unsigned)uni((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double2 uni(double2 x) { return make_double2(uni(x.x), uni(x.y)); }
template <class T> __device__ inline T* uni(T* p) {
    const unsigned long long b = (unsigned long long)p;
    const unsigned lo = (unsigned)uni((int)(unsigned)b), hi = (unsigned)uni((int)(unsigned)(b >> 32));
    return (T*)(((unsigned long long)hi << 32) | lo);
}

// Global-memory pointers as such (not generic), so that their loads and
// stores do not count against the LDS wait counter.
#ifdef __HIP_DEVICE_COMPILE__
typedef const __attribute__((address_space(1))) double2* gcp;
typedef __attribute__((address_space(1))) double2* gp;
#else
typedef const double2* gcp;
typedef double2* gp;
#endif

// ---------------------------------------------------------------------------
// One 16 x 16 tile of D = beta C + sum_t alpha_t op(A_t) op(B_t), by one wave.  op is
// in LDS.
__device__ void fused_tile(const GemmOp& op, int tile, int lane, Turn& XA, Turn& XB) {
    const OpRegs o(op, lane);
    const int m = o.head(offsetof(GemmOp, m) / 4), n = o.head(offsetof(GemmOp, n) / 4);
    const int tn = (n + 15) >> 4;
    int ti = 0;                                       // tile / tn, at most 4 rows of tiles
    while ((ti + 1) * tn <= tile) ++ti;
    const int i0 = ti * 16, j0 = (tile - ti * tn) * 16;
    const int q = lane & 15, kq = lane >> 4;
    double2 cv[4] = {};
    double2* C = op_c(o);
    if (C) {
        const int ldc = o.head(offsetof(GemmOp, ldc) / 4);
        const __amdgpu_buffer_rsrc_t rc = fused_rsrc(C, m, n, ldc);
#pragma unroll
        for (int r = 0; r < 4; ++r) cv[r] = load16(rc, (__mul24(i0 + kq + 4 * r, ldc) + j0 + q) * 16);
    }
    v4d re, im;
    tile16_sum(o, m, n, i0, j0, lane, XA, XB, re, im);
    const double2 beta = op_beta(o);
    const int ldd = o.head(offsetof(GemmOp, ldd) / 4);
    const __amdgpu_buffer_rsrc_t rd = fused_rsrc(op_d(o), m, n, ldd);
    if (j0 + q < n) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double2 v = make_double2(re[r], im[r]);
            if (C) cfma(v, beta, cv[r]);
            store16(rd, (__mul24(i0 + kq + 4 * r, ldd) + j0 + q) * 16, v);
        }
    }
}

// ---------------------------------------------------------------------------
// Block sum D = sum_j c_j op_j(X_j) (op_j = X_j^H when bit j of hmask is set;
// such an input is stored cols x rows and is not D).
template <int FT>
__device__ void fused_add(const AddOp& op, int tid) {
    const int rows = uni(op.rows), cols = uni(op.cols), nin = uni(op.nin);
    const unsigned hmask = (unsigned)uni((int)op.hmask);
    gp D = (gp)uni(op.D);
    for (int e = tid; e < rows * cols; e += FT) {
        const int r = e / cols, c = e - r * cols;
        double2 acc = make_double2(0.0, 0.0);
        for (int j = 0; j < nin; ++j) {
            gcp X = (gcp)uni(op.X[j]);
            double2 x;
            if ((hmask >> j) & 1u) {
                x = X[(size_t)c * rows + r];
                x.y = -x.y;
            } else {
                x = X[e];
            }
            cfma(acc, uni(op.c[j]), x);
        }
        D[e] = acc;
    }
}

// ---------------------------------------------------------------------------
// The records of the next step are read from memory while the current one runs
// and handed over through LDS, and the step after that is read meanwhile, so no
// step waits for its own description.
// FW waves per workgroup: 8 while every instance has a CU to itself, else 4 (one
// instance 1.12 against 1.30 ms; 512 of them 3.3 against 3.0).  With 4, 48 bytes a lane go
// to scratch, beside scalars kept in vector registers in both.
template <int FW>
__global__ __launch_bounds__(64 * FW)
void fused_solve(const FusedTask* __restrict__ tasks, const FusedStep* __restrict__ steps,
                 const FusedRec* __restrict__ recs, DevStatus* status) {
    constexpr int FT = 64 * FW;
    constexpr int kWords = sizeof(FusedRec) / 16;                 // uint4 per record
    constexpr int kPer = (kFusedStepRecs * kWords + FT - 1) / FT;
    union Work {                       // a step uses one of them
        SmallInvLds<FW, 1> inv;
        Turn turn[FW][2];
    };
    __shared__ Work L;
    __shared__ FusedRec srec[2][kFusedStepRecs];
    const FusedTask T = tasks[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    uint4 w[kPer];
    auto fetch = [&](const FusedStep& st) {
        const uint4* from = reinterpret_cast<const uint4*>(recs + st.first);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + FT * i;
            if (e < st.count * kWords) w[i] = from[e];
        }
    };
    auto hand_over = [&](const FusedStep& st, int buf) {
        uint4* to = reinterpret_cast<uint4*>(srec[buf]);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + FT * i;
            if (e < st.count * kWords) to[e] = w[i];
        }
    };
    if (T.count <= 0) return;
    FusedStep cur = steps[T.first], nxt = steps[T.first + min(1, T.count - 1)];
    fetch(cur);
    hand_over(cur, 0);
    __syncthreads();
    for (int q = 0; q < T.count; ++q) {
        const FusedRec* R = srec[q & 1];
        const bool more = q + 1 < T.count;
        if (more) fetch(nxt);
        const FusedStep after = steps[T.first + min(q + 2, T.count - 1)];
        if (cur.type == 0) {
            // the products' first tiles, one per lane
            const int begin = lane < cur.count ? R[lane].tile_begin : INT_MAX;
            for (int e = wave; e < cur.tiles; e += FW) {
                const int r = __popcll(__ballot(begin <= e)) - 1;
                fused_tile(*reinterpret_cast<const GemmOp*>(R[r].body), e - uni(R[r].tile_begin), lane,
                           L.turn[wave][0], L.turn[wave][1]);
            }
        } else if (cur.type == 1) {
            const FusedInv& J = *reinterpret_cast<const FusedInv*>(R[0].body);
            small_inverse<FW, 1>(uni(J.src), uni(J.dst), uni(J.d), uni(J.tag), L.inv, tid, status);
            __builtin_amdgcn_s_setprio(0);
        } else {
            fused_add<FT>(*reinterpret_cast<const AddOp*>(R[0].body), tid);
        }
        if (more) hand_over(nxt, (q + 1) & 1);
        // the step's global writes and LDS reads are complete
        __syncthreads();
        cur = nxt;
        nxt = after;
    }
}

hipError_t launch_fused(const FusedTask* d_tasks, int ntasks, const FusedStep* d_steps, const FusedRec* d_recs,
                        DevStatus* status, hipStream_t s) {
    if (ntasks <= 0) return hipSuccess;
    constexpr int kCUs = 256;
    if (ntasks <= kCUs)
        hipLaunchKernelGGL(fused_solve<8>, dim3(ntasks), dim3(512), 0, s, d_tasks, d_steps, d_recs, status);
    else
        hipLaunchKernelGGL(fused_solve<4>, dim3(ntasks), dim3(256), 0, s, d_tasks, d_steps, d_recs, status);
    return hipGetLastError();
}

}  // namespace btsq
