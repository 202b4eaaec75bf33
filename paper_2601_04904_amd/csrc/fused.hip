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
#include "gauss.h"
#include <climits>
#include <cstddef>

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
// A product's descriptor in the registers of a wave: lane l holds dwords l and
// 64 + l of the GemmOp, so it is read from LDS in one latency and a field is one
// lane read.
struct OpRegs {
    unsigned w0, w1;
    __device__ inline OpRegs(const GemmOp& op, int lane) {
        const unsigned* p = reinterpret_cast<const unsigned*>(&op);
        w0 = p[lane];
        w1 = p[64 + min(lane, (int)(sizeof(GemmOp) / 4) - 65)];
    }
    static __device__ inline int lane_of(unsigned w, int i) { return __builtin_amdgcn_readlane((int)w, i); }
    // dword i (a constant below 64)
    __device__ inline int head(int i) const { return lane_of(w0, i); }
    // dword f of term s
    __device__ inline int term(int s, int f) const {
        constexpr int kFirst = offsetof(GemmOp, t) / 4, kLen = sizeof(GemmTerm) / 4;
        const int i = kFirst + kLen * s + f;
        return i < 64 ? lane_of(w0, i) : lane_of(w1, i - 64);
    }
    static __device__ inline double real(int lo, int hi) {
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    }
    static __device__ inline double2* ptr(int lo, int hi) {
        return (double2*)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    }
};
static_assert(sizeof(GemmOp) / 4 > 64 && sizeof(GemmOp) / 4 <= 128, "two dwords per lane");
static_assert(kFusedMaxDim * kFusedMaxDim * sizeof(double2) < (1u << 30), "32-bit offsets");

// Operands, C and D are addressed through raw buffer resources with 32-bit byte
// offsets; an offset past the record count (the operand's extent) reads as zero
// and is not written, so rows outside the product need no clamp.
__device__ inline __amdgpu_buffer_rsrc_t fused_rsrc(double2* base, int rows, int cols, int ld) {
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, ((rows - 1) * ld + cols) * 16, 0x00020000);
}
__device__ inline double2 load16(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
typedef unsigned u4 __attribute__((ext_vector_type(4)));
__device__ inline void store16(__amdgpu_buffer_rsrc_t r, int off, double2 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off, 0, 0);
}

// Operands that run along k in memory (A as stored, B^H) are read 16 k of a row by
// 16 lanes and turned through a piece of LDS of the wave's own (no barrier).
typedef double2 Turn[16][17];

// One 16 x 16 tile of D = beta C + sum_t alpha_t op(A_t) op(B_t), by one wave.
// The k range of every term is taken 16 at a time; the next chunk's loads (of the
// same or the next term) are issued before the current chunk's MFMAs.  Entries
// of A and B past k are cleared; rows and columns outside the product only reach
// entries of D that are not stored.  op is in LDS.
__device__ void fused_tile(const GemmOp& op, int tile, int lane, Turn& XA, Turn& XB) {
    const OpRegs o(op, lane);
    const int m = o.head(offsetof(GemmOp, m) / 4), n = o.head(offsetof(GemmOp, n) / 4);
    const int nt = o.head(offsetof(GemmOp, nterms) / 4);
    const int tn = (n + 15) >> 4;
    int ti = 0;                                       // tile / tn, at most 4 rows of tiles
    while ((ti + 1) * tn <= tile) ++ti;
    const int i0 = ti * 16, j0 = (tile - ti * tn) * 16;
    const int q = lane & 15, kq = lane >> 4;
    v4d re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    double2 cv[4] = {};
    double2* C = OpRegs::ptr(o.head(offsetof(GemmOp, C) / 4), o.head(offsetof(GemmOp, C) / 4 + 1));
    if (C) {
        const int ldc = o.head(offsetof(GemmOp, ldc) / 4);
        const __amdgpu_buffer_rsrc_t rc = fused_rsrc(C, m, n, ldc);
#pragma unroll
        for (int r = 0; r < 4; ++r) cv[r] = load16(rc, (__mul24(i0 + kq + 4 * r, ldc) + j0 + q) * 16);
    }

    // The chunk to load next: term s at offset c0.  Element t of a lane lies along
    // k (row kq + 4 t of the tile, k = q) or across (row or column q, k = 4 t + kq):
    // byte offsets va + t da (vb + t db), from one chunk to the next ka (kb) more.
    int s = -1, c0 = 0, k = 0, va = 0, vb = 0, da = 0, db = 0, ka = 0, kb = 0;
    bool ah = false, bh = false;
    double2 alpha = make_double2(1.0, 0.0);
    __amdgpu_buffer_rsrc_t ra, rb;
    auto advance = [&]() {
        c0 += 16;
        if (c0 < k) {
            va += ka;
            vb += kb;
            return;
        }
        c0 = 0;
        do ++s; while (s < nt && o.term(s, offsetof(GemmTerm, k) / 4) <= 0);
        if (s >= nt) return;
        k = o.term(s, offsetof(GemmTerm, k) / 4);
        const int lda = o.term(s, offsetof(GemmTerm, lda) / 4), ldb = o.term(s, offsetof(GemmTerm, ldb) / 4);
        const int flags = o.term(s, offsetof(GemmTerm, flags) / 4);
        constexpr int kAl = offsetof(GemmTerm, alpha) / 4;
        alpha = make_double2(OpRegs::real(o.term(s, kAl), o.term(s, kAl + 1)),
                             OpRegs::real(o.term(s, kAl + 2), o.term(s, kAl + 3)));
        ah = flags & kTermAH;
        bh = flags & kTermBH;
        double2* A = OpRegs::ptr(o.term(s, 0), o.term(s, 1));
        double2* B = OpRegs::ptr(o.term(s, 2), o.term(s, 3));
        ra = ah ? fused_rsrc(A, k, m, lda) : fused_rsrc(A, m, k, lda);
        rb = bh ? fused_rsrc(B, n, k, ldb) : fused_rsrc(B, k, n, ldb);
        const int la = __mul24(kq, lda), lb = __mul24(kq, ldb);
        va = (la + q + (ah ? i0 : i0 * lda)) * 16;
        vb = (lb + q + (bh ? j0 * ldb : j0)) * 16;
        da = 64 * lda;
        db = 64 * ldb;
        ka = ah ? 256 * lda : 256;
        kb = bh ? 256 : 256 * ldb;
    };
    static_assert(offsetof(GemmTerm, A) == 0 && offsetof(GemmTerm, B) == 8, "pointers first");
    struct Chunk {
        double2 a[4], b[4];
        double2 alpha;         // of its term, as ah, bh
        bool ah, bh;
        int left;              // the k left in the term from its start
    } ch[2];
    auto load = [&](Chunk& c) {
        c.ah = ah;
        c.bh = bh;
        c.alpha = alpha;
        c.left = k - c0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            c.a[t] = load16(ra, va + t * da);
            c.b[t] = load16(rb, vb + t * db);
        }
    };
    auto turn = [&](double2* v, Turn& X) {
#pragma unroll
        for (int t = 0; t < 4; ++t) X[q][kq + 4 * t] = v[t];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = X[4 * t + kq][q];
    };
    auto flip = [](double v) {
        return __longlong_as_double(__double_as_longlong(v) ^ (long long)0x8000000000000000ull);
    };
    auto multiply = [&](Chunk& c) {
        const bool one = c.alpha.y == 0.0 && (c.alpha.x == 1.0 || c.alpha.x == -1.0);
        const bool neg = one && c.alpha.x < 0.0;
        if (!c.ah) turn(c.a, XA);
        if (c.bh) turn(c.b, XB);
        // conjugation and alpha, each behind a wave-uniform branch
        if (c.ah) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c.a[t].y = flip(c.a[t].y);
        }
        if (c.bh != neg) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c.b[t].y = flip(c.b[t].y);
        }
        if (neg) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c.b[t].x = flip(c.b[t].x);
        }
        if (!one) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c.b[t] = cmul_i(c.alpha, c.b[t]);
        }
        if (c.left < 16) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * t + kq >= c.left) c.a[t] = c.b[t] = make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (4 * t >= c.left) break;                 // wave-uniform
            re = mfma64(c.a[t].x, c.b[t].x, re);
            im = mfma64(c.a[t].x, c.b[t].y, im);
            re = mfma64_nega(c.a[t].y, c.b[t].y, re);
            im = mfma64(c.a[t].y, c.b[t].x, im);
        }
    };
    advance();
    if (s < nt) {
        load(ch[0]);
        for (;;) {
            advance();
            bool more = s < nt;
            if (more) load(ch[1]);
            multiply(ch[0]);
            if (!more) break;
            advance();
            more = s < nt;
            if (more) load(ch[0]);
            multiply(ch[1]);
            if (!more) break;
        }
    }
    constexpr int kBe = offsetof(GemmOp, beta) / 4;
    const double2 beta = make_double2(OpRegs::real(o.head(kBe), o.head(kBe + 1)),
                                      OpRegs::real(o.head(kBe + 2), o.head(kBe + 3)));
    const int ldd = o.head(offsetof(GemmOp, ldd) / 4);
    const __amdgpu_buffer_rsrc_t rd = fused_rsrc(OpRegs::ptr(o.head(0), o.head(1)), m, n, ldd);
    static_assert(offsetof(GemmOp, D) == 0, "D first");
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
// instance 1.12 against 1.30 ms; 512 of them 3.3 against 3.0).
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
