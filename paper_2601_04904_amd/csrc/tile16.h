// Descriptors in lane registers and buffer addressing of 16 x 16 tiles, shared by the
// fused small-instance kernel and the small-launch product kernel, and the fused
// kernel's tile: one wave's, operands going from memory to the layout of
// v_mfma_f64_16x16x4 without workgroup barriers.
#pragma once
#include "gauss.h"
#include <cstddef>

namespace btsq {

// A product's descriptor in the registers of a wave: lane l holds dwords l and
// 64 + l of the GemmOp, so it is read in one latency and a field is one lane read.
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
        const int a = lane_of(w0, i & 63), b = lane_of(w1, i & 63);    // both, so that there is no branch
        return i < 64 ? a : b;
    }
    static __device__ inline double real(int lo, int hi) {
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    }
    static __device__ inline double2* ptr(int lo, int hi) {
        return (double2*)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    }
};
static_assert(sizeof(GemmOp) / 4 > 64 && sizeof(GemmOp) / 4 <= 128, "two dwords per lane");
static_assert((size_t)kInvMaxDim * kInvMaxDim * sizeof(double2) < (1u << 30), "32-bit offsets");

// Operands, C and D are addressed through raw buffer resources with 32-bit byte
// offsets; an offset past the record count (the operand's extent) reads as zero
// and is not written, so rows outside the product need no clamp.
__device__ inline __amdgpu_buffer_rsrc_t fused_rsrc(double2* base, int rows, int cols, int ld) {
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, ((rows - 1) * ld + cols) * 16, 0x00020000);
}
__device__ inline double2 load16(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
__device__ inline void store16(__amdgpu_buffer_rsrc_t r, int off, double2 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off, 0, 0);
}

// Operands that run along k in memory (A as stored, B^H) are read 16 k of a row by
// 16 lanes and turned through a piece of LDS of the wave's own (no barrier).
typedef double2 Turn[16][17];

__device__ inline void turn16(double2* v, Turn& X, int q, int kq) {
#pragma unroll
    for (int t = 0; t < 4; ++t) X[q][kq + 4 * t] = v[t];
    wave_lds_fence();
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = X[4 * t + kq][q];
    wave_lds_fence();                    // before the next chunk's writes
}

typedef float v4f __attribute__((ext_vector_type(4)));

// sum_t alpha_t op(A_t) op(B_t) over the 16 x 16 tile at (i0, j0), by one wave:
// register r is row lane/16 + 4 r of column lane%16.  The k range of every term is
// taken 16 at a time; the next chunk's loads (of the same or the next term) are issued
// before the current chunk's MFMAs.  Entries of A and B past k are cleared; rows and
// columns outside the product only reach entries that are not stored.
__device__ inline void tile16_sum(const OpRegs& o, int m, int n, int i0, int j0, int lane, Turn& XA, Turn& XB, v4d& re,
                                  v4d& im) {
    const int nt = o.head(offsetof(GemmOp, nterms) / 4);
    const int q = lane & 15, kq = lane >> 4;
    re = im = v4d{};
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
    auto flip = [](double v) {
        return __longlong_as_double(__double_as_longlong(v) ^ (long long)0x8000000000000000ull);
    };
    auto multiply = [&](Chunk& c) {
        const bool one = c.alpha.y == 0.0 && (c.alpha.x == 1.0 || c.alpha.x == -1.0);
        const bool neg = one && c.alpha.x < 0.0;
        if (!c.ah) turn16(c.a, XA, q, kq);
        if (c.bh) turn16(c.b, XB, q, kq);
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
}

// beta of a product from its descriptor
__device__ inline double2 op_beta(const OpRegs& o) {
    constexpr int kBe = offsetof(GemmOp, beta) / 4;
    return make_double2(OpRegs::real(o.head(kBe), o.head(kBe + 1)), OpRegs::real(o.head(kBe + 2), o.head(kBe + 3)));
}
__device__ inline double2* op_c(const OpRegs& o) {
    return OpRegs::ptr(o.head(offsetof(GemmOp, C) / 4), o.head(offsetof(GemmOp, C) / 4 + 1));
}
__device__ inline double2* op_d(const OpRegs& o) {
    static_assert(offsetof(GemmOp, D) == 0, "D first");
    return OpRegs::ptr(o.head(0), o.head(1));
}

}  // namespace btsq
