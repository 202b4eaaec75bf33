// Grouped complex block products on CDNA4 matrix cores.
//
// Every block update of the forward and backward sweeps is a dense complex
// product (or a short sum of them) on b x b, b x a and a x a blocks.  One
// launch executes a list of independent products, each cut into complex output
// tiles of the launch's shape (64 x 64, 64 x 32, 32 x 32, or 16 x 16 for small
// launches); a workgroup owns one tile of one product.
//
// FP64 path: v_mfma_f64_16x16x4 on the real and imaginary parts, four MFMAs per
// 16 x 16 x 4 complex block (an element is one 16-byte (re, im) pair in memory,
// LDS and registers, so both parts come with one read).
//
// What bounds it: the FP64 matrix rate (77.5 TFLOP/s measured with operands in
// registers).  On 32 products of 512 x 512 with distinct random operands the
// 64 x 64 tile runs at 69.6 TFLOP/s (493 us), on 16 of 1024 at 71.5; with the
// 4x4x4 instruction, A replicated over its blocks, and the memory instructions
// of a stage issued in blocks of their own it was 51 to 60 (two 256-thread
// workgroups per CU).  The accumulators must stay in plain VGPRs: in the
// accumulator half of the register file the compiler copies them in and out
// around every stage, which halves the rate of the 16x16x4 instruction (36
// against 77.5 TFLOP/s in a loop of it alone).
//
// Mixed path: complex arithmetic on real MFMA by a 2 x 2 real embedding.  A
// complex m x k matrix A stored as interleaved (re, im) is read as the real
// m x 2k matrix A', and op(B) (k x n complex) is expanded on the fly into the
// real 2k x 2n matrix
//     B''[2p+c][2j+d] = Re B[p][j]  (c == d),  Im B[p][j] (c=0,d=1),
//                       -Im B[p][j] (c=1,d=0)
// so that A' B'' is the interleaved complex product.  Operands rounded to FP32
// while staging into LDS, v_mfma_f32_16x16x4f32 with FP32 accumulation, the
// result added to the FP64 output in FP64.
#include "tile16.h"

namespace btsq {

constexpr int kBK = 16;          // complex k per LDS stage
constexpr int kThreads = 256;    // 4 waves, 2 x 2 over the tile

// a b, with the same roundings in every kernel
__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// Global pointer in the global address space (the C operand's loads).
#ifdef __HIP_DEVICE_COMPILE__
typedef const __attribute__((address_space(1))) double2* gptr_t;
#else
typedef const double2* gptr_t;
#endif

// Operand loads go through raw buffer resources, one per operand of the
// current term: a lane's load address is base + its own 32-bit byte offset +
// a wave-uniform scalar offset for the stage's k.  A lane whose row, column
// or k lies outside the operand gets the offset kOOB instead; the record
// count of every resource (the operand's extent in bytes, below 2^31) is
// smaller than that, so the hardware returns zeros for it without accessing
// memory.  For every other lane the byte offset plus the scalar offset stays
// inside the operand, so no access leaves it whether or not the hardware's
// range check counts the scalar offset.
constexpr unsigned kOOB = 0x80000000u;
constexpr int kRsrcWord3 = 0x00020000;   // raw buffer, 32-bit data format

__device__ inline __amdgpu_buffer_rsrc_t operand_rsrc(const double2* base, int rows, int cols, int ld) {
    const int extent = ((rows - 1) * ld + cols) * 16;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double2*>(base), (short)0, extent, kRsrcWord3);
}

__device__ inline double2 load_b128(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// What a stage's operands need between load and LDS: conjugation of A and
// B, and alpha (folded into B).  Taken from the term, so wave-uniform.
struct StageFlags {
    bool ah, bh;
    int akind;            // alpha: 0 general, 1 exactly +1, 2 exactly -1
    double2 alpha;
};

__device__ inline StageFlags term_flags(const GemmTerm& T) {
    StageFlags f;
    f.ah = T.flags & kTermAH;
    f.bh = T.flags & kTermBH;
    f.alpha = T.alpha;
    f.akind = T.alpha.y != 0.0 ? 0 : T.alpha.x == 1.0 ? 1 : T.alpha.x == -1.0 ? 2 : 0;
    return f;
}

// Addressing of one thread's loads for one product term, fixed over all k
// stages of the term: the byte offset of each load at k = 0 (kOOB when its
// A row or B column lies outside the matrix) and the bytes per unit of k.
// The term's flags, k and alpha come from the op list in global memory at a
// uniform address, so they are wave-uniform and the choices on them are
// scalar.
template <int BM, int BN>
struct TermAddr {
    static constexpr int NA = BM * kBK / kThreads;
    static constexpr int NB = BN * kBK / kThreads;
    __amdgpu_buffer_rsrc_t ra, rb;
    unsigned va[NA], vb[NB];
    int ska, skb;
    StageFlags f;
};

// Coordinates of load e (= tid + kThreads q) inside the stage tile: A (i, p)
// and B (j, p), chosen so that consecutive threads read consecutive memory.
template <int BM> __device__ inline int a_i(bool ah, int e) { return ah ? (e % BM) : (e / kBK); }
template <int BM> __device__ inline int a_p(bool ah, int e) { return ah ? (e / BM) : (e % kBK); }
template <int BN> __device__ inline int b_j(bool bh, int e) { return bh ? (e / kBK) : (e % BN); }
template <int BN> __device__ inline int b_p(bool bh, int e) { return bh ? (e % kBK) : (e / BN); }

// op(A) is m x k: stored k x m (A^H) or m x k; op(B) is k x n: stored n x k
// (B^H) or k x n.  Element (i, p) of op(A) sits at p lda + i or i lda + p,
// element (p, j) of op(B) at j ldb + p or p ldb + j.
template <int BM, int BN>
__device__ inline void term_setup(const GemmTerm& T, int m, int n, int i0, int j0, int tid,
                                  TermAddr<BM, BN>& ta) {
    const bool ah = T.flags & kTermAH, bh = T.flags & kTermBH;
    ta.f = term_flags(T);
    ta.ska = (ah ? T.lda : 1) * 16;
    ta.skb = (bh ? 1 : T.ldb) * 16;
    ta.ra = ah ? operand_rsrc(T.A, T.k, m, T.lda) : operand_rsrc(T.A, m, T.k, T.lda);
    ta.rb = bh ? operand_rsrc(T.B, n, T.k, T.ldb) : operand_rsrc(T.B, T.k, n, T.ldb);
#pragma unroll
    for (int q = 0; q < ta.NA; ++q) {
        const int e = tid + kThreads * q;
        const int gi = i0 + a_i<BM>(ah, e);
        const unsigned off = (unsigned)((ah ? gi : gi * T.lda) * 16 + a_p<BM>(ah, e) * ta.ska);
        ta.va[q] = gi < m ? off : kOOB;
    }
#pragma unroll
    for (int q = 0; q < ta.NB; ++q) {
        const int e = tid + kThreads * q;
        const int gj = j0 + b_j<BN>(bh, e);
        const unsigned off = (unsigned)((bh ? gj * T.ldb : gj) * 16 + b_p<BN>(bh, e) * ta.skb);
        ta.vb[q] = gj < n ? off : kOOB;
    }
}

// Raw operands of one stage in flight, and the flags of the term they belong to.
template <int BM, int BN>
struct Stage {
    static constexpr int NA = BM * kBK / kThreads;
    static constexpr int NB = BN * kBK / kThreads;
    double2 ra[NA], rb[NB];
    StageFlags f;
};

// Where the loads stand: the term, the largest k still inside it counted from
// the stage's first k (negative when no stage is left), and the scalar byte
// offsets of the stage.  All wave-uniform.
struct Fetch {
    int t, lim, soa, sob;
};

// Steps to the stage after the current one, setting up the next term that has
// any k when the current one ends.  The last stage of a term whose k is not a
// multiple of the stage depth switches the lanes past k to kOOB for good (the
// next term sets the offsets up again): lim - p < 0 exactly there, and every
// in-range offset is below 2^31, so with the sign bit set it is at least kOOB.
// Past the last term lim stays negative and every lane is switched off: the
// register set is then defined (all zeros) without any memory access, so the
// loads are issued unconditionally.  All other stages take no vector
// arithmetic here or in load_elem.
template <int BM, int BN>
__device__ inline void next_stage(const GemmTerm* terms, int nterms, int m, int n, int i0, int j0, int tid,
                                  Fetch& f, TermAddr<BM, BN>& ta, int step = kBK) {
    f.lim -= step;
    f.soa += step * ta.ska;
    f.sob += step * ta.skb;
    if (f.lim < 0) {
        f.soa = f.sob = 0;
        while (f.t < nterms) {
            if (++f.t == nterms) break;
            if (terms[f.t].k > 0) {
                f.lim = terms[f.t].k - 1;
                term_setup<BM, BN>(terms[f.t], m, n, i0, j0, tid, ta);
                break;
            }
        }
    }
    if (f.lim < kBK - 1) {
#pragma unroll
        for (int q = 0; q < ta.NA; ++q)
            ta.va[q] |= (unsigned)(f.lim - a_p<BM>(ta.f.ah, tid + kThreads * q)) & kOOB;
#pragma unroll
        for (int q = 0; q < ta.NB; ++q)
            ta.vb[q] |= (unsigned)(f.lim - b_p<BN>(ta.f.bh, tid + kThreads * q)) & kOOB;
    }
}

// Load e of a stage (A's first, then B's).
template <int BM, int BN>
__device__ inline void load_elem(const TermAddr<BM, BN>& ta, const Fetch& f, Stage<BM, BN>& st, int e) {
    constexpr int NA = Stage<BM, BN>::NA;
    // wave-uniform by construction; readfirstlane lets the compiler keep them in SGPRs
    if (e < NA) st.ra[e] = load_b128(ta.ra, ta.va[e], __builtin_amdgcn_readfirstlane(f.soa));
    else st.rb[e - NA] = load_b128(ta.rb, ta.vb[e - NA], __builtin_amdgcn_readfirstlane(f.sob));
}

template <int BM, int BN>
__device__ inline void load_stage(const TermAddr<BM, BN>& ta, const Fetch& f, Stage<BM, BN>& st) {
#pragma unroll
    for (int e = 0; e < Stage<BM, BN>::NA + Stage<BM, BN>::NB; ++e) load_elem<BM, BN>(ta, f, st, e);
    st.f = ta.f;
}

__device__ inline double flip_sign(double v, unsigned long long mask) {
    return __longlong_as_double(__double_as_longlong(v) ^ (long long)mask);
}

// A general alpha is multiplied into B; +1 and -1 need no arithmetic (below).
template <int BM, int BN>
__device__ inline void scale_stage(Stage<BM, BN>& st) {
    if (st.f.akind == 0) {
#pragma unroll
        for (int q = 0; q < Stage<BM, BN>::NB; ++q) {
            if (st.f.bh) st.rb[q].y = -st.rb[q].y;
            st.rb[q] = cmul(st.f.alpha, st.rb[q]);
            if (st.f.bh) st.rb[q].y = -st.rb[q].y;
        }
    }
}

// A stage to LDS (out-of-range values are already zero), rounded to FP32 in the mixed
// path.  Conjugation and alpha = -1 are sign flips with wave-uniform masks.
__device__ inline void round_to(float2& to, double2 v) { to = make_float2((float)v.x, (float)v.y); }
__device__ inline void round_to(double2& to, double2 v) { to = v; }
template <int BM, int BN, class CT>
__device__ inline void store_stage(int tid, const Stage<BM, BN>& st, CT (*As)[BM + 1], CT (*Bs)[BN + 1]) {
    constexpr unsigned long long kSign = 0x8000000000000000ull;
    const StageFlags& f = st.f;
    const bool neg = f.akind == 2;
#pragma unroll
    for (int e = 0; e < Stage<BM, BN>::NA; ++e) {
        const int x = tid + kThreads * e;
        double2 v = st.ra[e];
        v.y = flip_sign(v.y, f.ah ? kSign : 0ull);
        round_to(As[a_p<BM>(f.ah, x)][a_i<BM>(f.ah, x)], v);
    }
#pragma unroll
    for (int e = 0; e < Stage<BM, BN>::NB; ++e) {
        const int x = tid + kThreads * e;
        double2 v = st.rb[e];
        v.x = flip_sign(v.x, neg ? kSign : 0ull);
        v.y = flip_sign(v.y, f.bh != neg ? kSign : 0ull);
        round_to(Bs[b_p<BN>(f.bh, x)][b_j<BN>(f.bh, x)], v);
    }
}

// FP64 path: where the elements of a stage go in an LDS buffer (byte offsets;
// they depend on which operands are read transposed only, so they are set up
// again only when that changes).
template <int BM, int BN>
struct LdsPlace {
    static constexpr int NA = Stage<BM, BN>::NA;
    static constexpr int NB = Stage<BM, BN>::NB;
    unsigned a[NA], b[NB];
    int layout = -1;
    __device__ inline void set(const StageFlags& f, int tid) {
        const int want = (f.ah ? 1 : 0) | (f.bh ? 2 : 0);
        if (want == layout) return;
        layout = want;
#pragma unroll
        for (int e = 0; e < NA; ++e) {
            const int x = tid + kThreads * e;
            a[e] = (a_p<BM>(f.ah, x) * (BM + 1) + a_i<BM>(f.ah, x)) * 16;
        }
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int x = tid + kThreads * e;
            b[e] = (b_p<BN>(f.bh, x) * (BN + 1) + b_j<BN>(f.bh, x)) * 16;
        }
    }
    __device__ inline void store(const Stage<BM, BN>& st, double2 (*As)[BM + 1], double2 (*Bs)[BN + 1], int e) const {
        if (e < NA) *reinterpret_cast<double2*>(reinterpret_cast<char*>(As) + a[e]) = st.ra[e];
        else *reinterpret_cast<double2*>(reinterpret_cast<char*>(Bs) + b[e - NA]) = st.rb[e - NA];
    }
};

// Conjugates what the stage's operands take as H.  (alpha = -1 costs nothing
// here: the accumulators change sign between terms instead.)
template <int BM, int BN>
__device__ inline void conj_stage(Stage<BM, BN>& st) {
    constexpr unsigned long long kSign = 0x8000000000000000ull;
    if (st.f.ah) {
#pragma unroll
        for (int q = 0; q < Stage<BM, BN>::NA; ++q) st.ra[q].y = flip_sign(st.ra[q].y, kSign);
    }
    if (st.f.bh) {
#pragma unroll
        for (int q = 0; q < Stage<BM, BN>::NB; ++q) st.rb[q].y = flip_sign(st.rb[q].y, kSign);
    }
}

// The accumulators of one wave and what it does with them: start (beta C),
// the multiply-adds of one LDS stage, and the store of its part of the tile.
// The 4 waves of a workgroup split the BM x BN complex tile 2 x 2.
template <bool MIXED, int BM, int BN> struct WaveTile;

// FP64: v_mfma_f64_16x16x4 on planar operands.  A lane reads its entry of A
// and B as one (re, im) pair, and a 16 x 16 x 4 complex block is
//     Re += Re A Re B - Im A Im B,   Im += Re A Im B + Im A Re B,
// four MFMAs on the two components; the minus sign is the instruction's
// negation of its first operand.  Layout (measured on gfx950): A[l%16][l/16],
// B[l/16][l%16], D row l/16 + 4r, column l%16 in register r.
template <int BM, int BN>
struct WaveTile<false, BM, BN> {
    static constexpr int RA = BM / 32;    // 16-row blocks of the wave
    static constexpr int CB = BN / 32;    // 16-column blocks of the wave
    v4d re[RA][CB], im[RA][CB];

    static __device__ inline v4d mfma(double a, double b, v4d c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline v4d mfma_nega(double a, double b, v4d c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
    }

    // Starts at beta C (C read before any of D is written, so C may be D), so
    // the epilogue only stores.
    __device__ inline void init(const GemmOp* op, int m, int n, int i0, int j0, int lane) {
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b) re[a][b] = im[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
        if (!op->C) return;
        const gptr_t Cp = (gptr_t)op->C;
        const int ldc = op->ldc;
        const double2 beta = op->beta;
        double2 cv[RA][CB][4];
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = min(i0 + a * 16 + 4 * r + (lane >> 4), m - 1);
                    const int col = min(j0 + b * 16 + (lane & 15), n - 1);
                    cv[a][b][r] = Cp[(size_t)row * ldc + col];
                }
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double2 c = cv[a][b][r];
                    const double2 v = cmul(beta, c);
                    re[a][b][r] = v.x;
                    im[a][b][r] = v.y;
                }
    }

    __device__ inline void negate() {
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    re[a][b][r] = -re[a][b][r];
                    im[a][b][r] = -im[a][b][r];
                }
    }

    // The wave's entries of one 4-deep k step: 16 x 4 blocks of A, 4 x 16 of B.
    struct Frag {
        double2 a[RA], b[CB];
    };
    static constexpr int kReads = RA + CB;
    static constexpr int kMfma = 4 * RA * CB;

    // read e of the fragment of step kk
    static __device__ inline void read(Frag& f, const double2 (*As)[BM + 1], const double2 (*Bs)[BN + 1], int r0,
                                       int c0, int lane, int kk, int e) {
        const int p = 4 * kk + (lane >> 4), q = lane & 15;
        if (e < RA) f.a[e] = As[p][r0 + e * 16 + q];
        else f.b[e - RA] = Bs[p][c0 + (e - RA) * 16 + q];
    }

    // The MFMAs of one step, with hook(i) run after the i-th: reads, loads and
    // LDS stores put there issue while the matrix core works (64 cycles per
    // MFMA), where in a block of their own they would leave it idle.
    template <class H>
    __device__ inline void step(const Frag& f, H hook) {
#pragma unroll
        for (int i = 0; i < kMfma; ++i) {
            const int half = i / (2 * RA * CB), j = i % (2 * RA * CB);
            const int b = j / (2 * RA), a = (j / 2) % RA;
            if (half == 0) {
                if (j & 1) im[a][b] = mfma(f.a[a].x, f.b[b].y, im[a][b]);
                else re[a][b] = mfma(f.a[a].x, f.b[b].x, re[a][b]);
            } else {
                if (j & 1) im[a][b] = mfma(f.a[a].y, f.b[b].x, im[a][b]);
                else re[a][b] = mfma_nega(f.a[a].y, f.b[b].y, re[a][b]);
            }
            hook(i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    __device__ inline void store(const GemmOp* op, int m, int n, int i0, int j0, int lane) {
        double2* D = op->D;
        const int ldd = op->ldd;
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = i0 + a * 16 + 4 * r + (lane >> 4);
                    const int col = j0 + b * 16 + (lane & 15);
                    if (row < m && col < n) D[(size_t)row * ldd + col] = make_double2(re[a][b][r], im[a][b][r]);
                }
    }
};

// Mixed: operands rounded to FP32 in LDS, v_mfma_f32_16x16x4f32 on the 2 x 2
// real embedding above, FP32 accumulation, beta C added in FP64 at the end.
template <int BM, int BN>
struct WaveTile<true, BM, BN> {
    static constexpr int RG = BM / 32;    // 16-row blocks of the wave
    static constexpr int NI = BN / 16;    // 16-column blocks of the wave (real columns)
    v4f acc[RG][NI];

    __device__ inline void init(const GemmOp*, int, int, int, int, int) {
#pragma unroll
        for (int a = 0; a < RG; ++a)
#pragma unroll
            for (int b = 0; b < NI; ++b) acc[a][b] = v4f{};
    }

    __device__ inline void stage(const float2 (*As)[BM + 1], const float2 (*Bs)[BN + 1], int r0, int c0, int lane) {
        const int cA = (lane >> 4) & 1;   // real k within the pair: 0 = re part of A, 1 = im part
        const int pOff = lane >> 5;       // complex k offset within the 4-wide real k step
        const int r16 = lane & 15;
        const int d = lane & 1;           // output component of this lane's B'' column
        const int negB = cA == 1 && d == 0 ? (int)0x80000000u : 0;
#pragma unroll
        for (int kk = 0; kk < kBK / 2; ++kk) {
            const int p = 2 * kk + pOff;
            float av[RG], bv[NI];
            // one component read per operand: A' takes component cA, B'' takes
            // component cA ^ d, negated for (cA, d) = (1, 0)
#pragma unroll
            for (int g = 0; g < RG; ++g)
                av[g] = reinterpret_cast<const float*>(&As[p][r0 + g * 16 + r16])[cA];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const float v = reinterpret_cast<const float*>(&Bs[p][c0 + ((ni * 16 + r16) >> 1)])[cA ^ d];
                bv[ni] = __int_as_float(__float_as_int(v) ^ negB);
            }
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[g][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[g], bv[ni], acc[g][ni], 0, 0, 0);
        }
    }

    // Lane holds real column lane%16 (component lane%2 of complex column
    // lane%16 / 2) of rows 4 (lane/16) + r of each 16-row block.
    __device__ inline void store(const GemmOp* op, int m, int n, int i0, int j0, int lane) {
        double* D = reinterpret_cast<double*>(op->D);
        const int ldd = op->ldd, ldc = op->ldc;
        const double2 beta = op->beta;
        const int d = lane & 1, rq = 4 * (lane >> 4), cq = lane & 15;
        double2 cv[RG][NI][4];
        if (op->C) {
            // all C loads first (clamped, unconditional), then the stores
            const gptr_t Cp = (gptr_t)op->C;
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = min(i0 + g * 16 + rq + r, m - 1);
                        const int col = min(j0 + ((ni * 16 + cq) >> 1), n - 1);
                        cv[g][ni][r] = Cp[(size_t)row * ldc + col];
                    }
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        asm volatile("" : "+v"(cv[g][ni][r].x), "+v"(cv[g][ni][r].y));
        }
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = i0 + g * 16 + rq + r;
                    const int col = j0 + ((ni * 16 + cq) >> 1);
                    double v = (double)acc[g][ni][r];
                    if (op->C) {
                        const double2 c = cmul(beta, cv[g][ni][r]);
                        v += d ? c.y : c.x;
                    }
                    if (row < m && col < n) D[2 * ((size_t)row * ldd + col) + d] = v;
                }
    }
};

// One workgroup computes a BM x BN complex tile of one product.
template <bool MIXED, int BM, int BN>
__global__ __launch_bounds__(kThreads)
void zgemm_grouped(const GemmOp* __restrict__ ops, const TileEntry* __restrict__ order) {
    typedef typename std::conditional<MIXED, float2, double2>::type CT;     // element in LDS
    __shared__ CT As[2][kBK][BM + 1];
    __shared__ CT Bs[2][kBK][BN + 1];

    // which tile of which product: from the launch's order, or all tiles of the only
    // product
    const TileEntry at = order ? order[blockIdx.x] : tile_entry(0, xcd_remap(blockIdx.x, gridDim.x));
    if (at == kNoTile) return;
    const GemmOp* op = ops + (uint32_t)(at >> 32);
    const int local = (int)(uint32_t)at;
    const int m = op->m, n = op->n, nterms = op->nterms;
    const int tm = local / op->tiles_n, tn = local - tm * op->tiles_n;
    const int i0 = tm * BM, j0 = tn * BN;
    const int tid = threadIdx.x;
    const GemmTerm* terms = op->t;     // uniform: read with scalar loads

    const int lane = tid & 63, wave = tid >> 6;
    const int r0 = (wave & 1) * (BM / 2), c0 = (wave >> 1) * (BN / 2);   // the wave's part of the tile
    WaveTile<MIXED, BM, BN> wt;
    wt.init(op, m, n, i0 + r0, j0 + c0, lane);

    // Stages are the terms' k ranges in order, kBK at a time.  Two register
    // sets hold the raw operands of the next two stages: while the stage in LDS
    // is multiplied, the loads of the stage after next are issued into one set
    // and the other set (loaded during the stage before) goes to the other LDS
    // buffer.
    Stage<BM, BN> st[2];
    TermAddr<BM, BN> ta;
    ta.ska = ta.skb = 0;
    Fetch fe{-1, -1, 0, 0};
    next_stage<BM, BN>(terms, nterms, m, n, i0, j0, tid, fe, ta, 0);
    bool cur = fe.lim >= 0, fly = false;
    if (cur) {
        load_stage<BM, BN>(ta, fe, st[0]);
        next_stage<BM, BN>(terms, nterms, m, n, i0, j0, tid, fe, ta);
        fly = fe.lim >= 0;
        load_stage<BM, BN>(ta, fe, st[1]);
        scale_stage<BM, BN>(st[0]);
    }
    constexpr int NL = Stage<BM, BN>::NA + Stage<BM, BN>::NB;

    if constexpr (MIXED) {
        if (cur) store_stage<BM, BN>(tid, st[0], As[0], Bs[0]);
        __syncthreads();
        // one stage: X = register set in flight (the next stage), Y = free set,
        // X - 1 the parity of the LDS buffer multiplied
        auto step = [&](auto xs) {
            constexpr int X = decltype(xs)::value, Y = 1 - X, buf = Y;
            next_stage<BM, BN>(terms, nterms, m, n, i0, j0, tid, fe, ta);
            load_stage<BM, BN>(ta, fe, st[Y]);
            // keep the order issue -> MFMAs -> conversion of the next stage, so
            // that the loads in flight have a whole stage of MFMAs to land
            __builtin_amdgcn_sched_barrier(0);
            wt.stage(As[buf], Bs[buf], r0, c0, lane);
            __builtin_amdgcn_sched_barrier(0);
            // unconditional like the loads: without a next stage st[X] holds
            // zeros from kOOB loads, stored to the buffer no later stage reads
            scale_stage<BM, BN>(st[X]);
            store_stage<BM, BN>(tid, st[X], As[buf ^ 1], Bs[buf ^ 1]);
            __syncthreads();
            cur = fly;
            fly = fe.lim >= 0;
        };
        while (cur) {
            step(std::integral_constant<int, 1>{});
            if (!cur) break;
            step(std::integral_constant<int, 0>{});
        }
    } else {
        // FP64: memory and LDS instructions run in the shadow of the MFMAs (64
        // cycles each).  Vector arithmetic does not: every place between two
        // MFMAs with any of it cost about one MFMA (a stage with address and
        // sign arithmetic at its 8 loads and 8 stores took 5600 cycles for 4096
        // of MFMAs), so the stage has one, which conjugates.  The first three k steps
        // of a stage carry the loads of the stage after next and the LDS stores
        // of the next one; the barrier comes before the last step, whose
        // operands are in registers by then, so that step's MFMAs cover the
        // first reads of the next stage.
        typedef WaveTile<MIXED, BM, BN> WT;
        constexpr int KS = kBK / 4, NR = WT::kReads, NM = WT::kMfma;
        typename WT::Frag fr[2];
        LdsPlace<BM, BN> place;
        bool neg = false, neg_lds = false;    // sign of the accumulators / of the stage in LDS
        if (cur) {
            place.set(st[0].f, tid);
            neg_lds = st[0].f.akind == 2;
            conj_stage<BM, BN>(st[0]);
#pragma unroll
            for (int e = 0; e < NL; ++e) place.store(st[0], As[0], Bs[0], e);
        }
        __syncthreads();
        if (cur) {
#pragma unroll
            for (int e = 0; e < NR; ++e) WT::read(fr[0], As[0], Bs[0], r0, c0, lane, 0, e);
        }
        auto step = [&](auto xs) {
            constexpr int X = decltype(xs)::value, Y = 1 - X, buf = Y;
            next_stage<BM, BN>(terms, nterms, m, n, i0, j0, tid, fe, ta);
            if (neg_lds != neg) {
                neg = neg_lds;
                wt.negate();
            }
            neg_lds = st[X].f.akind == 2;
            place.set(st[X].f, tid);
            st[Y].f = ta.f;
            __builtin_amdgcn_sched_barrier(0);
            auto kstep = [&](auto ks) {
                constexpr int kk = decltype(ks)::value;
                if constexpr (kk == KS - 1) {
                    __syncthreads();
                    wt.step(fr[kk & 1], [&](int i) {
                        if (i < NR) WT::read(fr[(kk + 1) & 1], As[buf ^ 1], Bs[buf ^ 1], r0, c0, lane, 0, i);
                    });
                } else {
                    if constexpr (kk == 1) {
                        scale_stage<BM, BN>(st[X]);
                        conj_stage<BM, BN>(st[X]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // after MFMA i: the next step's reads first; load e at slot
                    // (e + 1/2) / NL of the three steps, store e at e / NL of the
                    // last two
                    wt.step(fr[kk & 1], [&](int i) {
                        if (i < NR) WT::read(fr[(kk + 1) & 1], As[buf], Bs[buf], r0, c0, lane, kk + 1, i);
                        const int slot = kk * NM + i;
#pragma unroll
                        for (int e = 0; e < NL; ++e) {
                            if ((2 * e + 1) * (KS - 1) * NM / (2 * NL) == slot) load_elem<BM, BN>(ta, fe, st[Y], e);
                            if (NM + e * (KS - 2) * NM / NL == slot) place.store(st[X], As[buf ^ 1], Bs[buf ^ 1], e);
                        }
                    });
                }
            };
            [&]<int... K>(std::integer_sequence<int, K...>) {
                (kstep(std::integral_constant<int, K>{}), ...);
            }(std::make_integer_sequence<int, KS>{});
            cur = fly;
            fly = fe.lim >= 0;
        };
        while (cur) {
            step(std::integral_constant<int, 1>{});
            if (!cur) break;
            step(std::integral_constant<int, 0>{});
        }
        if (neg) wt.negate();
    }

    wt.store(op, m, n, i0 + r0, j0 + c0, lane);
}

// Launches with at most about one larger tile per CU (kSmallShape): one 16 x 16 tile per
// workgroup, four times the workgroups of 32 x 32 tiles.  What is left is the latency of
// the launch, of the descriptor (read in one go into the lanes of a wave) and of the first
// loads, then the chain of sums of one entry.  The waves share the tile's entries and
// not its k: v_mfma_f64_4x4x4 with A replicated over its four blocks is a 4-row x
// 16-column x 4-k product (A[lane%4][lane/16], B[lane/16][lane%16], D row lane/16,
// column lane%16), a quarter of the chain of the 16x16x4 instruction at the same rate, and
// both round as an ascending chain of fused multiply-adds (measured: no difference in
// 512000 sums of 64), so a product has the same bits in every shape and does not depend
// on what else is in its launch.  Mixed: the real embedding of the larger tiles, two waves
// of 8 columns.
// Against 32 x 32 tiles, us: 1 product of 32 4.1 -> 3.4, of 64 5.6 -> 4.0, of 128 8.3 ->
// 5.1, of 256 13.4 -> 7.7, 3 of 192 11.2 -> 9.4 (mixed 5.3 -> 3.5, 6.7 -> 4.3, 9.5 -> 5.6,
// 15.4 -> 8.6, 12.6 -> 9.0).  A wave per part of k, as an order of its own, would take 4.7
// and 6.9 us for one product of 128 and 256.
//
// G: chunks of kBK k's held in LDS at a time, all of whose loads are issued: 8, or as many
// as the longest term of the launch fills (8 for one product of 32: 4.2 us).
template <bool MIXED, int G>
__global__ __launch_bounds__(kThreads)
void zgemm_small(const GemmOp* __restrict__ ops, const TileEntry* __restrict__ order) {
    typedef typename std::conditional<MIXED, float2, double2>::type CT;
    __shared__ CT As[G][kBK][17], Bs[G][kBK][17];
    const TileEntry at = order ? order[blockIdx.x] : tile_entry(0, blockIdx.x);
    if (at == kNoTile) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const OpRegs o(ops[(uint32_t)(at >> 32)], lane);
    const int tile = (int)(uint32_t)at;
    const int m = o.head(offsetof(GemmOp, m) / 4), n = o.head(offsetof(GemmOp, n) / 4);
    const int nt = o.head(offsetof(GemmOp, nterms) / 4);
    const int tn = (n + 15) >> 4, ti = tile / tn;
    const int i0 = ti * 16, j0 = (tile - ti * tn) * 16;

    // this lane's entries of the tile: FP64 one of the wave's 4 rows, mixed 4 rows of one
    // component of a column of waves 0 and 1
    constexpr int NE = MIXED ? 4 : 1;
    const bool mine = !MIXED || wave < 2;
    const int row = i0 + (MIXED ? 4 * (lane >> 4) : 4 * wave + (lane >> 4));
    const int col = j0 + (MIXED ? 8 * wave + ((lane & 15) >> 1) : lane & 15);
    double2* C = op_c(o);
    double2 cv[NE];
    if (C && mine) {
        const int ldc = o.head(offsetof(GemmOp, ldc) / 4);
#pragma unroll
        for (int r = 0; r < NE; ++r)
            cv[r] = load16(fused_rsrc(C, m, n, ldc), (__mul24(row + r, ldc) + col) * 16);
    }

    // A step is up to G chunks of one term, multiplied from LDS while the loads of the
    // next one are in flight.
    double2 av[G], bv[G];
    TermAddr<16, 16> ta;
    int s = -1, lim = -1, soa = 0, sob = 0;      // term, largest k in it from the step's first on, scalar offsets
    const int ldd = o.head(offsetof(GemmOp, ldd) / 4);
    const __amdgpu_buffer_rsrc_t rd = fused_rsrc(op_d(o), m, n, ldd);
    ta.ra = ta.rb = rd;                          // (without any term: nothing is read through them)
    ta.va[0] = ta.vb[0] = kOOB;
    ta.ska = ta.skb = 0;
    ta.f = StageFlags{};
    // Loads the next step; returns how many chunks it has.  Entries
    // past k, and everything past the last term, are switched off by their offset: the
    // loads are unconditional, since a register loaded in a branch is waited for at its
    // end.
    auto load = [&]() {
        lim -= G * kBK;
        soa += G * kBK * ta.ska;
        sob += G * kBK * ta.skb;
        if (lim < 0) {
            soa = sob = 0;
            while (s < nt && ++s < nt) {
                GemmTerm T;
                T.k = o.term(s, offsetof(GemmTerm, k) / 4);
                if (T.k <= 0) continue;
                T.A = OpRegs::ptr(o.term(s, 0), o.term(s, 1));
                T.B = OpRegs::ptr(o.term(s, 2), o.term(s, 3));
                T.lda = o.term(s, offsetof(GemmTerm, lda) / 4);
                T.ldb = o.term(s, offsetof(GemmTerm, ldb) / 4);
                T.flags = o.term(s, offsetof(GemmTerm, flags) / 4);
                constexpr int kAl = offsetof(GemmTerm, alpha) / 4;
                T.alpha = make_double2(OpRegs::real(o.term(s, kAl), o.term(s, kAl + 1)),
                                       OpRegs::real(o.term(s, kAl + 2), o.term(s, kAl + 3)));
                term_setup<16, 16>(T, m, n, i0, j0, tid, ta);
                lim = T.k - 1;
                break;
            }
        }
        const int pa = a_p<16>(ta.f.ah, tid), pb = b_p<16>(ta.f.bh, tid);
#pragma unroll
        for (int c = 0; c < G; ++c) {
            const int left = lim - c * kBK;
            av[c] = load_b128(ta.ra, ta.va[0] | ((unsigned)(left - pa) & kOOB),
                                   __builtin_amdgcn_readfirstlane(left < 0 ? 0 : soa + c * kBK * ta.ska));
            bv[c] = load_b128(ta.rb, ta.vb[0] | ((unsigned)(left - pb) & kOOB),
                                   __builtin_amdgcn_readfirstlane(left < 0 ? 0 : sob + c * kBK * ta.skb));
        }
        return lim < 0 ? 0 : min(lim / kBK + 1, G);
    };
    // Operands as they are in memory but for conjugation and a general alpha; alpha = -1 is
    // a change of the accumulators' sign.
    unsigned pa = 0, pb = 0;                     // this thread's places in a chunk of As, Bs
    int layout = -1;
    bool neg = false, neg_lds = false;           // sign of the accumulators / of the step in LDS
    auto to_lds = [&](int g) {
        const int want = (ta.f.ah ? 1 : 0) | (ta.f.bh ? 2 : 0);
        if (want != layout) {
            layout = want;
            pa = (a_p<16>(ta.f.ah, tid) * 17 + a_i<16>(ta.f.ah, tid)) * sizeof(CT);
            pb = (b_p<16>(ta.f.bh, tid) * 17 + b_j<16>(ta.f.bh, tid)) * sizeof(CT);
        }
        neg_lds = ta.f.akind == 2;
#pragma unroll
        for (int c = 0; c < G; c += 2) {
            if (c >= 2 && c >= g) continue;
            Stage<16, 16> x[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                // not before here: earlier, it would wait for the loads
                asm volatile("" : "+v"(av[c + e].x), "+v"(av[c + e].y), "+v"(bv[c + e].x), "+v"(bv[c + e].y));
                x[e].ra[0] = av[c + e];
                x[e].rb[0] = bv[c + e];
                x[e].f = ta.f;
            }
            if (want != 0 || ta.f.akind == 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    scale_stage<16, 16>(x[e]);
                    conj_stage<16, 16>(x[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                round_to(*reinterpret_cast<CT*>(reinterpret_cast<char*>(As[c + e]) + pa), x[e].ra[0]);
                round_to(*reinterpret_cast<CT*>(reinterpret_cast<char*>(Bs[c + e]) + pb), x[e].rb[0]);
            }
        }
    };

    // accumulators: re, im of the lane's entry, or (mixed) its four entries' component
    double re = 0.0, im = 0.0;
    v4f acc = {};
    if constexpr (!MIXED) {
        if (C) {
            const double2 v = cmul(op_beta(o), cv[0]);
            re = v.x;
            im = v.y;
        }
    }
    auto negate = [&]() {
        re = -re;
        im = -im;
        if constexpr (MIXED) acc = -acc;
    };
    // A chunk's entries are read while the one before is multiplied (past g: whatever is
    // there, not used).  KS instructions of 4 real or (mixed) 2 complex k's.
    auto multiply = [&](int g) {
        constexpr int KS = MIXED ? kBK / 2 : kBK / 4;
        typedef typename std::conditional<MIXED, float, double2>::type Entry;
        Entry fa[2][KS], fb[2][KS];
        const int cA = (lane >> 4) & 1, d = lane & 1;          // mixed: as in the larger tiles
        const int sign = cA == 1 && d == 0 ? (int)0x80000000u : 0;
        auto read = [&](int c) {
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) {
                if constexpr (MIXED) {
                    const int p = 2 * kk + (lane >> 5);
                    fa[c & 1][kk] = reinterpret_cast<const float*>(&As[c][p][lane & 15])[cA];
                    fb[c & 1][kk] = reinterpret_cast<const float*>(&Bs[c][p][8 * wave + ((lane & 15) >> 1)])[cA ^ d];
                } else {
                    fa[c & 1][kk] = As[c][4 * kk + (lane >> 4)][4 * wave + (lane & 3)];
                    fb[c & 1][kk] = Bs[c][4 * kk + (lane >> 4)][lane & 15];
                }
            }
        };
        if (!mine) return;
        read(0);
#pragma unroll
        for (int c = 0; c < G; ++c) {
            if (c < g) {
                if (c + 1 < G) read(c + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    const Entry a = fa[c & 1][kk], b = fb[c & 1][kk];
                    if constexpr (MIXED) {
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, __int_as_float(__float_as_int(b) ^ sign), acc, 0, 0, 0);
                    } else {
                        re = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, b.x, re, 0, 0, 0);
                        im = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, b.y, im, 0, 0, 0);
                        re = __builtin_amdgcn_mfma_f64_4x4x4f64(a.y, b.y, re, 0, 0, 1);
                        im = __builtin_amdgcn_mfma_f64_4x4x4f64(a.y, b.x, im, 0, 0, 0);
                    }
                }
            }
        }
    };
    int cur = load();
    to_lds(cur);
    __syncthreads();
    while (cur > 0) {
        if (neg != neg_lds) {
            neg = neg_lds;
            negate();
        }
        const int next = load();
        multiply(cur);
        __syncthreads();
        if (next > 0) {
            to_lds(next);
            __syncthreads();
        }
        cur = next;
    }
    if (neg) negate();

    if constexpr (MIXED) {
        if (mine && col < n) {
            const int d = lane & 1;
            const double2 beta = op_beta(o);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double v = (double)acc[r];
                if (C) {
                    const double2 c = cmul(beta, cv[r]);
                    v += d ? c.y : c.x;
                }
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rd, (__mul24(row + r, ldd) + col) * 16 + 8 * d, 0, 0);
            }
        }
    } else {
        if (col < n) store16(rd, (__mul24(row, ldd) + col) * 16, make_double2(re, im));
    }
}

// Tile shapes of the grouped product (complex rows x complex columns).
// Every op of a launch is tiled with the launch's shape: tiles_n of the ops and
// the launch's tile order are those of that shape.
struct TileShape { int bm, bn; };
constexpr TileShape kShapes[kGemmShapes + 1] = {{32, 32}, {64, 32}, {64, 64}, {16, 16}};    // last: kSmallShape

int gemm_shape_bm(int shape) { return kShapes[shape].bm; }
int gemm_shape_bn(int shape) { return kShapes[shape].bn; }
int gemm_tiles_shape(int m, int n, int shape) {
    return ((m + kShapes[shape].bm - 1) / kShapes[shape].bm) * ((n + kShapes[shape].bn - 1) / kShapes[shape].bn);
}
int gemm_tiles_n_shape(int n, int shape) { return (n + kShapes[shape].bn - 1) / kShapes[shape].bn; }

template <bool MIXED>
static void launch_mixed(const GemmOp* d_ops, const TileEntry* d_order, int grid, int shape, int maxk, hipStream_t s) {
    switch (shape) {
        case 0: hipLaunchKernelGGL((zgemm_grouped<MIXED, 32, 32>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order); break;
        case 1: hipLaunchKernelGGL((zgemm_grouped<MIXED, 64, 32>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order); break;
        case kSmallShape:
            if (maxk <= 2 * kBK) hipLaunchKernelGGL((zgemm_small<MIXED, 2>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order);
            else if (maxk <= 4 * kBK) hipLaunchKernelGGL((zgemm_small<MIXED, 4>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order);
            else hipLaunchKernelGGL((zgemm_small<MIXED, 8>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order);
            break;
        default: hipLaunchKernelGGL((zgemm_grouped<MIXED, 64, 64>), dim3(grid), dim3(kThreads), 0, s, d_ops, d_order); break;
    }
}

// d_order: the launch's tile order (grid entries, gemm_tile_order), or null for a
// single product, whose tiles then are the grid.  maxk: the largest k of a term.
hipError_t launch_gemm_shape(const GemmOp* d_ops, const TileEntry* d_order, int grid, bool mixed, int shape, int maxk,
                             hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    if (shape < 0 || shape > kSmallShape) return hipErrorInvalidValue;
    if (mixed) launch_mixed<true>(d_ops, d_order, grid, shape, maxk, s);
    else launch_mixed<false>(d_ops, d_order, grid, shape, maxk, s);
    return hipGetLastError();
}

}  // namespace btsq
