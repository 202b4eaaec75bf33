// Gauss-Jordan elimination of column groups on FP64 matrix cores, shared by the
// panel-per-launch inverse and the one-workgroup inverse of small blocks.
#pragma once
#include "common.h"
#include "cplx.h"
#include <type_traits>
#include <utility>

namespace btsq {

constexpr int kGrp = 4;     // columns eliminated between two block updates

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ inline v4d mfma64(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline v4d mfma64_nega(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
}

// Between LDS writes and reads of the same places by different lanes of one wave: the
// wave's LDS instructions complete in order, so nothing waits, but per lane the
// addresses differ and the compiler would be free to change the order.
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Value of a double in lane src (wave-uniform), in every lane.
__device__ inline double lane_value(double x, int src) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, src);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), src);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double2 lane_value(double2 x, int src) {
    return make_double2(lane_value(x.x, src), lane_value(x.y, src));
}

// 4 x 4 transpose of (lane group l/16, register): v[c] of lane group i and v[i]
// of lane group c change places.
__device__ inline void swap_rows(double& a, double& b, bool halves) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32), yl = (unsigned)y, yh = (unsigned)(y >> 32);
    const auto l = halves ? __builtin_amdgcn_permlane32_swap(xl, yl, false, false)
                          : __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = halves ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false)
                          : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    a = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0]));
    b = __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}
__device__ inline void transpose4(double2* v) {
    swap_rows(v[0].x, v[2].x, true);
    swap_rows(v[0].y, v[2].y, true);
    swap_rows(v[1].x, v[3].x, true);
    swap_rows(v[1].y, v[3].y, true);
    swap_rows(v[0].x, v[1].x, false);
    swap_rows(v[0].y, v[1].y, false);
    swap_rows(v[2].x, v[3].x, false);
    swap_rows(v[2].y, v[3].y, false);
}

// The block of a panel workgroup: a wave's NRB row blocks in accumulator layout.
template <int NRB>
struct PanelBlock {
    v4d re[NRB], im[NRB];

    // Row m of block b, in the lanes that ask for it, to out[column]; then cleared.
    __device__ inline void take_row(int b, bool mine, int i, double2* out) {
        if (mine) {
#pragma unroll
            for (int r = 0; r < 4; ++r) out[4 * r + i] = make_double2(re[b][r], im[b][r]);
            re[b] = im[b] = v4d{0.0, 0.0, 0.0, 0.0};
        }
    }

    // += F G for one k step: f the row block's entry of F, g the entry of G
    __device__ inline void update(int b, double2 f, double2 g) {
        re[b] = mfma64(g.x, f.x, re[b]);
        im[b] = mfma64(g.x, f.y, im[b]);
        re[b] = mfma64_nega(g.y, f.y, re[b]);
        im[b] = mfma64(g.y, f.x, im[b]);
    }
};

// Elimination of a group of kGrp columns held one row per lane: u[q] are the four
// entries of row row0 + 64 q + lane, kmask / krow the key bits of the rows that may
// still be chosen (cleared here for the chosen ones), count the columns the group
// really has (the others are zero and left alone).  NW waves hold the rows, WR =
// 64 Q each; one wave alone needs no LDS and no barrier.  On return u is the
// eliminated group F, piv the pivot rows (-1 past count).
//
// Per column: the lane's candidate (largest key over its rows) and the wave
// maximum; the winner hands its reciprocal pivot and the three other entries of
// its row to every lane (several waves: through an LDS record per wave, written by
// the wave's best lane, then one barrier); every row takes
// U -= (U[s] / pivot) * pivot row, and slot s takes -U[s] / pivot.  Pivot rows are
// not rescaled when they are chosen: every row is kept as sc * U with sc = 1, or 1 /
// pivot in the pivot rows, and there U[s] lacks a 1 until the end of the group;
// neither is read by the other columns, so both are put right once, at the end.
template <int NW, int Q>
struct GroupRec {
    uint4 key[2][(NW + 3) / 4];                    // wave maxima, four to a read (0 past NW)
    double2 r[2][NW][kGrp];                        // reciprocal, the three other entries
};

template <int NW, int Q>
__device__ inline void eliminate_group(double2 (*u)[kGrp], unsigned* kmask, unsigned* krow, int count, int row0,
                                       int wave, int lane, GroupRec<NW, Q>* rec, int* piv, bool& bad) {
    constexpr int WR = 64 * Q;
    unsigned bk, wk;
    double2 bip;
    int bq;
    auto search = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        bk = pivot_key(u[0][s], kmask[0], krow[0]);
        bq = 0;
        double2 pv = u[0][s];
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const unsigned k = pivot_key(u[q][s], kmask[q], krow[q]);
            const bool take = k > bk;
            bk = take ? k : bk;
            bq = take ? q : bq;
            pv = sel2(take, u[q][s], pv);
        }
        bip = crecip(pv);
        wk = wave_umax(bk);
        // keeps the reciprocal here, beside the maximum's lane steps; left to
        // itself the compiler moves it behind them, next to its use
        asm volatile("" : "+v"(bip.x), "+v"(bip.y));
    };
    auto publish = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if constexpr (NW > 1) {
            double2* R = rec->r[s & 1][wave];
            if (lane == 0) reinterpret_cast<unsigned*>(rec->key[s & 1])[wave] = wk;
            if (wk != 0 && bk == wk) {
                R[0] = bip;
#pragma unroll
                for (int c = 0; c < kGrp; ++c) {
                    if (c == s) continue;
                    double2 x = u[0][c];
#pragma unroll
                    for (int q = 1; q < Q; ++q) x = sel2(q == bq, u[q][c], x);
                    R[1 + (c < s ? c : c - 1)] = x;
                }
            }
        }
    };
    double2 ips[kGrp];
    search(std::integral_constant<int, 0>{});
    publish(std::integral_constant<int, 0>{});
    auto column = [&](auto scst) {
        constexpr int s = decltype(scst)::value;
        piv[s] = -1;
        ips[s] = make_double2(1.0, 0.0);
        if (s >= count) return;
        unsigned gk = wk;
        int gr;
        double2 ip, v[kGrp];
        if constexpr (NW > 1) {
            __syncthreads();
            // the keys, then the winner's record, at the same address in every lane
            gk = 0;
#pragma unroll
            for (int w = 0; w < (NW + 3) / 4; ++w) {
                const uint4 k = rec->key[s & 1][w];
                gk = max(max(gk, max(k.x, k.y)), max(k.z, k.w));
            }
            const double2* R = rec->r[s & 1][min(key_row(gk) / WR, NW - 1)];
            ip = R[0];
#pragma unroll
            for (int c = 0; c < kGrp; ++c)
                if (c != s) v[c] = R[1 + (c < s ? c : c - 1)];
            gk = __builtin_amdgcn_readfirstlane(gk);
            gr = gk == 0 ? -1 : key_row(gk);
        } else {
            gr = gk == 0 ? -1 : key_row(gk);
            const int from = gr & 63;
            ip = lane_value(bip, from);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (q != max(gr - row0, 0) / 64) continue;          // wave-uniform
#pragma unroll
                for (int c = 0; c < kGrp; ++c)
                    if (c != s) v[c] = lane_value(u[q][c], from);
            }
        }
        bad = bad || gk == 0 || !(fabs(ip.x) + fabs(ip.y) <= DBL_MAX);
        piv[s] = gr < 0 ? 0 : gr;
        ips[s] = ip;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool pr = row0 + q * 64 + lane == gr;
            const double2 ng = sel2(pr, make_double2(0.0, 0.0), cmul_neg(u[q][s], ip));
            kmask[q] = pr ? 0u : kmask[q];
            krow[q] = pr ? 0u : krow[q];
#pragma unroll
            for (int c = 0; c < kGrp; ++c)
                if (c != s) cfma(u[q][c], ng, v[c]);
            u[q][s] = ng;
        }
        if constexpr (s + 1 < kGrp) {
            search(std::integral_constant<int, s + 1>{});
            if (s + 1 < count) publish(std::integral_constant<int, s + 1>{});
        }
    };
    [&]<int... S>(std::integer_sequence<int, S...>) {
        (column(std::integral_constant<int, S>{}), ...);
    }(std::make_integer_sequence<int, kGrp>{});
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        double2 sc = make_double2(1.0, 0.0);
        bool any = false;
#pragma unroll
        for (int s = 0; s < kGrp; ++s) {
            const bool pr = row0 + q * 64 + lane == piv[s];
            sc = sel2(pr, ips[s], sc);
            any = any || pr;
            u[q][s].x += pr ? 1.0 : 0.0;
        }
        if (any) {
#pragma unroll
            for (int c = 0; c < kGrp; ++c) u[q][c] = cmul_i(sc, u[q][c]);
        }
    }
}

// Row blocks 4 q .. 4 q + 3 of the rows row0 ..: the pivot rows of a group to G,
// then cleared in the block.
template <int NRB>
__device__ inline void take_group_rows(PanelBlock<NRB>& W, int row0, int m, int i, const int* piv, double2 (*G)[kInvNB]) {
#pragma unroll
    for (int b = 0; b < NRB; ++b) {
        const int r0 = row0 + b * 16;
        bool here = false;                       // wave-uniform, mostly false
#pragma unroll
        for (int s = 0; s < kGrp; ++s) here = here || (piv[s] >= r0 && piv[s] < r0 + 16);
        if (!here) continue;
        int s = -1;
#pragma unroll
        for (int c = 0; c < kGrp; ++c) s = piv[c] == r0 + m ? c : s;
        W.take_row(b, s >= 0, i, G[s & (kGrp - 1)]);
    }
}

// ---------------------------------------------------------------------------
// Inverse of one d x d block by one workgroup, the whole block in registers:
// wave w owns columns 16 w .. 16 w + 15 of M = A^T (all 64 Q rows, accumulator
// layout), so d <= 64 Q and d <= 16 NW.  The wave that owns the current group of
// four columns eliminates it alone, no barrier inside, and leaves F and the pivot
// rows in LDS; after one barrier every wave applies them to its own columns, whose
// pivot rows it holds itself.  Bound by the chain of columns of one wave:
// the other waves' updates run beside the owner's next group.
template <int NW, int Q>
struct SmallInvLds {
    double2 F[2][kGrp][64 * Q];
    double2 G[NW][kGrp][kInvNB];
    int piv[2][kGrp];
    int perm[64 * Q];
    int place[64 * Q];
};

template <int NW, int Q>
__device__ void small_inverse(const double2* src, double2* dst, int d, int tag, SmallInvLds<NW, Q>& L, int tid,
                              DevStatus* status) {
    constexpr int NRB = 4 * Q;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, i = lane >> 4;
    const int c0 = wave * kInvNB;
    const int nc = min(kInvNB, d - c0);               // may be <= 0: no columns
    PanelBlock<NRB> W;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + i;
        const double2* column = src + (size_t)min(c0 + c, d - 1) * d;
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            const double2 v = column[min(b * 16 + m, d - 1)];
            W.re[b][r] = c < nc ? v.x : 0.0;
            W.im[b][r] = c < nc ? v.y : 0.0;
        }
    }
    for (int e = tid; e < 64 * Q; e += 64 * NW) {
        L.perm[e] = 0;
        L.place[e] = 0;
    }
    unsigned kmask[Q], krow[Q];                        // rows not yet chosen; every owner keeps them up to date
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int r = q * 64 + lane;
        kmask[q] = r < d ? kKeyBits : 0u;
        krow[q] = r < d ? key_row_bits(r) : 0u;
    }
    bool bad = false;
    __syncthreads();
    for (int cw = 0; cw * kInvNB < d; ++cw) {
        auto group = [&](auto gc) {
            constexpr int grp = decltype(gc)::value;
            constexpr int buf = grp & 1;
            const int j0 = cw * kInvNB + grp * kGrp;
            if (j0 >= d) return;
            const int count = min(kGrp, d - j0);
            double2 u[Q][kGrp];
            int piv[kGrp];
            if (wave == cw) {
                __builtin_amdgcn_s_setprio(3);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) u[q][b] = make_double2(W.re[4 * q + b][grp], W.im[4 * q + b][grp]);
                    transpose4(u[q]);
                }
                eliminate_group<1, Q>(u, kmask, krow, count, 0, 0, lane, nullptr, piv, bad);
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int c = 0; c < kGrp; ++c) L.F[buf][c][q * 64 + lane] = u[q][c];
#pragma unroll
                for (int s = 0; s < kGrp; ++s)
                    if (lane == 0) {
                        L.piv[buf][s] = piv[s];
                        if (s < count) L.perm[j0 + s] = piv[s];
                    }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kGrp; ++s) piv[s] = __builtin_amdgcn_readfirstlane(L.piv[buf][s]);
            double2 f[NRB];
#pragma unroll
            for (int b = 0; b < NRB; ++b) f[b] = L.F[buf][i][b * 16 + m];
            if (wave != cw) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int s = 0; s < kGrp; ++s) {
                        const bool pr = q * 64 + lane == piv[s];
                        kmask[q] = pr ? 0u : kmask[q];
                        krow[q] = pr ? 0u : krow[q];
                    }
            }
            if (nc <= 0) return;
            const int next = j0 + kGrp;                // the next group's owner goes first where waves share a SIMD
            if (wave != next / kInvNB) __builtin_amdgcn_s_setprio(0);
            take_group_rows(W, 0, m, i, piv, L.G[wave]);      // (last group's reads: a barrier ago)
            wave_lds_fence();
            double2 g = L.G[wave][i][m];
            // columns the group has, and its own place in its owner's block
            if (i >= count || (wave == cw && (m >> 2) == grp)) g = make_double2(0.0, 0.0);
            if (wave == cw) {
#pragma unroll
                for (int b = 0; b < NRB; ++b) {
                    W.re[b][grp] = f[b].x;
                    W.im[b][grp] = f[b].y;
                }
            }
#pragma unroll
            for (int b = 0; b < NRB; ++b)
                if (b * 16 < d) W.update(b, f[b], g);
        };
        [&]<int... S>(std::integer_sequence<int, S...>) {
            (group(std::integral_constant<int, S>{}), ...);
        }(std::make_integer_sequence<int, kInvNB / kGrp>{});
    }
    if (bad && lane == 0 && atomicCAS(&status->code, 0, 3) == 0) status->tag = tag;
    // A^-1[perm[col]][pinv(r)] = W[r][col]  (place: cleared above, so after a
    // singular pivot every index stays in range)
    __syncthreads();
    for (int e = tid; e < d; e += 64 * NW) L.place[L.perm[e]] = e;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + i;
        if (c < nc) {
            double2* out = dst + (size_t)L.perm[c0 + c] * d;
#pragma unroll
            for (int b = 0; b < NRB; ++b) {
                const int row = b * 16 + m;
                if (row < d) out[L.place[row]] = make_double2(W.re[b][r], W.im[b][r]);
            }
        }
    }
}

}  // namespace btsq
