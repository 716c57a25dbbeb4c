// McMurchie-Davidson electron-repulsion kernels for one quartet class
// (bra pair class (LA, LB), ket pair class (LC, LD)), with the on-the-fly
// J/K digest of Eq. fock or a plain store of the contracted block.
//
// Per primitive quartet (bra primitive pair i, ket primitive pair j):
//   alpha = p q / (p + q),  R_PQ = P - Q,  T = alpha |R_PQ|^2
//   F_0..F_L(T)                                  (Boys, boys.h)
//   R^n_000 = (-2 alpha)^n F_n(T) / sqrt(p + q)  (Eq. Rn-definition, source;
//             the 1/sqrt(p+q) of the ERI prefactor rides along linearly)
//   R^0_tuv by Eq. R-recursion, in place
//   W_{tuv,cd} = sum_{tau nu phi} (-1)^{tau+nu+phi} E^{cd}_{tau nu phi} R^0_{t+tau,u+nu,v+phi}
//   (ab|cd)   += sum_{tuv} E^{ab}_{tuv} W_{tuv,cd}
// which is Eq. eri-tensor-contracted evaluated through the intermediate
// J_{tuv,k} of Sec. 2.5.  The pair tables carry the contraction
// coefficients and sqrt(2 pi^(5/2)) / p (resp. / q) of the prefactor of
// Eq. twoe-final, so the sum is already the contracted integral.
//
// Digest of a canonical quartet (ab|cd) with value v and degeneracy factor
// f = (1/2)^[a=b] (1/2)^[c=d] (1/2)^[ab=cd] into half-sums J', K':
//   J'_ab += 2 f v D_cd   J'_cd += 2 f v D_ab
//   K'_ac += f v D_bd     K'_bc += f v D_ad   K'_ad += f v D_bc   K'_bd += f v D_ac
// so that J = J' + J'^T and K = K' + K'^T (the eight permutational images of
// every canonical quartet then count once).
#pragma once

#include <type_traits>
#include <utility>

#include "boys.h"
#include "fsim_internal.h"

namespace fsim {

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (N > 0) static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <typename T>
__device__ __forceinline__ const T *etab(const PairTable &t);
template <>
__device__ __forceinline__ const double *etab<double>(const PairTable &t) { return t.E; }
template <>
__device__ __forceinline__ const float *etab<float>(const PairTable &t) { return t.Ef; }

template <typename T>
__device__ __forceinline__ const T *rtab(const PairTable &t);
template <>
__device__ __forceinline__ const double *rtab<double>(const PairTable &t) { return t.rE; }
template <>
__device__ __forceinline__ const float *rtab<float>(const PairTable &t) { return t.rEf; }

template <typename T>
__device__ __forceinline__ const T *stab(const PairTable &t);
template <>
__device__ __forceinline__ const double *stab<double>(const PairTable &t) { return t.S; }
template <>
__device__ __forceinline__ const float *stab<float>(const PairTable &t) { return t.Sf; }

// Pointers into the constant address space: loads at wave-uniform addresses
// become scalar loads into SGPRs, which the VALU takes as operands.  Only for
// tables no kernel of the launch writes.
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ ConstPtr<T> const_ptr(const T *p) {
    return (ConstPtr<T>)(unsigned long long)p;
}

// Index (0..7) of the XCD the calling wave runs on, from the XCC_ID
// hardware register (bits 3:0).
__device__ __forceinline__ int xcd_index() {
    return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 7;
}

// v of the lane the DPP control selects, 0 where it selects none.
template <int CTRL>
__device__ __forceinline__ double dpp_zero(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the wave, valid in lane 63.  Six DPP lane moves and adds on the
// VALU (row shifts by 1, 2, 4, 8, then the row broadcasts 15 and 31): the
// shuffle form took two LDS permutes and a wait per step.
__device__ __forceinline__ double wave_sum63(double v) {
    v += dpp_zero<0x111>(v);
    v += dpp_zero<0x112>(v);
    v += dpp_zero<0x114>(v);
    v += dpp_zero<0x118>(v);
    v += dpp_zero<0x142>(v);
    v += dpp_zero<0x143>(v);
    return v;
}

// In-place Hermite Coulomb recursion: on entry src[n] = R^n_000; on exit
// r[hidx(t,u,v)] = R^0_tuv for t + u + v <= L.  At step n the totals are
// rewritten from high to low, so every R^{n+1} value is read before its slot
// is overwritten.
template <int L, typename T>
__device__ __forceinline__ void hermite_r(const T *src, T X, T Y, T Z, T *r) {
    r[0] = src[L];
    static_for<L>([&](auto m_) {
        constexpr int n = L - 1 - decltype(m_)::value;
        static_for<L - n>([&](auto k_) {
            constexpr int s = L - n - decltype(k_)::value;
            constexpr int base = s == 0 ? 0 : nherm(s - 1);
            static_for<nherm(s) - base>([&](auto q_) {
                constexpr int id = base + decltype(q_)::value;
                constexpr int t = hidx_t(id), u = hidx_u(id), v = hidx_v(id);
                if constexpr (t > 0) {
                    if constexpr (t > 1)
                        r[id] = X * r[hidx(t - 1, u, v)] + T(t - 1) * r[hidx(t - 2, u, v)];
                    else
                        r[id] = X * r[hidx(t - 1, u, v)];
                } else if constexpr (u > 0) {
                    if constexpr (u > 1)
                        r[id] = Y * r[hidx(t, u - 1, v)] + T(u - 1) * r[hidx(t, u - 2, v)];
                    else
                        r[id] = Y * r[hidx(t, u - 1, v)];
                } else {
                    if constexpr (v > 1)
                        r[id] = Z * r[hidx(t, u, v - 1)] + T(v - 1) * r[hidx(t, u, v - 2)];
                    else
                        r[id] = Z * r[hidx(t, u, v - 1)];
                }
            });
        });
        r[0] = src[n];
    });
}

// Locate the tile's bra and ket range (Fock mode).  tile_start is the
// prefix sum of tiles per bra; the search is wave-uniform.
__device__ __forceinline__ int tile_bra(const TileList &tl, int tile) {
    int lo = 0, hi = tl.nbra - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tl.tile_start[mid] <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// ===========================================================================
// Kernel A: one lane per contracted quartet, everything unrolled at compile
// time.  A wave owns a tile (one bra pair, up to 64 consecutive kets), so the
// bra's exponents, centre and Hermite tensor are wave-uniform and the ket
// tables are read with unit stride across lanes.
//
// Loop order (the intermediate J_{tuv,k} of Sec. 2.5, summed over the ket
// primitives before the bra contraction):
//   for each bra primitive pair i:
//       W_{tuv,cd} = sum over ket primitive pairs j of (-1)^{..} E^{cd}_j R^0_ij
//       (ab|cd)   += sum_tuv E^{ab}_i W_{tuv,cd}
// The block is produced in chunks of CA bra components a and CDC ket
// component pairs cd, so that block, W and R^0 fit in registers; each chunk
// re-evaluates the Boys function and R^0 and is digested when complete.
// ===========================================================================
__host__ __device__ constexpr int cmin(int a, int b) { return a < b ? a : b; }

// live values per lane of a chunk: block + W + R^0
__host__ __device__ constexpr int lane_live(int la, int lb, int lc, int ld, int ca, int cdc) {
    return ca * ncart(lb) * cdc + nherm(la + lb) * cdc + nherm(la + lb + lc + ld);
}
// chunk sizes: halve the cd range, then the a range, until the live set fits
__host__ __device__ constexpr int chunk_cd(int la, int lb, int lc, int ld, int limit) {
    int ca = ncart(la), cdc = ncart(lc) * ncart(ld);
    while (lane_live(la, lb, lc, ld, ca, cdc) > limit) {
        if (cdc > 1) cdc = (cdc + 1) / 2;
        else if (ca > 1) ca = (ca + 1) / 2;
        else break;
    }
    return cdc;
}
__host__ __device__ constexpr int chunk_a(int la, int lb, int lc, int ld, int limit) {
    int ca = ncart(la), cdc = ncart(lc) * ncart(ld);
    while (lane_live(la, lb, lc, ld, ca, cdc) > limit) {
        if (cdc > 1) cdc = (cdc + 1) / 2;
        else if (ca > 1) ca = (ca + 1) / 2;
        else break;
    }
    return ca;
}
__host__ __device__ constexpr int n_chunks(int la, int lb, int lc, int ld, int limit) {
    const int ca = chunk_a(la, lb, lc, ld, limit), cdc = chunk_cd(la, lb, lc, ld, limit);
    return ((ncart(la) + ca - 1) / ca) * ((ncart(lc) * ncart(ld) + cdc - 1) / cdc);
}

// Digest of one chunk of a lane's block (components a in [A0, A1), ket
// component pairs in [CD0, CD1)) into the half-sums of Eq. fock:
// J'_ab += 2 v D_cd (wave-reduced), J'_cd += 2 v D_ab, K'_ac += v D_bd,
// K'_bc += v D_ad, K'_ad += v D_bc, K'_bd += v D_ac (fac: degeneracy factor,
// 0 for an idle lane).
//
// D_cd and J'_cd are kept in pair order (EriArgs::Dk, Jk): Dk, Jk point at
// the lane's ket and step by nk from component pair to component pair, Jb at
// the bra and steps by nb.  The 64 lanes hold consecutive kets, so each
// access is one run of 512 bytes; in the N x N matrices the same lanes met 64
// cache lines, and the J'_cd atomics 64 read-modify-writes of the L2.  With
// the DPP wave sum of J'_ab: 64 waters FP64 605 -> 557 ms per build, the
// stored-integral build of 10 waters 3.05 -> 1.79 ms, 64 C/H molecules in
// mixed precision 63.0 -> 46.6 ms.
//
// With kl, the K' terms go to the block's LDS rows instead (krow: row x < NA
// is K'_{f1 + x, .}, row NA + y is K'_{f2 + y, .}, kn doubles per row),
// which the kernel flushes to global memory once per segment of tiles.
template <int LA, int LB, int LC, int LD, typename T, int A0, int A1, int CD0, int CD1>
__device__ __forceinline__ void digest_chunk(const T (&out)[(A1 - A0) * ncart(LB)][CD1 - CD0],
                                             const double *__restrict__ D,
                                             const double *__restrict__ Dk,
                                             double *__restrict__ Jb, double *__restrict__ Jk,
                                             size_t nb, size_t nk,
                                             double *__restrict__ Kh, int N, int f1, int f2, int f3,
                                             int f4, double fac, bool active,
                                             double *__restrict__ krow = nullptr, int kn = 0,
                                             bool kl = false) {
    constexpr int NA = ncart(LA), NB = ncart(LB), NC = ncart(LC), ND = ncart(LD);
    constexpr int NAc = A1 - A0, NABc = NAc * NB, NCDc = CD1 - CD0;
    const int lane = threadIdx.x & 63;
    // J'_ab (partial over this chunk's cd): pre-reduced over the wave
    double dcd[NCDc];
#pragma unroll
    for (int x = 0; x < NCDc; ++x) dcd[x] = Dk[(size_t)(CD0 + x) * nk];
    static_for<NABc>([&](auto abl_) {
        constexpr int abl = decltype(abl_)::value;
        constexpr int ab = (A0 + abl / NB) * NB + abl % NB;
        double sum = 0.0;
        static_for<NCDc>([&](auto cdl_) {
            constexpr int cdl = decltype(cdl_)::value;
            sum += (double)out[abl][cdl] * dcd[cdl];
        });
        sum = wave_sum63(2.0 * fac * sum);
        if (lane == 63) atomicAdd(&Jb[(size_t)ab * nb], sum);
    });
    if (active) {
        // J'_cd (partial over this chunk's a)
        static_for<NCDc>([&](auto cdl_) {
            constexpr int cdl = decltype(cdl_)::value;
            double sum = 0.0;
            static_for<NABc>([&](auto abl_) {
                constexpr int abl = decltype(abl_)::value;
                constexpr int ia = A0 + abl / NB, ib = abl % NB;
                sum += (double)out[abl][cdl] * D[(size_t)(f1 + ia) * N + f2 + ib];
            });
            atomicAdd(&Jk[(size_t)(CD0 + cdl) * nk], 2.0 * fac * sum);
        });
        // K'_xc for x in {a (with D_bd), b (with D_ad)} and every c in the chunk
        static_for<NC>([&](auto c_) {
            constexpr int ic = decltype(c_)::value;
            constexpr bool has_c = ic * ND + ND > CD0 && ic * ND < CD1;
            if constexpr (has_c) {
                static_for<NAc>([&](auto al_) {
                    constexpr int al = decltype(al_)::value;
                    double sum = 0.0;
                    static_for<NB>([&](auto b_) {
                        constexpr int ib = decltype(b_)::value;
                        static_for<ND>([&](auto d_) {
                            constexpr int id = decltype(d_)::value;
                            constexpr int cd = ic * ND + id;
                            if constexpr (cd >= CD0 && cd < CD1)
                                sum += (double)out[al * NB + ib][cd - CD0] *
                                       D[(size_t)(f2 + ib) * N + f4 + id];
                        });
                    });
                    if (kl) atomicAdd(&krow[(A0 + al) * kn + f3 + ic], fac * sum);
                    else atomicAdd(&Kh[(size_t)(f1 + A0 + al) * N + f3 + ic], fac * sum);
                });
                static_for<NB>([&](auto b_) {
                    constexpr int ib = decltype(b_)::value;
                    double sum = 0.0;
                    static_for<NAc>([&](auto al_) {
                        constexpr int al = decltype(al_)::value;
                        static_for<ND>([&](auto d_) {
                            constexpr int id = decltype(d_)::value;
                            constexpr int cd = ic * ND + id;
                            if constexpr (cd >= CD0 && cd < CD1)
                                sum += (double)out[al * NB + ib][cd - CD0] *
                                       D[(size_t)(f1 + A0 + al) * N + f4 + id];
                        });
                    });
                    if (kl) atomicAdd(&krow[(NA + ib) * kn + f3 + ic], fac * sum);
                    else atomicAdd(&Kh[(size_t)(f2 + ib) * N + f3 + ic], fac * sum);
                });
            }
        });
        // K'_xd for x in {a (with D_bc), b (with D_ac)} and every d in the chunk
        static_for<ND>([&](auto d_) {
            constexpr int id = decltype(d_)::value;
            constexpr bool has_d = [] {
                for (int c = 0; c < NC; ++c)
                    if (c * ND + id >= CD0 && c * ND + id < CD1) return true;
                return false;
            }();
            if constexpr (has_d) {
                static_for<NAc>([&](auto al_) {
                    constexpr int al = decltype(al_)::value;
                    double sum = 0.0;
                    static_for<NB>([&](auto b_) {
                        constexpr int ib = decltype(b_)::value;
                        static_for<NC>([&](auto c_) {
                            constexpr int ic = decltype(c_)::value;
                            constexpr int cd = ic * ND + id;
                            if constexpr (cd >= CD0 && cd < CD1)
                                sum += (double)out[al * NB + ib][cd - CD0] *
                                       D[(size_t)(f2 + ib) * N + f3 + ic];
                        });
                    });
                    if (kl) atomicAdd(&krow[(A0 + al) * kn + f4 + id], fac * sum);
                    else atomicAdd(&Kh[(size_t)(f1 + A0 + al) * N + f4 + id], fac * sum);
                });
                static_for<NB>([&](auto b_) {
                    constexpr int ib = decltype(b_)::value;
                    double sum = 0.0;
                    static_for<NAc>([&](auto al_) {
                        constexpr int al = decltype(al_)::value;
                        static_for<NC>([&](auto c_) {
                            constexpr int ic = decltype(c_)::value;
                            constexpr int cd = ic * ND + id;
                            if constexpr (cd >= CD0 && cd < CD1)
                                sum += (double)out[al * NB + ib][cd - CD0] *
                                       D[(size_t)(f1 + A0 + al) * N + f3 + ic];
                        });
                    });
                    if (kl) atomicAdd(&krow[(NA + ib) * kn + f4 + id], fac * sum);
                    else atomicAdd(&Kh[(size_t)(f2 + ib) * N + f4 + id], fac * sum);
                });
            }
        });
    }
}

// How a launch over segments shares one tile out, so that a small molecule's
// few tiles still fill the GPU and no wave walks through all the primitives
// of 64 quartets: csplit groups of the tile's chunks, ksplit lanes per
// quartet, each with every ksplit-th ket primitive (a power of two up to 8; an
// item then covers 64 / ksplit kets, and the lanes' blocks are added up
// before the digest), and bsplit items with every bsplit-th bra primitive
// each (the digest is linear in the block: each item digests its own share).
struct TileShare {
    int tile, chunk = 0, csplit = 1;
    int k0 = 0, lane, ls = 0;   // first ket of the item in its tile, log2 ksplit
    int b0 = 0, bstep = 1;      // bra primitives b0, b0 + bstep, ...
    int j0 = 0, jstep = 1;      // ket primitives of the calling lane
    __device__ __forceinline__ explicit TileShare(int t) : tile(t), lane(threadIdx.x & 63) {}
    // item of the tiles from t0 on
    __device__ __forceinline__ TileShare(const EriArgs &a, int t0, int item) : TileShare(t0 + item) {
        if (a.shares == 1) return;   // a tile per item: the large launches
        ls = 31 - __builtin_clz(a.ksplit);
        csplit = a.csplit;
        bstep = a.bsplit;
        chunk = item % csplit;
        item /= csplit;
        b0 = item % bstep;
        item /= bstep;
        k0 = (item & (a.ksplit - 1)) * (64 >> ls);
        tile = t0 + (item >> ls);
        lane = (threadIdx.x & 63) >> ls;
        jstep = a.ksplit;
        j0 = threadIdx.x & (a.ksplit - 1);
    }
};

// Sum over the 1 << ls lanes of a quartet, in all of them (DPP: lane xor 1,
// lane xor 2, mirrored half rows).
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_other(T v) {
    if constexpr (sizeof(T) == 8) {
        return dpp_zero<CTRL>(v);
    } else {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
    }
}
template <int N, int M, typename T>
__device__ __forceinline__ void share_sum(T (&out)[N][M], int ls) {
    if (ls == 0) return;
#pragma unroll
    for (int x = 0; x < N; ++x)
#pragma unroll
        for (int y = 0; y < M; ++y) {
            out[x][y] += dpp_other<0xB1>(out[x][y]);
            if (ls > 1) out[x][y] += dpp_other<0x4E>(out[x][y]);
            if (ls > 2) out[x][y] += dpp_other<0x141>(out[x][y]);
        }
}

// Segment mode of the lane kernels (Fock builds): the block takes whole
// segments, each a run of tiles of one bra record, and its waves split the
// segment's tiles.  The K' terms of a quartet all lie in the rows of the
// bra's functions (K'_ac, K'_ad in the rows of a, K'_bc, K'_bd in those of
// b), so they are added into the block's LDS copy of those rows; after a
// block barrier the non-zero entries go to global K' with one atomic each
// and the rows are cleared.  Short lists share their tiles out (TileShare),
// and a.parts blocks take every parts-th item of a segment.  krow: (NA + NB) rows of a.kn doubles.
// The block's rows after segment sg: non-zero entries added to global K'
// and cleared (every thread of the block takes part; no barriers inside).
template <int NA, int NB>
__device__ __forceinline__ void segment_flush(const EriArgs &a, double *__restrict__ krow,
                                              long long xoff, int sg) {
    constexpr int NR = NA + NB;
    const int kn = a.kn;
    const int bra = a.tl.bra[a.tl.seg_rec[sg]];
    const int mol = a.bra.mol[bra];
    const int N = a.mol_n[mol];
    const int f1 = a.bra.bf1[bra], f2 = a.bra.bf2[bra];
    double *__restrict__ Kh = a.Kh + xoff + a.mol_off[mol];
    for (int x = threadIdx.x; x < NR * N; x += blockDim.x) {
        const int r = x / N, col = x - r * N;
        const double v = krow[r * kn + col];
        if (v != 0.0) {
            atomicAdd(&Kh[(size_t)(r < NA ? f1 + r : f2 + r - NA) * N + col], v);
            krow[r * kn + col] = 0.0;
        }
    }
}

template <int NA, int NB, typename Body>
__device__ __forceinline__ void run_segments(const EriArgs &a, double *__restrict__ krow,
                                             long long xoff, Body &&body) {
    constexpr int NR = NA + NB;
    const int wave = threadIdx.x >> 6, wpb = blockDim.x >> 6;
    for (int x = threadIdx.x; x < NR * a.kn; x += blockDim.x) krow[x] = 0.0;
    __syncthreads();
    for (int w = blockIdx.x; w < a.tl.nseg * a.parts; w += gridDim.x) {
        const int sg = w / a.parts, part = w - sg * a.parts;
        const int t0 = a.tl.seg_t0[sg], nt = a.tl.seg_nt[sg];
        const int items = nt * a.shares;
        for (int it = wave * a.parts + part; it < items; it += wpb * a.parts)
            body(t0, __builtin_amdgcn_readfirstlane(it));
        __syncthreads();
        segment_flush<NA, NB>(a, krow, xoff, sg);
        __syncthreads();
    }
}

// Minimum waves per SIMD the lane kernel is compiled for.  ds and dp bras
// with a live set of up to 128 FP64 values are held to two resident waves
// (256 registers each); every other kernel is left to the compiler, which
// measured faster for the s and p bras, and for the dd bras, whose staged
// ket entries spilled to scratch at two ((dd|ps) FP64, 64 waters: 13.9 ms
// with 340 bytes of scratch per lane, 5.1 ms without).
__host__ __device__ constexpr int lane_min_waves(int la, int lb, int lc, int ld, int ca, int cdc) {
    return la == 2 && lb < 2 && lane_live(la, lb, lc, ld, ca, cdc) <= 128 ? 2 : 1;
}

// Blocks of the lane kernel in segment mode: 8 waves where the kernel is held
// to two waves per SIMD (two blocks' worth of registers per CU), else 4.
__host__ __device__ constexpr int seg_waves(int la, int lb, int lc, int ld, int ca, int cdc) {
    return lane_min_waves(la, lb, lc, ld, ca, cdc) == 2 ? 8 : 4;
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE, int CA, int CDC, bool SEG,
          bool SHARED = false>
__global__ __launch_bounds__(SEG ? 64 * seg_waves(LA, LB, LC, LD, CA, CDC) : 256,
                             lane_min_waves(LA, LB, LC, LD, CA, CDC)) void k_eri_lane(EriArgs a) {
    constexpr int L = LA + LB + LC + LD, LAB = LA + LB;
    constexpr int NA = ncart(LA), NB = ncart(LB), NC = ncart(LC), ND = ncart(LD);
    constexpr int NCD = NC * ND, NHAB = nherm(LAB), NH = nherm(L);
    constexpr int NEB = n_entries(LA, LB), NEK = n_entries(LC, LD);
    constexpr int NCHA = (NA + CA - 1) / CA, NCHCD = (NCD + CDC - 1) / CDC;
    // Boys grid in LDS: FP64 for FP64 tiles, FP32 (5 terms, the Taylor step
    // only) for FP32 tiles
    constexpr bool F32 = std::is_same<T, float>::value;
    __shared__ __align__(16) std::conditional_t<F32, float, double> tab[F32 ? BOYS_LDS32 : BOYS_LDS];
    extern __shared__ __align__(16) unsigned char stage_lds[];
    if constexpr (F32) boys_stage32(tab, a.boys, L);
    else boys_stage(tab, a.boys, L);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int ntile = STORE ? a.st_ntile : a.tl.ntile;
    const T *__restrict__ Eb = etab<T>(a.bra);
    const T *__restrict__ Ek = etab<T>(a.ket);
    const size_t nb = a.bra.n, nk = a.ket.n;
    // The bra pair is the same for the whole wave.  For d bras (large Hermite
    // boxes, re-read in every chunk) its primitive data are copied once per
    // tile (or per group of ks primitive pairs) into this wave's LDS slice and
    // read back as broadcasts; s and p bras read them from global memory,
    // which measured faster for their small boxes.
    constexpr bool STAGE = LA == 2;
    const int ks = STAGE ? a.stage_prims : 1 << 20;
    double *__restrict__ sp = (double *)(stage_lds + (size_t)(threadIdx.x >> 6) * a.stage_bytes);
    T *__restrict__ se = (T *)(sp + 4 * ks);
    auto stage = [&](int bra_, int i0, int cnt) {
        // from the row copies, which a wave reads in whole cache lines
        const size_t r0 = (size_t)bra_ * a.bra.kmax + i0;
        for (int x = lane; x < cnt * 4; x += 64) sp[x] = a.bra.rp[r0 * 4 + x];
        for (int x = lane; x < cnt * NEB; x += 64) se[x] = rtab<T>(a.bra)[r0 * NEB + x];
        // the wave's own LDS writes complete before its reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // per-XCD private J'/K' copies keep each cache line's atomics on one XCD
    const long long xoff = (!STORE && a.xcd_stride) ? xcd_index() * a.xcd_stride : 0;

    // one tile; kl: K' rows into the block's LDS rows krow (segment mode)
    auto tile_body = [&](const TileShare sh, double *__restrict__ krow,
                         const bool kl) __attribute__((always_inline)) {
        const int tile = sh.tile;
        int bra, ket;
        bool active;
        if constexpr (STORE) {
            bra = __builtin_amdgcn_readfirstlane(a.st_bra[tile]);
            ket = a.st_ket[tile * 64 + lane];
            active = ket >= 0;
            if (!active) ket = 0;
        } else {
            const int b = tile_bra(a.tl, tile);
            bra = __builtin_amdgcn_readfirstlane(a.tl.bra[b]);
            const int k0 = a.tl.ket_lo[b] + (tile - a.tl.tile_start[b]) * TILE + sh.k0;
            if (k0 >= a.tl.ket_hi[b]) return;   // the whole wave: no kets in this item
            ket = k0 + sh.lane;
            active = ket < a.tl.ket_hi[b];
            if (!active) ket = k0;
        }
        const int nbp = __builtin_amdgcn_readfirstlane(a.bra.nprim[bra]);
        const int nkp = active ? a.ket.nprim[ket] : 0;
        const bool all_staged = nbp <= ks;
        // bra primitives are shared out only when all of them are staged
        if (!all_staged && sh.b0 > 0) return;
        const int bstep = all_staged ? sh.bstep : 1;
        if (STAGE && all_staged) stage(bra, 0, nbp);
        // the quartet's molecule block (bra and ket pairs share the molecule)
        const int mol = __builtin_amdgcn_readfirstlane(a.bra.mol[bra]);
        const long long mbase = STORE ? 0 : a.mol_off[mol];
        const int N = STORE ? 0 : a.mol_n[mol];
        const double *__restrict__ D = STORE ? nullptr : a.D + mbase;
        double *__restrict__ Jb = STORE ? nullptr : a.Jb + xoff + bra;
        double *__restrict__ Jk = STORE ? nullptr : a.Jk + xoff + ket;
        const double *__restrict__ Dk = STORE ? nullptr : a.Dk + ket;
        double *__restrict__ Kh = STORE ? nullptr : a.Kh + xoff + mbase;
        int f1 = 0, f2 = 0, f3 = 0, f4 = 0;
        double fac = 0.0;
        long long soff = 0;
        int st0 = 0, st1 = 0, st2 = 0, st3 = 0;
        if constexpr (STORE) {
            if (active) {
                const size_t q = (size_t)tile * 64 + lane;
                soff = a.st_off[q];
                st0 = a.st_stride[q * 4 + 0];
                st1 = a.st_stride[q * 4 + 1];
                st2 = a.st_stride[q * 4 + 2];
                st3 = a.st_stride[q * 4 + 3];
            }
        } else {
            f1 = __builtin_amdgcn_readfirstlane(a.bra.bf1[bra]);
            f2 = __builtin_amdgcn_readfirstlane(a.bra.bf2[bra]);
            f3 = a.ket.bf1[ket];
            f4 = a.ket.bf2[ket];
            active = active && sh.j0 == 0;   // one lane of each quartet digests
            fac = active ? 1.0 : 0.0;
            if (a.bra.sh1[bra] == a.bra.sh2[bra]) fac *= 0.5;
            if (a.ket.sh1[ket] == a.ket.sh2[ket]) fac *= 0.5;
            if (a.same_class && ket == bra) fac *= 0.5;
        }

        static_for<NCHA * NCHCD>([&](auto ch_) {
            constexpr int ch = decltype(ch_)::value;
            constexpr int A0 = (ch / NCHCD) * CA, A1 = cmin(A0 + CA, NA);
            constexpr int CD0 = (ch % NCHCD) * CDC, CD1 = cmin(CD0 + CDC, NCD);
            constexpr int NAc = A1 - A0, NABc = NAc * NB, NCDc = CD1 - CD0;
            if (NCHA * NCHCD > 1 && SHARED && ch % sh.csplit != sh.chunk) return;
            T out[NABc][NCDc];
#pragma unroll
            for (int x = 0; x < NABc; ++x)
#pragma unroll
                for (int y = 0; y < NCDc; ++y) out[x][y] = T(0);

            for (int i = sh.b0; i < nbp; i += bstep) {
                int il = i;
                if (STAGE && !all_staged) {
                    il = i % ks;
                    if (il == 0) stage(bra, i, nbp - i < ks ? nbp - i : ks);
                }
                const double p = STAGE ? sp[il * 4 + 0] : a.bra.p[(size_t)i * nb + bra];
                const double Px = STAGE ? sp[il * 4 + 1] : a.bra.P[((size_t)i * 3 + 0) * nb + bra];
                const double Py = STAGE ? sp[il * 4 + 2] : a.bra.P[((size_t)i * 3 + 1) * nb + bra];
                const double Pz = STAGE ? sp[il * 4 + 3] : a.bra.P[((size_t)i * 3 + 2) * nb + bra];
                T W[NCDc][NHAB];
#pragma unroll
                for (int x = 0; x < NCDc; ++x)
#pragma unroll
                    for (int h = 0; h < NHAB; ++h) W[x][h] = T(0);
                // d bras: ket primitive data, including this chunk's Hermite box
                // entries, loaded one primitive ahead of use (s and p bras load
                // them in place, which measured faster)
                constexpr int EK0 = box_off(LC, LD, CD0);
                constexpr int EK1 = CD1 < NCD ? box_off(LC, LD, CD1) : NEK;
                constexpr int NEKC = STAGE ? EK1 - EK0 : 1;
                double qn = 0.0, Kxn = 0.0, Kyn = 0.0, Kzn = 0.0;
                T ekn[NEKC];
                auto kload = [&](int j_) {
                    qn = a.ket.p[(size_t)j_ * nk + ket];
                    Kxn = a.ket.P[((size_t)j_ * 3 + 0) * nk + ket];
                    Kyn = a.ket.P[((size_t)j_ * 3 + 1) * nk + ket];
                    Kzn = a.ket.P[((size_t)j_ * 3 + 2) * nk + ket];
                    if constexpr (STAGE) {
                        const T *__restrict__ ekp = Ek + (size_t)j_ * NEK * nk + ket;
#pragma unroll
                        for (int e = 0; e < NEKC; ++e) ekn[e] = ekp[(size_t)(EK0 + e) * nk];
                    }
                };
                if (STAGE && sh.j0 < nkp) kload(sh.j0);
                for (int j = sh.j0; j < nkp; j += sh.jstep) {
                    if (!STAGE) kload(j);
                    const double q = qn;
                    const double X = Px - Kxn, Y = Py - Kyn, Z = Pz - Kzn;
                    T ekc[NEKC];
#pragma unroll
                    for (int e = 0; e < NEKC; ++e) ekc[e] = ekn[e];
                    if (STAGE && j + sh.jstep < nkp) kload(j + sh.jstep);
                    // 1/sqrt(p+q) once; 1/(p+q) and alpha = pq/(p+q) from it
                    T src[L + 1];
                    if constexpr (F32) {
                        // FP32 tile: FP32 Taylor step, FP64 recursion and
                        // prefactor, sources rounded to FP32
                        const double rs = rsqrt(p + q);
                        const double alpha = p * q * (rs * rs);
                        double F[L + 1];
                        boys_eval_mixed<L>(alpha * (X * X + Y * Y + Z * Z), tab, F);
                        double m = rs;
#pragma unroll
                        for (int n = 0; n <= L; ++n) {
                            src[n] = (float)(F[n] * m);
                            m *= -2.0 * alpha;
                        }
                    } else {
                        const double rs = rsqrt(p + q);
                        const double alpha = p * q * (rs * rs);
                        double F[L + 1];
                        boys_eval<L>(alpha * (X * X + Y * Y + Z * Z), tab, F);
                        double m = rs;
#pragma unroll
                        for (int n = 0; n <= L; ++n) {
                            src[n] = T(F[n] * m);
                            m *= -2.0 * alpha;
                        }
                    }
                    T r[NH];
                    hermite_r<L, T>(src, T(X), T(Y), T(Z), r);
                    const T *__restrict__ ek = Ek + (size_t)j * NEK * nk + ket;
                    static_for<NCDc>([&](auto cdl_) {
                        constexpr int cdl = decltype(cdl_)::value;
                        constexpr int cd = CD0 + cdl;
                        constexpr int bx = box_dim(LC, LD, cd, 0), by = box_dim(LC, LD, cd, 1),
                                      bz = box_dim(LC, LD, cd, 2);
                        constexpr int eo = box_off(LC, LD, cd);
                        static_for<bx + 1>([&](auto ta_) {
                            constexpr int ta = decltype(ta_)::value;
                            static_for<by + 1>([&](auto nu_) {
                                constexpr int nu = decltype(nu_)::value;
                                static_for<bz + 1>([&](auto ph_) {
                                    constexpr int ph = decltype(ph_)::value;
                                    constexpr int e = eo + (ta * (by + 1) + nu) * (bz + 1) + ph;
                                    T ev;
                                    if constexpr (STAGE) ev = ekc[e - EK0];
                                    else ev = ek[(size_t)e * nk];
                                    if constexpr ((ta + nu + ph) & 1) ev = -ev;
                                    static_for<NHAB>([&](auto h_) {
                                        constexpr int h = decltype(h_)::value;
                                        constexpr int ri = hidx(hidx_t(h) + ta, hidx_u(h) + nu,
                                                                hidx_v(h) + ph);
                                        W[cdl][h] = fma(ev, r[ri], W[cdl][h]);
                                    });
                                });
                            });
                        });
                    });
                }
                // bra contraction, once per bra primitive pair
                const T *__restrict__ eb = STAGE ? se + il * NEB : Eb + (size_t)i * NEB * nb + bra;
                const size_t es = STAGE ? 1 : nb;
                static_for<NABc>([&](auto abl_) {
                    constexpr int abl = decltype(abl_)::value;
                    constexpr int ab = (A0 + abl / NB) * NB + abl % NB;
                    constexpr int ax = box_dim(LA, LB, ab, 0), ay = box_dim(LA, LB, ab, 1),
                                  az = box_dim(LA, LB, ab, 2);
                    constexpr int ao = box_off(LA, LB, ab);
                    static_for<ax + 1>([&](auto t_) {
                        constexpr int t = decltype(t_)::value;
                        static_for<ay + 1>([&](auto u_) {
                            constexpr int u = decltype(u_)::value;
                            static_for<az + 1>([&](auto v_) {
                                constexpr int v = decltype(v_)::value;
                                constexpr int e = ao + (t * (ay + 1) + u) * (az + 1) + v;
                                const T ebv = eb[e * es];
                                static_for<NCDc>([&](auto cdl_) {
                                    constexpr int cdl = decltype(cdl_)::value;
                                    out[abl][cdl] = fma(ebv, W[cdl][hidx(t, u, v)], out[abl][cdl]);
                                });
                            });
                        });
                    });
                });
            }

            if constexpr (STORE) {
                if (active) {
                    static_for<NABc>([&](auto abl_) {
                        constexpr int abl = decltype(abl_)::value;
                        constexpr int ia = A0 + abl / NB, ib = abl % NB;
                        static_for<NCDc>([&](auto cdl_) {
                            constexpr int cdl = decltype(cdl_)::value;
                            constexpr int ic = (CD0 + cdl) / ND, id = (CD0 + cdl) % ND;
                            a.out[soff + ia * st0 + ib * st1 + ic * st2 + id * st3] =
                                (double)out[abl][cdl];
                        });
                    });
                }
            } else {
                if constexpr (SHARED) share_sum(out, sh.ls);
                digest_chunk<LA, LB, LC, LD, T, A0, A1, CD0, CD1>(
                    out, D, Dk, Jb, Jk, nb, nk, Kh, N, f1, f2, f3, f4, fac, active, krow, a.kn, kl);
            }
        });
    };
    if constexpr (SEG && !STORE) {
        double *__restrict__ krow = (double *)(stage_lds + (size_t)wpb * a.stage_bytes);
        run_segments<NA, NB>(a, krow, xoff, [&](int t0, int it) __attribute__((always_inline)) {
            if constexpr (SHARED) tile_body(TileShare(a, t0, it), krow, true);
            else tile_body(TileShare(t0 + it), krow, true);
        });
    } else {
        for (int tile0 = blockIdx.x * wpb + (threadIdx.x >> 6); tile0 < ntile;
             tile0 += gridDim.x * wpb)
            tile_body(TileShare(__builtin_amdgcn_readfirstlane(tile0)), nullptr, false);
    }
}

// ===========================================================================
// Kernel A, ket-outer order (ss, ps, pp and ds bras, dp bras with ss and ps
// kets; Fock or store mode).  The same lane-per-quartet tiles as k_eri_lane,
// with the primitive loops swapped: each ket
// primitive's data are loaded once and held in registers while the bra
// primitives (wave-uniform, read by scalar loads from the row tables; staged
// in LDS they cost the 64-water s/p build 312 ms against 292) run inside, and
// the bra contraction is applied per primitive quartet:
//   V_{tuv,cd} = sum_{tau nu phi} (-1)^{tau+nu+phi} E^{cd}_{tau nu phi} R^0_{t+tau,u+nu,v+phi}
//   (ab|cd)   += sum_tuv E^{ab}_{tuv} V_{tuv,cd}
// The ket entries are the scaled ones: the factor common to the last entry
// of every component pair's box goes into the sources R^n_000, and that entry
// is then 1, so that the ket step of a pair of p functions takes one FMA
// per value and direction less ((ps|: half of it) and loads fewer columns;
// the norms of d components are applied to the finished block.  64 waters,
// FP64: (pp|ps) 90.1 -> 82.7 ms, (ps|ps) 50.3 -> 46.7 ms.
// This trades the once-per-bra-primitive bra step for one per primitive
// quartet (cheap for small bra boxes, and see ko_sums) against loading every
// ket primitive once per quartet instead of once per bra primitive.
// ===========================================================================
// Boys-function providers of the ket-outer tile body: the class kernels
// stage the table of their own order L (boys.h); the persistent kernel
// stages raw F_n(T_k) for every order its classes need.
template <typename B>
struct BoysTable {
    const double *tab;
    template <int L>
    __device__ __forceinline__ void eval(double T, double *F) const { B::eval(T, tab, F); }
};

// The sums of a ps or pp bra.  With P - A = -beta AB and P - B = alpha AB,
//   (p_i s| = S_i - AB_i S0
//   (p_i p_j| = S_ij + delta_ij D - AB_i U_j + AB_j W_i - AB_i AB_j S0
// where, V the Hermite integrals over the bra's indices, the sums over the
// primitive quartets are
//   ps: S0 = sum c beta V_0, S_i = sum c h V_i                              (4)
//   pp: S0 = sum c alpha beta V_0, D = sum c h V_0, U_i = sum c beta h V_i,
//       W_i = sum c alpha h V_i, S_ij = sum c h^2 V_ij                     (14)
// so a primitive quartet takes 4 FMAs per ket component in place of the 6 of
// the components' boxes, 14 in place of 33.  FP64 classes whose block is taken
// in one chunk: (pp|pp) would need three chunks for its 14 x 9 sums, or two and
// spills (46.1 -> 46.5 or 49.0 ms, 1024 C/H molecules 107 -> 126 or 113).
// 64 waters without d shells, before and after: (pp|ps) 70.9 -> 59.6 ms, (pp|ss)
// 23.0 -> 21.5, (ps|ps) 40.7 -> 38.9, (ps|ss) 38.8 -> 37.7.
__host__ __device__ constexpr bool ko_sums(int la, int lb, int nchunk, bool f64) {
    return f64 && has_factors(la, lb) && nchunk == 1;
}
__host__ __device__ constexpr int bra_sums(int lb) { return lb == 0 ? 4 : 14; }
// S_ij (i <= j in the order xx xy xz yy yz zz) from 8 on
__host__ __device__ constexpr int sum_pp(int i, int j) {
    return i > j ? sum_pp(j, i) : 8 + i * 3 - i * (i + 1) / 2 + j;
}
// factor of sum k in the bra's row
__host__ __device__ constexpr int sum_factor(int lb, int k) {
    if (lb == 0) return k == 0 ? 0 : 1;
    return k < 2 ? k : (k < 5 ? 2 : (k < 8 ? 3 : 4));
}
// Hermite index of sum k
__host__ __device__ constexpr int sum_herm(int lb, int k) {
    const int unit[3] = {hidx(1, 0, 0), hidx(0, 1, 0), hidx(0, 0, 1)};
    if (lb == 0) return k == 0 ? hidx(0, 0, 0) : unit[k - 1];
    if (k < 2) return hidx(0, 0, 0);
    if (k < 8) return unit[(k - 2) % 3];
    const int pair[6] = {hidx(2, 0, 0), hidx(1, 1, 0), hidx(1, 0, 1),
                         hidx(0, 2, 0), hidx(0, 1, 1), hidx(0, 0, 2)};
    return pair[k - 8];
}

// One tile (one bra pair x up to 64 kets) of the ket-outer kernel.
template <int LA, int LB, int LC, int LD, typename T, bool STORE, int CA, int CDC,
          bool SHARED = false, typename BP>
__device__ __forceinline__ void ko_tile(const EriArgs &a, const TileShare sh, const BP &bp,
                                        double *__restrict__ krow = nullptr, bool kl = false) {
    constexpr int L = LA + LB + LC + LD, LAB = LA + LB;
    constexpr int NA = ncart(LA), NB = ncart(LB), NC = ncart(LC), ND = ncart(LD);
    constexpr int NCD = NC * ND, NHAB = nherm(LAB), NH = nherm(L);
    constexpr bool F32 = std::is_same<T, float>::value;
    // bra sums instead of components
    constexpr bool SUMS = ko_sums(LA, LB, (ncart(LC) * ncart(LD) + CDC - 1) / CDC, !F32);
    constexpr int NRB = F32 ? n_entries(LA, LB) : n_row(LA, LB), NSK = n_scaled(LC, LD);
    constexpr int NCHA = (NA + CA - 1) / CA, NCHCD = (NCD + CDC - 1) / CDC;
    static_assert(!SUMS || NCHA == 1, "the bra sums are for whole bras");
    const int lane = threadIdx.x & 63;
    const int tile = sh.tile;
    const T *__restrict__ Sk = stab<T>(a.ket);
    const size_t nb = a.bra.n, nk = a.ket.n;
    const long long xoff = (!STORE && a.xcd_stride) ? xcd_index() * a.xcd_stride : 0;
    int bra, ket;
    bool active;
    if constexpr (STORE) {
        bra = __builtin_amdgcn_readfirstlane(a.st_bra[tile]);
        ket = a.st_ket[tile * 64 + lane];
        active = ket >= 0;
        if (!active) ket = 0;
    } else {
        const int b = tile_bra(a.tl, tile);
        bra = __builtin_amdgcn_readfirstlane(a.tl.bra[b]);
        const int k0 = a.tl.ket_lo[b] + (tile - a.tl.tile_start[b]) * TILE + sh.k0;
        if (k0 >= a.tl.ket_hi[b]) return;   // the whole wave: no kets in this item
        ket = k0 + sh.lane;
        active = ket < a.tl.ket_hi[b];
        if (!active) ket = k0;
    }
    const int nbp = __builtin_amdgcn_readfirstlane(a.bra.nprim[bra]);
    const int nkp = active ? a.ket.nprim[ket] : 0;
    const int mol = __builtin_amdgcn_readfirstlane(a.bra.mol[bra]);
    const long long mbase = STORE ? 0 : a.mol_off[mol];
    const int N = STORE ? 0 : a.mol_n[mol];
    const double *__restrict__ D = STORE ? nullptr : a.D + mbase;
    double *__restrict__ Jb = STORE ? nullptr : a.Jb + xoff + bra;
    double *__restrict__ Jk = STORE ? nullptr : a.Jk + xoff + ket;
    const double *__restrict__ Dk = STORE ? nullptr : a.Dk + ket;
    double *__restrict__ Kh = STORE ? nullptr : a.Kh + xoff + mbase;
    const int f1 = __builtin_amdgcn_readfirstlane(a.bra.bf1[bra]);
    const int f2 = __builtin_amdgcn_readfirstlane(a.bra.bf2[bra]);
    const int f3 = a.ket.bf1[ket], f4 = a.ket.bf2[ket];
    if constexpr (SHARED) active = active && sh.j0 == 0;   // one lane of each quartet digests
    double fac = active ? 1.0 : 0.0;
    if (a.bra.sh1[bra] == a.bra.sh2[bra]) fac *= 0.5;
    if (a.ket.sh1[ket] == a.ket.sh2[ket]) fac *= 0.5;
    if (a.same_class && ket == bra) fac *= 0.5;
    long long soff = 0;
    int st0 = 0, st1 = 0, st2 = 0, st3 = 0;
    if constexpr (STORE) {
        if (active) {
            const size_t q = (size_t)tile * 64 + lane;
            soff = a.st_off[q];
            st0 = a.st_stride[q * 4 + 0];
            st1 = a.st_stride[q * 4 + 1];
            st2 = a.st_stride[q * 4 + 2];
            st3 = a.st_stride[q * 4 + 3];
        }
    }

    // the bra's primitive rows
    const ConstPtr<double> rp = const_ptr(a.bra.rp + (size_t)bra * a.bra.kmax * 4);
    const ConstPtr<T> re = const_ptr(rtab<T>(a.bra) + (size_t)bra * a.bra.kmax * NRB);

    static_for<NCHA * NCHCD>([&](auto ch_) {
        constexpr int ch = decltype(ch_)::value;
        constexpr int A0 = (ch / NCHCD) * CA, A1 = cmin(A0 + CA, NA);
        constexpr int CD0 = (ch % NCHCD) * CDC, CD1 = cmin(CD0 + CDC, NCD);
        constexpr int NAc = A1 - A0, NABc = NAc * NB, NCDc = CD1 - CD0;
        if (SHARED && NCHA * NCHCD > 1 && ch % sh.csplit != sh.chunk) return;
        constexpr int EK0 = scaled_off(LC, LD, CD0), EK1 = scaled_off(LC, LD, CD1);
        constexpr int NACC = SUMS ? bra_sums(LB) : NABc;
        T acc[NACC][NCDc];
        auto clear = [&](T (&v)[NACC][NCDc]) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NACC; ++x)
#pragma unroll
                for (int y = 0; y < NCDc; ++y) v[x][y] = T(0);
        };
        clear(acc);
        // FP32: the bra primitives of a ket primitive are added up apart.  Added
        // straight to the quartet's sum, its small terms are rounded away: K of
        // 64 C/H molecules was off by 1.5e-12 rms, now 5.2e-13 (bra-outer kernel,
        // which also sums in two steps, 6.3e-13).  64 waters mixed 325 -> 339 ms.
        T part[F32 ? NACC : 1][F32 ? NCDc : 1];

        for (int j = SHARED ? sh.j0 : 0; j < nkp; j += SHARED ? sh.jstep : 1) {
            // this ket primitive, held across the bra primitives
            const double q = a.ket.p[(size_t)j * nk + ket];
            const double Kx = a.ket.P[((size_t)j * 3 + 0) * nk + ket];
            const double Ky = a.ket.P[((size_t)j * 3 + 1) * nk + ket];
            const double Kz = a.ket.P[((size_t)j * 3 + 2) * nk + ket];
            const double s0 = a.ket.S0[(size_t)j * nk + ket];
            T ek[EK1 > EK0 ? EK1 - EK0 : 1];
            const T *__restrict__ ekp = Sk + (size_t)j * NSK * nk + ket;
#pragma unroll
            for (int e = EK0; e < EK1; ++e) ek[e - EK0] = ekp[(size_t)e * nk];
            if constexpr (F32) clear(part);
            auto &sum = [&]() -> auto & {
                if constexpr (F32) return part;
                else return acc;
            }();
            for (int i = SHARED ? sh.b0 : 0; i < nbp; i += SHARED ? sh.bstep : 1) {
                const double p = rp[i * 4 + 0];
                const double X = rp[i * 4 + 1] - Kx, Y = rp[i * 4 + 2] - Ky,
                             Z = rp[i * 4 + 3] - Kz;
                T src[L + 1];
                if constexpr (F32) {
                    // FP32 tile: FP32 Taylor step, FP64 recursion and
                    // prefactor, sources rounded to FP32
                    const double rs = rsqrt_pos(p + q);
                    const double alpha = p * q * (rs * rs);
                    double F[L + 1];
                    bp.template eval<L>(alpha * (X * X + Y * Y + Z * Z), F);
                    double m = rs * s0;
#pragma unroll
                    for (int n = 0; n <= L; ++n) {
                        src[n] = (float)(F[n] * m);
                        m *= -2.0 * alpha;
                    }
                } else {
                    const double rs = rsqrt_pos(p + q);
                    const double alpha = p * q * (rs * rs);
                    double F[L + 1];
                    bp.template eval<L>(alpha * (X * X + Y * Y + Z * Z), F);
                    double m = rs * s0;
#pragma unroll
                    for (int n = 0; n <= L; ++n) {
                        src[n] = T(F[n] * m);
                        m *= -2.0 * alpha;
                    }
                }
                T r[NH];
                hermite_r<L, T>(src, T(X), T(Y), T(Z), r);
                // one ket component at a time: its ket step, then its bra step
                const ConstPtr<T> eb = re + i * NRB + (SUMS ? row_factors(LA, LB) : 0);
                static_for<NCDc>([&](auto cdl_) {
                    constexpr int cdl = decltype(cdl_)::value;
                    constexpr int cd = CD0 + cdl;
                    constexpr int bx = box_dim(LC, LD, cd, 0), by = box_dim(LC, LD, cd, 1),
                                  bz = box_dim(LC, LD, cd, 2);
                    constexpr int eo = scaled_off(LC, LD, cd);
                    T V[NHAB];
                    static_for<NHAB>([&](auto h_) {
                        constexpr int h = decltype(h_)::value;
                        const T rt = r[hidx(hidx_t(h) + bx, hidx_u(h) + by, hidx_v(h) + bz)];
                        V[h] = ((bx + by + bz) & 1) ? -rt : rt;
                    });
                    static_for<bx + 1>([&](auto ta_) {
                        constexpr int ta = decltype(ta_)::value;
                        static_for<by + 1>([&](auto nu_) {
                            constexpr int nu = decltype(nu_)::value;
                            static_for<bz + 1>([&](auto ph_) {
                                constexpr int ph = decltype(ph_)::value;
                                if constexpr (ta < bx || nu < by || ph < bz) {
                                    constexpr int e = eo + (ta * (by + 1) + nu) * (bz + 1) + ph;
                                    T ev = ek[e - EK0];
                                    if constexpr ((ta + nu + ph) & 1) ev = -ev;
                                    static_for<NHAB>([&](auto h_) {
                                        constexpr int h = decltype(h_)::value;
                                        constexpr int ri = hidx(hidx_t(h) + ta, hidx_u(h) + nu,
                                                                hidx_v(h) + ph);
                                        V[h] = fma(ev, r[ri], V[h]);
                                    });
                                }
                            });
                        });
                    });
                    if constexpr (SUMS) {
                        static_for<NACC>([&](auto k_) {
                            constexpr int k = decltype(k_)::value;
                            constexpr int f = sum_factor(LB, k), h = sum_herm(LB, k);
                            sum[k][cdl] = fma(eb[f], V[h], sum[k][cdl]);
                        });
                    } else {
                        static_for<NABc>([&](auto abl_) {
                            constexpr int abl = decltype(abl_)::value;
                            constexpr int ab = (A0 + abl / NB) * NB + abl % NB;
                            constexpr int ax = box_dim(LA, LB, ab, 0), ay = box_dim(LA, LB, ab, 1),
                                          az = box_dim(LA, LB, ab, 2);
                            constexpr int ao = box_off(LA, LB, ab);
                            static_for<ax + 1>([&](auto t_) {
                                constexpr int t = decltype(t_)::value;
                                static_for<ay + 1>([&](auto u_) {
                                    constexpr int u = decltype(u_)::value;
                                    static_for<az + 1>([&](auto v_) {
                                        constexpr int v = decltype(v_)::value;
                                        constexpr int e = ao + (t * (ay + 1) + u) * (az + 1) + v;
                                        sum[abl][cdl] = fma(eb[e], V[hidx(t, u, v)], sum[abl][cdl]);
                                    });
                                });
                            });
                        });
                    }
                });
            }
            if constexpr (F32) {
#pragma unroll
                for (int x = 0; x < NACC; ++x)
#pragma unroll
                    for (int y = 0; y < NCDc; ++y) acc[x][y] += part[x][y];
            }
        }
        T out[NABc][NCDc];
        if constexpr (SUMS) {
            constexpr int ab0 = row_ab(LA, LB);
            const T AB[3] = {re[ab0], re[ab0 + 1], re[ab0 + 2]};
            static_for<NABc * NCDc>([&](auto x_) {
                constexpr int ab = decltype(x_)::value / NCDc, y = decltype(x_)::value % NCDc;
                constexpr int i = ab / NB, j = ab % NB;
                if constexpr (LB == 0) {
                    out[ab][y] = fma(-AB[i], acc[0][y], acc[1 + i][y]);
                } else {
                    constexpr int s2 = sum_pp(i, j);
                    T v = acc[s2][y];
                    if constexpr (i == j) v += acc[1][y];
                    v = fma(AB[j], acc[5 + i][y], v);
                    out[ab][y] = fma(-AB[i], fma(AB[j], acc[0][y], acc[2 + j][y]), v);
                }
            });
        } else {
#pragma unroll
            for (int x = 0; x < NABc; ++x)
#pragma unroll
                for (int y = 0; y < NCDc; ++y) out[x][y] = acc[x][y];
        }
        if constexpr (LC == 2) {
            // the norms the scaled entries leave out (1 for s and p)
            static_for<NCDc>([&](auto cdl_) {
                constexpr int cdl = decltype(cdl_)::value;
                constexpr double nrm = comp_norm(LC, (CD0 + cdl) / ND) * comp_norm(LD, (CD0 + cdl) % ND);
                if constexpr (nrm != 1.0)
                    static_for<NABc>([&](auto abl_) { out[decltype(abl_)::value][cdl] *= T(nrm); });
            });
        }
        if constexpr (STORE) {
            if (active) {
                static_for<NABc>([&](auto abl_) {
                    constexpr int abl = decltype(abl_)::value;
                    constexpr int ia = A0 + abl / NB, ib = abl % NB;
                    static_for<NCDc>([&](auto cdl_) {
                        constexpr int cdl = decltype(cdl_)::value;
                        constexpr int ic = (CD0 + cdl) / ND, id = (CD0 + cdl) % ND;
                        a.out[soff + ia * st0 + ib * st1 + ic * st2 + id * st3] =
                            (double)out[abl][cdl];
                    });
                });
            }
        } else {
            if constexpr (SHARED) share_sum(out, sh.ls);
            digest_chunk<LA, LB, LC, LD, T, A0, A1, CD0, CD1>(
                out, D, Dk, Jb, Jk, nb, nk, Kh, N, f1, f2, f3, f4, fac, active, krow, a.kn, kl);
        }
    });
}

// Chunks of the ket-outer kernel: block, R^0 and one ket component's V are
// live at a time; KO_LIVE values leave two waves per SIMD without spills
// ((pp|pp) in two chunks instead of three, (ds|ds) in one instead of two).
constexpr int KO_LIVE = 96;
// The bra classes it serves: ss, ps, pp, ds, and dp for s and ps kets, where
// the whole block and R^0 fit at once.  Their bra step of 108 entries runs
// per primitive quartet, where the bra-outer kernel runs it per bra
// primitive, but that one needs 300 to 400 registers per lane there and
// spends as many instructions moving them.
__host__ __device__ constexpr bool ko_serves(int la, int lb, int lc, int ld) {
    return pclass(la, lb) <= KO_PCLASS_MAX || (la == 2 && lb == 1 && pclass(lc, ld) <= 1);
}
__host__ __device__ constexpr int ko_chunk(int la, int lb, int lc, int ld, bool want_a) {
    int ca = ncart(la), cdc = ncart(lc) * ncart(ld);
    const int rest = nherm(la + lb) + nherm(la + lb + lc + ld);
    while (pclass(la, lb) <= KO_PCLASS_MAX && ca * ncart(lb) * cdc + rest > KO_LIVE) {
        if (cdc > 1) cdc = (cdc + 1) / 2;
        else if (ca > 1) ca = (ca + 1) / 2;
        else break;
    }
    return want_a ? ca : cdc;
}
__host__ __device__ constexpr int ko_ca(int la, int lb, int lc, int ld) {
    return ko_chunk(la, lb, lc, ld, true);
}
__host__ __device__ constexpr int ko_cdc(int la, int lb, int lc, int ld) {
    return ko_chunk(la, lb, lc, ld, false);
}

// Blocks of the ket-outer kernel in segment mode.  One block's K' rows fill
// most of a CU's LDS for large molecules, so the block has as many waves as
// the registers allow: a live set of up to 30 values runs in 128 registers
// (16 waves, four per SIMD), up to 60 in 168 (12, three per SIMD), the rest
// in 256 (8); FP32 kernels hold two sets of sums, of half the registers.  The
// classes of total angular momentum 0 and 1 have few enough
// rows for two blocks of 8.
__host__ __device__ constexpr int ko_seg_waves(int la, int lb, int lc, int ld, bool f64) {
    const int L = la + lb + lc + ld;
    const int cdc = ko_cdc(la, lb, lc, ld);
    const bool sums = ko_sums(la, lb, (ncart(lc) * ncart(ld) + cdc - 1) / cdc, f64);
    const int rows = sums ? bra_sums(lb) : ko_ca(la, lb, lc, ld) * ncart(lb) * (f64 ? 1 : 2);
    const int live = rows * cdc + nherm(la + lb) + nherm(L);
    if (L <= 1) return 8;
    return live <= (f64 ? 30 : 60) ? 16 : (live <= (f64 ? 60 : 90) ? 12 : 8);
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE, int CA, int CDC, bool SEG,
          bool SHARED = false>
__global__ __launch_bounds__(SEG ? 64 * ko_seg_waves(LA, LB, LC, LD, !std::is_same<T, float>::value)
                                 : 256)
void k_eri_lane_ko(EriArgs a) {
    constexpr int L = LA + LB + LC + LD;
    // Boys table in LDS: FP64 rows for FP64 tiles, FP32 (5 terms, the Taylor
    // step only) for FP32 tiles, each with the exp column
    using BT = std::conditional_t<std::is_same<T, float>::value, BoysLongMixed<L>, BoysLong<L>>;
    __shared__ __align__(16) double tab[BT::SIZE];
    extern __shared__ __align__(16) unsigned char row_lds[];
    BT::stage(tab, a.boys);
    __syncthreads();
    const int wpb = blockDim.x >> 6;
    const int ntile = STORE ? a.st_ntile : a.tl.ntile;
    const BoysTable<BT> bp{tab};
    if constexpr (SEG && !STORE) {
        // segment mode: the block's waves share the bra's K' rows
        double *__restrict__ krow = (double *)row_lds;
        const long long xoff = a.xcd_stride ? xcd_index() * a.xcd_stride : 0;
        run_segments<ncart(LA), ncart(LB)>(
            a, krow, xoff, [&](int t0, int it) __attribute__((always_inline)) {
                if constexpr (SHARED)
                    ko_tile<LA, LB, LC, LD, T, STORE, CA, CDC, true>(a, TileShare(a, t0, it), bp,
                                                                     krow, true);
                else
                    ko_tile<LA, LB, LC, LD, T, STORE, CA, CDC>(a, TileShare(t0 + it), bp, krow,
                                                               true);
            });
    } else {
        for (int tile0 = blockIdx.x * wpb + (threadIdx.x >> 6); tile0 < ntile;
             tile0 += gridDim.x * wpb)
            ko_tile<LA, LB, LC, LD, T, STORE, CA, CDC>(
                a, TileShare(__builtin_amdgcn_readfirstlane(tile0)), bp);
    }
}

// ===========================================================================
// Kernel B: one wave per contracted quartet for the high-L classes (d shells).
// R^0 is built level by level in LDS with the lanes over Hermite triples,
// W_{tuv,cd} is accumulated over ket primitives with the lanes over
// (tuv, cd), and the block with the lanes over (ab, cd).
// ===========================================================================
template <int LA, int LB, int LC, int LD, typename T, bool STORE>
__global__ __launch_bounds__(64) void k_eri_wave(EriArgs a) {
    constexpr int L = LA + LB + LC + LD, LAB = LA + LB;
    constexpr int NA = ncart(LA), NB = ncart(LB), NC = ncart(LC), ND = ncart(LD);
    constexpr int NAB = NA * NB, NCD = NC * ND, NHAB = nherm(LAB), NH = nherm(L);
    constexpr int NEB = n_entries(LA, LB), NEK = n_entries(LC, LD);
    constexpr int NW = NHAB * NCD, NWL = (NW + 63) / 64;
    constexpr int NO = NAB * NCD, NOL = (NO + 63) / 64;
    constexpr int NRL = (NH + 63) / 64;
    __shared__ __align__(16) double tab[BOYS_LDS];
    __shared__ T rbuf[2][NH];
    __shared__ T wl[NW];
    __shared__ T ebl[NEB], ekl[NEK];
    // digest staging: density elements D_ab, D_cd, D_bd, D_ad, D_bc, D_ac
    // (offsets DO_*) and the J'/K' targets (offsets TG_*)
    constexpr int DO_CD = NAB, DO_BD = DO_CD + NCD, DO_AD = DO_BD + NB * ND,
                  DO_BC = DO_AD + NA * ND, DO_AC = DO_BC + NB * NC, NDEN = DO_AC + NA * NC;
    constexpr int TG_JCD = NAB, TG_KAC = TG_JCD + NCD, TG_KBC = TG_KAC + NA * NC,
                  TG_KAD = TG_KBC + NB * NC, TG_KBD = TG_KAD + NA * ND, NTGT = TG_KBD + NB * ND;
    __shared__ double blk[STORE ? 1 : NO];
    __shared__ double den[STORE ? 1 : NDEN];
    boys_stage(tab, a.boys, L);
    const int lane = threadIdx.x;

    // per-lane decode of the owned Hermite triples, W entries and block entries
    int rt[NRL], ru[NRL], rv[NRL];
#pragma unroll
    for (int k = 0; k < NRL; ++k) {
        const int id = lane + 64 * k < NH ? lane + 64 * k : 0;
        rt[k] = hidx_t(id);
        ru[k] = hidx_u(id);
        rv[k] = hidx_v(id);
    }
    int wt[NWL], wu[NWL], wv[NWL], wcd[NWL], wbx[NWL], wby[NWL], wbz[NWL], wo[NWL];
#pragma unroll
    for (int k = 0; k < NWL; ++k) {
        const int e = lane + 64 * k < NW ? lane + 64 * k : 0;
        const int h = e / NCD, cd = e % NCD;
        wt[k] = hidx_t(h);
        wu[k] = hidx_u(h);
        wv[k] = hidx_v(h);
        wcd[k] = cd;
        wbx[k] = box_dim(LC, LD, cd, 0);
        wby[k] = box_dim(LC, LD, cd, 1);
        wbz[k] = box_dim(LC, LD, cd, 2);
        wo[k] = box_off(LC, LD, cd);
    }
    int oab[NOL], ocd[NOL], obx[NOL], oby[NOL], obz[NOL], oo[NOL];
#pragma unroll
    for (int k = 0; k < NOL; ++k) {
        const int e = lane + 64 * k < NO ? lane + 64 * k : 0;
        oab[k] = e / NCD;
        ocd[k] = e % NCD;
        obx[k] = box_dim(LA, LB, oab[k], 0);
        oby[k] = box_dim(LA, LB, oab[k], 1);
        obz[k] = box_dim(LA, LB, oab[k], 2);
        oo[k] = box_off(LA, LB, oab[k]);
    }
    __syncthreads();

    const int ntile = STORE ? a.st_ntile : a.tl.ntile;
    const T *__restrict__ Eb = etab<T>(a.bra);
    const T *__restrict__ Ek = etab<T>(a.ket);
    const size_t nb = a.bra.n, nk = a.ket.n;

    const int nsub = STORE ? 1 : a.ksplit;   // ket ranges of a tile, each an item of its own
    for (int item = blockIdx.x; item < ntile * nsub; item += gridDim.x) {
        const int tile = item / nsub, sub = item - tile * nsub;
        int bra, k0 = 0, k1 = 0;
        if constexpr (STORE) {
            bra = a.st_bra[tile];
            k1 = 64;
        } else {
            const int b = tile_bra(a.tl, tile);
            bra = a.tl.bra[b];
            k0 = a.tl.ket_lo[b] + (tile - a.tl.tile_start[b]) * TILE + sub * (TILE / nsub);
            k1 = min(k0 + TILE / nsub, a.tl.ket_hi[b]);
        }
        const int nbp = a.bra.nprim[bra];
        for (int kk = k0; kk < k1; ++kk) {
            int ket = kk;
            if constexpr (STORE) {
                ket = a.st_ket[tile * 64 + kk];
                if (ket < 0) continue;
            }
            const int nkp = a.ket.nprim[ket];
            T o[NOL];
#pragma unroll
            for (int k = 0; k < NOL; ++k) o[k] = T(0);
            for (int i = 0; i < nbp; ++i) {
                const double p = a.bra.p[i * nb + bra];
                const double Px = a.bra.P[(i * 3 + 0) * nb + bra];
                const double Py = a.bra.P[(i * 3 + 1) * nb + bra];
                const double Pz = a.bra.P[(i * 3 + 2) * nb + bra];
                for (int e = lane; e < NEB; e += 64) ebl[e] = Eb[((size_t)i * NEB + e) * nb + bra];
                T w[NWL];
#pragma unroll
                for (int k = 0; k < NWL; ++k) w[k] = T(0);
                for (int j = 0; j < nkp; ++j) {
                    const double q = a.ket.p[j * nk + ket];
                    const double X = Px - a.ket.P[(j * 3 + 0) * nk + ket];
                    const double Y = Py - a.ket.P[(j * 3 + 1) * nk + ket];
                    const double Z = Pz - a.ket.P[(j * 3 + 2) * nk + ket];
                    const double pq = p + q, alpha = p * q / pq;
                    double F[L + 1];
                    boys_eval<L>(alpha * (X * X + Y * Y + Z * Z), tab, F);
                    T src[L + 1];
                    double m = 1.0 / sqrt(pq);
#pragma unroll
                    for (int n = 0; n <= L; ++n) {
                        src[n] = T(F[n] * m);
                        m *= -2.0 * alpha;
                    }
                    for (int e = lane; e < NEK; e += 64)
                        ekl[e] = Ek[((size_t)j * NEK + e) * nk + ket];
                    // R^0 level by level (level n holds totals <= L - n)
                    int cur = 0;
                    if (lane == 0) rbuf[0][0] = src[L];
                    __syncthreads();
                    for (int n = L - 1; n >= 0; --n) {
                        const int nxt = cur ^ 1, cnt = nherm(L - n);
                        const T Xt = T(X), Yt = T(Y), Zt = T(Z);
#pragma unroll
                        for (int k = 0; k < NRL; ++k) {
                            const int id = lane + 64 * k;
                            if (id < cnt) {
                                const int t = rt[k], u = ru[k], v = rv[k];
                                T val;
                                if (id == 0) val = src[n];
                                else if (t > 0)
                                    val = Xt * rbuf[cur][hidx(t - 1, u, v)] +
                                          (t > 1 ? T(t - 1) * rbuf[cur][hidx(t - 2, u, v)] : T(0));
                                else if (u > 0)
                                    val = Yt * rbuf[cur][hidx(t, u - 1, v)] +
                                          (u > 1 ? T(u - 1) * rbuf[cur][hidx(t, u - 2, v)] : T(0));
                                else
                                    val = Zt * rbuf[cur][hidx(t, u, v - 1)] +
                                          (v > 1 ? T(v - 1) * rbuf[cur][hidx(t, u, v - 2)] : T(0));
                                rbuf[nxt][id] = val;
                            }
                        }
                        cur = nxt;
                        __syncthreads();
                    }
                    const T *R = rbuf[cur];
#pragma unroll
                    for (int k = 0; k < NWL; ++k) {
                        if (lane + 64 * k < NW) {
                            T acc = w[k];
                            int e = wo[k];
                            for (int ta = 0; ta <= wbx[k]; ++ta)
                                for (int nu = 0; nu <= wby[k]; ++nu)
                                    for (int ph = 0; ph <= wbz[k]; ++ph, ++e) {
                                        const T ev = ((ta + nu + ph) & 1) ? -ekl[e] : ekl[e];
                                        acc += ev * R[hidx(wt[k] + ta, wu[k] + nu, wv[k] + ph)];
                                    }
                            w[k] = acc;
                        }
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int k = 0; k < NWL; ++k)
                    if (lane + 64 * k < NW) wl[lane + 64 * k] = w[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < NOL; ++k) {
                    if (lane + 64 * k < NO) {
                        T acc = o[k];
                        int e = oo[k];
                        for (int t = 0; t <= obx[k]; ++t)
                            for (int u = 0; u <= oby[k]; ++u)
                                for (int v = 0; v <= obz[k]; ++v, ++e)
                                    acc += ebl[e] * wl[hidx(t, u, v) * NCD + ocd[k]];
                        o[k] = acc;
                    }
                }
                __syncthreads();
            }
            // write out or digest
            if constexpr (STORE) {
                const size_t q = (size_t)tile * 64 + kk;
                const long long off = a.st_off[q];
                const int s0 = a.st_stride[q * 4 + 0], s1 = a.st_stride[q * 4 + 1],
                          s2 = a.st_stride[q * 4 + 2], s3 = a.st_stride[q * 4 + 3];
#pragma unroll
                for (int k = 0; k < NOL; ++k) {
                    if (lane + 64 * k < NO) {
                        const int ia = oab[k] / NB, ib = oab[k] % NB, ic = ocd[k] / ND,
                                  id = ocd[k] % ND;
                        a.out[off + ia * s0 + ib * s1 + ic * s2 + id * s3] = (double)o[k];
                    }
                }
            } else {
                const int mol = a.bra.mol[bra];
                const long long mbase = a.mol_off[mol];
                const int N = a.mol_n[mol];
                const double *__restrict__ D = a.D + mbase;
                const long long xoff = a.xcd_stride ? xcd_index() * a.xcd_stride : 0;
                double *__restrict__ Jb = a.Jb + xoff + bra;
                double *__restrict__ Jk = a.Jk + xoff + ket;
                double *__restrict__ Kh = a.Kh + xoff + mbase;
                const int f1 = a.bra.bf1[bra], f2 = a.bra.bf2[bra];
                const int f3 = a.ket.bf1[ket], f4 = a.ket.bf2[ket];
                double fac = 1.0;
                if (a.bra.sh1[bra] == a.bra.sh2[bra]) fac *= 0.5;
                if (a.ket.sh1[ket] == a.ket.sh2[ket]) fac *= 0.5;
                if (a.same_class && ket == bra) fac *= 0.5;
                // Reduce before scattering: the scaled block and the density
                // elements it meets go to LDS, then every J'/K' target element
                // is summed once and added with a single atomic (adding each
                // block element separately would put up to NCD lanes of one
                // instruction on the same address).
#pragma unroll
                for (int k = 0; k < NOL; ++k)
                    if (lane + 64 * k < NO) blk[lane + 64 * k] = fac * (double)o[k];
                for (int x = lane; x < NDEN; x += 64) {
                    size_t r, c;
                    if (x < DO_CD) { r = f1 + x / NB; c = f2 + x % NB; }
                    else if (x < DO_BD) { r = f3 + (x - DO_CD) / ND; c = f4 + (x - DO_CD) % ND; }
                    else if (x < DO_AD) { r = f2 + (x - DO_BD) / ND; c = f4 + (x - DO_BD) % ND; }
                    else if (x < DO_BC) { r = f1 + (x - DO_AD) / ND; c = f4 + (x - DO_AD) % ND; }
                    else if (x < DO_AC) { r = f2 + (x - DO_BC) / NC; c = f3 + (x - DO_BC) % NC; }
                    else { r = f1 + (x - DO_AC) / NC; c = f3 + (x - DO_AC) % NC; }
                    den[x] = D[r * N + c];
                }
                __syncthreads();
                for (int t = lane; t < NTGT; t += 64) {
                    double sum = 0.0;
                    if (t < TG_JCD) {   // J'_ab += 2 sum_cd v D_cd
                        for (int cd = 0; cd < NCD; ++cd) sum += blk[t * NCD + cd] * den[DO_CD + cd];
                        atomicAdd(&Jb[(size_t)t * nb], 2.0 * sum);
                    } else if (t < TG_KAC) {   // J'_cd += 2 sum_ab v D_ab
                        const int cd = t - TG_JCD;
                        for (int ab = 0; ab < NAB; ++ab) sum += blk[ab * NCD + cd] * den[ab];
                        atomicAdd(&Jk[(size_t)cd * nk], 2.0 * sum);
                    } else if (t < TG_KBC) {   // K'_ac += sum_bd v D_bd
                        const int ia = (t - TG_KAC) / NC, ic = (t - TG_KAC) % NC;
                        for (int ib = 0; ib < NB; ++ib)
                            for (int id = 0; id < ND; ++id)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_BD + ib * ND + id];
                        atomicAdd(&Kh[(size_t)(f1 + ia) * N + f3 + ic], sum);
                    } else if (t < TG_KAD) {   // K'_bc += sum_ad v D_ad
                        const int ib = (t - TG_KBC) / NC, ic = (t - TG_KBC) % NC;
                        for (int ia = 0; ia < NA; ++ia)
                            for (int id = 0; id < ND; ++id)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_AD + ia * ND + id];
                        atomicAdd(&Kh[(size_t)(f2 + ib) * N + f3 + ic], sum);
                    } else if (t < TG_KBD) {   // K'_ad += sum_bc v D_bc
                        const int ia = (t - TG_KAD) / ND, id = (t - TG_KAD) % ND;
                        for (int ib = 0; ib < NB; ++ib)
                            for (int ic = 0; ic < NC; ++ic)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_BC + ib * NC + ic];
                        atomicAdd(&Kh[(size_t)(f1 + ia) * N + f4 + id], sum);
                    } else {   // K'_bd += sum_ac v D_ac
                        const int ib = (t - TG_KBD) / ND, id = (t - TG_KBD) % ND;
                        for (int ia = 0; ia < NA; ++ia)
                            for (int ic = 0; ic < NC; ++ic)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_AC + ia * NC + ic];
                        atomicAdd(&Kh[(size_t)(f2 + ib) * N + f4 + id], sum);
                    }
                }
                __syncthreads();
            }
        }
    }
}

// ===========================================================================
// Kernel C: one wave per contracted quartet with both E.R.E steps on the
// matrix cores (16x16x4 MFMA, FP64 or FP32).  Per primitive quartet,
//   W[h_ab][cd] += sum_{h_cd} R^0[h_ab + h_cd] Et[h_cd][cd]     (step 1)
// with Et the ket Hermite entries carrying (-1)^{tau+nu+phi} (zero outside a
// component pair's box); per bra primitive pair,
//   (ab|cd)     += sum_{h_ab} E[ab][h_ab] W[h_ab][cd]            (step 2).
// Both are dense products over the Hermite index, the J_{tuv,k} form of
// Sec. 2.5 (Eq. eri-tensor-contracted) written as matrix products.
// Operand layout of v_mfma_{f64,f32}_16x16x4 (lane l): A[l % 16][l / 16],
// B[l / 16][l % 16]; accumulator v of lane l holds D[l / 16 + 4 v][l % 16]
// for FP64 and D[4 (l / 16) + v][l % 16] for FP32.
// ===========================================================================
typedef double mfma_v4d __attribute__((ext_vector_type(4)));
typedef float mfma_v4f __attribute__((ext_vector_type(4)));
template <typename T>
struct MfmaOp;
template <>
struct MfmaOp<double> {
    using acc = mfma_v4d;
    static __device__ __forceinline__ acc mma(double x, double y, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};
template <>
struct MfmaOp<float> {
    using acc = mfma_v4f;
    static __device__ __forceinline__ acc mma(float x, float y, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// F_0..F_L at T from the FP64 grid in global memory (wave-uniform reads).
template <int L>
__device__ __forceinline__ void boys_eval_global(double T, const double *__restrict__ g, double *F) {
    if (T < BOYS_TMAX) {
        const int k = __double2int_rn(T * BOYS_INV_DT);
        const double d = k * BOYS_DT - T;
        const double *c = g + k * BOYS_NORD + L;
        double f = c[BOYS_NTAYLOR - 1] * inv_factorial(BOYS_NTAYLOR - 1);
#pragma unroll
        for (int j = BOYS_NTAYLOR - 2; j >= 0; --j) f = fma(f, d, c[j] * inv_factorial(j));
        F[L] = f;
        if constexpr (L > 0) {
            const double e = exp(-T), t2 = 2.0 * T;
#pragma unroll
            for (int n = L; n > 0; --n) F[n - 1] = fma(t2, F[n], e) * (1.0 / (2 * n - 1));
        }
    } else {
        F[0] = 0.88622692545275801365 * rsqrt(T);
        if constexpr (L > 0) {
            const double e = exp(-T), h = 0.5 / T;
#pragma unroll
            for (int n = 0; n < L; ++n) F[n + 1] = ((2 * n + 1) * F[n] - e) * h;
        }
    }
}

// Index maps of kernel C, evaluated at compile time: building them in every
// block cost a lone (dd|dd) quartet 0.61 ms (now 0.04).
template <int LA, int LB, int LC, int LD>
struct MfmaMaps {
    static constexpr int NHAB = nherm(LA + LB), NHCD = nherm(LC + LD);
    static constexpr int NH = nherm(LA + LB + LC + LD);
    static constexpr int NAB = ncart(LA) * ncart(LB), NCD = ncart(LC) * ncart(LD);
    static constexpr int MR1 = (NHAB + 15) / 16 * 16, KR = (NHCD + 3) / 4 * 4;
    static constexpr int NC16 = (NCD + 15) / 16 * 16;
    static constexpr int MR2 = (NAB + 15) / 16 * 16, KR2 = (NHAB + 3) / 4 * 4;
    short rmap[MR1 * KR] = {};     // R^0 index of (h_ab, h_cd), -1 in the padding
    short kmap[KR * NC16] = {};    // +-(ket entry + 1) with the Hermite sign, 0 outside
    short bmap[MR2 * KR2] = {};    // bra entry + 1, 0 outside
    int tuv[NH] = {};              // t | u << 8 | v << 16

    constexpr MfmaMaps() {
        constexpr int L = LA + LB + LC + LD;
        for (int t = 0; t <= L; ++t)
            for (int u = 0; u <= L - t; ++u)
                for (int v = 0; v <= L - t - u; ++v) tuv[hidx(t, u, v)] = t | u << 8 | v << 16;
        for (int r = 0; r < MR1; ++r)
            for (int k = 0; k < KR; ++k) {
                int id = -1;
                if (r < NHAB && k < NHCD) {
                    const int s = tuv[r] + tuv[k];   // the sums stay below 256
                    id = hidx(s & 255, (s >> 8) & 255, s >> 16);
                }
                rmap[r * KR + k] = (short)id;
            }
        int o = 0;
        for (int n = 0; n < NCD; ++n) {
            const int bx = box_dim(LC, LD, n, 0), by = box_dim(LC, LD, n, 1),
                      bz = box_dim(LC, LD, n, 2);
            for (int t = 0; t <= bx; ++t)
                for (int u = 0; u <= by; ++u)
                    for (int v = 0; v <= bz; ++v) {
                        ++o;
                        kmap[hidx(t, u, v) * NC16 + n] = (short)(((t + u + v) & 1) ? -o : o);
                    }
        }
        o = 0;
        for (int m = 0; m < NAB; ++m) {
            const int bx = box_dim(LA, LB, m, 0), by = box_dim(LA, LB, m, 1),
                      bz = box_dim(LA, LB, m, 2);
            for (int t = 0; t <= bx; ++t)
                for (int u = 0; u <= by; ++u)
                    for (int v = 0; v <= bz; ++v) bmap[m * KR2 + hidx(t, u, v)] = (short)++o;
        }
    }
};
template <int LA, int LB, int LC, int LD>
__device__ const MfmaMaps<LA, LB, LC, LD> mfma_maps{};

template <int LA, int LB, int LC, int LD, typename T, bool STORE>
__global__ __launch_bounds__(64) void k_eri_mfma(EriArgs a) {
    constexpr int L = LA + LB + LC + LD, LAB = LA + LB, LCD = LC + LD;
    constexpr int NA = ncart(LA), NB = ncart(LB), NC = ncart(LC), ND = ncart(LD);
    constexpr int NAB = NA * NB, NCD = NC * ND;
    constexpr int NHAB = nherm(LAB), NHCD = nherm(LCD), NH = nherm(L);
    constexpr int NEB = n_entries(LA, LB), NEK = n_entries(LC, LD);
    constexpr int MT1 = (NHAB + 15) / 16, NT = (NCD + 15) / 16, KS1 = (NHCD + 3) / 4;
    constexpr int MT2 = (NAB + 15) / 16, KS2 = (NHAB + 3) / 4;
    constexpr int KR = KS1 * 4, NC16 = NT * 16, MR2 = MT2 * 16, KR2 = KS2 * 4;
    constexpr int NO = NAB * NCD, NRL = (NH + 63) / 64;
    using M = MfmaOp<T>;
    using acc_t = typename M::acc;
    // digest staging (as kernel B): density blocks and J'/K' targets
    constexpr int DO_CD = NAB, DO_BD = DO_CD + NCD, DO_AD = DO_BD + NB * ND,
                  DO_BC = DO_AD + NA * ND, DO_AC = DO_BC + NB * NC, NDEN = DO_AC + NA * NC;
    constexpr int TG_JCD = NAB, TG_KAC = TG_JCD + NCD, TG_KBC = TG_KAC + NA * NC,
                  TG_KAD = TG_KBC + NB * NC, TG_KBD = TG_KAD + NA * ND, NTGT = TG_KBD + NB * ND;
    constexpr int NWST = (KR2 * NC16 * (int)sizeof(T) + 7) / 8;   // W staging, in doubles
    constexpr int NU = STORE ? NWST : (NWST > NO ? NWST : NO);
    __shared__ T rbuf[2][NH];
    __shared__ T ekl[NEK], ebl[NEB];
    constexpr int MR1 = MT1 * 16;
    __shared__ short rmap[MR1][KR];    // R^0 index of (h_ab, h_cd), -1 in the padding
    __shared__ short kmap[KR][NC16];   // +-(ket entry + 1) with the Hermite sign, 0 outside
    __shared__ short bmap[MR2][KR2];   // bra entry + 1, 0 outside
    __shared__ double ubuf[NU];        // W staging, then the scaled block for the digest
    __shared__ double den[STORE ? 1 : NDEN];
    T *wst = (T *)ubuf;
    const int lane = threadIdx.x;

    const MfmaMaps<LA, LB, LC, LD> &maps = mfma_maps<LA, LB, LC, LD>;
    for (int x = lane; x < KR * NC16; x += 64) (&kmap[0][0])[x] = maps.kmap[x];
    for (int x = lane; x < MR2 * KR2; x += 64) (&bmap[0][0])[x] = maps.bmap[x];
    for (int x = lane; x < MR1 * KR; x += 64) (&rmap[0][0])[x] = maps.rmap[x];
    // level decode of the R recursion (as kernel B)
    int rt[NRL], ru[NRL], rv[NRL];
#pragma unroll
    for (int k = 0; k < NRL; ++k) {
        const int q = maps.tuv[lane + 64 * k < NH ? lane + 64 * k : 0];
        rt[k] = q & 255;
        ru[k] = (q >> 8) & 255;
        rv[k] = q >> 16;
    }
    __syncthreads();

    const int ntile = STORE ? a.st_ntile : a.tl.ntile;
    const T *__restrict__ Eb = etab<T>(a.bra);
    const T *__restrict__ Ek = etab<T>(a.ket);
    const size_t nb = a.bra.n, nk = a.ket.n;

    const int nsub = STORE ? 1 : a.ksplit;   // ket ranges of a tile, each an item of its own
    for (int item = blockIdx.x; item < ntile * nsub; item += gridDim.x) {
        const int tile = item / nsub, sub = item - tile * nsub;
        int bra, k0 = 0, k1 = 0;
        if constexpr (STORE) {
            bra = a.st_bra[tile];
            k1 = 64;
        } else {
            const int b = tile_bra(a.tl, tile);
            bra = a.tl.bra[b];
            k0 = a.tl.ket_lo[b] + (tile - a.tl.tile_start[b]) * TILE + sub * (TILE / nsub);
            k1 = min(k0 + TILE / nsub, a.tl.ket_hi[b]);
        }
        const int nbp = a.bra.nprim[bra];
        for (int kk = k0; kk < k1; ++kk) {
            int ket = kk;
            if constexpr (STORE) {
                ket = a.st_ket[tile * 64 + kk];
                if (ket < 0) continue;
            }
            const int nkp = a.ket.nprim[ket];
            acc_t o[MT2][NT];
#pragma unroll
            for (int mt = 0; mt < MT2; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) o[mt][nt] = acc_t{};
            for (int i = 0; i < nbp; ++i) {
                const double p = a.bra.p[i * nb + bra];
                const double Px = a.bra.P[(i * 3 + 0) * nb + bra];
                const double Py = a.bra.P[(i * 3 + 1) * nb + bra];
                const double Pz = a.bra.P[(i * 3 + 2) * nb + bra];
                for (int e = lane; e < NEB; e += 64) ebl[e] = Eb[((size_t)i * NEB + e) * nb + bra];
                acc_t w[MT1][NT];
#pragma unroll
                for (int mt = 0; mt < MT1; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) w[mt][nt] = acc_t{};
                for (int j = 0; j < nkp; ++j) {
                    const double q = a.ket.p[j * nk + ket];
                    const double X = Px - a.ket.P[(j * 3 + 0) * nk + ket];
                    const double Y = Py - a.ket.P[(j * 3 + 1) * nk + ket];
                    const double Z = Pz - a.ket.P[(j * 3 + 2) * nk + ket];
                    const double pq = p + q, alpha = p * q / pq;
                    double F[L + 1];
                    boys_eval_global<L>(alpha * (X * X + Y * Y + Z * Z), a.boys, F);
                    T src[L + 1];
                    double m = 1.0 / sqrt(pq);
#pragma unroll
                    for (int n = 0; n <= L; ++n) {
                        src[n] = T(F[n] * m);
                        m *= -2.0 * alpha;
                    }
                    for (int e = lane; e < NEK; e += 64)
                        ekl[e] = Ek[((size_t)j * NEK + e) * nk + ket];
                    // R^0 level by level (level n holds totals <= L - n)
                    int cur = 0;
                    if (lane == 0) rbuf[0][0] = src[L];
                    __syncthreads();
                    for (int n = L - 1; n >= 0; --n) {
                        const int nxt = cur ^ 1, cnt = nherm(L - n);
                        const T Xt = T(X), Yt = T(Y), Zt = T(Z);
#pragma unroll
                        for (int k = 0; k < NRL; ++k) {
                            const int id = lane + 64 * k;
                            if (id < cnt) {
                                const int t = rt[k], u = ru[k], v = rv[k];
                                T val;
                                if (id == 0) val = src[n];
                                else if (t > 0)
                                    val = Xt * rbuf[cur][hidx(t - 1, u, v)] +
                                          (t > 1 ? T(t - 1) * rbuf[cur][hidx(t - 2, u, v)] : T(0));
                                else if (u > 0)
                                    val = Yt * rbuf[cur][hidx(t, u - 1, v)] +
                                          (u > 1 ? T(u - 1) * rbuf[cur][hidx(t, u - 2, v)] : T(0));
                                else
                                    val = Zt * rbuf[cur][hidx(t, u, v - 1)] +
                                          (v > 1 ? T(v - 1) * rbuf[cur][hidx(t, u, v - 2)] : T(0));
                                rbuf[nxt][id] = val;
                            }
                        }
                        cur = nxt;
                        __syncthreads();
                    }
                    const T *R = rbuf[cur];
                    // step 1 on the matrix cores (K steps not unrolled: the
                    // operands of one step are loaded just before its MFMAs)
#pragma unroll 1
                    for (int ks = 0; ks < KS1; ++ks) {
                        T bv[NT];
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const int mk = kmap[4 * ks + (lane >> 4)][16 * nt + (lane & 15)];
                            bv[nt] = mk == 0 ? T(0) : (mk > 0 ? ekl[mk - 1] : -ekl[-mk - 1]);
                        }
#pragma unroll
                        for (int mt = 0; mt < MT1; ++mt) {
                            const int ri = rmap[16 * mt + (lane & 15)][4 * ks + (lane >> 4)];
                            const T av = ri >= 0 ? R[ri] : T(0);
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) w[mt][nt] = M::mma(av, bv[nt], w[mt][nt]);
                        }
                    }
                    __syncthreads();   // rbuf and ekl are rewritten by the next ket primitive
                }
                // W to LDS in the B-operand order of step 2 (rows h_ab < KR2)
#pragma unroll
                for (int mt = 0; mt < MT1; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int r = 16 * mt + M::row(lane, v);
                            if (r < KR2) wst[r * NC16 + 16 * nt + (lane & 15)] = w[mt][nt][v];
                        }
                __syncthreads();
                // step 2 on the matrix cores
#pragma unroll 1
                for (int ks = 0; ks < KS2; ++ks) {
                    T bv[NT];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        bv[nt] = wst[(4 * ks + (lane >> 4)) * NC16 + 16 * nt + (lane & 15)];
#pragma unroll
                    for (int mt = 0; mt < MT2; ++mt) {
                        const int mb = bmap[16 * mt + (lane & 15)][4 * ks + (lane >> 4)];
                        const T av = mb ? ebl[mb - 1] : T(0);
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) o[mt][nt] = M::mma(av, bv[nt], o[mt][nt]);
                    }
                }
                __syncthreads();   // wst and ebl are rewritten by the next bra primitive
            }
            if constexpr (STORE) {
                const size_t qq = (size_t)tile * 64 + kk;
                const long long off = a.st_off[qq];
                const int s0 = a.st_stride[qq * 4 + 0], s1 = a.st_stride[qq * 4 + 1],
                          s2 = a.st_stride[qq * 4 + 2], s3 = a.st_stride[qq * 4 + 3];
#pragma unroll
                for (int mt = 0; mt < MT2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int ab = 16 * mt + M::row(lane, v), cd = 16 * nt + (lane & 15);
                            if (ab < NAB && cd < NCD)
                                a.out[off + (ab / NB) * s0 + (ab % NB) * s1 + (cd / ND) * s2 +
                                      (cd % ND) * s3] = (double)o[mt][nt][v];
                        }
            } else {
                const int mol = a.bra.mol[bra];
                const long long mbase = a.mol_off[mol];
                const int N = a.mol_n[mol];
                const double *__restrict__ D = a.D + mbase;
                const long long xoff = a.xcd_stride ? xcd_index() * a.xcd_stride : 0;
                double *__restrict__ Jb = a.Jb + xoff + bra;
                double *__restrict__ Jk = a.Jk + xoff + ket;
                double *__restrict__ Kh = a.Kh + xoff + mbase;
                const int f1 = a.bra.bf1[bra], f2 = a.bra.bf2[bra];
                const int f3 = a.ket.bf1[ket], f4 = a.ket.bf2[ket];
                double fac = 1.0;
                if (a.bra.sh1[bra] == a.bra.sh2[bra]) fac *= 0.5;
                if (a.ket.sh1[ket] == a.ket.sh2[ket]) fac *= 0.5;
                if (a.same_class && ket == bra) fac *= 0.5;
                double *blk = ubuf;
#pragma unroll
                for (int mt = 0; mt < MT2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int ab = 16 * mt + M::row(lane, v), cd = 16 * nt + (lane & 15);
                            if (ab < NAB && cd < NCD) blk[ab * NCD + cd] = fac * (double)o[mt][nt][v];
                        }
                for (int x = lane; x < NDEN; x += 64) {
                    size_t r, c;
                    if (x < DO_CD) { r = f1 + x / NB; c = f2 + x % NB; }
                    else if (x < DO_BD) { r = f3 + (x - DO_CD) / ND; c = f4 + (x - DO_CD) % ND; }
                    else if (x < DO_AD) { r = f2 + (x - DO_BD) / ND; c = f4 + (x - DO_BD) % ND; }
                    else if (x < DO_BC) { r = f1 + (x - DO_AD) / ND; c = f4 + (x - DO_AD) % ND; }
                    else if (x < DO_AC) { r = f2 + (x - DO_BC) / NC; c = f3 + (x - DO_BC) % NC; }
                    else { r = f1 + (x - DO_AC) / NC; c = f3 + (x - DO_AC) % NC; }
                    den[x] = D[r * N + c];
                }
                __syncthreads();
                for (int t = lane; t < NTGT; t += 64) {
                    double sum = 0.0;
                    if (t < TG_JCD) {   // J'_ab += 2 sum_cd v D_cd
#pragma unroll 2
                        for (int cd = 0; cd < NCD; ++cd) sum += blk[t * NCD + cd] * den[DO_CD + cd];
                        atomicAdd(&Jb[(size_t)t * nb], 2.0 * sum);
                    } else if (t < TG_KAC) {   // J'_cd += 2 sum_ab v D_ab
                        const int cd = t - TG_JCD;
#pragma unroll 2
                        for (int ab = 0; ab < NAB; ++ab) sum += blk[ab * NCD + cd] * den[ab];
                        atomicAdd(&Jk[(size_t)cd * nk], 2.0 * sum);
                    } else if (t < TG_KBC) {   // K'_ac += sum_bd v D_bd
                        const int ia = (t - TG_KAC) / NC, ic = (t - TG_KAC) % NC;
#pragma unroll 1
                        for (int ib = 0; ib < NB; ++ib)
                            for (int id = 0; id < ND; ++id)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_BD + ib * ND + id];
                        atomicAdd(&Kh[(size_t)(f1 + ia) * N + f3 + ic], sum);
                    } else if (t < TG_KAD) {   // K'_bc += sum_ad v D_ad
                        const int ib = (t - TG_KBC) / NC, ic = (t - TG_KBC) % NC;
#pragma unroll 1
                        for (int ia = 0; ia < NA; ++ia)
                            for (int id = 0; id < ND; ++id)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_AD + ia * ND + id];
                        atomicAdd(&Kh[(size_t)(f2 + ib) * N + f3 + ic], sum);
                    } else if (t < TG_KBD) {   // K'_ad += sum_bc v D_bc
                        const int ia = (t - TG_KAD) / ND, id = (t - TG_KAD) % ND;
#pragma unroll 1
                        for (int ib = 0; ib < NB; ++ib)
                            for (int ic = 0; ic < NC; ++ic)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_BC + ib * NC + ic];
                        atomicAdd(&Kh[(size_t)(f1 + ia) * N + f4 + id], sum);
                    } else {   // K'_bd += sum_ac v D_ac
                        const int ib = (t - TG_KBD) / ND, id = (t - TG_KBD) % ND;
#pragma unroll 1
                        for (int ia = 0; ia < NA; ++ia)
                            for (int ic = 0; ic < NC; ++ic)
                                sum += blk[(ia * NB + ib) * NCD + ic * ND + id] * den[DO_AC + ia * NC + ic];
                        atomicAdd(&Kh[(size_t)(f2 + ib) * N + f4 + id], sum);
                    }
                }
                __syncthreads();   // blk and den are rewritten by the next quartet
            }
        }
    }
}

// Launch variants.  Variants 0..2 fix the per-lane register budget of kernel
// A (live block + W + R^0 values; the chunking follows from it); variant 3 is
// kernel B; variant 4 is kernel A in ket-outer order (the classes ko_serves
// names; others run variant 1).  A budget whose chunking does not fit, or
// needs more than MAX_CHUNKS chunks, falls back to kernel B.  The autotuner
// picks a variant and the waves per block for every class and precision.
constexpr int NVARIANT = 7;
constexpr int VARIANT_WAVE = 3;
constexpr int VARIANT_KO = 4;
constexpr int VARIANT_WIDE = 5;   // kernel A at 192 live values, where 160 does not fit
constexpr int VARIANT_MFMA = 6;   // kernel C (matrix cores), classes with a d bra
constexpr int DEFAULT_VARIANT = 1;
__host__ __device__ constexpr int variant_budget(int v) {
    return v == 0 ? 96 : (v == 1 ? 128 : (v == 2 ? 160 : (v == VARIANT_WIDE ? 192 : 0)));
}
constexpr int MAX_CHUNKS = 24;

// LDS per wave for the staged bra primitives of the bra-outer lane kernel
constexpr int STAGE_BYTES = 3072;
template <int LA, int LB, int LC, int LD, int BUDGET>
__host__ __device__ constexpr bool lane_fits() {
    return BUDGET > 0 &&
           lane_live(LA, LB, LC, LD, chunk_a(LA, LB, LC, LD, BUDGET),
                     chunk_cd(LA, LB, LC, LD, BUDGET)) <= BUDGET &&
           n_chunks(LA, LB, LC, LD, BUDGET) <= MAX_CHUNKS;
}

// The widest budget at which a class has a lane kernel of its own (variant 5).
template <int LA, int LB, int LC, int LD>
__host__ __device__ constexpr int widest_budget() {
    constexpr int b2 = variant_budget(2), b5 = variant_budget(VARIANT_WIDE);
    if (!lane_fits<LA, LB, LC, LD, b2>()) return b5;
    return lane_fits<LA, LB, LC, LD, b5>() &&
                   n_chunks(LA, LB, LC, LD, b5) < n_chunks(LA, LB, LC, LD, b2)
               ? b5
               : b2;
}

// Launches of fewer than SHARE_WAVES tiles, three waves for every SIMD of the
// GPU, are shared out until they have about as many items: by chunks first,
// which repeat no work, then by ket primitives, then by bra primitives, which
// repeat the digest (nchunk = 0: not shared out).  Launch times summed, FP64:
// 3 waters 12.8 -> 0.79 ms, 10 waters 29.9 -> 6.1 ms, of which the kernels a
// class runs by default account for the step to 3.2 and 9.3 ms.  The kernels
// for it are instantiations of their own: with the loop bounds in registers
// the large launches ran up to a quarter slower ((dp|pp) 41.7 -> 49.6 ms).
constexpr int SHARE_WAVES = 3072;
inline void share_tiles(EriArgs &b, int nchunk, int waves) {
    long long n = b.tl.ntile;
    b.csplit = b.ksplit = b.bsplit = b.parts = b.shares = 1;
    if (n >= SHARE_WAVES || nchunk < 1) return;
    auto want = [&] { return (int)((SHARE_WAVES + n / 2) / n); };
    if (want() > 1) n *= b.csplit = cmin(nchunk, want());
    while (want() > 1 && b.ksplit < 8 && b.ksplit < b.ket.kmax) {
        b.ksplit *= 2;
        n *= 2;
    }
    if (want() > 1) n *= b.bsplit = cmin(b.bra.kmax > 1 ? b.bra.kmax : 1, want());
    // every part of a segment keeps an item for each of its waves
    const long long per = n / b.tl.nseg / waves;
    b.parts = per > 1 ? (int)per : 1;
    b.shares = b.csplit * b.ksplit * b.bsplit;
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE>
void launch_wave_kernel(int ntile, const EriArgs &a, hipStream_t s) {
    EriArgs b = a;
    b.ksplit = 1;
    if (!STORE)
        while (ntile * b.ksplit < SHARE_WAVES && b.ksplit < TILE) b.ksplit *= 2;
    int blocks = ntile * b.ksplit;
    if (blocks > 32768) blocks = 32768;
    hipLaunchKernelGGL((k_eri_wave<LA, LB, LC, LD, T, STORE>), dim3(blocks), dim3(64), 0, s, b);
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE>
void launch_mfma_kernel(int ntile, const EriArgs &a, hipStream_t s) {
    EriArgs b = a;
    b.ksplit = 1;
    if (!STORE)
        while (ntile * b.ksplit < SHARE_WAVES && b.ksplit < TILE) b.ksplit *= 2;
    int blocks = ntile * b.ksplit;
    if (blocks > 32768) blocks = 32768;
    hipLaunchKernelGGL((k_eri_mfma<LA, LB, LC, LD, T, STORE>), dim3(blocks), dim3(64), 0, s, b);
}

// LDS of one workgroup on gfx950.
constexpr size_t LDS_PER_CU = 160 * 1024;

// Segment mode of a lane-kernel launch (waves_per_block = 8 in a Fock build
// with a.kn > 0 and a segment list): blocks over segments, the dynamic LDS
// holding the waves' staging slices and the bra's K' rows.  False (the
// caller then launches the tile-mode kernel with kn = 0) when the rows do not
// fit next to the kernel's static LDS.
//
// cuw: waves a CU holds by the kernel's registers.  W comes in as the most a
// block may have and leaves as what it gets: 4 or 8 where enough such blocks
// fit the CU's LDS to keep it as full, since the waves of a block wait for
// each other at the end of every segment and the segments of small molecules
// are short (1024 C/H molecules, 5.8 tiles each: 362 -> 301 ms per build, 64 of
// them in mixed precision 44 -> 28).
template <int LA, int LB>
bool segment_fit(const void *kernel, int cuw, int &W, int nchunk, EriArgs &b, int &blocks,
                 size_t &dyn) {
    if (b.kn <= 0 || b.tl.nseg <= 0) return false;
    const size_t rows = (size_t)(ncart(LA) + ncart(LB)) * b.kn * sizeof(double);
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, kernel) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    auto lds = [&](int w) { return fa.sharedSizeBytes + (size_t)w * b.stage_bytes + rows; };
    if (lds(W) > LDS_PER_CU) return false;
    auto held = [&](int w) { return cmin(cuw / w, (int)(LDS_PER_CU / lds(w))) * w; };
    const int most = W;
    int best = held(most);
    for (int w = 4; w < most; w *= 2)
        if (held(w) > best) best = held(w);
    for (int w = 4; w < most; w *= 2)
        if (held(w) == best) {
            W = w;
            break;
        }
    dyn = (size_t)W * b.stage_bytes + rows;
    share_tiles(b, nchunk, W);
    const long long n = (long long)b.tl.nseg * b.parts;
    blocks = n < 8192 ? (int)n : 8192;
    return true;
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE, int BUDGET>
void launch_budget(int ntile, int wpb, const EriArgs &a, hipStream_t s) {
    if constexpr (lane_fits<LA, LB, LC, LD, BUDGET>()) {
        constexpr int CA = chunk_a(LA, LB, LC, LD, BUDGET), CDC = chunk_cd(LA, LB, LC, LD, BUDGET);
        int blocks = 0;
        // LDS stage of the bra primitives: up to STAGE_BYTES per wave
        constexpr int per_prim = 4 * (int)sizeof(double) + n_entries(LA, LB) * (int)sizeof(T);
        EriArgs b = a;
        b.stage_prims = STAGE_BYTES / per_prim < 1 ? 1 : STAGE_BYTES / per_prim;
        if (b.stage_prims > a.bra.kmax) b.stage_prims = a.bra.kmax > 0 ? a.bra.kmax : 1;
        b.stage_bytes = LA == 2 ? (b.stage_prims * per_prim + 15) / 16 * 16 : 0;
        if constexpr (!STORE) {
            if (wpb == 8) {
                int W = seg_waves(LA, LB, LC, LD, CA, CDC);
                // the shared form exists at the widest budget, the default's
                constexpr bool WIDEST = BUDGET == widest_budget<LA, LB, LC, LD>();
                const bool share = WIDEST && ntile < SHARE_WAVES;
                auto seg = share ? k_eri_lane<LA, LB, LC, LD, T, false, CA, CDC, true, WIDEST>
                                 : k_eri_lane<LA, LB, LC, LD, T, false, CA, CDC, true, false>;
                int sblocks = 0;
                size_t dyn = 0;
                if (segment_fit<LA, LB>((const void *)seg, W, W,
                                        share ? n_chunks(LA, LB, LC, LD, BUDGET) : 0, b, sblocks,
                                        dyn)) {
                    hipLaunchKernelGGL(seg, dim3(sblocks), dim3(64 * W), dyn, s, b);
                    return;
                }
            }
        }
        b.kn = 0;
        const int w = wpb > 4 ? 4 : wpb;
        blocks = (ntile + w - 1) / w;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL((k_eri_lane<LA, LB, LC, LD, T, STORE, CA, CDC, false>), dim3(blocks),
                           dim3(64 * w), (size_t)w * b.stage_bytes, s, b);
    } else {
        launch_wave_kernel<LA, LB, LC, LD, T, STORE>(ntile, a, s);
    }
}

template <int LA, int LB, int LC, int LD, typename T, bool STORE>
void launch_ko(int ntile, int wpb, const EriArgs &a, hipStream_t s) {
    if constexpr (ko_serves(LA, LB, LC, LD)) {
        constexpr int CA = ko_ca(LA, LB, LC, LD), CDC = ko_cdc(LA, LB, LC, LD);
        EriArgs b = a;
        b.stage_prims = b.stage_bytes = 0;
        if constexpr (!STORE) {
            if (wpb == 8) {
                auto seg = ntile < SHARE_WAVES
                               ? k_eri_lane_ko<LA, LB, LC, LD, T, false, CA, CDC, true, true>
                               : k_eri_lane_ko<LA, LB, LC, LD, T, false, CA, CDC, true, false>;
                int W = ko_seg_waves(LA, LB, LC, LD, !std::is_same<T, float>::value);
                int sblocks = 0;
                size_t dyn = 0;
                constexpr int NCH =
                    ((ncart(LA) + CA - 1) / CA) * ((ncart(LC) * ncart(LD) + CDC - 1) / CDC);
                const int cuw = LA + LB + LC + LD <= 1 ? 16 : W;
                if (segment_fit<LA, LB>((const void *)seg, cuw, W, NCH, b, sblocks, dyn)) {
                    hipLaunchKernelGGL(seg, dim3(sblocks), dim3(64 * W), dyn, s, b);
                    return;
                }
            }
        }
        b.kn = 0;
        const int w = wpb > 4 ? 4 : wpb;
        int blocks = (ntile + w - 1) / w;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL((k_eri_lane_ko<LA, LB, LC, LD, T, STORE, CA, CDC, false>), dim3(blocks),
                           dim3(64 * w), 0, s, b);
    } else {
        launch_budget<LA, LB, LC, LD, T, STORE, variant_budget(DEFAULT_VARIANT)>(ntile, wpb, a, s);
    }
}

// One variant in Fock mode (STORE = false) or store mode (the same kernel
// code writing the contracted blocks out instead of digesting them).
template <int LA, int LB, int LC, int LD, typename T, bool STORE>
void launch_variant(int ntile, int variant, int wpb, const EriArgs &a, hipStream_t s) {
    switch (variant) {
        case 0: launch_budget<LA, LB, LC, LD, T, STORE, variant_budget(0)>(ntile, wpb, a, s); break;
        case 1: launch_budget<LA, LB, LC, LD, T, STORE, variant_budget(1)>(ntile, wpb, a, s); break;
        case 2: launch_budget<LA, LB, LC, LD, T, STORE, variant_budget(2)>(ntile, wpb, a, s); break;
        case VARIANT_KO: launch_ko<LA, LB, LC, LD, T, STORE>(ntile, wpb, a, s); break;
        case VARIANT_WIDE:
            // a 192-value lane kernel for the classes whose smallest chunk
            // exceeds 160 live values, or that need fewer chunks at 192
            // ((ds|pp), (dp|pp), (dp|ds): each chunk re-evaluates Boys and
            // R, and these run at one wave per SIMD either way); every other
            // class runs variant 2
            launch_budget<LA, LB, LC, LD, T, STORE, widest_budget<LA, LB, LC, LD>()>(ntile, wpb, a,
                                                                                     s);
            break;
        case VARIANT_MFMA:
            // the matrix-core kernel serves classes with a d bra; the others
            // run the wave kernel
            if constexpr (LA == 2) launch_mfma_kernel<LA, LB, LC, LD, T, STORE>(ntile, a, s);
            else launch_wave_kernel<LA, LB, LC, LD, T, STORE>(ntile, a, s);
            break;
        default: launch_wave_kernel<LA, LB, LC, LD, T, STORE>(ntile, a, s); break;
    }
}

template <int LA, int LB, int LC, int LD, typename T>
hipError_t launch_class(bool store, int variant, int wpb, const EriArgs &a, hipStream_t s) {
    const int ntile = store ? a.st_ntile : a.tl.ntile;
    if (ntile <= 0) return hipSuccess;
    if (wpb != 1 && wpb != 2 && wpb != 4 && wpb != 8) wpb = 4;
    if (store) launch_variant<LA, LB, LC, LD, T, true>(ntile, variant, wpb, a, s);
    else launch_variant<LA, LB, LC, LD, T, false>(ntile, variant, wpb, a, s);
    return hipGetLastError();
}

}  // namespace fsim
