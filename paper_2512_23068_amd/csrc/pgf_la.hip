// libpgf: decaying linear attention with its tangent flow (App. F: linear
// transformers, RetNet and RWKV-6 as general linear recurrences) for gfx950.
//
// The state of one (batch, head) is a dk x dv matrix S.  A block owns 64 value
// columns of one head and takes a segment in chunks of 16 steps.  Within a
// chunk, with G_t the sum of g up to and including step t (per key), the steps
// are products of small matrices, on the f32 matrix cores:
//   o_t = (q_t e^{G_t}) S + sum_{s<=t} w_st v_s,  w_st = sum_keys q_t k_s e^{G_t - G_s},
//   S' = e^{G_16} S + sum_s (k_s e^{G_16 - G_s}) v_s^T,
// and the tangent along (dq, dk, dv, dg) is their product rule.  Every factor
// e^{..} and every difference of dG is formed from the steps between its ends
// alone (k_la_chunk), so a decay that underflows loses only what it has
// forgotten and no term cancels another.  A chunk with a value that is not
// finite, or so large or small that a product of q and k could leave the range
// of f32, is taken one step at a time by the same code (decay, k v, q S),
// which keeps a value that is not finite from the steps before it.
//
// Kernels, per host block of steps [t0, t0+len):
//   k_la_chunk<false>  zero-start segment aggregates (end states) and the
//                  segment sums of g and dg_k
//   k_la_carry     composes the block's segments, per lane and in order: a segment
//                  maps (S, dS_k) to (P S + S0, P dS_k + Q_k S + dS0_k) with
//                  P = exp(sum g), Q_k = P sum dg_k (multiplications only)
//   k_la_chunk<true>   rescan from the true entry states, writes o and do_k
// The sequential evaluation (enough columns to fill the GPU) runs
// k_la_chunk<true> only.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "pgf_exp.h"
#include "pgf_plan.h"
#include "pgf_timing.h"

namespace pgf {
namespace la {

constexpr int kThreads = 256;       // threads per block of the elementwise kernels
constexpr float kLog2eHi = 1.44269502162933349609375f;  // log2(e) rounded to f32
constexpr float kLog2eLo = 1.925963033500011079e-08f;   // log2(e) - kLog2eHi
constexpr float kLn2 = 0.693147180559945309f;

// e^v within a few ulp for moderate |v|: v*log2(e) split into p + lo (an fma
// recovers the rounding of p), 2^p from the hardware exponential and
// 2^lo ~ 1 + lo*ln2 as a correction; lo also carries the lift that cancels
// the hardware exponential's mean bias near 1 (pgf_exp.h), since the decay
// alpha = e^g of a long-memory key is close to 1.
__device__ __forceinline__ float exp_acc(float v) {
    const float p = v * kLog2eHi;
    const float lo = fmaf(v, kLog2eHi, -p) + fmaf(v, kLog2eLo, kExp2Lift);
    const float e = __builtin_amdgcn_exp2f(p);
    return fmaf(e, lo * kLn2, e);
}

// ---------------------------------------------------------------- scan
constexpr int kChunk = 16;       // steps per chunk
// Limits of the chunk form (beyond them a chunk goes step by step).  Its
// products associate as (q k) v where the recurrence takes q (k v): with
// |q|, |k| (and their tangents) up to kMaxQK, |dg| up to kMaxDg and a growth
// (positive g) of e^4 at most, the sums over 64 keys stay below 2^127; values
// so small that q k could leave the normal range while v brings the outputs
// back into it are kept out by kMinQ and kMinK (of a wave's largest value).
constexpr float kMaxQK = 0x1p40f, kMaxDg = 0x1p30f, kMaxGrow = 4.0f / kChunk;
constexpr float kMinQ = 0x1p-80f, kMinK = 0x1p-40f;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Access at a 32-bit element offset from a base that is the same for the whole
// wave (a host block has fewer than 2^30 elements per sequence and head).
__device__ __forceinline__ float ld(const float *base, uint32_t i) {
    return *(const float *)((const char *)base + (size_t)(i * 4u));
}
__device__ __forceinline__ void st(float *base, uint32_t i, float x) {
    *(float *)((char *)base + (size_t)(i * 4u)) = x;
}

// Block barrier that orders LDS only: the loads of the next chunk and the
// stores of the last one stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sums of two values over lane halves at once: rows of 32 (16) lanes of a and
// b are paired, so that lanes of even 32-halves (rows of 16) hold a's sum over
// the pair and those of odd ones b's.
__device__ __forceinline__ float pair_sum32(float a, float b) {
    const uintx2 r = __builtin_bit_cast(
        uintx2, __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false));
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_sum16(float a, float b) {
    const uintx2 r = __builtin_bit_cast(
        uintx2, __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false));
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over a row of 16 lanes, in every lane of the row.
template <int ROT>
__device__ __forceinline__ float add_ror(float v) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + ROT, 0xF,
                                                                     0xF, false));
}
__device__ __forceinline__ float row_sum(float v) { return add_ror<1>(add_ror<2>(add_ror<4>(add_ror<8>(v)))); }

// v_mfma_f32_16x16x4f32: lane (q, c) = (l/16, l%16) supplies A[c][q] and
// B[q][c] and receives D[4q + r][c] in accumulator r.  Wave w owns columns
// 16w .. 16w+15 of the block and every key: S[kt][r] is key 16kt + 4q + r of
// column c, so that each S[kt][r] is the B operand of the products with Q
// (k index q <-> key 16kt + 4q + r) as it lies.  Thread (tg, key) prepares SPT
// consecutive steps of one key.
//
// The weight of step s in the output of a later step t of the chunk is
// e^{g_{s+1} + .. + g_t} per key.  It is never formed as e^{G_t} e^{-G_s}:
// e^{-G} leaves the range of f32 for decays that models have, and the
// tangent's dG_t - dG_s cancels where one step decays strongly.  Instead the
// pairs are cut by the highest bit L in which s and t differ (8, 4, 2, 1):
// with c the first step of t's half of their block of 2L,
//   e^{..} = e^{g_{s+1} + .. + g_{c-1}} (with k_s)  e^{g_c + .. + g_t} (with q_t)
// and every factor, for S and the state's update too, is a product of the
// steps' own e^g (one exponential each) along a tree, every dG a sum of the
// steps' dg.  At each level a step is either a k (bit clear) or a q (bit set),
// so two levels fill the 16 rows and 16 columns of one product: rows and
// columns 0-7 hold level 8 (2), 8-15 level 4 (1), the quarters on the
// diagonal count.  q_t . k_t is summed over the keys by the vector unit.
// The parts of each key tile meet in sP, whose entry [16 (s/4) + t][s%4] is
// weight (s, t): the A operand of the product with v, without a transposition.
//
// Bound by the f32 matrix cores in the output pass (132 instructions of 32
// cycles per wave and chunk at dk = 64, one direction) and by memory in the
// aggregate pass (48).  At 32 heads x 32768 steps, dk = dv = 64, one direction,
// a call takes 1.33 ms and errs by 4.6e-7; a single reference per chunk
// (e^{G_t} e^{-G_s}, 120 instructions) took 1.20 ms and lost what is said
// above, the recurrence on the vector unit 2.38 ms at 6.7e-7.
template <int DK, int K, bool OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K == 1 && !OUT ? 4 : 2))) void k_la_chunk(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
    const float *__restrict__ g, const float *__restrict__ dq, const float *__restrict__ dk,
    const float *__restrict__ dv, const float *__restrict__ dg, const float *init, int64_t ibs, int64_t igs,
    int64_t ics, float *__restrict__ o, float *__restrict__ do_, float *end_state, float *__restrict__ agg_h,
    float *__restrict__ agg_s, int64_t BH, int64_t L, int64_t DV, int64_t t0, int64_t len, int64_t S, int G) {
    constexpr int KT = DK / 16;          // key tiles
    constexpr int NG = 256 / DK;         // thread groups over the steps of a chunk
    constexpr int SPT = kChunk / NG;     // steps per thread
    constexpr int P = DK + 4, PT = kChunk + 4;
    constexpr int O = 1 + K, NQ = OUT ? O : 1, RQ = OUT ? kChunk : 1;
    // With two directions at dk = 64 the two products share their operands'
    // LDS, one after the other, so that two blocks fit a CU.
    constexpr int SETS = K == 2 && DK == 64 ? 1 : 2;
    __shared__ __align__(16) float sQ[NQ][RQ][P];
    __shared__ __align__(16) float sLv[2][OUT ? SETS : 1][NQ][RQ][P];   // [k | q] of a level pair
    __shared__ floatx4 sP[NQ][OUT ? KT : 1][OUT ? 64 : 1];
    __shared__ __align__(16) float sKT[O][DK][PT];
    __shared__ __align__(16) float sEnd[O][DK];         // e^{G_16}, dG_16
    __shared__ float sTot[O][NG][DK];                   // products of e^g, sums of dg
    __shared__ float sSum[NG][DK];                      // sums of g
    __shared__ int sBad[2];

    const int tid = threadIdx.x;
    const int lane = tid % 64, c = lane % 16, qd = lane / 16;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int key = tid % DK, tg = DK == 64 ? w : tid / DK;
    const int64_t groups = DV / 64;
    const int64_t bh = blockIdx.x / groups;
    const int64_t cg = blockIdx.x % groups;
    const uint32_t cl = 16 * w + c;                    // this lane's column of the block
    const uint32_t DVu = (uint32_t)DV;
    const int gs = blockIdx.y;
    const int ts = (int)(gs * S);
    const int te = (int)(ts + S < len ? ts + S : len);
    if (ts >= te) return;   // uniform over the block
    const int64_t kst = BH * L;                        // rows between tangent directions
    const int64_t row0 = bh * L + t0;
    // wave-uniform bases: rows from step t0 of this head, columns of the block
    const float *qb = q + row0 * DK, *kb = k + row0 * DK, *gb = g + row0 * DK, *vb = v + row0 * DV + cg * 64;
    const float *dqb = dq + row0 * DK, *dkb = dk + row0 * DK, *dgb = dg + row0 * DK,
                *dvb = dv + row0 * DV + cg * 64;
    float *ob = o + row0 * DV + cg * 64, *dob = do_ + row0 * DV + cg * 64;
    const int64_t dks = kst * DK, dvs = kst * DV;

    floatx4 Sm[KT], dS[K][KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t e = (16 * kt + 4 * qd + r) * DVu + cl;
            const float *ib = init + bh * ibs + gs * igs + cg * 64;
            Sm[kt][r] = OUT ? ld(ib, e) : 0.0f;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dS[kk][kt][r] = OUT ? ld(ib + (1 + kk) * ics, e) : 0.0f;
        }
    if (tid < 2) sBad[tid] = 0;
    if constexpr (OUT) {
        // weights of s > t stay zero
        for (int i = tid; i < NQ * KT * 64; i += 256) (&sP[0][0][0])[i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // key-side inputs of this thread's steps and the value rows 4qd + m
    float rg[SPT], rk[SPT], rq[SPT], rdg[K][SPT], rdk[K][SPT], rdq[K][SPT], vn[4], dvn[K][4];
    auto fetch = [&](int tb) {
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const int t = tb + tg * SPT + j;
            const bool live = t < te;
            const uint32_t e = (uint32_t)((live ? t : te - 1) * DK + key);
            rg[j] = live ? ld(gb, e) : 0.0f;
            rk[j] = live ? ld(kb, e) : 0.0f;
            if constexpr (OUT) rq[j] = live ? ld(qb, e) : 0.0f;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                rdg[kk][j] = live ? ld(dgb + kk * dks, e) : 0.0f;
                rdk[kk][j] = live ? ld(dkb + kk * dks, e) : 0.0f;
                if constexpr (OUT) rdq[kk][j] = live ? ld(dqb + kk * dks, e) : 0.0f;
            }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int t = tb + 4 * qd + m;
            const bool live = t < te;
            const uint32_t e = (uint32_t)(live ? t : te - 1) * DVu + cl;
            vn[m] = live ? ld(vb, e) : 0.0f;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dvn[kk][m] = live ? ld(dvb + kk * dvs, e) : 0.0f;
        }
    };
    // S <- e S, dS <- e dS + dG S' for the decay in sEnd
    auto decay = [&]() {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const floatx4 e = *(const floatx4 *)&sEnd[0][16 * kt + 4 * qd];
#pragma unroll
            for (int r = 0; r < 4; ++r) Sm[kt][r] *= e[r];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const floatx4 d = *(const floatx4 *)&sEnd[1 + kk][16 * kt + 4 * qd];
#pragma unroll
                for (int r = 0; r < 4; ++r) dS[kk][kt][r] = fmaf(e[r], dS[kk][kt][r], d[r] * Sm[kt][r]);
            }
        }
    };
    // o += Q S and its tangents
    auto read_out = [&](floatx4 &ov, floatx4 (&dov)[K]) {
        if constexpr (OUT) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const floatx4 qa = *(const floatx4 *)&sQ[0][c][16 * kt + 4 * qd];
#pragma unroll
                for (int r = 0; r < 4; ++r) ov = mfma4(qa[r], Sm[kt][r], ov);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) {
                    const floatx4 dqa = *(const floatx4 *)&sQ[1 + kk][c][16 * kt + 4 * qd];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        dov[kk] = mfma4(dqa[r], Sm[kt][r], dov[kk]);
                        dov[kk] = mfma4(qa[r], dS[kk][kt][r], dov[kk]);
                    }
                }
            }
        }
    };
    // S += K v and its tangents
    auto update = [&](const float (&vv)[4], const float (&dvv)[K][4]) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const floatx4 ka = *(const floatx4 *)&sKT[0][16 * kt + c][4 * qd];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const floatx4 dka = *(const floatx4 *)&sKT[1 + kk][16 * kt + c][4 * qd];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    dS[kk][kt] = mfma4(dka[m], vv[m], dS[kk][kt]);
                    dS[kk][kt] = mfma4(ka[m], dvv[kk][m], dS[kk][kt]);
                }
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) Sm[kt] = mfma4(ka[m], vv[m], Sm[kt]);
        }
    };
    // stores rows lo <= row < hi of the chunk
    auto put_out = [&](int tb, int lo, int hi, floatx4 ov, const floatx4 (&dov)[K]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = 4 * qd + r;
            if (t >= lo && t < hi && tb + t < te) {
                const uint32_t e = (uint32_t)(tb + t) * DVu + cl;
                st(ob, e, ov[r]);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) st(dob + kk * dvs, e, dov[kk][r]);
            }
        }
    };
    // The weights of one level pair (set 0: levels 8 and 4, set 1: 2 and 1)
    // over one key tile, left in sP.
    auto weights = [&](int set, int kt) {
        if constexpr (OUT) {
            const float (*ks)[kChunk][P] = sLv[0][SETS == 2 ? set : 0], (*qs)[kChunk][P] = sLv[1][SETS == 2 ? set : 0];
            const floatx4 ka = *(const floatx4 *)&ks[0][c][16 * kt + 4 * qd];
            const floatx4 qa = *(const floatx4 *)&qs[0][c][16 * kt + 4 * qd];
            floatx4 pv[O];
#pragma unroll
            for (int cc = 0; cc < O; ++cc) pv[cc] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int r = 0; r < 4; ++r) pv[0] = mfma4(ka[r], qa[r], pv[0]);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const floatx4 dka = *(const floatx4 *)&ks[1 + kk][c][16 * kt + 4 * qd];
                const floatx4 dqa = *(const floatx4 *)&qs[1 + kk][c][16 * kt + 4 * qd];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pv[1 + kk] = mfma4(dka[r], qa[r], pv[1 + kk]);
                    pv[1 + kk] = mfma4(ka[r], dqa[r], pv[1 + kk]);
                }
            }
            // row 4qd + r is a k, column c a q of the packed rows
            const int h = c & 7;
#pragma unroll
            for (int cc = 0; cc < O; ++cc) {
                floatx4 *sp = sP[cc][kt];
                const floatx4 p = pv[cc];
                if (set == 0) {
                    if (qd < 2) {
                        if (c < 8) sp[16 * qd + 8 + c] = p;                        // s = 4qd + r, t = 8 + c
                    } else if (c / 4 == qd) {
                        sp[32 * (qd - 2) + 8 * (qd - 2) + 4 + (c & 3)] = p;        // s = 8(qd-2) + r
                    }
                } else if (qd < 2) {
                    if (c / 4 == qd) {                                             // s = 4(c/2) + {0, 1}
                        float *e = (float *)&sp[16 * (c / 2) + 4 * (c / 2) + 2 + (c & 1)];
                        e[0] = c & 2 ? p[2] : p[0];
                        e[1] = c & 2 ? p[3] : p[1];
                    }
                } else if (c / 4 == qd) {                                          // s = 2h, t = 2h + 1
                    float *e = (float *)&sp[16 * (h / 2) + 2 * h + 1];
                    e[2 * (h & 1)] = h & 2 ? (h & 1 ? p[3] : p[2]) : (h & 1 ? p[1] : p[0]);
                }
            }
        }
    };

    float sg = 0.0f, sdg[K];   // aggregate pass: sums of g and dg_k over this thread's steps
#pragma unroll
    for (int kk = 0; kk < K; ++kk) sdg[kk] = 0.0f;
    fetch(ts);
    int buf = 0;
    for (int tb = ts; tb < te; tb += kChunk, buf ^= 1) {
        float vv[4], dvv[K][4];
        float chk = 0.0f;        // NaN once a value below is not finite
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            vv[m] = vn[m];
            chk = fmaf(vv[m], 0.0f, chk);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                dvv[kk][m] = dvn[kk][m];
                chk = fmaf(dvv[kk][m], 0.0f, chk);
            }
        }
        // this thread's decays, their product and the sums of dg
        float a[SPT], grow = 0.0f, mag = 0.0f, mdg = 0.0f, qmax = 0.0f, kmax = 0.0f;
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            a[j] = exp_acc(rg[j]);
            chk = fmaf(a[j], 0.0f, chk);
            grow += fmaxf(rg[j], 0.0f);
            mag += fabsf(rk[j]);
            kmax = fmaxf(kmax, fabsf(rk[j]));
            if constexpr (OUT) {
                mag += fabsf(rq[j]);
                qmax = fmaxf(qmax, fabsf(rq[j]));
            }
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                mdg += fabsf(rdg[kk][j]);
                mag += fabsf(rdk[kk][j]);
                kmax = fmaxf(kmax, fabsf(rdk[kk][j]));
                if constexpr (OUT) {
                    mag += fabsf(rdq[kk][j]);
                    qmax = fmaxf(qmax, fabsf(rdq[kk][j]));
                }
            }
            if constexpr (!OUT) {
#pragma unroll
                for (int kk = 0; kk < K; ++kk) sdg[kk] += rdg[kk][j];
            }
        }
        float gsum = rg[0];      // of the chunk, once the other threads' are added
        {
            float T = a[0], D[K];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) D[kk] = rdg[kk][0];
#pragma unroll
            for (int j = 1; j < SPT; ++j) {
                T *= a[j];
                gsum += rg[j];
#pragma unroll
                for (int kk = 0; kk < K; ++kk) D[kk] += rdg[kk][j];
            }
            sTot[0][tg][key] = T;
            sSum[tg][key] = gsum;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) sTot[1 + kk][tg][key] = D[kk];
        }
        if constexpr (!OUT) sg += gsum;
        bool bad = !(mag <= kMaxQK) || !(mdg <= kMaxDg) || !(grow <= kMaxGrow * SPT) || !(chk == 0.0f);
        if constexpr (OUT) {
            // a wave whose q (k) are all tiny, not all zero
            const auto any = [](bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; };
            bad |= (any(qmax > 0.0f) && !any(qmax >= kMinQ)) || (any(kmax > 0.0f) && !any(kmax >= kMinK));
        }
        lds_barrier();          // also: every wave has left the last chunk's operands
        if (bad) sBad[buf] = 1;

        // Per step: the decay (p, inclusive) and dg from the start of its block
        // of 2^i steps, and (s, exclusive) to its end, doubling the block.
        float pf[SPT], sf[SPT], pd[K][SPT], sd[K][SPT];
        float lf[4][SPT], ld_[4][K][SPT];     // each level's factor: p of a q, s of a k
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            pf[j] = a[j];
            sf[j] = 1.0f;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                pd[kk][j] = rdg[kk][j];
                sd[kk][j] = 0.0f;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int Lv = 1 << i;
            if (Lv < SPT) {
                float tf[SPT], td[K][SPT];    // a block's totals, at its last step
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    tf[j] = pf[j];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) td[kk][j] = pd[kk][j];
                }
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const bool up = (j & Lv) != 0;
                    const int x = up ? (j & ~(Lv - 1)) - 1 : (j | (2 * Lv - 1));   // last step of the other half
                    lf[i][j] = up ? pf[j] : sf[j];
                    (up ? pf[j] : sf[j]) *= tf[x];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        ld_[i][kk][j] = up ? pd[kk][j] : sd[kk][j];
                        (up ? pd[kk][j] : sd[kk][j]) += td[kk][x];
                    }
                }
            } else {
                const int m = Lv / SPT;       // thread groups of a half
                const bool up = (tg & m) != 0;
                const int h0 = (tg ^ m) & ~(m - 1);
                float T = sTot[0][h0][key], D[K];
#pragma unroll
                for (int kk = 0; kk < K; ++kk) D[kk] = sTot[1 + kk][h0][key];
#pragma unroll
                for (int h = 1; h < m; ++h) {
                    T *= sTot[0][h0 + h][key];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) D[kk] += sTot[1 + kk][h0 + h][key];
                }
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    lf[i][j] = up ? pf[j] : sf[j];
                    pf[j] = up ? pf[j] * T : pf[j];
                    sf[j] = up ? sf[j] : sf[j] * T;
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        ld_[i][kk][j] = up ? pd[kk][j] : sd[kk][j];
                        pd[kk][j] = up ? pd[kk][j] + D[kk] : pd[kk][j];
                        sd[kk][j] = up ? sd[kk][j] : sd[kk][j] + D[kk];
                    }
                }
            }
        }
        // the operands of level i
        auto stage = [&](int i) {
            if constexpr (OUT) {
                const int Lv = 1 << i;
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const int t = tg * SPT + j;
                    const bool up = Lv < SPT ? (j & Lv) != 0 : (tg & (Lv / SPT)) != 0;
                    const int row = (t & (Lv - 1)) + t / (2 * Lv) * Lv + (i % 2 == 0 ? 8 : 0);
                    float *dst = &sLv[up][SETS == 2 && i < 2 ? 1 : 0][0][row][key];
                    const float x = up ? rq[j] : rk[j];
                    dst[0] = x * lf[i][j];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk)
                        dst[(1 + kk) * kChunk * P] =
                            fmaf(x, ld_[i][kk][j], up ? rdq[kk][j] : rdk[kk][j]) * lf[i][j];
                }
            }
        };
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const int t = tg * SPT + j;
            sKT[0][key][t] = rk[j] * sf[j];
            if constexpr (OUT) sQ[0][t][key] = rq[j] * pf[j];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                sKT[1 + kk][key][t] = fmaf(rk[j], sd[kk][j], rdk[kk][j]) * sf[j];
                if constexpr (OUT) sQ[1 + kk][t][key] = fmaf(rq[j], pd[kk][j], rdq[kk][j]) * pf[j];
            }
        }
        if (tg == NG - 1) {
            // The state's own decay is one exponential of the sum of g: over a
            // long memory 16 rounded factors a chunk add up (errors at the
            // RWKV sizes 1.1e-6 with their product, 4.5e-7 with this).
#pragma unroll
            for (int h = NG - 2; h >= 0; --h) gsum += sSum[h][key];
            sEnd[0][key] = exp_acc(gsum);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) sEnd[1 + kk][key] = pd[kk][SPT - 1];
        }
        if constexpr (OUT) {
            stage(3);
            stage(2);
            if (SETS == 2) {
                stage(1);
                stage(0);
            }
            // the weights of s = t: sums over the keys, four steps a wave, the
            // rows of 16 lanes holding one step each
#pragma unroll
            for (int cc = 0; cc < O; ++cc) {
                float z[SPT];
#pragma unroll
                for (int j = 0; j < SPT; ++j)
                    z[j] = cc == 0 ? rq[j] * rk[j]
                                   : fmaf(rdq[cc ? cc - 1 : 0][j], rk[j], rq[j] * rdk[cc ? cc - 1 : 0][j]);
                float sum;
                int t;
                if constexpr (SPT == 4) {
                    sum = pair_sum16(pair_sum32(z[0], z[1]), pair_sum32(z[2], z[3]));
                    t = 4 * w + ((qd & 1) << 1 | qd >> 1);
                } else if constexpr (SPT == 2) {
                    sum = pair_sum16(z[0], z[1]);
                    t = 4 * w + qd;
                } else {
                    sum = z[0];
                    t = 4 * w + qd;
                }
                sum = row_sum(sum);
                if (c == 0) ((float *)&sP[cc][0][16 * w + t])[t & 3] = sum;
            }
        }
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(sBad[buf]) == 0) {
            floatx4 ov = {0.0f, 0.0f, 0.0f, 0.0f}, dov[K];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dov[kk] = ov;
            if constexpr (OUT) {
                if constexpr (SETS == 1) {
                    weights(0, w);
                    lds_barrier();
                    stage(1);
                    stage(0);
                    fetch(tb + kChunk);
                    lds_barrier();
                    weights(1, w);
                } else {
                    fetch(tb + kChunk);
                    if constexpr (KT == 4) {
                        weights(0, w);
                        weights(1, w);
                    } else if (w < 2 * KT) {
                        weights(w / KT, w % KT);
                    }
                }
                read_out(ov, dov);
                lds_barrier();
                floatx4 pv[O];
#pragma unroll
                for (int cc = 0; cc < O; ++cc) {
                    pv[cc] = sP[cc][0][lane];
#pragma unroll
                    for (int kt = 1; kt < KT; ++kt) {
                        const floatx4 pw = sP[cc][kt][lane];
#pragma unroll
                        for (int r = 0; r < 4; ++r) pv[cc][r] += pw[r];
                    }
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    ov = mfma4(pv[0][m], vv[m], ov);
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        dov[kk] = mfma4(pv[1 + kk][m], vv[m], dov[kk]);
                        dov[kk] = mfma4(pv[0][m], dvv[kk][m], dov[kk]);
                    }
                }
                put_out(tb, 0, kChunk, ov, dov);
            } else {
                fetch(tb + kChunk);
            }
            decay();
            update(vv, dvv);
        } else {
            // one step at a time, as the recurrence has it: decay, k v, q S
            for (int sub = 0; sub < kChunk; ++sub) {
                lds_barrier();
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const int t = tg * SPT + j;
                    const bool on = t == sub;
                    sKT[0][key][t] = on ? rk[j] : 0.0f;
                    if constexpr (OUT) sQ[0][t][key] = rq[j];
                    if (on) sEnd[0][key] = exp_acc(rg[j]);
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        sKT[1 + kk][key][t] = on ? rdk[kk][j] : 0.0f;
                        if constexpr (OUT) sQ[1 + kk][t][key] = rdq[kk][j];
                        if (on) sEnd[1 + kk][key] = rdg[kk][j];
                    }
                }
                float vs[4], dvs_[K][4];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const bool on = 4 * qd + m == sub;
                    vs[m] = on ? vv[m] : 0.0f;
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) dvs_[kk][m] = on ? dvv[kk][m] : 0.0f;
                }
                lds_barrier();
                decay();
                update(vs, dvs_);
                floatx4 ov = {0.0f, 0.0f, 0.0f, 0.0f}, dov[K];
#pragma unroll
                for (int kk = 0; kk < K; ++kk) dov[kk] = ov;
                read_out(ov, dov);
                if constexpr (OUT) put_out(tb, sub, sub + 1, ov, dov);
            }
            fetch(tb + kChunk);
        }
        if (tid == 0) sBad[buf ^ 1] = 0;   // read two barriers later at the earliest
    }

    auto put_state = [&](float *dst, int64_t plane) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t e = (16 * kt + 4 * qd + r) * DVu + cl;
                st(dst + cg * 64, e, Sm[kt][r]);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) st(dst + cg * 64 + (1 + kk) * plane, e, dS[kk][kt][r]);
            }
    };
    if constexpr (OUT) {
        if (end_state) put_state(end_state + bh * ibs, ics);
    } else {
        put_state(agg_h + (bh * G + gs) * (1 + K) * DK * DV, DK * DV);
        // the segment sums, the thread groups' parts added in order
        lds_barrier();
        sTot[0][tg][key] = sg;
#pragma unroll
        for (int kk = 0; kk < K; ++kk) sTot[1 + kk][tg][key] = sdg[kk];
        lds_barrier();
        if (cg == 0 && tg == 0) {
#pragma unroll
            for (int cc = 0; cc <= K; ++cc) {
                float t = sTot[cc][0][key];
#pragma unroll
                for (int h = 1; h < NG; ++h) t += sTot[cc][h][key];
                agg_s[((bh * G + gs) * (1 + K) + cc) * DK + key] = t;
            }
        }
    }
}

// ---------------------------------------------------------------- carry
// The state entering each segment: per lane (bh, i, j) the segments' maps are
// composed one after the other.  state [(1+K)][BH][DK][DV] enters and leaves;
// seg [BH][G][(1+K)][DK][DV] holds each segment's zero-start end state on
// entry and is overwritten with the true state entering the segment.  sums
// [BH][G][(1+K)][DK] as written by k_la_chunk<false>.
// Only the chain is sequential: a block owns 64 lanes (of one head, grid x =
// BH * DK * DV / 64) and its waves take consecutive runs of GB segments each,
// load them and form P = exp(sum g) and P sum dg_k at the same time, and then
// pass the state from wave to wave through LDS.  One thread walking all
// segments of a lane took about 180 ns a segment: a call of one head of 131072
// steps in 64-step segments, dk = 64, 0.53 ms, now 0.37 (32-step segments 0.90
// and 0.57).
constexpr int kCarryWaves = 8;

template <int K>
__global__ __launch_bounds__(64 * kCarryWaves) __attribute__((amdgpu_waves_per_eu(4))) void k_la_carry(
    float *seg, const float *__restrict__ sums, float *__restrict__ state, int64_t BH, int64_t DK, int64_t DV, int G) {
    constexpr int CP = 1 + K, GB = K == 1 ? 8 : 4;
    __shared__ float s_st[CP][64];
    const int l = threadIdx.x % 64;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int W = (int)blockDim.x / 64;
    const int64_t per = DK * DV;                 // a multiple of 64
    const int64_t bh = blockIdx.x / (per / 64);
    const int64_t r0 = blockIdx.x % (per / 64) * 64;
    const int64_t i = r0 / DV;                   // 64 columns of one key
    const int64_t cs = BH * per;
    float *sb = state + bh * per + r0;
    if (w == 0) {
#pragma unroll
        for (int c = 0; c < CP; ++c) s_st[c][l] = sb[c * cs + l];
    }
    lds_barrier();
    for (int t0 = 0; t0 < G; t0 += W * GB) {
        const int g0 = t0 + w * GB;
        const int ng = G - g0 < GB ? G - g0 : GB;      // segments of this wave (may be <= 0)
        float *sg = seg + (bh * G + g0) * CP * per + r0;
        const float *sm = sums + (bh * G + g0) * CP * DK + i;
        float e[GB][CP], co[GB][CP];
#pragma unroll
        for (int j = 0; j < GB; ++j) {
            if (j < ng) {
#pragma unroll
                for (int c = 0; c < CP; ++c) {
                    e[j][c] = sg[(j * CP + c) * per + l];
                    co[j][c] = sm[(j * CP + c) * DK];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < GB; ++j) {
            if (j < ng) {
                co[j][0] = exp_series(co[j][0]);
#pragma unroll
                for (int c = 1; c < CP; ++c) co[j][c] *= co[j][0];
            }
        }
        for (int w0 = 0; w0 < W && t0 + w0 * GB < G; ++w0) {
            if (w == w0) {
                float s[CP];
#pragma unroll
                for (int c = 0; c < CP; ++c) s[c] = s_st[c][l];
#pragma unroll
                for (int j = 0; j < GB; ++j) {
                    if (j < ng) {
#pragma unroll
                        for (int c = 0; c < CP; ++c) sg[(j * CP + c) * per + l] = s[c];
#pragma unroll
                        for (int c = 1; c < CP; ++c) s[c] = fmaf(co[j][0], s[c], fmaf(co[j][c], s[0], e[j][c]));
                        s[0] = fmaf(co[j][0], s[0], e[j][0]);
                    }
                }
#pragma unroll
                for (int c = 0; c < CP; ++c) s_st[c][l] = s[c];
            }
            lds_barrier();
        }
    }
    if (w == 0) {
#pragma unroll
        for (int c = 0; c < CP; ++c) sb[c * cs + l] = s_st[c][l];
    }
}

// ---------------------------------------------------------------- state in/out
// dst[i] = src ? src[i] : 0 over n floats (the state layout is the ABI's).
__global__ __launch_bounds__(kThreads) void k_la_copy(const float *__restrict__ src, float *__restrict__ dst,
                                                      int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) dst[i] = src ? src[i] : 0.0f;
}

// ---------------------------------------------------------------- dispatch
struct LaLauncher {
    const LaPlan &q;
    const pgf_la_params &p;
    const float *qv, *kv, *vv, *gv, *dqv, *dkv, *dvv, *dgv;
    float *o, *dov;
    hipStream_t st;
    char *ws;

    float *state() const { return (float *)(ws + q.state); }
    float *agg_h() const { return (float *)(ws + q.agg_h); }
    float *agg_s() const { return (float *)(ws + q.agg_s); }

    template <int DK, int K>
    void block(int64_t t0, int64_t len) {
        const int64_t ND = DK * q.DV;
        const unsigned gx = (unsigned)(q.BH * q.DV / 64);
        const int64_t S = q.seg ? q.seg : len;
        const int G = (int)((len + S - 1) / S);
        if (q.seg == 0) {
            Timed tm(3, st);
            hipLaunchKernelGGL((k_la_chunk<DK, K, true>), dim3(gx, 1), dim3(256), 0, st, qv, kv, vv, gv, dqv, dkv, dvv,
                               dgv, (const float *)state(), ND, (int64_t)0, q.BH * ND, o, dov, state(),
                               (float *)nullptr, (float *)nullptr, q.BH, q.L, q.DV, t0, len, len, 1);
            return;
        }
        {
            Timed tm(1, st);
            hipLaunchKernelGGL((k_la_chunk<DK, K, false>), dim3(gx, (unsigned)G), dim3(256), 0, st, qv, kv, vv, gv,
                               dqv, dkv, dvv, dgv, (const float *)nullptr, (int64_t)0, (int64_t)0, (int64_t)0, o, dov,
                               (float *)nullptr, agg_h(), agg_s(), q.BH, q.L, q.DV, t0, len, S, G);
        }
        {
            constexpr int GB = K == 1 ? 8 : 4;   // (k_la_carry's)
            const int w = (G + GB - 1) / GB;
            Timed tm(2, st);
            hipLaunchKernelGGL((k_la_carry<K>), dim3((unsigned)(q.BH * ND / 64)),
                               dim3(64 * (w < kCarryWaves ? w : kCarryWaves)), 0, st, agg_h(),
                               (const float *)agg_s(), state(), q.BH, (int64_t)DK, q.DV, G);
        }
        {
            Timed tm(3, st);
            hipLaunchKernelGGL((k_la_chunk<DK, K, true>), dim3(gx, (unsigned)G), dim3(256), 0, st, qv, kv, vv, gv, dqv,
                               dkv, dvv, dgv, (const float *)agg_h(), (int64_t)G * (1 + K) * ND,
                               (int64_t)(1 + K) * ND, ND, o, dov, (float *)nullptr, (float *)nullptr,
                               (float *)nullptr, q.BH, q.L, q.DV, t0, len, S, G);
        }
    }

    template <int DK, int K>
    int run_t() {
        const int64_t nst = q.BH * DK * q.DV;   // floats per state component
        const unsigned gs = (unsigned)((nst + kThreads - 1) / kThreads);
        {
            Timed tm(4, st);
            hipLaunchKernelGGL(k_la_copy, dim3(gs), dim3(kThreads), 0, st, p.S_in, state(), nst);
            for (int kk = 0; kk < K; ++kk)
                hipLaunchKernelGGL(k_la_copy, dim3(gs), dim3(kThreads), 0, st,
                                   p.dS_in ? p.dS_in + kk * nst : (const float *)nullptr, state() + (1 + kk) * nst,
                                   nst);
        }
        for (int64_t t0 = 0; t0 < q.L; t0 += q.chunk_len) {
            const int64_t len = q.L - t0 < q.chunk_len ? q.L - t0 : q.chunk_len;
            block<DK, K>(t0, len);
        }
        if (p.S_out || p.dS_out) {
            Timed tm(4, st);
            if (p.S_out)
                hipLaunchKernelGGL(k_la_copy, dim3(gs), dim3(kThreads), 0, st, (const float *)state(), p.S_out, nst);
            if (p.dS_out)
                hipLaunchKernelGGL(k_la_copy, dim3((unsigned)((K * nst + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                                   st, (const float *)(state() + nst), p.dS_out, K * nst);
        }
        return hipGetLastError() == hipSuccess ? PGF_OK : PGF_ERR_HIP;
    }

    int run() {
        switch (q.DK * 10 + q.K) {
            case 161: return run_t<16, 1>();
            case 162: return run_t<16, 2>();
            case 321: return run_t<32, 1>();
            case 322: return run_t<32, 2>();
            case 641: return run_t<64, 1>();
            case 642: return run_t<64, 2>();
            default: return PGF_ERR_UNSUPPORTED;
        }
    }
};

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return na && nb && pa < pb + nb && pb < pa + na;
}

}  // namespace la
}  // namespace pgf

extern "C" int pgf_la_scan_jvp(const float *q, const float *k, const float *v, const float *g, const float *dq,
                               const float *dk, const float *dv, const float *dg, const pgf_la_params *p, float *o,
                               float *do_, void *stream) {
    using namespace pgf;
    LaPlan pl;
    const int rc = make_la_plan(p, &pl);
    if (rc != PGF_OK) return rc;
    if (!p->workspace || p->workspace_bytes < pl.total || ((uintptr_t)p->workspace & 255))
        return PGF_ERR_WORKSPACE;
    if (pl.L > 0) {
        if (!q || !k || !v || !g || !dq || !dk || !dv || !dg || !o || !do_) return PGF_ERR_INVALID_ARG;
        const size_t f = sizeof(float);
        const size_t nk = (size_t)pl.BH * pl.L * pl.DK * f, nv = (size_t)pl.BH * pl.L * pl.DV * f;
        const void *ins[8] = {q, k, v, g, dq, dk, dv, dg};
        const size_t sz[8] = {nk, nk, nv, nk, nk * pl.K, nk * pl.K, nv * pl.K, nk * pl.K};
        for (int i = 0; i < 8; ++i)
            if (la::overlap(o, nv, ins[i], sz[i]) || la::overlap(do_, nv * pl.K, ins[i], sz[i]) ||
                la::overlap(p->workspace, pl.total, ins[i], sz[i]))
                return PGF_ERR_INVALID_ARG;
        if (la::overlap(o, nv, do_, nv * pl.K) || la::overlap(o, nv, p->workspace, pl.total) ||
            la::overlap(do_, nv * pl.K, p->workspace, pl.total))
            return PGF_ERR_INVALID_ARG;
    }
    (void)hipGetLastError();
    la::LaLauncher l{pl, *p, q, k, v, g, dq, dk, dv, dg, o, do_, (hipStream_t)stream, (char *)p->workspace};
    return l.run();
}
