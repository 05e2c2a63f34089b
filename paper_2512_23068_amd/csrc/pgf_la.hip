// libpgf: decaying linear attention with its tangent flow (App. F: linear
// transformers, RetNet and RWKV-6 as general linear recurrences) for gfx950.
//
// The state of one (batch, head) is a dk x dv matrix S.  A block owns 64 value
// columns of one head and takes a segment in chunks of 16 steps.  Within a
// chunk, with G_t the sum of g up to and including step t (per key) and
//   Q_t = q_t e^{G_t},  K_s = k_s e^{-G_s},
// the steps are products of small matrices, on the f32 matrix cores:
//   o_t = Q_t S + sum_{s<=t} (Q_t . K_s) v_s,   S' = e^{G_16} (S + sum_s K_s v_s^T)
// and the tangent along (dq, dk, dv, dg) is their product rule with
//   dQ_t = (dq_t + q_t dG_t) e^{G_t},  dK_s = (dk_s - k_s dG_s) e^{-G_s},
//   dS' = e^{G_16} dS~ + dG_16 S',  S~ the bracket above.
// Where a chunk's |G| exceeds kMaxG, or a scaled operand or a value is not
// finite, its steps are taken one at a time by the same code (decay the state,
// then the products of one step), which needs no e^{-G} and keeps a value
// that is not finite from the steps before it.
//
// Kernels, per host block of steps [t0, t0+len):
//   k_la_chunk<false>  zero-start segment aggregates (end states) and the
//                  segment sums of g and dg_k
//   k_la_carry     sequential over the block's segments, per lane: a segment
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
constexpr float kMaxG = 60.0f;   // e^60 = 1e26: products with |k|, |q| below 1e12 stay finite

typedef float floatx4 __attribute__((ext_vector_type(4)));

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

// v_mfma_f32_16x16x4f32: lane (q, c) = (l/16, l%16) supplies A[c][q] and
// B[q][c] and receives D[4q + r][c] in accumulator r.  Wave w owns columns
// 16w .. 16w+15 of the block and every key: S[kt][r] is key 16kt + 4q + r of
// column c, so that each S[kt][r] is the B operand of the products with Q
// (k index q <-> key 16kt + 4q + r) as it lies.  The 16 x 16 products K_s . Q_t
// are formed by every wave with s in the rows, whose accumulators are then
// the A operand of the product with v (s = 4q + r), without a transposition.
// Thread (tg, key) prepares SPT consecutive steps of one key: K and Q as rows
// [t][key] and K also as [key][t] for the update of S.
//
// Bound by the f32 matrix cores in the output pass (120 instructions of 32
// cycles per wave and chunk at dk = 64, one direction) and by memory in the
// aggregate pass (48).
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
    constexpr int NQ = OUT ? 1 + K : 1;
    __shared__ __align__(16) float sQ[NQ][OUT ? kChunk : 1][P];
    __shared__ __align__(16) float sK[NQ][OUT ? kChunk : 1][P];
    __shared__ __align__(16) float sKT[1 + K][DK][PT];
    __shared__ __align__(16) float sEnd[1 + K][DK];     // e^{G_16}, dG_16
    __shared__ float sTot[1 + K][NG][DK];
    __shared__ int sBad[2];
    // K_s . Q_t and its tangents: with four key tiles each wave forms the part
    // of one tile and all add the four (36 of 156 products saved, for a barrier)
    constexpr bool PART = OUT && KT == 4;
    __shared__ floatx4 sP[PART ? 1 + K : 1][PART ? 4 : 1][PART ? 64 : 1];

    const int tid = threadIdx.x;
    const int lane = tid % 64, c = lane % 16, qd = lane / 16;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int key = tid % DK, tg = tid / DK;
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
    // This thread's rows of the operands from step j's scaled values.
    auto put = [&](int j, float kv, const float (&dkv)[K], float qv, const float (&dqv)[K]) {
        const int t = tg * SPT + j;
        sKT[0][key][t] = kv;
        if constexpr (OUT) {
            sK[0][t][key] = kv;
            sQ[0][t][key] = qv;
        }
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
            sKT[1 + kk][key][t] = dkv[kk];
            if constexpr (OUT) {
                sK[1 + kk][t][key] = dkv[kk];
                sQ[1 + kk][t][key] = dqv[kk];
            }
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
    // The products of one staged chunk: outputs of its rows (the values of
    // row 4qd + r, stored for rows lo <= row < hi of the chunk), then S~.
    auto products = [&](int tb, int lo, int hi, const float (&vv)[4], const float (&dvv)[K][4]) {
        if constexpr (OUT) {
            floatx4 ov = {0.0f, 0.0f, 0.0f, 0.0f}, dov[K], pv = ov, dpv[K];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dov[kk] = dpv[kk] = pv;
            auto inner = [&](int kt) {
                const floatx4 qa = *(const floatx4 *)&sQ[0][c][16 * kt + 4 * qd];
                const floatx4 ka = *(const floatx4 *)&sK[0][c][16 * kt + 4 * qd];
#pragma unroll
                for (int r = 0; r < 4; ++r) pv = mfma4(ka[r], qa[r], pv);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) {
                    const floatx4 dqa = *(const floatx4 *)&sQ[1 + kk][c][16 * kt + 4 * qd];
                    const floatx4 dka = *(const floatx4 *)&sK[1 + kk][c][16 * kt + 4 * qd];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        dpv[kk] = mfma4(dka[r], qa[r], dpv[kk]);
                        dpv[kk] = mfma4(ka[r], dqa[r], dpv[kk]);
                    }
                }
            };
            if constexpr (PART) {
                inner(w);
                sP[0][w][lane] = pv;
#pragma unroll
                for (int kk = 0; kk < K; ++kk) sP[1 + kk][w][lane] = dpv[kk];
            }
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                if constexpr (!PART) inner(kt);
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
            if constexpr (PART) {
                lds_barrier();
                pv = sP[0][0][lane];
#pragma unroll
                for (int kk = 0; kk < K; ++kk) dpv[kk] = sP[1 + kk][0][lane];
#pragma unroll
                for (int h = 1; h < 4; ++h) {
                    const floatx4 pw = sP[0][h][lane];
#pragma unroll
                    for (int r = 0; r < 4; ++r) pv[r] += pw[r];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        const floatx4 dpw = sP[1 + kk][h][lane];
#pragma unroll
                        for (int r = 0; r < 4; ++r) dpv[kk][r] += dpw[r];
                    }
                }
            }
            // pv[r] = K_s . Q_t, s = 4qd + r, t = c: only s <= t counts
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = 4 * qd + r <= c;
                pv[r] = in ? pv[r] : 0.0f;
#pragma unroll
                for (int kk = 0; kk < K; ++kk) dpv[kk][r] = in ? dpv[kk][r] : 0.0f;
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                ov = mfma4(pv[m], vv[m], ov);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) {
                    dov[kk] = mfma4(dpv[kk][m], vv[m], dov[kk]);
                    dov[kk] = mfma4(pv[m], dvv[kk][m], dov[kk]);
                }
            }
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
        }
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
        // G and dG within this thread's steps, then the steps before them
        float Gt[SPT], dGt[K][SPT];
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            Gt[j] = j ? Gt[j - 1] + rg[j] : rg[j];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dGt[kk][j] = j ? dGt[kk][j - 1] + rdg[kk][j] : rdg[kk][j];
        }
        if constexpr (!OUT) {
            sg += Gt[SPT - 1];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) sdg[kk] += dGt[kk][SPT - 1];
        }
        sTot[0][tg][key] = Gt[SPT - 1];
#pragma unroll
        for (int kk = 0; kk < K; ++kk) sTot[1 + kk][tg][key] = dGt[kk][SPT - 1];
        lds_barrier();          // also: every wave has left the last chunk's operands
        float g0 = 0.0f, dg0[K];
#pragma unroll
        for (int kk = 0; kk < K; ++kk) dg0[kk] = 0.0f;
#pragma unroll
        for (int h = 0; h < NG - 1; ++h) {
            const bool before = h < tg;
            g0 += before ? sTot[0][h][key] : 0.0f;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) dg0[kk] += before ? sTot[1 + kk][h][key] : 0.0f;
        }
        bool bad = false;
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const float Gj = g0 + Gt[j];
            bad |= !(fabsf(Gj) <= kMaxG);
            const float ei = exp_acc(-Gj), eq = OUT || j == SPT - 1 ? exp_acc(Gj) : 0.0f;
            const float kv = rk[j] * ei;
            const float qv = OUT ? rq[j] * eq : 0.0f;
            float dkv[K], dqv[K];
            chk = fmaf(kv, 0.0f, fmaf(qv, 0.0f, chk));
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const float dGj = dg0[kk] + dGt[kk][j];
                dkv[kk] = fmaf(-rk[j], dGj, rdk[kk][j]) * ei;
                dqv[kk] = OUT ? fmaf(rq[j], dGj, rdq[kk][j]) * eq : 0.0f;
                chk = fmaf(dkv[kk], 0.0f, fmaf(dqv[kk], 0.0f, chk));
                if (j == SPT - 1 && tg == NG - 1) sEnd[1 + kk][key] = dGj;
            }
            if (j == SPT - 1 && tg == NG - 1) sEnd[0][key] = eq;
            put(j, kv, dkv, qv, dqv);
        }
        if (bad || !(chk == 0.0f)) sBad[buf] = 1;
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(sBad[buf]) == 0) {
            fetch(tb + kChunk);
            products(tb, 0, kChunk, vv, dvv);
            decay();
        } else {
            // one step at a time: decay by the step, then its products alone
            for (int sub = 0; sub < kChunk; ++sub) {
                lds_barrier();
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const bool on = tg * SPT + j == sub;
                    float dkv[K], dqv[K];
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) {
                        dkv[kk] = on ? rdk[kk][j] : 0.0f;
                        dqv[kk] = OUT && on ? rdq[kk][j] : 0.0f;
                        if (on) sEnd[1 + kk][key] = rdg[kk][j];
                    }
                    if (on) sEnd[0][key] = exp_acc(rg[j]);
                    put(j, on ? rk[j] : 0.0f, dkv, OUT && on ? rq[j] : 0.0f, dqv);
                }
                float vs[4], dvs[K][4];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const bool on = 4 * qd + m == sub;
                    vs[m] = on ? vv[m] : 0.0f;
#pragma unroll
                    for (int kk = 0; kk < K; ++kk) dvs[kk][m] = on ? dvv[kk][m] : 0.0f;
                }
                lds_barrier();
                decay();
                products(tb, sub, sub + 1, vs, dvs);
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
// One thread per lane (bh, i, j), sequential over the block's segments.
// state [(1+K)][BH][DK][DV] enters and leaves; seg [BH][G][(1+K)][DK][DV]
// holds each segment's zero-start end state on entry and is overwritten with
// the true state entering the segment.  sums [BH][G][(1+K)][DK] as written
// by k_la_chunk<false>.
template <int K>
__global__ __launch_bounds__(kThreads) void k_la_carry(
    float *__restrict__ seg, const float *__restrict__ sums, float *__restrict__ state, int64_t BH, int64_t DK,
    int64_t DV, int G) {
    constexpr int GB = K == 1 ? 16 : 8;
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t per = DK * DV;
    if (idx >= BH * per) return;
    const int64_t bh = idx / per, r = idx % per, i = r / DV;
    const int64_t cs = BH * per;
    float s = state[idx], ds[K];
#pragma unroll
    for (int kk = 0; kk < K; ++kk) ds[kk] = state[(1 + kk) * cs + idx];
    for (int g0 = 0; g0 < G; g0 += GB) {
        float e0[GB], e1[K][GB], sg[GB], sdg[K][GB];
#pragma unroll
        for (int jj = 0; jj < GB; ++jj) {
            const int g = g0 + jj < G ? g0 + jj : G - 1;
            const int64_t base = (bh * G + g) * (1 + K);
            e0[jj] = seg[base * per + r];
            sg[jj] = sums[base * DK + i];
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                e1[kk][jj] = seg[(base + 1 + kk) * per + r];
                sdg[kk][jj] = sums[(base + 1 + kk) * DK + i];
            }
        }
#pragma unroll
        for (int jj = 0; jj < GB; ++jj) {
            if (g0 + jj >= G) break;
            const int64_t base = (bh * G + g0 + jj) * (1 + K);
            seg[base * per + r] = s;
#pragma unroll
            for (int kk = 0; kk < K; ++kk) seg[(base + 1 + kk) * per + r] = ds[kk];
            const float P = exp_series(sg[jj]);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) ds[kk] = fmaf(P, ds[kk], fmaf(P * sdg[kk][jj], s, e1[kk][jj]));
            s = fmaf(P, s, e0[jj]);
        }
    }
    state[idx] = s;
#pragma unroll
    for (int kk = 0; kk < K; ++kk) state[(1 + kk) * cs + idx] = ds[kk];
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
            const int64_t lanes = q.BH * ND;
            Timed tm(2, st);
            hipLaunchKernelGGL((k_la_carry<K>), dim3((unsigned)((lanes + kThreads - 1) / kThreads)), dim3(kThreads),
                               0, st, agg_h(), (const float *)agg_s(), state(), q.BH, (int64_t)DK, q.DV, G);
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
