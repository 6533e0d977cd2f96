// One galaxy (or chain) per workgroup of two waves: the approximate-path model for batches too
// small to fill the chip with a lane or two per galaxy.
//
// Same model, rules, operand rounding and summation order as approx_eval, so the results are the
// batched kernels'; only the FP64 total of the smooth mass is summed in another order.  A thread
// owns one age bin (its mass, derivatives and burst share stay in registers between the forward and
// the adjoint pass), and wave w takes every second block of 16 table rows (ages) of the contraction:
// the fragments of both z nodes are loaded into registers ahead of their use, the forward ones during
// the weights and the adjoint ones during the bands.  The galaxy fills all 16 rows of the matrix
// products, so every lane group holds its results.  The sums over bins run in the batched order, one
// sum per lane.  Nothing is shared between galaxies: no z sort, no record, no pass per z bucket.
//
// What bounds it: the serial chain of one evaluation (bins -> total -> contraction -> bands ->
// adjoint contraction -> sums) while the chip has free wave slots, then the wave slots and the 66 KB
// of table that each wave reads from L2.
#pragma once
#include "sps_eval.h"

namespace sps {

constexpr int PAIR_T = 2 * WAVE;
constexpr int PAIR_NB = 3;   // blocks of 16 table rows or ages per wave, at most

// ------------------------------------------------------------------ sums over a wave
template <int CTRL, int ROWS = 0xf>
__device__ inline double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}
__device__ inline float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double lane_value(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}
// the wave's sum, in every lane (all 64 lanes must call it): rotations by 8, 4, 2, 1 within each
// row of 16, then rows 1 and 3 take the row before them (row_bcast:15) and rows 2 and 3 row 1's
// total (row_bcast:31); lane 63 holds the sum
__device__ inline double wave_sum(double v) {
    v = dpp_add<0x128>(v);
    v = dpp_add<0x124>(v);
    v = dpp_add<0x122>(v);
    v = dpp_add<0x121>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return lane_value(v, 63);
}

// ------------------------------------------------------------------ per-workgroup state
// factors of the adjoint's sums over bins (see pair_sums)
enum { PX_NGBAR, PX_PSBAR, PX_BURST, PX_ONE, PX_COUNT };
enum { PY_PS, PY_D1, PY_D2, PY_D3, PY_PB, PY_DPB, PY_COUNT };
enum { PS_CBAR, PS_A0, PS_A1, PS_A2, PS_B0, PS_B1, PS_B2, PS_E1, PS_E2, PS_E3, PS_FBAR, PS_COUNT };

struct __attribute__((aligned(16))) PairLds {
    uint16_t hi[2][SLOT_W], lo[2][SLOT_W];   // contraction operands of the two nodes, BF16 hi and lo
    float t[SLOT_W];                         // T, then dP_age
    float px[PX_COUNT][SLOT_W], py[PY_COUNT][SLOT_W];
    float pz[NZ + 4], sum[PS_COUNT + 1];
    double S[2], d[2][4];
};

// a thread's age bin: fixed over a run
struct PairBin {
    float a_lo, a_hi, le_lo, le_hi;   // edges in Gyr and in log10 yr
    float up0, up1;                   // upper log-age edges of bins lane and lane + 64
    float met_hi, lam;                // lane j: upper edge of metallicity bin j, wavelength of band j
    bool own;
};
__device__ inline PairBin pair_bin(const DevConsts &k) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), i = min(tid, NA - 1);
    return PairBin{k.age_lo[i], k.age_hi[i], k.lage_lo[i], k.lage_hi[i], k.lage_hi[min(lane, NA - 1)],
                   k.lage_hi[min(lane + WAVE, NA - 1)], k.met_hi[min(lane, NZ - 1)],
                   k.lam_eff[min(lane, NB_MAX - 1)], tid < NA};
}
// log-age edge e (0 .. NA), from the lanes that hold the upper edges
__device__ inline float pair_edge(const PairBin &b, int e) {
    if (e == 0) return -INFINITY;
    return (e <= WAVE) ? lane_value(b.up0, e - 1) : lane_value(b.up1, e - 1 - WAVE);
}

// wave w's fragments (qf or qa of sps_internal.h) of nodes kb and kb + 1: blocks 2 t + w, BF16 hi and lo
struct PairTab {
    b8v h[2][PAIR_NB][KSTEPS], l[2][PAIR_NB][KSTEPS];
};
__device__ inline void pair_load(PairTab &t, const DevConsts &k, const uint16_t *q, int kb, int w, int lane, int nbk) {
    const uint16_t *b = q + (size_t)kb * QB_NODE + lane * 8;
    const size_t lo_off = (size_t)k.n_z * QB_NODE;
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) {
        if (2 * nb + w >= nbk) break;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
            for (int nd = 0; nd < 2; ++nd) {
                const size_t o = (size_t)((2 * nb + w) * KSTEPS + ks) * 512 + (size_t)nd * QB_NODE;
                t.h[nd][nb][ks] = *(const b8v *)(b + o);
                t.l[nd][nb][ks] = *(const b8v *)(b + lo_off + o);
            }
    }
}

__device__ inline void split_store(float x, uint16_t *hi, uint16_t *lo) {
    const __bf16 h = (__bf16)x, l = (__bf16)(x - (float)h);
    *hi = __builtin_bit_cast(uint16_t, h);
    *lo = __builtin_bit_cast(uint16_t, l);
}

// S.t[n] = sum over both nodes and k of operand[k] table[k][n], the wave's blocks of n (each
// accumulator takes its products in contract()'s order)
__device__ inline void pair_contract(const PairTab &t, PairLds &S, int w, int lane, int nbk) {
    const int x = lane & 15, lk = lane >> 4;
    v4f acc[PAIR_NB];
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) acc[nb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int o = 32 * ks + 8 * lk;
        const b8v a0h = *(const b8v *)(S.hi[0] + o), a0l = *(const b8v *)(S.lo[0] + o);
        const b8v a1h = *(const b8v *)(S.hi[1] + o), a1l = *(const b8v *)(S.lo[1] + o);
#pragma unroll
        for (int nb = 0; nb < PAIR_NB; ++nb) {
            if (2 * nb + w >= nbk) break;
            acc[nb] = mfma3(a0h, a0l, t.h[0][nb][ks], t.l[0][nb][ks], acc[nb]);
            acc[nb] = mfma3(a1h, a1l, t.h[1][nb][ks], t.l[1][nb][ks], acc[nb]);
        }
    }
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) {
        if (2 * nb + w >= nbk) break;
        if (lk == 0) S.t[16 * (2 * nb + w) + x] = acc[nb][0];
    }
}

// The adjoint's sums over the age bins, each in the batched kernels' order: with PG lanes per galaxy
// there, bins q, q + PG, ... in turn for each q, then the PG sums added.  Lane PG s + q of wave 0
// takes part q of sum s.
template <int PG>
__device__ inline void pair_sums(PairLds &S, int lane) {
    static_assert(PG * PS_COUNT <= WAVE, "a lane per partial sum");
    const int s = min(lane / PG, PS_COUNT - 1), q = lane % PG;
    const int xi = s == PS_FBAR ? PX_NGBAR : s <= PS_A2 ? PX_PSBAR : (s == PS_E1 || s == PS_E2) ? PX_BURST : PX_ONE;
    const int yi = (s == PS_CBAR || s == PS_FBAR) ? PY_PS : s <= PS_A2 ? PY_D1 + s - PS_A0
                   : s <= PS_B2 ? PY_D1 + s - PS_B0 : s == PS_E2 ? PY_PB : PY_DPB;
    const float *xp = S.px[xi], *yp = S.py[yi];
    float v = 0.0f;
    constexpr int STEP = 4;
#pragma unroll 4
    for (int i = 0; i < SLOT_W; i += STEP) {
        const v4f a = *(const v4f *)(xp + i), b = *(const v4f *)(yp + i);
#pragma unroll
        for (int e = 0; e < STEP; e += PG)
            v = (PG == 1) ? fmaf(a[e], b[e], v) : fmaf(q ? a[e + PG - 1] : a[e], q ? b[e + PG - 1] : b[e], v);
    }
    // the burst part of fbar follows its smooth part
    if (s == PS_FBAR) {
#pragma unroll 2
        for (int i = 0; i < SLOT_W; i += STEP) {
            const v4f a = *(const v4f *)(xp + i), b = *(const v4f *)(S.py[PY_PB] + i);
#pragma unroll
            for (int e = 0; e < STEP; e += PG)
                v = (PG == 1) ? fmaf(a[e], -b[e], v) : fmaf(q ? a[e + PG - 1] : a[e], q ? -b[e + PG - 1] : -b[e], v);
        }
    }
    if (PG == 2) v += __shfl_xor(v, 1, WAVE);
    if (q == 0 && lane < PG * PS_COUNT) S.sum[s] = v;
}

// ------------------------------------------------------------------ one evaluation
// Every thread of the workgroup calls it with the same galaxy.  q: the wave's forward fragments of
// nodes kb and kb + 1 on entry; the adjoint's are loaded into it (qa).  PK and PG: the columns'
// 24-bit rounding and the lanes per galaxy of the batched kernel that it stands in for (the one-shot
// kernels: true, 1; the samplers: false, 2).  ob, sg_f: lane b of each wave holds band b's
// observation and sigma (VJP: ob its adjoint).  MODE_MAGS: lane b gets band b's magnitude in
// `mag`.  Else: logl, and with MODE_LOGL_GRAD the gradient, in every thread.
template <int MODE, bool PK, int PG, bool VJP>
__device__ __forceinline__ void pair_eval(const DevConsts &k, const PairBin &bin, PairTab &q, const uint16_t *qa,
                                          int kb, PairLds &S, int sfh, const float (&th)[NP], float zf, float f,
                                          double t_obs, double m0, float ob, float sg_f, uint32_t mask, float &mag,
                                          double &logl, float (&gr)[NP]) {
    constexpr bool GRAD = (MODE == MODE_LOGL_GRAD);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & (WAVE - 1);
    const int nb = k.n_band;
    const float t_obs_f = (float)t_obs;
    const bool dpl = (sfh == SPS_SFH_DPL);

    // ---- weights: the thread's bin
    float m = 0.0f, d1 = 0.0f, d2 = 0.0f, d3 = 0.0f;
    if (bin.own) {
        if (dpl) {
            Dpl p = make_dpl(th[1], th[2], th[3]);
            dpl_at_obs(p, t_obs_f);
            dpl_bin<GRAD>(bin.a_lo, bin.a_hi, t_obs_f, p, m, d1, d2, d3);
        } else {
            logn_bin<GRAD>(bin.a_lo, bin.a_hi, t_obs_f, make_logn(th[1], th[2]), m, d1, d2);
        }
    }
    {
        const double s = wave_sum((double)m);
        if (lane == 0) S.S[w] = s;
    }
    // metallicity bin `lane` (both waves alike): its upper edge, the lower one from the lane before
    const float inv_sz = 1.0f / k.sigma_logz;
    float pz = 0.0f, dpz = 0.0f;
    {
        const bool top = lane >= NZ - 1;
        const float xe = top ? INFINITY : (bin.met_hi - th[6]) * inv_sz;
        const float te = top ? 0.0f : 0.5f * erfcf(0.7071067811865475f * fabsf(xe));
        const float de = top ? 0.0f : phi_f(xe);
        float xp = __shfl_up(xe, 1, WAVE), tp = __shfl_up(te, 1, WAVE), dp = __shfl_up(de, 1, WAVE);
        if (lane == 0) {
            xp = -INFINITY;
            tp = dp = 0.0f;
        }
        if (lane < NZ) {
            pz = (xp > 0.0f) ? tp - te : ((xe <= 0.0f) ? te - tp : 1.0f - tp - te);
            dpz = (dp - de) * inv_sz;
            if (w == 0) S.pz[lane] = pz;
        }
    }
    __syncthreads();
    const double Sm = S.S[0] + S.S[1];
    // burst: first bin of the window (every bin before it ends at or below the window's start)
    const float l_obs = (float)log10_split(t_obs * 1e9), mu = th[5], inv_s3 = 1.0f / (3.0f * k.burst_sig);
    const float v0 = mu - 3.0f * k.burst_sig;
    const unsigned long long above0 = __ballot(bin.up0 > v0), above1 = __ballot(bin.up1 > v0);
    const int i0 = above0 ? __builtin_ctzll(above0) : (above1 ? min(NA - 1, WAVE + __builtin_ctzll(above1)) : NA - 1);
    const int i_end = min(i0 + k.burst_nbins, NA);
    const float Zb = burst_mass(burst_edge_at<false>(pair_edge(bin, i0), l_obs, mu, inv_s3),
                                burst_edge_at<false>(pair_edge(bin, i_end), l_obs, mu, inv_s3));
    const BurstEdge b_lo = burst_edge_at<GRAD>(bin.le_lo, l_obs, mu, inv_s3);
    const BurstEdge b_hi = burst_edge_at<GRAD>(bin.le_hi, l_obs, mu, inv_s3);
    const bool in_win = bin.own && tid >= i0 && tid < i_end;
    const float bm = burst_mass(b_lo, b_hi);
    const float fb = th[4], sm = (1.0f - fb) * (float)(1.0 / Sm), bz = (Zb > 0.0f) ? fb / Zb : 0.0f;
    // the column holds P_age / scale, as in the batched kernels
    const float scale = (sm > 0.0f) ? sm : 1.0f, cb = (sm > 0.0f) ? bz / sm : bz;
    if (tid < SLOT_W) {
        float c = (sm > 0.0f) ? m : 0.0f;
        if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
        if (in_win) c = fmaf(cb, bm, c);
        if (!bin.own) c = 0.0f;
        if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
#pragma unroll
        for (int nd = 0; nd < 2; ++nd) split_store(c * ((nd ? f : 1.0f - f) * scale), &S.hi[nd][tid], &S.lo[nd][tid]);
    }
    __syncthreads();

    // ---- T, then the adjoint's fragments on their way
    pair_contract(q, S, w, lane, row_blocks(nb));
    if (GRAD) pair_load(q, k, qa, kb, w, lane, AGE_BLK);
    __syncthreads();

    // ---- bands: lane b of each wave (both waves alike)
    const int R = nb * NZ;
    const bool is_b = lane < nb;
    const int bl = is_b ? lane : 0;
    double ll = 0.0;
    float sbar = 0.0f, gm = 0.0f, fbar_b = 0.0f, f7 = 0.0f, f8 = 0.0f, f9 = 0.0f;
    {
        double sb = 0.0;
#pragma unroll
        for (int j = 0; j < NZ; ++j) sb += (double)S.pz[j] * (double)S.t[bl * NZ + j];
        const DustVal d = dust_at(bin.lam / ((1.0f + zf) * 5500.0f), th[7], th[8], th[9]);
        const double mg = m0 - 2.5 * log10_split((double)d.F * sb);
        mag = (float)mg;
        if (MODE == MODE_MAGS) return;
        if (is_b && ((mask >> bl) & 1u)) {
            if (VJP) {
                gm = ob;
            } else {
                const double sg = sg_f;
                const double r = (mg - (double)ob) / sg;
                ll = -0.5 * r * r - (double)logf(sg_f * 2.5066282746310002f);
                gm = (float)(-r / sg);
            }
            if (MODE != MODE_LOGL) {
                const float c = gm * (-2.5f / LN10F);
                sbar = (float)(c / sb);
                fbar_b = c / d.F;
                f7 = d.dF_tauv;
                f8 = d.dF_delta;
                f9 = d.dF_floor;
            }
        }
    }
    // sums over the bands in the batched order: bands q, q + PG, ... for each q < PG, then those added
    logl = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p) gr[p] = 0.0f;
#pragma unroll
    for (int q0 = 0; q0 < PG; ++q0) {
        double l = 0.0;
        float v0_ = 0.0f, v7 = 0.0f, v8 = 0.0f, v9 = 0.0f;
#pragma unroll
        for (int b = q0; b < NB_MAX; b += PG) {
            if (b >= nb) break;
            l += lane_value(ll, b);
            if (MODE == MODE_LOGL) continue;
            const float fbb = lane_value(fbar_b, b);
            v0_ += -2.5f * lane_value(gm, b);
            v7 = fmaf(fbb, lane_value(f7, b), v7);
            v8 = fmaf(fbb, lane_value(f8, b), v8);
            v9 = fmaf(fbb, lane_value(f9, b), v9);
        }
        logl += l;
        gr[0] += v0_;
        gr[7] += v7;
        gr[8] += v8;
        gr[9] += v9;
    }
    if (!GRAD) return;

    // ---- d/dmu_Z = sum_j dP_Z(j)/dmu sum_b sbar_b T[b][j], and the operands C = sbar_b P_Z(j)
    {
        const int j = min(lane, NZ - 1);
        float s = 0.0f;
#pragma unroll
        for (int q0 = 0; q0 < PG; ++q0) {
            float v = 0.0f;
#pragma unroll
            for (int b = q0; b < NB_MAX; b += PG) {
                if (b >= nb) break;
                v = fmaf(lane_value(sbar, b), S.t[b * NZ + j], v);
            }
            s += v;
        }
        float mbar = 0.0f;
#pragma unroll
        for (int t = 0; t < NZ; ++t) mbar = fmaf(lane_value(s, t), lane_value(dpz, t), mbar);
        gr[6] = mbar;
        const float wnode = w ? f : 1.0f - f;   // wave w writes node w's operands
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int r = lane + WAVE * t, rb = min(r / NZ, nb - 1), rj = r % NZ;
            const float sr = __shfl(sbar, rb, WAVE), pr = S.pz[rj];
            float c = (r < R) ? sr * pr : 0.0f;
            if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
            if (r < SLOT_W) split_store(c * wnode, &S.hi[w][r], &S.lo[w][r]);
        }
    }
    __syncthreads();

    // ---- dP_age
    pair_contract(q, S, w, lane, AGE_BLK);
    __syncthreads();

    // ---- weights adjoint: the thread's bin, then the sums over bins
    const float invS = (float)(1.0 / Sm), invZ = (Zb > 0.0f) ? 1.0f / Zb : 0.0f;
    if (tid < SLOT_W) {
        float gbar = S.t[tid];
        if (PK) gbar = __uint_as_float(round24(gbar) & 0xffffff00u);
        if (!bin.own) gbar = 0.0f;
        const float psbar = (1.0f - fb) * gbar;
        S.px[PX_NGBAR][tid] = -gbar;
        S.px[PX_PSBAR][tid] = psbar;
        S.px[PX_BURST][tid] = in_win ? fb * gbar : 0.0f;
        S.px[PX_ONE][tid] = 1.0f;
        S.py[PY_PS][tid] = dpl ? m * invS : (float)((double)m / Sm);
        S.py[PY_D1][tid] = d1;
        S.py[PY_D2][tid] = d2;
        S.py[PY_D3][tid] = d3;
        S.py[PY_PB][tid] = in_win ? bm * invZ : 0.0f;
        S.py[PY_DPB][tid] = in_win ? (b_lo.d - b_hi.d) * inv_s3 : 0.0f;
    }
    if (!dpl) {   // FP64 sums of the log-normal derivatives
        const double pb = (1.0f - fb) * (bin.own ? -S.px[PX_NGBAR][min(tid, SLOT_W - 1)] : 0.0f);
        const double v[4] = {pb * (double)d1, pb * (double)d2, (double)d1, (double)d2};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double s = wave_sum(v[j]);
            if (lane == 0) S.d[w][j] = s;
        }
    }
    __syncthreads();
    if (w == 0) pair_sums<PG>(S, lane);
    __syncthreads();
    const float cbar = S.sum[PS_CBAR];
    if (dpl) {
#pragma unroll
        for (int j = 0; j < 3; ++j) gr[1 + j] = (S.sum[PS_A0 + j] - cbar * S.sum[PS_B0 + j]) * invS;
    } else {
        gr[1] = (float)((S.d[0][0] + S.d[1][0] - (double)cbar * (S.d[0][2] + S.d[1][2])) / Sm);
        gr[2] = (float)((S.d[0][1] + S.d[1][1] - (double)cbar * (S.d[0][3] + S.d[1][3])) / Sm);
    }
    gr[4] = S.sum[PS_FBAR];
    gr[5] = (S.sum[PS_E1] - S.sum[PS_E2] * S.sum[PS_E3]) * invZ;
}

}  // namespace sps
