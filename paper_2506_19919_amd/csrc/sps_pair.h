// One galaxy (or chain) per workgroup of two waves: the approximate-path model for batches too
// small to fill the chip with a lane or two per galaxy.
//
// Same model, rules, operand rounding and FP32 summation order as approx_eval with one lane per galaxy (the
// samplers': with two), so the results are that kernel's; only the FP64 sums (the total of the smooth mass, the
// log-normal derivatives) are taken in another order.  A thread
// owns one age bin (its mass, derivatives and burst share stay in registers between the forward and
// the adjoint pass), and wave w takes every second block of 16 table rows (ages) of the contraction:
// the fragments of both z nodes are loaded into registers ahead of their use, the forward ones during
// the weights and the adjoint ones during the bands.  The galaxy fills all 16 rows of the matrix
// products, so every lane group holds its results.  The sums over bins run in the batched order, one
// sum per lane.  Nothing is shared between galaxies: no z sort, no record, no pass per z bucket.
//
// What bounds it: the serial chain of one evaluation (bins -> total -> contraction -> bands ->
// adjoint contraction -> sums) while the chip has free wave slots, then the wave slots and the table that
// each wave reads from L2, 36 KB per contraction.
#pragma once
#include "sps_eval.h"

namespace sps {

constexpr int PAIR_T = 2 * WAVE;
constexpr int PAIR_NB = AGE_BLK / 2;   // blocks of 16 table rows or ages per wave (rows past the bands are zero)

// ------------------------------------------------------------------ sums over a wave
template <int CTRL, int ROWS = 0xf>
__device__ inline float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
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
template <typename T>
__device__ inline T wave_sum(T v) {
    v = dpp_add<0x128>(v);
    v = dpp_add<0x124>(v);
    v = dpp_add<0x122>(v);
    v = dpp_add<0x121>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return lane_value(v, 63);
}

// Between LDS writes of some lanes of a wave and reads of the same words by others (all 64 lanes must
// call it).  A wave's LDS operations are done in order, so it emits nothing: it keeps the compiler from moving them
// past each other.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ per-workgroup state
// factors of the adjoint's sums over bins (see pair_sums)
enum { PX_NGBAR, PX_PSBAR, PX_BURST, PX_ONE, PX_INVS3, PX_COUNT };
enum { PY_PS, PY_D1, PY_D2, PY_D3, PY_PB, PY_DPB, PY_DD, PY_COUNT };
enum { PS_CBAR, PS_A0, PS_A1, PS_A2, PS_B0, PS_B1, PS_B2, PS_E1, PS_E2, PS_E3, PS_FBAR, PS_MET, PS_COUNT };

// rows of 100 floats: 16-byte aligned, and the sums' lanes, each on its own row, on different banks
constexpr int PAIR_ROW = SLOT_W + 4;
struct __attribute__((aligned(16))) PairLds {
    uint16_t hi[2][SLOT_W], lo[2][SLOT_W];   // contraction operands of the two nodes, BF16 hi and lo
    float t[SLOT_W];                         // T, then dP_age
    float px[PX_COUNT][PAIR_ROW], py[PY_COUNT][PAIR_ROW];
    float met[2][16];                        // dlogL/dP_Z and dP_Z/dmu, zero from NZ on
    float pz[16], th[12];
    float sbar[NB_MAX], bx[4][NB_MAX], by[4][NB_MAX];   // per band: dlogL/d(sum), and factors of gr 0, 7, 8, 9
    double ll[NB_MAX], S[2], d[2][4];
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

// wave w's fragments (qf or qa of sps_internal.h) of nodes kb and kb + 1: blocks 2 t + w, BF16 hi and
// lo.  The first PAIR_KRES k-steps are loaded ahead, the rest inside the contraction: one leaves 128
// registers, four waves per SIMD (value+gradient, us at 4096 / 8192 galaxies: 38 / 63; two ahead, three waves, 41 / 69;
// all three ahead, two waves, 44 / 75; at one galaxy the same).
constexpr int PAIR_KRES = 1;
struct PairTab {
    b8v h[PAIR_KRES][2][PAIR_NB], l[PAIR_KRES][2][PAIR_NB];
};
__device__ inline void pair_load_step(const DevConsts &k, const uint16_t *b, int ks, int w, b8v (&h)[2][PAIR_NB],
                                      b8v (&l)[2][PAIR_NB]) {
    const size_t lo_off = (size_t)k.n_z * QB_NODE;
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) {
#pragma unroll
        for (int nd = 0; nd < 2; ++nd) {
            const size_t o = (size_t)((2 * nb + w) * KSTEPS + ks) * 512 + (size_t)nd * QB_NODE;
            h[nd][nb] = *(const b8v *)(b + o);
            l[nd][nb] = *(const b8v *)(b + lo_off + o);
        }
    }
}
__device__ inline void pair_load(PairTab &t, const DevConsts &k, const uint16_t *q, int kb, int w, int lane) {
    const uint16_t *b = q + (size_t)kb * QB_NODE + lane * 8;
#pragma unroll
    for (int ks = 0; ks < PAIR_KRES; ++ks) pair_load_step(k, b, ks, w, t.h[ks], t.l[ks]);
}

__device__ inline void split_store(float x, uint16_t *hi, uint16_t *lo) {
    const __bf16 h = (__bf16)x, l = (__bf16)(x - (float)h);
    *hi = __builtin_bit_cast(uint16_t, h);
    *lo = __builtin_bit_cast(uint16_t, l);
}

// S.t[n] = sum over both nodes and k of operand[k] table[k][n], the wave's blocks of n (each
// accumulator takes its products in contract()'s order)
__device__ inline void pair_contract(const PairTab &t, const DevConsts &k, const uint16_t *q, int kb, PairLds &S, int w,
                                     int lane) {
    const int x = lane & 15, lk = lane >> 4;
    const uint16_t *qb = q + (size_t)kb * QB_NODE + lane * 8;
    b8v th[KSTEPS - PAIR_KRES + 1][2][PAIR_NB], tl[KSTEPS - PAIR_KRES + 1][2][PAIR_NB];
#pragma unroll
    for (int ks = PAIR_KRES; ks < KSTEPS; ++ks) pair_load_step(k, qb, ks, w, th[ks - PAIR_KRES], tl[ks - PAIR_KRES]);
    v4f acc[PAIR_NB];
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) acc[nb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int o = 32 * ks + 8 * lk;
        const b8v a0h = *(const b8v *)(S.hi[0] + o), a0l = *(const b8v *)(S.lo[0] + o);
        const b8v a1h = *(const b8v *)(S.hi[1] + o), a1l = *(const b8v *)(S.lo[1] + o);
        const auto &h = ks < PAIR_KRES ? t.h[ks < PAIR_KRES ? ks : 0] : th[ks < PAIR_KRES ? 0 : ks - PAIR_KRES];
        const auto &l = ks < PAIR_KRES ? t.l[ks < PAIR_KRES ? ks : 0] : tl[ks < PAIR_KRES ? 0 : ks - PAIR_KRES];
#pragma unroll
        for (int nb = 0; nb < PAIR_NB; ++nb) {
                acc[nb] = mfma3(a0h, a0l, h[0][nb], l[0][nb], acc[nb]);
            acc[nb] = mfma3(a1h, a1l, h[1][nb], l[1][nb], acc[nb]);
        }
    }
#pragma unroll
    for (int nb = 0; nb < PAIR_NB; ++nb) {
        if (lk == 0) S.t[16 * (2 * nb + w) + x] = acc[nb][0];
    }
}

// The adjoint's sums, each in the batched kernels' order with one fused multiply-add per term, as their
// loops compile to: with PG lanes per galaxy there, bins q, q + PG, ... in turn for each q, then the
// PG sums added.  Lane PG s + q of the wave takes part q of sum s; the sum is returned in lane PG s.
// Bin i's factors lie at pair_at(i): each part's bins are consecutive.
template <int PG>
__device__ inline int pair_at(int i) {
    return PG == 1 ? i : (i & 1) * (SLOT_W / 2) + (i >> 1);
}
template <int PG>
__device__ inline float pair_sums(const PairLds &S, int lane, int i0, int i_end) {
    static_assert(PG * PS_COUNT <= WAVE, "a lane per partial sum");
    constexpr int LEN = SLOT_W / PG, CH = 16 / PG;
    const int s = min(lane / PG, PS_COUNT - 1), q = lane % PG;
    const int xi = s == PS_FBAR ? PX_NGBAR : s <= PS_A2 ? PX_PSBAR : s <= PS_B2 ? PX_ONE : s == PS_E3 ? PX_INVS3 : PX_BURST;
    const int yi = (s == PS_CBAR || s == PS_FBAR) ? PY_PS : s <= PS_A2 ? PY_D1 + s - PS_A0
                   : s <= PS_B2 ? PY_D1 + s - PS_B0 : s == PS_E2 ? PY_PB : s == PS_E3 ? PY_DD : PY_DPB;
    const float *xp = S.px[xi] + q * LEN, *yp = S.py[yi] + q * LEN;
    float v = 0.0f;
#pragma unroll
    for (int c = 0; c < LEN; c += 24) {
        v4f a[6], b[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            a[e] = *(const v4f *)(xp + c + 4 * e);
            b[e] = *(const v4f *)(yp + c + 4 * e);
        }
#pragma unroll
        for (int e = 0; e < 24; ++e) v = fmaf(a[e / 4][e % 4], b[e / 4][e % 4], v);
    }
    // the burst part of fbar follows its smooth part, over the window's bins (zero around them); the
    // metallicity sum, in order
    if (s == PS_MET) v = 0.0f;
    const float *x2 = s == PS_MET ? S.met[0] : S.px[PX_NGBAR] + q * LEN;
    const float *y2 = s == PS_MET ? S.met[1] : S.py[PY_PB] + q * LEN;
    const int c0 = i0 / PG & ~(CH - 1), c1 = (i_end + PG - 1) / PG;
    if (s >= PS_FBAR) {
        for (int c = c0; c < c1; c += CH) {
            const bool met = s == PS_MET;
            if (met && c > c0) break;
            const int at = met ? 0 : c;
            v4f a[4], b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = (PG == 2 && !met && e >= 2) ? 0 : 4 * e;
                a[e] = *(const v4f *)(x2 + at + o);
                b[e] = *(const v4f *)(y2 + at + o);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (met ? e < NZ : e < CH) v = fmaf(met ? a[e / 4][e % 4] : -a[e / 4][e % 4], b[e / 4][e % 4], v);
            }
        }
    }
    if (PG == 2) {
        if (s == PS_MET && q != 0) v = 0.0f;   // one part holds the whole of it
        v += __shfl_xor(v, 1, WAVE);
    }
    return v;
}

// ------------------------------------------------------------------ one evaluation
// Every thread of the workgroup calls it with the same galaxy.  q: the wave's forward fragments of
// nodes kb and kb + 1 on entry; the adjoint's are loaded into it.  wz0, wz1: the nodes' z weights (1 - f and f, or 0 outside the table:
// T = 0, as in the batched kernels).  PK and PG: the columns'
// 24-bit rounding and the lanes per galaxy of the batched kernel that it stands in for (the one-shot
// kernels: true, 1; the samplers: false, 2).  ob, sg_f: lane b of wave 0 holds band b's
// observation and sigma (VJP: ob its adjoint).  Results in wave 0: MODE_MAGS: lane b gets band b's
// magnitude in `mag`.  Else: logl in every lane, and with MODE_LOGL_GRAD lane p gets gradient component p.
template <int MODE, bool PK, int PG, bool VJP>
__device__ __forceinline__ void pair_eval(const DevConsts &k, const PairBin &bin, PairTab &q, const uint16_t *qa,
                                          const uint16_t *qf, int kb, PairLds &S, int sfh, const float (&th)[NP],
                                          float zf, float wz0, float wz1, double t_obs, double m0, float ob, float sg_f, uint32_t mask, float &mag,
                                          double &logl, float &gp, bool fuse_odd = true) {
    constexpr bool GRAD = (MODE == MODE_LOGL_GRAD);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & (WAVE - 1);
    const int nb = k.n_band;
    const float t_obs_f = (float)t_obs;
    const bool dpl = (sfh == SPS_SFH_DPL);

    // ---- weights: the thread's bin.  Wave 1 holds the oldest bins, whose panels take longest: wave 0
    // does the per-galaxy work (metallicity, dust) meanwhile, and the bands later
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
    DustVal dust{};
    if (w == 0) {
        // metallicity bin `lane`: its upper edge, the lower one from the lane before
        const float inv_sz = 1.0f / k.sigma_logz;
        const bool top = lane >= NZ - 1;
        const float xe = top ? INFINITY : (bin.met_hi - th[6]) * inv_sz;
        const float te = top ? 0.0f : 0.5f * erfcf(0.7071067811865475f * fabsf(xe));
        constexpr float C = 0.3989422804014327f;
        const float ee = top ? 0.0f : expf(-0.5f * xe * xe), de = C * ee;
        float xp = __shfl_up(xe, 1, WAVE), tp = __shfl_up(te, 1, WAVE), ep = __shfl_up(ee, 1, WAVE);
        if (lane == 0) {
            xp = -INFINITY;
            tp = ep = 0.0f;
        }
        if (lane < NZ) {
            // met_weights' differences of densities, fused as its unrolled loop is: the odd edges' products,
            // or (k_hmc_init) each lower edge's
            S.met[1][lane] = ((lane & 1) && fuse_odd ? fmaf(-C, ee, C * ep) : fmaf(C, ep, -de)) * inv_sz;
            S.pz[lane] = (xp > 0.0f) ? tp - te : ((xe <= 0.0f) ? te - tp : 1.0f - tp - te);
        }
        dust = dust_at(bin.lam / ((1.0f + zf) * 5500.0f), th[7], th[8], th[9]);
    }
    // burst: first bin of the window (every bin before it ends at or below the window's start)
    const float l_obs = (float)log10_split(t_obs * 1e9), mu = th[5], inv_s3 = 1.0f / (3.0f * k.burst_sig);
    const float v0 = mu - 3.0f * k.burst_sig;
    const unsigned long long above0 = __ballot(bin.up0 > v0), above1 = __ballot(bin.up1 > v0);
    const int i0 = above0 ? __builtin_ctzll(above0) : (above1 ? min(NA - 1, WAVE + __builtin_ctzll(above1)) : NA - 1);
    const int i_end = min(i0 + k.burst_nbins, NA);
    const float Zb = burst_mass(burst_edge_at<false>(pair_edge(bin, i0), l_obs, mu, inv_s3),
                                burst_edge_at<false>(pair_edge(bin, i_end), l_obs, mu, inv_s3));
    const float fb = th[4], bz = (Zb > 0.0f) ? fb / Zb : 0.0f;
    const bool in_win = bin.own && tid >= i0 && tid < i_end;
    float bm = 0.0f, b_dd = 0.0f;   // the bin's burst mass and difference of edge densities
    if (in_win) {
        const BurstEdge b_lo = burst_edge_at<GRAD>(bin.le_lo, l_obs, mu, inv_s3);
        const BurstEdge b_hi = burst_edge_at<GRAD>(bin.le_hi, l_obs, mu, inv_s3);
        bm = burst_mass(b_lo, b_hi);
        b_dd = b_lo.d - b_hi.d;
    }
    __syncthreads();
    const double Sm = S.S[0] + S.S[1];
    const float sm = (1.0f - fb) * (float)(1.0 / Sm);
    // the column holds P_age / scale, as in the batched kernels
    const float scale = (sm > 0.0f) ? sm : 1.0f, cb = (sm > 0.0f) ? bz / sm : bz;
    if (tid < SLOT_W) {
        float c = (sm > 0.0f) ? m : 0.0f;
        if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
        if (in_win) c = fmaf(cb, bm, c);
        if (!bin.own) c = 0.0f;
        if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
#pragma unroll
        for (int nd = 0; nd < 2; ++nd) split_store(c * ((nd ? wz1 : wz0) * scale), &S.hi[nd][tid], &S.lo[nd][tid]);
    }
    __syncthreads();

    // ---- T, then the adjoint's fragments on their way
    pair_contract(q, k, qf, kb, S, w, lane);
    if (GRAD) pair_load(q, k, qa, kb, w, lane);
    __syncthreads();

    // ---- bands: lane b of wave 0
    gp = 0.0f;
    if (w == 0) {
        const int R = nb * NZ;
        const bool is_b = lane < nb;
        const int bl = is_b ? lane : 0;
        double sb = 0.0;
#pragma unroll
        for (int j = 0; j < NZ; ++j) sb += (double)S.pz[j] * (double)S.t[bl * NZ + j];
        const double mg = m0 - 2.5 * log10_split((double)dust.F * sb);
        mag = (float)mg;
        if (MODE != MODE_MAGS) {
            double ll = 0.0;
            float sbar = 0.0f, gm = 0.0f, fbar_b = 0.0f, f7 = 0.0f, f8 = 0.0f, f9 = 0.0f;
            if (is_b && ((mask >> bl) & 1u)) {
                if (VJP) {
                    gm = ob;
                } else {
                    const double sg = sg_f;
                    const double r = (mg - (double)ob) / sg;
                    ll = -0.5 * r * r - (double)logf(sg_f * 2.5066282746310002f);
                    gm = (float)(-r / sg);
                }
                const float c = gm * (-2.5f / LN10F);
                sbar = (float)(c / sb);
                fbar_b = c / dust.F;
                f7 = dust.dF_tauv;
                f8 = dust.dF_delta;
                f9 = dust.dF_floor;
            }
            if (lane < NB_MAX) {
                S.ll[lane] = ll;
                if (GRAD) {
                    S.sbar[lane] = sbar;
                    S.bx[0][lane] = -2.5f;
                    S.bx[1][lane] = S.bx[2][lane] = S.bx[3][lane] = fbar_b;
                    S.by[0][lane] = gm;
                    S.by[1][lane] = f7;
                    S.by[2][lane] = f8;
                    S.by[3][lane] = f9;
                }
            }
            wave_sync();
            // sums over the bands in the batched order: bands q, q + PG, ... for each q < PG, then those
            // added (the entries past the bands are zero)
            logl = 0.0;
            const int row = lane == 0 ? 0 : min(max(lane - 6, 1), 3);   // lane p = 0, 7, 8, 9: gr[p]
#pragma unroll
            for (int q0 = 0; q0 < PG; ++q0) {
                double l = 0.0;
                float v = 0.0f;
#pragma unroll
                for (int b = q0; b < NB_MAX; b += PG) {
                    l += S.ll[b];
                    if (GRAD) v = fmaf(S.bx[row][b], S.by[row][b], v);
                }
                logl += l;
                gp += v;
            }
        }
        if (GRAD) {
            // d/dmu_Z = sum_j dP_Z(j)/dmu sum_b sbar_b T[b][j] (the last sum in pair_sums), and the operands
            // C = sbar_b P_Z(j)
            const int j = min(lane, NZ - 1);
            float s = 0.0f;
#pragma unroll
            for (int q0 = 0; q0 < PG; ++q0) {
                float v = 0.0f;
#pragma unroll
                for (int b = q0; b < NB_MAX; b += PG) v = fmaf(S.sbar[b], S.t[b * NZ + j], v);
                s += v;
            }
            if (lane < NZ) S.met[0][lane] = s;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int r = lane + WAVE * t;
                float c = (r < R) ? S.sbar[min(r / NZ, NB_MAX - 1)] * S.pz[r % NZ] : 0.0f;
                if (PK) c = __uint_as_float(round24(c) & 0xffffff00u);
                if (r < SLOT_W) {
                    split_store(c * wz0, &S.hi[0][r], &S.lo[0][r]);
                    split_store(c * wz1, &S.hi[1][r], &S.lo[1][r]);
                }
            }
        }
    }
    if (!GRAD) return;
    __syncthreads();

    // ---- dP_age
    pair_contract(q, k, qa, kb, S, w, lane);
    __syncthreads();

    // ---- weights adjoint: the thread's bin, then the sums over bins
    const float invS = (float)(1.0 / Sm), invZ = (Zb > 0.0f) ? 1.0f / Zb : 0.0f;
    if (tid < SLOT_W) {
        float gbar = S.t[tid];
        if (PK) gbar = __uint_as_float(round24(gbar) & 0xffffff00u);
        if (!bin.own) gbar = 0.0f;
        const int at = pair_at<PG>(tid);
        S.px[PX_NGBAR][at] = -gbar;
        S.px[PX_PSBAR][at] = (1.0f - fb) * gbar;
        S.px[PX_BURST][at] = in_win ? fb * gbar : 0.0f;
        S.px[PX_ONE][at] = 1.0f;
        S.px[PX_INVS3][at] = inv_s3;
        S.py[PY_PS][at] = dpl ? m * invS : (float)((double)m / Sm);
        S.py[PY_D1][at] = d1;
        S.py[PY_D2][at] = d2;
        S.py[PY_D3][at] = d3;
        S.py[PY_PB][at] = bm * invZ;
        S.py[PY_DPB][at] = b_dd * inv_s3;
        S.py[PY_DD][at] = b_dd;
    }
    if (!dpl) {   // FP64 sums of the log-normal derivatives
        const double pb = (1.0f - fb) * (bin.own ? -S.px[PX_NGBAR][pair_at<PG>(min(tid, SLOT_W - 1))] : 0.0f);
        const double v[4] = {pb * (double)d1, pb * (double)d2, (double)d1, (double)d2};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double s = wave_sum(v[j]);
            if (lane == 0) S.d[w][j] = s;
        }
    }
    __syncthreads();
    if (w != 0) return;
    const float v = pair_sums<PG>(S, lane, i0, i_end);
    auto sum = [&](int s) { return lane_value(v, PG * s); };
    const float cbar = sum(PS_CBAR);
    if (dpl) {
#pragma unroll
        for (int j = 0; j < 3; ++j) gp = (lane == 1 + j) ? (sum(PS_A0 + j) - cbar * sum(PS_B0 + j)) * invS : gp;
    } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double a = S.d[0][j] + S.d[1][j], b = S.d[0][j + 2] + S.d[1][j + 2];
            gp = (lane == 1 + j) ? (float)((a - (double)cbar * b) / Sm) : gp;
        }
        gp = (lane == 3) ? 0.0f : gp;
    }
    gp = (lane == 4) ? sum(PS_FBAR) : gp;
    gp = (lane == 5) ? (sum(PS_E1) - sum(PS_E2) * sum(PS_E3)) * invZ : gp;
    gp = (lane == 6) ? sum(PS_MET) : gp;
}

}  // namespace sps
