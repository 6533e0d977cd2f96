// Exact photometry (Sec. 3, Eq. photo_integral_exact) as a dense contraction on MFMA.
//
//   SED[g][l]  = sum_s P_SSP[g][s] L[s][l]                   (galaxies x SSPs) . (SSPs x wavelengths)
//   num[g][b]  = sum_l SED[g][l] F_att(l; g) T_b((1+z_g) l) l q_l
//   N[g][b]    = sum_l T_b((1+z_g) l) q_l / l                 (photon-counting AB normaliser)
//   m[g][b]    = -2.5 log10 K(z_g) - 2.5 log10 M_g - 2.5 log10(num / N)
//
// The GEMM runs on MFMA (FP64 16x16x4, or BF16 16x16x32 accumulated in FP32: SPS_F32 splits
// both operands into three BF16 parts, which hold all 24 bits, and takes six products;
// SPS_BF16X into two, W = W_hi + W_lo, L = L_hi + L_lo, and takes three).  The attenuation, filter and quadrature weights are
// generated in the epilogue and reduced over each wavelength tile (16 wide on the
// FP64 path, 128 on the FP32 / BF16X paths) into per-tile partial sums; small
// kernels finish the sums per galaxy.  The FP32 / BF16X paths skip the wavelength
// tiles outside every band's 8-sigma support for a 128-galaxy row tile.
// Gradient (FP32 / BF16X): dlogL/dnum -> Rbar[g][l] -> second GEMM
// Wbar = Rbar . L^T -> dP_age, dP_Z -> the weights adjoint shared with the
// approximate path; dust derivatives come from extra epilogue partials.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "sps_pair.h"

namespace sps {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int NSSP = NZ * NA;
constexpr int EPI_PHOT = 0, EPI_PHOT_DUST = 1, EPI_STORE = 2;

__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }   // nearest even
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// FP32 as three BF16 values hi + mid + lo: exact (8 + 8 + 8 bits) down to 2^-110, below which the last runs out of
// range (the weights' parts that small do not reach FP32 sums, the table is scaled, Rbar carries l q); an
// infinity or NaN is carried by hi alone
__device__ inline void split3(float v, uint16_t &h, uint16_t &m, uint16_t &l) {
    h = f2bf(v);
    const bool fin = (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u;
    const float r = fin ? v - bf2f(h) : 0.0f;
    m = f2bf(r);
    l = f2bf(r - bf2f(m));
}


constexpr double GAUSS_K2 = 0.84932180028801904272;   // sqrt(log2(e) / 2): exp(-x^2 / 2) = exp2(-(K x)^2)
constexpr float LOG2E_F = 1.4426950408889634f;

struct FiltConst {
    double fc[NB_MAX], inv_fs[NB_MAX];   // band centres and 1 / widths (FP64, as in the forward epilogue)
    double lo8[NB_MAX], hi8[NB_MAX];     // c - 8 sigma, c + 8 sigma: the support the kernels keep
    double gk[NB_MAX];                   // sqrt(log2(e) / 2) / sigma
};
inline FiltConst filt_const(const double *fc, const double *fs) {
    FiltConst f;
    for (int b = 0; b < NB_MAX; ++b) {
        f.fc[b] = fc[b];
        f.inv_fs[b] = fs[b] > 0.0 ? 1.0 / fs[b] : 0.0;
        f.gk[b] = f.inv_fs[b] * GAUSS_K2;
        f.lo8[b] = fc[b] - 8.0 * fs[b];
        f.hi8[b] = fc[b] + 8.0 * fs[b];
    }
    return f;
}

constexpr int round_up(int x, int m) { return (x + m - 1) / m * m; }
static_assert(S_PAD % 128 == 0 && S_PAD >= NSSP, "SSP padding");

// ------------------------------------------------------------------ FP64 GEMM + photometry
// SED[g][l] = sum_s W[g][s] L[s][l] on v_mfma_f64_16x16x4, then the band partials of its wavelengths.
// A small batch is the rule (the parity batch is 64 galaxies), and a chain of loads, not the 4 us of
// products or bytes, is its time: a block takes D_ROWS galaxies x D_LAM wavelengths, so that 64
// galaxies x 2000 wavelengths fill the chip, its waves split the SSP axis, each reads its operands
// straight into the fragments with the next batch of loads in flight, and the waves' sums meet in LDS,
// where a thread owns one (galaxy, wavelength) for the transmissions.  (64 x 64 tiles with the SSP axis cut
// over 15 blocks repeated those exponentials 15 times: 60 us of 82 per call at 64 x 2000, 6 bands; these take 19.)
// Large batches take several wavelength tiles per block, which bounds the partials.
constexpr int D_ROWS = 32, D_LAM = 16, D_WAVES = 8, D_T = D_WAVES * WAVE;
constexpr int D_K = S_PAD / D_WAVES, D_G = D_K / 8, D_BATCH = 3;   // SSPs, groups of 8, groups per load batch
static_assert(S_PAD % (8 * D_WAVES) == 0 && D_G % D_BATCH == 0 && D_ROWS * D_LAM == D_T, "FP64 tile");
// wavelength tiles per block, and whether it takes them two at a time, each weight fragment then feeding
// two products (a CU holds one block at a time: from a block per CU on, fewer loads count for more than more
// blocks).  us per call at 2000 wavelengths, 6 bands, one at a time / two: 64 galaxies 29.9 / 33.4, 65
// 39.8 / 33.3, 500 136 / 94, 4096 998 / 605 (500 and 4096 galaxies on the tiles above: 192, 883).
constexpr int D_WIDE = 256;
static int f64_tiles(int n, int n_wave, bool *wide) {
    const int blocks = (n + D_ROWS - 1) / D_ROWS * ((n_wave + D_LAM - 1) / D_LAM);
    *wide = blocks > D_WIDE;
    return *wide ? std::min(4, std::max(2, blocks / 2048)) & ~1 : 1;
}
static int f64_parts(int n, int n_wave) {
    bool wide;
    const int t = f64_tiles(n, n_wave, &wide) * D_LAM;
    return (n_wave + t - 1) / t;
}
struct DArgs {
    int n, n_wave, n_band, tiles;   // tiles: wavelength tiles per block, a multiple of NT
    const double *w, *lum;          // [n][S_PAD], [NSSP][n_wave]
    const double *params, *z, *wave, *trap;
    FiltConst fl;
    double *part;                   // [blockIdx.x][n][2 n_band]: numerators, normalisers
};

template <int NT>
__global__ void __launch_bounds__(D_T, 2) k_exact_phot64(DArgs a) {
    __shared__ double red[NT][D_WAVES][D_ROWS * D_LAM];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), m0 = blockIdx.y * D_ROWS;
    // SSPs k0 + 8 t + 2 lk and + 1 of group t feed the k slots lk of two products, from A and B alike
    const int k0 = w * D_K + 2 * lk;
    const double *ap[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) ap[t] = a.w + (size_t)min(m0 + 16 * t + li, a.n - 1) * S_PAD + k0;
    const int row = m0 + (tid >> 4), g = min(row, a.n - 1);
    const double tauv = a.params[(size_t)7 * a.n + g], delta = a.params[(size_t)8 * a.n + g];
    const double ffl = a.params[(size_t)9 * a.n + g], opz = 1.0 + a.z[g];
    double num[NB_MAX], nrm[NB_MAX];
#pragma unroll
    for (int b = 0; b < NB_MAX; ++b) num[b] = nrm[b] = 0.0;
    const int l_end = min(a.n_wave, (int)(blockIdx.x + 1) * a.tiles * D_LAM);
    for (int l0 = blockIdx.x * a.tiles * D_LAM; l0 < l_end; l0 += NT * D_LAM) {
        const double *bp[NT];
        d4v acc[2][NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            bp[j] = a.lum + min(l0 + j * D_LAM + li, a.n_wave - 1);
            acc[0][j] = acc[1][j] = d4v{0, 0, 0, 0};
        }
        double av[2][D_BATCH][2][2], bv[2][D_BATCH][2][NT];
        auto load = [&](int q, int t0) {
#pragma unroll
            for (int u = 0; u < D_BATCH; ++u)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int ks = k0 + 8 * (t0 + u) + e;
#pragma unroll
                    for (int t = 0; t < 2; ++t) av[q][u][t][e] = ap[t][8 * (t0 + u) + e];
                    // the padding SSPs have weight 0
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        const double v = bp[j][(size_t)min(ks, NSSP - 1) * a.n_wave];
                        bv[q][u][e][j] = ks < NSSP ? v : 0.0;
                    }
                }
        };
        load(0, 0);
#pragma unroll
        for (int t0 = 0, q = 0; t0 < D_G; t0 += D_BATCH, q ^= 1) {
            if (t0 + D_BATCH < D_G) load(q ^ 1, t0 + D_BATCH);
#pragma unroll
            for (int u = 0; u < D_BATCH; ++u)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            acc[t][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q][u][t][e], bv[q][u][e][j], acc[t][j], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[j][w][(16 * t + 4 * r + lk) * D_LAM + li] = acc[t][j][r];
        __syncthreads();
#pragma unroll 1
        for (int j = 0; j < NT; ++j) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < D_WAVES; ++i) s += red[j][i][tid];
            const int l = l0 + j * D_LAM + (tid & (D_LAM - 1));
            if (l < a.n_wave) {
                const double lam = a.wave[l], q = a.trap[l];
                const double xd = exp(delta * log(lam * (1.0 / 5500.0))), F = ffl + (1.0 - ffl) * exp(-tauv * xd);
                const double wn = s * F * (lam * q), wq = q / lam;
#pragma unroll
                for (int b = 0; b < NB_MAX; ++b) {
                    if (b >= a.n_band) break;
                    const double x = (opz * lam - a.fl.fc[b]) * a.fl.inv_fs[b], y = -0.5 * x * x;
                    if (y > -746.0) {   // below, exp(y) = 0
                        const double tb = exp(y);
                        num[b] += tb * wn;
                        nrm[b] += tb * wq;
                    }
                }
            }
        }
        __syncthreads();   // the next tiles' sums take the slots
    }
    auto over_lambda = [](double v) {   // over the 16 lanes of a galaxy
        v = dpp_add<0x128>(v);
        v = dpp_add<0x124>(v);
        v = dpp_add<0x122>(v);
        return dpp_add<0x121>(v);
    };
    double *out = a.part + ((size_t)blockIdx.x * a.n + g) * 2 * a.n_band;
#pragma unroll
    for (int b = 0; b < NB_MAX; ++b) {
        if (b >= a.n_band) break;
        const double sn = over_lambda(num[b]), sw = over_lambda(nrm[b]);
        if ((tid & (D_LAM - 1)) == 0 && row < a.n) {
            out[b] = sn;
            out[a.n_band + b] = sw;
        }
    }
}

// ------------------------------------------------------------------ FP32 / BF16-split GEMM (gfx950)
// C = A . B^T with A [M][K] and B [N][K], both k-contiguous (row strides lda, ldb), K a
// multiple of 32, N a multiple of 128, A allocated to a multiple of 128 rows.  Block tile
// 128 x 128, 256 threads as 2 x 2 waves of 64 x 64 (4 x 4 MFMA tiles of 16 x 16); k-tiles
// of 32 staged through LDS (the next tile's global loads are in flight while the current tile's
// products issue).  Both precisions run on v_mfma_f32_16x16x32_bf16, lane l supplying k =
// 8 (l / 16) .. + 7, with FP32 accumulation, the operands split into XP BF16 parts that lie
// side by side per 32-element k chunk (bfx_at, bf3_at), so a k-tile of a row is XP 64-byte runs:
//   FP32:  hi + mid + lo, which hold all 24 bits (of values down to 2^-110, see split3 and
//          sps_ctx::lum32_exp); six products lo.hi + hi.lo + mid.mid + mid.hi +
//          hi.mid + hi.hi per tile pair (the three dropped ones are below 2^-26 of the product).
//          v_mfma_f32_16x16x4f32 takes 32 cycles for 4 k, these six 96 for 32: the GEMMs at 4096 x
//          5000 took 378 (forward) and 373 us (gradient) on the former.
//   BF16X: hi + lo; three products lo.hi + hi.lo + hi.hi.
// Blocks are mapped XCD-aware: consecutive dispatch slots go round-robin over the 8 XCDs, so
// slot b is remapped to tile (b % 8) * T / 8 + b / 8 and each XCD works through one
// contiguous run of tiles (tile_order for the built-in choice).
constexpr int XBM = 128, XBN = 128, XBK = 32;
template <int P> constexpr int x_parts() { return P == SPS_F32 ? 3 : 2; }
constexpr int XSUB = XBM * 64;                                                  // bytes of one part of an operand tile
template <int P> constexpr int x_stage() { return 2 * x_parts<P>() * XSUB; }     // 49,152 or 32,768 bytes
// K ranges of the gradient GEMM: its n/128 x 9 output tiles are split so that about XSPLIT_BLOCKS blocks
// run (three fit on a CU), each taking an equal part of its row tile's window
constexpr int XSPLIT_MAX = 8, XSPLIT_BLOCKS = 640;
constexpr int XBAND = 8;                                     // row tiles per band (tile order 3)

// a row tile's window (k_xwindows) packs the bands that the forward epilogue and Rbar must not skip over its first k-tile
__device__ inline int win_z(int4 w) { return w.z & 0xffffff; }
__device__ inline unsigned win_keep(int4 w) { return (unsigned)w.z >> 24; }

struct XArgs {
    int M, N, K;
    const void *A;             // BF16 parts interleaved, [M][3 lda] (bf3_at) or [M][2 lda] (bfx_at)
    int lda;
    const void *B;             // likewise [N][ldb]
    int ldb;
    int n_mt, n_nt;
    int k_splits;              // EPI_STORE: K is split into this many ranges, one partial C each
    size_t c_split;            // floats between the partial C of consecutive K ranges
    float *C;                  // EPI_STORE: transposed, [n_store][ldc] (ldc >= 128-padded M)
    int ldc, n_store;
    const float *dust, *z;     // photometry epilogue: tau_V, delta, F_floor [3][M] and z
    const double *wave;
    const float *wc;           // [N][4]: ln(l / 5500), l q, q / l, l
    int n_wave, n_band;
    double fc[NB_MAX], inv_fs[NB_MAX];
    float *part;               // [n_nt][npart][M] (quantity-major: the finish reads it coalesced)
    int npart;
    // per 128-galaxy row tile: the wavelength tiles (x, y: 128-wide, [x, y)) and k-tiles (win_z, w:
    // 32-wide) inside some band's 8-sigma filter support for some galaxy of the tile
    const int4 *win;
    // rows in z order: the forward epilogue skips, per wave, the bands farther than 8 sigma
    // from all of its wavelengths (a wave's galaxies then share nearly one redshift), but for the row tile's
    // win_keep
    int band_skip;
    // tile order: 1 M fastest, 2 N fastest, 3 bands of XBAND row tiles; xcd: one contiguous run of
    // tiles per XCD (1) or dispatch order (0).  Every order computes the same tiles the same way.
    int order, xcd;
};

// LDS stages, filled by direct global-to-LDS loads (no staging registers): one stage with three blocks
// per CU, whose products cover each other's loads; or for BF16X (RING = true, a launch choice) a ring
// of two stages with two blocks per CU.  The two BF16X forms multiply the same tiles in the same order
// (the same bits); which is faster depends on the shape (sps_autotune_exact): value+gradient, us, one stage /
// ring, 2000 wavelengths, 200 galaxies 105 / 99, 1000 121 / 117, 4096 171 / 175, 65,536 1224 / 1294; 5000
// wavelengths, 1000 141 / 134, 4096 257 / 278.
constexpr int RSTAGES = 2;
constexpr int RSTAGE = 2 * XBM * 128;   // A then B rows, 128 bytes (the k-tile's 32 hi + 32 lo) each
// the single stage is at least the epilogue's half SED tile with the wavelength constants
constexpr int XSED = XBM * (XBN / 2 + 1) * 4 + XBN * 16;
template <int P, bool RING> constexpr int x_smem() {
    return RING ? RSTAGES * RSTAGE : (x_stage<P>() > XSED ? x_stage<P>() : XSED);
}
template <int P, bool RING> constexpr int x_blocks() { return RING ? 2 : 3; }

#define SPS_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
// s_waitcnt immediate for "at most n vector-memory operations outstanding" (other counters free)
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// Ring stage of a k-tile: 32 loads of 1 KB, 8 per wave.  Waves 0 and 1 fill the A rows
// 0..63 and 64..127, waves 2 and 3 the B rows; load j of a wave covers 8 of its rows, its lane L
// writing the stage's bytes 1024 q + 16 L (q = 8 wave + j), i.e. slot L % 8 of stage row
// 8 q + L / 8, with the row's 16-byte chunk (L % 8) ^ (L / 8) (chunks 0..3 hi, 4..7 lo;
// (L / 8) = the stage row mod 8): the XOR swizzle that keeps the fragment reads free of bank
// conflicts.  The lane's source address is fixed but for the k offset, and which operand a wave
// loads is wave-uniform.
struct XRing {
    const uint16_t *src;   // this lane's chunk of its first row, k-tile 0 (uint16 units)
    size_t jstep;          // from one of the wave's loads to the next: 8 rows
};
__device__ inline XRing x_ring_setup(const XArgs &a, int tile_m, int tile_n, int wave, int lane) {
    const int w = __builtin_amdgcn_readfirstlane(wave);
    const bool isA = w < 2;
    const uint16_t *base = (const uint16_t *)(isA ? a.A : a.B);
    const int ld = isA ? a.lda : a.ldb, tile0 = isA ? tile_m : tile_n;
    const int row = (w & 1) * 64 + (lane >> 3), c = (lane & 7) ^ (lane >> 3);
    return XRing{base + (size_t)(tile0 + row) * 2 * ld + 8 * c, (size_t)16 * ld};
}
__device__ inline void x_ring_issue(const XRing &r, char *stage, int k0, int wave) {
    const int w = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        __builtin_amdgcn_global_load_lds((const void *)(r.src + j * r.jstep + 2 * k0),
                                         SPS_LDS_PTR(stage + 1024 * (8 * w + j)), 16, 0, 0);
}

// Single stage: part p of operand o (A, B) is 128 rows of 64 bytes at (o XP + p) XSUB.  A load covers
// 16 rows, lane L writing slot L % 4 of row L / 4 with the row's 16-byte chunk (L % 4) ^ x_swz(L / 16).
// A fragment read (16 bytes per lane, row lane % 16, chunk lane / 16) is served 16 lanes at a time,
// lanes 0-3, 12-15, 20-23, 24-27 together and 4-11, 16-19, 28-31: x_swz of the row's bits 2..3 puts each
// of those sets on all banks once (the plain XOR with those bits doubled the reads' cycles).  Wave w
// loads rows 32 w .. 32 w + 31 of every part.
__device__ inline int x_swz(int q) { return (((q ^ (q >> 1)) & 1) << 1) | (q >> 1); }   // 0, 2, 3, 1
// (base: wave-uniform, the wave's first row of the operand; off: the lane's bytes from there.)
template <int P>
__device__ inline void x_issue(const char *base, uint32_t off, int ld, int k0, char *stage) {
    constexpr int PARTS = x_parts<P>();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
            __builtin_amdgcn_global_load_lds(
                (const void *)(base + ((size_t)h * 16 * PARTS * ld + PARTS * k0 + 32 * p) * 2 + off),
                SPS_LDS_PTR(stage + p * XSUB + 1024 * h), 16, 0, 0);
}

template <int P, int EPI, bool RING>
__global__ void __launch_bounds__(256, (x_blocks<P, RING>())) k_xgemm(XArgs a) {
    static_assert(!RING || P == SPS_BF16X, "the ring form is the BF16X kernel's");
    __shared__ __attribute__((aligned(16))) char smem[x_smem<P, RING>()];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 15, lk = lane >> 4;
    // XCD-aware tile order; with a split K the slot also names the K range
    const int T = a.n_mt * a.n_nt, nsp = (EPI == EPI_STORE) ? a.k_splits : 1, total = T * nsp, b = blockIdx.x;
    int t = b;
    if (a.xcd && total % 8 == 0) t = (b % 8) * (total / 8) + b / 8;
    // the K range: between M and N, as the windows clip it (every XCD's run of tiles
    // then holds all ranges, so the mostly skipped last ones do not gather on a few XCDs, and
    // consecutive tiles still share their B rows and K range in L2)
    [[maybe_unused]] int sp = 0;
    if constexpr (EPI == EPI_STORE) {
        const int m_ = t % a.n_mt, rest = t / a.n_mt;
        sp = rest % nsp;
        t = (rest / nsp) * a.n_mt + m_;
    }
    const bool nfast = a.order == 2;
    int tile_m, tile_n;
    if (a.order == 3) {
        // bands of XBAND row tiles: M fastest inside a band, which sweeps every column tile, so
        // the blocks in flight on an XCD share a few A and B panels
        const int band = t / (XBAND * a.n_nt), w = t - band * XBAND * a.n_nt;
        const int bm = min(XBAND, a.n_mt - band * XBAND);
        tile_m = (band * XBAND + w % bm) * XBM;
        tile_n = (w / bm) * XBN;
    } else {
        tile_m = (nfast ? t / a.n_nt : t % a.n_mt) * XBM;
        tile_n = (nfast ? t % a.n_nt : t / a.n_mt) * XBN;
    }
    int klen = a.K, kbeg = 0;
    [[maybe_unused]] unsigned keep = 0;
    {
        // wavelengths outside every band's support for all of this tile's galaxies: the
        // forward tile's band sums are below exp(-32) of the band's: the tile is not computed
        // and the tile sum (k_exact_finish) skips it; the gradient GEMM's Rbar is exactly zero
        // there, so its K range is the window's
        const int4 w = a.win[tile_m / XBM];
        if constexpr (EPI == EPI_STORE) {
            const int nk_w = max(w.w - win_z(w), 0), k0 = win_z(w) + nk_w * sp / nsp, k1 = win_z(w) + nk_w * (sp + 1) / nsp;
            kbeg = k0 * XBK;
            klen = (k1 - k0) * XBK;
        } else {
            if (tile_n / XBN < w.x || tile_n / XBN >= w.y) return;   // k_exact_finish reads only the tiles inside
            keep = win_keep(w);
        }
    }

    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    const int nk = klen / XBK;
    if constexpr (RING) {
        // prologue: k-tile 0 in flight
        static_assert(RSTAGES == 2, "the next k-tile loads while this one's products issue");
        const XRing ring = x_ring_setup(a, tile_m, tile_n, wave, lane);
        if (nk > 0) x_ring_issue(ring, smem, kbeg, wave);
        for (int kt = 0; kt < nk; ++kt) {
            // this wave's loads of k-tile kt are done; the barrier then covers every wave's loads, and
            // every wave's reads of the stage that k-tile kt + 1 refills (k-tile kt - 1's)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + 1 < nk) x_ring_issue(ring, smem + ((kt + 1) % RSTAGES) * RSTAGE, kbeg + (kt + 1) * XBK, wave);
            const char *As = smem + (kt % RSTAGES) * RSTAGE, *Bs = As + XBM * 128;
            b8v ah[4], al[4], bh[4], bl[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ra = wm * 64 + i * 16 + li, rb = wn * 64 + i * 16 + li;
                ah[i] = *(const b8v *)(As + ra * 128 + ((lk ^ (ra & 7)) << 4));
                al[i] = *(const b8v *)(As + ra * 128 + (((lk + 4) ^ (ra & 7)) << 4));
                bh[i] = *(const b8v *)(Bs + rb * 128 + ((lk ^ (rb & 7)) << 4));
                bl[i] = *(const b8v *)(Bs + rb * 128 + (((lk + 4) ^ (rb & 7)) << 4));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();   // every wave is done with the ring before the epilogue reuses it
    } else {
    constexpr int PARTS = x_parts<P>();
    const int ws = __builtin_amdgcn_readfirstlane(wave);
    const int lch = 16 * ((lane & 3) ^ x_swz(lane >> 4));
    const char *pa = (const char *)a.A + (size_t)(tile_m + 32 * ws) * PARTS * a.lda * 2;
    const char *pb = (const char *)a.B + (size_t)(tile_n + 32 * ws) * PARTS * a.ldb * 2;
    const uint32_t oa = (uint32_t)(lane >> 2) * PARTS * a.lda * 2 + lch, ob = (uint32_t)(lane >> 2) * PARTS * a.ldb * 2 + lch;
    char *sa = smem + 2048 * ws, *sb = sa + PARTS * XSUB;
    const int frag = li * 64 + ((lk ^ x_swz(li >> 2)) << 4);
    if (nk > 0) {
        x_issue<P>(pa, oa, a.lda, kbeg, sa);
        x_issue<P>(pb, ob, a.ldb, kbeg, sb);
    }
    for (int kt = 0; kt < nk; ++kt) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __syncthreads();
        // the k-tile's fragments into registers, then the stage is free for the next k-tile, whose loads
        // run under this one's products
        const char *Ar = smem + opaque(frag) + 4096 * (ws >> 1), *Br = smem + opaque(frag) + PARTS * XSUB + 4096 * (ws & 1);
        auto next = [&]() {
            __syncthreads();
            if (kt + 1 < nk) {
                x_issue<P>(pa, oa, a.lda, kbeg + (kt + 1) * XBK, sa);
                x_issue<P>(pb, ob, a.ldb, kbeg + (kt + 1) * XBK, sb);
            }
        };
        b8v af[PARTS][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int p = 0; p < PARTS; ++p) af[p][i] = *(const b8v *)(Ar + i * 1024 + p * XSUB);
        // FP32 takes B's fragments in two halves (all of them would not fit beside A's in 168 registers)
        constexpr int JH = (P == SPS_F32) ? 2 : 4;
        constexpr int NPROD = (P == SPS_F32) ? 6 : 3;   // small products first
        constexpr int PA[6] = {PARTS - 1, 0, P == SPS_F32 ? 1 : 0, 1, 0, 0}, PB[6] = {0, PARTS - 1, P == SPS_F32 ? 1 : 0, 0, 1, 0};
#pragma unroll
        for (int j0 = 0; j0 < 4; j0 += JH) {
            b8v bf[PARTS][JH];
#pragma unroll
            for (int j = 0; j < JH; ++j)
#pragma unroll
                for (int p = 0; p < PARTS; ++p) bf[p][j] = *(const b8v *)(Br + (j0 + j) * 1024 + p * XSUB);
            if (j0 + JH == 4) next();
#pragma unroll
            for (int t = 0; t < NPROD; ++t)
#pragma unroll
                for (int j = 0; j < JH; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[PA[t]][i], bf[PB[t]][j], acc[i][j0 + j], 0, 0, 0);
        }
    }
    __syncthreads();   // every wave is done before the epilogue reuses the stage
    }

    if constexpr (EPI == EPI_STORE) {
        // C stored transposed, C[n][m] with row stride ldc >= the 128-padded M: a lane's four
        // accumulator rows are consecutive m, one 16-byte store
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = tile_m + wm * 64 + i * 16 + 4 * lk;
                const int n = tile_n + wn * 64 + j * 16 + li;
                if (n < a.n_store) *(v4f *)(a.C + sp * a.c_split + (size_t)n * a.ldc + m) = acc[i][j];
            }
        return;
    } else {
        // SED tile [128 galaxies][128 wavelengths] -> LDS in two passes of PW columns (row
        // stride PW + 1; one stage holds half the tile), two threads per galaxy reducing PW / 2
        // wavelengths each per pass into the band sums
        constexpr int NPASS = 2, PW = XBN / NPASS;
        float(*sed)[PW + 1] = reinterpret_cast<float(*)[PW + 1]>(smem);
        // the tile's wavelength constants (ln x, l q, q / l, l) in LDS after the SED columns:
        // read once per tile instead of one dependent global load per column and thread
        v4f *swc = reinterpret_cast<v4f *>(smem + XBM * (PW + 1) * 4);
        static_assert(XBM * (PW + 1) * 4 + XBN * 16 <= x_smem<P, RING>(), "SED columns fit the staging buffers");
        static_assert((XBM * (PW + 1) * 4) % 16 == 0, "aligned wavelength constants");
        const int row = tid >> 1, half = tid & 1, g = tile_m + row;
        constexpr int NPB = (EPI == EPI_PHOT_DUST) ? 5 : 2;   // num, N [, dnum/dtauV, dnum/ddelta, dnum/dFfloor]
        float accp[NB_MAX][NPB];
#pragma unroll
        for (int bb = 0; bb < NB_MAX; ++bb)
#pragma unroll
            for (int q = 0; q < NPB; ++q) accp[bb][q] = 0.0f;
        const int gg = g < a.M ? g : a.M - 1;
        const float tauv = a.dust[gg], delta = a.dust[(size_t)a.M + gg], ffl = a.dust[(size_t)2 * a.M + gg];
        const double opz = 1.0 + (double)a.z[gg];
        // the galaxy's filter offsets as one FP32 FMA per band and wavelength: t = l ta_b + tc_b
        // = x_b sqrt(log2(e) / 2) with x_b = ((1+z) l - c_b) / s_b, so T_b = exp2(-t^2); the
        // constants are formed in FP64 (|t| errs by ~1e-6 near a band, 3e-6 of T_b); the dust
        // exponents carry log2(e) too
        float ta[NB_MAX], tc[NB_MAX];
#pragma unroll
        for (int bb = 0; bb < NB_MAX; ++bb) {
            ta[bb] = (float)(opz * a.inv_fs[bb] * GAUSS_K2);
            tc[bb] = (float)(-a.fc[bb] * a.inv_fs[bb] * GAUSS_K2);
        }
        const float delta2 = delta * LOG2E_F, tauv2 = -tauv * LOG2E_F;
        // (beyond the grid the constants are zero, and so are the SED columns: those columns
        // add exact zeros)
        if (tid < XBN) swc[tid] = *(const v4f *)(a.wc + 4 * (size_t)(tile_n + tid));
#pragma unroll
        for (int pp = 0; pp < NPASS; ++pp) {
        if (pp > 0) __syncthreads();   // the previous pass's reads are done
        if (wn == pp) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) sed[wm * 64 + i * 16 + 4 * lk + q][j * 16 + li] = acc[i][j][q];
        }
        __syncthreads();
        // bands within 8 sigma of some redshifted wavelength of some thread of the wave: a
        // wave-uniform mask, so a skipped band is a scalar branch (all bands when the rows are
        // in arbitrary z order, where the test would rarely skip and only cost time)
        unsigned act = (1u << a.n_band) - 1u;
        if (a.band_skip) {
            const int l0 = tile_n + pp * PW + half * (PW / 2), l1 = min(l0 + PW / 2 - 1, a.n_wave - 1);
            const double u0 = opz * a.wave[min(l0, a.n_wave - 1)], u1 = opz * a.wave[l1];
            act = keep;
#pragma unroll
            for (int bb = 0; bb < NB_MAX; ++bb) {
                if (bb >= a.n_band) break;
                const double x0 = (u0 - a.fc[bb]) * a.inv_fs[bb], x1 = (u1 - a.fc[bb]) * a.inv_fs[bb];
                if (__ballot(l0 < a.n_wave && x0 < 8.0 && x1 > -8.0) != 0) act |= 1u << bb;
            }
        }
        // four columns at a time: their LDS reads issue together, and each band's sums take the
        // columns in order (the same sums as one column after another)
        for (int c4 = 0; c4 < PW / 2; c4 += 4) {
            v4f w[4];   // ln x, l q, q / l, l
            float xd[4], ee[4], F[4], sw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                w[u] = swc[pp * PW + half * (PW / 2) + c4 + u];
                sw[u] = sed[row][half * (PW / 2) + c4 + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                xd[u] = __builtin_amdgcn_exp2f(delta2 * w[u][0]);
                ee[u] = __builtin_amdgcn_exp2f(tauv2 * xd[u]);
                F[u] = ffl + (1.0f - ffl) * ee[u];
                sw[u] = sw[u] * w[u][1];
            }
#pragma unroll
            for (int bb = 0; bb < NB_MAX; ++bb) {
                if (bb >= a.n_band) break;
                if (!((act >> bb) & 1u)) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float t = fmaf(w[u][3], ta[bb], tc[bb]);
                    const float tb = __builtin_amdgcn_exp2f(-t * t);
                    const float stw = sw[u] * tb;
                    accp[bb][0] = fmaf(stw, F[u], accp[bb][0]);
                    accp[bb][1] = fmaf(tb, w[u][2], accp[bb][1]);
                    if constexpr (EPI == EPI_PHOT_DUST) {
                        const float dtv = -(1.0f - ffl) * xd[u] * ee[u];
                        accp[bb][2] = fmaf(stw, dtv, accp[bb][2]);
                        accp[bb][3] = fmaf(stw * dtv, tauv * w[u][0], accp[bb][3]);
                        accp[bb][4] = fmaf(stw, 1.0f - ee[u], accp[bb][4]);
                    }
                }
            }
        }
        }
#pragma unroll
        for (int bb = 0; bb < NB_MAX; ++bb)
#pragma unroll
            for (int q = 0; q < NPB; ++q) accp[bb][q] += __shfl_xor(accp[bb][q], 1, 64);
        if (half == 0 && g < a.M) {
            float *out = a.part + (size_t)(tile_n / XBN) * a.npart * a.M + g;
#pragma unroll
            for (int bb = 0; bb < NB_MAX; ++bb) {
                if (bb >= a.n_band) break;
#pragma unroll
                for (int q = 0; q < NPB; ++q) out[(size_t)(q * a.n_band + bb) * a.M] = accp[bb][q];
            }
        }
    }
}

// ------------------------------------------------------------------ FP64 weights rows P_SSP[g][s]
// FP64 weights from FP64 bin edges: closed-form log-normal or 8-point Gauss-Legendre DPL
// panels, closed-form triweight and normal CDFs (the FP64 parity path).  Its time is one bin's chain
// of FP64 functions, so a galaxy takes three waves: thread i < NA age bin i, the third wave the metallicity
// bins (one wave with two bins per lane took 12.5 us at 64 galaxies, these 7.1).
constexpr int W64_T = 192;
__global__ void __launch_bounds__(W64_T) k_exact_weights64(DevConsts k, int n, int sfh, const double *params_v,
                                                           const double *z_v, const double *edges, double *w_out) {
    static_assert(NA <= 2 * WAVE && NZ <= WAVE, "an age bin per thread of two waves, a metallicity bin per lane");
    __shared__ double spz[NZ], sum[2][2];
    const int tid = threadIdx.x, g = blockIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double *prm = params_v;
    const double *age_lo = edges, *age_hi = edges + NA, *lage_lo = edges + 2 * NA, *lage_hi = edges + 3 * NA;
    const double *met_lo = edges + 4 * NA, *met_hi = edges + 4 * NA + NZ;
    double th[NP], m = 0.0, bm = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p) th[p] = prm[(size_t)p * n + g];
    double *w = w_out + (size_t)g * S_PAD;
    if (wv < 2) {
        const double t_obs = age_universe_gyr(k, z_v[g]);
        if (tid < NA) {
            double a0, a1;
            if (sfh == SPS_SFH_LOGNORMAL) logn_bin_e<false>(age_lo[tid], age_hi[tid], t_obs, th[1], th[2], m, a0, a1);
            else m = dpl_bin_f64(k, age_lo[tid], age_hi[tid], t_obs, th[1], th[2], th[3]);
            const double l_obs = log10(t_obs * 1e9), s3 = 3.0 * k.burst_sig_d, lo = lage_lo[tid];
            if (lo < l_obs) {
                const double hi = fmin(lage_hi[tid], l_obs);
                auto cdf = [](double u) {
                    u = fmin(fmax(u, -1.0), 1.0);
                    const double u2 = u * u;
                    return 0.5 + 1.09375 * u * (1.0 - u2 + u2 * u2 * (0.6 - u2 / 7.0));
                };
                bm = cdf((hi - th[5]) / s3) - cdf((lo - th[5]) / s3);
            }
        }
        const double S = wave_sum(m), Zb = wave_sum(bm);
        if ((tid & 63) == 0) {
            sum[wv][0] = S;
            sum[wv][1] = Zb;
        }
    } else {
        const int j = tid - 2 * WAVE;
        if (j < NZ) {
            const double xl = (met_lo[j] - th[6]) / k.sigma_logz_d, xh = (met_hi[j] - th[6]) / k.sigma_logz_d;
            spz[j] = (xl > 0.0) ? Phic_d(xl) - Phic_d(xh) : Phi_d(xh) - Phi_d(xl);
        }
        for (int s = NSSP + j; s < S_PAD; s += WAVE) w[s] = 0.0;
    }
    __syncthreads();
    if (tid >= NA) return;
    const double S = sum[0][0] + sum[1][0], Zb = sum[0][1] + sum[1][1];
    const double pa = (1.0 - th[4]) * m / S + (Zb > 0.0 ? th[4] * bm / Zb : 0.0);
    for (int j = 0; j < NZ; ++j) w[j * NA + tid] = spz[j] * pa;
}

// ------------------------------------------------------------------ FP32 / BF16X weights, large batches
// From GPL_BIG_N galaxies on, GPL adjacent lanes share a galaxy (and its LDS column) and split its age
// bins; below, a wave takes each galaxy (k_exact_weights).  Four lanes: the chain of a lane's bins is the
// time of the weights and of their adjoint, us with two / four lanes: 16,384 galaxies 29 + 38 / 23 + 30,
// 20,011 32 + 43 / 25 + 33, 65,536 43 + 65 / 43 + 53.
// Per-galaxy results, SoA [slot][n]: slots 0..93 P_age, 96..107 P_Z, 108/109 the FP64 total
// smooth mass (low/high words), 110 the burst normaliser, 111 log10 t_obs, 112 the first
// burst bin (int bits).
constexpr int PW_SLOTS = 128, PW_PZ = 96, PW_S = 108, PW_ZB = 110, PW_LOBS = 111, PW_I0 = 112;
constexpr int GPL_BIG_N = 16384, GPL = 4;

__global__ void __launch_bounds__(64) k_exact_pw(DevConsts k, int n, int sfh, const float *params, const float *z,
                                                 float *pw) {
    __shared__ float lds[LDS_SLOTS * (64 / GPL)];
    __shared__ float ledge[NA + 1];
    stage_log_age_edges(k, ledge);
    const int lane = threadIdx.x, slot = lane / GPL, q = lane % GPL;
    const int g = blockIdx.x * (64 / GPL) + slot, gg = g < n ? g : n - 1;
    LdsColT<64 / GPL> col{lds + slot};
    float th[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) th[p] = params[(size_t)p * n + gg];
    const double t_obs = age_universe_gyr(k, (double)z[gg]);
    float pz[NZ];
    WeightsState ws;
    forward_weights<GPL>(k, ledge, sfh, th, t_obs, col, pz, ws, q);
    if (g >= n) return;
    for (int i = q; i < NA; i += GPL) pw[(size_t)i * n + g] = col[i];
    if (q == 0) {
#pragma unroll
        for (int j = 0; j < NZ; ++j) pw[(size_t)(PW_PZ + j) * n + g] = pz[j];
        pw[(size_t)PW_S * n + g] = __int_as_float(__double2loint(ws.S));
        pw[(size_t)(PW_S + 1) * n + g] = __int_as_float(__double2hiint(ws.S));
        pw[(size_t)PW_ZB * n + g] = ws.Zb;
        pw[(size_t)PW_LOBS * n + g] = ws.l_obs;
        pw[(size_t)PW_I0 * n + g] = __int_as_float(ws.i0);
    }
}

// weights rows W[g][s] = P_Z(j) P_age(i), s = j NA + i, zero for s >= NSSP.  A block takes
// XG galaxies: their P_age and P_Z columns (galaxy-contiguous in pw) are staged in LDS, one row
// of factors per galaxy, then the rows are written with consecutive threads on consecutive
// pairs of s (whole lines; a pair is one 4-byte store per BF16 part, and never
// straddles a metallicity, the padding or a 32-element chunk, NA, NSSP and S_PAD being even).
// The lanes of a wave read consecutive pairs of one galaxy's row, and the staging writes of
// consecutive galaxies fall in different banks (row length 106 words).
constexpr int XG = 16, XROWF = NA + NZ;
static_assert(NA % 2 == 0 && NSSP % 2 == 0 && S_PAD % 2 == 0 && XROWF % 2 == 0, "pairs of SSPs");
// elements sidx, sidx + 1 of row g from its factors (P_age, then P_Z)
template <int P>
__device__ inline void expand_pair(const float *f, int sidx, size_t g, void *w) {
    float v0 = 0.0f, v1 = 0.0f;
    if (sidx < NSSP) {
        const int j = sidx / NA, i = sidx - j * NA;
        const float pzj = f[NA + j];
        const float2 pa = *(const float2 *)&f[i];
        v0 = pzj * pa.x;
        v1 = pzj * pa.y;
    }
    if constexpr (P == SPS_F32) {
        uint16_t h0, m0, l0, h1, m1, l1;
        split3(v0, h0, m0, l0);
        split3(v1, h1, m1, l1);
        uint16_t *o = (uint16_t *)w + bf3_at(g, S_PAD, sidx);   // even
        *(uint32_t *)o = (uint32_t)h0 | ((uint32_t)h1 << 16);
        *(uint32_t *)(o + 32) = (uint32_t)m0 | ((uint32_t)m1 << 16);
        *(uint32_t *)(o + 64) = (uint32_t)l0 | ((uint32_t)l1 << 16);
    } else {
        const uint16_t h0 = f2bf(v0), h1 = f2bf(v1);
        const uint16_t l0 = f2bf(v0 - bf2f(h0)), l1 = f2bf(v1 - bf2f(h1));
        uint16_t *o = (uint16_t *)w + bfx_at(g, S_PAD, sidx);
        *(uint32_t *)o = (uint32_t)h0 | ((uint32_t)h1 << 16);
        *(uint32_t *)(o + 32) = (uint32_t)l0 | ((uint32_t)l1 << 16);
    }
}

template <int P>
__global__ void __launch_bounds__(256) k_expand(int n, const float *pw, void *w) {
    __shared__ __attribute__((aligned(8))) float sp[XG][XROWF];
    const int g0 = blockIdx.x * XG, tid = threadIdx.x;
    for (int e = tid; e < (NA + NZ) * XG; e += 256) {
        const int r = e / XG, t = e - r * XG, g = min(g0 + t, n - 1);
        sp[t][r] = pw[(size_t)(r < NA ? r : PW_PZ + (r - NA)) * n + g];
    }
    __syncthreads();
    const int ng = min(XG, n - g0);
    constexpr int HP = S_PAD / 2;
    for (int e = tid; e < ng * HP; e += 256) {
        const int t = e / HP;
        expand_pair<P>(sp[t], 2 * (e - t * HP), (size_t)(g0 + t), w);
    }
}

// ------------------------------------------------------------------ finish: magnitudes / likelihood
// FP32 / BF16X: the photometry partials [tile][quantity][rank] summed over the wavelength tiles of the
// row tile's window (the forward GEMM writes none outside it), then magnitudes, or log L (vjp: the
// caller's adjoints obs = dL/dm_b take the place of the residuals), the mass and dust derivatives and
// dlogL/dnum.  Eight lanes per galaxy, a band each; perm: the caller's index of a rank (null: the same).
// sums, with mag: the tile sums [g][5][n_band] of the numerator, the normaliser and the numerator's dust
// derivatives are kept for a later backward, which passes them with vjp in place of the partials; sperm:
// the caller's index of a rank for them.  k.kfac takes in the table's unit (sps_ctx::lum32_exp): only
// the magnitude sees it, dlogL/dnum and the table of the gradient GEMM share it.  A block's 32 galaxies share a row tile.  One thread per galaxy
// and a pass of its own for the tile sums took 28 + 9 us at 4096 galaxies.
template <bool GRAD>
__global__ void __launch_bounds__(256) k_exact_finish(DevConsts k, int n, int n_tiles, const int *perm,
                                                      const float *params, const float *z, const int4 *win,
                                                      const float *part, int npart, float *mag, const float *obs,
                                                      const float *sigma, const uint8_t *mask, float *logl,
                                                      float *grad, float *cnum, int vjp, float *sums,
                                                      const int *sperm) {
    static_assert(NB_MAX == 8, "a lane per band");
    const int r = blockIdx.x * 32 + (threadIdx.x >> 3), b = threadIdx.x & 7, nb = k.n_band;
    const bool valid = r < n, act = b < nb;
    const int rr = min(r, n - 1), g = perm ? perm[rr] : rr, bb = min(b, nb - 1);
    static_assert(XBM % 32 == 0, "a block's galaxies lie in one row tile");
    const int4 w = win[blockIdx.x * 32 / XBM];
    constexpr int NQ = GRAD ? 5 : 2;
    float v[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    const size_t so = (size_t)(sperm ? sperm[rr] : g) * 5 * nb + bb;
    if (GRAD && vjp && sums) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = sums[so + q * nb];
    } else {
        const float *pp = part + (size_t)bb * n + rr;
        const size_t qs = (size_t)nb * n, ts = (size_t)npart * n;
        const int t_end = min(w.y, n_tiles);
#pragma unroll 4
        for (int t = w.x; t < t_end; ++t) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[q] += pp[t * ts + q * qs];
        }
    }
    // the distance integral's nodes split over the eight lanes (mag_offset)
    const double zf = (double)z[rr];
    double chi = 0.0;
    const double ol = 1.0 - k.om, h = 0.5 * zf;
#pragma unroll
    for (int i = 0; i < NGL_DL; i += 8) {
        if (i + b < NGL_DL) {
            const double ep = 1.0 + h + h * k.gl_x[i + b], em = 1.0 + h - h * k.gl_x[i + b];
            chi += k.gl_w[i + b] * (1.0 / sqrt(k.om * ep * ep * ep + ol) + 1.0 / sqrt(k.om * em * em * em + ol));
        }
    }
    chi = group_sum<8>(chi);
    const double dl = (1.0 + zf) * k.dh_cm * h * chi;
    const double m0 = -2.5 * log10((1.0 + zf) * k.kfac) + 5.0 * log10(dl) - 2.5 * (double)params[g];
    const double num = v[0], m = m0 - 2.5 * log10(num / (double)v[1]);
    if (mag) {
        if (valid && act) mag[(size_t)g * nb + b] = (float)m;
        if (GRAD && sums && valid && act)
#pragma unroll
            for (int q = 0; q < NQ; ++q) sums[so + q * nb] = v[q];
        return;
    }
    const uint32_t mk = (vjp || !mask) ? 0xffffffffu : mask[g];
    double ll = 0.0, g0 = 0.0, g7 = 0.0, g8 = 0.0, g9 = 0.0, cb = 0.0;
    if (act && ((mk >> b) & 1u)) {
        double gm;   // d logL / d m_b
        if (vjp) {
            gm = (double)obs[(size_t)g * nb + b];
        } else {
            const double s = sigma[(size_t)g * nb + b], res = (m - (double)obs[(size_t)g * nb + b]) / s;
            ll = -0.5 * res * res - log(s * 2.5066282746310002);
            gm = -res / s;
        }
        g0 = -2.5 * gm;
        cb = gm * (-2.5 / 2.302585092994046) / num;   // d logL / d num_b
        g7 = cb * (double)v[2];
        g8 = cb * (double)v[3];
        g9 = cb * (double)v[4];
    }
    // a kept band (k_xwindows) whose sum is 0, or too small for 1 / sum, has no share
    if (((win_keep(w) >> b) & 1u) && (num == 0.0 || fabs(cb) > 3.4e38)) cb = 0.0;
    if (valid && cnum) cnum[(size_t)r * NB_MAX + b] = (float)cb;
    ll = group_sum<8>(ll);
    if (logl && valid && b == 0) logl[g] = (float)ll;
    if (!GRAD) return;
    g0 = group_sum<8>(g0);
    g7 = group_sum<8>(g7);
    g8 = group_sum<8>(g8);
    g9 = group_sum<8>(g9);
    if (valid && b < 4) grad[(size_t)(b == 0 ? 0 : 6 + b) * n + g] = (float)(b == 0 ? g0 : b == 1 ? g7 : b == 2 ? g8 : g9);
}

// Rbar[g][l] = sum_b (d logL / d num_b) F_att(l) T_b((1+z) l) l q_l  (zero beyond n_wave);
// bands more than 8 sigma from the redshifted wavelength contribute below FP32 resolution, but in a row
// tile with a win_keep, whose magnitudes are made of such terms: there none is left out.  (One limit for
// all bands, and seven waves on a SIMD: with a limit per band and 79 registers the gradient of 20,011 galaxies, 503
// us, took 514.)
// One block takes G consecutive galaxies (rows of one 128-row tile, so one filter-support
// window, all that the gradient GEMM reads) and walks their rows from the window's first k-tile to its
// last, two wavelengths per thread: the galaxies' constants are loaded
// together once, and each batch of wavelength constants serves all of the block's galaxies.
// G = 4 spares those loads, G = 1 keeps more blocks in flight: us with 1 / 4 galaxies, 6 bands, BF16X, 500
// x 2000 5.2 / 9.7, 4096 12.8 / 14.6, 15,900 31.8 / 30.1, 20,011 39.0 / 36.0, 65,536 122 / 99.  Bound by instructions (an
// exponential per band in reach and two for the dust); one wavelength per thread in whole chunks of 256
// around the window, a 2-byte store per part, took 63 us at 20,011 and 195 at 65,536.
constexpr int RBAR_G_BIG = 4, RBAR_BIG_MIN_GAL = 16384;
static_assert(XBM % RBAR_G_BIG == 0, "a block's galaxies share one row tile");
template <int P, int RBAR_G>
__global__ void __launch_bounds__(256, P == SPS_F32 ? 6 : 7) k_exact_rbar(int n, int n_wave, int ld, int nb, FiltConst fl,
                                                    const float *dust, const float *z, const float *wc,
                                                    const float *cnum, const int4 *win, void *rb) {
    const int g0 = blockIdx.x * RBAR_G, tid = threadIdx.x;
    const int ng = min(RBAR_G, n - g0);   // galaxies of this block (>= 1)
    const int4 wn = win[g0 / XBM];
    const int lo = win_z(wn) * XBK, hi = min(ld, wn.w * XBK);
    const float cut = win_keep(wn) ? INFINITY : 8.0f * GAUSS_K2;
    double opz[RBAR_G];
    float cb[RBAR_G][NB_MAX], ffl[RBAR_G], delta2[RBAR_G], tauv2[RBAR_G];
#pragma unroll
    for (int j = 0; j < RBAR_G; ++j) {
        const int g = min(g0 + j, n - 1);
        opz[j] = 1.0 + (double)z[g];
        const float tauv = dust[g], delta = dust[(size_t)n + g];
        ffl[j] = dust[(size_t)2 * n + g];
        delta2[j] = delta * LOG2E_F;
        tauv2[j] = -tauv * LOG2E_F;
#pragma unroll
        for (int b = 0; b < NB_MAX; ++b) cb[j][b] = (b < nb) ? cnum[(size_t)g * NB_MAX + b] : 0.0f;
    }
    float tc[NB_MAX];   // filter offsets as in the forward epilogue
#pragma unroll
    for (int b = 0; b < NB_MAX; ++b) tc[b] = (float)(-fl.fc[b] * fl.gk[b]);
    // bands are tested per pair (a wave's 128 wavelengths lie within a filter's reach of each other, so the
    // test rarely diverges)
    for (int l = lo + 2 * tid; l < hi; l += 512) {
        v4f w[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) w[e] = *(const v4f *)(wc + 4 * (size_t)min(l + e, n_wave - 1));   // ln x, l q, q / l, l
#pragma unroll
        for (int j = 0; j < RBAR_G; ++j) {
            if (j >= ng) break;
            const int g = g0 + j;
            float v[2], sum[2] = {0.0f, 0.0f};
#pragma unroll
            for (int b = 0; b < NB_MAX; ++b) {
                if (b >= nb) break;
                const float ta = (float)(opz[j] * fl.gk[b]), t0 = fmaf(w[0][3], ta, tc[b]), t1 = fmaf(w[1][3], ta, tc[b]);
                if (fminf(fabsf(t0), fabsf(t1)) < cut) {
                    sum[0] = fmaf(cb[j][b], __builtin_amdgcn_exp2f(-t0 * t0), sum[0]);
                    sum[1] = fmaf(cb[j][b], __builtin_amdgcn_exp2f(-t1 * t1), sum[1]);
                }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float F = ffl[j] + (1.0f - ffl[j]) * __builtin_amdgcn_exp2f(
                                                            tauv2[j] * __builtin_amdgcn_exp2f(delta2[j] * w[e][0]));
                v[e] = (l + e < n_wave && sum[e] != 0.0f) ? sum[e] * F * w[e][1] : 0.0f;
            }
            if (P == SPS_F32) {
                uint16_t *o = (uint16_t *)rb + bf3_at(g, ld, l);   // l is even
                uint16_t h[2], m[2], q[2];
                split3(v[0], h[0], m[0], q[0]);
                split3(v[1], h[1], m[1], q[1]);
                *(uint32_t *)o = h[0] | ((uint32_t)h[1] << 16);
                *(uint32_t *)(o + 32) = m[0] | ((uint32_t)m[1] << 16);
                *(uint32_t *)(o + 64) = q[0] | ((uint32_t)q[1] << 16);
            } else {
                uint16_t *o = (uint16_t *)rb + bfx_at(g, ld, l);   // interleaved hi / lo rows
                const uint16_t h0 = f2bf(v[0]), h1 = f2bf(v[1]);
                *(uint32_t *)o = h0 | ((uint32_t)h1 << 16);
                *(uint32_t *)(o + 32) = f2bf(v[0] - bf2f(h0)) | ((uint32_t)f2bf(v[1] - bf2f(h1)) << 16);
            }
        }
    }
}

// dP_age and dP_Z from Wbar = dlogL/dP_SSP (stored [s][ld], galaxies contiguous):
//   dP_age(i) = sum_j P_Z(j) Wbar[j NA + i],  dP_Z(j) = sum_i P_age(i) Wbar[j NA + i]
// over the n_split partial products of the gradient GEMM's K ranges (split elements apart).  Each Wbar
// element is read once; a group of ages' dP_age are complete, its dP_Z are partial sums written SoA
// pb[NA + grp NZ + j][n] and added by the weights adjoint.  Written SoA pb[r][n] (r < NA: dP_age).
// From GPL_BIG_N galaxies on (one partial product) a thread takes a galaxy and a group of 24 ages.
constexpr int WB_BIG = 4, WB_SMALL = 6;   // groups of ages
__global__ void __launch_bounds__(256) k_wbar_reduce(int n, const float *pw, const float *wbar, int ld, float *pb) {
    constexpr int AGES = (NA + WB_BIG - 1) / WB_BIG;
    const int g = blockIdx.x * 256 + threadIdx.x, grp = blockIdx.y;
    if (g >= n) return;
    float pz[NZ], dz[NZ];
#pragma unroll
    for (int j = 0; j < NZ; ++j) {
        pz[j] = pw[(size_t)(PW_PZ + j) * n + g];
        dz[j] = 0.0f;
    }
    const int i1 = min(NA, (grp + 1) * AGES);
#pragma unroll 1
    for (int i = grp * AGES; i < i1; ++i) {
        float w[NZ];
#pragma unroll
        for (int j = 0; j < NZ; ++j) w[j] = wbar[(size_t)(j * NA + i) * ld + g];
        const float pa = pw[(size_t)i * n + g];
        float da = 0.0f;
#pragma unroll
        for (int j = 0; j < NZ; ++j) {
            da = fmaf(pz[j], w[j], da);
            dz[j] = fmaf(pa, w[j], dz[j]);
        }
        pb[(size_t)i * n + g] = da;
    }
#pragma unroll
    for (int j = 0; j < NZ; ++j) pb[(size_t)(NA + grp * NZ + j) * n + g] = dz[j];
}

// Below GPL_BIG_N the chain of loads is the time, so each of a block's waves takes one age of its group
// for 64 galaxies, two partial products' loads in flight, and the group's dP_Z are summed in LDS.  us at 100 /
// 1500 / 4096 / 9600 galaxies (8 / 6 / 2 / 1 products): 7.8 / 9.2 / 8.5 / 11.5; a thread per group of 24
// ages, after a pass of its own for the partial products, 16.2 / 19.1 / 20.9 / 13.0.
constexpr int WB_AGES = (NA + WB_SMALL - 1) / WB_SMALL, WB_Q = 2;
__global__ void __launch_bounds__(WB_AGES * WAVE) k_wbar_reduce_wave(int n, const float *pw, const float *wbar, int ld,
                                                                    int n_split, size_t split, float *pb) {
    __shared__ float dz[WB_AGES][NZ][WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = blockIdx.y, i = grp * WB_AGES + wv, g = blockIdx.x * WAVE + lane, gg = min(g, n - 1);
    if (i < NA) {
        float w[NZ];
#pragma unroll
        for (int j = 0; j < NZ; ++j) w[j] = 0.0f;
        for (int q0 = 0; q0 < n_split; q0 += WB_Q) {   // WB_Q products' loads in flight
            float v[WB_Q][NZ];
#pragma unroll
            for (int u = 0; u < WB_Q; ++u)
#pragma unroll
                for (int j = 0; j < NZ; ++j)
                    v[u][j] = wbar[min(q0 + u, n_split - 1) * split + (size_t)(j * NA + i) * ld + gg];
#pragma unroll
            for (int u = 0; u < WB_Q; ++u)
#pragma unroll
                for (int j = 0; j < NZ; ++j)
                    if (q0 + u < n_split) w[j] += v[u][j];
        }
        const float pa = pw[(size_t)i * n + gg];
        float da = 0.0f;
#pragma unroll
        for (int j = 0; j < NZ; ++j) {
            da = fmaf(pw[(size_t)(PW_PZ + j) * n + gg], w[j], da);
            dz[wv][j][lane] = pa * w[j];
        }
        if (g < n) pb[(size_t)i * n + g] = da;
    }
    __syncthreads();
    const int ages = min(WB_AGES, NA - grp * WB_AGES);
    for (int j = wv; j < NZ; j += WB_AGES) {
        float v = 0.0f;
        for (int t = 0; t < ages; ++t) v += dz[t][j][lane];
        if (g < n) pb[(size_t)(NA + grp * NZ + j) * n + g] = v;
    }
}
static_assert((WB_SMALL - 1) * WB_AGES < NA, "no group without ages");

// FP64 magnitudes from the partials [t][g][quantity]: a block per galaxy, thread (r, q) sums every R-th
// partial of quantity q, then the R row sums of each quantity are added in LDS; meanwhile the last
// thread forms the magnitude offset.
__global__ void __launch_bounds__(256) k_exact_finish64(DevConsts k, int n, int n_parts, const double *params,
                                                        const double *z, const double *part, double *mag) {
    __shared__ double red[256], m0;
    const int nb = k.n_band, npart = 2 * nb, nt = 192;
    const int g = blockIdx.x, tid = threadIdx.x, R = nt / npart, r = tid / npart, q = tid % npart;
    double v = 0.0;
    if (r < R)
        for (int t = r; t < n_parts; t += R) v += part[((size_t)t * n + g) * npart + q];
    if (tid == 255) m0 = mag_offset(k, z[g]) - 2.5 * params[g];
    red[tid] = v;
    __syncthreads();
    if (tid < npart) {
        double acc = 0.0;
        for (int i = 0; i < R; ++i) acc += red[i * npart + tid];
        red[tid] = acc;   // read by this thread alone until the barrier
    }
    __syncthreads();
    if (tid < nb) mag[(size_t)g * nb + tid] = m0 - 2.5 * log10(red[tid] / red[nb + tid]);
}

// ------------------------------------------------------------------ weights and their adjoint, a wave per galaxy
// Below GPL_BIG_N galaxies: a lane takes age bins lane and lane + 64, so the serial chain of a galaxy
// is two bins instead of the twelve of eight lanes per galaxy, and the weights row is written by the
// wave that formed it.  A block takes XWG galaxies.  From GPL_BIG_N on the lanes that idle over short
// bins cost more than the chain.
constexpr int XWG = 8;

// age_universe_gyr to a few ulp with one square root pair and one log1p: asinh(y) = log1p(y + y^2 /
// (1 + sqrt(1 + y^2)))
__device__ inline double age_gyr_log1p(const DevConsts &k, double z) {
    const double ol = 1.0 - k.om, ep = 1.0 + z, a15 = 1.0 / (ep * sqrt(ep));
    if (!(ol > 0.0)) return 2.0 / (3.0 * k.h0_gyr) * a15;
    const double y = sqrt(ol / k.om) * a15, y2 = y * y;
    return 2.0 / (3.0 * k.h0_gyr * sqrt(ol)) * log1p(y + y2 / (1.0 + sqrt(1.0 + y2)));
}

struct WaveWeights {
    float m[2], d1[2], d2[2], d3[2], bm[2], dd[2];   // the lane's bins: mass, derivatives, burst mass, edge densities
    double S;
    float Zb, l_obs, pz, dpz;                        // pz, dpz: metallicity bin `lane`
};
template <bool DERIV>
__device__ inline WaveWeights wave_weights(const DevConsts &k, int sfh, const float (&th)[NP], double t_obs, int lane) {
    WaveWeights r{};
    const float t_obs_f = (float)t_obs;
    const bool two = lane + WAVE < NA;
    const int i1 = two ? lane + WAVE : NA - 1;
    const float up0 = k.lage_hi[lane], up1 = k.lage_hi[i1];
    if (sfh == SPS_SFH_DPL) {
        Dpl p = make_dpl(th[1], th[2], th[3]);
        dpl_at_obs(p, t_obs_f);
        dpl_bin<DERIV>(k.age_lo[lane], k.age_hi[lane], t_obs_f, p, r.m[0], r.d1[0], r.d2[0], r.d3[0]);
        if (two) dpl_bin<DERIV>(k.age_lo[i1], k.age_hi[i1], t_obs_f, p, r.m[1], r.d1[1], r.d2[1], r.d3[1]);
    } else {
        const Logn p = make_logn(th[1], th[2]);
        logn_bin<DERIV>(k.age_lo[lane], k.age_hi[lane], t_obs_f, p, r.m[0], r.d1[0], r.d2[0]);
        if (two) logn_bin<DERIV>(k.age_lo[i1], k.age_hi[i1], t_obs_f, p, r.m[1], r.d1[1], r.d2[1]);
    }
    r.S = wave_sum((double)r.m[0] + (double)r.m[1]);
    // burst window, as in forward_weights
    const float mu = th[5], inv_s3 = 1.0f / (3.0f * k.burst_sig), v0 = mu - 3.0f * k.burst_sig;
    r.l_obs = (float)log10_split(t_obs * 1e9);
    const unsigned long long a0 = __ballot(up0 > v0), a1 = __ballot(two && up1 > v0);
    const int i0 = a0 ? __builtin_ctzll(a0) : (a1 ? WAVE + __builtin_ctzll(a1) : NA - 1);
    const int i_end = min(i0 + k.burst_nbins, NA);
    auto edge = [&](int e) { return e == 0 ? -INFINITY : (e <= WAVE ? lane_value(up0, e - 1) : lane_value(up1, e - 1 - WAVE)); };
    r.Zb = burst_mass(burst_edge_at<false>(edge(i0), r.l_obs, mu, inv_s3),
                      burst_edge_at<false>(edge(i_end), r.l_obs, mu, inv_s3));
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int i = lane + WAVE * t;
        if (i >= i0 && i < i_end) {
            const BurstEdge lo = burst_edge_at<DERIV>(k.lage_lo[i], r.l_obs, mu, inv_s3);
            const BurstEdge hi = burst_edge_at<DERIV>(k.lage_hi[i], r.l_obs, mu, inv_s3);
            r.bm[t] = burst_mass(lo, hi);
            r.dd[t] = lo.d - hi.d;
        }
    }
    // metallicity bin `lane`: its upper edge, the lower one from the lane before
    const float inv_sz = 1.0f / k.sigma_logz;
    const bool top = lane >= NZ - 1;
    const float xe = top ? INFINITY : (k.met_hi[min(lane, NZ - 1)] - th[6]) * inv_sz;
    const float te = top ? 0.0f : 0.5f * erfcf(0.7071067811865475f * fabsf(xe)), de = top ? 0.0f : phi_f(xe);
    float xp = __shfl_up(xe, 1, WAVE), tp = __shfl_up(te, 1, WAVE), dp = __shfl_up(de, 1, WAVE);
    if (lane == 0) {
        xp = -INFINITY;
        tp = dp = 0.0f;
    }
    if (lane < NZ) {
        r.pz = (xp > 0.0f) ? tp - te : ((xe <= 0.0f) ? te - tp : 1.0f - tp - te);
        r.dpz = (dp - de) * inv_sz;
    }
    return r;
}
// galaxy g's parameters, in every lane
__device__ inline void wave_params(const float *params, int n, int g, int lane, float (&th)[NP]) {
    const float v = params[(size_t)min(lane, NP - 1) * n + g];
#pragma unroll
    for (int p = 0; p < NP; ++p) th[p] = lane_value(v, p);
}

// P_age, P_Z -> pw (slots as above), the weights row -> w (unless null), and the epilogue's inputs tau_V, delta,
// F_floor, z in rank order -> eg [4][n]
template <int P>
__global__ void __launch_bounds__(XWG * WAVE) k_exact_weights(DevConsts k, int n, int sfh, const int *perm,
                                                              const float *params, const float *z, float *pw,
                                                              float *eg, void *w) {
    __shared__ __attribute__((aligned(8))) float sp[XWG][XROWF];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & (WAVE - 1);
    const int r0 = blockIdx.x * XWG, r = min(r0 + wv, n - 1), g = perm ? perm[r] : r;
    float th[NP];
    wave_params(params, n, g, lane, th);
    const float zf = z[g];
    const WaveWeights ww = wave_weights<false>(k, sfh, th, age_gyr_log1p(k, (double)zf), lane);
    const float fb = th[4], sm = (1.0f - fb) * (float)(1.0 / ww.S), bz = (ww.Zb > 0.0f) ? fb / ww.Zb : 0.0f;
    sp[wv][lane] = fmaf(bz, ww.bm[0], ww.m[0] * sm);
    if (lane + WAVE < NA) sp[wv][lane + WAVE] = fmaf(bz, ww.bm[1], ww.m[1] * sm);
    if (lane < NZ) sp[wv][NA + lane] = ww.pz;
    __syncthreads();
    if (lane < 4) eg[(size_t)lane * n + r] = lane == 3 ? zf : th[7 + lane];
    for (int e = tid; e < XROWF * XWG; e += XWG * WAVE) {
        const int row = e / XWG, t = e % XWG;
        if (r0 + t < n) pw[(size_t)(row < NA ? row : PW_PZ + (row - NA)) * n + r0 + t] = sp[t][row];
    }
    if (r0 + wv >= n || !w) return;
    for (int e = lane; e < S_PAD / 2; e += WAVE) expand_pair<P>(sp[wv], 2 * e, (size_t)r, w);
}

// the weights adjoint -> grad slots 1..6
__global__ void __launch_bounds__(XWG * WAVE) k_exact_adjoint_wave(DevConsts k, int n, int sfh, const int *perm,
                                                                   const float *params, const float *z,
                                                                   const float *pb, float *grad) {
    constexpr int ROWS = NA + WB_SMALL * NZ;
    __shared__ float sp[XWG][ROWS];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & (WAVE - 1);
    const int r0 = blockIdx.x * XWG, r = min(r0 + wv, n - 1), g = perm ? perm[r] : r;
    for (int e = tid; e < ROWS * XWG; e += XWG * WAVE) {
        const int row = e / XWG, t = e % XWG;
        sp[t][row] = pb[(size_t)row * n + min(r0 + t, n - 1)];
    }
    float th[NP];
    wave_params(params, n, g, lane, th);
    const WaveWeights ww = wave_weights<true>(k, sfh, th, age_gyr_log1p(k, (double)z[g]), lane);
    __syncthreads();
    const float fb = th[4], invS = (float)(1.0 / ww.S), invZ = (ww.Zb > 0.0f) ? 1.0f / ww.Zb : 0.0f;
    const float inv_s3 = 1.0f / (3.0f * k.burst_sig);
    const bool dpl = sfh == SPS_SFH_DPL;
    float v[12] = {};   // fbar, cbar, e1, e2, e3, A0..2, B0..2, d/dmu_Z
    double dv[4] = {};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int i = lane + WAVE * t;
        const float gbar = i < NA ? sp[wv][i] : 0.0f, psbar = (1.0f - fb) * gbar;
        const float ps = dpl ? ww.m[t] * invS : (float)((double)ww.m[t] / ww.S);
        const float pb_i = ww.bm[t] * invZ, dpb = ww.dd[t] * inv_s3, pbbar = fb * gbar;
        v[0] += gbar * (pb_i - ps);
        v[1] = fmaf(psbar, ps, v[1]);
        v[2] = fmaf(pbbar, dpb, v[2]);
        v[3] = fmaf(pbbar, pb_i, v[3]);
        v[4] += dpb;
        if (dpl) {
            v[5] = fmaf(psbar, ww.d1[t], v[5]);
            v[6] = fmaf(psbar, ww.d2[t], v[6]);
            v[7] = fmaf(psbar, ww.d3[t], v[7]);
            v[8] += ww.d1[t];
            v[9] += ww.d2[t];
            v[10] += ww.d3[t];
        } else {
            dv[0] += (double)psbar * (double)ww.d1[t];
            dv[1] += (double)psbar * (double)ww.d2[t];
            dv[2] += (double)ww.d1[t];
            dv[3] += (double)ww.d2[t];
        }
    }
    if (lane < NZ) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < WB_SMALL; ++q) s += sp[wv][NA + q * NZ + lane];
        v[11] = s * ww.dpz;
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) v[j] = wave_sum(v[j]);
    float out = v[11];   // lane p: component p
    out = (lane == 4) ? v[0] : out;
    out = (lane == 5) ? (v[2] - v[3] * v[4]) * invZ : out;
    if (dpl) {
#pragma unroll
        for (int j = 0; j < 3; ++j) out = (lane == 1 + j) ? (v[5 + j] - v[1] * v[8 + j]) * invS : out;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) dv[j] = wave_sum(dv[j]);
#pragma unroll
        for (int j = 0; j < 2; ++j) out = (lane == 1 + j) ? (float)((dv[j] - (double)v[1] * dv[2 + j]) / ww.S) : out;
        out = (lane == 3) ? 0.0f : out;
    }
    if (r0 + wv < n && lane >= 1 && lane <= 6) grad[(size_t)lane * n + g] = out;
}

// the weights adjoint of large batches -> grad slots 1..6, GPL lanes per galaxy
__global__ void __launch_bounds__(64) k_exact_adjoint(DevConsts k, int n, int sfh, const float *params,
                                                      const float *z, const float *pw, const float *pb,
                                                      float *grad) {
    __shared__ float lds[LDS_SLOTS * (64 / GPL)];
    __shared__ float ledge[NA + 1];
    stage_log_age_edges(k, ledge);
    const int lane = threadIdx.x, slot = lane / GPL, q = lane % GPL;
    const int g = blockIdx.x * (64 / GPL) + slot, gg = g < n ? g : n - 1;
    LdsColT<64 / GPL> col{lds + slot};
    float th[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) th[p] = params[(size_t)p * n + gg];
    const double t_obs = age_universe_gyr(k, (double)z[gg]);
    WeightsState ws;
    ws.S = __hiloint2double(__float_as_int(pw[(size_t)(PW_S + 1) * n + gg]), __float_as_int(pw[(size_t)PW_S * n + gg]));
    ws.Zb = pw[(size_t)PW_ZB * n + gg];
    ws.l_obs = pw[(size_t)PW_LOBS * n + gg];
    ws.i0 = __float_as_int(pw[(size_t)PW_I0 * n + gg]);
    for (int i = q; i < NA; i += GPL) col[i] = pb[(size_t)i * n + gg];
    float pzbar[NZ];
#pragma unroll
    for (int j = 0; j < NZ; ++j) {
        float v = 0.0f;
        for (int q = 0; q < WB_BIG; ++q) v += pb[(size_t)(NA + q * NZ + j) * n + gg];
        pzbar[j] = v;
    }
    float gr[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) gr[p] = 0.0f;
    adjoint_weights<GPL>(k, ledge, sfh, th, t_obs, ws, col, pzbar, gr, q);
    if (g >= n || q != 0) return;
#pragma unroll
    for (int p = 1; p <= 6; ++p) grad[(size_t)p * n + g] = gr[p];
}

// ------------------------------------------------------------------ filter-support windows
// Per 128-galaxy row tile: the rest-frame wavelengths any band reaches within 8 sigma for any
// of the tile's galaxies, [min_b (c_b - 8 s_b) / (1 + z_max), max_b (c_b + 8 s_b) / (1 + z_min)],
// as 128-wide wavelength tiles and 32-wide k-tiles of the padded grid, one index of margin on
// each side (14.5 sigma, beyond which T is below the smallest FP32 number, for the bands that come no nearer than
// 5 sigma to the grid); and the bands that the forward epilogue and Rbar must not skip.  One block per row tile.
//
// 8 sigma leave out less than 5e-7 of a band over 0 <= tau_V <= 4, delta >= -1.5 at z <= 3.  Without a floor a steeper
// attenuation can outweigh the transmission (delta = -3: magnitudes up to 1.6 off): steep_bands' bit b is set for a
// galaxy whose term at 8 sigma exceeds 1e-5 of the largest of those at 0 and 4 sigma of band b (none can while exp(-32)
// is below 1e-5 of the floor or of the attenuation at the centre).  A row tile with such a galaxy takes a
// window of 14.5 sigma and skips no such band.  The check takes 0.2 us of k_xwindows' 4.
__device__ __forceinline__ unsigned steep_bands(const FiltConst &fl, int nb, float z, float tauv, float delta,
                                                double lam_first, double lam_last) {
    unsigned bits = 0;
    const float inv = __builtin_amdgcn_rcpf(1.0f + z), lo = (float)lam_first, hi = (float)lam_last;
#pragma unroll 1
    for (int b = 0; b < nb; ++b) {
        const float c = (float)fl.fc[b] * inv, s8 = 0.5f * (float)(fl.hi8[b] - fl.lo8[b]) * inv;
        auto log_term = [&](float l, float x2) {   // ln(T F) at l, x sigma from the centre
            const float a = tauv * __builtin_amdgcn_exp2f(delta * __builtin_amdgcn_logf(l * (1.0f / 5500.0f)));
            return (l >= lo && l <= hi) ? -0.5f * x2 - a : -INFINITY;
        };
        const float at_c = log_term(c, 0.0f);
        if (at_c > -20.0f) continue;
        const float most = fmaxf(at_c, fmaxf(log_term(c - 0.5f * s8, 16.0f), log_term(c + 0.5f * s8, 16.0f)));
        const float far = fmaxf(log_term(fmaxf(c - s8, lo), 64.0f), log_term(fminf(c + s8, hi), 64.0f));
        if (far > most - 11.5f) bits |= 1u << b;
    }
    return bits;
}

__global__ void __launch_bounds__(128) k_xwindows(int n, int n_wave, FiltConst fl, int nb, const float *z,
                                                  const float *dust, const double *wave, double lam_first,
                                                  double lam_last, float lc_lo, float lc_hi, unsigned dense, int4 *win) {
    __shared__ float zlo[2], zhi[2];
    __shared__ unsigned steep[2];
    const int tid = threadIdx.x, g = min((int)blockIdx.x * XBM + tid, n - 1);
    float mn = z[g], mx = mn;
    // first the bound above at the bluest and the reddest centre (log2 of their ratios to 5500 A): most row tiles pass it
    const float tauv = dust[g], delta = dust[(size_t)n + g], lz = __builtin_amdgcn_logf(1.0f + mn);
    const float a_max = tauv * fmaxf(__builtin_amdgcn_exp2f(delta * (lc_lo - lz)), __builtin_amdgcn_exp2f(delta * (lc_hi - lz)));
    const bool check = dust[(size_t)2 * n + g] < 1e-9f && a_max >= 20.0f;
    unsigned mine = 0;
    if (__builtin_expect(__any(check), 0)) {
        if (check) mine = steep_bands(fl, nb, mn, tauv, delta, lam_first, lam_last);
        for (int o = 32; o > 0; o >>= 1) mine |= __shfl_xor(mine, o, 64);
    }
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o, 64));
        mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    if ((tid & 63) == 0) {
        zlo[tid >> 6] = mn;
        zhi[tid >> 6] = mx;
        steep[tid >> 6] = mine;
    }
    __syncthreads();
    const double z0 = fmin(zlo[0], zlo[1]), z1 = fmax(zhi[0], zhi[1]);
    // far_bands: the bands that come no nearer than 5 sigma to a wavelength of the grid for some galaxy of the tile: past
    // either end of it at the tile's largest or smallest z, or in a grid too coarse for them (bit clear in dense:
    // the wavelength after one at or below (c - 5 s) / (1 + z) may lie above (c + 5 s) / (1 + z)).  Such a band's
    // magnitude is made of far terms, so the epilogue must skip none; of a nearer one's sum, the terms beyond 8
    // sigma are at most exp(-(64 - 25) / 2) = 3e-9.
    const unsigned steep_any = steep[0] | steep[1];
    unsigned far_bands = (~dense & ((1u << nb) - 1u)) | steep_any;
    double lo = 1e300, hi = 0.0;
#pragma unroll
    for (int b = 0; b < NB_MAX; ++b) {   // unrolled: the bands' limits are read together
        const double l8 = fl.lo8[b], h8 = fl.hi8[b];
        if (b >= nb) continue;
        // c - 5 s and c + 5 s
        if ((1.0 + z1) * lam_first >= 0.8125 * h8 + 0.1875 * l8 || (1.0 + z0) * lam_last <= 0.8125 * l8 + 0.1875 * h8)
            far_bands |= 1u << b;
        // of these, and with steep galaxies, 14.5 sigma
        const bool wide = steep_any || ((far_bands >> b) & 1u);
        lo = fmin(lo, (wide ? 1.40625 * l8 - 0.40625 * h8 : l8) / (1.0 + z1));
        hi = fmax(hi, (wide ? 1.40625 * h8 - 0.40625 * l8 : h8) / (1.0 + z0));
    }
    // the number of wavelengths below lo (wave 0) and up to hi (wave 1) on the ascending grid: 64 probes at
    // a time (a serial binary search waited out 26 loads, 7.6 us)
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    int a = 0, c = n_wave;
    while (a < c) {
        const int step = (c - a + 63) >> 6, i = a + lane * step;
        const double l = wave[min(i, n_wave - 1)];
        const int cnt = __popcll(__ballot(i < c && (wv ? l <= hi : l < lo)));
        c = min(c, a + cnt * step);
        a = cnt ? a + (cnt - 1) * step + 1 : a;
    }
    __shared__ int found[2];
    if (lane == 0) found[wv] = a;
    __syncthreads();
    if (tid != 0) return;
    const int l0 = max(found[0] - 1, 0);
    const int l1 = min(found[1], n_wave - 1);   // one past the last index <= hi, as margin
    win[blockIdx.x] = make_int4(l0 / XBN, l1 / XBN + 1, (int)((unsigned)(l0 / XBK) | far_bands << 24), l1 / XBK + 1);
}

// ------------------------------------------------------------------ launcher
// Byte offsets of the exact path's workspace for n rows: weights rows | per-galaxy weights |
// partial sums | their tile sums | filter windows | dlogL/dnum | Rbar | Wbar | dP.  logl: the
// likelihood outputs are wanted; grad: also the gradient; dust: magnitudes with the dust derivatives' sums.
struct ExactLayout {
    size_t o_w = 0, o_pw = 0, o_part = 0, o_eg = 0, o_win = 0, o_cn = 0, o_rb = 0, o_wb = 0, o_pb = 0;
    size_t bytes = 0;
};
// K ranges of the gradient GEMM for n galaxies, and the rows of its partial products for any batch up to n
static int grad_splits(int n) {
    const int tiles = round_up(n, XBM) / XBM * (S_PAD / XBN);
    return std::min(XSPLIT_MAX, std::max(1, (XSPLIT_BLOCKS + tiles / 2) / tiles));
}
static int wbar_rows(int n) {
    int most = 0;
    for (int m = XBM;; m += XBM) {   // the split falls to 1 within a few thousand rows
        const int k = grad_splits(std::min(m, n));
        most = std::max(most, k * std::min(m, round_up(n, XBM)));
        if (m >= n) return most;
        if (k == 1) return std::max(most, round_up(n, XBM));
    }
}

static ExactLayout exact_layout(const sps_ctx *c, int n, int prec, bool logl, bool grad, bool dust = false) {
    const int nw = c->n_wave, nb = c->n_band;
    const bool f64 = (prec == SPS_F64);
    const int n_parts = f64 ? f64_parts(n, nw) : c->lw / XBN;
    const int mp = round_up(n, XBM);              // A operands are read in whole 128-row tiles
    const bool want_grad = logl && grad;
    const int npart = (want_grad || dust ? 5 : 2) * nb;
    const int esz = f64 ? 8 : 4;
    const int tsz = f64 ? 8 : 2;   // a GEMM operand's element: FP64, or BF16 parts
    const int nsplit = f64 ? 1 : (prec == SPS_F32 ? 3 : 2);
    ExactLayout L;
    size_t off = 0;
    auto carve = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    L.o_w = carve((size_t)nsplit * mp * S_PAD * tsz);
    L.o_pw = f64 ? 0 : carve((size_t)PW_SLOTS * n * 4);
    L.o_part = carve((size_t)n_parts * n * npart * esz);
    L.o_eg = carve(f64 ? 0 : (size_t)4 * n * sizeof(float));
    L.o_win = f64 ? 0 : carve((size_t)(mp / XBM) * sizeof(int4));
    if (logl) {
        L.o_cn = carve((size_t)n * NB_MAX * 4);
        if (want_grad) {
            L.o_rb = carve((size_t)nsplit * mp * c->lw * tsz);
            L.o_wb = carve((size_t)wbar_rows(n) * S_PAD * 4);
            L.o_pb = carve((size_t)(NA + std::max(WB_BIG, WB_SMALL) * NZ) * n * 4);
        }
    }
    L.bytes = off;
    return L;
}

size_t exact_ws_bytes(const sps_ctx *c, int n, int prec, bool logl, bool grad) {
    if (prec != SPS_F64) return exact_layout(c, n, prec, logl, grad).bytes;
    // the FP64 partials shrink where the blocks take more tiles: size for the largest need of any batch
    // up to n, which for one number of tiles falls on a whole number of row tiles or on n
    size_t most = 0;
    for (int t = 1; t <= (n + D_ROWS - 1) / D_ROWS; ++t)
        most = std::max(most, exact_layout(c, std::min(t * D_ROWS, n), prec, logl, grad).bytes);
    return most;
}

// The built-in tile order (sps_launch_cfg): bands of row tiles, whose panels the blocks in flight share
// in L2; each XCD its own run of them from ORDER_XCD_MT row tiles on, below in dispatch order, where the
// row tiles' different windows would load the XCDs unevenly.  BF16X value+gradient, us, bands in runs /
// in dispatch order / M fastest in runs (N fastest forward): 4096 x 5000 303 / 269 / 276, 20,011 x 2000
// 499 / 511 / 532, 65,536 x 2000 1254 / 1352 / 1440.
constexpr int ORDER_XCD_MT = 64;
static void tile_order(const sps_ctx *c, XArgs &a) {
    const bool own = c->launch.exact_order == 0;
    a.order = own ? 3 : c->launch.exact_order;
    a.xcd = c->launch.exact_xcd && (!own || a.n_mt >= ORDER_XCD_MT);
}

// perm: the caller's index of each rank, or null where the arrays come in rank order (always from
// GPL_BIG_N galaxies on).  sums: with mag_out, the band sums that a backward starts from, to be kept; with vjp,
// those of an earlier call on the same inputs, whose forward GEMM is then not repeated; sperm: the caller's
// indices of the ranks for them.
static int exact_core(sps_ctx *c, hipStream_t s, int n, int sfh, int prec, const void *params, const void *z,
                      void *mag_out, const float *obs, const float *sigma, const uint8_t *mask, float *logl,
                      float *grad, bool zordered, bool vjp, const int *perm, float *sums, const int *sperm) {
    const int nw = c->n_wave, nb = c->n_band;
    const bool f64 = (prec == SPS_F64);
    const int n_tiles = c->lw / XBN;
    const int mp = round_up(n, XBM);              // A operands are read in whole 128-row tiles
    const bool want_grad = grad != nullptr, dust5 = want_grad || sums, given = vjp && sums;
    const int npart = (dust5 ? 5 : 2) * nb;
    const int lw = c->lw;                         // padded wavelength stride of Rbar
    const bool lik = logl != nullptr || vjp;     // the likelihood's (or the adjoints') finish
    const ExactLayout Lo = exact_layout(c, n, prec, lik, want_grad, dust5);
    const size_t o_w = Lo.o_w, o_pw = Lo.o_pw, o_part = Lo.o_part, o_eg = Lo.o_eg, o_win = Lo.o_win;
    const size_t o_cn = Lo.o_cn, o_rb = Lo.o_rb, o_wb = Lo.o_wb, o_pb = Lo.o_pb;
    if (c->work_bytes < Lo.bytes || n > c->max_exact)
        return set_error(SPS_E_STATE, "the exact path's workspace holds " + std::to_string(c->max_exact) +
                                          " rows, this call needs " + std::to_string(n) +
                                          " (call sps_reserve_exact)");
    char *W = (char *)c->d_work;
    int4 *win = nullptr;   // filter-support windows of the row tiles (FP32 / BF16X paths)
    void *w_hi = W + o_w;   // weights rows: FP64 [n][S_PAD], or BF16 parts interleaved [mp][3 or 2 S_PAD]

    float *pw = f64 ? nullptr : (float *)(W + o_pw);
    const bool big = n >= GPL_BIG_N;
    // the dust parameters and z in rank order (large batches come in rank order)
    float *eg = (float *)(W + o_eg);
    const float *dust = big ? (const float *)params + (size_t)7 * n : eg;
    const float *z_r = big ? (const float *)z : eg + (size_t)3 * n;
    if (f64) {
        hipLaunchKernelGGL(k_exact_weights64, dim3(n), dim3(W64_T), 0, s, c->k, n, sfh,
                           (const double *)params, (const double *)z, c->d_edges, (double *)w_hi);
    } else if (big) {
        hipLaunchKernelGGL(k_exact_pw, dim3((n + 64 / GPL - 1) / (64 / GPL)), dim3(64), 0, s, c->k, n, sfh,
                           (const float *)params, (const float *)z, pw);
        const dim3 ge((n + XG - 1) / XG), be(256);
        if (given) {   // no weights rows
        } else if (prec == SPS_F32) hipLaunchKernelGGL(k_expand<SPS_F32>, ge, be, 0, s, n, (const float *)pw, w_hi);
        else hipLaunchKernelGGL(k_expand<SPS_BF16X>, ge, be, 0, s, n, (const float *)pw, w_hi);
    } else {
        auto kw = prec == SPS_F32 ? k_exact_weights<SPS_F32> : k_exact_weights<SPS_BF16X>;
        hipLaunchKernelGGL(kw, dim3((n + XWG - 1) / XWG), dim3(XWG * WAVE), 0, s, c->k, n, sfh, perm,
                           (const float *)params, (const float *)z, pw, eg, given ? nullptr : w_hi);
    }
    float *part = (float *)(W + o_part);
    if (f64) {
        bool wide;
        const int np = f64_parts(n, nw), tiles = f64_tiles(n, nw, &wide);
        const DArgs a{n, nw, nb, tiles, (const double *)w_hi, c->d_lum64, (const double *)params,
                      (const double *)z, c->d_wave, c->d_trap, filt_const(c->h_fc, c->h_fs), (double *)part};
        hipLaunchKernelGGL((wide ? k_exact_phot64<2> : k_exact_phot64<1>), dim3(np, (n + D_ROWS - 1) / D_ROWS),
                           dim3(D_T), 0, s, a);
        hipLaunchKernelGGL(k_exact_finish64, dim3(n), dim3(256), 0, s, c->k, n, np, (const double *)params,
                           (const double *)z, (const double *)part, (double *)mag_out);
    } else {
        const FiltConst fl = filt_const(c->h_fc, c->h_fs);
        win = (int4 *)(W + o_win);
        unsigned dense = 0;
        for (int b = 0; b < nb; ++b)
            if ((c->h_fc[b] - 5.0 * c->h_fs[b]) * c->h_step < c->h_fc[b] + 5.0 * c->h_fs[b]) dense |= 1u << b;
        hipLaunchKernelGGL(k_xwindows, dim3(mp / XBM), dim3(128), 0, s, n, nw, fl, nb, z_r, dust, c->d_wave,
                           c->h_wave.front(), c->h_wave.back(), (float)std::log2(*std::min_element(c->h_fc, c->h_fc + nb) / 5500.0),
                           (float)std::log2(*std::max_element(c->h_fc, c->h_fc + nb) / 5500.0), dense, win);
        XArgs a{};
        a.win = win;
        a.band_skip = zordered ? 1 : 0;
        a.M = n;
        a.N = lw;
        a.K = S_PAD;
        a.A = w_hi;
        a.lda = S_PAD;
        a.B = (prec == SPS_F32) ? (const void *)c->d_lt_b3 : (const void *)c->d_lt_bx;
        a.ldb = S_PAD;
        a.n_mt = mp / XBM;
        a.n_nt = lw / XBN;
        a.dust = dust;
        a.z = z_r;
        a.wave = c->d_wave;
        a.wc = c->d_wc;
        a.n_wave = nw;
        a.n_band = nb;
        for (int b = 0; b < NB_MAX; ++b) { a.fc[b] = c->h_fc[b]; a.inv_fs[b] = 1.0 / c->h_fs[b]; }
        a.part = part;
        a.npart = npart;
        tile_order(c, a);
        const dim3 gx(a.n_mt * a.n_nt), bx(256);
        const bool ring = c->launch.exact_ring != 0;
        if (given) {   // the sums are the caller's
        } else if (prec == SPS_F32 && !dust5) hipLaunchKernelGGL((k_xgemm<SPS_F32, EPI_PHOT, false>), gx, bx, 0, s, a);
        else if (prec == SPS_F32) hipLaunchKernelGGL((k_xgemm<SPS_F32, EPI_PHOT_DUST, false>), gx, bx, 0, s, a);
        else if (!dust5 && ring) hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_PHOT, true>), gx, bx, 0, s, a);
        else if (!dust5) hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_PHOT, false>), gx, bx, 0, s, a);
        else if (ring) hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_PHOT_DUST, true>), gx, bx, 0, s, a);
        else hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_PHOT_DUST, false>), gx, bx, 0, s, a);
    }

    float *cn = lik ? (float *)(W + o_cn) : nullptr;
    if (!f64) {
        auto kf = dust5 ? k_exact_finish<true> : k_exact_finish<false>;
        DevConsts k = c->k;
        if (prec == SPS_F32) k.kfac = std::ldexp(k.kfac, -c->lum32_exp);
        hipLaunchKernelGGL(kf, dim3((n + 31) / 32), dim3(256), 0, s, k, n, n_tiles, perm,
                           (const float *)params, z_r, (const int4 *)win, (const float *)part, npart, (float *)mag_out,
                           obs, sigma, mask, logl, grad, cn, vjp ? 1 : 0, sums, sperm);
    }
    if (want_grad) {
        void *r_hi = W + o_rb;   // Rbar rows: BF16 parts interleaved [mp][3 or 2 lw]
        const bool many = n >= RBAR_BIG_MIN_GAL;
        dim3 gr(many ? (n + RBAR_G_BIG - 1) / RBAR_G_BIG : n), br(256);
        const FiltConst fl = filt_const(c->h_fc, c->h_fs);
        auto kr = (prec == SPS_F32) ? (many ? k_exact_rbar<SPS_F32, RBAR_G_BIG> : k_exact_rbar<SPS_F32, 1>)
                                    : (many ? k_exact_rbar<SPS_BF16X, RBAR_G_BIG> : k_exact_rbar<SPS_BF16X, 1>);
        hipLaunchKernelGGL(kr, gr, br, 0, s, n, nw, lw, nb, fl, dust, z_r, c->d_wc, cn, win, r_hi);
        XArgs b{};
        b.win = win;
        b.M = n;
        b.N = S_PAD;
        b.K = lw;
        b.A = r_hi;
        b.lda = lw;
        b.B = (prec == SPS_F32) ? (const void *)c->d_ls_b3 : (const void *)c->d_ls_bx;
        b.ldb = lw;
        b.n_mt = mp / XBM;
        b.n_nt = S_PAD / XBN;
        b.C = (float *)(W + o_wb);
        b.ldc = mp;
        b.n_store = S_PAD;
        b.k_splits = grad_splits(n);
        b.c_split = (size_t)S_PAD * mp;
        tile_order(c, b);
        const dim3 g2(b.n_mt * b.n_nt * b.k_splits), b2(256);
        if (prec == SPS_F32) hipLaunchKernelGGL((k_xgemm<SPS_F32, EPI_STORE, false>), g2, b2, 0, s, b);
        else if (c->launch.exact_ring) hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_STORE, true>), g2, b2, 0, s, b);
        else hipLaunchKernelGGL((k_xgemm<SPS_BF16X, EPI_STORE, false>), g2, b2, 0, s, b);
        float *pb = (float *)(W + o_pb);
        if (big) {
            static_assert(XSPLIT_BLOCKS < GPL_BIG_N / XBM * (S_PAD / XBN), "one partial product");
            hipLaunchKernelGGL(k_wbar_reduce, dim3((n + 255) / 256, WB_BIG), dim3(256), 0, s, n,
                               (const float *)pw, (const float *)b.C, mp, pb);
            hipLaunchKernelGGL(k_exact_adjoint, dim3((n + 64 / GPL - 1) / (64 / GPL)), dim3(64), 0, s, c->k, n, sfh,
                               (const float *)params, (const float *)z, (const float *)pw, (const float *)pb, grad);
        } else {
            hipLaunchKernelGGL(k_wbar_reduce_wave, dim3((n + WAVE - 1) / WAVE, WB_SMALL), dim3(WB_AGES * WAVE), 0, s, n,
                               (const float *)pw, (const float *)b.C, mp, b.k_splits, b.c_split, pb);
            hipLaunchKernelGGL(k_exact_adjoint_wave, dim3((n + XWG - 1) / XWG), dim3(XWG * WAVE), 0, s, c->k, n, sfh,
                               perm, (const float *)params, (const float *)z, (const float *)pb, grad);
        }
    }
    SPS_HIP(hipGetLastError());
    return SPS_OK;
}

// ------------------------------------------------------------------ z order
// Inputs of the galaxy of each rank (perm: rank -> galaxy) into rank order, and the outputs
// back to the caller's order; one thread per rank.
__global__ void __launch_bounds__(256) k_exact_order_in(int n, int nb, const int *perm, const float *params,
                                                        const float *z, const float *obs, const float *sigma,
                                                        const uint8_t *mask, float *params_s, float *z_s,
                                                        float *obs_s, float *sig_s, uint8_t *mask_s) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const int g = perm[r];
#pragma unroll
    for (int p = 0; p < NP; ++p) params_s[(size_t)p * n + r] = params[(size_t)p * n + g];
    z_s[r] = z[g];
    if (obs)
        for (int b = 0; b < nb; ++b) obs_s[(size_t)r * nb + b] = obs[(size_t)g * nb + b];
    if (sigma)
        for (int b = 0; b < nb; ++b) sig_s[(size_t)r * nb + b] = sigma[(size_t)g * nb + b];
    if (mask) mask_s[r] = mask[g];
}

__global__ void __launch_bounds__(256) k_exact_order_out(int n, int nb, const int *perm, const float *mag_s,
                                                         const float *logl_s, const float *grad_s, float *mag,
                                                         float *logl, float *grad) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const int g = perm[r];
    if (mag)
        for (int b = 0; b < nb; ++b) mag[(size_t)g * nb + b] = mag_s[(size_t)r * nb + b];
    if (logl) logl[g] = logl_s[r];
    if (grad)
#pragma unroll
        for (int p = 0; p < NP; ++p) grad[(size_t)p * n + g] = grad_s[(size_t)p * n + r];
}

// The FP32 / BF16X paths rank the galaxies by z first (by buckets of the z table's grid, or 64 over
// 0 <= z < 8 without a table): a 128-galaxy row tile then spans a narrow z range, its filter-support
// window (k_xwindows) covers about half of the wavelength grid instead of two thirds, and the forward
// epilogue skips the bands out of reach of a wave's galaxies.  From XSORT_MIN galaxies on the inputs
// are gathered and the outputs returned by passes of their own; below, one block ranks the batch
// (k_exact_rank) and the per-galaxy kernels read and write through the ranks.  A single row tile keeps
// its order.
constexpr int XSORT_MIN = 16384;
static_assert(XSORT_MIN == GPL_BIG_N, "batches with their own passes are the large ones");
// perm: the caller's indices ordered by z bucket, in their own order within a bucket (the same tiles and
// windows, so the same sums, on every run); n < XSORT_MIN, at most RANK_BK buckets.  Each wave ranks a
// contiguous part of the batch, 64 galaxies at a time: lanes of equal bucket are found by ballots over
// the bucket's bits, and the first of them advances the wave's count.
constexpr int RANK_T = 1024, RANK_BK = 1024, RANK_W = RANK_T / WAVE, RANK_PER = XSORT_MIN / RANK_T;
static_assert(RANK_BK == RANK_T && SORT_MAX_BUCKETS <= RANK_BK && XSORT_MIN <= 65536, "a thread per bucket, 16-bit counts");
__global__ void __launch_bounds__(RANK_T) k_exact_rank(DevConsts k, int n, const float *__restrict__ z,
                                                       int *__restrict__ perm) {
    __shared__ uint16_t cnt[RANK_W][RANK_BK];
    __shared__ int start[RANK_BK], wsum[RANK_W];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid >> 6, nbk = k.n_z;
    for (int w = 0; w < RANK_W; ++w) cnt[w][tid] = 0;
    const int per = ((n + RANK_W - 1) / RANK_W + WAVE - 1) / WAVE * WAVE, base = wv * per;   // per <= 64 RANK_PER
    const int bits = 32 - __clz(max(nbk - 1, 1));
    int bk[RANK_PER], at[RANK_PER];
#pragma unroll
    for (int t = 0; t < RANK_PER; ++t) {
        const int i = base + WAVE * t + lane;
        bk[t] = -1;
        if (WAVE * t < per && i < n) {
            float f;
            const int kk = z_bucket(k, z[i], &f);
            bk[t] = kk < 0 ? nbk - 1 : kk;
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RANK_PER; ++t) {
        at[t] = 0;
        unsigned long long same = __ballot(bk[t] >= 0);
        if (same == 0) continue;
        for (int bit = 0; bit < bits; ++bit) {
            const bool on = (bk[t] >> bit) & 1;
            const unsigned long long m = __ballot(on);
            same &= on ? m : ~m;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull)), c = bk[t] >= 0 ? cnt[wv][bk[t]] : 0;
        wave_sync();   // every lane has read its bucket's count before the bucket's first lane advances it
        at[t] = c + before;
        if (bk[t] >= 0 && before == 0) cnt[wv][bk[t]] = (uint16_t)(c + __popcll(same));
        wave_sync();
    }
    __syncthreads();
    // bucket tid: its waves' counts to offsets, and the exclusive scan of the totals
    int own = 0;
    for (int w = 0; w < RANK_W; ++w) {
        const int c = cnt[w][tid];
        cnt[w][tid] = (uint16_t)own;
        own += c;
    }
    int x = own;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int y = __shfl_up(x, o, WAVE);
        if (lane >= o) x += y;
    }
    if (lane == WAVE - 1) wsum[wv] = x;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wv; ++w) before += wsum[w];
    start[tid] = before + x - own;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RANK_PER; ++t)
        if (bk[t] >= 0) perm[start[bk[t]] + cnt[wv][bk[t]] + at[t]] = base + WAVE * t + lane;
}

struct XsortLayout {
    size_t o_par, o_z, o_obs, o_sig, o_msk, o_mag, o_ll, o_gr, bytes;
};
static XsortLayout xsort_layout(const sps_ctx *c, int n) {
    const int nb = c->n_band;
    XsortLayout x{};
    size_t off = 0;
    auto carve = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    x.o_par = carve((size_t)NP * n * 4);
    x.o_z = carve((size_t)n * 4);
    x.o_obs = carve((size_t)n * nb * 4);
    x.o_sig = carve((size_t)n * nb * 4);
    x.o_msk = carve((size_t)n);
    x.o_mag = carve((size_t)n * nb * 4);
    x.o_ll = carve((size_t)n * 4);
    x.o_gr = carve((size_t)NP * n * 4);
    x.bytes = off;
    return x;
}

size_t exact_xsort_bytes(const sps_ctx *c, int n) { return n >= XSORT_MIN ? xsort_layout(c, n).bytes : 0; }

int launch_exact(sps_ctx *c, hipStream_t s, int n, int sfh, int prec, const void *params, const void *z,
                 void *mag_out, const float *obs, const float *sigma, const uint8_t *mask, float *logl,
                 float *grad, bool ordered, bool vjp, float *sums) {
    if (prec == SPS_F64 || ordered)
        return exact_core(c, s, n, sfh, prec, params, z, mag_out, obs, sigma, mask, logl, grad,
                          ordered && prec != SPS_F64, vjp, nullptr, sums, nullptr);
    const DevConsts grid = z_sort_grid(c);
    if (n < XSORT_MIN) {
        const bool rank = n > XBM;
        if (rank) {
            hipLaunchKernelGGL(k_exact_rank, dim3(1), dim3(RANK_T), 0, s, grid, n, (const float *)z, c->d_perm);
            SPS_HIP(hipGetLastError());
        }
        return exact_core(c, s, n, sfh, prec, params, z, mag_out, obs, sigma, mask, logl, grad, rank, vjp,
                          rank ? c->d_perm : nullptr, sums, nullptr);
    }
    const int nb = c->n_band;
    const XsortLayout xl = xsort_layout(c, n);
    const size_t o_par = xl.o_par, o_z = xl.o_z, o_obs = xl.o_obs, o_sig = xl.o_sig, o_msk = xl.o_msk;
    const size_t o_mag = xl.o_mag, o_ll = xl.o_ll, o_gr = xl.o_gr;
    if (c->xsort_bytes < xl.bytes || n > c->max_gal)
        return set_error(SPS_E_STATE, "the exact path's z-order buffer is too small for " + std::to_string(n) +
                                          " galaxies (call sps_reserve_exact)");
    char *X = (char *)c->d_xsort;
    float *par_s = (float *)(X + o_par), *z_s = (float *)(X + o_z), *obs_s = (float *)(X + o_obs);
    float *sig_s = (float *)(X + o_sig), *mag_s = (float *)(X + o_mag), *ll_s = (float *)(X + o_ll);
    float *gr_s = (float *)(X + o_gr);
    uint8_t *msk_s = (uint8_t *)(X + o_msk);
    int rc = launch_bucket_sort(c, s, n, (const float *)z, nullptr, &grid);
    if (rc) return rc;
    const dim3 g1((n + 255) / 256), b1(256);
    hipLaunchKernelGGL(k_exact_order_in, g1, b1, 0, s, n, nb, (const int *)c->d_perm, (const float *)params,
                       (const float *)z, obs, sigma, mask, par_s, z_s, obs_s, sig_s, msk_s);
    rc = exact_core(c, s, n, sfh, prec, par_s, z_s, mag_out ? mag_s : nullptr, obs ? obs_s : nullptr,
                    sigma ? sig_s : nullptr, mask ? msk_s : nullptr, logl ? ll_s : nullptr, grad ? gr_s : nullptr,
                    true, vjp, nullptr, sums, c->d_perm);
    if (rc) return rc;
    hipLaunchKernelGGL(k_exact_order_out, g1, b1, 0, s, n, nb, (const int *)c->d_perm, mag_s, ll_s, gr_s,
                       (float *)mag_out, logl, grad);
    SPS_HIP(hipGetLastError());
    return SPS_OK;
}

}  // namespace sps
