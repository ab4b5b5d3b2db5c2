// Adjoint of the order-invariant sum on the matrix cores (gfx950): the sums of k_adjoint.hip for
// grids on which most terms are separable over a 16 x 16 sub-tile of frequencies (k_accum_mfma.hip
// has the separable form: term = X(u) Y(v) exp(-(a + j phi) t), t = u v / 56.25).
//
// For one Gaussian and wavelength, with w = v / 7.5 and W_k(u) = sum_v conj(Gs(u, v)) w^k Y(v),
//   Z_j(u) = sum_v conj(Gs) w^j Y exp(-a t) = sum_k c_k (u / 7.5)^k W_{k+j}(u),
// and every sum the gradient needs is sum_u X(u) u^p Z_j(u) with p + j <= 2.  W_k for 16
// Gaussians is a matrix product: A = conj(Gs) w^k (16 columns u by 16 rows v, real and imaginary
// parts along the contraction; the same for every Gaussian, so it is formed once per sub-tile
// in LDS), B = Y.  Per (Gaussian, sub-tile) and wavelength 32 complex factors are evaluated and
// 16 polynomials combined instead of 256 terms.
//
// A and B are fp16 pairs as in the forward (k <= 3: products h h, h l, l h; k >= 4, which only
// multiply c_3 and smaller or c_2 in Z_2, one product), accumulated in FP32.  Gs is scaled by
// a power of two per sub-tile and wavelength.  X, the polynomials and all sums are FP32.  W_k of a higher order
// than a Gaussian's class meets c_k = 0, so results do not depend on which 16 share a pass.
//
// Work.  A work-group of four wavefronts owns up to 512 consecutive sorted Gaussians and a range of
// tiles (the adjoint's items).  At an item's start the Gaussians are ordered by class.  Per
// sub-tile every thread tests its two Gaussians; the accepted ones go into an LDS list, the
// A operands into LDS, and each wavefront takes 16 listed Gaussians at a time: lane l holds
// Gaussian l % 16, evaluates X at columns 4 (l / 16) + j and Y at rows 4 (l / 16) + j (the
// layouts of the result and of B), and the sums over the four lane groups go to the Gaussian's
// LDS accumulators.  Every Gaussian is visited once per sub-tile, so the order of its sums is
// fixed.  Gaussians that fail the separable form's tests there, and all of them where a few frequencies
// of Gs stand out, are evaluated term by term.
//
// Bound: VALU issue (80 % of the busy cycles, the matrix units 21 %), 74 VALU instructions per
// (Gaussian, sub-tile) at three wavelengths against 212 term by term: about 50 evaluate and combine,
// the rest test the Gaussians and build the operands, once per sub-tile.  1e5 Gaussians at
// 1080 x 1920 x 3: 11.7 -> 7.1 ms.  Three wavefronts per SIMD (two: 8.6 ms for the backward instead of
// 7.6), which the opaque copies of indices make possible.  Gradients against FP64, 1000 Gaussians at
// 1080 x 1920 x 3: 2.2e-7 ... 6.8e-7 (3.4e-7 ... 1.7e-6 term by term).
#include "mfma_f16.h"

namespace gws {

constexpr int AM_T = 256;         // threads
constexpr int AM_YS = 5, AM_GS = 8;  // powers of two carried by Y and by the scaled Gs
constexpr int AM_MAXW = 8;        // W_0 ... W_7

// z += e w by component.
static __device__ __forceinline__ void fma4(float4_t &z, const float (&e)[4], float4_t w)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = fmaf(e[j], w[j], z[j]);
}
static __device__ __forceinline__ float4_t f4zero() { return (float4_t){0.0f, 0.0f, 0.0f, 0.0f}; }

// Index of the 16 x 16 sub-tile (column block h of tile tx, row block s of tile ty).
static __device__ __forceinline__ int sub_index(const AdjGeom &geo, int tx, int ty, int h, int s)
{
    return ((ty - geo.ty_min) * 4 + s) * (2 * geo.ntx) + (tx - geo.tx_min) * 2 + h;
}

// Gs sub-tile-major (zero outside the grid), the largest finite binary exponent per sub-tile and
// wavelength (a faint wavelength's Gs on a strong one's scale would lose its low fp16 parts), and per
// sub-tile whether a few of its frequencies stand out: a mean of the field gradient, a grating.  The
// separable form sums moments about the sub-tile's centre, where the weight such a frequency has (zero, on
// an axis) comes out as a difference, and fp16 pairs hold the rest on its scale: with a mean of ten times
// the spread the gradients of 20-pixel means were 1e-4 off.  A sub-tile whose largest component of Gs
// has a square above AM_SPIKE times the mean |Gs|^2 goes term by term: a single frequency five times
// the others' size still passes; of independent normal components 512 erfc(5) = 8e-10 of the
// sub-tiles do not.
// gexp: C exponents and that flag for each sub-tile.
constexpr float AM_SPIKE = 25.0f;
template <int C>
__global__ void __launch_bounds__(256) k_adj_pack_sub(Consts k, AdjGeom geo, const float2 *__restrict__ gspec,
                                                      float2 *__restrict__ gsub, int32_t *__restrict__ gexp)
{
    __shared__ float s_m[C][4], s_s[C][4];  // per wavefront: largest component, sum of |Gs|^2
    const int sub = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int x0 = (geo.tx_min * 2 + sub % (2 * geo.ntx)) * 16, y0 = (geo.ty_min * 4 + sub / (2 * geo.ntx)) * 16;
    const int mxp = x0 + (t & 15), myp = y0 + (t >> 4);
    const int hx = k.nx / 2, hy = k.ny / 2;
    const bool in = mxp >= -hx && mxp < hx && myp >= -hy && myp < hy;
    const int mx = mxp < 0 ? mxp + k.nx : mxp, my = myp < 0 ? myp + k.ny : myp;
    float2 v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = in ? gspec[((int64_t)c * k.ny + my) * k.nx + mx] : make_float2(0.0f, 0.0f);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        gsub[((int64_t)sub * C + c) * 256 + t] = v[c];
        float m = fmaxf(fabsf(v[c].x), fabsf(v[c].y));
        if (!(m <= 3.4028234663852886e38f)) m = 0.0f;
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
        if (lane == 0) s_m[c][wave] = m;
    }
    __syncthreads();
    float top[C];  // the largest component, 1 ... 2 on its own scale
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float m = fmaxf(fmaxf(s_m[c][0], s_m[c][1]), fmaxf(s_m[c][2], s_m[c][3]));
        const int e = m > 0.0f ? ilogbf(m) : -1000;
        if (t == 0) gexp[(int64_t)sub * (C + 1) + c] = e;
        top[c] = ldexpf(m, -e);
        const float x = ldexpf(v[c].x, -e), y = ldexpf(v[c].y, -e);
        float q = fmaf(x, x, y * y);
        for (int d = 32; d >= 1; d >>= 1) q += __shfl_xor(q, d);
        if (lane == 0) s_s[c][wave] = q;
    }
    __syncthreads();
    if (t == 0) {
        const float count = (float)((min(x0 + 16, hx) - max(x0, -hx)) * (min(y0 + 16, hy) - max(y0, -hy)));  // on the grid
        bool spike = false;
#pragma unroll
        for (int c = 0; c < C; ++c)
            spike |= top[c] * top[c] * count > AM_SPIKE * ((s_s[c][0] + s_s[c][1]) + (s_s[c][2] + s_s[c][3]));
        gexp[(int64_t)sub * (C + 1) + C] = spike;
    }
}

// Geometry of a sub-tile, the same for every scene (float words of its row of the table): the
// separable form's limits |z| <= zlim and the bound of phi per metre, then per wavelength k_z
// along the central row and column minus its centre's (16 each), D_c at the centre (a
// double), phi per metre of depth, k_z's slope and curvature along w.
constexpr int AS_HEAD = 4, AS_C = 40;
__host__ __device__ constexpr int adj_sub_floats(int c) { return AS_HEAD + AS_C * c; }

__global__ void __launch_bounds__(128) k_adj_sub_geo(Consts k, AdjGeom geo, float *__restrict__ table)
{
    const int sub = blockIdx.x, t = threadIdx.x, sx = sub % (2 * geo.ntx), sy = sub / (2 * geo.ntx);
    const int sx0 = (geo.tx_min * 2 + sx) * 16, sy0 = (geo.ty_min * 4 + sy) * 16;
    float *row = table + (int64_t)sub * adj_sub_floats(k.C);
    const double iWx = 1.0 / (k.nx * k.px), iWy = 1.0 / (k.ny * k.py);
    const double nx0 = (sx0 + 7.5) * iWx, ny0 = (sy0 + 7.5) * iWy;
    const int c = t >> 5, i = t & 15;
    if (c < k.C) {
        const bool along_y = t & 16;
        const double il = k.inv_lambda[c], nu = along_y ? (sy0 + i) * iWy : (sx0 + i) * iWx, nc = along_y ? nx0 : ny0;
        const double r0 = fmin(nx0 * nx0 + ny0 * ny0, il * il), D0 = dprop_m(r0, il), kz2 = fmax(il * il - r0, 1e-300);
        row[AS_HEAD + AS_C * c + (t & 31)] = (float)(dprop_m(fmin(nu * nu + nc * nc, il * il), il) - D0);
        if ((t & 31) == 0) {
            float *w = row + AS_HEAD + AS_C * c + 32;
            *reinterpret_cast<double *>(w) = D0;
            const double kz = sqrt(kz2), step = 7.5 * iWy;
            w[2] = (float)(353.4291735288517 * nx0 * ny0 * iWx * iWy / (kz2 * kz));
            w[3] = (float)(-ny0 / kz * step);
            w[4] = (float)(-0.5 / kz * (1.0 + ny0 * ny0 / kz2) * step * step);
        }
    }
    if (t == 0) {
        const double xm = fabs(nx0) + 7.5 * iWx, ym = fabs(ny0) + 7.5 * iWy;
        double zlim = 3.4e38, phimax = 0.0;
        for (int q = 0; q < k.C; ++q) {
            const double il = k.inv_lambda[q], wm = il * il - xm * xm - ym * ym;
            if (wm > 0.0) {
                const double k3 = 1.0 / (wm * sqrt(wm)), k5 = 3.0 * k3 / wm;
                phimax = fmax(phimax, 353.43 * iWx * iWy * xm * ym * k3);
                zlim = fmin(zlim, 1e-6 / (1326.0 * iWx * iWy * (iWx * ym * (k3 + k5 * xm * xm) + iWy * xm * (k3 + k5 * ym * ym))));
            } else {
                zlim = -1.0;
            }
        }
        row[0] = (float)zlim;
        row[1] = (float)phimax;
    }
}

int adj_sub_table_floats(int C) { return adj_sub_floats(C); }

hipError_t launch_adj_pack_sub(const Consts &k, const AdjGeom &geo, int n_scenes, const float2 *gspecs, float2 *gsub,
                               int32_t *gexp, float *table, hipStream_t s)
{
    const int nsub = 4 * geo.nreg;
    const int64_t M = (int64_t)k.nx * k.ny * k.C, per = (int64_t)nsub * k.C * 256;
    hipLaunchKernelGGL(k_adj_sub_geo, dim3(nsub), dim3(128), 0, s, k, geo, table);
#define GWS_PACK(CC)                                                                                              \
    hipLaunchKernelGGL(k_adj_pack_sub<CC>, dim3(nsub), dim3(256), 0, s, k, geo, gspecs + (int64_t)i * M,                \
                       gsub + (int64_t)i * per, gexp + (int64_t)i * nsub * (CC + 1))
    for (int i = 0; i < n_scenes; ++i)
        switch (k.C) {
        case 1: GWS_PACK(1); break;
        case 2: GWS_PACK(2); break;
        case 3: GWS_PACK(3); break;
        case 4: GWS_PACK(4); break;
        default: return hipErrorInvalidValue;
        }
#undef GWS_PACK
    return hipGetLastError();
}

// The sub-tile's tables in LDS.
template <int C, int NVP>
struct AmTile {
    uint32_t a[C][4][2][256];  // conj(Gs) w^k: [c][k][high, low][lane * 4 + r], r = re 01, re 23, im 01, im 23
    float geo[C][AS_C];        // the sub-tile's row of the geometry table
    float dd[C][256];          // D_c(nu) - D_c(centre), for the term-by-term entries
    int rel[C];                // exponent of the wavelength's Gs less the largest
    int ex[NVP];               // exponent of each sum
    __device__ __forceinline__ double d0(int c) const { return *reinterpret_cast<const double *>(&geo[c][32]); }
};

template <int C, bool DEPTH>
__global__ void __launch_bounds__(AM_T, DEPTH || C > 3 ? 2 : 3)
    k_adjoint_mfma(Consts k, const int32_t *__restrict__ tile_xy, const BwdScene *__restrict__ scenes,
                   const int32_t *__restrict__ prefix, int n_scenes, long long *__restrict__ queue, const float *__restrict__ sgeo, AdjGeom geo)
{
    constexpr int NV = adj_nv(C, DEPTH), NVP = (NV + 3) & ~3;
    __shared__ __attribute__((aligned(16))) AmTile<C, NVP> s_t;
    __shared__ float s_acc[ADJ_MFMA_G * NV];
    __shared__ uint16_t s_perm[ADJ_MFMA_G];         // Gaussians in class order
    __shared__ uint16_t s_tlist[ADJ_MFMA_G];        // those that reach the tile
    __shared__ uint16_t s_list[3][ADJ_MFMA_G];      // accepted: separable from the front, others from the back
    __shared__ int s_cnt[3], s_dcnt[3], s_next[3], s_tcnt[3], s_hist[8];
    __shared__ int s_item, s_scene;

    const int tid = threadIdx.x, lane = tid & 63;
    const int total_items = prefix[n_scenes];
    const int hx = k.nx / 2, hy = k.ny / 2;
    const float lim = uniform_f((float)(k.tau2 * (1.0 + 1e-5)) + 1e-4f);
    const float mrxf = uniform_f((float)k.mrx), mryf = uniform_f((float)k.mry);

    bool first = true;
    for (;;) {
        if (tid == 0) {
            const int q = next_item(first, queue);
            int sc = 0;
            if (q < total_items)
                while (sc + 1 < n_scenes && prefix[sc + 1] <= q) ++sc;
            s_item = q;
            s_scene = sc;
        }
        first = false;
        if (tid < 8) s_hist[tid] = 0;
        if (tid < 3) s_cnt[tid] = s_dcnt[tid] = s_next[tid] = s_tcnt[tid] = 0;
        __syncthreads();
        const int q = __builtin_amdgcn_readfirstlane(s_item), sc = __builtin_amdgcn_readfirstlane(s_scene);
        if (q >= total_items) break;
        const BwdScene &S = scenes[sc];
        const GRec *__restrict__ rec = S.rec;
        const float4 *__restrict__ poly = adj_poly(rec, S.n);
        const int64_t nvalid = S.n - S.counters[CTR_NCULLED];
        const BItem bi = S.bitems[q - prefix[sc]];
        const int CH = __builtin_amdgcn_readfirstlane(S.chunk);  // ADJ_MFMA_G at most
        const int64_t g0 = (int64_t)bi.chunk * CH;
        const int ng = (int)min((int64_t)CH, nvalid - g0);
        int pairs = 0;
        for (int i = tid; i < CH * NV; i += AM_T) s_acc[i] = 0.0f;
        // order by class (7 first)
        int cc[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int o = tid + r * AM_T;
            cc[r] = 7;
            if (o < ng) {
                const int cls = cross_class(fabsf(rec[g0 + o].beta2) * MM_A_OF_BETA2);
                cc[r] = cls ? 7 - cls : 5;
                atomicAdd(&s_hist[cc[r]], 1);
            }
        }
        __syncthreads();
        if (tid == 0) {
            int run = 0;
            for (int i = 0; i < 8; ++i) {
                const int c = s_hist[i];
                s_hist[i] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (cc[r] < 7) s_perm[atomicAdd(&s_hist[cc[r]], 1)] = (uint16_t)(tid + r * AM_T);
        __syncthreads();
        int par = 0, tpar = 0;
        const int k0t = __builtin_amdgcn_readfirstlane(bi.k0), k1t = __builtin_amdgcn_readfirstlane(bi.k1);
        for (int kt = k0t; kt < k1t; ++kt) {
            const int32_t txy = __builtin_amdgcn_readfirstlane(tile_xy[kt]);
            const int tx = (int)(int16_t)(txy & 0xffff), ty = txy >> 16;
            {
                // the Gaussians that reach the 32 x 64 tile (every later test is only theirs)
                const int tv = here_v(tid);
                const float x0 = (float)max(tx * TILEX, -hx) - mrxf, x1 = (float)min(tx * TILEX + TILEX - 1, hx - 1) - mrxf;
                const float y0 = (float)max(ty * ADJ_RH, -hy) - mryf, y1 = (float)min(ty * ADJ_RH + ADJ_RH - 1, hy - 1) - mryf;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    bool hit = false;
                    int o = 0;
                    if (tv + r * AM_T < ng) {
                        o = s_perm[tv + r * AM_T];
                        const float4_t r0 = load4(rec + g0 + o);
                        hit = ellipse_meets_rect_r(r0.x, r0.y, r0.z, 0.5f * __builtin_amdgcn_rcpf(r0.x),
                                                   0.5f * __builtin_amdgcn_rcpf(r0.z), lim, x0, x1, y0, y1);
                    }
                    const uint64_t bh = __ballot(hit);
                    int at = 0;
                    if (lane == 0 && bh) at = atomicAdd(&s_tcnt[tpar], __popcll(bh));
                    at = __builtin_amdgcn_readfirstlane(at);
                    if (hit) s_tlist[at + rank_below(bh)] = (uint16_t)o;
                }
            }
            __syncthreads();
            const int tcnt = __builtin_amdgcn_readfirstlane(s_tcnt[tpar]);
            // the previous tile's counter, used again two tiles from now
            if (tid == 0) s_tcnt[tpar == 0 ? 2 : tpar - 1] = 0;
            tpar = tpar == 2 ? 0 : tpar + 1;
            if (tcnt == 0) continue;  // uniform
        for (int st = 0; st < 8; ++st) {
            const int sx0 = tx * TILEX + (st & 1) * 16, sy0 = ty * ADJ_RH + (st >> 1) * 16;
            if (sx0 >= hx || sx0 + 16 <= -hx || sy0 >= hy || sy0 + 16 <= -hy) continue;  // uniform
            const int sub = sub_index(geo, tx, ty, st & 1, st >> 1);
            const float *srow = sgeo + (int64_t)sub * adj_sub_floats(C);
            {
                int sx = sx0, sy = sy0;
                asm volatile("" : "+s"(sx), "+s"(sy));
                const float phimax = srow[1];
                const bool spike = S.gexp[sub * (C + 1) + C] != 0;
                const float zlim = spike ? -1.0f : srow[0];  // |z| beyond it: term by term
                const float x0 = (float)max(sx, -hx) - mrxf, x1 = (float)min(sx + 15, hx - 1) - mrxf;
                const float y0 = (float)max(sy, -hy) - mryf, y1 = (float)min(sy + 15, hy - 1) - mryf;
                const float xe = (float)sx + 7.5f - mrxf, ye = (float)sy + 7.5f - mryf;
                const int tv = here_v(tid);
                for (int i0 = 0; i0 < tcnt; i0 += AM_T) {
                    bool hit = false, sep = false;
                    int o = 0;
                    if (i0 + tv < tcnt) {
                        o = s_tlist[i0 + tv];
                        const float4_t r0 = load4(rec + g0 + o);
                        hit = ellipse_meets_rect_r(r0.x, r0.y, r0.z, 0.5f * __builtin_amdgcn_rcpf(r0.x),
                                                   0.5f * __builtin_amdgcn_rcpf(r0.z), lim, x0, x1, y0, y1);
                        // the separable form's limits (see k_accum_mfma.hip)
                        const float ex = fmaf(r0.x, MM_P, fabsf(fmaf(2.0f * r0.x, xe, r0.y * ye)) * 7.5f);
                        const float ey = fmaf(r0.z, MM_P, fabsf(fmaf(2.0f * r0.z, ye, r0.y * xe)) * 7.5f);
                        const float az = fabsf(r0.w), ph = az * phimax, aa = fabsf(r0.y) * MM_A_OF_BETA2;
                        sep = aa <= MM_A7 && fmaxf(ex, ey) <= 10.0f && az <= zlim && ph <= 2e-4f && ph * aa <= 1e-6f;
                    }
                    const uint64_t bs = __ballot(hit && sep), bd = __ballot(hit && !sep);
                    int at = 0, ad = 0;
                    if (lane == 0) {
                        if (bs) at = atomicAdd(&s_cnt[par], __popcll(bs));
                        if (bd) ad = atomicAdd(&s_dcnt[par], __popcll(bd));
                    }
                    at = __builtin_amdgcn_readfirstlane(at);
                    ad = __builtin_amdgcn_readfirstlane(ad);
                    if (hit) {
                        if (sep) s_list[par][at + rank_below(bs)] = (uint16_t)o;
                        else s_list[par][ADJ_MFMA_G - 1 - ad - rank_below(bd)] = (uint16_t)o;
                        pairs += 4;
                    }
                }
            }
            __syncthreads();  // the list is complete; the previous sub-tile is done with the tables
            const int cnt = __builtin_amdgcn_readfirstlane(s_cnt[par]), dcnt = __builtin_amdgcn_readfirstlane(s_dcnt[par]);
            const int cur = par, prev = par == 0 ? 2 : par - 1;
            par = par == 2 ? 0 : par + 1;
            // the previous sub-tile's counters, used again two sub-tiles from now
            if (tid == 0) s_cnt[prev] = s_dcnt[prev] = s_next[prev] = 0;
            if (cnt + dcnt == 0) continue;  // uniform
            // exponents of the wavelengths' Gs (-1000: all zero) and the largest of them
            int et[C], etm = -1000;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                et[c] = __builtin_amdgcn_readfirstlane(S.gexp[sub * (C + 1) + c]);
                etm = max(etm, et[c]);
            }
            {
                const float2 *gs = S.gpack + (int64_t)sub * C * 256;
                const int tv = here_v(tid);
                for (int i = tv; i < C * 128; i += AM_T) {
                    const int c = i >> 7, u = i & 15, vp = (i >> 4) & 7;
                    int e = et[0];
#pragma unroll
                    for (int q = 1; q < C; ++q) e = c == q ? et[q] : e;
                    const int ng = AM_GS - e;
                    const float2_t p = load2(gs + c * 256 + 32 * vp + u), p2 = load2(gs + c * 256 + 32 * vp + 16 + u);
                    float r0 = ldexpf(p.x, ng), i0 = ldexpf(p.y, ng);
                    float r1 = ldexpf(p2.x, ng), i1 = ldexpf(p2.y, ng);
                    const float w0 = ((float)(2 * vp) - 7.5f) * (1.0f / 7.5f), w1 = ((float)(2 * vp) - 6.5f) * (1.0f / 7.5f);
                    const int at = (u + 16 * (vp >> 1)) * 4 + (vp & 1);
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        const half2_t hr = to_half2(r0, r1), hi = to_half2(i0, i1);
                        const float2_t lr = rest(r0, r1, hr), li = rest(i0, i1, hi);
                        s_t.a[c][o][0][at] = bits(hr);
                        s_t.a[c][o][0][at + 2] = bits(hi);
                        s_t.a[c][o][1][at] = half_pair(lr.x, lr.y);
                        s_t.a[c][o][1][at + 2] = half_pair(li.x, li.y);
                        r0 *= w0;
                        i0 *= w0;
                        r1 *= w1;
                        i1 *= w1;
                    }
                }
                if (tv < NVP) {
                    // sums of one wavelength have its exponent, those over all the largest
                    const int c = tv < C ? tv : (DEPTH && tv >= C + 5 ? (tv - 5) % C : C);
                    int e = etm;
#pragma unroll
                    for (int q = 0; q < C; ++q) e = c == q ? et[q] : e;
                    s_t.ex[tv] = e - AM_GS - AM_YS;
                    if (tv < C) s_t.rel[tv] = e - etm;
                }
                for (int i = tv; i < C * AS_C; i += AM_T) (&s_t.geo[0][0])[i] = srow[AS_HEAD + i];
                if (dcnt) {
                    int sx = sx0, sy = sy0;
                    asm volatile("" : "+s"(sx), "+s"(sy));
                    const double iWx = 1.0 / (k.nx * k.px), iWy = 1.0 / (k.ny * k.py);
                    const double nux = (sx + (tv & 15)) * iWx, nuy = (sy + (tv >> 4)) * iWy;
#pragma unroll 1
                    for (int c = 0; c < C; ++c) {
                        const double il = k.inv_lambda[c], D0 = *reinterpret_cast<const double *>(srow + AS_HEAD + AS_C * c + 32);
                        s_t.dd[c][tv] = (float)(dprop_m(fmin(nux * nux + nuy * nuy, il * il), il) - D0);
                    }
                }
            }
            __syncthreads();
            const int ngrp = (cnt + 15) >> 4;
            for (;;) {
                int un = 0;
                if (lane == 0) un = atomicAdd(&s_next[cur], 1);
                un = __builtin_amdgcn_readfirstlane(un);
                if (un >= ngrp + dcnt) break;
                const int ln = here_v(lane), g = ln >> 4;
                // opaque copies: uniform values are formed where they are used rather than held in vector
                // registers across the passes
                int sx = sx0, sy = sy0;
                asm volatile("" : "+s"(sx), "+s"(sy));
                if (un < ngrp) {
                    const int li = un * 16 + (ln & 15);
                    const bool on = li < cnt;
                    const int o = s_list[cur][on ? li : un * 16];
                    const GRec *rp = rec + g0 + o;
                    const float4_t r0 = load4(rp), r1 = load4(&rp->rx), kap = load4(rp->kappa), amv = load4(rp->amp);
                    const float a = r0.y * MM_A_OF_BETA2, z = r0.w;
                    const int cls = cross_class(fabsf(a));
                    const float4_t co = load4(poly + g0 + o);  // c1 / c0, c2 / c0, c3 / c0, c0
                    const int R = __ballot(cls == 7) ? 6 : (__ballot(cls >= 5) ? 5 : (__ballot(cls == 4) ? 4 : 3));
                    // c4 and c5 follow from c3, zero beyond the Gaussian's own class
                    const float a4 = cls > 4 ? a : 0.0f, a5 = cls == 7 ? a : 0.0f;
                    // q at the centre and its gradient, the phase base: FP64
                    float lx, ly, e0, base[C];
                    {
                        const double xe = sx + 7.5 - k.mrx, ye = sy + 7.5 - k.mry;
                        const double ax = (double)r0.x * xe, gy = (double)r0.z * ye, b2 = r0.y;
                        const double q0 = fmin(xe * (ax + b2 * ye) + gy * ye, 1e6), qr = rint(q0);
                        lx = (float)(2.0 * ax + b2 * ye);
                        ly = (float)(2.0 * gy + b2 * xe);
                        e0 = on ? co.w * ldexpf(__builtin_amdgcn_exp2f((float)(qr - q0)), -(int)qr) : 0.0f;
                        const int cx = sx + 8, cy = sy + 8;
                        const uint32_t ramp = (uint32_t)cx * __float_as_uint(r1.x) + (uint32_t)cy * __float_as_uint(r1.y);
                        const double ramp_rev = (double)ramp * (1.0 / 4294967296.0);
                        const float kv[4] = {kap.x, kap.y, kap.z, kap.w};
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            if (k.phase_mode == 1) {
                                const float v = kv[c] - ((float)cx * r1.z + (float)cy * r1.w) - z * (float)s_t.d0(c);
                                base[c] = v - floorf(v);
                            } else {
                                base[c] = (float)frac_m((double)kv[c] - ramp_rev - (double)z * s_t.d0(c));
                            }
                        }
                    }
                    const float u0 = (float)(4 * g) - 7.5f;
                    float Ex[4], Ey[4], tx[4], ty[4], e1[4], e2[4], e3[4];
                    {
                        const uint32_t rx = __float_as_uint(r1.x), ry = __float_as_uint(r1.y);
                        const float rxa = (float)(int32_t)(rx & 0xfffff000u) * 0x1p-32f, rxb = (float)(rx & 0xfffu) * 0x1p-32f;
                        const float rya = (float)(int32_t)(ry & 0xfffff000u) * 0x1p-32f, ryb = (float)(ry & 0xfffu) * 0x1p-32f;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float u = u0 + (float)j, d = u - 0.5f, w = u * (1.0f / 7.5f);
                            Ex[j] = e0 * __builtin_amdgcn_exp2f(-u * fmaf(r0.x, u, lx));
                            Ey[j] = __builtin_amdgcn_exp2f(fmaf(-u, fmaf(r0.z, u, ly), (float)AM_YS));
                            tx[j] = fmaf(d, rxb, __builtin_amdgcn_fractf(d * rxa));
                            ty[j] = fmaf(d, ryb, __builtin_amdgcn_fractf(d * rya));
                            e1[j] = co.x * w;
                            e2[j] = co.y * w * w;
                            e3[j] = co.z * w * w * w;
                        }
                    }
                    const uint32_t w01 = half_pair(u0 * (1.0f / 7.5f), (u0 + 1.0f) * (1.0f / 7.5f)),
                                   w23 = half_pair((u0 + 2.0f) * (1.0f / 7.5f), (u0 + 3.0f) * (1.0f / 7.5f));
                    // Gs_c is held on its own scale: the sums over wavelengths take it on the largest's
                    const float am[4] = {amv.x, amv.y, amv.z, amv.w};
                    float R0[4], I0[4], R1[4], I1[4], R2[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) R0[j] = I0[j] = R1[j] = I1[j] = R2[j] = 0.0f;
                    float x[NVP];
#pragma unroll
                    for (int i = 0; i < NVP; ++i) x[i] = 0.0f;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        __builtin_amdgcn_sched_barrier(0);  // one wavelength at a time: bounds the live registers
                        // B: (Yr, Yi, -Yr), high and low; the real part reads the first four registers,
                        // the imaginary part the last four
                        Frag6 bh, bl;
                        {
                            float yr[4], yi[4];
                            const float4_t gy = *reinterpret_cast<const float4_t *>(&s_t.geo[c][16 + 4 * g]);
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const float th = fmaf(-z, gy[j], -ty[j]);
                                yr[j] = Ey[j] * __builtin_amdgcn_cosf(th);
                                yi[j] = Ey[j] * __builtin_amdgcn_sinf(th);
                            }
                            split4(yr, yi, bh.r, bl.r);
                            bh.r[4] = bh.r[0] ^ 0x80008000u;
                            bh.r[5] = bh.r[1] ^ 0x80008000u;
                            bl.r[4] = bl.r[0] ^ 0x80008000u;
                            bl.r[5] = bl.r[1] ^ 0x80008000u;
                        }
                        // Z_0, Z_1, Z_2 take each W_k as it is formed
                        const float zp = z * s_t.geo[c][34] * (1.0f / 7.5f);
                        float4_t z0r, z0i, z1r, z1i, z2r, z2i;
                        Frag ah;
#pragma unroll
                        for (int o3 = 0; o3 < 4; ++o3) {
                            ah = *reinterpret_cast<const Frag *>(&s_t.a[c][o3][0][ln * 4]);
                            const Frag al = *reinterpret_cast<const Frag *>(&s_t.a[c][o3][1][ln * 4]);
                            float4_t wr = mfma16(ah, bh.im(), f4zero()), wi = mfma16(ah, bh.re(), f4zero());
                            wr = mfma16(al, bh.im(), wr);
                            wi = mfma16(al, bh.re(), wi);
                            wr = mfma16(ah, bl.im(), wr);
                            wi = mfma16(ah, bl.re(), wi);
                            if (o3 == 0) {
                                z0r = wr;
                                z0i = wi;
                            } else if (o3 == 1) {
                                // phi only reaches Z_0: in Z_1 its share is phi 7.5 / (2.6 |m_y|) of the sum, 2e-7 for
                                // |phi| <= 2e-4 where it is that large
                                z1r = wr;
                                z1i = wi;
                                fma4(z0r, e1, wr);
                                fma4(z0i, e1, wi);
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    const float ei = zp * (u0 + (float)j);
                                    z0r[j] = fmaf(-ei, wi[j], z0r[j]);
                                    z0i[j] = fmaf(ei, wr[j], z0i[j]);
                                }
                            } else if (o3 == 2) {
                                z2r = wr;
                                z2i = wi;
                                fma4(z0r, e2, wr);
                                fma4(z0i, e2, wi);
                                fma4(z1r, e1, wr);
                                fma4(z1i, e1, wi);
                            } else {
                                if (R > 3) {
                                    fma4(z0r, e3, wr);
                                    fma4(z0i, e3, wi);
                                }
                                fma4(z1r, e2, wr);
                                fma4(z1i, e2, wi);
                                fma4(z2r, e1, wr);
                                fma4(z2i, e1, wi);
                            }
                        }
                        float ek[4], el[4], em[4];  // e_k, e_(k-1), e_(k-2)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            ek[j] = e3[j] * a4 * (u0 + (float)j) * (-1.0f / 30.0f);
                            el[j] = e3[j];
                            em[j] = e2[j];
                        }
#pragma unroll
                        for (int o3 = 4; o3 < AM_MAXW; ++o3) {
                            if (o3 > R + 1) break;
                            ah.r[0] = pk_mul(ah.r[0], w01);
                            ah.r[1] = pk_mul(ah.r[1], w23);
                            ah.r[2] = pk_mul(ah.r[2], w01);
                            ah.r[3] = pk_mul(ah.r[3], w23);
                            const float4_t wr = mfma16(ah, bh.im(), f4zero()), wi = mfma16(ah, bh.re(), f4zero());
                            if (o3 < R) {
                                fma4(z0r, ek, wr);
                                fma4(z0i, ek, wi);
                            }
                            if (o3 <= R) {
                                fma4(z1r, el, wr);
                                fma4(z1i, el, wi);
                            }
                            fma4(z2r, em, wr);
                            fma4(z2i, em, wi);
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                em[j] = el[j];
                                el[j] = ek[j];
                                ek[j] *= a5 * (u0 + (float)j) * (-1.0f / 37.5f);
                            }
                        }
                        const float4_t gx = *reinterpret_cast<const float4_t *>(&s_t.geo[c][4 * g]);
                        const float amc = C > 1 ? ldexpf(am[c], s_t.rel[c]) : am[c];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float th = fmaf(-z, gx[j], base[c] - tx[j]);
                            const float Xr = Ex[j] * __builtin_amdgcn_cosf(th), Xi = Ex[j] * __builtin_amdgcn_sinf(th);
                            const float ar = amc * Xr, ai = amc * Xi;
                            x[c] = fmaf(-Xi, z0i[j], fmaf(Xr, z0r[j], x[c]));
                            if constexpr (DEPTH) {
                                const float p0i = fmaf(Xr, z0i[j], Xi * z0r[j]), p1i = fmaf(Xr, z1i[j], Xi * z1r[j]);
                                const float p2i = fmaf(Xr, z2i[j], Xi * z2r[j]);
                                x[C + 5 + c] += p0i;
                                x[2 * C + 5 + c] = fmaf(gx[j], p0i, fmaf(s_t.geo[c][35], p1i, fmaf(s_t.geo[c][36], p2i, x[2 * C + 5 + c])));
                            }
                            R0[j] = fmaf(-ai, z0i[j], fmaf(ar, z0r[j], R0[j]));
                            I0[j] = fmaf(ai, z0r[j], fmaf(ar, z0i[j], I0[j]));
                            R1[j] = fmaf(-ai, z1i[j], fmaf(ar, z1r[j], R1[j]));
                            I1[j] = fmaf(ai, z1r[j], fmaf(ar, z1i[j], I1[j]));
                            R2[j] = fmaf(-ai, z2i[j], fmaf(ar, z2r[j], R2[j]));
                            // taken here, not after the last wavelength (Z of every wavelength would stay live)
                            asm volatile("" : "+v"(R0[j]), "+v"(I0[j]), "+v"(R1[j]), "+v"(I1[j]), "+v"(R2[j]));
                        }
                        if constexpr (DEPTH) x[2 * C + 5 + c] = fmaf((float)s_t.d0(c), x[C + 5 + c], x[2 * C + 5 + c]);
                    }
                    {
                        float r0s = 0.0f, ru = 0.0f, ruu = 0.0f, i0s = 0.0f, iu = 0.0f, r1s = 0.0f, ruv = 0.0f, i1s = 0.0f, r2s = 0.0f;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float u = u0 + (float)j;
                            r0s += R0[j];
                            ru = fmaf(u, R0[j], ru);
                            ruu = fmaf(u * u, R0[j], ruu);
                            i0s += I0[j];
                            iu = fmaf(u, I0[j], iu);
                            r1s += R1[j];
                            ruv = fmaf(u, R1[j], ruv);
                            i1s += I1[j];
                            r2s += R2[j];
                        }
                        r1s *= 7.5f;
                        ruv *= 7.5f;
                        const float xe = (float)(sx + 7.5 - k.mrx), ye = (float)(sy + 7.5 - k.mry);
                        x[C + 0] = fmaf(xe, i0s, iu);
                        x[C + 1] = fmaf(ye, i0s, 7.5f * i1s);
                        x[C + 2] = fmaf(xe, fmaf(xe, r0s, 2.0f * ru), ruu);
                        x[C + 3] = fmaf(ye, fmaf(xe, r0s, ru), fmaf(xe, r1s, ruv));
                        x[C + 4] = fmaf(ye, fmaf(ye, r0s, 2.0f * r1s), 56.25f * r2s);
                        if constexpr (!DEPTH) x[C + 5] = i0s;
                    }
                    // sums over the four lane groups: register i of lane l then holds value
                    // (NVP / 4) (2 b5 + b4) + i.  The powers of two of Gs and Y come back last: in X they would take
                    // the factors of a small Gs out of FP32's normal range long before the sums
#pragma unroll
                    for (int i = 0; i < NVP / 2; ++i) {
                        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + NVP / 2]), false, false);
                        x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
                    }
                    const int v0 = (NVP / 4) * (here_v(lane) >> 4);
#pragma unroll
                    for (int i = 0; i < NVP / 4; ++i) {
                        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i + NVP / 4]), false, false);
                        x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
                        const int v = v0 + i;
                        if (on && v < NV) atomicAdd(&s_acc[o * NV + v], ldexpf(x[i], s_t.ex[v]));  // ds_add_f32, no return
                    }
                } else {
                    // term by term: lane l takes column l % 16 and rows l / 16 + 4 f
                    const int o = __builtin_amdgcn_readfirstlane((int)s_list[cur][ADJ_MFMA_G - 1 - (un - ngrp)]);
                    const GRec *rp = rec + g0 + o;
                    const float4_t r0 = load4(rp), r1 = load4(&rp->rx), kap = load4(rp->kappa), amv = load4(rp->amp);
                    const float kv[4] = {kap.x, kap.y, kap.z, kap.w}, am[4] = {amv.x, amv.y, amv.z, amv.w};
                    const int cx = sx + 8, cy = sy + 8, col = ln & 15;
                    const uint32_t ramp = (uint32_t)cx * __float_as_uint(r1.x) + (uint32_t)cy * __float_as_uint(r1.y);
                    const double ramp_rev = (double)ramp * (1.0 / 4294967296.0);
                    const float fmx = (float)((double)(sx + col) - k.mrx);
                    const float2 *gs = S.gpack + (int64_t)sub * C * 256;
                    float x[NV];
#pragma unroll
                    for (int i = 0; i < NV; ++i) x[i] = 0.0f;
#pragma unroll 1
                    for (int f = 0; f < 4; ++f) {
                        const int row = g + 4 * f;
                        const float my = (float)((double)(sy + row) - k.mry);
                        const float E = __builtin_amdgcn_exp2f(-fmaf(my, fmaf(r0.z, my, r0.y * fmx), r0.x * fmx * fmx));
                        float rr = 0.0f, ri = 0.0f;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            float bs;
                            if (k.phase_mode == 1) {
                                const float v = kv[c] - ((float)cx * r1.z + (float)cy * r1.w) - r0.w * (float)s_t.d0(c);
                                bs = v - floorf(v);
                            } else {
                                bs = (float)frac_m((double)kv[c] - ramp_rev - (double)r0.w * s_t.d0(c));
                            }
                            const float dD = s_t.dd[c][row * 16 + col];
                            const float2_t gv = load2(gs + c * 256 + row * 16 + col);
                            const float bx = __builtin_amdgcn_fractf(fmaf(-(float)(col - 8), r1.z, bs));
                            const float th = fmaf(-r0.w, dD, fmaf(-(float)(row - 8), r1.w, bx));
                            const float cs = E * __builtin_amdgcn_cosf(th), sn = E * __builtin_amdgcn_sinf(th);
                            const float pr = fmaf(gv.x, cs, gv.y * sn), pi = fmaf(gv.x, sn, -gv.y * cs);
                            x[c] += pr;
                            if constexpr (DEPTH) {
                                x[C + 5 + c] += pi;
                                x[2 * C + 5 + c] = fmaf((float)s_t.d0(c) + dD, pi, x[2 * C + 5 + c]);
                            }
                            rr = fmaf(am[c], pr, rr);
                            ri = fmaf(am[c], pi, ri);
                        }
                        x[C + 0] = fmaf(fmx, ri, x[C + 0]);
                        x[C + 1] = fmaf(my, ri, x[C + 1]);
                        x[C + 2] = fmaf(fmx * fmx, rr, x[C + 2]);
                        x[C + 3] = fmaf(fmx * my, rr, x[C + 3]);
                        x[C + 4] = fmaf(my * my, rr, x[C + 4]);
                        if constexpr (!DEPTH) x[C + 5] += ri;
                    }
                    reduce_into<NV>(x, s_acc + o * NV, lane);
                }
            }
        }
        }
        __syncthreads();
        const int chunk = __builtin_amdgcn_readfirstlane(S.chunk);
        float *dst = S.bpartials + (int64_t)bi.slot * chunk * NV;
        for (int i = tid; i < chunk * NV; i += AM_T) dst[i] = s_acc[i];
        const long long np = wave_sum_i64((long long)pairs) * 64;
        if (lane == 0 && np) atomicAdd((unsigned long long *)&S.counters[CTR_PAIRS], (unsigned long long)np);
        __syncthreads();  // s_acc and the counters are free again
    }
}

template <int C, bool DEPTH>
static const void *adj_mfma_ptr() { return (const void *)k_adjoint_mfma<C, DEPTH>; }

hipError_t launch_adjoint_mfma(const Plan &p, const Consts &k, const BwdScene *scenes, const int32_t *prefix, int n_scenes,
                               long long *queue, const float *sgeo, const AdjGeom &geo, int grid, hipStream_t s)
{
#define GWS_AM(CC, DD)                                                                                            \
    hipLaunchKernelGGL((k_adjoint_mfma<CC, DD>), dim3(grid), dim3(AM_T), 0, s, k, p.tile_xy, scenes, prefix, n_scenes, \
                       queue, sgeo, geo)
    const bool d = k.depth_grad != 0;
    switch (k.C) {
    case 1: if (d) GWS_AM(1, true); else GWS_AM(1, false); break;
    case 2: if (d) GWS_AM(2, true); else GWS_AM(2, false); break;
    case 3: if (d) GWS_AM(3, true); else GWS_AM(3, false); break;
    case 4: if (d) return hipErrorInvalidValue; else GWS_AM(4, false); break;
    default: return hipErrorInvalidValue;
    }
#undef GWS_AM
    return hipGetLastError();
}

int adjoint_mfma_occupancy(int C, int depth)
{
    const void *kp = nullptr;
    switch (C) {
    case 1: kp = depth ? adj_mfma_ptr<1, true>() : adj_mfma_ptr<1, false>(); break;
    case 2: kp = depth ? adj_mfma_ptr<2, true>() : adj_mfma_ptr<2, false>(); break;
    case 3: kp = depth ? adj_mfma_ptr<3, true>() : adj_mfma_ptr<3, false>(); break;
    default: kp = adj_mfma_ptr<4, false>(); break;
    }
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kp, AM_T, 0) != hipSuccess || nb < 1) nb = 1;
    return nb;
}

}  // namespace gws
