// Spectrum accumulation on the matrix cores (gfx950): the sum of k_accum.hip,
//   S_c[m] = sum_i A_{c,i} exp2(-q_i(m)) exp(j 2 pi Theta_{c,i}(m)),
// for grids on which most terms are separable over a 16 x 16 sub-tile of frequencies.
//
// What bounds the term-by-term kernel is VALU issue: 17 plain and 7 transcendental
// instructions per 64 (Gaussian, frequency) pairs at three wavelengths.  On a sub-tile of
// 16 x 16 frequencies, with u, v the offsets from its centre (-7.5 ... 7.5) and t = u v / 56.25,
// a term is X(u) Y(v) exp(-(a + j phi_c) t), where a = 56.25 ln2 beta2 comes from the
// covariance's cross term and phi_c from the (small) cross derivative of k_z; the rest of
// k_z's variation splits into a function of u plus one of v up to third derivatives, which
// a bound per sub-tile checks.  exp(-a t) is a polynomial in t, and t does not depend on the
// Gaussian, so with c_k(a) its coefficients
//   S(u, v) = sum_k t^k M_k(u, v),   M_k = sum_i [c_k(a_i) X_i(u)] Y_i(v):
// complex outer products summed over Gaussians -- a matrix product with the Gaussians as the
// contraction index.  Per (Gaussian, sub-tile) only 16 + 16 complex factors are evaluated per
// wavelength instead of 256 terms, and the products run on v_mfma_f32_16x16x32_f16.
// Orders 2 and up, small, fold u and v into their fp16 factors and share M_1.
//
// Precision.  Each FP32 factor is split into two fp16 numbers, both rounded to nearest
// (x = h + l, |x - h - l| <= 2^-23 |x| while l is a normal fp16 number, 2^-25 where it is not: below
// |x| = 2^-2 at the latest, against a strongest factor of about 2^4), the products h h, h l and l h
// are accumulated in FP32 (l l is at most 2^-22 of h h).  fp16's range is met by exact powers of two: the
// running exponent e of the wavelength's largest term met so far is taken out of the factors
// (accumulators are rescaled when it grows) and factors are kept in 2^+-15.  The polynomial is the Taylor
// polynomial with the next two orders projected onto it by least squares over the
// sub-tile's 256 points: relative rms error at most 1e-7 for |a| <= 0.0175, 0.08, 0.2, 0.35 with
// 3, 4, 5, 6 coefficients (2.4e-7 for one of five at |a| = 0.2 that shares a pass with six, whose
// sixth it then takes besides its projection).  q at the centre, its gradient and the phase base are formed in FP64
// by the staging lane, and the ramp m . r is exact.  Spectrum error against FP64, 40 Gaussians at
// 2400 x 1800 x 2: 3.4e-7 (6.0e-7 term by term); 1e6 at 2160 x 3840 x 3: 1.4e-6 (4.5e-6).
//
// A Gaussian that fails a test on a sub-tile (a too large, a steep envelope, a deep Gaussian
// where k_z curves fast, a nearly singular covariance, non-finite amplitude) is evaluated term by term into the same
// accumulators there (lane l of the MFMA result holds column l % 16 and rows l / 16 + 4 f, the
// term-by-term kernel's own layout).
//
// Layout.  v_mfma_f32_16x16x32_f16 takes row l % 16 of A and column l % 16 of B from lane l,
// eight consecutive k per 16-lane group.  k runs over (re / im, Gaussian): lane l evaluates
// X at column l % 16 and Y at row l % 16 of the four Gaussians l / 16 + 4 j, so the operands
// are formed in the lanes that feed them, with no exchange between lanes.  One pass takes 16
// Gaussians; what does not fill a pass stays in the wavefront's list for the next batch.
//
// Bound now: VALU issue (91 % of the busy cycles; the matrix units 23 %), 41 VALU instructions per
// (Gaussian, sub-tile) at three wavelengths, a fifth of them staging, against 146 term by
// term.  Forward of 1e6 at 2160 x 3840 x 3: 304 -> 120 ms; 3e5 at one wavelength 15.5 ms.  Three
// wavefronts per SIMD with seven registers spilt, outside the passes; accumulators for t^2 too
// would spill inside them.
#include "mfma_f16.h"

namespace gws {

constexpr int MF = 4;                    // 4-row blocks (and result registers) of a sub-tile
constexpr int MM_CAND = 1024;            // candidates tested per round
constexpr int MM_SLOTS = 96;             // a wavefront's list: up to 15 entries kept, 64 new, padding to 16
constexpr int MM_XS = 4, MM_YS = 5;      // powers of two carried by X and Y (kept inside fp16's normal range)
constexpr int MM_E_NONE = -100000;       // so far only zeros, which any power of two leaves
constexpr int MM_SLACK = 80;             // powers of two by which a term-by-term term may exceed the running exponent
constexpr int MM_EMIT = 32;              // passes after which a round's end moves the accumulators to the output

// An entry of a wavefront's list, 12 + 4 C floats.  Separable: lx, alpha, ly, gamma | r_x's upper
// 20 bits and the rest, r_y's | c1, 8 c2 / P, 8 c3 / c2 / P, 8 c4 / c3 / P | per wavelength base, A,
// c1 imaginary, z.  Term by term: alpha, beta2, gamma, z | rxf, ryf, rows, - |
// -- | per wavelength base, amp, -, -.
__host__ __device__ constexpr int mm_floats(int c) { return 12 + 4 * c; }

// The four Gaussians' factors times m0 ... m3.
static __device__ __forceinline__ void scale_pair(Frag &b, float m0, float m1, float m2, float m3)
{
    const uint32_t p = half_pair(m0, m1), q = half_pair(m2, m3);
    b.r[0] = pk_mul(b.r[0], p);
    b.r[1] = pk_mul(b.r[1], q);
    b.r[2] = pk_mul(b.r[2], p);
    b.r[3] = pk_mul(b.r[3], q);
}

template <int C>
struct MAcc {
    float4_t re[2][C], im[2][C];
};

// Per-lane constants of a sub-tile.
template <int C>
struct MLane {
    float u, v;            // column and row offset of the lane's X and Y factors
    float dx, dy;          // the same from the integer centre of the ramp
    float gx[C], gy[C];    // k_z along the sub-tile's central row and column, minus its centre's
};

// 16 separable Gaussians (entries first ... first + 15), evaluated as class R.
template <int C>
static __device__ __forceinline__ void mm_pass(const float (&ent)[MM_SLOTS][mm_floats(C)], int first, int R, int lane,
                                               const MLane<C> &L, MAcc<C> &M)
{
    const float(*e)[mm_floats(C)] = &ent[first + (lane >> 4)];
    float Ex[4], Ey[4], tx[4], ty[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float4_t e0 = *reinterpret_cast<const float4_t *>(&e[4 * j][0]);
        const float4_t e1 = *reinterpret_cast<const float4_t *>(&e[4 * j][4]);
        Ex[j] = __builtin_amdgcn_exp2f(-L.u * fmaf(e0.y, L.u, e0.x));
        Ey[j] = __builtin_amdgcn_exp2f(fmaf(-L.v, fmaf(e0.w, L.v, e0.z), (float)MM_YS));
        // the ramp m . r of the lane's column / row modulo 1: the product with r's upper 20 bits and
        // its fraction are exact
        tx[j] = fmaf(L.dx, e1.y, __builtin_amdgcn_fractf(L.dx * e1.x));
        ty[j] = fmaf(L.dy, e1.w, __builtin_amdgcn_fractf(L.dy * e1.z));
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        __builtin_amdgcn_sched_barrier(0);  // one wavelength's factors at a time: bounds the live registers
        Frag6 ah, al;
        Frag bh, bl, ch, cl;
        float Xr[4], Xi[4], Yr[4], Yi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4_t ec = *reinterpret_cast<const float4_t *>(&e[4 * j][12 + 4 * c]);
            const float thx = fmaf(-ec.w, L.gx[c], ec.x - tx[j]), thy = fmaf(ec.w, L.gy[c], ty[j]);
            const float ax = ec.y * Ex[j];
            Xr[j] = ax * __builtin_amdgcn_cosf(thx);
            Xi[j] = ax * __builtin_amdgcn_sinf(thx);
            // the conjugate of Y: Re = Xr Yr + Xi Yi, Im = Xi Yr - Xr Yi
            Yr[j] = Ey[j] * __builtin_amdgcn_cosf(thy);
            Yi[j] = Ey[j] * __builtin_amdgcn_sinf(thy);
        }
        split4(Yr, Yi, ah.r + 2, al.r + 2);
        ah.r[0] = ah.r[4] ^ 0x80008000u;
        ah.r[1] = ah.r[5] ^ 0x80008000u;
        al.r[0] = al.r[4] ^ 0x80008000u;
        al.r[1] = al.r[5] ^ 0x80008000u;
        split4(Xr, Xi, bh.r, bl.r);
        M.re[0][c] = mfma16(ah.re(), bh, M.re[0][c]);
        M.im[0][c] = mfma16(ah.im(), bh, M.im[0][c]);
        M.re[0][c] = mfma16(al.re(), bh, M.re[0][c]);
        M.im[0][c] = mfma16(al.im(), bh, M.im[0][c]);
        M.re[0][c] = mfma16(ah.re(), bl, M.re[0][c]);
        M.im[0][c] = mfma16(ah.im(), bl, M.im[0][c]);
        __builtin_amdgcn_sched_barrier(0);
        {
            float pr[4], pi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float cr = e[4 * j][8], ci = e[4 * j][14 + 4 * c];
                pr[j] = fmaf(Xr[j], cr, -Xi[j] * ci);
                pi[j] = fmaf(Xr[j], ci, Xi[j] * cr);
            }
            split4(pr, pi, ch.r, cl.r);
        }
        M.re[1][c] = mfma16(ah.re(), ch, M.re[1][c]);
        M.im[1][c] = mfma16(ah.im(), ch, M.im[1][c]);
        M.re[1][c] = mfma16(al.re(), ch, M.re[1][c]);
        M.im[1][c] = mfma16(al.im(), ch, M.im[1][c]);
        M.re[1][c] = mfma16(ah.re(), cl, M.re[1][c]);
        M.im[1][c] = mfma16(ah.im(), cl, M.im[1][c]);
        // c_k t^k = t (c_k u^(k-1)) (v^(k-1)), each order from the one before it, so only t^0 and
        // t^1 have accumulators.  Up to class 5 |c2| <= a^2 / 2 <= 7e-3 and one fp16 product is enough
        // (its relative error is 3e-4 of a term whose rms share is 0.2 c2); classes 6 and 7 keep both
        // parts.  |c3| <= a^3 / 6 <= 7e-3 and the orders above need one product; c5 / c4 is 4 / 5 of
        // c4 / c3 to the accuracy c5 t^5 (2e-6 at most in the mean) asks for.
        if (R < 6) {
            scale_pair(bh, e[0][9] * L.u, e[4][9] * L.u, e[8][9] * L.u, e[12][9] * L.u);
            const uint32_t v1 = half_pair(L.v * 0.125f, L.v * 0.125f);
#pragma unroll
            for (int i = 0; i < 6; ++i) ah.r[i] = pk_mul(ah.r[i], v1);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float m = e[4 * j][9] * L.u;
                asm volatile("" : "+v"(m));  // keeps this branch's products in the branch
                Xr[j] *= m;
                Xi[j] *= m;
            }
            split4(Xr, Xi, bh.r, bl.r);
            float yr[4], yi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float v8 = L.v * 0.125f;
                yr[j] = v8 * part(ah.r[2 + j / 2], j & 1) + v8 * part(al.r[2 + j / 2], j & 1);
                yi[j] = v8 * part(ah.r[4 + j / 2], j & 1) + v8 * part(al.r[4 + j / 2], j & 1);
            }
            split4(yr, yi, ah.r + 2, al.r + 2);
            ah.r[0] = ah.r[4] ^ 0x80008000u;
            ah.r[1] = ah.r[5] ^ 0x80008000u;
            al.r[0] = al.r[4] ^ 0x80008000u;
            al.r[1] = al.r[5] ^ 0x80008000u;
            M.re[1][c] = mfma16(al.re(), bh, M.re[1][c]);
            M.im[1][c] = mfma16(al.im(), bh, M.im[1][c]);
            M.re[1][c] = mfma16(ah.re(), bl, M.re[1][c]);
            M.im[1][c] = mfma16(ah.im(), bl, M.im[1][c]);
        }
        M.re[1][c] = mfma16(ah.re(), bh, M.re[1][c]);
        M.im[1][c] = mfma16(ah.im(), bh, M.im[1][c]);
        const uint32_t v1 = half_pair(L.v * 0.125f, L.v * 0.125f);
#pragma unroll
        for (int o = 3; o < 6; ++o) {
            if (o >= R || (o == 5 && R < 7)) break;
            const int w = o < 5 ? 7 + o : 11;
            const float uo = o < 5 ? L.u : 0.8f * L.u;
            scale_pair(bh, e[0][w] * uo, e[4][w] * uo, e[8][w] * uo, e[12][w] * uo);
#pragma unroll
            for (int i = 0; i < 6; ++i) ah.r[i] = pk_mul(ah.r[i], v1);
            M.re[1][c] = mfma16(ah.re(), bh, M.re[1][c]);
            M.im[1][c] = mfma16(ah.im(), bh, M.im[1][c]);
        }
    }
}

// Wavefronts per SIMD the kernel is compiled for (one wavelength: 3e5 Gaussians at 2160 x 3840 with four
// 15.5 ms, with three 16.7).
__host__ __device__ constexpr int mm_waves(int c) { return c == 1 ? 4 : c <= 3 ? 3 : 2; }

// Work items, tile order, chunks and partial-sum slots are k_accumulate's (F = 4).  Uniform values
// are taken through readfirstlane: held in vector registers they spilt the matrix passes.
template <int C>
__global__ void __launch_bounds__(WG, mm_waves(C)) k_accumulate_mfma(Consts k, const int32_t *__restrict__ tile_xy,
                                                           const FwdScene *__restrict__ scenes,
                                                           const int32_t *__restrict__ prefix, int n_scenes,
                                                           long long *__restrict__ queue)
{
    __shared__ __align__(16) float s_w[WAVES][MM_SLOTS][mm_floats(C)];
    __shared__ float s_dd[WAVES][MF][C][64];  // D_c(nu) - D_c(centre), for the term-by-term entries
    __shared__ int s_idx[MM_CAND];            // candidates that reach the tile, in order
    __shared__ double s_d0[WAVES][C];         // D_c at the sub-tile's centre
    __shared__ float s_phi[WAVES][C];         // -(c1's imaginary part) per metre of depth
    __shared__ int s_item, s_scene;
    __shared__ int s_cnt[MM_CAND / WG][WAVES];

    constexpr int TY = 2 * sub_h(MF);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int total_items = prefix[n_scenes];
    const int hx = k.nx / 2, hy = k.ny / 2;
    const float lim = uniform_f((float)(k.tau2 * (1.0 + 1e-5)) + 1e-4f);
    const float mrxf = uniform_f((float)k.mrx), mryf = uniform_f((float)k.mry);
    const int col = lane & (SUBX - 1), row0 = lane >> 4;
    const int yi = (col >> 2) + 4 * (col & 3);  // the row whose Y factor the lane forms: A row i is row i / 4 + 4 (i % 4)
    MLane<C> L;
    L.u = (float)col - 7.5f;
    L.v = (float)yi - 7.5f;
    L.dx = (float)(col - 8);
    L.dy = (float)(yi - 8);

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
        __syncthreads();
        const int gitem = __builtin_amdgcn_readfirstlane(s_item), scene = __builtin_amdgcn_readfirstlane(s_scene);
        __syncthreads();
        if (gitem >= total_items) break;
        const FwdScene &S = scenes[scene];
        const GRec *__restrict__ rec = S.rec;
        const Item it = S.items[gitem - prefix[scene]];
        const int slot = __builtin_amdgcn_readfirstlane(it.slot);
        const int CH = __builtin_amdgcn_readfirstlane((int)S.counters[CTR_CHUNK]);
        int pairs = 0;  // this item's evaluated pairs / 64, per lane
        const int32_t txy = __builtin_amdgcn_readfirstlane(tile_xy[it.tile]);
        const int tx = (int)(int16_t)(txy & 0xffff), ty = txy >> 16;
        const int c0 = __builtin_amdgcn_readfirstlane(it.chunk) * CH;
        const int c1 = min(c0 + CH, __builtin_amdgcn_readfirstlane(S.tile_L[it.tile]));
        const int sx0 = tx * TILEX + (wave & 1) * SUBX, sy0 = ty * TY + (wave >> 1) * SUBX;
        const bool wave_live = sx0 < hx && sx0 + SUBX > -hx && sy0 < hy && sy0 + SUBX > -hy;
        // k_z: along the central row and column (factors), the cross derivative (c1's imaginary
        // part), a bound of what is left (third derivatives, at the sub-tile's outer corner)
        float zlim = 3.4e38f, phimax = 0.0f;
        {
            const double iWx = 1.0 / (k.nx * k.px), iWy = 1.0 / (k.ny * k.py);
            const double xc = sx0 + 7.5, yc = sy0 + 7.5;
            const double nx0 = xc * iWx, ny0 = yc * iWy;
            const double xm = (fabs(xc) + 7.5) * iWx, ym = (fabs(yc) + 7.5) * iWy;
            const double nxu = (xc + L.u) * iWx, nyv = (yc + L.v) * iWy;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const double il = k.inv_lambda[c];
                // the centre can lie up to 7.5 indices beyond the grid, and there beyond the propagating disk:
                // any finite D0 will do then, every entry going term by term
                const double D0 = dprop_m(fmin(nx0 * nx0 + ny0 * ny0, il * il), il);
                s_d0[wave][c] = D0;
                const double wm = il * il - xm * xm - ym * ym;
                L.gx[c] = L.gy[c] = 0.0f;
                float phi = 0.0f;
                if (wm > 0.0) {
                    L.gx[c] = (float)(dprop_m(nxu * nxu + ny0 * ny0, il) - D0);
                    L.gy[c] = (float)(dprop_m(nx0 * nx0 + nyv * nyv, il) - D0);
                    // bounds and the (1e-3 at most) cross phase need no more than FP32
                    const float wf = (float)(il * il - nx0 * nx0 - ny0 * ny0), k3 = __builtin_amdgcn_rsqf((float)wm) / (float)wm;
                    phi = (float)(6.283185307179586 * 56.25 * nx0 * ny0 * iWx * iWy) * __builtin_amdgcn_rsqf(wf) / wf;
                    phimax = fmaxf(phimax, fabsf(phi));
                    const float k5 = 3.0f * k3 / (float)wm, xf = (float)xm, yf = (float)ym, fx = (float)iWx, fy = (float)iWy;
                    const float r = 1326.0f * fx * fy * (fx * yf * fmaf(k5 * xf, xf, k3) + fy * xf * fmaf(k5 * yf, yf, k3));
                    zlim = fminf(zlim, 1e-6f / r);
                } else {
                    zlim = -1.0f;  // the stencil leaves the propagating disk: every entry term by term
                }
                s_phi[wave][c] = phi;
            }
        }
        bool have_dd = false;
        MAcc<C> M;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c) M.re[r][c] = M.im[r][c] = (float4_t){0.0f, 0.0f, 0.0f, 0.0f};
        int erun[C];  // the accumulators of wavelength c hold sums times 2^(XS + YS - erun[c])
#pragma unroll
        for (int c = 0; c < C; ++c) erun[c] = MM_E_NONE;
        bool emitted = false;
        int npass = 0;  // passes in the accumulators
        int kept = 0, keptR = 3;  // entries of the list's front not yet evaluated (< 16), their class

        for (int base = c0; base < c1; base += MM_CAND) {
            // the candidates of this round that reach the tile, listed in order
            const int nr = min(MM_CAND / WG, (c1 - base + WG - 1) / WG);
            {
                const float X0 = (float)max(tx * TILEX, -hx) - mrxf, X1 = (float)min(tx * TILEX + TILEX - 1, hx - 1) - mrxf;
                const float Y0 = (float)max(ty * TY, -hy) - mryf, Y1 = (float)min(ty * TY + TY - 1, hy - 1) - mryf;
                uint64_t bal[MM_CAND / WG];
#pragma unroll
                for (int r = 0; r < MM_CAND / WG; ++r) {
                    const int gi = base + r * WG + tid;
                    bool pred = false;
                    if (r < nr && gi < c1) {
                        const float4_t r0 = load4(rec + gi);
                        pred = ellipse_meets_rect_r(r0.x, r0.y, r0.z, 0.5f * __builtin_amdgcn_rcpf(r0.x), 0.5f * __builtin_amdgcn_rcpf(r0.z),
                                             lim, X0, X1, Y0, Y1);
                    }
                    bal[r] = __ballot(pred);
                    if (lane == 0) s_cnt[r][wave] = __popcll(bal[r]);
                }
                __syncthreads();
                int off = 0;
#pragma unroll
                for (int r = 0; r < MM_CAND / WG; ++r)
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) {
                        if (w == wave && (bal[r] >> lane) & 1) s_idx[off + rank_below(bal[r])] = base + r * WG + tid;
                        off += s_cnt[r][w];
                    }
                if (tid == 0) s_item = off;
            }
            __syncthreads();
            const int total = __builtin_amdgcn_readfirstlane(s_item);
            const bool last = base + MM_CAND >= c1;
            for (int j0 = 0; wave_live && j0 < total; j0 += 64) {
                int cls = -1;  // -1 not on the sub-tile, 0 term by term, else the class of |a|
                int eq = 0, qi = 0;
                bool grows = false;
                float4_t r0 = {0.0f, 0.0f, 0.0f, 0.0f};
                float lx = 0.0f, ly = 0.0f, qf = 0.0f;  // gradient of q at the centre, q there = qi - qf
                const GRec *rp = rec + s_idx[min(j0 + lane, total - 1)];
                // the sub-tile's uniform values are formed again in every batch (opaque integers): held
                // across the matrix passes they would cost vector registers
                int sx = __builtin_amdgcn_readfirstlane(sx0), sy = __builtin_amdgcn_readfirstlane(sy0);
                asm volatile("" : "+s"(sx), "+s"(sy));
                const float x0 = (float)max(sx, -hx) - mrxf, x1 = (float)min(sx + SUBX - 1, hx - 1) - mrxf;
                const float y0 = (float)max(sy, -hy) - mryf, y1 = (float)min(sy + SUBX - 1, hy - 1) - mryf;
                if (j0 + lane < total) {
                    r0 = load4(rp);
                    const float4_t am = load4(rp->amp);
                    const float qmin = ellipse_min_q(r0.x, r0.y, r0.z, 0.5f * __builtin_amdgcn_rcpf(r0.x),
                                                     0.5f * __builtin_amdgcn_rcpf(r0.z), x0, x1, y0, y1);
                    if (qmin <= lim) {
                        const double xe = sx + 7.5 - k.mrx, ye = sy + 7.5 - k.mry;
                        const double ax = (double)r0.x * xe, gy = (double)r0.z * ye, b2 = r0.y;
                        const double q0 = fmin(xe * (ax + b2 * ye) + gy * ye, 1e6), qr = rint(q0);
                        qi = (int)qr;
                        qf = (float)(qr - q0);
                        lx = (float)(2.0 * ax + b2 * ye);
                        ly = (float)(2.0 * gy + b2 * xe);
                        const float aa = fabsf(r0.y) * MM_A_OF_BETA2, az = fabsf(r0.w);
                        const float ampmax = fmaxf(fmaxf(fabsf(am.x), fabsf(am.y)), fmaxf(fabsf(am.z), fabsf(am.w)));
                        const float ex = fmaf(r0.x, MM_P, fabsf(lx) * 7.5f), ey = fmaf(r0.z, MM_P, fabsf(ly) * 7.5f);
                        const float ph = az * phimax;
                        // near a singular covariance q is a small difference of large terms, and its
                        // rounding is part of the result: kept as the term-by-term kernel rounds it
                        const float ag4 = 4.0f * r0.x * r0.z;
                        const bool ok = fmaxf(ex, ey) <= 10.0f && az <= zlim && ph <= 1e-3f &&
                                        ph * aa <= 1e-6f && ampmax <= 1e30f && fmaf(-r0.y, r0.y, ag4) >= 0.04f * ag4;
                        cls = ok ? cross_class(aa) : 0;
                        // exponent of a separable entry's largest term, within 2^20: the one at the sub-tile's
                        // centre.  Any other entry is FP32 all through and only has to keep to its range: it
                        // asks for MM_SLACK less than its largest term (a steep envelope can fall by hundreds
                        // of powers of two from the sub-tile's edge to its centre), so that its factor
                        // 2^(XS + YS - erun) amp stays below 2^(8 + 32 + MM_SLACK)
                        eq = cls ? min(qi, 200) : (int)fminf(fmaxf(qmin, 0.0f), 32.0f) + MM_SLACK;
                        // a wavelength is a sum of its own, with a running exponent of its own: a faint one beside a
                        // strong one would otherwise lose its factors' low fp16 parts
#pragma unroll
                        for (int c = 0; c < C; ++c) grows |= fabsf(ldexpf(am[c], -eq - erun[c])) >= 1.0f;
                    }
                }
                const uint64_t b7 = __ballot(cls == 7), b6 = __ballot(cls == 6), b5 = __ballot(cls == 5), b4 = __ballot(cls == 4),
                               b3 = __ballot(cls == 3), bd = __ballot(cls == 0);
                if (__ballot(grows)) {
                    if (kept) {  // evaluated at the scale they were written for
                        if (lane < 16 - kept)
                            for (int i = 0; i < mm_floats(C); ++i) s_w[wave][kept + lane][i] = 0.0f;
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        mm_pass<C>(s_w[wave], 0, __builtin_amdgcn_readfirstlane(keptR), lane, L, M);
                        kept = 0;
                        keptR = 3;
                    }
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const float ac = rp->amp[c];
                        int ee = MM_E_NONE;
                        if (grows && __builtin_amdgcn_classf(ac, 0x198)) ee = __builtin_amdgcn_frexp_expf(ac) - eq;  // finite, not 0
#pragma unroll
                        for (int d = 32; d >= 1; d >>= 1) ee = max(ee, __shfl_xor(ee, d));
                        const int en = max(__builtin_amdgcn_readfirstlane(ee), erun[c]);
                        const float sc = erun[c] == MM_E_NONE ? 1.0f : ldexpf(1.0f, max(erun[c] - en, -200));
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            M.re[r][c] *= sc;
                            M.im[r][c] *= sc;
                        }
                        erun[c] = en;
                    }
                }
                const int n7 = kept + __popcll(b7), n6 = n7 + __popcll(b6), n5 = n6 + __popcll(b5), n4 = n5 + __popcll(b4), nf = n4 + __popcll(b3);
                const int nd = __popcll(bd);
                auto class_at = [&](int i) { return i < n7 ? 7 : i < n6 ? 6 : (i < n5 ? 5 : (i < n4 ? 4 : 3)); };  // of a new entry
                // the last batch's list is padded to 16 with entries of amplitude 0
                const bool flush = last && j0 + 64 >= total;
                const int npad = flush ? (nf + 15) & ~15 : nf;
                if (lane < npad - nf)
                    for (int i = 0; i < mm_floats(C); ++i) s_w[wave][nf + lane][i] = 0.0f;
                if (cls >= 0) {
                    const int pos = cls == 7   ? kept + rank_below(b7)
                                    : cls == 6 ? n7 + rank_below(b6)
                                    : cls == 5 ? n6 + rank_below(b5)
                                    : cls == 4 ? n5 + rank_below(b4)
                                    : cls == 3 ? n4 + rank_below(b3)
                                               : rank_below(bd) + npad;
                    float4_t *dst = reinterpret_cast<float4_t *>(&s_w[wave][pos][0]);
                    const float4_t r1 = load4(&rp->rx), kap = load4(rp->kappa), am = load4(rp->amp);
                    const uint32_t rx = __float_as_uint(r1.x), ry = __float_as_uint(r1.y);
                    float ik0 = 1.0f, e0 = 1.0f;  // the amplitude's factor is e0 2^(ne - erun): e0 near 1, the power beyond FP32's
                    int ne;                       // range for the smallest amplitudes, so it is applied to the amplitude itself
                    if (cls > 0) {
                        float k0, k1, k2, k3, k4;
                        cross_poly(r0.y * MM_A_OF_BETA2, cls, k0, k1, k2, k3, k4);
                        ik0 = __builtin_amdgcn_rcpf(k0);
                        e0 = k0 * __builtin_amdgcn_exp2f(qf);
                        ne = MM_XS - qi;
                        dst[0] = (float4_t){lx, r0.x, ly, r0.z};
                        const int32_t rx20 = (int32_t)(rx & 0xfffff000u), ry20 = (int32_t)(ry & 0xfffff000u);
                        dst[1] = (float4_t){(float)rx20 * 0x1p-32f, (float)(rx & 0xfffu) * 0x1p-32f,
                                            (float)ry20 * 0x1p-32f, (float)(ry & 0xfffu) * 0x1p-32f};
                        k2 *= ik0;
                        dst[2] = (float4_t){k1 * ik0, k2 * (8.0f / MM_P),
                                            cls > 3 ? k3 * ik0 * __builtin_amdgcn_rcpf(k2) * (8.0f / MM_P) : 0.0f,
                                            cls > 4 ? k4 * __builtin_amdgcn_rcpf(k3) * (8.0f / MM_P) : 0.0f};
                        pairs += SUBX * SUBX / 64;
                    } else {
                        const uint32_t rows = row_block_mask<MF>(r0.x, r0.y, r0.z, lim, x0, x1, sy, hy, mryf);
                        ne = MM_XS + MM_YS;
                        dst[0] = (float4_t){r0.x, r0.y, r0.z, r0.w};
                        dst[1] = (float4_t){r1.z, r1.w, __uint_as_float(rows), 0.0f};
                        pairs += __popc(rows);
                    }
                    // phase base at the centre: exact ramp in 0.32 fixed point, the rest in FP64
                    const int cx = sx + 8, cy = sy + 8;
                    const uint32_t ramp = (uint32_t)cx * rx + (uint32_t)cy * ry;
                    const double ramp_rev = (double)ramp * (1.0 / 4294967296.0);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        float bs;
                        if (k.phase_mode == 1) {
                            // plain FP32 phase (precision study only)
                            const float rr = (float)cx * r1.z + (float)cy * r1.w;
                            const float v = kap[c] - rr - r0.w * (float)s_d0[wave][c];
                            bs = v - floorf(v);
                        } else {
                            bs = (float)frac_m((double)kap[c] - ramp_rev - (double)r0.w * s_d0[wave][c]);
                        }
                        dst[3 + c] = (float4_t){bs, ldexpf(am[c], ne - erun[c]) * e0, r0.w * s_phi[wave][c] * ik0, r0.w};
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int nfull = flush ? npad : nf & ~15;
                npass += nfull >> 4;
                for (int e = 0; e < nfull; e += 16) {
                    int R = class_at(max(e, kept));  // the list is in descending order after the kept entries
                    if (e < kept) R = nf > kept ? max(R, keptR) : keptR;
                    mm_pass<C>(s_w[wave], e, __builtin_amdgcn_readfirstlane(R), lane, L, M);
                }
                if (nd && !have_dd) {
                    have_dd = true;
                    const double iWx = 1.0 / (k.nx * k.px), iWy = 1.0 / (k.ny * k.py);
#pragma unroll 1
                    for (int f = 0; f < MF; ++f) {
                        const double nux = (sx + col) * iWx, nuy = (sy + row0 + 4 * f) * iWy, nu2 = nux * nux + nuy * nuy;
#pragma unroll 1
                        for (int c = 0; c < C; ++c) {
                            const double il = k.inv_lambda[c];
                            s_dd[wave][f][c][lane] = nu2 < il * il ? (float)(dprop_m(nu2, il) - s_d0[wave][c]) : 0.0f;
                        }
                    }
                }
                for (int e = npad; e < npad + nd; ++e) {
                    const float *w = &s_w[wave][e][0];
                    const float alpha = w[0], beta2 = w[1], gamma = w[2], z = w[3], rxf = w[4], ryf = w[5];
                    const uint32_t rows = __builtin_amdgcn_readfirstlane(__float_as_uint(w[6]));
                    // opaque to the optimiser: these paths' per-lane values are formed here rather than
                    // held in registers through the matrix passes
                    int cl = col, rw = row0;
                    asm volatile("" : "+v"(cl), "+v"(rw));
                    const float fmx = (float)((double)(sx + cl) - k.mrx), dxf = (float)(cl - 8);
#pragma unroll
                    for (int f = 0; f < MF; ++f) {
                        if (!(rows & (1u << f))) continue;
                        const float fmy = (float)((double)(sy + rw + 4 * f) - k.mry);
                        const float E = __builtin_amdgcn_exp2f(
                            -fmaf(gamma, fmy * fmy, fmaf(beta2, fmx * fmy, alpha * (fmx * fmx))));
                        const float dyf = (float)(rw + 4 * f - 8);
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const float bx = __builtin_amdgcn_fractf(fmaf(-dxf, rxf, w[12 + 4 * c]));
                            const float th = fmaf(-z, s_dd[wave][f][c][lane], fmaf(-dyf, ryf, bx));
                            const float wgt = w[13 + 4 * c] * E;
                            M.re[0][c][f] = fmaf(wgt, __builtin_amdgcn_cosf(th), M.re[0][c][f]);
                            M.im[0][c][f] = fmaf(wgt, __builtin_amdgcn_sinf(th), M.im[0][c][f]);
                        }
                    }
                }
                // what does not fill a pass stays, moved to the list's front
                if (!flush) {
                    const int nk = nf - nfull;
                    __builtin_amdgcn_wave_barrier();
                    if (nfull) {
                        keptR = class_at(nfull);
                        if (lane < nk) {
                            float4_t t[mm_floats(C) / 4];
#pragma unroll
                            for (int i = 0; i < mm_floats(C) / 4; ++i)
                                t[i] = reinterpret_cast<const float4_t *>(&s_w[wave][nfull + lane][0])[i];
#pragma unroll
                            for (int i = 0; i < mm_floats(C) / 4; ++i)
                                reinterpret_cast<float4_t *>(&s_w[wave][lane][0])[i] = t[i];
                        }
                    } else {
                        keptR = max(keptR, nf > kept ? class_at(kept) : 3);
                    }
                    kept = nk;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (wave_live && last && total == 0 && kept) {
                // nothing new in the last round: evaluate what was kept
                if (lane < 16 - kept)
                    for (int i = 0; i < mm_floats(C); ++i) s_w[wave][kept + lane][i] = 0.0f;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                mm_pass<C>(s_w[wave], 0, __builtin_amdgcn_readfirstlane(keptR), lane, L, M);
                kept = 0;
            }
            // S = M_0 + t M_1 at the lane's four frequencies.  The matrix units' running FP32 sums round
            // less well than single additions, so after 500 Gaussians or more (looked at after a round of
            // candidates: 1500 at most) they move to the output and are added there (one sum over 1e5 Gaussians at 2160 x 3840 was 1.2e-5 off; it is
            // 1.4e-6 off this way, 4.5e-6 term by term).
            if (npass >= MM_EMIT || last) {
                int sx = sx0, sy = sy0, cl = col, rw = row0;
                asm volatile("" : "+s"(sx), "+s"(sy), "+v"(cl), "+v"(rw));  // formed here, as above
                const int mxp = sx + cl;
#pragma unroll
                for (int f = 0; f < MF; ++f) {
                    const int myp = sy + rw + 4 * f;
                    const bool valid = mxp >= -hx && mxp < hx && myp >= -hy && myp < hy;
                    const float t = ((float)cl - 7.5f) * ((float)(rw + 4 * f) - 7.5f) * (1.0f / MM_P);
                    const int mx = mxp < 0 ? mxp + k.nx : mxp, my = myp < 0 ? myp + k.ny : myp;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const int eo = erun[c] - MM_XS - MM_YS;
                        float2 v;
                        v.x = ldexpf(fmaf(t, M.re[1][c][f], M.re[0][c][f]), eo);
                        v.y = ldexpf(fmaf(t, M.im[1][c][f], M.im[0][c][f]), eo);
                        float2 *dst = slot < 0 ? S.spectrum + ((int64_t)c * k.ny + my) * k.nx + mx
                                               : S.partials + (((int64_t)slot * C + c) * MF + f) * WG + tid;
                        if (slot >= 0 || valid) {
                            if (emitted) {
                                const float2 w = *dst;
                                v.x += w.x;
                                v.y += w.y;
                            }
                            *dst = v;
                        }
                        M.re[0][c][f] = M.re[1][c][f] = M.im[0][c][f] = M.im[1][c][f] = 0.0f;
                    }
                }
                emitted = true;
                npass = 0;
            }
            __syncthreads();
        }
        const long long np = wave_sum_i64((long long)pairs) * 64;
        if (lane == 0 && np) atomicAdd((unsigned long long *)&S.counters[CTR_PAIRS], (unsigned long long)np);
    }
}

hipError_t launch_accumulate_mfma(const Plan &p, const Consts &k, const FwdScene *scenes, const int32_t *prefix,
                                  int n_scenes, long long *queue, int grid, hipStream_t s)
{
#define GWS_MM(CC)                                                                                               \
    hipLaunchKernelGGL((k_accumulate_mfma<CC>), dim3(grid), dim3(WG), 0, s, k, p.tile_xy, scenes, prefix, n_scenes, queue)
    switch (k.C) {
    case 1: GWS_MM(1); break;
    case 2: GWS_MM(2); break;
    case 3: GWS_MM(3); break;
    case 4: GWS_MM(4); break;
    default: return hipErrorInvalidValue;
    }
#undef GWS_MM
    return hipGetLastError();
}

int accumulate_mfma_occupancy(int C)
{
    const void *kp = nullptr;
    switch (C) {
    case 1: kp = (const void *)k_accumulate_mfma<1>; break;
    case 2: kp = (const void *)k_accumulate_mfma<2>; break;
    case 3: kp = (const void *)k_accumulate_mfma<3>; break;
    default: kp = (const void *)k_accumulate_mfma<4>; break;
    }
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kp, WG, 0) != hipSuccess || nb < 1) nb = 1;
    return nb;
}

}  // namespace gws
