// The 2D DFT as dense real GEMMs on the gfx950 matrix cores, with every FP32 operand split into
// a bf16 high part and a bf16 residual and three products per real product (hi*hi + hi*lo +
// lo*hi), accumulated in FP32 by v_mfma_f32_16x16x32_bf16.
//
// Along one axis, with N = R L (R = 4, or 2) and w_N = exp(+-j 2 pi / N), in FP32
//   y_p[n] = w_N^(n p) sum_j x[n + j L] w_R^(j p),   X[R q + p] = sum_n y_p[n] w_L^(n q),
// and for the dense sum over n = 0 ... L - 1 the symmetries of cosine (even) and sine (odd) in
// both n and q: with e[m] = y[m] + y[L - m], o[m] = y[m] - y[L - m] (a term without a partner
// stands alone)
//   C[q] = sum_m e[m] cos(2 pi m q / L),  S[q] = sum_m o[m] sin(2 pi m q / L),  m, q = 0 ... L / 2,
//   X_p[q] = C[q] +- j S[q],  X_p[L - q] = C[q] -+ j S[q].
// That leaves 1 / (4 R) of the complex products with the whole matrix F[m][n] = w_N^(m n), which
// bound the transform before (matrix units at 54 %): 3840 x 2160 x 3 took 3.08 ms, 0.73 now, of
// which the two folds' memory passes are 0.23; 1920 x 1080 x 3 0.55 -> 0.16, 256 x 256 0.058 -> 0.028.
// R = 1 with larger tiles: 2.5 ms.  Error against FP64 as before, 5.3e-6 (5.5e-6).
//
// k_dft_fold does the FP32 part and writes e and o as eight bf16 planes (hi and lo of Re e, Im e,
// Re o, Im o); k_dft_gemm computes all X_p of X [M][N], writing the result transposed, [N][M].
// Applied twice -- first to the rows of the image, then to the rows of the transposed
// intermediate, which stands in the output array -- they give the 2D transform in natural
// layout:  (S F_x)^T = T^T, (T^T F_y)^T = F_y S F_x.
//
// The cosine and sine matrices are built once per size on the host from exactly reduced phases
// (m q mod L) in FP64 and stored pre-split as four bf16 planes (cos hi, sin hi, cos lo, sin lo),
// [q][m], zero-padded to the block tile.
#include <math.h>
#include <string.h>

#include <vector>

#include "gws_internal.h"

namespace gws {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// Block tile 64 (rows of the data operand) x 64 (frequencies q) x 32 (m); four wavefronts in a
// 2 x 2 grid, each owning 32 x 32 as 2 x 2 MFMA tiles of 16 x 16, four sums each (C and S of Re
// and Im: 64 registers).  Two work-groups per CU (60 KB of LDS each), so one's loads and
// barriers overlap the other's products.  128 x 128 with four times the registers spilled.
constexpr int DBM = 64, DBN = 64, DBK = 32, DTHREADS = 256;
constexpr int DSTR = DBK + 8;  // padded LDS row stride (bf16 elements): conflict-free 16-byte fragment reads
constexpr int NPA = 8;         // data planes: hi of Re e, Im e, Re o, Im o, then lo
constexpr int NPB = 4;         // matrix planes: cos hi, sin hi, cos lo, sin lo

struct DftMats {
    int n, radix, len, npad, kpad;  // N, R, L = N / R; L / 2 + 1 padded to the block tile's columns and its k
    uint16_t *planes;               // [NPB][npad][kpad]
};

static __device__ __forceinline__ uint16_t f32_to_bf16_rne(float x)
{
    const uint32_t b = __float_as_uint(x);
    return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}
static __device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

static int radix_of(int n) { return n % 4 == 0 ? 4 : 2; }  // grids are even
static int kpad_of(int n) { return (n / radix_of(n) / 2 + 1 + DBK - 1) / DBK * DBK; }

struct Split2 {
    uint16_t h, l;
};
static __device__ __forceinline__ Split2 split_bf16(float x)
{
    Split2 r;
    r.h = f32_to_bf16_rne(x);
    r.l = f32_to_bf16_rne(x - bf16_to_f32(r.h));
    return r;
}

// The FP32 part along the rows: X [img][M][N] complex64 -> [img][R][8][M][kpad] bf16 planes (v = hi
// + lo, each rounded to nearest even), zero beyond L / 2.  tw[i] = exp(-j 2 pi i / N).  One thread per
// four m of a row, for every p; it reads the row at m + j L and L - m + j L.  Bound by memory:
// 8 bytes read and 8 written per element.
template <int R>
__global__ void __launch_bounds__(256) k_dft_fold(const float2 *__restrict__ X, uint16_t *__restrict__ P,
                                                  const float2 *__restrict__ tw, int dir, int M, int N, int kpad,
                                                  int64_t total)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int per_row = kpad / 4, L = N / R;
    const int64_t rowi = t / per_row;
    const int m0 = (int)(t - rowi * per_row) * 4;
    const int64_t img = rowi / M;
    const int row = (int)(rowi - img * M);
    const float2 *src = X + rowi * N;
    const float s = (float)dir;
    u16x4 pl[R][NPA];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + i;
        float2 y[2][R];  // y_p at m and at L - m
        const bool live = 2 * m <= L, pair = live && m != 0 && 2 * m != L;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool on = h ? pair : live;
            const int n = h ? L - m : m;
            float2 x[R];
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = on ? src[n + j * L] : make_float2(0.0f, 0.0f);
            if constexpr (R == 2) {
                y[h][0] = make_float2(x[0].x + x[1].x, x[0].y + x[1].y);
                y[h][1] = make_float2(x[0].x - x[1].x, x[0].y - x[1].y);
            } else {
                const float2 a = make_float2(x[0].x + x[2].x, x[0].y + x[2].y), b = make_float2(x[0].x - x[2].x, x[0].y - x[2].y);
                const float2 c = make_float2(x[1].x + x[3].x, x[1].y + x[3].y);
                const float2 d = make_float2(s * (x[3].y - x[1].y), s * (x[1].x - x[3].x));  // s j (x1 - x3)
                y[h][0] = make_float2(a.x + c.x, a.y + c.y);
                y[h][1] = make_float2(b.x + d.x, b.y + d.y);
                y[h][2] = make_float2(a.x - c.x, a.y - c.y);
                y[h][3] = make_float2(b.x - d.x, b.y - d.y);
            }
#pragma unroll
            for (int p = 1; p < R; ++p) {
                const float2 w = on ? tw[n * p] : make_float2(1.0f, 0.0f);  // n p < N
                const float wi = -s * w.y;
                y[h][p] = make_float2(fmaf(y[h][p].x, w.x, -y[h][p].y * wi), fmaf(y[h][p].x, wi, y[h][p].y * w.x));
            }
        }
#pragma unroll
        for (int p = 0; p < R; ++p) {
            const float2 u = y[0][p], v = y[1][p];
            const float q[4] = {u.x + v.x, u.y + v.y, pair ? u.x - v.x : 0.0f, pair ? u.y - v.y : 0.0f};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const Split2 sp = split_bf16(q[c]);
                pl[p][c][i] = sp.h;
                pl[p][c + 4][i] = sp.l;
            }
        }
    }
    const int64_t plane = (int64_t)M * kpad;
    uint16_t *dst = P + (img * R * NPA * M + row) * (int64_t)kpad + m0;
#pragma unroll
    for (int p = 0; p < R; ++p)
#pragma unroll
        for (int c = 0; c < NPA; ++c) *(u16x4 *)(dst + (p * NPA + c) * plane) = pl[p][c];
}

// Out [img][R L][M] complex64 for the data planes A [img][R][8][M][K] and the matrix planes Bt
// [4][npad][K]: row R q + p of image img from the planes (img, p).
//
// Block order.  Work-groups are dealt to the 8 XCDs round-robin (id % 8), each with its own L2,
// and one operand of a block streams while the other stays cached.  So each XCD takes a
// contiguous run of tiles, and within it tiles go down groups of GROUP_M block rows before the
// next block column: the ~32 blocks an XCD runs at once share a few block rows and columns.
constexpr int GROUP_M = 8;

template <int DIR>
__global__ void __launch_bounds__(DTHREADS, 2) k_dft_gemm(const uint16_t *__restrict__ A, const uint16_t *__restrict__ Bt,
                                                          float2 *__restrict__ out, int M, int R, int L, int K, int npad,
                                                          int mblocks, int rows_total, int per_xcd)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[NPA * DBM * DSTR];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[NPB * DBN * DSTR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // tile of this work-group: rows_total = batch x R x mblocks block rows, npad / DBN block columns
    const int nblocks = npad / DBN;
    const int T = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
    if (T >= rows_total * nblocks) return;
    const int per_group = GROUP_M * nblocks, grp = T / per_group, first = grp * GROUP_M;
    const int gm = min(rows_total - first, GROUP_M), w = T - grp * per_group;
    const int rowblk = first + w % gm, nb = w / gm;
    const int64_t ip = rowblk / mblocks;  // img R + p
    const int n0 = nb * DBN, m0 = (rowblk - (int)ip * mblocks) * DBM;
    const int64_t aplane = (int64_t)M * K, bplane = (int64_t)npad * K;
    const int wm = wave & 1, wn = wave >> 1;
    // staging: thread t moves 16 bytes (8 k) of row t / 4 of every plane; rows beyond M repeat the
    // last one (their results are not stored)
    const int srow = tid >> 2, sk = (tid & 3) * 8;
    const uint16_t *ga = A + ip * NPA * aplane + (int64_t)min(m0 + srow, M - 1) * K + sk;
    const uint16_t *gb = Bt + (int64_t)(n0 + srow) * K + sk;
    const int s_lds = srow * DSTR + sk;
    u16x8 ra[NPA], rb[NPB];
#pragma unroll
    for (int p = 0; p < NPA; ++p) ra[p] = *(const u16x8 *)(ga + p * aplane);
#pragma unroll
    for (int p = 0; p < NPB; ++p) rb[p] = *(const u16x8 *)(gb + p * bplane);
    f32x4 acc[2][2][4];  // [row tile][frequency tile][C of Re, C of Im, S of Re, S of Im]
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[t][u][q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int kk = (lane >> 4) * 8;
    const uint16_t *fa = As + (wm * 32 + (lane & 15)) * DSTR + kk, *fb = Bs + (wn * 32 + (lane & 15)) * DSTR + kk;
    for (int kc = 0; kc < K; kc += DBK) {
        __syncthreads();  // the previous k-step's fragments are read
#pragma unroll
        for (int p = 0; p < NPA; ++p) *(u16x8 *)(As + p * DBM * DSTR + s_lds) = ra[p];
#pragma unroll
        for (int p = 0; p < NPB; ++p) *(u16x8 *)(Bs + p * DBN * DSTR + s_lds) = rb[p];
        __syncthreads();
        if (kc + DBK < K) {  // prefetch the next k-step into registers
            ga += DBK;
            gb += DBK;
#pragma unroll
            for (int p = 0; p < NPA; ++p) ra[p] = *(const u16x8 *)(ga + p * aplane);
#pragma unroll
            for (int p = 0; p < NPB; ++p) rb[p] = *(const u16x8 *)(gb + p * bplane);
        }
        // the data's high parts with both parts of the matrix, then its low parts with the high
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 a[2][4];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    a[t][q] = *(const bf16x8 *)(fa + (4 * h + q) * DBM * DSTR + t * 16 * DSTR);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int l = 0; l < 2 - h; ++l) {
                    const bf16x8 bc = *(const bf16x8 *)(fb + (2 * l) * DBN * DSTR + u * 16 * DSTR);
                    const bf16x8 bs = *(const bf16x8 *)(fb + (2 * l + 1) * DBN * DSTR + u * 16 * DSTR);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            acc[t][u][q] =
                                __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][q], q < 2 ? bc : bs, acc[t][u][q], 0, 0, 0);
                }
        }
    }
    // D[row][col] of a 16 x 16 tile: row = (lane / 16) * 4 + i, col = lane % 16; written transposed
    const int64_t img = ip / R;
    const int p = (int)(ip - img * R);
    float2 *Yi = out + img * R * L * M;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int f = n0 + wn * 32 + u * 16 + (lane & 15);
        if (2 * f > L) continue;
        // the frequencies f and L - f
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            if (v && (f == 0 || 2 * f == L)) continue;
            float2 *Yr = Yi + ((int64_t)R * (v ? L - f : f) + p) * M;
            const float s = (DIR > 0) == (v == 0) ? 1.0f : -1.0f;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int row0 = m0 + wm * 32 + t * 16 + (lane >> 4) * 4;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (row0 + i < M)
                        Yr[row0 + i] = make_float2(fmaf(-s, acc[t][u][3][i], acc[t][u][0][i]),
                                                   fmaf(s, acc[t][u][2][i], acc[t][u][1][i]));
            }
        }
    }
}

static uint16_t host_bf16(float x)
{
    uint32_t b;
    memcpy(&b, &x, 4);
    return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}
static float host_bf16_f(uint16_t h)
{
    const uint32_t b = (uint32_t)h << 16;
    float f;
    memcpy(&f, &b, 4);
    return f;
}

static hipError_t build_mats_n(int n, DftMats *out)
{
    const int R = radix_of(n), L = n / R, half = L / 2 + 1, npad = (half + DBN - 1) / DBN * DBN, kpad = kpad_of(n);
    const size_t plane = (size_t)npad * kpad;
    std::vector<uint16_t> h(NPB * plane, 0);
    for (int f = 0; f < half; ++f)
        for (int m = 0; m < half; ++m) {
            const long long r = ((long long)f * m) % L;
            const double ph = 2.0 * M_PI * (double)r / (double)L;
            const double vals[2] = {cos(ph), sin(ph)};
            for (int part = 0; part < 2; ++part) {  // cos, sin
                const double x = vals[part];
                const uint16_t hi = host_bf16((float)x);
                const uint16_t lo = host_bf16((float)(x - (double)host_bf16_f(hi)));
                h[part * plane + (size_t)f * kpad + m] = hi;
                h[(2 + part) * plane + (size_t)f * kpad + m] = lo;
            }
        }
    out->n = n;
    out->radix = R;
    out->len = L;
    out->npad = npad;
    out->kpad = kpad;
    hipError_t e = hipMalloc(&out->planes, h.size() * sizeof(uint16_t));
    if (e != hipSuccess) return e;
    return hipMemcpy(out->planes, h.data(), h.size() * sizeof(uint16_t), hipMemcpyHostToDevice);
}

hipError_t build_dft_mats(Plan &p)
{
    if (p.dft_mats) return hipSuccess;
    DftMats *m = new DftMats[2];
    hipError_t e = build_mats_n(p.nx, &m[0]);
    if (e == hipSuccess) e = build_mats_n(p.ny, &m[1]);
    if (e != hipSuccess) {
        delete[] m;
        return e;
    }
    p.dft_mats = (void *)m;
    return hipSuccess;
}

void free_dft_mats(Plan &p)
{
    if (!p.dft_mats) return;
    DftMats *m = (DftMats *)p.dft_mats;
    (void)hipFree(m[0].planes);
    (void)hipFree(m[1].planes);
    delete[] m;
    p.dft_mats = nullptr;
}

// The data planes of one axis at a time, [batch][R][8][M][kpad] bf16: 8 bytes per complex element
// and a few percent of padding.
size_t dft_bf16x3_workspace(int nx, int ny, int batch)
{
    const size_t x = (size_t)ny * radix_of(nx) * kpad_of(nx), y = (size_t)nx * radix_of(ny) * kpad_of(ny);
    return (size_t)batch * std::max(x, y) * 2 * NPA + 256;
}

// Transform the rows of in [batch][M][F.n] into out [batch][F.n][M] (in == out is fine).
static void transform_rows(const DftMats &F, const float2 *tw, int dir, const float2 *in, float2 *out, uint16_t *planes,
                           int M, int batch, hipStream_t s)
{
    const int64_t total = (int64_t)batch * M * (F.kpad / 4);
    const dim3 fgrid((unsigned)((total + 255) / 256)), fblock(256);
#define GWS_DFT_FOLD(R) \
    hipLaunchKernelGGL(k_dft_fold<R>, fgrid, fblock, 0, s, in, planes, tw, dir, M, F.n, F.kpad, total)
    if (F.radix == 4) GWS_DFT_FOLD(4);
    else GWS_DFT_FOLD(2);
#undef GWS_DFT_FOLD
    const int mblocks = (M + DBM - 1) / DBM, rows_total = batch * F.radix * mblocks;
    const int tiles = rows_total * (F.npad / DBN), per_xcd = (tiles + 7) / 8;
    const dim3 grid((unsigned)(8 * per_xcd)), block(DTHREADS);
    if (dir > 0)
        hipLaunchKernelGGL((k_dft_gemm<1>), grid, block, 0, s, planes, F.planes, out, M, F.radix, F.len, F.kpad, F.npad,
                           mblocks, rows_total, per_xcd);
    else
        hipLaunchKernelGGL((k_dft_gemm<-1>), grid, block, 0, s, planes, F.planes, out, M, F.radix, F.len, F.kpad, F.npad,
                           mblocks, rows_total, per_xcd);
}

hipError_t launch_dft_bf16x3(Plan &p, int batch, int direction, const float2 *in, float2 *out, void *ws, hipStream_t s)
{
    hipError_t e = build_dft_mats(p);
    if (e != hipSuccess) return e;
    const DftMats *m = (const DftMats *)p.dft_mats;
    transform_rows(m[0], p.tw_x, direction, in, out, (uint16_t *)ws, p.ny, batch, s);   // (S F_x)^T [nx][ny]
    transform_rows(m[1], p.tw_y, direction, out, out, (uint16_t *)ws, p.nx, batch, s);  // F_y S F_x [ny][nx]
    return hipGetLastError();
}

}  // namespace gws
