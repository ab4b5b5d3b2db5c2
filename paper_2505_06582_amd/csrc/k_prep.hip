// Per-Gaussian preprocessing, depth sort and binning of spectral supports (gfx950).
//
// k_keys     one thread per Gaussian: validity, spectral-support radius bucket, sort key
//            (forward: support radius descending, then depth descending = front to back;
//            adjoint: level of the radius, then the support's shape).
// radix sort stable LSD radix sort of the keys, 8-bit digits, wave-ballot ranking.
// k_records  one thread per sorted Gaussian: the 64-byte record the accumulation reads,
//            with every large phase quantity reduced exactly in FP64 / fixed point.
// k_bin_*    one work-group per scene: candidate counts per tile, chunk size, work-item lists.
//
// Each launch takes up to PREP_GROUP scenes (blockIdx): bound by latency, they take hardly longer
// than one (six scenes of 1e4 Gaussians at 1280 x 1024: 860 us a scene after another, 290 together).
//
// The spectrum of Gaussian i (Sec. 4.1, Eq. 10, in-plane so det J = 1) has modulus
// 2 pi sqrt(det S) exp(-2 pi^2 nu^T S nu): an ellipse centred on DC.  In index units
// (nu_x = m_x'/(nx px), nu_y = m_y'/(ny py)) the exponent, written in powers of two, is
// q(m') = alpha m_x'^2 + beta2 m_x' m_y' + gamma m_y'^2 and the term is below eps of its
// peak outside q <= log2(1/eps).  The circumscribed circle of that ellipse has radius
// sqrt(log2(1/eps) / lambda_min) and sets the Gaussian's bucket.
#include "mfma_f16.h"

namespace gws {

static __device__ __forceinline__ bool finite_f(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

static __device__ __forceinline__ double frac_d(double v) { return v - floor(v); }

// The adjoint's order: its sums do not depend on it, so Gaussians whose ellipses cover the same
// sub-tiles stand together -- levels of the radius (LPO to the octave), then the ratio of the
// axes in four steps, then the axis' direction.  A level's largest radius bounds its tiles.
constexpr uint32_t KEY_CULLED = 0xffffu;  // upper 16 bits of an invalid Gaussian's key, above every valid one
constexpr int BWD_LPO = 4, BWD_LEVELS = 12 * BWD_LPO;
static __device__ __forceinline__ int bwd_level(int bucket)
{
    return min(BWD_LEVELS, (int)((float)BWD_LPO * log2f((float)(bucket + 1))));
}
static __device__ __forceinline__ int bwd_level_bucket(int level)
{
    return min(NBUCKET - 1, (int)exp2f((float)(level + 1) * (1.0f / BWD_LPO)) + 1);  // one above: log2f's rounding
}

// Also clears the scene's counters and bucket ends, which the next kernels write.
__global__ void __launch_bounds__(256) k_keys(PrepGroup grp, Consts k)
{
    const PrepScene &S = grp.s[blockIdx.y];
    const GView &g = S.g;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < CTR_COUNT) S.counters[i] = 0;
    if (i < NBUCKET) S.bucket_end[i] = 0;
    if (i >= g.n) return;
    const float sxx = g.cov_xx[i], sxy = g.cov_xy[i], syy = g.cov_yy[i];
    const float mx = g.mean_x[i], my = g.mean_y[i], z = g.depth[i], o = g.opacity[i], ph = g.phase[i];
    bool ok = finite_f(sxx) && finite_f(sxy) && finite_f(syy) && finite_f(mx) && finite_f(my) &&
              finite_f(z) && finite_f(o) && finite_f(ph);
    bool any_amp = false;
    for (int c = 0; c < k.C; ++c) {
        const float a = g.amplitude[(int64_t)c * g.amp_stride + i];
        ok = ok && finite_f(a);
        any_amp = any_amp || (a != 0.0f);
    }
    const double det = (double)sxx * syy - (double)sxy * sxy;
    ok = ok && sxx > 0.0f && det > 0.0;
    if (k.forward) ok = ok && o != 0.0f && any_amp;
    uint32_t hi, lo;
    if (ok) {
        const double Wx = k.nx * k.px, Wy = k.ny * k.py;
        const double a = k.K2 * sxx / (Wx * Wx), b = k.K2 * sxy / (Wx * Wy), c = k.K2 * syy / (Wy * Wy);
        const double rad = sqrt(0.25 * (a - c) * (a - c) + b * b), lmin = 0.5 * (a + c) - rad;
        int bucket = NBUCKET - 1;
        if (lmin > 0.0) {
            const double R = sqrt(k.tau2 / lmin);
            if (R < (double)(NBUCKET - 1)) bucket = (int)R;
        }
        if (k.forward) {
            hi = (uint32_t)(NBUCKET - 1 - bucket);
        } else {
            const int aspect = min(3, (int)(4.0f * sqrtf(fmaxf((float)lmin, 0.0f) / (float)(lmin + 2.0 * rad))));
            const float axis = 0.5f + 0.15915494309189535f * atan2f((float)(2.0 * b), (float)(a - c));  // [0, 1]
            hi = (uint32_t)(((BWD_LEVELS - bwd_level(bucket)) << 10) | (aspect << 8) | min(255, (int)(256.0f * axis)));
        }
    } else {
        hi = KEY_CULLED;
    }
    // depth, descending: map the float to an ascending unsigned key, then complement
    const uint32_t u = __float_as_uint(z);
    const uint32_t asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    lo = k.forward ? ~asc : 0u;
    S.keys_a[i] = ((uint64_t)hi << 32) | (uint64_t)lo;
    S.vals_a[i] = (uint32_t)i;
}

hipError_t launch_keys(const PrepGroup &grp, const Consts &k, hipStream_t s)
{
    const int64_t blocks = std::max<int64_t>((grp.max_n() + 255) / 256, NBUCKET / 256);
    hipLaunchKernelGGL(k_keys, dim3((unsigned)blocks, grp.n), dim3(256), 0, s, grp, k);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Stable LSD radix sort, 8-bit digits.  Each wavefront owns a run of consecutive keys and ranks
// them by ballots with its own running counts, so a digit takes two barriers, not one per row of
// keys.  Bound by latency.  Up to SORT_ONE keys: one work-group sorts them in LDS, all digits in one
// launch.  More: per digit a histogram and a scatter, where every block owns SORT_TILE keys and adds
// up the rows (256 counts per block) before its own itself; counting the next digit while
// scattering took longer (global atomics: 14 us per digit of 1e4 keys).
// ---------------------------------------------------------------------------------
constexpr int SORT_THREADS = 1024, SORT_WAVES = SORT_THREADS / 64, SORT_ITEMS = 4;
constexpr int SORT_TILE = SORT_THREADS * SORT_ITEMS;
// what fits one CU's LDS: 10 bytes a key and the wavefronts' counts
constexpr int SORT_ONE_ITEMS = 12, SORT_ONE = SORT_THREADS * SORT_ONE_ITEMS;
// above this many blocks, adding up the rows in each of them (256 KiB read per 256 rows) takes
// longer than a launch that does it once
constexpr int SORT_SELF_SCAN = 512;
static int sort_blocks(int64_t n) { return (int)std::max<int64_t>(1, (n + SORT_TILE - 1) / SORT_TILE); }
int64_t sort_table_words(int64_t n) { return (int64_t)256 * sort_blocks(n); }

// Rank of the lane's digit among the wavefront's keys so far; cnt is the wavefront's row of counts.
static __device__ __forceinline__ uint32_t sort_rank(uint32_t *cnt, uint32_t dg, bool valid)
{
    const uint64_t on = __ballot(valid);
    uint32_t lo = (uint32_t)on, hi = (uint32_t)(on >> 32);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const int32_t m = (int32_t)(dg << (31 - bit)) >> 31;  // the digit's bit in every position
        const uint64_t bb = __ballot(m);
        lo &= ~((uint32_t)bb ^ (uint32_t)m);
        hi &= ~((uint32_t)(bb >> 32) ^ (uint32_t)m);
    }
    const uint64_t same = ((uint64_t)hi << 32) | lo;
    const uint32_t below = (uint32_t)rank_below(same), old = cnt[dg];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) cnt[dg] = old + (uint32_t)__popcll(same);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return old + below;
}

// Exclusive prefix over the 256 digits (threads 0 ... 255; every thread calls).
static __device__ __forceinline__ uint32_t sort_digit_scan(uint32_t v, uint32_t *s_wave, int tid, int lane)
{
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63 && tid < 256) s_wave[tid >> 6] = incl;
    __syncthreads();
    uint32_t base = 0;
    for (int w = 0; w < (tid >> 6) && w < 4; ++w) base += s_wave[w];
    return base + incl - v;
}

template <int ITEMS>
__global__ void __launch_bounds__(SORT_THREADS) k_sort_one(PrepGroup grp, int first_digit, int last_digit)
{
    __shared__ uint64_t s_key[SORT_THREADS * ITEMS];
    __shared__ uint16_t s_idx[SORT_THREADS * ITEMS];
    __shared__ uint32_t s_off[SORT_WAVES][256];
    __shared__ uint32_t s_wave[4];
    __shared__ uint64_t s_diff[SORT_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = wave * (64 * ITEMS) + lane;
    const PrepScene &S = grp.s[blockIdx.x];
    if (S.g.n == 0 || S.g.n > SORT_THREADS * ITEMS) return;  // nothing, or in many blocks
    const int n = (int)S.g.n;
    uint64_t *const keys = S.keys_a;
    uint64_t key[ITEMS];
    uint32_t idx[ITEMS], rank[ITEMS];
    uint64_t diff = 0;
    const uint64_t key0 = keys[0];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int i = base + it * 64;
        idx[it] = (uint32_t)i;
        key[it] = i < n ? keys[i] : key0;
        diff |= key[it] ^ key0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) diff |= __shfl_xor(diff, o);
    if (lane == 0) s_diff[wave] = diff;
    __syncthreads();
    diff = 0;
#pragma unroll
    for (int w = 0; w < SORT_WAVES; ++w) diff |= s_diff[w];
    for (int dg = first_digit; dg <= last_digit; ++dg) {
        const int shift = 8 * dg;
        if (((diff >> shift) & 0xffu) == 0) continue;  // every key holds the same digit
        for (int j = lane; j < 256; j += 64) s_off[wave][j] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            rank[it] = sort_rank(s_off[wave], (uint32_t)(key[it] >> shift) & 0xffu, base + it * 64 < n);
        __syncthreads();
        uint32_t total = 0;
        if (tid < 256)
#pragma unroll
            for (int w = 0; w < SORT_WAVES; ++w) total += s_off[w][tid];
        uint32_t run = sort_digit_scan(total, s_wave, tid, lane);
        if (tid < 256)
#pragma unroll
            for (int w = 0; w < SORT_WAVES; ++w) {
                const uint32_t c = s_off[w][tid];
                s_off[w][tid] = run;
                run += c;
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (base + it * 64 < n) {
                const uint32_t pos = s_off[wave][(uint32_t)(key[it] >> shift) & 0xffu] + rank[it];
                s_key[pos] = key[it];
                s_idx[pos] = (uint16_t)idx[it];
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (base + it * 64 < n) {
                key[it] = s_key[base + it * 64];
                idx[it] = s_idx[base + it * 64];
            }
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (base + it * 64 < n) {
            keys[base + it * 64] = key[it];
            S.vals_a[base + it * 64] = idx[it];
        }
}

__global__ void __launch_bounds__(SORT_THREADS) k_sort_hist(PrepGroup grp, int shift, bool odd)
{
    const PrepScene &S = grp.s[blockIdx.y];
    const int64_t n = S.g.n;
    if (n <= SORT_ONE || (int64_t)blockIdx.x * SORT_TILE >= n) return;
    const uint64_t *__restrict__ keys = odd ? S.keys_b : S.keys_a;
    uint32_t *__restrict__ table = S.sort_table;
    __shared__ uint32_t s_cnt[SORT_WAVES][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int j = lane; j < 256; j += 64) s_cnt[wave][j] = 0;
    uint64_t key[SORT_ITEMS];
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        const int64_t i = (int64_t)blockIdx.x * SORT_TILE + it * SORT_THREADS + tid;
        key[it] = i < n ? keys[i] : 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it)
        sort_rank(s_cnt[wave], (uint32_t)(key[it] >> shift) & 0xffu,
                  (int64_t)blockIdx.x * SORT_TILE + it * SORT_THREADS + tid < n);
    __syncthreads();
    if (tid < 256) {
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) v += s_cnt[w][tid];
        table[(int64_t)blockIdx.x * 256 + tid] = v;
    }
}

// Thread 256 q + d: sum of digit d over the rows of quarter q, and over those before `me`.
static __device__ __forceinline__ void sort_rows(const uint32_t *__restrict__ table, int nb, int me, int d, int q,
                                                 uint32_t &total, uint32_t &before)
{
    const int r0 = nb * q >> 2, r1 = nb * (q + 1) >> 2;
    total = before = 0;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) {
        const uint32_t v = table[(int64_t)r * 256 + d];
        total += v;
        before += r < me ? v : 0u;
    }
}

// Many blocks: the table's rows become output offsets, in one block.
__global__ void __launch_bounds__(SORT_THREADS) k_sort_scan(PrepGroup grp)
{
    uint32_t *__restrict__ table = grp.s[blockIdx.x].sort_table;
    const int64_t n = grp.s[blockIdx.x].g.n;
    const int nb = (int)((n + SORT_TILE - 1) / SORT_TILE);
    if (nb <= SORT_SELF_SCAN) return;
    __shared__ uint32_t part[4][256], s_wave[4];
    const int tid = threadIdx.x, lane = tid & 63, d = tid & 255, q = tid >> 8;
    uint32_t total, before;
    sort_rows(table, nb, 0, d, q, total, before);
    part[q][d] = total;
    __syncthreads();
    const uint32_t all = part[0][d] + part[1][d] + part[2][d] + part[3][d];
    uint32_t run = sort_digit_scan(tid < 256 ? all : 0u, s_wave, tid, lane);
    if (tid < 256)
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = part[j][d];
            part[j][d] = run;
            run += v;
        }
    __syncthreads();
    run = part[q][d];
    const int r0 = nb * q >> 2, r1 = nb * (q + 1) >> 2;
    for (int r = r0; r < r1; ++r) {
        const uint32_t v = table[(int64_t)r * 256 + d];
        table[(int64_t)r * 256 + d] = run;
        run += v;
    }
}

// odd: from keys_b / vals_b to keys_a / vals_a, else the other way.
__global__ void __launch_bounds__(SORT_THREADS) k_sort_scatter(PrepGroup grp, int shift, bool odd)
{
    __shared__ uint32_t s_off[SORT_WAVES][256];  // per wavefront: digit counts, then output offsets
    __shared__ uint32_t s_part[2][4][256], s_wave[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, d = tid & 255, q = tid >> 8;
    const PrepScene &S = grp.s[blockIdx.y];
    const int64_t n = S.g.n;
    const int nb = (int)((n + SORT_TILE - 1) / SORT_TILE), me = blockIdx.x;
    if (n <= SORT_ONE || me >= nb) return;
    const uint64_t *__restrict__ keys_in = odd ? S.keys_b : S.keys_a;
    const uint32_t *__restrict__ vals_in = odd ? S.vals_b : S.vals_a, *__restrict__ table = S.sort_table;
    uint64_t *__restrict__ keys_out = odd ? S.keys_a : S.keys_b;
    uint32_t *__restrict__ vals_out = odd ? S.vals_a : S.vals_b;
    const bool SCANNED = nb > SORT_SELF_SCAN;
    const int64_t base = (int64_t)me * SORT_TILE + wave * (64 * SORT_ITEMS) + lane;
    uint64_t key[SORT_ITEMS];
    uint32_t val[SORT_ITEMS], rank[SORT_ITEMS];
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        const int64_t i = base + it * 64;
        key[it] = i < n ? keys_in[i] : 0;
        val[it] = i < n ? vals_in[i] : 0;
    }
    uint32_t total = 0, before = 0;
    if (SCANNED) {
        if (q == 0) before = table[(int64_t)me * 256 + d];
    } else {
        sort_rows(table, nb, me, d, q, total, before);
        s_part[0][q][d] = total;
        s_part[1][q][d] = before;
    }
    for (int j = lane; j < 256; j += 64) s_off[wave][j] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it)
        rank[it] = sort_rank(s_off[wave], (uint32_t)(key[it] >> shift) & 0xffu, base + it * 64 < n);
    __syncthreads();
    uint32_t run = before;
    if (!SCANNED) {
        total = s_part[0][0][d] + s_part[0][1][d] + s_part[0][2][d] + s_part[0][3][d];
        before = s_part[1][0][d] + s_part[1][1][d] + s_part[1][2][d] + s_part[1][3][d];
        run = before + sort_digit_scan(tid < 256 ? total : 0u, s_wave, tid, lane);
    }
    if (tid < 256)
        for (int w = 0; w < SORT_WAVES; ++w) {
            const uint32_t c = s_off[w][d];
            s_off[w][d] = run;
            run += c;
        }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it)
        if (base + it * 64 < n) {
            const uint32_t pos = s_off[wave][(uint32_t)(key[it] >> shift) & 0xffu] + rank[it];
            keys_out[pos] = key[it];
            vals_out[pos] = val[it];
        }
}

hipError_t radix_sort(const PrepGroup &grp, int first_digit, int last_digit, hipStream_t s)
{
    if ((last_digit - first_digit) % 2 == 0) return hipErrorInvalidValue;  // the result stands in keys_a
    const dim3 block(SORT_THREADS);
    int64_t one = 0, many = 0;  // the largest scene of each kind
    for (int i = 0; i < grp.n; ++i) {
        int64_t &m = grp.s[i].g.n > SORT_ONE ? many : one;
        m = std::max(m, grp.s[i].g.n);
    }
#define GWS_SORT_ONE(I) hipLaunchKernelGGL(k_sort_one<I>, dim3(grp.n), block, 0, s, grp, first_digit, last_digit)
    if (one > 8 * SORT_THREADS) GWS_SORT_ONE(SORT_ONE_ITEMS);
    else if (one > 4 * SORT_THREADS) GWS_SORT_ONE(8);
    else if (one > 2 * SORT_THREADS) GWS_SORT_ONE(4);
    else if (one > SORT_THREADS) GWS_SORT_ONE(2);
    else if (one > 0) GWS_SORT_ONE(1);
#undef GWS_SORT_ONE
    if (many > 0) {
        const int nb = sort_blocks(many);
        const dim3 grid(nb, grp.n);
        for (int dg = first_digit; dg <= last_digit; ++dg) {
            const bool odd = (dg - first_digit) & 1;
            hipLaunchKernelGGL(k_sort_hist, grid, block, 0, s, grp, 8 * dg, odd);
            if (nb > SORT_SELF_SCAN) hipLaunchKernelGGL(k_sort_scan, dim3(grp.n), block, 0, s, grp);
            hipLaunchKernelGGL(k_sort_scatter, grid, block, 0, s, grp, 8 * dg, odd);
        }
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Records, in sorted order.
// ---------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_records(PrepGroup grp, Consts k, bool poly)
{
    const PrepScene &S = grp.s[blockIdx.y];
    const GView &g = S.g;
    const uint64_t *__restrict__ keys = S.keys_a;
    const uint32_t *__restrict__ vals = S.vals_a;
    GRec *__restrict__ rec = S.rec;
    uint32_t *__restrict__ bucket_end = S.bucket_end;
    long long *__restrict__ counters = S.counters;
    const int64_t n = g.n;
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const uint32_t hi = (uint32_t)(keys[s] >> 32);
    if (hi == KEY_CULLED) {
        if (s == 0) counters[CTR_NCULLED] = n;
        return;
    }
    // where the keys change: the end of the bucket, of the valid Gaussians
    const uint32_t after = s + 1 < n ? (uint32_t)(keys[s + 1] >> 32) : KEY_CULLED;
    if (after == KEY_CULLED) counters[CTR_NCULLED] = n - (s + 1);
    if (k.forward && after != hi) bucket_end[NBUCKET - 1 - hi] = (uint32_t)(s + 1);
    const int64_t i = vals[s];
    const double sxx = g.cov_xx[i], sxy = g.cov_xy[i], syy = g.cov_yy[i];
    const double det = sxx * syy - sxy * sxy;
    const double Wx = k.nx * k.px, Wy = k.ny * k.py;
    GRec r;
    r.alpha = (float)(k.K2 * sxx / (Wx * Wx));
    r.beta2 = (float)(2.0 * k.K2 * sxy / (Wx * Wy));
    r.gamma = (float)(k.K2 * syy / (Wy * Wy));
    const float z = g.depth[i];
    r.z = z;
    // ramp: the centring factor (-1)^m' of the SLM-centred field is folded in as +1/2
    const double fx = frac_d((double)g.mean_x[i] / Wx + 0.5);
    const double fy = frac_d((double)g.mean_y[i] / Wy + 0.5);
    r.rx = (uint32_t)(uint64_t)llrint(fx * 4294967296.0);
    r.ry = (uint32_t)(uint64_t)llrint(fy * 4294967296.0);
    r.rxf = (float)((double)(int32_t)r.rx * (1.0 / 4294967296.0));
    r.ryf = (float)((double)(int32_t)r.ry * (1.0 / 4294967296.0));
    const double o = g.opacity[i];
    const double norm = 6.283185307179586 * sqrt(det) / (k.px * k.py * (double)k.nx * (double)k.ny);
    // carrier: the Gaussian's phase, the propagation's z / lambda, and under reference-wave
    // illumination (spectrum taken at nu - nu_r) the ramp's constant part +nu_r . mu
    const double phi_rev =
        frac_d((double)g.phase[i] * 0.15915494309189535 + k.nurx * (double)g.mean_x[i] + k.nury * (double)g.mean_y[i]);
    for (int c = 0; c < 4; ++c) {
        if (c < k.C) {
            r.kappa[c] = (float)frac_d(phi_rev - (double)z * k.inv_lambda[c]);
            r.amp[c] = (float)((double)g.amplitude[(int64_t)c * g.amp_stride + i] * o * norm);
        } else {
            r.kappa[c] = 0.0f;
            r.amp[c] = 0.0f;
        }
    }
    rec[s] = r;
    if (poly) {
        const float a = r.beta2 * MM_A_OF_BETA2;
        float k0, k1, k2, k3, k4;
        cross_poly(a, cross_class(fabsf(a)), k0, k1, k2, k3, k4);
        adj_poly(rec, n)[s] = make_float4(k1 / k0, k2 / k0, k3 / k0, k0);
    }
}

hipError_t launch_records(const PrepGroup &grp, const Consts &k, bool poly, hipStream_t s)
{
    const int64_t blocks = (grp.max_n() + 255) / 256;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_records, dim3((unsigned)blocks, grp.n), dim3(256), 0, s, grp, k, poly);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Forward binning.  Tiles are held in order of increasing distance rho from DC, so the
// candidates of tile k -- Gaussians whose support circle reaches the tile -- are a prefix
// L_k of the sorted Gaussians, and the heaviest tiles come first.  Each tile's
// candidates are split into chunks of CH; CH grows until the tiles with more than one
// chunk need at most max_slots partial-sum slots (bounded workspace).
// ---------------------------------------------------------------------------------
// Scans over the 1024 threads: shuffles within each wavefront, the sixteen totals through LDS
// (s_wave, free again on return).
template <class Op>
static __device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, Op op)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o);
        if ((int)(threadIdx.x & 63) >= o) v = op(v, t);
    }
    return v;
}

static __device__ uint32_t block_excl_scan_1024(uint32_t v, uint32_t *s_wave, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v, [](uint32_t x, uint32_t y) { return x + y; });
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const uint32_t t = s_wave[w];
        before += w < wave ? t : 0u;
        all += t;
    }
    *total = all;
    __syncthreads();
    return before + incl - v;
}

// Largest value of the threads before this one (0 for the first).
static __device__ uint32_t block_excl_max_1024(uint32_t v, uint32_t *s_wave)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v, [](uint32_t x, uint32_t y) { return max(x, y); });
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t m = __shfl_up(incl, 1);
    if (lane == 0) m = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) m = w < wave ? max(m, s_wave[w]) : m;
    __syncthreads();
    return m;
}

static __device__ unsigned long long block_sum_1024(unsigned long long v, unsigned long long *s_sum)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned long long all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) all += s_sum[w];
    return all;
}

__global__ void __launch_bounds__(1024) k_bin_forward(const int32_t *__restrict__ tile_bucket, int ntiles, PrepGroup grp)
{
    const PrepScene &S = grp.s[blockIdx.x];
    const uint32_t *__restrict__ bucket_end = S.bucket_end;
    uint32_t *__restrict__ cum = S.cum;
    int32_t *__restrict__ tile_L = S.tile_L;
    int2 *__restrict__ tile_slots = S.tile_slots;
    Item *__restrict__ items = S.items;
    const int64_t max_items = S.max_items, max_slots = S.max_slots;
    const int base_chunk = S.base_chunk;
    long long *__restrict__ counters = S.counters;
    __shared__ uint32_t tmp[16];
    __shared__ unsigned long long red[16];
    __shared__ int32_t chunk_sh;
    // cum[b] = number of valid Gaussians with bucket >= b: the largest end at or above b
    {
        const int per = NBUCKET / 1024;
        const int b0 = (1023 - threadIdx.x) * per;  // thread 0 owns the highest buckets
        uint32_t m = 0;
        for (int j = 0; j < per; ++j) m = max(m, bucket_end[b0 + j]);
        uint32_t run = block_excl_max_1024(m, tmp);
        for (int j = per - 1; j >= 0; --j) {
            run = max(run, bucket_end[b0 + j]);
            cum[b0 + j] = run;
        }
    }
    __syncthreads();
    // candidates per tile and their total
    unsigned long long sumL = 0;
    for (int t = threadIdx.x; t < ntiles; t += 1024) {
        const uint32_t L = cum[tile_bucket[t]];
        tile_L[t] = (int32_t)L;
        sumL += L;
    }
    const unsigned long long sum = block_sum_1024(sumL, red);
    if (threadIdx.x == 0) {
        // multi-chunk tiles need <= 2 sum / CH slots: the configured base chunk, grown to fit
        long long ch = base_chunk;
        const long long need = (long long)((2ull * sum + (unsigned long long)max_slots - 1) / (unsigned long long)max_slots);
        if (need > ch) ch = (need + 255) / 256 * 256;
        if (ch > (1ll << 30)) ch = 1ll << 30;
        chunk_sh = (int32_t)ch;
        counters[CTR_CHUNK] = ch;
        counters[CTR_CAND] = (long long)sum;
    }
    __syncthreads();
    const int CH = chunk_sh;
    // items per tile (tiles are processed in slices of 1024 with a running offset)
    uint32_t item_base = 0, slot_base = 0;
    for (int t0 = 0; t0 < ntiles; t0 += 1024) {
        const int t = t0 + threadIdx.x;
        const uint32_t L = t < ntiles ? (uint32_t)tile_L[t] : 0u;
        const uint32_t nk = (L + CH - 1) / CH;
        uint32_t tot_items, tot_slots;
        const uint32_t ex_items = block_excl_scan_1024(nk, tmp, &tot_items);
        const uint32_t ex_slots = block_excl_scan_1024(nk > 1 ? nk : 0u, tmp, &tot_slots);
        if (t < ntiles) tile_slots[t] = make_int2((int)nk, (int)(slot_base + ex_slots));
        for (uint32_t j = 0; j < nk; ++j) {
            const uint64_t it = (uint64_t)item_base + ex_items + j;
            if (it < (uint64_t)max_items) {
                Item e;
                e.tile = t;
                e.chunk = (int32_t)j;
                e.slot = nk > 1 ? (int32_t)(slot_base + ex_slots + j) : -1;
                e.pad = 0;
                items[it] = e;
            }
        }
        item_base += tot_items;
        slot_base += tot_slots;
    }
    if (threadIdx.x == 0) {
        counters[CTR_NITEMS] = (long long)(item_base < max_items ? item_base : max_items);
        counters[CTR_WORK] = 0;
    }
}

hipError_t launch_bin_forward(const Plan &p, const PrepGroup &grp, hipStream_t s)
{
    hipLaunchKernelGGL(k_bin_forward, dim3(grp.n), dim3(1024), 0, s, p.tile_bucket, p.ntiles, grp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Backward binning: chunk b of `chunk` sorted Gaussians reaches the first K_b sorted
// tiles (K_b = tiles whose bucket is at most the chunk's largest bucket).  Those tiles are
// split into ranges of TRB tiles (TRB grows until the items fit max_bitems).  Items are
// ordered range-major -- range r of every chunk that has one, then range r + 1 -- so the
// wavefronts in flight at any time read the same tiles of the field gradient (L2 reuse).
// Because K_b does not increase with b (chunks are sorted by support radius), the chunks
// that have range r form a prefix [0, P_r) and item (r, b) sits at range_base[r] + b.  Bound by
// latency: with the bisection in global memory and a thread writing all of its chunk's items
// 20 chunks took 88 us, 13 now.
// ---------------------------------------------------------------------------------
constexpr int BWD_K_LDS = 4096;
__global__ void __launch_bounds__(1024) k_bin_backward(const int32_t *__restrict__ tile_cum, int max_ranges, PrepGroup grp)
{
    const PrepScene &S = grp.s[blockIdx.x];
    const uint64_t *__restrict__ keys = S.keys_a;
    BItem *__restrict__ bitems = S.bitems;
    int2 *__restrict__ chunk_items = S.chunk_items;
    int32_t *__restrict__ range_base = S.range_base;
    const int64_t max_bitems = S.max_bitems, n = S.g.n;
    long long *__restrict__ counters = S.counters;
    const int chunk = S.chunk;
    __shared__ uint32_t tmp[16];
    __shared__ unsigned long long red[16];
    __shared__ int32_t trb_sh, nr_sh;
    __shared__ int32_t s_K[BWD_K_LDS];
    const int64_t nvalid = n - counters[CTR_NCULLED];
    const int nchunks = (int)((nvalid + chunk - 1) / chunk);
    // K_b of the first chunks (all of them up to 2 million Gaussians) in LDS: the bisection below reads them
    for (int b = threadIdx.x; b < min(nchunks, BWD_K_LDS); b += 1024)
        s_K[b] = tile_cum[bwd_level_bucket(BWD_LEVELS - (int)(keys[(int64_t)b * chunk] >> 42))];
    __syncthreads();
    auto K_of = [&](int b) {
        return b < BWD_K_LDS ? s_K[b] : tile_cum[bwd_level_bucket(BWD_LEVELS - (int)(keys[(int64_t)b * chunk] >> 42))];
    };
    unsigned long long sumK = 0;
    for (int b = threadIdx.x; b < nchunks; b += 1024) sumK += (unsigned long long)K_of(b);
    const unsigned long long sum = block_sum_1024(sumK, red);
    if (threadIdx.x == 0) {
        long long trb = 1;
        // items <= sum / TRB + nchunks <= max_bitems
        const long long room = max_bitems - nchunks;
        if (room > 0) {
            const long long need = (long long)((sum + (unsigned long long)room - 1) / (unsigned long long)room);
            if (need > trb) trb = need;
        } else {
            trb = 1 << 30;
        }
        trb_sh = (int32_t)trb;
        nr_sh = nchunks > 0 ? (int32_t)((K_of(0) + trb - 1) / trb) : 0;
        counters[CTR_TRB] = trb;
    }
    __syncthreads();
    const int TRB = trb_sh, NR = min(nr_sh, max_ranges);
    // P_r = number of chunks with more than r ranges (a prefix, found by bisection)
    uint32_t base = 0;
    for (int r0 = 0; r0 < NR; r0 += 1024) {
        const int r = r0 + threadIdx.x;
        uint32_t P = 0;
        if (r < NR) {
            int lo = 0, hi = nchunks;  // first b with ceil(K_b / TRB) <= r
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((K_of(mid) + TRB - 1) / TRB > r) lo = mid + 1;
                else hi = mid;
            }
            P = (uint32_t)lo;
        }
        uint32_t tot;
        const uint32_t ex = block_excl_scan_1024(P, tmp, &tot);
        if (r < NR) range_base[r] = (int32_t)(base + ex);
        base += tot;
    }
    if (threadIdx.x == 0) range_base[NR] = (int32_t)base;
    __syncthreads();
    for (int b = threadIdx.x; b < nchunks; b += 1024) chunk_items[b] = make_int2(0, min((K_of(b) + TRB - 1) / TRB, NR));
    // items: W threads take the chunks of a range, the work-group's 1024 / W groups its ranges
    int lw = 0;
    while (lw < 10 && (1 << lw) < nchunks) ++lw;
    for (int r = threadIdx.x >> lw; r < NR; r += 1024 >> lw) {
        const int64_t at = range_base[r];
        const int P = range_base[r + 1] - (int)at;
        for (int b = threadIdx.x & ((1 << lw) - 1); b < P; b += 1 << lw)
            if (at + b < max_bitems) {
                BItem e;
                e.chunk = b;
                e.k0 = r * TRB;
                e.k1 = min((r + 1) * TRB, K_of(b));
                e.slot = (int32_t)(at + b);
                bitems[at + b] = e;
            }
    }
    if (threadIdx.x == 0) {
        counters[CTR_NBITEMS] = (long long)(base < max_bitems ? base : max_bitems);
        counters[CTR_BWORK] = 0;
    }
}

hipError_t launch_bin_backward(const Plan &p, const PrepGroup &grp, int max_ranges, hipStream_t s)
{
    hipLaunchKernelGGL(k_bin_backward, dim3(grp.n), dim3(1024), 0, s, p.tile_cum, max_ranges, grp);
    return hipGetLastError();
}

// Scene tables: copy the by-value table to device memory and form the prefix sums of the
// per-scene work-item counts (so one persistent launch can walk every scene's items).
__global__ void k_fwd_table(FwdTab tab, FwdScene *__restrict__ dst, int32_t *__restrict__ prefix,
                            long long *__restrict__ queue)
{
    if (threadIdx.x == 0) {
        int32_t run = 0;
        for (int i = 0; i < tab.n; ++i) {
            dst[i] = tab.s[i];
            prefix[i] = run;
            run += (int32_t)tab.s[i].counters[CTR_NITEMS];
        }
        prefix[tab.n] = run;
        *queue = 0;
    }
}

__global__ void k_bwd_table(BwdTab tab, BwdScene *__restrict__ dst, int32_t *__restrict__ prefix,
                            long long *__restrict__ queue)
{
    if (threadIdx.x == 0) {
        int32_t run = 0;
        for (int i = 0; i < tab.n; ++i) {
            dst[i] = tab.s[i];
            prefix[i] = run;
            run += (int32_t)tab.s[i].counters[CTR_NBITEMS];
        }
        prefix[tab.n] = run;
        *queue = 0;
    }
}

hipError_t launch_fwd_table(const FwdTab &tab, FwdScene *dst, int32_t *prefix, long long *queue, hipStream_t s)
{
    hipLaunchKernelGGL(k_fwd_table, dim3(1), dim3(64), 0, s, tab, dst, prefix, queue);
    return hipGetLastError();
}

hipError_t launch_bwd_table(const BwdTab &tab, BwdScene *dst, int32_t *prefix, long long *queue, hipStream_t s)
{
    hipLaunchKernelGGL(k_bwd_table, dim3(1), dim3(64), 0, s, tab, dst, prefix, queue);
    return hipGetLastError();
}

struct CtrPtrs {
    int n;
    long long *p[MAX_SCENES];
};

// Statistics of a call: counters summed over its scenes.
__global__ void k_sum_counters(CtrPtrs src, long long *__restrict__ dst)
{
    const int t = threadIdx.x;
    if (t < CTR_COUNT) {
        long long v = 0;
        for (int i = 0; i < src.n; ++i) v += src.p[i][t];
        dst[t] = v;
    }
}

hipError_t launch_sum_counters(long long *const *src, int n, long long *dst, hipStream_t s)
{
    CtrPtrs c;
    c.n = n;
    for (int i = 0; i < n && i < MAX_SCENES; ++i) c.p[i] = src[i];
    hipLaunchKernelGGL(k_sum_counters, dim3(1), dim3(64), 0, s, c, dst);
    return hipGetLastError();
}

// Synthetic Gaussians for the autotuner, drawn on the device with a counter-based
// generator (SplitMix64 of seed, index and draw number): means uniform over the field,
// depth U(-10, 10) mm, standard deviations U(2, 20) pixels per axis, rotation U(0, pi),
// opacity U(0.1, 1), amplitudes U(0, 1), phase U(0, 2 pi).
static __device__ __forceinline__ double u01(uint64_t seed, uint64_t i, uint64_t d)
{
    uint64_t z = seed + 0x9e3779b97f4a7c15ull * (i * 16 + d + 1);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

__global__ void k_synth(float *__restrict__ base, int64_t n, uint64_t seed, Consts k)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double PI = 3.14159265358979323846;
    const double W = k.nx * k.px, H = k.ny * k.py;
    const double su = (2.0 + 18.0 * u01(seed, i, 3)) * k.px, sv = (2.0 + 18.0 * u01(seed, i, 4)) * k.py;
    const double th = PI * u01(seed, i, 5);
    const double c = cos(th), s = sin(th);
    float *mx = base, *my = base + n, *z = base + 2 * n, *sxx = base + 3 * n, *sxy = base + 4 * n, *syy = base + 5 * n;
    float *o = base + 6 * n, *ph = base + 7 * n, *amp = base + 8 * n;
    mx[i] = (float)((u01(seed, i, 0) - 0.5) * W);
    my[i] = (float)((u01(seed, i, 1) - 0.5) * H);
    z[i] = (float)((u01(seed, i, 2) - 0.5) * 0.02);
    sxx[i] = (float)(c * c * su * su + s * s * sv * sv);
    sxy[i] = (float)(c * s * (su * su - sv * sv));
    syy[i] = (float)(s * s * su * su + c * c * sv * sv);
    o[i] = (float)(0.1 + 0.9 * u01(seed, i, 6));
    ph[i] = (float)(2.0 * PI * u01(seed, i, 7));
    for (int ch = 0; ch < k.C; ++ch) amp[(int64_t)ch * n + i] = (float)u01(seed, i, 8 + ch);
}

hipError_t launch_synth(GView g, float *base, int64_t n, uint64_t seed, const Consts &k, hipStream_t s)
{
    (void)g;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_synth, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, base, n, seed, k);
    return hipGetLastError();
}

}  // namespace gws
