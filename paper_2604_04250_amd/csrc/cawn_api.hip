// Host side of libcawn: argument checks, workspace layout, the gate's fp32 breakpoints, the lane
// table kernel, the stand-alone Temporal Syntax Cache kernel and the parameter-gradient reduction.
#include <atomic>
#include <cmath>
#include <cstring>
#include <limits>

#include "cawn_internal.hpp"
#include "cawn_gate_host.hpp"

namespace cawn {

static std::atomic<uint32_t> g_spin_limit{1u << 20};   // polls (~1 us each): a second of waiting, far beyond any real wait

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static bool desc_ok(const cawn_desc *d)
{
    if (!d) return false;
    if (d->B <= 0 || d->L < 0 || d->H <= 0 || d->F <= 0) return false;
    if ((int64_t)d->H * d->F > (1 << 24)) return false;
    if (d->conv_k < 0) return false;
    if (d->gate_mode != 0 && d->gate_mode != 1) return false;
    if (d->ret_mode != 0 && d->ret_mode != 1) return false;
    if (d->hconv_k != 0 && d->hconv_k != 3) return false;
    return true;
}

// fwd_only: the layout of a workspace that only forward calls use (the allocation-free entry point):
// published words for the forward's tiles, no backward halo, no partial sums.
static WsLayout make_layout(const cawn_desc *d, bool fwd_only = false)
{
    WsLayout w{};
    w.J = d->H * d->F;
    w.Jp = (int)align_up(w.J, 64);
    w.Jp128 = (int)align_up(w.J, 256);   // covers the widest lane block of any kernel variant
    w.nT = (d->L + BwdGeom::TILE_T - 1) / BwdGeom::TILE_T;      // backward tiles (the finer of the two tilings)
    w.nTc = (d->L + CKPT_T - 1) / CKPT_T;
    const int kc = d->conv_k > MAX_KC ? MAX_KC : d->conv_k;
    const int nT_pub = fwd_only ? (d->L + FwdGeom::TILE_T - 1) / FwdGeom::TILE_T : w.nT;
    const size_t tiles_rows = (size_t)d->B * (nT_pub > 0 ? nT_pub : 1);
    size_t o = sizeof(WsHeader);
    w.off_table = o;
    o = align_up(o + (size_t)lane_rows(kc, d->hconv_k != 0) * w.Jp * sizeof(float), 256);
    w.off_agg = o;      // published words are 8 bytes each: value + tag
    o = align_up(o + tiles_rows * 2 * w.Jp128 * sizeof(tagged_t), 256);
    w.off_pre = o;
    o = align_up(o + tiles_rows * 2 * w.Jp128 * sizeof(tagged_t), 256);
    w.off_halo = o;
    if (!fwd_only) o = align_up(o + tiles_rows * (kc > 1 ? kc - 1 : 0) * 2 * w.Jp128 * sizeof(tagged_t), 256);
    w.off_part = o;
    if (!fwd_only) o = align_up(o + tiles_rows * part_rows(kc, d->hconv_k != 0) * w.Jp128 * sizeof(float), 256);
    w.off_vpart = o;    // gate_mode 1: per-group sums of the valve's gradient terms, [B][groups][L]
    if (d->gate_mode == 1 && !fwd_only)
        o = align_up(o + (size_t)d->B * (size_t)(d->H * (d->F >= 32 ? d->F / 32 : 1)) * (size_t)(d->L > 0 ? d->L : 1) * sizeof(float), 256);
    w.off_aggp = o;     // ret_mode 1: third chained word of a tile's aggregate (product of its retentions)
    if (d->ret_mode == 1) o = align_up(o + tiles_rows * w.Jp128 * sizeof(tagged_t), 256);
    w.off_rpart = o;    // ret_mode 1: per-group sums of the retention logits' gradient terms, [B][groups][L]
    if (d->ret_mode == 1 && !fwd_only)
        o = align_up(o + (size_t)d->B * (size_t)(d->H * (d->F >= 32 ? d->F / 32 : 1)) * (size_t)(d->L > 0 ? d->L : 1) * sizeof(float), 256);
    w.off_dbg = o;
#ifdef CAWN_TIMING
    o += (size_t)MAX_TILES * 16 * sizeof(unsigned long long);
#endif
    w.total = o;
    return w;
}

// lanes of a 32-lane block that share a valve: heads of F >= 32 lanes span whole blocks
static bool valve_shape_ok(const cawn_desc *d) { return d->F % 32 == 0 || d->F == 16 || d->F == 8; }
static int valve_groups(const cawn_desc *d) { return d->H * (d->F >= 32 ? d->F / 32 : 1); }   // per token

// ------------------------------------------------------------------------------------ kernels
// gate_mode 1: dvalve[b][t][h] = sig (1 - sig) * (sum over the head's groups of vpart[b][g][t]),
// sig = sigmoid(valve - 3): the straight-through gradient of Sec. 3.3.  One thread per (b, h, t),
// t fastest; the groups of a head are summed in index order.  valve == nullptr: the plain sum (the
// retention logits' gradient, whose terms already carry their sigmoid factor per lane).  The calling
// threads share the elements: thread `first` of `stride`.  (A call has at most 2^18 tiles of 128 tokens and 4 heads:
// 32-bit indices, whose divisions take a fifth of the instructions of 64-bit ones.)
__device__ __forceinline__ void logit_reduce(const float *__restrict__ vpart, const float *__restrict__ valve,
                                             float *__restrict__ dvalve, uint32_t B, uint32_t L, uint32_t H, uint32_t G,
                                             uint32_t first, uint32_t stride)
{
    const uint32_t n = B * H * L;
    const uint32_t gph = G / H;       // groups per head
    for (uint32_t e = first; e < n; e += stride) {
        const uint32_t r = e / L, t = e - r * L;      // r = b H + h: the head's groups follow each other in vpart
        const uint32_t b = r / H, h = r - b * H;
        const size_t o = ((size_t)b * L + t) * H + h;
        const float vl = valve ? valve[o] : 0.f;      // (asked for with the terms)
        const float *src = vpart + (size_t)r * gph * L + t;
        float sum = 0.f;
        for (uint32_t g = 0; g < gph; g += 8) {
            float x[8];
#pragma unroll
            for (uint32_t q = 0; q < 8; ++q) x[q] = g + q < gph ? src[(size_t)(g + q) * L] : 0.f;
#pragma unroll
            for (uint32_t q = 0; q < 8; ++q) sum += x[q];
        }
        if (valve) {
            const float sg = 1.0f / (1.0f + expf(-(vl - 3.0f)));
            sum *= sg * (1.0f - sg);
        }
        dvalve[o] = sum;
    }
}

__global__ void fill_zero_kernel(uint32_t *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// sin and cos in fp64 of an angle of at most 33 significant bits.  Up to 2^20 radians: two-term Cody-Waite reduction by multiples of pi/2 (the
// fused products round once each, at the size of their result), then the Taylor series to r^17 and r^16, whose next terms
// are below 1e-17 on [-pi/4, pi/4].  (The library's functions carry the reduction of any argument: far more code, which a
// table built between two large kernels fetches anew each time.)
__device__ __forceinline__ void sincos_f64(double x, double &s, double &c)
{
    if (!(__builtin_fabs(x) < 1048576.0)) {
        s = sin(x);
        c = cos(x);
        return;
    }
    const double k = __builtin_rint(x * 0.63661977236758134308);         // 2 / pi
    double r = __builtin_fma(-k, 1.57079632679489661923, x);             // fp64(pi / 2)
    r = __builtin_fma(-k, 6.12323399573676603587e-17, r);                // pi / 2 - fp64(pi / 2)
    const double q = r * r;
    double ps = 1.0 / 355687428096000.0, pc = 1.0 / 20922789888000.0;    // 1 / 17!, 1 / 16!
    const double fs[8] = {1.0, -1.0 / 6, 1.0 / 120, -1.0 / 5040, 1.0 / 362880, -1.0 / 39916800, 1.0 / 6227020800.0, -1.0 / 1307674368000.0};
    const double fc[8] = {1.0, -1.0 / 2, 1.0 / 24, -1.0 / 720, 1.0 / 40320, -1.0 / 3628800, 1.0 / 479001600, -1.0 / 87178291200.0};
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        ps = __builtin_fma(ps, q, fs[i]);
        pc = __builtin_fma(pc, q, fc[i]);
    }
    ps *= r;
    const int n = (int)k & 3;
    s = (n & 1) ? pc : ps;
    c = (n & 1) ? ps : pc;
    s = (n & 2) ? -s : s;
    c = ((n + 1) & 2) ? -c : c;
}

// Every per-lane constant the scan kernels need, formed in fp64.  One thread per (lane, slot): a slot is one power of
// lambda, or one of the values that are copied into the table.  A call's cost is its longest chain of dependent reads and
// arithmetic, all cold behind the kernels of a training step: one thread copying a lane's taps, each read behind the last
// one's store, and library pow, sin and cos took 4.2 - 4.7 us at 120 and 256 lanes and 5.8 - 6.6 us in large steps (an empty
// kernel 1.6); a slot for every value, powers by squaring: 3.3 and 4.7 - 4.8.
// (One thread per lane, working through all powers in turn, took 24 us.)
// gamma == nullptr (data-dependent retention): the table is built with gamma = 1, i.e. its powers
// are pure rotations, and row R_RBIAS receives the static retention bias b_k of the lane's harmonic.
constexpr int LANE_TABLE_POWERS = 3 + FwdGeom::NSEG + BwdGeom::NSEG;
inline int lane_table_slots(int conv_k, bool hconv) { return LANE_TABLE_POWERS + 3 + 2 * conv_k + (hconv ? HC_ROWS : 0); }
__global__ __launch_bounds__(128) void lane_table_kernel(const float *__restrict__ gamma, const float *__restrict__ theta,
                                  const float *__restrict__ conv_w, const float *__restrict__ conv_b,
                                  const float *__restrict__ ret_bias, int F,
                                  const float *__restrict__ hconv_w, const float *__restrict__ hconv_b,
                                  float *__restrict__ table, int J, int Jp, int conv_k)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int slot = blockIdx.y;
    if (j >= Jp) return;
    const bool live = j < J;
    if (slot >= LANE_TABLE_POWERS) {        // copies: retention bias, conv biases, taps, the harmonic convolution's constants
        const int r = slot - LANE_TABLE_POWERS, w0 = 3, h0 = w0 + 2 * conv_k;
        const float *src = nullptr;
        int row = R_RBIAS;
        if (r == 0) {
            if (ret_bias) src = ret_bias + j % F;
        } else if (r < w0) {
            row = r == 1 ? R_BIAS_M : R_BIAS_A;
            if (conv_b && conv_k > 0) src = conv_b + (size_t)(r - 1) * J + j;
        } else if (r < h0) {
            const int q = r - w0, sidx = q >= conv_k ? 1 : 0;
            row = R_W0 + q;
            src = conv_w + ((size_t)sidx * J + j) * conv_k + (q - sidx * conv_k);
        } else {                            // taps [2][H][3] and biases [2][H] of the lane's head
            const int q = r - h0, H = J / F, h = j / F;
            row = R_W0 + 2 * conv_k + q;
            if (q < 6) src = hconv_w + ((size_t)(q / 3) * H + h) * 3 + q % 3;
            else if (hconv_b) src = hconv_b + (size_t)(q - 6) * H + h;
        }
        table[(size_t)row * Jp + j] = live && src ? *src : 0.0f;
        return;
    }
    auto put = [&](int row, double v) { table[(size_t)row * Jp + j] = (float)v; };
    const double g = live ? (gamma ? (double)gamma[j] : 1.0) : 0.0;
    const bool fwd = slot >= 3 && slot - 3 < FwdGeom::NSEG;
    const int sgi = fwd ? slot - 3 : slot - 3 - FwdGeom::NSEG;
    const bool rem64 = fwd && sgi == 0;     // (lambda^0 needs no rows: they hold what fp32 drops of lambda^64)
    const int n = slot == 0 ? 1 : slot == 1 ? FwdGeom::TILE_T : slot == 2 ? BwdGeom::TILE_T : rem64 ? FwdShort::TILE_T
                                                            : sgi * (fwd ? FwdGeom::NSTEP : BwdGeom::NSTEP);
    double c, s;
    sincos_f64(n * (live ? (double)theta[j] : 0.0), s, c);      // (n <= 256: the product is exact)
    // gamma^n by squaring, highest bit of n first, carried as the sum of two fp64 numbers: exact to the last bit of the result
    double m = 1.0, ml = 0.0;
    auto times = [&](double f, double fl) {
        const double p = m * f, e = __builtin_fma(m, f, -p) + __builtin_fma(m, fl, ml * f);
        m = p + e;
        ml = e - (m - p);
    };
    for (int bit = 31 - __builtin_clz(n | 1); bit >= 0; --bit) {     // (n is the same for the whole block)
        times(m, ml);
        if (n >> bit & 1) times(g, 0.0);
    }
    if (!(__builtin_fabs(m) < __builtin_inf())) {       // (the remainder of an infinite product is a NaN: without it)
        m = 1.0;
        for (int bit = 31 - __builtin_clz(n | 1); bit >= 0; --bit) m *= n >> bit & 1 ? m * g : m;
    }
    const double re = m * c, im = m * s;
    if (slot == 0) {
        put(R_LR, re);
        put(R_LI, im);
        put(R_COS, c);
        put(R_SIN, s);
        put(R_GAMMA, g);
    } else if (slot <= 2) {                 // lambda^(tile length) as a double-float: forward, backward
        const float hr = (float)re, hi = (float)im;
        put(slot == 1 ? R_PT_HR : R_PTB_HR, hr);
        put(slot == 1 ? R_PT_HI : R_PTB_HI, hi);
        put(slot == 1 ? R_PT_LR : R_PTB_LR, re - (double)hr);
        put(slot == 1 ? R_PT_LI : R_PTB_LI, im - (double)hi);
    } else if (rem64) {
        put(R_PT64_LR, re - (double)(float)re);
        put(R_PT64_LI, im - (double)(float)im);
    } else {                                // lambda^(segment start): forward segments, then backward segments
        put((fwd ? R_PSEG : R_PSEGB) + 2 * sgi, re);
        put((fwd ? R_PSEG : R_PSEGB) + 2 * sgi + 1, im);
    }
}

// Stand-alone Temporal Syntax Cache: one thread per (V adjacent channels, run of NS tokens).
// Bound by HBM: 4 bytes in, 4 out per element.  V = 4 (16-byte accesses) wherever shapes, strides and pointers allow
// it, single channels otherwise.  The HALO rows before a run are those of the run before it: runs that follow each other
// in time go to the same XCD (workgroup i runs on XCD i mod 8), whose L2 then serves them.  The carried history is
// written by the threads that read it (the first run of each channel), so one launch does everything, also where
// hist_in and hist_out are the same buffer.  B4 L2048 C768: one channel a thread and a second launch for the history
// took 12.4 - 13.3 us; now 10.9 with default-policy stores, 10.1 with streamed ones (5.0 TB/s; runs of 4 and 16 tokens:
// 11.5 and 10.0 us, and 8 leave a short call twice the threads of 16).
constexpr int CONV_NS = 8;      // tokens per thread
template <int V> struct ConvVec;
template <> struct ConvVec<1> { typedef float type; };
template <> struct ConvVec<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <int KC, int V>
__global__ __launch_bounds__(256) void syntax_conv_kernel(const float *__restrict__ x, const float *__restrict__ w,
                                                          const float *__restrict__ bias,
                                                          const float *hist_in, float *__restrict__ y,
                                                          float *hist_out, int L, int C, long long xsb, long long xst,
                                                          long long ysb, long long yst, float cc, unsigned runs, unsigned runs_z)
{
    constexpr int NS = CONV_NS, HALO = KC - 1;
    typedef typename ConvVec<V>::type vec;
    auto at = [](const vec &v, int q) -> float { if constexpr (V == 1) return v; else return v[q]; };
    auto ld = [](const float *p) { return *reinterpret_cast<const vec *>(p); };
    // thread -> (run of tokens, channels), channels fastest; each XCD takes a contiguous eighth of the workgroups
    const unsigned n = gridDim.x, xcd = blockIdx.x % 8u, k8 = blockIdx.x / 8u;
    const unsigned per = n / 8u, rem = n % 8u;
    const unsigned id = xcd * per + (xcd < rem ? xcd : rem) + k8;
    const unsigned e = id * 256u + threadIdx.x, cq = (unsigned)(C / V);
    const unsigned in_z = e / cq, run = blockIdx.z * runs_z + in_z;
    if (in_z >= runs_z || run >= runs) return;
    const int c = (int)(e - in_z * cq) * V, t0 = (int)run * NS;
    const int b = blockIdx.y;
    const float *xb = x + (size_t)b * xsb + c;
    float *yb = y + (size_t)b * ysb + c;
    vec u[NS + HALO];
#pragma unroll
    for (int r = 0; r < NS + HALO; ++r) {
        const int t = t0 - HALO + r;
        vec v = {};
        if (t >= 0 && t < L) v = ld(xb + (size_t)t * xst);
        else if (t < 0 && hist_in && t + HALO >= 0) v = ld(hist_in + ((size_t)b * HALO + (t + HALO)) * C + c);
        u[r] = v;
    }
    float wk[V][KC], bs[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
        bs[q] = bias ? bias[c + q] : 0.0f;
#pragma unroll
        for (int i = 0; i < KC; ++i) wk[q][i] = w[(size_t)(c + q) * KC + i];
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int t = t0 + i;
        if (t >= L) break;
        vec o;
#pragma unroll
        for (int q = 0; q < V; ++q) {
            float z = bs[q];
#pragma unroll
            for (int k = 0; k < KC; ++k) z = __builtin_fmaf(wk[q][k], at(u[i + k], q), z);
            const float zc = clampf(z, cc), r = zc * sigmoid_fast(zc);
            if constexpr (V == 1) o = r; else o[q] = r;
        }
        __builtin_nontemporal_store(o, reinterpret_cast<vec *>(yb + (size_t)t * yst));
    }
    // the last HALO pre-conv rows; what is older than this call comes from hist_in, of which every row my channels
    // have is in u[0 .. HALO-1] already (in place is fine)
    if (HALO > 0 && hist_out && t0 == 0) {
        vec rows[HALO > 0 ? HALO : 1];
#pragma unroll
        for (int q = 0; q < HALO; ++q) {
            const int t = L - HALO + q;
            rows[q] = vec{};
            if (t >= 0) rows[q] = ld(xb + (size_t)t * xst);
            else {
#pragma unroll
                for (int r = 0; r < HALO; ++r)
                    if (r == t + HALO) rows[q] = u[r];
            }
        }
#pragma unroll
        for (int q = 0; q < HALO; ++q) *reinterpret_cast<vec *>(hist_out + ((size_t)b * HALO + q) * C + c) = rows[q];
    }
}

template <int KC>
static void launch_conv(bool vec4, dim3 grid, hipStream_t s, const float *x, const float *w, const float *bias,
                        const float *hist_in, float *y, float *hist_out, int L, int C, long long xsb, long long xst,
                        long long ysb, long long yst, float cc, unsigned runs, unsigned runs_z)
{
    if (vec4) hipLaunchKernelGGL((syntax_conv_kernel<KC, 4>), grid, dim3(256), 0, s, x, w, bias, hist_in, y, hist_out, L, C, xsb, xst, ysb, yst, cc, runs, runs_z);
    else hipLaunchKernelGGL((syntax_conv_kernel<KC, 1>), grid, dim3(256), 0, s, x, w, bias, hist_in, y, hist_out, L, C, xsb, xst, ysb, yst, cc, runs, runs_z);
}

// Sum the backward tiles' parameter partials in a fixed order.  The partials are [lane block][row][chain][32 lanes]
// (chain = position-in-time * B + b): what a block reads is one run of memory.  Block = 8 threads of four lanes each x 32
// groups: group g sums chains g, g+32, ... of its lanes in increasing order, then the 32 sub-sums meet in LDS
// and are added in index order -- the association is fixed, so results are bitwise repeatable.
// (The partials as [chain][lane block][row][32], which a tile writes in one run and a block of 1024 threads read 128 bytes
// at a time, and 64-bit divisions for the logits: B2 L4096 J4096 8.7 us, now 5.4; B8 L8192 J768 5.9, now 5.0; B7 L1024 J256 of
// the paper's layer 4.7, now 4.1.)
constexpr int RG = 32, EPI_NT = 8 * RG;       // groups and threads of a reduction block
typedef float v4f __attribute__((ext_vector_type(4)));
// the sums of group g's chains of four lanes of one (lane block, row): `acc` continues
template <class A>
__device__ __forceinline__ void sum_chains(const float *__restrict__ src, int chains, int g, A (&acc)[4])
{
    auto add = [&](const v4f &v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += (A)v[q];
    };
    // (eight independent reads in flight per thread; the sum keeps its order)
    int c = g;
    for (; c + 7 * RG < chains; c += 8 * RG) {
        v4f v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const v4f *>(src + (size_t)(c + u * RG) * 32);
#pragma unroll
        for (int u = 0; u < 8; ++u) add(v[u]);
    }
    if (c >= chains) return;
    v4f v[7];
#pragma unroll
    for (int u = 0; u < 7; ++u) v[u] = *reinterpret_cast<const v4f *>(src + (size_t)(c + u * RG < chains ? c + u * RG : c) * 32);
#pragma unroll
    for (int u = 0; u < 7; ++u)
        if (c + u * RG < chains) add(v[u]);
}
__device__ __forceinline__ void reduce_partials(const float *__restrict__ part, float *__restrict__ out0,
                                                float *__restrict__ out1, float *__restrict__ out2,
                                                float *__restrict__ out3, int rows, int conv_k,
                                                int J, int chains, int accumulate, int bx,
                                                int row, float (*sm)[33])
{
    // one block per (32 lanes, row): bx, row
    const int l4 = threadIdx.x % 8 * 4, g = threadIdx.x / 8;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    sum_chains(part + ((size_t)bx * rows + row) * chains * 32 + l4, chains, g, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) sm[g][l4 + q] = acc[q];
    __syncthreads();
    const int lane = threadIdx.x, j = bx * 32 + lane;
    if (lane < 32 && j < J) {
        float s = 0.0f;
#pragma unroll
        for (int qq = 0; qq < RG; ++qq) s += sm[qq][lane];
        // rows: 0 dgamma, 1 dtheta, 2 dbias_m, 3 dbias_a, 4 + s*conv_k + i: dw[s][j][i]
        float *dst = nullptr;
        if (row == 0) dst = out0 ? out0 + j : nullptr;
        else if (row == 1) dst = out1 ? out1 + j : nullptr;
        else if (row < 4) dst = out3 ? out3 + (size_t)(row - 2) * J + j : nullptr;
        else {
            const int sidx = row - 4 >= conv_k ? 1 : 0, i = row - 4 - sidx * conv_k;
            dst = out2 ? out2 + ((size_t)sidx * J + j) * conv_k + i : nullptr;
        }
        if (dst) *dst = accumulate ? *dst + s : s;
    }
}

// Harmonic convolution (Sec. 3.6): its taps and biases belong to a (plane, head) channel.  One block per output: q = 0 .. 5
// taps (plane, tap), 6, 7 biases, and head h.  The threads of a group sum its chains over the head's 32-lane blocks, four lanes
// each, the groups meet in LDS in index order and the 32 lane sums (F <= 32: those of the head) in a butterfly of lane
// exchanges (both partners add the same two values): the association is fixed, the result repeatable.  (As a kernel of
// its own behind per-lane sums in memory this cost 4.0 - 4.8 us a call.)
// One output sums up to 8 times the terms of a lane's, and one thread those of all of a head's blocks: in fp32 that added
// to the error (F = 64, L = 8192: 3.7e-7 -> 4.7e-7 of the taps' gradients).  The sums are taken in fp64 and rounded once;
// the reads bound the loop either way.
__device__ __forceinline__ void reduce_hconv(const float *__restrict__ part, float *__restrict__ dw, float *__restrict__ db,
                                             int rows, int hc_row0, int H, int F, int chains,
                                             int accumulate, int q, int h, double (*sm)[33])
{
    const int l4 = threadIdx.x % 8 * 4, g = threadIdx.x / 8;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < (F >= 32 ? F / 32 : 1); ++k)
        sum_chains(part + ((size_t)((h * F) / 32 + k) * rows + hc_row0 + q) * chains * 32 + l4, chains, g, acc);
#pragma unroll
    for (int k = 0; k < 4; ++k) sm[g][l4 + k] = acc[k];
    __syncthreads();
    const int lane = threadIdx.x, l0 = (h * F) % 32;
    if (lane >= 32) return;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < RG; ++k) s += sm[k][lane];
    if (F < 32 && (lane < l0 || lane >= l0 + F)) s = 0.0;
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) s += __shfl_xor(s, o, 32);
    if (lane == 0) {
        float *dst = q < 6 ? (dw ? dw + ((size_t)(q / 3) * H + h) * 3 + q % 3 : nullptr)
                           : (db ? db + (size_t)(q - 6) * H + h : nullptr);
        if (dst) *dst = accumulate ? (float)((double)*dst + s) : (float)s;
    }
}

// What follows the backward kernel, in one launch: blocks [0, nbx * rows_lane) sum the parameter partials, nhc blocks behind them the harmonic convolution's, the
// rest share the logit gradients of the valve and of the retention (nsets of them, nb blocks each).
struct EpilogueArgs {
    const float *part;
    float *out0, *out1, *out2, *out3, *dhw, *dhb;
    int rows, rows_lane, conv_k, J, chains, accumulate, nbx, nhc;
    const float *lpart[2], *logit[2];
    float *lout[2];
    int nsets, nb, B, L, H, F, G;
};
__global__ __launch_bounds__(EPI_NT, 8) void bwd_epilogue_kernel(const EpilogueArgs p)
{
    static_assert(BwdLPR == 32, "reduction blocks take a lane block's 32 lanes");
    __shared__ union { float f[RG][33]; double d[RG][33]; } sm;
    const int nA = p.nbx * p.rows_lane;
    if ((int)blockIdx.x < nA) {
        reduce_partials(p.part, p.out0, p.out1, p.out2, p.out3, p.rows, p.conv_k, p.J, p.chains,
                        p.accumulate, (int)blockIdx.x % p.nbx, (int)blockIdx.x / p.nbx, sm.f);
        return;
    }
    if ((int)blockIdx.x < nA + p.nhc) {
        const int e = (int)blockIdx.x - nA;
        reduce_hconv(p.part, p.dhw, p.dhb, p.rows, p.rows - HC_PART_ROWS, p.H, p.F, p.chains, p.accumulate, e / p.H, e % p.H, sm.d);
        return;
    }
    const int bid = (int)blockIdx.x - nA - p.nhc, set = bid / p.nb, blk = bid % p.nb;
    logit_reduce(p.lpart[set], p.logit[set], p.lout[set], p.B, p.L, p.H, p.G, (uint32_t)blk * blockDim.x + threadIdx.x,
                 (uint32_t)p.nb * blockDim.x);
}

// Plain streaming copy with the forward's traffic shape: two fp32 streams in, two out, 8 bytes read and
// 8 bytes written per element, 16-byte non-temporal accesses, every byte touched once.  What this
// kernel reaches is the practical ceiling of the HBM roofline on the chip at hand; it computes nothing.
// (Of the shapes tried at 50 MB .. 1.2 GB -- grid-stride and slab-per-workgroup, 1/2/4 loads in flight,
// 2 .. 32 workgroups per CU, one element per thread -- this one was at or within 3 % of the best.)
__global__ __launch_bounds__(256) void stream_copy_kernel(const v4f *__restrict__ a0, const v4f *__restrict__ a1,
                                                          v4f *__restrict__ o0, v4f *__restrict__ o1, size_t n4)
{
    constexpr int U = 4;     // independent 16-byte loads in flight per stream and thread
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + (U - 1) * stride < n4; i += U * stride) {
        v4f x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = __builtin_nontemporal_load(a0 + i + u * stride);
            y[u] = __builtin_nontemporal_load(a1 + i + u * stride);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            __builtin_nontemporal_store(x[u], o0 + i + u * stride);
            __builtin_nontemporal_store(y[u], o1 + i + u * stride);
        }
    }
    for (; i < n4; i += stride) {
        o0[i] = a0[i];
        o1[i] = a1[i];
    }
}

static hipError_t build_table(const cawn_desc *d, const WsLayout &w, char *ws, const float *gamma,
                              const float *theta, const float *conv_w, const float *conv_b,
                              const float *ret_bias, hipStream_t s, const float *hconv_w = nullptr,
                              const float *hconv_b = nullptr)
{
    float *table = reinterpret_cast<float *>(ws + w.off_table);
    const int threads = 128;
    hipLaunchKernelGGL(lane_table_kernel, dim3((w.Jp + threads - 1) / threads, lane_table_slots(d->conv_k, hconv_w != nullptr)), dim3(threads), 0, s,
                       gamma, theta, conv_w, conv_b, ret_bias, d->F, hconv_w, hconv_b, table, w.J, w.Jp, d->conv_k);
    return hipGetLastError();
}

static bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace cawn

using namespace cawn;

extern "C" {

size_t cawn_state_bytes(const cawn_desc *d)
{
    if (!desc_ok(d)) return 0;
    const size_t J = (size_t)d->H * d->F;
    const size_t halo = d->conv_k > 1 ? d->conv_k - 1 : 0;
    return (size_t)d->B * 2 * J * sizeof(float) * (1 + halo);
}

size_t cawn_workspace_bytes(const cawn_desc *d)
{
    if (!desc_ok(d)) return 0;
    return make_layout(d).total;
}

size_t cawn_ckpt_bytes(const cawn_desc *d)
{
    if (!desc_ok(d)) return 0;
    const size_t nT = (d->L + CKPT_T - 1) / CKPT_T;
    return (size_t)d->B * nT * 2 * d->H * d->F * sizeof(float);
}

int32_t cawn_tile_len(void) { return CKPT_T; }

const char *cawn_status_string(int st)
{
    switch (st) {
    case CAWN_OK: return "ok";
    case CAWN_EINVAL: return "invalid argument";
    case CAWN_EUNSUPPORTED: return "unsupported configuration";
    case CAWN_EWORKSPACE: return "workspace too small or misaligned";
    case CAWN_ELAUNCH: return "HIP launch or copy failed";
    case CAWN_ETIMEOUT: return "a tile gave up waiting for its predecessor's carry";
    default: return "unknown status";
    }
}

__global__ void init_header_kernel(WsHeader *h, unsigned long long bytes)
{
    h->bytes_lo = (uint32_t)bytes;
    h->bytes_hi = (uint32_t)(bytes >> 32);
}

int cawn_workspace_init(void *workspace, size_t bytes, void *stream)
{
    if (!workspace) return CAWN_EINVAL;
    if (bytes < sizeof(WsHeader) || !aligned(workspace, 256)) return CAWN_EWORKSPACE;
    // the whole buffer: a word counts as published only when its tag matches, and tag 0 never does
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<uint32_t *>(workspace), bytes / sizeof(uint32_t));
    hipLaunchKernelGGL(init_header_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream,
                       reinterpret_cast<WsHeader *>(workspace), (unsigned long long)bytes);
    return hipGetLastError() == hipSuccess ? CAWN_OK : CAWN_ELAUNCH;
}

int cawn_workspace_status(void *workspace, void *stream)
{
    if (!workspace) return CAWN_EINVAL;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return CAWN_ELAUNCH;
    uint32_t err = 0;
    WsHeader *h = reinterpret_cast<WsHeader *>(workspace);
    if (hipMemcpy(&err, &h->error, sizeof(err), hipMemcpyDeviceToHost) != hipSuccess) return CAWN_ELAUNCH;
    if (err) {
        uint32_t zero = 0;
        if (hipMemcpy(&h->error, &zero, sizeof(zero), hipMemcpyHostToDevice) != hipSuccess) return CAWN_ELAUNCH;
        return CAWN_ETIMEOUT;
    }
    return CAWN_OK;
}

void cawn_set_spin_limit(uint32_t polls) { g_spin_limit.store(polls); }

int cawn_theta_init(int32_t H, int32_t F, float *theta_host)
{
    if (H <= 0 || F <= 0 || !theta_host) return CAWN_EINVAL;
    const int64_t J = (int64_t)H * F;
    for (int64_t j = 0; j < J; ++j)
        theta_host[j] = (float)std::pow(10000.0, -2.0 * (double)j / (double)J);
    return CAWN_OK;
}

int cawn_syntax_conv(const cawn_desc *d, int32_t C, const float *x, const float *w, const float *bias,
                     const float *conv_state_in, float *y, float *conv_state_out, void *stream)
{
    if (!d || d->B <= 0 || d->L < 0 || C <= 0 || !w) return CAWN_EINVAL;
    if (d->conv_k < 1) return CAWN_EINVAL;
    if (d->conv_k > MAX_KC) return CAWN_EUNSUPPORTED;
    if (d->L > 0 && (!x || !y)) return CAWN_EINVAL;
    const long long xst = d->in_stride_t ? d->in_stride_t : C, xsb = d->in_stride_b ? d->in_stride_b : (long long)d->L * C;
    const long long yst = d->out_stride_t ? d->out_stride_t : C, ysb = d->out_stride_b ? d->out_stride_b : (long long)d->L * C;
    if (xst < C || yst < C) return CAWN_EINVAL;
    if (d->conv_k == 1) conv_state_out = nullptr;      // no history
    if (d->L == 0 && !conv_state_out) return CAWN_OK;
    // 16-byte accesses: every row of x, y and the histories starts on 16 bytes
    const bool vec4 = C % 4 == 0 && xst % 4 == 0 && xsb % 4 == 0 && yst % 4 == 0 && ysb % 4 == 0 && aligned(x, 16) &&
                      aligned(y, 16) && aligned(conv_state_in, 16) && aligned(conv_state_out, 16);
    const long long runs = d->L > 0 ? ((long long)d->L + CONV_NS - 1) / CONV_NS : 1;     // (no tokens: the history alone)
    const long long cq = vec4 ? C / 4 : C;
    const long long most = 0xffffff00LL / cq;       // threads of one grid row are counted in 32 bits: more runs go to grid.z
    const long long runs_z = runs < most ? runs : most, nz = (runs + runs_z - 1) / runs_z;
    if (nz > 65535 || d->B > 65535) return CAWN_EUNSUPPORTED;
    const dim3 grid((unsigned)((runs_z * cq + 255) / 256), d->B, (unsigned)nz);
    hipStream_t s = (hipStream_t)stream;
    switch (d->conv_k) {
    case 1: launch_conv<1>(vec4, grid, s, x, w, bias, conv_state_in, y, conv_state_out, d->L, C, xsb, xst, ysb, yst, d->conv_clamp, (unsigned)runs, (unsigned)runs_z); break;
    case 2: launch_conv<2>(vec4, grid, s, x, w, bias, conv_state_in, y, conv_state_out, d->L, C, xsb, xst, ysb, yst, d->conv_clamp, (unsigned)runs, (unsigned)runs_z); break;
    case 3: launch_conv<3>(vec4, grid, s, x, w, bias, conv_state_in, y, conv_state_out, d->L, C, xsb, xst, ysb, yst, d->conv_clamp, (unsigned)runs, (unsigned)runs_z); break;
    default: launch_conv<4>(vec4, grid, s, x, w, bias, conv_state_in, y, conv_state_out, d->L, C, xsb, xst, ysb, yst, d->conv_clamp, (unsigned)runs, (unsigned)runs_z); break;
    }
    return hipGetLastError() == hipSuccess ? CAWN_OK : CAWN_ELAUNCH;
}

// The gate's breakpoints depend on four scalars of the descriptor only and cost 60 - 100 fp64 exponentials (1.2 us; the
// valve's threshold 0.5 us): a thread keeps the last ones it computed, by the scalars' bits.
static bool gate_set_of(bool fused, int amp_mode, float conv_clamp, float tau, GateSet *out)
{
    struct Key { uint32_t fused, amp, cc, tau; };
    static thread_local Key last{~0u, 0, 0, 0};
    static thread_local GateSet set;
    Key k{fused ? 1u : 0u, (uint32_t)amp_mode, 0, 0};
    memcpy(&k.cc, &conv_clamp, 4);
    memcpy(&k.tau, &tau, 4);
    if (memcmp(&k, &last, sizeof k) != 0) {
        if (!make_gate_set(fused, amp_mode, (double)conv_clamp, tau, &set)) {
            last.fused = ~0u;
            return false;
        }
        last = k;
    }
    *out = set;
    // The second of two intervals is the increasing end of |A(SiLU(x))| or of |x|: it has no upper end.  Without one, nothing
    // is above a2.
    const float inf = std::numeric_limits<float>::infinity();
    if (!(set.a2 <= set.b2)) out->a2 = std::numeric_limits<float>::quiet_NaN();
    else if (set.b2 != inf) return false;
    return true;
}
static float valve_threshold_of(float eps)
{
    static thread_local bool known = false;
    static thread_local uint32_t last;
    static thread_local float thr;
    uint32_t k;
    memcpy(&k, &eps, 4);
    if (!known || k != last) {
        thr = valve_threshold(eps);
        last = k;
        known = true;
    }
    return thr;
}

// Short tiles (64 tokens, 8 per thread) for calls whose 256-token tiles would leave much of the chip idle: as long as
// every short tile has a workgroup of its own on the chip (4 per compute unit, 1 of twice the threads with the harmonic
// convolution; beyond that a workgroup's second tile, and all draws on one counter, double a call's time), and while a tile's
// way to its carry is not too long.  A short tile reads the aggregates of all tiles before it in its chain, and the tiles of a call
// cost where they start and leave; long tiles cost nearly the same whatever the call.  So the line between them is where
//     (tiles in a chain) x per + (tiles)  =  most,
// set from 394 calls of ten kinds (1 - 64 chains of 6 - 64 short tiles, conv 3).  us a call, long / short tiles, tiles a chain in front:
//   fp32, 2 chains  10: 10.2 / 8.1  36: 11.3 / 10.5  50: 11.2 / 11.7;  12 chains  10: 10.7 / 8.6  24: 11.3 / 10.5  36: 11.9 / 12.4  64: 12.3 / 15.5;
//     24 chains  16: 11.1 / 10.2  36: 12.4 / 15.1;  with valve and retentions, 2 chains  36: 13.2 / 12.2  50: 13.2 / 13.7;  24 chains  16: 13.1 / 12.0  36: 14.4 / 18.4
//   bf16 (long tiles of 64 lanes), 8 chains  36: 12.5 / 12.2, with the valve 50: 13.5 / 13.4;  24 chains  16: 11.9 / 10.0  24: 12.7 / 11.9  36: 13.6 / 15.1
//   harmonic convolution (up to 256 tiles)  4 chains  16: 11.5 / 9.7  50: 13.3 / 13.4  64: 13.6 / 14.8, of the paper's layer 64: 15.5 / 15.5;  16 chains  16: 11.7 / 10.8
// With the harmonic convolution and retentions only the chain's length and the tiles in all bound the choice.  Long / short there (conv 3;
// fp32, fp32 with the valve, bf16 with the valve): 1 chain 64: 13.3 / 14.1, 13.1 / 14.3, 13.5 / 14.5;  2 chains 56: 13.4 / 14.0, 13.5 / 14.2, 13.7 / 14.4  64: 13.6 /
//   14.7, 13.6 / 14.9, 13.7 / 15.0;  4 chains 48: 13.8 / 13.6, 13.9 / 13.8, 14.2 / 13.9  64: 14.1 / 15.4, 14.3 / 15.6, 14.5 / 15.8;  5 chains 51: 15.5 / 14.3, 15.4 / 14.5,
//   15.6 / 14.7;  8 chains 32: 13.6 / 12.5, 13.5 / 12.6, 13.7 / 12.9;  16 chains 16: 12.6 / 11.4, 12.6 / 11.7, 12.8 / 11.5
// A short tile is closer to the exact result where the state reaches far back: it steps 8 instead of 32 tokens by lambda rounded to fp32.  With a
// constant retention up to 0.9999 its outputs' error is 1.8e-7 against 4.1e-7; with retentions from the data 1.2e-7 in both at 0.73, 2.8e-7
// against 4.1e-7 at 0.95 on lanes whose lambda rounds worst.  Calls therefore stay on short tiles to where these used to be ahead of
// long ones (`closer`), although between that line and the one above long tiles are faster, by the figures above.
// The words short tiles publish (aggregates, no prefixes) must fit where the workspace's layout has the long tiles' and,
// behind those, the backward's: always so at cawn_workspace_bytes(); where the array of the allocation-free call is too
// small for them the long tiles stay.
static bool use_short_tiles(const cawn_desc *d, bool bf16, const WsLayout &w, int JB, size_t workspace_bytes)
{
    if (d->hconv_k != 0 && d->F > FwdShortHead::JB) return false;      // (a row is a whole head)
    const size_t nT = ((size_t)d->L + FwdShort::TILE_T - 1) / FwdShort::TILE_T;
    const size_t tiles = (size_t)d->B * nT * (((size_t)w.J + JB - 1) / JB);
    const bool ret = d->ret_mode == 1, hc = d->hconv_k != 0;
    if (nT > (size_t)FwdShort::MAX_CHAIN || tiles > 256u * (hc ? 1 : 4)) return false;
    const size_t per = hc ? 6 : bf16 ? 12 : 17, most = hc ? 510 : bf16 ? 960 : 880;
    const size_t per8 = !ret ? 24 : bf16 ? 16 : 40, most8 = !ret ? 1608 : bf16 ? 1056 : 1480;
    const bool ahead = nT * per + tiles <= most, closer = hc || nT * per8 + tiles <= most8;
    if (!ahead && !closer) return false;
    return w.off_agg + tiles * JB * (ret ? 3 : 2) * sizeof(tagged_t) <= workspace_bytes;
}

static int fwd_impl(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                    const float *ret, const float *ret_bias, const float *gamma, const float *theta, const float *conv_w, const float *conv_b,
                    const void *state_in, float *z_re, float *z_im, void *state_out, void *ckpt,
                    uint32_t *gate_mask, void *workspace, size_t workspace_bytes, void *stream, bool bf16 = false,
                    const float *hconv_w = nullptr, const float *hconv_b = nullptr, bool fwd_only_ws = false)
{
    if (d->conv_k > MAX_KC || (d->amp_mode != 0 && d->amp_mode != 1)) return CAWN_EUNSUPPORTED;
    // the harmonic convolution belongs to its own entry point (which passes the taps)
    if ((d->hconv_k != 0) != (hconv_w != nullptr)) return CAWN_EINVAL;
    // heads are whole inside a 32-lane block, or made of whole blocks (and whole inside the 256 lanes of
    // a short call's workgroup)
    if (d->hconv_k != 0 && !(d->F <= 32 ? 32 % d->F == 0 : (d->F % 32 == 0 && 256 % d->F == 0))) return CAWN_EUNSUPPORTED;
    if (d->hconv_k != 0 && (d->gate_mode == 1 || d->ret_mode == 1) && d->F < 32) return CAWN_EUNSUPPORTED;   // LDS
    if ((d->gate_mode == 1 || d->ret_mode == 1) && !valve_shape_ok(d)) return CAWN_EUNSUPPORTED;
    if (d->gate_mode == 1 && d->ret_mode == 1 && d->F < 16) return CAWN_EUNSUPPORTED;   // LDS for both logit tiles
    hipStream_t s = (hipStream_t)stream;
    const WsLayout w = make_layout(d, fwd_only_ws);
    const long long J = w.J;
    if (d->L == 0) {   // nothing to scan: the state passes through
        if (state_out && state_out != state_in) {
            const size_t nb = cawn_state_bytes(d);
            hipError_t e;
            if (state_in) {
                e = hipMemcpyAsync(state_out, state_in, nb, hipMemcpyDeviceToDevice, s);
            } else {   // a fill kernel rather than a memset node: safe under graph capture
                hipLaunchKernelGGL(fill_zero_kernel, dim3(64), dim3(256), 0, s,
                                   reinterpret_cast<uint32_t *>(state_out), nb / sizeof(uint32_t));
                e = hipGetLastError();
            }
            if (e != hipSuccess) return CAWN_ELAUNCH;
        }
        return CAWN_OK;
    }
    if (!mag || !ang || !theta || !z_re || !z_im || !workspace) return CAWN_EINVAL;
    if (d->ret_mode == 1 ? (!ret || !ret_bias) : !gamma) return CAWN_EINVAL;
    if (d->gate_mode == 1 && !valve) return CAWN_EINVAL;
    if (d->conv_k > 0 && !conv_w) return CAWN_EINVAL;
    // tile indices and tickets are bounded: B x (tiles per sequence) x (32-lane blocks) <= 2^18 per call
    if ((unsigned long long)d->B * ((d->L + FwdGeom::TILE_T - 1) / FwdGeom::TILE_T) * ((J + FwdGeom::JB - 1) / FwdGeom::JB) > MAX_TILES)
        return CAWN_EUNSUPPORTED;
    if (workspace_bytes < w.total || !aligned(workspace, 256)) return CAWN_EWORKSPACE;
    const long long ist = d->in_stride_t ? d->in_stride_t : J, isb = d->in_stride_b ? d->in_stride_b : (long long)d->L * J;
    const long long ost = d->out_stride_t ? d->out_stride_t : J, osb = d->out_stride_b ? d->out_stride_b : (long long)d->L * J;
    if (ist < J || ost < J || isb < 0 || osb < 0) return CAWN_EINVAL;
    if (ist > (1ll << 21) || ost > (1ll << 21)) return CAWN_EUNSUPPORTED;   // in-tile offsets are 32-bit
    // bf16 rows are staged as four-byte words: an even number of lanes, even strides, aligned rows
    if (bf16 && (J % 2 || ist % 2 || isb % 2 || !aligned(mag, 4) || !aligned(ang, 4))) return CAWN_EUNSUPPORTED;

    FwdArgs a{};
    a.bf16 = bf16 ? 1 : 0;
    a.hconv = d->hconv_k != 0 ? 1 : 0;
    if (d->gate_mode == 1) {
        const float INF = std::numeric_limits<float>::infinity();
        a.gs = GateSet{-INF, INF, INF, -INF};        // no per-lane threshold in this mode
        a.valve = valve;
        a.valve_thr = valve_threshold_of(d->valve_eps);
    } else if (!gate_set_of(d->conv_k > 0, d->amp_mode, d->conv_clamp, d->gate_tau, &a.gs)) {
        return CAWN_EUNSUPPORTED;
    }
    // the tile: 32-lane rows, with the harmonic convolution 64-lane rows (the same number of token-lanes)
    const bool short_tiles = use_short_tiles(d, bf16, w, hconv_w ? FwdHead::JB : FwdGeom::JB, workspace_bytes);
    const bool head = hconv_w || (bf16 && !short_tiles);
    const bool wide = hconv_w && d->F > FwdHead::JB;      // 128 or 256: a row is a head
    static_assert(FwdWide128::TILE_T == 64 && FwdWide256::TILE_T == 64, "");
    const int JB = wide ? d->F : head ? FwdHead::JB : FwdGeom::JB;
    const int TT = short_tiles ? FwdShort::TILE_T : wide ? FwdWide128::TILE_T : (head ? FwdHead::TILE_T : FwdGeom::TILE_T);
    a.short_tiles = short_tiles ? 1 : 0;
    a.H = d->H; a.F = d->F;
    a.gpb = d->F >= JB ? (d->F % JB ? 2 : 1) : JB / d->F;
    if (d->ret_mode == 1) {
        a.ret = ret;
        a.aggp = reinterpret_cast<tagged_t *>(reinterpret_cast<char *>(workspace) + w.off_aggp);
    }
    const int nLB = (int)((J + JB - 1) / JB);
    const int nTf = (d->L + TT - 1) / TT;
    const size_t tiles = (size_t)d->B * nTf * nLB;

    char *ws = reinterpret_cast<char *>(workspace);
    if (!d->lane_consts_cached) {
        if (build_table(d, w, ws, d->ret_mode == 1 ? nullptr : gamma, theta, conv_w, conv_b,
                        d->ret_mode == 1 ? ret_bias : nullptr, s, hconv_w, hconv_b) != hipSuccess) return CAWN_ELAUNCH;
    }
    a.mag = mag; a.ang = ang;
    a.table = reinterpret_cast<const float *>(ws + w.off_table);
    a.state_in = reinterpret_cast<const float *>(state_in);
    a.z_re = z_re; a.z_im = z_im;
    a.state_out = reinterpret_cast<float *>(state_out);
    a.ckpt = reinterpret_cast<float *>(ckpt);
    a.mask = gate_mask;
    a.hdr = reinterpret_cast<WsHeader *>(ws);
    a.agg = reinterpret_cast<tagged_t *>(ws + w.off_agg);
    a.pre = reinterpret_cast<tagged_t *>(ws + w.off_pre);
    if (short_tiles) {      // aggregates only, the products behind them: the layout's later regions are the backward's
        a.pre = nullptr;
        a.aggp = a.agg + tiles * 2 * JB;
    }
    if (wide) {             // twice the tiles the layout's regions are for: aggregates, prefixes and products in a row
        a.pre = a.agg + tiles * 2 * JB;
        a.aggp = a.pre + tiles * 2 * JB;
        if (w.off_agg + tiles * JB * (d->ret_mode == 1 ? 5 : 4) * sizeof(tagged_t) > workspace_bytes) return CAWN_EWORKSPACE;
    }
    a.clear_from = w.off_agg;
    a.B = d->B; a.L = d->L; a.J = (int)J; a.Jp = w.Jp; a.nT = nTf; a.nTc = w.nTc; a.nLB = nLB;
    a.amp_mode = d->amp_mode;
    a.small_angle = (d->conv_k > 0 && d->conv_clamp <= 256.0f) ? 1 : 0;   // |angle| <= SiLU(clamp) <= 41 revolutions
    a.stage16 = (J % 4 == 0 && ist % 4 == 0 && isb % 4 == 0 && aligned(mag, 16) && aligned(ang, 16) &&
                 (!state_in || aligned(state_in, 16))) ? 1 : 0;
    if (bf16) a.stage16 = (J % 8 == 0 && ist % 8 == 0 && isb % 8 == 0 && aligned(mag, 16) && aligned(ang, 16)) ? 1 : 0;
    a.isb = isb; a.ist = ist; a.osb = osb; a.ost = ost;
    a.conv_clamp = d->conv_clamp; a.out_clamp = d->out_clamp;
    a.spin_limit = g_spin_limit.load();
    a.total_tiles = (uint32_t)tiles;
    a.dbg = reinterpret_cast<unsigned long long *>(ws + w.off_dbg);
    if (launch_fwd(a, d->conv_k, s) != hipSuccess) return CAWN_ELAUNCH;
    return CAWN_OK;
}

int cawn_phase_accumulate_fwd(const cawn_desc *d, const float *mag, const float *ang, const float *gamma,
                              const float *theta, const float *conv_w, const float *conv_b,
                              const void *state_in, float *z_re, float *z_im, void *state_out, void *ckpt,
                              uint32_t *gate_mask, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->gate_mode != 0 || d->ret_mode != 0) return CAWN_EINVAL;      // those modes have entry points of their own
    return fwd_impl(d, mag, ang, nullptr, nullptr, nullptr, gamma, theta, conv_w, conv_b, state_in, z_re, z_im, state_out, ckpt,
                    gate_mask, workspace, workspace_bytes, stream);
}

int cawn_phase_accumulate_valve_fwd(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                                    const float *gamma, const float *theta, const float *conv_w,
                                    const float *conv_b, const void *state_in, float *z_re, float *z_im,
                                    void *state_out, void *ckpt, uint32_t *gate_mask, void *workspace,
                                    size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->gate_mode != 1 || d->ret_mode != 0) return CAWN_EINVAL;
    return fwd_impl(d, mag, ang, valve, nullptr, nullptr, gamma, theta, conv_w, conv_b, state_in, z_re, z_im,
                    state_out, ckpt, gate_mask, workspace, workspace_bytes, stream);
}

int cawn_phase_accumulate_ret_fwd(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                                  const float *ret, const float *ret_bias, const float *theta,
                                  const float *conv_w, const float *conv_b, const void *state_in, float *z_re,
                                  float *z_im, void *state_out, void *ckpt, uint32_t *gate_mask, void *workspace,
                                  size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->ret_mode != 1) return CAWN_EINVAL;
    return fwd_impl(d, mag, ang, d->gate_mode == 1 ? valve : nullptr, ret, ret_bias, nullptr, theta, conv_w, conv_b,
                    state_in, z_re, z_im, state_out, ckpt, gate_mask, workspace, workspace_bytes, stream);
}

static int bwd_impl(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                    const float *ret, const float *ret_bias,
                    const float *gamma, const float *theta, const float *conv_w, const float *conv_b,
                    const void *state_in, const void *ckpt, const float *dz_re, const float *dz_im,
                    const void *dstate_out, float *dmag, float *dang, float *dvalve, float *dret, float *dgamma,
                    float *dtheta, float *dconv_w, float *dconv_b, void *dstate_in, void *workspace,
                    size_t workspace_bytes, void *stream, bool bf16 = false, const float *hconv_w = nullptr,
                    const float *hconv_b = nullptr, float *dhconv_w = nullptr, float *dhconv_b = nullptr)
{
    if (d->conv_k > MAX_KC || (d->amp_mode != 0 && d->amp_mode != 1)) return CAWN_EUNSUPPORTED;
    // gradients of the convolved output: the harmonic convolution's own entry point only
    const bool hc = d->hconv_k != 0;
    if (hc != (hconv_w != nullptr)) return CAWN_EINVAL;
    if (hc && !(d->F <= 32 ? 32 % d->F == 0 : (d->F % 32 == 0 && 256 % d->F == 0))) return CAWN_EUNSUPPORTED;   // as in the forward
    if (hc && (d->gate_mode == 1 || d->ret_mode == 1) && d->F < 32) return CAWN_EUNSUPPORTED;                   // as in the forward
    if ((d->gate_mode == 1 || d->ret_mode == 1) && !valve_shape_ok(d)) return CAWN_EUNSUPPORTED;
    if (d->gate_mode == 1 && d->ret_mode == 1 && d->F < 16) return CAWN_EUNSUPPORTED;   // as in the forward
    hipStream_t s = (hipStream_t)stream;
    const WsLayout w = make_layout(d);
    const long long J = w.J;
    const int kc = d->conv_k;
    const bool want_w = kc > 0 && (dconv_w || dconv_b);
    // (the retention kernels rebuild the forward state in any case and always emit their partials)
    // (the harmonic convolution's tap gradients need the clamped state: state rebuilt, partials always emitted)
    const bool want_param = dgamma || dtheta || want_w || d->ret_mode == 1 || hc;
    if (d->L == 0) {   // no tokens: the state gradient passes through, parameter gradients are zero
        auto zero = [&](void *p, size_t nfloat) {
            if (!p || !nfloat) return hipSuccess;
            hipLaunchKernelGGL(fill_zero_kernel, dim3(64), dim3(256), 0, s, reinterpret_cast<uint32_t *>(p), nfloat);
            return hipGetLastError();
        };
        const size_t nb = cawn_state_bytes(d);
        hipError_t e = hipSuccess;
        if (dstate_in && dstate_in != dstate_out)
            e = dstate_out ? hipMemcpyAsync(dstate_in, dstate_out, nb, hipMemcpyDeviceToDevice, s)
                           : zero(dstate_in, nb / 4);
        if (e == hipSuccess && !d->accumulate_param_grads) {
            e = zero(dgamma, J);
            if (e == hipSuccess) e = zero(dtheta, J);
            if (e == hipSuccess && kc > 0) e = zero(dconv_w, 2 * J * kc);
            if (e == hipSuccess && kc > 0) e = zero(dconv_b, 2 * J);
            if (e == hipSuccess && hc) e = zero(dhconv_w, (size_t)2 * d->H * 3);
            if (e == hipSuccess && hc) e = zero(dhconv_b, (size_t)2 * d->H);
        }
        return e == hipSuccess ? CAWN_OK : CAWN_ELAUNCH;
    }
    if (!mag || !ang || !theta || !dz_re || !dz_im || !dmag || !dang || !workspace) return CAWN_EINVAL;
    if (d->ret_mode == 1 ? (!ret || !ret_bias || dgamma) : !gamma) return CAWN_EINVAL;
    if (d->gate_mode == 1 && !valve) return CAWN_EINVAL;
    if (kc > 0 && !conv_w) return CAWN_EINVAL;
    if ((dgamma || dtheta || d->ret_mode == 1 || hc) && !ckpt) return CAWN_EINVAL;
    // tile indices and tickets are bounded: B x (tiles per sequence) x (32-lane blocks) <= 2^18 per call
    if ((unsigned long long)d->B * w.nT * ((J + BwdLPR - 1) / BwdLPR) > MAX_TILES) return CAWN_EUNSUPPORTED;
    if (workspace_bytes < w.total || !aligned(workspace, 256)) return CAWN_EWORKSPACE;
    const long long ist = d->in_stride_t ? d->in_stride_t : J, isb = d->in_stride_b ? d->in_stride_b : (long long)d->L * J;
    const long long ost = d->out_stride_t ? d->out_stride_t : J, osb = d->out_stride_b ? d->out_stride_b : (long long)d->L * J;
    if (ist < J || ost < J || isb < 0 || osb < 0) return CAWN_EINVAL;
    if (ist > (1ll << 21) || ost > (1ll << 21)) return CAWN_EUNSUPPORTED;   // in-tile offsets are 32-bit
    // bf16 rows are staged as four-byte words: an even number of lanes, even strides, aligned rows
    if (bf16 && (J % 2 || ist % 2 || isb % 2 || ost % 2 || osb % 2 || !aligned(mag, 4) || !aligned(ang, 4) ||
                 !aligned(dz_re, 4) || !aligned(dz_im, 4))) return CAWN_EUNSUPPORTED;

    BwdArgs a{};
    a.bf16 = bf16 ? 1 : 0;
    if (d->gate_mode == 1) {
        const float INF = std::numeric_limits<float>::infinity();
        a.gs = GateSet{-INF, INF, INF, -INF};        // no per-lane threshold in this mode
        a.valve = valve;
        a.valve_thr = valve_threshold_of(d->valve_eps);
        a.vpart = dvalve ? reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + w.off_vpart) : nullptr;
    } else if (!gate_set_of(d->conv_k > 0, d->amp_mode, d->conv_clamp, d->gate_tau, &a.gs)) {
        return CAWN_EUNSUPPORTED;
    }
    a.H = d->H; a.F = d->F;
    a.gpb = d->F >= 32 ? 1 : 32 / d->F;
    a.G = valve_groups(d);
    if (d->ret_mode == 1) {
        a.ret = ret;
        a.rpart = dret ? reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + w.off_rpart) : nullptr;
        a.aggp = reinterpret_cast<tagged_t *>(reinterpret_cast<char *>(workspace) + w.off_aggp);
    }
    const bool vec = (J % BwdV == 0) && (ist % BwdV == 0) && (isb % BwdV == 0) && (ost % BwdV == 0) &&
                     (osb % BwdV == 0) && aligned(mag, 8) && aligned(ang, 8) && aligned(dz_re, 8) &&
                     aligned(dz_im, 8) && aligned(dmag, 8) && aligned(dang, 8) &&
                     (!state_in || aligned(state_in, 8)) && (!ckpt || aligned(ckpt, 8)) &&
                     (!dstate_out || aligned(dstate_out, 8)) && (!dstate_in || aligned(dstate_in, 8));
    const int JB = (vec ? BwdV : 1) * BwdLPR;
    const int nLB = (int)((J + JB - 1) / JB);
    const size_t tiles = (size_t)d->B * w.nT * nLB;
    if (tiles > MAX_TILES) return CAWN_EUNSUPPORTED;

    char *ws = reinterpret_cast<char *>(workspace);
    if (!d->lane_consts_cached) {
        if (build_table(d, w, ws, d->ret_mode == 1 ? nullptr : gamma, theta, conv_w, conv_b,
                        d->ret_mode == 1 ? ret_bias : nullptr, s, hconv_w, hconv_b) != hipSuccess) return CAWN_ELAUNCH;
    }
    a.hconv = hc ? 1 : 0;
    a.out_clamp = d->out_clamp;
    a.mag = mag; a.ang = ang; a.dz_re = dz_re; a.dz_im = dz_im;
    a.table = reinterpret_cast<const float *>(ws + w.off_table);
    a.state_in = reinterpret_cast<const float *>(state_in);
    a.ckpt = reinterpret_cast<const float *>(ckpt);
    a.dstate_out = reinterpret_cast<const float *>(dstate_out);
    a.dmag = dmag; a.dang = dang;
    a.dstate_in = reinterpret_cast<float *>(dstate_in);
    a.hdr = reinterpret_cast<WsHeader *>(ws);
    a.agg = reinterpret_cast<tagged_t *>(ws + w.off_agg);
    a.pre = reinterpret_cast<tagged_t *>(ws + w.off_pre);
    a.clear_from = w.off_agg;
    a.halo = reinterpret_cast<tagged_t *>(ws + w.off_halo);
    a.part = reinterpret_cast<float *>(ws + w.off_part);
    a.B = d->B; a.L = d->L; a.J = (int)J; a.Jp = w.Jp; a.nT = w.nT; a.nTc = w.nTc; a.nLB = nLB;
    a.amp_mode = d->amp_mode; a.want_param = want_param ? 1 : 0;
    a.small_angle = (kc > 0 && d->conv_clamp <= 256.0f) ? 1 : 0;
    a.stage16 = (J % 4 == 0 && ist % 4 == 0 && isb % 4 == 0 && aligned(mag, 16) && aligned(ang, 16) &&
                 (!state_in || aligned(state_in, 16))) ? 1 : 0;
    if (bf16) a.stage16 = (J % 8 == 0 && ist % 8 == 0 && isb % 8 == 0 && aligned(mag, 16) && aligned(ang, 16)) ? 1 : 0;
    const long long zq = bf16 ? 8 : 4;       // elements per 16 bytes
    a.stage16z = (J % zq == 0 && ost % zq == 0 && osb % zq == 0 && aligned(dz_re, 16) && aligned(dz_im, 16)) ? 1 : 0;
    a.isb = isb; a.ist = ist; a.osb = osb; a.ost = ost;
    a.conv_clamp = d->conv_clamp; a.grad_clamp = d->grad_clamp;
    a.spin_limit = g_spin_limit.load();
    a.total_tiles = (uint32_t)tiles;
    a.dbg = reinterpret_cast<unsigned long long *>(ws + w.off_dbg);
    if (launch_bwd(a, kc, vec, s) != hipSuccess) return CAWN_ELAUNCH;
    {
        EpilogueArgs p{};
        p.rows = part_rows(kc, hc);
        if (dgamma || dtheta || want_w) {
            p.rows_lane = part_rows(kc);
            p.nbx = (int)((J + 31) / 32);
        }
        p.part = a.part;
        p.out0 = dgamma; p.out1 = dtheta; p.out2 = dconv_w; p.out3 = dconv_b; p.dhw = dhconv_w; p.dhb = dhconv_b;
        p.nhc = hc && (dhconv_w || dhconv_b) ? HC_PART_ROWS * d->H : 0;
        p.conv_k = kc > 0 ? kc : 1;
        p.J = (int)J; p.chains = d->B * w.nT; p.accumulate = d->accumulate_param_grads;
        p.F = d->F;
        if (a.vpart) { p.lpart[p.nsets] = a.vpart; p.logit[p.nsets] = valve; p.lout[p.nsets] = dvalve; ++p.nsets; }
        if (a.rpart) { p.lpart[p.nsets] = a.rpart; p.logit[p.nsets] = nullptr; p.lout[p.nsets] = dret; ++p.nsets; }
        const long long n = (long long)d->B * d->H * d->L;
        const long long nb = (n + EPI_NT - 1) / EPI_NT;
        p.nb = p.nsets ? (int)(nb < 4096 ? nb : 4096) : 0;
        p.B = d->B; p.L = d->L; p.H = d->H; p.G = a.G;
        const unsigned blocks = (unsigned)(p.nbx * p.rows_lane + p.nhc + p.nb * p.nsets);
        if (blocks) {
            hipLaunchKernelGGL(bwd_epilogue_kernel, dim3(blocks), dim3(EPI_NT), 0, s, p);
            if (hipGetLastError() != hipSuccess) return CAWN_ELAUNCH;
        }
    }
    return CAWN_OK;
}

int cawn_phase_accumulate_bwd(const cawn_desc *d, const float *mag, const float *ang, const float *gamma,
                              const float *theta, const float *conv_w, const float *conv_b,
                              const void *state_in, const void *ckpt, const float *dz_re, const float *dz_im,
                              const void *dstate_out, float *dmag, float *dang, float *dgamma, float *dtheta,
                              float *dconv_w, float *dconv_b, void *dstate_in, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->gate_mode != 0 || d->ret_mode != 0) return CAWN_EINVAL;      // those modes have entry points of their own
    return bwd_impl(d, mag, ang, nullptr, nullptr, nullptr, gamma, theta, conv_w, conv_b, state_in, ckpt, dz_re, dz_im, dstate_out,
                    dmag, dang, nullptr, nullptr, dgamma, dtheta, dconv_w, dconv_b, dstate_in, workspace, workspace_bytes,
                    stream);
}

int cawn_phase_accumulate_valve_bwd(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                                    const float *gamma, const float *theta, const float *conv_w,
                                    const float *conv_b, const void *state_in, const void *ckpt,
                                    const float *dz_re, const float *dz_im, const void *dstate_out, float *dmag,
                                    float *dang, float *dvalve, float *dgamma, float *dtheta, float *dconv_w,
                                    float *dconv_b, void *dstate_in, void *workspace, size_t workspace_bytes,
                                    void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->gate_mode != 1 || d->ret_mode != 0) return CAWN_EINVAL;
    return bwd_impl(d, mag, ang, valve, nullptr, nullptr, gamma, theta, conv_w, conv_b, state_in, ckpt, dz_re, dz_im,
                    dstate_out, dmag, dang, dvalve, nullptr, dgamma, dtheta, dconv_w, dconv_b, dstate_in, workspace,
                    workspace_bytes, stream);
}

int cawn_phase_accumulate_bf16_fwd(const cawn_desc *d, const uint16_t *mag, const uint16_t *ang, const float *valve,
                                   const float *ret, const float *ret_bias, const float *gamma, const float *theta,
                                   const float *conv_w, const float *conv_b, const void *state_in, uint16_t *z_re,
                                   uint16_t *z_im, void *state_out, void *ckpt, uint32_t *gate_mask, void *workspace,
                                   size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    return fwd_impl(d, reinterpret_cast<const float *>(mag), reinterpret_cast<const float *>(ang),
                    d->gate_mode == 1 ? valve : nullptr, d->ret_mode == 1 ? ret : nullptr,
                    d->ret_mode == 1 ? ret_bias : nullptr, d->ret_mode == 1 ? nullptr : gamma, theta, conv_w, conv_b,
                    state_in, reinterpret_cast<float *>(z_re), reinterpret_cast<float *>(z_im), state_out, ckpt,
                    gate_mask, workspace, workspace_bytes, stream, true);
}

int cawn_phase_accumulate_hconv_fwd(const cawn_desc *d, const void *mag, const void *ang, const float *valve,
                                    const float *ret, const float *ret_bias, const float *gamma, const float *theta,
                                    const float *conv_w, const float *conv_b, const float *hconv_w,
                                    const float *hconv_b, const void *state_in, void *zc_re, void *zc_im,
                                    void *state_out, void *ckpt, uint32_t *gate_mask, void *workspace,
                                    size_t workspace_bytes, int32_t activations_bf16, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->hconv_k != 3 || !hconv_w) return CAWN_EINVAL;
    return fwd_impl(d, reinterpret_cast<const float *>(mag), reinterpret_cast<const float *>(ang),
                    d->gate_mode == 1 ? valve : nullptr, d->ret_mode == 1 ? ret : nullptr,
                    d->ret_mode == 1 ? ret_bias : nullptr, d->ret_mode == 1 ? nullptr : gamma, theta, conv_w, conv_b,
                    state_in, reinterpret_cast<float *>(zc_re), reinterpret_cast<float *>(zc_im), state_out, ckpt,
                    gate_mask, workspace, workspace_bytes, stream, activations_bf16 != 0, hconv_w, hconv_b);
}

int cawn_phase_accumulate_hconv_bwd(const cawn_desc *d, const void *mag, const void *ang, const float *valve,
                                    const float *ret, const float *ret_bias, const float *gamma, const float *theta,
                                    const float *conv_w, const float *conv_b, const float *hconv_w, const float *hconv_b,
                                    const void *state_in, const void *ckpt, const void *dc_re, const void *dc_im,
                                    const void *dstate_out, void *dmag, void *dang, float *dvalve, float *dret,
                                    float *dgamma, float *dtheta, float *dconv_w, float *dconv_b, float *dhconv_w,
                                    float *dhconv_b, void *dstate_in, void *workspace, size_t workspace_bytes,
                                    int32_t activations_bf16, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->hconv_k != 3 || !hconv_w) return CAWN_EINVAL;
    const bool valved = d->gate_mode == 1, rmode = d->ret_mode == 1;
    return bwd_impl(d, reinterpret_cast<const float *>(mag), reinterpret_cast<const float *>(ang),
                    valved ? valve : nullptr, rmode ? ret : nullptr, rmode ? ret_bias : nullptr, rmode ? nullptr : gamma,
                    theta, conv_w, conv_b, state_in, ckpt, reinterpret_cast<const float *>(dc_re),
                    reinterpret_cast<const float *>(dc_im), dstate_out, reinterpret_cast<float *>(dmag),
                    reinterpret_cast<float *>(dang), valved ? dvalve : nullptr, rmode ? dret : nullptr, dgamma, dtheta,
                    dconv_w, dconv_b, dstate_in, workspace, workspace_bytes, stream, activations_bf16 != 0, hconv_w,
                    hconv_b, dhconv_w, dhconv_b);
}

int cawn_phase_accumulate_bf16_bwd(const cawn_desc *d, const uint16_t *mag, const uint16_t *ang, const float *valve,
                                   const float *ret, const float *ret_bias, const float *gamma, const float *theta,
                                   const float *conv_w, const float *conv_b, const void *state_in, const void *ckpt,
                                   const uint16_t *dz_re, const uint16_t *dz_im, const void *dstate_out, uint16_t *dmag,
                                   uint16_t *dang, float *dvalve, float *dret, float *dgamma, float *dtheta,
                                   float *dconv_w, float *dconv_b, void *dstate_in, void *workspace,
                                   size_t workspace_bytes, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    const bool valved = d->gate_mode == 1, rmode = d->ret_mode == 1;
    return bwd_impl(d, reinterpret_cast<const float *>(mag), reinterpret_cast<const float *>(ang),
                    valved ? valve : nullptr, rmode ? ret : nullptr, rmode ? ret_bias : nullptr,
                    rmode ? nullptr : gamma, theta, conv_w, conv_b, state_in, ckpt,
                    reinterpret_cast<const float *>(dz_re), reinterpret_cast<const float *>(dz_im), dstate_out,
                    reinterpret_cast<float *>(dmag), reinterpret_cast<float *>(dang), valved ? dvalve : nullptr,
                    rmode ? dret : nullptr, rmode ? nullptr : dgamma, dtheta, dconv_w, dconv_b, dstate_in, workspace,
                    workspace_bytes, stream, true);
}

int cawn_phase_accumulate_ret_bwd(const cawn_desc *d, const float *mag, const float *ang, const float *valve,
                                  const float *ret, const float *ret_bias, const float *theta,
                                  const float *conv_w, const float *conv_b, const void *state_in, const void *ckpt,
                                  const float *dz_re, const float *dz_im, const void *dstate_out, float *dmag,
                                  float *dang, float *dvalve, float *dret, float *dtheta, float *dconv_w,
                                  float *dconv_b, void *dstate_in, void *workspace, size_t workspace_bytes,
                                  void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->ret_mode != 1) return CAWN_EINVAL;
    const bool valved = d->gate_mode == 1;
    return bwd_impl(d, mag, ang, valved ? valve : nullptr, ret, ret_bias, nullptr, theta, conv_w, conv_b, state_in,
                    ckpt, dz_re, dz_im, dstate_out, dmag, dang, valved ? dvalve : nullptr, dret, nullptr, dtheta,
                    dconv_w, dconv_b, dstate_in, workspace, workspace_bytes, stream);
}

int cawn_stream_copy(const float *in0, const float *in1, float *out0, float *out1, size_t n, void *stream)
{
    if (!in0 || !in1 || !out0 || !out1) return CAWN_EINVAL;
    if (n % 4 || !aligned(in0, 16) || !aligned(in1, 16) || !aligned(out0, 16) || !aligned(out1, 16)) return CAWN_EUNSUPPORTED;
    if (n == 0) return CAWN_OK;
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return CAWN_ELAUNCH;
        cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
    }
    const size_t n4 = n / 4;
    size_t blocks = (n4 + 255) / 256;
    const size_t resident = (size_t)cus * 2;       // two workgroups of 4 waves per CU
    if (blocks > resident) blocks = resident;
    hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<const v4f *>(in0), reinterpret_cast<const v4f *>(in1),
                       reinterpret_cast<v4f *>(out0), reinterpret_cast<v4f *>(out1), n4);
    return hipGetLastError() == hipSuccess ? CAWN_OK : CAWN_ELAUNCH;
}

// ---------------------------------------------------------------------- allocation-free forward
// The workspace of this entry point is a static device array instead of caller memory.  `scratch`
// names the array for device code only: on the host it is a stand-in, never an address.  The device
// address is asked for once per device (hipGetSymbolAddress, with that device current) and kept;
// every launch and fill below takes that pointer.
#ifndef CAWN_STATIC_WS_BYTES
#define CAWN_STATIC_WS_BYTES (8u << 20)
#endif
static __device__ __align__(256) unsigned char scratch[CAWN_STATIC_WS_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::atomic<void *> g_scratch_ptr[MAX_DEVICES];      // per device: the array's address there, once known
}

int cawn_phase_accumulate_fwd_static(const cawn_desc *d, const float *mag, const float *ang, const float *gamma,
                                     const float *theta, const float *conv_w, const float *conv_b,
                                     const void *state_in, float *z_re, float *z_im, void *state_out, void *ckpt,
                                     uint32_t *gate_mask, void *stream)
{
    if (!desc_ok(d)) return CAWN_EINVAL;
    if (d->gate_mode != 0 || d->ret_mode != 0 || d->hconv_k != 0) return CAWN_EINVAL;
    // sizes beyond the static array are refused before anything touches the device
    if (make_layout(d, true).total > (size_t)CAWN_STATIC_WS_BYTES) return CAWN_EWORKSPACE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return CAWN_ELAUNCH;
    void *ws = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ws) {
        // first call on this device.  The array is zero when the module is loaded (no word carries a
        // tag); only the header's size field, read when the epoch wraps, has to be written.  Two
        // threads racing here find the same address and enqueue the same idempotent store.
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CAWN_ELAUNCH;
        hipLaunchKernelGGL(init_header_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream,
                           reinterpret_cast<WsHeader *>(p), (unsigned long long)CAWN_STATIC_WS_BYTES);
        if (hipGetLastError() != hipSuccess) return CAWN_ELAUNCH;
        g_scratch_ptr[dev].store(p, std::memory_order_release);
        ws = p;
    }
    return fwd_impl(d, mag, ang, nullptr, nullptr, nullptr, gamma, theta, conv_w, conv_b, state_in, z_re, z_im,
                    state_out, ckpt, gate_mask, ws, (size_t)CAWN_STATIC_WS_BYTES, stream, false, nullptr, nullptr, true);
}

}  // extern "C"
