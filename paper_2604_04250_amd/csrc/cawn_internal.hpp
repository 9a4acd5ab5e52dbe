// Internal definitions shared by the libcawn translation units (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cawn.h"
#include "cawn_gate_host.hpp"

namespace cawn {

// ------------------------------------------------------------------------------------ geometry
// One tile = JB lanes x TILE_T tokens of one batch row, processed by one workgroup at a time.  A
// thread owns V adjacent lanes and NSTEP consecutive tokens ("segment"); NSEG segments make the
// tile.  The two kernels pick their own shape:
//   forward : long tiles.  Its tiles of one chain are joined by memory round trips, so the fewer
//             tiles a chain has the better; it keeps only 2 values per token-lane in registers,
//             which allows 32 tokens per thread.  With the harmonic convolution a tile is 64 lanes
//             wide: heads of up to 64 harmonics lie inside one wave's lanes, and neighbours are a DPP
//             shift away.  Heads of 128 and 256 have rows of their own width, whose waves exchange
//             their outermost lanes in LDS.  (32-lane
//             rows: a head of 64 was two tiles of one workgroup, one after the other, with four LDS
//             exchanges per token.  Against that: B1 L333 J256 35.8 -> 17.5 us, the training step of
//             B8 L8192 H4 F64 329 -> 299 us, of B8 L8192 H12 F64 623 -> 544 us, F = 256 156 -> 100 us;
//             heads of up to 32 on J = 96 and 160, whose last block is half empty: 1.7 % slower.)
//   backward: keeps ~10 values per token-lane, hence 8 tokens per thread and one lane per thread
//             (4 waves per SIMD).
// Checkpoints of the scan state are kept every CKPT_T tokens = one backward segment: a backward
// thread starts the forward state of its tokens from the checkpoint of its own segment (one more
// byte per token-lane each way; without it every tile had to join its segments' states in LDS).
#ifndef CAWN_BWD_TILE_T
#define CAWN_BWD_TILE_T 128
#endif
#ifndef CAWN_BWD_NSTEP
#define CAWN_BWD_NSTEP 8
#endif
#ifndef CAWN_BWD_V
#define CAWN_BWD_V 1
#endif
#ifndef CAWN_BWD_LPR
#define CAWN_BWD_LPR 32
#endif
#ifndef CAWN_FWD_WAVES
#define CAWN_FWD_WAVES 2      // waves per SIMD the forward kernel's register budget is set for
#endif
#ifndef CAWN_BWD_WAVES
#define CAWN_BWD_WAVES 4
#endif
// NSTEP tokens per thread, JB lanes (= threads) per row, NT threads
template <int NSTEP_, int JB_, int NT_> struct FwdTile {
    static constexpr int NSTEP = NSTEP_, JB = JB_, NT = NT_, NSEG = NT / JB, TILE_T = NSEG * NSTEP;
    static constexpr bool SHORT = NSTEP < 32;
    static constexpr int MAX_CHAIN = 64;       // most short tiles of a chain (one group)
};
using FwdGeom = FwdTile<32, 32, 256>;      // 256 tokens x 32 lanes
using FwdHead = FwdTile<32, 64, 256>;      // 128 tokens x 64 lanes: harmonic convolution
using FwdWide128 = FwdTile<32, 128, 256>;  // 64 tokens x 128 lanes: harmonic convolution, heads of 128
using FwdWide256 = FwdTile<32, 256, 512>;  // 64 tokens x 256 lanes: heads of 256
using FwdShort = FwdTile<8, 32, 256>;      // 64 tokens x 32 lanes: calls that leave the chip idle otherwise
using FwdShortHead = FwdTile<8, 64, 512>;  // 64 tokens x 64 lanes: the same with the harmonic convolution
static_assert(FwdShort::TILE_T == FwdShortHead::TILE_T, "one table row for both");
struct BwdGeom {
    static constexpr int TILE_T = CAWN_BWD_TILE_T, NSTEP = CAWN_BWD_NSTEP, NSEG = TILE_T / NSTEP;
};
constexpr int CKPT_T = BwdGeom::NSTEP;
static_assert(FwdGeom::NSTEP % CKPT_T == 0, "a forward segment spans whole checkpoint intervals");
static_assert(BwdGeom::TILE_T % CKPT_T == 0, "backward tiles start on checkpoints");
constexpr int BwdV = CAWN_BWD_V, BwdLPR = CAWN_BWD_LPR;
constexpr int MAX_KC = 4;
constexpr uint32_t MAX_TILES = 1u << 18;   // most tiles one call may have (tile indices, tickets)

// ---------------------------------------------------------------------------------- lane table
// Per-lane constants, struct-of-arrays, each row Jp floats (Jp = J rounded up to 64), built in
// fp64 by a small kernel from gamma, theta, conv_w, conv_b.
enum LaneRow : int {
    R_COS = 0, R_SIN, R_GAMMA, // e^{i theta}, gamma
    R_PT_HR, R_PT_HI,          // lambda^256 (FwdGeom::TILE_T), leading fp32 part
    R_PT_LR, R_PT_LI,          //                          remainder (double-float)
    R_PTB_HR, R_PTB_HI,        // the same for the backward tile length
    R_PTB_LR, R_PTB_LI,
    R_PSEGB,                   // R_PSEGB + 2*s (+1): re (im) of lambda^(NSTEP*s), backward segments
    // The rows below are what a forward tile's threads keep in registers; they are contiguous so
    // that a tile stages them in LDS with a few wide loads (R_LR .. R_W0 + 2*conv_k - 1).
    R_LR = R_PSEGB + 2 * BwdGeom::NSEG, R_LI,   // lambda = gamma e^{i theta}
    R_PSEG,                    // R_PSEG + 2*s (+1): lambda^(32 s), the long forward tiles' segments, s >= 1
    // (s = 0 would be 1: its rows hold the remainder of lambda^64, the short tiles' length, whose leading part is s = 2)
    R_PT64_LR = R_PSEG, R_PT64_LI, R_PT64_HR = R_PSEG + 4, R_PT64_HI,
    R_BIAS_M = R_PSEG + 2 * FwdGeom::NSEG, R_BIAS_A,
    R_RBIAS,                   // ret_mode 1: the lane's static retention bias b_k (k = j mod F)
    R_W0                       // R_W0 + s*conv_k + i : tap i of stream s
};
// Harmonic convolution (Sec. 3.6): HC_ROWS more rows behind the temporal conv's taps, per lane the
// constants of its head's two channels: R_W0 + 2*conv_k + 3*plane + i = tap i, + 6 + plane = bias.
constexpr int HC_ROWS = 8;
inline __host__ __device__ int lane_rows(int conv_k, bool hconv = false) { return R_W0 + 2 * conv_k + (hconv ? HC_ROWS : 0); }

// ----------------------------------------------------------------------------------- workspace
// Workspace: [header 1 KiB][lane table][aggregates][prefixes][backward conv halo][backward parameter
// partials].  Everything tiles publish to each other (aggregates, prefixes, halo rows) is stored as
// 8-byte words {value, tag}: the tag is make_tag(epoch of the call), so a word is valid exactly
// when its tag matches -- no separate status words, no ordering between stores, one memory round trip
// from publication to use.  Words left by earlier calls (whatever their descriptor) carry other tags
// and read as "not published"; cawn_workspace_init zeroes the whole buffer (a zero word is never a tag).
// Region offsets depend on the descriptor, so a call may find fp32 data of an earlier call with another
// descriptor (lane-table rows, partial sums) where it expects published words.  Tags are therefore the
// bit patterns of negative NaNs with a non-zero payload (0xFF800001 .. 0xFFFFFFFF): no finite value,
// infinity or hardware-made NaN (0x7FC00000) an fp32 computation leaves behind equals one.
// Nothing is cleared per tile or per call: the workgroup that leaves last resets the tickets and
// advances the epoch.
constexpr int MAX_QUEUES = 8;
struct WsHeader {
    uint32_t q01[64];              // ticket and finished counters (ticket_word, done_word)
    uint32_t done;                 // workgroups, or groups of them, finished
    uint32_t error;                // sticky: a tile gave up waiting
    uint32_t epoch;                // calls completed on this workspace (mod EPOCH_MOD): make_tag() of it marks published words
    uint32_t bytes_lo, bytes_hi;   // size given to cawn_workspace_init (what an epoch wrap has to clear)
    uint32_t q27[256 - 64 - 5];
};
static_assert(sizeof(WsHeader) == 1024, "header size");
// Counters of queue q, as word indices into the header: one 128-byte line each (queue 2 shares its line with `done`)
inline __host__ __device__ uint32_t ticket_word(uint32_t q) { return q == 2 ? 80u : q * 32u; }
inline __host__ __device__ uint32_t done_word(uint32_t q) { return ticket_word(q) + 8u; }

// How a call's tiles are handed out.  Atomics on one address complete one after the other, 11.4 ns each here (on
// addresses 128 bytes apart side by side): the 384 workgroups of a 4096-token call on 768 lanes had their first tickets
// after 4.4 us, their second ones (which only tell them that there is nothing left) 4.4 us later, and their last
// count took as long again.  So:
//   * a call whose workgroups take one tile each draws no second ticket, and its U chains are dealt to eight counters:
//     U / 8 adjacent ones each (one more to the first U mod 8 counters), and a counter's n-th draw is tile n / C of its chain number
//     n mod C (C chains of this counter); tile numbers stay what they are (tile in time x U + chain), a chain belongs to one counter,
//     and a tile still only waits for tiles with a lower ticket of its own counter, which a running workgroup holds.  Workgroup w
//     draws from counter (w mod U) mod 8: as many draws as the counter has tiles.  (Dealt to 2^k counters only where 2^k divides U, an
//     odd number of chains had one counter: a draw then took 2.3 us on average and 4.3 at most in a grid of 384 workgroups, 3.1 and
//     6.0 in one of 512; with eight 0.9 - 1.0 and 1.6.  Forward calls of 7 - 66 chains with a few tiles more than fit: 3 - 14 % of
//     the call.)  Where eight divides U, workgroups of a counter are those of one XCD, whose L2 then sees adjacent lane blocks of a
//     row: the words of the gate mask, four bytes a block, are joined there, and no XCD is bound to one class of addresses (with
//     chain c at counter c mod 8, every eighth block of 128 bytes): B4 L2048 J768 with a mask 25.4 -> 24.2 us;
//   * a call with more tiles than workgroups keeps one counter: its draws are spread over the call and cost nothing
//     (eight counters with a second choice where one ran dry were slower: training step 431 -> 454 us, bf16 B2 L4096
//     J4096 284 -> 298; the first tickets' delay keeps the workgroups out of step, and loads beside arithmetic);
//   * the many workgroups of such a one-tile-each call are counted in two levels, in the middle of their tile (counts_early).
struct TileQueues { uint32_t units, one_each, group; };     // group: tiles of a chain between two prefixes (see chain_carry)
// Tiles between two prefixes in the forward: 8; 16 where there are so few chains that passing prefixes on bounds the call.
// us a call with 2 / 4 / 8 / 16: B1 L4096 J768 20.5 / 18.8 / 18.1 / 19.2; B1 L32768 J256 of the paper's layer in bf16 109 /
// 71 / 52 / 49, with the harmonic convolution 111 / 73 / 58 / 56; B2 L4096 J4096 bf16 84.5 / 83.6 / 84.8 / 86.9.
// Between them, 8 against 16 at U = 4 / 8 / 10 / 12 / 16 chains: L32700 bf16 50.1 and 45.4 / 64.4 and 62.0 / 73.2 and 72.1 /
// 78.9 and 78.2 / 98.5 and 99.6, with retentions 48.9 and 46.5 / 71.2 and 74.1 / 83.1 and 87.5 / 95.7 and 101 / 120 and 129;
// fp32 with a workgroup a tile 28.1 and 24.9 / 22.2 and 21.4 / 24.3 and 23.8 / 28.6 and 28.4 / 20.6 and 20.9.  (conv 3)
// 1 (a prefix per tile, look_back) for 32-lane rows whose workgroups take several tiles (MANY): there the nearest prefix has nearly
// always arrived, and one pair of words is cheaper than a fold: B16 L1000 J768 55.0 against 56.2, paper's layer B8 L8192
// J256 74.4 against 77.4 (with bf16 or the harmonic convolution, on 64-lane rows, the fold is ahead there too).
inline TileQueues make_queues(uint32_t U, uint32_t nT, long long workgroups)
{
    return TileQueues{U, workgroups >= (long long)U * nT ? 1u : 0u, U <= 8 ? 16u : 8u};
}

struct WsLayout {
    int J, Jp, Jp128, nT, nTc;     // nT: backward tiles per sequence, nTc: checkpoint intervals
    size_t off_table, off_agg, off_pre, off_halo, off_part, off_vpart, off_aggp, off_rpart, off_dbg, total;
};

constexpr uint32_t EPOCH_MOD = (1u << 23) - 1u;     // epochs 0 .. 2^23 - 2
typedef unsigned long long tagged_t;     // {fp32 value (low half), tag (high half)}
inline __host__ __device__ uint32_t make_tag(uint32_t epoch) { return 0xFF800001u + epoch; }

// (GateSet, the gate as a union of two closed fp32 intervals, comes from cawn_gate_host.hpp)

struct FwdArgs {
    const float *mag, *ang;
    const float *table;          // lane table
    const float *state_in;       // may be null
    float *z_re, *z_im;
    float *state_out;            // may be null
    float *ckpt;                 // may be null
    uint32_t *mask;              // may be null
    WsHeader *hdr;
    tagged_t *agg, *pre;
    TileQueues tq;
    int B, L, J, Jp, nT, nLB;    // nT: forward tiles per sequence
    int nTc;                     // checkpoint intervals per sequence
    int stage16;                 // input rows may be staged with 16-byte loads (alignment, J % 4 == 0)
    int amp_mode;
    int small_angle;             // angles are bounded (conv clamp): skip the two-term range reduction
    long long isb, ist, osb, ost;
    float conv_clamp, out_clamp;
    GateSet gs;
    uint32_t spin_limit;
    uint32_t total_tiles;
    size_t clear_from;           // byte offset of the first published word (cleared when the epoch wraps)
    unsigned long long *dbg;     // -DCAWN_TIMING builds only
    // (kept behind everything else: the kernels that do not use them fetch none of this)
    // gate_mode 1 (per-head input valve, Sec. 3.3): logits [B][L][H]; a lane block of JB lanes
    // touches at most gpb heads (groups): JB / F whole ones, a part of one, or two where heads of more than JB lanes
    // end inside a block (F an odd multiple of 32, 64-lane blocks); the valve is open when the logit >= valve_thr
    const float *valve;          // null: gate_mode 0
    int H, F, gpb;
    float valve_thr;
    // ret_mode 1 (data-dependent retention, Sec. 3.3 item 4): logits [B][L][H], staged like the valve's;
    // the lane table is then built with gamma = 1 (its powers are pure rotations) and a tile's
    // aggregate has a third chained word, the product of the tile's retentions: aggp [tile][JB]
    const float *ret;            // null: ret_mode 0
    tagged_t *aggp;
    // activations are bfloat16 in memory (mag, ang, z_re, z_im then point to 2-byte elements; strides
    // are in elements); J and the strides are even
    int bf16;
    int hconv;                   // harmonic convolution of the output before it is stored (Sec. 3.6, three taps)
    int short_tiles;             // FwdShort / FwdShortHead instead of FwdGeom / FwdHead
};

struct BwdArgs {
    const float *mag, *ang, *dz_re, *dz_im;
    const float *table;
    const float *state_in;       // may be null
    const float *ckpt;           // may be null when no dgamma/dtheta
    const float *dstate_out;     // may be null
    float *dmag, *dang;
    float *dstate_in;            // may be null
    WsHeader *hdr;
    tagged_t *agg, *pre, *halo;
    TileQueues tq;
    float *part;
    int B, L, J, Jp, nT, nLB;
    int nTc;                     // checkpoint intervals per sequence
    int small_angle;
    int stage16;                 // input rows may be staged with 16-byte loads (alignment, J % 4 == 0)
    int stage16z;                // the same for the upstream-gradient rows
    int amp_mode, want_param;
    long long isb, ist, osb, ost;
    float conv_clamp, grad_clamp;
    GateSet gs;
    uint32_t spin_limit;
    uint32_t total_tiles;
    size_t clear_from;           // byte offset of the first published word (cleared when the epoch wraps)
    unsigned long long *dbg;     // -DCAWN_TIMING builds only
    // (kept behind everything else: the kernels that do not use them fetch none of this)
    // gate_mode 1 (per-head input valve): see FwdArgs; vpart [B][G][L] receives, per valve group
    // (a head, or the 32-lane slice of a head) and token, the sum over the group's lanes of
    // a Re(conj(dp) e^{i phi}); G groups per token
    const float *valve;          // null: gate_mode 0
    float *vpart;                // null: no valve gradient wanted
    int H, F, gpb, G;
    float valve_thr;
    // ret_mode 1 (data-dependent retention): see FwdArgs; rpart like vpart, for the retention logits
    const float *ret;            // null: ret_mode 0
    float *rpart;                // null: no gradient of the retention logits wanted
    tagged_t *aggp;
    int bf16;                    // activations (mag, ang, dz_*, dmag, dang) are bfloat16 in memory: see FwdArgs
    // harmonic convolution behind the output clamp (Sec. 3.6): dz_re / dz_im are then the gradients of the
    // CONVOLVED output; the kernel applies the transposed convolution as it reads them and emits, per lane,
    // the terms of the tap and bias gradients (rows behind the conv front-end's in `part`)
    int hconv;
    float out_clamp;
};

// Number of per-lane partial sums a backward tile emits: dgamma, dtheta, dbias[2], dw[2][conv_k]; with the
// harmonic convolution 8 more: its taps' terms [2 planes][3], then its biases' [2 planes].
constexpr int HC_PART_ROWS = 8;
inline __host__ __device__ int part_rows(int conv_k, bool hconv = false) { return 4 + 2 * conv_k + (hconv ? HC_PART_ROWS : 0); }

hipError_t launch_fwd(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_bwd(const BwdArgs &a, int conv_k, bool vec, hipStream_t s);

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)
// ------------------------------------------------------------------------------ device helpers
__device__ __forceinline__ float clampf(float v, float c) { return __builtin_amdgcn_fmed3f(v, -c, c); }

// Streamed data -- the activations a call reads once and the outputs it writes once -- moves with the
// non-temporal cache policy: it does not displace what is read again (lane table, published words, halo rows,
// and the checkpoints, which the backward of the same step reads back: those keep the default policy).
// Measured on the training-step shape: backward 275 -> 258 us, a 4096-token chunk 25.3 -> 23.5 us.
__device__ __forceinline__ void st_stream(float *p, float v) { __builtin_nontemporal_store(v, p); }
constexpr int DMA_STREAM = 2;      // cache-policy operand of the direct-to-LDS loads of staged rows: nt

// An element of a bf16 output row, LINES: of rows of whole 128-byte lines, which are streamed (B8 L2048 J768 42.5 -> 39.2 us, the paper's
// layer behind the harmonic convolution B1 L32768 J256 44.9 -> 43.4).  Of others the cache joins a line's parts, which neighbouring
// tiles store (streamed: 32-lane tiles 155 against 136 us, B3 L11401 J1200 training step 391 against 381, B8 L2048 J96 12.7 against 12.1).
template <bool LINES> __device__ __forceinline__ void st_row16(char *p, uint16_t v)
{
    if constexpr (LINES) __builtin_nontemporal_store(v, reinterpret_cast<uint16_t *>(p));
    else *reinterpret_cast<uint16_t *>(p) = v;
}
// bfloat16 in memory: the upper half of an fp32; to bf16 with the hardware's round-to-nearest-even.
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t to_bf16(float x)
{
    const __bf16 h = (__bf16)x;
    return __builtin_bit_cast(uint16_t, h);
}

// sigmoid(z) with the hardware exp2 / reciprocal (both ~1 ulp).
__device__ __forceinline__ float sigmoid_fast(float z)
{
    float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * z);
    return __builtin_amdgcn_rcpf(1.0f + e);
}

// sin and cos of an angle in radians: two-term Cody-Waite reduction to [-pi, pi] (exact products
// through fma), then the hardware sin/cos, which take revolutions.
__device__ __forceinline__ void sincos_fast(float phi, float &s, float &c)
{
    const float INV_2PI = 0.15915494309189535f;
    const float TWO_PI_HI = 6.2831854820251465f;      // fp32(2 pi)
    const float TWO_PI_LO = -1.7484555314695172e-07f; // 2 pi - TWO_PI_HI
    float k = __builtin_rintf(phi * INV_2PI);
    float r = __builtin_fmaf(-k, TWO_PI_HI, phi);
    r = __builtin_fmaf(-k, TWO_PI_LO, r);
    float x = r * INV_2PI;
    s = __builtin_amdgcn_sinf(x);
    c = __builtin_amdgcn_cosf(x);
}

// Same, for angles known to be small (a few revolutions): the hardware reduces the range itself.
__device__ __forceinline__ void sincos_small(float phi, float &s, float &c)
{
    const float x = phi * 0.15915494309189535f;
    s = __builtin_amdgcn_sinf(x);
    c = __builtin_amdgcn_cosf(x);
}
// The reduced angle in revolutions those two hand to the hardware (a caller short of registers
// keeps this one value and asks the hardware for sin and cos again).
__device__ __forceinline__ float revolutions_fast(float phi)
{
    const float INV_2PI = 0.15915494309189535f;
    const float TWO_PI_HI = 6.2831854820251465f;
    const float TWO_PI_LO = -1.7484555314695172e-07f;
    float k = __builtin_rintf(phi * INV_2PI);
    float r = __builtin_fmaf(-k, TWO_PI_HI, phi);
    r = __builtin_fmaf(-k, TWO_PI_LO, r);
    return r * INV_2PI;
}
__device__ __forceinline__ float revolutions_small(float phi) { return phi * 0.15915494309189535f; }

__device__ __forceinline__ float softplus_fast(float m)
{
    // log(1 + e^m) = max(m, 0) + log(1 + e^-|m|)
    float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * __builtin_fabsf(m));
    return __builtin_fmaxf(m, 0.0f) + 0.6931471805599453f * __builtin_amdgcn_logf(1.0f + e);
}

// softplus(m) as above, and its derivative sigmoid(m) from the same exponential
__device__ __forceinline__ float softplus_sigmoid_fast(float m, float &sig)
{
    const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * __builtin_fabsf(m)), t = 1.0f + e;
    const float r = __builtin_amdgcn_rcpf(t);
    sig = m >= 0.0f ? r : e * r;
    return __builtin_fmaxf(m, 0.0f) + 0.6931471805599453f * __builtin_amdgcn_logf(t);
}

// (a second interval has no upper end, see gate_set_of: three comparisons)
__device__ __forceinline__ bool in_gate(const GateSet &g, float x)
{
    // bitwise on purpose: short-circuit forms compile to divergent branches
    return (bool)(((int)(x >= g.a1) & (int)(x <= g.b1)) | (int)(x >= g.a2));
}

// Whole-wave shifts by one lane (DPP wave_shr:1 / wave_shl:1): lane i takes lane i-1's (i+1's) value, the
// first (last) lane zero.  (By the shift's own rule for lanes without a source: keeping the lane's own value, or writing into
// a register cleared before, is a second instruction.)
__device__ __forceinline__ float wave_shift_up0(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_shift_down0(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, true));
}

// Two tokens' outputs of both planes += w[plane][0] * (lane i-1's z) + w[plane][2] * (lane i+1's z), zero beyond the wave's
// ends: the shift is the multiply-add's own operand modifier, which the compiler does not form for it (it moves first: two
// instructions a neighbour instead of one; with a cleared destination, as the shifts above were once written, three).  Two
// wait states stand between a vector write and a shifted read of it.  Every lane of the wave must be active.
__device__ __forceinline__ void fma_neighbours(float &r0, float &i0, float &r1, float &i1, float zr0, float zi0, float zr1, float zi1,
                                               const float (&w)[2][3])
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 1\n"
                 "v_fmac_f32_dpp %0, %4, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %1, %5, %9 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %2, %6, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %3, %7, %9 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %0, %4, %10 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %1, %5, %11 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %2, %6, %10 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
                 "v_fmac_f32_dpp %3, %7, %11 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
                 : "+&v"(r0), "+&v"(i0), "+&v"(r1), "+&v"(i1)
                 : "v"(zr0), "v"(zi0), "v"(zr1), "v"(zi1), "v"(w[0][0]), "v"(w[1][0]), "v"(w[0][2]), "v"(w[1][2]));
#endif
}

// Cross-tile publication.  Tiles of one chain may run on different XCDs, whose L2 caches are not
// coherent with each other.  Payload and status words therefore move with agent-scope relaxed
// atomics (sc1 accesses, which go to the memory-side coherence point), and ordering is by waiting
// for the stores to complete (vmcnt) before the status word is written.  Acquire/release atomics
// are avoided on purpose: at agent scope they write back / invalidate the whole L2 on every use,
// which a spin loop next to streaming stores cannot afford.
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }
// Wait until at most N of this wave's vector memory operations are outstanding.  They complete in
// issue order (loads, stores and direct-to-LDS loads alike), so this waits for everything except
// the N youngest.  The builtin (not inline assembly) lets the compiler's own wait insertion see it.
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    compiler_fence();
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);   // expcnt, lgkmcnt: no wait
    compiler_fence();
}
__device__ __forceinline__ void wait_stores_done() { wait_vm<0>(); }
// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains every outstanding
// global load and store of every wave, which would serialise a tile's output stores and the next
// tile's staging loads with the barrier; global data here is never exchanged inside a workgroup.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// The same barrier for a point where direct-to-LDS loads are still in flight: there the compiler
// makes the fences above wait for those loads.  Hardware barrier only; LDS accesses of this wave
// are waited for explicitly and the compiler may not move memory accesses across.
__device__ __forceinline__ void lds_barrier_raw()
{
    compiler_fence();
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt, expcnt: no wait
    __builtin_amdgcn_s_barrier();
    compiler_fence();
}

// Stage the pre-conv input rows of one tile in LDS with direct global->LDS loads (no registers):
// rows tile_t0-HALO .. tile_t0+TT-1 of the magnitude stream, then the same rows of the angle
// stream, JB lanes each, row-major; each stream occupies staged_rows<TT, JB, HALO>() rows (padded
// to whole load instructions).  Called by `nwaves` waves (index `wave` among them).  Rows outside
// [0, L) and lanes beyond J read a clamped (valid) address: their values never reach a result (the
// scan is causal, a lane only reads its own LDS column; rows before a sequence start are zeroed at
// the point of use).  Rows before the call's first token come from the carried conv history when
// there is one.  LB: bytes per lane per load (16 needs 16-byte aligned rows).
template <int TT, int JB, int HALO>
__host__ __device__ constexpr int staged_rows()
{
    constexpr int g = 256 / JB > 0 ? 256 / JB : 1;      // rows per instruction of the widest load
    return (TT + HALO + g - 1) / g * g;
}
template <int TT, int JB, int HALO, int LB>
__device__ __forceinline__ void stage_rows(float *sU, const float *mag, const float *ang, const float *tail_in,
                                           int b, int tile_t0, int lb, int J, int L, long long isb, int ist,
                                           int wave, int nwaves, int lane)
{
    constexpr int NRT = TT + HALO;
    // rows whose segment fills a 128-byte line are streamed; half lines (bf16 on 32-lane rows) keep the default policy,
    // so that the cache can serve the neighbouring lane block's half of the line
    [[maybe_unused]] constexpr int POL = JB * 4 >= 128 ? DMA_STREAM : 0;
    constexpr int NRTP = staged_rows<TT, JB, HALO>();
    constexpr int LR = JB * 4 / LB;                // lanes per row
    if constexpr (LR <= 64) {
        constexpr int RPI = 64 / LR;               // rows per wave instruction
        static_assert(NRTP % RPI == 0, "a stream is a whole number of load instructions");
        constexpr int NIS = NRTP / RPI;            // instructions per stream
        const int t_first = tile_t0 - HALO;
        // wave-uniform bases of the two streams at the first staged row
        const float *base_m = mag + (size_t)b * isb + (long long)t_first * ist;
        const float *base_a = ang + (size_t)b * isb + (long long)t_first * ist;
        const int r_in = lane / LR, c_in = (lane % LR) * (LB / 4);      // my row within an instruction, my lane
        if (t_first >= 0 && t_first + NRT <= L && (lb + 1) * JB <= J) {
            // every staged row exists: uniform base + one per-lane byte offset
            const uint32_t loff = (uint32_t)(r_in * ist + lb * JB + c_in) * 4u;
            for (int i = wave; i < 2 * NIS; i += nwaves) {
                const int sidx = i >= NIS ? 1 : 0, ii = i - sidx * NIS;
                const float *ub = (sidx ? base_a : base_m) + (long long)(ii * RPI) * ist;
                const float *src = reinterpret_cast<const float *>(reinterpret_cast<const char *>(ub) + loff);
                if (ii * RPI + r_in >= NRT) continue;      // padding rows of a stream's last instruction: not fetched
#if defined(__HIP_DEVICE_COMPILE__)
                if constexpr (LB == 16) __builtin_amdgcn_global_load_lds(src, sU + (size_t)(sidx * NRTP + ii * RPI) * JB, 16, 0, POL);
                else __builtin_amdgcn_global_load_lds(src, sU + (size_t)(sidx * NRTP + ii * RPI) * JB, 4, 0, POL);
#else
                (void)src;
#endif
            }
            return;
        }
        int j = lb * JB + c_in;
        if (j >= J) j = 0;
        const bool hist = HALO > 0 && tile_t0 == 0 && tail_in != nullptr;
        for (int i = wave; i < 2 * NIS; i += nwaves) {
            const int sidx = i >= NIS ? 1 : 0, ii = i - sidx * NIS;
            int rr = ii * RPI + r_in;
            if (rr >= NRT) rr = NRT - 1;
            const int t = t_first + rr;
            const int tc = t < 0 ? 0 : (t >= L ? L - 1 : t);
            const float *src = (sidx ? base_a : base_m) + ((tc - t_first) * ist + j);
            if (hist && t < 0) src = tail_in + ((size_t)(b * HALO + rr) * 2 + sidx) * J + j;
#if defined(__HIP_DEVICE_COMPILE__)
            if constexpr (LB == 16) __builtin_amdgcn_global_load_lds(src, sU + (size_t)(sidx * NRTP + ii * RPI) * JB, 16, 0, POL);
            else __builtin_amdgcn_global_load_lds(src, sU + (size_t)(sidx * NRTP + ii * RPI) * JB, 4, 0, POL);
#else
            (void)src;
#endif
        }
    }
}
// A valve logit's factor of the amplitude: sigmoid(logit - 3), -1 where the valve is closed.
__device__ __forceinline__ float valve_factor(float logit, float thr) { return logit >= thr ? sigmoid_fast(logit - 3.0f) : -1.0f; }
// Stage the valve logits of one tile (gate_mode 1): entry (group, token) of the tile lands at
// sV[group * TT + token]; the lane block's groups are the gpb heads from the one its first lane lies in on.
// 4 bytes per lane per load; called by one wave.
template <int TT, int JB>
__device__ __forceinline__ void stage_valve(float *sV, const float *valve, int b, int tile_t0, int lb, int L, int H,
                                            int F, int gpb, int lane)
{
    const int h0 = (lb * JB) / F;
    for (int i = 0; i < TT * gpb / 64; ++i) {
        const int idx = i * 64 + lane;
        int t = tile_t0 + idx % TT, h = h0 + idx / TT;
        t = t < L ? t : L - 1;          // rows past the end, heads past the last: a valid address,
        h = h < H ? h : H - 1;          // the value is never used
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_global_load_lds(valve + ((size_t)b * L + t) * H + h, sV + i * 64, 4, 0, 0);
#else
        (void)sV;
        (void)valve;
#endif
    }
}

// ... and once they have landed, the same wave turns them into factors.  One element a lane
// instead of one a lane, token and head: in the front-end, where every lane of a head formed the same factor, this was 8 of
// its 45 instructions, two of them transcendental.
template <int TT>
__device__ __forceinline__ void valve_factors(float *sV, float thr, int gpb, int lane)
{
    for (int i = 0; i < TT * gpb / 64; ++i) sV[i * 64 + lane] = valve_factor(sV[i * 64 + lane], thr);
}

__device__ __forceinline__ void flag_store(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t flag_load(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Published words.  One 8-byte relaxed agent-scope store carries a value and the call's tag; the
// reader takes the value only from a word whose tag matches.  8-byte naturally aligned accesses are
// single-copy atomic, so a reader sees either the whole new word or an old one.
__device__ __forceinline__ void tagged_store(tagged_t *p, float v, uint32_t tag)
{
    __hip_atomic_store(p, (tagged_t)__float_as_uint(v) | ((tagged_t)tag << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ tagged_t tagged_load(const tagged_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tagged_ok(tagged_t w, uint32_t tag) { return (uint32_t)(w >> 32) == tag; }
__device__ __forceinline__ float tagged_value(tagged_t w) { return __uint_as_float((uint32_t)w); }

__device__ __forceinline__ uint32_t *hdr_word(WsHeader *h, uint32_t w) { return reinterpret_cast<uint32_t *>(h) + w; }
constexpr uint32_t NO_TICKET = 0x7fffffffu;     // beyond every call's tiles
// the first tile of workgroup `wg`: see TileQueues
__device__ __forceinline__ uint32_t first_ticket(WsHeader *h, const TileQueues &t, uint32_t wg)
{
    auto draw = [&](uint32_t q) { return __hip_atomic_fetch_add(hdr_word(h, ticket_word(q)), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (!t.one_each) return draw(0);
    constexpr uint32_t Q = MAX_QUEUES;
    // (as many workgroups of a period of `units` draw at a counter as it has chains)
    const uint32_t q = t.units % Q ? wg % t.units % Q : wg % Q, C = (t.units - q + Q - 1) / Q, n = draw(q);
    // n / C: n < 2^18, so that the reciprocal's error is below the distance of (n + 1/2) / C from a whole number
    const uint32_t tt = (uint32_t)(((float)n + 0.5f) * __builtin_amdgcn_rcpf((float)C)), rest = t.units % Q;
    return tt * t.units + q * (t.units / Q) + (q < rest ? q : rest) + (n - tt * C);
}
// ... and the next ones (calls with one counter)
__device__ __forceinline__ uint32_t next_ticket_of(WsHeader *h)
{
    return __hip_atomic_fetch_add(hdr_word(h, ticket_word(0)), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A workgroup leaves the call: the count is asked for (leave_ask), and its answer says whether it was the last one of the
// grid (leave_last).  96 and more workgroups that take one tile each, and so are counted at about the same time, are counted
// in two levels (a second round trip, 0.4 us, for the last of them; 96 counts on one address take 1.1 us); those of larger
// calls are spread by their draws.
__device__ __forceinline__ bool leave_two_levels(const TileQueues &t, uint32_t grid) { return t.one_each && grid >= 96; }
__device__ __forceinline__ uint32_t leave_ask(WsHeader *h, const TileQueues &t, uint32_t wg, uint32_t grid)
{
    uint32_t *w = leave_two_levels(t, grid) ? hdr_word(h, done_word(wg % MAX_QUEUES)) : &h->done;
    return __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool leave_last(WsHeader *h, const TileQueues &t, uint32_t wg, uint32_t grid, uint32_t before)
{
    if (!leave_two_levels(t, grid)) return before + 1u == grid;
    if (before + 1u != (grid - wg % MAX_QUEUES + MAX_QUEUES - 1) / MAX_QUEUES) return false;
    return __hip_atomic_fetch_add(&h->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (uint32_t)MAX_QUEUES;
}
// Workgroups that take one tile each have drawn all they will ever draw, and read the epoch, before they start on it: they
// are counted in the middle of the tile, by a wave that waits for the carry, and the last one counted resets the counters
// while tiles are still at work.  Counted behind its output stores, a call ended with these round trips: B1 L333 J256 with the
// harmonic convolution 11.0 -> 10.5 us, a training step of B7 L1024 J256 43.4 -> 41.9, of B3 L1777 J120 36.1 -> 34.3.
// Only the call that wraps the epoch is counted at its end: it clears published words.
__device__ __forceinline__ bool counts_early(const TileQueues &t, uint32_t epoch) { return t.one_each && epoch + 1u != EPOCH_MOD; }

__device__ __forceinline__ void reset_header(WsHeader *hdr, uint32_t next_epoch, uint32_t tid, uint32_t nthreads)
{
    for (uint32_t q = tid; q < (uint32_t)MAX_QUEUES; q += nthreads) {
        flag_store(hdr_word(hdr, ticket_word(q)), 0u);
        flag_store(hdr_word(hdr, done_word(q)), 0u);
    }
    if (tid == 0) {
        flag_store(&hdr->done, 0u);
        flag_store(&hdr->epoch, next_epoch);
    }
}
// End of a call, run by thread `tid` of the `nthreads` of the workgroup that left last: tickets and
// the finished-workgroup count return to zero and the epoch advances.  When the epoch wraps, words of
// EPOCH_MOD calls ago would become valid again: everything behind the lane table is cleared then
// (`clear_from`: byte offset of this call's first published word) but what `keep` says of a word's address: the partial
// sums that a backward's epilogue has yet to read, every word of which this call wrote.
template <class Keep>
__device__ __forceinline__ void finish_call(WsHeader *hdr, size_t clear_from, uint32_t epoch, uint32_t tid,
                                            uint32_t nthreads, Keep keep)
{
    const uint32_t next = (epoch + 1) % EPOCH_MOD;
    if (next == 0) {
        const size_t bytes = (size_t)hdr->bytes_lo | ((size_t)hdr->bytes_hi << 32);
        uint32_t *base = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(hdr) + clear_from);
        const size_t n = bytes > clear_from ? (bytes - clear_from) / sizeof(uint32_t) : 0;
        for (size_t i = tid; i < n; i += nthreads)
            if (!keep(base + i)) flag_store(base + i, 0u);
    }
    reset_header(hdr, next, tid, nthreads);
}

// One link of a tile chain: P = T + M c, with M = lambda^TILE_T held as a double-float (h + q) and
// conjugated for the adjoint chain.  Published prefixes, look_back and chain_carry are all made of it.
template <bool CONJ>
__device__ __forceinline__ void chain_step(float Tr, float Ti, float hr, float hi, float qr, float qi,
                                           float cr, float ci, float &Pr, float &Pi)
{
    if (!CONJ) {
        const float lo_r = __builtin_fmaf(qr, cr, -qi * ci);
        const float lo_i = __builtin_fmaf(qi, cr, qr * ci);
        Pr = __builtin_fmaf(hr, cr, __builtin_fmaf(-hi, ci, Tr + lo_r));
        Pi = __builtin_fmaf(hi, cr, __builtin_fmaf(hr, ci, Ti + lo_i));
    } else {
        const float lo_r = __builtin_fmaf(qr, cr, qi * ci);
        const float lo_i = __builtin_fmaf(qr, ci, -qi * cr);
        Pr = __builtin_fmaf(hr, cr, __builtin_fmaf(hi, ci, Tr + lo_r));
        Pi = __builtin_fmaf(hr, ci, __builtin_fmaf(-hi, cr, Ti + lo_i));
    }
}

// Whether all lanes of my group say yes: a half of the wave, or all of it.  (Not the ballot shifted right by a register: one
// kernel's gate masks came out wrong now and then while it shifted 64-bit ballots by its last allocated vector register, the last of a
// block of eight too, and have been right since no such shift was left.  That is what was seen; no trace of the instruction was taken.)
template <int LANES>
__device__ __forceinline__ bool group_all(bool ok)
{
    static_assert(LANES >= 32, "half a wave, or whole waves");
    const unsigned long long all = __builtin_amdgcn_ballot_w64(ok);
    if (LANES >= 64) return all == ~0ull;
    const bool lower = (uint32_t)all == ~0u, upper = (uint32_t)(all >> 32) == ~0u;
    return (threadIdx.x & 32) ? upper : lower;
}

// The carry of a tile: what the tiles before it in its chain leave behind.  Run by one group of JB consecutive threads of
// a wave, or by each of the JB / 64 waves of a wider row for its own lanes.  A chain's tiles form groups of G (a power of two).  Every tile publishes its aggregate as soon as it has it
// (the chain's first tile its prefix, in the same place), the last tile of a group also its prefix.  A tile reads the
// aggregates of the r tiles before it in its group, NB per round trip, and folds them, in order, into one link
//   carry = E + P M^r c      (P: RET, the product of the r tiles' retentions)
// while the prefix c of the previous group is on its way; the first group needs none (its E is the carry).  So a
// prefix is passed on once per G tiles, and only that is a chain of round trips: with a prefix per tile, long chains of
// few rows advanced by 0.22 us a tile, and walking back over aggregates instead read every one of them in every tile.
// The association is fixed by G and the tile's position alone: results do not depend on timing.  (Tile length and G follow
// from the whole call's sizes: the same row in a call of another batch may be rounded differently.)  For the forward chains.
// `id` is the tile's index, `stride` the distance to its predecessor's, tt >= 1 its position in the chain.  M is
// lambda^TILE_T as a double-float; its power is formed in fp64.  Every wait is bounded: false if one gave up (the carry
// is then meaningless).
//
// The fold of a group's aggregates, one at a time in order; LINK: and the power of M, for the link on the prefix before them.
struct ChainFold {
    float Er = 0.f, Ei = 0.f, P = 1.f;
    double mr = 1.0, mi = 0.0;
    template <bool RET, bool CONJ>
    __device__ __forceinline__ void add(bool first, bool link, float tr, float ti, float p, float hr, float hi, float qr, float qi)
    {
        if constexpr (RET) {
            Er *= p;
            Ei *= p;
            P *= p;
        }
        if (first) {
            Er = tr;
            Ei = ti;
        } else {
            float nr, ni;
            chain_step<CONJ>(tr, ti, hr, hi, qr, qi, Er, Ei, nr, ni);
            Er = nr;
            Ei = ni;
        }
        if (link) {
            const double Mr = (double)hr + (double)qr, Mi = (double)hi + (double)qi, t = mr * Mr - mi * Mi;
            mi = mr * Mi + mi * Mr;
            mr = t;
        }
    }
    template <bool RET, bool CONJ>
    __device__ __forceinline__ void link(float cr, float ci, float &Pr, float &Pi)      // E + P M^r c
    {
        const float ar = (float)mr, ai = (float)mi;
        if constexpr (RET) { cr *= P; ci *= P; }
        chain_step<CONJ>(Er, Ei, ar, ai, (float)(mr - (double)ar), (float)(mi - (double)ai), cr, ci, Pr, Pi);
    }
};
template <int JB, int NB, bool RET, bool PRE>
__device__ __forceinline__ bool chain_carry(const tagged_t *agg, const tagged_t *aggp, const tagged_t *pre, uint32_t id,
                                            uint32_t stride, int tt, int G, int lv, float hr, float hi, float qr, float qi,
                                            uint32_t spin_limit, uint32_t tag, float &cr, float &ci)
{
    const int r = tt & (G - 1);
    const bool first_group = tt == r;
    const uint32_t first = id - (uint32_t)r * stride;
    uint32_t spins = 0;
    ChainFold f;
    // (PRE: the prefix is asked for with the first aggregates: where it is already there, one round trip brings both)
    const tagged_t *src = pre + (size_t)(first - stride) * 2 * JB + lv;
    tagged_t w0 = 0, w1 = 0;
    if (PRE && !first_group) {
        w0 = tagged_load(src);
        w1 = tagged_load(src + JB);
    }
    for (int base = 0; base < r; base += NB) {
        tagged_t wr[NB], wi[NB], wp[RET ? NB : 1];
        while (true) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const size_t t = first + (uint32_t)(base + k < r ? base + k : r - 1) * stride;   // (past the end: the last again)
                wr[k] = tagged_load(agg + t * 2 * JB + lv);
                wi[k] = tagged_load(agg + t * 2 * JB + JB + lv);
                if constexpr (RET) wp[k] = tagged_load(aggp + t * JB + lv);
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                ok = ok && tagged_ok(wr[k], tag) && tagged_ok(wi[k], tag);
                // (the chain's first tile publishes no product: nothing comes before it)
                if constexpr (RET) ok = ok && (tagged_ok(wp[k], tag) || (first_group && (base + k < r ? base + k : r - 1) == 0));
            }
            if (group_all<JB>(ok)) break;
            if (++spins > spin_limit) return false;
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k)
            if (base + k < r)
                f.add<RET, false>(base + k == 0, !first_group, tagged_value(wr[k]), tagged_value(wi[k]), RET ? tagged_value(wp[RET ? k : 0]) : 1.f, hr, hi, qr, qi);
    }
    cr = f.Er;
    ci = f.Ei;
    if (first_group) return true;
    while (!group_all<JB>(tagged_ok(w0, tag) && tagged_ok(w1, tag))) {
        if (++spins > spin_limit) return false;
        __builtin_amdgcn_s_sleep(1);
        w0 = tagged_load(src);
        w1 = tagged_load(src + JB);
    }
    cr = tagged_value(w0);
    ci = tagged_value(w1);
    if (r > 0) f.link<RET, false>(cr, ci, cr, ci);
    return true;
}

// The same with all of a workgroup's segments reading: segment `seg` of NSEG takes tiles seg, seg + NSEG, ... of the r before this
// one in its group, NB per round trip, and leaves them in LDS (out [tile][2 or 3][JB]), where the fold finds them behind a barrier.
// One or two round trips for the whole group, by waves that would only wait: a group of 16 or a short chain of up to 64 took
// one per NB tiles.  False if a wait gave up (what it leaves is then meaningless).
template <int JB, int NB, int NSEG, bool RET>
__device__ __forceinline__ bool read_aggregates(float *out, const tagged_t *agg, const tagged_t *aggp, uint32_t id, uint32_t stride, int tt,
                                                int r, int seg, int lv, uint32_t spin_limit, uint32_t tag)
{
    const uint32_t first = id - (uint32_t)r * stride;
    uint32_t spins = 0;
    for (int base = seg; base < r; base += NB * NSEG) {
        tagged_t wr[NB], wi[NB], wp[RET ? NB : 1];
        while (true) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const size_t t = first + (uint32_t)(base + k * NSEG < r ? base + k * NSEG : base) * stride;     // (past the end: the first again)
                wr[k] = tagged_load(agg + t * 2 * JB + lv);
                wi[k] = tagged_load(agg + t * 2 * JB + JB + lv);
                if constexpr (RET) wp[k] = tagged_load(aggp + t * JB + lv);
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                ok = ok && tagged_ok(wr[k], tag) && tagged_ok(wi[k], tag);
                if constexpr (RET) ok = ok && (tagged_ok(wp[k], tag) || (tt == r && (base + k * NSEG < r ? base + k * NSEG : base) == 0));
            }
            if (group_all<JB>(ok)) break;
            if (++spins > spin_limit) return false;
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int t = base + k * NSEG;
            if (t < r) {
                float *o = out + (size_t)t * (RET ? 3 : 2) * JB + lv;
                o[0] = tagged_value(wr[k]);
                o[JB] = tagged_value(wi[k]);
                if constexpr (RET) o[2 * JB] = tagged_value(wp[k]);
            }
        }
    }
    return true;
}
template <int JB, bool RET, bool CONJ>
__device__ __forceinline__ bool fold_aggregates(const float *in, const tagged_t *pre, uint32_t id, uint32_t stride, int tt, int r, int lv,
                                                tagged_t w0, tagged_t w1, float hr, float hi, float qr, float qi, uint32_t spin_limit,
                                                uint32_t tag, float &cr, float &ci)
{
    const bool first_group = tt == r;
    ChainFold f;
#pragma unroll 4
    for (int t = 0; t < r; ++t) {
        const float *o = in + (size_t)t * (RET ? 3 : 2) * JB + lv;
        f.add<RET, CONJ>(t == 0, !first_group, o[0], o[JB], RET ? o[RET ? 2 * JB : 0] : 1.f, hr, hi, qr, qi);
    }
    cr = f.Er;
    ci = f.Ei;
    if (first_group) return true;
    const tagged_t *src = pre + (size_t)(id - (uint32_t)(r + 1) * stride) * 2 * JB + lv;
    for (uint32_t spins = 0; !group_all<JB>(tagged_ok(w0, tag) && tagged_ok(w1, tag));) {
        if (++spins > spin_limit) return false;
        __builtin_amdgcn_s_sleep(1);
        w0 = tagged_load(src);
        w1 = tagged_load(src + JB);
    }
    cr = tagged_value(w0);
    ci = tagged_value(w1);
    if (r > 0) f.link<RET, CONJ>(cr, ci, cr, ci);
    return true;
}

// Decoupled look-back, run by one group of LPR consecutive threads of a wave (thread lv of the
// group owns V lanes at lane offset `lo` of the tile slots; a slot is [2][JB] tagged words).
// `pred` is the chain predecessor's tile index, `depth` the number of tiles before this one in the
// chain (the chain's first tile always publishes a prefix).
//   The group reads the prefixes AND aggregates of the next NB predecessors in one round trip; a
//   tile's words count only when all of the group's lanes found their tags valid.  It stops at the
//   nearest tile with a valid prefix, provided every nearer tile has a valid aggregate; it waits
//   (bounded, polling one word per lane) on the nearest tile that has published nothing yet.  Then it walks forward from that
//   prefix through the aggregates with chain_step(), from the registers of the last window and, for
//   nearer tiles seen in earlier windows, by reading them again (published words never change
//   within a call).  In the common case -- a prefix within NB tiles -- that is one round trip.
// Returns false if a wait gave up (the carry is then meaningless).
// RET (data-dependent retention): an aggregate has a third word per lane, the product of the tile's
// retentions (aggp, [tile][JB]); a link then is P = T + product * M c.
template <int V, bool CONJ, int LPR, int NB, bool RET = false>
__device__ __forceinline__ bool look_back(const tagged_t *agg, const tagged_t *pre, uint32_t pred, uint32_t stride,
                                          int depth, int JB, int lo, int lv, const float (&hr)[V],
                                          const float (&hi)[V], const float (&qr)[V], const float (&qi)[V],
                                          uint32_t spin_limit, uint32_t tag, float (&cr)[V], float (&ci)[V],
                                          const tagged_t *aggp = nullptr)
{
    int base = 0;       // tiles at distance < base are known to hold aggregates
    uint32_t spins = 0;
    float ar[NB][V], ai[NB][V];      // aggregates of the current window
    float ap[RET ? NB : 1][V];
    int found = -1;                  // position of the prefix in the current window
    while (true) {
        const int w = depth - base < NB ? depth - base : NB;
        bool pok[NB], aok[NB];
        float pr_[NB][V], pi_[NB][V];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int dd = n < w ? base + n : base;      // (positions past the chain's start repeat a valid one)
            const size_t slot = (size_t)(pred - (uint32_t)dd * stride) * 2 * JB + lo;
            pok[n] = aok[n] = true;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const tagged_t w0 = tagged_load(pre + slot + v), w1 = tagged_load(pre + slot + JB + v);
                const tagged_t w2 = tagged_load(agg + slot + v), w3 = tagged_load(agg + slot + JB + v);
                pok[n] = pok[n] && tagged_ok(w0, tag) && tagged_ok(w1, tag);
                aok[n] = aok[n] && tagged_ok(w2, tag) && tagged_ok(w3, tag);
                pr_[n][v] = tagged_value(w0); pi_[n][v] = tagged_value(w1);
                ar[n][v] = tagged_value(w2);  ai[n][v] = tagged_value(w3);
                if constexpr (RET) {
                    const tagged_t w4 = tagged_load(aggp + (size_t)(pred - (uint32_t)dd * stride) * JB + lo + v);
                    aok[n] = aok[n] && tagged_ok(w4, tag);
                    ap[n][v] = tagged_value(w4);
                }
            }
        }
        compiler_fence();
        int stall = -1;
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            if (found < 0 && stall < 0 && n < w) {
                if (group_all<LPR>(pok[n])) {
                    found = n;
#pragma unroll
                    for (int v = 0; v < V; ++v) { cr[v] = pr_[n][v]; ci[v] = pi_[n][v]; }
                } else if (!group_all<LPR>(aok[n])) {
                    stall = n;
                }
            }
        }
        if (found >= 0) break;
        if (stall >= 0) {           // the tile at base + stall has published nothing yet
            base += stall;
            // wait for it on one word per lane (a light poll), then read the window again.  The
            // chain's first tile publishes a prefix only; every other tile publishes its aggregate first.
            const tagged_t *probe = (base == depth - 1 ? pre : agg) + (size_t)(pred - (uint32_t)base * stride) * 2 * JB + lo;
            while (true) {
                if (++spins > spin_limit) return false;
                __builtin_amdgcn_s_sleep(1);
                if (group_all<LPR>(tagged_ok(tagged_load(probe), tag))) break;
            }
        } else {
            base += w;              // aggregates only: look further back
            if (base >= depth) return false;   // cannot happen: the chain's first tile publishes a prefix
        }
    }
    // forward again: first the aggregates of the last window, nearest last
#pragma unroll
    for (int n = NB - 1; n >= 0; --n) {
        if (n < found) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                float nr, ni;
                if constexpr (RET) { cr[v] *= ap[n][v]; ci[v] *= ap[n][v]; }
                chain_step<CONJ>(ar[n][v], ai[n][v], hr[v], hi[v], qr[v], qi[v], cr[v], ci[v], nr, ni);
                cr[v] = nr;
                ci[v] = ni;
            }
        }
    }
    // then the tiles of earlier windows (nearer than `base`)
    for (int d = base - 1; d >= 0; d -= NB) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int dd = d - n < 0 ? 0 : d - n;
            const size_t slot = (size_t)(pred - (uint32_t)dd * stride) * 2 * JB + lo;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                ar[n][v] = tagged_value(tagged_load(agg + slot + v));
                ai[n][v] = tagged_value(tagged_load(agg + slot + JB + v));
                if constexpr (RET)
                    ap[n][v] = tagged_value(tagged_load(aggp + (size_t)(pred - (uint32_t)dd * stride) * JB + lo + v));
            }
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            if (d - n >= 0) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float nr, ni;
                    if constexpr (RET) { cr[v] *= ap[n][v]; ci[v] *= ap[n][v]; }
                    chain_step<CONJ>(ar[n][v], ai[n][v], hr[v], hi[v], qr[v], qi[v], cr[v], ci[v], nr, ni);
                    cr[v] = nr;
                    ci[v] = ni;
                }
            }
        }
    }
    return true;
}
#endif

}  // namespace cawn
