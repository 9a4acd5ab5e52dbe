// Fused forward: Temporal Syntax Cache conv -> clamp -> SiLU -> gate -> phasor -> causal phase
// accumulation -> clamp, single pass over HBM (Sec. 3.2 - 3.5 of the paper).
//
// Parallel structure.  The recurrence S[t] = p[t] + lambda S[t-1] has a per-lane constant
// multiplier, so a run of n tokens acts on an incoming state as  S_out = E + lambda^n S_in,
// with E the run's result from a zero state.  Three levels use that:
//   thread    : one lane x NSTEP consecutive tokens, serial, phasors kept in registers;
//   workgroup : NSEG such segments = one tile of TILE_T tokens; segment results meet in LDS;
//   grid      : tiles of one (batch row, lane block) form a chain in time.  A tile publishes its
//               aggregate E and finds its carry in one of two ways: it folds the aggregates before it
//               in its group of tiles into one link on the prefix of the group before (chain_carry; on
//               short tiles the whole chain is one group, and no prefix is passed on), or, in calls on
//               32-lane rows whose workgroups take several tiles, it looks back over earlier tiles until it
//               meets one that already knows its inclusive prefix, and publishes its own (look_back).
// After the carry is known each thread replays its NSTEP tokens from the true incoming state,
// clamps and stores.  Per token-lane HBM traffic: 8 bytes in, 8 bytes out.
//
// Scheduling.  Small calls have a workgroup for every tile, whose threads read their rows into registers (short tiles
// have theirs staged in LDS); larger ones run
// the persistent kernel (MANY, see launch_fwd_tile for the line): about as many workgroups as fit on the chip are launched
// and each loops over tiles, handed out by atomic tickets in the order (time tile, batch row,
// lane block) (see TileQueues).  Tickets go out in time order, so a tile only ever waits for tiles that a running
// workgroup already holds; all chains advance together, so tiles that happen to be slow (some
// address classes of the 128-byte lane-block rows are, by a quarter) are spread over every
// workgroup instead of leaving a few chains to finish alone; and the lane blocks of one row are
// in flight together, which keeps DRAM pages busy.  The ticket, the input rows and the lane
// constants of the NEXT tile are fetched while the current tile is in its communication phase,
// whose memory round trips would otherwise leave the SIMDs idle.
#pragma once
#include <atomic>
#include <type_traits>

#include "cawn_internal.hpp"

namespace cawn {

// Tuning aid, compiled only with -DCAWN_TIMING: per-tile time stamps (100 MHz counter) of the
// chain-owning thread, written behind the parameter partials in the workspace.
#ifdef CAWN_TIMING
#define CAWN_STAMP(k) do { if (tid == (NSEG - 1) * LPR) a.dbg[(size_t)id * 16 + (k)] = wall_clock64(); } while (0)
#else
#define CAWN_STAMP(k) do { } while (0)
#endif

typedef float v4f __attribute__((ext_vector_type(4)));
template <int V> struct Vec;
template <> struct Vec<1> {
    static __device__ __forceinline__ void ld(float (&d)[1], const float *p) { d[0] = *p; }
    static __device__ __forceinline__ void st(float *p, const float (&s)[1]) { *p = s[0]; }
};

// Position of a ticket in the problem: tickets count (time tile, batch row, lane block), lane block fastest.
struct TileId {
    int lb, b, tt;
    uint32_t id;     // unique tile index (workspace slot); the chain predecessor is id - B
};
__device__ __forceinline__ TileId decode_tile(uint32_t ticket, int nLB, int B, int nT)
{
    const uint32_t per_tt = (uint32_t)B * nLB;
    const uint32_t tt = ticket / per_tt, r = ticket - tt * per_tt;
    TileId t;
    t.tt = (int)tt;
    t.b = (int)(r / nLB);
    t.lb = (int)(r - (uint32_t)t.b * nLB);
    t.id = ((uint32_t)t.lb * nT + t.tt) * B + t.b;
    return t;
}

// The lane constants a forward tile keeps in registers, staged in LDS: lambda, lambda^(NSTEP s) for s = 1 .. NSEG - 1
// (segment 0 starts at the tile's first token: its power is 1), biases, retention bias, taps (HC: and the harmonic
// convolution's).  C_* are rows of the staged copy; the table's rows are in the same order with other powers between.
template <class G> struct FwdConsts {
    static constexpr int C_LR = 0, C_LI = 1, C_P = 2, C_BIAS_M = C_P + 2 * (G::NSEG - 1), C_BIAS_A = C_BIAS_M + 1,
                         C_RBIAS = C_BIAS_M + 2, C_W0 = C_BIAS_M + 3;
    static __device__ __forceinline__ int table_row(int r)
    {
        if (!G::SHORT)      // (the table's order with gaps)
            return R_LR + r + (r < C_P ? 0 : 2) + (r < C_BIAS_M ? 0 : R_BIAS_M - R_PSEG - 2 * G::NSEG);
        return r < C_P ? R_LR + r : (r < C_BIAS_M ? R_PSEGB + 2 + (r - C_P) : R_BIAS_M + (r - C_BIAS_M));
    }
};
// 16 bytes per lane per load: JB / 4 lanes cover a row.  Called by one wave.  Table rows are 256-byte aligned and
// padded, so every address is valid.
// Rows NCM .. NCR - 1: lambda^TILE_T as a double-float (table rows PT, PT + 1, PTL, PTL + 1).
// RUNS: two rows more in front of those, lambda^RUN (the table's first step between backward segments).
template <class G, int NCM, int PT, int PTL, bool RUNS>
__device__ __forceinline__ int const_row(int r)
{
    if (r < NCM) return FwdConsts<G>::table_row(r);
    r -= NCM;
    if (RUNS && r < 2) return R_PSEGB + 2 + r;
    r -= RUNS ? 2 : 0;
    return r < 2 ? PT + r : PTL + (r - 2);
}
template <class G, int NCR, int NCM, int PT, int PTL, bool RUNS>
__device__ __forceinline__ void stage_consts(float *sC, const float *table, int Jp, int lb, int lane)
{
    constexpr int JB = G::JB, LR = JB / 4, RPI = 64 / LR;      // lanes per row, rows per instruction
    const int r_in = lane / LR, c_in = (lane % LR) * 4;
#pragma unroll
    for (int i = 0; i < (NCR + RPI - 1) / RPI; ++i) {
        const int r = i * RPI + r_in;
        if (r < NCR) {
            const float *src = table + ((size_t)const_row<G, NCM, PT, PTL, RUNS>(r) * Jp + (size_t)lb * JB + c_in);
#if defined(__HIP_DEVICE_COMPILE__)
            __builtin_amdgcn_global_load_lds(src, sC + (size_t)(i * RPI) * JB, 16, 0, 0);
#else
            (void)src;
            (void)sC;
#endif
        }
    }
}

// VALVE: gate_mode 1, the per-head input valve of Sec. 3.3 in place of the per-lane threshold.
// RET: ret_mode 1, the retention of Sec. 3.3 item 4: gamma[t] = sigmoid(logit[t][head] + b_k) scales
// what arrives from token t-1 (accumulation equations of Sec. 3.4, printed with gamma_{t,j}).  A run of
// tokens then acts on an incoming state as S_out = E + (product of the run's gammas) e^{i n theta} S_in:
// the lane table holds pure rotations and every level carries the real product beside its aggregate.
// BF: activations (mag, ang in; z_re, z_im out) are bfloat16 in memory; arithmetic, state and
// checkpoints stay fp32 (Sec. 3.5 / Sec. 6.1 of the paper: the network runs in bf16, the accumulator in
// fp32).  A staged row of JB bf16 lanes is handled as JB/2 four-byte words; outputs are rounded to
// nearest even by the hardware conversion.
// (with bf16 rows the staged tile is half as large and a third workgroup fits a CU's LDS; the variants
// without the per-token retentions also fit its registers)
// HC: the depth-wise harmonic convolution of Sec. 3.6 applied to the clamped output before it is
// stored: channel = (plane, head), three taps along the harmonics of the head, zeros beyond its ends.
// Neighbouring harmonics are neighbouring lanes of a row (rows of 64 lanes here: one wave each).  A head
// of 128 or 256 lanes is a row of its own width (WIDE): the waves side by side leave the values of their outermost lanes in LDS
// between the recurrence and the convolution, which therefore run one after the other, the clamped states waiting in the
// registers of the phasors.  Every row is stored whole, by one workgroup.
// MANY: workgroups take several tiles (launch_fwd_tile); on 32-lane rows these calls pass a prefix on per tile (EACH).
// Long tiles without it: a workgroup for every tile (ONE).
template <class G, int KC, bool VALVE, bool RET, bool BF, bool HC, bool MANY>
__global__ __launch_bounds__(G::NT, G::SHORT ? (HC ? 2 : 4) : ((MANY ? BF : !BF && !VALVE) && !RET && !HC) ? CAWN_FWD_WAVES + 1 : CAWN_FWD_WAVES) void fwd_kernel(const FwdArgs a)
{
    constexpr int V = 1;                           // lanes per thread
    constexpr int TILE_T = G::TILE_T, NSTEP = G::NSTEP, NSEG = G::NSEG, LPR = G::JB;
    constexpr int JB = G::JB;
    constexpr int MW = JB / 32;                    // gate-mask words of a row
    static_assert(MW * NSTEP <= JB, "the gate mask: every word of a segment has a lane that keeps it");
    static_assert(!HC || JB >= 64, "harmonic convolution: a row is a wave, or a head of several");
    static_assert(!MANY || !G::SHORT, "short tiles: one a workgroup");
    constexpr bool WIDE = JB > 64;                 // a row is one head of WPS waves
    constexpr int WPS = WIDE ? JB / 64 : 1;
    static_assert(!WIDE || (HC && !G::SHORT), "rows of several waves: wide heads behind the harmonic convolution");
    constexpr bool EACH = MANY && JB == 32, ONE = !MANY && !G::SHORT;
    // One tile a workgroup, known at compile time: no loop, nothing kept across it.  On short tiles of 32 lanes the loop cost
    // 20 - 30 registers and, with retentions, 2 - 10 spilled ones: training step B3 L1777 J120 34.5 -> 33.5 us.
    constexpr bool SINGLE = !MANY;
    // (64-lane rows with retentions and several tiles a workgroup: at the register limit, the count in the middle spilled 6 more values; the paper's layer
    // in bf16, B1 L32768, 56.1 -> 57.3 us)
    constexpr bool COUNT_EARLY = !EACH && !(JB >= 64 && MANY && RET);
    // RUNS: a segment of 32 tokens is four runs of RUN, joined by the exact power lambda^RUN as segments are by theirs.  Within a
    // run the rounding of lambda to fp32 adds up, coherently over its tokens; short tiles hold it to 8 of them, and calls of
    // heads of 128 and 256 that short tiles once took run here: their rows are as wide as a head.  (The state's error, of its rms, on
    // lanes whose lambda rounds worst: 1.14e-6 in runs of 32, now 2.2e-7, short tiles 2.3e-7; with retentions of 0.95 from the data 4.0e-7 and
    // less than 3.4e-7.)  An instruction a token-lane and 8 - 10 registers, which these kernels have: B8 L8192 J768 F128 178.2 -> 178.6 us, bf16
    // 155.2 -> 156.0, F256 188.0 -> 189.3, B1 L700 13.7 both, with retentions 15.6 -> 15.5, F256 18.6 -> 18.4.  Not where retentions meet several tiles a
    // workgroup, calls that were never short: 13 registers more, conv 4 on rows of 128 leaves one wave a SIMD.  On rows of 32 and 64
    // lanes they cost the third workgroup of a compute unit, or spill 17: such calls keep their short tiles instead.
    constexpr int RUN = BwdGeom::NSTEP;
    constexpr bool RUNS = WIDE && (ONE || !RET);
    static_assert(!RUNS || NSTEP % RUN == 0, "whole runs");
    constexpr int HALO = KC > 0 ? KC - 1 : 0;
    constexpr int KC1 = KC > 0 ? KC : 1;
    constexpr int NT = G::NT;                      // threads
    constexpr int NW = NT / 64;                    // waves
    constexpr int JBS = BF ? JB / 2 : JB;          // four-byte words per staged row
    constexpr int NRTP = staged_rows<TILE_T, JBS, HALO>();   // staged rows per stream: time tile_t0-HALO+rr
    static_assert(JB <= 256 && 256 % JB == 0, "a staged row must fit a wave");
    static_assert(NW > WPS, "the last segment's waves own the chain, the others stage the next tile");

    // One tile a workgroup: the aggregates of a group's tiles, read by all segments where one group of threads would need more
    // than a round trip (NB tiles each); over the staged rows, which are dead by then
    constexpr int NB = G::SHORT ? (RET ? (HC ? 6 : 4) : (HC ? 8 : 6)) : (HC && RET ? 2 : (BF && !RET && !HC ? 4 : 7));
    // (not in the kernel of which three workgroups fit a compute unit: its registers are taken, 12 - 36 spilled)
    constexpr bool ALL_READ = SINGLE && (G::SHORT || BF || VALVE || RET || HC);
    constexpr int N_AGG = ALL_READ ? (G::SHORT ? FwdShort::MAX_CHAIN : 16) * (RET ? 3 : 2) * JB : 1, N_U = ONE ? 1 : 2 * NRTP * JBS;
    __shared__ __attribute__((aligned(16))) float sPoolU[N_AGG > N_U ? N_AGG : N_U];
    // ONE: a thread reads its rows from memory itself (see the loads below)
    float (*sU)[JBS] = reinterpret_cast<float (*)[JBS]>(&sPoolU[0]);  // [stream*NRTP + rr][lane]
    // element (row, lane) of the staged rows as fp32
    auto su = [&](int r, int l) -> float {
        if constexpr (BF) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(&sU[r][0])[l] << 16);
        else return sU[r][l];
    };
    __shared__ float sE[NSEG - 1][2][JB];          // (the last segment's is nobody's predecessor inside the tile)
    __shared__ float sCarry[2][JB];
    typedef FwdConsts<G> CR;
    // staged lane-constant rows.  ALL_READ: and lambda^TILE_T, which other kernels load where they need it -- a load on one of
    // several paths there, which the compiler waits for where the paths meet, behind the stores of the aggregate.  (The plain
    // fp32 kernel, three workgroups a compute unit: staged 26.2 us, loaded 25.4 for B4 L2048 J768 with a mask, inputs not cached)
    constexpr int NCM = CR::C_W0 + 2 * KC + (HC && !WIDE ? HC_ROWS : 0), C_RUN = NCM, C_PT = NCM + (RUNS ? 2 : 0),
                  NCR = C_PT + (ALL_READ ? 4 : 0);
    __shared__ __attribute__((aligned(16))) float sC[NCR][JB];
    // lambda^TILE_T as a double-float: leading part re, im, remainder re, im
    constexpr int PT = TILE_T == 64 ? R_PT64_HR : (TILE_T == FwdGeom::TILE_T ? R_PT_HR : R_PTB_HR);
    constexpr int PTL = TILE_T == 64 ? R_PT64_LR : PT + 2;
    static_assert(G::SHORT ? TILE_T == 64 && NSTEP == BwdGeom::NSTEP && NSEG <= BwdGeom::NSEG
                           : (TILE_T == FwdGeom::TILE_T || TILE_T == BwdGeom::TILE_T || TILE_T == 64) && NSTEP == FwdGeom::NSTEP,
                  "powers the lane table holds");
    // valve / retention groups per lane block: F >= 8, or F >= 16 with both (LDS: two workgroups per CU)
    // (HC: F >= 32, i.e. two groups of a 64-lane block)
    constexpr bool FACTORS = VALVE && !G::SHORT;         // the staged logits become factors in LDS (short tiles: on the way to every call's end)
    constexpr int GPB_MAX = WIDE ? 1 : HC ? 2 : ((VALVE && RET) ? 2 : 4) * (JB / 32);
    __shared__ float sV[VALVE ? TILE_T * GPB_MAX : 1];
    __shared__ float sR[RET ? TILE_T * GPB_MAX : 1];     // retention logits, laid out like sV
    __shared__ float sP[RET ? NSEG - 1 : 1][JB];                  // product of each segment's retentions
    // WIDE: the head's taps and biases, and the clamped states of the lanes on either side of a boundary between waves,
    // [plane][boundary][0: the lane below, 1: the lane above][token]
    __shared__ float sHW[WIDE ? HC_ROWS : 1];
    constexpr int NBD = WIDE ? WPS - 1 : 1;
    __shared__ __attribute__((aligned(16))) float sEdge[2][NBD][2][WIDE ? TILE_T : 1];
    __shared__ uint32_t sTicket[2], sLast, sEpoch;

    const int tid = threadIdx.x;
    const int lv = tid % LPR, seg = tid / LPR;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;   // (wave index: scalar)
    const uint32_t qtiles = (uint32_t)a.nLB * a.B * a.nT;     // all tiles of the call
    const bool is_tail_seg = seg == NSEG - 1;
    const bool owner_wave = wave >= NW - WPS;      // the waves holding the last segment own the chain
    const float *tail_in = a.state_in ? a.state_in + (size_t)a.B * 2 * a.J : nullptr;

    if (tid == 0) {
        const uint32_t e = flag_load(&a.hdr->epoch);     // both round trips at once
        const uint32_t t = EACH ? next_ticket_of(a.hdr) : first_ticket(a.hdr, a.tq, blockIdx.x);
        sEpoch = e;
        sTicket[0] = t;
        sLast = 0;
    }
    __syncthreads();
    uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)sTicket[0]);   // wave-uniform: index math stays scalar
    const uint32_t epoch = (uint32_t)__builtin_amdgcn_readfirstlane((int)sEpoch);
    const uint32_t tag = make_tag(epoch);      // of every word this call publishes

    // From here on the kernel's arguments are read from the kernel-argument segment again in every
    // phase of a tile (scalar loads next to their use; `ARGS_AGAIN()` makes the compiler forget what it
    // loaded) instead of living in scalar registers across the loop: kept there, they and what the
    // compiler derives from them overflow the scalar register file, and every overflowing value costs
    // vector registers and lane moves.
    typedef const __attribute__((address_space(4))) FwdArgs *KArgs;
    KArgs ap = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
#define a (*ap)
#define ARGS_AGAIN() asm volatile("" : "+s"(ap))
    // Stage a tile's input rows in LDS.  The chain-owning wave stays out of it: a wave's memory
    // operations complete in order, and its polls of other tiles must not queue behind a tile's
    // worth of HBM reads.
    const int ist32 = (int)a.ist;
    auto stage_tile = [&](const TileId &T) {
        if (owner_wave) return;
        if (wave == 0) stage_consts<G, NCR, NCM, PT, PTL, RUNS>(&sC[0][0], a.table, a.Jp, T.lb, lane);
#if defined(__HIP_DEVICE_COMPILE__)
        if (WIDE && wave == 0 && lane < HC_ROWS)
            __builtin_amdgcn_global_load_lds(a.table + ((size_t)(R_W0 + 2 * KC + lane) * a.Jp + (size_t)T.lb * JB), &sHW[0], 4, 0, 0);
#endif
        if (VALVE && wave == 0) stage_valve<TILE_T, JB>(&sV[0], a.valve, T.b, T.tt * TILE_T, T.lb, a.L, a.H, a.F, a.gpb, lane);
        if (RET && wave == 0) stage_valve<TILE_T, JB>(&sR[0], a.ret, T.b, T.tt * TILE_T, T.lb, a.L, a.H, a.F, a.gpb, lane);
        // (bf16: rows of J/2 words at half the strides; the fp32 conv history is read at its point of use)
        if (a.stage16)
            stage_rows<TILE_T, JBS, HALO, 16>(&sU[0][0], a.mag, a.ang, BF ? nullptr : tail_in, T.b, T.tt * TILE_T, T.lb,
                                      BF ? a.J / 2 : a.J, a.L, BF ? a.isb / 2 : a.isb, BF ? ist32 / 2 : ist32, wave, NW - WPS, lane);
        else
            stage_rows<TILE_T, JBS, HALO, 4>(&sU[0][0], a.mag, a.ang, BF ? nullptr : tail_in, T.b, T.tt * TILE_T, T.lb,
                                     BF ? a.J / 2 : a.J, a.L, BF ? a.isb / 2 : a.isb, BF ? ist32 / 2 : ist32, wave, NW - WPS, lane);
    };

    TileId T{};
    if (ticket < qtiles) {
        T = decode_tile(ticket, a.nLB, a.B, a.nT);
        if constexpr (!ONE) stage_tile(T);
    }

    // ONE: the rows of my segment, HALO of the one before it among them, straight into registers.  Nothing has to be
    // staged ahead in such a call, a thread's rows are its own, and the first of them are worked on while the
    // last are on their way; without the staged tile in LDS a third workgroup fits a compute unit.  Staged, such a call went
    // through its loads, its arithmetic and its stores one after the other on the whole chip, and 768 tiles of B4 L2048 J768
    // took two rounds: 35.2 -> 25.1 us with this; B1 L4096 J768 17.8 -> 16.2.  (The KC - 1 rows that two
    // segments share are read by both, the second time from a cache.)
    constexpr int NRD = ONE ? NSTEP + HALO : 1;
    typedef std::conditional_t<BF, uint16_t, float> elem;
    elem dm[NRD], da[NRD];
    uint32_t dmh[KC1], dah[KC1];   // BF: the HALO first rows as the four-byte words that hold them, or the history's fp32 values
    bool from_hist = false;
    if constexpr (ONE) {
        // What the tile's threads share -- lane constants, logits -- goes to LDS by way of registers, asked for ahead of the
        // rows: direct-to-LDS loads in flight would make the compiler wait for everything at the first read of LDS.
        constexpr int NCQ = (NCR * JB / 4 + NT - 1) / NT, NLG = (TILE_T * GPB_MAX + NT - 1) / NT;
        v4f cv[NCQ];
        float lgv[VALVE ? NLG : 1], lgr[RET ? NLG : 1], hcv = 0.f;
        if (WIDE && tid < HC_ROWS) hcv = a.table[(size_t)(R_W0 + 2 * KC + tid) * a.Jp + (size_t)T.lb * JB];
#pragma unroll
        for (int q = 0; q < NCQ; ++q) {
            const int w = q * NT + tid < NCR * JB / 4 ? q * NT + tid : 0;
            cv[q] = *reinterpret_cast<const v4f *>(a.table + (size_t)const_row<G, NCM, PT, PTL, RUNS>(w / (JB / 4)) * a.Jp + (size_t)T.lb * JB + w % (JB / 4) * 4);
        }
        auto logit = [&](const float *p, int i) {       // (beyond the end: a valid address, never used)
            const int t = T.tt * TILE_T + i % TILE_T, g = i / TILE_T, h = (T.lb * JB) / a.F + (g < a.gpb ? g : 0);
            return p[((size_t)T.b * a.L + (t < a.L ? t : a.L - 1)) * a.H + (h < a.H ? h : a.H - 1)];
        };
#pragma unroll
        for (int q = 0; q < NLG; ++q) {
            if constexpr (VALVE) lgv[q] = logit(a.valve, q * NT + tid);
            if constexpr (RET) lgr[q] = logit(a.ret, q * NT + tid);
        }
        compiler_fence();       // (the rows in their order behind these, and)
        // Rows outside the call have the address of one inside it (a row before the first token wraps to the last one's):
        // their values are not used.  One straight path, no branch between a load and its use: the compiler's waits are
        // exact only there.
        constexpr uint32_t ESZ = BF ? 2u : 4u;
        const int jl = T.lb * JB + lv;
        const uint32_t jc = (uint32_t)(jl < a.J ? jl : 0), istb = (uint32_t)ist32 * ESZ;
        const int first = T.tt == 0 ? 0 : T.tt * TILE_T - HALO, end = (T.tt + 1) * TILE_T < a.L ? (T.tt + 1) * TILE_T : a.L;
        const uint32_t last = (uint32_t)(end - 1 - first) * istb + jc * ESZ, off0 = (uint32_t)(seg * NSTEP - (T.tt == 0 ? HALO : 0)) * istb + jc * ESZ;
        const long long at = ((long long)T.b * a.isb + (long long)first * a.ist) * (long long)ESZ;
        const char *um = reinterpret_cast<const char *>(a.mag) + at, *ua = reinterpret_cast<const char *>(a.ang) + at;
        // the rows before the first token: the carried history's
        from_hist = HALO > 0 && tail_in && T.tt == 0 && seg == 0;
        const char *hm = tail_in ? reinterpret_cast<const char *>(tail_in + (size_t)T.b * HALO * 2 * a.J) : um;
        auto ld = [](const char *p) { return __builtin_nontemporal_load(reinterpret_cast<const elem *>(p)); };
#pragma unroll
        for (int r = 0; r < NRD; ++r) {
            uint32_t off = off0 + (uint32_t)r * istb;
            off = off < last ? off : last;
            const uint32_t h = ((uint32_t)(r * 2) * (uint32_t)a.J + jc) * 4u;
            if (BF && r < HALO) {
                dmh[r] = *reinterpret_cast<const uint32_t *>(from_hist ? hm + h : um + (off & ~3u));
                dah[r] = *reinterpret_cast<const uint32_t *>(from_hist ? hm + h + (uint32_t)a.J * 4u : ua + (off & ~3u));
            } else {
                const bool fh = r < HALO && from_hist;
                dm[r] = ld(fh ? hm + h : um + off);
                da[r] = ld(fh ? hm + h + (uint32_t)a.J * 4u : ua + off);
            }
        }
        compiler_fence();       // (all of it on its way before anything is waited for)
        if (WIDE && tid < HC_ROWS) sHW[tid] = hcv;
#pragma unroll
        for (int q = 0; q < NCQ; ++q) {
            const int w = q * NT + tid;
            if (w < NCR * JB / 4) *reinterpret_cast<v4f *>(&sC[w / (JB / 4)][w % (JB / 4) * 4]) = cv[q];
        }
#pragma unroll
        for (int q = 0; q < NLG; ++q) {
            if (VALVE && q * NT + tid < TILE_T * GPB_MAX) sV[q * NT + tid] = valve_factor(lgv[VALVE ? q : 0], a.valve_thr);
            if (RET && q * NT + tid < TILE_T * GPB_MAX) sR[q * NT + tid] = lgr[RET ? q : 0];
        }
    } else {
        wait_vm<0>();     // the first tile's staged rows
        if (FACTORS && wave == 0) valve_factors<TILE_T>(&sV[0], a.valve_thr, a.gpb, lane);
    }

    float lr[V], li[V], pfr[V], pfi[V], psr[V], psi[V];
    float prr[V], pri[V];                          // RUNS: lambda^RUN
    float wm[KC1][V], wa[KC1][V], bm[V], ba[V];
    float rb[V];                                   // RET: static retention bias of my lanes
    float hw[2][3], hb[2];                         // HC: taps and bias of my lane's two channels

    for (int it = 0; ticket < qtiles; ++it) {
        ARGS_AGAIN();
        const GateSet gs_ = {a.gs.a1, a.gs.b1, a.gs.a2, a.gs.b2};
        const uint32_t id = T.id;
        const int b = T.b, tt = T.tt;
        const int j0 = T.lb * JB + lv * V;
        const bool active = j0 < a.J;
        const int t0 = tt * TILE_T + seg * NSTEP;

        // ticket of the next tile: asked for now, parked in LDS after the front-end (the round trip
        // of the atomic stays off the path to the barrier below)
        uint32_t ticket_ahead;   // (only thread 0's copy is ever set or read; no initialiser, so no
                             // merge of values that would wait for the atomic right here)
        if (tid == 0) {
            if (SINGLE || (!EACH && a.tq.one_each)) ticket_ahead = NO_TICKET;
            else ticket_ahead = next_ticket_of(a.hdr);
        }

        // ---- the staged rows have landed (each wave waited for its own loads: before the loop, or
        //      at the end of the previous iteration)
        lds_barrier();
        CAWN_STAMP(0);

        // ---- lane constants of this tile's lane block, staged with its rows
        {
            auto cst = [&](float(&d)[V], int r) {
#pragma unroll
                for (int v = 0; v < V; ++v) d[v] = sC[r][lv * V + v];
            };
            cst(lr, CR::C_LR);
            cst(li, CR::C_LI);
            if (RUNS) {
                cst(prr, RUNS ? C_RUN : 0);
                cst(pri, RUNS ? C_RUN + 1 : 0);
            }
            cst(pfr, CR::C_P);                    // lambda^NSTEP
            cst(pfi, CR::C_P + 1);
            cst(psr, CR::C_P + 2 * (seg > 0 ? seg - 1 : 0));           // lambda^(NSTEP*seg)
            cst(psi, CR::C_P + 2 * (seg > 0 ? seg - 1 : 0) + 1);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                psr[v] = seg > 0 ? psr[v] : 1.f;
                psi[v] = seg > 0 ? psi[v] : 0.f;
                bm[v] = ba[v] = 0.f;
#pragma unroll
                for (int k = 0; k < KC1; ++k) wm[k][v] = wa[k][v] = 0.f;
            }
            if (RET) cst(rb, CR::C_RBIAS);
            if (HC) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    hb[p] = WIDE ? sHW[WIDE ? 6 + p : 0] : sC[WIDE ? 0 : CR::C_W0 + 2 * KC + 6 + p][lv];
#pragma unroll
                    for (int k = 0; k < 3; ++k) hw[p][k] = WIDE ? sHW[WIDE ? 3 * p + k : 0] : sC[WIDE ? 0 : CR::C_W0 + 2 * KC + 3 * p + k][lv];
                }
            }
            if (KC > 0) {
                cst(bm, CR::C_BIAS_M);
                cst(ba, CR::C_BIAS_A);
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    cst(wm[k], CR::C_W0 + k);
                    cst(wa[k], CR::C_W0 + KC + k);
                }
            }
        }

        // ---- front-end, phasors, local scan from zero.  Rows come from LDS as a sliding window.
        float pr[NSTEP][V], pi[NSTEP][V];
        float Er[V], Ei[V];
        constexpr int NER = RUNS ? NSTEP / RUN - 1 : 1;
        float er[NER][V], ei[NER][V], rp[NER][V]; // RUNS: what each run but the last adds, from zero, and RET: its retentions' product
        // (a run's step: R = (its retentions' product) lambda^RUN R + what it adds)
        auto run_step = [&](float &Rr_, float &Ri_, float q, float x, float y, int v) {
            const float ar = Rr_, ai = Ri_;
            if (RET) {
                const float rr = __builtin_fmaf(prr[v], ar, -pri[v] * ai);
                const float ri = __builtin_fmaf(pri[v], ar, prr[v] * ai);
                Rr_ = __builtin_fmaf(q, rr, x);
                Ri_ = __builtin_fmaf(q, ri, y);
            } else {
                Rr_ = __builtin_fmaf(prr[v], ar, __builtin_fmaf(-pri[v], ai, x));
                Ri_ = __builtin_fmaf(pri[v], ar, __builtin_fmaf(prr[v], ai, y));
            }
        };
        float gm[RET ? NSTEP : 1][V], Pth[V];     // RET: retention of each token, product over my tokens
        uint32_t mword = 0;                       // gate mask: my 32 lanes' word of my segment's token lv % 32
        const bool zero_hist = HALO > 0 && !tail_in && tt == 0 && seg == 0;   // rows before a sequence start
        // bf16: the carried conv history is fp32 and is not staged; the one segment that needs it reads it
        // here (and waits for it here, so that no wait for it lands in the common path)
        float hwm[KC1][V], hwa[KC1][V];
#pragma unroll
        for (int k = 0; k < KC1; ++k)
#pragma unroll
            for (int v = 0; v < V; ++v) hwm[k][v] = hwa[k][v] = 0.f;
        const bool hist_bf = !ONE && BF && HALO > 0 && tail_in && tt == 0 && seg == 0;
        if (hist_bf) {
#pragma unroll
            for (int k = 0; k < HALO; ++k) {
                const size_t o = ((size_t)(b * HALO + k) * 2) * a.J + (active ? j0 : 0);
                hwm[k][0] = tail_in[o];
                hwa[k][0] = tail_in[o + a.J];
            }
            wait_vm<0>();
        }
        // (my lane's logits: a block holds whole heads, a part of one, or, where a head ends inside it, the end of one and
        // the start of the next)
        const int vgroup = a.F < JB ? (lv * V) / a.F : (JB > 32 && !HC && lv >= a.F - (T.lb * JB) % a.F ? 1 : 0);
        const int vbase = (VALVE || RET) ? vgroup * TILE_T + seg * NSTEP : 0;
        // row r of my segment, HALO of the segment before it first
        auto own = [&](int r, const elem(&d)[NRD], const uint32_t(&dh)[KC1]) -> float {
            if constexpr (!BF) return d[r];
            else if (r >= HALO) return from_bf16(d[r]);
            else return __uint_as_float(from_hist ? dh[r] : (lv & 1) ? dh[r] & 0xffff0000u : dh[r] << 16);   // (even strides: odd lanes are the upper halves)
        };
        auto row_m = [&](int r) -> float { if constexpr (ONE) return own(r, dm, dmh); else return su(seg * NSTEP + r, lv); };
        auto row_a = [&](int r) -> float { if constexpr (ONE) return own(r, da, dah); else return su(NRTP + seg * NSTEP + r, lv); };
        // The mode switches are uniform over the launch; each combination gets its own straight-line
        // copy of the loop, so that the tokens' dependent chains (exp -> rcp -> sin/cos) interleave.
        auto front_end = [&](auto amp_c, auto small_c, auto mask_c) {
            constexpr bool AMP = decltype(amp_c)::value, SMALL = decltype(small_c)::value;
            constexpr bool MASK = decltype(mask_c)::value;
            float wnm[KC1][V], wna[KC1][V];           // window: rows i .. i+KC-1 of my segment
            // (row r of my segment lives in slot r % KC1: no register shuffling as the window slides)
#pragma unroll
            for (int k = 0; k < KC1 - 1; ++k) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    wnm[k % KC1][v] = zero_hist ? 0.f : (hist_bf ? hwm[k][v] : row_m(k));
                    wna[k % KC1][v] = zero_hist ? 0.f : (hist_bf ? hwa[k][v] : row_a(k));
                }
            }
#pragma unroll
            for (int v = 0; v < V; ++v) { Er[v] = Ei[v] = 0.f; Pth[v] = 1.f; }
            float Ar[V], Ai[V], Qr[V];                // RUNS: the segment up to my run's start; RET: the product of my run's retentions
#pragma unroll
            for (int v = 0; v < V; ++v) Qr[v] = 1.f;
#pragma unroll
            for (int i = 0; i < NSTEP; ++i) {
                if (RUNS && i > 0 && i % RUN == 0) {
                    const int k = RUNS ? i / RUN - 1 : 0;
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        er[k][v] = Er[v];
                        ei[k][v] = Ei[v];
                        rp[k][v] = Qr[v];
                        if (k > 0) {
                            run_step(Ar[v], Ai[v], Qr[v], Er[v], Ei[v], v);
                        } else {
                            Ar[v] = Er[v];
                            Ai[v] = Ei[v];
                        }
                        Pth[v] *= Qr[v];
                        Qr[v] = 1.f;
                        Er[v] = Ei[v] = 0.f;
                    }
                }
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    wnm[(i + HALO) % KC1][v] = row_m(i + HALO);
                    wna[(i + HALO) % KC1][v] = row_a(i + HALO);
                }
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float zm, xm, phi;
                    if (KC > 0) {
                        zm = bm[v];
                        float za = ba[v];
#pragma unroll
                        for (int k = 0; k < KC; ++k) {
                            zm = __builtin_fmaf(wm[k][v], wnm[(i + k) % KC1][v], zm);
                            za = __builtin_fmaf(wa[k][v], wna[(i + k) % KC1][v], za);
                        }
                        const float cm = clampf(zm, a.conv_clamp), ca = clampf(za, a.conv_clamp);
                        xm = cm * sigmoid_fast(cm);
                        phi = ca * sigmoid_fast(ca);
                    } else {
                        zm = wnm[i % KC1][v];
                        xm = zm;
                        phi = wna[i % KC1][v];
                    }
                    const float amp = AMP ? __builtin_fminf(softplus_fast(xm), 10.0f) : xm;
                    bool g;
                    float ag;
                    if (VALVE) {      // beta = sigmoid(logit - 3), zero when the valve is closed
                        const float beta = FACTORS ? sV[vbase + i] : valve_factor(sV[vbase + i], a.valve_thr);
                        g = beta >= 0.0f;
                        ag = g ? amp * beta : 0.0f;
                    } else {
                        g = in_gate(gs_, zm);
                        ag = g ? amp : 0.0f;
                    }
                    float s, c;
                    if (SMALL) sincos_small(phi, s, c);
                    else sincos_fast(phi, s, c);
                    pr[i][v] = ag * c;
                    pi[i][v] = ag * s;
                    if (MASK) {
                        // The comparison's result is already a 64-bit lane mask: its two halves are the words of
                        // this token (32-lane rows: in the wave's two segments), and lane i of 32 keeps token i's.  (Packed
                        // by five lane exchanges per token, the mask took 7 of a tile's 15 us: B4 L2048 J768 with
                        // a mask 46.2 -> 35.4 us; then a select of the half and of the lane, five instructions, now two.)
                        [[maybe_unused]] const unsigned long long bal = __builtin_amdgcn_ballot_w64(g & active);
#if defined(__HIP_DEVICE_COMPILE__)
                        asm("s_nop 1\n"      // (wait states, should a vector instruction have written the mask)
                            "v_writelane_b32 %0, %1, %3\n"
                            "v_writelane_b32 %0, %2, %4"
                            : "+v"(mword) : "s"((uint32_t)bal), "s"((uint32_t)(bal >> 32)), "i"(i), "i"(32 + i));
#endif
                    }
                    float nr, ni;
                    if (RET) {
                        const float gmv = sigmoid_fast(sR[vbase + i] + rb[v]);
                        gm[i][v] = gmv;
                        (RUNS ? Qr[v] : Pth[v]) *= gmv;
                        const float rr = __builtin_fmaf(lr[v], Er[v], -li[v] * Ei[v]);
                        const float ri = __builtin_fmaf(li[v], Er[v], lr[v] * Ei[v]);
                        nr = __builtin_fmaf(gmv, rr, pr[i][v]);
                        ni = __builtin_fmaf(gmv, ri, pi[i][v]);
                    } else {
                        nr = __builtin_fmaf(lr[v], Er[v], __builtin_fmaf(-li[v], Ei[v], pr[i][v]));
                        ni = __builtin_fmaf(li[v], Er[v], __builtin_fmaf(lr[v], Ei[v], pi[i][v]));
                    }
                    Er[v] = nr;
                    Ei[v] = ni;
                }
            }
            if (RUNS) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    run_step(Ar[v], Ai[v], Qr[v], Er[v], Ei[v], v);
                    Er[v] = Ar[v];
                    Ei[v] = Ai[v];
                    Pth[v] *= Qr[v];
                }
            }
        };
        {
            using T_ = std::true_type;
            using F_ = std::false_type;
            switch ((a.amp_mode ? 4 : 0) | (a.small_angle ? 2 : 0) | (a.mask ? 1 : 0)) {
            case 0: front_end(F_{}, F_{}, F_{}); break;
            case 1: front_end(F_{}, F_{}, T_{}); break;
            case 2: front_end(F_{}, T_{}, F_{}); break;
            case 3: front_end(F_{}, T_{}, T_{}); break;
            case 4: front_end(T_{}, F_{}, F_{}); break;
            case 5: front_end(T_{}, F_{}, T_{}); break;
            case 6: front_end(T_{}, T_{}, F_{}); break;
            default: front_end(T_{}, T_{}, T_{}); break;
            }
        }
        CAWN_STAMP(2);

        ARGS_AGAIN();
        // ---- segments meet in LDS; after this barrier nobody reads the staged rows any more
        if (!is_tail_seg) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                sE[seg][0][lv * V + v] = Er[v];
                sE[seg][1][lv * V + v] = Ei[v];
                if (RET) sP[seg][lv * V + v] = Pth[v];
            }
        }
        if (!SINGLE && tid == 0) sTicket[(it + 1) & 1] = ticket_ahead;
        lds_barrier();
        CAWN_STAMP(3);

        // ---- start staging the next tile (it lands during this tile's communication phase)
        const uint32_t next_ticket = SINGLE ? NO_TICKET : (uint32_t)__builtin_amdgcn_readfirstlane((int)sTicket[(it + 1) & 1]);
        TileId Tn{};
        if (!SINGLE && next_ticket < qtiles) {
            Tn = decode_tile(next_ticket, a.nLB, a.B, a.nT);
            stage_tile(Tn);
        }

        ARGS_AGAIN();
        float Xr[V], Xi[V];   // state entering my segment, from a zero tile input
        float Cs[V];          // RET: product of the retentions of the segments before mine
#pragma unroll
        for (int v = 0; v < V; ++v) { Xr[v] = Xi[v] = 0.f; Cs[v] = 1.f; }
        for (int qq = 0; qq < seg; ++qq) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float er = sE[qq][0][lv * V + v], ei = sE[qq][1][lv * V + v];
                float nr, ni;
                if (RET) {
                    const float pq = sP[qq][lv * V + v];
                    const float rr = __builtin_fmaf(pfr[v], Xr[v], -pfi[v] * Xi[v]);
                    const float ri = __builtin_fmaf(pfi[v], Xr[v], pfr[v] * Xi[v]);
                    nr = __builtin_fmaf(pq, rr, er);
                    ni = __builtin_fmaf(pq, ri, ei);
                    Cs[v] *= pq;
                } else {
                    nr = __builtin_fmaf(pfr[v], Xr[v], __builtin_fmaf(-pfi[v], Xi[v], er));
                    ni = __builtin_fmaf(pfi[v], Xr[v], __builtin_fmaf(pfr[v], Xi[v], ei));
                }
                Xr[v] = nr;
                Xi[v] = ni;
            }
        }

        // (the last tile of a workgroup that is counted early: by a wave that waits for the owner's carry)
        if constexpr (COUNT_EARLY) {
            const TileQueues tq_ = {a.tq.units, a.tq.one_each, a.tq.group};
            if (next_ticket >= qtiles && counts_early(tq_, epoch) && tid == 0 &&
                leave_last(a.hdr, tq_, blockIdx.x, gridDim.x, leave_ask(a.hdr, tq_, blockIdx.x, gridDim.x)))
                reset_header(a.hdr, epoch + 1u, 0u, 1u);
        }

        // ---- chain.  The threads of the last segment own the tile aggregate: they publish it, do
        //      the look-back and publish the prefix, all within their own wave (stores are waited
        //      for with that wave's vmcnt, so no workgroup barrier sits on the publication path).
        const size_t slot = (size_t)id * 2 * JB + lv * V;
        // (what this tile publishes: its aggregate, the chain's first tile its prefix instead; the last of a
        // group also its prefix; the chain's last tile nothing)
        // (EACH: a prefix per tile, the first tile's with the others)
        const int group = EACH ? 1 : (int)a.tq.group;
        const bool feeds = tt + 1 < a.nT, ends_group = EACH || (tt & (group - 1)) == group - 1;
        const int before = tt & (group - 1);                     // tiles before this one in its group
        const bool all_read = ALL_READ && before > NB;           // (uniform over the workgroup)
        float Tr[V], Ti[V], hr[V], hi[V], qr[V], qi[V];
        float Pt[V];      // RET: product of the whole tile's retentions
        tagged_t w0 = 0, w1 = 0;
        if (is_tail_seg) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if (RET) {
                    const float rr = __builtin_fmaf(pfr[v], Xr[v], -pfi[v] * Xi[v]);
                    const float ri = __builtin_fmaf(pfi[v], Xr[v], pfr[v] * Xi[v]);
                    Tr[v] = __builtin_fmaf(Pth[v], rr, Er[v]);
                    Ti[v] = __builtin_fmaf(Pth[v], ri, Ei[v]);
                    Pt[v] = Cs[v] * Pth[v];
                } else {
                    Tr[v] = __builtin_fmaf(pfr[v], Xr[v], __builtin_fmaf(-pfi[v], Xi[v], Er[v]));
                    Ti[v] = __builtin_fmaf(pfi[v], Xr[v], __builtin_fmaf(pfr[v], Xi[v], Ei[v]));
                    Pt[v] = 1.f;
                }
                hr[v] = hi[v] = qr[v] = qi[v] = 0.f;
            }
            if constexpr (ALL_READ) {
                hr[0] = sC[ALL_READ ? C_PT : 0][lv];
                hi[0] = sC[ALL_READ ? C_PT + 1 : 0][lv];
                qr[0] = sC[ALL_READ ? C_PT + 2 : 0][lv];
                qi[0] = sC[ALL_READ ? C_PT + 3 : 0][lv];
            } else if (active) {   // lambda^TILE_T as a double-float
                const float *tb = a.table + j0;
                Vec<V>::ld(hr, tb + (size_t)PT * a.Jp);
                Vec<V>::ld(hi, tb + (size_t)(PT + 1) * a.Jp);
                Vec<V>::ld(qr, tb + (size_t)PTL * a.Jp);
                Vec<V>::ld(qi, tb + (size_t)(PTL + 1) * a.Jp);
            }
            if (tt > 0 && feeds && (EACH || !ends_group)) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    tagged_store(a.agg + slot + v, Tr[v], tag);
                    tagged_store(a.agg + slot + JB + v, Ti[v], tag);
                    if (RET) tagged_store(a.aggp + (size_t)id * JB + lv * V + v, Pt[v], tag);
                }
            }
            if (all_read && tt != before) {       // (the prefix is asked for ahead of the aggregates)
                const tagged_t *src = a.pre + (size_t)(id - (uint32_t)(before + 1) * (uint32_t)a.B) * 2 * JB + lv;
                w0 = tagged_load(src);
                w1 = tagged_load(src + JB);
            }
        }
        bool read_ok = true;
        if constexpr (ALL_READ) {
            if (all_read) {
                read_ok = read_aggregates<JB, HC && RET ? 2 : 4, NSEG, RET>(&sPoolU[0], a.agg, a.aggp, id, (uint32_t)a.B, tt, before, seg, lv,
                                                                           a.spin_limit, tag);
                if (!read_ok && lv % 64 == 0) __hip_atomic_store(&a.hdr->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lds_barrier();
            }
        }
        if (is_tail_seg) {
            float cr[V], ci[V];
#pragma unroll
            for (int v = 0; v < V; ++v) cr[v] = ci[v] = 0.f;
            if (tt == 0) {
                if (a.state_in && active) {
                    Vec<V>::ld(cr, a.state_in + ((size_t)b * 2 + 0) * a.J + j0);
                    Vec<V>::ld(ci, a.state_in + ((size_t)b * 2 + 1) * a.J + j0);
                }
            } else {
                bool got;
                if constexpr (EACH)
                    got = look_back<V, false, LPR, 2, RET>(a.agg, a.pre, id - (uint32_t)a.B, (uint32_t)a.B, tt, JB, lv * V, lv, hr, hi,
                                                           qr, qi, a.spin_limit, tag, cr, ci, a.aggp);
                else if (all_read)
                    got = fold_aggregates<JB, RET, false>(&sPoolU[0], a.pre, id, (uint32_t)a.B, tt, before, lv, w0, w1, hr[0], hi[0], qr[0], qi[0],
                                                   a.spin_limit, tag, cr[0], ci[0]);
                else
                    got = chain_carry<JB, NB, RET, !G::SHORT && !(HC && RET)>(a.agg, a.aggp, a.pre, id, (uint32_t)a.B, tt, group, lv, hr[0], hi[0], qr[0],
                                                     qi[0], a.spin_limit, tag, cr[0], ci[0]);
                if (!got) {
                    // gave up: flag the workspace, keep going so that every wave exits.  (Rows of 128 and 256 lanes: each
                    // wave waits for its own lanes, and gives up by itself)
                    if (lv % 64 == 0) __hip_atomic_store(&a.hdr->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            CAWN_STAMP(5);
            // Every load of this block is complete from here on, on every path: a load that some path
            // never uses would stay "in flight" in the compiler's bookkeeping and cost a full wait
            // where its register is reused -- in the replay below, behind the prefix stores.
#pragma unroll
            for (int v = 0; v < V; ++v) asm volatile("" ::"v"(hr[v]), "v"(hi[v]), "v"(qr[v]), "v"(qi[v]));
#pragma unroll
            for (int v = 0; v < V; ++v) {
                sCarry[0][lv * V + v] = cr[v];
                sCarry[1][lv * V + v] = ci[v];
            }
            if (feeds && (tt == 0 || ends_group)) {   // the tile's inclusive prefix for the chain
                tagged_t *pre = tt == 0 && !EACH ? a.agg : a.pre;
                float P_r[V], P_i[V];
#pragma unroll
                for (int v = 0; v < V; ++v)
                    chain_step<false>(Tr[v], Ti[v], hr[v], hi[v], qr[v], qi[v], RET ? Pt[v] * cr[v] : cr[v],
                                      RET ? Pt[v] * ci[v] : ci[v], P_r[v], P_i[v]);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    tagged_store(pre + slot + v, P_r[v], tag);
                    tagged_store(pre + slot + JB + v, P_i[v], tag);
                }
            }
        }
        lds_barrier_raw();     // the next tile's rows are still on their way
        CAWN_STAMP(6);

        ARGS_AGAIN();
        // ---- true state entering my segment
        float Sr[V], Si[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float cr = sCarry[0][lv * V + v], ci = sCarry[1][lv * V + v];
            if (RET) {
                const float rr = __builtin_fmaf(psr[v], cr, -psi[v] * ci);
                const float ri = __builtin_fmaf(psi[v], cr, psr[v] * ci);
                Sr[v] = __builtin_fmaf(Cs[v], rr, Xr[v]);
                Si[v] = __builtin_fmaf(Cs[v], ri, Xi[v]);
            } else {
                Sr[v] = __builtin_fmaf(psr[v], cr, __builtin_fmaf(-psi[v], ci, Xr[v]));
                Si[v] = __builtin_fmaf(psi[v], cr, __builtin_fmaf(psr[v], ci, Xi[v]));
            }
        }

        // RUNS: the state at the next run's start, behind the run that ends with token i
        float Rr[V], Ri[V];
#pragma unroll
        for (int v = 0; v < V; ++v) { Rr[v] = Sr[v]; Ri[v] = Si[v]; }
        auto next_run = [&](int i) {
            if constexpr (RUNS) {
                if ((i + 1) % RUN != 0 || i + 1 >= NSTEP) return;
                const int k = (i + 1) / RUN - 1;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    run_step(Rr[v], Ri[v], rp[k][v], er[k][v], ei[k][v], v);
                    Sr[v] = Rr[v];
                    Si[v] = Ri[v];
                }
            }
        };

        // ---- optional gate mask: bit j%32 of word j/32, one word per thread (behind the look-back, whose polls
        //      would queue behind these stores; ahead of the output stores, which may stay in flight)
        if (a.mask && lv % 32 < NSTEP && t0 + lv % 32 < a.L) {
            const int W = (a.J + 31) >> 5, wd = T.lb * MW + lv / 32;
            if (MW == 1 || wd < W) a.mask[((size_t)b * a.L + t0 + lv % 32) * W + wd] = mword;
        }

        // ---- checkpoints for the backward pass: the state before every CKPT_T-th token.  The one at
        //      the start of my segment goes out here, the others from inside the replay.
        float *ckp = a.ckpt ? a.ckpt + (((size_t)b * a.nTc + t0 / CKPT_T) * 2) * a.J + (active ? j0 : 0) : nullptr;
        const uint32_t ck_step = (uint32_t)a.J * 2u * 4u;       // bytes from one checkpoint of a lane to the next
        if (ckp && active && t0 < a.L) {
            Vec<V>::st(ckp, Sr);
            Vec<V>::st(ckp + a.J, Si);
        }

        // ---- replay from the true state, clamp, store.  Addresses are a wave-uniform base plus a
        //      32-bit offset; a tile that lies wholly inside the tensor stores without per-row checks.
        {
            constexpr uint32_t ES = BF ? 2u : 4u;          // bytes per output element
            const size_t obase = ((size_t)b * a.osb + (size_t)(tt * TILE_T) * a.ost + (size_t)T.lb * JB) * ES;
            float *zre = reinterpret_cast<float *>(reinterpret_cast<char *>(a.z_re) + obase);
            float *zim = reinterpret_cast<float *>(reinterpret_cast<char *>(a.z_im) + obase);
            const uint32_t ost32 = (uint32_t)a.ost;
            uint32_t off = ((uint32_t)(seg * NSTEP) * ost32 + (uint32_t)(lv * V)) * ES;   // bytes
            const bool full = (tt + 1) * TILE_T <= a.L && (T.lb + 1) * JB <= a.J;
            const bool plain = full && !(a.state_out && tt == a.nT - 1);   // no per-row checks at all
            // HC: whether my lane is the first or the last of its head
            const int hk = HC && !WIDE ? j0 % a.F : 0;
            const bool h_first = hk == 0, h_last = hk == a.F - 1;
            // WIDE: a lane beside a boundary between waves has one neighbour in another wave
            const int blk = WIDE ? lv / 64 : 0;
            const bool e_lo = WIDE && lane == 0 && blk > 0, e_hi = WIDE && lane == 63 && blk + 1 < WPS;
            const int bnd = e_lo ? blk - 1 : (e_hi ? blk : 0);
            // bf16 rows of 64 and more lanes are whole 128-byte lines, where strides and bases say so: st_row16 streams them then
            const bool lines = BF && ((ost32 * 2 | (uint32_t)a.osb * 2 | (uint32_t)reinterpret_cast<uintptr_t>(a.z_re) |
                                       (uint32_t)reinterpret_cast<uintptr_t>(a.z_im)) & 127) == 0;
            auto replay = [&](auto plain_c, auto whole_c, auto ck_c, auto lines_c) {
                constexpr bool PLAIN = decltype(plain_c)::value;
                constexpr bool LINES = decltype(lines_c)::value;
                constexpr bool CK = decltype(ck_c)::value;       // checkpoints wanted (uniform over the launch)
                constexpr bool WHOLE = decltype(whole_c)::value; // a wave's 64 lanes are one head, or a part of one
                if constexpr (HC) {
                    // The harmonic convolution, four tokens at a time: the recurrence of the four, then all
                    // their lane exchanges, then outputs.  No branch in here, so the steps stay one block of code.
                    constexpr int CH = 4;
                    static_assert(NSTEP % CH == 0, "whole chunks");
                    auto states = [&](int c0, float (&z_r)[CH], float (&z_i)[CH]) {
#pragma unroll
                        for (int k = 0; k < CH; ++k) {
                            const int i = c0 + k;
                            float nr, ni;
                            if (RET) {
                                const float rr = __builtin_fmaf(lr[0], Sr[0], -li[0] * Si[0]);
                                const float ri = __builtin_fmaf(li[0], Sr[0], lr[0] * Si[0]);
                                nr = __builtin_fmaf(gm[i][0], rr, pr[i][0]);
                                ni = __builtin_fmaf(gm[i][0], ri, pi[i][0]);
                            } else {
                                nr = __builtin_fmaf(lr[0], Sr[0], __builtin_fmaf(-li[0], Si[0], pr[i][0]));
                                ni = __builtin_fmaf(li[0], Sr[0], __builtin_fmaf(lr[0], Si[0], pi[i][0]));
                            }
                            Sr[0] = nr;
                            Si[0] = ni;
                            next_run(i);
                            if (CK && (i + 1) % CKPT_T == 0 && i + 1 < NSTEP && (PLAIN || (active && t0 + i + 1 < a.L))) {
                                float *cq = reinterpret_cast<float *>(reinterpret_cast<char *>(ckp) + (uint32_t)((i + 1) / CKPT_T) * ck_step);
                                cq[0] = Sr[0];       // (checkpoints are read back by the backward of the same step: cached stores)
                                cq[a.J] = Si[0];
                            }
                            z_r[k] = clampf(nr, a.out_clamp);
                            z_i[k] = clampf(ni, a.out_clamp);
                            if (!PLAIN && t0 + i == a.L - 1 && a.state_out && active) {
                                a.state_out[((size_t)b * 2 + 0) * a.J + j0] = nr;
                                a.state_out[((size_t)b * 2 + 1) * a.J + j0] = ni;
                            }
                        }
                    };
                    if constexpr (WIDE) {
#pragma unroll
                        for (int c0 = 0; c0 < NSTEP; c0 += CH) {
                            float z_r[CH], z_i[CH];
                            states(c0, z_r, z_i);
#pragma unroll
                            for (int k = 0; k < CH; ++k) {
                                pr[c0 + k][0] = z_r[k];
                                pi[c0 + k][0] = z_i[k];
                            }
                        }
                        if (e_lo || e_hi) {
                            const int side = e_hi ? 0 : 1;
#pragma unroll
                            for (int i = 0; i < NSTEP; ++i) {
                                sEdge[0][bnd][side][seg * NSTEP + i] = pr[i][0];
                                sEdge[1][bnd][side][seg * NSTEP + i] = pi[i][0];
                            }
                        }
                        lds_barrier_raw();     // (the next tile's rows may be on their way)
                    }
#pragma unroll
                    for (int c0 = 0; c0 < NSTEP; c0 += CH) {
                        float z_r[CH], z_i[CH], c_r[CH], c_i[CH];
                        if constexpr (WIDE) {
#pragma unroll
                            for (int k = 0; k < CH; ++k) {
                                z_r[k] = pr[c0 + k][0];
                                z_i[k] = pi[c0 + k][0];
                            }
                        } else {
                            states(c0, z_r, z_i);
                        }
                        if constexpr (WHOLE) {      // the shift itself brings the zeros beyond the wave's ends
#pragma unroll
                            for (int k = 0; k < CH; ++k) {
                                c_r[k] = __builtin_fmaf(hw[0][1], z_r[k], hb[0]);
                                c_i[k] = __builtin_fmaf(hw[1][1], z_i[k], hb[1]);
                            }
#pragma unroll
                            for (int k = 0; k < CH; k += 2)
                                fma_neighbours(c_r[k], c_i[k], c_r[k + 1], c_i[k + 1], z_r[k], z_i[k], z_r[k + 1], z_i[k + 1], hw);
                            if (WIDE && (e_lo || e_hi)) {
                                const int side = e_hi ? 1 : 0;
                                const float w_r = e_hi ? hw[0][2] : hw[0][0], w_i = e_hi ? hw[1][2] : hw[1][0];
#pragma unroll
                                for (int k = 0; k < CH; ++k) {
                                    c_r[k] = __builtin_fmaf(w_r, sEdge[0][bnd][side][WIDE ? seg * NSTEP + c0 + k : 0], c_r[k]);
                                    c_i[k] = __builtin_fmaf(w_i, sEdge[1][bnd][side][WIDE ? seg * NSTEP + c0 + k : 0], c_i[k]);
                                }
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < CH; ++k) {
                                // (the shifts are statements of their own: every lane executes them)
                                const float lzr = wave_shift_up0(z_r[k]), lzi = wave_shift_up0(z_i[k]);
                                const float rzr = wave_shift_down0(z_r[k]), rzi = wave_shift_down0(z_i[k]);
                                const float l_r = h_first ? 0.f : lzr, l_i = h_first ? 0.f : lzi;
                                const float r_r = h_last ? 0.f : rzr, r_i = h_last ? 0.f : rzi;
                                c_r[k] = __builtin_fmaf(hw[0][2], r_r, __builtin_fmaf(hw[0][1], z_r[k], __builtin_fmaf(hw[0][0], l_r, hb[0])));
                                c_i[k] = __builtin_fmaf(hw[1][2], r_i, __builtin_fmaf(hw[1][1], z_i[k], __builtin_fmaf(hw[1][0], l_i, hb[1])));
                            }
                        }
#pragma unroll
                        for (int k = 0; k < CH; ++k) {
                            if (PLAIN || (active && t0 + c0 + k < a.L)) {
                                char *pr_ = reinterpret_cast<char *>(zre) + off, *pi_ = reinterpret_cast<char *>(zim) + off;
                                if constexpr (BF) {
                                    st_row16<LINES>(pr_, to_bf16(c_r[k]));
                                    st_row16<LINES>(pi_, to_bf16(c_i[k]));
                                } else {
                                    st_stream(reinterpret_cast<float *>(pr_), c_r[k]);
                                    st_stream(reinterpret_cast<float *>(pi_), c_i[k]);
                                }
                            }
                            off += ost32 * ES;
                        }
                    }
                } else {
#pragma unroll
                for (int i = 0; i < NSTEP; ++i) {
                    const int t = t0 + i;
                    float zr[V], zi[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        float nr, ni;
                        if (RET) {
                            const float rr = __builtin_fmaf(lr[v], Sr[v], -li[v] * Si[v]);
                            const float ri = __builtin_fmaf(li[v], Sr[v], lr[v] * Si[v]);
                            nr = __builtin_fmaf(gm[i][v], rr, pr[i][v]);
                            ni = __builtin_fmaf(gm[i][v], ri, pi[i][v]);
                        } else {
                            nr = __builtin_fmaf(lr[v], Sr[v], __builtin_fmaf(-li[v], Si[v], pr[i][v]));
                            ni = __builtin_fmaf(li[v], Sr[v], __builtin_fmaf(lr[v], Si[v], pi[i][v]));
                        }
                        Sr[v] = nr;
                        Si[v] = ni;
                        zr[v] = clampf(nr, a.out_clamp);
                        zi[v] = clampf(ni, a.out_clamp);
                    }
                    if (!PLAIN && t == a.L - 1 && a.state_out && active) {
                        Vec<V>::st(a.state_out + ((size_t)b * 2 + 0) * a.J + j0, Sr);
                        Vec<V>::st(a.state_out + ((size_t)b * 2 + 1) * a.J + j0, Si);
                    }
                    next_run(i);
                    if (CK && (i + 1) % CKPT_T == 0 && i + 1 < NSTEP && (PLAIN || (active && t + 1 < a.L))) {
                        float *cq = reinterpret_cast<float *>(reinterpret_cast<char *>(ckp) + (uint32_t)((i + 1) / CKPT_T) * ck_step);
                        Vec<V>::st(cq, Sr);       // the state before token t + 1
                        Vec<V>::st(cq + a.J, Si);
                    }
                    if (PLAIN || (active && t < a.L)) {
                        if constexpr (BF) {
                            st_row16<LINES>(reinterpret_cast<char *>(zre) + off, to_bf16(zr[0]));
                            st_row16<LINES>(reinterpret_cast<char *>(zim) + off, to_bf16(zi[0]));
                        } else {
                            static_assert(V == 1, "streamed output stores: one lane per thread");
                            st_stream(reinterpret_cast<float *>(reinterpret_cast<char *>(zre) + off), zr[0]);
                            st_stream(reinterpret_cast<float *>(reinterpret_cast<char *>(zim) + off), zi[0]);
                        }
                    }
                    off += ost32 * ES;
                }
                }
            };
            // What is still in flight ahead of this tile's output stores must be complete now: the next
            // tile's staged rows (needed after the next barrier).  The output stores themselves (the
            // 2 * NSTEP youngest operations when no row needed a check) are left in flight.
            using T_ = std::true_type;
            using F_ = std::false_type;
            auto replay_ck = [&](auto plain_c, auto whole_c) {
                auto replay_to = [&](auto lines_c) {
                    if (ckp) replay(plain_c, whole_c, T_{}, lines_c);
                    else replay(plain_c, whole_c, F_{}, lines_c);
                };
                if constexpr (BF && JB >= 64 && decltype(plain_c)::value && (!HC || decltype(whole_c)::value)) {
                    if (lines) replay_to(T_{});
                    else replay_to(F_{});
                } else {
                    replay_to(F_{});
                }
            };
            auto replay_hc = [&](auto plain_c) {
                if constexpr (WIDE) replay_ck(plain_c, T_{});
                else if (HC && a.F == JB) replay_ck(plain_c, T_{});
                else replay_ck(plain_c, F_{});
            };
            if (plain) {
                replay_hc(T_{});
                wait_vm<(2 * NSTEP < 63 ? 2 * NSTEP : 63)>();
            } else {
                replay_hc(F_{});
                wait_vm<0>();
            }
        }
        CAWN_STAMP(8);

        // ---- conv history for the next call: last HALO pre-conv rows (written by the last tile,
        //      after its carry arrived, i.e. after the first tile has consumed state_in: safe in place)
        if (HALO > 0 && a.state_out && tt == a.nT - 1 && is_tail_seg && active) {
            float *tail_out = a.state_out + (size_t)a.B * 2 * a.J;
            for (int r = 0; r < HALO; ++r) {
                const int t = a.L - HALO + r;
                float vm[V], va[V];
#pragma unroll
                for (int v = 0; v < V; ++v) vm[v] = va[v] = 0.f;
                if (t >= 0) {
                    const size_t off = (size_t)b * a.isb + (size_t)t * a.ist + j0;
                    if constexpr (BF) {
                        vm[0] = from_bf16(reinterpret_cast<const uint16_t *>(a.mag)[off]);
                        va[0] = from_bf16(reinterpret_cast<const uint16_t *>(a.ang)[off]);
                    } else {
                        Vec<V>::ld(vm, a.mag + off);
                        Vec<V>::ld(va, a.ang + off);
                    }
                } else if (tail_in) {
                    const size_t off = ((size_t)(b * HALO + (t + HALO)) * 2) * a.J + j0;
                    Vec<V>::ld(vm, tail_in + off);
                    Vec<V>::ld(va, tail_in + off + a.J);
                }
                const size_t o = ((size_t)(b * HALO + r) * 2) * a.J + j0;
                Vec<V>::st(tail_out + o, vm);
                Vec<V>::st(tail_out + o + a.J, va);
            }
        }

        if (SINGLE) break;
        // (the next tile's logits have landed: waited for above)
        if (FACTORS && wave == 0 && next_ticket < qtiles) valve_factors<TILE_T>(&sV[0], a.valve_thr, a.gpb, lane);
        ticket = next_ticket;
        T = Tn;
    }

#undef a
#undef ARGS_AGAIN
    // ---- the workgroup that leaves last resets the tickets and advances the epoch for the next call.
    //      Workgroups are counted, not tiles: every one of the grid has then drawn its last ticket.
    if (COUNT_EARLY && counts_early(a.tq, epoch)) return;      // (counted in its last tile)
    if (tid == 0)
        sLast = leave_last(a.hdr, a.tq, blockIdx.x, gridDim.x, leave_ask(a.hdr, a.tq, blockIdx.x, gridDim.x)) ? 1u : 0u;
    __syncthreads();
    if (sLast) finish_call(a.hdr, a.clear_from, epoch, tid, blockDim.x, [](const uint32_t *) { return false; });
}

// Compute units of the device, and workgroups of a kernel that fit on it (asked once per kernel); 0: the runtime would not say
static inline long long fwd_cus()
{
    static std::atomic<long long> known{0};
    if (known.load(std::memory_order_relaxed) == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        known.store(prop.multiProcessorCount, std::memory_order_relaxed);
    }
    return known.load(std::memory_order_relaxed);
}
template <class G, int KC, bool VALVE, bool RET, bool BF, bool HC, bool MANY>
static long long fwd_resident()
{
    static std::atomic<long long> known{0};
    if (known.load(std::memory_order_relaxed) == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fwd_kernel<G, KC, VALVE, RET, BF, HC, MANY>, G::NT, 0) != hipSuccess)
            return 0;
        known.store((long long)(n > 0 ? n : 1) * fwd_cus(), std::memory_order_relaxed);
    }
    return known.load(std::memory_order_relaxed);
}

template <class G, int KC, bool VALVE, bool RET, bool BF, bool HC, bool MANY>
static hipError_t launch_fwd_chain(const FwdArgs &a, uint32_t units, long long wgs, hipStream_t s)
{
    FwdArgs b = a;
    b.tq = make_queues(units, (uint32_t)a.nT, wgs);
    if (G::SHORT) b.tq.group = 64;      // (one group: no prefixes)
    hipLaunchKernelGGL((fwd_kernel<G, KC, VALVE, RET, BF, HC, MANY>), dim3((unsigned)wgs), dim3(G::NT), 0, s, b);
    return hipGetLastError();
}

// Two kernels of long tiles.  ONE: a workgroup for every tile, rows straight into registers, the carry by groups of tiles.
// MANY: as many workgroups as fit on the chip, each with the next tile's rows on their way to LDS while it works on one; on
// 32-lane rows a prefix per tile (see make_queues).  (Both schemes in one kernel: the first kind 1 - 2.5 % slower, B16 L1000 J768
// 53.9 us against 52.4, the second 4 %.)
// A call may have more tiles than fit as workgroups of ONE at a time: the others start as these end, and still draw in
// the chains' order.  They start with nothing on its way, and where there are many of them MANY is ahead.
// Time ONE / time MANY, conv 3 if not said, 3100 calls (chains in brackets; with fewer than four counters for the first draws of ONE where the
// chains are no multiple of four, which cost it up to a seventh where there are few more tiles than fit at a time -- with eight for any
// number of chains 595 such calls, 513 - 620 and 770 - 1020 tiles, are 0.85 - 1.03 of what MANY took):
//   32 lanes, constant retention (768 fit at a time): 770 - 1020 tiles 0.55 - 0.97 (1 - 66); 1150 tiles 0.90 (22 - 128), 1400 tiles 0.96 - 1.01,
//     1536 and more 1.02 - 1.25
//   32 lanes, retentions: 560 - 1020 tiles 0.79 - 0.95 (even), 0.94 - 1.00 (odd); 1150 tiles 0.92, 1400 tiles 0.96; 1536 1.04 with the valve
//   64 lanes, no retentions: bf16 800 - 1750 tiles 0.68 - 0.97, 2000 0.87 - 1.01, 3000 0.92 - 1.18, with the valve at 1280 0.90, at 1500 0.89 -
//     1.03; harmonic convolution 560 - 2300 tiles 0.77 - 1.00, 3000 0.86 - 1.04, 4500 0.83 - 1.14
//   64 lanes, retentions: 800 - 2300 tiles 0.80 - 1.01, 3000 0.84 - 1.03, 4500 0.84 - 1.13; with the valve, since adjacent chains share an XCD,
//     conv 3 (8 - 128 chains): harmonic convolution bf16 2300 tiles 0.88 - 0.91, 3072 0.93, 4096 0.85 - 0.96, 4608 1.00, fp32 2300 0.95 - 0.97,
//     3072 0.98, 4096 0.90 - 1.01, 6144 1.03; bf16 alone, conv 4, 2300 0.91 - 0.92, 3072 0.94, 4096 0.93 - 0.98, 6144 1.01; 43 drawn calls of
//     conv 1 - 4 with 2060 - 3072 (4096) tiles 0.81 - 1.01, mean 0.95; bf16 alone with conv 1 and many chains 1.06
//   64 lanes, no conv (less arithmetic to hide the loads of MANY behind), more than 32 chains: at 1300 / 1400 - 1600 / 1700 - 1800 tiles, mean,
//     bf16 with retentions 0.98 / 1.06 / 1.02, fp32 harmonic convolution 1.00 / 1.03 / 1.06, in bf16 0.92 / 1.01 / 1.05, with retentions 0.96 / 1.00 /
//     1.05; the other kinds 0.80 - 1.12, mean 0.98 (0.97 with conv 1), with retentions at 2020 tiles 1.02: B4 L3741 J1088 fp32 with retentions and the
//     harmonic convolution 67 us MANY, 72 - 75 ONE.  Up to 32 chains 0.81 - 1.07, mean 0.95.  Up to conv 2 768 of ONE fit behind the harmonic
//     convolution without retentions, and 800 - 1010 tiles are 1.00 - 1.10 (15, 49)
// bf16 without retentions needs fewer registers in MANY, of which 768 workgroups fit, than in ONE, of which 512 do: in
// between every workgroup of MANY has one tile and ONE takes a second round, B1 L8192 J768 (768) 28.8 / 31.1.
// Heads of 128 and 256 harmonics behind the harmonic convolution (rows of their own width, 64 tokens a tile): a workgroup of
// 128-lane rows is half a compute unit, and of 256-lane rows, which need twice the waves, a whole one, which has nothing else to do while
// its rows are on their way.  Time ONE / time MANY, conv 3, the means of four kinds in fp32 and bf16:
//   128 lanes: up to 2500 tiles 0.86 - 0.97 (2496 tiles of 24 chains 1.05 and 1.02), 2900 - 6000 tiles 0.86 - 0.90 (6 chains), 0.92 -
//     1.00 (16), 1.02 - 1.15 (64; bf16 with retentions 0.97 - 1.00)
//   256 lanes: up to 256 tiles 0.93 - 0.98, beyond 1.01 - 1.23 (where a few tiles more than 256 take a second round most)
// MANY stages 16 bytes a load only: rows that start elsewhere go to ONE.  (Blocks of 64 lanes of such a head one after the other in one
// workgroup, which handed the outermost lanes on in LDS, as it was: a call's blocks of one head in series, and where the
// workgroup was one of few all of its tiles too: B1 L6532 H1 F256 bf16 with retentions 2104 us, now 28; B8 L465 H16 F256 84, now 66;
// B2 L16025 H6 F128 122, now 119.)
template <class G, int KC, bool VALVE, bool RET, bool BF, bool HC>
static hipError_t launch_fwd_tile(const FwdArgs &a, hipStream_t s)
{
    // (the host divided the call by the tile it chose: the same one, or nothing is launched)
    if (a.nLB != (a.J + G::JB - 1) / G::JB || a.nT != (a.L + G::TILE_T - 1) / G::TILE_T) return hipErrorInvalidValue;
    const uint32_t units = (uint32_t)a.nLB * a.B;
    const long long jobs = (long long)units * a.nT;
    if constexpr (!G::SHORT) {
        constexpr bool W64 = G::JB == 64, W128 = G::JB > 64;
        const long long one = fwd_resident<G, KC, VALVE, RET, BF, HC, false>(), many = fwd_resident<G, KC, VALVE, RET, BF, HC, true>(), cus = fwd_cus();
        if (one <= 0 || many <= 0) return hipErrorUnknown;
        const bool light = KC == 0 && !VALVE && (RET ? BF : HC) && units > 32;
        const int per_cu = !W64 || (BF && VALVE && !RET && !HC) ? 4 : light ? 5 : RET && KC > 0 ? (VALVE && (HC || KC > 1) ? (BF ? 16 : 12) : 8) : 7;      // (tiles a compute unit)
        const bool wide_many = a.stage16 && (G::JB == 256 ? jobs > one : units > 32 && jobs > 9 * cus && !(RET && BF));
        if (W128) return wide_many ? launch_fwd_chain<G, KC, VALVE, RET, BF, HC, true>(a, units, jobs < many ? jobs : many, s)
                                   : launch_fwd_chain<G, KC, VALVE, RET, BF, HC, false>(a, units, jobs, s);
        if (jobs > per_cu * cus || (jobs > one && jobs <= many))
            return launch_fwd_chain<G, KC, VALVE, RET, BF, HC, true>(a, units, jobs < many ? jobs : many, s);   // persistent: what fits on the chip
        return launch_fwd_chain<G, KC, VALVE, RET, BF, HC, false>(a, units, jobs, s);
    } else {
        return launch_fwd_chain<G, KC, VALVE, RET, BF, HC, false>(a, units, jobs, s);
    }
}

// The tile shape of a call (the host computed nT and nLB from the same rule): 64-lane rows with the harmonic
// convolution, 128 or 256 for heads of that width, 32-lane rows without.
template <bool SHORT, int KC, bool VALVE, bool RET, bool BF, bool HC>
static hipError_t launch_fwd_k(const FwdArgs &a, hipStream_t s)
{
    using std::conditional_t;
    if constexpr (HC) {
        if constexpr (!SHORT) {
            if (a.F == FwdWide128::JB) return launch_fwd_tile<FwdWide128, KC, VALVE, RET, BF, true>(a, s);
            if (a.F == FwdWide256::JB) return launch_fwd_tile<FwdWide256, KC, VALVE, RET, BF, true>(a, s);
        }
        return launch_fwd_tile<conditional_t<SHORT, FwdShortHead, FwdHead>, KC, VALVE, RET, BF, true>(a, s);
    } else {
        return launch_fwd_tile<conditional_t<SHORT, FwdShort, conditional_t<BF, FwdHead, FwdGeom>>, KC, VALVE, RET, BF, false>(a, s);
    }
}

// Tuning aid: -DCAWN_DEV_KC=<k> compiles only the conv_k = k kernels and -DCAWN_DEV_PLAIN only the
// threshold-mode fp32 ones without the harmonic convolution (a build for timing one variant in
// seconds; every other variant then fails to launch with hipErrorInvalidValue).  The library is
// always built without them.
template <bool SHORT, bool VALVE, bool RET, bool HC, bool BF>
static hipError_t launch_fwd_act(const FwdArgs &a, int conv_k, hipStream_t s)
{
#ifdef CAWN_DEV_PLAIN
    if constexpr (VALVE || RET || BF || HC) return hipErrorInvalidValue; else
#endif
    switch (conv_k) {
#ifdef CAWN_DEV_KC
    case CAWN_DEV_KC: return launch_fwd_k<SHORT, CAWN_DEV_KC, VALVE, RET, BF, HC>(a, s);
#else
    case 0: return launch_fwd_k<SHORT, 0, VALVE, RET, BF, HC>(a, s);
    case 1: return launch_fwd_k<SHORT, 1, VALVE, RET, BF, HC>(a, s);
    case 2: return launch_fwd_k<SHORT, 2, VALVE, RET, BF, HC>(a, s);
    case 3: return launch_fwd_k<SHORT, 3, VALVE, RET, BF, HC>(a, s);
    case 4: return launch_fwd_k<SHORT, 4, VALVE, RET, BF, HC>(a, s);
#endif
    default: return hipErrorInvalidValue;
    }
}

// One translation unit per family of forward kernels (tile length x gate mode x retention mode, long tiles x harmonic
// convolution): they compile side by side.
template <bool SHORT, bool VALVE, bool RET, bool HC>
static hipError_t launch_fwd_family(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return a.bf16 ? launch_fwd_act<SHORT, VALVE, RET, HC, true>(a, conv_k, s) : launch_fwd_act<SHORT, VALVE, RET, HC, false>(a, conv_k, s);
}
hipError_t launch_fwd_plain(const FwdArgs &a, int conv_k, hipStream_t s);        // threshold gate, constant retention
hipError_t launch_fwd_valve(const FwdArgs &a, int conv_k, hipStream_t s);        // per-head valve, constant retention
hipError_t launch_fwd_ret(const FwdArgs &a, int conv_k, hipStream_t s);          // threshold gate, data-dependent retention
hipError_t launch_fwd_valve_ret(const FwdArgs &a, int conv_k, hipStream_t s);    // valve and data-dependent retention
hipError_t launch_fwd_hconv_plain(const FwdArgs &a, int conv_k, hipStream_t s);  // the same four with the harmonic convolution
hipError_t launch_fwd_hconv_valve(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_fwd_hconv_ret(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_fwd_hconv_valve_ret(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_fwd_short_plain(const FwdArgs &a, int conv_k, hipStream_t s);  // and on short tiles, with and without it
hipError_t launch_fwd_short_valve(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_fwd_short_ret(const FwdArgs &a, int conv_k, hipStream_t s);
hipError_t launch_fwd_short_valve_ret(const FwdArgs &a, int conv_k, hipStream_t s);

}  // namespace cawn
