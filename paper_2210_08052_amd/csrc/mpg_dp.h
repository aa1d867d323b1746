// Device helpers and the templated DP kernel, shared by the per-K
// translation units (mpg_dp_k1/k2/k4.hip) and the other kernels.
#pragma once

#include <climits>

#include "mpg_internal.h"
#include "mpg_walk.h"

// Occupancy targets of the DP kernels (waves per SIMD; 1 = no cap).  An fp32
// subtraction issues beside another wavefront's max, so more wavefronts pair
// more of them (cycles per instruction of an even mix: 3.0 at three waves per
// SIMD, 2.5 at four, 2.35 at eight).  Score-only kernels of width <= 2 and
// width 1 with traceback run four (128 VGPRs, 10,240 B of LDS each); width 2
// with traceback three, which its LDS caps; width 4 keeps the registers it
// needs.
#ifndef MPG_SCORE_WAVES
#define MPG_SCORE_WAVES 4
#endif
#ifndef MPG_TB_WAVES
#define MPG_TB_WAVES 3
#endif
#ifndef MPG_TB1_WAVES
#define MPG_TB1_WAVES 4
#endif
#ifndef MPG_K4_WAVES
#define MPG_K4_WAVES 1
#endif
template <int K, bool TB>
struct WavesPerEu {
    static constexpr int value =
        K > 2 ? MPG_K4_WAVES : (TB ? (K == 2 ? MPG_TB_WAVES : MPG_TB1_WAVES) : MPG_SCORE_WAVES);
};

namespace mpg {
namespace dev {


constexpr int kShr1 = 0x138;  // DPP wave_shr:1

static __constant__ uint8_t kAaOfLetter[26] = {0,  20, 4,  3,  6,  13, 7,  8,  9,  22, 11, 10, 12,
                                        2,  22, 14, 5,  1,  15, 16, 22, 19, 17, 22, 18, 21};

__device__ __forceinline__ int dna_code(uint32_t ch) {
    switch (ch | 0x20u) {
        case 'a': return 0;
        case 'c': return 1;
        case 'g': return 2;
        case 't': return 3;
        default: return 4;
    }
}

__device__ __forceinline__ int aa_code(uint32_t ch) {
    if (ch == '*') return 23;
    uint32_t u = (ch | 0x20u) - 'a';
    return u < 26u ? kAaOfLetter[u] : 22;
}

__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int imax3(int a, int b, int c) { return imax(imax(a, b), c); }

__device__ __forceinline__ int shr1(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, kShr1, 0xF, 0xF, false);
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
        uint32_t olo = __shfl_xor((int)lo, o, 64), ohi = __shfl_xor((int)hi, o, 64);
        uint64_t w = ((uint64_t)ohi << 32) | olo;
        v = w > v ? w : v;
    }
    return v;
}

// End-cell key: larger is better; score desc, then row asc, then column asc.
__device__ __forceinline__ uint64_t end_key(int score, int row, int col) {
    return ((uint64_t)(uint32_t)(score + (1 << 27)) << 36) |
           ((uint64_t)(uint32_t)((1 << 21) - 1 - row) << 15) | (uint64_t)((1 << 15) - 1 - col);
}

// Modes whose H floors at 0 in every cell (a path may start anywhere), and
// modes read at the single end cell (n, m).
__host__ __device__ constexpr bool floor_mode(int mode) {
    return mode == MPG_LOCAL || mode == MPG_EXTEND_LEFT;
}
__host__ __device__ constexpr bool fixed_end_mode(int mode) {
    return mode == MPG_GLOBAL || mode == MPG_EXTEND_LEFT;
}

__device__ __forceinline__ int neg_for(int mode, bool tb) {
    return floor_mode(mode) ? (tb ? -(1 << 29) : -(1 << 25)) : -(1 << 30);
}

// ------------------------------------------------------------ prepasses
// Rows per thread: a block covers 256 * kPrepassRows consecutive rows, so its
// owner search and table staging are shared by that many rows, and a thread
// reads one window of bases for its consecutive rows.
constexpr int kPrepassRows = 4;
static_assert(64 % kPrepassRows == 0 && kDescLo % kPrepassRows == 0 &&
                  kDescHi % kPrepassRows == 0,
              "a thread's rows must lie in one pair");

// The last index p in [0, n) with start[p] <= g (start ascending, start[0] <=
// g), found by wave 0 of the block 64 probes at a time: each round reads 64
// positions spread over the remaining range at once and keeps the part between
// the last probe at or below g and the next one, so 10^5 entries take 3 rounds
// of dependent loads instead of 17.  Must be called by all 64 lanes of a wave.
__device__ __forceinline__ int wave_find_owner(const int64_t* __restrict__ start, int n, int64_t g) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = n - 1;  // start[lo] <= g; the answer is in [lo, hi]
    while (hi > lo) {
        const int64_t span = hi - lo;
        // probe l: lo + ceil(span * (l + 1) / 64), ascending in l, probe 63 = hi
        const int pl = lo + (int)((span * (lane + 1) + 63) / 64);
        const unsigned long long ok = __ballot(start[pl] <= g);
        const int nk = __popcll(ok);  // ok holds for probes 0 .. nk-1
        const int nlo = nk ? lo + (int)((span * nk + 63) / 64) : lo;
        const int nhi = nk < 64 ? lo + (int)((span * (nk + 1) + 63) / 64) - 1 : hi;
        lo = nlo;
        hi = nhi;
    }
    return lo;
}

// ---------------------------------------------------------------------- DP
//
// Score-only layout (TB = false): plain values, descriptor {tr, z, r+d(i+1),
// a(i)}; r+d(i), r+d(i-1), a(i-1), a(i-2) are carried in registers.
// Traceback layout (TB = true): H is 16*H; I, D, A, B, C are 16*v + their
// fixed nibble (13, 12, 7, 6, 5); descriptor {tr, z+15, 5-16(r+d(i+1)),
// 16a(i)}, the same rows carried: C opens at H - 16(r+d(i+1)) + 5, B at
// H - 16(r+d(i)) + 6 (the previous row's field plus one), A at
// H - 16(r+d(i-1)) + 7 (the field of two rows up plus two), one three-input
// add each.
// H winner codes: 0 start, 1 M, 2 I, 3 D, 4 F1, 5 F2, 6 G1, 7 G2, 8 A, 9 B,
// 10 C; nibble = 15 - code.

// SEG: the kernel also runs two pairs' last strips on lane segments of one
// wavefront; the second pair's descriptor ring follows the other areas, and
// its incoming boundary takes the outgoing boundary's area (a last strip
// publishes no boundary).
template <int K, bool TB, bool SEG = false>
struct LdsLayout {
    static constexpr int DS = 16;              // descriptor bytes per row
    static constexpr int PS = TB ? 2 : 1;      // profile score bytes
    static constexpr int PE = K * PS;          // a lane's scores for one amino acid
    static constexpr int PB = PE < 4 ? 4 : PE; // a lane's block of a profile row
    static constexpr int PN = PB / PE;         // amino acids of one row
    static constexpr int SW = 64 * K;          // strip width
    static constexpr int RING = 128 * DS;      // two chunks of descriptors
    static constexpr int PROF = (25 + PN - 1) / PN * 64 * PB;  // 24 aa + poison row
    static constexpr int IN = 64 * 8;          // incoming boundary of the chunk
    // outgoing boundary (64 rows), then the slots through which each lane
    // hands its last column to the lane on its right (one per lane and step)
    static constexpr int OUT = 192 * 8;
    static constexpr int MAT = 640;            // substitution matrix, then the letter codes
    static constexpr int RING2 = RING + PROF + IN + OUT + MAT;  // SEG: second ring
    static constexpr int WAVE = RING2 + (SEG ? RING : 0);
};

// The profile in LDS: a lane's scores of one amino acid for its K columns lie
// together, in a block of at least 4 bytes of its own, so that the 64 lanes,
// each with the amino acid of its own row, read 64 different banks.  (Rows of
// 64 one-byte scores put four lanes on a bank and several amino acids on the
// same one.)  The row descriptors hold the byte offset of their amino acid
// within lane 0's block, for the pair's own width and kind.  Each column is
// one read and one add: both columns in one read need sub-dword operands
// (SDWA), whose instructions, like DPP, issue beside no other wavefront's
// (10k batch 11.5 -> 13.3 ms).
__host__ __device__ __forceinline__ int prof_offset(int K, bool tb, int tr) {
    const int pe = K * (tb ? 2 : 1);
    if (pe >= 4) return tr * 64 * pe;
    return pe == 2 ? (tr >> 1) * 256 + (tr & 1) * 2 : (tr >> 2) * 256 + (tr & 3);
}

// How a value v (in score-only units, or the 16x units of the traceback
// layout) is held in a 32-bit register.
//
// F32 = false: the integer v itself.
//
// F32 = true: the bits of the fp32 number BIAS + v, an exact integer in
// [2^23, 2^24), where neighbouring integers are neighbouring bit patterns: a
// 32-bit integer add to the bits (the substitution score) is the same sum,
// the low bits are the integer's own (the winner nibble), and integer max and
// compare of the bits order the numbers.  Penalties are subtracted with
// v_sub_f32, exactly.  The point: on gfx950 an fp32 add or subtract issues
// beside another wavefront's v_max / v_max3 / v_alignbit, an integer add or
// subtract does not.  Measured per SIMD at four wavefronts, alternating the
// two kinds: 2.5 cycles per instruction with v_sub_f32 and v_max3_i32, 4.5
// with v_sub_u32; about half of a cell's instructions are subtractions.
// The planner (f32_ok) proves that every reachable value fits; other pairs
// run the integer form.  Values below BIAS in LOCAL mode (never on a path)
// and the sentinel (2^22, or 2^21 without a floor) lie below 2^23 and stay
// positive numbers, so the order of the bits still holds.
//
// The floor modes keep -infinity small enough that a shifted end-tracking key
// of any sentinel-derived value stays below every reachable cell's.
template <int MODE, bool TB, bool F32 = false>
struct Sentinel {
    static constexpr bool LOC = MODE == MPG_LOCAL;
    static constexpr int NEG = F32 ? (LOC ? kF32NegLocal : kF32Neg)
                                   : (floor_mode(MODE) ? (TB ? -(1 << 29) : -(1 << 25)) : -(1 << 30));
    static constexpr int UNREACH = F32 ? kF32Unreach : (floor_mode(MODE) ? NEG / 2 : -(1 << 29));
    static constexpr int ZERO = F32 ? (LOC ? kF32ZeroLocal : kF32Zero) : 0;  // the value 0
    // the score of a reachable H
    static __device__ __forceinline__ int score(int h) { return (h - ZERO) >> (TB ? 4 : 0); }
};

template <bool F32>
__device__ __forceinline__ int vsub(int a, int b) {
    return F32 ? __float_as_int(__int_as_float(a) - __int_as_float(b)) : a - b;
}
template <bool F32>
__device__ __forceinline__ int vadd(int a, int b) {
    return F32 ? __float_as_int(__int_as_float(a) + __int_as_float(b)) : a + b;
}
// A per-lane penalty in the register form (the uniform ones come in DevParams).
template <bool F32>
__device__ __forceinline__ int vnum(int v) {
    return F32 ? __float_as_int((float)v) : v;
}
// End-tracking keys of a chunk: the cell's H above, 63 - step in the low 6
// bits, so that one max keeps the first best cell.  F32: compared unsigned;
// the bits of H shifted out at the top are the same for every value an H can
// take (exponents of 2^21 to 2^24).
// The keys of two consecutive steps enter one three-input max: an even step
// leaves its key in kp, the odd one takes both (64 steps: none is left over).
// Each is kept in its step: left free, the compiler takes the maxima of a
// chunk's 64 keys at its end and spills every step's H until then (widths 1
// and 2 hold 128 or 168 VGPRs; integer form at width 2, 10,000 pairs: 19.8 ms
// with 127 spilled, 15.2 so).  The integer form of width 4 runs one wavefront
// per SIMD with registers to spare, where free maxima cover latency (3,000
// pairs 5.9 ms, kept 7.9).
template <int K, bool F32>
struct PinKeys {
    static constexpr bool value = F32 || K <= 2;
};
template <int K, bool TB, bool F32>
__device__ __forceinline__ void key_push(int& bk, int& kp, int h, int t) {
    const int k = (int)(((uint32_t)h << (TB ? 2 : 6)) | (uint32_t)(63 - t));
    if (!PinKeys<K, F32>::value) {
        bk = imax(k, bk);
        return;
    }
    if (t & 1) {
        if (F32) {
            const uint32_t q = (uint32_t)kp > (uint32_t)k ? (uint32_t)kp : (uint32_t)k;
            bk = (int)(q > (uint32_t)bk ? q : (uint32_t)bk);
        } else {
            bk = imax3(kp, k, bk);
        }
        asm volatile("" : "+v"(bk));
    } else {
        kp = k;
        asm volatile("" : "+v"(kp));
    }
}
template <bool TB, bool F32>
__device__ __forceinline__ int key_value(int bk) {
    if (F32)
        return TB ? (int)((((uint32_t)bk >> 6) << 4) | 0x40000000u)
                  : (int)(((uint32_t)bk >> 6) | 0x48000000u);
    return TB ? (bk >> 6) << 4 : bk >> 6;
}
template <bool F32>
__host__ __device__ constexpr int key_none() {
    return F32 ? 0 : INT_MIN;
}

// a + b + k in one instruction (left to itself, the compiler shares b + k
// between a lane's columns and spends two)
template <int k>
__device__ __forceinline__ int add3k(int a, int b) {
    int r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "i"(k));
    return r;
}

// acc = 2*acc + (diff < 0) in every lane, one funnel shift: the choice of a
// gap or intron state, one bit per step, most recent step in bit 0.  diff =
// extension - opening, so the bit is 1 where the state opened (opening
// strictly better: extension wins ties).  All values lie within 2^31 of each
// other (planner's score bound), so the difference never overflows.
__device__ __forceinline__ uint32_t push_open(uint32_t acc, int diff) {
    return __builtin_amdgcn_alignbit(acc, (uint32_t)diff, 31);
}

// Issue priority of a wavefront whose strip runs `nchunks` chunks, on the scale
// `most`: 3 from half of it on, 0 below an eighth.  In a batch `most` is that of
// the launch's pair with most work: its longest chains go first.  Serving gives
// 0 to its short lanes (every strip 3) and more than any strip has to its long
// ones (every strip 0): a short job does not wait behind the long strips on its
// SIMD (24,000 jobs/s: short jobs p99 2.8 ms, at one priority 5.8; long jobs
// p50 35 ms, 32).
__device__ __forceinline__ void strip_priority(int nchunks, int most) {
    if (2 * nchunks >= most) __builtin_amdgcn_s_setprio(3);
    else if (4 * nchunks >= most) __builtin_amdgcn_s_setprio(2);
    else if (8 * nchunks >= most) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// Per-pair state shared by the waves that work on the pair's strips.
struct PairState {
    unsigned long long key;  // best end-cell key over the finished strips
    int done;                // strips finished
    int gsc;                 // GLOBAL: H(n, m)
    int bad;                 // a bounded wait gave up
    int pad;
};

// Device-scope relaxed atomics: coherent across every CU and XCD without
// cache-wide fences (loads and stores carry the device-scope cache bits).
__device__ __forceinline__ int ld_dev(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int2 ld_dev2(const int2* p) {
    const unsigned long long v = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return make_int2((int)(uint32_t)v, (int)(uint32_t)(v >> 32));
}
__device__ __forceinline__ void st_dev2(int2* p, int2 v) {
    const unsigned long long u = (unsigned long long)(uint32_t)v.x |
                                 ((unsigned long long)(uint32_t)v.y << 32);
    __hip_atomic_store((unsigned long long*)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// s_waitcnt encoding (gfx9 family): vmcnt in bits 3:0 and 15:14, expcnt in
// 6:4, lgkmcnt in 11:8.  vmcnt(1) with the other counters left free: every
// vector memory operation but the most recent one has completed (they retire
// in issue order).
constexpr int kWaitVm1 = 0x0F71;

// Write a result record, its status last (after a system-scope fence when the
// record lives in host memory that the host polls).
__device__ __forceinline__ void publish(mpg_dev_result* rec, const mpg_dev_result& R, int system) {
    rec->score = R.score;
    rec->g_beg = R.g_beg;
    rec->g_end = R.g_end;
    rec->p_beg = R.p_beg;
    rec->p_end = R.p_end;
    rec->ops_off = R.ops_off;
    rec->ops_len = R.ops_len;
    rec->_pad = 0;
    if (system) {
        __threadfence_system();
        __hip_atomic_store(&rec->status, R.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        // read only after the kernel has ended (by later kernels or the
        // host): no fence
        rec->status = R.status;
    }
}

// Bounded wait until the left strip has published `target` chunks.  Gives up
// after `limit` polls (kMaxPolls: well under a second) so no wave can spin
// forever; the pair then reports MPG_E_DEVICE.  A limit of 0 gives up at
// once (the host sets it to exercise that path).
// The polled value goes through readfirstlane: the loop exit is then uniform
// for the compiler too, so the wave never runs it in divergent form.
__device__ __forceinline__ bool wait_prog(const int* flag, int target, int limit) {
    for (int it = 0; it < limit; ++it) {
        if (__builtin_amdgcn_readfirstlane(ld_dev(flag)) >= target) return true;
        __builtin_amdgcn_s_sleep(2);
    }
    return false;
}

// Result record of a LOCAL score-only pair from its end key (score, -i, -j).
__device__ __forceinline__ void local_record(mpg_dev_result& R, const PairJob& J,
                                             unsigned long long ku, bool bad) {
    R.g_beg = -1;
    R.p_beg = -1;
    R.ops_off = J.ops_off;
    R.ops_len = 0;
    R._pad = 0;
    if (bad) {
        R.status = MPG_E_DEVICE;
        R.score = 0;
        R.g_end = -1;
        R.p_end = -1;
    } else {
        R.status = MPG_OK;
        R.score = (int)(ku >> 36) - (1 << 27);
        R.g_end = (1 << 21) - 1 - (int)((ku >> 15) & ((1u << 21) - 1));
        R.p_end = (1 << 15) - 1 - (int)(ku & ((1u << 15) - 1));
    }
}

// Two LOCAL pairs' last strips on lane segments of one wavefront (a strip
// that fills only part of its lanes leaves the rest idle for all its steps).
// item = (pair A, -1 - (pair B << 6 | split)): pair A's last strip in lanes
// [0, split), pair B's in [split, 64); both strips run the same number of
// chunks.  Each lane works on its own pair's rows (the segment's lane k at
// step s on row s - k), reads its pair's descriptors from that pair's LDS
// ring and takes its left neighbour's H and I through the same LDS slots as a
// whole-wave strip; the first lane of each segment reads its pair's incoming
// boundary instead, by its own address.  A pair of one
// strip starts from the -infinity column; otherwise its previous strip
// streams the boundary through HBM as for any strip.  With traceback (batch
// calls, walked afterwards by the walk kernel) each lane stores its direction
// bits into its own pair's block of the strip at its lane within the
// segment: the layout of a whole-wave strip.
template <int K, bool TB, bool NOI, bool NOF, bool F32>
__device__ __forceinline__ void seg_item(const int2 item, const PairJob* __restrict__ jobs,
                                         PairState* __restrict__ pst, int* __restrict__ prog_g,
                                         const uint8_t* __restrict__ prot,
                                         const uint8_t* __restrict__ desc, int2* __restrict__ bnd,
                                         uint8_t* __restrict__ tbbuf, const DpSink& sink,
                                         const DevParams& P, uint8_t* smem, const int8_t* smat,
                                         const uint8_t* saa) {
    using LY = LdsLayout<K, TB, true>;
    using SV = Sentinel<MPG_LOCAL, TB, F32>;
    constexpr int NEG = SV::NEG;
    constexpr int UNREACH = SV::UNREACH;
    // F32 traceback: the carried donor fields include the nibble difference of
    // the state that reads them (one add per row; the integer form adds it in
    // the three-input add that opens the state)
    constexpr bool DDN = F32 && TB;
    constexpr int kOne = F32 ? 0x3F800000 : 1, kTwo = F32 ? 0x40000000 : 2;
    constexpr int kNone = key_none<F32>();
    const int lane = threadIdx.x & 63;
    const int code = -1 - item.y;
    const int ja = item.x, jb = code >> 6, split = code & 63;
    const PairJob JA = jobs[ja], JB = jobs[jb];
    const bool sg = lane >= split;            // lane of pair B
    const bool first = lane == 0 || lane == split;
    const int kk = sg ? lane - split : lane;  // lane within its segment
    const int nA = JA.n, nB = JB.n;
    const int n_l = sg ? nB : nA, m_l = sg ? JB.m : JA.m;
    const int nchunks = JA.nchunks;
    const int stripA = JA.nstrips - 1, stripB = JB.nstrips - 1;
    const int col0 = (sg ? stripB : stripA) * LY::SW + kk * K;
    const uint8_t* dscA = desc + JA.desc_off;
    const uint8_t* dscB = desc + JB.desc_off;
    const uint8_t* dsc_l = sg ? dscB : dscA;
    const uint8_t* Pa = prot + (sg ? JB.prot_off : JA.prot_off);
    const int2* bndA = bnd + JA.bnd_off;
    const int2* bndB = bnd + JB.bnd_off;
    const int* progA = prog_g + JA.prog_off;
    const int* progB = prog_g + JB.prog_off;
    const bool leftA = stripA > 0, leftB = stripB > 0;
    // traceback: this lane's direction-bit blocks (its pair's last strip)
    uint8_t* tb_l = TB ? tbbuf + (sg ? JB.tb_off : JA.tb_off) +
                             (int64_t)(sg ? stripB : stripA) * nchunks * (kTbBlockBytes * K)
                       : nullptr;
    uint8_t* ringA = smem;
    uint8_t* ringB = smem + LY::RING2;
    uint8_t* prof = smem + LY::RING;
    const uint8_t* const prof_l = prof + lane * LY::PB;
    int2* inbA = (int2*)(smem + LY::RING + LY::PROF);
    int2* inbB = (int2*)(smem + LY::RING + LY::PROF + LY::IN);
    // penalties in the layout of the variant (as in the whole-wave strips)
    const int cq = P.pen[F32][TB][kPenI];
    const int cqD = P.pen[F32][TB][kPenD];
    const int ce = P.pen[F32][TB][kPenExt];
    const int cf = P.pen[F32][TB][kPenFs];
    int cf11 = P.pen[F32][TB][kPenF1];
    int cf9 = P.pen[F32][TB][kPenG1];
    asm volatile("" : "+s"(cf11), "+s"(cf9));
    const int2 neg2 = make_int2(NEG, NEG);

    // profile of this lane's columns (its own pair's residues)
#pragma unroll
    for (int c = 0; c < K; ++c) {
        const int j = col0 + c;
        int pc = -1;
        if (j >= 1 && j <= m_l) {
            const uint32_t ch = Pa[j - 1];
            const uint32_t u = (ch | 0x20u) - 'a';
            pc = ch == '*' ? 23 : (u < 26u ? saa[u] : 22);
        }
        int sv[24];
#pragma unroll
        for (int tr = 0; tr < 24; ++tr) sv[tr] = pc < 0 ? 0 : (int)smat[tr * 24 + pc];
#pragma unroll
        for (int tr = 0; tr < 25; ++tr) {
            const bool poison = pc < 0 || tr == 24;
            const int v = tr < 24 ? sv[tr < 24 ? tr : 0] : 0;
            uint8_t* at = prof + prof_offset(K, TB, tr) + lane * LY::PB + c * LY::PS;
            if (TB) *(int16_t*)at = (int16_t)(poison ? -32768 : 16 * v + 14);
            else *(int8_t*)at = (int8_t)(poison ? -128 : v);
        }
    }
    int h1[K], h2[K], h3[K], d1[K], d2[K], d3[K], a1[K], b1[K], c1[K];
    int best[K], bstep[K], bk[K], kp[K], fp[K];
    uint32_t nacc[K], xacc[5][K];
#pragma unroll
    for (int c = 0; c < K; ++c) {
        h1[c] = h2[c] = h3[c] = NEG;
        d1[c] = d2[c] = d3[c] = NEG;
        a1[c] = b1[c] = c1[c] = NEG;
        best[c] = NEG;
        bstep[c] = 0;
        bk[c] = kp[c] = kNone;
        fp[c] = TB ? vsub<F32>(NEG, cf11) : vsub<F32>(NEG, cf);
        nacc[c] = 0;
#pragma unroll
        for (int x = 0; x < 5; ++x) xacc[x][c] = 0;
    }
    int hl1 = NEG, hl2 = NEG, hl3 = NEG;
    int Hout = NEG, Iout = NEG;
    int dd0, ddm1, aam1, aam2;
    {
        const int4 u = *(const int4*)(dsc_l + (int64_t)(-kk - 1 + kDescLo) * LY::DS);
        const int4 v = *(const int4*)(dsc_l + (int64_t)(-kk - 2 + kDescLo) * LY::DS);
        aam1 = u.w; aam2 = v.w;
        dd0 = DDN ? vadd<F32>(u.z, kOne) : u.z;
        ddm1 = DDN ? vadd<F32>(v.z, kTwo) : v.z;
    }
    // both rings: rows -64..-1 then 0..63 of each pair
    {
        const int4 a0 = *(const int4*)(dscA + (int64_t)(lane - 64 + kDescLo) * LY::DS);
        const int4 a1v = *(const int4*)(dscA + (int64_t)(lane + kDescLo) * LY::DS);
        const int4 b0 = *(const int4*)(dscB + (int64_t)(lane - 64 + kDescLo) * LY::DS);
        const int4 b1v = *(const int4*)(dscB + (int64_t)(lane + kDescLo) * LY::DS);
        *(int4*)(ringA + lane * LY::DS) = a0;
        *(int4*)(ringA + (64 + lane) * LY::DS) = a1v;
        *(int4*)(ringB + lane * LY::DS) = b0;
        *(int4*)(ringB + (64 + lane) * LY::DS) = b1v;
    }
    inbA[lane] = neg2;
    inbB[lane] = neg2;
    bool failed = false;
    int2 nbA = neg2, nbB = neg2;
    int seenA = 0, seenB = 0;
    if (leftA) {
        if (!wait_prog(&progA[stripA - 1], nchunks < 2 ? nchunks : 2, P.max_polls)) failed = true;
        nbA = ld_dev2(&bndA[kBndLo + lane]);
        seenA = ld_dev(&progA[stripA - 1]);
    }
    if (leftB) {
        if (!wait_prog(&progB[stripB - 1], nchunks < 2 ? nchunks : 2, P.max_polls)) failed = true;
        nbB = ld_dev2(&bndB[kBndLo + lane]);
        seenB = ld_dev(&progB[stripB - 1]);
    }
    int4 pfA = make_int4(0, 0, 0, 0), pfB = make_int4(0, 0, 0, 0);
    // this lane's ring, the slot it hands its last column through, and where
    // it finds its left neighbour's (step t: row t of its pair's incoming
    // boundary, or the slot that lane wrote one step before), as LDS offsets
    // opaque to the compiler: it would distribute the selects over the steps'
    // addresses, which are invariant across chunks, and hoist all of them
    // into registers
    int ring_off = sg ? LY::RING2 : 0;
    int out_off = LY::RING + LY::PROF + LY::IN + (64 + lane) * 8;
    int in_off = first ? (sg ? LY::RING + LY::PROF + LY::IN : LY::RING + LY::PROF)
                       : LY::RING + LY::PROF + LY::IN + (62 + lane) * 8;
    asm volatile("" : "+v"(ring_off), "+v"(in_off), "+v"(out_off));
    const uint8_t* ring_l = smem + ring_off;
    const int2* in_l = (const int2*)(smem + in_off);
    int2* out_l = (int2*)(smem + out_off);

    for (int ch = 0; ch < nchunks && !failed; ++ch) {
        // incoming boundary rows ch*64 .. ch*64+63 of each pair with a left strip
        if (leftA) {
            inbA[lane] = ch * 64 + lane > nA ? neg2 : nbA;
            if (ch + 1 < nchunks) {
                const int need = ch + 3 < nchunks ? ch + 3 : nchunks;
                if (__builtin_amdgcn_readfirstlane(seenA) < need &&
                    !wait_prog(&progA[stripA - 1], need, P.max_polls)) {
                    failed = true;
                    break;
                }
                nbA = ld_dev2(&bndA[kBndLo + (ch + 1) * 64 + lane]);
                seenA = ld_dev(&progA[stripA - 1]);
            }
        }
        if (leftB) {
            inbB[lane] = ch * 64 + lane > nB ? neg2 : nbB;
            if (ch + 1 < nchunks) {
                const int need = ch + 3 < nchunks ? ch + 3 : nchunks;
                if (__builtin_amdgcn_readfirstlane(seenB) < need &&
                    !wait_prog(&progB[stripB - 1], need, P.max_polls)) {
                    failed = true;
                    break;
                }
                nbB = ld_dev2(&bndB[kBndLo + (ch + 1) * 64 + lane]);
                seenB = ld_dev(&progB[stripB - 1]);
            }
        }
        if (ch > 0) {
            const int4 oA = *(const int4*)(ringA + (64 + lane) * LY::DS);
            const int4 oB = *(const int4*)(ringB + (64 + lane) * LY::DS);
            *(int4*)(ringA + lane * LY::DS) = oA;
            *(int4*)(ringA + (64 + lane) * LY::DS) = pfA;
            *(int4*)(ringB + lane * LY::DS) = oB;
            *(int4*)(ringB + (64 + lane) * LY::DS) = pfB;
        }
        pfA = *(const int4*)(dscA + (int64_t)((ch + 1) * 64 + lane + kDescLo) * LY::DS);
        pfB = *(const int4*)(dscB + (int64_t)((ch + 1) * 64 + lane + kDescLo) * LY::DS);
        const uint8_t* rb = ring_l + (64 - kk) * LY::DS;
        auto ld_prof = [&](const int4& x0, int* scv) {
            const uint8_t* pr = prof_l + x0.x;
#pragma unroll
            for (int c = 0; c < K; ++c)
                scv[c] = TB ? (int)*(const int16_t*)(pr + c * LY::PS)
                            : (int)*(const int8_t*)(pr + c * LY::PS);
        };
        uint8_t* tbblk = TB ? tb_l + (int64_t)ch * (kTbBlockBytes * K) : nullptr;
        int4 cd0 = *(const int4*)(rb), nd0 = *(const int4*)(rb + LY::DS);
        int csc[K];
        ld_prof(cd0, csc);
        // step 0: the neighbour's last step of the chunk before
        // (shifted in every lane, then selected: a shift reads nothing from a
        // lane that a branch has masked off)
        const int hs = shr1(NEG, Hout), is = shr1(NEG, Iout);
        const int2 in0 = in_l[0];
        int2 cin = make_int2(first ? in0.x : hs, first ? in0.y : is);
#pragma unroll
        for (int t = 0; t < 64; ++t) {
            int4 fd0 = make_int4(0, 0, 0, 0);
            if (t + 2 < 64) fd0 = *(const int4*)(rb + (t + 2) * LY::DS);
            int nsc[K];
            if (t + 1 < 64) ld_prof(nd0, nsc);
            const int4 ds0 = cd0;
            int hl0 = cin.x, il0 = cin.y;
            const int z = ds0.y;
            int Hn[K], In[K], Dn[K], An[K], Bn[K], Cn[K];
            // First every term that does not need the left lane's values of this row,
            // for all columns, then I and H: the hand-off's latency lies under the first
            // part (left to itself the compiler waits for it after a few
            // instructions).
            int xw[K], xy[K];  // maxima of H's candidates but I
#pragma unroll
            for (int c = 0; c < K; ++c) {
                const int L1 = c ? h1[c - 1] : hl1;
                const int L3 = c ? h3[c - 1] : hl3;
                const int zc = z;
                if (!TB) {
                    const int D = vsub<F32>(imax(vsub<F32>(h3[c], cq), d3[c]), ce);
                    const int M = L3 + csc[c];
                    // frameshifts: F1 and G1 of this row cost f each, and F2, G2 are the
                    // previous row's F1, G1 (H two rows up is the history one row up), so
                    // one max per cell covers all four
                    int pf = 0;
                    if (!NOF) {
                        pf = vsub<F32>(imax(L1, h1[c]), cf);
                        // opaque to the next row: the compiler would otherwise expand
                        // fp - ... back into four candidates there
                        asm("" : "+v"(pf));
                    }
                    if (!NOI) {
                        const int A = imax(vsub<F32>(h1[c], ddm1), a1[c]);
                        const int B = imax(vsub<F32>(L1, dd0), b1[c]);
                        const int C = imax(vsub<F32>(L1, ds0.z), c1[c]);
                        An[c] = A; Bn[c] = B; Cn[c] = C;
                        const int x = imax3(D, vsub<F32>(A, ds0.w), vsub<F32>(B, aam2));
                        xw[c] = imax3(M, zc, x);
                        const int y = vsub<F32>(C, aam1);
                        xy[c] = NOF ? y : imax3(y, pf, fp[c]);
                    } else {
                        xw[c] = NOF ? D : imax3(D, pf, fp[c]);
                        xy[c] = imax(M, zc);
                    }
                    if (!NOF) fp[c] = pf;
                    Dn[c] = D;
                } else {
                    const int oD = vsub<F32>(h3[c], cqD), xD = vsub<F32>(d3[c], ce);
                    xacc[1][c] = push_open(xacc[1][c], vsub<F32>(xD, oD));
                    int D = imax(oD, xD);
                    const int M = L3 + csc[c];
                    // F1 (nibble 11) and G1 (9) of this row; F2 (10) and G2 (8) are the
                    // previous row's F1 and G1 less one, so their maximum is the previous
                    // row's maximum less one
                    int p1 = 0, p2 = 0;
                    if (!NOF) {
                        p1 = imax(vsub<F32>(L1, cf11), vsub<F32>(h1[c], cf9));
                        // opaque to the next row: the compiler would otherwise expand
                        // fp - 1 back into four candidates there
                        asm("" : "+v"(p1));
                        p2 = vsub<F32>(fp[c], kOne);
                        fp[c] = p1;
                    }
                    // the states enter H's maximum as they are: left visible, the
                    // compiler may also build H from their two halves in a second tree
                    // (seen at one column per lane)
                    asm("" : "+v"(D));
                    if (!NOI) {
                        const int oA = DDN ? vadd<F32>(h1[c], ddm1) : add3k<2>(h1[c], ddm1);
                        xacc[2][c] = push_open(xacc[2][c], vsub<F32>(a1[c], oA));
                        int A = imax(oA, a1[c]);
                        const int oB = DDN ? vadd<F32>(L1, dd0) : add3k<1>(L1, dd0);
                        xacc[3][c] = push_open(xacc[3][c], vsub<F32>(b1[c], oB));
                        int B = imax(oB, b1[c]);
                        const int oC = vadd<F32>(L1, ds0.z);
                        xacc[4][c] = push_open(xacc[4][c], vsub<F32>(c1[c], oC));
                        int C = imax(oC, c1[c]);
                        asm("" : "+v"(A), "+v"(B), "+v"(C));
                        An[c] = A; Bn[c] = B; Cn[c] = C;
                        const int x = imax3(D, vsub<F32>(A, ds0.w), vsub<F32>(B, aam2));
                        xw[c] = imax3(M, zc, x);
                        const int y = vsub<F32>(C, aam1);
                        xy[c] = NOF ? y : imax3(y, p1, p2);
                    } else {
                        xw[c] = NOF ? D : imax3(D, p1, p2);
                        xy[c] = imax(M, zc);
                    }
                    Dn[c] = D;
                }
            }
#pragma unroll
            for (int c = 0; c < K; ++c) asm("" : "+v"(hl0), "+v"(il0) : "v"(xw[c]), "v"(xy[c]));
#pragma unroll
            for (int c = 0; c < K; ++c) {
                const int L0 = c ? Hn[c - 1] : hl0;
                const int IL = c ? In[c - 1] : il0;
                const int oI = vsub<F32>(L0, cq);
                if (!TB) {
                    const int I = vsub<F32>(imax(oI, IL), ce);
                    Hn[c] = imax3(xw[c], xy[c], I);
                    In[c] = I;
                } else {
                    const int xI = vsub<F32>(IL, ce);
                    xacc[0][c] = push_open(xacc[0][c], vsub<F32>(xI, oI));
                    int I = imax(oI, xI);
                    asm("" : "+v"(I));
                    const int Hk = imax3(xw[c], xy[c], I);
                    nacc[c] = __builtin_amdgcn_alignbit(Hk, nacc[c], 4);
                    Hn[c] = Hk & ~15;
                    In[c] = I;
                }
            }
            Hout = Hn[K - 1];
            Iout = In[K - 1];
            // (the hand-off as in the whole-wave strips)
            __builtin_amdgcn_sched_barrier(0);
            out_l[t] = make_int2(Hout, Iout);
            if (t + 1 < 64) cin = in_l[t + 1];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < K; ++c)
                key_push<K, TB, F32>(bk[c], kp[c], Hn[c], t);
            if (TB && (t & 7) == 7) {
#pragma unroll
                for (int c = 0; c < K; ++c)
                    *(uint32_t*)(tbblk + (((t >> 3) * K + c) * 64 + kk) * 4) = nacc[c];
            }
            if (TB && (t & 31) == 31) {
#pragma unroll
                for (int x = 0; x < 5; ++x) {
                    if (NOI && x >= 2) continue;
#pragma unroll
                    for (int c = 0; c < K; ++c)
                        *(uint32_t*)(tbblk + 2048 * K +
                                     (((x * K + c) * 2 + (t >> 5)) * 64 + kk) * 4) = xacc[x][c];
                }
            }
            hl3 = hl2; hl2 = hl1; hl1 = hl0;
#pragma unroll
            for (int c = 0; c < K; ++c) {
                h3[c] = h2[c]; h2[c] = h1[c]; h1[c] = Hn[c];
                d3[c] = d2[c]; d2[c] = d1[c]; d1[c] = Dn[c];
                if (!NOI) { a1[c] = An[c]; b1[c] = Bn[c]; c1[c] = Cn[c]; }
            }
            ddm1 = DDN ? vadd<F32>(dd0, kOne) : dd0;
            dd0 = DDN ? vadd<F32>(ds0.z, kOne) : ds0.z;
            aam2 = aam1; aam1 = ds0.w;
            cd0 = nd0; nd0 = fd0;
#pragma unroll
            for (int c = 0; c < K; ++c) csc[c] = nsc[c];
        }
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const int v = key_value<TB, F32>(bk[c]);
            const int tt = 63 - (bk[c] & 63);
            if (v > best[c]) { best[c] = v; bstep[c] = ch * 64 + tt; }
            bk[c] = kNone;
        }
    }

    // each pair's best cell over its own lanes, folded into the pair
    uint64_t key = 0;
#pragma unroll
    for (int c = 0; c < K; ++c) {
        const int row = bstep[c] - kk, col = col0 + c;
        if (col <= m_l && row >= 0 && row <= n_l && best[c] > UNREACH) {
            const uint64_t k2 = end_key(SV::score(best[c]), row, col);
            key = k2 > key ? k2 : key;
        }
    }
    const uint64_t keyA = wave_max_u64(sg ? 0 : key), keyB = wave_max_u64(sg ? key : 0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const PairJob& J = q ? JB : JA;
        PairState* ps = pst + (q ? jb : ja);
        const unsigned long long k = q ? keyB : keyA;
        const bool solo = J.nstrips == 1;
        int done = 0;
        if (!solo) {
            if (lane == 0) {
                if (failed) atomicMax(&ps->bad, 1);
                else if (k) atomicMax(&ps->key, k);
            }
            __builtin_amdgcn_s_waitcnt(0);
            if (lane == 0)
                done = __hip_atomic_fetch_add(&ps->done, 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
            done = __builtin_amdgcn_readfirstlane(done);
        }
        if (done == J.nstrips - 1) {
            const unsigned long long kf =
                solo ? k : __hip_atomic_load(&ps->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool bad =
                solo ? failed : __builtin_amdgcn_readfirstlane(ld_dev(&ps->bad)) != 0;
            const uint32_t khi = __builtin_amdgcn_readfirstlane((uint32_t)(kf >> 32));
            const uint32_t klo = __builtin_amdgcn_readfirstlane((uint32_t)kf);
            mpg_dev_result R;
            local_record(R, J, ((unsigned long long)khi << 32) | klo, bad);
            if (lane == 0) publish(sink.out + J.res, R, sink.system);
        }
    }
}

// The DP kernel.  Persistent single-wavefront workgroups take (pair, strip)
// work items from one queue ordered longest pair first, strips in order.  A
// strip streams its left boundary (H and I of the previous strip's last
// column) from HBM as the previous strip publishes it chunk by chunk, so the
// strips of a long pair run as a pipeline spread over many CUs, and every
// wavefront slot stays busy until the queue is empty.  Dependencies only point
// to items taken earlier by running wavefronts, so the waits always end.
// PRO: the query is a position-specific profile block (prof_scores /
// prof_gaps) instead of protein letters and one matrix.
template <int K, int MODE, bool TB, bool NOI, bool NOF, bool PRO, bool F32>
__global__ void __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(WavesPerEu<K, TB>::value)))
dp_kernel(const PairJob* __restrict__ jobs, const int2* __restrict__ items, int nitems,
          int* __restrict__ qhead, PairState* __restrict__ pst, int* __restrict__ prog_g,
          const uint8_t* __restrict__ prot, const uint8_t* __restrict__ desc,
          int2* __restrict__ bnd, uint8_t* __restrict__ tbbuf, DpSink sink, DevParams P) {
    // LOCAL launches also run lane-segment items (two pairs' last strips in
    // one wavefront)
    constexpr bool SEGOK = MODE == MPG_LOCAL && !PRO;
    using LY = LdsLayout<K, TB, SEGOK>;
    // the mixed variant runs EXTEND and fixed-end pairs (per-pair modes)
    constexpr bool MIXED = MODE == kModeMixed;
    constexpr int SM = MIXED ? (int)MPG_GLOBAL : MODE;  // mode of the sentinels and the floor
    using SV = Sentinel<SM, TB, F32>;
    constexpr int NEG = SV::NEG;
    constexpr int UNREACH = SV::UNREACH;
    // F32 traceback: the carried donor fields include the nibble difference of
    // the state that reads them (one add per row; the integer form adds it in
    // the three-input add that opens the state)
    constexpr bool DDN = F32 && TB;
    constexpr int kOne = F32 ? 0x3F800000 : 1, kTwo = F32 ? 0x40000000 : 2;
    constexpr int kNone = key_none<F32>();
    constexpr int ZN = TB ? 15 : 0;  // nibble of the start candidate
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    uint8_t* ring = smem;
    uint8_t* prof = smem + LY::RING;
    const uint8_t* const prof_l = prof + lane * LY::PB;
    int2* inb = (int2*)(smem + LY::RING + LY::PROF);
    int2* outb = (int2*)(smem + LY::RING + LY::PROF + LY::IN);
    // A lane hands its last column's H and I to the lane on its right through
    // LDS: lane l < 63 writes slot 64 + l + t at step t, the next lane reads
    // that slot for step t + 1 (LDS operations of a wavefront run in order),
    // and lane 0 reads row t + 1 of the incoming boundary with the same
    // instruction.  Lane 63 writes the outgoing boundary, slot t.  A shift by
    // DPP takes two instructions that issue beside no other wavefront's, and
    // a select in packed strips; this read takes the place of the broadcast
    // read of the boundary row, and the step's other terms cover its latency.
    // One base per lane, the step in the immediate offset.  Without introns
    // or at one column without traceback there are too few other terms (25
    // instructions per step): a call that leaves the device idle waits for the
    // hand-off, so those kernels shift by DPP (rescoring 800 pairs 1.21 ->
    // 1.05 ms, 1,000 profiles 2.55 -> 2.41; one column with traceback gains 2%
    // alone and loses 7% on 1,500 pairs).
    constexpr bool XLDS = !NOI && (K > 1 || TB);
    // whether the hand-off is pinned to its place in the step (see below);
    // the mixed variant is 4% slower with it
    constexpr bool EARLY = XLDS && !MIXED;
    int out_off = LY::RING + LY::PROF + LY::IN + (lane == 63 ? 0 : 64 + lane) * 8;
    int in_off = lane ? LY::RING + LY::PROF + LY::IN + (62 + lane) * 8 : LY::RING + LY::PROF;
    asm volatile("" : "+v"(in_off), "+v"(out_off));
    const int2* const in_l = (const int2*)(smem + in_off);
    int2* const out_l = (int2*)(smem + out_off);
    int8_t* smat = (int8_t*)(smem + LY::RING + LY::PROF + LY::IN + LY::OUT);
    uint8_t* saa = (uint8_t*)(smat + 24 * 24);
    // the matrix and the letter codes, read with per-lane indices when a
    // strip's profile is built, are staged in LDS once per launch
    for (int k = lane; k < 24 * 24 / 4; k += 64)
        ((int*)smat)[k] = ((const int*)P.mat)[k];  // 4-byte aligned in both
    if (lane < 26) saa[lane] = kAaOfLetter[lane];
    __syncthreads();
    auto aa_lds = [&](uint32_t ch) -> int {
        if (ch == '*') return 23;
        const uint32_t u = (ch | 0x20u) - 'a';
        return u < 26u ? saa[u] : 22;
    };

    // penalties in the layout of this variant
    const int cq = P.pen[F32][TB][kPenI];   // I open  (TB: nibble 13)
    const int cqD = P.pen[F32][TB][kPenD];  // D open  (TB: nibble 12)
    const int ce = P.pen[F32][TB][kPenExt];
    const int cf = P.pen[F32][TB][kPenFs];
    // traceback: the F1 and G1 candidates' offsets (16f less their nibbles),
    // kept opaque so that the compiler does not share H - 16f between them
    // and add each nibble with a separate instruction
    int cf11 = P.pen[F32][TB][kPenF1];
    int cf9 = P.pen[F32][TB][kPenG1];
    asm volatile("" : "+s"(cf11), "+s"(cf9));

    // Items are taken when the previous one is done (claiming ahead would
    // hold a strip that the next strip of its pair then waits for).
    for (;;) {
        // take the next item without a divergent branch: lane 0 adds 1, the
        // other lanes add 0, so lane 0 always receives the old head; its value
        // through readfirstlane is wave-uniform, which keeps the loop exit
        // uniform, so no cross-lane operation below ever runs with part of
        // the wave masked off
        const int it = __builtin_amdgcn_readfirstlane(atomicAdd(qhead, lane == 0 ? 1 : 0));
        if (it >= nitems) break;
        const int2 item = items[it];
        strip_priority(jobs[item.x].nchunks, P.prio_chunks);
        if constexpr (SEGOK) {
            if (item.y < 0) {
                seg_item<K, TB, NOI, NOF, F32>(item, jobs, pst, prog_g, prot, desc, bnd, tbbuf, sink,
                                          P, smem, smat, saa);
                continue;
            }
        }
        const PairJob J = jobs[item.x];
        const int strip = item.y;
        const int n = J.n, m = J.m;
        const int nchunks = J.nchunks, nstrips = J.nstrips;
        const uint8_t* dsc_g = desc + J.desc_off;  // row r at (r + kDescLo) * DS
        int2* bnd_g = bnd + J.bnd_off;             // row r at r + kBndLo
        const uint8_t* Pa = prot + J.prot_off;
        uint8_t* tbp = tbbuf + J.tb_off;
        int* prog = prog_g + J.prog_off;           // chunks published, per strip
        PairState* ps = pst + item.x;
        const bool has_next = strip + 1 < nstrips;
        const int col0 = strip * LY::SW + lane * K;  // DP column of this lane's first column
        bool failed = false;
        uint64_t best_key = 0;

        // ---- strip set-up: profile, registers, first descriptors and boundary
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const int j = col0 + c;
            const int pc = (j >= 1 && j <= m) ? (PRO ? 0 : aa_lds(Pa[j - 1])) : -1;
            // all 24 entries are read before any is stored, so the reads
            // overlap
            int sv[24];
#pragma unroll
            for (int tr = 0; tr < 24; ++tr)
                sv[tr] = pc < 0 ? 0
                                : (PRO ? (int)prof_scores(Pa)[24 * (j - 1) + tr]
                                       : (int)smat[tr * 24 + pc]);
#pragma unroll
            for (int tr = 0; tr < 25; ++tr) {
                const bool poison = pc < 0 || tr == 24;
                const int v = tr < 24 ? sv[tr < 24 ? tr : 0] : 0;
                uint8_t* at = prof + prof_offset(K, TB, tr) + lane * LY::PB + c * LY::PS;
                if (TB) *(int16_t*)at = (int16_t)(poison ? -32768 : 16 * v + 14);
                else *(int8_t*)at = (int8_t)(poison ? -128 : v);
            }
        }

        // gap costs of this lane's columns in the layout of the variant (a
        // profile's own per column; columns beyond m take column m's)
        int cqv[K], cqDv[K], cev[K], ceDv[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
            if (PRO) {
                const int16_t* g = prof_gaps(Pa, m) + 4 * imin(col0 + c, m);
                const int oi = g[0], ei = g[1], od = g[2], ed = g[3];
                cqv[c] = vnum<F32>(TB ? 16 * (oi + ei) - 13 : oi);
                cev[c] = vnum<F32>(TB ? 16 * ei : ei);
                cqDv[c] = vnum<F32>(TB ? 16 * (od + ed) - 12 : od);
                ceDv[c] = vnum<F32>(TB ? 16 * ed : ed);
            } else {
                cqv[c] = cq;
                cev[c] = ce;
                cqDv[c] = cqD;
                ceDv[c] = ce;
            }
        }
        inb[lane] = make_int2(NEG, NEG);
        int h1[K], h2[K], h3[K], d1[K], d2[K], d3[K], a1[K], b1[K], c1[K];
        int zl[K], best[K], bstep[K], bk[K], bkt[K], hn[K], kp[K];
        int fp[K];  // previous row's frameshift term (F1/G1 maximum)
        uint32_t nacc[K];
        uint32_t xacc[5][K];  // extension decisions of the last steps, per lane
        // The fixed-end kernel also runs EXTEND_LEFT pairs: their start term
        // is the row's own (0 on every valid row), so the column term is
        // lifted out of the minimum.
        const bool floor0 = (MIXED || fixed_end_mode(MODE)) && J.mode == MPG_EXTEND_LEFT;
        // the pair ends at (n, m) (a compile-time constant but in the mixed variant)
        const bool fixed = MIXED ? J.mode != MPG_EXTEND : fixed_end_mode(MODE);
#pragma unroll
        for (int c = 0; c < K; ++c) {
            h1[c] = h2[c] = h3[c] = NEG;
            d1[c] = d2[c] = d3[c] = NEG;
            a1[c] = b1[c] = c1[c] = NEG;
            zl[c] = floor0 ? INT_MAX : ((col0 + c == 0) ? SV::ZERO + ZN : NEG + ZN);
            best[c] = NEG;
            bstep[c] = 0;
            bk[c] = kp[c] = kNone;
            bkt[c] = 0;
            hn[c] = NEG;
            // the frameshift term of the row above the strip's first (every
            // H there is -infinity)
            fp[c] = TB ? vsub<F32>(NEG, cf11) : vsub<F32>(NEG, cf);
            nacc[c] = 0;
#pragma unroll
            for (int x = 0; x < 5; ++x) xacc[x][c] = 0;
        }
        int hl1 = NEG, hl2 = NEG, hl3 = NEG;
        int Hout = NEG, Iout = NEG;
        // registers carrying the previous two rows' donor and acceptor fields
        // (score-only: r+d(i), r+d(i-1), a(i-1), a(i-2))
        int dd0 = 0, ddm1 = 0, aam1 = 0, aam2 = 0;
        {
            const int4 u = *(const int4*)(dsc_g + (int64_t)(-lane - 1 + kDescLo) * LY::DS);
            const int4 v = *(const int4*)(dsc_g + (int64_t)(-lane - 2 + kDescLo) * LY::DS);
            aam1 = u.w; aam2 = v.w;
            dd0 = DDN ? vadd<F32>(u.z, kOne) : u.z;
            ddm1 = DDN ? vadd<F32>(v.z, kTwo) : v.z;
        }
        // descriptor ring: rows -64..-1 then 0..63
        int4 pf0 = make_int4(0, 0, 0, 0);
        {
            // all loads first, then the stores
            const uint8_t* src = dsc_g + (int64_t)(lane - 64 + kDescLo) * LY::DS;
            const uint8_t* src2 = dsc_g + (int64_t)(lane + kDescLo) * LY::DS;
            const int4 r0 = *(const int4*)src, r2 = *(const int4*)src2;
            *(int4*)(ring + lane * LY::DS) = r0;
            *(int4*)(ring + (64 + lane) * LY::DS) = r2;
        }
        int2 nb = make_int2(NEG, NEG);
        // the left strip's last column arrives from HBM as that strip
        // publishes it; rows of chunk c need its chunks c and c+1.  Its
        // progress counter is read one chunk ahead, so the check at a chunk
        // start normally finds the value loaded long before and never waits.
        const bool from_left = strip > 0;
        int seen = 0;
        if (from_left) {
            if (!wait_prog(&prog[strip - 1], nchunks < 2 ? nchunks : 2, P.max_polls))
                failed = true;
            nb = ld_dev2(&bnd_g[kBndLo + lane]);
            seen = ld_dev(&prog[strip - 1]);
        }

        for (int ch = 0; ch < nchunks && !failed; ++ch) {
            {
                // incoming boundary rows ch*64 .. ch*64+63 (rows beyond n hold
                // garbage-row values or were never written: -infinity)
                const bool beyond = ch * 64 + lane > n;
                if (from_left) {
                    inb[lane] = beyond ? make_int2(NEG, NEG) : nb;
                    if (ch + 1 < nchunks) {
                        const int need = ch + 3 < nchunks ? ch + 3 : nchunks;
                        if (__builtin_amdgcn_readfirstlane(seen) < need &&
                            !wait_prog(&prog[strip - 1], need, P.max_polls)) {
                            failed = true;
                            break;
                        }
                        nb = ld_dev2(&bnd_g[kBndLo + (ch + 1) * 64 + lane]);
                        seen = ld_dev(&prog[strip - 1]);
                    }
                }
                if (ch > 0) {
                    // slide the descriptor ring: current chunk -> previous half
                    const int4 o0 = *(const int4*)(ring + (64 + lane) * LY::DS);
                    *(int4*)(ring + lane * LY::DS) = o0;
                    *(int4*)(ring + (64 + lane) * LY::DS) = pf0;
                }
                pf0 = *(const int4*)(dsc_g + (int64_t)((ch + 1) * 64 + lane + kDescLo) * LY::DS);
                const uint8_t* rb = ring + (64 - lane) * LY::DS;
                uint8_t* tbblk = tbp + ((int64_t)strip * nchunks + ch) * (kTbBlockBytes * K);
                const int srow_n = ch * 64 - n;  // GLOBAL: lane == t + srow_n  <=>  row == n

                // Software pipeline: descriptors are read two steps ahead, the
                // profile entries and the incoming boundary value one step ahead.
                auto ld_desc = [&](int tt, int4& x0) { x0 = *(const int4*)(rb + tt * LY::DS); };
                auto ld_prof = [&](const int4& x0, int* scv) {
                    const uint8_t* pr = prof_l + x0.x;
#pragma unroll
                    for (int c = 0; c < K; ++c)
                        scv[c] = TB ? (int)*(const int16_t*)(pr + c * LY::PS)
                                    : (int)*(const int8_t*)(pr + c * LY::PS);
                };
                int4 cd0, nd0;
                ld_desc(0, cd0);
                ld_desc(1, nd0);
                int csc[K];
                ld_prof(cd0, csc);
                // step 0: the neighbour's last step of the chunk before
                const int2 in0 = inb[0];
                int2 cin = XLDS ? make_int2(shr1(in0.x, Hout), shr1(in0.y, Iout)) : in0;

#pragma unroll
                for (int t = 0; t < 64; ++t) {
                    // ---- prefetch for steps t+1 and t+2
                    int4 fd0 = make_int4(0, 0, 0, 0);
                    if (t + 2 < 64) ld_desc(t + 2, fd0);
                    int nsc[K];
                    if (t + 1 < 64) ld_prof(nd0, nsc);
                    int2 nin = make_int2(0, 0);
                    if (!XLDS && t + 1 < 64) nin = inb[t + 1];
                    const int4 ds0 = cd0;
                    int hl0 = XLDS ? cin.x : shr1(cin.x, Hout);
                    int il0 = XLDS ? cin.y : shr1(cin.y, Iout);
                    const int zr = ds0.y;
                    int Hn[K], In[K], Dn[K], An[K], Bn[K], Cn[K];
                    // First every term that does not need the left lane's values of this row,
                    // for all columns, then I and H: the hand-off's latency lies under the first
                    // part (left to itself the compiler waits for it after a few instructions:
                    // 10k batch 10.2 -> 9.98 ms, one traced pair 0.376 -> 0.370).
                    // (Kernels that do not pin the hand-off do one column after the other.)
                    int xw[K], xy[K], xm[K];  // maxima of H's candidates but I; M
                    auto terms = [&](int c) {
                        const int L1 = c ? h1[c - 1] : hl1;
                        const int L3 = c ? h3[c - 1] : hl3;
                        const int zc = (floor_mode(SM) ? zr : imin(zr, zl[c]));
                        if (!TB) {
                            const int D = vsub<F32>(imax(vsub<F32>(h3[c], cqDv[c]), d3[c]), ceDv[c]);
                            const int M = L3 + csc[c];
                            xm[c] = M;
                            // frameshifts: F1 and G1 of this row cost f each, and F2, G2 are the
                            // previous row's F1, G1 (H two rows up is the history one row up), so
                            // one max per cell covers all four
                            int pf = 0;
                            if (!NOF) {
                                pf = vsub<F32>(imax(L1, h1[c]), cf);
                                // opaque to the next row: the compiler would otherwise expand
                                // fp - ... back into four candidates there
                                asm("" : "+v"(pf));
                            }
                            if (!NOI) {
                                const int A = imax(vsub<F32>(h1[c], ddm1), a1[c]);
                                const int B = imax(vsub<F32>(L1, dd0), b1[c]);
                                const int C = imax(vsub<F32>(L1, ds0.z), c1[c]);
                                An[c] = A; Bn[c] = B; Cn[c] = C;
                                const int x = imax3(D, vsub<F32>(A, ds0.w), vsub<F32>(B, aam2));
                                xw[c] = EARLY ? imax3(M, zc, x) : x;
                                const int y = vsub<F32>(C, aam1);
                                xy[c] = NOF ? y : imax3(y, pf, fp[c]);
                            } else {
                                xw[c] = NOF ? D : imax3(D, pf, fp[c]);
                                xy[c] = EARLY ? imax(M, zc) : xw[c];
                            }
                            if (!NOF) fp[c] = pf;
                            Dn[c] = D;
                        } else {
                            const int oD = vsub<F32>(h3[c], cqDv[c]), xD = vsub<F32>(d3[c], ceDv[c]);
                            xacc[1][c] = push_open(xacc[1][c], vsub<F32>(xD, oD));
                            int D = imax(oD, xD);
                            const int M = L3 + csc[c];
                            xm[c] = M;
                            // F1 (nibble 11) and G1 (9) of this row; F2 (10) and G2 (8) are the
                            // previous row's F1 and G1 less one, so their maximum is the previous
                            // row's maximum less one
                            int p1 = 0, p2 = 0;
                            if (!NOF) {
                                p1 = imax(vsub<F32>(L1, cf11), vsub<F32>(h1[c], cf9));
                                // opaque to the next row: the compiler would otherwise expand
                                // fp - 1 back into four candidates there
                                asm("" : "+v"(p1));
                                p2 = vsub<F32>(fp[c], kOne);
                                fp[c] = p1;
                            }
                            // the states enter H's maximum as they are: left visible, the
                            // compiler may also build H from their two halves in a second tree
                            // (seen at one column per lane)
                            asm("" : "+v"(D));
                            if (!NOI) {
                                const int oA = DDN ? vadd<F32>(h1[c], ddm1) : add3k<2>(h1[c], ddm1);
                                xacc[2][c] = push_open(xacc[2][c], vsub<F32>(a1[c], oA));
                                int A = imax(oA, a1[c]);
                                const int oB = DDN ? vadd<F32>(L1, dd0) : add3k<1>(L1, dd0);
                                xacc[3][c] = push_open(xacc[3][c], vsub<F32>(b1[c], oB));
                                int B = imax(oB, b1[c]);
                                const int oC = vadd<F32>(L1, ds0.z);
                                xacc[4][c] = push_open(xacc[4][c], vsub<F32>(c1[c], oC));
                                int C = imax(oC, c1[c]);
                                asm("" : "+v"(A), "+v"(B), "+v"(C));
                                An[c] = A; Bn[c] = B; Cn[c] = C;
                                const int x = imax3(D, vsub<F32>(A, ds0.w), vsub<F32>(B, aam2));
                                xw[c] = EARLY ? imax3(M, zc, x) : x;
                                const int y = vsub<F32>(C, aam1);
                                xy[c] = NOF ? y : imax3(y, p1, p2);
                            } else {
                                xw[c] = NOF ? D : imax3(D, p1, p2);
                                xy[c] = EARLY ? imax(M, zc) : xw[c];
                            }
                            Dn[c] = D;
                        }
                    };
                    auto best_of = [&](int c, int I) {
                        if (EARLY) return imax3(xw[c], xy[c], I);
                        const int z = floor_mode(SM) ? zr : imin(zr, zl[c]);
                        if (NOI) return imax(xw[c], imax3(xm[c], I, z));
                        return imax3(xw[c], xy[c], imax3(xm[c], I, z));
                    };
                    auto finish = [&](int c) {
                        const int L0 = c ? Hn[c - 1] : hl0;
                        const int IL = c ? In[c - 1] : il0;
                        const int oI = vsub<F32>(L0, cqv[c]);
                        if (!TB) {
                            const int I = vsub<F32>(imax(oI, IL), cev[c]);
                            Hn[c] = best_of(c, I);
                            In[c] = I;
                        } else {
                            const int xI = vsub<F32>(IL, cev[c]);
                            xacc[0][c] = push_open(xacc[0][c], vsub<F32>(xI, oI));
                            int I = imax(oI, xI);
                            asm("" : "+v"(I));
                            const int Hk = best_of(c, I);
                            nacc[c] = __builtin_amdgcn_alignbit(Hk, nacc[c], 4);
                            Hn[c] = Hk & ~15;
                            In[c] = I;
                        }
                    };
#pragma unroll
                    for (int c = 0; c < K; ++c) {
                        terms(c);
                        if (!EARLY) finish(c);
                    }
                    if (EARLY) {
#pragma unroll
                        for (int c = 0; c < K; ++c) asm("" : "+v"(hl0), "+v"(il0) : "v"(xw[c]), "v"(xy[c]));
#pragma unroll
                        for (int c = 0; c < K; ++c) finish(c);
                    }
                    Hout = Hn[K - 1];
                    Iout = In[K - 1];
                    if (EARLY) {
                        // the hand-off at once, and in this order: what follows
                        // it here and the next step's first part cover its latency
                        __builtin_amdgcn_sched_barrier(0);
                        out_l[t] = make_int2(Hout, Iout);
                        if (t + 1 < 64) cin = in_l[t + 1];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // end-cell tracking (chunk-local, merged after the chunk)
                    if constexpr (MIXED) {
                        // the best cell, over every cell (EXTEND) or the
                        // cells of row n (fixed end)
                        const bool take = !fixed || lane == t + srow_n;
#pragma unroll
                        for (int c = 0; c < K; ++c) {
                            const int v = take ? Hn[c] : NEG;
                            if (F32) {  // one key, as in LOCAL
                                key_push<K, TB, F32>(bk[c], kp[c], v, t);
                                continue;
                            }
                            const bool gt = v > bk[c];
                            bk[c] = gt ? v : bk[c];
                            bkt[c] = gt ? t : bkt[c];
                            if (PinKeys<K, F32>::value)
                                asm volatile("" : "+v"(bk[c]), "+v"(bkt[c]));
                        }
                    } else if (fixed_end_mode(MODE)) {
                        const bool at_n = (lane == t + srow_n);
#pragma unroll
                        for (int c = 0; c < K; ++c) {
                            hn[c] = at_n ? Hn[c] : hn[c];
                            // keep the select in this step: left free, the
                            // compiler defers all 64 of them to the chunk's
                            // end, holding every step's H and mask live
                            // (about 100 more VGPRs, one wave per SIMD)
                            asm volatile("" : "+v"(hn[c]));
                        }
                    } else if (MODE == MPG_LOCAL || F32) {
#pragma unroll
                        for (int c = 0; c < K; ++c)
                            key_push<K, TB, F32>(bk[c], kp[c], Hn[c], t);
                    } else {
#pragma unroll
                        for (int c = 0; c < K; ++c) {
                            const bool gt = Hn[c] > bk[c];
                            bk[c] = gt ? Hn[c] : bk[c];
                            bkt[c] = gt ? t : bkt[c];
                            if (PinKeys<K, F32>::value)
                                asm volatile("" : "+v"(bk[c]), "+v"(bkt[c]));
                        }
                    }
                    if (TB && (t & 7) == 7) {
#pragma unroll
                        for (int c = 0; c < K; ++c)
                            *(uint32_t*)(tbblk + (((t >> 3) * K + c) * 64 + lane) * 4) = nacc[c];
                    }
                    if (TB && (t & 31) == 31) {
                        // each lane's state choices of the last 32 steps, bit
                        // 31 - (t & 31) for step t, 1 = opened
#pragma unroll
                        for (int x = 0; x < 5; ++x) {
                            if (NOI && x >= 2) continue;
#pragma unroll
                            for (int c = 0; c < K; ++c)
                                *(uint32_t*)(tbblk + 2048 * K +
                                             (((x * K + c) * 2 + (t >> 5)) * 64 + lane) * 4) =
                                    xacc[x][c];
                        }
                    }
                    // shift histories
                    hl3 = hl2; hl2 = hl1; hl1 = hl0;
#pragma unroll
                    for (int c = 0; c < K; ++c) {
                        h3[c] = h2[c]; h2[c] = h1[c]; h1[c] = Hn[c];
                        d3[c] = d2[c]; d2[c] = d1[c]; d1[c] = Dn[c];
                        if (!NOI) { a1[c] = An[c]; b1[c] = Bn[c]; c1[c] = Cn[c]; }
                    }
                    ddm1 = DDN ? vadd<F32>(dd0, kOne) : dd0;
                    dd0 = DDN ? vadd<F32>(ds0.z, kOne) : ds0.z;
                    aam2 = aam1; aam1 = ds0.w;
                    if (!EARLY) {
                        out_l[t] = make_int2(Hout, Iout);
                        if (!XLDS) cin = nin;
                        else if (t + 1 < 64) cin = in_l[t + 1];
                    }
                    // rotate the pipeline
                    cd0 = nd0; nd0 = fd0;
#pragma unroll
                    for (int c = 0; c < K; ++c) csc[c] = nsc[c];
                }  // steps

                // merge the chunk's best into the strip's best (first maximum)
                if (MIXED || !fixed_end_mode(MODE)) {
#pragma unroll
                    for (int c = 0; c < K; ++c) {
                        int v, tt;
                        if (MODE == MPG_LOCAL || F32) {
                            v = key_value<TB, F32>(bk[c]);
                            tt = 63 - (bk[c] & 63);
                        }
                        else { v = bk[c]; tt = bkt[c]; }
                        if (v > best[c]) { best[c] = v; bstep[c] = ch * 64 + tt; }
                        bk[c] = kNone;
                    }
                }
                // publish the strip's last column for rows ch*64-63+lane.  The
                // counter lags one chunk: once every memory operation but this
                // store has completed, the previous chunk's rows are at the
                // coherence point, so chunks 0..ch-1 are announced without
                // waiting for the store just issued.
                if (has_next) {
                    const int orow = ch * 64 - 63 + lane;
                    st_dev2(&bnd_g[kBndLo + orow], outb[lane]);
                    __builtin_amdgcn_s_waitcnt(kWaitVm1);
                    if (lane == 0 && ch > 0) st_dev(&prog[strip], ch);
                }
            }
        }  // chunks
        if (has_next && !failed) {
            __builtin_amdgcn_s_waitcnt(0);  // the last chunk's rows, then the count
            if (lane == 0) st_dev(&prog[strip], nchunks);
        }
        if (failed) {
            // let the strips to the right drain quickly; the pair reports an error
            if (lane == 0) {
                st_dev(&prog[strip], nchunks);
                atomicMax(&ps->bad, 1);
            }
        }

        // ---- strip epilogue: best cell of the strip, folded into the pair.
        // A pair of one strip keeps it in registers: no pair state, no
        // atomics.
        const bool solo = nstrips == 1;
        unsigned long long solo_key = 0;
        int solo_gsc = NEG;
        if (!failed) {
            if (fixed) {
                // H(n, m): tracked on its own, or (mixed variant) the best
                // cell of row n
                int hv[K];
#pragma unroll
                for (int c = 0; c < K; ++c) hv[c] = MIXED ? best[c] : hn[c];
                if (solo) {
                    int v = NEG;
#pragma unroll
                    for (int c = 0; c < K; ++c)
                        if (col0 + c == m) v = hv[c];
                    // one lane holds column m
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) v = imax(v, __shfl_xor(v, o, 64));
                    solo_gsc = v;
                } else {
#pragma unroll
                    for (int c = 0; c < K; ++c)
                        if (col0 + c == m) st_dev(&ps->gsc, hv[c]);
                }
            } else {
                uint64_t key = 0;
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    const int row = bstep[c] - lane;
                    const int col = col0 + c;
                    const int v = SV::score(best[c]);
                    if (col <= m && row >= 0 && row <= n && best[c] > UNREACH) {
                        const uint64_t k2 = end_key(v, row, col);
                        key = k2 > key ? k2 : key;
                    }
                }
                key = wave_max_u64(key);
                best_key = key > best_key ? key : best_key;
                if (solo) solo_key = best_key;
                else if (lane == 0 && best_key)
                    atomicMax(&ps->key, (unsigned long long)best_key);
            }
        }
        // the wave that finishes the pair's last strip writes the result.
        // Its end key and H(n, m) are device-scope atomics that completed
        // before the count (the wait), so the finishing wave reads them
        // after its own count; when the traceback is walked in this kernel
        // the count is also acquire-release, so that the walking wave sees
        // every strip's direction bits.
        int done = 0;
        if (!solo) {
            __builtin_amdgcn_s_waitcnt(0);
            if (lane == 0)
                done = (TB && sink.walk)
                           ? __hip_atomic_fetch_add(&ps->done, 1, __ATOMIC_ACQ_REL,
                                                    __HIP_MEMORY_SCOPE_AGENT)
                           : __hip_atomic_fetch_add(&ps->done, 1, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
            done = __builtin_amdgcn_readfirstlane(done);
        }
        if (done == nstrips - 1) {
            const unsigned long long k =
                solo ? solo_key
                     : __hip_atomic_load(&ps->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int gv =
                __builtin_amdgcn_readfirstlane(solo ? solo_gsc : ld_dev(&ps->gsc));
            const int bad = solo ? 0 : __builtin_amdgcn_readfirstlane(ld_dev(&ps->bad));
            mpg_dev_result R;
            R.g_beg = -1;
            R.p_beg = -1;
            R.ops_off = J.ops_off;
            R.ops_len = 0;
            R._pad = 0;
            if (bad) {
                R.status = MPG_E_DEVICE;
                R.score = 0;
                R.g_end = -1;
                R.p_end = -1;
            } else if (fixed) {
                if (gv < UNREACH) {
                    R.status = MPG_E_NOALN;
                    R.score = 0;
                    R.g_end = -1;
                    R.p_end = -1;
                } else {
                    R.status = MPG_OK;
                    R.score = SV::score(gv);
                    R.g_end = n;
                    R.p_end = m;
                }
            } else {
                const uint32_t khi = __builtin_amdgcn_readfirstlane((uint32_t)(k >> 32));
                const uint32_t klo = __builtin_amdgcn_readfirstlane((uint32_t)k);
                const unsigned long long ku = ((unsigned long long)khi << 32) | klo;
                R.status = MPG_OK;
                R.score = (int)(ku >> 36) - (1 << 27);
                R.g_end = (1 << 21) - 1 - (int)((ku >> 15) & ((1u << 21) - 1));
                R.p_end = (1 << 15) - 1 - (int)(ku & ((1u << 15) - 1));
            }
            if (TB && sink.walk) {
                if (solo) {
                    // this wave's own direction bits: complete, then read
                    // past the vector cache
                    __builtin_amdgcn_s_waitcnt(0);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
                // walk the traceback now: the pair completes without a second kernel
                char* txt = sink.ops + J.ops_off;
                if (R.status == MPG_OK) {
                    const TbView V{tbbuf + J.tb_off, J.K, J.nchunks};
                    const int64_t end = 2LL * (n + m);
                    OpWriter W{txt, end};
                    int bi = -1, bj = -1;
                    const bool ok = walk_wave(V, R.g_end, R.p_end, n, m, W, lane, bi, bj);
                    if (!ok || W.overflow) {
                        R.status = MPG_E_DEVICE;
                        if (lane == 0) txt[0] = 0;
                    } else {
                        if (lane == 0) txt[end] = 0;
                        R.g_beg = bi;
                        R.p_beg = bj;
                        R.ops_off = J.ops_off + W.pos;
                        R.ops_len = (int32_t)(end - W.pos);
                    }
                } else if (lane == 0) {
                    txt[0] = 0;
                }
            }
            if (lane == 0) publish(sink.out + J.res, R, sink.system);
        }
    }  // queue
}

template <int K, int MODE, bool TB, bool PRO, bool F32>
hipError_t launch_dp_t(hipStream_t s, int ncu, const DevParams& P, const PairJob* jobs,
                       const int2* items, int nitems, int* qhead, PairState* pst, int* prog,
                       const uint8_t* prot, const uint8_t* desc, int2* bnd, uint8_t* tbbuf,
                       const DpSink& sink) {
    const bool noi = (P.flags & MPG_NO_INTRON) != 0;
    const bool nof = (P.flags & MPG_NO_FRAMESHIFT) != 0;
    const size_t lds = (size_t)LdsLayout<K, TB, MODE == MPG_LOCAL && !PRO>::WAVE;
    dim3 b(64);
    // persistent grid: as many waves as ncu compute units hold at once for
    // this kernel, never more than there are items
#define MPG_LAUNCH(NI, NF)                                                                      \
    do {                                                                                        \
        static int per_cu = 0;                                                                  \
        if (per_cu <= 0 &&                                                                      \
            hipOccupancyMaxActiveBlocksPerMultiprocessor(                                       \
                &per_cu, dp_kernel<K, MODE, TB, NI, NF, PRO, F32>, 64, lds) != hipSuccess)           \
            per_cu = 0;                                                                         \
        const int waves = per_cu > 0 ? per_cu * ncu : 8 * ncu;                                \
        dim3 g(nitems < waves ? nitems : waves);                                                \
        hipLaunchKernelGGL((dp_kernel<K, MODE, TB, NI, NF, PRO, F32>), g, b, lds, s, jobs, items,   \
                           nitems, qhead, pst, prog, prot, desc, bnd, tbbuf, sink, P);          \
    } while (0)
    if (!noi && !nof) MPG_LAUNCH(false, false);
    else if (noi && !nof) MPG_LAUNCH(true, false);
    else if (!noi && nof) MPG_LAUNCH(false, true);
    else MPG_LAUNCH(true, true);
#undef MPG_LAUNCH
    return hipGetLastError();
}

template <int K, bool PRO, bool F32>
hipError_t launch_dp_k(hipStream_t s, int ncu, bool tb, const DevParams& P, const PairJob* jobs,
                       const int2* items, int nitems, int* qhead, PairState* pst, int* prog,
                       const uint8_t* prot, const uint8_t* desc, int2* bnd, uint8_t* tbbuf,
                       const DpSink& sink) {
#define MPG_MODE(M)                                                                             \
    return tb ? launch_dp_t<K, M, true, PRO, F32>(s, ncu, P, jobs, items, nitems, qhead, pst, prog, \
                                             prot, desc, bnd, tbbuf, sink)                      \
              : launch_dp_t<K, M, false, PRO, F32>(s, ncu, P, jobs, items, nitems, qhead, pst, prog, \
                                              prot, desc, bnd, tbbuf, sink)
    switch (P.mode) {
        case MPG_LOCAL: MPG_MODE(MPG_LOCAL);
        case MPG_EXTEND: MPG_MODE(MPG_EXTEND);
        case kModeMixed:
            if constexpr (!PRO) MPG_MODE(kModeMixed);
            return hipErrorInvalidValue;  // profile queries come in one mode per call
        default: MPG_MODE(MPG_GLOBAL);  // GLOBAL and EXTEND_LEFT (per-pair start term)
    }
#undef MPG_MODE
}

}  // namespace dev
}  // namespace mpg
