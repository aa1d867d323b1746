// Chaining of seed anchors on gfx950 (Methods, "Chaining" of Li 2022):
// Eq. (gap) on a genome binned in 256-bp bins (or, in the second round, the
// base-resolution gap 3*dy - dx), the chaining recurrence
//   f(j) = max(k, max_{i<j} f(i) + min(y_j - y_i, k) - gamma(g(i,j)))
// with the gap penalty of Eq. (gap-pen), then the extraction of chains and
// their ranking.
//
// One workgroup per anchor set: one wavefront, or four when the launch's
// largest set has 512 anchors or more (its chain of anchors is the launch's
// critical path).  Anchors go 64 at a time, one per lane.  First every lane
// takes the candidates before the block (the wavefronts share them, nearest
// first): all lanes look at the same candidate at once, so nothing is reduced
// across lanes, and a candidate costs one comparison unless some lane may
// still gain by it: its value is at most f(i) + k, since the gap penalty is
// never negative, and only a candidate that may reach a lane's best pays for
// the gap and its log2.  The scan ends where the genome distance alone
// exceeds G.  Then the block's own anchors are settled one after another, each
// offered to the lanes behind it.  (One anchor at a time, the lanes striding
// over its candidates and an arg-max over the workgroup, took 3.4 us per
// anchor of the largest set: 2.42 ms for 3,000 sets of up to 700 anchors; now
// 1.07 ms.)
//
// f of the set's anchors lives in LDS (fp64), or, for a set too large for it,
// in the f output in HBM, read and written with device-scope atomics so that
// no wavefront reads a stale copy from its vector cache.  Extraction takes the
// unused anchor of largest f again and again and follows its predecessors; the
// ranking takes the best chain again and again.  A set held in LDS does both
// in one wavefront, each lane keeping the best of every 64th anchor or chain,
// so that a round is one arg-max and a rescan of the lanes that lost an
// anchor; a larger set scans all its anchors in every round.
#include "mpg_internal.h"

namespace mpg {
namespace dev {

// Eq. (gap) (binned) or 3*dy - dx (base resolution).
__device__ __forceinline__ long long chain_gap(long long dx, long long dy, int binned) {
    if (!binned) return 3 * dy - dx;
    const long long lo = 256 * (dx - 1), hi = 256 * (dx + 1);
    if (3 * dy < lo) return 3 * dy - lo;
    if (3 * dy > hi) return 3 * dy - hi;
    return 0;
}

// Eq. (gap-pen) for |g| < G.  Each operation rounds on its own (no fused
// multiply-add), in the order the equation is written.
__device__ __forceinline__ double chain_gamma(long long g, double beta) {
#pragma clang fp contract(off)
    if (g == 0) return 0.0;
    const double a = (double)(g < 0 ? -g : g);
    const double third = a / 3.0;
    const double lg = beta * log2(a + 1.0);
    if (g > 0) return third + lg;
    return third < lg ? third : lg;
}

// A number not above chain_gamma(g, beta): its terms in fp32, less more than
// their rounding (every term is at least 1/3 or beta, the relative errors of
// the conversions, products and log2 are below 1e-6 in all).
__device__ __forceinline__ double gamma_low(long long g, float beta) {
    if (g == 0) return 0.0;
    const float a = (float)(g < 0 ? -g : g);
    const float third = a * 0.333333f, lg = beta * __log2f(a + 1.0f);
    return (double)((g > 0 ? third + lg : fminf(third, lg)) * 0.99999f);
}

// Wave-wide arg-max of (v, i): the larger v, ties the smaller i (i < 0: none).
__device__ __forceinline__ void wave_argmax(double& v, int& i) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v2 = __shfl_xor(v, o);
        const int i2 = __shfl_xor(i, o);
        const bool take = i2 >= 0 && (i < 0 || v2 > v || (v2 == v && i2 < i));
        v = take ? v2 : v;
        i = take ? i2 : i;
    }
}

// Arg-max of (v, i) over the workgroup's W wavefronts (the larger v, ties
// the smaller i); every thread receives it.  rv, ri: W slots in LDS.
template <int W>
__device__ __forceinline__ void block_argmax(double& v, int& i, double* rv, int* ri) {
    wave_argmax(v, i);
    if constexpr (W > 1) {
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            rv[w] = v;
            ri[w] = i;
        }
        __syncthreads();
        v = rv[0];
        i = ri[0];
#pragma unroll
        for (int q = 1; q < W; ++q) {
            const double v2 = rv[q];
            const int i2 = ri[q];
            const bool take = i2 >= 0 && (i < 0 || v2 > v || (v2 == v && i2 < i));
            v = take ? v2 : v;
            i = take ? i2 : i;
        }
        __syncthreads();  // the slots are free again
    }
}

// Wave-wide maximum of an unsigned value (row shifts, then row broadcasts;
// lanes without a source keep 0, the identity).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define MPG_DPP_MAX(CTRL)                                                                   \
    {                                                                                       \
        const uint32_t o =                                                                  \
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);        \
        v = o > v ? o : v;                                                                  \
    }
    MPG_DPP_MAX(0x111)  // row_shr:1
    MPG_DPP_MAX(0x112)
    MPG_DPP_MAX(0x114)
    MPG_DPP_MAX(0x118)
    MPG_DPP_MAX(0x142)  // row_bcast:15
    MPG_DPP_MAX(0x143)  // row_bcast:31
#undef MPG_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Arg-max over the wavefront of (v, i), i < 0: none: the larger v, ties the
// smaller i.  A double's bits, the sign bit set (positive) or all inverted
// (negative), order the numbers as unsigned integers.
__device__ __forceinline__ int wave_best(double v, int i) {
    const long long b = __double_as_longlong(v);
    const unsigned long long u =
        i < 0 ? 0ull : (unsigned long long)b ^ (b < 0 ? ~0ull : 1ull << 63);
    const uint32_t hi = (uint32_t)(u >> 32), lo = (uint32_t)u;
    const uint32_t mh = wave_max_u32(hi);
    const uint32_t ml = wave_max_u32(hi == mh ? lo : 0u);
    // the smallest index is the largest complement; none: 0
    return (int)~wave_max_u32(i >= 0 && hi == mh && lo == ml ? ~(uint32_t)i : 0u);
}

__device__ __forceinline__ double ld_f64_dev(const double* p) {
    const unsigned long long u = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return __longlong_as_double((long long)u);
}
__device__ __forceinline__ void st_f64_dev(double* p, double v) {
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W>
__global__ void __launch_bounds__(64 * W) chain_kernel(const ChainSetJob* __restrict__ sets,
                                                       int nsets, const int2* __restrict__ anchors,
                                                       ChainCfg cfg, double* __restrict__ f_out,
                                                       int* __restrict__ pred_out,
                                                       ChainRec* __restrict__ recs,
                                                       int* __restrict__ idx_out,
                                                       mpg_chain_out* __restrict__ top,
                                                       int* __restrict__ ntop) {
    constexpr int NT = 64 * W;
    if ((int)blockIdx.x >= nsets) return;
    const int tid = threadIdx.x;
    // the jobs come largest set first (the launch's makespan is the largest
    // sets' sequential work); id is the set's own index
    const ChainSetJob S = sets[blockIdx.x];
    const int s = S.id;
    const int n = S.n;
    extern __shared__ __align__(16) uint8_t smem[];
    // LDS: the reduction slots, then f (if it fits), then (staged) the
    // anchors and the predecessors, then the used flags.  The anchor reads
    // of the candidate loop and the predecessor walk of the extraction are on
    // the set's sequential path, so staging them takes a global-memory
    // latency off every step of it.
    const bool f_lds = cfg.f_lds != 0;
    const bool stage = cfg.stage != 0;
    double* rv = (double*)smem;
    int* ri = (int*)(smem + 8 * W);
    size_t off = kChainRedBytes;
    double* f = (double*)(smem + off);
    if (f_lds) off += 8 * (size_t)cfg.max_n;
    int2* sA = (int2*)(smem + off);
    int* spo = (int*)(smem + off + 8 * (size_t)cfg.max_n);
    if (stage) off += 12 * (size_t)cfg.max_n;
    uint8_t* used = smem + off;
    const int2* A = anchors + S.off;
    double* fo = f_out + S.off;
    int* po = pred_out + S.off;
    auto fget = [&](int i) -> double { return f_lds ? f[i] : ld_f64_dev(fo + i); };
    if (S.status != MPG_OK) {
        if (tid == 0) ntop[s] = S.status;
        return;
    }
    if (stage) {
        for (int i = tid; i < n; i += NT) sA[i] = A[i];
        __syncthreads();
    }
    const int2* AA = stage ? (const int2*)sA : A;
    const double kd = (double)cfg.k;
    // ---- the DP, 64 anchors at a time
    const int lane = tid & 63, wave = tid >> 6;
    double* mv = (double*)(smem + kChainRedBytes - 64 * 12 * 3);  // the other wavefronts' bests
    int* mi = (int*)(mv + 64 * 3);
    // beyond this genome distance (in x units) |g| >= G whatever the residues
    long long ylo = 0, yhi = 0;
    for (int i = lane; i < n; i += 64) {
        const long long y = AA[i].y;
        if (i == lane) ylo = yhi = y;
        ylo = y < ylo ? y : ylo;
        yhi = y > yhi ? y : yhi;
    }
    if (lane >= n) ylo = yhi = n ? AA[0].y : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const long long a = __shfl_xor(ylo, o), b = __shfl_xor(yhi, o);
        ylo = a < ylo ? a : ylo;
        yhi = b > yhi ? b : yhi;
    }
    const long long reach = (long long)cfg.G + 3 * (yhi - ylo);
    auto too_far = [&](long long dx) { return (cfg.binned ? 256 * (dx - 1) : dx) >= reach; };
    // (a beta beyond fp32 bounds nothing: 0 is a bound too)
    const float beta_f = cfg.beta < 1e30 ? (float)cfg.beta : 0.0f;
    for (int j0 = 0; j0 < n; j0 += 64) {
        const int j = j0 + lane;
        const bool live = j < n;
        const int2 aj = AA[live ? j : n - 1];
        double bv = kd;
        int bi = -1;
        // candidate i = (ai, fi) offered to the lanes in `open`; `last`: of
        // equal values the one offered later wins (smaller i: descending scan)
        auto offer = [&](const int2 ai, double fi, int i, bool open, bool last) {
            const bool may = open && (last ? fi + kd >= bv : fi + kd > bv);
            if (!__any(may)) return;
            bool ok = may && aj.x >= ai.x && aj.y > ai.y;
            if (!__any(ok)) return;
            const long long dx = (long long)aj.x - ai.x, dy = (long long)aj.y - ai.y;
            const long long g = chain_gap(dx, dy, cfg.binned);
            const double u = fi + (double)(int)(dy < cfg.k ? dy : cfg.k);
            ok = ok && g < cfg.G && -g < cfg.G;
            // the exact penalty (a division and a log2 in fp64) only where a
            // lower bound of it leaves the candidate in
            const double most = u - gamma_low(g, beta_f);
            ok = ok && (last ? most >= bv : most > bv);
            if (!__any(ok)) return;
            double v = u;
            if (__any(ok && g != 0)) v = u - chain_gamma(ok ? g : 0, cfg.beta);
            if (ok && (v > bv || (last && v == bv && bi >= 0))) {
                bv = v;
                bi = i;
            }
        };
        // the anchors before the block, in chunks of 64, nearest first
        const int x0 = AA[j0].x;
        for (int c = j0 / 64 - 1 - wave; c >= 0; c -= W) {
            if (too_far((long long)x0 - AA[c * 64 + 63].x)) break;
            for (int q = 56; q >= 0; q -= 8) {
                int2 ai[8];
                double fi[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    ai[r] = AA[c * 64 + q + r];
                    fi[r] = fget(c * 64 + q + r);
                }
#pragma unroll
                for (int r = 7; r >= 0; --r) offer(ai[r], fi[r], c * 64 + q + r, live, true);
            }
        }
        if constexpr (W > 1) {
            if (wave > 0) {
                mv[(wave - 1) * 64 + lane] = bv;
                mi[(wave - 1) * 64 + lane] = bi;
            }
            __syncthreads();
        }
        if (wave == 0) {
#pragma unroll
            for (int w = 0; w + 1 < W; ++w) {
                const double v2 = mv[w * 64 + lane];
                const int i2 = mi[w * 64 + lane];
                if (i2 >= 0 && (v2 > bv || (v2 == bv && i2 < bi))) {
                    bv = v2;
                    bi = i2;
                }
            }
            // the block's own anchors, each once it is settled
            const int cnt = n - j0 < 64 ? n - j0 : 64;
            for (int t = 0; t + 1 < cnt; ++t) {
                const long long fb = __double_as_longlong(bv);
                const int flo = __builtin_amdgcn_readlane((int)fb, t);
                const int fhi = __builtin_amdgcn_readlane((int)(fb >> 32), t);
                const double fi = __longlong_as_double(((long long)fhi << 32) | (uint32_t)flo);
                const int2 ai = make_int2(__builtin_amdgcn_readlane(aj.x, t),
                                          __builtin_amdgcn_readlane(aj.y, t));
                offer(ai, fi, j0 + t, live && lane > t, false);
            }
            if (live) {
                if (f_lds) {
                    f[j] = bv;
                    fo[j] = bv;
                } else {
                    st_f64_dev(fo + j, bv);
                }
                po[j] = bi;
                if (stage) spo[j] = bi;
            }
        }
        __syncthreads();
    }
    if (stage) {
        // ---- extraction and ranking in one wavefront; a used anchor's f is
        // negated in LDS, and the chains' scores take the anchors' place
        if (wave > 0) return;
        double* sc = (double*)sA;
        ChainRec* R = recs + S.off;  // at most n chains
        int* idx = idx_out + S.off;
        double lv = 0.0;
        int li = -1;  // the best unused anchor among lane, lane + 64, ...
        auto rescan = [&]() {
            lv = 0.0;
            li = -1;
            int i = lane;
            for (; i + 7 * 64 < n; i += 8 * 64) {  // eight reads in flight
                double fi[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) fi[r] = f[i + 64 * r];
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (fi[r] > lv) {
                        lv = fi[r];
                        li = i + 64 * r;
                    }
            }
            for (; i < n; i += 64) {
                const double fi = f[i];
                if (fi > lv) {
                    lv = fi;
                    li = i;
                }
            }
        };
        rescan();
        int nc = 0, pos = 0;
        for (;;) {
            const int bi = wave_best(lv, li);
            if (bi < 0) break;
            // every lane follows the chain; lane 0 marks it
            const double top_f = f[bi];
            int len = 0, t = bi;
            unsigned long long lost = 0;
            double stop_f = 0.0;
            while (t >= 0) {
                const double ft = f[t];
                if (!(ft > 0.0)) {
                    stop_f = -ft;
                    break;
                }
                if (lane == 0) f[t] = -ft;
                lost |= 1ull << (t & 63);
                ++len;
                t = spo[t];
            }
            // indices ascending: written from the end of the chain's range
            int u = bi;
            for (int q = len - 1; q >= 0; --q) {
                if (lane == 0) idx[pos + q] = u;
                u = spo[u];
            }
            const double score = top_f - stop_f;
            if (lane == 0) {
                sc[nc] = score;
                ChainRec c;
                c.score = score;
                c.first = pos;
                c.len = len;
                R[nc] = c;
            }
            pos += len;
            ++nc;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if ((lost >> lane) & 1) rescan();
        }
        const int keep = nc < cfg.max_chains ? nc : cfg.max_chains;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        auto rescan_chains = [&]() {
            lv = -INFINITY;
            li = -1;
            for (int c = lane; c < nc; c += 64) {
                const double v = sc[c];
                if (v > lv) {  // -infinity: taken
                    lv = v;
                    li = c;
                }
            }
        };
        rescan_chains();
        for (int r = 0; r < keep; ++r) {
            const int bc = wave_best(lv, li);
            if (bc < 0) break;
            if (lane == (bc & 63)) {
                const ChainRec c = R[bc];
                mpg_chain_out o;
                o.score = c.score;
                o.first = c.first;
                o.len = c.len;
                top[(int64_t)s * cfg.max_chains + r] = o;
                sc[bc] = -INFINITY;
                rescan_chains();
            }
        }
        if (lane == 0) ntop[s] = keep;
        return;
    }
    // ---- extraction: the unused anchor of largest f starts a chain that
    // follows the predecessors until -1 or a used anchor
    for (int i = tid; i < n; i += NT) used[i] = 0;
    __syncthreads();
    ChainRec* R = recs + S.off;  // at most n chains
    int* idx = idx_out + S.off;
    int* slen = ri + W;  // one more slot: the chain's length for every thread
    int nc = 0, pos = 0;
    for (;;) {
        double bv = 0.0;
        int bi = -1;
        for (int i = tid; i < n; i += NT)
            if (!used[i]) {
                const double fi = fget(i);
                if (bi < 0 || fi > bv) {
                    bv = fi;
                    bi = i;
                }
            }
        block_argmax<W>(bv, bi, rv, ri);
        if (bi < 0) break;
        if (tid == 0) {
            int len = 0;
            int t = bi;
            const int* P = stage ? (const int*)spo : po;
            while (t >= 0 && !used[t]) {
                used[t] = 1;
                ++len;
                t = P[t];
            }
            // indices ascending: write from the end of the chain's range
            int u = bi;
            for (int q = len - 1; q >= 0; --q) {
                idx[pos + q] = u;
                u = P[u];
            }
            ChainRec c;
            c.score = fget(bi) - (t >= 0 ? fget(t) : 0.0);
            c.first = pos;
            c.len = len;
            R[nc] = c;
            *slen = len;
        }
        __syncthreads();
        pos += *slen;
        ++nc;
        __syncthreads();  // slen is written again by the next chain
    }
    // ---- ranking: the max_chains best chains (ties: extracted first)
    const int keep = nc < cfg.max_chains ? nc : cfg.max_chains;
    for (int r = 0; r < keep; ++r) {
        double bv = 0.0;
        int bi = -1;
        for (int c = tid; c < nc; c += NT)
            if (R[c].len > 0 && (bi < 0 || R[c].score > bv)) {
                bv = R[c].score;
                bi = c;
            }
        block_argmax<W>(bv, bi, rv, ri);
        if (tid == 0) {
            mpg_chain_out o;
            o.score = R[bi].score;
            o.first = R[bi].first;
            o.len = R[bi].len;
            top[(int64_t)s * cfg.max_chains + r] = o;
            R[bi].len = -R[bi].len - 1;  // taken
        }
        __syncthreads();
    }
    if (tid == 0) ntop[s] = keep;
}

}  // namespace dev

hipError_t launch_chain(hipStream_t st, const ChainSetJob* sets, int nsets, const int2* anchors,
                        const ChainCfg& cfg, double* f, int* pred, ChainRec* recs, int* idx,
                        mpg_chain_out* top, int* ntop) {
    if (nsets <= 0) return hipSuccess;
    const size_t lds = chain_lds_bytes(cfg);
    if (cfg.waves == 4)
        hipLaunchKernelGGL(dev::chain_kernel<4>, dim3(nsets), dim3(256), lds, st, sets, nsets,
                           anchors, cfg, f, pred, recs, idx, top, ntop);
    else
        hipLaunchKernelGGL(dev::chain_kernel<1>, dim3(nsets), dim3(64), lds, st, sets, nsets,
                           anchors, cfg, f, pred, recs, idx, top, ntop);
    return hipGetLastError();
}

}  // namespace mpg
