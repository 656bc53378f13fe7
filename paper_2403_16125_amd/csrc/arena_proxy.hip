// HIP kernel of the proxy-plan planner (gfx950).
//
// For every (job, GPU type, GPU count) cell, the load-aware planner of
// Sec. 3.3 without execution:
//   * the job's layers form O = min(L, n_ops) clustered operators; each
//     operator's load is its roofline time (Eq. 2: FLOPs over the attainable
//     rate at its arithmetic intensity) and its GPU share is proportional to
//     the load;
//   * every pipeline degree s is a grid (Sec. 3.2); in it every contiguous
//     grouping of the operators into s stages is normalised to power-of-two
//     stage GPU counts summing to n with the least computation bias (Eq. 3);
//   * per microbatch count B, among groupings whose stages fit memory, the
//     proxy plan has the least bias, then the least communication load
//     (Eq. 4) with each stage's intra-stage (dp, tp) chosen for the least
//     communication; it is priced by the 1F1B model with per-stage GPU
//     counts (Sec. 3.4);
//   * the cell keeps the fastest grid (ties within the tie window: fewer
//     stages, then fewer microbatches).
//
// One workgroup of 4 waves per cell; the waves take its pipeline degrees from an
// LDS counter and each works through a degree on its own (no block barrier
// between set-up and the cell's choice).  A degree's least-bias groupings are
// found by branch and bound instead of scanning every grouping's multisets:
//   * bias bound: stage shares and stage GPU counts both sum to n, so for any
//     multiplier l the bias sum_j (2^e_j - D_j)^2 equals sum_j (2^e_j - D_j)^2 +
//     l (2^e_j - D_j), and dropping the constraint that the 2^e_j sum to n gives
//     a lower bound that is a sum over the stages of table entries
//     min_e (2^e - D)^2 + l (2^e - D); the largest over kLam multipliers is used;
//   * memory bound, per microbatch count B: a stage needs at least the smallest
//     power of two of GPUs at which B divides and the stage fits, so a grouping
//     whose stages need more than n GPUs together does not fit at B;
//   * limits: a shortest-path pass over the same table gives, per multiplier,
//     the grouping of least bound of every degree; those groupings' biases bound
//     the answer of every B they fit at.
// Only groupings within both bounds for some B have their multisets scanned;
// they are collected to fill the lanes, each lane (or a power of two of lanes,
// when few are left) taking one grouping.  The choice is the plain
// enumeration's: a bound only drops a grouping whose bias is strictly larger
// than that of a grouping that fits.  Measured on 96 trace-like jobs x 4 types
// x 35 counts (16 operators): 75.6 ms scanning every grouping, 11.8 ms so; of
// these 3.4 ms set-up and walk, 0.8 ms limits, 6.3 ms scans (nearly all at B
// where every grouping of the degree overflows), 0.8 ms pricing.
//
// Multisets of (n, s) are lexicographically descending, so the first least
// cost wins ties.  Every B is tested for memory with the largest admissible
// tensor degree (memory falls with tp and admissibility only gets easier, so
// that tp fits iff some tp does).  Arithmetic of every decision is fp64 in the
// operation order of a plain evaluation (left-to-right stage sums, the bias
// summed over stages in stage order), so every decision is reproducible; the
// bounds are fp32, rounded down with a margin.
#include <math.h>

#include "arena_internal.h"

namespace arena {
namespace {

constexpr int kPxThreads = 256;
constexpr int kPxWaves = kPxThreads / 64;
constexpr double kInfP = __builtin_huge_val();
constexpr int kLam = 7;                   // multipliers of the bias bound, as fractions of n
constexpr int kTri = 136;                 // operator ranges [lo, hi) of 16 operators
constexpr int kNeeds = 696;               // (range, stages after it) of 16 operators: sum of hi max(1, 16 - hi)
constexpr unsigned kNoFit = 2047u;        // GPUs a stage that never fits is counted with (> n; 16 of them < 2^16)

// A range's bias-bound terms (one per multiplier) and the place of its GPU
// needs: one 32-byte entry, so a stage costs two LDS reads.
struct alignas(16) RangeBound {
    float t[kLam];
    int32_t need;                         // first entry of S.need for this range
};

// One wave's degree: NB microbatch counts.
template <int NB>
struct alignas(16) PxWave {
    float lim[NB];                        // a grouping whose bound passes this cannot win at B (-inf: B closed)
    unsigned long long bdexp[NB];         // per B: stage GPU exponents of the least-bias grouping
    double bkey[NB];                      //   its squared bias (+inf: none fits)
    double tkey[NB];                      //   ties: least communication load
    int32_t tidx[NB];                     //   and its rank key
    int32_t bidx[NB];                     //   rank key of the least-bias grouping
    uint32_t bmask[NB];                   //   its stage starts
    uint16_t cand[128];                   // groupings waiting for a scan
};

template <int NB>
struct ProxyLds {
    // sums of the operator quantities over every range [lo, hi), left to right
    double ss[6][kTri];
    RangeBound rb[17 * 16];                      // range [lo, hi) at hi * 16 + lo
    alignas(16) uint16_t need[kNeeds][NB];       // least GPUs of a stage by (range, stages after it) and B
    // operator sums (left to right over their layers)
    double od[kProxyMaxOps], oT[kProxyMaxOps], oX[kProxyMaxOps], oE[kProxyMaxOps];
    double oP[kProxyMaxOps], oA[kProxyMaxOps], oxl[kProxyMaxOps], oload[kProxyMaxOps];
    int32_t binom[16][16];
    int32_t mval[kMaxM];
    double bt[11][kMaxM];                        // replica samples at dp = 2^e, m_values[k]; -1: not a divisor
    int32_t emax[kMaxM];                         // largest stage GPU exponent at which m_values[k] divides, -1: none
    unsigned long long gD[kProxyMaxOps + 1][NB]; // stage GPU exponents of each grid's proxy at each B
    unsigned long long gP[kProxyMaxOps + 1][NB]; // its stage tensor-degree exponents
    double gT[kProxyMaxOps + 1][NB];             // its T (inf: none fits)
    uint32_t gM[kProxyMaxOps + 1][NB];           // its stage starts (0xffffffff: no grouping fits)
    float path[kLam][2][17];                     // least bound of a prefix of operators, by parity of the stage count
    uint8_t from[kLam][17][17];                  // [multiplier][stages][end]: start of the last stage
    int32_t next_s;
    int32_t no_load;                             // every operator has zero load: no proxy plan
    PxWave<NB> w[kPxWaves];
};

// The cell's constants.
struct Cell {
    int L, Bg, O, n, gpn;
    double speed, mem, bwi, bwe, kap;
};

// Orders the LDS accesses of the lanes of one wave (its memory operations
// execute in order: the fences only stop the compiler from moving accesses).
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (key, idx) of another lane picked by one DPP control; lanes of the rows
// the row mask leaves out read the identity (+inf, INT_MAX).
template <int CTRL, int ROWS>
__device__ __forceinline__ void dpp_pair(double k, int i, double& ok, int& oi)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(k);
    const unsigned long long e = (unsigned long long)__double_as_longlong(kInfP);
    const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)e, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(e >> 32), (int)(unsigned)(b >> 32), CTRL, ROWS,
                                               0xf, false);
    ok = __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                          (unsigned long long)(unsigned)lo));
    oi = __builtin_amdgcn_update_dpp(0x7fffffff, i, CTRL, ROWS, 0xf, false);
}

__device__ __forceinline__ void take_less(double& k, int& i, double ok, int oi)
{
    const bool t = (ok < k) | ((ok == k) & (oi < i));
    k = t ? ok : k;
    i = t ? oi : i;
}

// Least (key, idx) of the wave (smaller key, then smaller idx), in every
// lane: quad swaps and row rotations give each row its least pair, row
// broadcasts carry it to the last row, lane 63 hands the result out.  DPP
// moves need no lane addresses (a shuffle's would be held in registers).
__device__ __forceinline__ void wave_argmin(double& k, int& i)
{
    double ok;
    int oi;
    dpp_pair<0xB1, 0xf>(k, i, ok, oi);    // quad_perm [1,0,3,2]
    take_less(k, i, ok, oi);
    dpp_pair<0x4E, 0xf>(k, i, ok, oi);    // quad_perm [2,3,0,1]
    take_less(k, i, ok, oi);
    dpp_pair<0x124, 0xf>(k, i, ok, oi);   // row_ror:4
    take_less(k, i, ok, oi);
    dpp_pair<0x128, 0xf>(k, i, ok, oi);   // row_ror:8
    take_less(k, i, ok, oi);
    dpp_pair<0x142, 0xa>(k, i, ok, oi);   // row_bcast:15 into rows 1 and 3
    take_less(k, i, ok, oi);
    dpp_pair<0x143, 0xc>(k, i, ok, oi);   // row_bcast:31 into rows 2 and 3
    take_less(k, i, ok, oi);
    const unsigned long long b = (unsigned long long)__double_as_longlong(k);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned)b, 63);
    const int hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
    k = __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                         (unsigned long long)(unsigned)lo));
    i = __builtin_amdgcn_readlane(i, 63);
}

// Stage-start mask (bit i: a stage starts at operator i, i >= 1) of the
// grouping of rank r among those of O operators into s stages, cut vectors
// in lexicographic order.
template <class Lds>
__device__ __forceinline__ unsigned unrank(int r, int O, int s, const Lds& S)
{
    unsigned mask = 0u;
    const int N = O - 1, t = s - 1;
    int c = 1;
    for (int q = 0; q < t; ++q) {
        for (;;) {
            const int cnt = S.binom[N - c][t - 1 - q];
            if (r < cnt) break;
            r -= cnt;
            ++c;
        }
        mask |= 1u << c;
        ++c;
    }
    return mask;
}

// The grouping after `mask` in lexicographic order of cut vectors (t cuts
// among operators 1..O-1): the last cut moves up if it can; otherwise the
// cuts packed against the end follow the highest cut that can still move.
__device__ __forceinline__ unsigned next_grouping(unsigned mask, int O, int t)
{
    const int top = O - 1;
    int r = 0;
    while (r < t && ((mask >> (top - r)) & 1u)) ++r;
    if (r == 0) {
        const int c = 31 - __clz(mask);
        return mask ^ (1u << c) ^ (1u << (c + 1));
    }
    const unsigned rest = mask & ~(((1u << r) - 1u) << (top - r + 1));
    const int c = 31 - __clz(rest);
    return (rest ^ (1u << c)) | (1u << (c + 1)) | (((1u << r) - 1u) << (c + 2));
}

// End (exclusive) of the stage starting at `lo`: the next stage start, or O.
__device__ __forceinline__ int stage_end(unsigned mask, int lo, int O)
{
    const unsigned rest = mask & ~((2u << lo) - 1u);
    return rest ? __ffs(rest) - 1 : O;
}

// Operator quantities kept as range sums.
enum { kQd = 0, kQT, kQX, kQE, kQP, kQA };

__device__ __forceinline__ int tri(int lo, int hi)
{
    return ((hi * (hi - 1)) >> 1) + lo;
}

template <class Lds>
__device__ __forceinline__ double ssum(const Lds& S, int qn, int lo, int hi)
{
    return S.ss[qn][tri(lo, hi)];
}

// Squared bias of multiset m (exponents at bits 4p, largest first) with
// stage j taking position q_j, summed over the stages in stage order (S
// stages, a compile-time count so the sum has no branches).
template <int S>
__device__ __forceinline__ double bias(unsigned long long m, const double (&D)[16], const int (&q)[16])
{
    const unsigned lo = (unsigned)m, hi = (unsigned)(m >> 32);
    double cost = 0.0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        // the exponent of position q_j, then 2^e from its exponent field (e <= 10)
        const unsigned e = __builtin_amdgcn_ubfe(q[j] < 8 ? lo : hi, (unsigned)(4 * q[j]) & 31u, 4u);
        const double diff = __hiloint2double((int)((e << 20) + 0x3ff00000u), 0) - D[j];   // 2^e - share
        cost += diff * diff;
    }
    return cost;
}

// The least bias over multisets k = first, first + step, ... below K (the
// table is lexicographically descending, so among equal costs the smallest k
// wins) and that k (-1 if none).
template <int S>
__device__ __forceinline__ double normalise_s(const double (&D)[16], const int (&q)[16], int K, int first,
                                              int step, const unsigned long long* __restrict__ ms, int& bk)
{
    double best = kInfP;
    bk = -1;
    // two multisets per iteration (independent sums), compared in order
    int k = first;
    for (; k + step < K; k += 2 * step) {
        const unsigned long long m0 = ms[k], m1 = ms[k + step];
        const double c0 = bias<S>(m0, D, q);
        const double c1 = bias<S>(m1, D, q);
        if (c0 < best) {
            best = c0;
            bk = k;
        }
        if (c1 < best) {
            best = c1;
            bk = k + step;
        }
    }
    if (k < K) {
        const double c0 = bias<S>(ms[k], D, q);
        if (c0 < best) {
            best = c0;
            bk = k;
        }
    }
    return best;
}

// Stage shares D_j (stage order) and each stage's sorted position q_j
// (largest share first, ties to the lower stage) for a compile-time stage
// count; static indices so both stay in registers.
template <int S, class Lds>
__device__ __forceinline__ void shares_s(unsigned mask, int O, const Lds& Ls, double (&D)[16], int (&q)[16])
{
    int lo = 0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const int hi = stage_end(mask, lo, O);
        D[j] = ssum(Ls, kQd, lo, hi);
        lo = hi;
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
        int r = 0;
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (i != j && (D[i] > D[j] || (D[i] == D[j] && i < j))) ++r;
        q[j] = r;
    }
}

// The stage exponents (4 bits per stage, stage order) multiset m assigns.
template <int S>
__device__ __forceinline__ unsigned long long stage_exps(unsigned long long m, const int (&q)[16])
{
    unsigned long long dexp = 0ull;
#pragma unroll
    for (int j = 0; j < S; ++j) dexp |= ((m >> (4 * q[j])) & 15ull) << (4 * j);
    return dexp;
}

// The least bias of grouping `mask` over multisets first, first + step, ...
// of ms[0..K), the smallest such multiset index bk (kNoMs: none) and the
// stage exponents it assigns.
constexpr int kNoMs = 0x7fffffff;

template <int S, class Lds>
__device__ __forceinline__ double group_bias(unsigned mask, int O, int K, int first, int step, const Lds& Ls,
                                             const unsigned long long* __restrict__ ms, int& bk,
                                             unsigned long long& dexp)
{
    double D[16];
    int q[16];
    shares_s<S>(mask, O, Ls, D, q);
    const double best = normalise_s<S>(D, q, K, first, step, ms, bk);
    dexp = bk >= 0 ? stage_exps<S>(ms[bk], q) : 0ull;
    if (bk < 0) bk = kNoMs;
    return best;
}

template <class Lds>
__device__ __forceinline__ double group_bias(int s, unsigned mask, int O, int K, int first, int step, const Lds& Ls,
                                             const unsigned long long* __restrict__ ms, int& bk,
                                             unsigned long long& dexp)
{
    switch (s) {
#define ARENA_PX_CASE(n) case n: return group_bias<n>(mask, O, K, first, step, Ls, ms, bk, dexp);
        ARENA_PX_CASE(1) ARENA_PX_CASE(2) ARENA_PX_CASE(3) ARENA_PX_CASE(4)
        ARENA_PX_CASE(5) ARENA_PX_CASE(6) ARENA_PX_CASE(7) ARENA_PX_CASE(8)
        ARENA_PX_CASE(9) ARENA_PX_CASE(10) ARENA_PX_CASE(11) ARENA_PX_CASE(12)
        ARENA_PX_CASE(13) ARENA_PX_CASE(14) ARENA_PX_CASE(15) ARENA_PX_CASE(16)
#undef ARENA_PX_CASE
        default: bk = kNoMs; dexp = 0ull; return kInfP;
    }
}

// Per-replica samples of a stage with D GPUs at tensor degree tp and B
// microbatches, or -1 when dp B does not divide the batch.
__device__ __forceinline__ double replica_batch(int Bg, int D, int tp, int B)
{
    const int dp = D / tp;
    if (Bg % (dp * B)) return -1.0;
    return (double)Bg / (double)(dp * B);
}

__device__ __forceinline__ double stage_mem(double P, double A, int tp, double b, int inflight)
{
    return 4.0 * P / (double)tp + (double)inflight * b * A / (double)tp;
}

// Intra-stage communication per microbatch (C) and gradient all-reduce per
// iteration (AR) of a stage with operator range [lo, hi), D GPUs, degree tp.
template <class Lds>
__device__ __forceinline__ void stage_comm(const Cell c, const Lds& S, int lo, int hi, int D, int tp,
                                           double b, double& C, double& AR)
{
    const double X = ssum(S, kQX, lo, hi), E = ssum(S, kQE, lo, hi), P = ssum(S, kQP, lo, hi);
    double per_sample = 0.0;
    if (tp > 1) per_sample += c.kap * 8.0 * (double)(tp - 1) / (double)tp * X / c.bwi;
    if (D > 1) per_sample += c.kap * E / c.bwe;
    C = b * per_sample;
    const int dp = D / tp;
    const double B_dp = (D <= c.gpn && c.gpn % D == 0) ? c.bwi : c.bwe;
    AR = 0.0;
    if (dp > 1) AR = c.kap * 2.0 * (double)(dp - 1) / (double)dp * (P / (double)tp) / B_dp;
}

// Every stage's tp (least communication B C + AR within memory, ties to the
// smaller tp) and the communication load (Eq. 4); false if a stage has none.
template <class Lds>
__device__ __forceinline__ bool plan_lcomm(const Cell c, const Lds& S, unsigned mask, int s, int B,
                           unsigned long long dexp, unsigned long long& texp, double& lcomm)
{
    double cmax = 0.0, csum = 0.0, arsum = 0.0;
    texp = 0ull;
    int lo = 0;
    for (int j = 0; j < s; ++j) {
        const int hi = stage_end(mask, lo, c.O);
        const int D = 1 << (int)((dexp >> (4 * j)) & 15ull);
        const int inflight = B < s - j ? B : s - j;
        const double P = ssum(S, kQP, lo, hi), A = ssum(S, kQA, lo, hi);
        int best = 0;
        double best_cost = 0.0, bC = 0.0, bAR = 0.0;
        for (int tp = 1; tp <= D; tp *= 2) {
            if (D % tp || c.gpn % tp) continue;
            const double b = replica_batch(c.Bg, D, tp, B);
            if (b < 0.0) continue;
            if (stage_mem(P, A, tp, b, inflight) > c.mem) continue;
            double C, AR;
            stage_comm(c, S, lo, hi, D, tp, b, C, AR);
            const double cost = (double)B * C + AR;
            if (best == 0 || cost < best_cost) {
                best = tp;
                best_cost = cost;
                bC = C;
                bAR = AR;
            }
        }
        if (best == 0) return false;
        texp |= (unsigned long long)(__ffs(best) - 1) << (4 * j);
        if (bC > cmax) cmax = bC;
        csum += bC;
        arsum += bAR;
        lo = hi;
    }
    lcomm = (double)(B - 1) * cmax + csum + arsum;
    return true;
}

// The 1F1B iteration time with per-stage (dp_j, tp_j).
template <class Lds>
__device__ __forceinline__ double price(const Cell c, const Lds& S, unsigned mask, int s, int B, unsigned long long dexp,
                        unsigned long long texp)
{
    const double B_pp = (c.n <= c.gpn) ? c.bwi : c.bwe;
    double fill = 0.0, wmax = 0.0, armax = 0.0;
    int lo = 0;
    for (int j = 0; j < s; ++j) {
        const int hi = stage_end(mask, lo, c.O);
        const int D = 1 << (int)((dexp >> (4 * j)) & 15ull);
        const int tp = 1 << (int)((texp >> (4 * j)) & 15ull);
        const int dp = D / tp;
        const double b = replica_batch(c.Bg, D, tp, B);
        if (b < 0.0) return kInfP;
        const int inflight = B < s - j ? B : s - j;
        const double T = ssum(S, kQT, lo, hi), X = ssum(S, kQX, lo, hi), E = ssum(S, kQE, lo, hi);
        const double P = ssum(S, kQP, lo, hi), A = ssum(S, kQA, lo, hi);
        if (stage_mem(P, A, tp, b, inflight) > c.mem) return kInfP;
        double per_sample = T / ((double)c.Bg * c.speed * (double)tp);
        if (tp > 1) per_sample += c.kap * 8.0 * (double)(tp - 1) / (double)tp * X / c.bwi;
        if (D > 1) per_sample += c.kap * E / c.bwe;
        const double W = b * per_sample;
        double p2p = 0.0;
        if (j < s - 1) {
            const int Dn = 1 << (int)((dexp >> (4 * (j + 1))) & 15ull);
            const int tpn = 1 << (int)((texp >> (4 * (j + 1))) & 15ull);
            const int dpn = Dn / tpn;
            const int dmin = dp < dpn ? dp : dpn;
            p2p = c.kap * 2.0 * ((double)c.Bg / (double)(dmin * B)) * S.oxl[hi - 1] / B_pp;
        }
        const double B_dp = (D <= c.gpn && c.gpn % D == 0) ? c.bwi : c.bwe;
        double AR = 0.0;
        if (dp > 1) AR = c.kap * 2.0 * (double)(dp - 1) / (double)dp * (P / (double)tp) / B_dp;
        fill += W + p2p;
        if (W > wmax) wmax = W;
        if (AR > armax) armax = AR;
        lo = hi;
    }
    return fill + (double)(B - 1) * wmax + armax;
}

// Position of a grouping among those of its degree in lexicographic order of
// cut vectors, as a key: at the first cut where two groupings differ the one
// that starts a stage there comes first.
__device__ __forceinline__ int rank_key(unsigned mask)
{
    return (int)((~__brev(mask)) & 0x7fffffffu);
}

// One degree of the cell, worked on by one wave.
struct PxDegree {
    const unsigned long long* ms;        // its multisets
    int s, K;
    unsigned open;                       // microbatch counts some grouping may fit at
    unsigned ties;                       // counts at which several groupings share the least bias
};

enum PxMode { kPxLimits, kPxSearch, kPxTies };

// Scans the multisets of the first c (<= 64) waiting groupings, one per group
// of tpg lanes, tests every B of `open` for memory and takes the results up:
//   kPxLimits  lowers the limits of the B a grouping fits at;
//   kPxSearch  the least (bias, rank) per B, and which B had ties;
//   kPxTies    among groupings of the least bias: the least communication load.
template <int NB>
__device__ __forceinline__ void px_scan(const Cell& c, ProxyLds<NB>& S, PxWave<NB>& W, PxDegree& d, int mode,
                                        int lane, int cnt, int gpe)
{
    int tpg = 1;
    while (tpg * 2 * cnt <= 64) tpg *= 2;
    const int sub = lane & (tpg - 1);
    const int gi = lane / tpg;
    const bool live = gi < cnt;
    const unsigned mask = live ? (unsigned)W.cand[gi] : 0u;
    double best = kInfP;
    int bk = kNoMs;
    unsigned long long dexp = 0ull;
    if (live) best = group_bias(d.s, mask, c.O, d.K, sub, tpg, S, d.ms, bk, dexp);
    for (int off = 1; off < tpg; off <<= 1) {
        const double ob = __shfl_xor(best, off);
        const int ok = __shfl_xor(bk, off);
        const unsigned long long od = __shfl_xor(dexp, off);
        if (ob < best || (ob == best && ok < bk)) {
            best = ob;
            bk = ok;
            dexp = od;
        }
    }
    unsigned fm = 0u;
    if (live && sub == 0) {
        // memory test per B at the largest admissible tensor degree (replica
        // samples from the per-cell table; dividing by the power-of-two tp is
        // scaling by its exact reciprocal, so the memory is bitwise the plain
        // formula's)
        fm = d.open;
        int lo = 0;
        for (int j = 0; j < d.s && fm; ++j) {
            const int hi = stage_end(mask, lo, c.O);
            const int ej = (int)((dexp >> (4 * j)) & 15ull);
            const int te = ej < gpe ? ej : gpe;                  // log2 of the largest tp
            const double itp = __hiloint2double((1023 - te) << 20, 0);
            const double P = ssum(S, kQP, lo, hi), Aj = ssum(S, kQA, lo, hi);
            const double pmem = 4.0 * P * itp;
            const double* bt = S.bt[ej - te];
            for (unsigned left = fm; left; left &= left - 1u) {
                const int k = __ffs(left) - 1;
                const int B = S.mval[k];
                const double b = bt[k];
                const int inflight = B < d.s - j ? B : d.s - j;
                if (b < 0.0 || pmem + (double)inflight * b * Aj * itp > c.mem) fm &= ~(1u << k);
            }
            lo = hi;
        }
    }
    const int rk = rank_key(mask);
    for (unsigned left = d.open; left; left &= left - 1u) {
        const int k = __ffs(left) - 1;
        const bool fits = ((fm >> k) & 1u) != 0u;
        if (mode == kPxTies) {
            if (!((d.ties >> k) & 1u)) continue;
            double lc = kInfP;
            int li = 0x7fffffff;
            unsigned long long texp;
            if (fits && best == W.bkey[k]) {
                double v;
                if (plan_lcomm(c, S, mask, d.s, S.mval[k], dexp, texp, v) && v <= kInfP) {
                    lc = v;
                    li = rk;
                }
            }
            const double mine = lc;
            const int mi = li;
            wave_argmin(lc, li);
            const double tk = W.tkey[k];
            const int ti = W.tidx[k];
            wave_fence();
            if (li != 0x7fffffff && (lc < tk || (lc == tk && li < ti)) && mine == lc && mi == li) {
                W.tkey[k] = lc;
                W.tidx[k] = li;
                W.bmask[k] = mask;
                W.bdexp[k] = dexp;
            }
            wave_fence();
            continue;
        }
        double kk = fits ? best : kInfP;
        int ii = fits ? rk : 0x7fffffff;
        const double mine = kk;
        const int mi = ii;
        wave_argmin(kk, ii);
        if (!(kk < kInfP)) continue;
        // the limit on the bound: the bias, rounded up
        const float lim = __double2float_ru(kk);
        if (mode == kPxLimits) {
            if (lane == 0) W.lim[k] = fminf(W.lim[k], lim);
        } else {
            const unsigned long long same = __ballot(fits && mine == kk);
            const double bk0 = W.bkey[k];
            const int bi0 = W.bidx[k];
            wave_fence();
            if (kk < bk0) d.ties &= ~(1u << k);
            if (kk == bk0 || (kk <= bk0 && (same & (same - 1ull)))) d.ties |= 1u << k;
            if (kk < bk0 || (kk == bk0 && ii < bi0)) {
                if (mine == kk && mi == ii) {
                    W.bkey[k] = kk;
                    W.bidx[k] = ii;
                    W.bmask[k] = mask;
                    W.bdexp[k] = dexp;
                }
                if (lane == 0) W.lim[k] = fminf(W.lim[k], lim);
            }
        }
        wave_fence();
    }
}

// One pass over the degree.  kPxLimits scans the kLam groupings waiting in
// W.cand; kPxSearch and kPxTies walk every grouping and scan those whose bounds
// leave them a chance at some B, lane l a run of consecutive ranks.  The walk is
// bound by VALU issue: per stage four instructions find the range, two LDS
// reads give its terms and one its GPU needs, then kLam + NB / 2 adds (two
// 16-bit needs per register).
template <int NB>
__device__ __forceinline__ void px_pass(const Cell& c, ProxyLds<NB>& S, PxWave<NB>& W, PxDegree& d, int mode,
                                        int lane, int gpe, float margin)
{
    const int nparts = S.binom[c.O - 1][d.s - 1];
    const int chunk = mode == kPxLimits ? 0 : (nparts + 63) >> 6;
    const int r0 = lane * chunk;
    unsigned mask = chunk > 0 && r0 < nparts ? unrank(r0, c.O, d.s, S) : 0u;
    const unsigned n16 = (unsigned)c.n;
    int cnt = mode == kPxLimits ? kLam : 0;
    for (int it = 0;; ++it) {
        if (it < chunk) {
            bool pass = false;
            if (r0 + it < nparts) {
                if (it) mask = next_grouping(mask, c.O, d.s - 1);
                float lb[kLam];
                unsigned nd[NB / 2];
#pragma unroll
                for (int l = 0; l < kLam; ++l) lb[l] = 0.0f;
#pragma unroll
                for (int k = 0; k < NB / 2; ++k) nd[k] = 0u;
                unsigned rest = (mask | (1u << c.O)) >> 1;     // stage ends past `lo`, the next one first
                int lo = 0;
                for (int j = 0; j < d.s; ++j) {
                    const int z = __ffs(rest);
                    const int hi = lo + z;
                    rest >>= z;
                    const RangeBound& r = S.rb[hi * 16 + lo];
                    const int after = d.s - j - 2;
                    const unsigned* need = (const unsigned*)S.need[r.need + (after > 0 ? after : 0)];
#pragma unroll
                    for (int l = 0; l < kLam; ++l) lb[l] += r.t[l];
#pragma unroll
                    for (int k = 0; k < NB / 2; ++k) nd[k] += need[k];
                    lo = hi;
                }
                float b = lb[0];
#pragma unroll
                for (int l = 1; l < kLam; ++l) b = fmaxf(b, lb[l]);
                b -= margin;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const unsigned need = k & 1 ? nd[k >> 1] >> 16 : nd[k >> 1] & 0xffffu;
                    pass |= need <= n16 && b <= W.lim[k];
                }
            }
            const unsigned long long pm = __ballot(pass);
            if (pm) {
                if (pass)
                    W.cand[cnt + __builtin_amdgcn_mbcnt_hi((unsigned)(pm >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((unsigned)pm, 0u))] =
                        (uint16_t)mask;
                cnt += __popcll(pm);
                wave_fence();
            }
        }
        // full lanes, or the end of the walk
        const bool last = it + 1 >= chunk;
        while (cnt >= 64 || (last && cnt > 0)) {
            const int take = cnt < 64 ? cnt : 64;
            px_scan<NB>(c, S, W, d, mode, lane, take, gpe);
            cnt -= take;
            const uint16_t v = W.cand[64 + lane];
            wave_fence();
            if (lane < cnt) W.cand[lane] = v;
            wave_fence();
        }
        if (last) break;
    }
}

// The degree a cell's tk-th task takes: the middle ones, which have the most
// groupings and multisets, first (1 <= degree <= smax <= O).
__device__ __forceinline__ int degree_of(int tk, int smax, int O)
{
    int mid = (O + 1) / 2 + 1;
    mid = mid < smax ? mid : smax;
    const int up = smax - mid, down = mid - 1;
    const int both = 2 * (up < down ? up : down);
    if (tk <= both) return tk & 1 ? mid + (tk + 1) / 2 : mid - tk / 2;
    return up > down ? mid + (tk - down) : mid - (tk - up);
}

// The bias bound's multipliers, as fractions of n.
__device__ __forceinline__ double lam_of(int l)
{
    const double mag = l < 3 ? 1.0 / 80.0 : (l < 5 ? 1.0 / 32.0 : 1.0 / 12.0);
    return l == 0 ? 0.0 : (l & 1 ? mag : -mag);
}

template <int NB>
__device__ __forceinline__ void proxy_cell(const ProxyArgs& A, ProxyLds<NB>& S, int cell)
{
    // the thread index passes through an empty asm statement once per cell, so
    // nothing derived from it is hoisted out of the cell loop and held in
    // registers across every cell (it would be spilled)
    int tid;
    __asm__ volatile("" : "=v"(tid) : "0"((int)threadIdx.x));
    const int ci = cell % A.n_counts;
    const int g = (cell / A.n_counts) % A.n_types;
    const int jb = cell / (A.n_counts * A.n_types);

    Cell c;
    const int off0 = A.layer_offset[jb];
    c.L = A.layer_offset[jb + 1] - off0;
    c.Bg = A.batch[jb];
    c.O = c.L < A.n_ops ? c.L : A.n_ops;
    c.n = A.counts[ci];
    const TypeDev ty = A.types[g];
    c.speed = ty.speed;
    c.mem = ty.mem;
    c.bwi = ty.bw_intra;
    c.bwe = ty.bw_inter;
    c.gpn = ty.gpn;
    c.kap = (double)A.kappa[g * A.n_counts + ci];
    const double hbm = A.hbm[g];
    const int gpe = __ffs(c.gpn) - 1;             // log2 of the largest power of two dividing the node size
    const int etop = 31 - __clz(c.n);             // largest stage GPU exponent

    // operator sums, loads and shares; binomials; microbatch counts
    if (tid < c.O) {
        const int lo = (int)(((long long)tid * c.L) / c.O), hi = (int)(((long long)(tid + 1) * c.L) / c.O);
        double T = 0.0, X = 0.0, E = 0.0, P = 0.0, Ac = 0.0, M = 0.0;
        for (int l = off0 + lo; l < off0 + hi; ++l) {
            T += (double)A.t[l];
            X += (double)A.x[l];
            E += (double)A.q[l];
            P += (double)A.p[l];
            Ac += (double)A.a[l];
            M += (double)A.p[l] + (double)c.Bg * (double)A.a[l];
        }
        S.oT[tid] = T;
        S.oX[tid] = X;
        S.oE[tid] = E;
        S.oP[tid] = P;
        S.oA[tid] = Ac;
        S.oxl[tid] = (double)A.x[off0 + hi - 1];
        const double flops = A.f_ref * T;
        const double compute = flops / (c.speed * A.f_ref);
        const double memory = M / hbm;
        S.oload[tid] = compute > memory ? compute : memory;
    }
    {
        const int a = tid >> 4, b = tid & 15;
        int v = 0;
        if (b <= a) {          // C(a, b) by the multiplicative formula (exact in 32 bits for a <= 15)
            v = 1;
            for (int k = 1; k <= b; ++k) v = v * (a - b + k) / k;
        }
        S.binom[a][b] = v;
    }
    if (tid < A.n_m) S.mval[tid] = A.m_values[tid];
    if (tid < 11 * A.n_m) {
        const int e = tid / A.n_m, k = tid - e * A.n_m;
        S.bt[e][k] = replica_batch(c.Bg, 1 << e, 1, A.m_values[k]);
    }
    for (int z = tid; z < (kProxyMaxOps + 1) * NB; z += kPxThreads) {
        (&S.gT[0][0])[z] = kInfP;
        (&S.gM[0][0])[z] = 0xffffffffu;
    }
    if (tid == 0) S.next_s = 0;
    __syncthreads();
    if (tid < kProxyMaxOps) {
        double lsum = 0.0;
        for (int i = 0; i < c.O; ++i) lsum += S.oload[i];
        if (tid < c.O) S.od[tid] = (S.oload[tid] / lsum) * (double)c.n;
        if (tid == 0) S.no_load = lsum > 0.0 ? 0 : 1;
    } else if (tid >= 64 && tid < 64 + A.n_m) {
        const int k = tid - 64;
        int em = -1;
        for (int e = 0; e <= etop; ++e)
            if (S.bt[e < gpe ? 0 : e - gpe][k] >= 0.0) em = e;
        S.emax[k] = em;
    }
    __syncthreads();
    for (int task = tid; task < 6 * 256; task += kPxThreads) {
        const int qn = task >> 8, lo = task & 15, hi = ((task >> 4) & 15) + 1;
        const double* v = qn == kQd ? S.od : qn == kQT ? S.oT : qn == kQX ? S.oX : qn == kQE ? S.oE
                         : qn == kQP ? S.oP : S.oA;
        if (lo < hi) {
            double acc = 0.0;
            if (hi <= c.O)
                for (int i = lo; i < hi; ++i) acc += v[i];
            S.ss[qn][tri(lo, hi)] = acc;
        }
    }
    __syncthreads();
    // the ranges' bias-bound terms (rounded down) and their GPU needs
    {
        const int lo = tid & 15, hi = (tid >> 4) + 1;
        if (lo < hi && hi <= c.O) {
            const double D = ssum(S, kQd, lo, hi);
            RangeBound& r = S.rb[hi * 16 + lo];
#pragma unroll
            for (int l = 0; l < kLam; ++l) {
                const double lam = lam_of(l) * (double)c.n;
                double best = kInfP;
                for (int e = 0; e <= etop; ++e) {
                    const double x = __hiloint2double((1023 + e) << 20, 0) - D;
                    best = fmin(best, x * x + lam * x);
                }
                r.t[l] = __double2float_rd(best);
            }
            // ranges ending at h < hi take h max(1, O - h) entries, those ending
            // at hi and starting before lo max(1, O - hi) each
            int base = 0;
            for (int h = 1; h < hi; ++h) base += h * (c.O > h ? c.O - h : 1);
            r.need = base + lo * (c.O > hi ? c.O - hi : 1);
        }
    }
    // a stage over [lo, hi) with `after` stages behind it (none for hi = O,
    // 1 .. O - hi otherwise) fits at B with 2^e GPUs when B divides there and the
    // memory at the largest tensor degree is within the GPU's (the test of the
    // scan, term by term)
    for (int task = tid; task < kNeeds; task += kPxThreads) {
        int t = task, hi = 1;
        while (hi < c.O && t >= hi * (c.O - hi)) {
            t -= hi * (c.O - hi);
            ++hi;
        }
        const int wdt = c.O > hi ? c.O - hi : 1;
        const int lo = t / wdt, after = t - lo * wdt + (hi < c.O ? 1 : 0);
        if (lo < hi) {
            const double P = ssum(S, kQP, lo, hi), Aj = ssum(S, kQA, lo, hi);
            for (int k = 0; k < NB; ++k) {
                unsigned v = kNoFit;
                if (k < A.n_m) {
                    const int B = S.mval[k];
                    const int inflight = B < after + 1 ? B : after + 1;
                    for (int e = S.emax[k]; e >= 0; --e) {
                        const int te = e < gpe ? e : gpe;
                        const double itp = __hiloint2double((1023 - te) << 20, 0);
                        const double b = S.bt[e - te][k];
                        if (!(b < 0.0) && !(4.0 * P * itp + (double)inflight * b * Aj * itp > c.mem)) v = 1u << e;
                    }
                }
                S.need[task][k] = (uint16_t)v;
            }
        }
    }
    __syncthreads();
    const int smax = S.no_load ? 0 : (c.O < c.n ? c.O : c.n);
    // per multiplier and stage count: the grouping of least bound (its last
    // stage's start by prefix end), 32 lanes of one wave per multiplier
    if (smax > 0) {
        const int l = tid >> 5, i = tid & 31;
        if (l < kLam) {
            if (i <= c.O) S.path[l][0][i] = i == 0 ? 0.0f : __builtin_huge_valf();
            for (int t = 1; t <= smax; ++t) {
                wave_fence();
                float best = __builtin_huge_valf();
                int from = 0;
                if (i >= t && i <= c.O)
                    for (int lo = t - 1; lo < i; ++lo) {
                        const float v = S.path[l][(t - 1) & 1][lo] + S.rb[i * 16 + lo].t[l];
                        if (v < best) {
                            best = v;
                            from = lo;
                        }
                    }
                if (i <= c.O) {
                    S.path[l][t & 1][i] = best;
                    S.from[l][t][i] = (uint8_t)from;
                }
            }
        }
    }
    __syncthreads();

    // the waves take the degrees, those with the most groupings first
    const int lane = tid & 63;
    PxWave<NB>& W = S.w[__builtin_amdgcn_readfirstlane(tid >> 6)];
    const float margin = (float)c.n * (float)c.n * 1e-6f;
    for (;;) {
        int tk = 0;
        if (lane == 0) tk = atomicAdd(&S.next_s, 1);
        tk = __builtin_amdgcn_readfirstlane(tk);
        if (tk >= smax) break;
        // middle degrees first: (O + 1) / 2, then the nearest on either side
        const int s = degree_of(tk, smax, c.O);
        const int mo = A.mset_off[ci * 17 + s];
        PxDegree d;
        d.s = s;
        d.ms = A.msets + mo;
        d.K = A.mset_off[ci * 17 + s + 1] - mo;
        if (d.K <= 0) continue;                    // no s powers of two sum to n
        d.open = 0u;
        d.ties = 0u;
        for (int k = 0; k < A.n_m; ++k)
            if (S.emax[k] >= 0 && (s << S.emax[k]) >= c.n) d.open |= 1u << k;
        if (!d.open) continue;                     // no count divides with stages small enough
        if (lane < NB) {
            W.lim[lane] = ((d.open >> lane) & 1u) ? __builtin_huge_valf() : -__builtin_huge_valf();
            W.bkey[lane] = kInfP;
            W.bidx[lane] = 0x7fffffff;
            W.bmask[lane] = 0xffffffffu;
        }
        wave_fence();
        if (lane < kLam) {
            unsigned m = 0u;
            int i = c.O;
            for (int t = s; t > 1; --t) {
                i = S.from[lane][t][i];
                m |= 1u << i;
            }
            W.cand[lane] = (uint16_t)m;
        }
        wave_fence();
        for (int mode = kPxLimits; mode <= kPxTies; ++mode) {
            if (mode == kPxTies) {
                // several groupings of the least bias: the least communication load decides
                if (!d.ties) break;
                if (lane < NB) {
                    W.tkey[lane] = kInfP;
                    W.tidx[lane] = 0x7fffffff;
                    if (!((d.ties >> lane) & 1u)) W.lim[lane] = -__builtin_huge_valf();
                    else W.bmask[lane] = 0xffffffffu;
                }
                wave_fence();
            }
            px_pass<NB>(c, S, W, d, mode, lane, gpe, margin);
        }
        if (lane < NB) {
            S.gM[s][lane] = W.bmask[lane];
            S.gD[s][lane] = W.bdexp[lane];
        }
        wave_fence();
    }
    __syncthreads();

    // each grid's proxy at each B priced by its own thread
    for (int z = tid; z < smax * NB; z += kPxThreads) {
        const int s = z / NB + 1, k = z & (NB - 1);
        const unsigned mask = S.gM[s][k];
        if (mask == 0xffffffffu) continue;
        const unsigned long long dexp = S.gD[s][k];
        const int B = S.mval[k];
        unsigned long long texp;
        double lc;
        if (plan_lcomm(c, S, mask, s, B, dexp, texp, lc)) {
            S.gT[s][k] = price(c, S, mask, s, B, dexp, texp);
            S.gP[s][k] = texp;
        }
    }
    __syncthreads();

    // the fastest grid; ties within the window: fewer stages, then fewer microbatches
    if (tid < 64) {
        double tl = kInfP;
        int dummy = 0;
        for (int z = tid; z < smax * NB; z += 64) tl = fmin(tl, (&S.gT[1][0])[z]);
        wave_argmin(tl, dummy);
        unsigned long long w0 = 0ull, w1 = 0ull, w2 = 0ull;
        float tout = __builtin_huge_valf(), thout = 0.0f;
        if (tl < kInfP) {
            const double lim = tl * (1.0 + A.tie_eps);
            double key = kInfP;                        // s * 128 + B: exact
            int at = 0x7fffffff;
            for (int z = tid; z < smax * NB; z += 64)
                if ((&S.gT[1][0])[z] <= lim) {
                    const double v = (double)((z / NB + 1) * 128 + S.mval[z & (NB - 1)]);
                    if (v < key) {
                        key = v;
                        at = z;
                    }
                }
            wave_argmin(key, at);
            const int bs = at / NB + 1, bk = at & (NB - 1);
            const double T = S.gT[bs][bk];
            tout = (float)T;
            thout = (float)((double)c.Bg / T);
            w0 = (unsigned long long)(S.gM[bs][bk] >> 1) | ((unsigned long long)bs << 16) |
                 ((unsigned long long)S.mval[bk] << 24) | (1ull << 31);
            w1 = S.gD[bs][bk];
            w2 = S.gP[bs][bk];
        }
        if (tid == 0) {
            A.t_iter[cell] = tout;
            A.thr[cell] = thout;
            A.plan[(size_t)cell * kProxyPlanWords + 0] = w0;
            A.plan[(size_t)cell * kProxyPlanWords + 1] = w1;
            A.plan[(size_t)cell * kProxyPlanWords + 2] = w2;
        }
    }
}

// Resident blocks take cells from a device queue until none is left: a
// dispatcher that places block b on XCD b % 8 in order would otherwise leave
// CUs idle while a block waits for room on its XCD.  NB: microbatch counts
// the LDS tables hold (8, or 16 when the plan space lists more than 8).
template <int NB>
__global__ __launch_bounds__(kPxThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void proxy_kernel(ProxyArgs A,
                                                                                                    int n_cells)
{
    __shared__ ProxyLds<NB> S;
    __shared__ int slot;
    for (;;) {
        if (threadIdx.x == 0) {
            const unsigned long long q = atomicAdd(A.queue, 1ull);
            slot = q < (unsigned long long)n_cells ? (int)q : -1;
        }
        __syncthreads();
        const int cell = slot;
        __syncthreads();
        if (cell < 0) break;
        proxy_cell<NB>(A, S, cell);
        __syncthreads();          // the next cell reuses the LDS
    }
}

template <int NB>
hipError_t launch(const ProxyArgs& args, long long cells, hipStream_t stream)
{
    int per_cu = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, proxy_kernel<NB>, kPxThreads, 0);
    if (e != hipSuccess) return e;
    const long long resident = (long long)(args.n_cus > 0 ? args.n_cus : 1) * (per_cu > 0 ? per_cu : 1);
    const unsigned blocks = (unsigned)(cells < resident ? cells : resident);
    hipLaunchKernelGGL((proxy_kernel<NB>), dim3(blocks), dim3(kPxThreads), 0, stream, args, (int)cells);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_proxy(const ProxyArgs& args, hipStream_t stream)
{
    const long long cells = (long long)args.n_jobs * args.n_types * args.n_counts;
    if (cells <= 0) return hipSuccess;
    return args.n_m <= 8 ? launch<8>(args, cells, stream) : launch<16>(args, cells, stream);
}

}  // namespace arena
