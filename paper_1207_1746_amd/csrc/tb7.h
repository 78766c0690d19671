// Temporal blocking for the 7-point weighted Jacobi sweep and for red-black
// relaxation: k sweeps (or k colour passes) per pass over HBM (wide ghost
// zones).
//
// A block owns a working region of 64 columns x 32 rows and marches it through
// z; a group of lanes holds two rows of it.  FP64 Jacobi: the group is a wave,
// each lane one column; the x neighbours are a wave-wide DPP shift away.
// Otherwise ("pairs") the group is half a wave, each lane two adjacent columns
// (an even x and the next); the x neighbours inside a pair are in the lane, the
// others a shift away (a shift across the halves only fills ghost columns): half
// the shifts, but twice the registers per lane, which in FP64 leave Jacobi two
// waves per SIMD (1.5 us a step of 4 levels; four rows of one column 1.47; 16
// waves of two rows 1.37).  The y neighbour inside the two rows is in the lane,
// and only the row of the next group up or down goes through LDS.  The region is
// the output tile grown by k cells on every side (pairs: columns by k rounded up
// to even): level t (the grid after t sweeps) is needed on the tile grown by
// k - t cells, so after k levels the inner points are exact and are the only
// ones written.
//
// At march step s the block holds input plane s (level 0) and computes, for
// t = 1..k, level t at plane s - t: its z neighbours are the thread's own
// level t-1 values at planes s-t-1, s-t (registers) and s-t+1 (computed
// earlier in the same step); every lane stages its level t-1 rows for the
// half-waves above and below at the start of the step.  Every input plane is
// read from HBM once per k sweeps.  Level t is first needed at plane
// z0 - (k - t), which it reaches in step z0 - k + 2t; earlier steps leave it
// out, so a chunk of cz planes costs k cz + k (k - 1) level steps.  Steps are
// written out in groups of the period of the register windows, which makes
// their shifts renamings.
//
// Outside the domain, levels take the Dirichlet value; under the periodic
// rule the loads wrap and the computed values are the periodic extension.
// The per-point arithmetic is the plain sweep's operator, so the result is
// the one k separate sweeps produce, bit for bit.
//
// Red-black levels (RB): level t is one colour pass of level t-1, colour
// (c0 + t - 1) mod 2 with c0 = p[3], using the in-place pass's operator.  An
// in-place colour pass reads only points of the other colour, which it does
// not change, so k levels are k in-place passes, bit for bit, and a pass of 2m
// levels is m full red-black sweeps.  Here a level updates its colour in place
// in the registers of its plane: of a lane's pair in a row exactly one point
// has the colour, the same one at every level of a step, and it alternates
// from row to row and from step to step; so the march starts on a step of
// fixed parity and the point is known at compile time.  Half the points of a
// level are computed, staged and shifted.
//
// Bound: the issue of vector instructions (FP32 and FP64 alike 4 cycles per
// wave; per block and step of 4 levels 1600 in FP32, 2300 in FP64, 1070
// red-black, 45-70% of the time of a step) and the LDS rows, which the barrier
// keeps from overlapping much.  Figures beside tb_pick_chunk.
#pragma once

#include <algorithm>
#include <type_traits>

#include "ops.h"

namespace gk {

struct TBArgs {
    Geo g;
    const void* u;    // input grid (level 0)
    const void* f;    // right-hand side (may be null)
    void* out;        // level k
    double p[8];      // operator parameters of the plain sweep (RB: p[3] = first colour)
    int k;            // sweeps (colour passes) per pass, 1..TB_KMAX (the
                      // kernels take it as the template parameter K)
    int ntx, nty, ncz, cz;
    int operand;
    RedArgs ra;
};

constexpr int TB_KMAX = 4;  // most levels of a pass
constexpr int TB_COLS = 64, TB_ROWS = 32;

// Whether a kernel's lanes hold pairs of columns, and its waves.
constexpr bool tb_pairs(bool f64, bool rb) { return rb || !f64; }
constexpr int tb_waves(bool pairs) { return pairs ? 8 : 16; }

// Output tile of a k-level block (pairs: ghost columns are whole pairs).
__host__ __device__ constexpr int tb_ghost_x(int k, bool pairs) { return pairs ? (k + 1) & ~1 : k; }
__host__ __device__ constexpr int tb_out_x(int k, bool pairs) { return TB_COLS - 2 * tb_ghost_x(k, pairs); }
__host__ __device__ constexpr int tb_out_y(int k) { return TB_ROWS - 2 * k; }

// Waves per SIMD that a K-level kernel is compiled for: two blocks per CU
// (8 waves: 128 VGPRs) where the LDS rows of two fit the 160 KB and the windows
// the registers, else one (8 waves: 256, 16: 128).  (Spilled windows are worse than one block less:
// their reloads wait for every load in flight.  Red-black, FP64, K = 4, 192^3:
// 35 us per pass with 181 VGPRs, 48 with 128 and 40 spilled.)
template <class T, int K, bool RB>
constexpr int tb_waves_per_eu() {
    if (!tb_pairs(sizeof(T) == 8, RB)) return 4;
    return sizeof(T) == 4 || K == 1 ? 4 : 2;
}

// z chunk of a launch whose chunk no one has set: the blocks of all chunks
// share 256 CUs, and a block's time is its planes plus its warm-up, which
// counts as `lead` planes (FP64 6.5, FP32 5; red-black 11, whose steps are
// shorter but load as much).  One block per CU and round; where two fit
// (FP32), a round of two takes 1.6 times one.  tiles(cz) is the number of
// blocks with chunks of cz planes.  Measured per pass of 4 levels with a
// right-hand side, us at the chunk taken (before: 16-wave blocks, one column
// per lane, power-of-two chunks):
//           Jacobi FP64      Jacobi FP32      red-black FP64
//    32^3   13.8 -> 10.6     10.7 ->  7.8     14.4 ->  7.7
//    96^3   21.4 -> 15.6     19.2 -> 11.1     22.6 -> 11.7
//   192^3   64.5 -> 45       42.6 -> 29.0     71.4 -> 35
//   256^3   117  -> 113      69.3 -> 57       139  -> 106
template <class Tiles>
inline int tb_pick_chunk(int nz, int64_t max_blocks, bool rb, bool f64, int k, Tiles&& tiles) {
    const double lead = (rb ? 11.0 : f64 ? 6.5 : 5.0) * k / TB_KMAX;
    int best = 0;
    double best_cost = 0.0;
    for (int cz = 1; cz <= std::min(nz, 128); ++cz) {
        const int64_t n = tiles(cz);
        if (n > max_blocks) continue;
        const double rounds = f64 ? (double)((n + 255) / 256) : 1.6 * (double)(n / 512) + (n % 512 == 0 ? 0.0 : n % 512 <= 256 ? 1.0 : 1.6);
        const double cost = rounds * (cz + lead);
        if (best == 0 || cost <= best_cost) {
            best = cz;
            best_cost = cost;
        }
    }
    return best;
}

// Blocks of a pass in chunks of cz planes.
inline int64_t tb_blocks(const Geo& g, int k, int cz, bool pairs) {
    const int ox = tb_out_x(k, pairs), oy = tb_out_y(k);
    return (int64_t)((g.nx + ox - 1) / ox) * ((g.ny + oy - 1) / oy) * ((g.nz + cz - 1) / cz);
}

// z chunk of a launch: the one set for its extents, else the one that balances
// the blocks over the chip.  A fused reduction takes a partial per block: the
// choice never needs more of them than the nominal chunk does or 2048.
inline int tb_launch_chunk(const Geo& g, int k, int nominal, bool set, bool rb, bool f64) {
    if (set) return nominal;
    const bool pairs = tb_pairs(f64, rb);
    const int cz = tb_pick_chunk(g.nz, std::max<int64_t>(tb_blocks(g, k, nominal, pairs), 2048), rb, f64, k,
                                 [&](int q) { return tb_blocks(g, k, q, pairs); });
    return cz ? cz : nominal;
}

// z chunks of grids that share one launch (a batch): one chunk for all, chosen
// like a single launch's.  A grid's rule, if it has one, is the least chunk while
// the rules' chunks make at least 512 tiles (two blocks per CU), and the most
// after that (the tail of a stream, which shorter chunks spread over the CUs).
// On a full chip a longer balanced chunk beats the rule's: 64 grids of 80^3,
// FP32, ms a step of 64 sweeps: 3.25 balanced; held at 4, 8, 16 and 32 planes
// 5.56, 4.47, 3.76 and 3.41.
struct TBShare {
    int cols, nz;  // tiles of a plane, planes
    int rule;      // rule's chunk (0: none)
    int cz;        // out
};
inline void tb_share_chunks(TBShare* s, int n, bool rb, bool f64, int k) {
    auto tiles = [&](auto&& chunk) {
        int64_t t = 0;
        for (int i = 0; i < n; ++i) t += (int64_t)s[i].cols * ((s[i].nz + chunk(s[i]) - 1) / chunk(s[i]));
        return t;
    };
    auto within = [](const TBShare& g, int cz) { return std::max(1, std::min(cz, g.nz)); };
    int nzmax = 1;
    for (int i = 0; i < n; ++i) nzmax = std::max(nzmax, s[i].nz);
    const bool full = tiles([&](const TBShare& g) { return within(g, g.rule > 0 ? g.rule : 16); }) >= 512;
    auto most = [&](const TBShare& g, int cz) { return within(g, !full && g.rule > 0 ? std::min(g.rule, cz) : cz); };
    const int cz = tb_pick_chunk(nzmax, INT32_MAX, rb, f64, k, [&](int q) {
        return tiles([&](const TBShare& g) { return most(g, q); });
    });
    for (int i = 0; i < n; ++i) s[i].cz = full ? within(s[i], std::max(s[i].rule, cz)) : most(s[i], cz);
}

// The count that a fused reduction into fixed scratch of `limit` partials is
// held against: nominal chunks of tiles with exactly k ghost columns.  A launch
// whose count is within the limit has at most 2 * limit blocks (and 2048): a
// pair layout's tiles put out two columns less at odd k, 56 instead of 58 or 60
// instead of 62, so a row takes at most twice as many.
inline int64_t tb_nominal_blocks(const Geo& g, int k, int nominal) { return tb_blocks(g, k, nominal, false); }

// Value of the lane below (lane - 1) or above (lane + 1) in the wave, by
// wave-wide DPP shifts (wave_shr:1 / wave_shl:1); lanes without a source get 0.
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
constexpr int DPP_WAVE_SHR1 = 0x138, DPP_WAVE_SHL1 = 0x130;

// a * b rounded once, never fused with a later sum
template <class T>
__device__ __forceinline__ T exact_mul(T a, T b) {
#pragma clang fp contract(off)
    return a * b;
}

// this lane's bit of a wave mask
__device__ __forceinline__ bool lane_of(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// (((((xp + xm) + yp) + ym) + zp) + zm), the order of the plain sweeps
template <class T>
__device__ __forceinline__ T near_sum(T xp, T xm, T yp, T ym, T zp, T zm) {
#pragma clang fp contract(off)
    T s = xp + xm;
    s = s + yp;
    s = s + ym;
    s = s + zp;
    return s + zm;
}

// What a block keeps of its tile while it marches (see tb7_tile).
// SPLIT: the wrap of an odd row length splits pairs (periodic rule).
template <class T, bool HAS_F, int K, bool RED, bool RB, bool SPLIT>
struct TBMarch {
    static constexpr bool PAIRS = tb_pairs(sizeof(T) == 8, RB);
    // rows and columns of a lane, lanes of a group and of a block
    static constexpr int R = 2, NV = PAIRS ? 2 : 1, GROUP = PAIRS ? 32 : 64, NL = 64 * tb_waves(PAIRS);
    // values staged per row: red-black only those of one colour
    static constexpr int NE = RB ? 1 : NV;
    // period of the register windows, in steps: even (the parity of the LDS
    // copies, of the two-plane windows and of the red-black points), and at
    // least the planes a window spans, K + 4 with two of them being loaded
    static constexpr int PER = (K + 5) / 2 * 2;
    // planes requested ahead of the one being computed (one where two and the
    // reduction do not fit the registers of 16 waves)
    static constexpr int LA = !PAIRS && RED ? 1 : 2;
    static constexpr int NH = RB ? PER : 2 * K;  // planes held
    // Without a fused reduction the right-hand side is held as h^2 f, formed
    // once per loaded value instead of once per level, and the operator is
    // given h^2 = 1: the product it forms is then exact, so every level
    // rounds as the plain sweep does.  (A fused residual needs f itself.)
    static constexpr bool PRE_H2 = HAS_F && !RED;
    using Lds = T[2][K][R][NE][NL];

    const TBArgs& a;
    Lds& lds;
    double& acc;
    const T* ub;
    const T* fb;
    T* ob;
    int z0, z1, s_end;
    int idx, dn, up;             // LDS slots of this lane and of the same columns in the rows below / above
    uint32_t roff[R];            // byte offset of this lane's columns in a plane
    int d1;                      // SPLIT: byte distance to the pair's second column
    bool whole;                  // rows are whole pairs
    bool dir;                    // Dirichlet rule
    // lane masks (scalar registers): inside the grid in x and y (periodic
    // rule: any); the pair's points are written
    uint64_t keep[R][NV], out[R][NV];
    T bcv, omega, h2;
    // RB: plane p in slot p mod PER (by the step's phase); else level L's two
    // newest planes in 2 L, 2 L + 1, and nu the two planes being loaded
    T u[NH][R][NV];
    T nu[2][R][NV];
    T fq[PER][R][NV];            // h^2 f (or f) of plane p in slot p mod PER

    // Plane offsets (elements): the input's next plane is zn, kept wrapped
    // under the periodic rule and clamped at use under Dirichlet's; the
    // right-hand side follows one plane behind, at foff.
    int zn;
    int64_t foff;
    __device__ __forceinline__ int64_t next_off() {
        const int nz = a.g.nz;
        const int zz = dir ? min(max(zn, 0), nz - 1) : zn;
        ++zn;
        if (!dir && zn == nz) zn = 0;
        return (int64_t)zz * a.g.pz;
    }
    __device__ __forceinline__ void load_row(const char* pl, int i, T (&v)[NV]) const {
        if constexpr (SPLIT) {
            v[0] = *reinterpret_cast<const T*>(pl + roff[i]);
            v[NV - 1] = *reinterpret_cast<const T*>(pl + (uint32_t)((int)roff[i] + d1));
        } else {
            const Vec<T, NV> q = *reinterpret_cast<const Vec<T, NV>*>(pl + roff[i]);
#pragma unroll
            for (int e = 0; e < NV; ++e) v[e] = q.v[e];
        }
    }
    // Request the next plane of the input (PH: the phase of its step) and the
    // plane before it of the right-hand side.
    template <int PH, bool F>
    __device__ __forceinline__ void load_next() {
        const int64_t off = next_off();
        const char* pu = reinterpret_cast<const char*>(ub + off);
#pragma unroll
        for (int i = 0; i < R; ++i) load_row(pu, i, RB ? u[RB ? PH % PER : 0][i] : nu[PH & 1][i]);
        if (HAS_F && F) {
            const char* pf = reinterpret_cast<const char*>(fb + foff);
#pragma unroll
            for (int i = 0; i < R; ++i) load_row(pf, i, fq[(PH + PER - 1) % PER][i]);
        }
        foff = off;
    }

    // Step s; PH = step index mod PER.  WARM: a step of the first group, whose
    // levels are not all needed.
    template <int PH, bool WARM>
    __device__ __forceinline__ void step(const int s) {
        // slot of plane s - j
        auto slot = [](int j) constexpr { return ((PH - j) % PER + PER) % PER; };
        constexpr int par = PH & 1;
        // plane s arrives: boundary values, and h^2 f of plane s - 1
        T cur[R][NV];  // Jacobi: level 0 of plane s
        {
            const bool z_in = !dir || ((unsigned)s < (unsigned)a.g.nz);
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int e = 0; e < NV; ++e) {
                    T& v = RB ? u[RB ? slot(0) : 0][i][e] : nu[par][i][e];
                    cur[i][e] = v = lane_of(z_in ? keep[i][e] : 0) ? v : bcv;
                    if (PRE_H2) fq[slot(1)][i][e] = exact_mul(h2, fq[slot(1)][i][e]);
                }
        }
        // request plane s + LA of the input, the one before of the right-hand side
        // (redefined each step: the 64-bit form of the offsets is then not kept
        // in registers, and accesses take a scalar base and a 32-bit offset)
#pragma unroll
        for (int i = 0; i < R; ++i) asm volatile("" : "+v"(roff[i]));
        load_next<PH + LA, true>();
        const int lv = WARM ? (s - (z0 - K)) >> 1 : K;  // levels needed so far
        // stage level t-1 of plane s - t (RB: the points this step does not update)
        auto& lb = lds[par];
#pragma unroll
        for (int t = 1; t <= K; ++t)
            if (!WARM || t <= lv) {
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int e = 0; e < NE; ++e)  // (a pair in two rows of the copy: no bank conflicts)
                        lb[t - 1][i][e][idx] =
                            RB ? u[RB ? slot(t) : 0][i][NV - 1 - ((i + PH) & 1)] : u[RB ? 0 : 2 * (t - 1) + 1][i][e];
            }
        __syncthreads();
        const T inv = T(1) / T(6), h2l = PRE_H2 ? T(1) : h2;
#pragma unroll
        for (int t = 1; t <= K; ++t) {
            const int zp = s - t;
            const bool z_in = !dir || ((unsigned)zp < (unsigned)a.g.nz);
            T c[R][NV], val[R][NV];
            double rv[R][NV];
            if (!RB) {
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int e = 0; e < NV; ++e) val[i][e] = c[i][e] = u[RB ? 0 : 2 * (t - 1) + 1][i][e];
            }
            if (!WARM || t <= lv) {
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int e = 0; e < NV; ++e) {
                        if (RB && e != ((i + PH) & 1)) continue;
                        T old, sum;
                        if (RB) {
                            auto& q = u[RB ? slot(t) : 0];
                            const T xs = q[i][NV - 1 - e];
                            const T xm = e == 0 ? lane_shift<DPP_WAVE_SHR1>(xs) : xs;
                            const T xp = e == 0 ? xs : lane_shift<DPP_WAVE_SHL1>(xs);
                            const T ym = i > 0 ? q[0][e] : lb[t - 1][1][0][dn];
                            const T yp = i > 0 ? lb[t - 1][0][0][up] : q[1][e];
                            sum = near_sum(xp, xm, yp, ym, u[RB ? slot(t - 1) : 0][i][e], u[RB ? slot(t + 1) : 0][i][e]);
                            old = q[i][e];
                        } else {
                            const T xm = e == 0 ? lane_shift<DPP_WAVE_SHR1>(c[i][NV - 1]) : c[i][0];
                            const T xp = e == NV - 1 ? lane_shift<DPP_WAVE_SHL1>(c[i][0]) : c[i][NV - 1];
                            const T ym = i > 0 ? c[0][e] : lb[t - 1][1][RB ? 0 : e][dn];
                            const T yp = i > 0 ? lb[t - 1][0][RB ? 0 : e][up] : c[1][e];
                            sum = near_sum(xp, xm, yp, ym, cur[i][e], u[RB ? 0 : 2 * (t - 1)][i][e]);
                            old = c[i][e];
                        }
                        const T fv = HAS_F ? fq[slot(t)][i][e] : T(0);
                        const T un = relax_point(old, sum, fv, omega, h2l, inv);
                        if (RED && t == K) {
#pragma clang fp contract(off)
                            if (a.operand == RV_RESIDUAL)
                                rv[i][e] = (double)(fv - (sum - T(6) * old) * (T)a.p[2]);
                            else
                                rv[i][e] = a.operand == RV_UPDATE ? (double)(un - old) : (double)un;
                        }
                        if (RB)
                            u[RB ? slot(t) : 0][i][e] = lane_of(z_in ? keep[i][e] : 0) ? un : old;
                        else
                            val[i][e] = lane_of(z_in ? keep[i][e] : 0) ? un : bcv;
                    }
            }
            if (t == K && zp >= z0) {  // (zp < z1 always)
                char* po = reinterpret_cast<char*>(ob + (int64_t)zp * a.g.pz);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    Vec<T, NV> q;
#pragma unroll
                    for (int e = 0; e < NV; ++e) {
                        q.v[e] = RB ? u[RB ? slot(t) : 0][i][e] : val[i][e];
                        // keep the computation out of the branches below
                        asm volatile("" : "+v"(q.v[e]));
                    }
                    if (!PAIRS || whole) {
                        if (lane_of(out[i][0])) *reinterpret_cast<Vec<T, NV>*>(po + roff[i]) = q;
                    } else {
#pragma unroll
                        for (int e = 0; e < NV; ++e)
                            if (lane_of(out[i][e])) *reinterpret_cast<T*>(po + roff[i] + e * sizeof(T)) = q.v[e];
                    }
                    if (RED) {
#pragma unroll
                        for (int e = 0; e < NV; ++e) {
                            if (RB && e != ((i + PH) & 1)) continue;
                            if (lane_of(out[i][e])) acc = red_acc(acc, rv[i][e], a.ra.op);
                        }
                    }
                }
            }
            if (!RB) {
                // shift the level t-1 window; the new level t value is the
                // z + 1 neighbour of level t + 1 in this step
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int e = 0; e < NV; ++e) {
                        u[RB ? 0 : 2 * (t - 1)][i][e] = c[i][e];
                        u[RB ? 0 : 2 * (t - 1) + 1][i][e] = cur[i][e];
                        cur[i][e] = val[i][e];
                    }
            }
        }
    }

    // Steps PH .. PER - 1 of a group from step s on; true once s_end is reached.
    template <int PH, bool WARM>
    __device__ __forceinline__ bool group(int& s) {
        step<PH, WARM>(s);
        if (++s >= s_end) return true;
        if constexpr (PH + 1 < PER) return group<PH + 1, WARM>(s);
        return false;
    }
};

// One output tile (index `tile` of a.ntx x a.nty x a.ncz): K levels over its
// z chunk; with RED, the fused operand of level K is added to acc.  Every
// thread of the block calls it.
template <class T, bool HAS_F, int K, bool RED, bool RB, bool SPLIT = false>
__device__ __forceinline__ void tb7_tile(const TBArgs& a, const int tile, double& acc) {
    using M = TBMarch<T, HAS_F, K, RED, RB, SPLIT>;
    // the rows every lane stages per level, in two copies alternating by
    // step: a step's staging writes the copy the previous step did not read,
    // so one barrier per step suffices
    __shared__ typename M::Lds lds;
    constexpr int R = M::R, NV = M::NV, G = tb_ghost_x(K, M::PAIRS), GROUP = M::GROUP;
    const Geo& g = a.g;
    M m{a, lds, acc};
    m.ub = static_cast<const T*>(a.u);
    m.fb = static_cast<const T*>(a.f);
    m.ob = static_cast<T*>(a.out);
    const int xt = tile % a.ntx, rest = tile / a.ntx, yt = rest % a.nty, zc = rest / a.nty;
    m.z0 = zc * a.cz;
    m.z1 = min(m.z0 + a.cz, g.nz);
    m.dir = g.bc == BC_DIRICHLET;
    m.bcv = (T)g.bcv;
    m.omega = (T)a.p[0];
    m.h2 = (T)a.p[1];
    const int rg = M::PAIRS ? threadIdx.x / GROUP : __builtin_amdgcn_readfirstlane(threadIdx.x / GROUP);
    const int l = threadIdx.x % GROUP;
    m.idx = threadIdx.x;
    // (the region's edge rows read their own: they lie in the ghost zone)
    m.dn = rg > 0 ? m.idx - GROUP : m.idx;
    m.up = rg < TB_ROWS / R - 1 ? m.idx + GROUP : m.idx;
    const int x = xt * tb_out_x(K, M::PAIRS) - G + NV * l;  // pairs: even
    const int rule = m.dir ? BC_CLAMP : g.bc;
    m.whole = (g.nx & 1) == 0;
    // a pair inside the grid, or starting at its last column (the second point
    // is then the row's padding, never used), is contiguous; columns outside
    // under the Dirichlet rule are read anywhere in the row and replaced
    const int xs = (unsigned)x < (unsigned)g.nx ? x : (m.dir ? (x < 0 ? 0 : (g.nx - 1) & -NV) : wrap_idx(x, g.nx, rule));
    m.d1 = SPLIT ? (wrap_idx(x + 1, g.nx, rule) - xs) * (int)sizeof(T) : 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = rg * R + i, y = yt * tb_out_y(K) - K + row;
        const bool y_in = (unsigned)y < (unsigned)g.ny;
        const int ys = y_in ? y : wrap_idx(y, g.ny, rule);
        m.roff[i] = (uint32_t)(((int64_t)ys * g.py + xs) * (int64_t)sizeof(T));
        const bool out = row >= K && row < TB_ROWS - K && y_in && l >= G / NV && l < (TB_COLS - G) / NV;
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const bool x_in = (unsigned)(x + e) < (unsigned)g.nx;
            m.keep[i][e] = __ballot(!m.dir || (y_in && x_in));
            m.out[i][e] = __ballot(out && x_in);
        }
    }
#pragma unroll
    for (int j = 0; j < M::NH; ++j)
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int e = 0; e < NV; ++e) m.u[j][i][e] = T(0);
#pragma unroll
    for (int j = 0; j < M::PER; ++j)
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int e = 0; e < NV; ++e) m.fq[j][i][e] = T(0);

    // Level K is first needed at plane z0 in step z0 + K; steps from z0 - K on
    // fill the windows.  RB: the point (x + e, y, s - t) of row i has colour
    // (e + i + K + s - t) mod 2 (x is even, y = i + K mod 2) and level t updates
    // colour (c0 + t - 1) mod 2, so the point of step s is
    // e = (i + K + s + c0 + 1) mod 2: start where that is i mod 2.
    int s = m.z0 - K;
    if (RB && ((s + K + (int)a.p[3] + 1) & 1)) --s;
    m.s_end = m.z1 + K;
    m.zn = m.dir ? s : wrap_idx(s, g.nz, BC_PERIODIC);
    m.template load_next<0, false>();
    if constexpr (M::LA == 2) m.template load_next<1, true>();
    // (a group is at least 2 K steps)
    if (m.template group<0, true>(s)) return;
    while (!m.template group<0, false>(s)) {
    }
}

template <class T, bool HAS_F, int K, bool RED, bool RB, bool SPLIT>
__global__ __launch_bounds__(64 * tb_waves(tb_pairs(sizeof(T) == 8, RB)), (tb_waves_per_eu<T, K, RB>())) void tb7_sweep(TBArgs a) {
    const int tile = xcd_remap(blockIdx.x, a.ntx * a.nty * a.ncz);
    double acc = 0.0;
    tb7_tile<T, HAS_F, K, RED, RB, SPLIT>(a, tile, acc);
    if (RED) block_reduce(acc, a.ra, tile);
}

}  // namespace gk
