// The diamond iteration space (Section 3: cells (i-1, j) and (i, j-1) are
// processed before cell (i, j); 2D, every layer independent).  The operators:
//   RECUR: out(i, j) = a out(i-1, j) + b out(i, j-1) + c   (seed outside)
//   GS2D:  lexicographic Gauss-Seidel / SOR on the 5-point problem, in place:
//          u <- (1 - omega) u + omega (W + S + E + N - h^2 f) / 4 with W and S
//          already updated, E and N not yet (Dirichlet value outside).
#include "launch.h"

namespace gk {

// Tiled wavefront: tiles of 64 x 64 or 64 x 32 cells of every layer, one launch per tile
// anti-diagonal D = I + J.  Tile (I, J) reads only tiles (I-1, J) and
// (I, J-1), finished by earlier launches (the new W and S values), and
// (I+1, J), (I, J+1), which later launches change (the old E and N values);
// never a tile of its own diagonal, so those run in parallel.  A block of
// DNW waves owns a tile: the waves load the tile and its one-cell halo into
// LDS with row-contiguous accesses (each wave nine rows, all requested
// together), the first wave alone walks the tile's anti-diagonals, and all
// waves store the tile back.
//
// In the walk lane t owns column t: cell (t, j) is computed at step t + j from
// its S neighbour (the lane's own previous result) and its W neighbour (lane
// t-1's previous result, by a wave-wide DPP shift), so the dependency chain
// never goes through LDS.  The other operands do not depend on the walk: they
// are read four steps at a time, four steps ahead, and what a step waits for is
// its chain of dependent operations alone.  One wave issues an instruction every
// four cycles at best, so the offsets of a step are formed once and shared by
// its accesses, and lanes without a cell compute on clamped rows and store to a
// spare slot rather than branch.  (A tile of 2 x 840 x 821, RECUR FP64, one per
// launch: 21 -> 15 us.)  During the walk the halo tile in LDS is only read (E, N and
// the centre are old values; a step's N is the next step's centre), and each
// result goes to the LDS slot of the cell's own pointwise input, which only its
// lane reads, before: so the walk needs no barrier.  The per-cell arithmetic is
// the operators' above, in the same order.  Rows are 66 elements apart in LDS,
// so lanes on different rows of the same anti-diagonal spread over the banks.
//
// Bound: on many layers by memory and the overlap of the blocks on a CU (GS2D
// FP64, 1024 x 256^2: 766 -> 480 us, 3.4 TB/s); on few by the time of a tile, one
// per tile diagonal (2 x 840 x 821, RECUR FP64: 576 -> 401 us).
constexpr int DT = 64, DNW = 8;

// value of lane t-1, lane 0 its own `first`: wave_shr:1
__device__ __forceinline__ float from_lane_below(float v, float first) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first),
                                                                 __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ double from_lane_below(double v, double first) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned long long f = __builtin_bit_cast(unsigned long long, first);
    const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)f, (int)(unsigned)b, 0x138, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(f >> 32), (int)(unsigned)(b >> 32), 0x138, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

template <class T, int KIND, int DY>
__global__ __launch_bounds__(64 * DNW) void diamond_tile(DiamondArgs a, int D, int i_lo, int count) {
#pragma clang fp contract(off)
    constexpr int LW = DT + 2, RB = (DY + 2 + DNW - 1) / DNW;
    constexpr int NP = KIND == DIAMOND_RECUR ? 3 : 1;  // pointwise inputs: a, b, c or f
    // the tile's values with a one-cell halo ring (RECUR: row 0 and column 0 of it)
    constexpr bool GS = KIND == DIAMOND_GS2D;
    __shared__ T U[GS ? DY + 2 : 1][LW];
    __shared__ T U0[GS ? 1 : DY + 2];
    __shared__ T P[NP][DY][DT];     // pointwise inputs of the tile's cells; P[0] then the results
    __shared__ T idle[DT];          // where lanes without a cell put theirs
    const int t = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int I = i_lo + (int)(blockIdx.x % (unsigned)count), J = D - I;
    const int64_t base = (int64_t)(blockIdx.x / (unsigned)count) * a.pz;
    const int nx = a.nx, ny = a.ny;
    const int64_t py = a.py;
    const int x0 = I * DT, y0 = J * DY;
    const int tw = min(DT, nx - x0), th = min(DY, ny - y0);
    T* out = static_cast<T*>(a.out);
    const T* fsrc = static_cast<const T*>(a.in[1]);
    // boundary values: the Dirichlet value (GS2D) or the seed (RECUR, W and S only)
    const T edge = GS ? (T)a.p[2] : (T)a.p[0];

    // load: halo ring from the grid being computed (W and S new, E and N old;
    // GS2D also the tile's own old values), pointwise inputs of the cells.
    // Columns t and t + 64 of LDS rows r0 .. r0 + RB - 1.
    {
        const int r0 = w * RB;
        T uv[RB][2], pv[RB][NP];
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const int r = r0 + k, y = y0 - 1 + r;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = t + 64 * h, x = x0 - 1 + c;
                const bool ring = r == 0 || c == 0;
                const bool in = r < th + 2 && c < tw + 2 && (unsigned)x < (unsigned)nx && (unsigned)y < (unsigned)ny &&
                                (GS || ring);
                uv[k][h] = in ? out[base + (int64_t)y * py + x] : edge;
            }
            // the cell of column t (LDS column t + 1) in row r
            const bool cell = r >= 1 && r <= th && t < tw;
            const int64_t p = base + (int64_t)y * py + (x0 + t);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const T* src = KIND == DIAMOND_RECUR ? static_cast<const T*>(a.in[i]) : fsrc;
                pv[k][i] = (cell && src) ? src[p] : T(0);
            }
        }
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const int r = r0 + k;
            if (r >= th + 2) break;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = t + 64 * h;
                if (c >= LW) continue;
                if (GS || r == 0) U[GS ? r : 0][c] = uv[k][h];
                else if (c == 0) U0[r] = uv[k][h];
            }
            if (r >= 1 && r <= th && t < tw) {
#pragma unroll
                for (int i = 0; i < NP; ++i) P[i][r - 1][t] = pv[k][i];
            }
        }
    }
    __syncthreads();
    const T omega = (T)a.p[0], h2 = (T)a.p[1];
    // the walk: first wave only (the others wait at the barrier below)
    if (w == 0) {
        constexpr int W = 4, S = (int)sizeof(T);
        // byte offsets of the lane's row jl = d - t, clamped to the tile: of
        // U[jl][t] (the cell's neighbours lie at fixed distances from it) and
        // of P[.][jl][t]
        const int ku = t * S - t * LW * S, ulo = t * S, uhi = ulo + (DY - 1) * LW * S;
        const int kp = t * S - t * DT * S, phi = ulo + (DY - 1) * DT * S;
        const unsigned rows = t < tw ? th : 0;
        const char* const ub = reinterpret_cast<const char*>(&U[0][0]);
        char* const pb = reinterpret_cast<char*>(&P[0][0][0]);
        const int spare = (int)(reinterpret_cast<char*>(&idle[t]) - pb);
        struct In { T e, n, wb, p[NP]; int o; };
        // operands of step d: E, N, the W of lane 0 (others read their old W),
        // the pointwise inputs
        auto fetch = [&](int d, In& v) __attribute__((always_inline)) {
            if (GS) {
                const char* q = ub + min(max(d * LW * S + ku, ulo), uhi);
                v.e = *reinterpret_cast<const T*>(q + (LW + 2) * S);
                v.n = *reinterpret_cast<const T*>(q + (2 * LW + 1) * S);
                v.wb = *reinterpret_cast<const T*>(q + LW * S);
            } else {
                v.wb = U0[GS ? 0 : min(d, DY - 1) + 1];
            }
            const int o = min(max(d * DT * S + kp, ulo), phi);
#pragma unroll
            for (int i = 0; i < NP; ++i) v.p[i] = *reinterpret_cast<const T*>(pb + o + i * DY * DT * S);
            v.o = (unsigned)(d - t) < rows ? o : spare;
        };
        const T s0 = U[0][t + 1], c0 = GS ? U[GS ? 1 : 0][t + 1] : T(0);
        T last = s0;  // this lane's result at the previous step (its next cell's S)
        T ctr = c0;
        const T om1 = T(1) - omega;
        auto run = [&](int d, const In& v, auto fill) __attribute__((always_inline)) {
#pragma clang fp contract(off)
            const T wv = from_lane_below(last, v.wb);  // lane t-1's previous result (every lane shifts)
            T res;
            if (GS) {
                T sum = wv + last;
                sum = sum + v.e;
                sum = sum + v.n;
                res = om1 * ctr + omega * ((sum - h2 * v.p[0]) / T(4));
            } else {
                res = v.p[0] * wv + v.p[NP > 1 ? 1 : 0] * last + v.p[NP > 2 ? 2 : 0];
            }
            *reinterpret_cast<T*>(pb + v.o) = res;
            // before a lane's first cell its S and centre are those of that cell
            const bool begun = !decltype(fill)::value || d >= t;
            last = begun ? res : s0;
            ctr = begun ? v.n : c0;
        };
        In cur[W], nxt[W];
#pragma unroll
        for (int u = 0; u < W; ++u) fetch(u, cur[u]);
        const int steps = tw + th - 1;
        auto group = [&](int d0, auto fill) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < W; ++u) fetch(d0 + W + u, nxt[u]);
#pragma unroll
            for (int u = 0; u < W; ++u) run(d0 + u, cur[u], fill);
#pragma unroll
            for (int u = 0; u < W; ++u) cur[u] = nxt[u];
        };
        int d0 = 0;
        for (; d0 < min(steps, DT); d0 += W) group(d0, std::true_type{});
        for (; d0 < steps; d0 += W) group(d0, std::false_type{});
    }
    __syncthreads();
    if (t < tw) {
        for (int r = 1 + w; r <= th; r += DNW) out[base + (int64_t)(y0 - 1 + r) * py + (x0 + t)] = P[0][r - 1][t];
    }
}

template <class T, int KIND, int DY>
static hipError_t run_tiled(DiamondArgs& a, hipStream_t s) {
    const int ntx = (a.nx + DT - 1) / DT, nty = (a.ny + DY - 1) / DY;
    for (int D = 0; D <= ntx + nty - 2; ++D) {
        const int i_lo = std::max(0, D - (nty - 1)), i_hi = std::min(D, ntx - 1);
        const int count = i_hi - i_lo + 1;
        hipLaunchKernelGGL((diamond_tile<T, KIND, DY>), dim3((unsigned)count * (unsigned)a.nl), dim3(64 * DNW), 0, s, a, D,
                           i_lo, count);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Tiles of 64 x 32 where a diagonal of them fills the chip: their LDS lets four
// blocks (FP64 RECUR: three) share a CU where 64 x 64 tiles leave two (one), and
// blocks that load and store cover those that walk (GS2D FP64, 1024 x 256^2: 581
// us on 64 x 64, 480 on 64 x 32).  Elsewhere 64 x 64: fewer diagonals; also where
// a diagonal of 64 x 32 has more threads than a launch dimension holds, 2^32.
template <class T, int KIND>
static hipError_t pick_tiles(DiamondArgs& a, hipStream_t s) {
    const int64_t wide = std::min((a.nx + DT - 1) / DT, (a.ny + 31) / 32);
    const int64_t blocks = wide * a.nl;
    return blocks >= 512 && blocks * (64 * DNW) < (int64_t)1 << 32 ? run_tiled<T, KIND, 32>(a, s) : run_tiled<T, KIND, 64>(a, s);
}

template <class T>
static hipError_t run_diamond(DiamondArgs& a, int kind, hipStream_t s) {
    if (a.nl == 0 || a.nx == 0 || a.ny == 0) return hipSuccess;
    if (kind == DIAMOND_RECUR) return pick_tiles<T, DIAMOND_RECUR>(a, s);
    if (kind == DIAMOND_GS2D) return pick_tiles<T, DIAMOND_GS2D>(a, s);
    return hipErrorInvalidValue;
}

hipError_t launch_diamond(DiamondArgs& a, int dtype, int kind, hipStream_t s) {
    if (dtype == 0) return run_diamond<double>(a, kind, s);
    if (dtype == 1) return run_diamond<float>(a, kind, s);
    return hipErrorInvalidValue;
}

}  // namespace gk
