// Generic do_all for a linear operator given as a term list (Section 3: an
// operator reads grids at fixed offsets from the core element and writes the
// core element), any offsets, any boundary rule per grid.
//
// A wave owns 64 * V consecutive points of R rows; its lanes hold V points of
// each and read every term as one V-wide access per row.  A term's rows
// (y + dy, z + dz) are the same for the whole wave, so the boundary rule in y
// and z and the addresses are scalar work: a row of the grid, a wrapped or
// clamped row, or (Dirichlet) the boundary value without a load.  Only lanes
// whose shifted columns leave the row take an element-by-element branch, and
// only for terms with dx != 0.
//
// Bound: each grid is read from HBM once (counters: reads 1.06 x algorithmic
// on 250^3), but every term is a read of the L1, whose 64 B/clk per CU alone
// takes 30 us there, and of the L2 where the L1 has lost the row; waves wait
// for one term's loads at a time, so occupancy (8 waves per SIMD) matters more
// than loads in flight per wave: reading 2, 4 or 7 terms together measured
// 76, 88 and 110 us against 75.  Measured, seven-term operator of Fig. 1b,
// FP64, per call: 250^3 170 -> 75 us (1.5 -> 3.3 TB/s), 512^3 588 us
// (3.7 TB/s); before, one point per thread walked the list with per-point
// bounds checks.
#include "launch.h"

namespace gk {

// V elements at an address aligned to one element only
template <class T, int V> struct __attribute__((packed, aligned(sizeof(T)))) UVec { T v[V]; };

// One output's sums over its terms [t, t1) at points x .. x + V - 1 of rows
// y .. y + R - 1 of plane z.  INNER: every row the terms read lies inside the
// grid.
template <class T, int V, int R, bool INNER>
__device__ __forceinline__ void linear_sum(const LArgs& a, int t, const int t1, int64_t row, int x0, int xl, int y, int z,
                                           bool xin, T (&s)[R][V]) {
    const Geo& g = a.g;
    const int x = x0 + xl;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < V; ++i) s[r][i] = T(0);
    for (; t < t1; ++t) {
        const LinTerm tm = a.t[t];
        const int dx = (int8_t)tm.d;
        T v[R][V];
        const T* src[R];  // column 0 of the shifted rows
        bool have[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            src[r] = static_cast<const T*>(tm.src) + (row + r * g.py);
            have[r] = true;
            if (!INNER) {
                const int yy = y + r + (int8_t)(tm.d >> 8), zz = z + (int8_t)(tm.d >> 16);
                if (y + r >= g.ny) {
                    have[r] = false;  // not a row of the grid
                } else if ((unsigned)yy >= (unsigned)g.ny || (unsigned)zz >= (unsigned)g.nz) {
                    const int gi = tm.grid & 255, bc = a.bc[gi];
                    have[r] = bc != BC_DIRICHLET;
                    if (have[r])
                        src[r] = static_cast<const T*>(a.in[gi]) + dx + (int64_t)wrap_idx(zz, g.nz, bc) * g.pz +
                                 (int64_t)wrap_idx(yy, g.ny, bc) * g.py;
                }
                if (!have[r]) {
                    const T bcv = (T)a.bcv[tm.grid & 255];
#pragma unroll
                    for (int i = 0; i < V; ++i) v[r][i] = bcv;
                }
            }
        }
        if (dx == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!have[r]) continue;
                const Vec<T, V> q = vload<T, V>(row_at(src[r] + x0, xl));
#pragma unroll
                for (int i = 0; i < V; ++i) v[r][i] = q.v[i];
            }
        } else if (xin) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!have[r]) continue;
                const UVec<T, V> q = *reinterpret_cast<const UVec<T, V>*>(row_at(src[r] + x0, xl));
#pragma unroll
                for (int i = 0; i < V; ++i) v[r][i] = q.v[i];
            }
        } else {
            const int gi = tm.grid & 255, bc = a.bc[gi];
            const T bcv = (T)a.bcv[gi];
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const int xi = x + i + dx;
                const bool in = (unsigned)xi < (unsigned)g.nx;
                const int xs = in ? xi : wrap_idx(xi, g.nx, bc == BC_DIRICHLET ? BC_CLAMP : bc);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (!have[r]) continue;
                    const T q = (src[r] - dx)[xs];
                    v[r][i] = in || bc != BC_DIRICHLET ? q : bcv;
                }
            }
        }
        const T wt = (T)tm.w;
        if (const int ci = tm.grid >> 8) {
            const T* cp = static_cast<const T*>(a.in[ci - 1]) + row;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!INNER && y + r >= g.ny) continue;
                const Vec<T, V> c = vload<T, V>(row_at(cp + r * g.py + x0, xl));
#pragma unroll
                for (int i = 0; i < V; ++i) s[r][i] = fma(wt * c.v[i], v[r][i], s[r][i]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < V; ++i) s[r][i] = fma(wt, v[r][i], s[r][i]);
        }
    }
}

template <class T, int V, int R, bool RED>
__global__ __launch_bounds__(256, 8) void linear_kernel(LArgs a) {
    const Geo& g = a.g;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (id >= a.nblocks) return;
    const int b = xcd_remap((int)id, a.nblocks);
    // x tile, then row group of the strip, then plane, then strip
    const int xt = b % a.nxt;
    int rest = b / a.nxt;
    const int strip = rest / (a.strip * g.nz);
    const int rows = min(a.strip, a.nyt - strip * a.strip);  // row groups of this strip (the last may be short)
    rest -= strip * a.strip * g.nz;
    const int z = rest / rows, y = ((strip * a.strip + rest % rows) * 4 + w) * R;
    const int x0 = xt * 64 * V, xl = lane * V, x = x0 + xl;
    double acc = 0.0;
    if (y < g.ny && x < g.nx) {
        const bool inner = y >= a.ry && y + R - 1 < g.ny - a.ry && z >= a.rz && z < g.nz - a.rz;
        const bool xin = x >= a.rx && x + V + a.rx <= g.nx;
        const int64_t row = (int64_t)z * g.pz + (int64_t)y * g.py;
        T first[R][V];
        int t = 0;
        for (int o = 0; o < a.nout; ++o) {
            const int t1 = a.tend[o];
            T s[R][V];
            if (inner) linear_sum<T, V, R, true>(a, t, t1, row, x0, xl, y, z, xin, s);
            else linear_sum<T, V, R, false>(a, t, t1, row, x0, xl, y, z, xin, s);
            t = t1;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (y + r >= g.ny) continue;
                T* dst = static_cast<T*>(a.out[o]) + (row + r * g.py);
                if (x + V <= g.nx) {
                    Vec<T, V> q;
#pragma unroll
                    for (int i = 0; i < V; ++i) q.v[i] = s[r][i];
                    vstore_nt<T, V>(row_at(dst + x0, xl), q);
                } else {
#pragma unroll
                    for (int i = 0; i < V; ++i)
                        if (x + i < g.nx) dst[x + i] = s[r][i];
                }
                if (RED && o == 0) {
#pragma unroll
                    for (int i = 0; i < V; ++i) first[r][i] = s[r][i];
                }
            }
        }
        if (RED) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (y + r >= g.ny) continue;
                const T* u0 = static_cast<const T*>(a.in[0]) + (row + r * g.py);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    if (x + i >= g.nx) continue;
                    double v = (double)first[r][i];
                    if (a.operand == 1) v = v - (double)u0[x + i];
                    acc = red_acc(acc, v, a.ra.op);
                }
            }
        }
    }
    if (RED) block_reduce(acc, a.ra, b);
}

template <class T, int V, int R>
static hipError_t run_linear(LArgs& a, bool red, hipStream_t s, int* nblocks) {
    a.nxt = (a.g.nx + 64 * V - 1) / (64 * V);
    a.nyt = (a.g.ny + 4 * R - 1) / (4 * R);
    // Rows of a strip: an XCD works through a strip plane by plane, so the
    // planes its terms reach (2 rz + 1 per grid) should stay in its 4 MB L2
    // with room for the streams (512^3 FP64, Fig. 1b: strips of 0.25, 0.5, 1,
    // 2, 4 MB of them and whole planes 624, 608, 589, 588, 650, 678 us).
    const int64_t group = (int64_t)a.g.py * 4 * R * sizeof(T) * (2 * a.rz + 1) * a.nin;
    a.strip = (int)std::max<int64_t>(1, std::min<int64_t>(a.nyt, (2 << 20) / std::max<int64_t>(group, 1)));
    const int64_t n = (int64_t)a.nxt * a.nyt * a.g.nz;
    if (n > INT32_MAX) return hipErrorInvalidValue;
    *nblocks = a.nblocks = (int)n;
    if (n == 0) return hipSuccess;
    // a launch dimension holds under 2^32 threads
    constexpr int64_t GX = 1 << 20;
    const dim3 grid((unsigned)std::min<int64_t>(n, GX), (unsigned)((n + GX - 1) / GX));
    if (red) hipLaunchKernelGGL((linear_kernel<T, V, R, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((linear_kernel<T, V, R, false>), grid, dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !red) return e;
    return launch_reduce_finish(a.ra, *nblocks, s);
}

template <class T, int V>
static hipError_t pick_rows(LArgs& a, bool red, hipStream_t s, int* nb) {
    // two rows per wave share the scalar work of a term (250^3 FP64 104 -> 75
    // us), one where that would leave the chip short of waves (64^3)
    const int64_t waves = ((int64_t)a.g.nx + 64 * V - 1) / (64 * V) * a.g.ny * a.g.nz;
    return waves >= 16384 ? run_linear<T, V, 2>(a, red, s, nb) : run_linear<T, V, 1>(a, red, s, nb);
}

hipError_t launch_linear(LArgs& a, int dtype, bool red, hipStream_t s, int* nblocks) {
    // 16 bytes per lane where a row fills at least one such wave
    if (dtype == 0)
        return a.g.nx > 64 ? pick_rows<double, 2>(a, red, s, nblocks) : pick_rows<double, 1>(a, red, s, nblocks);
    if (dtype == 1) {
        if (a.g.nx > 128) return pick_rows<float, 4>(a, red, s, nblocks);
        return a.g.nx > 64 ? pick_rows<float, 2>(a, red, s, nblocks) : pick_rows<float, 1>(a, red, s, nblocks);
    }
    return hipErrorInvalidValue;
}

}  // namespace gk
