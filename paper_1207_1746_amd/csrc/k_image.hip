// Integer image filters on uint8 planes (Section 1: basic image-processing
// filters are stencil computations), clamp-to-edge:
//   box = floor((S + 12) / 25), S the 5x5 window sum   (uint8 out)
//   lap = N + S + E + W - 4 C  (or 8-neighbour - 8 C)    (int16 out)
//
// Each lane owns 16 consecutive pixels of a row and marches through a chunk of
// rows, with two rows of loads in flight ahead of the row being filtered.
// Chunks are mapped to XCDs in contiguous ranges and march in alternating
// directions (even chunks down, odd chunks up; both filters are symmetric in
// y), so the two halo rows a chunk reads past each end are requested in the
// same steps as the neighbouring chunk requests them as its own rows, and come
// from the shared L2 instead of HBM.  A 5-row queue holds the raw bytes (the
// lane's 16 plus 4 on each side), vertical window sums are kept as running
// sums of packed 16-bit pairs (even / odd byte lanes of each dword, so 32-bit
// adds never carry between halves), the horizontal 5-sum uses funnel shifts
// across neighbouring dwords, and the divide by 25 is an exact multiply-shift:
// floor((S+12)/25) = (S*41944 + 12*41944) >> 20 for every S in [0, 6375].
//
// Any width: rows start 16-byte aligned and their pitch is a multiple of 16
// bytes, so the last lane's 16-byte load stays inside the row's allocation;
// the wave that holds the end of a row replaces the bytes past it by the last
// pixel (one bit-select per dword, precomputed masks) and its last lane stores
// its 1..15 pixels as 8, 4, 2 and 1.  Bound by HBM (1 B read, 3 B written per
// pixel): 4 x 8192^2 225 us on fresh buffers, 4.8 TB/s (a device copy of that
// size reaches 5.2).  Rows of up to 512 pixels share a wave: 2, 4 or 8 chunks of
// rows, each on as many lanes as its row needs (4 x 137 x 4145: 18.9 us with a
// row per wave, 16.7 with a thread per pixel, 9.7 so).  8 x 1918 x 1078, 8-neighbour Laplacian: 76.7 -> 20.5 us
// (before, widths that are not a multiple of 16 and the 8-neighbour Laplacian
// ran one thread per pixel with 25 byte loads).  Small images still do: see
// image_by_pixel.
#include "launch.h"

namespace gk {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

struct Row6 {
    uint32_t d[6];  // d[0]: bytes x-4..x-1, d[1..4]: x..x+15, d[5]: x+16..x+19
};

__device__ __forceinline__ uint32_t rep_byte(uint32_t b) { return b * 0x01010101u; }

// x < g.nx.  TAIL: the wave holds the end of the row; m[k] selects the bytes of
// d[k + 1] inside it, and the others become the last pixel.
template <bool TAIL>
__device__ __forceinline__ Row6 load_row6(const uint8_t* img, const Geo& g, int x, int y, int z, const uint32_t (&m)[5]) {
    const int yc = y < 0 ? 0 : (y >= g.ny ? g.ny - 1 : y);
    const uint8_t* row = img + (int64_t)z * g.pz + (int64_t)yc * g.py;
    Row6 r;
    const uint4 c = *reinterpret_cast<const uint4*>(row + x);
    r.d[1] = c.x;
    r.d[2] = c.y;
    r.d[3] = c.z;
    r.d[4] = c.w;
    r.d[0] = x >= 4 ? *reinterpret_cast<const uint32_t*>(row + x - 4) : rep_byte(c.x & 0xFFu);
    if (TAIL) {
        const uint32_t e = rep_byte(row[g.nx - 1]);
        r.d[5] = x + 16 < g.nx ? *reinterpret_cast<const uint32_t*>(row + x + 16) : e;
#pragma unroll
        for (int k = 0; k < 5; ++k) r.d[k + 1] = (r.d[k + 1] & m[k]) | (e & ~m[k]);
    } else {
        r.d[5] = *reinterpret_cast<const uint32_t*>(row + x + 16);
    }
    return r;
}

__device__ __forceinline__ uint32_t evn(uint32_t d) { return d & 0x00FF00FFu; }
__device__ __forceinline__ uint32_t odd(uint32_t d) { return (d >> 8) & 0x00FF00FFu; }
// (hi half of a, lo half of b): the pair shifted by one position
__device__ __forceinline__ uint32_t funnel(uint32_t lo_src, uint32_t hi_src) {
    return __builtin_amdgcn_alignbit(hi_src, lo_src, 16);
}
__device__ __forceinline__ uint32_t box1(uint32_t s) { return (__umul24(s, 41944u) + 503328u) >> 20; }
__device__ __forceinline__ uint32_t pk_sub16(uint32_t a, uint32_t b) {
    u16x2 va = __builtin_bit_cast(u16x2, a), vb = __builtin_bit_cast(u16x2, b);
    return __builtin_bit_cast(uint32_t, va - vb);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// The 16 int16 values of lane t of P are segments 2 t, 2 t + 1 (16 bytes each) of
// the P lanes' 32 P bytes: hand them round so that lane t holds segments t
// and P + t and each store instruction writes 16 P bytes contiguously (stored as
// they lie, every other 16 bytes per instruction, streaming stores leave
// half-written lines: writes 1.12 x algorithmic and 254 us against 165 on
// 4 x 8192^2).
template <int P>
__device__ __forceinline__ void exchange(const uint32_t (&lo)[8], u32x4& s0, u32x4& s1) {
    const int lane = threadIdx.x & 63, src = (lane & ~(P - 1)) + (lane % P >> 1);
    const bool hi = lane & 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t a0 = (uint32_t)__shfl((int)lo[k], src), b0 = (uint32_t)__shfl((int)lo[4 + k], src);
        const uint32_t a1 = (uint32_t)__shfl((int)lo[k], src + P / 2), b1 = (uint32_t)__shfl((int)lo[4 + k], src + P / 2);
        s0[k] = hi ? b0 : a0;
        s1[k] = hi ? b1 : a1;
    }
}

// n (0..8) int16 values of a 16-byte segment, as 8, 4, 2 and 1
__device__ __forceinline__ void store_seg(int16_t* p, const u32x4& v, int n) {
    if (n >= 8) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
        return;
    }
    if (n & 4) *reinterpret_cast<u32x2*>(p) = u32x2{v[0], v[1]};
    if (n & 2) *reinterpret_cast<uint32_t*>(p + (n & 4)) = (n & 4) ? v[2] : v[0];
    if (n & 1) p[n & 6] = (int16_t)((n & 4) ? ((n & 2) ? v[3] : v[2]) : ((n & 2) ? v[1] : v[0]));
}

// A march of P lanes x 16 pixels over the n rows ys, ys + dir, ... (the wave's
// other lanes march over rows of their own, all of them `steps` steps).
template <bool LAP8, bool TAIL, int P>
__device__ __forceinline__ void image_march(const uint8_t* __restrict__ img, uint8_t* __restrict__ box,
                                            int16_t* __restrict__ lap, const Geo& g, int xw, int z, int ys, int dir,
                                            int n, int steps) {
    const int lane = threadIdx.x % P;
    const int xl = xw + lane * 16;
    const int nv = min(g.nx - xl, 16);         // this lane's pixels (<= 0: none)
    const int x = TAIL && nv <= 0 ? xw : xl;   // lanes past the end repeat the first lane's loads
    uint32_t m[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int in = g.nx - x - 4 * k;       // bytes of the dword inside the row
        m[k] = in >= 4 ? 0xFFFFFFFFu : (in <= 0 ? 0u : (1u << (8 * in)) - 1u);
    }

    Row6 q[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) q[i] = load_row6<TAIL>(img, g, x, ys + dir * (i - 2), z, m);
    uint32_t VE[6], VO[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        VE[k] = evn(q[0].d[k]) + evn(q[1].d[k]) + evn(q[2].d[k]) + evn(q[3].d[k]) + evn(q[4].d[k]);
        VO[k] = odd(q[0].d[k]) + odd(q[1].d[k]) + odd(q[2].d[k]) + odd(q[3].d[k]) + odd(q[4].d[k]);
    }

    // two rows in flight ahead of the one being consumed
    Row6 nxt1, nxt2;
    if (1 < steps) nxt1 = load_row6<TAIL>(img, g, x, ys + dir * 3, z, m);
    for (int s = 0; s < steps; ++s) {
        const int y = ys + dir * s;
        const bool more = s + 1 < steps;
        if (s + 2 < steps) nxt2 = load_row6<TAIL>(img, g, x, ys + dir * (s + 4), z, m);

        // box: horizontal 5-sums of the vertical sums, columns 4k..4k+3
        uint32_t AE[5], AO[5];  // AE[k+1] = (hi VE[k], lo VE[k+1]), k = -1..3
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            AE[k] = funnel(VE[k], VE[k + 1]);
            AO[k] = funnel(VO[k], VO[k + 1]);
        }
        uint32_t bo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t t = AO[k] + VE[k + 1] + VO[k + 1] + AE[k + 1];
            const uint32_t he = t + AE[k];      // columns 4k, 4k+2
            const uint32_t ho = t + AO[k + 1];  // columns 4k+1, 4k+3
            bo[k] = box1(he & 0xFFFFu) | (box1(ho & 0xFFFFu) << 8) | (box1(he >> 16) << 16) |
                    (box1(ho >> 16) << 24);
        }
        const int64_t row = (int64_t)z * g.pz + (int64_t)y * g.py;
        const bool own = P == 64 || s < n;
        if (!TAIL || (own && nv == 16)) {
            u32x4 vb = {bo[0], bo[1], bo[2], bo[3]};
            __builtin_nontemporal_store(vb, reinterpret_cast<u32x4*>(box + row + x));
        } else if (own && nv > 0) {
            uint8_t* p = box + row + x;
            if (nv & 8) *reinterpret_cast<u32x2*>(p) = u32x2{bo[0], bo[1]};
            const uint32_t w0 = (nv & 8) ? bo[2] : bo[0], w1 = (nv & 8) ? bo[3] : bo[1];
            if (nv & 4) *reinterpret_cast<uint32_t*>(p + (nv & 8)) = w0;
            const uint32_t w = (nv & 4) ? w1 : w0;
            if (nv & 2) *reinterpret_cast<uint16_t*>(p + (nv & 12)) = (uint16_t)w;
            if (nv & 1) p[nv & 14] = (uint8_t)((nv & 2) ? w >> 16 : w);
        }

        // Laplacian from rows y -+ 1 (q[1], q[3]) and y (q[2]), a bias per half
        // (the sums stay positive): 4-neighbour + 1024, 8-neighbour + 2048
        uint32_t lo[8];
        constexpr uint32_t BIAS = LAP8 ? 0x08000800u : 0x04000400u;
        uint32_t ne[6], no[6];  // column sums a horizontal neighbour adds: the row itself, or all three rows
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            ne[k] = evn(q[2].d[k]);
            no[k] = odd(q[2].d[k]);
            if (LAP8) {
                ne[k] += evn(q[1].d[k]) + evn(q[3].d[k]);
                no[k] += odd(q[1].d[k]) + odd(q[3].d[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t ce = evn(q[2].d[k + 1]), co = odd(q[2].d[k + 1]);
            const uint32_t left_e = funnel(no[k], no[k + 1]);       // columns 4k-1, 4k+1
            const uint32_t right_o = funnel(ne[k + 1], ne[k + 2]);  // columns 4k+2, 4k+4
            const uint32_t pe = evn(q[1].d[k + 1]) + evn(q[3].d[k + 1]) + left_e + no[k + 1];
            const uint32_t po = odd(q[1].d[k + 1]) + odd(q[3].d[k + 1]) + ne[k + 1] + right_o;
            const uint32_t le = pe + BIAS - (ce << (LAP8 ? 3 : 2));
            const uint32_t lq = po + BIAS - (co << (LAP8 ? 3 : 2));
            // int16 outputs in column order: (4k, 4k+1) and (4k+2, 4k+3)
            lo[2 * k] = pk_sub16(__builtin_amdgcn_perm(lq, le, 0x05040100u), BIAS);
            lo[2 * k + 1] = pk_sub16(__builtin_amdgcn_perm(lq, le, 0x07060302u), BIAS);
        }
        u32x4 s0, s1;
        exchange<P>(lo, s0, s1);
        int16_t* lp = lap + row + xw;  // the lanes' segment: 16-byte pieces lane and P + lane
        if (TAIL) {
            if (own) {
                store_seg(lp + 8 * lane, s0, max(min(g.nx - xw - 8 * lane, 8), 0));
                store_seg(lp + 8 * P + 8 * lane, s1, max(min(g.nx - xw - 8 * P - 8 * lane, 8), 0));
            }
        } else {
            __builtin_nontemporal_store(s0, reinterpret_cast<u32x4*>(lp) + lane);
            __builtin_nontemporal_store(s1, reinterpret_cast<u32x4*>(lp) + 64 + lane);
        }

        if (more) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                VE[k] = VE[k] + evn(nxt1.d[k]) - evn(q[0].d[k]);
                VO[k] = VO[k] + odd(nxt1.d[k]) - odd(q[0].d[k]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) q[i] = q[i + 1];
            q[4] = nxt1;
            nxt1 = nxt2;
        }
    }
}

template <bool LAP8, int P>
__global__ __launch_bounds__(256) void image_kernel(const uint8_t* __restrict__ img, uint8_t* __restrict__ box,
                                                    int16_t* __restrict__ lap, Geo g, int cy, int gyn, int ntiles,
                                                    int nblocks) {
    const int id = blockIdx.y * gridDim.x + blockIdx.x;
    if (id >= nblocks) return;
    const int block = xcd_remap(id, nblocks);
    // launched as waves x chunks: a wave's tile is (x wave, chunk, layer); in
    // rows of at most 16 P < 1024 pixels, 64 / P tiles (chunk, layer)
    if constexpr (P < 64) {
        const int wave = block * (blockDim.x >> 6) + (threadIdx.x >> 6);
        const int first = wave * (64 / P);
        if (first >= ntiles) return;
        const int t = min(first + (int)(threadIdx.x & 63) / P, ntiles - 1);  // (the last wave's spare lanes repeat its last)
        const int by = t % gyn, z = t / gyn, y0 = by * cy, y1 = min(y0 + cy, g.ny);
        const int dir = (by & 1) ? -1 : 1;
        image_march<LAP8, true, P>(img, box, lap, g, 0, z, dir > 0 ? y0 : y1 - 1, dir, y1 - y0, min(cy, g.ny));
        return;
    }
    const int nxw = (g.nx + 1023) / 1024;
    const int nw = blockDim.x >> 6;
    const int tile = block * nw + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= ntiles) return;
    const int xw = (tile % nxw) * 1024, by = (tile / nxw) % gyn, z = tile / (nxw * gyn);
    const int y0 = by * cy, y1 = min(y0 + cy, g.ny);
    // march direction and first row; row i of the queue is ys + dir * (s + i - 2)
    // at step s (the queue is symmetric in y, so the filters are unchanged)
    const int dir = (by & 1) ? -1 : 1;
    const int ys = dir > 0 ? y0 : y1 - 1;
    // the dword after the wave's last lane lies in the row: no lane needs the edge rule
    if (xw + 1024 + 4 <= g.nx) image_march<LAP8, false, 64>(img, box, lap, g, xw, z, ys, dir, y1 - y0, y1 - y0);
    else image_march<LAP8, true, 64>(img, box, lap, g, xw, z, ys, dir, y1 - y0, y1 - y0);
}

// One thread per pixel, 25 byte loads each, all in flight together: the chain
// of a small image is one load's latency, where a march's is its first five
// rows, the filters of 16 pixels and an exchange of lanes.
__global__ __launch_bounds__(256) void image_pixels(const uint8_t* __restrict__ img, uint8_t* __restrict__ box,
                                                    int16_t* __restrict__ lap, Geo g, int lap_kind) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int z = blockIdx.z;
    if (x >= g.nx || y >= g.ny) return;
    const uint8_t* pl = img + (int64_t)z * g.pz;
    auto at = [&](int xx, int yy) -> int {
        xx = xx < 0 ? 0 : (xx >= g.nx ? g.nx - 1 : xx);
        yy = yy < 0 ? 0 : (yy >= g.ny ? g.ny - 1 : yy);
        return pl[(int64_t)yy * g.py + xx];
    };
    uint32_t s = 0;
    for (int dy = -2; dy <= 2; ++dy)
        for (int dx = -2; dx <= 2; ++dx) s += at(x + dx, y + dy);
    const int c = at(x, y);
    int l;
    if (lap_kind == 8) {
        l = -9 * c;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) l += at(x + dx, y + dy);
    } else {
        l = at(x, y - 1) + at(x, y + 1) + at(x - 1, y) + at(x + 1, y) - 4 * c;
    }
    const int64_t off = (int64_t)z * g.pz + (int64_t)y * g.py + x;
    box[off] = (uint8_t)box1(s);
    lap[off] = (int16_t)l;
}

template <int P>
static void run_image(const uint8_t* img, uint8_t* box, int16_t* lap, const Geo& g, bool lap8, int cy, int gyn, int n,
                      hipStream_t s) {
    const int nb = (n + 256 / P - 1) / (256 / P);
    // a launch dimension holds under 2^32 threads
    constexpr int GX = 1 << 20;
    const dim3 grid((unsigned)std::min(nb, GX), (unsigned)((nb + GX - 1) / GX));
    if (lap8) hipLaunchKernelGGL((image_kernel<true, P>), grid, dim3(256), 0, s, img, box, lap, g, cy, gyn, n, nb);
    else hipLaunchKernelGGL((image_kernel<false, P>), grid, dim3(256), 0, s, img, box, lap, g, cy, gyn, n, nb);
}

hipError_t launch_image(const uint8_t* img, uint8_t* box, int16_t* lap, const Geo& g,
                        int lap_kind, int cy, hipStream_t s) {
    if (g.nx == 0 || g.ny == 0 || g.nz == 0) return hipSuccess;
    if (cy == 0) {
        const dim3 grid((g.nx + 63) / 64, (g.ny + 3) / 4, g.nz);
        hipLaunchKernelGGL(image_pixels, grid, dim3(256), 0, s, img, box, lap, g, lap_kind);
        return hipGetLastError();
    }
    cy = std::min(cy, g.ny);
    auto tiles = [&] { return (int64_t)((g.nx + 1023) / 1024) * ((g.ny + cy - 1) / cy) * g.nz; };
    // tile indices are 32-bit: longer chunks of rows where there are too many
    while (tiles() > (int64_t)1 << 30 && cy < g.ny) cy = (int)std::min<int64_t>(2 * (int64_t)cy, g.ny);
    const int gyn = (g.ny + cy - 1) / cy;
    const int64_t n = tiles();
    if (n > (int64_t)1 << 30) return hipErrorInvalidValue;
    const bool lap8 = lap_kind == 8;
    switch (image_lanes(g.nx)) {
        case 8: run_image<8>(img, box, lap, g, lap8, cy, gyn, (int)n, s); break;
        case 16: run_image<16>(img, box, lap, g, lap8, cy, gyn, (int)n, s); break;
        case 32: run_image<32>(img, box, lap, g, lap8, cy, gyn, (int)n, s); break;
        default: run_image<64>(img, box, lap, g, lap8, cy, gyn, (int)n, s); break;
    }
    return hipGetLastError();
}

}  // namespace gk
