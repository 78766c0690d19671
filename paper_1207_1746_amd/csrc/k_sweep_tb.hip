// Temporally blocked instantiations: weighted Jacobi (k sweeps per pass) and
// red-black relaxation (k colour passes per pass).
#include "launch.h"
#include "tb7.h"

namespace gk {

template <class T, bool HAS_F, int K, bool RB>
static hipError_t run_tb(TBArgs& a, bool red, hipStream_t s, int* nblocks) {
    const int n = (int)tb_blocks(a.g, K, a.cz, tb_pairs(sizeof(T) == 8, RB));
    constexpr int OX = tb_out_x(K, tb_pairs(sizeof(T) == 8, RB));
    a.ntx = (a.g.nx + OX - 1) / OX;
    a.nty = (a.g.ny + tb_out_y(K) - 1) / tb_out_y(K);
    a.ncz = (a.g.nz + a.cz - 1) / a.cz;
    *nblocks = n;
    if (n == 0) return hipSuccess;
    // the wrap of an odd row length splits pairs of columns
    constexpr bool PAIRS = tb_pairs(sizeof(T) == 8, RB), CAN_SPLIT = PAIRS && !RB;
    const bool split = CAN_SPLIT && a.g.bc == BC_PERIODIC && (a.g.nx & 1);
    const dim3 blk(64 * tb_waves(PAIRS));
    if (red) {
        if (split) hipLaunchKernelGGL((tb7_sweep<T, HAS_F, K, true, RB, CAN_SPLIT>), dim3(n), blk, 0, s, a);
        else hipLaunchKernelGGL((tb7_sweep<T, HAS_F, K, true, RB, false>), dim3(n), blk, 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_reduce_finish(a.ra, n, s);
    }
    if (split) hipLaunchKernelGGL((tb7_sweep<T, HAS_F, K, false, RB, CAN_SPLIT>), dim3(n), blk, 0, s, a);
    else hipLaunchKernelGGL((tb7_sweep<T, HAS_F, K, false, RB, false>), dim3(n), blk, 0, s, a);
    return hipGetLastError();
}

template <class T, bool HAS_F, bool RB>
static hipError_t run_tb_k(TBArgs& a, bool red, hipStream_t s, int* nb) {
    static_assert(TB_KMAX == 4, "one instantiation per level count");
    switch (a.k) {
    case 1: return run_tb<T, HAS_F, 1, RB>(a, red, s, nb);
    case 2: return run_tb<T, HAS_F, 2, RB>(a, red, s, nb);
    case 3: return run_tb<T, HAS_F, 3, RB>(a, red, s, nb);
    case 4: return run_tb<T, HAS_F, 4, RB>(a, red, s, nb);
    default: return hipErrorInvalidValue;
    }
}

template <bool RB>
static hipError_t dispatch_tb(TBArgs& a, int dtype, bool has_f, bool red, hipStream_t s, int* nb) {
    if (a.k < 1 || a.k > TB_KMAX) return hipErrorInvalidValue;
    if (dtype == 0)
        return has_f ? run_tb_k<double, true, RB>(a, red, s, nb) : run_tb_k<double, false, RB>(a, red, s, nb);
    if (dtype == 1)
        return has_f ? run_tb_k<float, true, RB>(a, red, s, nb) : run_tb_k<float, false, RB>(a, red, s, nb);
    return hipErrorInvalidValue;
}

hipError_t launch_wjacobi_tb(TBArgs& a, int dtype, bool has_f, bool red, hipStream_t s, int* nb) {
    return dispatch_tb<false>(a, dtype, has_f, red, s, nb);
}

hipError_t launch_rbgs_tb(TBArgs& a, int dtype, bool has_f, bool red, hipStream_t s, int* nb) {
    if (a.g.bc != BC_DIRICHLET) return hipErrorInvalidValue;
    return dispatch_tb<true>(a, dtype, has_f, red, s, nb);
}

}  // namespace gk
