// Register-tile passes over all grids of a batch in one launch: the passes of
// k2r_impl.h (standard form, fixed counts, no current), a workgroup's grid
// and tile found from a prefix sum of the grids' tiles.  A batch of small
// grids is bound as one grid of their cells is: by the latency of its passes
// while the tiles are few, by VALU issue and the tiles' rims above.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {

template <typename T, int R, int NW, int KIND>
__global__ __launch_bounds__(64 * NW, (min_waves<T, 1, R, FM_STD>())) __attribute__((amdgpu_num_sgpr(80)))
void kb_reg(const GridDesc<T> *desc, int ng, const int *tiles, RegBatchPass p, int W, int H, int n)
{
    __shared__ __attribute__((aligned(16))) char lds[lds_bytes<T, 1, NW>()];
    __shared__ double sh[1][2];
    __shared__ int stop;
    const int id = xcd_map(blockIdx.x, gridDim.x);
    const int wid = id >= n ? id - n : id;   // the first n workgroups TE, the rest TM
    // grid: the number of prefix sums (of the grids before the next) at or
    // below wid, 64 at a time
    int g = 0;
    for (int g0 = 0; g0 < ng; g0 += 64) {
        const int i = g0 + (int)(threadIdx.x & 63);
        const int c = __popcll(__ballot(i < ng && tiles[i + 1] <= wid));
        g += c;
        if (c < 64) break;
    }
    g = __builtin_amdgcn_readfirstlane(g);
    const GridDesc<T> &d = desc[g];
    const Coef<T> c = d.c;
    RegArgs<T> a{};
    for (int q = 0; q < 3; q++) {
        a.E[q] = d.E[q];
        a.Bin[q] = d.B[p.bin][q];
        a.B[q] = d.B[p.bin ^ 1][q];
        a.dEp[q] = d.dEp[q];
        a.rhs[q] = d.dEp[q];
        a.x_in[q] = p.first ? d.dEp[q] : d.X[p.xout ^ 1][q];
        a.x_out[q] = d.X[p.xout][q];
        a.Bs[q] = p.hand ? d.B[1][q] : nullptr;
        a.Bd[q] = p.hand ? d.B[0][q] : nullptr;
    }
    a.first = p.first;
    a.k = p.k;
    const int t = __builtin_amdgcn_readfirstlane(wid - tiles[g]), ntx = (c.nx + W - 1) / W;
    if (id >= n) reg_pass<T, 2, 1, R, NW, KIND, FM_STD, false>(c, a, ntx, W, H, t, lds, sh, &stop);
    else reg_pass<T, 1, 1, R, NW, KIND, FM_STD, false>(c, a, ntx, W, H, t, lds, sh, &stop);
}

template <typename T, int R, int NW>
hipError_t launch_batch(const GridDesc<T> *d, int ng, const int *tiles, int n, const RegBatchPass &p, hipStream_t s)
{
    const int W = 64 - 2 * p.cut - (p.kind == RK_FRONT ? 3 : 0), H = NW * R - 2 * p.cut;
    if (W < 1 || H < 1 || p.k > p.cut || p.cut > 16 || n < 1) return hipErrorInvalidValue;
    const dim3 g(2 * n), b(64 * NW);
    if (p.kind == RK_FRONT) hipLaunchKernelGGL((kb_reg<T, R, NW, RK_FRONT>), g, b, 0, s, d, ng, tiles, p, W, H, n);
    else if (p.kind == RK_MID) hipLaunchKernelGGL((kb_reg<T, R, NW, RK_MID>), g, b, 0, s, d, ng, tiles, p, W, H, n);
    else hipLaunchKernelGGL((kb_reg<T, R, NW, RK_LAST>), g, b, 0, s, d, ng, tiles, p, W, H, n);
    return hipGetLastError();
}

}  // namespace reg2d

template <typename T>
hipError_t launch_reg_batch(const GridDesc<T> *d, int ng, const int *tiles, int n, int geo, const RegBatchPass &p,
                            hipStream_t s)
{
    using namespace reg2d;
    switch (geo) {
    case 0: return launch_batch<T, 2, 16>(d, ng, tiles, n, p, s);
    case 1: return launch_batch<T, 4, 8>(d, ng, tiles, n, p, s);
    case 2: return launch_batch<T, 4, 16>(d, ng, tiles, n, p, s);
    default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_reg_batch<float>(const GridDesc<float> *, int, const int *, int, int, const RegBatchPass &,
                                            hipStream_t);
template hipError_t launch_reg_batch<double>(const GridDesc<double> *, int, const int *, int, int, const RegBatchPass &,
                                             hipStream_t);

}  // namespace mx
