// k_halo.hip -- periodic boundary condition: the 2-point halo of a padded
// field is filled from the interior at the wrapped indices (i mod ni,
// j mod nj), corners included.  The sources are interior points only, so
// one pass over the halo ring of every level is race free.
#include "launch.hpp"

namespace gt4mi {

__device__ __forceinline__ int wrap_index(int i, int n) {
  const int r = i % n;
  return r < 0 ? r + n : r;
}

// Fields of one layout and domain, each given at domain point (0,0,0); blockIdx.z
// picks one, blockIdx.y a level.  Ring of a level: rows -2, -1 and nj, nj+1 over
// i in [-2, ni+2), then columns -2, -1, ni, ni+1 of rows 0 .. nj-1.  Latency bound
// (FP64 256x256x80 moves 3 MB): no loop over levels up to the grid's limit, and
// both states of a time loop in one launch.
template <typename T>
struct HaloPair {
  T* p[2];
  int64_t sj[2], sk[2];
};

template <typename T>
__global__ void __launch_bounds__(kWG) k_halo_periodic(HaloPair<T> f, int ni, int nj, int nk) {
  const int W = ni + 4, r = blockIdx.x * kWG + threadIdx.x;
  if (r >= 4 * W + 4 * nj) return;
  int i, j;
  if (r < 4 * W) {  // the two rows above and the two below
    const int row = r / W;
    i = r - row * W - 2;
    j = row < 2 ? row - 2 : nj + row - 2;
  } else {  // the side columns of the interior rows
    const int s = r - 4 * W;
    j = s >> 2;
    const int c = s & 3;
    i = c < 2 ? c - 2 : ni + c - 2;
  }
  const bool second = blockIdx.z != 0;  // uniform
  T* const p = second ? f.p[1] : f.p[0];
  const int64_t sj = second ? f.sj[1] : f.sj[0], sk = second ? f.sk[1] : f.sk[0];
  const int64_t from = (int64_t)wrap_index(j, nj) * sj + wrap_index(i, ni), to = (int64_t)j * sj + i;
  for (int k = blockIdx.y; k < nk; k += gridDim.y) p[(int64_t)k * sk + to] = p[(int64_t)k * sk + from];
}

template <typename T>
static hipError_t launch(const HaloPair<T>& f, int fields, int ni, int nj, int nk, hipStream_t s) {
  if (ni <= 0 || nj <= 0 || nk <= 0) return hipSuccess;
  const int64_t ring = 4 * (int64_t)(ni + 4) + 4 * (int64_t)nj;
  const dim3 grid((unsigned)((ring + kWG - 1) / kWG), nk < 65535 ? nk : 65535, fields);
  hipLaunchKernelGGL(k_halo_periodic<T>, grid, dim3(kWG), 0, s, f, ni, nj, nk);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_halo_periodic(T* p, int64_t sj, int64_t sk, int ni, int nj, int nk, hipStream_t s) {
  return launch(HaloPair<T>{{p, p}, {sj, sj}, {sk, sk}}, 1, ni, nj, nk, s);
}
template <typename T>
hipError_t launch_halo_periodic_pair(T* p, int64_t p_sj, int64_t p_sk, T* q, int64_t q_sj, int64_t q_sk, int ni, int nj,
                                     int nk, hipStream_t s) {
  return launch(HaloPair<T>{{p, q}, {p_sj, q_sj}, {p_sk, q_sk}}, 2, ni, nj, nk, s);
}

template hipError_t launch_halo_periodic<float>(float*, int64_t, int64_t, int, int, int, hipStream_t);
template hipError_t launch_halo_periodic<double>(double*, int64_t, int64_t, int, int, int, hipStream_t);
template hipError_t launch_halo_periodic_pair<float>(float*, int64_t, int64_t, float*, int64_t, int64_t, int, int, int,
                                                     hipStream_t);
template hipError_t launch_halo_periodic_pair<double>(double*, int64_t, int64_t, double*, int64_t, int64_t, int, int, int,
                                                      hipStream_t);

}  // namespace gt4mi
