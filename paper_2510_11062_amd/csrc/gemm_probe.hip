// Measurement aid: the tile loop of the head kernels run as plain bf16 GEMMs, without any epilogue work, so that the
// loop itself can be compared with a vendor GEMM on the shapes the library uses.
//
//   gemm_probe <variant> M N K
//     nt    C[m][n] = sum_k A[m][k] B[n][k]   both operands contiguous along k (forward, exponentials, dZ)
//     km    C[m][n] = sum_k A[k][m] B[k][n]   both operands k-major (dW)
//     mx    C[m][n] = sum_k A[k][m] B[n][k]   A k-major, B contiguous along k (dHidden on untransposed weights)
//   each with a suffix for the wavefront grid: 8 = 4 x 2, t = 2 x 4, 4 = 2 x 2 wavefronts
// M, N multiples of 256, K a multiple of 64.  Prints the time per launch, the achieved TFLOP/s and the shader clock
// (cycle counter against the 100 MHz wall clock) after checking 600 sampled outputs of a 512 x 512 corner against fp64
// sums.  Not part of the library.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "gemm_bf16.hpp"
#include "tile_order.hpp"

#define CHECK(x)                                                            \
  do {                                                                      \
    hipError_t e_ = (x);                                                    \
    if (e_ != hipSuccess) {                                                 \
      printf("HIP error %s at line %d\n", hipGetErrorString(e_), __LINE__); \
      exit(1);                                                              \
    }                                                                       \
  } while (0)

namespace {

using namespace atg;

constexpr size_t kClockSlot = (size_t{16} << 20) - 1;   // float index in C where workgroup 0 leaves the clock

// AK / BK: the operand is k-major; lda / ldb: row strides in bytes
template <typename G, bool AK, bool BK>
__global__ __launch_bounds__(G::kThreads) void k_probe(const char* __restrict__ A, const char* __restrict__ B,
                                                       float* __restrict__ C, int M, int N, int K, size_t lda, size_t ldb,
                                                       int write_c) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const long long clk0 = clock64(), wall0 = wall_clock64();
  const TileOrder ord{M / kTile16, N / kTile16, 8};
  float sink = 0.f;
  for (int t = logical_workgroup(); t < ord.total(); t += gridDim.x) {
    int ta, tb;
    ord.decode(t, &ta, &tb);
    const Coord16<G> co;
    floatx4 acc[G::kIB][G::kJB];
    typename std::conditional<AK, KMajorPanel<G::kLoadsA>, RowPanel<G::kLoadsA>>::type pa;
    typename std::conditional<BK, KMajorPanel<G::kLoadsB>, RowPanel<G::kLoadsB>>::type pb;
    if constexpr (AK) pa.init(A + static_cast<size_t>(ta) * kTile16 * 2, co.wave, co.lane, lda, 31);
    else pa.init(A + static_cast<size_t>(ta) * kTile16 * lda, co.wave, co.lane, [&](int r) { return static_cast<uint32_t>(r * lda); });
    if constexpr (BK) pb.init(B + static_cast<size_t>(tb) * kTile16 * 2, co.wave, co.lane, ldb, 31);
    else pb.init(B + static_cast<size_t>(tb) * kTile16 * ldb, co.wave, co.lane, [&](int r) { return static_cast<uint32_t>(r * ldb); });
    gemm16<G>(acc, pa, pb, K / kStepK, smem, co);
    const Coord16<G> ce;
    if (write_c) {
#pragma unroll
      for (int i = 0; i < G::kIB; ++i)
#pragma unroll
        for (int j = 0; j < G::kJB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            C[static_cast<size_t>(ta * kTile16 + ce.a_row(i) + r) * N + tb * kTile16 + ce.b_row(j)] = acc[i][j][r];
    } else {
#pragma unroll
      for (int i = 0; i < G::kIB; ++i)
#pragma unroll
        for (int j = 0; j < G::kJB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) sink += acc[i][j][r];
    }
  }
  if (!write_c && sink == 12345.678f) C[threadIdx.x] = sink;   // keeps the contraction alive
  if (!write_c && blockIdx.x == 0 && threadIdx.x == 0)
    C[kClockSlot] = static_cast<float>(clock64() - clk0) / static_cast<float>(wall_clock64() - wall0) * 100.f;
}

// pseudo-random bf16 in [-0.5, 0.5)
__global__ void k_init(uint16_t* p, size_t n, uint32_t seed) {
  for (size_t i = blockIdx.x * size_t{256} + threadIdx.x; i < n; i += gridDim.x * size_t{256}) {
    uint32_t x = static_cast<uint32_t>(i) * 2654435761u + seed;
    x = (x ^ (x >> 15)) * 2246822519u;
    x = (x ^ (x >> 13)) * 3266489917u;
    p[i] = f32_to_bf16(static_cast<float>((x >> 8) & 0xffff) / 65536.f - 0.5f).bits;
  }
}

__global__ void k_reference(const uint16_t* A, const uint16_t* B, const float* C, int K, size_t lda, size_t ldb, int ak,
                            int bk, float* err) {
  const int q = blockIdx.x, i = (q * 131) % 512, j = (q * 977 + 13) % 512;
  double s = 0;
  for (int k = threadIdx.x; k < K; k += 64) {
    const uint16_t a = ak ? A[k * (lda / 2) + i] : A[i * (lda / 2) + k], b = bk ? B[k * (ldb / 2) + j] : B[j * (ldb / 2) + k];
    s += static_cast<double>(bf16_to_f32(bf16_t{a})) * bf16_to_f32(bf16_t{b});
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (threadIdx.x == 0) err[q] = static_cast<float>(fabs(s - C[static_cast<size_t>(i) * 512 + j]));
}

template <typename G, bool AK, bool BK>
int bench(const char* variant, int M, int N, int K) {
  char *dA, *dB;
  float *dC, *dE;
  const size_t na = static_cast<size_t>(M) * K, nb = static_cast<size_t>(N) * K;
  const size_t lda = static_cast<size_t>(AK ? M : K) * 2, ldb = static_cast<size_t>(BK ? N : K) * 2;
  CHECK(hipMalloc(&dA, na * 2));
  CHECK(hipMalloc(&dB, nb * 2));
  CHECK(hipMalloc(&dC, size_t{64} << 20));
  CHECK(hipMalloc(&dE, 600 * 4));
  hipLaunchKernelGGL(k_init, dim3(4096), dim3(256), 0, 0, reinterpret_cast<uint16_t*>(dA), na, 1u);
  hipLaunchKernelGGL(k_init, dim3(4096), dim3(256), 0, 0, reinterpret_cast<uint16_t*>(dB), nb, 77u);
  auto kern = k_probe<G, AK, BK>;
  CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kRingBytes));
  hipLaunchKernelGGL(kern, dim3(8), dim3(G::kThreads), kRingBytes, 0, dA, dB, dC, 512, 512, K, lda, ldb, 1);
  hipLaunchKernelGGL(k_reference, dim3(600), dim3(64), 0, 0, reinterpret_cast<uint16_t*>(dA), reinterpret_cast<uint16_t*>(dB),
                     dC, K, lda, ldb, AK ? 1 : 0, BK ? 1 : 0, dE);
  std::vector<float> err(600);
  CHECK(hipMemcpy(err.data(), dE, 600 * 4, hipMemcpyDeviceToHost));
  float maxerr = 0.f;
  for (float e : err) maxerr = e > maxerr ? e : maxerr;
  if (!(maxerr < 1e-3 * sqrt(static_cast<double>(K)))) {
    printf("%s: WRONG RESULT, max abs err %.3e\n", variant, maxerr);
    return 1;
  }
  printf("%s check: max abs err %.3e on 600 sampled outputs\n", variant, maxerr);
  hipEvent_t e0, e1;
  CHECK(hipEventCreate(&e0));
  CHECK(hipEventCreate(&e1));
  const int iters = 5;
  for (int it = 0; it < 2 + iters; ++it) {
    if (it == 2) CHECK(hipEventRecord(e0));
    hipLaunchKernelGGL(kern, dim3(256), dim3(G::kThreads), kRingBytes, 0, dA, dB, dC, M, N, K, lda, ldb, 0);
  }
  CHECK(hipEventRecord(e1));
  CHECK(hipDeviceSynchronize());
  float ms = 0.f, mhz = 0.f;
  CHECK(hipEventElapsedTime(&ms, e0, e1));
  ms /= iters;
  CHECK(hipMemcpy(&mhz, dC + kClockSlot, 4, hipMemcpyDeviceToHost));
  printf("{\"variant\": \"%s\", \"M\": %d, \"N\": %d, \"K\": %d, \"ms\": %.4f, \"tflops\": %.1f, \"shader_clock_mhz\": %.0f}\n",
         variant, M, N, K, ms, 2.0 * M * N * K / ms / 1e9, mhz);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 5) {
    printf("usage: gemm_probe nt8|ntt|nt4|km8|kmt|km4|mx8|mxt|mx4 M N K\n");
    return 2;
  }
  const char* v = argv[1];
  const int M = atoi(argv[2]), N = atoi(argv[3]), K = atoi(argv[4]);
  if (M % 256 || N % 256 || K % 64 || M < 512 || N < 512 || K < 64) {
    printf("unsupported shape\n");
    return 2;
  }
  using G8 = Grid16<4, 2>;
  using GT = Grid16<2, 4>;
  using G4 = Grid16<2, 2>;
  if (!strcmp(v, "nt8")) return bench<G8, false, false>(v, M, N, K);
  if (!strcmp(v, "ntt")) return bench<GT, false, false>(v, M, N, K);
  if (!strcmp(v, "nt4")) return bench<G4, false, false>(v, M, N, K);
  if (!strcmp(v, "km8")) return bench<G8, true, true>(v, M, N, K);
  if (!strcmp(v, "kmt")) return bench<GT, true, true>(v, M, N, K);
  if (!strcmp(v, "km4")) return bench<G4, true, true>(v, M, N, K);
  if (!strcmp(v, "mx8")) return bench<G8, true, false>(v, M, N, K);
  if (!strcmp(v, "mxt")) return bench<GT, true, false>(v, M, N, K);
  if (!strcmp(v, "mx4")) return bench<G4, true, false>(v, M, N, K);
  printf("unknown variant\n");
  return 2;
}
