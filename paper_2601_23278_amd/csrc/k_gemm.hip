// Dense projections  C[M, N] = A[M, K] * W[N, K]^T  (activations times [out, in] weights), fp32 accumulate.
//
// Kernels:
//   k_gemm_valu  any element type, any shape: LDS-tiled 64x64x16, 4x4 outputs per lane on the vector ALU.
//                Used for large fp32 products and for shapes the matrix-core kernels do not take.
//   k_gemm_f32   small fp32 products on the matrix cores (full fp32 products and sums).
//   k_gemm_pipe, k_gemm_mfma  bf16 on the matrix cores (see below).
// M is read from device memory when the row count is only known on the device (packed batch after eviction).
#include <algorithm>

#include "focus_internal.h"

namespace fk {

template <typename T> __device__ __forceinline__ float to_f(T v) { return (float)v; }

template <typename T, int EPI>
__device__ __forceinline__ void store_out(void *out, size_t idx, float acc) {
  if (EPI == EPI_STORE) ((T *)out)[idx] = (T)acc;
  else if (EPI == EPI_ADD_F32) ((float *)out)[idx] += acc;
  else ((float *)out)[idx] = acc;
}

template <typename T, int EPI>
__global__ __launch_bounds__(256) void k_gemm_valu(const T *__restrict__ A, const T *__restrict__ W, int N, int K, Rows rows,
                                                   void *out, int ldo) {
  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  __shared__ float As[16][65], Ws[16][65];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int i = threadIdx.x; i < 1024; i += 256) {
      int rr = i >> 4, kk = i & 15;
      int gm = m0 + rr, gn = n0 + rr, gk = k0 + kk;
      As[kk][rr] = (gm < M && gk < K) ? to_f(A[(size_t)gm * K + gk]) : 0.f;
      Ws[kk][rr] = (gn < N && gk < K) ? to_f(W[(size_t)gn * K + gk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i], w[i] = Ws[kk][tx * 4 + i];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * w[j];
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i) {
    int gm = m0 + ty * 4 + i;
    if (gm >= M) continue;
    for (int j = 0; j < 4; ++j) {
      int gn = n0 + tx * 4 + j;
      if (gn < N) store_out<T, EPI>(out, (size_t)gm * ldo + gn, acc[i][j]);
    }
  }
}

template <typename T>
static void launch_valu(hipStream_t s, const void *A, const void *W, int N, int K, Rows rows, int epi, void *out, int ldo) {
  dim3 grid((N + 63) / 64, (rows.cap + 63) / 64);
  if (epi == EPI_STORE)
    k_gemm_valu<T, EPI_STORE><<<grid, 256, 0, s>>>((const T *)A, (const T *)W, N, K, rows, out, ldo);
  else if (epi == EPI_ADD_F32)
    k_gemm_valu<T, EPI_ADD_F32><<<grid, 256, 0, s>>>((const T *)A, (const T *)W, N, K, rows, out, ldo);
  else
    k_gemm_valu<T, EPI_STORE_F32><<<grid, 256, 0, s>>>((const T *)A, (const T *)W, N, K, rows, out, ldo);
}

// ---------------------------------------------------------------------------------------------
// fp32 on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums).  The fp32 models are small, so a launch is bound by
// latency: 64 x 64 tiles gave 64 rows x 256 columns four workgroups that walked K = 1024 alone (65 us).  Here a tile is 16 rows x 16
// columns and the workgroup's wavefronts share its K: wavefront w takes the 16-wide K pieces w, w + NW, ..., U = four in flight, straight
// from global memory (a 16-byte load per operand feeds four products; both operands permute k alike), and the partial tiles are added in
// wavefront order through LDS: 5.2 us.  (Eight in flight hold twice the registers: 512 rows of a 512-wide model 985 us a step, 863 with four.)
// SiLU*up: the workgroup computes the gate and the up tile of the same columns and stores silu(gate) * up.
// NORM: A holds rows of the residual stream and the product is that of their RMSNorm: each workgroup first adds up the squares of its rows
// (for 256 columns in the order of k_rmsnorm, so that the sums are the same bit for bit) and scales the rows it holds in registers, so it
// has to hold all of K at once: NW * U pieces.  The norm's own launch, 2.8 to 3.5 us in a chain of such launches, is gone; what every
// workgroup does again for its rows decides whether that pays (gemm_fuses_rmsnorm).
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int NW, int U, int EPI, bool NORM>
__global__ __launch_bounds__(NW * 64) void k_gemm_f32(const float *__restrict__ A, const float *__restrict__ W, int N, int K, Rows rows,
                                                      float *out, int ldo, const float *__restrict__ norm_w, float eps) {
  constexpr int NB = EPI == EPI_SILU_MUL ? 2 : 1;
  __shared__ f32x4 part[NB][NW][64];
  __shared__ float squares[NORM ? NW : 1][64];
  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  const int ncol = N / NB, n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, kq = (lane >> 4) * 4;
  const float *pa = A + (size_t)min(m0 + r, M - 1) * K, *pw[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) pw[b] = W + (size_t)(b * ncol + min(n0 + r, ncol - 1)) * K;
  f32x4 acc[NB], va[U], vw[NB][U], vn[U];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto load = [&](int c) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c + u * NW) * 16 + kq;
      const bool in = k < K;                              // K is a multiple of 4: a piece is inside or outside as a whole
      va[u] = in ? *(const f32x4 *)(pa + k) : zero;
      if (NORM) vn[u] = in ? *(const f32x4 *)(norm_w + k) : zero;
#pragma unroll
      for (int b = 0; b < NB; ++b) vw[b][u] = in ? *(const f32x4 *)(pw[b] + k) : zero;
    }
  };
  if (m0 >= M) return;                                    // first: a launch without rows (blocks that are not finished) ends 1 us earlier
  load(wave);
  float old[4];                                           // EPI_ADD_F32: what the first wavefront adds to
  if (EPI == EPI_ADD_F32 && wave == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i) old[i] = out[(size_t)min(m0 + kq + i, M - 1) * ldo + min(n0 + r, ncol - 1)];
  loads_asked_for();
  float inv = 0.f;                                        // of row r
  if (NORM) {
    float q[U], qw[NW];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = va[u][0] * va[u][0] + va[u][1] * va[u][1] + va[u][2] * va[u][2] + va[u][3] * va[u][3];
#pragma unroll
    for (int h = U / 2; h > 0; h /= 2)
#pragma unroll
      for (int u = 0; u < h; ++u) q[u] += q[u + h];
    squares[wave][lane] = q[0];
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) qw[w] = squares[w][lane];
#pragma unroll
    for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
      for (int w = 0; w < h; ++w) qw[w] += qw[w + h];
    float ss = qw[0] + __shfl_xor(qw[0], 32);
    ss += __shfl_xor(ss, 16);
    inv = 1.0f / sqrtf(ss / (float)K + eps);
  }
  for (int c = wave; c * 16 < K; c += NW * U) {
    if (c != wave) load(c);
    if (NORM)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) va[u][e] = va[u][e] * inv * vn[u][e];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u][e], vw[b][u][e], acc[b], 0, 0, 0);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) part[b][wave][lane] = acc[b];
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 1; w < NW; ++w)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] += part[b][w][lane];
  // register i of lane l is C[4 * (l / 16) + i][l % 16]
  const int gn = n0 + r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int gm = m0 + kq + i;
    if (gm >= M || gn >= ncol) continue;
    float *o = out + (size_t)gm * ldo + gn;
    if (EPI == EPI_SILU_MUL) *o = acc[0][i] / (1.0f + __expf(-acc[0][i])) * acc[NB - 1][i];
    else if (EPI == EPI_ADD_F32) *o = old[i] + acc[0][i];
    else *o = acc[0][i];
  }
}

template <int NW, int U, bool NORM>
static void launch_f32(hipStream_t s, const float *A, const float *W, int N, int K, Rows rows, int epi, float *out, int ldo, const float *norm_w = nullptr,
                       float eps = 0.f) {
  const dim3 grid(((epi == EPI_SILU_MUL ? N / 2 : N) + 15) / 16, (rows.cap + 15) / 16);
  if (epi == EPI_SILU_MUL) k_gemm_f32<NW, U, EPI_SILU_MUL, NORM><<<grid, NW * 64, 0, s>>>(A, W, N, K, rows, out, ldo, norm_w, eps);
  else if (epi == EPI_ADD_F32) k_gemm_f32<NW, U, EPI_ADD_F32, NORM><<<grid, NW * 64, 0, s>>>(A, W, N, K, rows, out, ldo, norm_w, eps);
  else k_gemm_f32<NW, U, EPI_STORE_F32, NORM><<<grid, NW * 64, 0, s>>>(A, W, N, K, rows, out, ldo, norm_w, eps);
}
// 16-byte loads need K a multiple of 4 and aligned operands.  A workgroup reads its operands without sharing them, so from about 1024
// tiles of 64 x 64 on k_gemm_valu is the faster one (rows x N x K, us, valu / this: 64 x 1024 x 1024 136 / 6, 1024 x 1024 x 1024
// 181 / 60, 256 x 4096 x 2048 366 / 117, 1024 x 4096 x 2048 428 / 449, 4096 x 4096 x 2048 1394 / 1772).
static bool takes_f32(const void *A, const void *W, int N, int K, int rows_cap) {
  return K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0 && (long)((rows_cap + 63) / 64) * ((N + 63) / 64) < 1024;
}

// ---------------------------------------------------------------------------------------------
// bf16 on the matrix cores.
//
// Workgroup = 4 wavefronts (2 x 2), macro tile BM x BN x 64; each wavefront owns a (BM/2) x (BN/2) patch as
// 32x32 accumulator tiles of v_mfma_f32_32x32x16_bf16.  Both operands are K-contiguous, so A rows and W rows
// feed the instruction the same way: lane l supplies row l % 32, eight consecutive k starting at 8 * (l / 32).
//
// LDS holds one K-slab of each operand, rows of 64 bf16 = 128 B = eight 16-byte chunks; chunk c of row r is
// stored at chunk position c ^ ((r >> 1) & 7), so the 32 rows read by one ds_read_b128 spread over all banks and
// the 8 lanes that fill a row write distinct chunks.  The next K-slab is fetched from global memory into
// registers while the current one is multiplied (two workgroups per CU overlap each other's barriers).
//
// Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; the id is remapped so that each XCD
// works on one contiguous range of tiles (ordered in groups of 8 tile rows), which keeps the A and W panels a
// range touches inside that XCD's own L2.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int EPI>
__global__ __launch_bounds__(256, 2) void k_gemm_mfma(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W, int N, int K,
                                                      Rows rows, void *out, int ldo, int tiles_m, int tiles_n) {
  constexpr int BK = 64, WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;
  constexpr int CA = BM * 8 / 256, CB = BN * 8 / 256;      // 16-byte chunks per thread and K-slab
  __shared__ __attribute__((aligned(16))) unsigned char As[BM * 128];
  __shared__ __attribute__((aligned(16))) unsigned char Bs[BN * 128];

  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  // XCD-aware tile order over the tile rows that hold valid rows (the grid is sized for rows.cap; with a row count that
  // only the device knows, the live tiles still spread over all 8 XCDs and the workgroups beyond them exit)
  tiles_m = min(tiles_m, (M + BM - 1) / BM);
  const int total = tiles_m * tiles_n;
  const int per_xcd = (total + 7) / 8;
  const int tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (blockIdx.x / 8 >= per_xcd || tile >= total) return;
  constexpr int GROUP = 8;
  const int in_group = tile % (GROUP * tiles_n), first_m = (tile / (GROUP * tiles_n)) * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int m0 = (first_m + in_group % gsz) * BM, n0 = (in_group / gsz) * (EPI == EPI_SILU_MUL ? BN / 2 : BN);
  if (m0 >= M) return;
  static_assert(EPI != EPI_SILU_MUL || BN == 128, "the fused SiLU*up epilogue pairs the two column tiles of a wavefront");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;

  // global -> register -> LDS staging: chunk id = tid + 256 * i -> (row, chunk)
  const bf16_t *ga[CA], *gb[CB];
  int sa[CA], sb[CB];
#pragma unroll
  for (int i = 0; i < CA; ++i) {
    int c = tid + 256 * i, r = c >> 3, ch = c & 7;
    ga[i] = A + (size_t)min(m0 + r, M - 1) * K + ch * 8;
    sa[i] = r * 128 + ((ch ^ ((r >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    int c = tid + 256 * i, r = c >> 3, ch = c & 7;
    // fused SiLU*up: the two 32-column accumulator tiles of a wavefront are the gate and the up projection of
    // the same 32 activation columns, so LDS row r holds gate row n0 + ... for even 32-row groups and the
    // matching up row (F rows further) for odd ones
    const int wrow = EPI == EPI_SILU_MUL ? ((r >> 5) & 1) * (N / 2) + n0 + (r / WN) * 32 + (r & 31) : n0 + r;
    gb[i] = W + (size_t)min(wrow, N - 1) * K + ch * 8;
    sb[i] = r * 128 + ((ch ^ ((r >> 1) & 7)) << 4);
  }
  u32x4 ra[CA], rb[CB];
#pragma unroll
  for (int i = 0; i < CA; ++i) ra[i] = *(const u32x4 *)(ga[i]);
#pragma unroll
  for (int i = 0; i < CB; ++i) rb[i] = *(const u32x4 *)(gb[i]);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment addresses: row = base + (lane & 31), logical chunk = 2 * ks + (lane >> 5)
  const int frow = lane & 31, fch = lane >> 5;
  const int nk = K / BK;
  for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
    for (int i = 0; i < CA; ++i) *(u32x4 *)(As + sa[i]) = ra[i];
#pragma unroll
    for (int i = 0; i < CB; ++i) *(u32x4 *)(Bs + sb[i]) = rb[i];
    __syncthreads();
    {
      // the last iteration re-reads its own slab: an unconditional load keeps the staging registers in VGPRs
      const size_t koff = (size_t)min(kt + 1, nk - 1) * BK;
#pragma unroll
      for (int i = 0; i < CA; ++i) ra[i] = *(const u32x4 *)(ga[i] + koff);
#pragma unroll
      for (int i = 0; i < CB; ++i) rb[i] = *(const u32x4 *)(gb[i] + koff);
    }
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        int r = wm + i * 32 + frow;
        af[i] = *(const bf16x8 *)(As + r * 128 + (((2 * ks + fch) ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        int r = wn + j * 32 + frow;
        bfr[j] = *(const bf16x8 *)(Bs + r * 128 + (((2 * ks + fch) ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // epilogue: accumulator register r of lane l is C[8 * (r / 4) + 4 * (l / 32) + r % 4][l % 32] of its 32x32 tile
  if (EPI == EPI_SILU_MUL) {
    const int gn = n0 + (wn / WN) * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int gm = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const float g = acc[i][0][r], u = acc[i][TN - 1][r];
        if (gm < M && gn < N / 2) ((bf16_t *)out)[(size_t)gm * ldo + gn] = (bf16_t)(g / (1.0f + __expf(-g)) * u);
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int gn = n0 + wn + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int gm = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (gm < M && gn < N) store_out<bf16_t, EPI>(out, (size_t)gm * ldo + gn, acc[i][j][r]);
      }
    }
}

template <int BM, int BN>
static void launch_mfma(hipStream_t s, const void *A, const void *W, int N, int K, Rows rows, int epi, void *out, int ldo) {
  const int tiles_m = (rows.cap + BM - 1) / BM;
  const int tiles_n = epi == EPI_SILU_MUL ? (N / 2 + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
  const int grid = ((tiles_m * tiles_n + 7) / 8) * 8;
  const bf16_t *a = (const bf16_t *)A, *w = (const bf16_t *)W;
  if (epi == EPI_SILU_MUL) k_gemm_mfma<BM, BN, EPI_SILU_MUL><<<grid, 256, 0, s>>>(a, w, N, K, rows, out, ldo, tiles_m, tiles_n);
  else if (epi == EPI_STORE) k_gemm_mfma<BM, BN, EPI_STORE><<<grid, 256, 0, s>>>(a, w, N, K, rows, out, ldo, tiles_m, tiles_n);
  else if (epi == EPI_ADD_F32) k_gemm_mfma<BM, BN, EPI_ADD_F32><<<grid, 256, 0, s>>>(a, w, N, K, rows, out, ldo, tiles_m, tiles_n);
  else k_gemm_mfma<BM, BN, EPI_STORE_F32><<<grid, 256, 0, s>>>(a, w, N, K, rows, out, ldo, tiles_m, tiles_n);
}

// ---------------------------------------------------------------------------------------------
// BM x 256 x 64 tiles, four wavefronts, one workgroup per CU, K-slabs loaded straight into LDS
// (buffer_load_dwordx4 ... lds: lane l of an instruction fills the 16-byte slot l of a 1 KB block = 8 tile rows, so
// the bank swizzle is applied by choosing which chunk a lane fetches; rows beyond the matrix fall outside the buffer
// descriptor and read as zero), software-pipelined by hand:
//   * the fragments of k-step s + 1 are read from LDS while the MFMAs of step s run (two register sets);
//   * one barrier per slab, placed before the last k-step: by then every wavefront has read all of the current slab
//     and the next one has landed, so the stage of the current slab can be filled again right behind the barrier;
//   * three LDS stages of the weights, and of the rows where they fit (up to 160 of them: 156 KB; above two: 160 KB at 256), so that
//     loads have a whole slab's time more to arrive.  With two stages every height took the same 0.95 us or more for a slab, which
//     is how long a slab takes to come from memory, whatever there was to multiply: 4096 columns, K = 12288, weights from HBM, 256
//     tiles of 64 / 96 / 128 / 160 / 192 / 256 rows 188 / 201 / 214 / 225 / 244 / 322 us, now 140 / 158 / 180 / 204 / 235 / 312.  At 192
//     rows and above it is power that binds (1.6 GHz of 2.4 under real values; the matrix cores busy in 86 % of the cycles of a slab);
//   * loads are spread evenly between the MFMAs (a burst of 8 direct-to-LDS loads per wavefront stalls the matrix pipe for
//     longer than the loads take on their own: measured 37 % of the MFMA rate against 100 % when interleaved), and they
//     take their slab and stage offsets from scalar registers: next to no vector ALU work competes with the MFMAs for issue slots.
// The waits for the loads are explicit, and so is the barrier: the compiler does not order LDS reads behind direct-to-LDS loads, but it
// lets a workgroup fence wait for all of them.
// LDS layout: the stages of the rows, then those of the weights.
#define FK_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// Workgroup barrier that orders LDS traffic only: outstanding global loads (which the kernel waits for by count) are
// not drained, unlike with __syncthreads().
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lane exchanges inside a row of 16 lanes without LDS: CTRL is a data-parallel-primitive pattern (0xB1 / 0x4E: lanes l ^ 1 / l ^ 2
// of a quad, 0x141: lane 7 - l of eight, 0x140: lane 15 - l of sixteen).  All four are permutations, so every lane has a source.
template <int CTRL> __device__ __forceinline__ float lane_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ void lane_max_step(float &m, int &mi) {
  const float om = lane_dpp<CTRL>(m);
  const int oi = __builtin_amdgcn_update_dpp(0, mi, CTRL, 0xF, 0xF, false);
  if (om > m || (om == m && oi < mi)) { m = om; mi = oi; }     // equal maxima: the lower column
}

constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }   // s_waitcnt vmcnt(n) only
constexpr int pipe_stages_a(int bm) { return bm <= 160 ? 3 : 2; }
constexpr int kPipeStagesW = 3;
constexpr int kNonTemporal = 2;      // cache policy of a load (NT bit): what is read once does not push other lines out

// ONE: the launch has one row of tiles, so that every weight is read by one workgroup only, past the caches (151936 columns, K = 4096:
// 8 rows 217 us, 232 with plain loads; 128 rows 233 and 248; with two and more rows of tiles it is the same or slower, 374 -> 382)
template <int BM, int EPI, int BN = 256, bool ONE = false>
__global__ __launch_bounds__(256, 1) void k_gemm_pipe(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W, int N, int K,
                                                      Rows rows, void *out, int ldo, int tiles_m, int tiles_n, int splits,
                                                      size_t split_stride, float *logits) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer-resource builtins exist in the device pass only
  // splits > 1: the K range is cut into `splits` parts, one workgroup each; part s writes its fp32 sums to
  // out + s * split_stride and a second kernel adds the parts in order (EPI is then EPI_STORE_F32 or EPI_PARTIAL_SILU)
  constexpr bool SILU_W = EPI == EPI_SILU_MUL || EPI == EPI_PARTIAL_SILU;
  // BM = 256: wavefronts 2 x 2, each 128 x BN/2 (the fewest LDS reads per MFMA; accumulators in the 256 accumulation registers a lone
  // wavefront per SIMD can have).  Otherwise the wavefronts lie side by side, each BM x 64, so that BM may be any multiple of 32: the
  // height that fits the row count.  (Eight wavefronts, 2 x 4, were slower at every height: 2048 x 4096 x 12288, K cut in two, 185 us
  // against 176; BM = 128 229 against 208.)
  // BN = 192 exists for launches whose 256-wide tiles would leave a quarter of the CUs idle
  constexpr int NW = 4, WROWS = BM == 256 ? 2 : 1;
  constexpr int BK = 64, WCOLS = NW / WROWS, WM = BM / WROWS, WN = BN / WCOLS, TM = WM / 32, TN = WN / 32;
  static_assert(WM % 32 == 0 && WN % 32 == 0 && (BM / 8) % NW == 0 && (BN / 8) % NW == 0 && (!SILU_W || TN % 2 == 0), "tile shape");
  constexpr int IA = BM / 8 / NW, IB = BN / 8 / NW, NI = IA + IB;
  constexpr int SA = pipe_stages_a(BM), SW = kPipeStagesW;
  constexpr int ASTAGE = BM * 128, WSTAGE = BN * 128, WBASE = SA * ASTAGE, NMF = TM * TN;
  // Loads of a window (barrier to barrier, four k-steps): the rows first, then the weights, a quarter in each k-step
  constexpr int L0 = (NI + 3) / 4, L1 = (NI - L0 + 2) / 3, L2 = (NI - L0 - L1 + 1) / 2, L3 = NI - L0 - L1 - L2;
  static_assert(L0 <= NMF && TM + TN <= NMF, "one load and one fragment read per MFMA at most");
  // Loads that may still be on their way at the barrier.  The slab that comes next was asked for in the window before this one, but with
  // two stages its rows in this window: so those behind them, all of this window's or the weights.
  constexpr int FLY = SA > 2 ? NI : IB;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_pipe[];
  unsigned char *const lds = lds_pipe;
  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  // the tile list covers the tile rows that hold valid rows: the grid is sized for rows.cap, and with a row count that only the
  // device knows the live tiles still spread evenly over the 8 XCDs (workgroups beyond them exit at once)
  tiles_m = min(tiles_m, (M + BM - 1) / BM);
  const int total = tiles_m * tiles_n * splits;
  const int per_xcd = (total + 7) / 8;
  const int work = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (blockIdx.x / 8 >= per_xcd || work >= total) return;
  const int tile = work / splits, split = work % splits;
  constexpr int GROUP = 8;
  const int in_group = tile % (GROUP * tiles_n), first_m = (tile / (GROUP * tiles_n)) * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int m0 = (first_m + in_group % gsz) * BM, n0 = (in_group / gsz) * (SILU_W ? BN / 2 : BN);
  if (m0 >= M) return;
  out = (void *)((float *)out + (size_t)split * split_stride);   // (split is 0 unless the output is fp32 partial sums)
  const int nk = K / BK / splits;                                 // slabs of this workgroup
  const unsigned k_base = (unsigned)split * (unsigned)nk * (BK * 2);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / WCOLS) * WM, wn = (wave % WCOLS) * WN;
  // raw buffers over the valid rows: an offset at or beyond the size reads zero without touching memory
  __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc((void *)A, 0, (unsigned)M * (unsigned)K * 2u, 0x00020000);
  __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, (unsigned)N * (unsigned)K * 2u, 0x00020000);
  // per-lane byte offsets of this wavefront's load instructions: instruction q covers tile rows (wave * I + q) * 8 .. + 7
  unsigned voa[IA], vob[IB];
#pragma unroll
  for (int q = 0; q < IA; ++q) {
    const int r = (wave * IA + q) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    voa[q] = (unsigned)(m0 + r) * (unsigned)K * 2u + k_base + c * 16;
  }
#pragma unroll
  for (int q = 0; q < IB; ++q) {
    const int r = (wave * IB + q) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    // fused SiLU*up: LDS rows 64 c .. 64 c + 31 hold the gate rows of output columns 32 c .. 32 c + 31, the next 32 rows the
    // matching up rows, so that a wavefront's column tiles 2 p and 2 p + 1 are gate and up of the same columns
    const int wrow = SILU_W ? ((r >> 5) & 1) * (N / 2) + n0 + (r / 64) * 32 + (r & 31) : n0 + r;
    vob[q] = (unsigned)wrow * (unsigned)K * 2u + k_base + c * 16;
  }
  // load instruction i (A: 0 .. IA-1, W: IA .. NI-1) of the slabs at byte offsets so_a, so_w into the stages at byte offsets st_a, st_w
  auto gl = [&](int i, unsigned so_a, int st_a, unsigned so_w, int st_w) {
    if (i < IA)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, FK_LDS_PTR(lds + st_a + (wave * IA + (i < IA ? i : 0)) * 1024), 16, voa[i < IA ? i : 0], so_a, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, FK_LDS_PTR(lds + WBASE + st_w + (wave * IB + (i < IA ? 0 : i - IA)) * 1024), 16,
                                               vob[i < IA ? 0 : i - IA], so_w, 0, ONE ? kNonTemporal : 0);
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // fragment addresses: row = base + (lane & 31), logical chunk 2 * ks + (lane >> 5), swizzled with the row (all 32-row
  // tiles start at a multiple of 32, so the swizzle depends on the lane only)
  const int frow = lane & 31, fch = lane >> 5, sw = (frow >> 1) & 7;
  const unsigned char *pa[4], *pb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    pa[ks] = lds + (wm + frow) * 128 + (((2 * ks + fch) ^ sw) << 4);
    pb[ks] = lds + WBASE + (wn + frow) * 128 + (((2 * ks + fch) ^ sw) << 4);
  }
  bf16x8 fa[2][TM], fb[2][TN];
  auto rd = [&](int s, int ks, int st_a, int st_w, int slot) {   // s-th fragment read of a k-step, in the order the MFMAs need them
    const int f = s == 0 ? TM : (s == 1 ? 0 : (s <= TN ? TM + s - 1 : s - TN));   // W0, A0, W1 .. W(TN-1), A1 .. A(TM-1)
    if (f < TM) fa[slot][f < TM ? f : 0] = *(const bf16x8 *)(pa[ks] + st_a + (f < TM ? f : 0) * 4096);
    else fb[slot][f < TM ? 0 : f - TM] = *(const bf16x8 *)(pb[ks] + st_w + (f < TM ? 0 : f - TM) * 4096);
  };
  auto slab_off = [&](int kt) { return kt < nk ? (unsigned)kt * (BK * 2) : 0x80000000u; };   // beyond the last slab nothing is moved
  // before the loop: the rows of slabs 0 .. SA - 2 and the weights of slabs 0 .. SW - 2, and the first k-step's share of the window that
  // ends at the first barrier
#pragma unroll
  for (int q = 0; q < SW - 1; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (i >= IA || q < SA - 1) gl(i, slab_off(q), q * ASTAGE, slab_off(q), q * WSTAGE);
#pragma unroll
  for (int i = 0; i < L0; ++i) gl(i, slab_off(SA - 1), (SA - 1) * ASTAGE, slab_off(SW - 1), (SW - 1) * WSTAGE);
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(L0 + (SW - 2) * IB + (SA - 2) * IA));   // slab 0 has landed
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int s = 0; s < TM + TN; ++s) rd(s, 0, 0, 0, 0);

  // one k-step: the MFMAs on register set `cur`; behind MFMA s, fragment read s of the next k-step, and (when nl > 0)
  // a load on every NMF / nl-th MFMA
#define FK_STEP(cur, next_ks, ra, rw, nl, lfirst, so_a, st_a, so_w, st_w)                               \
  {                                                                                                     \
    _Pragma("unroll") for (int s = 0; s < NMF; ++s) {                                                   \
      const int i = s / TN, j = s % TN;                                                                 \
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);  \
      if (s < TM + TN) rd(s, next_ks, ra, rw, (cur) ^ 1);                                               \
      if ((nl) > 0 && s % (NMF / ((nl) > 0 ? (nl) : 1)) == NMF / ((nl) > 0 ? (nl) : 1) - 1 && s / (NMF / ((nl) > 0 ? (nl) : 1)) < (nl)) \
        gl((lfirst) + s / (NMF / ((nl) > 0 ? (nl) : 1)), so_a, st_a, so_w, st_w);                       \
      __builtin_amdgcn_sched_barrier(0);                                                                \
    }                                                                                                   \
  }
  int ra = 0, rw = 0;                                       // stages of the slab that is multiplied
  int la = (SA - 1) * ASTAGE, lw = (SW - 1) * WSTAGE;       // stages that are filled: the ones the slab before it has left
  for (int kt = 0; kt < nk; ++kt) {
    unsigned so_a = slab_off(kt + SA - 1), so_w = slab_off(kt + SW - 1);
    FK_STEP(0, 1, ra, rw, L1, L0, so_a, la, so_w, lw)
    FK_STEP(1, 2, ra, rw, L2, L0 + L1, so_a, la, so_w, lw)
    FK_STEP(0, 3, ra, rw, L3, L0 + L1 + L2, so_a, la, so_w, lw)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(FLY));                     // this wavefront's part of the next slab has landed
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // ... and everyone's; everyone has read all of this slab
    la = ra; lw = rw;
    ra = ra == (SA - 1) * ASTAGE ? 0 : ra + ASTAGE;
    rw = rw == (SW - 1) * WSTAGE ? 0 : rw + WSTAGE;
    so_a = slab_off(kt + SA); so_w = slab_off(kt + SW);
    FK_STEP(1, 0, ra, rw, L0, 0, so_a, la, so_w, lw)
  }
#undef FK_STEP
  __builtin_amdgcn_s_waitcnt(0x0F70);
  // epilogue: accumulator register r of lane l is C[8 * (r / 4) + 4 * (l / 32) + r % 4][l % 32] of its 32x32 tile.
  // A tile that lies inside the matrix takes the path without per-element bounds checks.
  const bool inside = m0 + BM <= M && n0 + (SILU_W ? BN / 2 : BN) <= (SILU_W ? N / 2 : N);
  const int erow = m0 + wm + 4 * (lane >> 5), ecol = lane & 31;
  if (EPI == EPI_SILU_MUL) {
#pragma unroll
    for (int jp = 0; jp < TN / 2; ++jp) {
      const int gn = n0 + (wn / 64 + jp) * 32 + ecol;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int gm = erow + i * 32 + 8 * (r >> 2) + (r & 3);
          const float g = acc[i][2 * jp][r], u = acc[i][2 * jp + 1][r];
          if (inside || (gm < M && gn < N / 2)) ((bf16_t *)out)[(size_t)gm * ldo + gn] = (bf16_t)(g / (1.0f + __expf(-g)) * u);
        }
    }
    return;
  }
  if (EPI == EPI_PARTIAL_SILU) {   // fp32 partial sums in weight-row order: gate of column c at c, up at N / 2 + c
#pragma unroll
    for (int jp = 0; jp < TN / 2; ++jp) {
      const int gn = n0 + (wn / 64 + jp) * 32 + ecol;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int gm = erow + i * 32 + 8 * (r >> 2) + (r & 3);
          if (inside || (gm < M && gn < N / 2)) {
            ((float *)out)[(size_t)gm * ldo + gn] = acc[i][2 * jp][r];
            ((float *)out)[(size_t)gm * ldo + N / 2 + gn] = acc[i][2 * jp + 1][r];
          }
        }
    }
    return;
  }
  if (EPI == EPI_CONF || EPI == EPI_CONF_LOGITS) {
    // per row: (maximum, sum exp(x - maximum), lowest column of the maximum) over this wavefront's WN columns.  The accumulators
    // hold a row spread over 32 lanes; each 32 x WN patch goes through a private LDS area (the operand stages are free: every
    // load has landed) and comes back with two lanes per row, each holding half of the row's columns in order, so that the
    // reductions run inside a lane and one exchange with the neighbour lane finishes them.
    if (EPI == EPI_CONF_LOGITS) {
      // the products themselves are wanted too, [M, N] (276 rows x 151936: 58 us less than reading them again); the descriptor ends at the
      // last valid row, as below
      const __amdgpu_buffer_rsrc_t rs_l = __builtin_amdgcn_make_buffer_rsrc(logits + (size_t)m0 * N, 0, (unsigned)min(BM, M - m0) * (unsigned)N * 4u, 0x00020000);
      unsigned at[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int gn = n0 + wn + j * 32 + ecol;
        at[j] = gn < N ? ((unsigned)(erow - m0) * (unsigned)N + (unsigned)gn) * 4u : 0x80000000u;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r]), rs_l, at[j], (unsigned)(i * 32 + 8 * (r >> 2) + (r & 3)) * (unsigned)N * 4u, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    constexpr int XS = WN + 4;                               // padded row: two lanes per row read 16-byte pieces
    static_assert(NW * 32 * XS * 4 <= 2 * (BM + BN) * 128, "transpose area");
    lds_barrier();                                           // everybody's loads have landed, nobody reads operands any more
    float *xp = (float *)lds + wave * (32 * XS);
    const int slot = (n0 / BN) * WCOLS + wn / WN;
    const int xrow = lane >> 1, xpart = lane & 1;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const bool ok = n0 + wn + j * 32 + ecol < N;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          xp[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * XS + j * 32 + ecol] = ok ? acc[i][j][r] : -INFINITY;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
      const float4 *src = (const float4 *)(xp + xrow * XS + xpart * (WN / 2));
      float4 v[WN / 8];
#pragma unroll
      for (int k = 0; k < WN / 8; ++k) v[k] = src[k];
      float m = -INFINITY;
      int mi = 0x7fffffff;
      const int c0 = n0 + wn + xpart * (WN / 2);
#pragma unroll
      for (int k = 0; k < WN / 8; ++k) {                     // ascending columns: the first maximum stays
        if (v[k].x > m) { m = v[k].x; mi = c0 + 4 * k; }
        if (v[k].y > m) { m = v[k].y; mi = c0 + 4 * k + 1; }
        if (v[k].z > m) { m = v[k].z; mi = c0 + 4 * k + 2; }
        if (v[k].w > m) { m = v[k].w; mi = c0 + 4 * k + 3; }
      }
      lane_max_step<0xB1>(m, mi);                            // the row's other half (lane l ^ 1)
      float sum = 0.f;
      if (m > -INFINITY) {
#pragma unroll
        for (int k = 0; k < WN / 8; ++k) sum += __expf(v[k].x - m) + __expf(v[k].y - m) + __expf(v[k].z - m) + __expf(v[k].w - m);
      }
      sum += lane_dpp<0xB1>(sum);
      const int gm = m0 + wm + i * 32 + xrow;
      if (xpart == 0 && gm < M) {
        float *p = (float *)out + ((size_t)gm * ldo + slot) * 3;
        p[0] = m; p[1] = sum; p[2] = __int_as_float(mi);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();                       // the patch is rewritten by the next row tile
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    }
    return;
  }
  if (EPI == EPI_ADD_F32) {
    // through a descriptor that ends at the last valid row (a column beyond N is moved beyond its end): what lies outside the matrix
    // reads as zero and is not stored, so that full and remainder tiles alike read a whole row of 32x32 tiles before they add and
    // store (element by element under a bounds check, a remainder tile waited for memory once per accumulator: 4096 columns, K = 4096,
    // weights from HBM, 2185 rows 105 us, now 78; 3800 rows 180, now 115; K = 12288 247 / 215 and 394 / 302)
    const __amdgpu_buffer_rsrc_t rs_o =
        __builtin_amdgcn_make_buffer_rsrc((float *)out + (size_t)m0 * ldo, 0, (unsigned)min(BM, M - m0) * (unsigned)ldo * 4u, 0x00020000);
    unsigned col[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int gn = n0 + wn + j * 32 + ecol;
      col[j] = gn < N ? ((unsigned)(erow - m0) * (unsigned)ldo + (unsigned)gn) * 4u : 0x80000000u;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float old[TN][16];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          old[j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_o, col[j] + (unsigned)(i * 32 + 8 * (r >> 2) + (r & 3)) * (unsigned)ldo * 4u, 0, 0));
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(old[j][r] + acc[i][j][r]), rs_o,
                                                col[j] + (unsigned)(i * 32 + 8 * (r >> 2) + (r & 3)) * (unsigned)ldo * 4u, 0, 0);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int gn = n0 + wn + j * 32 + ecol;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int gm = erow + i * 32 + 8 * (r >> 2) + (r & 3);
        if (inside || (gm < M && gn < N)) store_out<bf16_t, EPI == EPI_PARTIAL_SILU ? EPI_STORE_F32 : EPI>(out, (size_t)gm * ldo + gn, acc[i][j][r]);
      }
    }
#endif
}

// Adds the fp32 partial sums of a K-split projection in split order and applies the epilogue.  Bound by the partial sums.  The row count may
// lie far below the bound that the parts are laid out for, so it is read first (722 of 8192 rows, 4096 columns: 102 us when every row of the
// bound was read before the count, 11.5 now).  There are workgroups for the expected rows, at most the kReduceGroups that run at once: each
// waits for the count once, not in every round (1600 rows 18.9 us, 20.4 with all workgroups).  The first kReduceEarly of them ask for their loads
// before the count, 10 MB for two parts, so that memory is busy meanwhile.  FEW (at most kFewRows rows): one trip, all loads before the count; a
// step of one request gains half a percent.
constexpr size_t kReduceGroups = 2048;
constexpr unsigned kReduceEarly = 512;
template <int EPI, bool FEW>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float *__restrict__ part, int splits, size_t split_stride, Rows rows, int N,
                                                       void *out, int ldo) {
  constexpr int U = 4;
  const int ncol = EPI == EPI_SILU_MUL ? N / 2 : N, per_row = ncol / 4;
  size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  float4 v[U], u[U];
  float old[4];
  auto load = [&](int m, int c, int s0) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const float *q = part + (size_t)m * N + c + (size_t)min(s0 + i, splits - 1) * split_stride;
      v[i] = *(const float4 *)q;
      if (EPI == EPI_SILU_MUL) u[i] = *(const float4 *)(q + N / 2);
    }
    if (EPI == EPI_ADD_F32 && s0 == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) old[i] = ((const float *)out)[(size_t)m * ldo + c + i];
  };
  bool early = FEW || blockIdx.x < kReduceEarly;
  if (early) load(min((int)(idx / per_row), rows.cap - 1), (int)(idx % per_row) * 4, 0);
  loads_asked_for();
  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  for (;; idx += (size_t)gridDim.x * 256) {
    const int m = (int)(idx / per_row), c = (int)(idx % per_row) * 4;
    if (m >= M) return;
    if (!early) load(m, c, 0);
    early = false;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    for (int s0 = 0; s0 < splits; s0 += U) {
      if (s0 > 0) load(m, c, s0);
#pragma unroll
      for (int i = 0; i < U; ++i)
        if (s0 + i < splits) {
          a.x += v[i].x; a.y += v[i].y; a.z += v[i].z; a.w += v[i].w;
          if (EPI == EPI_SILU_MUL) { b.x += u[i].x; b.y += u[i].y; b.z += u[i].z; b.w += u[i].w; }
        }
    }
    const float r[4] = {a.x, a.y, a.z, a.w}, up[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t o = (size_t)m * ldo + c + i;
      if (EPI == EPI_SILU_MUL) ((bf16_t *)out)[o] = (bf16_t)(r[i] / (1.0f + __expf(-r[i])) * up[i]);
      else if (EPI == EPI_ADD_F32) ((float *)out)[o] = old[i] + r[i];
      else store_out<bf16_t, EPI>(out, o, r[i]);
    }
    if (FEW) return;
  }
}

template <int BM, int EPI, int BN = 256, bool ONE = false>
static bool launch_pipe(hipStream_t s, const bf16_t *a, const bf16_t *w, int N, int K, Rows rows, void *out, int ldo, int splits = 1,
                        size_t split_stride = 0, float *logits = nullptr) {
  constexpr int kLds = (pipe_stages_a(BM) * BM + kPipeStagesW * BN) * 128;
  constexpr bool SILU_W = EPI == EPI_SILU_MUL || EPI == EPI_PARTIAL_SILU;
  if constexpr (!ONE && BM <= 128 && (EPI == EPI_CONF || EPI == EPI_CONF_LOGITS || EPI == EPI_STORE_F32 || EPI == EPI_PARTIAL_SILU))      // projections of few rows
    if (rows.expected() <= BM) return launch_pipe<BM, EPI, BN, true>(s, a, w, N, K, rows, out, ldo, splits, split_stride, logits);
  static bool ready = false;             // the dynamic LDS size has to be allowed once per kernel
  if (!ready) {
    if (hipFuncSetAttribute((const void *)k_gemm_pipe<BM, EPI, BN, ONE>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess) return false;
    ready = true;
  }
  const int tiles_m = (rows.cap + BM - 1) / BM, tiles_n = SILU_W ? (N / 2 + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
  const int grid = ((tiles_m * tiles_n * splits + 7) / 8) * 8;
  k_gemm_pipe<BM, EPI, BN, ONE><<<grid, 256, kLds, s>>>(a, w, N, K, rows, out, ldo, tiles_m, tiles_n, splits, split_stride, logits);
  return true;
}

template <int BM>
static bool launch_pipe_epi(hipStream_t s, const bf16_t *a, const bf16_t *w, int N, int K, Rows rows, int epi, void *out, int ldo, int splits,
                            size_t split_stride, float *logits) {
  switch (epi) {
    case EPI_STORE: return launch_pipe<BM, EPI_STORE>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_ADD_F32: return launch_pipe<BM, EPI_ADD_F32>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_STORE_F32: return launch_pipe<BM, EPI_STORE_F32>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_SILU_MUL: return launch_pipe<BM, EPI_SILU_MUL>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_PARTIAL_SILU: return launch_pipe<BM, EPI_PARTIAL_SILU>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_CONF: return launch_pipe<BM, EPI_CONF>(s, a, w, N, K, rows, out, ldo, splits, split_stride);
    case EPI_CONF_LOGITS:
      if constexpr (BM < 256) return launch_pipe<BM, EPI_CONF_LOGITS>(s, a, w, N, K, rows, out, ldo, splits, split_stride, logits);
      else return false;
  }
  return false;
}

// Shape of a pipelined launch: tile height, tile width and parts of K.
struct PipeShape { int bm, bn, splits; };

static bool launch_shape(hipStream_t s, PipeShape p, const void *A, const void *W, int N, int K, Rows rows, int epi, void *out, int ldo,
                         size_t split_stride = 0, float *logits = nullptr) {
  const bf16_t *a = (const bf16_t *)A, *w = (const bf16_t *)W;
  if (p.bn == 192)
    return epi == EPI_STORE     ? launch_pipe<256, EPI_STORE, 192>(s, a, w, N, K, rows, out, ldo)
           : epi == EPI_ADD_F32 ? launch_pipe<256, EPI_ADD_F32, 192>(s, a, w, N, K, rows, out, ldo)
                                : launch_pipe<256, EPI_STORE_F32, 192>(s, a, w, N, K, rows, out, ldo);
  switch (p.bm) {
    case 64: return launch_pipe_epi<64>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
    case 96: return launch_pipe_epi<96>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
    case 128: return launch_pipe_epi<128>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
    case 160: return launch_pipe_epi<160>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
    case 192: return launch_pipe_epi<192>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
    case 224: return launch_pipe_epi<224>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
  }
  return launch_pipe_epi<256>(s, a, w, N, K, rows, epi, out, ldo, p.splits, split_stride, logits);
}

// The shape with the least estimated time.  A compute unit takes one tile at a time and spends about 0.30 + 0.0046 BM us (0.08 more at
// height 64) on a 64-wide slab of a BM x 256 tile, up to a fifth less when part of the chip is idle; K cut into parts costs writing the
// fp32 partial sums and reading them back (about 4.4 TB/s), 2.5 us for one more launch, and a microsecond per part.
// Fitted to 207 problems of 129 to 8192 rows (2048 to 24576 columns, K 2048 to 12288, eight weight matrices in turn): the shape taken is
// on average 0.2 % slower than the best one (at most 10 %).  A few of them, us: 2048 x 4096 x 12288 171 in 128 rows, 1310 rows of it 121
// in two parts of 192, 1024 rows 97 in four of 256, 1536 x 6144 x 4096 68 in 160 rows, 777 x 24576 x 4096 138 in 160, 2048 x 2048 x 2048
// 23 in 64.
// (Shapes are chosen for the expected row count; the grids cover rows.cap.)
static PipeShape pipe_shape(int N, int K, Rows rows, int epi, size_t scratch_bytes) {
  static const int heights[] = {256, 224, 192, 160, 128, 96, 64};
  const bool silu = epi == EPI_SILU_MUL;
  const int nk = K / 64, est = rows.expected();
  const double out_mb = (double)est * (silu ? N / 2 : N) * (epi == EPI_ADD_F32 ? 8 : epi == EPI_STORE_F32 ? 4 : 2) * 1e-6;
  PipeShape best{256, 256, 1};
  double best_us = 1e30;
  auto consider = [&](PipeShape p, long tiles, double slab_us) {
    const double rounds = (double)((tiles * p.splits + 255) / 256), idle = 1 - std::min(1.0, tiles * p.splits / 256.0);
    const double us = 4 + rounds * (nk / p.splits) * slab_us * (1 - 0.185 * idle) +
                      (p.splits > 1 ? 2.5 + p.splits + (p.splits * (double)est * N * 4e-6 + out_mb) / 4.4 : 0);
    if (us < best_us) { best_us = us; best = p; }
  };
  for (int bm : heights) {
    const long tiles = (long)((est + bm - 1) / bm) * (silu ? (N / 2 + 127) / 128 : (N + 255) / 256);
    for (int splits = 1; splits <= 16; splits *= 2) {
      // at least four slabs per part; an even number of them, which the kernel does not need but every shape that was measured had; sums in
      // 16-byte pieces
      if (splits > 1 && (nk % (splits * 2) || nk / splits < 4 || N % 8 || (size_t)splits * rows.cap * N * 4 > scratch_bytes)) break;
      consider(PipeShape{bm, 256, splits}, tiles, 0.30 + 0.0046 * bm + (bm == 64 ? 0.075 : 0));
    }
  }
  if (N % 192 == 0 && (epi == EPI_STORE || epi == EPI_ADD_F32 || epi == EPI_STORE_F32))
    consider(PipeShape{256, 192, 1}, (long)((est + 255) / 256) * (N / 192), 1.115);
  return best;
}

// K-split launch for problems with too few tiles to occupy the chip (few rows: the projection is bound by streaming W,
// and a CU cannot pull more than a fraction of a percent of the HBM bandwidth on its own): `splits` workgroups per tile
// write fp32 partial sums to the scratch buffer, k_splitk_reduce adds them in a fixed order.
template <bool FEW> static void launch_reduce(hipStream_t s, int N, Rows rows, int epi, void *out, int ldo, int splits, const float *scratch) {
  const size_t stride = (size_t)rows.cap * N;
  const size_t quads = (size_t)(FEW ? rows.cap : rows.expected()) * ((epi == EPI_SILU_MUL ? N / 2 : N) / 4);
  const unsigned grid = (unsigned)(FEW ? (quads + 255) / 256 : std::min((quads + 255) / 256, kReduceGroups));
  if (epi == EPI_SILU_MUL) k_splitk_reduce<EPI_SILU_MUL, FEW><<<grid, 256, 0, s>>>(scratch, splits, stride, rows, N, out, ldo);
  else if (epi == EPI_STORE) k_splitk_reduce<EPI_STORE, FEW><<<grid, 256, 0, s>>>(scratch, splits, stride, rows, N, out, ldo);
  else if (epi == EPI_ADD_F32) k_splitk_reduce<EPI_ADD_F32, FEW><<<grid, 256, 0, s>>>(scratch, splits, stride, rows, N, out, ldo);
  else k_splitk_reduce<EPI_STORE_F32, FEW><<<grid, 256, 0, s>>>(scratch, splits, stride, rows, N, out, ldo);
}
static void launch_reduce(hipStream_t s, int N, Rows rows, int epi, void *out, int ldo, int splits, const float *scratch) {
  if (rows.cap <= kFewRows) launch_reduce<true>(s, N, rows, epi, out, ldo, splits, scratch);
  else launch_reduce<false>(s, N, rows, epi, out, ldo, splits, scratch);
}

// Byte offsets of rows, and inside an fp32 output tile, within 32 bits.  An even number of slabs: the kernel takes any, but no shape with an odd
// number was measured, and those stay with k_gemm_mfma.
static bool takes_pipe(int N, int K, int rows_cap) {
  return (double)std::max(rows_cap + 256, N + 256) * K * 2 < 4.0e9 && K % 128 == 0 && N <= 1 << 21;
}

bool gemm_conf_partials(hipStream_t s, int dtype, const void *A, const void *W, int N, int K, Rows rows, float *part, size_t part_bytes,
                        int *n_slots, float *logits) {
  if (rows.cap <= 0 || dtype != FOCUS_BF16 || K % 64 || (((uintptr_t)A | (uintptr_t)W) & 15) || !takes_pipe(N, K, rows.cap)) return false;
  if ((long)((rows.expected() + 127) / 128) * ((N + 255) / 256) < 160) return false;   // a small vocabulary: K-split and materialised logits
  const PipeShape p = pipe_shape(N, K, rows, EPI_CONF, 0);
  if (logits && p.bm == 256) return false;                         // the epilogue that also stores does not fit the registers at that height
  const int slots = (N + 255) / 256 * (p.bm == 256 ? 2 : 4);       // one per wavefront column
  if ((size_t)rows.cap * slots * 12 > part_bytes) return false;
  *n_slots = slots;
  return launch_shape(s, p, A, W, N, K, rows, logits ? EPI_CONF_LOGITS : EPI_CONF, part, slots, 0, logits);
}

bool gemm_fuses_silu_mul(int dtype, const void *A, const void *W, int N, int K, int rows_cap) {
  if (dtype == FOCUS_F32) return N % 2 == 0 && takes_f32(A, W, N, K, rows_cap);
  return dtype == FOCUS_BF16 && K % 64 == 0 && N % 2 == 0 && ((uintptr_t)A & 15) == 0 && ((uintptr_t)W & 15) == 0;
}

// The norm belongs into the projection where a workgroup holds all of K at once and there are few workgroups to do it again: with 512 columns
// up to about 1024 (a step of 128 rows, 4 layers, 321 us fused and 329 apart; 256 rows 508 and 510, 512 rows 886 and 863), with 1024 columns,
// whose pieces fill the registers, 256 (16 rows 294 and 305, 32 rows 402 and 383); with 256 columns always (8 rows 140 and 158, 512 rows 359
// and 378, 2048 rows 1065 and 1069).  K in several trips, each row read twice, never paid (2048 columns, 64 rows: 1483 and 940).
bool gemm_fuses_rmsnorm(int dtype, const float *x, const void *norm_w, const void *W, int N, int K, int rows_cap, int epilogue) {
  if (dtype != FOCUS_F32 || !takes_f32(x, W, N, K, rows_cap) || ((uintptr_t)norm_w & 15)) return false;
  const long tiles = (long)((rows_cap + 15) / 16) * (((epilogue == EPI_SILU_MUL ? N / 2 : N) + 15) / 16);
  return K <= 256 || (K <= 512 && tiles <= 1024) || (K <= 1024 && tiles <= 256);
}
void gemm_of_rmsnorm(hipStream_t s, const float *x, const void *norm_w, float eps, const void *W, int N, int K, Rows rows, int epilogue, void *out, int ldo) {
  if (rows.cap <= 0) return;
  const float *w = (const float *)W, *nw = (const float *)norm_w;
  if (K <= 256) launch_f32<4, 4, true>(s, x, w, N, K, rows, epilogue, (float *)out, ldo, nw, eps);
  else if (K <= 512) launch_f32<8, 4, true>(s, x, w, N, K, rows, epilogue, (float *)out, ldo, nw, eps);
  else launch_f32<8, 8, true>(s, x, w, N, K, rows, epilogue, (float *)out, ldo, nw, eps);
}

void gemm(hipStream_t s, int dtype, const void *A, const void *W, int N, int K, Rows rows, int epilogue,
          void *out, int ldo, Scratch scratch) {
  if (rows.cap <= 0) return;
  if (dtype == FOCUS_F32) {
    if (!takes_f32(A, W, N, K, rows.cap)) launch_valu<float>(s, A, W, N, K, rows, epilogue, out, ldo);
    else if (K >= 512) launch_f32<8, 4, false>(s, (const float *)A, (const float *)W, N, K, rows, epilogue, (float *)out, ldo);
    else launch_f32<4, 4, false>(s, (const float *)A, (const float *)W, N, K, rows, epilogue, (float *)out, ldo);
    return;
  }
  const bool aligned = K % 64 == 0 && ((uintptr_t)A & 15) == 0 && ((uintptr_t)W & 15) == 0;
  if (!aligned) { launch_valu<bf16_t>(s, A, W, N, K, rows, epilogue, out, ldo); return; }
  // one tile of rows and fewer column tiles than CUs: pure weight streaming.  The expert-projection kernel (two workgroups per CU, two
  // weight slabs in flight each) with K cut so that about one workgroup per CU exists (64 rows x 4096 x 4096 16.4 us, 21 with two)
  const int est = rows.expected();
  const bool pipe = takes_pipe(N, K, rows.cap);
  // Up to 32 rows, weights of 96 MB and more in at least 32 column tiles: 64-row tiles of the pipelined kernel with parts of 16 slabs keep
  // more loads in flight (8 rows x 24576 x 4096 41.4 us by the expert-projection kernel, 36.8 in this; x 12288 27.0 and 21.3, x 32768 58 and
  // 47; 32 rows x 24576 42.3 and 39.2; from 64 rows on either may be the faster one, and so with fewer weights).  Whole pairs of parts: measured
  // with two, four and more.
  if (pipe && scratch.ptr && N % 8 == 0 && rows.cap <= 32 && (double)N * K >= 48e6 && N >= 32 * 256 && K % 2048 == 0 &&
      (size_t)(K / 1024) * rows.cap * N * 4 <= scratch.bytes) {
    const bool silu = epilogue == EPI_SILU_MUL;
    const int parts = K / 1024;
    if (launch_shape(s, PipeShape{64, 256, parts}, A, W, N, K, rows, silu ? EPI_PARTIAL_SILU : EPI_STORE_F32, scratch.ptr, N, (size_t)rows.cap * N)) {
      launch_reduce(s, N, rows, epilogue, out, ldo, parts, (const float *)scratch.ptr);
      return;
    }
  }
  if (pipe && scratch.ptr && N % 8 == 0 && rows.cap <= 128 && (epilogue == EPI_SILU_MUL ? (N / 2 + 127) / 128 : (N + 255) / 256) < 160) {
    const int nk = K / 64, tn = epilogue == EPI_SILU_MUL ? (N / 2 + 63) / 64 : (N + 127) / 128;
    int splits = 1;
    while (splits < 16 && (long)tn * (splits * 2) <= 256 && nk % (splits * 2) == 0 && nk / (splits * 2) >= 4 &&
           (size_t)(splits * 2) * rows.cap * N * 4 <= scratch.bytes)
      splits *= 2;
    if ((size_t)splits * rows.cap * N * 4 <= scratch.bytes &&
        gemm_stream_partial(s, A, W, N, K, rows, epilogue == EPI_SILU_MUL, splits, (float *)scratch.ptr)) {
      launch_reduce(s, N, rows, epilogue, out, ldo, splits, (const float *)scratch.ptr);
      return;
    }
  }
  if (pipe) {
    const PipeShape p = pipe_shape(N, K, rows, epilogue, scratch.ptr ? scratch.bytes : 0);
    if (p.splits == 1) {
      if (launch_shape(s, p, A, W, N, K, rows, epilogue, out, ldo)) return;
    } else if (launch_shape(s, p, A, W, N, K, rows, epilogue == EPI_SILU_MUL ? EPI_PARTIAL_SILU : EPI_STORE_F32, scratch.ptr, N, (size_t)rows.cap * N)) {
      launch_reduce(s, N, rows, epilogue, out, ldo, p.splits, (const float *)scratch.ptr);
      return;
    }
  }
  const long tiles_big = (long)((est + 255) / 256) * ((N + 127) / 128);
  if (tiles_big >= 512) launch_mfma<256, 128>(s, A, W, N, K, rows, epilogue, out, ldo);
  else launch_mfma<128, 128>(s, A, W, N, K, rows, epilogue, out, ldo);
}

}  // namespace fk
