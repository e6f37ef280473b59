// Synthesis imaging of calibrated visibilities for gfx950 (arXiv 2604.20640
// Sec. 8.1: gridding, Fourier inversion to a dirty image and synthesized
// beam, Hogbom CLEAN deconvolution).
//
// Conventions (n a power of two; cell = image pixel in radians;
// du = 1 / (n cell) wavelengths):
//   * gridding: nearest cell, iu = floor(u/du + 1/2) + n/2 (likewise v),
//     the product u * (n cell) formed in float64; the conjugate visibility
//     goes to the mirrored cell (n - iu, n - iv); a sample is dropped unless
//     both cells lie in [0, n).  The grid is indexed [iu][iv]; W, the total
//     gridded weight (both copies), is accumulated in float64.
//   * inversion: I[il][im] = Re sum G[iu][iv] e^{+2 pi i ((iu-n/2)(il-n/2) +
//     (iv-n/2)(im-n/2)) / n} / W.  With X = (-1)^(iu+iv) G, the sum is
//     (-1)^(il+im) conj(FFT2(conj X)) (forward FFTs of the LDS Stockham
//     engine), so I = (-1)^(il+im) Re FFT2(conj X) / W.  The 2-D transform
//     is rows, a tiled transpose, rows again; the final step reads the
//     transposed result back.
//   * Hogbom CLEAN in one launch, float32: each iteration subtracts the
//     previous component's beam g * psf[(p - peak + (n/2, n/2)) mod n]
//     (product and difference rounded separately: no contraction) and,
//     in the same sweep, finds the next peak: largest |residual|, ties to
//     the smallest flat index il * n + im.  g = gain * peak (rounded).
//     Stops when |peak| < threshold or after max_iter components.  Every
//     thread owns the same pixels in every sweep, so the only cross-thread
//     step is the reduction of the peak.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "qc.h"
#include "qc_fft.h"
#include "qc_internal.h"

namespace qc {

namespace {

// Gridding takes four consecutive samples per thread.  Neighbouring samples
// (channels of one baseline) mostly share a cell, so runs of equal cells are
// summed first, in the thread and then over the wave, and one atomic per run
// and component reaches memory.  Only the cell itself is added to here; the
// conjugates follow from the finished sums (image_mirror_kernel).  Bound: the
// atomics: 8.1 M samples of 32 antennas onto 1024 x 1024 took 2.3 ms with four
// per sample (14 G/s); runs leave about one sample in nine and the conjugates
// none, 62 us and 6 us for the mirror pass (2.1 TB/s of samples).  Few samples
// are done before a mirror pass would have been launched: they add their
// conjugates themselves (DIRECT).
constexpr int GRID_PER = 4;

template <bool VEC, bool DIRECT>
__global__ void __launch_bounds__(256)
image_grid_kernel(const float* __restrict__ u, const float* __restrict__ v, const float2* __restrict__ vis,
                  const float* __restrict__ weight, int64_t n_vis, int n, double inv_du,
                  float2* __restrict__ grid, double* __restrict__ wsum) {
  __shared__ double red[4];
  const int lane = threadIdx.x & 63;
  double wacc = 0.0;
  auto add = [&](int cell, float2 z) {
    if (cell < 0) return;
    float* const a = reinterpret_cast<float*>(grid + cell);
    atomicAdd(a, z.x);
    atomicAdd(a + 1, z.y);
    if constexpr (DIRECT) {  // (n - iu, n - iv)
      float* const b = reinterpret_cast<float*>(grid + ((int64_t)n * n + n - cell));
      atomicAdd(b, z.x);
      atomicAdd(b + 1, -z.y);
    }
  };
  // whole waves run each step: the scan needs every lane
  const int64_t wave_step = (int64_t)gridDim.x * blockDim.x * GRID_PER;
  for (int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63)) * GRID_PER; w0 < n_vis;
       w0 += wave_step) {
    const int64_t k0 = w0 + lane * GRID_PER;
    float uu[GRID_PER], vv[GRID_PER], ww[GRID_PER];
    float2 zz[GRID_PER];
    if (VEC && k0 + GRID_PER <= n_vis) {
      const float4 a = *reinterpret_cast<const float4*>(u + k0), b = *reinterpret_cast<const float4*>(v + k0);
      const float4 c = *reinterpret_cast<const float4*>(vis + k0), d = *reinterpret_cast<const float4*>(vis + k0 + 2);
      const float4 f = weight ? *reinterpret_cast<const float4*>(weight + k0) : make_float4(1.f, 1.f, 1.f, 1.f);
      uu[0] = a.x, uu[1] = a.y, uu[2] = a.z, uu[3] = a.w;
      vv[0] = b.x, vv[1] = b.y, vv[2] = b.z, vv[3] = b.w;
      ww[0] = f.x, ww[1] = f.y, ww[2] = f.z, ww[3] = f.w;
      zz[0] = make_float2(c.x, c.y), zz[1] = make_float2(c.z, c.w);
      zz[2] = make_float2(d.x, d.y), zz[3] = make_float2(d.z, d.w);
    } else {
#pragma unroll
      for (int j = 0; j < GRID_PER; ++j) {
        const int64_t k = k0 + j < n_vis ? k0 + j : n_vis - 1;
        uu[j] = u[k], vv[j] = v[k], zz[j] = vis[k];
        ww[j] = weight ? weight[k] : 1.f;
      }
    }
    int cell[GRID_PER];
#pragma unroll
    for (int j = 0; j < GRID_PER; ++j) {
      const int64_t iu = (int64_t)floor((double)uu[j] * inv_du + 0.5) + n / 2;
      const int64_t iv = (int64_t)floor((double)vv[j] * inv_du + 0.5) + n / 2;
      // the mirrored cell n - i lies in [0, n) for i in [1, n]
      const bool in = k0 + j < n_vis && iu >= 1 && iu < n && iv >= 1 && iv < n;
      cell[j] = in ? (int)(iu * n + iv) : -1;
      zz[j] = in ? make_float2(ww[j] * zz[j].x, ww[j] * zz[j].y) : make_float2(0.f, 0.f);
      if (in) wacc += 2.0 * (double)ww[j];
    }
    // runs inside the thread; the last one goes on to the wave
    int run = cell[0];
    float2 sum = zz[0];
    bool whole = true;
#pragma unroll
    for (int j = 1; j < GRID_PER; ++j) {
      const bool same = cell[j] == run;
      if (!same) {
        add(run, sum);
        whole = false;
      }
      sum = make_float2(same ? sum.x + zz[j].x : zz[j].x, same ? sum.y + zz[j].y : zz[j].y);
      run = cell[j];
    }
    // segmented sum over lanes: a lane of one run continues its predecessor's
    // segment if the cells agree
    const int before = __shfl_up(run, 1);
    const uint64_t heads = __ballot(lane == 0 || !whole || before != run);
    const int start = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
    for (int d = 1; d < 64; d <<= 1) {
      const float x = __shfl_up(sum.x, d), y = __shfl_up(sum.y, d);
      if (lane - d >= start) sum.x += x, sum.y += y;
    }
    if (lane == 63 || (heads >> (lane + 1)) & 1) add(run, sum);
  }
  for (int d = 32; d >= 1; d >>= 1) wacc += __shfl_down(wacc, d);
  if (lane == 0) red[threadIdx.x >> 6] = wacc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(wsum, red[0] + red[1] + red[2] + red[3]);
}

// Adds to each cell the conjugate of its mirror's sum: grid[c] = A[c] +
// conj A[mirror c], mirror (iu, iv) -> (n - iu, n - iv), in place.  A thread
// takes a cell and its mirror; row and column 0 have no mirror and stay zero.
__global__ void __launch_bounds__(256) image_mirror_kernel(float2* __restrict__ grid, int n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int iu = (int)(e / n), iv = (int)(e % n);
  if (iu < 1 || iu > n / 2 || iv < 1 || (iu == n / 2 && iv > n / 2)) return;
  const int64_t m = (int64_t)(n - iu) * n + (n - iv);
  const float2 a = grid[e], b = grid[m];
  grid[e] = make_float2(a.x + b.x, a.y - b.y);
  if (m != e) grid[m] = make_float2(b.x + a.x, b.y - a.y);
}

__global__ void image_zero_kernel(float2* __restrict__ grid, int64_t npix, double* __restrict__ wsum) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < npix) grid[e] = make_float2(0.f, 0.f);
  if (e == 0) *wsum = 0.0;
}

// X = conj((-1)^(iu+iv) G), into a work buffer.
__global__ void image_prep_kernel(const float2* __restrict__ g, int n, float2* __restrict__ x) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int iu = (int)(e / n), iv = (int)(e % n);
  const float s = ((iu + iv) & 1) ? -1.f : 1.f;
  const float2 z = g[e];
  x[e] = make_float2(s * z.x, -s * z.y);
}

// In-place forward FFT of `rows` contiguous rows of length N, S rows per
// workgroup (S N = 4096 values in LDS, one row for N >= 4096).
template <int N>
struct RowCfg {
  static constexpr int S = N >= 4096 ? 1 : 4096 / N;
  static constexpr int NT = S * N / 16;
  static constexpr int LDS = lds_padded_size(S * N);
};

template <int N>
__global__ void __launch_bounds__(RowCfg<N>::NT)
image_rows_fft_kernel(float2* __restrict__ x, int rows, const float2* __restrict__ tw) {
  using C = RowCfg<N>;
  extern __shared__ float2 buf[];
  const int r0 = blockIdx.x * C::S;
  for (int i = threadIdx.x; i < C::S * N; i += C::NT) {
    const int r = r0 + i / N;
    buf[lds_pad(i)] = r < rows ? x[(int64_t)r * N + (i % N)] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  fft_lds<N, C::NT>(buf, tw, threadIdx.x);
  for (int i = threadIdx.x; i < C::S * N; i += C::NT) {
    const int r = r0 + i / N;
    if (r < rows) x[(int64_t)r * N + (i % N)] = buf[lds_pad(i)];
  }
}

// y[c][r] = x[r][c] for an n x n complex matrix, 32 x 32 tiles through LDS.
__global__ void __launch_bounds__(256) image_transpose_kernel(const float2* __restrict__ x, int n,
                                                              float2* __restrict__ y) {
  __shared__ float2 t[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int j = ty; j < 32; j += 8) t[j][tx] = x[(int64_t)(by + j) * n + bx + tx];
  __syncthreads();
  for (int j = ty; j < 32; j += 8) y[(int64_t)(bx + j) * n + by + tx] = t[tx][j];
}

// image[il][im] = (-1)^(il+im) Re(Y[il][im]) / W with Y held transposed:
// yt[im][il] = Y[il][im].
__global__ void image_final_kernel(const float2* __restrict__ yt, int n, const double* __restrict__ wsum,
                                   float* __restrict__ image) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int il = (int)(e / n), im = (int)(e % n);
  const double W = *wsum;
  const float s = ((il + im) & 1) ? -1.f : 1.f;
  const float re = yt[(int64_t)im * n + il].x;
  image[e] = W > 0.0 ? (float)((double)(s * re) / W) : 0.f;
}

template <int N>
hipError_t launch_rows(float2* x, int rows, const float2* tw, hipStream_t s) {
  using C = RowCfg<N>;
  const size_t lds = sizeof(float2) * C::LDS;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(image_rows_fft_kernel<N>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(image_rows_fft_kernel<N>, dim3((unsigned)((rows + C::S - 1) / C::S)), dim3(C::NT), lds, s,
                     x, rows, tw);
  return hipGetLastError();
}

hipError_t rows_fft(float2* x, int n, const float2* tw, hipStream_t s) {
  switch (n) {
    case 64: return launch_rows<64>(x, n, tw, s);
    case 128: return launch_rows<128>(x, n, tw, s);
    case 256: return launch_rows<256>(x, n, tw, s);
    case 512: return launch_rows<512>(x, n, tw, s);
    case 1024: return launch_rows<1024>(x, n, tw, s);
    case 2048: return launch_rows<2048>(x, n, tw, s);
    case 4096: return launch_rows<4096>(x, n, tw, s);
  }
  return hipErrorInvalidValue;
}

// ---- Hogbom CLEAN ----------------------------------------------------------
//
// One launch of G workgroups runs every iteration.  Each thread owns the same
// pixels throughout, so the residual needs no exchange; what crosses
// workgroups is one 64-bit candidate peak each per iteration, written and
// polled with agent-scope accesses (the compute dies' L2 caches are not
// coherent with each other).  A candidate carries the iteration's tag, so the
// poll is reduction and barrier in one: a workgroup that has seen every tag
// of iteration i knows all have finished it.  Keys are kept for two iterations
// (by parity): a workgroup writes i + 2 over i only after it has seen every
// i + 1, which each workgroup writes after its last read of i.
//
// Bound: at 1024 x 1024 the sweep reads 4 MiB of beam (the residual stays in
// registers) and the exchange costs two trips to memory.  One workgroup on one
// CU took 0.65 ms per component there, bound by that CU's load path; 64
// workgroups take 4.6 us, about half of it the exchange.
//
// All G workgroups have to be resident together, which other launches on the
// GPU can prevent.  So they check in before anything is changed: the first
// workgroup lets the others go on once it has seen all of them; if one is
// missing after CLEAN_GATHER_US the first does the whole image alone and the
// others leave.  Once all are resident none can keep another away; a wait is
// bounded in time all the same, and a launch whose wait expires reports
// n_comp = -1.
constexpr int CLEAN_NT = 1024;
constexpr int CLEAN_MAX_WG = 64;
constexpr int CLEAN_SLOTS = 16;  // launches in flight with an exchange area of their own
constexpr uint64_t CLEAN_TICKS_US = 100;                           // of the 100 MHz wall clock
constexpr uint64_t CLEAN_WAIT_TICKS = 10000000 * CLEAN_TICKS_US;  // 10 s
constexpr int64_t CLEAN_GATHER_US = 20000;

enum { CLEAN_GATHER = 0, CLEAN_TOGETHER = 1, CLEAN_ALONE = 2 };
// Sixteen workgroups' keys share a cache line, and the lines lie on different
// memory channels (256 bytes apart): 64 workgroups 4.5 us a component at
// 1024 x 1024, 4.7 with the keys in a row; 16 at 256 x 256 2.4 us, 2.7 where
// they straddle two lines.
constexpr int CLEAN_KEYS = 32 * (CLEAN_MAX_WG / 16);
__device__ __forceinline__ int clean_at(int wg) { return 32 * (wg >> 4) + (wg & 15); }

struct alignas(256) CleanSlot {
  uint64_t key[2][CLEAN_KEYS];
  int busy, verdict, abort, count, done;
};
__device__ CleanSlot g_clean_slots[CLEAN_SLOTS];

template <class T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void agent_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Claims one of the first `areas` exchange areas for the launch that follows on
// the stream and hands it on in n_comp as -2 - index (-1: all taken; the launch
// then runs on one workgroup).  Workgroups that start after the others are done
// find the count there, which is no area either.
__global__ void __launch_bounds__(CLEAN_MAX_WG) image_clean_claim_kernel(int* __restrict__ n_comp, int areas) {
  __shared__ int slot_s;
  if (threadIdx.x == 0) {
    int slot = -1;
    for (int i = 0; i < areas && slot < 0; ++i)
      if (atomicCAS(&g_clean_slots[i].busy, 0, 1) == 0) slot = i;
    slot_s = slot;
    *n_comp = slot < 0 ? -1 : -2 - slot;
  }
  __syncthreads();
  if (slot_s < 0) return;  // no area of its own
  CleanSlot& c = g_clean_slots[slot_s];
  for (int q = 0; q < 2; ++q) agent_store(&c.key[q][clean_at(threadIdx.x)], (uint64_t)0);
  if (threadIdx.x == 0) {
    agent_store(&c.verdict, (int)CLEAN_GATHER);
    agent_store(&c.abort, 0);
    agent_store(&c.done, 0);
  }
}

// Candidate: |v| (31 bits), 2^26 - pixel (27), sign (1), tag (5): the largest is
// the largest |v|, of those the smallest pixel (n <= 8192).  A NaN is no
// candidate; 0 stands for none, which no pixel's key is.
constexpr uint64_t CLEAN_TAG = 31;
constexpr uint64_t CLEAN_ARRIVED = 31;  // the check-in's tag; iterations go through 1 to 30
__device__ __forceinline__ uint64_t clean_key(float v, int p) {
  const uint32_t bits = __float_as_uint(v);
  return ((uint64_t)(bits & 0x7fffffffu) << 33) | ((uint64_t)((1 << 26) - p) << 6) | ((uint64_t)(bits >> 31) << 5);
}

// Check-in of workgroup wg of G, by its first wave: true if all run together.
// The arrivals carry a tag of their own in the second set of keys; one
// word decides for all, whoever is the first to.
__device__ __forceinline__ bool clean_gather(CleanSlot* ex, int G, int wg, uint64_t gather_ticks) {
  const int lane = threadIdx.x & 63;
  if (lane == 0) agent_store(&ex->key[1][clean_at(wg)], CLEAN_ARRIVED);
  const uint64_t began = wall_clock64();
  int verdict = CLEAN_GATHER;
  while (verdict == CLEAN_GATHER) {
    const bool all = wg == 0 && __all(lane >= G || agent_load(&ex->key[1][clean_at(lane < G ? lane : 0)]) == CLEAN_ARRIVED);
    const bool late = wall_clock64() - began >= gather_ticks;
    if (all || late) {
      if (lane == 0) atomicCAS(&ex->verdict, (int)CLEAN_GATHER, (int)(all ? CLEAN_TOGETHER : CLEAN_ALONE));
    }
    verdict = __builtin_amdgcn_readfirstlane(agent_load(&ex->verdict));
  }
  return verdict == CLEAN_TOGETHER;
}

// Leaves the area: the last of G workgroups to do so, which has seen every
// other past its last read of the area, hands out the count and gives it back.
__device__ __forceinline__ void clean_leave(CleanSlot* ex, int G, int* n_comp) {
  const int left = __hip_atomic_fetch_add(&ex->done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  if (left != G - 1) return;
  *n_comp = agent_load(&ex->abort) ? -1 : agent_load(&ex->count);
  __hip_atomic_store(&ex->busy, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t key_max(uint64_t a, uint64_t b) { return a > b ? a : b; }

// The beam subtraction rounds the product and the difference separately: no
// contraction into a fused multiply-add in this kernel (the pragma covers
// expressions written here, not inlined library helpers, so the arithmetic
// is spelled out).
#pragma clang fp contract(off)

// PX > 0: PX pixels per thread held in registers (G * CLEAN_NT * PX >= n^2);
// PX = 0: any number, read from and written to memory each iteration.
template <int PX>
__global__ void __launch_bounds__(CLEAN_NT)
image_clean_kernel(float* __restrict__ r, const float* __restrict__ psf, int log2n, float gain, float thr,
                   int max_iter, uint64_t gather_ticks, int* __restrict__ comp_pix,
                   float* __restrict__ comp_flux, int* __restrict__ n_comp) {
  __shared__ uint64_t wkey[CLEAN_NT / 64];
  __shared__ uint64_t all_s;
  __shared__ int slot_s, stop_s, together_s;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int n = 1 << log2n, mask = n - 1, h = n / 2;
  const int npix = 1 << (2 * log2n);
  int G = gridDim.x, wg = blockIdx.x;
  if (wave == 0) {
    const int handed = G > 1 ? __builtin_amdgcn_readfirstlane(*n_comp) : -1;
    const bool together = handed <= -2 && clean_gather(g_clean_slots + (-2 - handed), G, wg, gather_ticks);
    if (t == 0) {
      slot_s = handed <= -2 ? -2 - handed : -1;
      together_s = together;
    }
  }
  __syncthreads();
  const int slot = __builtin_amdgcn_readfirstlane(slot_s);
  CleanSlot* const ex = g_clean_slots + (slot < 0 ? 0 : slot);
  if (G > 1 && !__builtin_amdgcn_readfirstlane(together_s)) {  // the first workgroup does it all
    if (wg > 0) {
      if (t == 0 && slot >= 0) clean_leave(ex, G, n_comp);
      return;
    }
    G = 1;
  }
  const int first = wg * CLEAN_NT + t, stride = G * CLEAN_NT;
  const bool regs = PX > 0 && G == (int)gridDim.x;
  float own[PX > 0 ? PX : 1];
  if (regs) {
#pragma unroll
    for (int j = 0; j < PX; ++j) {
      const int p = first + j * stride;
      own[j] = p < npix ? r[p] : 0.f;
    }
  }
  float g = 0.f;  // flux of the component whose beam is still to subtract
  int pl = 0, pm = 0;
  int it = 0;
  bool failed = false;
  for (;; ++it) {
    // subtract the previous component's beam (none before the first peak)
    // and find the next peak in the same sweep
    float best = -1.f, bv = 0.f;  // largest |residual| and its signed value
    int bi = 0;
    auto beam = [&](int p) -> float {
      return psf[((((p >> log2n) - pl + h) & mask) << log2n) + (((p & mask) - pm + h) & mask)];
    };
    auto visit = [&](float v, float b, int p, bool in) -> float {
      const float prod = g * b;      // rounded product
      v = it > 0 ? v - prod : v;     // rounded difference
      const bool more = in && fabsf(v) > best;
      best = more ? fabsf(v) : best;  // p increases along the thread's sweep: ties keep the first
      bv = more ? v : bv;
      bi = more ? p : bi;
      return v;
    };
    if (regs) {
      float b[PX > 0 ? PX : 1];
#pragma unroll
      for (int j = 0; j < PX; ++j) b[j] = beam((first + j * stride) & (npix - 1));
#pragma unroll
      for (int j = 0; j < PX; ++j) own[j] = visit(own[j], b[j], first + j * stride, first + j * stride < npix);
    } else {
      constexpr int U = 8;
      for (int p0 = first; p0 < npix; p0 += U * stride) {
        float v[U], b[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int p = (p0 + j * stride) & (npix - 1);
          v[j] = r[p];
          b[j] = beam(p);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int p = p0 + j * stride;
          v[j] = visit(v[j], b[j], p, p < npix);
          if (it > 0 && p < npix) r[p] = v[j];
        }
      }
    }
    uint64_t key = best < 0.f ? 0ull : clean_key(bv, bi);
    for (int d = 32; d >= 1; d >>= 1) key = key_max(key, __shfl_xor((unsigned long long)key, d));
    if (lane == 0) wkey[wave] = key;
    __syncthreads();
    if (wave == 0) {
      key = lane < CLEAN_NT / 64 ? wkey[lane] : 0ull;
      for (int d = 8; d >= 1; d >>= 1) key = key_max(key, __shfl_xor((unsigned long long)key, d));
      int stop = 0;
      if (G > 1) {
        const uint64_t tag = (uint64_t)(it % 30 + 1);
        uint64_t* const at = ex->key[it & 1];
        if (lane == 0) agent_store(&at[clean_at(wg)], key | tag);
        uint64_t began = 0;
        for (unsigned spin = 0;; ++spin) {
          key = lane < G ? agent_load(&at[clean_at(lane)]) : tag;
          if (__all((key & CLEAN_TAG) == tag)) break;
          if ((spin & 255u) == 255u) {
            const uint64_t now = wall_clock64();
            if (began == 0) began = now;
            if (now - began > CLEAN_WAIT_TICKS || agent_load(&ex->abort) != 0) {
              stop = 1;
              break;
            }
          }
        }
        if (stop && lane == 0) agent_store(&ex->abort, 1);
        key &= ~CLEAN_TAG;
        for (int d = 32; d >= 1; d >>= 1) key = key_max(key, __shfl_xor((unsigned long long)key, d));
      }
      if (lane == 0) {
        all_s = key;
        stop_s = stop;
      }
    }
    __syncthreads();
    // block-uniform, read from LDS (written again only after the next
    // iteration's first barrier): scalar for the compiler, so that the loop,
    // which holds barriers, is a scalar loop
    const uint64_t top = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(all_s >> 32)) << 32) |
                         (uint32_t)__builtin_amdgcn_readfirstlane((int)all_s);
    failed = __builtin_amdgcn_readfirstlane(stop_s) != 0;
    const bool none = top == 0ull;
    const int pi = none ? 0x7fffffff : (1 << 26) - (int)((top >> 6) & ((1u << 27) - 1));
    const float peak = none ? 0.f : __uint_as_float((uint32_t)(top >> 33) | ((uint32_t)((top >> 5) & 1u) << 31));
    if (failed || it >= max_iter || !(fabsf(peak) >= thr)) break;
    g = gain * peak;
    pl = pi >> log2n;
    pm = pi & mask;
    if (wg == 0 && t == 0) {
      comp_pix[it] = pi;
      comp_flux[it] = g;
    }
  }
  if (regs) {
#pragma unroll
    for (int j = 0; j < PX; ++j) {
      const int p = first + j * stride;
      if (p < npix) r[p] = own[j];
    }
  }
  if (t == 0) {
    if (slot >= 0) {
      if (wg == 0) agent_store(&ex->count, it);
      clean_leave(ex, (int)gridDim.x, n_comp);
    } else {
      *n_comp = it;
    }
  }
}

#pragma clang fp contract(on)

// What qc_image_clean_limits sets; read at each launch.
std::atomic<int> g_clean_areas{CLEAN_SLOTS};
std::atomic<int64_t> g_clean_gather_us{CLEAN_GATHER_US};

}  // namespace

}  // namespace qc

namespace {

bool img_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

}  // namespace

extern "C" qc_status qc_image_grid(const float* u, const float* v, const float* vis, const float* weight,
                                   int64_t n_vis, int32_t n, double cell_rad, float* grid, double* wsum,
                                   void* stream) {
  qc::api_clear_error();
  if (!img_pow2(n) || n < 64 || n > 4096)
    return qc::api_fail(QC_EINVAL, "n must be a power of two in [64, 4096] (got %d)", n);
  if (!(cell_rad > 0.0)) return qc::api_fail(QC_EINVAL, "cell_rad must be positive");
  if (n_vis < 0) return qc::api_fail(QC_EINVAL, "n_vis must be >= 0");
  if (n_vis > 0 && (!u || !v || !vis)) return qc::api_fail(QC_EINVAL, "u, v and vis must be non-null");
  if (!grid || !wsum) return qc::api_fail(QC_EINVAL, "grid and wsum must be non-null");
  if ((reinterpret_cast<uintptr_t>(vis) | reinterpret_cast<uintptr_t>(grid)) & 7u)
    return qc::api_fail(QC_EINVAL, "vis and grid must be 8-byte aligned");
  if (reinterpret_cast<uintptr_t>(wsum) & 7u) return qc::api_fail(QC_EINVAL, "wsum must be 8-byte aligned");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int64_t npix = (int64_t)n * n;
  hipLaunchKernelGGL(qc::image_zero_kernel, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<float2*>(grid), npix, wsum);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return qc::api_fail(QC_EHIP, "zero kernel: %s", hipGetErrorString(e));
  if (n_vis > 0) {
    const int64_t per = 256 * qc::GRID_PER;
    const int64_t blocks = (n_vis + per - 1) / per < 2048 ? (n_vis + per - 1) / per : 2048;
    const bool vec = ((reinterpret_cast<uintptr_t>(u) | reinterpret_cast<uintptr_t>(v) |
                       reinterpret_cast<uintptr_t>(vis) | reinterpret_cast<uintptr_t>(weight)) & 15u) == 0;
    // a mirror pass costs 2.4 us of launch and 16 B a pixel, two more atomics a
    // sample less than that up to here: 40000 samples onto 64 x 64 13.3 us (15.7
    // with the pass), 60000 16.6 (15.7); onto 4096 x 4096 3000 28 us (70), 500000
    // 119 (118)
    const bool direct = n_vis <= 45056 + npix / 32;
    hipLaunchKernelGGL((vec ? direct ? qc::image_grid_kernel<true, true> : qc::image_grid_kernel<true, false>
                            : direct ? qc::image_grid_kernel<false, true> : qc::image_grid_kernel<false, false>),
                       dim3((unsigned)blocks), dim3(256), 0, s, u, v, reinterpret_cast<const float2*>(vis), weight,
                       n_vis, (int)n, (double)n * cell_rad, reinterpret_cast<float2*>(grid), wsum);
    e = hipGetLastError();
    if (e != hipSuccess) return qc::api_fail(QC_EHIP, "grid kernel: %s", hipGetErrorString(e));
    if (!direct)
      hipLaunchKernelGGL(qc::image_mirror_kernel, dim3((unsigned)((npix / 2 + n + 255) / 256)), dim3(256), 0, s,
                         reinterpret_cast<float2*>(grid), (int)n);
    e = hipGetLastError();
    if (e != hipSuccess) return qc::api_fail(QC_EHIP, "grid kernel: %s", hipGetErrorString(e));
  }
  return QC_OK;
}

extern "C" qc_status qc_image_invert(const float* grid, const double* wsum, int32_t n, float* work,
                                     float* image, void* stream) {
  qc::api_clear_error();
  if (!img_pow2(n) || n < 64 || n > 4096)
    return qc::api_fail(QC_EINVAL, "n must be a power of two in [64, 4096] (got %d)", n);
  if (!grid || !wsum || !work || !image) return qc::api_fail(QC_EINVAL, "null buffer");
  if ((reinterpret_cast<uintptr_t>(grid) | reinterpret_cast<uintptr_t>(work)) & 7u)
    return qc::api_fail(QC_EINVAL, "grid and work must be 8-byte aligned");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  float2* tw = nullptr;
  qc_status st = qc::api_twiddles(n, &tw);
  if (st != QC_OK) return st;
  const int64_t npix = (int64_t)n * n;
  float2* x = reinterpret_cast<float2*>(work);
  float2* y = x + npix;
  const unsigned blocks = (unsigned)((npix + 255) / 256);
  hipLaunchKernelGGL(qc::image_prep_kernel, dim3(blocks), dim3(256), 0, s,
                     reinterpret_cast<const float2*>(grid), (int)n, x);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = qc::rows_fft(x, n, tw, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(qc::image_transpose_kernel, dim3(n / 32, n / 32), dim3(256), 0, s, x, (int)n, y);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = qc::rows_fft(y, n, tw, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(qc::image_final_kernel, dim3(blocks), dim3(256), 0, s, y, (int)n, wsum, image);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return qc::api_fail(QC_EHIP, "inversion kernels: %s", hipGetErrorString(e));
  return QC_OK;
}

extern "C" qc_status qc_image_clean_limits(int32_t areas, int64_t gather_us) {
  qc::api_clear_error();
  if (areas > qc::CLEAN_SLOTS) return qc::api_fail(QC_EINVAL, "at most %d exchange areas", qc::CLEAN_SLOTS);
  if (gather_us > 1000000) return qc::api_fail(QC_EINVAL, "gather_us must be at most 10^6");
  qc::g_clean_areas = areas < 0 ? qc::CLEAN_SLOTS : areas;
  qc::g_clean_gather_us = gather_us < 0 ? qc::CLEAN_GATHER_US : gather_us;
  return QC_OK;
}

extern "C" qc_status qc_image_clean(float* residual, const float* psf, int32_t n, float gain, float threshold,
                                    int32_t max_iter, int32_t* comp_pix, float* comp_flux, int32_t* n_comp,
                                    void* stream) {
  qc::api_clear_error();
  if (!img_pow2(n) || n < 2 || n > 8192)
    return qc::api_fail(QC_EINVAL, "n must be a power of two in [2, 8192] (got %d)", n);
  if (!(gain > 0.f && gain <= 1.f)) return qc::api_fail(QC_EINVAL, "gain must be in (0, 1]");
  if (!(threshold >= 0.f)) return qc::api_fail(QC_EINVAL, "threshold must be >= 0");
  if (max_iter < 0) return qc::api_fail(QC_EINVAL, "max_iter must be >= 0");
  if (!residual || !psf || !n_comp || (max_iter > 0 && (!comp_pix || !comp_flux)))
    return qc::api_fail(QC_EINVAL, "null buffer");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  // Workgroups by image size: 4 pixels per thread until 64 workgroups are
  // reached at n = 512 (one workgroup and no exchange up to n = 64), then 16
  // at n = 1024; larger images would need more than the 128 registers a thread
  // of a full workgroup has, and keep the residual in memory.
  int log2n = 0;
  while ((1 << log2n) < n) ++log2n;
  int* const pix = reinterpret_cast<int*>(comp_pix);
  int* const count = reinterpret_cast<int*>(n_comp);
  auto launch = [&](auto kernel, int wgs) {
    if (wgs > 1)
      hipLaunchKernelGGL(qc::image_clean_claim_kernel, dim3(1), dim3(qc::CLEAN_MAX_WG), 0, s, count,
                         qc::g_clean_areas.load(std::memory_order_relaxed));
    hipLaunchKernelGGL(kernel, dim3(wgs), dim3(qc::CLEAN_NT), 0, s, residual, psf, log2n, gain, threshold,
                       (int)max_iter, (uint64_t)qc::g_clean_gather_us.load(std::memory_order_relaxed) * qc::CLEAN_TICKS_US,
                       pix, comp_flux, count);
  };
  if (log2n <= 6) launch(qc::image_clean_kernel<4>, 1);
  else if (log2n == 7) launch(qc::image_clean_kernel<4>, 4);
  else if (log2n == 8) launch(qc::image_clean_kernel<4>, 16);
  else if (log2n == 9) launch(qc::image_clean_kernel<4>, 64);
  else if (log2n == 10) launch(qc::image_clean_kernel<16>, 64);
  else launch(qc::image_clean_kernel<0>, 64);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return qc::api_fail(QC_EHIP, "clean kernel: %s", hipGetErrorString(e));
  return QC_OK;
}
