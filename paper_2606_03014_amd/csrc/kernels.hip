// gfx950 (CDNA4) kernels of the ragged MoA generation step.
//
// One engine step runs every co-resident model's rows as one ragged batch:
// rows of the same model are contiguous, and each kernel class is launched
// once per layer for all models (grouped over models), so the weights of each
// active model stream from HBM once per step. The kernels are written for
// 64-wide wavefronts; the dense contractions use the bf16 MFMA
// v_mfma_f32_16x16x32_bf16 with fp32 accumulation.
#include "kernels.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>

namespace moa {

// Scratch for the kernels of allocation-free calls: partial sums only (every
// byte is written before it is read within a call, so nothing is cleared).
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(void** out) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return err;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// Optional event pair attached to the next launch (hipExtLaunchKernel
// timestamps the dispatch itself, so the measured span is the kernel's).
static hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;


void set_launch_events(hipEvent_t start, hipEvent_t stop) {
  g_ev_start = start;
  g_ev_stop = stop;
}

template <typename... KArgs, typename... Args>
static void klaunch_shm(void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned shm, hipStream_t st,
                        Args... args) {
  if (g_ev_start)
    hipExtLaunchKernelGGL(kernel, grid, block, shm, st, g_ev_start, g_ev_stop, 0, args...);
  else
    kernel<<<grid, block, shm, st>>>(args...);
}

template <typename... KArgs, typename... Args>
static void klaunch(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t st, Args... args) {
  klaunch_shm(kernel, grid, block, 0u, st, args...);
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// (a, b) -> two bf16 in one word (a low), round to nearest even: one
// v_cvt_pk_bf16_f32 on gfx950.
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}
// Split-bf16 pair: hi = bf16(a, b); lo = bf16 of the remainders.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& hi, unsigned& lo) {
  hi = pack_bf16(a, b);
  lo = pack_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

// fp32 -> bf16, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Split-bf16 store: v ~= hi + lo with hi = bf16(v), lo = bf16(v - hi); the
// pair carries ~16 significant bits, so a GEMM fed hi and lo (two MFMAs per
// weight fragment) sees the fp32 activation almost exactly while the weights
// stay bf16.
__device__ __forceinline__ void store_split(uint16_t* p, size_t lo, size_t i, float v) {
  const uint16_t h = f2bf(v);
  p[i] = h;
  p[i + lo] = f2bf(v - bf2f(h));
}

// silu(gate) * up, rounded once more before it is split: without the pragma one
// kernel would fuse the product into the split's subtraction and another not.
__device__ __forceinline__ float silu_mul(float g, float up) {
#pragma clang fp contract(off)
  return g / (1.f + __expf(-g)) * up;
}

// The norm's and RoPE's arithmetic, with every fused operation written out: the
// kernels that share it give the same bits whatever the compiler would fuse.
__device__ __forceinline__ float sumsq4(float4 v) {
  return fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.x, v.x, v.y * v.y)));
}
// split pairs of (v * scale) * g for four elements: h01, h23 | l01, l23
__device__ __forceinline__ u32x4 norm_split4(float4 v, float scale, const float g[4]) {
#pragma clang fp contract(off)
  const float t0 = v.x * scale, t1 = v.y * scale, t2 = v.z * scale, t3 = v.w * scale;
  const unsigned h0 = pack_bf16(t0 * g[0], t1 * g[1]), h1 = pack_bf16(t2 * g[2], t3 * g[3]);
  const unsigned l0 = pack_bf16(fmaf(t0, g[0], -__uint_as_float(h0 << 16)), fmaf(t1, g[1], -__uint_as_float(h0 & 0xffff0000u)));
  const unsigned l1 = pack_bf16(fmaf(t2, g[2], -__uint_as_float(h1 << 16)), fmaf(t3, g[3], -__uint_as_float(h1 & 0xffff0000u)));
  return u32x4{h0, h1, l0, l1};
}
__device__ __forceinline__ float2 rotate(float x1, float x2, float2 cs) {
#pragma clang fp contract(off)
  return make_float2(fmaf(x1, cs.x, -(x2 * cs.y)), fmaf(x2, cs.x, x1 * cs.y));
}

// Order this wavefront's LDS writes before its later LDS reads (no workgroup barrier).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ const void* pick(const ModelPtrs& mp, int m) {
  const void* r = mp.p[0];
#pragma unroll
  for (int i = 1; i < kMaxModels; ++i)
    if (i == m) r = mp.p[i];
  return r;
}

// Cross-lane moves inside a row of 16 lanes as DPP operand modifiers (plain
// VALU, no LDS crossbar): quad_perm [1,0,3,2] = lane ^ 1, quad_perm [2,3,0,1]
// = lane ^ 2, row_half_mirror = lane 7 - i within each 8 lanes (after the
// two quad steps every lane of a quad holds the quad's value, so the mirror
// brings in the other quad), row_ror:8 = lane ^ 8 within 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum8(float v) {       // over lanes 8k..8k+7
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  return v + dpp<0x141>(v);
}
__device__ __forceinline__ float sum16(float v) {      // over lanes 16k..16k+15
  v = sum8(v);
  return v + dpp<0x128>(v);
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  return fmaxf(v, dpp<0x128>(v));
}
// lane ^ 16 (within 32 lanes) through ds_swizzle's bit mode
__device__ __forceinline__ float swz_xor16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
}

// Sum over the 64 lanes (every lane gets it): DPP within rows of 16, a
// swizzle across the two rows of each half, one exchange across the halves.
__device__ __forceinline__ float wave_sum(float v) {
  v = sum16(v);
  v += swz_xor16(v);
  return v + __shfl_xor(v, 32, 64);
}

// Sum over a 256-thread block; every thread gets the result.
__device__ __forceinline__ float block_sum256(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------- embedding
// x[t] = E_model[tok] in fp32 (the residual stream is fp32 in every mode).
template <bool BF>
__global__ __launch_bounds__(256) void k_embed(const int* __restrict__ tok_store,
                                               const int* __restrict__ row_tok,
                                               const int* __restrict__ row_model, ModelPtrs embed,
                                               float* __restrict__ x, int d) {
  const int t = blockIdx.x;
  const int tok = tok_store[row_tok[t]];
  const void* E = pick(embed, row_model[t]);
  float* xr = x + (size_t)t * d;
  // 16-byte loads, all of a thread's issued before the first store (d % 256 == 0)
  if (BF) {
    const uint16_t* e = (const uint16_t*)E + (size_t)tok * d;
#pragma unroll 2
    for (int i = threadIdx.x * 8; i < d; i += 256 * 8) {
      const uint4 u = *(const uint4*)(e + i);
      *(float4*)(xr + i) = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                                       __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
      *(float4*)(xr + i + 4) = make_float4(__uint_as_float(u.z << 16), __uint_as_float(u.z & 0xffff0000u),
                                           __uint_as_float(u.w << 16), __uint_as_float(u.w & 0xffff0000u));
    }
  } else {
    const float* e = (const float*)E + (size_t)tok * d;
#pragma unroll 4
    for (int i = threadIdx.x * 4; i < d; i += 256 * 4) *(float4*)(xr + i) = *(const float4*)(e + i);
  }
}

// ------------------------------------------------- residual add + RMSNorm
// x[r] += sum_s part[s][r] (split-K partial sums of the previous projection),
// out[j] = x[r] * rsqrt(mean(x[r]^2) + eps) * gamma, r = gather ? gather[j] : j.
// One workgroup per row, V4 float4s of the row per thread, thread t owning
// float4s t, t + blockDim, ...: two per thread when d is a multiple of 2048
// (256 threads at d = 2048, 512 at 4096: the smaller workgroup finds room
// beside another stream's kernels sooner, and at 4096 it is as fast alone),
// else one (d / 4 threads, at most 1024).
// The partial-sum loads of a thread are all in flight before they are added.
template <bool BF, int V4>
__global__ __launch_bounds__(1024) void k_add_rmsnorm(float* __restrict__ x, const float* __restrict__ part,
                                                      int nsplit, size_t split_stride,
                                                      const int* __restrict__ gather,
                                                      const int* __restrict__ row_model, ModelPtrs gamma,
                                                      void* __restrict__ out, size_t out_lo, int d, float eps) {
  __shared__ float red[16];
  const int j = blockIdx.x;
  const int r = gather ? gather[j] : j;
  // the row's gain is fetched first, so its dependent loads (model id, gain
  // pointer, gains) overlap the partial-sum loads instead of following the
  // block reduction
  const void* g = pick(gamma, row_model[r]);
  float gv[V4][4];
#pragma unroll
  for (int k = 0; k < V4; ++k) {
    const int i = (threadIdx.x + k * blockDim.x) * 4;
    if (BF) {
      const uint2 gb = *(const uint2*)((const uint16_t*)g + i);
      gv[k][0] = __uint_as_float(gb.x << 16); gv[k][1] = __uint_as_float(gb.x & 0xffff0000u);
      gv[k][2] = __uint_as_float(gb.y << 16); gv[k][3] = __uint_as_float(gb.y & 0xffff0000u);
    } else {
      const float4 gf = *(const float4*)((const float*)g + i);
      gv[k][0] = gf.x; gv[k][1] = gf.y; gv[k][2] = gf.z; gv[k][3] = gf.w;
    }
  }
  float* xrow = x + (size_t)r * d;
  float4 v[V4];
#pragma unroll
  for (int k = 0; k < V4; ++k) v[k] = *(const float4*)(xrow + (threadIdx.x + k * blockDim.x) * 4);
  if (nsplit) {
    const float* prow = part + (size_t)r * d;
#pragma unroll 8
    for (int s = 0; s < nsplit; ++s) {
#pragma unroll
      for (int k = 0; k < V4; ++k) {
        const float4 p = *(const float4*)(prow + (size_t)s * split_stride + (threadIdx.x + k * blockDim.x) * 4);
        v[k].x += p.x; v[k].y += p.y; v[k].z += p.z; v[k].w += p.w;
      }
    }
#pragma unroll
    for (int k = 0; k < V4; ++k) *(float4*)(xrow + (threadIdx.x + k * blockDim.x) * 4) = v[k];
  }
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < V4; ++k) ss += sumsq4(v[k]);
  ss = wave_sum(ss);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int k = 0; k < nw; ++k) tot += red[k];
  const float scale = rsqrtf(tot / (float)d + eps);
#pragma unroll
  for (int k = 0; k < V4; ++k) {
    const int i = (threadIdx.x + k * blockDim.x) * 4;
    if (BF) {
      // split-bf16 pairs packed in hardware, one 8-byte store per plane
      const u32x4 y = norm_split4(v[k], scale, gv[k]);
      uint16_t* o = (uint16_t*)out + (size_t)j * d + i;
      *(uint2*)o = make_uint2(y.x, y.y);
      *(uint2*)(o + out_lo) = make_uint2(y.z, y.w);
    } else {
      *(float4*)((float*)out + (size_t)j * d + i) = make_float4(v[k].x * scale * gv[k][0], v[k].y * scale * gv[k][1],
                                                                v[k].z * scale * gv[k][2], v[k].w * scale * gv[k][3]);
    }
  }
}

// ------------------------------------------------------------ bf16 GEMMs
// Y = X . W^T for every group (model) of rows, on bf16 MFMA with fp32
// accumulation; X arrives as a split-bf16 pair (hi + lo planes), so each
// weight fragment meets two MFMAs.
//
// Weights are stored tile-shuffled so that one MFMA B-fragment (16 columns x
// 32 k) is 1 KB contiguous, lane-ordered: a wave's weight read is a single
// fully coalesced 1 KB burst per fragment, and a 16-column tile streams
// K*32 bytes contiguously.
//
// 16x16x32 operand layout (lane l of 64): A = rows l%16, k = 8*(l/16)..+8;
// B = column l%16, same k; D = column l%16, rows 4*(l/16)..+4.
//
// ------------------------------------------ bf16 GEMM, small row counts
// Up to 16 rows per model (and, at up to 64 rows per chunk, the widths and grids
// the medium-M kernel below does not take): the launch is a stream of weights
// that nothing but latency should slow down.
//  * A workgroup owns 16 * MT rows x 16 * NW * CT columns of one k-split, each of its
//    NW waves CT column tiles, and runs the split's k-steps in order, hi plane
//    before lo: one chain per output and split, so the sums are those of any
//    other kernel on the same split, bit for bit.
//  * Weights go straight to registers, R stages of four k-steps ahead, the same
//    loads every stage (clamped to the last), so the waits stay exact. A chain over
//    all of K (gate-up, LM head) has few waves, so each keeps up to 32 KB in flight.
//  * The activations (both planes, in MFMA A order) pass through registers into a
//    two-slot LDS ring that the waves share: loaded as far ahead as the weights
//    (vector loads complete in order, so waiting for a younger load waits for every
//    older one), written a stage ahead, one barrier per stage that leaves them in flight.
//  * Workgroup ids are remapped so that each XCD streams one contiguous range
//    of columns, and row chunks sharing weights run side by side on it.
// us per launch, 128-column workgroups with the next stage's loads issued together
// and copied -> this: 8B gate-up 50.4 -> 37.8 at 8 rows, 52.8 -> 39.8 at 16 (6.2 and
// 5.9 TB/s); o and down (mean) 23.7 -> 19.6, 25.0 -> 20.4; qkv 12.0 -> 12.3, 12.6 ->
// 13.3; a head of 4,096 40.8 -> 16.0. 1B gate-up 23.9 -> 14.1, 25.2 -> 14.6; o and
// down 12.1 -> 7.6, 12.8 -> 8.4; qkv 5.2 -> 5.7; head 20.6 -> 10.1. Measured and not
// kept: four stages ahead (1B gate-up 17.8), activations from L2 straight to
// registers (level up to 8 rows, 10-20% slower steps at 16), sums of four waves'
// quarters of a split (up to 10% faster, but another order: other last bits).
__device__ __forceinline__ u32x4 load_stream(const u32x4* p) { return __builtin_nontemporal_load(p); }

template <int MT, int CT, int NW, int R, int EPI>
__global__ __launch_bounds__(64 * NW, 2) void k_gemm_sm(GemmArgs a, int nblk) {
  constexpr int UK = 4;                              // k-steps per stage
  constexpr int PER = 2 * MT * UK / NW;              // activation fragments per wave and stage
  __shared__ __align__(16) unsigned char sA[2][2 * MT * UK * 1024];
  const int per = (nblk + 7) / 8;
  const int blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= nblk) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const void* Wg = a.g[0].W;
  int row0 = a.g[0].row0, nrows = a.g[0].nrows, n_mc = a.g[0].n_mc, item0 = a.g[0].item0;
#pragma unroll
  for (int i = 1; i < kMaxGroups; ++i) {
    if (i < a.ngroups && a.g[i].item0 <= blk) {
      Wg = a.g[i].W; row0 = a.g[i].row0; nrows = a.g[i].nrows; n_mc = a.g[i].n_mc; item0 = a.g[i].item0;
    }
  }
  // a group's workgroups: (column block, split), row chunk fastest
  const int idx = blk - item0;
  const int mc = idx % n_mc;
  const int s = idx / n_mc % a.S, nb = idx / n_mc / a.S;
  const int tile0 = (nb * NW + w) * CT;              // this wave's first 16-column tile
  const int KS = a.K >> 5, ns = a.ksteps / UK, ks0 = s * a.ksteps;
  const int rbase = row0 + mc * MT * 16, rend = row0 + nrows;
  const u32x4* bp = (const u32x4*)Wg + ((size_t)tile0 * KS + ks0) * 64 + lane;
  const size_t wt = (size_t)KS * 64;                 // u32x4 between weight tiles
  // fragment f of a stage is (plane, row tile, k-step) = (f / (MT * UK), f / UK % MT, f % UK)
  const uint16_t* ap[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = w * PER + i, pl = f / (MT * UK), m = f / UK % MT, u = f % UK;
    const int row = min(rbase + 16 * m + (lane & 15), rend - 1);
    ap[i] = (const uint16_t*)a.X + (size_t)pl * a.x_lo + (size_t)row * a.K + (size_t)(ks0 + u) * 32 + 8 * (lane >> 4);
  }
  u32x4 ga[R][PER], b[R][UK][CT];
  auto loadA = [&](int st, int d) {
#pragma unroll
    for (int i = 0; i < PER; ++i) ga[d][i] = *(const u32x4*)(ap[i] + min(st, ns - 1) * (UK * 32));
  };
  auto writeA = [&](int st, int d) {
#pragma unroll
    for (int i = 0; i < PER; ++i) *(u32x4*)(sA[st & 1] + (w * PER + i) * 1024 + lane * 16) = ga[d][i];
  };
  auto loadB = [&](int st, int d, int u) {
    const size_t o = (size_t)(min(st, ns - 1) * UK + u) * 64;
#pragma unroll
    for (int j = 0; j < CT; ++j) b[d][u][j] = load_stream(bp + j * wt + o);
  };
  // LDS only: the loads in flight stay in flight
  auto barrier = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  f32x4_t acc[MT][CT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[m][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  loadA(0, 0);
#pragma unroll
  for (int d = 0; d < R; ++d) {
#pragma unroll
    for (int u = 0; u < UK; ++u) loadB(d, d, u);
    if (d + 1 < R) loadA(d + 1, d + 1);
  }
  writeA(0, 0);
  loadA(R, 0);
  barrier();
  // Stage st reads slot st & 1 while the other slot takes stage st + 1; the one
  // barrier per stage makes that slot visible and frees the one just read.
  for (int st0 = 0; st0 < ns; st0 += R) {
#pragma unroll
    for (int d = 0; d < R; ++d) {
      const int st = st0 + d;
      if (st >= ns) break;                           // the same for all waves
      const unsigned char* sl = sA[st & 1] + lane * 16;
#pragma unroll
      for (int u = 0; u < UK; ++u) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const u32x4 av = *(const u32x4*)(sl + ((p * MT + m) * UK + u) * 1024);
#pragma unroll
            for (int j = 0; j < CT; ++j)
              acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av),
                                                                  __builtin_bit_cast(bf16x8_t, b[d][u][j]), acc[m][j], 0, 0, 0);
          }
        loadB(st + R, d, u);
        __builtin_amdgcn_sched_barrier(0);           // a fragment's registers are free before they are loaded again
      }
      writeA(st + 1, (d + 1) % R);
      loadA(st + 1 + R, (d + 1) % R);
      barrier();
    }
  }
  // register i of lane l of a tile is row 4 (l / 16) + i, column l % 16
  const int col = lane & 15, rq = (lane >> 4) * 4;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = rbase + 16 * m + rq + i;
      if (row >= rend) continue;
      if (EPI == EPI_F32) {
#pragma unroll
        for (int j = 0; j < CT; ++j)
          a.out[(size_t)s * a.out_split + (size_t)row * a.N + (tile0 + j) * 16 + col] = acc[m][j][i];
      } else {
        // tiles (2p, 2p+1) are (gate, up) of the same 16 hidden units
#pragma unroll
        for (int p = 0; p < CT / 2; ++p)
          store_split(a.hout, a.h_lo, (size_t)row * (a.N >> 1) + ((tile0 >> 1) + p) * 16 + col,
                      silu_mul(acc[m][2 * p][i], acc[m][2 * p + 1][i]));
      }
    }
}

// ---------------------------------------- wait, LDS and direct-load helpers
// Explicit waits, LDS addressing and untracked LDS reads shared by the GEMM
// and attention kernels below. Direct global->LDS loads
// (global_load_lds_dwordx4) move one 1 KB MFMA fragment per instruction.
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }
#define MOA_LDS(p) ((__attribute__((address_space(3))) void*)(p))
// 32-bit LDS address of a pointer into shared memory
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) void*)p;
}
// Two 8-byte LDS reads at addr + 8*O0 and addr + 8*O1 into one register
// quad. The compiler does not track it: pair it with lgkm_wait_for().
template <int O0, int O1>
__device__ __forceinline__ u32x4 ds_read2_b64(unsigned addr) {
  u32x4 v;
  asm volatile("ds_read2_b64 %0, %1 offset0:%2 offset1:%3" : "=v"(v) : "v"(addr), "i"(O0), "i"(O1));
  return v;
}
// Two transposed 8-byte LDS reads (ds_read_b64_tr_b16) at addr + O0 and
// addr + O1 into one register quad; untracked like ds_read2_b64 above.
template <int O0, int O1>
__device__ __forceinline__ u32x4 ds_read_tr16_pair(unsigned addr) {
  u32x2_t a, b;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(a) : "v"(addr), "i"(O0));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(b) : "v"(addr), "i"(O1));
  return u32x4{a.x, a.y, b.x, b.y};
}
// One 4-byte LDS store the compiler does not track (ordered by "memory" and by
// the explicit LDS waits before each barrier).
__device__ __forceinline__ void ds_write_b32(unsigned addr, unsigned v) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
// Wait for every outstanding LDS access; tying v makes its later uses follow.
__device__ __forceinline__ void lgkm_wait_for(u32x4& v) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v)); }

// -------------------------------- row GEMMs of steps with very few rows
// Up to 8 rows per model, a layer of nine launches spends as long on launches
// and the short kernels between the GEMMs (5 us each for a norm or RoPE) as on the
// 1B weights. Here a workgroup holds all S k-splits of its columns, a wave each
// (wave w < S * CG: split w % S of column group w / S), so its epilogue has finished
// sums:
//  * O and down add them to the residual;
//  * qkv owns both halves of its rotation pairs (tiles hd / 2 columns apart) and
//    writes q and the KV cache;
//  * qkv and gate-up normalise their model's rows themselves, every workgroup all
//    of them, into LDS as split pairs (d * 4 bytes a row), with eight waves at
//    least, while the weights' first loads are in flight.
// A layer is then qkv, attention (and its combine), O, gate-up, down. All sums run
// in the order of the kernels that this replaces (a split's k-steps in one chain,
// splits added in order to the residual, the norm's lanes and waves as in its own
// launch), so the step's bits are theirs.
// O and down read their rows' fragments from L2. Rows 0-7 of an A operand are the
// hi plane and rows 8-15 the lo plane, so one load brings both; the other operand is
// the same with the halves of 16 lanes swapped. Output rows 8-15 are not used.
// us per launch at 1 and 6 rows, 1B: qkv 7.4 and 9.6 (norm, GEMM and RoPE launches
// 14.7 and 15.1 at 8), gate-up 13.7 and 17.1 (18.6), down 9.0 and 12.4 (7.6 and a
// norm); 8B at 6 rows: qkv 15.0, O 8.4, gate-up 42.4, down 22.8.
constexpr int kRowPad = 4;                           // words between rows in LDS: other banks for each row
template <int CT, int D, int EPI>
__global__ __launch_bounds__(EPI == ROW_RES && D > 8 ? 256 : 1024) void k_gemm_row(GemmArgs a, RowArgs f, int ncb, int CG) {
  extern __shared__ __align__(16) unsigned char row_smem[];
  const int nblk = ncb * a.ngroups;
  const int per = (nblk + 7) / 8;
  const int blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= nblk) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int g = blk / ncb, cb = blk - g * ncb;
  const void* Wg = a.g[0].W;
  const void* gam = f.gamma.p[0];
  int row0 = a.g[0].row0, nrows = a.g[0].nrows;
#pragma unroll
  for (int i = 1; i < kMaxGroups; ++i)
    if (i == g) { Wg = a.g[i].W; row0 = a.g[i].row0; nrows = a.g[i].nrows; gam = f.gamma.p[i]; }
  const int S = a.S, s = w % S, cg = w / S;
  const bool mine = cg < CG;                         // the other waves only help to normalise
  const int KS = a.K >> 5, nk = a.ksteps, ks0 = s * nk;
  const int c0 = cb * CG + (mine ? cg : 0);          // this wave's columns
  auto tile_of = [&](int c, int j) {                 // their j-th 16-column tile
    if constexpr (EPI == ROW_ROPE) {
      const int ph = f.hd / 32, head = c / ph;
      return head * (f.hd / 16) + (c - head * ph) + j * ph;
    } else {
      return c * CT + j;
    }
  };
  float* red = (float*)row_smem;                     // [wave][tile][256], where the rows were
  const int d = f.d, stride = d + kRowPad;
  float* xr = (float*)row_smem;                      // [row][stride]: x, then per 4 columns h01, h23, l01, l23
  float* sums = xr + (size_t)nrows * stride;         // [row][norm wave]
  // the norm launch's shape: waves of 64 lanes, V4 float4s per lane
  const int v4 = (d % 2048 == 0) ? 2 : 1, nt = d / (4 * v4), nvw = nt >> 6;
  uint2 gb[2];                                       // gains of columns 4 * (thread, thread + blockDim)
  if constexpr (EPI != ROW_RES) {
    for (int u = w; u < nrows * (d >> 8); u += nw) {
      const int r = u / (d >> 8), c = (u - r * (d >> 8)) * 256;
      __builtin_amdgcn_global_load_lds((const void*)(f.x + (size_t)(row0 + r) * d + c + 4 * lane),
                                       MOA_LDS(xr + r * stride + c), 16, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = (threadIdx.x + k * blockDim.x) * 4;
      gb[k] = i < d ? *(const uint2*)((const uint16_t*)gam + i) : make_uint2(0, 0);
    }
  }
  const u32x4* bp[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) bp[j] = (const u32x4*)Wg + ((size_t)tile_of(c0, j) * KS + ks0) * 64 + lane;
  u32x4 b[D][CT], av[D];
  const uint16_t* ap = (const uint16_t*)a.X + (size_t)((lane >> 3) & 1) * a.x_lo +
                       (size_t)(row0 + min(lane & 7, nrows - 1)) * a.K + (size_t)ks0 * 32 + 8 * (lane >> 4);
  auto load = [&](int st, int q) {
#pragma unroll
    for (int j = 0; j < CT; ++j) b[q][j] = load_stream(bp[j] + (size_t)st * 64);
    if constexpr (EPI == ROW_RES) av[q] = *(const u32x4*)(ap + st * 32);
  };
  // LDS only: the loads in flight stay in flight
  auto barrier = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  if constexpr (EPI != ROW_RES) wait_vmcnt<0>();     // this wave's part of the rows is in LDS
  if (mine) {
#pragma unroll
    for (int q = 0; q < D; ++q) load(min(q, nk - 1), q);
  }
  if constexpr (EPI != ROW_RES) {
    barrier();
    for (int u = w; u < nrows * nvw; u += nw) {
      const int r = u / nvw, t = (u - r * nvw) * 64 + lane;
      const float* x = xr + r * stride + t * 4;
      float ss = sumsq4(*(const float4*)x);
      if (v4 == 2) ss += sumsq4(*(const float4*)(x + nt * 4));
      ss = wave_sum(ss);
      if (lane == 0) sums[r * 16 + (u - r * nvw)] = ss;
    }
    barrier();
    float scale = 0.f;                               // of row `lane`
    if (lane < nrows) {
      float tot = 0.f;
      for (int k = 0; k < nvw; ++k) tot += sums[lane * 16 + k];
      scale = rsqrtf(tot / (float)d + f.eps);
    }
    for (int r = 0; r < nrows; ++r) {
      const float sr = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, scale), r));
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int i = (threadIdx.x + k * blockDim.x) * 4;
        if (i < d) {
          const float gv[4] = {__uint_as_float(gb[k].x << 16), __uint_as_float(gb[k].x & 0xffff0000u),
                               __uint_as_float(gb[k].y << 16), __uint_as_float(gb[k].y & 0xffff0000u)};
          float* e = xr + r * stride + i;
          *(u32x4*)e = norm_split4(*(const float4*)e, sr, gv);
        }
      }
    }
    barrier();
  }
  const uint2* ax = (const uint2*)(xr + min(lane & 15, nrows - 1) * stride + ks0 * 32 + 8 * (lane >> 4));
  f32x4_t acc[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto mul = [&](int st, int q) {
    u32x4 x[2];
    if constexpr (EPI == ROW_RES) {
      x[0] = av[q];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[1][k] = __builtin_amdgcn_mov_dpp(av[q][k], 0x128, 0xF, 0xF, true);   // lane ^ 8 of 16
    } else {
      const uint2 h0 = ax[st * 16], l0 = ax[st * 16 + 1], h1 = ax[st * 16 + 2], l1 = ax[st * 16 + 3];
      x[0] = u32x4{h0.x, h0.y, h1.x, h1.y};
      x[1] = u32x4{l0.x, l0.y, l1.x, l1.y};
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int j = 0; j < CT; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[p]),
                                                         __builtin_bit_cast(bf16x8_t, b[q][j]), acc[j], 0, 0, 0);
  };
  if (mine) {
    int st = 0;
    for (; st + D < nk; st += D) {
#pragma unroll
      for (int q = 0; q < D; ++q) {
        mul(st + q, q);
        load(min(st + D + q, nk - 1), q);
        __builtin_amdgcn_sched_barrier(0);           // a fragment's registers are free before they are loaded again
      }
    }
#pragma unroll
    for (int q = 0; q < D; ++q)
      if (st + q < nk) mul(st + q, q);
  }
  if constexpr (EPI == ROW_SWIGLU) {
    // S = 1: the wave's own sums; register i of lane l is row 4 (l / 16) + i, column l % 16
    const int col = lane & 15, rq = (lane >> 4) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (mine && rq + i < nrows)
#pragma unroll
        for (int p = 0; p < CT / 2; ++p)
          store_split(a.hout, a.h_lo, (size_t)(row0 + rq + i) * (a.N >> 1) + (c0 * (CT / 2) + p) * 16 + col,
                      silu_mul(acc[2 * p][i], acc[2 * p + 1][i]));
    return;
  }
  if constexpr (EPI != ROW_RES) barrier();           // every wave has read its rows
  if (mine)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[(w * CT + j) * 256 + i * 64 + lane] = acc[j][i];
  barrier();
  // output t of the workgroup: column group t / 128, row t / 16 % 8, column t % 16
  for (int t = threadIdx.x; t < 128 * CG; t += blockDim.x) {
    const int oc = t >> 7, rr = (t >> 4) & 7, col = t & 15;
    if (rr >= nrows) continue;
    const int row = row0 + rr;
    const float* rp = red + (size_t)oc * S * CT * 256 + (rr & 3) * 64 + (rr >> 2) * 16 + col;
    if constexpr (EPI == ROW_RES) {
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        float* o = f.x + (size_t)row * d + tile_of(cb * CG + oc, j) * 16 + col;
        float v = *o;
        for (int k = 0; k < S; ++k) v += rp[(k * CT + j) * 256];
        *o = v;
      }
    } else {
      const int c = cb * CG + oc, ph = f.hd / 32, head = c / ph;
      const int half = f.hd >> 1, jj = (c - head * ph) * 16 + col;
      float x1 = 0.f, x2 = 0.f;
      for (int k = 0; k < S; ++k) {
        x1 += rp[k * CT * 256];
        x2 += rp[(k * CT + CT - 1) * 256];
      }
      const int pos = f.row_pos[row];
      const size_t hs = (size_t)2 * kBlock * f.hd;
      float2 y = make_float2(x1, x2);
      if (head < f.n_h + f.n_kv) y = rotate(x1, x2, f.rope_tab[(size_t)pos * half + jj]);
      if (head < f.n_h) {
        const size_t o = ((size_t)row * f.n_h + head) * f.hd + jj;
        f.q[o] = y.x;
        f.q[o + half] = y.y;
      } else {
        const int kh = (head - f.n_h) % f.n_kv, kv_sel = (head - f.n_h) / f.n_kv;
        const int bk = f.bt_store[f.row_bt[row] + (pos >> 4)];
        const size_t o = (((size_t)f.layer * f.num_blocks + bk) * f.n_kv + kh) * hs + (size_t)kv_sel * kBlock * f.hd +
                         (pos & 15) * f.hd + jj;
        ((uint16_t*)f.kv)[o] = f2bf(y.x);
        ((uint16_t*)f.kv)[o + half] = f2bf(y.y);
      }
    }
  }
}

// -------------------------------------- medium-M GEMM (16x16x32 MFMA)
// A few dozen to a few hundred rows per model. Every weight byte feeds only that
// many rows of MFMA work, so the GEMM must stream the weights at HBM speed, and
// keeping the weights out of LDS leaves the LDS to the activations. A workgroup of NW waves owns one row chunk of a
// group (mrows rows, at most 16*RT: a group of up to that many rows is one
// chunk, so each weight tile leaves HBM once per step; a larger group is cut
// into chunks whose items for one column block run side by side on one XCD)
// x NW * CT * 16 columns x one k-split.
//  * The split-bf16 activation block of a 32-k stage (2*RT fragments of 1 KB,
//    both planes) is shared by the waves: it goes HBM/L2 -> LDS by direct
//    loads into a ring of D + 1 slots.
//  * Each wave streams its own CT weight tiles (1 KB fragments) straight into
//    a register ring D stages deep (a stage's loads are issued once its
//    registers have fed the MFMAs: issuing them before, from a ring one
//    stage deeper, measured ~10% slower at 100+ rows), so the LDS holds only
//    activations: the planner sizes the grid to the resident slots
//    (a grid of more items than slots ran at half the streaming rate in its
//    last, partly empty round).
//  * Per stage a wave reads its hi-plane fragments, multiplies them, then the
//    lo plane (other waves on the SIMD fill the read latency); the RT x CT
//    accumulators form that many independent MFMA chains (16x16x32 needs
//    about 16 to reach its rate).
//  * Loads complete in issue order: stage s's activation loads, then its
//    weight loads, so waiting until D - 1 stages' worth of loads are
//    outstanding makes stage s resident.
//  * k-splits take KS / S k-steps each, rounded (any S).
// N 16-byte LDS reads at addr + OFF + 1024 * i and the wait for them, in
// one asm statement: the compiler sees the registers only once they hold
// the data (an asm read whose wait came later let it copy a register that
// was still in flight when registers were scarce).
template <int N, int OFF>
__device__ __forceinline__ void lds_frags(u32x4 (&v)[N], unsigned addr) {
  static_assert(N == 2 || N == 4 || N == 8, "fragment count");
  if constexpr (N == 2) {
    asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]) : "v"(addr), "i"(OFF), "i"(OFF + 1024));
  } else if constexpr (N == 4) {
    asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\t"
                 "ds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                 : "v"(addr), "i"(OFF), "i"(OFF + 1024), "i"(OFF + 2048), "i"(OFF + 3072));
  } else {
    asm volatile("ds_read_b128 %0, %8 offset:%9\n\tds_read_b128 %1, %8 offset:%10\n\t"
                 "ds_read_b128 %2, %8 offset:%11\n\tds_read_b128 %3, %8 offset:%12\n\t"
                 "ds_read_b128 %4, %8 offset:%13\n\tds_read_b128 %5, %8 offset:%14\n\t"
                 "ds_read_b128 %6, %8 offset:%15\n\tds_read_b128 %7, %8 offset:%16\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]),
                   "=&v"(v[7])
                 : "v"(addr), "i"(OFF), "i"(OFF + 1024), "i"(OFF + 2048), "i"(OFF + 3072), "i"(OFF + 4096),
                   "i"(OFF + 5120), "i"(OFF + 6144), "i"(OFF + 7168));
  }
}

template <int RT, int CT, int NW, int D, int EPI>
__global__ __launch_bounds__(64 * NW) void k_gemm_mm(GemmArgs a, int nwg) {
  constexpr int P = D + 1;
  constexpr int FA = 2 * RT;                         // activation fragments per stage (plane, row tile)
  constexpr int DPW = FA / NW;                       // activation loads per wave per stage
  static_assert(FA % NW == 0, "activation fragments per wave");
  constexpr int PER = DPW + CT;                      // loads per wave per stage
  constexpr unsigned SLOT = FA * 1024;
  extern __shared__ __align__(1024) unsigned char smem[];
  const int per = (nwg + 7) / 8;
  const int blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= a.total_items) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const void* Wg = a.g[0].W;
  int row0 = a.g[0].row0, nrows = a.g[0].nrows, n_mc = a.g[0].n_mc, item0 = a.g[0].item0, mrows = a.g[0].mrows;
#pragma unroll
  for (int i = 1; i < kMaxGroups; ++i) {
    if (i < a.ngroups && a.g[i].item0 <= blk) {
      Wg = a.g[i].W; row0 = a.g[i].row0; nrows = a.g[i].nrows; n_mc = a.g[i].n_mc; item0 = a.g[i].item0;
      mrows = a.g[i].mrows;
    }
  }
  // items of a group: ((split, column block), row chunk), row chunks
  // fastest: the chunks of one weight column block are neighbours, so they
  // run together on one XCD and its L2 serves the block to all of them
  const int ncol = a.N / (NW * CT * 16);
  const int idx = blk - item0;
  const int mc = idx % n_mc;
  const int nb = (idx / n_mc) % ncol;
  const int s = idx / (n_mc * ncol);
  const int KS = a.K >> 5;
  const int ks0 = (s * KS) / a.S, nk = ((s + 1) * KS) / a.S - ks0;
  const int crows = mrows > 0 ? mrows : RT * 16;
  const int rbase = row0 + mc * crows;
  const int rend = min(row0 + nrows, rbase + crows);  // this chunk's rows end
  const int nrt = min(RT, (rend - rbase + 15) >> 4); // row tiles holding rows (the rest are padding:
                                                     // still loaded, so every wave's load count per
                                                     // stage stays PER, but neither read nor multiplied)
  const int nt0 = (nb * NW + w) * CT;                // this wave's first 16-column weight tile

  const unsigned char* asrc[DPW];
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int f = w * DPW + i;
    const int p = f / RT, r = f % RT;
    const int row = min(rbase + 16 * r + (lane & 15), rend - 1);
    asrc[i] = (const unsigned char*)((const uint16_t*)a.X + (size_t)p * a.x_lo + (size_t)row * a.K +
                                     (size_t)ks0 * 32 + 8 * (lane >> 4));
  }
  const u32x4* bsrc = (const u32x4*)Wg + ((size_t)nt0 * KS + ks0) * 64 + lane;
  const size_t btile = (size_t)KS * 64;              // u32x4 between weight tiles
  // Every stage issues the same loads, past the last stage too (clamped to
  // it; those activation copies land in ring slots nobody reads again and
  // the weight copies are dropped), so the number of loads in flight is the
  // same at every wait and the compiler never has to drain the whole queue
  // to make a register of the ring safe to read.
  auto issueA = [&](int st) {
    const int sk = min(st, nk - 1);
    unsigned char* sl = smem + (st % P) * SLOT;
#pragma unroll
    for (int i = 0; i < DPW; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(asrc[i] + (size_t)sk * 64), MOA_LDS(sl + (w * DPW + i) * 1024),
                                       16, 0, 0);
  };
  auto loadB = [&](int st, u32x4* dst) {
    const size_t sk = (size_t)min(st, nk - 1) * 64;
#pragma unroll
    for (int c = 0; c < CT; ++c) dst[c] = bsrc[c * btile + sk];
  };

  f32x4_t acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  u32x4 breg[D][CT];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    issueA(d);
    loadB(d, breg[d]);
  }
  const unsigned lbase = lds_addr(smem) + lane * 16;
  for (int st0 = 0; st0 < nk; st0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int st = st0 + d;
      // stage st resident (D - 1 newer stages in flight); every wave done
      // with stage st - 1, whose slot is refilled next
      wait_vmcnt<(D - 1) * PER>();
      wait_lgkm0();
      asm volatile("s_barrier" ::: "memory");
      issueA(st + D);
      if (st < nk) {
        const unsigned sb = lbase + (unsigned)(st % P) * SLOT;
        u32x4 ah[RT], al[RT];
        lds_frags<RT, 0>(ah, sb);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (r < nrt) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
              acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ah[r]),
                                                                  __builtin_bit_cast(bf16x8_t, breg[d][c]), acc[r][c], 0, 0, 0);
          }
        lds_frags<RT, RT * 1024>(al, sb);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (r < nrt) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
              acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, al[r]),
                                                                  __builtin_bit_cast(bf16x8_t, breg[d][c]), acc[r][c], 0, 0, 0);
          }
      }
      loadB(st + D, breg[d]);
    }
  }
  wait_vmcnt<0>();                                   // no load may land in LDS after the workgroup ends

  const int col = lane & 15;
  const int rq = (lane >> 4) * 4;
  if (EPI == EPI_F32) {
    float* out = a.out + (size_t)s * a.out_split;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = rbase + r * 16 + rq + i;
          if (row < rend) out[(size_t)row * a.N + (nt0 + c) * 16 + col] = acc[r][c][i];
        }
  } else {
    // tiles (2p, 2p+1) are (gate, up) of the same 16 hidden units
    const int half = a.N >> 1;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int q = 0; q < CT / 2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = rbase + r * 16 + rq + i;
          if (row < rend) {
            const float g = acc[r][2 * q][i], u = acc[r][2 * q + 1][i];
            store_split(a.hout, a.h_lo, (size_t)row * half + ((nt0 >> 1) + q) * 16 + col, silu_mul(g, u));
          }
        }
  }
}

// ------------------------------------------- large-M GEMM (16x16x32 MFMA)
// Prefill chunks and wide decode batches are bound by the matrix cores. Same
// tiles as the medium-M kernel at RT = 8 (128 rows x 8 waves of 16 * CT columns,
// the same products in the same order), fed so that the MFMAs need not wait:
//  * activations go through registers into a two-slot LDS ring (loaded a stage
//    before they are written, written a stage before they are read), so the
//    compiler can follow every LDS access and no read waits for a load in flight;
//  * a stage's 16 fragment reads are spread between its MFMAs by scheduling
//    groups: eight reads ahead, then one read per CT MFMAs. With all of a plane's
//    reads and one wait in front of its 32 MFMAs the matrix cores were 64% busy.
// Same clocks, same launches: 8B qkv at 2,048 rows 184 -> 166 us, o 109 -> 105,
// gate-up 764 -> 736, down 350 -> 336; at 8,192 rows gate-up 2,920 -> 2,779 (692
// TFLOP/s useful, twice that on the MFMA for the split activations). Measured and
// not kept: 32x32x16 MFMAs (5-10% slower), 64-row waves over 128 columns
// (10-20%), two 4-wave workgroups per CU (12-18%), raised wave priority (8-10%).
template <int CT, int EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_big(GemmArgs a, int nwg) {
  constexpr int RT = 8, NW = 8, D = 3;
  constexpr unsigned SLOT = 2 * RT * 1024;
  __shared__ __align__(1024) unsigned char smem[2 * SLOT];
  const int per = (nwg + 7) / 8;
  const int blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= a.total_items) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const void* Wg = a.g[0].W;
  int row0 = a.g[0].row0, nrows = a.g[0].nrows, n_mc = a.g[0].n_mc, item0 = a.g[0].item0, mrows = a.g[0].mrows;
#pragma unroll
  for (int i = 1; i < kMaxGroups; ++i) {
    if (i < a.ngroups && a.g[i].item0 <= blk) {
      Wg = a.g[i].W; row0 = a.g[i].row0; nrows = a.g[i].nrows; n_mc = a.g[i].n_mc; item0 = a.g[i].item0;
      mrows = a.g[i].mrows;
    }
  }
  const int ncol = a.N / (NW * CT * 16);
  const int idx = blk - item0;
  const int mc = idx % n_mc;
  const int nb = (idx / n_mc) % ncol;
  const int s = idx / (n_mc * ncol);
  const int KS = a.K >> 5;
  const int ks0 = (s * KS) / a.S, nk = ((s + 1) * KS) / a.S - ks0;
  const int crows = mrows > 0 ? mrows : RT * 16;
  const int rbase = row0 + mc * crows;
  const int rend = min(row0 + nrows, rbase + crows);
  const int nrt = min(RT, (rend - rbase + 15) >> 4); // row tiles holding rows; the rest are not multiplied
  const int nt0 = (nb * NW + w) * CT;                // this wave's first 16-column weight tile

  const unsigned char* asrc[2];                      // this wave's two of the stage's 16 fragments
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int f = w * 2 + i, p = f / RT, r = f % RT;
    const int row = min(rbase + 16 * r + (lane & 15), rend - 1);
    asrc[i] = (const unsigned char*)((const uint16_t*)a.X + (size_t)p * a.x_lo + (size_t)row * a.K +
                                     (size_t)ks0 * 32 + 8 * (lane >> 4));
  }
  const u32x4* bsrc = (const u32x4*)Wg + ((size_t)nt0 * KS + ks0) * 64 + lane;
  const size_t btile = (size_t)KS * 64;              // u32x4 between weight tiles
  u32x4 ga[2], b[D][CT];
  auto loadA = [&](int st) {
    const size_t o = (size_t)min(st, nk - 1) * 64;
#pragma unroll
    for (int i = 0; i < 2; ++i) ga[i] = *(const u32x4*)(asrc[i] + o);
  };
  auto writeA = [&](int st) {
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4*)(smem + (st & 1) * SLOT + (w * 2 + i) * 1024 + lane * 16) = ga[i];
  };
  auto loadB = [&](int st, u32x4* dst) {
    const size_t o = (size_t)min(st, nk - 1) * 64;
#pragma unroll
    for (int c = 0; c < CT; ++c) dst[c] = bsrc[c * btile + o];
  };
  // LDS only: the loads in flight stay in flight
  auto barrier = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  f32x4_t acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  loadA(0);
#pragma unroll
  for (int d = 0; d < D; ++d) loadB(d, b[d]);
  writeA(0);
  loadA(1);
  barrier();
  // Stage st reads slot st & 1 while the other slot takes stage st + 1; the one
  // barrier per stage makes that slot visible and frees the one just read.
  auto loop = [&](auto full) {
    for (int st0 = 0; st0 < nk; st0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int st = st0 + d;
        if (st >= nk) break;
        const unsigned char* sl = smem + (st & 1) * SLOT + lane * 16;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            if (!full.value && r >= nrt) continue;
            const u32x4 av = *(const u32x4*)(sl + (p * RT + r) * 1024);
#pragma unroll
            for (int c = 0; c < CT; ++c)
              acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av),
                                                                  __builtin_bit_cast(bf16x8_t, b[d][c]), acc[r][c], 0, 0, 0);
          }
          if (p == 0) {
            writeA(st + 1);
            loadA(st + 2);
          }
        }
        loadB(st + D, b[d]);
        if (full.value) {
          __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);      // LDS reads
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, CT, 0);   // MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
        }
        barrier();
      }
    }
  };
  if (nrt == RT) loop(std::true_type{});
  else loop(std::false_type{});

  const int col = lane & 15;
  const int rq = (lane >> 4) * 4;
  if (EPI == EPI_F32) {
    float* out = a.out + (size_t)s * a.out_split;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = rbase + r * 16 + rq + i;
          if (row < rend) out[(size_t)row * a.N + (nt0 + c) * 16 + col] = acc[r][c][i];
        }
  } else {
    // tiles (2p, 2p+1) are (gate, up) of the same 16 hidden units
    const int half = a.N >> 1;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int q = 0; q < CT / 2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = rbase + r * 16 + rq + i;
          if (row < rend) {
            const float g = acc[r][2 * q][i], u = acc[r][2 * q + 1][i];
            store_split(a.hout, a.h_lo, (size_t)row * half + ((nt0 >> 1) + q) * 16 + col, silu_mul(g, u));
          }
        }
  }
}

// ------------------------------------------------------------ fp32 GEMM
// The fp32 engine mode: Y = X . W^T on the fp32 MFMA (16x16x4, exact fp32
// products), W row-major [N][K]. Small models' fp32 steps are bound by latency
// (their weights fit the caches), so the work of a launch is spread wide and
// every lane keeps 16-byte loads in flight:
//  * a workgroup owns 16 rows x CT 16-column tiles, its four waves a quarter
//    of K each; their sums meet in LDS in fixed order;
//  * lane l loads 4 consecutive k of row (A) or column (B) l % 16 at
//    k = 16 j + 4 (l / 16): element i of that quad feeds the i-th of four
//    MFMAs, which permutes k the same way in A and B and changes no product.
// K is a multiple of 64 (d_model, n_heads * head_dim and ffn_dim all are).
// EPI_SWIGLU (gate-up, rows of W are [gate(F) | up(F)]): tiles 2p and 2p + 1 are
// the gate and up columns of the same 16 hidden units, and h = silu(gate) * up
// is written by the same launch.
// Before: one lane per column walking K alone, 4 rows per lane: 62.8 us per
// launch over the tiny fp32 mixture's passes (d 256, ffn 1024, 1-32 rows).
template <int CT, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs a) {
  constexpr int SUB = 4 / CT;                        // workgroups per 64-column item
  __shared__ float red[4][CT][256];
  const int item = blockIdx.x / SUB, sub = blockIdx.x % SUB;
  const void* Wg = a.g[0].W;
  int row0 = a.g[0].row0, nrows = a.g[0].nrows, n_mc = a.g[0].n_mc, item0 = a.g[0].item0;
#pragma unroll
  for (int i = 1; i < kMaxGroups; ++i) {
    if (i < a.ngroups && a.g[i].item0 <= item) {
      Wg = a.g[i].W; row0 = a.g[i].row0; nrows = a.g[i].nrows; n_mc = a.g[i].n_mc; item0 = a.g[i].item0;
    }
  }
  const int idx = item - item0;
  const int mc = idx % n_mc, nb = idx / n_mc;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int tile0 = nb * 4 + sub * CT;               // first 16-column tile (SWIGLU: unit tile tile0 / 2)
  const int half = a.N >> 1;
  const int rbase = row0 + mc * 16;
  const int rend = row0 + nrows;
  auto col0 = [&](int c) { return EPI == EPI_SWIGLU ? (tile0 / 2 + c / 2) * 16 + (c & 1) * half : (tile0 + c) * 16; };
  const int kq = a.K >> 2;
  const size_t ko = (size_t)w * kq + 4 * (lane >> 4);
  const float* xp = (const float*)a.X + (size_t)min(rbase + (lane & 15), rend - 1) * a.K + ko;
  const float* wp[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) wp[c] = (const float*)Wg + (size_t)(col0(c) + (lane & 15)) * a.K + ko;
  f32x4_t acc[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k = 0; k < kq; k += 16) {
    const f32x4_t x = *(const f32x4_t*)(xp + k);
    f32x4_t b[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) b[c] = *(const f32x4_t*)(wp[c] + k);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], b[c][i], acc[c], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[w][c][(4 * (lane >> 4) + i) * 16 + (lane & 15)] = acc[c][i];
  __syncthreads();
  const int row = rbase + (threadIdx.x >> 4), cc = threadIdx.x & 15;
  if (row >= rend) return;
  float y[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
    y[c] = (red[0][c][threadIdx.x] + red[1][c][threadIdx.x]) + (red[2][c][threadIdx.x] + red[3][c][threadIdx.x]);
  if (EPI == EPI_F32) {
#pragma unroll
    for (int c = 0; c < CT; ++c) a.out[(size_t)row * a.N + col0(c) + cc] = y[c];
  } else {
#pragma unroll
    for (int c = 0; c + 1 < CT; c += 2) a.out[(size_t)row * half + col0(c) + cc] = y[c] / (1.f + expf(-y[c])) * y[c + 1];
  }
}

// ------------------------------------------------------ RoPE + KV append
// Reduces the QKV partial sums, rotates q and k (pairs (i, i + hd/2) turned by
// pos * theta^(-2i/hd), table precomputed in fp64 and rounded to fp32), stores
// q (fp32), and writes k, v (rounded to the cache type) into the row's paged-KV slot: block bt[pos / 16], slot
// pos % 16. Pool layout: [layer][block][kv_head][K|V][16][hd].
template <bool BF>
__global__ __launch_bounds__(256) void k_rope_kv(const float* __restrict__ part, int nsplit, size_t split_stride,
                                                 const int* __restrict__ row_pos, const int* __restrict__ row_bt,
                                                 const int* __restrict__ bt_store, const float2* __restrict__ tab,
                                                 float* __restrict__ qv, void* __restrict__ kvv, int layer, int NB,
                                                 int n_h, int n_kv, int hd) {
  // work items of a row: (n_h + n_kv) * hd/2 rotation pairs, then n_kv * hd v elements
  const int t = blockIdx.x;
  const int item = blockIdx.y * 256 + threadIdx.x;
  const int half = hd >> 1;
  const int npairs = (n_h + n_kv) * half;
  if (item >= npairs + n_kv * hd) return;
  const int pos = row_pos[t];
  const int qkv = (n_h + 2 * n_kv) * hd;
  const float* pr = part + (size_t)t * qkv;
  const int blk = bt_store[row_bt[t] + (pos >> 4)];
  const int off = pos & 15;
  const size_t hs = (size_t)2 * kBlock * hd;
  const size_t lbase = ((size_t)layer * NB + blk) * n_kv * hs;
  if (item < npairs) {
    const int head = item / half, jj = item - head * half;
    const int c = head * hd + jj;
    const float2 cs = tab[(size_t)pos * half + jj];   // in flight with the partial sums
    float x1 = 0.f, x2 = 0.f;
#pragma unroll 16
    for (int s = 0; s < nsplit; ++s) {
      x1 += pr[(size_t)s * split_stride + c];
      x2 += pr[(size_t)s * split_stride + c + half];
    }
    const float2 y = rotate(x1, x2, cs);
    const float y1 = y.x, y2 = y.y;
    if (head < n_h) {
      const size_t o = ((size_t)t * n_h + head) * hd + jj;
      qv[o] = y1;
      qv[o + half] = y2;
    } else {
      const size_t o = lbase + (size_t)(head - n_h) * hs + off * hd + jj;
      if (BF) { ((uint16_t*)kvv)[o] = f2bf(y1); ((uint16_t*)kvv)[o + half] = f2bf(y2); }
      else { ((float*)kvv)[o] = y1; ((float*)kvv)[o + half] = y2; }
    }
  } else {
    const int i = item - npairs;
    const int kh = i / hd, dd = i - kh * hd;
    const int c = (n_h + n_kv) * hd + i;
    float v = 0.f;
#pragma unroll 16
    for (int s = 0; s < nsplit; ++s) v += pr[(size_t)s * split_stride + c];
    const size_t o = lbase + (size_t)kh * hs + kBlock * hd + off * hd + dd;
    if (BF) ((uint16_t*)kvv)[o] = f2bf(v);
    else ((float*)kvv)[o] = v;
  }
}

// ------------------------------------------------ paged attention (split-KV)
// One workgroup = one query row x one KV head x one key range [k0, k1); its
// GQ wavefronts are the GQ query heads that share the KV head, so each K/V
// tile is read from HBM once for the whole group. The range's block ids are
// first copied to LDS (dynamic shared memory sized by the host), then tiles
// of 64 keys are staged in LDS with 16-byte coalesced loads (a 16-slot block
// of one KV head is contiguous); the next tile's loads are issued into
// registers before the current tile is computed. In a tile, lane l owns key
// 8*p + l/8 (p = 0..7) and head-dim chunk l%8: q.k partial dots are combined
// across the 8 lanes of a key with xor-shuffles, the tile max across the
// wavefront with shuffles, and P.V accumulates per lane on its own keys and
// dims (combined once at the end). Softmax runs in base 2 on scores
// pre-scaled by log2(e)/sqrt(hd).
#ifndef ATTN_WPE
#define ATTN_WPE 1
#endif
template <int HD, int GQ, bool BF, int TK>
__global__ __launch_bounds__(GQ * 64, ATTN_WPE) void k_attn(const AttnItem* __restrict__ items, const float* __restrict__ qv,
                                                  const void* __restrict__ kvv, const int* __restrict__ bt_store,
                                                  const int* __restrict__ row_bt, int layer, int NB, int n_h,
                                                  int n_kv, float scale_log2, void* __restrict__ outv,
                                                  size_t out_lo, float* __restrict__ pacc, float* __restrict__ pml) {
  constexpr int CH = HD / 8;
  constexpr int ESZ = BF ? 2 : 4;
  constexpr int ROWB = HD * ESZ;
  constexpr int CPR = ROWB / 16;                 // 16-byte chunks per key row
  constexpr int NCH = 2 * TK * CPR;              // chunks per tile (K and V)
  constexpr int NT = GQ * 64;
  constexpr int PER = (NCH + NT - 1) / NT;       // chunks per thread
  __shared__ __align__(16) unsigned char sK[TK * ROWB];
  __shared__ __align__(16) unsigned char sV[TK * ROWB];
  extern __shared__ unsigned long long sbo[];    // byte offsets of the key range's blocks in the layer's pool

  const AttnItem it = items[blockIdx.x];
  const int kvh = blockIdx.y;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g8 = lane >> 3, c8 = lane & 7;
  const int h = kvh * GQ + w;

  const size_t hs = (size_t)2 * kBlock * HD;     // elements per (block, kv head)
  const unsigned char* pool = (const unsigned char*)kvv + ((size_t)layer * NB * n_kv + kvh) * hs * ESZ;
  const unsigned long long blk_stride = (unsigned long long)n_kv * hs * ESZ;
  const int b0 = it.k0 >> 4, nb = ((it.k1 - 1) >> 4) - b0 + 1;
  {
    const int* bt = bt_store + it.bt_off;
    for (int i = threadIdx.x; i < nb; i += NT) sbo[i] = (unsigned long long)bt[i] * blk_stride;
  }
  // bf16 cache: q enters the dot products as a split-bf16 pair (hi + lo,
  // pre-scaled by log2(e)/sqrt(hd)) through v_dot2_f32_bf16, which multiplies
  // bf16 pairs exactly and accumulates in fp32; fp32 cache: plain fp32 q.
  float q[BF ? 1 : CH];
  unsigned qh[BF ? CH / 2 : 1], ql[BF ? CH / 2 : 1];
  {
    const size_t qo = ((size_t)it.row * n_h + h) * HD + c8 * CH;
    if (BF) {
#pragma unroll
      for (int i = 0; i < CH / 2; ++i)
        split_pair(qv[qo + 2 * i] * scale_log2, qv[qo + 2 * i + 1] * scale_log2, qh[i], ql[i]);
    } else {
#pragma unroll
      for (int i = 0; i < CH; ++i) q[i] = qv[qo + i];
    }
  }
  float m = -INFINITY, l = 0.f, acc[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) acc[i] = 0.f;

  // loop-invariant part of every chunk this thread moves: key in the tile,
  // byte offset inside its 16-slot block, LDS destination
  int ckey[PER];
  unsigned coff[PER];
  unsigned char* cdst[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int c = min((int)threadIdx.x + j * NT, NCH - 1);
    const int isV = c / (TK * CPR);
    const int rem = c - isV * (TK * CPR);
    const int key = rem / CPR, cc = rem - key * CPR;
    ckey[j] = (threadIdx.x + j * NT < NCH) ? key : (1 << 29);     // out-of-tile chunks never load
    coff[j] = (unsigned)((isV * kBlock * HD + (key & 15) * HD) * ESZ + cc * 16);
    cdst[j] = (isV ? sV : sK) + rem * 16;
  }
  __syncthreads();

  uint4 pre[PER];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int p = t0 + ckey[j];
      uint4 val = make_uint4(0u, 0u, 0u, 0u);
      if (p < it.k1) val = *(const uint4*)(pool + sbo[(p >> 4) - b0] + coff[j]);
      pre[j] = val;
    }
  };
  fetch(it.k0);
  for (int t0 = it.k0; t0 < it.k1; t0 += TK) {
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (threadIdx.x + j * NT < NCH) *(uint4*)cdst[j] = pre[j];
    __syncthreads();
    if (t0 + TK < it.k1) fetch(t0 + TK);

    constexpr int NP = TK / 8;                   // keys per lane group
    float s[NP];
#pragma unroll
    for (int p8 = 0; p8 < NP; ++p8) {
      const int key = p8 * 8 + g8;
      float dot = 0.f;
      if (BF) {
        const unsigned* kr = (const unsigned*)(sK + key * ROWB + c8 * CH * 2);
#pragma unroll
        for (int i = 0; i < CH / 2; ++i) {
          const bf16x2_t kp = __builtin_bit_cast(bf16x2_t, kr[i]);
          dot = __builtin_amdgcn_fdot2_f32_bf16(kp, __builtin_bit_cast(bf16x2_t, qh[i]), dot, false);
          dot = __builtin_amdgcn_fdot2_f32_bf16(kp, __builtin_bit_cast(bf16x2_t, ql[i]), dot, false);
        }
        dot = sum8(dot);
      } else {
        const float* kr = (const float*)(sK + key * ROWB) + c8 * CH;
#pragma unroll
        for (int i = 0; i < CH; ++i) dot = fmaf(q[i], kr[i], dot);
        dot = sum8(dot) * scale_log2;
      }
      s[p8] = (t0 + key < it.k1) ? dot : -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int p8 = 1; p8 < NP; ++p8) mx = fmaxf(mx, s[p8]);
    mx = fmaxf(mx, dpp<0x128>(mx));
    mx = fmaxf(mx, swz_xor16(mx));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx);
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    l *= alpha;
#pragma unroll
    for (int i = 0; i < CH; ++i) acc[i] *= alpha;
#pragma unroll
    for (int p8 = 0; p8 < NP; ++p8) {
      const float pj = __builtin_amdgcn_exp2f(s[p8] - mnew);
      l += pj;
      const int key = p8 * 8 + g8;
      if (BF) {
        const uint16_t* vr = (const uint16_t*)(sV + key * ROWB) + c8 * CH;
#pragma unroll
        for (int i = 0; i < CH; ++i) acc[i] = fmaf(pj, bf2f(vr[i]), acc[i]);
      } else {
        const float* vr = (const float*)(sV + key * ROWB) + c8 * CH;
#pragma unroll
        for (int i = 0; i < CH; ++i) acc[i] = fmaf(pj, vr[i], acc[i]);
      }
    }
    m = mnew;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    acc[i] += __shfl_xor(acc[i], 8, 64);
    acc[i] += __shfl_xor(acc[i], 16, 64);
    acc[i] += __shfl_xor(acc[i], 32, 64);
  }
  l += __shfl_xor(l, 8, 64);
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (g8 == 0) {
    if (it.slot < 0) {
      const float inv = 1.f / l;
      const size_t o = ((size_t)it.row * n_h + h) * HD + c8 * CH;
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        if (BF) store_split((uint16_t*)outv, out_lo, o + i, acc[i] * inv);
        else ((float*)outv)[o + i] = acc[i] * inv;
      }
    } else {
      const size_t o = ((size_t)it.slot * n_h + h) * HD + c8 * CH;
#pragma unroll
      for (int i = 0; i < CH; ++i) pacc[o + i] = acc[i];
      if (c8 == 0) {
        pml[((size_t)it.slot * n_h + h) * 2] = m;
        pml[((size_t)it.slot * n_h + h) * 2 + 1] = l;
      }
    }
  }
}

// x combined with the other half-wave's (lane ^ 32), without an LDS round trip
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float add_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// ------------------------------------------ causal prefill attention (MFMA)
// Causal prefill attention on the 32x32x16 MFMA. A workgroup is one query
// head and up to kPrefillRows consecutive positions of one request, four
// wavefronts of 32 query rows each; key tiles of 32 keys cover [0, pos0 + nq).
// Scores are formed transposed, S^T = K Q^T (A = K tile, B = the wave's q
// rows), so lane l of a wave holds the 16 scores of query row l%32 for keys
// 8(e/4) + 4(l/32) + e%4 of the tile: the online softmax is per lane (plus
// one exchange with lane l^32), and those 16 probabilities are directly the
// B operand of O^T = V^T P^T, with the key order inside each 16-key step
// permuted identically in A (V^T, read from LDS) and B (P^T, in registers).
// q and P enter the MFMAs as split bf16 (hi + lo, two MFMAs each). K and V tiles
// reach LDS by direct global->LDS loads into three-stage rings, K in MFMA fragment
// order, V in its rows, read transposed.
// Bound by issue: per tile a wave owes 32 MFMAs and ~190 VALU instructions, and
// the SIMD's two waves together keep the matrix cores 58% and the VALU 55% busy.
// So both are kept short and side by side:
//  * the next tile's scores are multiplied between this tile's softmax
//    instructions, two MFMAs and a share of the softmax at a time, and half of P
//    is split between the MFMAs of P V;
//  * addresses: wave-uniform parts are scalar, block ids are read an iteration
//    ahead in units of one head's block.
// Mean launch over 9,001- and 17,003-token prompts at 32 heads of 128 (16k-row
// chunks): 3,281 us with scores, softmax and P V one after the other, 2,878 so.
// Starting the scores' sums from minus the reference maximum and running q hi and
// q lo in one chain would save 37 us more, but loses precision (see below).
#ifndef PREFILL_WPE
#define PREFILL_WPE 2
#endif
template <int HD>
__global__ __launch_bounds__(256, PREFILL_WPE) void k_prefill_attn(const PrefillItem* __restrict__ items,
                                                      const float* __restrict__ qv, const uint16_t* __restrict__ kv,
                                                      const int* __restrict__ bt_store, int layer, int NB, int n_h,
                                                      int n_kv, float scale_log2, uint16_t* __restrict__ out,
                                                      size_t out_lo) {
  constexpr int TK = 32;                    // keys per tile
  constexpr int DS = HD / 16;               // 16-wide dim steps of S^T = K Q^T
  constexpr int DT = HD / 32;               // 32-dim tiles of O^T
  constexpr int KFR = DS;                   // K fragments (1 KB) per tile
  constexpr int KPW = KFR / 4;              // K fragments loaded per wave
  constexpr int ROWB = HD * 2;              // bytes per V row
  constexpr int CPR = ROWB / 16;            // 16-byte chunks per V row
  constexpr int KPF = 1024 / ROWB;          // V rows per 1 KB fragment
  constexpr int VFR = TK * ROWB / 1024;     // V fragments per tile
  constexpr int VPW = VFR / 4;              // V fragments loaded per wave
  constexpr int NKS = 3;                    // ring stages (K and V)
  static_assert(KPW >= 1 && KPW * 4 == KFR && VPW >= 1 && VPW * 4 == VFR, "tile shape");
  // One dynamic LDS block (sized by the launcher): the K ring (NKS x KFR KB),
  // the V ring (NKS x VFR KB), then the block ids of keys [0, kmax).
  extern __shared__ __align__(1024) unsigned char sKd[];
  unsigned char* sV = sKd + NKS * KFR * 1024;
  int* sbt = (int*)(sV + NKS * VFR * 1024);

  const PrefillItem it = items[blockIdx.x];
  const int h = blockIdx.y;
  const int kvh = h / (n_h / n_kv);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c32 = lane & 31, hf = lane >> 5;
  const int kmax = it.pos0 + it.nq;          // keys [0, kmax)
  const int ntile = (kmax + TK - 1) / TK;
  constexpr unsigned HS = 2 * kBlock * HD;   // elements of one head's K and V of a block
  const uint16_t* pool = kv + ((size_t)layer * NB * n_kv + kvh) * HS;
  // The block ids live in LDS for the whole item: a K/V address then never
  // waits on a global load, which (vector loads complete in order) would also
  // wait for every tile already in flight.
  {
    const int* bt = bt_store + it.bt_off;
    const int nblk = (kmax + kBlock - 1) / kBlock;
    for (int i = threadIdx.x; i < nblk; i += 256) sbt[i] = bt[i] * n_kv;   // in units of HS
    __syncthreads();
  }

  // B operand of S^T: query row 32w + l%32 (rows past nq read row nq-1 and
  // are never stored), dims 16s + 8(l/32) .. +8, scaled to log2 units, split
  u32x4 qh[DS], ql[DS];
  {
    const int r = min(32 * w + c32, it.nq - 1);
    const float* qrow = qv + ((size_t)(it.row0 + r) * n_h + h) * HD + 8 * hf;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
      unsigned hv[4], lv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        split_pair(qrow[16 * s + 2 * j] * scale_log2, qrow[16 * s + 2 * j + 1] * scale_log2, hv[j], lv[j]);
      qh[s] = u32x4{hv[0], hv[1], hv[2], hv[3]};
      ql[s] = u32x4{lv[0], lv[1], lv[2], lv[3]};
    }
  }
  const int qpos = it.pos0 + 32 * w + c32;   // this lane's query position

  // Tiles of K and V go by direct loads into their rings (tile t in slot t % NKS).
  // K fragment s holds key t*32 + l%32, dims 16s + 8(l/32) .. +8 in lane l.
  // V keeps its natural [key][dim] rows; the 16-byte chunk c of row r sits at
  // chunk position c ^ 2(r % 4), so the four rows a transposed read touches
  // fall on different LDS banks. The block ids of the next loads (kid, vid) are
  // read an iteration before their addresses are formed. The eight rows of V that
  // a wave brings lie in one block (rows past kmax - 1 repeat that one, which is
  // then among them or all of them).
  const int vrow_in = lane / CPR, vcp = lane % CPR;
  auto k_key = [&](int t) { return min(t * TK + c32, kmax - 1); };
  auto v_key = [&](int t, int i) { return min(t * TK + (w * VPW + i) * KPF + vrow_in, kmax - 1); };
  static_assert(VPW * KPF == 8, "V rows per wave");
  unsigned kid, vid;
  auto ids = [&](int tk, int tv) {
    kid = sbt[k_key(tk) >> 4];
    vid = sbt[min(tv * TK + 8 * w, kmax - 1) >> 4];
  };
  auto issue_k = [&](int t) {
    const uint16_t* base = pool + (size_t)kid * HS + (k_key(t) & 15) * HD + 8 * hf;
    unsigned char* sl = sKd + (t % NKS) * KFR * 1024;
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const int s = w * KPW + i;
      __builtin_amdgcn_global_load_lds((const void*)(base + 16 * s), MOA_LDS(sl + s * 1024), 16, 0, 0);
    }
  };
  auto issue_v = [&](int t) {
    unsigned char* vs = sV + (t % NKS) * VFR * 1024;
    const uint16_t* base = pool + (size_t)(unsigned)__builtin_amdgcn_readfirstlane(vid) * HS + kBlock * HD;
#pragma unroll
    for (int i = 0; i < VPW; ++i) {
      const int f = w * VPW + i;
      const int r = f * KPF + vrow_in;                    // row of the tile this lane fills
      const int gc = vcp ^ ((r & 3) << 1);                // chunk of the key's row it brings
      const uint16_t* src = base + (unsigned)((v_key(t, i) & 15) * HD + gc * 8);
      __builtin_amdgcn_global_load_lds((const void*)src, MOA_LDS(vs + f * 1024), 16, 0, 0);
    }
  };
  // Transposed V reads (ds_read_b64_tr_b16: within each 16 lanes, lane 4b+e
  // receives element e of the 8-byte reads of lanes 4a+b, a = 0..3). Lane
  // 4a+b of group g reads row 16u + 4(l/32) + a (+8), dims
  // 32d + 16(g%2) + 4b .. +4; after the transpose lane l holds dim 32d + l%32
  // of rows 16u + 4(l/32) + 0..3 (+8): the A operand of O^T = V^T P^T with the
  // slot order of P below.
  const int ta = (lane & 15) >> 2, tb = lane & 3, tg = lane >> 4;
  unsigned vcol[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d)
    vcol[d] = (unsigned)((((4 * d + 2 * (tg & 1) + (tb >> 1)) ^ (2 * ta)) * 16) + 8 * (tb & 1));
  const unsigned vrowoff = (unsigned)((4 * hf + ta) * ROWB);
  auto barrier = [] {
    wait_lgkm0();
    asm volatile("s_barrier" ::: "memory");
  };

  f32x16_t O[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) O[d] = f32x16_t{};
  float m = -INFINITY, l = 0.f;

  // One 16-dim step of a tile's scores, in two chains that both grow from zero:
  // a sum that starts at the reference maximum rounds every product at that
  // magnitude, the small q lo ones too (2.6x the rounding error at head_dim 128).
  f32x16_t A, A2;                            // q hi, q lo
  auto kfrag = [&](int t, int s) { return *(const u32x4*)(sKd + ((t % NKS) * KFR + s) * 1024 + lane * 16); };
  auto score = [&](int s, const u32x4& ka) {
    A = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ka), __builtin_bit_cast(bf16x8_t, qh[s]), s ? A : f32x16_t{}, 0, 0, 0);
    A2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ka), __builtin_bit_cast(bf16x8_t, ql[s]), s ? A2 : f32x16_t{}, 0, 0, 0);
  };
  // causal mask (only tiles that reach past the wave's first query or past
  // kmax need it) for query qpos (element e: key kb + 8(e/4) + e%4)
  auto mask = [&](int t, f32x16_t& S) {
    const int kb = t * TK + 4 * hf;
    if (t * TK + TK - 1 > it.pos0 + 32 * w || t * TK + TK > kmax) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = kb + 8 * (e >> 2) + (e & 3);
        if (key > qpos || key >= kmax) S[e] = -INFINITY;
      }
    }
  };
  // Every iteration issues the same loads, past the last tile too (keys are
  // clamped to kmax - 1, so those read valid memory and land in slots nobody
  // reads): the number of loads in flight is then the same at every point of
  // the loop, and each wait below is exact rather than a full drain. Iteration t
  // multiplies K of tile t + 1 and V of tile t, so K is issued three tiles
  // ahead and V two, each into the slot that iteration t - 1 read.
  ids(0, 0);
  issue_k(0);
  ids(1, 0);
  issue_k(1);
  issue_v(0);
  ids(2, 1);
  issue_k(2);
  issue_v(1);
  ids(3, 2);
  wait_vmcnt<2 * (KPW + VPW)>();
  barrier();
#pragma unroll
  for (int s = 0; s < DS; ++s) score(s, kfrag(0, s));
  f32x16_t S = A + A2;
  mask(0, S);
  auto step = [&](int t, auto more) {
    // K of tile t + 1 and V of tile t landed (issued after them: K t+2, V t+1)
    wait_vmcnt<KPW + VPW>();
    barrier();                               // visible; the slots of iteration t - 1 are free
    // The next tile's scores beside this tile's softmax, two MFMAs and a share of
    // the softmax at a time: the matrix cores work while the VALU does, in one wave.
    float ts = 0.f, base, alpha;
    u32x4 ph[2], pl[2];                        // P as the B operand: slot j of 16-key step u is key 16u + 8(j/4) + 4(l/32) + j%4
    // The reference maximum moves only when a score exceeds it by more than
    // 2^8 (log2 units): probabilities then stay below 256, exact in the split
    // and harmless in fp32, and the rescale of O below is rare.
    auto reference = [&] {
      float mx = S[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
      mx = max_halves(mx);
      const float mn = (mx > m + 8.f) ? mx : m;
      base = (mn == -INFINITY) ? 0.f : mn;     // a row with no score yet keeps m = -inf
      alpha = __builtin_amdgcn_exp2f(m - base);
      m = mn;
      if (!__all(alpha == 1.f)) {              // no row's maximum moved: nothing to rescale
#pragma unroll
        for (int d = 0; d < DT; ++d) O[d] *= alpha;
      }
    };
    auto split = [&](int j) {
      unsigned hv, lv;
      split_pair(S[2 * j], S[2 * j + 1], hv, lv);
      asm volatile("" : "+v"(hv), "+v"(lv));   // here and not beside their use
      ph[j >> 2][j & 3] = hv;
      pl[j >> 2][j & 3] = lv;
    };
    auto pair = [&](int j) {
#pragma unroll
      for (int e = 2 * j; e < 2 * j + 2; ++e) {
        S[e] = __builtin_amdgcn_exp2f(S[e] - base);
        ts += S[e];
      }
      asm volatile("" : "+v"(ts));
      if (j < 4) split(j);                     // the others beside the first half of P V
    };
    if constexpr (more.value) {
      u32x4 kf[3] = {kfrag(t + 1, 0), kfrag(t + 1, 1), u32x4{}};
#pragma unroll
      for (int s = 0; s < DS; ++s) {
        if (s + 2 < DS) kf[(s + 2) % 3] = kfrag(t + 1, s + 2);
        score(s, kf[s % 3]);
        if (s == 1) issue_k(t + 3);
        if (s == 2) issue_v(t + 2);
        if (s == 3) ids(t + 4, t + 3);
        if (s == 0) reference();
        else
#pragma unroll
          for (int j = (s - 1) * 8 / (DS - 1); j < s * 8 / (DS - 1); ++j) pair(j);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      reference();
#pragma unroll
      for (int j = 0; j < 8; ++j) pair(j);
    }
    l = l * alpha + add_halves(ts);
    // O^T += V^T P^T over two 16-key steps.
    // The V reads are explicit LDS instructions with an explicit wait tied to
    // their registers: the compiler, which cannot tell them from the ring
    // slots the direct loads are filling, would otherwise wait for every load
    // in flight (the tile two ahead included) before the first of them.
    const unsigned vb = lds_addr(sV + (t % NKS) * VFR * 1024) + vrowoff;
    u32x4 va[2][DT];
#pragma unroll
    for (int d = 0; d < DT; ++d) {
      va[0][d] = ds_read_tr16_pair<0 * ROWB, 8 * ROWB>(vb + vcol[d]);
      va[1][d] = ds_read_tr16_pair<16 * ROWB, 24 * ROWB>(vb + vcol[d]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int d = 0; d < DT; ++d) lgkm_wait_for(va[u][d]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int d = 0; d < DT; ++d)
        O[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, va[u][d]), __builtin_bit_cast(bf16x8_t, ph[u]), O[d], 0, 0, 0);
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        O[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, va[u][d]), __builtin_bit_cast(bf16x8_t, pl[u]), O[d], 0, 0, 0);
        if (u == 0)
#pragma unroll
          for (int j = 4 + d * 4 / DT; j < 4 + (d + 1) * 4 / DT; ++j) split(j);
      }
      if (u == 0) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (more.value) {
      S = A + A2;
      mask(t + 1, S);
    }
  };
  for (int t = 0; t + 1 < ntile; ++t) step(t, std::true_type{});
  step(ntile - 1, std::false_type{});
  wait_vmcnt<0>();                           // no load may land in LDS after this workgroup ends
  // normalise and store: element e of O[d] is dim 32d + 8(e/4) + 4(l/32) + e%4 of row 32w + l%32
  const int r = 32 * w + c32;
  if (r < it.nq) {
    const float inv = 1.f / l;
    const size_t o = ((size_t)(it.row0 + r) * n_h + h) * HD + 4 * hf;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int e = 0; e < 16; ++e) store_split(out, out_lo, o + 32 * d + 8 * (e >> 2) + (e & 3), O[d][e] * inv);
  }
}

// Combine the key-range partials of one row (fixed order over ranges).
template <bool BF>
__global__ __launch_bounds__(256) void k_attn_reduce(const ReduceItem* __restrict__ red, const float* __restrict__ pacc,
                                                     const float* __restrict__ pml, void* __restrict__ outv,
                                                     size_t out_lo, int n_h, int hd) {
  // One workgroup per (row, head); G = 256 / hd groups of hd lanes take every
  // G-th slot in one pass, each with its own running maximum (its sums are
  // rescaled when a slot's maximum exceeds it), so no pass over the slots
  // waits for another; then the G groups are merged in fixed order.
  __shared__ float sm[4], sl[4];
  __shared__ float so[256];
  const ReduceItem it = red[blockIdx.y];
  const int h = blockIdx.x;
  const int G = 256 / hd;
  const int g = threadIdx.x / hd, dd = threadIdx.x % hd;
  float M = -INFINITY, L = 0.f, o = 0.f;
#pragma unroll 4
  for (int s = g; s < it.nslots; s += G) {
    const size_t b = (size_t)(it.slot0 + s) * n_h + h;
    const float ms = pml[b * 2], ls = pml[b * 2 + 1], as = pacc[b * hd + dd];
    const float mn = fmaxf(M, ms);
    const float wa = __builtin_amdgcn_exp2f(M - mn), wb = __builtin_amdgcn_exp2f(ms - mn);
    L = L * wa + ls * wb;
    o = o * wa + as * wb;
    M = mn;
  }
  so[threadIdx.x] = o;
  if (dd == 0) { sm[g] = M; sl[g] = L; }
  __syncthreads();
  if (g == 0) {
    float Mt = sm[0];
    for (int k = 1; k < G; ++k) Mt = fmaxf(Mt, sm[k]);
    float Lt = 0.f, ot = 0.f;
    for (int k = 0; k < G; ++k) {
      const float w = __builtin_amdgcn_exp2f(sm[k] - Mt);   // a group without slots: -inf -> 0
      Lt += sl[k] * w;
      ot += so[k * hd + dd] * w;
    }
    const size_t oo = ((size_t)it.row * n_h + h) * hd + dd;
    if (BF) store_split((uint16_t*)outv, out_lo, oo, ot / Lt);
    else ((float*)outv)[oo] = ot / Lt;
  }
}

// ------------------------------------------------------------------ argmax
// Greedy sampler: the largest fp32 logit, ties to the lowest token id; the
// token is written into the device token store (it feeds the next step).
__global__ __launch_bounds__(1024) void k_argmax(const float* __restrict__ logits, int V,
                                                 const int* __restrict__ lm_dst, int* __restrict__ tok) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const int r = blockIdx.x;
  const float* lr = logits + (size_t)r * V;
  float best = -INFINITY;
  int bi = INT_MAX;
  // V % 4 == 0: each thread scans float4 groups in increasing index order, so a
  // strict '>' keeps the lowest index among its equal maxima.
  // Eight groups' loads are issued before any of them is compared.
  constexpr int B = 8;
  for (int v0 = threadIdx.x; v0 < V / 4; v0 += 1024 * B) {
    float4 xs[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int v4 = v0 + 1024 * k;
      xs[k] = (v4 < V / 4) ? *(const float4*)(lr + 4 * v4) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int v4 = v0 + 1024 * k;
      const float4 x = xs[k];
      if (x.x > best) { best = x.x; bi = 4 * v4; }
      if (x.y > best) { best = x.y; bi = 4 * v4 + 1; }
      if (x.z > best) { best = x.z; bi = 4 * v4 + 2; }
      if (x.w > best) { best = x.w; bi = 4 * v4 + 3; }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sv[w] = best; si[w] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    best = sv[0];
    bi = si[0];
    for (int k = 1; k < 16; ++k)
      if (sv[k] > best || (sv[k] == best && si[k] < bi)) { best = sv[k]; bi = si[k]; }
    tok[lm_dst[r]] = (bi == INT_MAX) ? 0 : bi;
  }
}

// ------------------------------------------------------ injected history
template <typename T>
__global__ __launch_bounds__(256) void k_kv_scatter(const T* __restrict__ src, T* __restrict__ kv,
                                                    const int* __restrict__ blocks, int p0, int n, int layer,
                                                    int kv_sel, int NB, int n_kv, int hd) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t per = (size_t)n_kv * hd;
  if (e >= (size_t)n * per) return;
  const int p = p0 + (int)(e / per);
  const int rem = (int)(e % per);
  const int h = rem / hd, d = rem - h * hd;
  const size_t hs = (size_t)2 * kBlock * hd;
  const size_t o = (((size_t)layer * NB + blocks[p >> 4]) * n_kv + h) * hs + (size_t)kv_sel * kBlock * hd +
                   (p & 15) * hd + d;
  kv[o] = src[e];
}

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
  return x;
}

// One workgroup per (KV block of 16 positions, layer) of every filled request
// of a step: the block's K and V of all heads are one contiguous run, written 16
// bytes per lane. Before: a launch per request, one 2-byte store per lane: 24 us
// a request of 200 to 8,000 positions (8B shape, two layers), 250 requests one
// after the other.
template <bool BF, int HD>
__global__ __launch_bounds__(256) void k_kv_fill(void* __restrict__ kvv, const int* __restrict__ bt_store,
                                                 const FillReq* __restrict__ reqs, int nreqs, int NB, int n_kv) {
  const int item = blockIdx.x, layer = blockIdx.y;
  int lo = 0, hi = nreqs - 1;                        // the last entry with item0 <= item
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (reqs[mid].item0 <= item) lo = mid;
    else hi = mid - 1;
  }
  const FillReq rq = reqs[lo];
  const int b = item - rq.item0;
  constexpr int EL = BF ? 8 : 4;                     // elements per 16-byte store
  const size_t run = (size_t)n_kv * 2 * kBlock * HD;
  const size_t base = ((size_t)layer * NB + bt_store[rq.bt_off + b]) * run;
  const uint32_t tg = rq.tag * 0x9e3779b9u;
  for (int e = threadIdx.x * EL; e < (int)run; e += 256 * EL) {
    const int head = e / (2 * kBlock * HD), kv_sel = (e / (kBlock * HD)) & 1, slot = (e / HD) & (kBlock - 1);
    const int p = b * kBlock + slot;
    if (p >= rq.ctx) continue;
    const uint32_t hp = tg ^ mix32(((uint32_t)(layer * 2 + kv_sel) << 24) ^ (uint32_t)p);
    const int rem = head * HD + e % HD;
    float v[EL];
#pragma unroll
    for (int i = 0; i < EL; ++i) {
      const uint32_t u = mix32(hp ^ (uint32_t)((rem + i) * 0x85ebca6bu));
      v[i] = (float)(int)(u >> 8) * (1.0f / 8388608.0f) - 1.0f;
    }
    if constexpr (BF)
      *(uint4*)((uint16_t*)kvv + base + e) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                                        pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    else
      *(float4*)((float*)kvv + base + e) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// --------------------------------------------- host <-> device small copies
// A step's metadata, prompts and block lists (and a collect's tokens) are many
// short runs; one launch moves them all straight from (to) pinned host memory,
// a workgroup per run of at most kCopyInts. As one copy command each they took
// 2-4 us of stream time apiece and 5 us of host time: 1,024 of them to admit 512
// calls, 512 to collect them.
__global__ __launch_bounds__(256) void k_upload(const int* __restrict__ host, const CopyEntry* __restrict__ entries,
                                                CopyBases base) {
  const CopyEntry c = entries[blockIdx.x];
  int* dst = (c.to == 0 ? base.p[0] : (c.to == 1 ? base.p[1] : base.p[2])) + c.dst;
  const int* src = host + c.src;
  int v[kCopyInts / 256];
#pragma unroll
  for (int i = 0; i < kCopyInts / 256; ++i) {
    const int k = threadIdx.x + 256 * i;
    v[i] = k < c.n ? src[k] : 0;
  }
#pragma unroll
  for (int i = 0; i < kCopyInts / 256; ++i) {
    const int k = threadIdx.x + 256 * i;
    if (k < c.n) dst[k] = v[i];
  }
}

__global__ __launch_bounds__(256) void k_gather(const int* __restrict__ store, const CopyEntry* __restrict__ entries,
                                                int* __restrict__ host) {
  const CopyEntry c = entries[blockIdx.x];
  for (int k = threadIdx.x; k < c.n; k += 256) host[c.dst + k] = store[c.src + k];
}

// =============================================================== launchers

hipError_t launch_kv_scatter(hipStream_t st, bool bf16, const void* src, void* kv, const int* blocks, int p0, int n,
                             int layer, int kv_sel, int num_blocks, int n_kv, int hd) {
  const size_t total = (size_t)n * n_kv * hd;
  if (total == 0) return hipSuccess;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (bf16)
    klaunch(k_kv_scatter<uint16_t>, grid, dim3(256), st, (const uint16_t*)src, (uint16_t*)kv, blocks, p0, n, layer,
            kv_sel, num_blocks, n_kv, hd);
  else
    klaunch(k_kv_scatter<float>, grid, dim3(256), st, (const float*)src, (float*)kv, blocks, p0, n, layer, kv_sel,
            num_blocks, n_kv, hd);
  return hipGetLastError();
}

hipError_t launch_kv_fill(hipStream_t st, bool bf16, void* kv, const int* bt_store, const FillReq* reqs, int nreqs,
                          int nitems, int n_layers, int num_blocks, int n_kv, int hd) {
  if (nitems <= 0) return hipSuccess;
  if (nreqs < 1 || (hd != 64 && hd != 128) || n_layers > 65535) return hipErrorInvalidValue;
  const dim3 grid(nitems, n_layers), blk(256);
  if (bf16 && hd == 64) klaunch(k_kv_fill<true, 64>, grid, blk, st, kv, bt_store, reqs, nreqs, num_blocks, n_kv);
  else if (bf16) klaunch(k_kv_fill<true, 128>, grid, blk, st, kv, bt_store, reqs, nreqs, num_blocks, n_kv);
  else if (hd == 64) klaunch(k_kv_fill<false, 64>, grid, blk, st, kv, bt_store, reqs, nreqs, num_blocks, n_kv);
  else klaunch(k_kv_fill<false, 128>, grid, blk, st, kv, bt_store, reqs, nreqs, num_blocks, n_kv);
  return hipGetLastError();
}

hipError_t launch_upload(hipStream_t st, const int* host, const CopyEntry* entries, int nentries, CopyBases base) {
  if (nentries <= 0) return hipSuccess;
  klaunch(k_upload, dim3(nentries), dim3(256), st, host, entries, base);
  return hipGetLastError();
}

hipError_t launch_gather(hipStream_t st, const int* store, const CopyEntry* entries, int nentries, int* host) {
  if (nentries <= 0) return hipSuccess;
  klaunch(k_gather, dim3(nentries), dim3(256), st, store, entries, host);
  return hipGetLastError();
}

hipError_t launch_embed(hipStream_t st, bool bf16, const int* tok_store, const int* row_tok,
                        const int* row_model, ModelPtrs embed, float* x, int T, int d) {
  if (T <= 0) return hipSuccess;
  if (bf16) klaunch(k_embed<true>, dim3(T), dim3(256), st, tok_store, row_tok, row_model, embed, x, d);
  else klaunch(k_embed<false>, dim3(T), dim3(256), st, tok_store, row_tok, row_model, embed, x, d);
  return hipGetLastError();
}

hipError_t launch_add_rmsnorm(hipStream_t st, bool bf16, float* x, const float* part, int nsplit,
                              size_t split_stride, const int* gather, const int* row_model, int nrows,
                              ModelPtrs gamma, void* out, size_t out_lo, int d, float eps) {
  if (nrows <= 0) return hipSuccess;
  if (d % 256 || d > 4096) return hipErrorInvalidValue;
  // V4 float4s per thread (d % 256 == 0: whole waves, at most 1024 threads)
  const int v4 = (d % 2048 == 0) ? 2 : 1;
  const int threads = d / (4 * v4);
  auto go = [&](auto kern) {
    klaunch(kern, dim3(nrows), dim3(threads), st, x, part, nsplit, split_stride, gather, row_model, gamma, out,
            out_lo, d, eps);
  };
  if (bf16) {
    if (v4 == 1) go(k_add_rmsnorm<true, 1>);
    else go(k_add_rmsnorm<true, 2>);
  } else {
    if (v4 == 1) go(k_add_rmsnorm<false, 1>);
    else go(k_add_rmsnorm<false, 2>);
  }
  return hipGetLastError();
}

template <int RT, int CT, int NW, int D, int EPI>
static hipError_t gemm_mm(hipStream_t st, const GemmArgs& a) {
  constexpr unsigned shm = 2 * RT * 1024 * (D + 1);
  static bool attr = false;                           // one attribute call per instantiation
  if (!attr) {
    hipError_t e = hipFuncSetAttribute((const void*)k_gemm_mm<RT, CT, NW, D, EPI>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const int nwg = a.total_items;
  klaunch_shm(k_gemm_mm<RT, CT, NW, D, EPI>, dim3((nwg + 7) / 8 * 8), dim3(64 * NW), shm, st, a, nwg);
  return hipGetLastError();
}

template <int CT, int EPI>
static hipError_t gemm_big(hipStream_t st, const GemmArgs& a) {
  const int nwg = a.total_items;
  klaunch(k_gemm_big<CT, EPI>, dim3((nwg + 7) / 8 * 8), dim3(512), st, a, nwg);
  return hipGetLastError();
}

// nt: CT (4 waves), 8 + CT (8 waves), 16 + CT (8 waves, three-stage weight ring)
// or 24 + CT (8 waves, the large-M kernel); see kMmTile
template <int RT, int EPI>
static hipError_t gemm_mm_nt(hipStream_t st, const GemmArgs& a, int nt) {
  if constexpr (RT <= 4)                          // 4 waves x RT = 8 x CT = 4: one wave per SIMD
    if (nt == 4) return gemm_mm<RT, 4, 4, 3, EPI>(st, a);
  if (nt == 2) return gemm_mm<RT, 2, 4, 4, EPI>(st, a);
  if constexpr (RT >= 4) {
    if (nt == 12) return gemm_mm<RT, 4, 8, (RT >= 8 ? 2 : 3), EPI>(st, a);
    if constexpr (RT >= 8) {
      if (nt == 10) return gemm_mm<RT, 2, 8, 3, EPI>(st, a);
      if constexpr (EPI == EPI_SWIGLU) {
        if (nt == 18) return gemm_mm<RT, 2, 8, 3, EPI>(st, a);
        if (nt == 20) return gemm_mm<RT, 4, 8, 3, EPI>(st, a);
      }
      if (nt == 26) return gemm_big<2, EPI>(st, a);
      if (nt == 28) return gemm_big<4, EPI>(st, a);
    }
  }
  return hipErrorInvalidValue;
}

bool gemm_accepts(bool bf16, const GemmArgs& a, int epi, int mt, int nt) {
  if (!bf16) return a.K % 64 == 0 && a.N % 64 == 0;
  if (mt > kMmTile && mt <= kMmTile + 8) {           // 16*RT rows x (16 * NW * CT) columns
    const int rt = mt - kMmTile;
    const bool big = nt == 26 || nt == 28;
    const int ct = nt < 8 ? nt : nt % 8;
    if (rt != 2 && rt != 4 && rt != 8) return false;
    if (nt != 2 && !(nt == 4 && rt <= 4) && !(nt == 12 && rt >= 4) && !(nt == 10 && rt == 8) &&
        !((nt == 18 || nt == 20) && rt == 8 && epi == EPI_SWIGLU) && !(big && rt == 8))
      return false;
    if (a.S < 1 || a.S > (a.K >> 5) || a.N % ((nt < 8 ? 4 : 8) * 16 * ct) != 0) return false;
    for (int g = 0; g < a.ngroups; ++g) {
      if (a.g[g].mrows < 0 || a.g[g].mrows % 16 != 0 || a.g[g].mrows > 16 * rt) return false;
      if (big && a.g[g].nrows > 0 && a.g[g].mrows != 128) return false;
    }
    return true;
  }
  const int m = mt - kWgTile;                        // row tiles of a workgroup
  if ((m != 1 && m != 2 && m != 4) || (nt != 8 && nt != 4 && (nt != 2 || epi != EPI_F32))) return false;
  // whole stages of four k-steps, equal splits
  return a.N % (16 * nt) == 0 && a.S >= 1 && a.ksteps >= 4 && a.ksteps % 4 == 0 && a.ksteps * a.S * 32 == a.K;
}

hipError_t launch_gemm(hipStream_t st, bool bf16, const GemmArgs& a, int epi, int mt, int nt) {
  if (a.total_items <= 0) return hipSuccess;
  if (!gemm_accepts(bf16, a, epi, mt, nt)) return hipErrorInvalidValue;
  if (bf16 && mt > kMmTile && mt <= kMmTile + 8) {
    const int rt = mt - kMmTile;
    if (epi == EPI_SWIGLU) {
      if (rt == 2) return gemm_mm_nt<2, EPI_SWIGLU>(st, a, nt);
      if (rt == 4) return gemm_mm_nt<4, EPI_SWIGLU>(st, a, nt);
      if (rt == 8) return gemm_mm_nt<8, EPI_SWIGLU>(st, a, nt);
    } else {
      if (rt == 2) return gemm_mm_nt<2, EPI_F32>(st, a, nt);
      if (rt == 4) return gemm_mm_nt<4, EPI_F32>(st, a, nt);
      if (rt == 8) return gemm_mm_nt<8, EPI_F32>(st, a, nt);
    }
    return hipErrorInvalidValue;
  }
  if (bf16 && mt >= kWgTile) {
    const int m = mt - kWgTile;
    auto go = [&](auto kern, int nw) {
      klaunch(kern, dim3((a.total_items + 7) / 8 * 8), dim3(64 * nw), st, a, a.total_items);
    };
    auto tile = [&](auto wr, auto ct, auto nw, auto e) {
      constexpr int M = decltype(wr)::value, CT = decltype(ct)::value, NW = decltype(nw)::value, E = decltype(e)::value;
      // two stages of weights ahead where there are few waves with long chains (one
      // 1B model with ffn 6528, whose down has 128 waves of 204 k-steps: 299 us a step
      // at 12 rows, 313 with one stage); more waves want the registers (1B, 16 rows:
      // 254, 251 with one)
      if (a.ksteps >= 12 && a.total_items * NW < 512) go(k_gemm_sm<M, CT, NW, 2, E>, NW);
      else go(k_gemm_sm<M, CT, NW, 1, E>, NW);
    };
    auto rows = [&](auto wr) {
      using One = std::integral_constant<int, 1>;
      using Two = std::integral_constant<int, 2>;
      using Four = std::integral_constant<int, 4>;
      const std::integral_constant<int, EPI_SWIGLU> swiglu;
      const std::integral_constant<int, EPI_F32> f32;
      if (epi == EPI_SWIGLU) {
        if (nt == 8) tile(wr, Two{}, Four{}, swiglu);
        else tile(wr, Two{}, Two{}, swiglu);
      } else {
        if (nt == 8) tile(wr, Two{}, Four{}, f32);
        else if (nt == 4) tile(wr, One{}, Four{}, f32);
        else tile(wr, One{}, Two{}, f32);
      }
    };
    if (m == 1) rows(std::integral_constant<int, 1>{});
    else if (m == 2) rows(std::integral_constant<int, 2>{});
    else rows(std::integral_constant<int, 4>{});
    return hipGetLastError();
  }
  if (!bf16) {
    // four column tiles per workgroup once that fills the chip four times over
    // (it reads each activation row a quarter as often), else one (SwiGLU: two)
    const bool wide = a.total_items >= 1024;
    const dim3 b(256);
    if (epi == EPI_SWIGLU) {
      if (wide) klaunch(k_gemm_f32<4, EPI_SWIGLU>, dim3(a.total_items), b, st, a);
      else klaunch(k_gemm_f32<2, EPI_SWIGLU>, dim3(2 * a.total_items), b, st, a);
    } else {
      if (wide) klaunch(k_gemm_f32<4, EPI_F32>, dim3(a.total_items), b, st, a);
      else klaunch(k_gemm_f32<1, EPI_F32>, dim3(4 * a.total_items), b, st, a);
    }
    return hipGetLastError();
  }
  return hipErrorInvalidValue;                        // no bf16 kernel for this tile code
}

bool row_gemm_shape(const GemmArgs& a, const RowArgs& f, int epi, RowShape& s) {
  if (a.ngroups < 1 || a.S < 1 || a.S > 16 || a.ksteps < 1 || a.S * a.ksteps * 32 != a.K || a.N % 128 != 0) return false;
  if (f.d % 256 != 0 || f.d > 4096) return false;
  int rows = 0;
  for (int g = 0; g < a.ngroups; ++g) {
    if (a.g[g].nrows < 1 || a.g[g].nrows > kRowMax) return false;
    rows = std::max(rows, a.g[g].nrows);
  }
  // the rows and their sums (at most 129 KB), or after them the waves' partial sums
  const unsigned norm = (unsigned)(rows * (f.d + kRowPad) + kRowMax * 16) * 4;
  if (epi == ROW_RES && a.N == f.d) {
    // a column tile per workgroup; few splits are long chains in few waves, which
    // keep 16 k-steps in flight
    s = {1, 1, a.S, (unsigned)a.S * 1024, a.S <= 4 && a.ksteps >= 16 ? 16 : (a.ksteps >= 8 ? 8 : 4)};
  } else if (epi == ROW_SWIGLU && a.K == f.d && a.S == 1) {
    // 128 columns per workgroup, 64 where that leaves CUs idle
    s = {2, a.ngroups * (a.N / 128) >= 224 ? 4 : 2, 8, norm, a.ksteps >= 8 ? 8 : 4};
  } else if (epi == ROW_ROPE && a.K == f.d && a.N == (f.n_h + 2 * f.n_kv) * f.hd && f.hd % 64 == 0) {
    const int cg = a.S >= 4 ? 1 : 4 / a.S;
    s = {2, cg, std::max(8, a.S * cg), std::max(norm, (unsigned)(2 * a.S * cg) * 1024), a.ksteps >= 8 ? 8 : 4};
  } else {
    return false;
  }
  return a.N % (16 * s.ct * s.cg) == 0;
}

hipError_t launch_gemm_row(hipStream_t st, const GemmArgs& a, const RowArgs& f, int epi) {
  if (a.ngroups < 1) return hipSuccess;
  RowShape s;
  if (!row_gemm_shape(a, f, epi, s)) return hipErrorInvalidValue;
  static bool attr = false;                // one attribute call per process for the kernels that hold rows in LDS
  if (!attr) {
    for (const void* k : {(const void*)k_gemm_row<2, 8, ROW_SWIGLU>, (const void*)k_gemm_row<2, 4, ROW_SWIGLU>,
                          (const void*)k_gemm_row<2, 8, ROW_ROPE>, (const void*)k_gemm_row<2, 4, ROW_ROPE>}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 144 * 1024);
      if (e != hipSuccess) return e;
    }
    attr = true;
  }
  const int ncb = a.N / (16 * s.ct * s.cg), nblk = ncb * a.ngroups;
  auto go = [&](auto kern) {
    klaunch_shm(kern, dim3((nblk + 7) / 8 * 8), dim3(64 * s.waves), s.lds, st, a, f, ncb, s.cg);
    return hipGetLastError();
  };
  if (epi == ROW_RES) {
    if (s.depth == 16) return go(k_gemm_row<1, 16, ROW_RES>);
    if (s.depth == 8) return go(k_gemm_row<1, 8, ROW_RES>);
    return go(k_gemm_row<1, 4, ROW_RES>);
  }
  if (epi == ROW_SWIGLU) {
    if (s.depth == 8) return go(k_gemm_row<2, 8, ROW_SWIGLU>);
    return go(k_gemm_row<2, 4, ROW_SWIGLU>);
  }
  if (s.depth == 8) return go(k_gemm_row<2, 8, ROW_ROPE>);
  return go(k_gemm_row<2, 4, ROW_ROPE>);
}

hipError_t launch_rope_kv(hipStream_t st, bool bf16, const float* part, int nsplit, size_t split_stride,
                          const int* row_pos, const int* row_bt, const int* bt_store,
                          const float2* rope_tab, float* q, void* kv, int layer, int num_blocks,
                          int n_h, int n_kv, int hd, int T) {
  if (T <= 0) return hipSuccess;
  const int items = (n_h + n_kv) * (hd / 2) + n_kv * hd;
  const dim3 grid(T, (items + 255) / 256);
  if (bf16)
    klaunch(k_rope_kv<true>, grid, dim3(256), st, part, nsplit, split_stride, row_pos, row_bt, bt_store, rope_tab, q, kv,
                                       layer, num_blocks, n_h, n_kv, hd);
  else
    klaunch(k_rope_kv<false>, grid, dim3(256), st, part, nsplit, split_stride, row_pos, row_bt, bt_store, rope_tab, q, kv,
                                        layer, num_blocks, n_h, n_kv, hd);
  return hipGetLastError();
}

#ifndef ATTN_TK64
#define ATTN_TK64 64
#endif
template <int HD, bool BF, int TK = (HD == 64 && BF) ? ATTN_TK64 : 64>
static hipError_t attn_gq(hipStream_t st, int gq, dim3 grid, unsigned shm, const AttnItem* items, const float* q,
                          const void* kv, const int* bt, const int* row_bt, int layer, int NB, int n_h, int n_kv,
                          float sl2, void* out, size_t out_lo, float* pacc, float* pml) {
  switch (gq) {
    case 1: klaunch_shm(k_attn<HD, 1, BF, TK>, grid, dim3(64), shm, st, items, q, kv, bt, row_bt, layer, NB, n_h, n_kv, sl2, out, out_lo, pacc, pml); break;
    case 2: klaunch_shm(k_attn<HD, 2, BF, TK>, grid, dim3(128), shm, st, items, q, kv, bt, row_bt, layer, NB, n_h, n_kv, sl2, out, out_lo, pacc, pml); break;
    case 4: klaunch_shm(k_attn<HD, 4, BF, TK>, grid, dim3(256), shm, st, items, q, kv, bt, row_bt, layer, NB, n_h, n_kv, sl2, out, out_lo, pacc, pml); break;
    case 8: klaunch_shm(k_attn<HD, 8, BF, TK>, grid, dim3(512), shm, st, items, q, kv, bt, row_bt, layer, NB, n_h, n_kv, sl2, out, out_lo, pacc, pml); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attention(hipStream_t st, bool bf16, const AttnItem* items, int nitems, int max_item_blocks,
                            const float* q, const void* kv, const int* bt_store, const int* row_bt,
                            int layer, int num_blocks, int n_h, int n_kv, int hd, float scale,
                            void* out, size_t out_lo, float* pacc, float* pml) {
  if (nitems <= 0) return hipSuccess;

  const unsigned shm = (unsigned)max_item_blocks * 8u;   // one 64-bit block offset per block of an item
  if (shm > 48u * 1024u) return hipErrorInvalidValue;
  const int gq = n_h / n_kv;
  const float sl2 = scale * 1.4426950408889634f;
  dim3 grid(nitems, n_kv);
  if (hd == 64) {
    return bf16 ? attn_gq<64, true>(st, gq, grid, shm, items, q, kv, bt_store, row_bt, layer, num_blocks, n_h, n_kv, sl2, out, out_lo, pacc, pml)
                : attn_gq<64, false>(st, gq, grid, shm, items, q, kv, bt_store, row_bt, layer, num_blocks, n_h, n_kv, sl2, out, out_lo, pacc, pml);
  }
  if (hd == 128) {
    return bf16 ? attn_gq<128, true>(st, gq, grid, shm, items, q, kv, bt_store, row_bt, layer, num_blocks, n_h, n_kv, sl2, out, out_lo, pacc, pml)
                : attn_gq<128, false>(st, gq, grid, shm, items, q, kv, bt_store, row_bt, layer, num_blocks, n_h, n_kv, sl2, out, out_lo, pacc, pml);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_prefill_attention(hipStream_t st, const PrefillItem* items, int nitems, int max_keys,
                                   const float* q, const void* kv, const int* bt_store, int layer, int num_blocks,
                                   int n_h, int n_kv, int hd, float scale, void* out, size_t out_lo) {
  if (nitems <= 0) return hipSuccess;
  // K ring (3 stages of hd/16 1 KB fragments), V ring (3 tiles of 32 rows of
  // hd values), the block ids of the longest item
  const unsigned shm = 3u * (unsigned)(hd / 16) * 1024u + 3u * 32u * (unsigned)hd * 2u +
                       (unsigned)((max_keys + kBlock - 1) / kBlock) * 4u;
  if (max_keys < 1 || shm > kPrefillLdsMax) return hipErrorInvalidValue;
  const dim3 grid(nitems, n_h), blk(256);
  const float sl2 = scale * 1.4426950408889634f;
  static bool attr = false;                // one attribute call per process for both instantiations
  if (!attr) {
    for (const void* f : {(const void*)k_prefill_attn<64>, (const void*)k_prefill_attn<128>}) {
      hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPrefillLdsMax);
      if (e != hipSuccess) return e;
    }
    attr = true;
  }
  if (hd == 64)
    klaunch_shm(k_prefill_attn<64>, grid, blk, shm, st, items, q, (const uint16_t*)kv, bt_store, layer, num_blocks,
                n_h, n_kv, sl2, (uint16_t*)out, out_lo);
  else if (hd == 128)
    klaunch_shm(k_prefill_attn<128>, grid, blk, shm, st, items, q, (const uint16_t*)kv, bt_store, layer, num_blocks,
                n_h, n_kv, sl2, (uint16_t*)out, out_lo);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_attn_reduce(hipStream_t st, bool bf16, const ReduceItem* red, int nred,
                              const float* pacc, const float* pml, void* out, size_t out_lo, int n_h,
                              int hd) {
  if (nred <= 0) return hipSuccess;
  if (hd < 64 || hd > 256 || 256 % hd || nred > 65535) return hipErrorInvalidValue;
  dim3 grid(n_h, nred);                    // heads fastest: a row's heads start together
  if (bf16) klaunch(k_attn_reduce<true>, grid, dim3(256), st, red, pacc, pml, out, out_lo, n_h, hd);
  else klaunch(k_attn_reduce<false>, grid, dim3(256), st, red, pacc, pml, out, out_lo, n_h, hd);
  return hipGetLastError();
}

hipError_t launch_argmax(hipStream_t st, const float* logits, int R, int V, const int* lm_dst, int* tok_store) {
  if (R <= 0) return hipSuccess;
  if (V % 4) return hipErrorInvalidValue;
  klaunch(k_argmax, dim3(R), dim3(1024), st, logits, V, lm_dst, tok_store);
  return hipGetLastError();
}

}  // namespace moa
