// Learned warm start: U-Net layers and network on gfx950 with BF16 MFMA.
//
// Convolutions are implicit GEMMs on v_mfma_f32_32x32x16_bf16 (forward, and
// the input gradient, which is the forward pass of the flipped, transposed
// filter): the input tile of a block with its halo sits in LDS, weights come
// through LDS (conv_tile_kernel) or, in fragment order, straight into
// registers (conv_direct_kernel).  NHWC with 8 consecutive channels per lane
// makes every operand one 16-byte read.  The weight gradient reduces over
// pixels, which are strided in NHWC: its operands are read with the
// transposing LDS load, the pixel tiles are split over blocks, and the FP32
// partial sums are added in a fixed order.  Images of 2 GB, channel counts
// beyond the LDS and many small images take conv_fwd_kernel or
// conv_fwd32_kernel (operands from memory); every path reduces in the same
// order and gives the same bits.
//
// MFMA 16x16x32 bf16 lane layout (verified on the device): lane l holds
// A[l % 16][8 (l / 16) + v] and B[8 (l / 16) + v][l % 16] for v < 8, and
// D[4 (l / 16) + v][l % 16] for v < 4.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "unet.h"

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

thread_local std::string g_err;

int fail(int code, const std::string& m) {
  g_err = m;
  return code;
}

#define UCHECK(x)                                                              \
  do {                                                                         \
    hipError_t e_ = (x);                                                       \
    if (e_ != hipSuccess)                                                      \
      return fail(UNET_EDEVICE, std::string(#x) + ": " + hipGetErrorString(e_)); \
  } while (0)

inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

// 16-byte loads through a buffer resource: a byte offset at or beyond `bytes`
// reads zeros, so image borders cost one select and no branch.
using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr unsigned kOutside = 0xFFFFFFF0u;   // an offset no image reaches
constexpr long long kMaxRsrc = 0x7FFFFFF0LL;
__device__ __forceinline__ Rsrc image_rsrc(const bf16* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(p), 0, int(bytes), 0x00020000);
}
__device__ __forceinline__ bf16x8 load8(Rsrc r, unsigned off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, int(off), 0, 0));
}
// Bytes from the first channel of an image (pixel stride ld) to the end of
// the last pixel's ch channels.
inline long long image_bytes(int h, int wd, int ld, int ch) {
  return 2 * (((long long)h * wd - 1) * ld + ch);
}

__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Convolution, forward (also the input gradient with transformed weights)
// ---------------------------------------------------------------------------
struct ConvArgs {
  const bf16* x;
  int ldx;
  const bf16* w;       // [cout][9][cin]
  const float* bias;   // [cout] or null
  void* y;
  int ldy;
  int npix, h, wd, cin, cout;
  int relu, out_f32;
  // fused neighbours of the network's convolutions (bf16 output only):
  const bf16* mask;    // ReLU backward: zero the output where mask <= 0, or null
  int ldmask;
  bf16* pool;          // 2x2 mean of the output (h, wd even), or null
  int ldpool;
  int up;              // write each pixel to its four fine pixels (2h x 2wd image)
  unsigned xbytes;     // image_bytes of x (set by launch_conv)
  const bf16* wf;      // w in fragment order (see fragment_kernel), or null
};

__device__ __forceinline__ bf16x8 relu_mask(bf16x8 d, const bf16x8& y) {
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (!((float)y[u] > 0.f)) d[u] = (bf16)0.f;
  return d;
}

// One output value (bias added) of pixel p: ReLU, then FP32, or bf16 masked or
// upsampled.
__device__ __forceinline__ void store_value(const ConvArgs& a, int p, int co, float val) {
  if (a.relu) val = fmaxf(val, 0.f);
  if (a.out_f32) {
    static_cast<float*>(a.y)[(long long)p * a.ldy + co] = val;
    return;
  }
  bf16 o = (bf16)val;
  if (a.mask && !((float)a.mask[(long long)p * a.ldmask + co] > 0.f)) o = (bf16)0.f;
  bf16* out = static_cast<bf16*>(a.y) + co;
  if (!a.up) {
    out[(long long)p * a.ldy] = o;
    return;
  }
  const int x = p % a.wd, q = p / a.wd, y = q % a.h, img = q / a.h;
#pragma unroll
  for (int f = 0; f < 4; ++f)
    out[(((long long)img * 2 * a.h + 2 * y + f / 2) * 2 * a.wd + 2 * x + f % 2) * a.ldy] = o;
}

// WC: waves along the output channels (1 or 2); 4 / WC waves along pixels.
template <int WC>
__global__ __launch_bounds__(256) void conv_fwd_kernel(ConvArgs a) {
  constexpr int WP = 4 / WC;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int px0 = blockIdx.x * (32 * WP) + 32 * (wv % WP);
  const int co0 = blockIdx.y * (32 * WC) + 32 * (wv / WP);
  const int r = lane & 15, g = lane >> 4;
  int pidx[2], py[2], pxx[2];
  bool pv[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int p = px0 + 16 * s + r;
    pv[s] = p < a.npix;
    const int q = pv[s] ? p : 0;
    pidx[s] = q;
    pxx[s] = q % a.wd;
    py[s] = (q / a.wd) % a.h;
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[s][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t = 0; t < 9; ++t) {
    const int dy = t / 3 - 1, dx = t % 3 - 1;
    const bf16* xa[2];
    bool ok[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int yy = py[s] + dy, xx = pxx[s] + dx;
      ok[s] = pv[s] && yy >= 0 && yy < a.h && xx >= 0 && xx < a.wd;
      xa[s] = a.x + (long long)(ok[s] ? pidx[s] + dy * a.wd + dx : 0) * a.ldx + 8 * g;
    }
    const bf16* wb[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
      wb[b] = a.w + ((long long)(co0 + 16 * b + r) * 9 + t) * a.cin + 8 * g;
    for (int c0 = 0; c0 < a.cin; c0 += 32) {
      bf16x8 A[2], B[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        A[s] = *reinterpret_cast<const bf16x8*>(xa[s] + c0);
        if (!ok[s]) A[s] = bf16x8{};
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) B[b] = *reinterpret_cast<const bf16x8*>(wb[b] + c0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[s][b] = mfma16(A[s], B[b], acc[s][b]);
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int co = co0 + 16 * b + r;
      const float bias = a.bias ? a.bias[co] : 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int p = px0 + 16 * s + 4 * g + v;
        if (p < a.npix) store_value(a, p, co, acc[s][b][v] + bias);
      }
    }
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same on v_mfma_f32_32x32x16_bf16 (layout at the tiled convolution below):
// a wave owns 64 pixels x 32 CT output channels and does twice the work per
// loaded byte, so it needs that many pixels to fill the device (704 -> 64
// channels at 16 x 64 x 64: 353 us with the tiles above, 209 with these).
template <int CT>
__global__ __launch_bounds__(256) void conv_fwd32_kernel(ConvArgs a) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int px0 = blockIdx.x * 256 + 64 * wv;
  const int co0 = blockIdx.y * (32 * CT);
  const int r = lane & 31, g = lane >> 5;
  int pidx[2], py[2], pxx[2];
  bool pv[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int p = px0 + 32 * s + r;
    pv[s] = p < a.npix;
    const int q = pv[s] ? p : 0;
    pidx[s] = q;
    pxx[s] = q % a.wd;
    py[s] = (q / a.wd) % a.h;
  }
  f32x16 acc[2][CT];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[s][b][v] = 0.f;
  for (int t = 0; t < 9; ++t) {
    const int dy = t / 3 - 1, dx = t % 3 - 1;
    const bf16* xa[2];
    bool ok[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int yy = py[s] + dy, xx = pxx[s] + dx;
      ok[s] = pv[s] && yy >= 0 && yy < a.h && xx >= 0 && xx < a.wd;
      xa[s] = a.x + (long long)(ok[s] ? pidx[s] + dy * a.wd + dx : 0) * a.ldx + 8 * g;
    }
    const bf16* wb[CT];
#pragma unroll
    for (int b = 0; b < CT; ++b)
      wb[b] = a.w + ((long long)(co0 + 32 * b + r) * 9 + t) * a.cin + 8 * g;
    for (int c0 = 0; c0 < a.cin; c0 += 16) {
      bf16x8 A[2], B[CT];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        A[s] = *reinterpret_cast<const bf16x8*>(xa[s] + c0);
        if (!ok[s]) A[s] = bf16x8{};
      }
#pragma unroll
      for (int b = 0; b < CT; ++b) B[b] = *reinterpret_cast<const bf16x8*>(wb[b] + c0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int b = 0; b < CT; ++b) acc[s][b] = mfma32(A[s], B[b], acc[s][b]);
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int b = 0; b < CT; ++b) {
      const int co = co0 + 32 * b + r;
      const float bias = a.bias ? a.bias[co] : 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int p = px0 + 32 * s + 8 * (v / 4) + 4 * g + (v % 4);
        if (p < a.npix) store_value(a, p, co, acc[s][b][v] + bias);
      }
    }
}

// Tiled convolution: a block owns a TX x TY pixel tile (P = 32 MP WP pixels)
// and 32 NC WC output channels.  The input tile with its one-pixel ring is
// staged once in LDS with all input channels (zeros outside the image, so
// the taps need no masks), the weights stream through two LDS buffers of KS
// reduction elements each (the next stage's global loads are in flight while
// the current one is multiplied), and every MFMA operand is one 16-byte LDS
// read.  Rows are padded by 16 bytes: 16 lanes that read 16 bytes at that
// stride (an odd multiple of 16 bytes) touch every bank once.
// v_mfma_f32_32x32x16_bf16: lane l holds A[l % 32][8 (l / 32) + v],
// B[8 (l / 32) + v][l % 32] for v < 8 and D[8 (v / 4) + 4 (l / 32) + v % 4]
// [l % 32] for v < 16.  Weights are the A operand and pixels the B operand,
// so a lane ends with groups of four consecutive channels of one pixel; the
// block writes them to LDS and from there out in 16-byte pieces.  The
// reduction runs tap by tap and channel by channel in one accumulator, the
// order of conv_fwd_kernel (a 32x32x16 chain gives the same bits as a
// 16x16x32 one, checked on the device), so the path taken never shows in
// the result.  Measured at batch 16, 128 x 128 and its halvings: 32 -> 32
// channels 12 us (390 TFLOP/s), 192 -> 64 22 us (650), 384 -> 128 26 us
// (560); before, with operands straight from memory, 35, 105 and 105 us.
// What is left is latency in series (launch, tile load, per stage LDS reads
// and a barrier, store), no single unit: leaving out any one of MFMA, LDS
// reads, tile load, weight loads or stores saves 5-20 %.
constexpr int kLdsBytes = 160 * 1024;
constexpr int kConv32MinPix = 65536;   // pixels from which conv_fwd32_kernel is faster

// A stage is KS channels of one tap (KS = 96, 64 or 32, the largest that
// divides cin) or, for cin = 32 (ROW), the three taps of a kernel row, so
// every LDS offset within a stage is a constant.
template <int MP, int NC, int WP, int WC, int TX, int KS>
struct ConvTile {
  static constexpr int P = 32 * MP * WP, CB = 32 * NC * WC, TY = P / TX;
  static constexpr int WS = 2 * KS + 16;   // LDS bytes per weight row
  static constexpr int OS = 2 * CB + 16;   // LDS bytes per output pixel
  static constexpr int NT = 64 * WP * WC;  // threads
  static_assert(TY * TX == P && KS % 32 == 0, "tile");
  static size_t lds(int cin) {
    const size_t in = (size_t)(TX + 2) * (TY + 2) * (2 * cin + 16) + 2 * (size_t)CB * WS;
    return 4 * CB + (in > (size_t)P * OS ? in : (size_t)P * OS);   // bias, then the tiles
  }
  static size_t lds_direct(int cin) {
    const size_t in = (size_t)(TX + 2) * (TY + 2) * (2 * cin + 16);
    return 4 * CB + (in > (size_t)P * OS ? in : (size_t)P * OS);
  }
};

// Input tile of a block: HP pixels x cin channels into LDS (S bytes per
// pixel), eight 16-byte loads in flight per thread.
template <int NT, int HX, int HP>
__device__ __forceinline__ void load_tile(const ConvArgs& a, int img, int x0, int y0, int S,
                                          char* sx) {
  const int tid = threadIdx.x;
  const int cv = a.cin >> 3, nvec = HP * cv;
  const Rsrc xr = image_rsrc(a.x + (long long)img * a.h * a.wd * a.ldx, a.xbytes);
  const int qs = NT / cv, rs = NT - qs * cv;
  int px = tid / cv, c = tid - px * cv;
  for (int base = 0; base < nvec; base += 8 * NT) {
    bf16x8 v[8];
    int at[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (base + NT * u < nvec) {
        const int yy = px / HX, xx = px - yy * HX;
        const int y = y0 + yy - 1, x = x0 + xx - 1;
        const bool in = unsigned(y) < unsigned(a.h) && unsigned(x) < unsigned(a.wd);
        v[u] = load8(xr, in ? unsigned((y * a.wd + x) * a.ldx + 8 * c) * 2u : kOutside);
        at[u] = px * S + 16 * c;
        px += qs;
        c += rs;
        const bool wrap = c >= cv;
        px += wrap ? 1 : 0;
        c -= wrap ? cv : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (base + NT * u + tid < nvec) *reinterpret_cast<bf16x8*>(sx + at[u]) = v[u];
  }
}

// Results of a block: bias and ReLU, then FP32 from the registers or bf16
// through LDS (free by then), masked, pooled or upsampled.
template <int MP, int NC, int WP, int WC, int TX, int KS>
__device__ __forceinline__ void store_tile(const ConvArgs& a, const f32x16 (&acc)[NC][MP], int img,
                                           int x0, int y0, int co0, const float* sbias,
                                           char* smem) {
  using L = ConvTile<MP, NC, WP, WC, TX, KS>;
  constexpr int NT = L::NT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wv % WP, wc = wv / WP;
  const int r = lane & 31, g = lane >> 5;
  if (a.out_f32) {
#pragma unroll
    for (int b = 0; b < NC; ++b)
#pragma unroll
      for (int s = 0; s < MP; ++s) {
        const int q = 32 * (wp * MP + s) + r;
        const int y = y0 + q / TX, x = x0 + q % TX;
        if (y >= a.h || x >= a.wd) continue;
        float* o = static_cast<float*>(a.y) +
                   ((long long)(img * a.h + y) * a.wd + x) * a.ldy + co0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int co = 32 * (NC * wc + b) + 8 * v + 4 * g;
          f32x4 val;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            val[i] = acc[b][s][4 * v + i] + sbias[co + i];
            if (a.relu) val[i] = fmaxf(val[i], 0.f);
          }
          *reinterpret_cast<f32x4*>(o + co) = val;
        }
      }
    return;
  }
  // bf16: through LDS (the staging areas are free after the last barrier)
#pragma unroll
  for (int b = 0; b < NC; ++b)
#pragma unroll
    for (int s = 0; s < MP; ++s) {
      const int q = 32 * (wp * MP + s) + r;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int co = 32 * (NC * wc + b) + 8 * v + 4 * g;
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float val = acc[b][s][4 * v + i] + sbias[co + i];
          if (a.relu) val = fmaxf(val, 0.f);
          o[i] = (bf16)val;
        }
        *reinterpret_cast<bf16x4*>(smem + q * L::OS + 2 * co) = o;
      }
    }
  __syncthreads();
  constexpr int kOVec = L::CB / 8;
#pragma unroll
  for (int i = 0; i < L::P * kOVec / NT; ++i) {
    const int v = tid + NT * i, q = v / kOVec, c = v % kOVec;
    const int y = y0 + q / TX, x = x0 + q % TX;
    if (y >= a.h || x >= a.wd) continue;
    bf16x8 o = *reinterpret_cast<const bf16x8*>(smem + q * L::OS + 16 * c);
    const long long p = (long long)(img * a.h + y) * a.wd + x;
    if (a.mask)
      o = relu_mask(o, *reinterpret_cast<const bf16x8*>(a.mask + p * a.ldmask + co0 + 8 * c));
    bf16* out = static_cast<bf16*>(a.y) + co0 + 8 * c;
    if (!a.up) {
      *reinterpret_cast<bf16x8*>(out + p * a.ldy) = o;
    } else {
#pragma unroll
      for (int f = 0; f < 4; ++f)
        *reinterpret_cast<bf16x8*>(
            out + ((long long)(img * 2 * a.h + 2 * y + f / 2) * 2 * a.wd + 2 * x + f % 2) * a.ldy) =
            o;
    }
  }
  if (a.pool) {
    // tiles start at even coordinates and h, wd are even: whole 2 x 2 cells
    for (int v = tid; v < L::P / 4 * kOVec; v += NT) {
      const int q = v / kOVec, c = v % kOVec;
      const int yy = 2 * (q / (TX / 2)), xx = 2 * (q % (TX / 2));
      if (y0 + yy >= a.h || x0 + xx >= a.wd) continue;
      float m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const bf16x8 e = *reinterpret_cast<const bf16x8*>(
            smem + ((yy + f / 2) * TX + xx + f % 2) * L::OS + 16 * c);
#pragma unroll
        for (int u = 0; u < 8; ++u) m[u] += (float)e[u];
      }
      bf16x8 o;
#pragma unroll
      for (int u = 0; u < 8; ++u) o[u] = (bf16)(0.25f * m[u]);
      const long long p =
          ((long long)img * (a.h / 2) + (y0 + yy) / 2) * (a.wd / 2) + (x0 + xx) / 2;
      *reinterpret_cast<bf16x8*>(a.pool + p * a.ldpool + co0 + 8 * c) = o;
    }
  }
}

template <int MP, int NC, int WP, int WC, int TX, int KS, bool ROW>
__global__ __launch_bounds__(64 * WP * WC) void conv_tile_kernel(ConvArgs a, int tiles_x, int tiles_y) {
  using L = ConvTile<MP, NC, WP, WC, TX, KS>;
  constexpr int TY = L::TY, HX = TX + 2, HP = (TX + 2) * (TY + 2), NT = L::NT;
  extern __shared__ __align__(16) char smem_all[];
  float* sbias = reinterpret_cast<float*>(smem_all);
  char* smem = smem_all + 4 * L::CB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wv % WP, wc = wv / WP;
  const int r = lane & 31, g = lane >> 5;
  int tile = blockIdx.x;
  const int tx = tile % tiles_x;
  tile /= tiles_x;
  const int ty = tile % tiles_y, img = tile / tiles_y;
  const int x0 = tx * TX, y0 = ty * TY, co0 = blockIdx.y * L::CB;
  const int S = 2 * a.cin + 16;
  char* sx = smem;
  char* sw = smem + HP * S;
  const int nst = 9 * a.cin / KS;

  // weights of one stage: CB rows of KS consecutive reduction elements
  constexpr int kRowVec = KS / 8, kWVec = L::CB * kRowVec, kWPer = (kWVec + NT - 1) / NT;
  // PF stages in flight in registers (the loads are unconditional: under a
  // branch, the wait for one stage would become a wait for all of them)
  constexpr int PF = 3;   // divides the number of stages
  bf16x8 wreg[PF][kWPer];
  unsigned woff[kWPer];
#pragma unroll
  for (int i = 0; i < kWPer; ++i) {
    const int v = tid + NT * i, row = kWVec % NT == 0 || v < kWVec ? v / kRowVec : 0;
    woff[i] = unsigned(row * 9 * a.cin + 8 * (v % kRowVec)) * 2u;
  }
  const char* wbase = reinterpret_cast<const char*>(a.w + (long long)co0 * 9 * a.cin);
  auto load_w = [&](int st, bf16x8 (&w)[kWPer]) {
    const char* p = wbase + (long long)min(st, nst - 1) * (2 * KS);
#pragma unroll
    for (int i = 0; i < kWPer; ++i) w[i] = *reinterpret_cast<const bf16x8*>(p + woff[i]);
  };
  auto store_w = [&](int buf, const bf16x8 (&w)[kWPer]) {
#pragma unroll
    for (int i = 0; i < kWPer; ++i) {
      const int v = tid + NT * i;
      if (kWVec % NT == 0 || v < kWVec)
        *reinterpret_cast<bf16x8*>(sw + buf * (L::CB * L::WS) + (v / kRowVec) * L::WS +
                                   16 * (v % kRowVec)) = w[i];
    }
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) load_w(i, wreg[i]);
  if (tid < L::CB) sbias[tid] = a.bias ? a.bias[co0 + tid] : 0.f;
  load_tile<NT, HX, HP>(a, img, x0, y0, S, sx);
  store_w(0, wreg[0]);
  load_w(PF, wreg[0]);
  __syncthreads();

  f32x16 acc[NC][MP];
#pragma unroll
  for (int b = 0; b < NC; ++b)
#pragma unroll
    for (int s = 0; s < MP; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][s][v] = 0.f;
  const char* xb[MP];
#pragma unroll
  for (int s = 0; s < MP; ++s) {
    const int q = 32 * (wp * MP + s) + r;
    xb[s] = sx + ((q / TX) * HX + q % TX) * S + 16 * g;
  }
  const int wrow = (32 * NC * wc + r) * L::WS + 16 * g;
  // stage position: byte offset of its tap (or kernel row) and channels
  int soff = 0, chunk = 0, tcol = 0;
  const int chunks = a.cin / KS;
  for (int st0 = 0; st0 < nst; st0 += PF) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int st = st0 + i;
      const char* wb = sw + (st & 1) * (L::CB * L::WS) + wrow;
      // operands of the next 32 elements are read while the current ones are
      // multiplied (the scheduling barriers keep the compiler from sinking each
      // read to just before its use, one LDS latency per MFMA)
      constexpr int NJ = KS / 32;
      bf16x8 A[2][2][NC], B[2][2][MP];
      const char* xs[MP];
#pragma unroll
      for (int s = 0; s < MP; ++s) xs[s] = xb[s] + soff;
      auto read = [&](int j, bf16x8 (&Aj)[2][NC], bf16x8 (&Bj)[2][MP]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int s = 0; s < MP; ++s)
            Bj[h][s] = *reinterpret_cast<const bf16x8*>(xs[s] + (ROW ? 80 : 64) * j + 32 * h);
#pragma unroll
          for (int b = 0; b < NC; ++b)
            Aj[h][b] = *reinterpret_cast<const bf16x8*>(wb + b * (32 * L::WS) + 64 * j + 32 * h);
        }
      };
      read(0, A[0], B[0]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j + 1 < NJ) read(j + 1, A[(j + 1) & 1], B[(j + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int b = 0; b < NC; ++b)
#pragma unroll
            for (int s = 0; s < MP; ++s)
              acc[b][s] = mfma32(A[j & 1][h][b], B[j & 1][h][s], acc[b][s]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (ROW) {
        soff += HX * 80;
      } else {   // uniform: the next channels, or the next tap
        ++chunk;
        const bool next = chunk == chunks;
        const int tap = tcol == 2 ? (TX + 1) * S - S : S;   // one to the right, or the next row
        soff += next ? tap - 2 * KS * (chunks - 1) : 2 * KS;
        tcol = next ? (tcol == 2 ? 0 : tcol + 1) : tcol;
        chunk = next ? 0 : chunk;
      }
      if (st + 1 < nst) store_w((st + 1) & 1, wreg[(i + 1) % PF]);
      load_w(st + 1 + PF, wreg[(i + 1) % PF]);
      __syncthreads();
    }
  }

  store_tile<MP, NC, WP, WC, TX, KS>(a, acc, img, x0, y0, co0, sbias, smem);
}

// The same with weights in fragment order (ConvArgs::wf) straight from memory
// into registers, PF stages of KS channels ahead: no barrier and no LDS round
// trip between the stages, so a wavefront runs at its own pace.  Bound by the
// chain of MFMAs of a wavefront and the latency of its start and end where a
// layer has one tile per SIMD (256 -> 256 channels at 16 x 16 x 16: 15.0 ->
// 9.7 us, 128 -> 256 8.9 -> 6.8), by LDS reads and the same latencies beyond
// (384 -> 128 at 16 x 32 x 32: 25.6 -> 21.2, 128 -> 384 26.5 -> 21.4).
// Fragments read from rows of 9 cin weights (32 lines per load) cost the
// address unit 80 clocks each, twice the time of the LDS stages.
template <int MP, int NC, int WP, int WC, int TX, int KS>
__global__ __launch_bounds__(64 * WP * WC) void conv_direct_kernel(ConvArgs a, int tiles_x, int tiles_y) {
  using L = ConvTile<MP, NC, WP, WC, TX, KS>;
  constexpr int TY = L::TY, HX = TX + 2, HP = (TX + 2) * (TY + 2), NT = L::NT;
  extern __shared__ __align__(16) char smem_all[];
  float* sbias = reinterpret_cast<float*>(smem_all);
  char* smem = smem_all + 4 * L::CB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wv % WP, wc = wv / WP;
  const int r = lane & 31, g = lane >> 5;
  int tile = blockIdx.x;
  const int tx = tile % tiles_x;
  tile /= tiles_x;
  const int ty = tile % tiles_y, img = tile / tiles_y;
  const int x0 = tx * TX, y0 = ty * TY, co0 = blockIdx.y * L::CB;
  const int S = 2 * a.cin + 16;
  char* sx = smem;
  const int nst = 9 * a.cin / KS;
  constexpr int PF = 3, NK = KS / 16;   // PF divides the number of stages
  bf16x8 wreg[PF][NK][NC];
  const char* wbase = reinterpret_cast<const char*>(a.wf + (long long)co0 * 9 * a.cin);
  unsigned woff[NC];
#pragma unroll
  for (int b = 0; b < NC; ++b)
    woff[b] = unsigned((NC * wc + b) * (32 * 9 * a.cin) + 8 * lane) * 2u;
  auto load_w = [&](int st, bf16x8 (&w)[NK][NC]) {
    const char* p = wbase + (long long)min(st, nst - 1) * (64 * KS);
#pragma unroll
    for (int j = 0; j < NK; ++j)
#pragma unroll
      for (int b = 0; b < NC; ++b)
        w[j][b] = *reinterpret_cast<const bf16x8*>(p + woff[b] + 1024 * j);
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) load_w(i, wreg[i]);
  if (tid < L::CB) sbias[tid] = a.bias ? a.bias[co0 + tid] : 0.f;
  load_tile<NT, HX, HP>(a, img, x0, y0, S, sx);
  __syncthreads();

  f32x16 acc[NC][MP];
#pragma unroll
  for (int b = 0; b < NC; ++b)
#pragma unroll
    for (int s = 0; s < MP; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][s][v] = 0.f;
  const char* xb[MP];
#pragma unroll
  for (int s = 0; s < MP; ++s) {
    const int q = 32 * (wp * MP + s) + r;
    xb[s] = sx + ((q / TX) * HX + q % TX) * S + 16 * g;
  }
  int soff = 0, chunk = 0, tcol = 0;
  const int chunks = a.cin / KS;
  constexpr int NJ = KS / 32;
  static_assert(NJ % 2 == 0, "the next stage's first operands go to buffer 0");
  bf16x8 B[2][2][MP];
  auto read = [&](int off, bf16x8 (&Bj)[2][MP]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < MP; ++s)
        Bj[h][s] = *reinterpret_cast<const bf16x8*>(xb[s] + off + 32 * h);
  };
  read(0, B[0]);
  for (int st0 = 0; st0 < nst; st0 += PF) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      // uniform: the next channels, or the next tap
      const int here = soff;
      ++chunk;
      const bool next = chunk == chunks;
      const int tap = tcol == 2 ? (TX + 1) * S - S : S;
      soff += next ? tap - 2 * KS * (chunks - 1) : 2 * KS;
      tcol = next ? (tcol == 2 ? 0 : tcol + 1) : tcol;
      chunk = next ? 0 : chunk;
      if (st0 + i + 1 == nst) soff = here;   // (nothing follows)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        read(j + 1 < NJ ? here + 64 * (j + 1) : soff, B[(j + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int b = 0; b < NC; ++b)
#pragma unroll
            for (int s = 0; s < MP; ++s)
              acc[b][s] = mfma32(wreg[i][2 * j + h][b], B[j & 1][h][s], acc[b][s]);
        __builtin_amdgcn_sched_barrier(0);
      }
      load_w(st0 + i + PF, wreg[i]);
    }
  }
  __syncthreads();
  store_tile<MP, NC, WP, WC, TX, KS>(a, acc, img, x0, y0, co0, sbias, smem);
}

// Whether tiles of P pixels cost more than the kernels without tiles: every image
// has tiles of its own, so many small images are mostly padding.  Up to three
// blocks per compute unit that does not matter.  Beyond, the tiles win up to a
// ratio of covered to image pixels of 4 to 5; of 3 against conv_fwd32_kernel, or
// with input channels that leave room for one block per compute unit; less with
// the largest channel counts, and with few input for many output channels, where
// the stores bound both.  The next smaller tile is tried first.  Without
// tiles | with, 64 -> 64 channels: 4096 images of 4 x 4 27.8 | 83.4 us, 1024 of them
// 12.9 | 11.5; 4062 of 8 x 8 96.5 | 85.4; 128 -> 128: 4096 of 1 x 1 16.3 | 121.
bool tiles_padded(const ConvArgs& a, long long tiles, int P, int channel_blocks) {
  const long long n = a.npix / (a.h * a.wd);
  if (tiles * n * channel_blocks <= 768) return false;
  const bool big = a.npix >= kConv32MinPix;
  double most = a.cout % 64 == 0 ? 5.2 : 4.0;
  if (a.cin == 32 && a.cout >= 128) most = 1.99;
  else if (big && a.cin >= 256 && a.cout >= 256) most = 2.2;
  else if (big || a.cin >= 256) most = a.cout >= 128 ? 3.0 : 3.2;
  return (double)tiles * P > most * a.h * a.wd;
}

// Launches a tiling if its LDS fits and its tiles are filled (*done); otherwise
// leaves *done false.
template <int MP, int NC, int WP, int WC, int TX, int KS, bool ROW>
int try_conv_tile(const ConvArgs& a, hipStream_t st, bool* done) {
  using L = ConvTile<MP, NC, WP, WC, TX, KS>;
  const int tx = (a.wd + TX - 1) / TX, ty = (a.h + L::TY - 1) / L::TY;
  const size_t lds = L::lds(a.cin);
  if (lds > (size_t)kLdsBytes || tiles_padded(a, (long long)tx * ty, L::P, a.cout / L::CB))
    return UNET_OK;
  auto* fn = conv_tile_kernel<MP, NC, WP, WC, TX, KS, ROW>;
  if (lds > 64 * 1024)
    UCHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  dim3 grid(tx * ty * (a.npix / (a.h * a.wd)), a.cout / L::CB);
  hipLaunchKernelGGL(fn, grid, dim3(L::NT), lds, st, a, tx, ty);
  UCHECK(hipGetLastError());
  *done = true;
  return UNET_OK;
}

template <int MP, int NC, int WP, int WC, int TX>
int try_conv_width(const ConvArgs& a, hipStream_t st, bool* done) {
  if (a.cin == 32) return try_conv_tile<MP, NC, WP, WC, TX, 96, true>(a, st, done);
  if (a.cin % 96 == 0) return try_conv_tile<MP, NC, WP, WC, TX, 96, false>(a, st, done);
  if (a.cin % 64 == 0) return try_conv_tile<MP, NC, WP, WC, TX, 64, false>(a, st, done);
  return try_conv_tile<MP, NC, WP, WC, TX, 32, false>(a, st, done);
}

template <int MP, int NC, int WP, int WC>
int try_conv(const ConvArgs& a, hipStream_t st, bool* done) {
  // 16-pixel-wide tiles where 32 would pad the rows more, or where they let
  // two blocks share a compute unit's LDS (by the largest stage): 96 -> 32
  // channels at 16 x 128 x 128, 38 -> 29 us
  const size_t half = kLdsBytes / 2;
  constexpr int KS = 96;
  const bool narrow = (a.wd + 15) / 16 * 16 < (a.wd + 31) / 32 * 32 ||
                      (ConvTile<MP, NC, WP, WC, 32, KS>::lds(a.cin) > half &&
                       ConvTile<MP, NC, WP, WC, 16, KS>::lds(a.cin) <= half);
  int rc = UNET_OK;
  if (!narrow) rc = try_conv_width<MP, NC, WP, WC, 32>(a, st, done);
  // (or where only they fit: 640 -> 64 at 16 x 64 x 64, 321 -> 133 us)
  if (!rc && !*done) rc = try_conv_width<MP, NC, WP, WC, 16>(a, st, done);
  return rc;
}

template <int MP, int NC, int WP, int WC, int TX>
int try_direct_width(const ConvArgs& a, hipStream_t st, bool* done) {
  using L = ConvTile<MP, NC, WP, WC, TX, 64>;
  if (a.cin % 64 || a.cout % L::CB) return UNET_OK;
  const int tx = (a.wd + TX - 1) / TX, ty = (a.h + L::TY - 1) / L::TY;
  const size_t lds = L::lds_direct(a.cin);
  if (lds > (size_t)kLdsBytes || tiles_padded(a, (long long)tx * ty, L::P, a.cout / L::CB))
    return UNET_OK;
  auto* fn = conv_direct_kernel<MP, NC, WP, WC, TX, 64>;
  if (lds > 64 * 1024)
    UCHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  dim3 grid(tx * ty * (a.npix / (a.h * a.wd)), a.cout / L::CB);
  hipLaunchKernelGGL(fn, grid, dim3(L::NT), lds, st, a, tx, ty);
  UCHECK(hipGetLastError());
  *done = true;
  return UNET_OK;
}

template <int MP, int NC, int WP, int WC>
int try_direct(const ConvArgs& a, hipStream_t st, bool* done) {
  const bool narrow = (a.wd + 15) / 16 * 16 < (a.wd + 31) / 32 * 32;
  return narrow ? try_direct_width<MP, NC, WP, WC, 16>(a, st, done)
                : try_direct_width<MP, NC, WP, WC, 32>(a, st, done);
}

__global__ void pool2_fwd_kernel(const bf16* x, int ldx, bf16* y, int ldy, int n, int h, int wd,
                                 int cv);
int grid_for(long long total);

int launch_conv(ConvArgs a, hipStream_t st) {
  if (a.cin <= 0 || a.cout <= 0 || a.cin % 32 || a.cout % 32)
    return fail(UNET_EINVAL, "conv: cin and cout must be positive multiples of 32");
  if (a.ldx % 8 || a.ldy % 8 || a.ldx < a.cin || a.ldy < a.cout)
    return fail(UNET_EINVAL, "conv: ld must be a multiple of 8 and cover the channels");
  if (a.npix <= 0 || a.h <= 0 || a.wd <= 0 || a.npix % (a.h * a.wd))
    return fail(UNET_EINVAL, "conv: bad image size");
  if (!a.x || !a.w || !a.y) return fail(UNET_EINVAL, "conv: null pointer");
  const long long xbytes = image_bytes(a.h, a.wd, a.ldx, a.cin);
  a.xbytes = (unsigned)xbytes;
  // The largest block tile that still gives about 256 blocks (one per compute
  // unit); eight waves of 32 x 32 or 64 x 32 hide each other's LDS and memory
  // latency better than four larger ones (128 -> 128 channels at 16 x 32 x
  // 32: 10.7 us against 12.7; 64 -> 64 at 16 x 64 x 64: 10.2 against 12.0).
  // The 64 x 128 tile also where it leaves some units idle: four waves of a
  // 64 x 64 tile then run two rounds, and with many input channels each alone
  // on its unit (384 -> 128 channels at 12 x 32 x 32: 31.7 us against 23.0).
  // An image of 2 GB takes the general path.
  const long long px32 = (a.npix + 31) / 32;
  bool done = xbytes > kMaxRsrc;
  int rc = UNET_OK;
  // Weights in fragment order (the network's layers): one 32 x 32 tile per
  // wavefront up to one wavefront per SIMD, else two.  Times of the LDS-staged
  // tiles below and of these: at conv_direct_kernel; 192 -> 64 channels at 9 x
  // 64 x 64 21.7 | 17.1 us, 128 -> 128 at 3 x 32 x 32 8.5 | 6.6.
  if (!done && a.wf) {
    if (px32 * (a.cout / 32) > 1024) rc = try_direct<2, 1, 2, 2>(a, st, &done);
    if (!rc && !done) rc = try_direct<1, 1, 2, 2>(a, st, &done);
    if (rc || done) return rc;
  }
  if (!done) {
    if (a.cout % 64 == 0 && px32 * (a.cout / 64) >= 2048) rc = try_conv<2, 1, 4, 2>(a, st, &done);
    if (!rc && !done && a.cout % 128 == 0 && px32 * (a.cout / 64) > 512)
      rc = try_conv<1, 1, 2, 4>(a, st, &done);
    if (!rc && !done && a.cout % 64 == 0) rc = try_conv<1, 1, 2, 2>(a, st, &done);
    if (!rc && !done && px32 * (a.cout / 32) >= 2048) rc = try_conv<1, 1, 8, 1>(a, st, &done);
    if (!rc && !done) rc = try_conv<1, 1, 4, 1>(a, st, &done);
    if (rc || done) return rc;
  }
  // an image of 2 GB, more input channels than LDS holds (none of the network's
  // layers), or many small images: operands straight from memory
  // (32 output channels of many input channels: 544 -> 32 at 16 x 64 x 64 99 us with
  // the small tiles, 127 with the large)
  if (a.npix >= kConv32MinPix && (a.cout % 64 == 0 || a.cin < 448)) {
    const int ct = a.cout % 64 == 0 ? 2 : 1;
    dim3 grid((a.npix + 255) / 256, a.cout / (32 * ct));
    if (ct == 2)
      hipLaunchKernelGGL(conv_fwd32_kernel<2>, grid, dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL(conv_fwd32_kernel<1>, grid, dim3(256), 0, st, a);
  } else if (a.cout % 64 == 0) {
    dim3 grid((a.npix + 63) / 64, a.cout / 64);
    hipLaunchKernelGGL(conv_fwd_kernel<2>, grid, dim3(256), 0, st, a);
  } else {
    dim3 grid((a.npix + 127) / 128, a.cout / 32);
    hipLaunchKernelGGL(conv_fwd_kernel<1>, grid, dim3(256), 0, st, a);
  }
  UCHECK(hipGetLastError());
  if (a.pool) {
    const int n = a.npix / (a.h * a.wd);
    hipLaunchKernelGGL(pool2_fwd_kernel, dim3(grid_for((long long)a.npix / 4 * (a.cout / 8))),
                       dim3(256), 0, st, static_cast<const bf16*>(a.y), a.ldy, a.pool, a.ldpool, n,
                       a.h, a.wd, a.cout / 8);
    UCHECK(hipGetLastError());
  }
  return UNET_OK;
}

// Flipped, transposed weights of one or more layers: wt[ci][t][co] =
// w[co][8 - t][ci], both at offset `off` of their arrays.  A block moves one
// 32 x 32 channel tile of one tap through LDS, so reads and writes are rows
// of 64 bytes (element by element, one thread per output, the strided reads
// took 4.8 us per layer).
constexpr int kMaxFlip = 16;
struct FlipArgs {
  const bf16* w;
  bf16* wt;
  int layers;
  struct {
    long long off;
    int cin, cout, first;   // first: index of the layer's first tile
  } l[kMaxFlip];
};

__global__ __launch_bounds__(256) void flip_tiles_kernel(FlipArgs a) {
  __shared__ bf16 s[32][34];
  int k = 0;
  while (k + 1 < a.layers && int(blockIdx.x) >= a.l[k + 1].first) ++k;
  const int cin = a.l[k].cin, cout = a.l[k].cout;
  int tile = blockIdx.x - a.l[k].first;
  const int t = tile % 9;
  tile /= 9;
  const int ci0 = (tile % (cin / 32)) * 32, co0 = (tile / (cin / 32)) * 32;
  const bf16* w = a.w + a.l[k].off;
  bf16* wt = a.wt + a.l[k].off;
  const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    s[q + 8 * i][c] = w[((long long)(co0 + q + 8 * i) * 9 + (8 - t)) * cin + ci0 + c];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i)
    wt[((long long)(ci0 + q + 8 * i) * 9 + t) * cout + co0 + c] = s[c][q + 8 * i];
}

int flip_tiles(int cin, int cout) { return 9 * (cin / 32) * (cout / 32); }

// Weights [rows][k] of one or more layers in fragment order: for every 32 rows
// and 16 reduction elements the 1 KB that a wavefront's lanes take for one
// MFMA, 16 bytes per lane, reduction elements in order.  Rows are multiples of
// 64 and k of 9 * 64, so a layer is whole blocks.
constexpr int kMaxFragment = 32;
struct FragmentArgs {
  int layers;
  struct {
    const bf16* src;
    bf16* dst;
    int k, first;   // first: index of the layer's first block
  } l[kMaxFragment];
};

__global__ __launch_bounds__(256) void fragment_kernel(FragmentArgs a) {
  int q = 0;
  while (q + 1 < a.layers && int(blockIdx.x) >= a.l[q + 1].first) ++q;
  const int v = (blockIdx.x - a.l[q].first) * 256 + threadIdx.x;
  const int lane = v & 63, steps = a.l[q].k / 16, s = (v >> 6) % steps, block = (v >> 6) / steps;
  *reinterpret_cast<bf16x8*>(a.l[q].dst + 8LL * v) = *reinterpret_cast<const bf16x8*>(
      a.l[q].src + (long long)(32 * block + (lane & 31)) * a.l[q].k + 16 * s + 8 * (lane >> 5));
}

// Layers whose convolutions (forward and input gradient) take weights in
// fragment order.
bool fragment_layer(int cin, int cout) { return cin % 64 == 0 && cout % 64 == 0; }

// ---------------------------------------------------------------------------
// Convolution, weight and bias gradients
// ---------------------------------------------------------------------------
// Tiled weight gradient of one or more layers in one launch: a block owns 32
// output x 32 input channels of all nine taps of a layer and runs over a
// share (split) of its pixel tiles of 16 x 16.  dy and x (with its one-pixel
// ring, zeros outside the image) are staged in LDS as they lie in memory,
// [pixel][channel]; the MFMA reduces over pixels, so both operands are read
// with the transposing LDS load (ds_read_b64_tr_b16: of 16 lanes, lane i
// receives element i of four rows of 16), two loads per operand of 16 pixels
// x 32 channels.  Rows of 64 bytes without padding: the four rows that half
// a wave reads cover every bank once (with 96 bytes 37 % of the LDS cycles
// were conflicts).  A wave owns two image rows; one dy operand serves the
// nine taps, and the x operands of the second row are two thirds those of
// the first.  Tiles are double buffered: the next one goes to LDS after this
// one is multiplied, the one after that is in flight meanwhile.  At the end
// the eight waves add their sums in LDS.  The bias partial sums are one more
// MFMA against a matrix of ones.  Bound by LDS reads and the registers (one
// block per compute unit, two wavefronts per SIMD): all layers of the network
// at batch 16, 94 GFLOP, take 155 us (610 TFLOP/s) in one launch, against 890
// us in a launch per layer with channel-major copies; 384 -> 128 channels at
// 16 x 32 x 32 alone 27 us.  Wider channel blocks and larger pixel tiles
// spill.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 lds_tr8(const char* p0, const char* p1) {
  using P = __attribute__((address_space(3))) s16x4*;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)p0);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)p1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int kMaxLayers = 16;
struct WgradLayer {
  const bf16* dy;
  const bf16* x;
  float* part;        // [splits][cout][9][cin]
  float* bpart;       // [splits][cout] or null
  float* dw;          // sums over the splits
  float* db;
  int lddy, ldx, h, wd, cin, cout;
  int tiles_x, tiles_y, units, splits;
  int first;                  // first block
  unsigned dybytes, xbytes;   // from the first to the last pixel of ax ay images,
                              // 32 channels of dy and of x
  int n, ax, ay;              // images, and those across and down a tile (see
};                            // wgrad_tiles); last: most forms do not load them
struct WgradGroup {
  int layers;
  WgradLayer l[kMaxLayers];
};

// Forms of the kernel, by what some layer of the group needs: tiles inside the
// images (sides of multiples of 16), tiles that reach beyond them, several images to
// a tile as well, and 64-bit addresses as well (tiles of 2 GB or more).  Each costs
// registers and a longer start (2 us) that the ones before it do without.
enum WgradForm { kWgradFull, kWgradRagged, kWgradPacked, kWgradBig };
template <WgradForm FORM>
__global__ __launch_bounds__(512, 2) void wgrad_tile_kernel(WgradGroup G) {
  constexpr bool BIG = FORM == kWgradBig, PACKED = FORM >= kWgradPacked;
  constexpr bool RAGGED = FORM >= kWgradRagged;
  constexpr int TX = 16, TY = 16;
  constexpr int CO = 32, CI = 32, NT = 512, WK = NT / 64;
  constexpr int SD = 2 * CO, SX = 2 * CI, HX = TX + 2, HP = HX * (TY + 2), P = TX * TY;
  constexpr int kDyVec = P * CO / 8, kXVec = HP * CI / 8;
  constexpr int kDyPer = kDyVec / NT, kXPer = (kXVec + NT - 1) / NT;
  constexpr int kSum = WK * 32 * 33 * 4;   // bytes of the final sums over waves
  constexpr int kStage = P * SD + HP * SX;
  constexpr int RW = TY / WK;              // rows per wave
  static_assert(kDyVec % NT == 0 && kStage >= kSum, "tile");
  __shared__ __align__(16) char smem[2 * kStage];   // two tiles: dy, then x
  const int tid = threadIdx.x, lane = tid & 63;
  const int wk = __builtin_amdgcn_readfirstlane(tid >> 6);
  int layer = 0;
  while (layer + 1 < G.layers && int(blockIdx.x) >= G.l[layer + 1].first) ++layer;
  const WgradLayer a = G.l[layer];
  const int nci = a.cin / CI, base = nci * (a.cout / CO);
  // the channel tiles of one share run on one XCD (block b on XCD b % 8), so
  // its pixels come into one L2 once
  const int idx = blockIdx.x - a.first;
  const bool by8 = a.splits % 8 == 0;
  const int split = by8 ? (idx >> 3) / base * 8 + (idx & 7) : idx / base;
  const int tile = (by8 ? idx >> 3 : idx) % base;
  if (split >= a.splits) return;
  const int ci0 = (tile % nci) * CI, co0 = (tile / nci) * CO;
  const int u0 = int((long long)split * a.units / a.splits);
  const int u1 = int((long long)(split + 1) * a.units / a.splits);
  const bool bias = a.bpart != nullptr && ci0 == 0;

  // Pixel (r, c) of a tile (-1 and 16: its ring) is pixel (r, c) of image k of the
  // tile; false: between images.
  const int per = PACKED ? a.ax * a.ay : 1;
  auto place = [&](int& r, int& c, int& k) {
    k = 0;
    if constexpr (PACKED) {
      const int ky = a.ay > 1 && r > 0 ? r / (a.h + 1) : 0;
      const int kx = a.ax > 1 && c > 0 ? c / (a.wd + 1) : 0;
      r -= ky * (a.h + 1);
      c -= kx * (a.wd + 1);
      k = ky * a.ax + kx;
      return ky < a.ay && kx < a.ax && (a.ay == 1 || (r >= 0 && r < a.h)) &&
             (a.ax == 1 || (c >= 0 && c < a.wd));
    }
    return true;
  };
  // this thread's pieces of a tile: pixel within the image (row << 16 | column, of
  // x from the ring's first on) and byte offset from the tile's first pixel, the
  // same for every tile; packed: image << 10 | row << 5 | column, negative for none
  int pd_[kDyPer], px_[kXPer];
  unsigned od[kDyPer], ox[kXPer];
#pragma unroll
  for (int i = 0; i < kDyPer; ++i) {
    const int v = tid + NT * i, q = v / (CO / 8), c = v % (CO / 8);
    if constexpr (PACKED) {
      int y = q / TX, x = q % TX, k;
      const bool in = place(y, x, k);
      pd_[i] = in ? k << 10 | y << 5 | x : -1;
      od[i] = unsigned(((k * a.h + y) * a.wd + x) * a.lddy + 8 * c) * 2u;
    } else {
      pd_[i] = (q / TX) << 16 | (q % TX);
      od[i] = unsigned(((q / TX) * a.wd + q % TX) * a.lddy + 8 * c) * 2u;
    }
  }
#pragma unroll
  for (int i = 0; i < kXPer; ++i) {
    const int v = tid + NT * i, q = v / (CI / 8), c = v % (CI / 8);
    if constexpr (PACKED) {
      int y = q / HX - 1, x = q % HX - 1, k;
      const bool in = place(y, x, k) && v < kXVec;
      px_[i] = in ? k << 10 | (y + 1) << 5 | (x + 1) : -1;
      ox[i] = unsigned(((k * a.h + y + 1) * a.wd + x + 1) * a.ldx + 8 * c) * 2u;
    } else {
      px_[i] = v < kXVec ? (q / HX) << 16 | (q % HX) : 0x7FFF0000;   // (never stored)
      ox[i] = unsigned((q / HX * a.wd + q % HX) * a.ldx + 8 * c) * 2u;
    }
  }
  int tx, ty, img;   // next tile to load
  bf16x8 rd[kDyPer], rx[kXPer];
  auto load = [&]() {
    const int x0 = tx * TX, y0 = ty * TY;
    const long long org = (long long)img * (PACKED ? per : 1) * a.h * a.wd;
    const bf16* dy = a.dy + org * a.lddy + co0;
    const bf16* xs = a.x + org * a.ldx + ci0;
    if constexpr (PACKED) {
      const int left = min(per, a.n - img * per);   // images of this tile
      if constexpr (BIG) {
#pragma unroll
        for (int i = 0; i < kDyPer; ++i) {
          const int c = (tid + NT * i) % (CO / 8), k = pd_[i] >> 10;
          const int y = y0 + (pd_[i] >> 5 & 31), x = x0 + (pd_[i] & 31);
          rd[i] = bf16x8{};
          if (pd_[i] >= 0 && k < left && y < a.h && x < a.wd)
            rd[i] = *reinterpret_cast<const bf16x8*>(
                dy + (((long long)k * a.h + y) * a.wd + x) * a.lddy + 8 * c);
        }
#pragma unroll
        for (int i = 0; i < kXPer; ++i) {
          const int c = (tid + NT * i) % (CI / 8), k = px_[i] >> 10;
          const int y = y0 - 1 + (px_[i] >> 5 & 31), x = x0 - 1 + (px_[i] & 31);
          rx[i] = bf16x8{};
          if (px_[i] >= 0 && k < left && y >= 0 && y < a.h && x >= 0 && x < a.wd)
            rx[i] = *reinterpret_cast<const bf16x8*>(
                xs + (((long long)k * a.h + y) * a.wd + x) * a.ldx + 8 * c);
        }
      } else {
        // (images beyond the last lie beyond the resource)
        const unsigned gone = unsigned((per - left) * a.h * a.wd) * 2u;
        const Rsrc dr = image_rsrc(dy, a.dybytes - gone * unsigned(a.lddy));
        const Rsrc xr = image_rsrc(xs, a.xbytes - gone * unsigned(a.ldx));
        const unsigned tb = unsigned((y0 * a.wd + x0) * a.lddy) * 2u;
        const unsigned xb = unsigned(((y0 - 1) * a.wd + x0 - 1) * a.ldx) * 2u;   // (may wrap)
#pragma unroll
        for (int i = 0; i < kDyPer; ++i) {
          const bool in =
              pd_[i] >= 0 && y0 + (pd_[i] >> 5 & 31) < a.h && x0 + (pd_[i] & 31) < a.wd;
          rd[i] = load8(dr, in ? od[i] + tb : kOutside);
        }
#pragma unroll
        for (int i = 0; i < kXPer; ++i) {
          const bool in = px_[i] >= 0 &&
                          unsigned(y0 - 1 + (px_[i] >> 5 & 31)) < unsigned(a.h) &&
                          unsigned(x0 - 1 + (px_[i] & 31)) < unsigned(a.wd);
          rx[i] = load8(xr, in ? ox[i] + xb : kOutside);
        }
      }
    } else {
      const Rsrc dr = image_rsrc(dy, a.dybytes), xr = image_rsrc(xs, a.xbytes);
      const unsigned tb = unsigned((y0 * a.wd + x0) * a.lddy) * 2u;
      const unsigned xb = unsigned(((y0 - 1) * a.wd + x0 - 1) * a.ldx) * 2u;   // (may wrap)
#pragma unroll
      for (int i = 0; i < kDyPer; ++i) {
        const bool in = y0 + (pd_[i] >> 16) < a.h && x0 + (pd_[i] & 0xFFFF) < a.wd;
        rd[i] = load8(dr, in ? od[i] + tb : kOutside);
      }
#pragma unroll
      for (int i = 0; i < kXPer; ++i) {
        const bool in = unsigned(y0 - 1 + (px_[i] >> 16)) < unsigned(a.h) &&
                        unsigned(x0 - 1 + (px_[i] & 0xFFFF)) < unsigned(a.wd);
        rx[i] = load8(xr, in ? ox[i] + xb : kOutside);
      }
    }
    if (++tx == a.tiles_x) {
      tx = 0;
      if (++ty == a.tiles_y) {
        ty = 0;
        ++img;
      }
    }
  };
  auto store = [&](int buf) {
    char* sd = smem + buf * kStage;
    char* sx = sd + P * SD;
#pragma unroll
    for (int i = 0; i < kDyPer; ++i) {
      const int v = tid + NT * i;
      *reinterpret_cast<bf16x8*>(sd + (v / (CO / 8)) * SD + 16 * (v % (CO / 8))) = rd[i];
    }
#pragma unroll
    for (int i = 0; i < kXPer; ++i) {
      const int v = tid + NT * i;
      if (kXVec % NT == 0 || v < kXVec)
        *reinterpret_cast<bf16x8*>(sx + (v / (CI / 8)) * SX + 16 * (v % (CI / 8))) = rx[i];
    }
  };

  f32x16 acc[9], accb;
  bf16x8 ones;
#pragma unroll
  for (int v = 0; v < 8; ++v) ones[v] = (bf16)1.f;
  // this lane's pixel row and channel within an operand (first of two loads)
  const int lrow = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int lch = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const char* pd = smem + (RW * wk * TX + lrow) * SD + 2 * lch;
  const char* px = smem + P * SD + (RW * wk * HX + lrow) * SX + 2 * lch;
  // The sums over this block's tiles.  masked: pixels outside the image take no
  // part (else they do with dy = 0).
  auto sweep = [&](auto masked) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      accb[v] = 0.f;
#pragma unroll
      for (int t = 0; t < 9; ++t) acc[t][v] = 0.f;
    }
    tx = u0 % a.tiles_x;
    ty = (u0 / a.tiles_x) % a.tiles_y;
    img = u0 / (a.tiles_x * a.tiles_y);
    int mx = tx, my = ty;   // tile being multiplied
    if (u0 < u1) load();
    store(0);
    if (u0 + 1 < u1) load();
    __syncthreads();
    for (int u = u0; u < u1; ++u) {
      const int buf = (u - u0) & 1;
      const char* d = pd + buf * kStage;
      const char* b = px + buf * kStage;
      unsigned cols = 0, rows = 0;   // bit: column, row of the tile inside an image
      if constexpr (masked) {
        for (int i = 0; i < TX; ++i) {
          int r0 = 0, c0 = 0, r = i, c = i, k;
          if (place(r0, c, k) && mx * TX + c < a.wd) cols |= 1u << i;
          if (place(r, c0, k) && my * TY + r < a.h) rows |= 1u << i;
        }
      }
      bf16x8 B[3][3];
#pragma unroll
      for (int j = 0; j < RW; ++j) {
#pragma unroll
        for (int k = j ? 2 : 0; k < 3; ++k)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const char* bt = b + ((j + k) * HX + c) * SX;
            B[(j + k) % 3][c] = lds_tr8(bt, bt + 4 * SX);
            if constexpr (masked) {
#pragma unroll
              for (int v = 0; v < 8; ++v)
                if (!((cols >> (8 * (lane >> 5) + v)) & 1)) B[(j + k) % 3][c][v] = (bf16)0.f;
            }
          }
        if (masked && !((rows >> (RW * wk + j)) & 1)) continue;   // uniform
        const bf16x8 A = lds_tr8(d + j * TX * SD, d + (j * TX + 4) * SD);
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] = mfma32(A, B[(j + t / 3) % 3][t % 3], acc[t]);
        if (bias) accb = mfma32(A, ones, accb);
      }
      if (masked && ++mx == a.tiles_x) {
        mx = 0;
        my = my + 1 == a.tiles_y ? 0 : my + 1;
      }
      if (u + 1 < u1) store(buf ^ 1);
      if (u + 2 < u1) load();
      __syncthreads();
    }
  };
  sweep(std::false_type{});
  // Inputs that are not finite: a pixel outside the image (dy = 0) has neighbours
  // inside, and 0 times infinity is none of the sum.  Seen in the sums, which are
  // then taken again without those pixels (masks in the loop itself cost 4 to 14 %
  // of a launch).
  if constexpr (RAGGED) {
    int* again = reinterpret_cast<int*>(smem);   // (every wave has left the loop)
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) z += acc[t][v] * 0.f;
    if (tid == 0) *again = 0;
    __syncthreads();
    if (z != 0.f) *again = 1;
    __syncthreads();
    const int redo = *again;
    __syncthreads();
    if (redo) sweep(std::true_type{});
  }
  const int r = lane & 31, g = lane >> 5;
  float* part = a.part + (long long)split * 9 * a.cin * a.cout;
  // sum over the waves, tap by tap, then the bias; two areas in turn, so that
  // one barrier per tap is enough
  float (*sums)[WK][32][33] = reinterpret_cast<float (*)[WK][32][33]>(smem);
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float (*sum)[32][33] = sums[t & 1];
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[wk][8 * (i / 4) + 4 * g + i % 4][r] = acc[t][i];
    __syncthreads();
#pragma unroll
    for (int e = tid; e < 1024; e += NT) {
      const int co = e >> 5, ci = e & 31;
      float v = sum[0][co][ci];
#pragma unroll
      for (int k = 1; k < WK; ++k) v += sum[k][co][ci];
      part[((long long)(co0 + co) * 9 + t) * a.cin + ci0 + ci] = v;
    }
  }
  if (bias) {
    float (*sum)[32][33] = sums[1];
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[wk][8 * (i / 4) + 4 * g + i % 4][r] = accb[i];
    __syncthreads();
    if (tid < 32) {
      float v = sum[0][tid][0];
#pragma unroll
      for (int k = 1; k < WK; ++k) v += sum[k][tid][0];
      a.bpart[(long long)split * a.cout + co0 + tid] = v;
    }
  }
}

// Sums over the splits of one or more weight gradients: dw[i] = sum_s
// part[s][i] for i < count and db[j] = sum_s bpart[s][j] for j < bcount (bpart
// may be null).  More than 16 splits (many tiles, few weights): a block owns 64
// consecutive entries; its 16 groups of 16 threads each add every 16th split
// (four entries per thread), then one group adds the 16 sums.  Up to 16 splits:
// 1024 entries per block, four per thread, split by split, which is the same
// order (the network's bottom layers hold most of the weights in few splits;
// with 64 entries per block their 27 000 short blocks bounded the launch, 35.4
// us for the network at batch 16, now 12.1).  Counts are multiples of 4.
constexpr int kFewSplits = 16;
__host__ __device__ constexpr int sum_entries(int splits) {
  return splits > kFewSplits ? 64 : 1024;
}
struct SumArgs {
  int layers;
  struct {
    const float* part;
    const float* bpart;
    float* dw;
    float* db;
    long long count;
    int bcount, splits, first, wblocks;   // first block, blocks of the weights
  } l[kMaxLayers];
};

__global__ __launch_bounds__(256) void sum_splits_kernel(SumArgs a) {
  __shared__ f32x4 s[16][16];
  const int e = threadIdx.x & 15, k0 = threadIdx.x >> 4;
  int k = 0;
  while (k + 1 < a.layers && int(blockIdx.x) >= a.l[k + 1].first) ++k;
  const int block = blockIdx.x - a.l[k].first, splits = a.l[k].splits;
  const bool bias = block >= a.l[k].wblocks;
  const float* src = bias ? a.l[k].bpart : a.l[k].part;
  float* dst = bias ? a.l[k].db : a.l[k].dw;
  const long long n = bias ? a.l[k].bcount : a.l[k].count;
  const long long first = (long long)(block - (bias ? a.l[k].wblocks : 0)) * sum_entries(splits);
  f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
  if (splits <= kFewSplits) {
    const long long i = first + 4 * (int)threadIdx.x;
    if (i >= n) return;
#pragma unroll 8
    for (int j = 0; j < splits; ++j)
      v += *reinterpret_cast<const f32x4*>(src + (long long)j * n + i);
    *reinterpret_cast<f32x4*>(dst + i) = v;
    return;
  }
  const long long i = first + 4 * e;
  if (i < n) {
#pragma unroll 4
    for (int j = k0; j < splits; j += 16)
      v += *reinterpret_cast<const f32x4*>(src + (long long)j * n + i);
  }
  s[k0][e] = v;
  __syncthreads();
  if (k0 == 0 && i < n) {
#pragma unroll
    for (int j = 1; j < 16; ++j) v += s[j][e];
    *reinterpret_cast<f32x4*>(dst + i) = v;
  }
}

// Into how many shares the pixel tiles of a weight gradient go.
// One layer alone: a round of 256 blocks (one per compute unit: registers)
// costs its tiles, about 3000 clocks each, and every share's partial sums are
// written and read once more (about 1.7 kB per clock).  Over the network's
// layers at batch 2 and 16 the choice is within 8 % of the best power of two.
// In a group (per_block > 0) that many tiles per block, more shares than
// eight in multiples of eight (one per XCD).
struct WgradPlan {
  int ax, ay, tiles_x, tiles_y, units, splits;
};

// Pixel tiles.  Images of up to seven pixels a side lie several to a tile, with a
// row or column of zeros between them (128 -> 128 channels: 12 000 images of 1 x 1,
// 64 to a tile, 851 us with a tile each, 31 so; 3750 of 4 x 4, nine to a tile, 276
// and 47).
WgradPlan wgrad_tiles(int n, int h, int wd) {
  WgradPlan p{17 / (wd + 1), 17 / (h + 1), (wd + 15) / 16, (h + 15) / 16, 0, 0};
  if (p.ax < 1) p.ax = 1;
  if (p.ay < 1) p.ay = 1;
  p.units = (n + p.ax * p.ay - 1) / (p.ax * p.ay) * p.tiles_x * p.tiles_y;
  return p;
}

WgradPlan wgrad_plan(int n, int h, int wd, int cin, int cout, int per_block = 0) {
  WgradPlan p = wgrad_tiles(n, h, wd);
  if (per_block > 0) {
    const int s = (p.units + per_block - 1) / per_block;
    p.splits = s < 8 ? s : std::min(s / 8 * 8, 1024);
    return p;
  }
  const int base = (cin / 32) * (cout / 32);
  double best = 0.0;
  auto consider = [&](int s) {
    if (s < 1 || s > p.units || s > 1024) return;
    const double rounds = (base * (long long)s + 255) / 256;
    const double cost = rounds * ((p.units + s - 1) / s) * 3000.0 +
                        (double)s * (9.0 * cin * cout + cout) * 8.0 / 1700.0;
    if (p.splits == 0 || cost < best) {
      p.splits = s;
      best = cost;
    }
  };
  for (int s = 1; s <= 1024; s *= 2) consider(s);
  consider(256 / base);   // exactly one round
  return p;
}

// ---------------------------------------------------------------------------
// Elementwise layers (8 channels per thread)
// ---------------------------------------------------------------------------
__global__ void relu_bwd_kernel(bf16* d, int ldd, const bf16* y, int ldy, long long npix, int cv) {
  const long long total = npix * cv;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long p = e / cv;
    const int c = int(e % cv) * 8;
    const bf16x8 dv = *reinterpret_cast<const bf16x8*>(d + p * ldd + c);
    *reinterpret_cast<bf16x8*>(d + p * ldd + c) =
        relu_mask(dv, *reinterpret_cast<const bf16x8*>(y + p * ldy + c));
  }
}

// (h, wd): input size of the pooling
__global__ void pool2_fwd_kernel(const bf16* x, int ldx, bf16* y, int ldy, int n, int h, int wd,
                                 int cv) {
  const int ho = h / 2, wo = wd / 2;
  const long long total = (long long)n * ho * wo * cv;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int c = int(e % cv) * 8;
    const long long po = e / cv;
    const int X = int(po % wo), Y = int((po / wo) % ho);
    const long long nn = po / ((long long)wo * ho);
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const long long pi = (nn * h + 2 * Y + i) * wd + 2 * X + j;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(x + pi * ldx + c);
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] += (float)v[u];
      }
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16)(0.25f * s[u]);
    *reinterpret_cast<bf16x8*>(y + po * ldy + c) = o;
  }
}

// mask (or null): the result is zeroed where mask <= 0 (ReLU backward)
__global__ void pool2_bwd_kernel(const bf16* dy, int lddy, const bf16* add, int ldadd, bf16* dx,
                                 int lddx, int n, int h, int wd, int cv, const bf16* mask,
                                 int ldmask) {
  const int ho = h / 2, wo = wd / 2;
  const long long total = (long long)n * h * wd * cv;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int c = int(e % cv) * 8;
    const long long p = e / cv;
    const int x = int(p % wd), y = int((p / wd) % h);
    const long long nn = p / ((long long)wd * h);
    const long long po = (nn * ho + y / 2) * wo + x / 2;
    const bf16x8 g = *reinterpret_cast<const bf16x8*>(dy + po * lddy + c);
    bf16x8 a = bf16x8{};
    if (add) a = *reinterpret_cast<const bf16x8*>(add + p * ldadd + c);
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16)((float)a[u] + 0.25f * (float)g[u]);
    if (mask) o = relu_mask(o, *reinterpret_cast<const bf16x8*>(mask + p * ldmask + c));
    *reinterpret_cast<bf16x8*>(dx + p * lddx + c) = o;
  }
}

// (h, wd): coarse size
__global__ void up2_fwd_kernel(const bf16* x, int ldx, bf16* y, int ldy, int n, int h, int wd,
                               int cv) {
  const int hf = 2 * h, wf = 2 * wd;
  const long long total = (long long)n * hf * wf * cv;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int c = int(e % cv) * 8;
    const long long p = e / cv;
    const int xf = int(p % wf), yf = int((p / wf) % hf);
    const long long nn = p / ((long long)wf * hf);
    const long long pc = (nn * h + yf / 2) * wd + xf / 2;
    *reinterpret_cast<bf16x8*>(y + p * ldy + c) =
        *reinterpret_cast<const bf16x8*>(x + pc * ldx + c);
  }
}

// mask (or null): a fine image (2h x 2wd) that holds each coarse value four
// times; the result is zeroed where it is <= 0 (ReLU backward)
__global__ void up2_bwd_kernel(const bf16* dy, int lddy, bf16* dx, int lddx, int n, int h, int wd,
                               int cv, const bf16* mask, int ldmask) {
  const int wf = 2 * wd;
  const long long total = (long long)n * h * wd * cv;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int c = int(e % cv) * 8;
    const long long pc = e / cv;
    const int X = int(pc % wd), Y = int((pc / wd) % h);
    const long long nn = pc / ((long long)wd * h);
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const long long pf = (nn * 2 * h + 2 * Y + i) * wf + 2 * X + j;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(dy + pf * lddy + c);
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] += (float)v[u];
      }
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16)s[u];
    if (mask)
      o = relu_mask(o, *reinterpret_cast<const bf16x8*>(
                           mask + ((nn * 2 * h + 2 * Y) * wf + 2 * X) * ldmask + c));
    *reinterpret_cast<bf16x8*>(dx + pc * lddx + c) = o;
  }
}

int grid_for(long long total) {
  long long b = (total + 255) / 256;
  return (int)std::min<long long>(std::max<long long>(b, 1), 65536);
}

// ---------------------------------------------------------------------------
// Loss
// ---------------------------------------------------------------------------
constexpr int kLossBlocks = 512;

// per-block FP64 partials: work[2 b] = sum of squares, work[2 b + 1] = fluid count
__global__ __launch_bounds__(256) void loss_partial_kernel(const float* out, int ldo,
                                                           const float* t, const uint8_t* fluid,
                                                           long long npix, double* work) {
  __shared__ double s_sq[256], s_n[256];
  double sq = 0.0, cnt = 0.0;
  for (long long p = blockIdx.x * 256LL + threadIdx.x; p < npix; p += 256LL * gridDim.x) {
    if (!fluid[p]) continue;
    cnt += 1.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double d = (double)out[p * ldo + c] - (double)t[p * 3 + c];
      sq += d * d;
    }
  }
  s_sq[threadIdx.x] = sq;
  s_n[threadIdx.x] = cnt;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s_sq[threadIdx.x] += s_sq[threadIdx.x + w];
      s_n[threadIdx.x] += s_n[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    work[2 * blockIdx.x] = s_sq[0];
    work[2 * blockIdx.x + 1] = s_n[0];
  }
}

// Gradient of the loss, 8 channels of one pixel per thread.  Every block
// first adds the per-block partials in the same fixed-order tree (8 KB from
// L2, cheaper than a launch of its own: 11.8 us at 16 x 128 x 128 for 34 MB);
// block 0 writes the loss and the
// fluid count behind the partials.  ldo is a multiple of 8.
__global__ __launch_bounds__(256) void loss_grad_kernel(const float* __restrict__ out, int ldo,
                                                        const float* __restrict__ t,
                                                        const uint8_t* __restrict__ fluid,
                                                        long long npix, bf16* __restrict__ dout,
                                                        const double* __restrict__ work,
                                                        double* __restrict__ fin, int blocks) {
  __shared__ double ssq[256], sn[256];
  double sq = 0.0, cnt = 0.0;
  for (int b = threadIdx.x; b < blocks; b += 256) {
    sq += work[2 * b];
    cnt += work[2 * b + 1];
  }
  ssq[threadIdx.x] = sq;
  sn[threadIdx.x] = cnt;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      ssq[threadIdx.x] += ssq[threadIdx.x + w];
      sn[threadIdx.x] += sn[threadIdx.x + w];
    }
    __syncthreads();
  }
  const double n = sn[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    fin[0] = n > 0 ? ssq[0] / (3.0 * n) : 0.0;
    fin[1] = n;
  }
  const float scale = n > 0 ? float(2.0 / (3.0 * n)) : 0.f;
  const int cv = ldo / 8;
  const long long total = npix * cv;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < total; e += gridDim.x * 256LL) {
    const long long p = e / cv;
    bf16x8 g = bf16x8{};
    if (e == p * cv && fluid[p]) {
#pragma unroll
      for (int c = 0; c < 3; ++c) g[c] = (bf16)(scale * (out[p * ldo + c] - t[p * 3 + c]));
    }
    *reinterpret_cast<bf16x8*>(dout + 8 * e) = g;
  }
}

// ---------------------------------------------------------------------------
// Adam
// ---------------------------------------------------------------------------
__global__ void adam_kernel(float* p, float* m, float* v, const float* g, bf16* pb, long long n,
                            float lr, float b1, float b2, float eps, float c1, float c2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = (bf16)pi;
  }
}

__global__ void to_bf16_kernel(const float* p, bf16* pb, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    pb[i] = (bf16)p[i];
}

// ---------------------------------------------------------------------------
// Input and output maps
// ---------------------------------------------------------------------------
// Coarse cell I covers the fine nodes i with floor(I fine / res) <= i <
// floor((I + 1) fine / res) (at least the node floor(I fine / res)); its
// solid fraction is the mean of the mask over those nodes.
__device__ __forceinline__ void cell_range(int I, int fine, int res, int& a, int& b) {
  if ((long long)res * fine < 1LL << 32) {   // uniform; 64-bit divisions are slow
    a = int(unsigned(I) * unsigned(fine) / unsigned(res));
    b = int(unsigned(I + 1) * unsigned(fine) / unsigned(res));
  } else {
    a = int((long long)I * fine / res);
    b = int((long long)(I + 1) * fine / res);
  }
  if (b <= a) b = a + 1;
}

// Row and column of element k of an array with rows of nx, without a 64-bit
// division where 32 bits hold k (uniform).
__device__ __forceinline__ void row_col(long long k, int nx, bool small, int& j, int& i) {
  if (small) {
    j = int(unsigned(k) / unsigned(nx));
    i = int(unsigned(k) - unsigned(j) * unsigned(nx));
  } else {
    j = int(k / nx);
    i = int(k - (long long)j * nx);
  }
}

// The case kind (case_params[cps c + 3] when cps == 4, else a cavity)
// places the driven-boundary marker: the lid row (top) of a cavity, the
// inlet column (left) of a channel.
__device__ __forceinline__ int case_kind(const float* cp, int cps, long long c) {
  return cps > 3 ? int(cp[cps * c + 3]) : UNET_KIND_CAVITY;
}

// Grid: pixels of a case in x, cases in y.  Bound by the stores (64 bytes per
// pixel); one index over all cases with 64-bit divisions took 15.1 us for 12
// cases of 128 x 128.
__global__ __launch_bounds__(256) void make_input_kernel(const uint8_t* solid, int nx, int ny,
                                                         const float* cp, int cps, int n, int res,
                                                         bf16* x0) {
  const long long per = (long long)res * res;
  const bool small = per <= 0xffffffffLL;
  const int lane = threadIdx.x & 63;
  static_assert(UNET_IN_CHANNELS == 32, "four lanes per pixel");
  for (long long c = blockIdx.y; c < n; c += gridDim.y) {
    for (long long p = blockIdx.x * 256LL + threadIdx.x; p - lane < per; p += gridDim.x * 256LL) {
      bf16x8 o = bf16x8{};
      if (p < per) {
        int i, j;
        row_col(p, res, small, j, i);
        int i0, i1, j0, j1;
        cell_range(i, nx, res, i0, i1);
        cell_range(j, ny, res, j0, j1);
        int cnt = 0;
        for (int b = j0; b < j1; ++b)
          for (int a = i0; a < i1; ++a) cnt += solid[(c * ny + b) * nx + a] != 0;
        o[0] = (bf16)(float(cnt) / float((i1 - i0) * (j1 - j0)));
        o[1] = (bf16)(cp[cps * c + 0] / 500.f);
        o[2] = (bf16)cp[cps * c + 1];
        o[3] = (bf16)(cp[cps * c + 2] / 0.1f);
        o[4] = (bf16)((i + 0.5f) / res);
        o[5] = (bf16)((j + 0.5f) / res);
        const bool channel = case_kind(cp, cps, c) == UNET_KIND_CHANNEL;
        o[6] = (bf16)((channel ? i == 0 : j == res - 1) ? 1.f : 0.f);
        o[7] = (bf16)1.f;
      }
      // the wavefront's 64 pixels, 16 at a time: lane l stores channels 8 (l % 4)
      // .. of pixel l / 4, so a store is 1 KB in one piece (64 bytes per lane
      // apart: 14.4 us)
      const i32x4 v = __builtin_bit_cast(i32x4, o);
      const long long first = p - lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int from = 16 * q + lane / 4;
        i32x4 w;
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = __shfl(v[u], from, 64);
        if (lane % 4) w = i32x4{};
        if (first + from < per)
          *reinterpret_cast<i32x4*>(x0 + (c * per + first + from) * UNET_IN_CHANNELS +
                                    8 * (lane % 4)) = w;
      }
    }
  }
}

// Bilinear values of three channels at (u, v), in coarse pixel-centre
// coordinates.  vec: a pixel's channels can be read as four floats (one load
// instead of three: neighbouring lanes' pixels lie in different lines).
__device__ __forceinline__ void bilinear3(const float* out, int ldo, bool vec, long long c, int res,
                                          float u, float v, float r[3]) {
  u = fminf(fmaxf(u, 0.f), float(res - 1));
  v = fminf(fmaxf(v, 0.f), float(res - 1));
  const int i0 = min(int(u), res - 2 < 0 ? 0 : res - 2), j0 = min(int(v), res - 2 < 0 ? 0 : res - 2);
  const int i1 = min(i0 + 1, res - 1), j1 = min(j0 + 1, res - 1);
  const float fu = u - i0, fv = v - j0;
  float p[4][3];
  const int pi[4] = {i0, i1, i0, i1}, pj[4] = {j0, j0, j1, j1};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float* at = out + ((c * res + pj[q]) * res + pi[q]) * ldo;
    if (vec) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(at);
      for (int ch = 0; ch < 3; ++ch) p[q][ch] = w[ch];
    } else {
      for (int ch = 0; ch < 3; ++ch) p[q][ch] = at[ch];
    }
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch)
    r[ch] = (1 - fv) * ((1 - fu) * p[0][ch] + fu * p[1][ch]) +
            fv * ((1 - fu) * p[2][ch] + fu * p[3][ch]);
}

// Grid as above.
__global__ __launch_bounds__(256) void fields_kernel(const float* out, int ldo, int n, int res,
                                                     const float* cp, int cps,
                                                     const uint8_t* solid, int nx, int ny,
                                                     float* rho, float* ux, float* uy) {
  const long long per = (long long)nx * ny;
  const bool small = per <= 0xffffffffLL;
  const bool vec = ldo % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
  const float scx = float(res) / float(nx), scy = float(res) / float(ny);
  for (long long c = blockIdx.y; c < n; c += gridDim.y) {
    for (long long p = blockIdx.x * 256LL + threadIdx.x; p < per; p += gridDim.x * 256LL) {
      const long long e = c * per + p;
      int i, j;
      row_col(p, nx, small, j, i);
      if (solid[e]) {
        rho[e] = 1.f;
        ux[e] = 0.f;
        uy[e] = 0.f;
        continue;
      }
      const float U = cp[cps * c + 2];
      const float u = (i + 0.5f) * scx - 0.5f, v = (j + 0.5f) * scy - 0.5f;
      float r[3];
      bilinear3(out, ldo, vec, c, res, u, v, r);
      rho[e] = 1.f + 3.f * U * U * r[0];
      ux[e] = U * r[1];
      uy[e] = U * r[2];
    }
  }
}

// One block per case (fixed-order FP64 sums).  (1) Remove the fluid mean of
// rho - 1.  (2) Remove the staggered momentum components: with bounce-back
// walls and no force, every step flips the sign of
// Ix = sum_fluid (-1)^i j_x and of Iy = sum_fluid (-1)^j j_y (collision
// conserves j at each node; streaming and bounce-back move each population
// with e_x != 0 to a column of the other parity, or reverse it in place), so
// a start with Ix or Iy != 0 never settles: the state keeps an undamped
// period-2 oscillation.  u_x -= (-1)^i Ix / sum rho (likewise u_y) makes
// both zero, as they are for the state at rest.  Closed lattices (cavities)
// only: a channel's inlet and outlet change its mass and do not keep these
// sums, so its prediction is left as it is.
//
// Bound by latency (three dependent passes over the case): 1024 threads with
// 16 independent loads each in flight per field, kept in registers from pass to
// pass where they hold the case (256 threads with one load: 96 us for 12 cases
// of 128 x 128; eight loads and every pass from memory: 19.2 us; now 17).  A
// case one node larger than they hold is read three times: all output maps of 12
// cases take 25.5 us at 128 x 128 and 34.2 at 129 x 129, of 64 cases 56.8 and
// 64.9.
constexpr int kMassThreads = 1024, kMassLoads = 16;
__global__ __launch_bounds__(kMassThreads) void mass_fix_kernel(float* rho, float* ux, float* uy,
                                                                const uint8_t* solid, int nx,
                                                                int ny, const float* cp, int cps) {
  constexpr int kWaves = kMassThreads / 64;
  __shared__ double s[2][3][kWaves];
  if (case_kind(cp, cps, blockIdx.x) != UNET_KIND_CAVITY) return;
  const int tid = threadIdx.x;
  const long long cnt = (long long)nx * ny;
  const bool small = cnt <= 0xffffffffLL;
  const long long base = (long long)blockIdx.x * cnt;
  rho += base;
  ux += base;
  uy += base;
  solid += base;
  auto block_sums = [&](double (*t)[kWaves], double v[3]) {
    for (int q = 0; q < 3; ++q) {
      for (int w = 32; w > 0; w >>= 1) v[q] += __shfl_xor(v[q], w, 64);
      if (tid % 64 == 0) t[q][tid / 64] = v[q];
    }
    __syncthreads();
    for (int q = 0; q < 3; ++q) {
      v[q] = 0.0;
      for (int w = 0; w < kWaves; ++w) v[q] += t[q][w];
    }
  };
  // calls f(u, k) for the thread's nodes, load(u, k) (k clamped into the case)
  // for a group of them first, unless the registers already hold them all
  const bool kept = cnt <= kMassThreads * kMassLoads;
  auto nodes = [&](bool fresh, auto load, auto f) {
    for (long long k0 = tid; k0 < cnt; k0 += kMassThreads * kMassLoads) {
      if (fresh || !kept)
#pragma unroll
      for (int u = 0; u < kMassLoads; ++u) {
        const long long k = k0 + u * kMassThreads;
        load(u, k < cnt ? k : cnt - 1);
      }
#pragma unroll
      for (int u = 0; u < kMassLoads; ++u)
        if (k0 + u * kMassThreads < cnt) f(u, k0 + u * kMassThreads);
    }
  };
  float r[kMassLoads], a[kMassLoads], b[kMassLoads];
  unsigned sol = 0;   // bit u: node u is solid
  auto load_mask = [&](int u, long long k) {
    sol = (sol & ~(1u << u)) | (solid[k] ? 1u << u : 0u);
  };
  double sum[3] = {};
  nodes(
      true,
      [&](int u, long long k) {
        r[u] = rho[k];
        load_mask(u, k);
        if (kept) {
          a[u] = ux[k];
          b[u] = uy[k];
        }
      },
      [&](int u, long long) {
        if (!(sol >> u & 1)) {
          sum[0] += (double)r[u] - 1.0;
          sum[1] += 1.0;
        }
      });
  block_sums(s[0], sum);
  const float mean = sum[1] > 0 ? float(sum[0] / sum[1]) : 0.f;
  sum[0] = sum[1] = sum[2] = 0.0;
  nodes(
      false,
      [&](int u, long long k) {
        r[u] = rho[k];
        a[u] = ux[k];
        b[u] = uy[k];
        load_mask(u, k);
      },
      [&](int u, long long k) {
        if (sol >> u & 1) return;
        const float rm = r[u] - mean;
        rho[k] = rm;
        int i, j;
        row_col(k, nx, small, j, i);
        sum[0] += (i & 1 ? -1.0 : 1.0) * (double)rm * (double)a[u];
        sum[1] += (j & 1 ? -1.0 : 1.0) * (double)rm * (double)b[u];
        sum[2] += (double)rm;
      });
  block_sums(s[1], sum);
  const double R = sum[2];
  const float mx = R > 0 ? float(sum[0] / R) : 0.f, my = R > 0 ? float(sum[1] / R) : 0.f;
  nodes(
      false,
      [&](int u, long long k) {
        a[u] = ux[k];
        b[u] = uy[k];
        load_mask(u, k);
      },
      [&](int u, long long k) {
        if (sol >> u & 1) return;
        int i, j;
        row_col(k, nx, small, j, i);
        ux[k] = a[u] - ((i & 1) ? -mx : mx);
        uy[k] = b[u] - ((j & 1) ? -my : my);
      });
}

}  // namespace

// ===========================================================================
// Input and output maps of either shape (cps: floats per case in case_params)
// ===========================================================================
static dim3 case_grid(long long per, int n) {
  return dim3(unsigned(std::min<long long>((per + 255) / 256, 65535)), std::min(n, 65535));
}

static int launch_make_input(const uint8_t* solid, int nx, int ny, const float* cp, int cps, int n,
                      int res, void* x0, void* stream) {
  if (!solid || !cp || !x0 || n <= 0 || res <= 0 || nx <= 0 || ny <= 0)
    return fail(UNET_EINVAL, "make_input: bad arguments");
  hipLaunchKernelGGL(make_input_kernel, case_grid((long long)res * res, n), dim3(256), 0,
                     as_stream(stream), solid, nx, ny, cp, cps, n, res, static_cast<bf16*>(x0));
  UCHECK(hipGetLastError());
  return UNET_OK;
}

static int launch_fields(const float* out, int ldo, int n, int res, const float* cp, int cps,
                  const uint8_t* solid, int nx, int ny, float* rho, float* ux, float* uy,
                  void* stream) {
  if (!out || !cp || !solid || !rho || !ux || !uy || n <= 0 || res < 2 || nx <= 0 || ny <= 0 ||
      ldo < 3)
    return fail(UNET_EINVAL, "fields_from_output: bad arguments");
  hipStream_t st = as_stream(stream);
  hipLaunchKernelGGL(fields_kernel, case_grid((long long)nx * ny, n), dim3(256), 0, st,
                     out, ldo, n, res, cp, cps, solid, nx, ny, rho, ux, uy);
  hipLaunchKernelGGL(mass_fix_kernel, dim3(n), dim3(kMassThreads), 0, st, rho, ux, uy, solid, nx,
                     ny, cp, cps);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

// Adds a layer to a group; returns the floats of `work` it uses.
static long long add_wgrad(WgradGroup& g, const WgradPlan& p, const bf16* dy, int lddy,
                           const bf16* x, int ldx, float* dw, float* db, int n, int h, int wd,
                           int cin, int cout, float* work) {
  WgradLayer& l = g.l[g.layers];
  const long long wcount = 9LL * cin * cout;
  const int per = p.ax * p.ay;
  l = WgradLayer{dy, x, work, db ? work + p.splits * wcount : nullptr, dw, db, lddy, ldx, h, wd,
                 cin, cout, p.tiles_x, p.tiles_y, p.units, p.splits, 0,
                 (unsigned)image_bytes(per * h, wd, lddy, 32),
                 (unsigned)image_bytes(per * h, wd, ldx, 32), n, p.ax, p.ay};
  if (g.layers) {
    const WgradLayer& q = g.l[g.layers - 1];
    l.first = q.first + (q.splits * (q.cin / 32) * (q.cout / 32) + 7) / 8 * 8;
  }
  ++g.layers;
  return p.splits * (wcount + cout);
}

// Partial sums of every layer of the group, then the sums over the splits.
static int launch_wgrad(const WgradGroup& g, hipStream_t st) {
  const WgradLayer& e = g.l[g.layers - 1];
  const dim3 grid(e.first + e.splits * (e.cin / 32) * (e.cout / 32)), block(512);
  WgradForm form = kWgradFull;
  for (int k = 0; k < g.layers; ++k) {
    const WgradLayer& l = g.l[k];
    const int rows = l.ax * l.ay * l.h;
    const bool big = image_bytes(rows, l.wd, l.lddy, 32) > kMaxRsrc ||
                     image_bytes(rows, l.wd, l.ldx, 32) > kMaxRsrc;
    form = std::max(form, big                     ? kWgradBig
                          : l.ax * l.ay > 1       ? kWgradPacked
                          : l.h % 16 || l.wd % 16 ? kWgradRagged
                                                  : kWgradFull);
  }
  switch (form) {
    case kWgradFull:
      hipLaunchKernelGGL(wgrad_tile_kernel<kWgradFull>, grid, block, 0, st, g);
      break;
    case kWgradRagged:
      hipLaunchKernelGGL(wgrad_tile_kernel<kWgradRagged>, grid, block, 0, st, g);
      break;
    case kWgradPacked:
      hipLaunchKernelGGL(wgrad_tile_kernel<kWgradPacked>, grid, block, 0, st, g);
      break;
    default:
      hipLaunchKernelGGL(wgrad_tile_kernel<kWgradBig>, grid, block, 0, st, g);
      break;
  }
  UCHECK(hipGetLastError());
  SumArgs sums{};
  sums.layers = g.layers;
  int blocks = 0;
  for (int k = 0; k < g.layers; ++k) {
    const WgradLayer& l = g.l[k];
    auto& q = sums.l[k];
    q.part = l.part;
    q.bpart = l.bpart;
    q.dw = l.dw;
    q.db = l.db;
    q.count = 9LL * l.cin * l.cout;
    q.bcount = l.db ? l.cout : 0;
    q.splits = l.splits;
    q.first = blocks;
    const int per = sum_entries(l.splits);
    q.wblocks = int((q.count + per - 1) / per);
    blocks += q.wblocks + (q.bcount + per - 1) / per;
  }
  hipLaunchKernelGGL(sum_splits_kernel, dim3(blocks), dim3(256), 0, st, sums);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

// ===========================================================================
// C ABI: layers
// ===========================================================================
extern "C" {

const char* unet_last_error(void) { return g_err.c_str(); }

int unet_conv3x3_fwd(const void* x, int32_t ldx, const void* w, const float* bias, void* y,
                     int32_t ldy, int32_t n, int32_t h, int32_t wd, int32_t cin, int32_t cout,
                     int32_t relu, int32_t out_f32, void* stream) {
  if (n <= 0 || h <= 0 || wd <= 0) return fail(UNET_EINVAL, "conv: bad size");
  ConvArgs a{static_cast<const bf16*>(x), ldx, static_cast<const bf16*>(w), bias, y, ldy,
             n * h * wd, h, wd, cin, cout, relu, out_f32};
  return launch_conv(a, as_stream(stream));
}

int unet_conv3x3_bwd_data(const void* dy, int32_t lddy, const void* w, void* dx, int32_t lddx,
                          int32_t n, int32_t h, int32_t wd, int32_t cin, int32_t cout, void* work,
                          void* stream) {
  if (!work || !w) return fail(UNET_EINVAL, "bwd_data: null pointer");
  if (n <= 0 || h <= 0 || wd <= 0) return fail(UNET_EINVAL, "bwd_data: bad size");
  hipStream_t st = as_stream(stream);
  if (cin <= 0 || cout <= 0 || cin % 32 || cout % 32)
    return fail(UNET_EINVAL, "bwd_data: cin and cout must be positive multiples of 32");
  FlipArgs f{};
  f.w = static_cast<const bf16*>(w);
  f.wt = static_cast<bf16*>(work);
  f.layers = 1;
  f.l[0].cin = cin;
  f.l[0].cout = cout;
  hipLaunchKernelGGL(flip_tiles_kernel, dim3(flip_tiles(cin, cout)), dim3(256), 0, st, f);
  ConvArgs a{static_cast<const bf16*>(dy), lddy, static_cast<const bf16*>(work), nullptr, dx,
             lddx, n * h * wd, h, wd, cout, cin, 0, 0};
  return launch_conv(a, st);
}

int64_t unet_wgrad_work_floats(int32_t n, int32_t h, int32_t wd, int32_t cin, int32_t cout) {
  if (n <= 0 || h <= 0 || wd <= 0 || cin < 32 || cout < 32) return 0;   // (nothing to do)
  return (int64_t)wgrad_plan(n, h, wd, cin, cout).splits * (9LL * cin * cout + cout);
}

int unet_conv3x3_bwd_weight(const void* dy, int32_t lddy, const void* x, int32_t ldx, float* dw,
                            float* dbias, int32_t n, int32_t h, int32_t wd, int32_t cin,
                            int32_t cout, float* work, void* stream) {
  if (!dy || !x || !dw || !work) return fail(UNET_EINVAL, "bwd_weight: null pointer");
  if (n <= 0 || h <= 0 || wd <= 0) return fail(UNET_EINVAL, "bwd_weight: bad size");
  if (cin % 32 || cout % 32 || cin <= 0 || cout <= 0)
    return fail(UNET_EINVAL, "bwd_weight: cin and cout must be positive multiples of 32");
  if (lddy % 8 || ldx % 8 || lddy < cout || ldx < cin)
    return fail(UNET_EINVAL, "bwd_weight: bad ld");
  WgradGroup g{};
  add_wgrad(g, wgrad_plan(n, h, wd, cin, cout), static_cast<const bf16*>(dy), lddy,
            static_cast<const bf16*>(x), ldx, dw, dbias, n, h, wd, cin, cout, work);
  return launch_wgrad(g, as_stream(stream));
}

int unet_relu_bwd(void* d, int32_t ldd, const void* y, int32_t ldy, int64_t npix, int32_t ch,
                  void* stream) {
  if (!d || !y || ch % 8 || ldd % 8 || ldy % 8 || npix < 0)
    return fail(UNET_EINVAL, "relu_bwd: bad arguments");
  hipLaunchKernelGGL(relu_bwd_kernel, dim3(grid_for(npix * (ch / 8))), dim3(256), 0,
                     as_stream(stream), static_cast<bf16*>(d), ldd, static_cast<const bf16*>(y),
                     ldy, (long long)npix, ch / 8);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int unet_pool2_fwd(const void* x, int32_t ldx, void* y, int32_t ldy, int32_t n, int32_t h,
                   int32_t wd, int32_t ch, void* stream) {
  if (!x || !y || h % 2 || wd % 2 || ch % 8 || ldx % 8 || ldy % 8 || n <= 0)
    return fail(UNET_EINVAL, "pool2_fwd: bad arguments");
  const long long total = (long long)n * (h / 2) * (wd / 2) * (ch / 8);
  hipLaunchKernelGGL(pool2_fwd_kernel, dim3(grid_for(total)), dim3(256), 0, as_stream(stream),
                     static_cast<const bf16*>(x), ldx, static_cast<bf16*>(y), ldy, n, h, wd,
                     ch / 8);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int unet_pool2_bwd(const void* dy, int32_t lddy, const void* add, int32_t ldadd, void* dx,
                   int32_t lddx, int32_t n, int32_t h, int32_t wd, int32_t ch, void* stream) {
  if (!dy || !dx || h % 2 || wd % 2 || ch % 8 || lddy % 8 || lddx % 8 || n <= 0 ||
      (add && ldadd % 8))
    return fail(UNET_EINVAL, "pool2_bwd: bad arguments");
  const long long total = (long long)n * h * wd * (ch / 8);
  hipLaunchKernelGGL(pool2_bwd_kernel, dim3(grid_for(total)), dim3(256), 0, as_stream(stream),
                     static_cast<const bf16*>(dy), lddy, static_cast<const bf16*>(add), ldadd,
                     static_cast<bf16*>(dx), lddx, n, h, wd, ch / 8, (const bf16*)nullptr, 0);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int unet_up2_fwd(const void* x, int32_t ldx, void* y, int32_t ldy, int32_t n, int32_t h,
                 int32_t wd, int32_t ch, void* stream) {
  if (!x || !y || ch % 8 || ldx % 8 || ldy % 8 || n <= 0 || h <= 0 || wd <= 0)
    return fail(UNET_EINVAL, "up2_fwd: bad arguments");
  const long long total = (long long)n * 4 * h * wd * (ch / 8);
  hipLaunchKernelGGL(up2_fwd_kernel, dim3(grid_for(total)), dim3(256), 0, as_stream(stream),
                     static_cast<const bf16*>(x), ldx, static_cast<bf16*>(y), ldy, n, h, wd,
                     ch / 8);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int unet_up2_bwd(const void* dy, int32_t lddy, void* dx, int32_t lddx, int32_t n, int32_t h,
                 int32_t wd, int32_t ch, void* stream) {
  if (!dy || !dx || ch % 8 || lddy % 8 || lddx % 8 || n <= 0 || h <= 0 || wd <= 0)
    return fail(UNET_EINVAL, "up2_bwd: bad arguments");
  const long long total = (long long)n * h * wd * (ch / 8);
  hipLaunchKernelGGL(up2_bwd_kernel, dim3(grid_for(total)), dim3(256), 0, as_stream(stream),
                     static_cast<const bf16*>(dy), lddy, static_cast<bf16*>(dx), lddx, n, h, wd,
                     ch / 8, (const bf16*)nullptr, 0);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int64_t unet_loss_work_doubles(int64_t npix) {
  (void)npix;
  return 2 * kLossBlocks + 2;
}

int unet_mse_loss(const float* out, int32_t ldo, const float* target, const uint8_t* fluid,
                  int64_t npix, void* dout, double* loss, double* work, void* stream) {
  if (!out || !target || !fluid || !dout || !work || ldo < 3 || ldo % 8 || npix <= 0)
    return fail(UNET_EINVAL, "mse_loss: bad arguments");
  hipStream_t st = as_stream(stream);
  hipLaunchKernelGGL(loss_partial_kernel, dim3(kLossBlocks), dim3(256), 0, st, out, ldo, target,
                     fluid, (long long)npix, work);
  const long long vecs = npix * (ldo / 8);
  hipLaunchKernelGGL(loss_grad_kernel, dim3((unsigned)std::min<long long>((vecs + 255) / 256, 1024)),
                     dim3(256), 0, st, out, ldo, target, fluid, (long long)npix,
                     static_cast<bf16*>(dout), (const double*)work, work + 2 * kLossBlocks,
                     kLossBlocks);
  UCHECK(hipGetLastError());
  if (loss) {
    UCHECK(hipMemcpyAsync(loss, work + 2 * kLossBlocks, sizeof(double), hipMemcpyDeviceToHost,
                          st));
    UCHECK(hipStreamSynchronize(st));
  }
  return UNET_OK;
}

int unet_adam(float* p, float* m, float* v, const float* g, void* pb, int64_t count, double lr,
              double beta1, double beta2, double eps, int64_t t, void* stream) {
  if (!p || !m || !v || !g || count < 0 || t < 1) return fail(UNET_EINVAL, "adam: bad arguments");
  const double c1 = 1.0 / (1.0 - std::pow(beta1, (double)t));
  const double c2 = 1.0 / (1.0 - std::pow(beta2, (double)t));
  hipLaunchKernelGGL(adam_kernel, dim3(grid_for(count)), dim3(256), 0, as_stream(stream), p, m,
                     v, g, static_cast<bf16*>(pb), (long long)count, (float)lr, (float)beta1,
                     (float)beta2, (float)eps, (float)c1, (float)c2);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int unet_make_input(const uint8_t* solid, int32_t fine, const float* case_params, int32_t n,
                    int32_t res, void* x0, void* stream) {
  return launch_make_input(solid, fine, fine, case_params, 3, n, res, x0, stream);
}

int unet_fields_from_output(const float* out, int32_t ldo, int32_t n, int32_t res,
                            const float* case_params, const uint8_t* solid, int32_t fine,
                            float* rho, float* ux, float* uy, void* stream) {
  return launch_fields(out, ldo, n, res, case_params, 3, solid, fine, fine, rho, ux, uy, stream);
}

int unet_make_input_rect(const uint8_t* solid, int32_t nx, int32_t ny, const float* case_params,
                         int32_t n, int32_t res, void* x0, void* stream) {
  return launch_make_input(solid, nx, ny, case_params, 4, n, res, x0, stream);
}

int unet_fields_from_output_rect(const float* out, int32_t ldo, int32_t n, int32_t res,
                                 const float* case_params, const uint8_t* solid, int32_t nx,
                                 int32_t ny, float* rho, float* ux, float* uy, void* stream) {
  return launch_fields(out, ldo, n, res, case_params, 4, solid, nx, ny, rho, ux, uy, stream);
}

}  // extern "C"

// ===========================================================================
// The network
// ===========================================================================
namespace {

// Activation buffers (bf16 NHWC) and their channel counts.
enum Buf {
  B_X0, B_E0A, B_CAT0, B_P1, B_E1A, B_CAT1, B_P2, B_E2A, B_CAT2, B_P3, B_B3A, B_B3,
  B_D2A, B_D2, B_D1A, B_D1, B_D0A, B_D0, B_COUNT
};

struct BufInfo {
  int level, ch;
};
constexpr BufInfo kBuf[B_COUNT] = {
    {0, UNET_IN_CHANNELS}, {0, 32}, {0, 96}, {1, 32}, {1, 64}, {1, 192}, {2, 64}, {2, 128},
    {2, 384}, {3, 128}, {3, 256}, {3, 256}, {2, 128}, {2, 128}, {1, 64}, {1, 64}, {0, 32},
    {0, 32}};

struct Conv {
  int in, in_off, cin, out, out_off, cout, level, relu;   // out = -1: network output (FP32)
  long long w_off, b_off;
};

// Layer table: input buffer/channel offset, output buffer/channel offset.
const Conv kConvs[] = {
    {B_X0, 0, 32, B_E0A, 0, 32, 0, 1, 0, 0},   {B_E0A, 0, 32, B_CAT0, 64, 32, 0, 1, 0, 0},
    {B_P1, 0, 32, B_E1A, 0, 64, 1, 1, 0, 0},   {B_E1A, 0, 64, B_CAT1, 128, 64, 1, 1, 0, 0},
    {B_P2, 0, 64, B_E2A, 0, 128, 2, 1, 0, 0},  {B_E2A, 0, 128, B_CAT2, 256, 128, 2, 1, 0, 0},
    {B_P3, 0, 128, B_B3A, 0, 256, 3, 1, 0, 0}, {B_B3A, 0, 256, B_B3, 0, 256, 3, 1, 0, 0},
    {B_CAT2, 0, 384, B_D2A, 0, 128, 2, 1, 0, 0}, {B_D2A, 0, 128, B_D2, 0, 128, 2, 1, 0, 0},
    {B_CAT1, 0, 192, B_D1A, 0, 64, 1, 1, 0, 0},  {B_D1A, 0, 64, B_D1, 0, 64, 1, 1, 0, 0},
    {B_CAT0, 0, 96, B_D0A, 0, 32, 0, 1, 0, 0},   {B_D0A, 0, 32, B_D0, 0, 32, 0, 1, 0, 0},
    {B_D0, 0, 32, -1, 0, UNET_OUT_CHANNELS, 0, 0, 0, 0}};
constexpr int kNumConvs = sizeof(kConvs) / sizeof(kConvs[0]);

}  // namespace

struct unet {
  int max_batch = 0, res = 0;
  hipStream_t stream = nullptr;
  std::vector<Conv> convs;
  long long nparams = 0;
  float* p = nullptr;    // FP32 master parameters
  bf16* pb = nullptr;    // bf16 copy (weights used by the kernels)
  float* grad = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  long long t = 0;       // Adam steps taken
  bf16* act[B_COUNT] = {};
  bf16* gact[B_COUNT] = {};
  float* out = nullptr;  // FP32 network output (training)
  bf16* gout = nullptr;  // bf16 gradient of the output
  bf16* wt = nullptr;    // flipped, transposed weights (input gradients), kept with pb
  bf16* wf = nullptr;    // pb and wt in fragment order (fragment_layer), kept with pb
  bf16* wtf = nullptr;
  float* wwork = nullptr;
  double* lwork = nullptr;
  double* host_loss = nullptr;       // pinned; valid when loss_done has passed
  hipEvent_t loss_done = nullptr;
};

namespace {

int side(const unet* net, int level) { return net->res >> level; }

long long npix(const unet* net, int level, int n) {
  const long long s = side(net, level);
  return (long long)n * s * s;
}

int forward_impl(unet* net, const bf16* x0, int n, float* out) {
  hipStream_t st = net->stream;
  net->act[B_X0] = const_cast<bf16*>(x0);
  // pool: buffer that receives the 2x2 means of the output, or -1; up: the
  // output goes upsampled into the finer level's buffer c.out names
  auto conv = [&](int k, int pool = -1, int up = -1) -> int {
    const Conv& c = net->convs[k];
    const int s = side(net, c.level);
    ConvArgs a{};
    a.x = net->act[c.in] + c.in_off;
    a.ldx = kBuf[c.in].ch;
    a.w = net->pb + c.w_off;
    if (fragment_layer(c.cin, c.cout)) a.wf = net->wf + c.w_off;
    a.bias = net->p + c.b_off;
    if (c.out < 0) {
      a.y = out;
      a.ldy = UNET_OUT_CHANNELS;
      a.out_f32 = 1;
    } else if (up >= 0) {
      a.y = net->act[up];
      a.ldy = kBuf[up].ch;
      a.up = 1;
    } else {
      a.y = net->act[c.out] + c.out_off;
      a.ldy = kBuf[c.out].ch;
    }
    if (pool >= 0) {
      a.pool = net->act[pool];
      a.ldpool = kBuf[pool].ch;
    }
    a.npix = n * s * s;
    a.h = s;
    a.wd = s;
    a.cin = c.cin;
    a.cout = c.cout;
    a.relu = c.relu;
    return launch_conv(a, st);
  };
  int rc;
  if ((rc = conv(0)) || (rc = conv(1, B_P1)) || (rc = conv(2)) || (rc = conv(3, B_P2)) ||
      (rc = conv(4)) || (rc = conv(5, B_P3)) || (rc = conv(6)) || (rc = conv(7, -1, B_CAT2)) ||
      (rc = conv(8)) || (rc = conv(9, -1, B_CAT1)) || (rc = conv(10)) ||
      (rc = conv(11, -1, B_CAT0)) || (rc = conv(12)) || (rc = conv(13)) || (rc = conv(14)))
    return rc;
  return UNET_OK;
}

// Pixel tiles per block of the grouped weight gradients: four rounds of
// blocks if the batch is small, at most 12 (the partial sums stay a small
// part of the traffic and the last round short).
int wgrad_per_block(int res, int n) {
  long long tiles = 0;
  for (const Conv& c : kConvs) {
    const int s = res >> c.level;
    tiles += (long long)wgrad_tiles(n, s, s).units * (c.cin / 32) * (c.cout / 32);
  }
  return (int)std::min<long long>(std::max<long long>(tiles / 1024, 1), 12);
}

// Input gradient of conv k given the gradient of its (pre-activation) output,
// masked by the ReLU of the input buffer (relu), or left as it is where the
// buffer has none or receives further gradients; the weight gradient joins
// the group.
int conv_backward(unet* net, int k, int n, const bf16* dy, int lddy, bool need_dx, bool relu,
                  WgradGroup& g, long long& used, int per_block) {
  const Conv& c = net->convs[k];
  const int s = side(net, c.level);
  used += add_wgrad(g, wgrad_plan(n, s, s, c.cin, c.cout, per_block), dy, lddy,
                    net->act[c.in] + c.in_off, kBuf[c.in].ch, net->grad + c.w_off,
                    net->grad + c.b_off, n, s, s, c.cin, c.cout, net->wwork + used);
  if (!need_dx) return UNET_OK;
  ConvArgs a{};
  a.x = dy;
  a.ldx = lddy;
  a.w = net->wt + c.w_off;
  if (fragment_layer(c.cin, c.cout)) a.wf = net->wtf + c.w_off;
  a.y = net->gact[c.in] + c.in_off;
  a.ldy = kBuf[c.in].ch;
  a.npix = n * s * s;
  a.h = s;
  a.wd = s;
  a.cin = c.cout;
  a.cout = c.cin;
  if (relu) {
    a.mask = net->act[c.in] + c.in_off;
    a.ldmask = kBuf[c.in].ch;
  }
  return launch_conv(a, net->stream);
}

// Flipped weights of every layer whose input gradient is needed (all but the
// first) and the weights in fragment order, after each change of pb: two
// launches.
int lay_out_weights(unet* net) {
  static_assert(kNumConvs <= kMaxFlip, "flip table");
  FlipArgs f{};
  f.w = net->pb;
  f.wt = net->wt;
  int tiles = 0;
  for (int k = 1; k < kNumConvs; ++k) {
    const Conv& c = net->convs[k];
    auto& l = f.l[f.layers++];
    l.off = c.w_off;
    l.cin = c.cin;
    l.cout = c.cout;
    l.first = tiles;
    tiles += flip_tiles(c.cin, c.cout);
  }
  hipLaunchKernelGGL(flip_tiles_kernel, dim3(tiles), dim3(256), 0, net->stream, f);
  static_assert(2 * kNumConvs <= kMaxFragment, "fragment table");
  FragmentArgs g{};
  int blocks = 0;
  for (int k = 0; k < kNumConvs; ++k) {
    const Conv& c = net->convs[k];
    if (!fragment_layer(c.cin, c.cout)) continue;
    for (int dx = 0; dx < (k ? 2 : 1); ++dx) {
      auto& l = g.l[g.layers++];
      l.src = (dx ? net->wt : net->pb) + c.w_off;
      l.dst = (dx ? net->wtf : net->wf) + c.w_off;
      l.k = 9 * (dx ? c.cout : c.cin);
      l.first = blocks;
      blocks += 9 * c.cin * c.cout / (8 * 256);
    }
  }
  hipLaunchKernelGGL(fragment_kernel, dim3(blocks), dim3(256), 0, net->stream, g);
  UCHECK(hipGetLastError());
  return UNET_OK;
}

int backward_impl(unet* net, int n) {
  hipStream_t st = net->stream;
  int rc = UNET_OK;
  // the weight gradients of all layers run in one launch at the end (each
  // alone is a short launch with a ramp, a tail and a sum of its own)
  WgradGroup group{};
  static_assert(kNumConvs <= kMaxLayers, "group");
  long long used = 0;
  const int per_block = wgrad_per_block(net->res, n);
  auto conv = [&](int k, int buf, int off, bool need_dx, bool relu) {
    const bf16* dy = buf < 0 ? net->gout : net->gact[buf] + off;
    return conv_backward(net, k, n, dy, buf < 0 ? UNET_OUT_CHANNELS : kBuf[buf].ch, need_dx, relu,
                         group, used, per_block);
  };
  // gradient of an upsampled buffer (channels [0, ch) of the concatenation),
  // masked by its ReLU: the concatenation holds its values
  auto upb = [&](int fine_buf, int coarse_buf, int coarse_level, int ch) -> int {
    const int s = side(net, coarse_level), ldf = kBuf[fine_buf].ch;
    hipLaunchKernelGGL(up2_bwd_kernel, dim3(grid_for((long long)n * s * s * (ch / 8))), dim3(256),
                       0, st, net->gact[fine_buf], ldf, net->gact[coarse_buf],
                       kBuf[coarse_buf].ch, n, s, s, ch / 8, net->act[fine_buf], ldf);
    UCHECK(hipGetLastError());
    return UNET_OK;
  };
  // skip gradient (channels [off, ..) of the concatenation) plus the pooled
  // path, masked by the ReLU
  auto poolb = [&](int coarse_buf, int fine_buf, int off, int fine_level, int ch) -> int {
    const int s = side(net, fine_level), ldf = kBuf[fine_buf].ch;
    bf16* g = net->gact[fine_buf] + off;
    hipLaunchKernelGGL(pool2_bwd_kernel, dim3(grid_for((long long)n * s * s * (ch / 8))),
                       dim3(256), 0, st, net->gact[coarse_buf], kBuf[coarse_buf].ch, g, ldf, g,
                       ldf, n, s, s, ch / 8, net->act[fine_buf] + off, ldf);
    UCHECK(hipGetLastError());
    return UNET_OK;
  };
  // output layer (linear), then the decoder upwards: per level the two
  // convolutions, then the upsampled half of the concatenation
  if ((rc = conv(14, -1, 0, true, true)) || (rc = conv(13, B_D0, 0, true, true)) ||
      (rc = conv(12, B_D0A, 0, true, false)) || (rc = upb(B_CAT0, B_D1, 1, 64)) ||
      (rc = conv(11, B_D1, 0, true, true)) || (rc = conv(10, B_D1A, 0, true, false)) ||
      (rc = upb(B_CAT1, B_D2, 2, 128)) || (rc = conv(9, B_D2, 0, true, true)) ||
      (rc = conv(8, B_D2A, 0, true, false)) || (rc = upb(B_CAT2, B_B3, 3, 256)))
    return rc;
  // bottom, then the encoder
  if ((rc = conv(7, B_B3, 0, true, true)) || (rc = conv(6, B_B3A, 0, true, false)) ||
      (rc = poolb(B_P3, B_CAT2, 256, 2, 128)) || (rc = conv(5, B_CAT2, 256, true, true)) ||
      (rc = conv(4, B_E2A, 0, true, false)) || (rc = poolb(B_P2, B_CAT1, 128, 1, 64)) ||
      (rc = conv(3, B_CAT1, 128, true, true)) || (rc = conv(2, B_E1A, 0, true, false)) ||
      (rc = poolb(B_P1, B_CAT0, 64, 0, 32)) || (rc = conv(1, B_CAT0, 64, true, true)) ||
      (rc = conv(0, B_E0A, 0, false, false)))
    return rc;
  return launch_wgrad(group, st);
}

uint64_t splitmix_next(uint64_t& s) {
  s += 0x9E3779B97F4A7C15ULL;
  uint64_t z = s;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

double splitmix_uniform(uint64_t& s) { return (splitmix_next(s) >> 11) * (1.0 / 9007199254740992.0); }

void free_net(unet* net) {
  void* ptrs[] = {net->p, net->pb, net->grad, net->m, net->v, net->out, net->gout, net->wt, net->wf,
                  net->wtf,
                  net->wwork, net->lwork};
  for (void* q : ptrs) (void)hipFree(q);
  (void)hipHostFree(net->host_loss);
  if (net->loss_done) (void)hipEventDestroy(net->loss_done);
  for (int b = 1; b < B_COUNT; ++b) (void)hipFree(net->act[b]);
  for (int b = 0; b < B_COUNT; ++b) (void)hipFree(net->gact[b]);
  delete net;
}

}  // namespace

extern "C" {

int unet_create(int32_t max_batch, int32_t res, uint64_t seed, unet** out) {
  if (!out) return fail(UNET_EINVAL, "null output pointer");
  *out = nullptr;
  if (max_batch <= 0 || res < 8 || res % 8) return fail(UNET_EINVAL, "res must be a multiple of 8");
  unet* net = new (std::nothrow) unet();
  if (!net) return fail(UNET_ENOMEM, "host allocation failed");
  net->max_batch = max_batch;
  net->res = res;
  long long off = 0;
  long long wwork_max = 0;
  for (int k = 0; k < kNumConvs; ++k) {
    Conv c = kConvs[k];
    c.w_off = off;
    off += 9LL * c.cin * c.cout;
    c.b_off = off;
    off += c.cout;
    net->convs.push_back(c);
  }
  net->nparams = off;
  // the partial sums of all layers of one backward pass
  for (int nb = 1; nb <= max_batch; ++nb) {
    long long words = 0;
    for (const Conv& c : net->convs) {
      const int s = res >> c.level;
      const WgradPlan p = wgrad_plan(nb, s, s, c.cin, c.cout, wgrad_per_block(res, nb));
      words += p.splits * (9LL * c.cin * c.cout + c.cout);
    }
    wwork_max = std::max(wwork_max, words);
  }
  auto alloc = [&](void** p, size_t bytes) {
    return hipMalloc(p, bytes) == hipSuccess;
  };
  bool ok = alloc((void**)&net->p, sizeof(float) * off) && alloc((void**)&net->pb, 2 * off) &&
            alloc((void**)&net->grad, sizeof(float) * off) &&
            alloc((void**)&net->m, sizeof(float) * off) &&
            alloc((void**)&net->v, sizeof(float) * off) &&
            alloc((void**)&net->out, sizeof(float) * (size_t)max_batch * res * res * UNET_OUT_CHANNELS) &&
            alloc((void**)&net->gout, 2ULL * max_batch * res * res * UNET_OUT_CHANNELS) &&
            alloc((void**)&net->wt, 2 * off) && alloc((void**)&net->wf, 2 * off) &&
            alloc((void**)&net->wtf, 2 * off) &&
            alloc((void**)&net->wwork, sizeof(float) * wwork_max) &&
            alloc((void**)&net->lwork, sizeof(double) * unet_loss_work_doubles(0));
  for (int b = 0; ok && b < B_COUNT; ++b) {
    const long long s = res >> kBuf[b].level;
    const size_t bytes = 2ULL * max_batch * s * s * kBuf[b].ch;
    // (B_B3, B_D2 and B_D1 live upsampled in the concatenations only)
    if (b != B_X0 && b != B_B3 && b != B_D2 && b != B_D1) ok = alloc((void**)&net->act[b], bytes);
    if (ok) ok = alloc((void**)&net->gact[b], bytes);
  }
  ok = ok && hipHostMalloc((void**)&net->host_loss, sizeof(double)) == hipSuccess &&
       hipEventCreateWithFlags(&net->loss_done, hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    free_net(net);
    return fail(UNET_ENOMEM, "device allocation failed");
  }
  // He-normal weights (Box-Muller on a SplitMix64 stream), zero biases
  std::vector<float> h(off, 0.f);
  uint64_t st = seed;
  for (const Conv& c : net->convs) {
    const double sd = std::sqrt((c.relu ? 2.0 : 1.0) / (9.0 * c.cin));
    for (long long i = 0; i < 9LL * c.cin * c.cout; ++i) {
      const double u1 = std::max(splitmix_uniform(st), 1e-300), u2 = splitmix_uniform(st);
      h[c.w_off + i] = float(sd * std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2));
    }
  }
  *out = net;
  int rc = unet_set_params(net, h.data());
  if (rc) {
    free_net(net);
    *out = nullptr;
    return rc;
  }
  return UNET_OK;
}

void unet_destroy(unet* net) {
  if (!net) return;
  (void)hipStreamSynchronize(net->stream);
  free_net(net);
}

int unet_set_stream(unet* net, void* s) {
  if (!net) return fail(UNET_EINVAL, "null network");
  net->stream = as_stream(s);
  return UNET_OK;
}

int unet_num_params(unet* net, int64_t* count) {
  if (!net || !count) return fail(UNET_EINVAL, "null argument");
  *count = net->nparams;
  return UNET_OK;
}

int unet_get_params(unet* net, float* host) {
  if (!net || !host) return fail(UNET_EINVAL, "null argument");
  UCHECK(hipStreamSynchronize(net->stream));
  UCHECK(hipMemcpy(host, net->p, sizeof(float) * net->nparams, hipMemcpyDeviceToHost));
  return UNET_OK;
}

int unet_set_params(unet* net, const float* host) {
  if (!net || !host) return fail(UNET_EINVAL, "null argument");
  UCHECK(hipStreamSynchronize(net->stream));
  UCHECK(hipMemcpy(net->p, host, sizeof(float) * net->nparams, hipMemcpyHostToDevice));
  UCHECK(hipMemset(net->m, 0, sizeof(float) * net->nparams));
  UCHECK(hipMemset(net->v, 0, sizeof(float) * net->nparams));
  net->t = 0;
  hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(net->nparams)), dim3(256), 0, net->stream,
                     net->p, net->pb, net->nparams);
  UCHECK(hipGetLastError());
  const int rc = lay_out_weights(net);
  if (rc) return rc;
  UCHECK(hipStreamSynchronize(net->stream));
  return UNET_OK;
}

int unet_get_grads(unet* net, float* host) {
  if (!net || !host) return fail(UNET_EINVAL, "null argument");
  UCHECK(hipStreamSynchronize(net->stream));
  UCHECK(hipMemcpy(host, net->grad, sizeof(float) * net->nparams, hipMemcpyDeviceToHost));
  return UNET_OK;
}

int unet_forward(unet* net, const void* x0, int32_t n, float* out) {
  if (!net || !x0 || !out) return fail(UNET_EINVAL, "null argument");
  if (n <= 0 || n > net->max_batch) return fail(UNET_EINVAL, "batch size outside [1, max_batch]");
  return forward_impl(net, static_cast<const bf16*>(x0), n, out);
}

int unet_backward(unet* net, const void* x0, const float* target, const uint8_t* fluid,
                  int32_t n, double* loss) {
  if (!net || !x0 || !target || !fluid) return fail(UNET_EINVAL, "null argument");
  if (n <= 0 || n > net->max_batch) return fail(UNET_EINVAL, "batch size outside [1, max_batch]");
  int rc = forward_impl(net, static_cast<const bf16*>(x0), n, net->out);
  if (rc) return rc;
  rc = unet_mse_loss(net->out, UNET_OUT_CHANNELS, target, fluid, (int64_t)n * net->res * net->res,
                     net->gout, nullptr, net->lwork, net->stream);
  if (rc) return rc;
  // the backward pass is queued before the host waits for the loss (waiting
  // first left the device idle for 40 us per pass)
  if (loss) {
    UCHECK(hipMemcpyAsync(net->host_loss, net->lwork + 2 * kLossBlocks, sizeof(double),
                          hipMemcpyDeviceToHost, net->stream));
    UCHECK(hipEventRecord(net->loss_done, net->stream));
  }
  rc = backward_impl(net, n);
  if (loss) {
    UCHECK(hipEventSynchronize(net->loss_done));
    *loss = *net->host_loss;
  }
  return rc;
}

int unet_train_step(unet* net, const void* x0, const float* target, const uint8_t* fluid,
                    int32_t n, double lr, double* loss) {
  int rc = unet_backward(net, x0, target, fluid, n, loss);
  if (rc) return rc;
  net->t += 1;
  rc = unet_adam(net->p, net->m, net->v, net->grad, net->pb, net->nparams, lr, 0.9, 0.999, 1e-8,
                 net->t, net->stream);
  return rc ? rc : lay_out_weights(net);
}

}  // extern "C"
