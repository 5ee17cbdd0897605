// V quantisation for the FP8 attention variant (gfx950).
//
// §3.4 quantises V on the GPU before attention on every step. Here every
// (batch, head, channel d) gets a power-of-two scale 2^e_d,
//     e_d = max(-127, min{e : amax_d * 2^-e <= 448}),
// amax_d = max |V[., d]| over the head's tokens, and every element is
// rounded to OCP E4M3 (round to nearest even): code = E4M3(V * 2^-e_d). The
// scaling is exact, so the codes are exactly the format's rounding of V / 2^e_d.
//
// Output layout (one 16 KB tile per block, the attention kernel's PV operand
// order): V8[b][h][j] is 128 rows (channel d) x 128 bytes (key position p);
// byte (d, p) is the code of channel d of the block's packed real key
//     kap(p) = 64 hb + 32 (t / 2) + 8 g + 4 (t % 2) + r,
//     p = 32 g + 16 hb + 4 t + r  (g, t in 0..3; hb in 0..1; r in 0..3),
// and 0 for positions past the block's real keys. Lane group g of the
// attention kernel holds the E4M3 probabilities of its S^T accumulators in
// exactly this order (byte 16 hb + 4 t + r of its 32-byte fp8 MFMA operand),
// and reads bytes 32 g .. 32 g + 31 of each channel row as the V^T operand,
// so the two meet without any shuffle.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "fva_common.h"
#include "fva_geometry.h"
#include "fva_internal.h"

namespace fva {
namespace {

__global__ void v8_clear_kernel(uint32_t* __restrict__ amax, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) amax[i] = 0u;
}

// amax over the tokens r0 .. r0 + 255 of one head: 16 lanes per 256-byte row, 16
// rows per step, all 16 steps' loads in flight (rows past the end re-read the
// last one), one atomic max per channel (non-negative floats order like their
// bit patterns).
constexpr int kAmaxRows = 256;

__device__ __forceinline__ void amax_rows(const uint16_t* __restrict__ Vh, int tokens, int64_t sn, int r0,
                                          uint32_t* __restrict__ amax, float (&red)[16][128]) {
  const int c = threadIdx.x & 15;
  const int rg = threadIdx.x >> 4;
  uint4 v[16];
#pragma unroll
  for (int s = 0; s < 16; ++s)
    v[s] = *reinterpret_cast<const uint4*>(Vh + (int64_t)min(r0 + 16 * s + rg, tokens - 1) * sn + 8 * c);
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = 0.f;
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const uint32_t w[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      m[2 * e] = fmaxf(m[2 * e], fabsf(bf16_lo(w[e])));
      m[2 * e + 1] = fmaxf(m[2 * e + 1], fabsf(bf16_hi(w[e])));
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rg][8 * c + e] = m[e];
  __syncthreads();
  if (threadIdx.x < 128) {
    float mx = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) mx = fmaxf(mx, red[g][threadIdx.x]);
    atomicMax(&amax[threadIdx.x], __float_as_uint(mx));
  }
}

// e_d from amax_d: amax = 1.f * 2^(E - 127) with biased exponent E and
// fraction f; amax * 2^-e <= 448 = 1.75 * 2^8 first holds at
// e = E - 135 when 1.f <= 1.75, at e = E - 134 otherwise. Zero and
// subnormal amax (and anything below) give the floor -127.
__device__ __forceinline__ int v8_exponent(uint32_t amax_bits) {
  const int E = (int)((amax_bits >> 23) & 255u);
  const uint32_t f = amax_bits & 0x7FFFFFu;
  const int e = E - 135 + (f > 0x600000u ? 1 : 0);
  return E == 0 ? -127 : (e < -127 ? -127 : e);
}

// One block of one head, 256 threads. Four keys that are neighbours in the tile's
// order (kap = 4x .. 4x + 3) are one 32-bit word of a channel's row, so a thread
// takes the same eight channels of four such rows and converts them to eight
// words without any transposition; the words meet in LDS, where a channel's
// 128 bytes become whole, and go out as 16-byte stores, 4 KB per instruction.
// LDS: channel d at row d ^ (d / 64), its 16-byte chunk q at q ^ (d / 8) % 8: a
// wave writes one word of sixteen channels 8 apart and of one chunk's four
// words, all in distinct banks.
__device__ __forceinline__ void quantize_block(const uint16_t* __restrict__ Vh, int64_t sn, const Geometry& g, int j,
                                               const uint32_t* __restrict__ amax, uint8_t* __restrict__ tile,
                                               int32_t* __restrict__ vexp, uint32_t (&words)[128 * 32]) {
  const BlockBox box = block_box(g, j);
  const int c = threadIdx.x & 15;            // channels 8c .. 8c + 7
  const int t = (threadIdx.x >> 4) & 3;      // word of the chunk
  const int wave = threadIdx.x >> 6;
  uint4 v[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = wave + 4 * i;  // chunk 2g + hb
    const int kap0 = 64 * (q & 1) + 32 * (t >> 1) + 8 * (q >> 1) + 4 * (t & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // rows past the block re-read its last one and count as zero below
      const int row = min(kap0 + r, box.n - 1);
      v[i][r] = *reinterpret_cast<const uint4*>(Vh + (int64_t)box_token(g, box, row) * sn + 8 * c);
      if (kap0 + r >= box.n) v[i][r] = make_uint4(0, 0, 0, 0);
    }
  }
  // 2^-e of the eight channels as floats: e in [-127, 120] keeps the biased
  // exponent in [7, 254]
  float inv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) inv[e] = __uint_as_float((uint32_t)(127 - v8_exponent(amax[8 * c + e])) << 23);
  if (j == 0 && threadIdx.x < 128) vexp[threadIdx.x] = v8_exponent(amax[threadIdx.x]);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = wave + 4 * i;
    const uint32_t w[4][4] = {{v[i][0].x, v[i][0].y, v[i][0].z, v[i][0].w},
                              {v[i][1].x, v[i][1].y, v[i][1].z, v[i][1].w},
                              {v[i][2].x, v[i][2].y, v[i][2].z, v[i][2].w},
                              {v[i][3].x, v[i][3].y, v[i][3].z, v[i][3].w}};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = ((e & 1) ? bf16_hi(w[r][e >> 1]) : bf16_lo(w[r][e >> 1])) * inv[e];
      int o = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false);
      o = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], o, true);
      const int d = 8 * c + e;
      words[(d ^ (d >> 6)) * 32 + 4 * (q ^ (c & 7)) + t] = (uint32_t)o;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int o = threadIdx.x + 256 * k;  // 16-byte piece of the tile
    const int d = o >> 3, q = o & 7;
    const uint4 piece = *reinterpret_cast<const uint4*>(&words[(d ^ (d >> 6)) * 32 + 4 * (q ^ ((d >> 3) & 7))]);
    *reinterpret_cast<uint4*>(tile + 16 * o) = piece;
  }
}

// One pass of the quantisation: the amax of n_amax heads from a0 on, and the
// tiles of n_quant heads from q0 on, whose amax the launch before has finished.
// V is read twice, 774 MB each time at 720p; heads go through in groups small
// enough (kGroupBytes of V) that the second reading finds them in the 256 MB
// last-level cache, and one launch holds the second reading of a group and the
// first of the next, so that the memory is busy with both. Workgroups are dealt
// out in turns of the two kinds. With a pass for each kind, the tiles built by
// 16-bit column reads of a staged block: 418 us (amax 152, tiles 272).
__global__ __launch_bounds__(256) void v8_pass_kernel(const uint16_t* __restrict__ V, int heads, int tokens, int64_t sb,
                                                      int64_t sh, int64_t sn, Geometry g, int a0, int n_amax, int q0,
                                                      int n_quant, uint32_t* __restrict__ amax,
                                                      uint8_t* __restrict__ V8, int32_t* __restrict__ vexp) {
  __shared__ __align__(16) union {
    float red[16][128];
    uint32_t words[128 * 32];
  } lds;
  const int na = n_amax * ((tokens + kAmaxRows - 1) / kAmaxRows);
  const int nq = n_quant * g.nb;
  // workgroup b does amax item k exactly when floor((b + 1) na / (na + nq)) > k = floor(b na / (na + nq))
  const int64_t n = (int64_t)na + nq;
  const int before = (int)((int64_t)blockIdx.x * na / n);
  const bool is_amax = (int)(((int64_t)blockIdx.x + 1) * na / n) > before;
  const int item = is_amax ? before : (int)blockIdx.x - before;
  const int per = is_amax ? (tokens + kAmaxRows - 1) / kAmaxRows : g.nb;
  const int bh = (is_amax ? a0 : q0) + item / per;
  const int k = item % per;
  const int b = bh / heads;
  const int h = bh - b * heads;
  const uint16_t* Vh = V + (int64_t)b * sb + (int64_t)h * sh;
  uint32_t* am = amax + (int64_t)bh * 128;
  if (is_amax)
    amax_rows(Vh, tokens, sn, k * kAmaxRows, am, lds.red);
  else
    quantize_block(Vh, sn, g, k, am, V8 + ((int64_t)bh * g.nb + k) * kV8TileBytes, vexp + (int64_t)bh * 128,
                   lds.words);
}

// V bytes of a group of heads. fva_quantize_v at 40 heads of 720p (19 MB a head) /
// the long clip (29 MB) / 480p (8 MB): 366 / 519 / 175 us in one group, 348 /
// 500 / 166 at 100 MB, 357 / 548 / 159 at 80 MB (two heads of the long clip: too
// little for a launch), 386 / 545 / 166 at 160 MB (V and the tiles no longer
// fit the cache together). The two readings and the writing go through the
// fabric at 5.7 TB/s at 720p.
constexpr int64_t kGroupBytes = (int64_t)100 << 20;

}  // namespace

size_t quantize_v_workspace_bytes(int batch, int heads) {
  return (((size_t)batch * heads * 128 * 4) + 255) & ~(size_t)255;
}

hipError_t launch_quantize_v(const QuantizeArgs& a) {
  (void)hipGetLastError();
  const Geometry g = make_geometry(a.T, a.H, a.W, a.bt, a.bh, a.bw);
  const int nbh = a.batch * a.heads;
  if (nbh == 0) return hipSuccess;
  uint32_t* amax = static_cast<uint32_t*>(a.workspace);
  const int n = nbh * 128;
  const uint16_t* V = static_cast<const uint16_t*>(a.V);
  v8_clear_kernel<<<(n + 255) / 256, 256, 0, a.stream>>>(amax, n);
  const int group = (int)std::max<int64_t>(1, std::min<int64_t>(nbh, kGroupBytes / ((int64_t)a.tokens * kHeadDim * 2)));
  const int per_head = (a.tokens + kAmaxRows - 1) / kAmaxRows;
  for (int q0 = -group; q0 < nbh; q0 += group) {
    const int a0 = q0 + group;
    const int n_amax = std::max(0, std::min(group, nbh - a0));
    const int n_quant = q0 < 0 ? 0 : std::min(group, nbh - q0);
    const int64_t n = (int64_t)n_amax * per_head + (int64_t)n_quant * g.nb;
    v8_pass_kernel<<<(unsigned)n, 256, 0, a.stream>>>(V, a.heads, a.tokens, a.stride_b, a.stride_h, a.stride_n, g, a0,
                                                      n_amax, q0, n_quant, amax, a.V8, a.vexp);
  }
  return hipGetLastError();
}

}  // namespace fva
