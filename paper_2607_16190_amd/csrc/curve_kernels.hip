// Hilbert-curve token order and row permutation (gfx950).
//
// §3.1 (routing frontend) reorders blocks along a Hilbert curve so that
// tokens close in the latent video fall into nearby blocks at every scale.
// Here the tokens of the T x H x W grid are ranked along J. Skilling's 3D
// Hilbert curve ("Programming the Hilbert curve", AIP Conf. Proc. 707, 2004)
// on the cube of side 2^k >= max(T, H, W), with (t, y, x) as the curve's
// axes 0, 1, 2 (axis 0 the most significant bit of each 3-bit digit).
// Cutting the ranked sequence into runs of B tokens gives blocks that are all
// full except the last; the routing and attention kernels then run unchanged
// on the permuted rows with the one-dimensional tiling {1, 1, N, 1, 1, B}.
//
// The rank of a token is the number of grid points with a smaller curve
// index. The curve passes a cube's eight octants one after the other, so that
// number is, over the levels of the octree, the grid points in the octants of
// the token's cube that come before its own: boxes clipped by the grid, whose
// sizes are products. Every thread ranks its token by itself, in one launch;
// with a bitmap of the marked indices, its popcount prefix and a rank pass (four
// launches, one of them a single workgroup) fva_curve_order took 79 us at 720p
// and 22 us at 480p; this way 10 us either way, 4 of them the kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fva_internal.h"

namespace fva {
namespace {

constexpr int kRowsPerThread = 4;

// Rank of the token with coordinates (a0, a1, a2) among the points of the grid
// e0 x e1 x e2, `bits` levels. Skilling's transform, top level first: a set bit
// on axis i inverts the lower bits of axis 0, a clear one exchanges the lower
// bits of axes 0 and i. Carried down the levels that is a permutation of the
// axes (here of their records: coordinate, extent) and a flip of each. The
// level's three bits, Gray-encoded and flipped by the parity `fix` of the levels
// above, are the digit of the curve index, most significant first: where a digit
// bit is set, the half in which it is clear comes before the token.
__device__ __forceinline__ int curve_rank(int a0, int a1, int a2, int e0, int e1, int e2, int bits) {
  int n[3] = {a0, a1, a2};
  int ext[3] = {e0, e1, e2};
  uint32_t flip[3] = {0u, 0u, 0u};
  uint32_t fix = 0u;
  int rank = 0;
  for (int q = bits - 1; q >= 0; --q) {
    const int s = 1 << q;
    uint32_t b[3];
    int mine[3], other[3];  // grid points of the axis in the token's half of the cube and in the other
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int org = n[i] & ~(2 * s - 1);
      const int lo = min(ext[i] - org, s);  // (the token's cube starts inside the grid)
      const int hi = min(max(ext[i] - org - s, 0), s);
      const uint32_t o = (uint32_t)(n[i] >> q) & 1u;
      mine[i] = o ? hi : lo;
      other[i] = o ? lo : hi;
      b[i] = o ^ flip[i];
    }
    const uint32_t g0 = b[0], g1 = g0 ^ b[1], g2 = g1 ^ b[2];
    const int last2 = mine[2] + other[2];
    rank += (g0 ^ fix) ? other[0] * (mine[1] + other[1]) * last2 : 0;
    rank += (g1 ^ fix) ? mine[0] * other[1] * last2 : 0;
    rank += (g2 ^ fix) ? mine[0] * mine[1] * other[2] : 0;
    fix ^= g2;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (b[i]) {
        flip[0] ^= 1u;
      } else if (i > 0) {
        const int tn = n[0], te = ext[0];
        const uint32_t tf = flip[0];
        n[0] = n[i];
        n[i] = tn;
        ext[0] = ext[i];
        ext[i] = te;
        flip[0] = flip[i];
        flip[i] = tf;
      }
    }
  }
  return rank;
}

__global__ __launch_bounds__(256) void curve_order_kernel(int T, int H, int W, int bits, int32_t* __restrict__ perm) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  const int HW = H * W;
  if (n >= T * HW) return;
  const int t = n / HW;
  const int rem = n - t * HW;
  const int y = rem / W;
  const int x = rem - y * W;
  perm[curve_rank(t, y, x, T, H, W, bits)] = n;
}

// Row permutation of a [batch, heads, tokens, 128] bf16 tensor: 16 lanes
// move one 256-byte row as 16-byte pieces; each thread moves kRowsPerThread
// rows, all loads issued before the stores. TO_CURVE gathers
// dst[r] = src[perm[r]], FROM_CURVE scatters dst[perm[r]] = src[r]; a perm
// entry outside [0, tokens) zeroes the gathered row or drops the scattered one.
__global__ __launch_bounds__(256) void permute_rows_kernel(const uint16_t* __restrict__ src,
                                                           uint16_t* __restrict__ dst, int heads, int tokens,
                                                           int64_t sb, int64_t sh, int64_t sn,
                                                           const int32_t* __restrict__ perm, int direction) {
  const int bh = blockIdx.y;
  const int b = bh / heads;
  const int h = bh - b * heads;
  const int64_t base = (int64_t)b * sb + (int64_t)h * sh + (threadIdx.x & 15) * 8;
  const int r0 = blockIdx.x * (16 * kRowsPerThread) + (threadIdx.x >> 4);
  uint4 v[kRowsPerThread];
  int to[kRowsPerThread];
#pragma unroll
  for (int u = 0; u < kRowsPerThread; ++u) {
    const int r = r0 + 16 * u;
    int from = -1;
    to[u] = -1;
    if (r < tokens) {
      const int p = perm[r];
      const bool ok = p >= 0 && p < tokens;
      from = direction == 0 ? (ok ? p : -1) : r;
      to[u] = direction == 0 ? r : (ok ? p : -1);
    }
    v[u] = from >= 0 ? *reinterpret_cast<const uint4*>(src + base + (int64_t)from * sn) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < kRowsPerThread; ++u)
    if (to[u] >= 0) *reinterpret_cast<uint4*>(dst + base + (int64_t)to[u] * sn) = v[u];
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

int bits_for(int T, int H, int W) {
  int m = T > H ? T : H;
  m = m > W ? m : W;
  int k = 0;
  while ((1 << k) < m) ++k;
  return k;
}

int bitmap_words(int bits) {
  const int64_t cells = (int64_t)1 << (3 * bits);
  return (int)(cells >= 32 ? cells / 32 : 1);
}

}  // namespace

size_t curve_workspace_bytes(int T, int H, int W) {
  const int words = bitmap_words(bits_for(T, H, W));
  const int64_t N = (int64_t)T * H * W;
  return al256((size_t)words * 4) * 2 + al256((size_t)N * 4);
}

// (The workspace is part of the interface and checked there; the ranks need none.)
hipError_t launch_curve_order(int T, int H, int W, int32_t* perm, void* workspace, hipStream_t stream) {
  (void)workspace;
  const int N = T * H * W;
  curve_order_kernel<<<(N + 255) / 256, 256, 0, stream>>>(T, H, W, bits_for(T, H, W), perm);
  return hipGetLastError();
}

hipError_t launch_permute_rows(const void* src, void* dst, int batch, int heads, int tokens, int64_t sb, int64_t sh,
                               int64_t sn, const int32_t* perm, int direction, hipStream_t stream) {
  if (batch * heads == 0) return hipSuccess;
  const dim3 grid((tokens + 16 * kRowsPerThread - 1) / (16 * kRowsPerThread), batch * heads);
  permute_rows_kernel<<<grid, 256, 0, stream>>>(static_cast<const uint16_t*>(src), static_cast<uint16_t*>(dst), heads,
                                                tokens, sb, sh, sn, perm, direction);
  return hipGetLastError();
}

}  // namespace fva
