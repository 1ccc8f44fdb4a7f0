// Pressure-Poisson apply on uniform, lexicographically numbered 3D meshes in
// one kernel, with no shared-node slots and no combine pass.
//
// Bound: FP64 issue.  A wave64 FP64 instruction takes 2.2 to 2.4 ns of its
// SIMD under load (measured; the clock falls to about 2 GHz), a leaf layer
// about 130 of them, and at 128^3 the tiles evaluate 1.43 times the leaves
// (their rims and the layer below each chunk), which costs less than the
// second kernel that would complete shared nodes.  FP64 apply, bricks with
// slots and combine before -> this kernel: 128^3 39.4 -> 22.1 us, 256^3
// 295 -> 175 us, 16^3 12.1 -> 8.5 us (two launches -> one).  Measured and not
// taken: the hand-over of the corner sums delayed by one leaf layer (24.8
// against 23.5 us, the extra registers), four waves per SIMD (spills, 52 us).
#pragma once
#include "march.h"

namespace chns {

// A workgroup computes 17 x 15 columns of leaves (255 of its 256 lanes, one
// column per lane) and completes the 16 x 14 node columns inside them: the
// leaves on its lower rim are computed by the neighbouring tile as well.
// 17 leaves give 16 nodes, so tiles of x divide every 2^l + 1 grid with l >= 4
// (the last tile also owns the last node).
constexpr int kTileX = 16, kTileY = 14;  // nodes a tile owns
constexpr int kTileLX = kTileX + 1, kTileLY = kTileY + 1;  // its leaf columns

template <typename T>
struct TileArgs {
  const T* x;
  const T* phi;
  T* y;
  double ratio;        // rho-/rho+
  int joint;           // see march::pp_joint
  int side, level;     // leaves per edge, their level
  int tx, ty, nz, own;  // tiles, chunks of node layers and layers per chunk
  // damped-Jacobi sweep: y = x + sm_w sm_d (sm_r - A x); or the product
  const T* sm_r;
  const T* sm_d;
  T sm_w;
  double* partials;  // fused x.y partial per block, or null
  const int* done;
  int blocks() const { return tx * ty * nz; }
};

template <typename T>
void tile_geometry(TileArgs<T>& a, int side, int own) {
  a.side = side;
  a.tx = (side + kTileX - 1) / kTileX;
  a.ty = (side + kTileY - 1) / kTileY;
  a.own = own < 1 ? 1 : own;
  a.nz = (side + a.own) / a.own;  // ceil((side + 1) / own)
}

template <typename T, bool SM>
__global__ __launch_bounds__(256) void k_pp_tile(TileArgs<T> a) {
  // corner sums handed to the lane that owns the node, double-buffered; the
  // extra column and row stay zero
  constexpr int LS = kTileLX + 1;
  __shared__ T ex[2][3][(kTileLY + 1) * LS];
  __shared__ double sh[4];
  if (a.done && *a.done) return;
  const int l = threadIdx.x;
  for (int i = l; i < 2 * 3 * (kTileLY + 1) * LS; i += 256) (&ex[0][0][0])[i] = T(0);
  // contiguous tiles on one XCD (blocks are dealt to the 8 XCDs in turn)
  const uint32_t g = gridDim.x, b = blockIdx.x, per = g / 8, rem = g % 8, xc = b % 8;
  const uint32_t t = xc * per + (xc < rem ? xc : rem) + b / 8;
  const int tx = t % a.tx, ty = (t / a.tx) % a.ty, tz = t / (a.tx * a.ty);
  const int S = a.side, sy = S + 1;
  const int lx = l % kTileLX, ly = l / kTileLX;
  const int cx = kTileX * tx - 1 + lx, cy = kTileY * ty - 1 + ly;  // leaf column
  const bool leaf = cx >= 0 && cx < S && cy >= 0 && cy < S && ly < kTileLY;
  // the lane owns the node at its leaf's upper corner
  const bool owner = cx < S && cy < S && ly < kTileLY && (lx < kTileX || cx == S - 1) && (ly < kTileY || cy == S - 1);
  const int qx = min(max(cx, 0), S - 1), qy = min(max(cy, 0), S - 1);
  // byte offsets in a node layer (32 bits; the layer's address is uniform)
  const uint32_t i0 = (uint32_t)(qx + qy * sy) * sizeof(T), i1 = i0 + (uint32_t)sy * sizeof(T);
  const uint32_t io = (uint32_t)((cx + 1) + (cy + 1) * sy) * sizeof(T);
  auto at = [](const T* base, uint32_t off) -> const T& { return *(const T*)((const char*)base + off); };
  const int64_t sz = (int64_t)sy * sy;
  const int z0 = tz * a.own, z1 = min(z0 + a.own, S + 1);
  const int zb = max(z0 - 1, 0), ze = min(z1, S);
  T u[4], p[4];
  auto load = [&](int z) {
    const T* px = a.x + (int64_t)z * sz;
    const T* pp = a.phi + (int64_t)z * sz;
    u[0] = at(px, i0);
    u[1] = at(px + 1, i0);
    u[2] = at(px, i1);
    u[3] = at(px + 1, i1);
    p[0] = at(pp, i0);
    p[1] = at(pp + 1, i0);
    p[2] = at(pp, i1);
    p[3] = at(pp + 1, i1);
  };
  const int me = ly * LS + lx;
  double dot = 0.0;
  int buf = 0;
  // x, r and D^-1 at the owned node of layer z, for the sweep and the dot
  const bool need_x = SM || a.partials;
  T xo = T(0), rr = T(0), dd = T(0);
  auto load_own = [&](int z) {
    if (!owner || !need_x) return;
    xo = at(a.x + (int64_t)z * sz, io);
    if constexpr (SM) {
      rr = at(a.sm_r + (int64_t)z * sz, io);
      dd = at(a.sm_d + (int64_t)z * sz, io);
    }
  };
  auto emit = [&](int z, const T* r) {
    if (leaf) {
      ex[buf][0][me] = r[2];
      ex[buf][1][me] = r[1];
      ex[buf][2][me] = r[0];
    }
    __syncthreads();
    if (owner) {
      // corner 0 first, as the bricks' node sums
      const T s = ((ex[buf][2][me + LS + 1] + ex[buf][1][me + LS]) + ex[buf][0][me + 1]) + (leaf ? r[3] : T(0));
      const T o = SM ? xo + a.sm_w * dd * (rr - s) : s;
      *(T*)((char*)(a.y + (int64_t)z * sz) + io) = o;
      if (a.partials) dot += (double)xo * (double)o;
    }
    buf ^= 1;
  };
  const march::PpCoef<T> cf = march::pp_coef3<T>(a.ratio, a.level, a.joint != 0);
  march::PpMarch<T> M;
  T r[4];
  load(zb);
  M.start(u, p);
  load(zb + 1);
  __syncthreads();
  // the leaf layer below the chunk: only its upper half counts
  if (z0 > zb) M.step(u, p, cf, r, [&] { load(min(z0 + 1, S)); });
  // two leaf layers per trip: the loop-carried layer state then changes
  // registers without moves
  int z = z0;
  auto leaf_layer = [&]() {
    load_own(z);
    M.step(u, p, cf, r, [&] { load(min(z + 2, S)); });
    emit(z, r);
  };
  while (z < ze) {
    leaf_layer();
    if (++z >= ze) break;
    leaf_layer();
    ++z;
  }
  if (z1 == S + 1) {
    load_own(S);
    M.finish(r);
    emit(S, r);
  }
  if (a.partials) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o, 64);
    if ((l & 63) == 0) sh[l >> 6] = dot;
    __syncthreads();
    if (l == 0) a.partials[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  }
}

}  // namespace chns
