// Multi-grid (pyramid) passes of the two-level force (section 5.2,
// Algorithms 2 and 3).  REDUCE convolves with the 3-D B-spline of order 6
// (the tensor product of the 1-D weights C(6, k) / 64, k = 0..6) and keeps
// every second cell per axis; EXPAND is its transpose times 8, i.e. zeros
// inserted between cells and the same kernel times 2 per axis.  Boundaries
// wrap (one device holds the whole periodic mesh); coarse cell i sits on fine
// cell 2 i.  Every field is x-blocked by 8.
//
// One level is one launch: a workgroup stages its tile's cells and their halo
// in LDS, filters along z, then y, then x there, and stores runs of eight x.
// The fine field is read once (the halos from L2) and nothing is written in
// between.  As three one-axis passes per level, each a stream over its
// intermediate, REDUCE and EXPAND of a 512^3 force took 1268 and 1413 us, of
// its density 724.
#include "layout.h"
#include "pyramid.h"

namespace pmk {
namespace {

// consecutive tiles of one launch on one XCD (they share halos)
__device__ __forceinline__ int xcd_tile(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int xcd = b & 7, slot = b >> 3;
  return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

// Tile (tx, ty, tz) of a cube, tiles XB blocks wide along x, along the Morton
// curve: neighbours in all three directions are staged soon after each other,
// while the halo they share is in L2.  XB = 2: the tiles (tx, y, z) of one
// half-resolution cube cell, y and z bits interleaved below the rest.
template <int XB>
__device__ __forceinline__ void tile_coords(int& tx, int& ty, int& tz) {
  const uint32_t t = (uint32_t)xcd_tile(blockIdx.x, gridDim.x), m = XB == 2 ? t >> 2 : t;
  auto compact = [](uint32_t v) {   // bit 3 i -> bit i
    v &= 0x09249249u;
    v = (v ^ (v >> 2)) & 0x030C30C3u;
    v = (v ^ (v >> 4)) & 0x0300F00Fu;
    v = (v ^ (v >> 8)) & 0xFF0000FFu;
    return (int)((v ^ (v >> 16)) & 0x000003FFu);
  };
  tx = compact(m);
  ty = compact(m >> 1);
  tz = compact(m >> 2);
  if (XB == 2) {
    ty = 2 * ty + (int)(t & 1);
    tz = 2 * tz + (int)(t >> 1 & 1);
  }
}

__device__ __forceinline__ long xoff(int x, int y, int z, int ny, int nz) {
  return ((((long)(x >> 3) * ny + y) * nz + z) << 3) + (x & 7);
}

// Four consecutive floats.  Only a caller's force checkpoint can lie off the
// 16-byte grid (al, uniform).
__device__ __forceinline__ float4 load4(const float* p, bool al) {
  return al ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ void store4(float* p, float4 v, bool al) {
  if (al) {
    *reinterpret_cast<float4*>(p) = v;
  } else {
    p[0] = v.x;
    p[1] = v.y;
    p[2] = v.z;
    p[3] = v.w;
  }
}
__device__ __forceinline__ bool aligned16(const PyrField& f) { return (reinterpret_cast<uintptr_t>(f.p[0]) & 15) == 0; }

// Writes a run of memory floats v of cells (dst block of eight x, channels in
// the field's order), combined with what is there as `mode` says.
__device__ __forceinline__ void combine4(float* d, float4 v, int mode, const float* aux, float alpha, bool al) {
  if (mode == PYR_ADD || mode == PYR_SUB) {
    const float4 w = load4(d, al);
    const float sg = mode == PYR_ADD ? 1.f : -1.f;
    v = make_float4(w.x + sg * v.x, w.y + sg * v.y, w.z + sg * v.z, w.w + sg * v.w);
  } else if (mode == PYR_COMBINE) {   // aux: the values of these four cells and channel
    v = make_float4(alpha * aux[0] - v.x, alpha * aux[3] - v.y, alpha * aux[6] - v.z, alpha * aux[9] - v.w);
  }
  store4(d, v, al);
}

// n outputs of a line of 2 n + 5 inputs: out(o) = sum_t C(6, t) / 64 in(2 o + t)
template <int N>
__device__ __forceinline__ void reduce_line(const float (&a)[2 * N + 5], float (&o)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    o[i] = (20.f / 64.f) * a[2 * i + 3] + (15.f / 64.f) * (a[2 * i + 2] + a[2 * i + 4]) +
           (6.f / 64.f) * (a[2 * i + 1] + a[2 * i + 5]) + (1.f / 64.f) * (a[2 * i] + a[2 * i + 6]);
}
// 2 n outputs of a line of n + 3 inputs (input 1 sits on output 0)
template <int N>
__device__ __forceinline__ void expand_line(const float (&a)[N + 3], float (&o)[2 * N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    o[2 * i] = (40.f / 64.f) * a[i + 1] + (12.f / 64.f) * (a[i] + a[i + 2]);
    o[2 * i + 1] = (30.f / 64.f) * (a[i + 1] + a[i + 2]) + (2.f / 64.f) * (a[i] + a[i + 3]);
  }
}

// Stages rows of cells in LDS: x in [xa, xa + NXG) with xa % 4 == 0 and NXG a
// multiple of 4, of which [X0, X0 + NX) are kept, y in [y0, y0 + NY), z in
// [z0, z0 + NZ), all wrapped, at ((c YS + y) NX + x) ZS + z.  Four cells of a
// block of eight x are one 16-byte access (three when interleaved); a thread
// keeps its x and z and walks y, so that the loop has no index arithmetic
// (cell by cell, with three divisions each, the staging took 520 us of a
// 512^3 level that moves 0.6 GB), and has all its loads in flight at once.
template <int CH, bool IL, int TH, int NXG, int X0, int NX, int NY, int NZ, int YS, int ZS>
__device__ __forceinline__ void stage(const PyrField& f, int xa, int y0, int z0, float* __restrict__ lds) {
  constexpr int Q = CH * NXG / 4, ROWS = TH / (Q * NZ), K = (NY + ROWS - 1) / ROWS;
  static_assert(ROWS >= 1, "a row of every z per pass");
  const int t = threadIdx.x, q = t % Q, z = t / Q % NZ, yy = t / (Q * NZ);
  if (yy < ROWS) {
    const bool al = aligned16(f);
    // four-cell group g of the row, sixteen-byte part of it, channel (separate fields)
    const int g = IL ? q / CH : q % (NXG / 4), part = IL ? q % CH : 0, ch = IL ? 0 : q / (NXG / 4);
    const int x = (xa + 4 * g) & (f.nx - 1), zz = (z0 + z) & (f.nz - 1);
    const float* src = f.p[0];
    if (CH > 1 && !IL) src = ch == 0 ? f.p[0] : (ch == 1 ? f.p[1] : f.p[2]);
    constexpr int C = IL ? CH : 1;   // floats per cell in memory
    src += ((long)(x >> 3) * f.ny * f.nz + zz) * (8 * C) + (x & 7) * C + 4 * part;
    const long sy = (long)f.nz * (8 * C);
    float4 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int y = yy + k * ROWS < NY ? yy + k * ROWS : NY - 1;   // past the end: the last row again
      v[k] = load4(src + ((y0 + y) & (f.ny - 1)) * sy, al);
    }
    int o[4];   // LDS slots in row y = 0; -1: not kept
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = 4 * part + j, xi = 4 * g + (IL ? e / CH : e) - X0, c = IL ? e % CH : ch;
      o[j] = xi >= 0 && xi < NX ? (c * YS * NX + xi) * ZS + z : -1;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int y = yy + k * ROWS;
      if (y < NY) {
        const float w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (o[j] >= 0) lds[o[j] + y * (NX * ZS)] = w[j];
      }
    }
  }
  __syncthreads();
}

// REDUCE of one level of one channel: tiles of 8^3 destination cells.  Lines
// are filtered in place (each by one thread), with a line stride of 21 words that
// keeps the lanes of a wave on different banks.  (Its rows of eight cells are
// 32 bytes: the lines of z of the three-channel kernel below would fetch them
// one by one, 191 us a level pair against 149.)
__global__ __launch_bounds__(256) void k_pyr_reduce1(PyrField src, PyrField dst, int mode) {
  constexpr int NX = 21, NZ = 21, NY = 21, TH = 256;
  __shared__ float lds[NY * NX * NZ];
  int tx, ty, tz;
  tile_coords<1>(tx, ty, tz);
  stage<1, false, TH, 24, 1, NX, NY, NZ, NY, NZ>(src, 16 * tx - 4, 16 * ty - 3, 16 * tz - 3, lds);
  for (int l = threadIdx.x; l < NY * NX; l += TH) {   // along z
    float a[21], o[8];
    float* p = lds + l * NZ;
#pragma unroll
    for (int i = 0; i < 21; ++i) a[i] = p[i];
    reduce_line<8>(a, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = o[i];
  }
  __syncthreads();
  for (int l = threadIdx.x; l < NX * 8; l += TH) {    // along y
    float a[NY], o[8];
    float* p = lds + (l >> 3) * NZ + (l & 7);
#pragma unroll
    for (int i = 0; i < NY; ++i) a[i] = p[i * NX * NZ];
    reduce_line<8>(a, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i * NX * NZ] = o[i];
  }
  __syncthreads();
  const bool al = aligned16(dst);
  for (int l = threadIdx.x; l < 64; l += TH) {         // along x, stored
    const int y = l >> 3, z = l & 7;
    float a[21], o[8];
#pragma unroll
    for (int i = 0; i < 21; ++i) a[i] = lds[(y * NX + i) * NZ + z];
    reduce_line<8>(a, o);
    float* d = dst.p[0] + xoff(8 * tx, 8 * ty + y, 8 * tz + z, dst.ny, dst.nz);
    combine4(d, make_float4(o[0], o[1], o[2], o[3]), mode, nullptr, 0.f, al);
    combine4(d + 4, make_float4(o[4], o[5], o[6], o[7]), mode, nullptr, 0.f, al);
  }
}

// REDUCE of one level of three channels: tiles of 8 XB x 8 x 8 destination cells.  A thread
// loads a whole line of 21 z, four floats wide, and filters it in registers,
// so that LDS holds only an eighth of the tile's cells (25 KB per channel at
// XB = 2) and the loads of two workgroups run beside each other.  What bounds
// it is the halo: 2.15 cells are fetched per cell at XB = 2, 2.58 at XB = 1.
// With the cells staged first (111 KB, one workgroup per CU, XB = 1) a 512^3
// level of three channels took 1064 us, 704 of them without its arithmetic.
template <bool SIL, bool DIL, int XB, int TH>
__global__ __launch_bounds__(TH) void k_pyr_reduce(PyrField src, PyrField dst, int mode,
                                                   const float* __restrict__ aux, float alpha) {
  constexpr int CH = 3, NX = 16 * XB + 5, NY = 21, ZS = 8;
  constexpr int G = (16 * XB + 8) / 4, Q = CH * G;   // four-cell groups of a row, 16-byte words of it
  static_assert(Q * NY <= TH, "one line per thread");
  __shared__ __align__(16) float lds[CH * NY * NX * ZS];
  int tx, ty, tz;
  tile_coords<XB>(tx, ty, tz);
  const int t = threadIdx.x, q = t % Q, y = t / Q;
  if (y < NY) {
    const bool al = aligned16(src);
    const int g = SIL ? q / CH : q % G, part = SIL ? q % CH : 0, ch = SIL ? 0 : q / G;
    constexpr int C = SIL ? CH : 1;   // floats per cell in memory
    const int x = (16 * XB * tx - 4 + 4 * g) & (src.nx - 1), yy = (16 * ty - 3 + y) & (src.ny - 1);
    const float* base = src.p[0];
    if (CH > 1 && !SIL) base = ch == 0 ? src.p[0] : (ch == 1 ? src.p[1] : src.p[2]);
    base += ((long)(x >> 3) * src.ny + yy) * src.nz * (8 * C) + (x & 7) * C + 4 * part;
    float4 v[21];
#pragma unroll
    for (int k = 0; k < 21; ++k) v[k] = load4(base + (long)((16 * tz - 3 + k) & (src.nz - 1)) * (8 * C), al);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = 4 * part + j, xi = 4 * g + (SIL ? e / CH : e) - 1, c = SIL ? e % CH : ch;
      float a[21], o[8];
#pragma unroll
      for (int k = 0; k < 21; ++k) a[k] = j == 0 ? v[k].x : (j == 1 ? v[k].y : (j == 2 ? v[k].z : v[k].w));
      reduce_line<8>(a, o);
      if (xi >= 0 && xi < NX) {
        float4* d = reinterpret_cast<float4*>(lds + ((c * NY + y) * NX + xi) * ZS);
        d[0] = make_float4(o[0], o[1], o[2], o[3]);
        d[1] = make_float4(o[4], o[5], o[6], o[7]);
      }
    }
  }
  __syncthreads();
  for (int l = t; l < CH * NX * 8; l += TH) {    // along y, in place
    float a[NY], o[8];
    float* p = lds + l / (NX * 8) * (NY * NX * ZS) + l % (NX * 8);
#pragma unroll
    for (int i = 0; i < NY; ++i) a[i] = p[i * NX * ZS];
    reduce_line<8>(a, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i * NX * ZS] = o[i];
  }
  __syncthreads();
  const bool al = aligned16(dst);
  for (int l = t; l < XB * 64; l += TH) {        // along x, stored
    const int b = l >> 6, yo = l >> 3 & 7, zo = l & 7;
    float o[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      float a[21];
#pragma unroll
      for (int i = 0; i < 21; ++i) a[i] = lds[((c * NY + yo) * NX + 16 * b + i) * ZS + zo];
      reduce_line<8>(a, o[c]);
    }
    const long e = xoff(8 * (XB * tx + b), 8 * ty + yo, 8 * tz + zo, dst.ny, dst.nz);
    if constexpr (DIL) {   // PYR_STORE, ADD or SUB
#pragma unroll
      for (int w = 0; w < CH * 2; ++w) {
        const int f = 4 * w;
        combine4(dst.p[0] + CH * e + f, make_float4(o[f % CH][f / CH], o[(f + 1) % CH][(f + 1) / CH],
                                                    o[(f + 2) % CH][(f + 2) / CH], o[(f + 3) % CH][(f + 3) / CH]),
                 mode, nullptr, 0.f, al);
      }
    } else {
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          combine4(dst.p[c] + e + 4 * h, make_float4(o[c][4 * h], o[c][4 * h + 1], o[c][4 * h + 2], o[c][4 * h + 3]),
                   mode, aux ? aux + 3 * (e + 4 * h) + c : nullptr, alpha, al);
    }
  }
}

// EXPAND of one level: tiles of 16^3 destination cells.  The outputs go
// through LDS once more, block of eight x by block, so that the stores (and
// the loads of a destination that is added to) are whole contiguous rows.
template <int CH, bool SIL, bool DIL, int TH>
__global__ __launch_bounds__(TH) void k_pyr_expand(PyrField src, PyrField dst, int mode) {
  constexpr int NX = 11, NY = 11, NZ = 11, ZS = 17;   // room for 16 outputs per line
  constexpr int LINES = CH * 16 * NX * ZS, OUT = 16 * 16 * 8 * CH;
  __shared__ __align__(16) float lds[LINES > OUT ? LINES : OUT];
  int tx, ty, tz;
  tile_coords<1>(tx, ty, tz);
  const bool al = aligned16(dst), add = mode == PYR_ADD || mode == PYR_SUB;
  constexpr int C = DIL ? CH : 1, ROW = 16 * 8 * C / 4;    // 16-byte words of a row (x block, y), 16 z
  constexpr int W = OUT / 4, K = (W + TH - 1) / TH;
  // word e of the tile's block b of eight x (separate fields: rows of channel e / (16 ROW))
  auto word = [&](int b, int e) {
    const int r = e / ROW, yy = r & 15, c = r >> 4;
    float* base = DIL || c == 0 ? dst.p[0] : (c == 1 ? dst.p[1] : dst.p[2]);
    return base + xoff(16 * tx + 8 * b, 16 * ty + yy, 16 * tz, dst.ny, dst.nz) * C + 4 * (e % ROW);
  };
  float4 old[2][K];   // what the outputs are added to, in flight beside the filters
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int e = (int)threadIdx.x + k * TH;
      old[b][k] = add ? load4(word(b, e < W ? e : W - 1), al) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  stage<CH, SIL, TH, 16, 3, NX, NY, NZ, 16, ZS>(src, 8 * tx - 4, 8 * ty - 1, 8 * tz - 1, lds);
  for (int l = threadIdx.x; l < CH * NY * NX; l += TH) {   // along z
    float a[11], o[16];
    float* p = lds + ((l / (NY * NX)) * 16 * NX + l % (NY * NX)) * ZS;
#pragma unroll
    for (int i = 0; i < 11; ++i) a[i] = p[i];
    expand_line<8>(a, o);
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = o[i];
  }
  __syncthreads();
  for (int l = threadIdx.x; l < CH * NX * 16; l += TH) {   // along y
    float a[11], o[16];
    float* p = lds + ((l / (NX * 16)) * 16 * NX + l / 16 % NX) * ZS + (l & 15);
#pragma unroll
    for (int i = 0; i < 11; ++i) a[i] = p[i * NX * ZS];
    expand_line<8>(a, o);
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i * NX * ZS] = o[i];
  }
  __syncthreads();
  const int y = threadIdx.x >> 4, z = threadIdx.x & 15;    // along x: 256 lines
  float o[CH][16];
  if (threadIdx.x < 256) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      float a[11];
#pragma unroll
      for (int i = 0; i < 11; ++i) a[i] = lds[((c * 16 + y) * NX + i) * ZS + z];
      expand_line<8>(a, o[c]);
    }
  }
  const float sg = mode == PYR_SUB ? -1.f : 1.f;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    __syncthreads();   // the lines, or the first block's outputs, are read
    if (threadIdx.x < 256) {
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          lds[DIL ? ((y * 16 + z) * 8 + i) * CH + c : ((c * 16 + y) * 16 + z) * 8 + i] = o[c][8 * b + i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int e = (int)threadIdx.x + k * TH;
      if (e < W) {
        const float4 v = reinterpret_cast<const float4*>(lds)[e], w = old[b][k];
        store4(word(b, e), make_float4(w.x + sg * v.x, w.y + sg * v.y, w.z + sg * v.z, w.w + sg * v.w), al);
      }
    }
  }
}

template <int CH, bool SIL, bool DIL>
void launch_level(bool expand, const PyrField& src, const PyrField& dst, int mode, const float* aux, float alpha,
                  hipStream_t s) {
  if (expand) {
    constexpr int TH = CH == 1 ? 256 : 320;
    const dim3 grid((unsigned)((long)dst.nx * dst.ny * dst.nz >> 12));
    hipLaunchKernelGGL((k_pyr_expand<CH, SIL, DIL, TH>), grid, dim3(TH), 0, s, src, dst, mode);
  } else {
    const dim3 grid((unsigned)((long)dst.nx * dst.ny * dst.nz >> 9));
    if constexpr (CH == 1)
      hipLaunchKernelGGL(k_pyr_reduce1, grid, dim3(256), 0, s, src, dst, mode);
    else if (dst.nx >= 16)
      hipLaunchKernelGGL((k_pyr_reduce<SIL, DIL, 2, 640>), dim3(grid.x / 2), dim3(640), 0, s, src, dst, mode, aux, alpha);
    else
      hipLaunchKernelGGL((k_pyr_reduce<SIL, DIL, 1, 384>), grid, dim3(384), 0, s, src, dst, mode, aux, alpha);
  }
}

}  // namespace

void launch_pyr_level(bool expand, int ch, const PyrField& src, const PyrField& dst, int mode, const float* aux,
                      float alpha, hipStream_t s) {
  const bool si = src.kind == PYR_INTERLEAVED, di = dst.kind == PYR_INTERLEAVED;
  if (ch == 1)
    launch_level<1, false, false>(expand, src, dst, mode, aux, alpha, s);
  else if (si && di)
    launch_level<3, true, true>(expand, src, dst, mode, aux, alpha, s);
  else if (si)
    launch_level<3, true, false>(expand, src, dst, mode, aux, alpha, s);
  else if (di)
    launch_level<3, false, true>(expand, src, dst, mode, aux, alpha, s);
  else
    launch_level<3, false, false>(expand, src, dst, mode, aux, alpha, s);
}

}  // namespace pmk
