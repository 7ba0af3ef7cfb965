// Tiled software rasterizer for gfx950: two kernels per render launch.
//
// raster_setup_kernel, one workgroup per camera image:
//   1. body poses, read in place from the physics state buffer, with R(q),
//      and the mesh templates go to LDS;
//   2. every template vertex of every body (and the ground) is transformed
//      once -- world = p + R (s v), clip = VP world, perspective divide,
//      viewport, snap to 24.8 fixed point -- into an LDS vertex cache;
//   3. culling: a triangle is dropped if a vertex in front of the near plane
//      is outside the guard band, if it is back-facing or degenerate (integer
//      area <= 0), or if its bounding box holds no pixel centre; one that
//      crosses the near plane is cut along it into one or two pieces (the
//      polygon in front, split as a fan), each culled the same way;
//      survivors are compacted into lists;
//   4. the tiles of each survivor's box are counted with LDS atomics;
//   5. a workgroup prefix scan of the counts places each 16x16 tile's bin;
//      then each survivor gets a setup record in the image's raster scratch
//      (snapped vertices in edge order, depths, 1/area, primitive and flat
//      Lambert colour), and its pairs with the tiles of its box, a lane each,
//      append its record id to their bins, after an exact corner test of the
//      edge functions where its box in the tile is large, flagged when the
//      triangle covers the whole tile.
//   Each wave keeps the survivors it finds to itself from step 3 on.
// raster_tile_kernel, one, two or four waves per workgroup over a run of tiles
//   of a row, each wave a tile at a time; a lane owns four horizontally
//   adjacent pixels.  The bin is read in batches of 64 records.  Small triangles (at most kSmallMax pixels of their box in the
//   tile) are expanded into fragments, one pixel per lane across several
//   triangles, whose keys meet in an LDS z-buffer through atomic minimum;
//   large ones are tested by every lane on its own four pixels, keeping the
//   minimum in registers.  Edge functions are exact (32-bit integers for
//   triangles of up to 120 pixels, else integer values carried in fp64); a
//   pixel centre is covered if every edge value is > 0, or == 0
//   on a top-left edge.  Depth is interpolated in fp32 and quantised to 24
//   bits, and the minimum key (depth << 40 | primitive << 24 | RGB8) wins,
//   so the result depends neither on bin order nor on which lane tests which
//   pixel.  The winner's colour comes from its record; depth and RGB8 leave
//   in 16- and 12-byte stores.
// An image whose bins exceed their capacity, or whose tile table does not fit
// the setup kernel's LDS, is marked unbinned: each of its tiles then tests
// every record of the image -- slower, with the same output.
#include <cstddef>

#include <type_traits>

#include "vuda_internal.h"

#pragma clang fp contract(off)

namespace vuda {
namespace {

constexpr int kMaxLdsTiles = 4096;  // tile table held in the setup kernel's LDS
// Box pixels in the tile of a fragment-packed triangle: a window of 64
// fragments takes 70 vector instructions (1.1 a pixel), a large triangle 110
// to 130 a tile, so they meet near 104.  (64, when a large one took 199: at two
// 256x256 cameras of 64 bodies 1,902 us a launch against 1,873.)
constexpr int kSmallMax = 104;
constexpr int kWide = 8;            // triangles over more tiles are binned by their whole wave
__host__ __device__ inline int align16(int x) { return (x + 15) & ~15; }

struct SetupLayout {
  // byte offsets into the setup (or fused) kernel's dynamic LDS
  int tpl, body, vis, cvis, own, pmap, vxy, vz, tiles, misc, lrec, lbin, total;
  int nmax, vmax, tw, rec_cap, bin_cap, vis_cap;
};

// The regions the setup alone uses (templates, poses, survivor lists, maps)
// come first, and at least zone0 bytes are reserved for them: the fused
// kernel's tile pass keeps its z-buffers there once the setup is done.  Then
// the vertex cache, the tile table and counters, and (fused kernel) rec_cap
// compact records and bin_cap bin entries.  threads: the workgroup's size
// (its waves keep their survivors in lists of their own).
__host__ __device__ inline SetupLayout setup_layout(int max_bodies, int max_verts, int max_tiles,
                                                    int max_tris, bool near_clip, int threads, int tpl_words,
                                                    int zone0 = 0, int rec_cap = 0, int bin_cap = 0) {
  SetupLayout L;
  L.nmax = max_bodies + 1;
  L.vmax = max_verts;
  L.tw = max_tiles < kMaxLdsTiles ? max_tiles : kMaxLdsTiles;
  L.rec_cap = rec_cap;
  L.bin_cap = bin_cap;
  L.vis_cap = (max_tris + threads - 1) / threads * 64;  // survivors of one wave
  int o = 0;
  L.tpl = o;    o += 4 * tpl_words;
  L.body = o;   o += 80 * L.nmax;
  L.vis = o;    o += align16(2 * L.vis_cap * (threads / 64));
  L.cvis = o;   o += near_clip ? align16(40 * kClipRecs) : 0;  // near-plane pieces: X[3] Y[3] z[3], primitive
  L.own = o;    o += 2 * threads;
  L.pmap = o;   o += align16(max_tris);   // primitive -> body map of the env
  if (o < zone0) o = align16(zone0);
  L.vxy = o;    o += align16(8 * L.vmax);  // (X, Y) per vertex
  L.vz = o;     o += align16(4 * L.vmax);  // depth per vertex
  L.tiles = o;  o += align16(4 * (3 * L.tw + 1));
  L.misc = o;   o += 192;  // [2] record count, [3] near-plane pieces, [4] queue slot,
                           // [5] a vertex behind the near plane, [6] fused: bit 0 records
                           // and bins in LDS, bit 1 binned; [8, 24) scan totals; [24, 40)
                           // survivors of each wave
  L.lrec = o;   o += 16 * rec_cap;
  L.lbin = o;   o += align16(2 * bin_cap);
  L.total = o;
  return L;
}

// A body in LDS: five quads, so that a lane takes what it needs of one in a
// few loads (arrays by component took 17 per vertex).
struct BodyLDS {
  float4* R;     // [3][nmax] rows of R(q), each with that component of the position
  float4* e;     // [nmax] half-extents along the body axes (x, y, z, 0); a radius thrice for a sphere
  int4* id;      // [nmax] vertex base and primitive base (env-local), albedo, type
};

// The mesh templates in LDS and the descriptor's constants.
struct Tpl {
  const uint32_t* w;
  int cv, gv, sn, cn, sf, cf, gf;  // word offsets (Templates::at_*)
  float near_w, guard, ground_albedo, ground_uv_scale, light[3];
  __device__ __forceinline__ float3 vec(int at, int i) const {
    const float* p = (const float*)w + at + 3 * i;
    return make_float3(p[0], p[1], p[2]);
  }
  __device__ __forceinline__ float3 vertex(bool cube, int i) const { return vec(cube ? cv : kTplSphereV, i); }
  __device__ __forceinline__ float3 normal(bool cube, int i) const { return vec(cube ? cn : sn, i); }
  __device__ __forceinline__ float3 albedo(int i) const { return vec(0, i); }
};

__device__ __forceinline__ Tpl tpl_view(const Templates* g, const uint32_t* lds) {
  Tpl t;
  t.w = lds;
  t.cv = uniform_ld(&g->at_cube_v);
  t.gv = uniform_ld(&g->at_ground_v);
  t.sn = uniform_ld(&g->at_sphere_n);
  t.cn = uniform_ld(&g->at_cube_n);
  t.sf = uniform_ld(&g->at_sphere_f);
  t.cf = uniform_ld(&g->at_cube_f);
  t.gf = uniform_ld(&g->at_ground_f);
  t.near_w = uniform_ld(&g->near_w);
  t.guard = uniform_ld(&g->guard);
  t.ground_albedo = uniform_ld(&g->ground_albedo);
  t.ground_uv_scale = uniform_ld(&g->ground_uv_scale);
#pragma unroll
  for (int k = 0; k < 3; ++k) t.light[k] = uniform_ld(&g->light[k]);
  return t;
}

// v turned by the rows r0, r1, r2
__device__ __forceinline__ float3 turned(float4 r0, float4 r1, float4 r2, float3 v) {
  return make_float3((r0.x * v.x + r0.y * v.y) + r0.z * v.z, (r1.x * v.x + r1.y * v.y) + r1.z * v.z,
                     (r2.x * v.x + r2.y * v.y) + r2.z * v.z);
}

// Rotation matrix of a unit quaternion, row-major, element k at m[k * stride]
__device__ __forceinline__ void quat_rot(float w, float x, float y, float z, float* m, int stride) {
  const float xx = x * x, yy = y * y, zz = z * z;
  const float xy = x * y, xz = x * z, yz = y * z;
  const float wx = w * x, wy = w * y, wz = w * z;
  m[0] = 1.0f - 2.0f * (yy + zz);
  m[stride] = 2.0f * (xy - wz);
  m[2 * stride] = 2.0f * (xz + wy);
  m[3 * stride] = 2.0f * (xy + wz);
  m[4 * stride] = 1.0f - 2.0f * (xx + zz);
  m[5 * stride] = 2.0f * (yz - wx);
  m[6 * stride] = 2.0f * (xz - wy);
  m[7 * stride] = 2.0f * (yz + wx);
  m[8 * stride] = 1.0f - 2.0f * (xx + yy);
}

constexpr int32_t kInvalid = (int32_t)0x80000000;  // in front, outside the guard band
constexpr int32_t kBehind = (int32_t)0x80000001;   // behind the near plane (clip w < near)

// Snapped screen-space triangle in edge order (vertices 0, 2, 1 of the face).
struct Tri {
  int32_t X[3], Y[3];
  float z[3];
  bool ok;
};

// vertex indices (env-local) of primitive `prim` whose body (from the map) is
// b; *body = -1 for the ground
__device__ __forceinline__ void prim_vertices(const Tpl& T, const BodyLDS& B, int b, int prim, int* body, int vid[3]) {
  int at = T.gf + prim, vb = 0;
  *body = -1;
  if (b != kGroundBody) {
    const int4 id = B.id[b];
    at = (id.w ? T.cf : T.sf) + (prim - id.y);
    vb = id.x;
    *body = b;
  }
  const uint32_t f = T.w[at];
  vid[0] = vb + (int)(f & 0xFFu);
  vid[1] = vb + (int)((f >> 8) & 0xFFu);
  vid[2] = vb + (int)(f >> 16);
}

// Snapped corners in edge order (vertices 0, 2, 1 of the face) from the vertex
// cache; ok: all in front of the near plane and inside the guard band.
__device__ __forceinline__ Tri load_tri(const int2* V, const int vid[3]) {
  Tri t;
  const int ord[3] = {0, 2, 1};
  t.ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int2 q = V[vid[ord[k]]];
    t.X[k] = q.x;
    t.Y[k] = q.y;
    t.z[k] = 0.0f;
    if (t.X[k] <= kBehind) t.ok = false;  // kInvalid or kBehind
  }
  return t;
}

__device__ __forceinline__ int64_t tri_area(const int32_t* X, const int32_t* Y) {
  return (int64_t)(X[1] - X[0]) * (int64_t)(Y[2] - Y[0]) -
         (int64_t)(Y[1] - Y[0]) * (int64_t)(X[2] - X[0]);
}

// Pixel range whose centres 256p+128 lie inside the bounding box, clipped
// to the image; returns false if empty.
__device__ __forceinline__ bool tri_pixels(const int32_t* X, const int32_t* Y, int W, int H, int* x0,
                                           int* x1, int* y0, int* y1) {
  const int xmin = min(X[0], min(X[1], X[2])), xmax = max(X[0], max(X[1], X[2]));
  const int ymin = min(Y[0], min(Y[1], Y[2])), ymax = max(Y[0], max(Y[1], Y[2]));
  *x0 = max(0, (xmin + 127) >> 8);
  *x1 = min(W - 1, (xmax - 128) >> 8);
  *y0 = max(0, (ymin + 127) >> 8);
  *y1 = min(H - 1, (ymax - 128) >> 8);
  return *x0 <= *x1 && *y0 <= *y1;
}

// Viewport transform and 24.8 snap of clip coordinates c: X = kBehind when
// near_test and c.w < near, kInvalid outside the guard band.
__device__ __forceinline__ void snap_clip(float4 c, float fW, float fH, const Tpl& T, bool near_test,
                                          int32_t* X, int32_t* Y, float* z) {
  *X = kInvalid;
  *Y = kInvalid;
  *z = 0.0f;
  if (near_test && c.w < T.near_w) {
    *X = *Y = kBehind;
    return;
  }
  const float nx = c.x / c.w, ny = c.y / c.w, nz = c.z / c.w;
  const float px = (nx * 0.5f + 0.5f) * fW;
  const float py = (0.5f - ny * 0.5f) * fH;
  if (!(fabsf(px) > T.guard || fabsf(py) > T.guard)) {
    *X = (int32_t)rintf(px * 256.0f);
    *Y = (int32_t)rintf(py * 256.0f);
    *z = nz;
  }
}

// The point where the edge from a (in front) to b (behind) meets the plane
// w = near, taken from the vertex in front so that both triangles sharing
// the edge cut it at the same point.
__device__ __forceinline__ float4 near_cut(float4 a, float4 b, float near_w) {
  const float t = (near_w - a.w) / (b.w - a.w);
  return make_float4(a.x + t * (b.x - a.x), a.y + t * (b.y - a.y), a.z + t * (b.z - a.z), a.w + t * (b.w - a.w));
}

// Piece s (0 or 1) of the part of a triangle in front of the near plane (c:
// clip coordinates of its vertices in face order, at least one in front and
// none in front outside the guard band): the polygon in front, in face
// order, split as a fan from its first vertex; the piece in edge order.
// Returns false if there is no piece s; t->ok is false if a cut point falls
// outside the guard band.
__device__ __forceinline__ bool near_piece(const float4 c[3], int s, float fW, float fH, const Tpl& T, Tri* t) {
  // the polygon's candidate points in cycle order: vertex k (if in front),
  // then the cut of edge k -> k+1 (if it crosses); selected with static
  // indices only, so that everything stays in registers
  float4 val[6];
  bool has[6], cut[6];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int k1 = k == 2 ? 0 : k + 1;
    const bool ik = !(c[k].w < T.near_w), ik1 = !(c[k1].w < T.near_w);
    val[2 * k] = c[k];
    has[2 * k] = ik;
    cut[2 * k] = false;
    val[2 * k + 1] = ik ? near_cut(c[k], c[k1], T.near_w) : near_cut(c[k1], c[k], T.near_w);
    has[2 * k + 1] = ik != ik1;
    cut[2 * k + 1] = true;
  }
  int m = 0;
#pragma unroll
  for (int j = 0; j < 6; ++j) m += has[j] ? 1 : 0;
  if (s + 2 >= m) return false;
  const int want[3] = {0, s + 2, s + 1};  // the piece (q0, q[s+1], q[s+2]) in edge order
  t->ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float4 q = val[0];
    bool qc = false;
    int n = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (has[j] && n == want[k]) {
        q = val[j];
        qc = cut[j];
      }
      n += has[j] ? 1 : 0;
    }
    snap_clip(q, fW, fH, T, !qc, &t->X[k], &t->Y[k], &t->z[k]);
    if (t->X[k] == kInvalid || t->X[k] == kBehind) t->ok = false;
  }
  return true;
}

__device__ __forceinline__ bool top_left(int32_t dx, int32_t dy) {
  return dy < 0 || (dy == 0 && dx > 0);
}

// Classify the pixel centres of the block [x0..x1] x [y0..y1] against the
// edges of a snapped triangle (edge order): 0 none can be covered, 1 some may
// be, 2 all are.  Edge values are affine in the pixel centre, so their
// extremes over the block are at its corners.  V: the type that holds them
// exactly: int32_t for a narrow triangle and a block inside its box, else
// double.
template <class V>
__device__ __forceinline__ int tile_class(const int32_t* X, const int32_t* Y, int x0, int x1, int y0, int y1) {
  const int32_t Px = 256 * x0 + 128, Py = 256 * y0 + 128;
  const V wx = (V)(256 * (x1 - x0)), wy = (V)(256 * (y1 - y0));
  bool all = true, none = false;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int a = (e + 1) % 3, b = (e + 2) % 3;
    const int32_t dx = X[b] - X[a], dy = Y[b] - Y[a];
    const V E = (V)dx * (V)(Py - Y[a]) - (V)dy * (V)(Px - X[a]);
    const V ax = -(V)dy * wx, ay = (V)dx * wy, zero = 0;
    const V emin = E + (ax < zero ? ax : zero) + (ay < zero ? ay : zero);
    const V emax = E + (ax < zero ? zero : ax) + (ay < zero ? zero : ay);
    const V thr = top_left(dx, dy) ? 0 : 1;  // covered from this value on
    none |= emax < thr;
    all &= emin >= thr;
  }
  return none ? 0 : (all ? 2 : 1);
}

// Flat Lambert colour of face `face` of body `body` (-1: ground), RGB8 packed.
__device__ __forceinline__ uint32_t face_color(const Tpl& T, const BodyLDS& B, int nmax, int body, int face) {
  float3 n = make_float3(0.0f, 0.0f, 1.0f), al = make_float3(T.ground_albedo, T.ground_albedo, T.ground_albedo);
  if (body >= 0) {
    const int4 id = B.id[body];
    n = turned(B.R[body], B.R[nmax + body], B.R[2 * nmax + body], T.normal(id.w != 0, face));
    al = T.albedo(id.z);
  }
  const float l = fmaxf(0.0f, (n.x * T.light[0] + n.y * T.light[1]) + n.z * T.light[2]);
  const float a[3] = {al.x, al.y, al.z};
  uint32_t rgb = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float col = a[c] * (0.2f + 0.8f * l);
    rgb |= (uint32_t)fminf(255.0f, rintf(col * 255.0f)) << (8 * c);
  }
  return rgb;
}

// Inclusive wave64 scans with DPP row shifts and row broadcasts: each step is
// a VALU operation reading a neighbour lane, with no LDS round trip.  Lanes
// whose source is outside the row read the identity (0; values are >= 0).
__device__ __forceinline__ int wave_incl_add(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}
// lanes of the mask m below this one
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Exclusive prefix sum over the workgroup of one value per thread.
__device__ __forceinline__ int wg_excl_scan(int v, int32_t* tmp, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int x = wave_incl_add(v);
  if (lane == 63) tmp[wave] = x;
  __syncthreads();
  int base = 0, tot = 0;
  for (int k = 0; k < nw; ++k) {
    const int t = tmp[k];
    base += k < wave ? t : 0;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + x - v;
}

// toff[t] = sum of cnt[0..t), toff[n] = total, with every thread of the group.
__device__ __forceinline__ int tile_scan(const int32_t* cnt, int32_t* toff, int n, int32_t* tmp) {
  const int nthr = blockDim.x;
  const int per = (n + nthr - 1) / nthr;
  const int t0 = min(n, (int)threadIdx.x * per), t1 = min(n, t0 + per);
  int s = 0;
  for (int t = t0; t < t1; ++t) s += cnt[t];
  int total;
  int acc = wg_excl_scan(s, tmp, &total);
  for (int t = t0; t < t1; ++t) {
    toff[t] = acc;
    acc += cnt[t];
  }
  if (threadIdx.x == 0) toff[n] = total;
  __syncthreads();
  return total;
}

// A small triangle's edge values over its box, in 32-bit integers: when the
// triangle spans at most kNarrow units (120 pixels) on both axes, every edge
// value at a pixel centre in its box is at most 2 kNarrow^2 < 2^31 in
// magnitude and the steps per pixel, 256 dx and 256 dy, stay below 2^23, so
// 24-bit multiply-adds are exact.
constexpr int kNarrow = 120 * 256;

// Flags of a triangle's setup record: bit e set when edge e is not top-left
// (a pixel centre on it is outside), bit 3 set when the triangle is narrow.
__device__ __forceinline__ int rec_flags(const Tri& t) {
  int flags = 0;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int a0 = (e + 1) % 3, b0 = (e + 2) % 3;
    if (!top_left(t.X[b0] - t.X[a0], t.Y[b0] - t.Y[a0])) flags |= 1 << e;
  }
  const bool narrow = max(t.X[0], max(t.X[1], t.X[2])) - min(t.X[0], min(t.X[1], t.X[2])) <= kNarrow &&
                      max(t.Y[0], max(t.Y[1], t.Y[2])) - min(t.Y[0], min(t.Y[1], t.Y[2])) <= kNarrow;
  if (narrow) flags |= 8;
  return flags;
}

// Setup record of a triangle in the image's raster scratch (64 bytes): what
// every tile it is binned to needs, so that the tile kernel recomputes none
// of it.  Word 2 of the last quad holds the flags.
__device__ __forceinline__ void store_rec(int4* recs, int r, const Tri& t, int prim, float invA,
                                          uint32_t rgb, int flags, int x0, int x1, int y0, int y1) {
  int4* p = recs + 4 * r;
  p[0] = make_int4(t.X[0], t.Y[0], t.X[1], t.Y[1]);
  p[1] = make_int4(t.X[2], t.Y[2], prim, __float_as_int(t.z[0]));
  p[2] = make_int4(__float_as_int(t.z[1]), __float_as_int(t.z[2]), __float_as_int(invA), (int32_t)rgb);
  p[3] = make_int4(x0 | (x1 << 16), y0 | (y1 << 16), flags, 0);
}

// ---------------------------------------------------------------------------
// setup kernel
// ---------------------------------------------------------------------------

// Clip coordinates of env-local vertex vi of body b (from the map): the
// body's pose applied to the scaled template vertex (the ground's vertices as
// they are), then the camera's view-projection (row dot products summed left
// to right, then the translation).
__device__ __forceinline__ float4 vertex_clip(const Tpl& T, const BodyLDS& B, int S, int b, int vi, const float* vp) {
  float wx, wy, wz;
  if (b == kGroundBody) {
    const float3 g = T.vec(T.gv, vi);
    wx = g.x;
    wy = g.y;
    wz = g.z;
  } else {
    const int4 id = B.id[b];
    const float3 tv = T.vertex(id.w != 0, vi - id.x);
    const float4 e = B.e[b], r0 = B.R[b], r1 = B.R[S + b], r2 = B.R[2 * S + b];
    const float3 t = turned(r0, r1, r2, make_float3(e.x * tv.x, e.y * tv.y, e.z * tv.z));
    wx = r0.w + t.x;
    wy = r1.w + t.y;
    wz = r2.w + t.z;
  }
  return make_float4(((vp[0] * wx + vp[1] * wy) + vp[2] * wz) + vp[3], ((vp[4] * wx + vp[5] * wy) + vp[6] * wz) + vp[7],
                     ((vp[8] * wx + vp[9] * wy) + vp[10] * wz) + vp[11],
                     ((vp[12] * wx + vp[13] * wy) + vp[14] * wz) + vp[15]);
}

// Attribute record r of a triangle for smooth shading (face `face` of body
// `body`, -1 the ground; vid its vertices in face order): the world normal
// and the reciprocal clip w of each vertex in edge order (face vertices 0, 2,
// 1), and the albedo.  A sphere's vertex normal is its unit template vertex
// turned by R, a cube's or box's the face normal, the ground's +z.
__device__ __forceinline__ void store_attr(float4* ga, float4* gt, int r, const Tpl& T, const BodyLDS& B,
                                           int S, int body, int face, const int vid[3], const float* vp) {
  const int ord[3] = {0, 2, 1};
  float iw[3];
  float3 n[3], al = make_float3(T.ground_albedo, T.ground_albedo, T.ground_albedo);
  const int4 id = B.id[body < 0 ? 0 : body];
  const bool cube = id.w != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int v = vid[ord[k]];
    iw[k] = 1.0f / vertex_clip(T, B, S, body < 0 ? (int)kGroundBody : body, v, vp).w;
    n[k] = make_float3(0.0f, 0.0f, 1.0f);
    if (body >= 0)
      n[k] = turned(B.R[body], B.R[S + body], B.R[2 * S + body], cube ? T.normal(true, face) : T.vertex(false, v - id.x));
  }
  if (body >= 0) al = T.albedo(id.z);
  float4* p = ga + 4 * r;
  p[0] = make_float4(n[0].x, n[0].y, n[0].z, n[1].x);
  p[1] = make_float4(n[1].y, n[1].z, n[2].x, n[2].y);
  p[2] = make_float4(n[2].z, iw[0], iw[1], iw[2]);
  p[3] = make_float4(al.x, al.y, al.z, 0.0f);
  if (!gt) return;
  // textured worlds: the texture coordinates of the vertices in edge order
  // (the ground: world x, y scaled; a cube or box face: the unit square over
  // the face's tangent axes of the body frame) and whether to sample
  float uv[3][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}};
  float textured = 0.0f;
  if (body < 0) {
    textured = 1.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float3 g = T.vec(T.gv, vid[ord[k]]);
      uv[k][0] = g.x * T.ground_uv_scale;
      uv[k][1] = g.y * T.ground_uv_scale;
    }
  } else if (cube) {
    textured = 1.0f;
    const float3 fn = T.normal(true, face);
    const int a = fabsf(fn.x) > 0.5f ? 0 : (fabsf(fn.y) > 0.5f ? 1 : 2);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float3 tv = T.vertex(true, vid[ord[k]] - id.x);
      uv[k][0] = ((a == 0 ? tv.y : tv.x) + 1.0f) * 0.5f;
      uv[k][1] = ((a == 2 ? tv.y : tv.z) + 1.0f) * 0.5f;
    }
  }
  float4* q = gt + 2 * r;
  q[0] = make_float4(uv[0][0], uv[0][1], uv[1][0], uv[1][1]);
  q[1] = make_float4(uv[2][0], uv[2][1], textured, 0.0f);
}

// CLIP: cut triangles crossing the near plane (else they are culled whole,
// and none of that code is compiled in).  FUSED: the fused kernel's setup,
// which keeps the image's records and bins in LDS when they fit (16-byte
// records: the vertex-cache indices of the corners in edge order, the
// primitive, 1/area, RGB8 and the flags), else writes them to the raster
// scratch as the setup kernel does; the tile table stays in LDS either way.
template <bool CLIP, bool FUSED>
__device__ void setup_image(unsigned char* lds, const SetupLayout& Lo, const WorldDev& W,
                            const RasterLaunch& L, int cam_id) {
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
  const CamDev cam = uniform_copy(W.cams + cam_id);
  const EnvDev ed = uniform_copy(W.envs + cam.env);
  const int n = ed.n_bodies;
  const int ntris = ed.n_tris;
  const int64_t cap = W.cap_bodies;
  const float* st = W.state[L.parity];
  // the env's primitive map (16-byte aligned and padded), read once into LDS:
  // the phases below look it up per triangle
  const uint8_t* gpmap = (const uint8_t*)(lds + Lo.pmap);
  const uint8_t* gvmap = W.vert_body + ed.vert_map;
  const int Wd = cam.w, Ht = cam.h;
  const int tsh = L.tile_shift, TS = 1 << tsh;  // tile edge in pixels
  const int ntx = (Wd + TS - 1) >> tsh;
  const int ntiles = tiles_of(Wd, Ht, tsh);
  // the image's scratch as the host laid it out (a tile table with room
  // for the smallest tiles)
  unsigned char* rs = W.rscratch + cam.rs_off + (int64_t)L.parity * cam.rs_total;  // one scratch per state buffer
  int32_t* hdr = (int32_t*)rs;
  int2* ttab = (int2*)(rs + 64);
  int4* grec = (int4*)(rs + cam.rs_recs);
  uint16_t* bins = (uint16_t*)(rs + cam.rs_bins);
  const int rs_bin_cap = kBinsPerTri * (cam.n_tris + kClipRecs);
  const int bin_cap = (L.bin_limit > 0 && L.bin_limit < rs_bin_cap) ? L.bin_limit : rs_bin_cap;

  const int S = Lo.nmax;
  BodyLDS B;
  B.R = (float4*)(lds + Lo.body);
  B.e = B.R + 3 * S;
  B.id = (int4*)(B.R + 4 * S);
  int2* V = (int2*)(lds + Lo.vxy);
  float* Vz = (float*)(lds + Lo.vz);
  uint16_t* vis = (uint16_t*)(lds + Lo.vis) + wave * Lo.vis_cap;  // this wave's survivors
  int32_t* cvis = (int32_t*)(lds + Lo.cvis);  // 10 words per piece
  uint8_t* start = lds + Lo.own + 128 * wave;  // this wave's marks where an owner's pairs start in the window
  uint8_t* owner = start + 64;                 // and 4 lane of the owners, in lane order
  int32_t* tcount = (int32_t*)(lds + Lo.tiles);
  int32_t* toff = tcount + Lo.tw;
  int32_t* tend = toff + Lo.tw + 1;
  int32_t* misc = (int32_t*)(lds + Lo.misc);
  const Tpl T = tpl_view(W.tpl, (const uint32_t*)(lds + Lo.tpl));

  // 1. templates, primitive map and bodies.  A thread asks for all it needs of
  // a body, and for its first quads of the templates and the map, before it
  // uses any (held together, else the compiler loads and waits one by one: at
  // 1,024 images 6,600 cycles of 64,500).
  for (int b = tid; b < n; b += nthr) {
    const int g = ed.body_off + b;
    float s7[7] = {st[QW * cap + g], st[QX * cap + g], st[QY * cap + g], st[QZ * cap + g],
                   st[PX * cap + g], st[PY * cap + g], st[PZ * cap + g]};
    const float* bx = W.box + 6 * (int64_t)g;
    float x = bx[0], y = bx[1], z = bx[2];
    int vb = W.vert_base[g], pb = W.prim_base[g], al = W.albedo[g], ty = W.type[g];
    asm volatile("" : "+v"(s7[0]), "+v"(s7[1]), "+v"(s7[2]), "+v"(s7[3]), "+v"(s7[4]), "+v"(s7[5]), "+v"(s7[6]),
                      "+v"(x), "+v"(y), "+v"(z), "+v"(vb), "+v"(pb), "+v"(al), "+v"(ty));
    float R[9];
    quat_rot(s7[0], s7[1], s7[2], s7[3], R, 1);
    B.R[b] = make_float4(R[0], R[1], R[2], s7[4]);
    B.R[S + b] = make_float4(R[3], R[4], R[5], s7[5]);
    B.R[2 * S + b] = make_float4(R[6], R[7], R[8], s7[6]);
    B.e[b] = make_float4(x, y, z, 0.0f);
    B.id[b] = make_int4(vb, pb, al, ty);
  }
  int body_next = gvmap[min(tid, ed.n_verts - 1)];
  {
    const int4* tsrc = (const int4*)W.tpl->data;
    const int4* psrc = (const int4*)(W.prim_body + ed.prim_map);
    int4* tdst = (int4*)(lds + Lo.tpl);
    int4* pdst = (int4*)(lds + Lo.pmap);
    const int nt = L.tpl_words / 4, np = (ntris + 15) / 16;  // at least 1 each
    const int t0 = min(tid, nt - 1), t1 = min(tid + nthr, nt - 1), p0 = min(tid, np - 1), p1 = min(tid + nthr, np - 1);
    int4 a = tsrc[t0], b = tsrc[t1], c = psrc[p0], d = psrc[p1];
    asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w),
                      "+v"(c.x), "+v"(c.y), "+v"(c.z), "+v"(c.w), "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w));
    // (threads past the end write the last quad again)
    tdst[t0] = a;
    tdst[t1] = b;
    pdst[p0] = c;
    pdst[p1] = d;
    for (int i = tid + 2 * nthr; i < nt; i += nthr) tdst[i] = tsrc[i];
    for (int i = tid + 2 * nthr; i < np; i += nthr) pdst[i] = psrc[i];
  }
  const bool tiled = ntiles <= Lo.tw;
  if (tid == 0) misc[3] = misc[5] = 0;
  if (tiled)
    for (int t = tid; t < ntiles; t += nthr) tcount[t] = 0;
  __syncthreads();

  // 2. vertices
  const float* vp = cam.vp;
  const float fW = (float)Wd, fH = (float)Ht;
  // (the body of a lane's next vertex is on its way while this one is transformed)
  for (int vi = tid; vi < ed.n_verts; vi += nthr) {
    const int b = body_next;
    body_next = gvmap[min(vi + nthr, ed.n_verts - 1)];
    int32_t X, Y;
    float z;
    snap_clip(vertex_clip(T, B, S, b, vi, vp), fW, fH, T, true, &X, &Y, &z);
    if (CLIP && X == kBehind) misc[5] = 1;  // some vertex of the image is behind the near plane
    V[vi] = make_int2(X, Y);
    Vz[vi] = z;
  }
  __syncthreads();

  // 3. visibility.  A triangle survives if every vertex is in front of the
  // near plane and inside the guard band, its integer area is > 0 (front
  // facing, not degenerate) and its box holds a pixel centre.  Each wave
  // compacts its survivors into a list of its own (a ballot, no atomic), so
  // that the costlier steps below run on full waves.  A triangle that crosses
  // the near plane (and has no vertex in front outside the guard band) is cut
  // along it: its surviving pieces go to cvis, and become the records after
  // the whole triangles.
  // (two versions of the pass: images with no vertex behind the near plane,
  // nearly all of them, run the one without the cut)
  int nmine = 0;  // this wave's survivors
  const auto visibility = [&](auto cut_tag) {
  for (int base = 0; base < ntris; base += nthr) {
    const int pr = base + tid;
    bool keep = false;
    if (pr < ntris) {
      int body, vid[3];
      prim_vertices(T, B, gpmap[pr], pr, &body, vid);
      const Tri t = load_tri(V, vid);
      int x0, x1, y0, y1;
      keep = t.ok && tri_area(t.X, t.Y) > 0 && tri_pixels(t.X, t.Y, Wd, Ht, &x0, &x1, &y0, &y1);
      if constexpr (decltype(cut_tag)::value) {
      int behind = 0, outside = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        behind += t.X[k] == kBehind;
        outside += t.X[k] == kInvalid;
      }
      if (behind > 0 && behind < 3 && outside == 0) {
        float4 c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) c[k] = vertex_clip(T, B, S, body < 0 ? (int)kGroundBody : body, vid[k], vp);
        for (int sp = 0; sp < 2; ++sp) {
          Tri q;
          q.ok = false;
          if (near_piece(c, sp, fW, fH, T, &q) && q.ok && tri_area(q.X, q.Y) > 0 &&
              tri_pixels(q.X, q.Y, Wd, Ht, &x0, &x1, &y0, &y1)) {
            // the piece itself is kept, so that the record and binning
            // passes need not cut again
            const int slot = atomicAdd(&misc[3], 1);
            if (slot < kClipRecs) {
              int32_t* o = cvis + 10 * slot;
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                o[k] = q.X[k];
                o[3 + k] = q.Y[k];
                o[6 + k] = __float_as_int(q.z[k]);
              }
              o[9] = pr;
            }
          }
        }
      }
      }
    }
    const uint64_t m = __ballot(keep);
    if (keep) vis[nmine + lanes_below(m)] = (uint16_t)pr;
    nmine += __popcll(m);
  }
  };
  if constexpr (CLIP) {
    if (misc[5]) visibility(std::true_type{});
    else visibility(std::false_type{});
  } else {
    visibility(std::false_type{});
  }
  if (lane == 0) misc[24 + wave] = nmine;
  int npieces = 0;
  if constexpr (CLIP) {
    // the pieces are the first wave's, after its whole triangles
    __syncthreads();
    npieces = min(misc[3], kClipRecs);
    if (tid == 0 && misc[3] > kClipRecs) raise_flag(W, cam.env, kFlagClipOverflow);
  }
  const int mine = nmine + (wave == 0 ? npieces : 0);  // records this wave makes
  // the wave's record i: whole triangle vis[i], or piece cvis[i - nmine]; vid
  // its face's vertices in face order
  const auto record_tri = [&](int i, int* pr, int* body, int vid[3], Tri* t) {
    const int32_t* o = cvis + 10 * (i - nmine);
    const bool whole = !CLIP || i < nmine;
    *pr = whole ? (int)vis[i] : o[9];
    prim_vertices(T, B, gpmap[*pr], *pr, body, vid);
    if (whole) {
      *t = load_tri(V, vid);
      return;
    }
    t->ok = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      t->X[k] = o[k];
      t->Y[k] = o[3 + k];
      t->z[k] = __int_as_float(o[6 + k]);
    }
  };
  // the tiles [tx0, tx0 + nx) x [ty0, ty0 + ny) of a triangle's box
  struct Box {
    int x0, x1, y0, y1, tx0, ty0, nx, ny;
  };
  const auto box_of = [&](const Tri& t) -> Box {
    Box q;
    tri_pixels(t.X, t.Y, Wd, Ht, &q.x0, &q.x1, &q.y0, &q.y1);
    q.tx0 = q.x0 >> tsh;
    q.ty0 = q.y0 >> tsh;
    q.nx = (q.x1 >> tsh) - q.tx0 + 1;
    q.ny = (q.y1 >> tsh) - q.ty0 + 1;
    return q;
  };

  // 4. tile counts, one surviving triangle per lane.  A triangle whose box
  // spans more than kWide tiles is counted by its whole wave, one tile per
  // lane, so that one lane never walks a long tile list alone.
  if (tiled) {
    for (int base = 0; base < mine; base += 64) {
      const int i = base + lane;
      Box q{};
      if (i < mine) {
        int pr, body, vid[3];
        Tri t;
        record_tri(i, &pr, &body, vid, &t);
        q = box_of(t);
      }
      const bool wide = q.nx * q.ny > kWide;
      if (!wide)
        for (int qy = 0; qy < q.ny; ++qy)
          for (int qx = 0; qx < q.nx; ++qx) atomicAdd(&tcount[(q.ty0 + qy) * ntx + q.tx0 + qx], 1);
      uint64_t m = __ballot(wide);
      while (m) {
        const int j = __ffsll((unsigned long long)m) - 1;
        m &= m - 1ull;
        const int jx0 = __builtin_amdgcn_readlane(q.tx0, j), jy0 = __builtin_amdgcn_readlane(q.ty0, j);
        const int jnx = __builtin_amdgcn_readlane(q.nx, j), jn = jnx * __builtin_amdgcn_readlane(q.ny, j);
        for (int k = lane; k < jn; k += 64) {
          const int qy = k / jnx;
          atomicAdd(&tcount[(jy0 + qy) * ntx + jx0 + (k - qy * jnx)], 1);
        }
      }
    }
  }
  __syncthreads();
  // records are numbered wave by wave
  int first = 0, nrec = npieces;
  for (int k = 0; k < nwaves; ++k) {
    const int c = misc[24 + k];
    first += k < wave ? c : 0;
    nrec += c;
  }
  if (wave > 0) first += npieces;
  // bin entries hold 15-bit record ids
  bool binned = tiled && nrec <= 32768;
  int total = 0;
  if (binned) total = tile_scan(tcount, toff, ntiles, misc + 8);
  bool local = false;
  if constexpr (FUSED) local = nrec <= Lo.rec_cap && (!binned || total <= Lo.bin_cap);
  if (binned && total > (local ? Lo.bin_cap : bin_cap)) binned = false;
  int4* lrec = (int4*)(lds + Lo.lrec);
  uint16_t* bout = local ? (uint16_t*)(lds + Lo.lbin) : bins;
  if (binned) {
    for (int t = tid; t < ntiles; t += nthr) tend[t] = toff[t];
    __syncthreads();
  }

  // 5. a setup record (with the face colour) per surviving triangle, and its
  // record id scattered into the bins.  Record slots are in no key, which
  // orders by depth, then primitive.
  for (int base = 0; base < mine; base += 64) {
    const int i = base + lane, r = first + i;
    Box q{};
    Tri t{};
    int flags = 0;
    if (i < mine) {
      int pr, body, vid[3];
      record_tri(i, &pr, &body, vid, &t);
      q = box_of(t);
      const int64_t A = tri_area(t.X, t.Y);
      const int face = body < 0 ? pr : pr - B.id[body].y;
      uint32_t rgb;
      if (L.smooth) {
        // the key carries the record instead of a colour; the pixel's colour
        // comes from the record's attributes in the tile kernel
        rgb = (uint32_t)r;
        store_attr((float4*)(rs + cam.rs_attr), W.texture ? (float4*)(rs + cam.rs_tuv) : nullptr, r, T, B, S, body,
                   face, vid, vp);
      } else {
        rgb = face_color(T, B, S, body, face);
      }
      const float invA = 1.0f / (float)(double)A;
      flags = rec_flags(t);
      if (FUSED && local) {
        lrec[r] = make_int4((int32_t)((uint32_t)vid[0] | ((uint32_t)vid[2] << 16)),
                            (int32_t)((uint32_t)vid[1] | ((uint32_t)pr << 16)), __float_as_int(invA),
                            (int32_t)(rgb | ((uint32_t)flags << 24)));
      } else {
        if (!CLIP || i < nmine) {
          t.z[0] = Vz[vid[0]];
          t.z[1] = Vz[vid[2]];
          t.z[2] = Vz[vid[1]];
        }
        store_rec(grec, r, t, pr, invA, rgb, flags, q.x0, q.x1, q.y0, q.y1);
      }
    }
    if (!binned) continue;
    // Every (triangle, tile of its box) pair takes a lane: pair f belongs to
    // the lane j with off_j <= f < off_j + n_j, found by marking where each
    // range starts and counting the marks (as the tile pass finds a fragment's
    // triangle).  A lane walking its triangle's tiles one after the other left
    // the others waiting for the longest: the pass took 28,000 of 70,000 cycles
    // at 540 triangles.
    // A pair's entry is rejected if the triangle's edges miss the tile, and
    // flagged if they cover it, where its box in the tile holds more than
    // kSmallMax pixels (the tile kernel goes over the whole tile then; a
    // smaller one is expanded into its box's pixels there anyway).
    const int cnt = q.nx * q.ny;
    int incl = wave_incl_add(cnt);
    asm("" : "+v"(incl));  // (else off is summed anew from the scan's parts)
    const int pairs = __builtin_amdgcn_readlane(incl, 63);
    const int off = incl - cnt;
    const float rnx = __builtin_amdgcn_rcpf((float)q.nx);
    const int bxx = q.x0 | (q.x1 << 16), byy = q.y0 | (q.y1 << 16);
    const uint64_t have = __ballot(cnt > 0);
    if (cnt > 0) owner[lanes_below(have)] = 4 * lane;
    int before = -1;  // owners that start before the window, less one
    for (int f0 = 0; f0 < pairs; f0 += 64) {
      start[lane] = 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      if (cnt > 0 && off >= f0 && off < f0 + 64) start[off - f0] = 1;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const uint64_t starts = __ballot(start[lane] != 0);
      const int nth = before + (int)(starts & 1) + lanes_below(starts >> 1);  // marks up to and at this lane
      before += __popcll(starts);
      const int j4 = owner[nth];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int f = f0 + lane;
      const auto own = [&](int v) { return __builtin_amdgcn_ds_bpermute(j4, v); };
      const int k = f - own(off);
      const int xx = own(bxx), yy = own(byy);
      const int jx0 = (xx & 0xFFFF) >> tsh, jy0 = (yy & 0xFFFF) >> tsh;
      const int jnx = (xx >> 16 >> tsh) - jx0 + 1;
      // k / jnx exactly: k < 2^18 tiles and jnx <= 512, so the quotient's
      // fraction is at least 1/1024 away from an integer and its rounding
      // error below 2^-12
      const int qy = (int)(((float)k + 0.5f) * __int_as_float(own(__float_as_int(rnx))));
      const int tx = jx0 + k - qy * jnx, ty = jy0 + qy;
      const int px = tx << tsh, py = ty << tsh;
      const int bx0 = max(xx & 0xFFFF, px), bx1 = min(xx >> 16, px + TS - 1);
      const int by0 = max(yy & 0xFFFF, py), by1 = min(yy >> 16, py + TS - 1);
      const bool live = f < pairs;
      const bool large = live && (bx1 - bx0 + 1) * (by1 - by0 + 1) > kSmallMax;
      int cls = 1;
      if (__ballot(large)) {
        int32_t JX[3], JY[3];
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          JX[v] = own(t.X[v]);
          JY[v] = own(t.Y[v]);
        }
        const bool narrow = (own(flags) & 8) != 0;
        const bool alone = jnx == 1 && yy >> 16 >> tsh == jy0;  // a single tile is never missed
        if (large && !alone) {
          if (narrow) cls = tile_class<int32_t>(JX, JY, bx0, bx1, by0, by1);
          else cls = tile_class<double>(JX, JY, bx0, bx1, by0, by1);
        }
      }
      if (live && cls != 0) {
        const bool whole = cls == 2 && bx0 == px && by0 == py && bx1 == min(Wd - 1, px + TS - 1) &&
                           by1 == min(Ht - 1, py + TS - 1);
        const int jr = first + base + (j4 >> 2);
        bout[atomicAdd(&tend[ty * ntx + tx], 1)] = (uint16_t)(jr | (whole ? 0x8000 : 0));
      }
    }
  }
  if constexpr (FUSED) {
    // the tile pass reads the table from LDS after the caller's barrier
    if (tid == 0) {
      misc[2] = nrec;
      misc[6] = (local ? 1 : 0) | (binned ? 2 : 0);
    }
    return;
  }
  __syncthreads();
  if (binned)
    for (int t = tid; t < ntiles; t += nthr) ttab[t] = make_int2(toff[t], tend[t] - toff[t]);
  if (tid == 0) {
    hdr[0] = nrec;
    hdr[1] = binned ? 1 : 0;
  }
}

// Held to 72 VGPRs (seven waves per SIMD), so that a slot a tile wave leaves can
// take one of its waves when the render overlaps the next step.  The price is 13
// VGPRs spilled to scratch, and 112 SGPRs to lanes of VGPRs (299 of its 1,544
// vector instructions move them).  Bound by latency: at 1,024 images of 540
// visible triangles (128 threads each) it takes 36.7 us; when it took 37.9, and
// 37.1 at 80 VGPRs, the pipelined iteration was 81 us with the one and 88 with the
// other (now 77; 4,096 envs of two 256x256 cameras and 2,048 envs of mixed sizes
// measure the same either way).  With the cut of the near plane seven waves spill
// 22 VGPRs and 133 SGPRs and lose, so it has 80 (six waves): the setup of 1,024
// images of 64x64, 8 bodies, 18.4 us against 19.8 with 72; 1,920 of 256x256, 20
// bodies, 45.6 against 49.9; the pipelined iteration of 1,024 envs of 32 bodies
// 76.4 against 78.8, of 2,048 envs of mixed sizes 213 and 228.
template <bool CLIP>
__global__ void __attribute__((amdgpu_waves_per_eu(CLIP ? 6 : 7))) raster_setup_kernel(WorldDev W, RasterLaunch L) {
  extern __shared__ __align__(16) unsigned char lds[];
  // At the end of a step this kernel shares CUs with the render's tile
  // waves; a higher issue priority keeps its chains of dependent steps moving.
  switch (L.prio) {
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 3: __builtin_amdgcn_s_setprio(3); break;
    default: break;
  }
  const SetupLayout Lo = setup_layout(L.max_bodies, L.max_verts, L.max_tiles, L.max_tris, CLIP, (int)blockDim.x, L.tpl_words);
  // one copy of the setup for both launch forms (14 KB of code; the instruction
  // cache is shared with the step's and the tiles' kernels)
  int32_t* slot = (int32_t*)(lds + Lo.misc) + 4;
  int wi = (int)blockIdx.x;
  for (;;) {
    if (L.persistent) {
      __syncthreads();
      if (threadIdx.x == 0) *slot = atomicAdd(L.queue, 1);
      __syncthreads();
      wi = *slot;
    }
    if (wi >= L.n_work) return;
    setup_image<CLIP, false>(lds, Lo, W, L, uniform_ld(L.work + wi));
    if (!L.persistent) return;
  }
}

// ---------------------------------------------------------------------------
// tile kernel
// ---------------------------------------------------------------------------

// A tile of TS x TS pixels per wave: each lane owns a block of BW x BH
// pixels, BW adjacent in a row (4, or 1 for 8x8 tiles), BH rows (4 for
// 32x32 tiles, else 1).
template <int TS>
struct TileGeo {
  static constexpr int BW = TS >= 16 ? 4 : 1;
  static constexpr int LPR = TS / BW;              // lanes per row of blocks
  static constexpr int BH = TS * TS / (64 * BW);
  static constexpr int NPX = BW * BH;              // pixels per lane
  static_assert(LPR * (64 / LPR) == 64 && (64 / LPR) * BH == TS, "tile shape");
};

template <int TS>
struct TileWaveLDS {
  uint64_t zb[TS * TS];  // z-buffer of the small-triangle fragments
  uint8_t start[64];     // marks where an owner's fragments start in the window
  uint8_t owner[64];     // 4 lane of the small triangles, in lane order
};

// Key of a primitive's fragment below its depth: primitive << 24 | RGB8.
// Primitives number at most 65535 per env, so no key equals the empty ~0.
__device__ __forceinline__ uint64_t prim_key(int prim, uint32_t rgb) {
  return ((uint64_t)(uint32_t)prim << 24) | (uint64_t)(rgb & 0xFFFFFFu);
}

// Quantised depth key of a covered pixel from its three edge values; the
// 24-bit depth decides, then the primitive (unique in an image), so the
// colour carried in the low bits never does.
__device__ __forceinline__ uint64_t depth_key(float e0, float e1, float e2, float z0, float z1, float z2,
                                              float invA, uint64_t key) {
  const float zz = ((e0 * z0 + e1 * z1) + e2 * z2) * invA;
  // the interpolated depth is finite, so the median equals the clamp to [0, 1]
  const uint32_t D = (uint32_t)rintf(__builtin_amdgcn_fmed3f(zz, 0.0f, 1.0f) * 16777215.0f);
  // (by halves: the upper one is a shift and an or in one instruction)
  return ((uint64_t)((D << 8) | (uint32_t)(key >> 32)) << 32) | (uint32_t)key;
}

// Smooth shading of pixel (px, py) won by record r: the attribute record's
// vertex normals interpolated with weights E_k / w_k at the pixel centre
// (exact edge values), normalized, and Lambert-shaded; RGB8 packed.
__device__ __forceinline__ uint32_t smooth_color(const int4* grec, const float4* gattr, const float4* gtuv,
                                                 const uint8_t* tex, const Templates* T, int r, int px, int py) {
  const int4 a = grec[4 * r], b = grec[4 * r + 1];
  const float4 g0 = gattr[4 * r], g1 = gattr[4 * r + 1], g2 = gattr[4 * r + 2], g3 = gattr[4 * r + 3];
  const int32_t X[3] = {a.x, a.z, b.x}, Y[3] = {a.y, a.w, b.y};
  const float iw[3] = {g2.y, g2.z, g2.w};
  const int Px = 256 * px + 128, Py = 256 * py + 128;
  float u[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int a0 = (e + 1) % 3, b0 = (e + 2) % 3;
    const int32_t dx = X[b0] - X[a0], dy = Y[b0] - Y[a0];
    const double E = fma(-(double)dy, (double)(Px - X[a0]), (double)dx * (double)(Py - Y[a0]));
    u[e] = (float)E * iw[e];
  }
  const float mx = (u[0] * g0.x + u[1] * g0.w) + u[2] * g1.z;
  const float my = (u[0] * g0.y + u[1] * g1.x) + u[2] * g1.w;
  const float mz = (u[0] * g0.z + u[1] * g1.y) + u[2] * g2.x;
  const float l2 = (mx * mx + my * my) + mz * mz;
  float nx = 0.0f, ny = 0.0f, nz = 0.0f;
  if (l2 > 0.0f) {
    const float l = sqrtf(l2);
    nx = mx / l;
    ny = my / l;
    nz = mz / l;
  }
  const float lam = fmaxf(0.0f, (nx * T->light[0] + ny * T->light[1]) + nz * T->light[2]);
  float al[3] = {g3.x, g3.y, g3.z};
  if (gtuv) {
    // textured worlds: the albedo times the texel (nearest, repeating) at
    // the texture coordinates interpolated with the weights above
    const float4 t0 = gtuv[2 * r], t1 = gtuv[2 * r + 1];
    if (t1.z != 0.0f) {
      const float s = (u[0] + u[1]) + u[2];
      float U = 0.0f, V = 0.0f;
      if (s > 0.0f) {
        U = ((u[0] * t0.x + u[1] * t0.z) + u[2] * t1.x) / s;
        V = ((u[0] * t0.y + u[1] * t0.w) + u[2] * t1.y) / s;
      }
      float fu = U - floorf(U), fv = V - floorf(V);
      if (!(fu >= 0.0f)) fu = 0.0f;
      if (!(fv >= 0.0f)) fv = 0.0f;
      const int i = min((int)(fu * (float)T->tex_w), T->tex_w - 1);
      const int j = min((int)(fv * (float)T->tex_h), T->tex_h - 1);
      const uint8_t* p = tex + 3 * ((int64_t)j * T->tex_w + i);
#pragma unroll
      for (int c = 0; c < 3; ++c) al[c] = al[c] * ((float)p[c] / 255.0f);
    }
  }
  uint32_t rgb = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float col = al[c] * (0.2f + 0.8f * lam);
    rgb |= (uint32_t)fminf(255.0f, rintf(col * 255.0f)) << (8 * c);
  }
  return rgb;
}

// Where the tile pass finds an image's records and bins.  GlobalRecs: the
// 64-byte records and the bins in the raster scratch.  LdsRecs (fused
// kernel): 16-byte records and bins in LDS, the corners read from the
// vertex cache and the pixel box recomputed, so that fetch() returns the
// four quads of the 64-byte record.
// kScalar: a wave may read one record with scalar loads, which is for records
// that an earlier kernel wrote (the tile kernel).  Scalar loads neither see nor
// wait for vector stores of the kernel they are in, not even across a workgroup
// barrier, so the fused kernel, which writes the records it reads, takes them
// from its lanes' registers.
template <bool kScalar>
struct GlobalRecs {
  static constexpr bool kUniform = kScalar;
  const int4* rec;
  const uint16_t* bins;
  __device__ __forceinline__ int bin(int k) const { return bins[k]; }
  __device__ __forceinline__ void fetch(int r, int4& a, int4& b, int4& c, int4& d) const {
    a = rec[4 * r];
    b = rec[4 * r + 1];
    c = rec[4 * r + 2];
    d = rec[4 * r + 3];
  }
};

struct LdsRecs {
  static constexpr bool kUniform = false;
  const int4* rec;
  const int2* V;
  const float* z;
  const uint16_t* bins;
  int w, h;
  __device__ __forceinline__ int bin(int k) const { return bins[k]; }
  __device__ __forceinline__ void fetch(int r, int4& a, int4& b, int4& c, int4& d) const {
    const int4 q = rec[r];
    const int i0 = q.x & 0xFFFF, i1 = (int)((uint32_t)q.x >> 16), i2 = q.y & 0xFFFF;
    const int2 v0 = V[i0], v1 = V[i1], v2 = V[i2];
    a = make_int4(v0.x, v0.y, v1.x, v1.y);
    b = make_int4(v2.x, v2.y, (int32_t)((uint32_t)q.y >> 16), __float_as_int(z[i0]));
    c = make_int4(__float_as_int(z[i1]), __float_as_int(z[i2]), q.z, q.w & 0xFFFFFF);
    const int32_t X[3] = {v0.x, v1.x, v2.x}, Y[3] = {v0.y, v1.y, v2.y};
    int x0, x1, y0, y1;
    tri_pixels(X, Y, w, h, &x0, &x1, &y0, &y1);
    d = make_int4(x0 | (x1 << 16), y0 | (y1 << 16), (int32_t)((uint32_t)q.w >> 24), 0);
  }
};

typedef short short2v __attribute__((ext_vector_type(2)));

// Registers of no particular value (no instruction): for lanes that hold no
// record.  (One statement, so that the four are different registers.)
__device__ __forceinline__ void no_value(int4& a, int4& b, int4& c, int4& d) {
  asm(""
      : "=v"(a.x), "=v"(a.y), "=v"(a.z), "=v"(a.w), "=v"(b.x), "=v"(b.y), "=v"(b.z), "=v"(b.w), "=v"(c.x),
        "=v"(c.y), "=v"(c.z), "=v"(c.w), "=v"(d.x), "=v"(d.y), "=v"(d.z), "=v"(d.w));
}

// The key of a pixel no triangle covers, above every other (primitives stay
// below 0xFFFF); its colour bits are the background's.
constexpr uint64_t kNoKey = 0xFFFFFFFFFF000000ull;

// Four pixels of a row from pixel `pix` of an image on: depth, and RGB packed in
// three words.  Where an image's width is no multiple of 4, most rows start off
// 16 and 4 bytes; global memory takes such stores whole (the types say what
// alignment there is), and stored pixel by pixel, a word and three bytes each,
// they bound the pass: 400 images of 337x211 174 us, 63 like this; 1,000 of
// 129x127 131 and 56.
struct __attribute__((packed, aligned(4))) Depth4 {
  uint32_t d[4];
};
struct __attribute__((packed, aligned(1))) Rgb4 {
  uint32_t c[3];
};
__device__ __forceinline__ void store_four(uint32_t* depth, uint8_t* image, uint32_t pix, Depth4 d, Rgb4 c) {
  *(Depth4*)((char*)depth + 4 * pix) = d;
  *(Rgb4*)(image + 3 * pix) = c;
}

// One tile of an image: records k0 .. k1 of the tile's bin (binned), or
// every record k0 .. k1 of the image.  rs: the image's raster scratch (smooth
// shading reads its attribute records there).
//
// Bound by VALU issue (three quarters of the cycles issue one), so it is the
// instructions per tile that count: empty tiles leave at once, lanes past the
// bin hold no values, a fragment finds its owner by counting marks and takes 14
// words of it, a large triangle's record comes by scalar loads that no branch
// surrounds and its edge values from integers where they fit.  At 8,192 images
// of 256x256 (64 bodies) 393 -> 353 vector instructions per tile, 1,985 ->
// 1,800 us a launch (1,635 in runs of tiles); at 1,024 of 128x128 (32 bodies)
// 65.8 -> 56.
template <bool DBG, bool SMOOTH, int TS, class Src>
__device__ __forceinline__ void raster_tile(const WorldDev& W, const CamDev& cam, const Src& src, bool binned,
                                            int k0, int k1, int tx, int ty, TileWaveLDS<TS>& S, int32_t* cov,
                                            const unsigned char* rs) {
  using G = TileGeo<TS>;
  constexpr int BW = G::BW, BH = G::BH, NPX = G::NPX;
  const int lane = threadIdx.x & 63;
  const int Wd = cam.w, Ht = cam.h;
  const int tx0 = tx * TS, ty0 = ty * TS;
  const int tx1 = min(tx0 + TS - 1, Wd - 1), ty1 = min(ty0 + TS - 1, Ht - 1);
  // this lane's pixels: (px0 + i, py0 + j) for i < BW, j < BH, z-buffer
  // entries zrow (j) + i
  const int bx = lane % G::LPR, by = lane / G::LPR;
  const int px0 = tx0 + BW * bx, py0 = ty0 + BH * by;
  const auto zidx = [&](int i, int j) { return (BH * by + j) * TS + BW * bx + i; };
  // the image's outputs: a uniform base and 32-bit pixel offsets (4096^2 at most)
  uint32_t* const depth = W.depth + cam.pix_off;
  uint8_t* const image = W.rgb + 3 * cam.pix_off;
  const uint32_t row0 = (uint32_t)(py0 * Wd + px0);
  uint64_t* zb = S.zb;
  if (!DBG && BW == 4 && BH == 1 && k0 >= k1) {
    // an empty bin (a third of the tiles of a settled scene): the background
    if (py0 <= ty1 && px0 + 3 <= tx1) {
      store_four(depth, image, row0, Depth4{{~0u, ~0u, ~0u, ~0u}}, Rgb4{{0u, 0u, 0u}});
      return;
    }
    if (py0 <= ty1)
      for (int i = 0; i < 4 && px0 + i <= tx1; ++i) {
        depth[row0 + i] = ~0u;
        for (int q = 0; q < 3; ++q) image[3 * (row0 + i) + q] = 0;
      }
    return;
  }
  // The LDS z-buffer is only for small triangles' fragments: it is cleared
  // before the first fragment window and read back only if it was.  A tile
  // that holds large triangles alone, such as the open ground, never touches
  // it.
  bool zused = false;
  if (DBG) {
#pragma unroll
    for (int j = 0; j < BH; ++j)
#pragma unroll
      for (int i = 0; i < BW; ++i) cov[zidx(i, j)] = 0;
  }
  uint64_t kreg[NPX];
  int creg[NPX];
#pragma unroll
  for (int q = 0; q < NPX; ++q) {
    kreg[q] = kNoKey;
    creg[q] = 0;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

  for (int kb = k0; kb < k1; kb += 64) {
    // One record per lane, kept in registers: a small triangle's fragments
    // fetch their owner's values with cross-lane reads (ds_bpermute, which
    // needs no LDS of its own), a large triangle's record is read uniformly.
    // So the tile keeps little LDS, and the step's waves find room beside it
    // on the CU.  Lanes past the bin hold no values (and no instructions
    // clear them): their area is 0.
    const int k = kb + lane;
    int ent = 0;  // record, bit 31 set when its triangle covers the tile
    int4 ra, rb, rc, rd;
    no_value(ra, rb, rc, rd);
    if (k < k1) {
      ent = k;
      if (binned) {
        const int e = src.bin(k);
        ent = (e & 0x7FFF) | ((e >> 15) << 31);
      }
      src.fetch(ent & 0x7FFFFFFF, ra, rb, rc, rd);
    }
    const int32_t X[3] = {ra.x, ra.z, rb.x}, Y[3] = {ra.y, ra.w, rb.y};
    // the triangle's pixel box (never empty) clipped to the tile
    const int fx0 = max(rd.x & 0xFFFF, tx0), fy0 = max(rd.y & 0xFFFF, ty0);
    const int bw = min(rd.x >> 16, tx1) - fx0 + 1, bh = min(rd.y >> 16, ty1) - fy0 + 1;
    const int area = ((k < k1) & (bw > 0) & (bh > 0)) ? __mul24(bw, bh) : 0;
    const bool big = area > ((rd.z & 8) ? kSmallMax : 0);  // a wide triangle's edge values need more than 32 bits
    // small triangles: edge values at the centre of pixel (fx0, fy0), and the
    // steps per row and column over 256, dx and -dy, in one register (a narrow
    // triangle's are below 2^15); (E > 0 or E == 0 on a top-left edge) ==
    // (E >= flag bit).  Other lanes' values are unused.
    int E0[3], step2[3];
    {
      const int Px = 256 * fx0 + 128, Py = 256 * fy0 + 128;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int a0 = (e + 1) % 3, b0 = (e + 2) % 3;
        const int32_t dx = X[b0] - X[a0], dy = Y[b0] - Y[a0];
        E0[e] = __mul24(dx, Py - Y[a0]) - __mul24(dy, Px - X[a0]);
        step2[e] = (dx & 0xFFFF) | (-dy << 16);
      }
    }
    // fragments packed over lanes: fragment f belongs to the lane j with
    // off_j <= f < off_j + a_j; per window of 64 fragments each owner marks
    // where its range starts, and the marks up to a fragment count its owner.
    const int a = big ? 0 : area;
    int incl = wave_incl_add(a);
    asm("" : "+v"(incl));  // (else off is summed anew from the scan's parts)
    const int F = __builtin_amdgcn_readlane(incl, 63);
    const int off = incl - a;
    // what a fragment needs of its owner's box: the first pixel in the tile,
    // the width, the edge flags and where the fragments start
    const int box = ((fy0 - ty0) * TS + fx0 - tx0) | (bw << 10) | ((rd.z & 7) << 16) | (off << 19);
    static_assert(TS <= 32 && 64 * kSmallMax < 1 << 13, "fields of box");
    const float rbw = __builtin_amdgcn_rcpf((float)bw);
    const uint32_t keylo = ((uint32_t)rb.z << 24) | ((uint32_t)rc.w & 0xFFFFFFu), keyhi = (uint32_t)rb.z >> 8;
    // The record of the first large triangle of the mask m (of lane 63, which
    // may hold record 0, if there is none: no branch surrounds the load, so
    // nothing waits for it before its first use).  Where records
    // are in memory these are scalar loads: no vector instruction, and
    // neighbouring tiles' waves find the record in the scalar cache; the first
    // one is asked for here, ahead of the fragments, the others one triangle
    // ahead.
    struct LargeRec {
      int4 a, b, c;
      int flags, ent;
    };
    const auto large_rec = [&](uint64_t m) -> LargeRec {
      const int j = (__ffsll((unsigned long long)m) - 1) & 63;
      LargeRec q;
      q.ent = __builtin_amdgcn_readlane(ent, j);
      if constexpr (Src::kUniform) {
        const int4* p = src.rec + 4 * (int64_t)(q.ent & 0x7FFFFFFF);
        q.a = uniform_copy(p);
        q.b = uniform_copy(p + 1);
        q.c = uniform_copy(p + 2);
        q.flags = uniform_ld((const int32_t*)(p + 3) + 2);
      } else {
        const auto rl = [&](int v) { return __builtin_amdgcn_readlane(v, j); };
        q.a = make_int4(rl(ra.x), rl(ra.y), rl(ra.z), rl(ra.w));
        q.b = make_int4(rl(rb.x), rl(rb.y), rl(rb.z), rl(rb.w));
        q.c = make_int4(rl(rc.x), rl(rc.y), rl(rc.z), rl(rc.w));
        q.flags = rl(rd.z);
      }
      return q;
    };
    uint64_t m = __ballot(big);
    LargeRec next = large_rec(m);
    if (F > 0) {
      const uint64_t own = __ballot(a > 0);
      if (a > 0) S.owner[lanes_below(own)] = 4 * lane;
    }
    if (F > 0 && !zused) {
#pragma unroll
      for (int j = 0; j < BH; ++j)
#pragma unroll
        for (int i = 0; i < BW; ++i) zb[zidx(i, j)] = kNoKey;
      zused = true;
    }
    int before = -1;  // owners that start before the window, less one
    for (int f0 = 0; f0 < F; f0 += 64) {
      S.start[lane] = 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      if (a > 0 && off >= f0 && off < f0 + 64) S.start[off - f0] = 1;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const uint64_t starts = __ballot(S.start[lane] != 0);
      // marks up to and at this lane: those below it of the mask less its
      // first bit
      const int first = before + (int)(starts & 1);
      const int nth = __builtin_amdgcn_mbcnt_hi((uint32_t)(starts >> 33),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)(starts >> 1), first));
      before += __popcll(starts);
      const int f = f0 + lane;
      // the owner's values (lanes past F read the last owner's, unused)
      const int j4 = S.owner[nth];
      const auto own = [&](int v) { return __builtin_amdgcn_ds_bpermute(j4, v); };
      const auto ownf = [&](float v) { return __int_as_float(own(__float_as_int(v))); };
      const int jbox = own(box);
      const int rr = f - (int)((uint32_t)jbox >> 19), jbw = (jbox >> 10) & 63;
      // rr / jbw exactly: rr < kSmallMax <= 128 and jbw <= 32 (a box in a
      // tile of at most 32 pixels) keep the quotient's fraction at least
      // 1/64 away from an integer, far above the reciprocal's rounding
      const int qy = (int)(((float)rr + 0.5f) * ownf(rbw));
      const int qx = rr - __mul24(qy, jbw);
      const short2v q2 = __builtin_bit_cast(short2v, qy | (qx << 16));
      const auto edge = [&](int k) {
        return own(E0[k]) + 256 * __builtin_amdgcn_sdot2(__builtin_bit_cast(short2v, own(step2[k])), q2, 0, false);
      };
      const int e0 = edge(0), e1 = edge(1), e2 = edge(2);
      const float z0 = ownf(__int_as_float(rb.w)), z1 = ownf(__int_as_float(rc.x));
      const float z2 = ownf(__int_as_float(rc.y)), invA = ownf(__int_as_float(rc.z));
      const uint64_t key = ((uint64_t)(uint32_t)own((int)keyhi) << 32) | (uint32_t)own((int)keylo);
      if ((f < F) & (e0 >= ((jbox >> 16) & 1)) & (e1 >= ((jbox >> 17) & 1)) & (e2 >= ((jbox >> 18) & 1))) {
        const uint64_t kk = depth_key((float)e0, (float)e1, (float)e2, z0, z1, z2, invA, key);
        const int pp = (jbox & 1023) + qy * TS + qx;
        atomicMin((unsigned long long*)&zb[pp], (unsigned long long)kk);
        if (DBG) atomicAdd(&cov[pp], 1);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    }
    // large triangles: every lane on its own pixels, the record uniform
    while (m) {
      const LargeRec q = next;
      m &= m - 1ull;
      next = large_rec(m);  // on its way while this one is rasterized
      const bool jfull = q.ent < 0;  // uniform
      const int4 qa = q.a, qb = q.b, qc = q.c;
      const int jflags = q.flags;
      const int32_t JX[3] = {qa.x, qa.z, qb.x}, JY[3] = {qa.y, qa.w, qb.y};
      const float z0 = __int_as_float(qb.w), z1 = __int_as_float(qc.x), z2 = __int_as_float(qc.y);
      const float invA = __int_as_float(qc.z);
      const uint64_t key = prim_key(qb.z, (uint32_t)qc.w);
      // one row of the lane's pixels from the edge values E at its first,
      // step per pixel; a pixel is covered if every value reaches thr (0, or
      // 1 on an edge that is not top-left)
      const auto row = [&](auto full, int j, auto E0, auto E1, auto E2, auto s0, auto s1, auto s2) {
#pragma unroll
        for (int i = 0; i < BW; ++i) {
          const int q = j * BW + i;
          const uint64_t kk = depth_key((float)E0, (float)E1, (float)E2, z0, z1, z2, invA, key);
          if constexpr (decltype(full)::value) {
            kreg[q] = kk < kreg[q] ? kk : kreg[q];
            if (DBG) creg[q] += 1;
          } else {
            const bool in = (E0 >= (jflags & 1)) & (E1 >= ((jflags >> 1) & 1)) & (E2 >= ((jflags >> 2) & 1));
            const bool take = in & (kk < kreg[q]);
            const uint32_t hi = take ? (uint32_t)(kk >> 32) : (uint32_t)(kreg[q] >> 32);
            kreg[q] = ((uint64_t)hi << 32) | (take ? (uint32_t)kk : (uint32_t)kreg[q]);
            if (DBG) creg[q] += in ? 1 : 0;
          }
          E0 += s0;
          E1 += s1;
          E2 += s2;
        }
      };
      if (TS <= 16 && (jflags & 8)) {
        // A narrow triangle's edge values stay below 2^31 over the whole of a
        // tile of at most 16 pixels that its box touches: 2 kNarrow (kNarrow
        // + 16 * 256).  The value at the tile's corner and the steps are
        // scalar work, so a lane starts with a multiply-add per axis.
        int E[3], step[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const int a0 = (e + 1) % 3, b0 = (e + 2) % 3;
          const int32_t dx = JX[b0] - JX[a0], dy = JY[b0] - JY[a0];
          const int32_t corner = dx * (256 * ty0 + 128 - JY[a0]) - dy * (256 * tx0 + 128 - JX[a0]);
          step[e] = -256 * dy;
          E[e] = corner + __mul24(by, 256 * dx) + __mul24(BW * bx, step[e]);
        }
        if (jfull) row(std::true_type{}, 0, E[0], E[1], E[2], step[0], step[1], step[2]);
        else row(std::false_type{}, 0, E[0], E[1], E[2], step[0], step[1], step[2]);
      } else {
        // edge values at the lane's first pixel, one pixel right, one row
        // down: exact integers in fp64, so stepping is exact
        double Er[3], step[3], down[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const int a0 = (e + 1) % 3, b0 = (e + 2) % 3;
          const int32_t dx = JX[b0] - JX[a0], dy = JY[b0] - JY[a0];
          Er[e] = fma(-(double)dy, (double)(256 * px0 + 128 - JX[a0]), (double)dx * (double)(256 * py0 + 128 - JY[a0]));
          step[e] = -(double)dy * 256.0;
          down[e] = (double)dx * 256.0;
        }
#pragma unroll
        for (int r = 0; r < BH; ++r) {
          if (jfull) row(std::true_type{}, r, Er[0], Er[1], Er[2], step[0], step[1], step[2]);
          else row(std::false_type{}, r, Er[0], Er[1], Er[2], step[0], step[1], step[2]);
#pragma unroll
          for (int e = 0; e < 3; ++e) Er[e] += down[e];
        }
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // resolve: the fragment z-buffer against the registers, then the winners'
  // colours and the stores, one row of the lane's block at a time
  if (zused) {
#pragma unroll
    for (int j = 0; j < BH; ++j)
#pragma unroll
      for (int i = 0; i < BW; ++i) {
        const uint64_t zk = zb[zidx(i, j)];
        const int q = j * BW + i;
        kreg[q] = zk < kreg[q] ? zk : kreg[q];
      }
  }
#pragma unroll
  for (int j = 0; j < BH; ++j) {
    const int py = py0 + j;
    uint32_t D[BW], rgb[BW];
    int32_t win[BW];
#pragma unroll
    for (int i = 0; i < BW; ++i) {
      const uint64_t key = kreg[j * BW + i];
      const bool hit = key != kNoKey;
      D[i] = hit ? (uint32_t)(key >> 40) : 0xFFFFFFFFu;
      rgb[i] = (uint32_t)key & 0xFFFFFFu;  // the winner's colour travels in its key
      win[i] = hit ? (int32_t)((key >> 24) & 0xFFFFu) : -1;
      if constexpr (SMOOTH) {
        // the key's low bits name the winning record
        if (hit)
          rgb[i] = smooth_color(src.rec, (const float4*)(rs + cam.rs_attr),
                                W.texture ? (const float4*)(rs + cam.rs_tuv) : nullptr, W.texture, W.tpl,
                                (int)rgb[i], px0 + i, py);
      }
    }
    if (py > ty1) continue;
    const uint32_t pix = row0 + (uint32_t)(j * Wd);
    if constexpr (BW == 4) {
      if (px0 + 3 <= tx1) {
        store_four(depth, image, pix, Depth4{{D[0], D[1], D[2], D[3]}},
                   Rgb4{{rgb[0] | (rgb[1] << 24), (rgb[1] >> 8) | (rgb[2] << 16), (rgb[2] >> 16) | (rgb[3] << 8)}});
      } else {
#pragma unroll
        for (int i = 0; i < BW; ++i) {
          if (px0 + i > tx1) continue;
          depth[pix + i] = D[i];
          image[3 * (pix + i)] = (uint8_t)(rgb[i] & 0xFF);
          image[3 * (pix + i) + 1] = (uint8_t)((rgb[i] >> 8) & 0xFF);
          image[3 * (pix + i) + 2] = (uint8_t)((rgb[i] >> 16) & 0xFF);
        }
      }
    } else {
      if (px0 <= tx1) {
        depth[pix] = D[0];
        image[3 * pix] = (uint8_t)(rgb[0] & 0xFF);
        image[3 * pix + 1] = (uint8_t)((rgb[0] >> 8) & 0xFF);
        image[3 * pix + 2] = (uint8_t)((rgb[0] >> 16) & 0xFF);
      }
    }
    if (DBG) {
#pragma unroll
      for (int i = 0; i < BW; ++i) {
        if (px0 + i > tx1) continue;
        W.winners[cam.pix_off + pix + i] = win[i];
        W.coverage[cam.pix_off + pix + i] = cov[zidx(i, j)] + creg[j * BW + i];
      }
    }
  }
}

// A job, a run of tiles of a row, per workgroup of TW waves, which take its
// tiles in turn.  Tiles of 16 pixels could run eight waves per SIMD, but keep to
// seven (and take 69 VGPRs of the 72 that leaves): the eighth slot is where the
// step's and the setup's workgroups start beside a full chip of tiles (an
// iteration of 1,024 envs at 128x128, pipelined: 81.1 us with seven, 89.7 with
// eight, 80.3 with six; 4,096 envs of 2x256x256, bound by the tiles: 2,136,
// 2,103 and 2,238).
template <bool DBG, bool SMOOTH, int TS, int TW>
__global__ void __launch_bounds__(64 * TW)
    __attribute__((amdgpu_waves_per_eu(TS == 16 && !DBG ? 7 : 1, TS == 16 && !DBG ? 7 : 8)))
    raster_tile_kernel(WorldDev W, RasterLaunch L) {
  __shared__ TileWaveLDS<TS> S[TW];
  __shared__ int32_t C[DBG ? TW : 1][DBG ? TS * TS : 1];
  // beside the step's kernels, a higher issue priority keeps the render
  // (the longer phase) from stretching
  switch (L.prio) {
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 3: __builtin_amdgcn_s_setprio(3); break;
    default: break;
  }
  // A wave's bookkeeping is uniform and takes three rounds of loads (the job,
  // the camera, then the image's header and the bin ranges of the first tiles
  // together) before the first bin entry is read.
  const int2 job = uniform_ld(L.tiles + blockIdx.x);
  if (job.x < 0) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int last = job.x >> kJobTilesShift;  // of the job's tiles
  if (wave > last) return;  // past the row's last tile; no workgroup barrier follows
  const CamDev* cp = W.cams + (job.x & kJobCamMask);
  CamDev cam;  // the fields the tile pass reads
  cam.w = uniform_ld(&cp->w);
  cam.h = uniform_ld(&cp->h);
  cam.pix_off = uniform_ld(&cp->pix_off);
  cam.rs_off = uniform_ld(&cp->rs_off);
  cam.rs_recs = uniform_ld(&cp->rs_recs);
  cam.rs_bins = uniform_ld(&cp->rs_bins);
  cam.rs_total = uniform_ld(&cp->rs_total);
  cam.rs_attr = uniform_ld(&cp->rs_attr);
  cam.rs_tuv = uniform_ld(&cp->rs_tuv);
  const int ntx = (cam.w + TS - 1) / TS;
  const int tx = job.y & 0xFFFF, ty = job.y >> 16;
  const unsigned char* rs = W.rscratch + cam.rs_off + (int64_t)L.parity * cam.rs_total;
  // the tile table has room for the image's tiles at the smallest tile
  // edge, so its entries are read before the header says the image is binned
  const int2 hdr = uniform_ld((const int2*)rs);
  const int2* table = (const int2*)(rs + 64) + (ty * ntx + tx);
  // The bin ranges of a run's next two tiles are asked for ahead of their turn,
  // but for 8-pixel tiles, whose single ones lost more by the extra loads (a wait
  // for a scalar load takes in every one under way) than runs gained: 5,600
  // images of 64x64 in single tiles 144 us ahead and 137 not, in runs 127 and 120;
  // 400 of 256x256 153 and 143, 125 and 119.
  constexpr bool kAhead = TS > 8;
  int2 te = uniform_ld(table + wave), next = te;
  if constexpr (kAhead) next = uniform_ld(table + min(wave + TW, last));
  const bool binned = hdr.y != 0;
  const GlobalRecs<true> src{(const int4*)(rs + cam.rs_recs), (const uint16_t*)(rs + cam.rs_bins)};
  for (int t = wave;; t += TW) {
    int2 after = te;
    if constexpr (kAhead) after = uniform_ld(table + min(t + 2 * TW, last));
    const int k0 = binned ? te.x : 0, k1 = binned ? te.x + te.y : hdr.x;
    raster_tile<DBG, SMOOTH, TS>(W, cam, src, binned, k0, k1, tx + t, ty, S[wave], DBG ? C[wave] : nullptr, rs);
    if (t + TW > last) return;
    te = kAhead ? next : uniform_ld(table + t + TW);
    next = after;
  }
}

// The tiles wave, wave + nw, ... of an image whose setup is done, from
// records and bins in src.
template <bool DBG, int TS, class Src>
__device__ __forceinline__ void fused_tiles(const WorldDev& W, const CamDev& cam, const Src& src, bool binned,
                                            int nrec, const int32_t* toff, const int32_t* tend, int wave,
                                            int nw, TileWaveLDS<TS>* S, int32_t* C, const unsigned char* rs) {
  static_assert(!Src::kUniform, "the records are written by this kernel");
  const int ntx = (cam.w + TS - 1) / TS, ntiles = ntx * ((cam.h + TS - 1) / TS);
  for (int t = wave; t < ntiles; t += nw) {
    const int k0 = binned ? toff[t] : 0, k1 = binned ? tend[t] : nrec;
    raster_tile<DBG, false, TS>(W, cam, src, binned, k0, k1, t % ntx, t / ntx, S[wave],
                                DBG ? C + wave * TS * TS : nullptr, rs);
  }
}

// Setup and tiles of one image per workgroup (flat shading, no near-plane
// clipping): the setup pass as above, then every wave rasterizes tiles
// wave, wave + nw, ... of the image from the records and bins in LDS, its
// z-buffer in the setup-only region.  Records and bins that do not fit go
// through the raster scratch instead, with the same results.
template <bool DBG, int TS>
__global__ void __launch_bounds__(1024) raster_fused_kernel(WorldDev W, RasterLaunch L) {
  extern __shared__ __align__(16) unsigned char lds[];
  const SetupLayout Lo = setup_layout(L.max_bodies, L.max_verts, L.max_tiles, L.max_tris, false, (int)blockDim.x,
                                      L.tpl_words, L.lds_zone0, L.lrec_cap, L.lbin_cap);
  const int nw = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  TileWaveLDS<TS>* S = (TileWaveLDS<TS>*)lds;
  int32_t* C = (int32_t*)(lds + nw * sizeof(TileWaveLDS<TS>));  // debug coverage, TS * TS per wave
  int32_t* misc = (int32_t*)(lds + Lo.misc);
  const int32_t* toff = (const int32_t*)(lds + Lo.tiles) + Lo.tw;
  const int32_t* tend = toff + Lo.tw + 1;
  int wi = (int)blockIdx.x;
  for (;;) {
    if (L.persistent > 0) {
      __syncthreads();
      if (threadIdx.x == 0) misc[4] = atomicAdd(L.queue, 1);
      __syncthreads();
      wi = misc[4];
    }
    if (wi >= L.n_work) return;
    const int cam_id = uniform_ld(L.work + wi);
    setup_image<false, true>(lds, Lo, W, L, cam_id);
    __syncthreads();
    const CamDev cam = uniform_copy(W.cams + cam_id);
    const int nrec = misc[2], mode = misc[6];
    const bool binned = (mode & 2) != 0;
    const unsigned char* rs = W.rscratch + cam.rs_off + (int64_t)L.parity * cam.rs_total;
    if (mode & 1) {
      const LdsRecs src{(const int4*)(lds + Lo.lrec), (const int2*)(lds + Lo.vxy), (const float*)(lds + Lo.vz),
                        (const uint16_t*)(lds + Lo.lbin), cam.w, cam.h};
      fused_tiles<DBG, TS>(W, cam, src, binned, nrec, toff, tend, wave, nw, S, C, rs);
    } else {
      const GlobalRecs<false> src{(const int4*)(rs + cam.rs_recs), (const uint16_t*)(rs + cam.rs_bins)};
      fused_tiles<DBG, TS>(W, cam, src, binned, nrec, toff, tend, wave, nw, S, C, rs);
    }
    if (L.persistent == 0) return;
    __syncthreads();  // the next image's setup reuses the LDS
  }
}

}  // namespace

size_t raster_lds_bytes(const RasterLaunch& l) {
  return (size_t)setup_layout(l.max_bodies, l.max_verts, l.max_tiles, l.max_tris, l.near_clip != 0, l.threads,
                              l.tpl_words)
      .total;
}

// The fused kernel's LDS for workgroups of l.threads: the tile pass's
// z-buffers (and debug coverage) over the setup-only region, and as many
// compact records as LDS allows up to half the primitives plus 64 (a convex
// closed mesh seen from outside shows at most about half its faces), with
// four bin entries each (at most max_recs records if max_recs > 0); 0 if
// fewer than min(64, max_recs) fit.
size_t raster_fused_plan(RasterLaunch* l, bool debug, int max_recs) {
  const int ts = 1 << l->tile_shift;
  const int nw = l->threads / 64;
  const size_t wave_lds = ts == 8 ? sizeof(TileWaveLDS<8>) : ts == 32 ? sizeof(TileWaveLDS<32>)
                                                                       : sizeof(TileWaveLDS<16>);
  l->lds_zone0 = (int32_t)(nw * (wave_lds + (debug ? 4 * ts * ts : 0)));
  int cap = (l->max_tris + 1) / 2 + 64;
  if (max_recs > 0 && max_recs < cap) cap = max_recs;
  for (const int least = cap < 64 ? cap : 64; cap >= least; cap /= 2) {
    const SetupLayout Lo = setup_layout(l->max_bodies, l->max_verts, l->max_tiles, l->max_tris, false, l->threads,
                                        l->tpl_words, l->lds_zone0, cap, 4 * cap);
    if (Lo.total <= kFusedLdsMax) {
      l->lrec_cap = cap;
      l->lbin_cap = 4 * cap;
      return (size_t)Lo.total;
    }
  }
  return 0;
}

hipError_t raster_fused_configure(size_t lds_bytes) {
  const void* k[] = {(const void*)raster_fused_kernel<false, 8>, (const void*)raster_fused_kernel<false, 16>,
                     (const void*)raster_fused_kernel<false, 32>, (const void*)raster_fused_kernel<true, 8>,
                     (const void*)raster_fused_kernel<true, 16>, (const void*)raster_fused_kernel<true, 32>};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool DBG>
static const void* fused_fn(int tile_shift) {
  if (tile_shift == 3) return (const void*)raster_fused_kernel<DBG, 8>;
  if (tile_shift == 5) return (const void*)raster_fused_kernel<DBG, 32>;
  return (const void*)raster_fused_kernel<DBG, 16>;
}

template <bool DBG>
static void launch_fused(const WorldDev& w, const RasterLaunch& l, int grid, size_t lds, hipStream_t s,
                         LaunchEvents* ev) {
  const dim3 g(grid), b(l.threads);
  if (l.tile_shift == 3) timed_launch(ev, true, true, raster_fused_kernel<DBG, 8>, g, b, (uint32_t)lds, s, w, l);
  else if (l.tile_shift == 5) timed_launch(ev, true, true, raster_fused_kernel<DBG, 32>, g, b, (uint32_t)lds, s, w, l);
  else timed_launch(ev, true, true, raster_fused_kernel<DBG, 16>, g, b, (uint32_t)lds, s, w, l);
}

hipError_t launch_raster_fused(const WorldDev& w, const RasterLaunch& l0, size_t lds, hipStream_t s,
                               LaunchEvents* ev) {
  if (l0.n_work <= 0) return hipSuccess;
  RasterLaunch l = l0;
  int grid = l.n_work;
  if (l.persistent != 0) {
    hipError_t e = persistent_grid(l.persistent, l.n_work, w.winners ? fused_fn<true>(l.tile_shift)
                                                                     : fused_fn<false>(l.tile_shift),
                                   l.threads, lds, &grid);
    if (e != hipSuccess) return e;
    l.persistent = grid;  // the kernel only tells 0 from the rest
    e = launch_reset_queue(l.queue, s);
    if (e != hipSuccess) return e;
  }
  if (w.winners) launch_fused<true>(w, l, grid, lds, s, ev);
  else launch_fused<false>(w, l, grid, lds, s, ev);
  return hipGetLastError();
}

hipError_t raster_configure(size_t lds_bytes) {
  const hipError_t e = hipFuncSetAttribute((const void*)raster_setup_kernel<false>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)raster_setup_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds_bytes);
}

hipError_t launch_raster_setup(const WorldDev& w, const RasterLaunch& l0, hipStream_t s, LaunchEvents* ev) {
  if (l0.n_work <= 0) return hipSuccess;
  RasterLaunch l = l0;
  const size_t lds = raster_lds_bytes(l);
  int grid = l.n_work;
  if (l.persistent != 0) {
    hipError_t e = persistent_grid(l.persistent, l.n_work,
                                   l.near_clip ? (const void*)raster_setup_kernel<true>
                                               : (const void*)raster_setup_kernel<false>,
                                   l.threads, lds, &grid);
    if (e != hipSuccess) return e;
    l.persistent = grid;  // the kernel only tells 0 from the rest
    e = launch_reset_queue(l.queue, s);
    if (e != hipSuccess) return e;
  }
  if (l.near_clip)
    timed_launch(ev, true, true, raster_setup_kernel<true>, dim3(grid), dim3(l.threads), (uint32_t)lds, s, w, l);
  else
    timed_launch(ev, true, true, raster_setup_kernel<false>, dim3(grid), dim3(l.threads), (uint32_t)lds, s, w, l);
  return hipGetLastError();
}

template <int TS, int TW>
static void launch_tiles(const WorldDev& w, const RasterLaunch& l, hipStream_t s, LaunchEvents* ev) {
  const dim3 g(l.n_tile_groups), b(64 * TW);
  if (l.smooth) {
    if (w.winners) timed_launch(ev, true, true, raster_tile_kernel<true, true, TS, TW>, g, b, 0, s, w, l);
    else timed_launch(ev, true, true, raster_tile_kernel<false, true, TS, TW>, g, b, 0, s, w, l);
  } else {
    if (w.winners) timed_launch(ev, true, true, raster_tile_kernel<true, false, TS, TW>, g, b, 0, s, w, l);
    else timed_launch(ev, true, true, raster_tile_kernel<false, false, TS, TW>, g, b, 0, s, w, l);
  }
}

template <int TS>
static void launch_tiles(const WorldDev& w, const RasterLaunch& l, hipStream_t s, LaunchEvents* ev) {
  if (l.tile_waves == 1) launch_tiles<TS, 1>(w, l, s, ev);
  else if (l.tile_waves == 2) launch_tiles<TS, 2>(w, l, s, ev);
  else launch_tiles<TS, 4>(w, l, s, ev);
}

hipError_t launch_raster_tiles(const WorldDev& w, const RasterLaunch& l, hipStream_t s, LaunchEvents* ev) {
  if (l.n_tile_groups <= 0) return hipSuccess;
  if (l.tile_shift == 3) launch_tiles<8>(w, l, s, ev);
  else if (l.tile_shift == 5) launch_tiles<32>(w, l, s, ev);
  else launch_tiles<16>(w, l, s, ev);
  return hipGetLastError();
}

}  // namespace vuda
