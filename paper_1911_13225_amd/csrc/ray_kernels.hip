// Ray bookkeeping kernels: generation and unit-sphere initialisation, the
// coarse-to-fine split, finalisation of the rendered
// maps, normals, and the gradient-sample list of the backward pass.  All of
// them are memory-bound (a few tens of bytes per ray) and use wave64 ballots
// with one atomic per workgroup for list appends.
#include <algorithm>

#include "dist_internal.h"
#include "ray_kernels.h"

namespace dist {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
// Append `value` to list for every thread with flag set; one atomic per
// block of NT threads.  Must be called by all threads of the block.  Returns the
// list position of a flagged thread's entry (-1 for the others); the entry at
// position i is stored at list[dir * i], so dir = -1 fills backwards from the
// element `list` points at.
template <int NT = 256>
__device__ __forceinline__ int block_append(bool flag, int value, int* list, int* counter, int dir = 1) {
  __shared__ int wcnt[NT / 64];
  __shared__ int base;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long m = __ballot(flag);
  const int within = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) wcnt[w] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) tot += wcnt[i];
    base = tot ? atomicAdd(counter, tot) : 0;
  }
  __syncthreads();
  int off = base;
  for (int i = 0; i < w; ++i) off += wcnt[i];
  if (flag) list[dir * (off + within)] = value;
  __syncthreads();
  return flag ? off + within : -1;
}

// Level-`lvl` ray through the centre of block (U, V): unit world direction and
// the normalised image coordinates (xt, yt) = K^-1 (x, y) of that centre.
__device__ __forceinline__ void level_ray(const ImgDesc& im, int lvl, int U, int V, float3& d, float& xt, float& yt) {
  const float sc = (float)(1 << lvl);
  const float u = sc * (float)U + 0.5f * sc;
  const float v = sc * (float)V + 0.5f * sc;
  xt = (u - im.cx) / im.fx;
  yt = (v - im.cy) / im.fy;
  const float nrm = sqrtf(xt * xt + yt * yt + 1.f);
  const float a = xt / nrm, b = yt / nrm, c = 1.f / nrm;
  d.x = im.R[0] * a + im.R[1] * b + im.R[2] * c;
  d.y = im.R[3] * a + im.R[4] * b + im.R[5] * c;
  d.z = im.R[6] * a + im.R[7] * b + im.R[8] * c;
}

// Unit-sphere interval of the ray c + t d (Sec. 3.2 initialisation).
__device__ __forceinline__ bool sphere_interval(const ImgDesc& im, float3 d, float& t_lo, float& t_hi) {
  const float b = im.c[0] * d.x + im.c[1] * d.y + im.c[2] * d.z;
  const float cc = im.c[0] * im.c[0] + im.c[1] * im.c[1] + im.c[2] * im.c[2];
  const float disc = b * b - (cc - 1.f);
  const float sq = sqrtf(fmaxf(disc, 0.f));
  t_lo = fmaxf(-b - sq, im.near_);
  t_hi = fminf(-b + sq, im.far_);
  // the camera is outside the sphere, so both roots share a sign: the ray
  // meets the sphere only if they lie ahead of it (b < 0)
  return disc > 0.f && b < 0.f;
}

// Distance from the origin to the ray c + t v, t >= 0 (b = c . v): the foot of
// the perpendicular if it lies ahead, else the camera centre (App. A.3).
__device__ __forceinline__ float ray_origin_distance(float cc, float b) {
  return b < 0.f ? sqrtf(fmaxf(cc - b * b, 0.f)) : sqrtf(cc);
}

__device__ __forceinline__ void init_ray(const RayPool& pl, const ImgDesc& im, int img, int r, float3 d, float t,
                                         float t_lo, float t_hi, bool inside, int step) {
  pl.d[r] = make_float4(d.x, d.y, d.z, t);
  pl.b[r] = make_float2(t_lo, t_hi);
  pl.img[r] = img;
  pl.st[r] = inside ? ST_ACTIVE : ST_MISS;
  pl.n[r] = (uint8_t)step;
  pl.flast[r] = 0.f;
  for (int k = 0; k < im.K; ++k) {
    pl.rec_f[(size_t)k * pl.cap + r] = INFINITY;
    pl.rec_t[(size_t)k * pl.cap + r] = 0.f;
    pl.rec_n[(size_t)k * pl.cap + r] = 0;
  }
}

// ---------------------------------------------------------------------------
// Coarsest level: one ray per 2^L x 2^L block, starting at the sphere entry.
// grid: (blocks over rays of the largest image, n_images)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init_level(RayPool pl, const ImgDesc* imgs, int* list,
                                                    int* counter) {
  const int img = blockIdx.y;
  const ImgDesc& im = imgs[img];
  const int lvl = im.levels;
  const int Wl = im.W >> lvl, Hl = im.H >> lvl;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool act = false;
  int r = 0;
  if (i < Wl * Hl) {
    const int V = i / Wl, U = i - V * Wl;
    float3 d;
    float xt, yt, t_lo, t_hi;
    level_ray(im, lvl, U, V, d, xt, yt);
    const bool inside = sphere_interval(im, d, t_lo, t_hi);
    r = im.slot_base + im.lvl_off[lvl] + i;
    init_ray(pl, im, img, r, d, t_lo, t_lo, t_hi, inside, 0);
    act = inside;
  }
  block_append(act, r, list, counter);
}

// ---------------------------------------------------------------------------
// Coarse-to-fine split (Sec. 3.2, Fig. 3a): every ray of level lvl+1 becomes
// four rays of level lvl.  A child starts from the parent's t clamped into its
// own unit-sphere interval (from its own entry if the parent missed) and is
// re-activated whatever the parent's state; its records start empty.
// With counter_tail the list is filled from both ends: children of rays that
// graze the surface (the ones that need the most further steps) from the
// front, the others backwards from list[tail_end - 1], so a consumer that
// takes the rays in order starts the long ones first.  A ray still marching at
// the split grazes if the march left |flast| < kGraze (f'' f - f'^2 / 2 of its
// last three queries): a tenth of the rays, where "still marching" held for
// half of them, and 98-99% of those that take more than 12 further steps.
// March of 4 x 256^2 (bf16): see k_march_run.
// ---------------------------------------------------------------------------
constexpr float kGraze = 0.02f;

__global__ __launch_bounds__(1024) void k_split(RayPool pl, const ImgDesc* imgs, int child_lvl, int child_step,
                                               int* list, int* counter, int* counter_tail,
                                               int tail_end) {
  const int img = blockIdx.y;
  const ImgDesc& im = imgs[img];
  const int Wl = im.W >> child_lvl, Hl = im.H >> child_lvl;
  const int Wp = im.W >> (child_lvl + 1);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool act = false, longest = false;
  int r = 0;
  if (i < Wl * Hl) {
    const int V = i / Wl, U = i - V * Wl;
    float3 d;
    float xt, yt, t_lo, t_hi;
    level_ray(im, child_lvl, U, V, d, xt, yt);
    const bool inside = sphere_interval(im, d, t_lo, t_hi);
    const int pr = im.slot_base + im.lvl_off[child_lvl + 1] + (V >> 1) * Wp + (U >> 1);
    const uint8_t pst = pl.st[pr];
    const float tp = pst == ST_MISS ? t_lo : pl.d[pr].w;
    const float t = fminf(fmaxf(tp, t_lo), t_hi);
    r = im.slot_base + im.lvl_off[child_lvl] + i;
    init_ray(pl, im, img, r, d, t, t_lo, t_hi, inside, child_step);
    act = inside;
    longest = counter_tail && pst == ST_ACTIVE && fabsf(pl.flast[pr]) < kGraze;
  }
  // 1024-thread blocks: a quarter of the atomics on the list counters
  if (counter_tail) {
    block_append<1024>(act && longest, r, list, counter);
    block_append<1024>(act && !longest, r, list + tail_end - 1, counter_tail, -1);
  } else {
    block_append<1024>(act, r, list, counter);
  }
}

// ---------------------------------------------------------------------------
// Finalise level-0 rays into the output maps (Sec. 3.3, App. A.3).
// grid: (1024-pixel blocks over H*W, n_images); one list atomic per block
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_finalize(RayPool pl, const ImgDesc* imgs, const int* imgs_list,
                                                  FinalizeOut o) {
  const int img = imgs_list ? imgs_list[blockIdx.y] : blockIdx.y;
  const ImgDesc& im = imgs[img];
  const int hw = im.H * im.W;
  const int pix = blockIdx.x * blockDim.x + threadIdx.x;
  bool hit = false;
  int r = 0;
  if (pix < hw) {
    r = im.slot_base + im.lvl_off[0] + pix;
    const uint8_t st = pl.st[r];
    const size_t q = (size_t)im.out_base + pix;
    const int V = pix / im.W, U = pix - V * im.W;
    float3 dd;
    float xt, yt;
    level_ray(im, 0, U, V, dd, xt, yt);
    const float4 d = pl.d[r];
    hit = st == ST_HIT;
    float depth = INFINITY, dist = INFINITY, sil;
    if (hit) {
      dist = d.w + pl.flast[r];
      depth = dist / sqrtf(xt * xt + yt * yt + 1.f);
    }
    if (st == ST_MISS) {
      const float b = im.c[0] * d.x + im.c[1] * d.y + im.c[2] * d.z;
      const float cc = im.c[0] * im.c[0] + im.c[1] * im.c[1] + im.c[2] * im.c[2];
      sil = ray_origin_distance(cc, b) - 1.f;
    } else if (st == ST_ERROR) {
      sil = INFINITY;                      // a non-finite query: background
    } else {
      sil = fabsf(pl.rec_f[r]) - im.eps;
    }
    if (o.depth) o.depth[q] = depth;
    if (o.dist) o.dist[q] = dist;
    if (o.sil) o.sil[q] = sil;
    if (o.status) o.status[q] = st;
    if (o.nsteps) o.nsteps[q] = st == ST_MISS ? 0 : pl.n[r];
    if (o.normal && !hit) { o.normal[3 * q] = 0.f; o.normal[3 * q + 1] = 0.f; o.normal[3 * q + 2] = 0.f; }
    if (o.nraw) o.nraw[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (o.queries && blockIdx.x == 0 && threadIdx.x == 0) o.queries[blockIdx.y] = (int64_t)o.qcount[blockIdx.y];
  const int h = block_append<1024>(hit && o.want_hits, r, o.hits, o.hit_count);
  if (o.hit_pix && pix < hw) o.hit_pix[(size_t)im.out_base + pix] = h;
}

// Normals from the six central-difference queries of each hit (Sec. 3.3).
__global__ void k_normals(const RayPool pl, const ImgDesc* imgs, const int* hits, const int* hit_count,
                          const float* fv, float delta, float* normal, float4* nraw) {
  const int h = blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= *hit_count) return;
  const int r = hits[h];
  const ImgDesc& im = imgs[pl.img[r]];
  const int pix = r - im.slot_base - im.lvl_off[0];
  const size_t q = (size_t)im.out_base + pix;
  const float* f = fv + 6ll * h;
  const float inv = 1.f / (2.f * delta);
  const float nx = (f[0] - f[1]) * inv, ny = (f[2] - f[3]) * inv, nz = (f[4] - f[5]) * inv;
  const float len = sqrtf(nx * nx + ny * ny + nz * nz);
  if (nraw) nraw[q] = make_float4(nx, ny, nz, len);
  if (normal) {
    const float s = len > 0.f ? 1.f / len : 0.f;
    normal[3 * q] = nx * s;
    normal[3 * q + 1] = ny * s;
    normal[3 * q + 2] = nz * s;
  }
}

// ---------------------------------------------------------------------------
// Backward: gradient samples (Sec. 3.4 Eq. 2 first term; App. B.2)
// ---------------------------------------------------------------------------
struct PixSamples {
  int nd, base, nn;      // depth records used, samples at records, normal samples
};

__device__ __forceinline__ PixSamples pixel_samples(const RayPool& pl, const ImgDesc& im, int r, size_t q,
                                                    const SeedIn& in) {
  PixSamples ps{0, 0, 0};
  const uint8_t st = pl.st[r];
  if (st == ST_MISS || st == ST_ERROR) return ps;     // no samples on a ray that met a non-finite query
  const float gd = in.g_depth ? in.g_depth[q] : 0.f;
  const float gs = in.g_sil ? in.g_sil[q] : 0.f;
  if (in.hit_mode) {
    ps.base = (st == ST_HIT && gd != 0.f) ? 1 : 0;
    return ps;
  }
  if (in.imp_gv) {
    // silhouette sample at the minimum-|f| query, depth sample at the Eq. 1 point
    ps.base = ((gs != 0.f && pl.rec_f[r] != INFINITY) ? 1 : 0) + ((st == ST_HIT && gd != 0.f && in.imp_gv[q] != 0.f) ? 1 : 0);
  } else if (st == ST_HIT && gd != 0.f) {
    for (int k = 0; k < im.K; ++k) ps.nd += (pl.rec_f[(size_t)k * pl.cap + r] != INFINITY) ? 1 : 0;
  }
  if (!in.imp_gv) {
    const int ns = (gs != 0.f && pl.rec_f[r] != INFINITY) ? 1 : 0;
    ps.base = ps.nd > ns ? ps.nd : ns;
  }
  if (st == ST_HIT && in.g_normal && in.nraw) {
    const float* g = in.g_normal + 3 * q;
    if ((g[0] != 0.f || g[1] != 0.f || g[2] != 0.f) && in.nraw[q].w > 0.f) ps.nn = 6;
  }
  return ps;
}

// Per block of 256 pixels: the number of gradient samples.  With bsum2 (the
// split layout) the record samples and the normal-stencil samples are counted
// for two separate lists; otherwise a pixel's stencil samples follow its
// record samples in one list.
__global__ __launch_bounds__(256) void k_samples_count(RayPool pl, const ImgDesc* imgs, const int* img_order,
                                                       SeedIn in, int* bsum, int* bsum2) {
  __shared__ int red[256], red2[256];
  const int img = img_order[blockIdx.y];
  const ImgDesc& im = imgs[img];
  const int hw = im.H * im.W;
  const int pix = blockIdx.x * 256 + threadIdx.x;
  int c = 0, c2 = 0;
  if (pix < hw) {
    const PixSamples ps = pixel_samples(pl, im, im.slot_base + im.lvl_off[0] + pix, (size_t)im.out_base + pix, in);
    c = bsum2 ? ps.base : ps.base + ps.nn;
    c2 = ps.nn;
  }
  red[threadIdx.x] = c;
  red2[threadIdx.x] = c2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      red[threadIdx.x] += red[threadIdx.x + s];
      red2[threadIdx.x] += red2[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    bsum[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
    if (bsum2) bsum2[blockIdx.y * gridDim.x + blockIdx.x] = red2[0];
  }
}

// One workgroup: exclusive scan of the block sums in image order, restarting
// the padding at every latent segment so that each segment starts at a
// multiple of the adjoint tile.  seg_* are indexed by latent id.  The list
// starts at *pos0 (0 if null); n_out[0] receives its end, n_out[1] its length.
// The padding samples at the end of a segment are written here: zero seed, the
// segment's latent; stencil index 0 (split layout), a valid entry whose
// contribution the zero seed cancels.
struct PadOut {
  float4* samples;
  int* sample_lat;
  int* sample_idx;                 // each of the last three may be null
  int4* sample_cam;
  float4* cseed;
};
__global__ __launch_bounds__(1024) void k_samples_scan(const int* bsum, int n_img, int bpi, const int* img_order,
                                                       const int* img_latent, int lat_fixed, int tile, int n_lat,
                                                       int* boff, int* seg_base, int* seg_total, int* seg_padded,
                                                       const int* pos0, int* n_out, PadOut out) {
  __shared__ int buf[1024];
  __shared__ int carry_s;
  const int tid = threadIdx.x;
  const int start = pos0 ? *pos0 : 0;
  for (int l = tid; l < n_lat; l += 1024) { seg_base[l] = start; seg_total[l] = 0; seg_padded[l] = 0; }
  __syncthreads();
  int pos = start;          // running padded offset (uniform)
  int i0 = 0;
  while (i0 < n_img) {
    const int lat = img_latent ? img_latent[img_order[i0]] : lat_fixed;
    int i1 = i0;
    while (i1 < n_img && (img_latent ? img_latent[img_order[i1]] : lat_fixed) == lat) ++i1;
    // scan blocks of images [i0, i1)
    const int nb = (i1 - i0) * bpi;
    const int b0 = i0 * bpi;
    if (tid == 0) carry_s = 0;
    __syncthreads();
    for (int c0 = 0; c0 < nb; c0 += 1024) {
      const int v = (c0 + tid < nb) ? bsum[b0 + c0 + tid] : 0;
      buf[tid] = v;
      __syncthreads();
      for (int off = 1; off < 1024; off <<= 1) {
        const int x = tid >= off ? buf[tid - off] : 0;
        __syncthreads();
        buf[tid] += x;
        __syncthreads();
      }
      const int carry = carry_s;
      if (c0 + tid < nb) boff[b0 + c0 + tid] = pos + carry + buf[tid] - v;
      __syncthreads();
      if (tid == 1023) carry_s = carry + buf[1023];
      __syncthreads();
    }
    const int total = carry_s;
    const int padded = (total + tile - 1) / tile * tile;
    if (tid == 0) { seg_base[lat] = pos; seg_total[lat] = total; seg_padded[lat] = padded; }
    for (int i = pos + total + tid; i < pos + padded; i += 1024) {
      out.samples[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      out.sample_lat[i] = lat;
      if (out.sample_idx) out.sample_idx[i] = 0;
      if (out.sample_cam) out.sample_cam[i] = make_int4(-1, 0, 0, 0);
      if (out.cseed) out.cseed[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    pos += padded;
    i0 = i1;
    __syncthreads();
  }
  if (tid == 0) {
    n_out[0] = pos;
    n_out[1] = pos - start;
  }
}

// Block-wide exclusive prefix of c over the 256 threads (all threads call).
__device__ __forceinline__ int block_excl_scan(int c, int* buf) {
  buf[threadIdx.x] = c;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const int x = threadIdx.x >= off ? buf[threadIdx.x - off] : 0;
    __syncthreads();
    buf[threadIdx.x] += x;
    __syncthreads();
  }
  return buf[threadIdx.x] - c;
}

// Writes each pixel's samples at the offsets of the scans.  With boff2 (split
// layout) the stencil samples go to the second list, each with its stencil
// index 6 h + j (h = the pixel's hit index in the forward's hit list), so that
// their adjoint can use the masks the forward kept.
__global__ __launch_bounds__(256) void k_samples_write(RayPool pl, const ImgDesc* imgs, const int* img_order,
                                                       SeedIn in, const int* boff, const int* boff2, float4* samples,
                                                       int* sample_lat, int* sample_idx, int4* sample_cam) {
  __shared__ int buf[256];
  const int img = img_order[blockIdx.y];
  const ImgDesc& im = imgs[img];
  const int hw = im.H * im.W;
  const int pix = blockIdx.x * 256 + threadIdx.x;
  PixSamples ps{0, 0, 0};
  int r = 0;
  size_t q = 0;
  if (pix < hw) {
    r = im.slot_base + im.lvl_off[0] + pix;
    q = (size_t)im.out_base + pix;
    ps = pixel_samples(pl, im, r, q, in);
  }
  const int blk = blockIdx.y * gridDim.x + blockIdx.x;
  const int c = boff2 ? ps.base : ps.base + ps.nn;
  int o = boff[blk] + block_excl_scan(c, buf);
  int o2 = 0;
  if (boff2) {
    __syncthreads();
    o2 = boff2[blk] + block_excl_scan(ps.nn, buf);
  }
  if (ps.base + ps.nn == 0) return;
  const float4 d = pl.d[r];
  const float cx = im.c[0], cy = im.c[1], cz = im.c[2];
  const int V = pix / im.W, U = pix - V * im.W;
  float3 dd;
  float xt, yt;
  level_ray(im, 0, U, V, dd, xt, yt);
  const float gd = in.g_depth ? in.g_depth[q] : 0.f;
  const float gs = in.g_sil ? in.g_sil[q] : 0.f;
  const float dseed = im.alpha * gd / sqrtf(xt * xt + yt * yt + 1.f);
  const float dist_eq1 = d.w + pl.flast[r];
  if (in.hit_mode || in.imp_gv) {
    const float f0 = pl.rec_f[r];
    if (in.imp_gv && gs != 0.f && f0 != INFINITY) {
      const float t0 = pl.rec_t[r];
      samples[o] = make_float4(fmaf(t0, d.x, cx), fmaf(t0, d.y, cy), fmaf(t0, d.z, cz),
                               gs * (f0 > 0.f ? 1.f : (f0 < 0.f ? -1.f : 0.f)));
      sample_lat[o] = im.latent;
      if (sample_cam) sample_cam[o] = make_int4(img, pix, __float_as_int(t0), 0);
      ++o;
    }
    const bool dep = pl.st[r] == ST_HIT && gd != 0.f && (in.hit_mode || in.imp_gv[q] != 0.f);
    if (dep) {
      const float seed = in.hit_mode ? 1.f : -gd / sqrtf(xt * xt + yt * yt + 1.f) / in.imp_gv[q];
      samples[o] = make_float4(fmaf(dist_eq1, d.x, cx), fmaf(dist_eq1, d.y, cy), fmaf(dist_eq1, d.z, cz), seed);
      sample_lat[o] = im.latent;
      if (sample_cam) sample_cam[o] = make_int4(img, pix, __float_as_int(dist_eq1), 0);
      ++o;
    }
  }
  for (int k = 0; k < ((in.hit_mode || in.imp_gv) ? 0 : ps.base); ++k) {
    const float tk = pl.rec_t[(size_t)k * pl.cap + r];
    float seed = k < ps.nd ? dseed : 0.f;
    if (k == 0 && gs != 0.f) {
      const float f0 = pl.rec_f[r];
      seed += gs * (f0 > 0.f ? 1.f : (f0 < 0.f ? -1.f : 0.f));
    }
    samples[o] = make_float4(fmaf(tk, d.x, cx), fmaf(tk, d.y, cy), fmaf(tk, d.z, cz), seed);
    sample_lat[o] = im.latent;
    if (sample_cam) sample_cam[o] = make_int4(img, pix, __float_as_int(tk), 0);
    ++o;
  }
  if (ps.nn) {
    const float4 nr = in.nraw[q];
    const float inv = 1.f / nr.w;
    const float nx = nr.x * inv, ny = nr.y * inv, nz = nr.z * inv;
    const float* g = in.g_normal + 3 * q;
    const float gn = g[0] * nx + g[1] * ny + g[2] * nz;
    const float gv[3] = {(g[0] - gn * nx) * inv, (g[1] - gn * ny) * inv, (g[2] - gn * nz) * inv};
    const float dist = d.w + pl.flast[r];
    const float p[3] = {fmaf(dist, d.x, cx), fmaf(dist, d.y, cy), fmaf(dist, d.z, cz)};
    const float s2 = 1.f / (2.f * in.delta);
    const int h = boff2 ? in.hit_pix[q] : 0;
    for (int j = 0; j < 6; ++j) {
      const int ax = j >> 1;
      float qv[3] = {p[0], p[1], p[2]};
      qv[ax] = (j & 1) ? qv[ax] - in.delta : qv[ax] + in.delta;
      const float seed = (j & 1) ? -gv[ax] * s2 : gv[ax] * s2;
      const int at = boff2 ? o2++ : o++;
      samples[at] = make_float4(qv[0], qv[1], qv[2], seed);
      sample_lat[at] = im.latent;
      if (boff2) sample_idx[at] = 6 * h + j;
    }
  }
}

// Camera-extrinsic gradient of one view (blockIdx.y), fixed summation order:
// every depth/silhouette sample of the view's images adds s grad_p f(p) to
// dL/dc and s t grad_p f(p) u^T to dL/dR (p = c + t R u, t detached), with
// s grad_p f = s 0.5 p/|p| + the adjoint's per-wave partials; every pixel whose
// ray misses the unit sphere adds dL/dS dS/d(c, R) of S = sqrt(|c|^2 -
// (c.v)^2) - 1 (App. A.3).  Workgroup b of the view's B takes every B-th run
// of 256 samples and pixels; its sums (dL/dc, dL/dR row-major) go to out[v][b]
// and k_cam_sum adds them in order.  One workgroup per view took 118 us for two
// views of 192^2; 64 take 12 us and their sum 5.
__global__ __launch_bounds__(256) void k_cam_reduce(RayPool pl, const ImgDesc* imgs, const int* img_view, int n_img,
                                                    const float4* samples, const int4* sample_cam,
                                                    const float* gp_part, const int* n_samples, const float* g_sil,
                                                    float* out) {
  __shared__ float red[256];
  const int v = blockIdx.y, i0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  float acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.f;
  const int ns = *n_samples;
  for (int i = i0; i < ns; i += step) {
    const int4 sc = sample_cam[i];
    if (sc.x < 0 || img_view[sc.x] != v) continue;
    const ImgDesc& im = imgs[sc.x];
    const float4 smp = samples[i];
    const float rn = sqrtf(smp.x * smp.x + smp.y * smp.y + smp.z * smp.z);
    const float h = rn > 0.f ? 0.5f * smp.w / rn : 0.f;
    float g[3] = {h * smp.x, h * smp.y, h * smp.z};
    const float* pp = gp_part + (size_t)i * 3 * kGpSlots;
    for (int w = 0; w < kGpSlots; ++w) {
      g[0] += pp[3 * w];
      g[1] += pp[3 * w + 1];
      g[2] += pp[3 * w + 2];
    }
    const int V = sc.y / im.W, U = sc.y - V * im.W;
    float3 d;
    float xt, yt;
    level_ray(im, 0, U, V, d, xt, yt);
    const float nrm = sqrtf(xt * xt + yt * yt + 1.f);
    const float u[3] = {xt / nrm, yt / nrm, 1.f / nrm};
    const float t = __int_as_float(sc.z);
    for (int a = 0; a < 3; ++a) {
      acc[a] += g[a];
      for (int b = 0; b < 3; ++b) acc[3 + 3 * a + b] = fmaf(g[a] * t, u[b], acc[3 + 3 * a + b]);
    }
  }
  if (g_sil) {
    for (int img = 0; img < n_img; ++img) {
      if (img_view[img] != v) continue;
      const ImgDesc& im = imgs[img];
      const int hw = im.H * im.W;
      for (int pix = i0; pix < hw; pix += step) {
        const int r = im.slot_base + im.lvl_off[0] + pix;
        const float gs = g_sil[(size_t)im.out_base + pix];
        if (pl.st[r] != ST_MISS || gs == 0.f) continue;
        const int V = pix / im.W, U = pix - V * im.W;
        float3 d;
        float xt, yt;
        level_ray(im, 0, U, V, d, xt, yt);
        const float nrm = sqrtf(xt * xt + yt * yt + 1.f);
        const float u[3] = {xt / nrm, yt / nrm, 1.f / nrm};
        const float c[3] = {im.c[0], im.c[1], im.c[2]};
        const float dv[3] = {d.x, d.y, d.z};
        const float b0 = c[0] * dv[0] + c[1] * dv[1] + c[2] * dv[2];
        // S = (distance from the origin to the ray) - 1: with the foot of the
        // perpendicular behind the camera it is |c| - 1 (b enters as 0)
        const float b = b0 < 0.f ? b0 : 0.f;
        const float q = ray_origin_distance(c[0] * c[0] + c[1] * c[1] + c[2] * c[2], b0);
        if (!(q > 0.f)) continue;
        const float w = gs / q;
        for (int a = 0; a < 3; ++a) {
          acc[a] = fmaf(w, c[a] - b * dv[a], acc[a]);
          const float da = -w * b * c[a];
          for (int bb = 0; bb < 3; ++bb) acc[3 + 3 * a + bb] = fmaf(da, u[bb], acc[3 + 3 * a + bb]);
        }
      }
    }
  }
  // fixed-order tree reduction of each of the 12 sums
  for (int k = 0; k < 12; ++k) {
    red[threadIdx.x] = acc[k];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
      if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[((size_t)v * gridDim.x + blockIdx.x) * 12 + k] = red[0];
    __syncthreads();
  }
}

__global__ __launch_bounds__(64) void k_cam_sum(const float* part, int B, float* g_cam) {
  const int v = blockIdx.x, k = threadIdx.x;
  if (k >= 12) return;
  float s = 0.f;
  for (int b = 0; b < B; b += 16) {
    float p[16];                           // in flight together, added in order
#pragma unroll
    for (int u = 0; u < 16; ++u) p[u] = b + u < B ? part[((size_t)v * B + b + u) * 12 + k] : 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) s += p[u];
  }
  g_cam[12 * (size_t)v + k] = s;
}

// g_z[l] = W0_z^T S0 + Ws_z^T Ss with S = sum over the latent's tiles.  The
// sum runs in two fixed-order passes: k_gz_fold adds each run of 64 tiles into
// the run's first tile, k_gz_reduce adds the run heads and applies W_z^T.
// Bitwise reproducible.
// Both keep several tiles' loads in flight per thread (the chains are bound by
// memory latency, not bandwidth) and add them in tile order.
constexpr int kFold = 64;

// blockIdx.z: the column sums of one row group of layer 0 or of the skip layer
// (the groups that the kernel did not write are left out).  A latent's runs are
// dealt to gridDim.x workgroups (see launch_gz_reduce).
__global__ __launch_bounds__(512) void k_gz_fold(float* partial, int kmax, int tile, const int* seg_base,
                                                 const int* seg_padded, int lat0, int mg0) {
  const int l = lat0 + blockIdx.y;
  const int t0 = seg_base[l] / tile, nt = seg_padded[l] / tile;
  const int i = threadIdx.x;
  if (i >= kmax) return;
  const int width = 4 * kmax, z = blockIdx.z;
  for (int c0 = blockIdx.x * kFold; c0 < nt; c0 += gridDim.x * kFold) {
    const int c1 = min(c0 + kFold, nt);
    float* p = partial + (size_t)(t0 + c0) * width + (z < mg0 ? z : 2 + z - mg0) * kmax + i;
    float a = 0.f;
    int t = 0;
    for (; t + 16 <= c1 - c0; t += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = p[(size_t)(t + u) * width];
#pragma unroll
      for (int u = 0; u < 16; ++u) a += v[u];
    }
    for (; t < c1 - c0; ++t) a += p[(size_t)t * width];
    *p = a;
  }
}

// One workgroup per latent and 64 values of its gradient (blockIdx.y).  The
// run heads of a column are summed in two halves (each in head order, added
// half 0 + half 1), and each output of the latent code in four quarters of the
// contracted rows [W0_z; Ws_z] (each in row order, added in quarter order), so
// every chain is short and the order is fixed.  The column sums are summed
// again by each of the latent's workgroups: with one workgroup for the whole
// code its 1 MB of W_z came through one CU (30 us for 256 values; 16 us by four).
__global__ __launch_bounds__(1024) void k_gz_reduce(const float* partial, int kmax, int tile, const int* seg_base,
                                                    const int* seg_padded, int w0, int mg0, const float* W0z,
                                                    int ws, int mgs, const float* Wsz, int L, float* gz, int lat0,
                                                    int accumulate) {
  __shared__ float S0[512];
  __shared__ float Ss[512];
  __shared__ float ph[2][2][512];
  __shared__ float pq[4][64];
  const int l = lat0 + blockIdx.x;
  const int t0 = seg_base[l] / tile, nt = seg_padded[l] / tile;
  const int nheads = (nt + kFold - 1) / kFold;
  {
    const int half = threadIdx.x >> 9, n = threadIdx.x & 511;
    const int h1 = half ? nheads : nheads / 2;
    int h = half ? nheads / 2 : 0;
    float a = 0.f, b = 0.f;
    for (; h + 8 <= h1; h += 8) {
      float va[8][2], vb[8][2];            // eight run heads (up to two row groups each) in flight
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* pt = partial + (size_t)(t0 + (h + u) * kFold) * 4 * kmax;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          va[u][g] = (g < mg0 && n < w0) ? pt[g * kmax + n] : 0.f;
          vb[u][g] = (Wsz && g < mgs && n < ws) ? pt[(2 + g) * kmax + n] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        for (int g = 0; g < mg0; ++g) a += va[u][g];
        if (Wsz)
          for (int g = 0; g < mgs; ++g) b += vb[u][g];
      }
    }
    for (; h < h1; ++h) {
      const float* pt = partial + (size_t)(t0 + h * kFold) * 4 * kmax;
      for (int g = 0; g < mg0; ++g) a += (n < w0) ? pt[g * kmax + n] : 0.f;
      if (Wsz)
        for (int g = 0; g < mgs; ++g) b += (n < ws) ? pt[(2 + g) * kmax + n] : 0.f;
    }
    ph[0][half][n] = a;
    ph[1][half][n] = b;
  }
  __syncthreads();
  if (threadIdx.x < 512) {
    S0[threadIdx.x] = ph[0][0][threadIdx.x] + ph[0][1][threadIdx.x];
    Ss[threadIdx.x] = ph[1][0][threadIdx.x] + ph[1][1][threadIdx.x];
  }
  __syncthreads();
  const int q = threadIdx.x >> 6, jl = threadIdx.x & 63, j = blockIdx.y * 64 + jl;
  if (q < 4) {
    const int rows = w0 + (Wsz ? ws : 0);
    const int r1 = (q + 1) * rows / 4;
    int r = q * rows / 4;
    float acc = 0.f;
    if (j < L) {
      for (; r + 32 <= r1; r += 32) {
        float w[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) {
          const int rr = r + u;
          w[u] = rr < w0 ? W0z[(size_t)rr * L + j] : Wsz[(size_t)(rr - w0) * L + j];
        }
#pragma unroll
        for (int u = 0; u < 32; ++u) {
          const int rr = r + u;
          acc = fmaf(w[u], rr < w0 ? S0[rr] : Ss[rr - w0], acc);
        }
      }
      for (; r < r1; ++r)
        acc = fmaf(r < w0 ? W0z[(size_t)r * L + j] : Wsz[(size_t)(r - w0) * L + j], r < w0 ? S0[r] : Ss[r - w0], acc);
    }
    pq[q][jl] = acc;
  }
  __syncthreads();
  if (q == 0 && j < L) {
    const float v = ((pq[0][jl] + pq[1][jl]) + pq[2][jl]) + pq[3][jl];
    gz[(size_t)l * L + j] = accumulate ? gz[(size_t)l * L + j] + v : v;
  }
}

// ---------------------------------------------------------------------------
// Serving: a tick's header and table come from, and its counts go to, pinned
// host memory by kernels of the tick itself (see TickIo).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tick_begin(TickIo io, int* zero, int n_zero) {
  const int i0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  for (int i = i0; i < n_zero; i += step) zero[i] = 0;
  const int words = io.hdr_words + io.entry_words * min(io.h_hdr[0], io.cap_entries);
  for (int i = i0; i < words; i += step) io.hdr[i] = io.h_hdr[i];
}

__global__ __launch_bounds__(256) void k_tick_end(TickIo io) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < io.stat_words; i += gridDim.x * 256) io.h_stat[i] = io.stat[i];
}

// ---------------------------------------------------------------------------
// Serving: the rays that start this tick, the children of images that split
// and the coarsest rays of newly (re)started images, join the pooled active
// list behind the rays that the last march left active.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_advance_new(RayPool pl, const ImgDesc* imgs, int* out_list, int* out_count,
                                                     const AdvEntry* table, const int* hdr) {
  const int n_tab = hdr[0], n_new = hdr[1];
  for (int base = blockIdx.x * 256; base < n_new; base += gridDim.x * 256) {
    const int j = base + threadIdx.x;
    bool keep = false;
    int r = 0;
    if (j < n_new) {
      int lo = 0, hi = n_tab - 1;          // last entry with begin <= j
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (table[mid].begin <= j) lo = mid; else hi = mid - 1;
      }
      const AdvEntry e = table[lo];
      const ImgDesc& im = imgs[e.img];
      const int c = j - e.begin;
      const int lvl = e.lvl;
      const int Wl = im.W >> lvl;
      const int V = c / Wl, U = c - V * Wl;
      float3 d;
      float xt, yt, t_lo, t_hi;
      level_ray(im, lvl, U, V, d, xt, yt);
      const bool inside = sphere_interval(im, d, t_lo, t_hi);
      float t = t_lo;
      if (e.split) {
        const int Wp = im.W >> (lvl + 1);
        const int pr = im.slot_base + im.lvl_off[lvl + 1] + (V >> 1) * Wp + (U >> 1);
        const float tp = pl.st[pr] == ST_MISS ? t_lo : pl.d[pr].w;
        t = fminf(fmaxf(tp, t_lo), t_hi);
      }
      r = im.slot_base + im.lvl_off[lvl] + c;
      init_ray(pl, im, e.img, r, d, t, t_lo, t_hi, inside, e.step);
      keep = inside;
    }
    block_append(keep, r, out_list, out_count);
  }
}

// Image-space loss of inverse optimisation and its gradient w.r.t. the
// rendered maps, one workgroup per image (fixed summation order, no atomics):
//   L_i = 1/HW [ w_d sum_{fg_r & fg_t} |z_c - z_c*|                 (Sec. 4.2.1 L1 depth)
//              + w_s sum_pix S* max(0, S) + (1 - S*) max(0, -S)     (App. A.3 hinge)
//              + w_n sum_{fg_r & fg_t} (-n . n*) ]                  (App. B.3 normal term)
// fg_r: S < 0 (the rendered binary silhouette), fg_t: S* > 0.5.  sign(0) = 0
// and max'(0) = 0; a hinge term whose weight S* or 1 - S* is zero adds
// nothing.  Gradient outputs may be null (not written); normals are read
// only when w_n != 0.
// V pixels per thread and step: 4 with 16-byte accesses where every map starts
// and every image's map ends on a 16-byte boundary, else 1.  The loss of an
// image is one workgroup's sum (blockIdx.y = 0), so its order is fixed; of an
// image of more than kLossRun pixels the gradients are written by further
// workgroups of kLossRun pixels each.  Four 256^2 images with normals: 61 us by
// one pixel at a time, 45 us by four, 16 us with the gradients apart.
constexpr int kLossRun = 4096;

template <int V>
__device__ __forceinline__ void ld_map(const float* p, size_t i, float (&v)[V]) {
  if constexpr (V == 4) {
    const float4 x = *(const float4*)(p + i);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  } else {
    v[0] = p[i];
  }
}
template <int V>
__device__ __forceinline__ void st_map(float* p, size_t i, const float (&v)[V]) {
  if constexpr (V == 4) *(float4*)(p + i) = make_float4(v[0], v[1], v[2], v[3]);
  else p[i] = v[0];
}
template <int V>
__global__ __launch_bounds__(1024) void k_render_loss(const float* depth, const float* normal, const float* sil,
                                                      const float* depth_t, const float* normal_t,
                                                      const float* sil_t, int hw, float w_d, float w_s, float w_n,
                                                      float* loss, float* g_depth, float* g_normal, float* g_sil) {
  __shared__ float red[1024];
  const size_t base = (size_t)blockIdx.x * hw;
  const float inv = 1.f / (float)hw;
  const float cd = w_d * inv, cs = w_s * inv, cn = w_n * inv;
  const bool nrm = w_n != 0.f;
  const bool sum = blockIdx.y == 0, grad = gridDim.y == 1 || !sum;
  const int p0 = sum ? 0 : (blockIdx.y - 1) * kLossRun, p1 = sum ? hw : min(p0 + kLossRun, hw);
  float acc = 0.f;
  for (int p = p0 + V * threadIdx.x; p < p1; p += V * 1024) {
    const size_t i = base + p;
    float S[V], St[V], d[V], dt[V], gd[V], gs[V], ls[V];
    float nr[3][V], nt[3][V];           // 3 V consecutive floats each
    ld_map<V>(sil, i, S);
    ld_map<V>(sil_t, i, St);
    ld_map<V>(depth, i, d);
    ld_map<V>(depth_t, i, dt);
    if (nrm) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        ld_map<V>(normal, 3 * i + V * k, nr[k]);
        ld_map<V>(normal_t, 3 * i + V * k, nt[k]);
      }
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const bool fg = S[u] < 0.f && St[u] > 0.5f;
      const float dd = fg ? d[u] - dt[u] : 0.f;
      float l = cd * fabsf(dd);
      l += cs * ((St[u] > 0.f ? St[u] * fmaxf(S[u], 0.f) : 0.f) + (St[u] < 1.f ? (1.f - St[u]) * fmaxf(-S[u], 0.f) : 0.f));
      if (nrm) {
        float dot = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          float& n = nt[(3 * u + k) / V][(3 * u + k) % V];
          if (!fg) n = 0.f;
          const float x = nr[(3 * u + k) / V][(3 * u + k) % V] * n;
          dot = k == 0 ? x : dot + x;
        }
        if (fg) l -= cn * dot;
      }
      gd[u] = cd * (dd > 0.f ? 1.f : (dd < 0.f ? -1.f : 0.f));
      gs[u] = cs * (St[u] * (S[u] > 0.f ? 1.f : 0.f) - (1.f - St[u]) * (S[u] < 0.f ? 1.f : 0.f));
      ls[u] = l;
    }
    if constexpr (V == 4) acc += (ls[0] + ls[1]) + (ls[2] + ls[3]);
    else acc += ls[0];
    if (!grad) continue;
    if (g_depth) st_map<V>(g_depth, i, gd);
    if (g_sil) st_map<V>(g_sil, i, gs);
    if (g_normal) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        float gn[V];
#pragma unroll
        for (int u = 0; u < V; ++u) gn[u] = nrm ? -cn * nt[k][u] : -cn * 0.f;
        st_map<V>(g_normal, 3 * i + V * k, gn);
      }
    }
  }
  if (!sum) return;
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[blockIdx.x] = red[0];
}

// out[0] = sum of a[0..n) in index order (one thread).
__global__ void k_sum_ordered(const float* a, int n, float* out) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    float s = 0.f;
    for (int i = 0; i < n; ++i) s += a[i];
    out[0] = s;
  }
}

// Adam (paper App. B.4: Adam, learning rate 1e-2) on one latent code.
__global__ void k_adam(float* z, float* m, float* v, const float* g, int L, float lr, float b1, float b2, float eps,
                       int t) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= L) return;
  const float gj = g[j];
  const float mj = b1 * m[j] + (1.f - b1) * gj;
  const float vj = b2 * v[j] + (1.f - b2) * gj * gj;
  m[j] = mj;
  v[j] = vj;
  const float mh = mj / (1.f - powf(b1, (float)t));
  const float vh = vj / (1.f - powf(b2, (float)t));
  z[j] -= lr * mh / (sqrtf(vh) + eps);
}

__global__ void k_fill_i32(int* p, int v, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void k_fill_u64(unsigned long long* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

// ---------------------------------------------------------------------------
// Exact gradient through the unrolled march (Eq. 2 with both terms), in
// reverse over the marching steps.  lam[r] is the adjoint of ray r's current
// t: dL/dt after the step being processed.  A ray's query at step n gets the
// seed
//   a = alpha lam[r]            if the step moved t (t += alpha f)
//     + dL/dd / |(xt, yt, 1)|   at a level-0 hit's last step (d = t + f)
//     + dL/dS sign f            at a level-0 ray's minimum-|f| step,
// the decoder's VJP at that point adds a df/dz to dL/dz, and lam[r] gains
// a grad_p f . v (the same query's dependence on t through p = c + t v).
//
// Only the scalar adjoint of t runs from step to step; the decoder's
// derivatives at a query do not depend on it.  A launch per step would leave
// the chip to a few rays for most of the steps, so steps of few rays are taken
// in chunks: one launch recomputes and back-propagates all their queries with
// unit seeds and keeps the point gradients and, at layer 0 and the skip layer,
// the rows of delta; a thread per ray then runs the recurrence over its steps
// (k_ul_lambda), and the column sums are made with the resulting seeds, from the
// rows (k_ul_colsum) or, where there is no memory for them, from the ReLU masks
// by a second VJP.  A step
// that fills the chip by itself is a chunk of its own: its seeds are known, and
// the first launch makes the column sums as well.
//   What is added up, and in which order, depends neither on the chunks nor on
// the images beside: a latent's rays at one step are a segment of their own,
// padded to whole tiles, every ray that can have a seed at the step is in it,
// and the tiles' sums are added in order of step and tile.  So the chunks may
// be as long as the memory at hand allows, and the gradient of an image is the
// same bit for bit with any of them.
//   The backward of two images of 96^2 (8 x 512 decoder) takes 1.12 ms in bf16
// and 4.0 in float32 (a launch per step: 10.5 and 39.7), of eight of 256^2 18.1
// in bf16 (24.4); recompute and VJP are 80% of it and 97%.
// ---------------------------------------------------------------------------
struct UlRay {
  float alpha, dterm, sterm;       // the depth term at step `last`, the silhouette term at step `near`
  int last, near;
  bool stays;                      // the last step moved no t (hit, or the step limit)
};
__device__ __forceinline__ UlRay ul_ray(const RayPool& pl, const ImgDesc& im, int r, int pix, const UlLevel& lv) {
  const uint8_t st = pl.st[r];
  UlRay y{im.alpha, 0.f, 0.f, (int)pl.n[r] - 1, -1, st == ST_HIT || st == ST_UNCONVERGED};
  if (lv.lvl == 0) {
    const size_t q = (size_t)im.out_base + pix;
    if (st == ST_HIT && lv.g_depth) {
      const int V = pix / im.W, U = pix - V * im.W;
      float3 dd;
      float xt, yt;
      level_ray(im, 0, U, V, dd, xt, yt);
      y.dterm = lv.g_depth[q] / sqrtf(xt * xt + yt * yt + 1.f);
    }
    const float f0 = pl.rec_f[r];
    if (lv.g_sil && f0 != INFINITY) {
      y.sterm = lv.g_sil[q] * (f0 > 0.f ? 1.f : (f0 < 0.f ? -1.f : 0.f));
      y.near = pl.rec_n[r];
    }
  }
  return y;
}
__device__ __forceinline__ float ul_seed(const UlRay& y, int step, float lam) {
  float a = step == y.last && y.stays ? 0.f : y.alpha * lam;
  if (step == y.last) a += y.dterm;
  if (step == y.near) a += y.sterm;
  return a;
}

__global__ __launch_bounds__(1024) void k_ul_slots(const int* img_order, const int* img_latent, int n_img,
                                                   int* img_slot, int* slot_lat) {
  __shared__ int buf[1024];
  const int tid = threadIdx.x;
  int carry = -1;                           // slot of the last image so far
  for (int i0 = 0; i0 < n_img; i0 += 1024) {
    const int i = i0 + tid;
    const int lat = i < n_img ? img_latent[img_order[i]] : -1;
    const int first = i < n_img && (i == 0 || img_latent[img_order[i - 1]] != lat) ? 1 : 0;
    buf[tid] = first;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int x = tid >= o ? buf[tid - o] : 0;
      __syncthreads();
      buf[tid] += x;
      __syncthreads();
    }
    if (i < n_img) {
      img_slot[i] = carry + buf[tid];
      if (first) slot_lat[carry + buf[tid]] = lat;
    }
    carry += buf[1023];
    __syncthreads();
  }
}

// Coarse-to-fine split in reverse: the adjoints of ray i's (level plvl) four
// children (fixed order) whose start was its t, i.e. it did not miss the sphere
// and the clamp into the child's interval (computed exactly as the forward's
// split) did not bind.
__device__ __forceinline__ float ul_split(const RayPool& pl, const ImgDesc& im, int plvl, int i, const float* lam) {
  const int Wp = im.W >> plvl, Wc = im.W >> (plvl - 1);
  const float tp = pl.d[im.slot_base + im.lvl_off[plvl] + i].w;
  const int Vp = i / Wp, Up = i - Vp * Wp;
  float acc = 0.f;
  for (int dy = 0; dy < 2; ++dy)
    for (int dx = 0; dx < 2; ++dx) {
      const int U = 2 * Up + dx, V = 2 * Vp + dy;
      float3 d;
      float xt, yt, t_lo, t_hi;
      level_ray(im, plvl - 1, U, V, d, xt, yt);
      const bool inside = sphere_interval(im, d, t_lo, t_hi);
      if (inside && tp > t_lo && tp < t_hi) acc += lam[im.slot_base + im.lvl_off[plvl - 1] + V * Wc + U];
    }
  return acc;
}

// The adjoints that reach the level through its split, the steps at which each
// ray can have a seed (top), and per workgroup of 256 rays and step the number
// of them.  A ray with an adjoint has one at all of its
// steps; nothing reaches the others from above, so a level-0 ray's first seed
// is at its minimum-|f| step (a hit's depth term is in lam from the start), and
// a coarser ray has none.
__global__ __launch_bounds__(256) void k_ul_top(RayPool pl, const ImgDesc* imgs, const int* img_order, UlLevel lv) {
  __shared__ int cnt[256];
  const int tid = threadIdx.x, pos = blockIdx.y;
  const ImgDesc& im = imgs[img_order[pos]];
  const int nr = (im.H >> lv.lvl) * (im.W >> lv.lvl);
  const int i = blockIdx.x * 256 + tid;
  int top = 0;
  if (i < nr) {
    const int r = im.slot_base + im.lvl_off[lv.lvl] + i;
    const uint8_t st = pl.st[r];
    float lam = lv.lam[r];
    if (lv.lvl > 0 && st != ST_MISS) lv.lam[r] = lam += ul_split(pl, im, lv.lvl, i, lv.lam);
    if (st != ST_MISS && st != ST_ERROR) {
      int hi = (int)pl.n[r] - 1;
      if (lam == 0.f)
        hi = lv.lvl == 0 && lv.g_sil && pl.rec_f[r] != INFINITY && lv.g_sil[(size_t)im.out_base + i] != 0.f
                 ? min(hi, (int)pl.rec_n[r]) : -1;
      top = min(max(hi - lv.first + 1, 0), lv.S);
    }
    lv.top[(size_t)pos * nr + i] = (uint8_t)top;
  }
  cnt[tid] = 0;
  __syncthreads();
  if (top) atomicAdd(&cnt[top - 1], 1);
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {       // rays with a sample at step tid: those of top > tid
    const int x = tid + o < 256 ? cnt[tid + o] : 0;
    __syncthreads();
    cnt[tid] += x;
    __syncthreads();
  }
  if (tid < lv.S) lv.off[(size_t)tid * lv.n_img * lv.blk + (size_t)pos * lv.blk + blockIdx.x] = cnt[tid];
}

// Exclusive prefix of v over 1024 threads; *total receives the sum.
__device__ __forceinline__ int scan1024(int v, int* buf, int* total) {
  const int tid = threadIdx.x;
  __syncthreads();                          // (the last scan's buf has been read)
  buf[tid] = v;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int x = tid >= o ? buf[tid - o] : 0;
    __syncthreads();
    buf[tid] += x;
    __syncthreads();
  }
  *total = buf[1023];
  return buf[tid] - v;
}

// Per step (blockIdx.x): the counts of k_ul_top become ranks within the segment
// of their latent, and the segments get their tiles in slot order.
__global__ __launch_bounds__(1024) void k_ul_scan(UlLevel lv, int tile) {
  __shared__ int buf[1024];
  const int tid = threadIdx.x, s = blockIdx.x;
  int* off = lv.off + (size_t)s * lv.n_img * lv.blk;
  int* rays = lv.seg_rays + (size_t)s * lv.n_slot;
  for (int i0 = 0; i0 < lv.n_img;) {
    const int slot = lv.img_slot[i0];
    int i1 = i0 + 1;
    while (i1 < lv.n_img && lv.img_slot[i1] == slot) ++i1;
    const long long b0 = (long long)i0 * lv.blk, nb = (long long)(i1 - i0) * lv.blk;
    int carry = 0;
    for (long long c0 = 0; c0 < nb; c0 += 1024) {
      const bool in = c0 + tid < nb;
      int tot;
      const int x = scan1024(in ? off[b0 + c0 + tid] : 0, buf, &tot);
      if (in) off[b0 + c0 + tid] = carry + x;
      carry += tot;
    }
    if (tid == 0) rays[slot] = carry;
    i0 = i1;
  }
  __syncthreads();
  int carry = 0;
  for (int l0 = 0; l0 < lv.n_slot; l0 += 1024) {
    const bool in = l0 + tid < lv.n_slot;
    int tot;
    const int x = scan1024(in ? (rays[l0 + tid] + tile - 1) / tile : 0, buf, &tot);
    if (in) lv.seg_base[(size_t)s * lv.n_slot + l0 + tid] = carry + x;
    carry += tot;
  }
  if (tid == 0) lv.step_tiles[s] = carry;
}

// Whole steps to chunks, the last step first (one workgroup).
__global__ __launch_bounds__(256) void k_ul_chunks(UlLevel lv, UlChunks k, int rounds) {
  __shared__ int T[256];
  const int tid = threadIdx.x;
  if (tid < lv.S) T[tid] = lv.step_tiles[tid];
  for (int c = tid; c < rounds; c += 256) lv.chunk[c] = make_int4(0, 0, 0, 0);
  __syncthreads();
  if (tid) return;
  int c = 0;
  for (int s = lv.S - 1; s >= 0;) {
    const int hi = s;
    int sum = T[s];
    lv.step_base[s--] = 0;
    if (sum < k.big)
      for (; s >= 0 && T[s] < k.big && sum + T[s] <= k.cap; --s) {
        lv.step_base[s] = sum;
        sum += T[s];
      }
    if (sum > 0 && c < rounds) lv.chunk[c++] = make_int4(hi, s + 1, sum, hi > s + 1);   // (rounds suffice: ul_rounds)
  }
}
int ul_rounds(int S, long long t1, const UlChunks& k) {
  if (t1 >= k.big) return S;
  if (S * t1 <= k.cap) return 1;
  // no step is big; a chunk ends where the next step would not fit (or is the last)
  return (int)std::min<long long>(S, S * t1 / (k.cap - t1 + 1) + 1);
}

// Where the samples of a workgroup's 256 rays lie in a chunk: per step the first
// sample of each wave.  Prepared for all steps at once (one barrier; a barrier
// per step made each wait for the loads of the one before).
struct UlSlots {
  int at[256][4];
};
__device__ __forceinline__ void ul_slots(const UlLevel& lv, const int4& c, int pos, int blk, int slot, int top, int tile,
                                         UlSlots& u) {
  const int tid = threadIdx.x, w = tid >> 6;
  for (int s = c.y; s <= c.x; ++s) {
    const int n = __popcll(__ballot(top > s));
    if ((tid & 63) == 0) u.at[s][w] = n;
  }
  __syncthreads();
  const int s = c.y + tid;
  if (s <= c.x) {
    int o = (lv.step_base[s] + lv.seg_base[(size_t)s * lv.n_slot + slot]) * tile +
            lv.off[(size_t)s * lv.n_img * lv.blk + (size_t)pos * lv.blk + blk];
    for (int k = 0; k < 4; ++k) {
      const int n = u.at[s][k];
      u.at[s][k] = o;
      o += n;
    }
  }
  __syncthreads();
}
// This thread's sample at step s (if top > s).
__device__ __forceinline__ int ul_at(const UlSlots& u, int s, int top) {
  const unsigned long long bal = __ballot(top > s);
  return u.at[s][threadIdx.x >> 6] + __popcll(bal & ((1ull << (threadIdx.x & 63)) - 1ull));
}

// One sample per ray and step of the chunk; zero seeds in the segments' padding.
__device__ __forceinline__ void ul_write(const RayPool& pl, const ImgDesc* imgs, const int* img_order,
                                         const UlLevel& lv, const int4& c, int blk, int pos, int tile, float4* samples,
                                         int* sample_lat, UlSlots& u) {
  const ImgDesc& im = imgs[img_order[pos]];
  const int nr = (im.H >> lv.lvl) * (im.W >> lv.lvl);
  const int tid = threadIdx.x, i = blk * 256 + tid;
  const int r = im.slot_base + im.lvl_off[lv.lvl] + i;
  const int top = i < nr ? lv.top[(size_t)pos * nr + i] : 0;
  const int slot = lv.img_slot[pos];
  const float lam = top ? lv.lam[r] : 0.f;
  const float4 d = top ? pl.d[r] : make_float4(0.f, 0.f, 0.f, 0.f);
  const UlRay y = top && !c.w ? ul_ray(pl, im, r, i, lv) : UlRay{};
  ul_slots(lv, c, pos, blk, slot, top, tile, u);
  for (int s = c.x; s >= c.y; --s) {
    const int o = ul_at(u, s, top);
    if (top <= s) continue;
    const float t = lv.t_hist[(size_t)(lv.first + s) * lv.t_stride + r];
    samples[o] = make_float4(fmaf(t, d.x, im.c[0]), fmaf(t, d.y, im.c[1]), fmaf(t, d.z, im.c[2]),
                             c.w ? 1.f : ul_seed(y, lv.first + s, lam));
    sample_lat[o] = im.latent;
  }
  if (blk != 0 || (pos > 0 && lv.img_slot[pos - 1] == slot)) return;
  for (int s = c.y + (tid >> 6); s <= c.x; s += 4) {       // the segment's first workgroup: a wave per step
    const size_t seg = (size_t)s * lv.n_slot + slot;
    const int n = lv.seg_rays[seg], o = (lv.step_base[s] + lv.seg_base[seg]) * tile;
    for (int k = n + (tid & 63); k < (n + tile - 1) / tile * tile; k += 64) {
      samples[o + k] = make_float4(0.f, 0.f, 0.f, 0.f);
      sample_lat[o + k] = im.latent;
    }
  }
}

// The tiles of a slot's segments, latest step first, added to its sums in
// kUlChains interleaved chains (one wave each, a lane per column), in 64 bits:
// a chain of additions over all tiles of all steps.
__device__ __forceinline__ void ul_sum(const UlLevel& lv, const int4& c, int slot, int colblk, int tile,
                                       const UlSums& a, int (&tb)[256], int (&nt)[256]) {
  const int q = threadIdx.x >> 6, col = colblk * 64 + (threadIdx.x & 63);
  const int s0 = c.y + threadIdx.x;
  if (s0 <= c.x) {
    const size_t seg = (size_t)s0 * lv.n_slot + slot;
    tb[s0] = lv.step_base[s0] + lv.seg_base[seg];
    nt[s0] = (lv.seg_rays[seg] + tile - 1) / tile;
  }
  __syncthreads();
  const int which = col < a.w0 ? 0 : 1, n = which ? col - a.w0 : col, mg = which ? a.mgs : a.mg0;
  const float* p = a.partial + (size_t)(2 * which) * a.kmax + n;
  double* out = a.sums + ((size_t)(slot * kUlChains + q) * 2 + which) * a.kmax + n;
  double acc = *out;
  constexpr int D = 16;                      // tiles in flight
  int s = c.x + 1, t = 0, end = 0, base = 0;
  auto settle = [&]() {                      // to the chain's next tile, in the next segment that has one
    while (t >= end && s > c.y) {
      --s;
      t = q;
      end = __builtin_amdgcn_readfirstlane(nt[s]);
      base = __builtin_amdgcn_readfirstlane(tb[s]);
    }
  };
  settle();
  while (t < end) {
    float v[D][2];
#pragma unroll
    for (int u = 0; u < D; ++u) {
      v[u][0] = v[u][1] = 0.f;
      if (t >= end) continue;
      const float* x = p + (size_t)(base + t) * 4 * a.kmax;
      v[u][0] = x[0];
      if (mg > 1) v[u][1] = x[a.kmax];
      t += kUlChains;
      settle();
    }
#pragma unroll
    for (int u = 0; u < D; ++u) {
      acc += v[u][0];
      acc += v[u][1];
    }
  }
  *out = acc;
}

// Both in one launch, by workgroup: the samples of chunk `next` and the sums of
// chunk `done` (either may be null).
__global__ __launch_bounds__(256) void k_ul_step(RayPool pl, const ImgDesc* imgs, const int* img_order, UlLevel lv,
                                                 const int4* next, const int4* done, int tile, float4* samples,
                                                 int* sample_lat, int* n_samples, UlSums sum) {
  __shared__ union {
    UlSlots slots;
    int seg[2][256];
  } sh;
  const int wb = next ? lv.n_img * lv.blk : 0, b = blockIdx.x;
  if (b < wb) {
    const int4 c = *next;
    if (b == 0 && threadIdx.x == 0) {
      n_samples[0] = c.z * tile;
      n_samples[1] = c.w ? c.z * tile : 0;
    }
    if (c.z) ul_write(pl, imgs, img_order, lv, c, b % lv.blk, b / lv.blk, tile, samples, sample_lat, sh.slots);
  } else {
    const int4 c = *done;
    const int cols = (sum.w0 + sum.ws) / 64;
    if (c.z) ul_sum(lv, c, (b - wb) / cols, (b - wb) % cols, tile, sum, sh.seg[0], sh.seg[1]);
  }
}

// The recurrence over the chunk's steps of each ray, latest first: the seed of
// its query (written to the sample), then lam += a grad_p f . v, with grad_p f
// the residual term's p / (2 |p|) plus the adjoint's per-wave partials.  Only
// lam and the seed run from step to step; the loads of four steps are in flight.
__global__ __launch_bounds__(256) void k_ul_lambda(RayPool pl, const ImgDesc* imgs, const int* img_order, UlLevel lv,
                                                   const int4* chunk, int tile, float4* samples,
                                                   const float* gp_part) {
  __shared__ UlSlots u;
  const int4 c = *chunk;
  if (c.z == 0) return;
  const int pos = blockIdx.y;
  const ImgDesc& im = imgs[img_order[pos]];
  const int nr = (im.H >> lv.lvl) * (im.W >> lv.lvl);
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int r = im.slot_base + im.lvl_off[lv.lvl] + i;
  const int top = i < nr ? lv.top[(size_t)pos * nr + i] : 0;
  float lam = top ? lv.lam[r] : 0.f;
  const float4 d = top ? pl.d[r] : make_float4(0.f, 0.f, 0.f, 0.f);
  const UlRay y = top ? ul_ray(pl, im, r, i, lv) : UlRay{};
  ul_slots(lv, c, pos, blockIdx.x, lv.img_slot[pos], top, tile, u);
  constexpr int G = 4, V = 3 * kGpSlots / 4;
  for (int s1 = c.x; s1 >= c.y; s1 -= G) {
    int o[G];
    float4 smp[G], gp[G][V];
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int s = max(s1 - k, c.y);        // (past the chunk: its first step again, not used)
      o[k] = ul_at(u, s, top);
      if (top <= s) continue;
      smp[k] = samples[o[k]];
#pragma unroll
      for (int v = 0; v < V; ++v) gp[k][v] = ((const float4*)(gp_part + (size_t)o[k] * 3 * kGpSlots))[v];
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int s = s1 - k;
      if (s < c.y || top <= s) continue;
      const float4 p = smp[k];
      const float rn = sqrtf(p.x * p.x + p.y * p.y + p.z * p.z);
      const float h = rn > 0.f ? 0.5f / rn : 0.f;
      float g[3] = {h * p.x, h * p.y, h * p.z};
#pragma unroll
      for (int w = 0; w < 3 * kGpSlots; ++w) {
        const float4 x = gp[k][w / 4];
        g[w % 3] += w % 4 == 0 ? x.x : (w % 4 == 1 ? x.y : (w % 4 == 2 ? x.z : x.w));
      }
      const float a = ul_seed(y, lv.first + s, lam);
      samples[o[k]].w = a;
      lam += a * (g[0] * d.x + g[1] * d.y + g[2] * d.z);
    }
  }
  if (top > c.y) lv.lam[r] = lam;
}

// Column sums of each tile of 64 delta rows weighted with the seeds' factors, in
// the order of the adjoint's epilogue (ep_vjp): a lane holds rows r and, where a
// wave covers the whole tile (one row group), r + 32, added in that order; then
// the lanes in pairs 16, 8, 4, 2 and 1 apart.  A thread owns four columns; the
// rows are read once, 16 bytes per lane.
template <int BIT, bool TWO>
__device__ __forceinline__ float4 ul_tree(const float* p, int dw, const float* wgt, int r) {
  if constexpr (BIT == 32) {
    const float4 x = *(const float4*)(p + (size_t)r * dw);
    float4 a = make_float4(fmaf(wgt[r], x.x, 0.f), fmaf(wgt[r], x.y, 0.f), fmaf(wgt[r], x.z, 0.f),
                           fmaf(wgt[r], x.w, 0.f));
    if constexpr (TWO) {
      const float4 y = *(const float4*)(p + (size_t)(r + 32) * dw);
      const float w = wgt[r + 32];
      a = make_float4(fmaf(w, y.x, a.x), fmaf(w, y.y, a.y), fmaf(w, y.z, a.z), fmaf(w, y.w, a.w));
    }
    return a;
  } else {
    const float4 a = ul_tree<2 * BIT, TWO>(p, dw, wgt, r), b = ul_tree<2 * BIT, TWO>(p, dw, wgt, r + BIT);
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  }
}
__global__ __launch_bounds__(256) void k_ul_colsum(const int4* chunk, const float* __restrict__ delta,
                                                   const float4* __restrict__ samples,
                                                   const float* __restrict__ dtanh, float* __restrict__ partial,
                                                   int kmax, int w0, int mg0, int ws, int mgs) {
  __shared__ float wgt[64];
  const int4 c = *chunk;
  if (!c.w) return;
  const int dw = w0 + ws, col = 4 * threadIdx.x, which = col < w0 ? 0 : 1, n = which ? col - w0 : col;
  for (int tile = blockIdx.x; tile < c.z; tile += gridDim.x) {
    const size_t row = (size_t)tile * 64;
    if (threadIdx.x < 64) wgt[threadIdx.x] = samples[row + threadIdx.x].w * 0.05f * dtanh[row + threadIdx.x];
    __syncthreads();
    if (col < dw) {
      const float* p = delta + row * dw + col;
      float* out = partial + (size_t)tile * 4 * kmax + 2 * which * kmax + n;
      if ((which ? mgs : mg0) == 1) {
        *(float4*)out = ul_tree<1, true>(p, dw, wgt, 0);
      } else {
        *(float4*)out = ul_tree<1, false>(p, dw, wgt, 0);
        *(float4*)(out + kmax) = ul_tree<1, false>(p + (size_t)32 * dw, dw, wgt + 32, 0);
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_ul_total(const int* slot_lat, int n_slot, int n_lat, int tile,
                                                  const double* sums, int kmax, float* partial, int* seg_base,
                                                  int* seg_padded) {
  for (int l = blockIdx.x * 256 + threadIdx.x; l < n_lat; l += gridDim.x * 256) {
    int lo = 0, hi = n_slot - 1;             // slot_lat ascends
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (slot_lat[mid] < l) lo = mid + 1; else hi = mid;
    }
    const bool used = slot_lat[lo] == l;
    seg_base[l] = used ? lo * tile : 0;
    seg_padded[l] = used ? tile : 0;
  }
  for (int slot = blockIdx.x; slot < n_slot; slot += gridDim.x)
    for (int k = threadIdx.x; k < 2 * kmax; k += 256) {
      double a = 0.0;
      for (int q = 0; q < kUlChains; ++q) a += sums[(size_t)(slot * kUlChains + q) * 2 * kmax + k];
      partial[(size_t)slot * 4 * kmax + (k < kmax ? k : kmax + k)] = (float)a;
    }
}

// Initial adjoints: dL/dd / |(xt, yt, 1)| for level-0 hits (d = t + f, so the
// last t carries the depth gradient directly), 0 for every other ray slot; and
// zero sums.
__global__ __launch_bounds__(256) void k_ul_init(RayPool pl, const ImgDesc* imgs, const float* g_depth, int spi,
                                                 float* lam, double* sums, long long n_sums) {
  const ImgDesc& im = imgs[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  for (long long k = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; k < n_sums;
       k += (long long)gridDim.x * gridDim.y * 256)
    sums[k] = 0.0;
  if (i >= spi) return;
  const int r = im.slot_base + i;
  float v = 0.f;
  const int pix = i - im.lvl_off[0];
  if (g_depth && pix >= 0 && pix < im.H * im.W && pl.st[r] == ST_HIT) {
    const int V = pix / im.W, U = pix - V * im.W;
    float3 dd;
    float xt, yt;
    level_ray(im, 0, U, V, dd, xt, yt);
    v = g_depth[(size_t)im.out_base + pix] / sqrtf(xt * xt + yt * yt + 1.f);
  }
  lam[r] = v;
}

// ---------------------------------------------------------------------------
// Colour at the hits: the list of hit rays, and the backward's samples (one
// per hit with a nonzero colour gradient: its Eq. 1 point and the gradient).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_color_hits(RayPool pl, const ImgDesc* imgs, int* list, int* counter) {
  const ImgDesc& im = imgs[blockIdx.y];
  const int pix = blockIdx.x * 256 + threadIdx.x;
  const int r = im.slot_base + im.lvl_off[0] + pix;
  const bool hit = pix < im.H * im.W && pl.st[r] == ST_HIT;
  block_append(hit, r, list, counter);
}

__device__ __forceinline__ bool color_sample(const RayPool& pl, const ImgDesc& im, int pix, const float* g) {
  if (pix >= im.H * im.W || pl.st[im.slot_base + im.lvl_off[0] + pix] != ST_HIT) return false;
  const float* gq = g + 3 * ((size_t)im.out_base + pix);
  return gq[0] != 0.f || gq[1] != 0.f || gq[2] != 0.f;
}

__global__ __launch_bounds__(256) void k_color_count(RayPool pl, const ImgDesc* imgs, const int* img_order,
                                                     const float* g_rgb, int* bsum) {
  __shared__ int red[256];
  const ImgDesc& im = imgs[img_order[blockIdx.y]];
  const int pix = blockIdx.x * 256 + threadIdx.x;
  red[threadIdx.x] = color_sample(pl, im, pix, g_rgb) ? 1 : 0;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_color_write(RayPool pl, const ImgDesc* imgs, const int* img_order,
                                                     const float* g_rgb, const int* boff, float4* samples,
                                                     float4* cseed, int* sample_lat) {
  __shared__ int buf[256];
  const ImgDesc& im = imgs[img_order[blockIdx.y]];
  const int pix = blockIdx.x * 256 + threadIdx.x;
  const bool take = color_sample(pl, im, pix, g_rgb);
  const int o = boff[blockIdx.y * gridDim.x + blockIdx.x] + block_excl_scan(take ? 1 : 0, buf);
  if (!take) return;
  const int r = im.slot_base + im.lvl_off[0] + pix;
  const float4 d = pl.d[r];
  const float dd = d.w + pl.flast[r];                   // Eq. 1 ray distance
  const float* gq = g_rgb + 3 * ((size_t)im.out_base + pix);
  samples[o] = make_float4(fmaf(dd, d.x, im.c[0]), fmaf(dd, d.y, im.c[1]), fmaf(dd, d.z, im.c[2]), 0.f);
  cseed[o] = make_float4(gq[0], gq[1], gq[2], 0.f);
  sample_lat[o] = im.latent;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblk(long long n, int b) { return (unsigned)((n + b - 1) / b); }

void launch_init_level(const RayPool& pl, const ImgDesc* imgs, int n_img, int max_rays, int* list, int* counter,
                       hipStream_t s) {
  if (n_img <= 0 || max_rays <= 0) return;
  hipLaunchKernelGGL(k_init_level, dim3(nblk(max_rays, 256), n_img), dim3(256), 0, s, pl, imgs, list, counter);
}
void launch_split(const RayPool& pl, const ImgDesc* imgs, int n_img, int max_children, int child_lvl, int child_step,
                  int* list, int* counter, hipStream_t s, int* counter_tail, int tail_end) {
  if (n_img <= 0 || max_children <= 0) return;
  hipLaunchKernelGGL(k_split, dim3(nblk(max_children, 1024), n_img), dim3(1024), 0, s, pl, imgs, child_lvl, child_step,
                     list, counter, counter_tail, tail_end);
}
void launch_finalize(const RayPool& pl, const ImgDesc* imgs, const int* imgs_list, int n_img, int hw,
                     const FinalizeOut& o, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize, dim3(nblk(hw, 1024), n_img), dim3(1024), 0, s, pl, imgs, imgs_list, o);
}
void launch_normals(const RayPool& pl, const ImgDesc* imgs, const int* hits, const int* hit_count, int max_hits,
                    const float* fv, float delta, float* normal, float4* nraw, hipStream_t s) {
  if (max_hits <= 0) return;
  hipLaunchKernelGGL(k_normals, dim3(nblk(max_hits, 256)), dim3(256), 0, s, pl, imgs, hits, hit_count, fv, delta,
                     normal, nraw);
}
void launch_samples(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const int* img_latent, int n_img,
                    int hw, int n_lat, int tile, const SeedIn& in, int* bsum, int* boff, int* seg_base,
                    int* seg_total, int* seg_padded, int* n_samples, float4* samples, int* sample_lat, hipStream_t s,
                    int lat_fixed, const SplitList* sl, int4* sample_cam) {
  const int bpi = (int)nblk(hw, 256);
  const bool split = sl != nullptr && in.hit_pix != nullptr;
  hipLaunchKernelGGL(k_samples_count, dim3(bpi, n_img), dim3(256), 0, s, pl, imgs, img_order, in, bsum,
                     split ? sl->bsum : nullptr);
  hipLaunchKernelGGL(k_samples_scan, dim3(1), dim3(1024), 0, s, bsum, n_img, bpi, img_order, img_latent, lat_fixed,
                     tile, n_lat, boff, seg_base, seg_total, seg_padded, nullptr, n_samples,
                     PadOut{samples, sample_lat, nullptr, sample_cam, nullptr});
  if (split)
    hipLaunchKernelGGL(k_samples_scan, dim3(1), dim3(1024), 0, s, sl->bsum, n_img, bpi, img_order, img_latent,
                       lat_fixed, tile, n_lat, sl->boff, sl->seg_base, sl->seg_total, sl->seg_padded, n_samples,
                       n_samples + 2, PadOut{samples, sample_lat, sl->sample_idx, nullptr, nullptr});
  hipLaunchKernelGGL(k_samples_write, dim3(bpi, n_img), dim3(256), 0, s, pl, imgs, img_order, in, boff,
                     split ? sl->boff : nullptr, samples, sample_lat, split ? sl->sample_idx : nullptr, sample_cam);
}
// grad_p f . v at each hit's Eq. 1 point (unit seeds): the adjoint's per-wave
// partials plus the residual term 0.5 p / |p|; 0 where the ray grazes the
// surface (|grad f . v| <= 1e-2 |grad f|), which then gets no implicit depth term.
__global__ void k_hit_gv(RayPool pl, const ImgDesc* imgs, const float4* samples, const int4* sample_cam,
                         const float* gp_part, const int* n_samples, float* gv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *n_samples) return;
  const int4 sc = sample_cam[i];
  if (sc.x < 0) return;
  const ImgDesc& im = imgs[sc.x];
  const float4 smp = samples[i];
  const float rn = sqrtf(smp.x * smp.x + smp.y * smp.y + smp.z * smp.z);
  const float h = rn > 0.f ? 0.5f * smp.w / rn : 0.f;
  float g[3] = {h * smp.x, h * smp.y, h * smp.z};
  const float* pp = gp_part + (size_t)i * 3 * kGpSlots;
  for (int w = 0; w < kGpSlots; ++w) {
    g[0] += pp[3 * w];
    g[1] += pp[3 * w + 1];
    g[2] += pp[3 * w + 2];
  }
  const float4 d = pl.d[im.slot_base + im.lvl_off[0] + sc.y];
  const float dv = g[0] * d.x + g[1] * d.y + g[2] * d.z;
  const float gn = sqrtf(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
  gv[(size_t)im.out_base + sc.y] = fabsf(dv) > 1e-2f * gn ? dv : 0.f;
}

void launch_hit_gv(const RayPool& pl, const ImgDesc* imgs, const float4* samples, const int4* sample_cam,
                   const float* gp_part, const int* n_samples, int max_samples, float* gv, hipStream_t s) {
  if (max_samples <= 0) return;
  hipLaunchKernelGGL(k_hit_gv, dim3(nblk(max_samples, 256)), dim3(256), 0, s, pl, imgs, samples, sample_cam, gp_part,
                     n_samples, gv);
}

void launch_cam_reduce(const RayPool& pl, const ImgDesc* imgs, const int* img_view, int n_img, int n_views,
                       const float4* samples, const int4* sample_cam, const float* gp_part, const int* n_samples,
                       const float* g_sil, float* scratch, size_t scratch_floats, float* g_cam, hipStream_t s) {
  // as many workgroups per view as the scratch holds sums for; one writes g_cam itself
  const int B = (int)std::max<size_t>(1, std::min<size_t>(64, scratch_floats / (12 * (size_t)n_views)));
  hipLaunchKernelGGL(k_cam_reduce, dim3(B, n_views), dim3(256), 0, s, pl, imgs, img_view, n_img, samples, sample_cam,
                     gp_part, n_samples, g_sil, B > 1 ? scratch : g_cam);
  if (B > 1) hipLaunchKernelGGL(k_cam_sum, dim3(n_views), dim3(64), 0, s, scratch, B, g_cam);
}
void launch_gz_reduce(float* partial, int kmax, int tile, int max_tiles, const int* seg_base,
                      const int* seg_padded, int n_lat, int w0, int mg0, const float* W0z, int ws, int mgs,
                      const float* Wsz, int L, float* gz, hipStream_t s, int lat0, int accumulate) {
  // A latent may own every run of the list, but all of them together own one
  // list: workgroups for every run of every latent are nearly all empty where
  // the latents are many (200,000 samples of 60,000 latents: 117 M workgroups,
  // 30 of 61 ms).  kFoldWgs in all, each over several runs if need be.
  constexpr unsigned kFoldWgs = 16384;
  const unsigned per_lat = std::min(nblk(max_tiles, kFold), std::max(1u, kFoldWgs / n_lat));
  hipLaunchKernelGGL(k_gz_fold, dim3(per_lat, n_lat, mg0 + (Wsz ? mgs : 0)), dim3(512), 0, s, partial, kmax, tile,
                     seg_base, seg_padded, lat0, mg0);
  hipLaunchKernelGGL(k_gz_reduce, dim3(n_lat, nblk(L, 64)), dim3(1024), 0, s, partial, kmax, tile, seg_base,
                     seg_padded, w0, mg0, W0z, ws, mgs, Wsz, L, gz, lat0, accumulate);
}
void launch_advance(const RayPool& pl, const ImgDesc* imgs, int* list, int* count, const AdvEntry* table,
                    const int* hdr, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_advance_new, dim3(grid), dim3(256), 0, s, pl, imgs, list, count, table, hdr);
}
void launch_tick_begin(const TickIo& io, int* zero, int n_zero, hipStream_t s) {
  hipLaunchKernelGGL(k_tick_begin, dim3(nblk(n_zero, 256)), dim3(256), 0, s, io, zero, n_zero);
}
void launch_tick_end(const TickIo& io, hipStream_t s) {
  hipLaunchKernelGGL(k_tick_end, dim3(nblk(io.stat_words, 256)), dim3(256), 0, s, io);
}
void launch_render_loss(const float* depth, const float* normal, const float* sil, const float* depth_t,
                        const float* normal_t, const float* sil_t, int n_img, int hw, float w_d, float w_s, float w_n,
                        float* loss, float* g_depth, float* g_normal, float* g_sil, hipStream_t s) {
  uintptr_t any = 0;
  for (const void* p : {(const void*)depth, (const void*)sil, (const void*)depth_t, (const void*)sil_t,
                        (const void*)g_depth, (const void*)g_normal, (const void*)g_sil})
    any |= (uintptr_t)p;
  if (w_n != 0.f) any |= (uintptr_t)normal | (uintptr_t)normal_t;
  bool apart = hw > kLossRun && (g_depth || g_normal || g_sil);
  for (const float* g : {g_depth, g_normal, g_sil})       // a gradient in its map's place: each pixel read first
    for (const float* p : {depth, normal, sil, depth_t, normal_t, sil_t})
      if (g && g == p) apart = false;
  const dim3 grid(n_img, apart ? 1 + nblk(hw, kLossRun) : 1);
  if (hw % 4 == 0 && any % 16 == 0)
    hipLaunchKernelGGL(k_render_loss<4>, grid, dim3(1024), 0, s, depth, normal, sil, depth_t, normal_t, sil_t, hw,
                       w_d, w_s, w_n, loss, g_depth, g_normal, g_sil);
  else
    hipLaunchKernelGGL(k_render_loss<1>, grid, dim3(1024), 0, s, depth, normal, sil, depth_t, normal_t, sil_t, hw,
                       w_d, w_s, w_n, loss, g_depth, g_normal, g_sil);
}
void launch_sum_ordered(const float* a, int n, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_ordered, dim3(1), dim3(64), 0, s, a, n, out);
}
void launch_adam(float* z, float* m, float* v, const float* g, int L, float lr, float b1, float b2, float eps, int t,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(nblk(L, 256)), dim3(256), 0, s, z, m, v, g, L, lr, b1, b2, eps, t);
}

void launch_ul_init(const RayPool& pl, const ImgDesc* imgs, int n_img, int spi, const float* g_depth, float* lam,
                    double* sums, long long n_sums, hipStream_t s) {
  hipLaunchKernelGGL(k_ul_init, dim3(nblk(spi, 256), n_img), dim3(256), 0, s, pl, imgs, g_depth, spi, lam, sums, n_sums);
}
void launch_ul_slots(const int* img_order, const int* img_latent, int n_img, int* img_slot, int* slot_lat,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_ul_slots, dim3(1), dim3(1024), 0, s, img_order, img_latent, n_img, img_slot, slot_lat);
}
void launch_ul_plan(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv, int tile,
                    const UlChunks& k, int rounds, hipStream_t s) {
  hipLaunchKernelGGL(k_ul_top, dim3(lv.blk, lv.n_img), dim3(256), 0, s, pl, imgs, img_order, lv);
  hipLaunchKernelGGL(k_ul_scan, dim3(lv.S), dim3(1024), 0, s, lv, tile);
  hipLaunchKernelGGL(k_ul_chunks, dim3(1), dim3(256), 0, s, lv, k, rounds);
}
void launch_ul_step(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv, const int4* next,
                    const int4* done, int tile, float4* samples, int* sample_lat, int* n_samples, const UlSums& sum,
                    hipStream_t s) {
  const unsigned grid = (next ? (unsigned)lv.n_img * lv.blk : 0) + (done ? (unsigned)lv.n_slot * ((sum.w0 + sum.ws) / 64) : 0);
  hipLaunchKernelGGL(k_ul_step, dim3(grid), dim3(256), 0, s, pl, imgs, img_order, lv, next, done, tile, samples,
                     sample_lat, n_samples, sum);
}
void launch_ul_lambda(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv,
                      const int4* chunk, int tile, float4* samples, const float* gp_part, hipStream_t s) {
  hipLaunchKernelGGL(k_ul_lambda, dim3(lv.blk, lv.n_img), dim3(256), 0, s, pl, imgs, img_order, lv, chunk, tile,
                     samples, gp_part);
}
void launch_ul_colsum(const int4* chunk, int max_tiles, const float* delta, const float4* samples, const float* dtanh,
                      float* partial, int kmax, int w0, int mg0, int ws, int mgs, hipStream_t s) {
  hipLaunchKernelGGL(k_ul_colsum, dim3(std::max(1, std::min(max_tiles, 2048))), dim3(256), 0, s, chunk, delta, samples,
                     dtanh, partial, kmax, w0, mg0, ws, mgs);
}
void launch_ul_total(const int* slot_lat, int n_slot, int n_lat, int tile, const double* sums, int kmax, float* partial,
                     int* seg_base, int* seg_padded, hipStream_t s) {
  hipLaunchKernelGGL(k_ul_total, dim3(std::min(std::max(n_slot, (int)nblk(n_lat, 256)), 1024)), dim3(256), 0, s,
                     slot_lat, n_slot, n_lat, tile, sums, kmax, partial, seg_base, seg_padded);
}
void launch_color_hits(const RayPool& pl, const ImgDesc* imgs, int n_img, int hw, int* list, int* counter,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_color_hits, dim3(nblk(hw, 256), n_img), dim3(256), 0, s, pl, imgs, list, counter);
}
void launch_color_samples(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const int* img_latent,
                          int n_img, int hw, int n_lat, int tile, const float* g_rgb, int* bsum, int* boff,
                          int* seg_base, int* seg_total, int* seg_padded, int* n_samples, float4* samples,
                          float4* cseed, int* sample_lat, hipStream_t s) {
  const int bpi = (int)nblk(hw, 256);
  hipLaunchKernelGGL(k_color_count, dim3(bpi, n_img), dim3(256), 0, s, pl, imgs, img_order, g_rgb, bsum);
  hipLaunchKernelGGL(k_samples_scan, dim3(1), dim3(1024), 0, s, bsum, n_img, bpi, img_order, img_latent, 0, tile,
                     n_lat, boff, seg_base, seg_total, seg_padded, nullptr, n_samples,
                     PadOut{samples, sample_lat, nullptr, nullptr, cseed});
  hipLaunchKernelGGL(k_color_write, dim3(bpi, n_img), dim3(256), 0, s, pl, imgs, img_order, g_rgb, boff, samples,
                     cseed, sample_lat);
}
void launch_fill_i32(int* p, int v, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_i32, dim3(nblk(n, 256)), dim3(256), 0, s, p, v, n);
}
void launch_fill_u64(unsigned long long* p, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_u64, dim3(nblk(n, 256)), dim3(256), 0, s, p, n);
}

}  // namespace dist
