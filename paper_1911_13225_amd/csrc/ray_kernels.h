// Launchers of the ray bookkeeping kernels (ray_kernels.hip).
#pragma once
#include "dist_internal.h"

namespace dist {

struct FinalizeOut {
  float* depth;
  float* dist;
  float* sil;
  float* normal;
  uint8_t* status;
  uint8_t* nsteps;
  float4* nraw;      // per pixel (nx, ny, nz, |n|), zeroed here, filled by the normal pass
  int* hits;
  int* hit_count;
  int want_hits;
  int* hit_pix;      // per output pixel: its index in hits, -1 if none (or null)
  const unsigned long long* qcount;   // per image in launch order: decoder queries, copied to
  int64_t* queries;                   // this output (or null)
};

// One image that starts rays this tick: split into level `lvl` (split = 1) or
// (re)started at its coarsest level `lvl` (split = 0); its new rays occupy
// positions [begin, begin + count) of the tick's new-ray range.
struct AdvEntry {
  int img, lvl, step, split, begin, count;
};

struct SeedIn {
  const float* g_depth;
  const float* g_normal;
  const float* g_sil;
  const float4* nraw;
  float delta;
  const int* hit_pix;  // split layout: per output pixel, its index in the forward's hit list
  // exact depth gradient: 1 = only one unit-seed sample per hit with a depth
  // gradient, at its Eq. 1 point (to measure grad f . v there); with imp_gv
  // the depth term of a hit is one sample at that point with seed
  // -dL/dz_c / |(xt, yt, 1)| / (grad f . v) (imp_gv[q] = 0: no depth term)
  int hit_mode;
  const float* imp_gv;
};

// The gradient through the unrolled march, one coarse-to-fine level of it: the
// rays of level lvl of n_img images (in latent order, blk workgroups of 256 rays
// per image), at their S steps first, first + 1, ...  Steps are indexed from
// first below; "slots" are the distinct latents of the images.
struct UlLevel {
  int lvl, first, S, n_img, blk, n_slot;
  const float* g_depth;
  const float* g_sil;
  const float* t_hist;             // t of every ray slot at every global step [step][t_stride]
  size_t t_stride;
  float* lam;                      // adjoint of every ray slot's current t
  const int* img_slot;             // [n_img] slot of the image's latent
  const int* slot_lat;             // [n_slot]
  uint8_t* top;                    // [n_img][rays]: steps at whose queries the ray may have a seed (0 .. top - 1)
  int* off;                        // [S][n_img blk]: rank of the workgroup's first ray in its segment
  int* seg_rays;                   // [S][n_slot]: rays of a segment (the rays of one latent at one step)
  int* seg_base;                   // [S][n_slot]: its first tile, from the step's first
  int* step_tiles;                 // [S]
  int* step_base;                  // [S]: the step's first tile, from its chunk's first
  int4* chunk;                     // [rounds] (last step, first step, tiles, more than one step); tiles 0: none
};
// img_slot and slot_lat of the images in latent order
void launch_ul_slots(const int* img_order, const int* img_latent, int n_img, int* img_slot, int* slot_lat,
                     hipStream_t s);
// Tiles: a step of `big` or more is a chunk of its own, others share chunks of
// at most `cap` (big <= (cap + 1) / 2).
struct UlChunks {
  int big, cap;
};
// Bound on the chunks of a level of S steps of at most t1 tiles each.
int ul_rounds(int S, long long t1, const UlChunks& k);
// The adjoints that reach the level through its split (lvl > 0), the level's
// samples (which ray has one at which step) and the chunks.
void launch_ul_plan(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv, int tile,
                    const UlChunks& k, int rounds, hipStream_t s);
// The samples of chunk `next` (or null), with their seeds if it is a single step
// and unit seeds else, its length in n_samples[0] and, if it has several steps,
// in n_samples[1]; and the column sums of chunk `done` (or null) join sums
// [slot][kUlChains][S0, Sskip][kmax].
constexpr int kUlChains = 4;
struct UlSums {
  const float* partial;
  int kmax, w0, mg0, ws, mgs;
  double* sums;
};
void launch_ul_step(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv, const int4* next,
                    const int4* done, int tile, float4* samples, int* sample_lat, int* n_samples, const UlSums& sum,
                    hipStream_t s);
// With the adjoint's point gradients (of unit seeds): every sample's seed, and
// the rays' adjoints before the chunk's steps.
void launch_ul_lambda(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const UlLevel& lv,
                      const int4* chunk, int tile, float4* samples, const float* gp_part, hipStream_t s);
// Column sums of a chunk of several steps from the rows of delta that the adjoint
// kept, bit for bit those of its own epilogue.
void launch_ul_colsum(const int4* chunk, int max_tiles, const float* delta, const float4* samples, const float* dtanh,
                      float* partial, int kmax, int w0, int mg0, int ws, int mgs, hipStream_t s);
// The sums as one tile per latent, for launch_gz_reduce.
void launch_ul_total(const int* slot_lat, int n_slot, int n_lat, int tile, const double* sums, int kmax, float* partial,
                     int* seg_base, int* seg_padded, hipStream_t s);

// Second sample list of the split layout (normal-stencil samples).
struct SplitList {
  int* bsum;
  int* boff;
  int* seg_base;
  int* seg_total;
  int* seg_padded;
  int* sample_idx;
};

void launch_init_level(const RayPool& pl, const ImgDesc* imgs, int n_img, int max_rays, int* list, int* counter,
                       hipStream_t s);
void launch_split(const RayPool& pl, const ImgDesc* imgs, int n_img, int max_children, int child_lvl, int child_step,
                  int* list, int* counter, hipStream_t s, int* counter_tail = nullptr, int tail_end = 0);
void launch_finalize(const RayPool& pl, const ImgDesc* imgs, const int* imgs_list, int n_img, int hw,
                     const FinalizeOut& o, hipStream_t s);
void launch_normals(const RayPool& pl, const ImgDesc* imgs, const int* hits, const int* hit_count, int max_hits,
                    const float* fv, float delta, float* normal, float4* nraw, hipStream_t s);
void launch_samples(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const int* img_latent, int n_img,
                    int hw, int n_lat, int tile, const SeedIn& in, int* bsum, int* boff, int* seg_base,
                    int* seg_total, int* seg_padded, int* n_samples, float4* samples, int* sample_lat, hipStream_t s,
                    int lat_fixed = 0, const SplitList* split = nullptr, int4* sample_cam = nullptr);
void launch_gz_reduce(float* partial, int kmax, int tile, int max_tiles, const int* seg_base,
                      const int* seg_padded, int n_lat, int w0, int mg0, const float* W0z, int ws, int mgs,
                      const float* Wsz, int L, float* gz, hipStream_t s, int lat0 = 0, int accumulate = 0);
void launch_cam_reduce(const RayPool& pl, const ImgDesc* imgs, const int* img_view, int n_img, int n_views,
                       const float4* samples, const int4* sample_cam, const float* gp_part, const int* n_samples,
                       const float* g_sil, float* scratch, size_t scratch_floats, float* g_cam, hipStream_t s);
void launch_hit_gv(const RayPool& pl, const ImgDesc* imgs, const float4* samples, const int4* sample_cam,
                   const float* gp_part, const int* n_samples, int max_samples, float* gv, hipStream_t s);
void launch_ul_init(const RayPool& pl, const ImgDesc* imgs, int n_img, int spi, const float* g_depth, float* lam,
                    double* sums, long long n_sums, hipStream_t s);
void launch_color_hits(const RayPool& pl, const ImgDesc* imgs, int n_img, int hw, int* list, int* counter,
                       hipStream_t s);
void launch_color_samples(const RayPool& pl, const ImgDesc* imgs, const int* img_order, const int* img_latent,
                          int n_img, int hw, int n_lat, int tile, const float* g_rgb, int* bsum, int* boff,
                          int* seg_base, int* seg_total, int* seg_padded, int* n_samples, float4* samples,
                          float4* cseed, int* sample_lat, hipStream_t s);
// What a serving tick reads from and writes to pinned host memory, in 4-byte
// words: the header and the entries it counts, and the counts the scheduler
// reads.  The tick's own kernels move them, which spares two copies and the
// gaps around them (10 us a tick).
struct TickIo {
  const int* h_hdr;
  int* hdr;
  int hdr_words, entry_words, cap_entries;
  const int* stat;
  int* h_stat;
  int stat_words;
};
void launch_tick_begin(const TickIo& io, int* zero, int n_zero, hipStream_t s);
void launch_tick_end(const TickIo& io, hipStream_t s);
// The rays that start this tick (split children and (re)started images) join the list.
void launch_advance(const RayPool& pl, const ImgDesc* imgs, int* list, int* count, const AdvEntry* table,
                    const int* hdr, int grid, hipStream_t s);
// Per-image loss of inverse optimisation (L1 depth, silhouette hinge, normal
// term) and its map gradients; one workgroup per image, fixed order.
void launch_render_loss(const float* depth, const float* normal, const float* sil, const float* depth_t,
                        const float* normal_t, const float* sil_t, int n_img, int hw, float w_d, float w_s, float w_n,
                        float* loss, float* g_depth, float* g_normal, float* g_sil, hipStream_t s);
void launch_sum_ordered(const float* a, int n, float* out, hipStream_t s);
void launch_adam(float* z, float* m, float* v, const float* g, int L, float lr, float b1, float b2, float eps, int t,
                 hipStream_t s);
void launch_fill_i32(int* p, int v, int n, hipStream_t s);
void launch_fill_u64(unsigned long long* p, int n, hipStream_t s);

}  // namespace dist
