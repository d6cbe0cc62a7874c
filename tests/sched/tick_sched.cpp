// The serving loop's scheduler core on a device model that keeps every ray, at
// the cadence of the HIP backend (kStepsPerTick steps per tick): a tick marches
// the listed rays, keeps the full-resolution ones that are still active, and
// joins the rays that the next tick's table starts.  Checks that no ray slot is
// listed twice or without its job, that a coarse ray lives for exactly one tick
// and is split at the step it reached, and that a job completes when, and only
// when, each of its full-resolution rays has stopped or reached the step limit.
// Built with ThreadSanitizer by tests/test_sched_tick.py; prints "ok <name>" and
// exits 0, or prints the failed check and exits 1.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "sched_core.h"

using namespace dist::sched;

#define CHECK(c)                                                              \
  do {                                                                        \
    if (!(c)) {                                                               \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c);    \
      std::exit(1);                                                           \
    }                                                                         \
  } while (0)

struct Ray {
  uint64_t job = 0;             // 0: the slot is free
  int img = -1, lvl = 0, n = 0, life = 0;
  bool active = false;
};

struct Img {
  Job* job = nullptr;
  int base = 0;                 // first ray slot; level l starts at base + off(l)
  int64_t q = 0;
  int act = 0;
  int first = 0;                // the render's first tick
};

struct RayBackend : Backend {
  RayBackend(int cap_rays, int cap_imgs) : rays(cap_rays), imgs(cap_imgs), g(3) {}
  std::vector<Ray> rays;
  std::vector<Img> imgs;
  std::vector<int> list;        // rays that the last tick left active
  std::mt19937 g;
  int ticks = 0, fail_at = -1, renders = 0, limited = 0;

  static int off(const Job* j, int lvl) {
    int o = 0;
    for (int l = 0; l < lvl; ++l) o += (j->H >> l) * (j->W >> l);
    return o;
  }
  bool acquire(Job*) override { return true; }
  void release(Job*) override {}
  void begin(Job* j) override {
    for (int v = 0; v < j->n_views; ++v) {
      Img& im = imgs[j->imgs[v]];
      CHECK(im.job == nullptr);
      im = Img{j, j->slot_base + v * j->spi, 0, 0, 0};
      for (int i = 0; i < j->spi; ++i) {
        CHECK(rays[im.base + i].job == 0);
        rays[im.base + i] = Ray{j->ticket, j->imgs[v], 0, 0, 0, false};
      }
    }
  }
  int tick(const std::vector<TickEntry>& table, int n_new) override {
    if (++ticks == fail_at) return DIST_EHIP;
    std::vector<int> in = list;
    int sum = 0;
    for (const TickEntry& e : table) {
      Img& im = imgs[e.img];
      const Job* j = im.job;
      CHECK(j && e.begin == sum && e.count == (j->H >> e.lvl) * (j->W >> e.lvl));
      CHECK(e.split == (e.step > 0) && e.step == kStepsPerTick * (j->levels - e.lvl));
      sum += e.count;
      if (!e.split) im.first = ticks;
      if (e.split)                // the parents took all their steps, or stopped before
        for (int i = 0; i < e.count / 4; ++i) {
          const Ray& p = rays[im.base + off(j, e.lvl + 1) + i];
          CHECK(p.lvl == e.lvl + 1 && !p.active && (p.n == e.step || p.n == p.life));
        }
      for (int i = 0; i < e.count; ++i) {
        const int r = im.base + off(j, e.lvl) + i;
        const bool meets = g() % 5 != 0;             // the others miss the sphere
        rays[r] = Ray{j->ticket, e.img, e.lvl, e.step, meets ? e.step + 1 + (int)(g() % 40) : e.step, meets};
        if (meets) in.push_back(r);
      }
    }
    CHECK(sum == n_new);
    CHECK(std::set<int>(in.begin(), in.end()).size() == in.size());       // no slot twice
    for (Img& im : imgs) im.act = 0;
    list.clear();
    for (int r : in) {
      Ray& y = rays[r];
      Img& im = imgs[y.img];
      CHECK(y.active && im.job && im.job->ticket == y.job);
      CHECK(r >= im.base && r < im.base + im.job->spi);
      CHECK(y.lvl == 0 || y.n == kStepsPerTick * (im.job->levels - y.lvl));   // a coarse ray begins its only tick
      for (int s = 0; s < kStepsPerTick && y.active; ++s) {
        ++y.n;
        ++im.q;
        y.active = y.n < y.life && y.n < im.job->max_steps;
      }
      if (!y.active) continue;
      if (y.lvl > 0) y.active = false;               // the split that follows takes over
      else {
        list.push_back(r);
        ++im.act;
      }
    }
    return DIST_OK;
  }
  int active(int img) const override { return imgs[img].act; }
  int64_t queries(int img) const override { return imgs[img].q; }
  void complete(Job* j) override {
    for (int img : j->imgs) {
      const Img& im = imgs[img];
      CHECK(ticks - im.first < (j->max_steps + kStepsPerTick - 1) / kStepsPerTick);     // and no later
      for (int i = 0; i < j->hw; ++i) {
        const Ray& y = rays[im.base + i];
        CHECK(y.lvl == 0 && !y.active && y.n == std::min(y.life, j->max_steps));
        limited += y.life > j->max_steps;
      }
    }
    ++renders;
    if (j->kind == DIST_REQ_ZOPT && ++j->iter < j->iters) {
      for (int img : j->imgs) imgs[img].q = 0;
      j->restart();
    } else {
      j->finished = true;
    }
  }
  void settle(Job* j) override {
    for (int img : j->imgs) {
      for (int i = 0; i < j->spi; ++i) rays[imgs[img].base + i] = Ray{};
      imgs[img] = Img{};
    }
  }
  void drop_rays() override { list.clear(); }
  void idle() override { std::this_thread::sleep_for(std::chrono::microseconds(50)); }
};

static Job* make_job(std::mt19937& g, int i) {
  Job* j = new Job();
  j->kind = i % 4 == 3 ? DIST_REQ_ZOPT : DIST_REQ_RENDER;
  j->n_views = 1 + (int)(g() % 3);
  j->H = 4 << (g() % 3);
  j->W = 4 << (g() % 3);
  j->hw = j->H * j->W;
  j->levels = i % 3;
  for (int l = 0; l <= j->levels; ++l) j->spi += (j->H >> l) * (j->W >> l);
  // step limits around the ticks: one, two and three steps past the last split, and more
  const int more[6] = {1, 2, 3, 4, 17, 50};
  j->max_steps = 3 * j->levels + more[g() % 6];
  j->iters = j->kind == DIST_REQ_ZOPT ? 1 + (int)(g() % 3) : 1;
  return j;
}

static void rays(int fail_at) {
  RayBackend be(3000, 12);
  be.fail_at = fail_at;
  Core core(&be, 3000, 12, 12, 4096);
  core.start();
  std::mt19937 g(17);
  std::vector<uint64_t> tks;
  for (int i = 0; i < 150; ++i) {
    uint64_t t = 0;
    CHECK(core.submit(make_job(g, i), &t) == DIST_OK);
    tks.push_back(t);
  }
  int ok = 0;
  for (uint64_t t : tks) {
    dist_result r{};
    CHECK(core.poll(t, &r, -1) == DIST_OK);
    CHECK(r.status == DIST_OK || (fail_at > 0 && r.status == DIST_EHIP));
    ok += r.status == DIST_OK;
  }
  core.shutdown();
  CHECK(be.list.empty() && be.renders >= ok && be.limited > 0);
  CHECK(fail_at > 0 ? ok > 0 && ok < 150 : ok == 150);
  for (const Ray& y : be.rays) CHECK(y.job == 0);
}

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  if (s == "rays") rays(-1);
  else if (s == "failed") rays(20);
  else return 2;
  std::printf("ok %s\n", s.c_str());
  return 0;
}
