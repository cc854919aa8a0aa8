// Launch shapes of flat and list calls, on the CPU.
#include <cstdio>
#include <vector>

#include "zo_plan.h"

using namespace zo;

static int failed = 0;
#define CHECK(cond, ...)                                             \
  do {                                                               \
    if (!(cond)) {                                                   \
      std::fprintf(stderr, "line %d: %s: ", __LINE__, #cond);        \
      std::fprintf(stderr, __VA_ARGS__);                             \
      std::fprintf(stderr, "\n");                                    \
      ++failed;                                                      \
    }                                                                \
  } while (0)

static Sweep update_of(uint32_t groups) {
  static const std::vector<float> c(ZO_K_MAX, 0.5f);
  Sweep w{};
  if (make_update_sweep(w, 0, 8 * groups, c.data(), 1e-3f, nullptr) != ZO_OK || w.n_groups != groups) ++failed;
  return w;
}

// A list of `tensors` equal tensors of `bytes` each, 512-byte aligned, with an empty one after every seventh.
static std::vector<zo_segment> list_of(uint32_t tensors, uint64_t bytes, size_t elem) {
  std::vector<zo_segment> segs;
  const uint64_t stride = (bytes + 511) / 512 * 512;
  for (uint32_t i = 0; i < tensors; ++i) {
    segs.push_back({reinterpret_cast<void*>(0x7f0000000000ull + i * stride), i * (bytes / elem), bytes / elem});
    if (i % 7 == 6) segs.push_back({nullptr, 0, 0});
  }
  return segs;
}

// Every launch of a list call that streams as a whole: updates of five and more groups take workgroups of
// more than 256 threads only where the launch's own tensors are 256 MiB and more; every tensor is planned
// once, in order.
static void check_lists() {
  for (size_t elem : {(size_t)2, (size_t)4})
    for (uint32_t groups = 1; groups <= 17; ++groups)
      for (uint32_t tensors : {1u, 40u, 64u, 65u, 150u, 300u, 1200u, 12000u})
        for (uint64_t total : {300ull << 20, 1100ull << 20, 40000ull << 20}) {
          const std::vector<zo_segment> segs = list_of(tensors, total / tensors / elem * elem, elem);
          const Sweep w = update_of(groups);
          uint32_t planned = 0;
          const int rc = plan_list<kSegsPerLaunch>(segs.data(), static_cast<uint32_t>(segs.size()), elem, w,
                                                   [&](const Plans<kSegsPerLaunch>& ps, const Shape& sh) {
            uint64_t bytes = 0;
            for (uint32_t s = 0; s < ps.count; ++s, ++planned) {
              bytes += (ps.p[s].hi - ps.p[s].lo) * elem;
              CHECK(reinterpret_cast<uintptr_t>(ps.p[s].base) == 0x7f0000000000ull + planned * ((total / tensors / elem * elem + 511) / 512 * 512),
                    "tensor %u", planned);
            }
            CHECK(ps.chunk_groups == sh.chunk_groups, "chunks of another shape");
            CHECK(sh.chunks_per_wave <= 1, "%u chunks per stream", sh.chunks_per_wave);
            if (groups >= 5 && bytes < kStreamBytes)
              CHECK(sh.block == kBlock && sh.copies == 0,
                    "elem %zu, %u groups, a launch of %llu MiB in workgroups of %u threads", elem, groups,
                    (unsigned long long)(bytes >> 20), sh.block);
            if (groups >= 5 && bytes < kShortLaunchBytes) CHECK(sh.chunk_groups * kGroupElems * elem == 4096, "chunks");
            const bool fixed = groups <= (elem == 2 ? 16u : 8u);
            if (groups >= 5 && fixed && bytes >= kStreamBytes) CHECK(sh.block > kBlock, "%u groups", groups);
            return static_cast<int>(ZO_OK);
          });
          CHECK(rc == ZO_OK && planned == tensors, "%u of %u tensors", planned, tensors);
        }
}

// Flat updates in large workgroups, one to a CU: the chunks they walk one after another on the busiest CU
// are at most 2% (fp32 10%, for the table builds saved) more than with the better of one and four chunks per
// stream, wherever the buffer lies.
static void check_rounds() {
  for (size_t elem : {(size_t)2, (size_t)4})
    for (uint32_t groups = 5; groups <= (elem == 2 ? 16u : 8u); ++groups) {
      const Sweep w = update_of(groups);
      for (uintptr_t addr : {0x7f0000000000ull, 0x7f0000000000ull + 512 * 77, 0x7f0000000000ull + (300ull << 10) + 2 * elem})
        for (uint64_t mib = 256; mib < 20000; mib += mib < 2000 ? 1 : 23) {
          const uint64_t n = (mib << 20) / elem;
          const Shape sh = shape_for(n, elem, w, addr);
          if (elem == 4 && groups < 8) {
            CHECK(sh.chunks_per_wave == 1, "%u fp32 groups", groups);
            continue;
          }
          auto steps = [&](uint32_t chunks) {  // as the launch itself counts its workgroups
            Shape s = sh;
            s.chunks_per_wave = chunks;
            Plans<1> ps{};
            ps.chunk_groups = s.chunk_groups;
            add_plan(ps, make_plan(reinterpret_cast<void*>(addr), 0, n, elem, s.chunk_groups), elem, streams_per_block(s));
            return static_cast<double>(chunks * ((plans_grid(ps, s) + 255) / 256));
          };
          const double best = steps(1) < steps(4) ? steps(1) : steps(4);
          CHECK(sh.chunks_per_wave == 1 || sh.chunks_per_wave == 4, "%u chunks", sh.chunks_per_wave);
          CHECK(steps(sh.chunks_per_wave) <= best * (elem == 2 ? 1.021 : 1.101), "elem %zu, %u groups, %llu MiB at %llx: %u chunks per stream",
                elem, groups, (unsigned long long)mib, (unsigned long long)addr, sh.chunks_per_wave);
        }
    }
}

// Misaligned tensors: element by element in small launches, on row groups in larger ones; aligned ones
// always on row groups; and the line rises with the probe groups.
static void check_misaligned() {
  for (size_t elem : {(size_t)2, (size_t)4}) {
    uint64_t last = 0;
    for (uint32_t groups : {1u, 2u, 3u, 4u, 8u, 16u, 17u, 40u, 128u}) {
      const Sweep w = update_of(groups);
      const uint64_t from = any_alignment_from(elem, w);
      CHECK(from >= last && from <= 1ull << 23, "%u groups from %llu weights", groups, (unsigned long long)from);
      last = from;
      for (uint32_t tensors : {1u, 10u, 64u, 200u})
        for (uint64_t weights : {from / 2, from ? from - 1 : 3000, from, 4 * from + 100000}) {
          if (weights < tensors) continue;
          std::vector<zo_segment> segs;
          for (uint32_t i = 0; i < tensors; ++i)  // every other tensor misaligned
            segs.push_back({reinterpret_cast<void*>(0x7f0000000000ull + i * (weights * elem + 4096) + (i % 2) * elem), 0,
                            weights / tensors + (i == 0 ? weights % tensors : 0)});
          plan_list<kSegsPerLaunch>(segs.data(), tensors, elem, w, [&](const Plans<kSegsPerLaunch>& ps, const Shape&) {
            uint64_t n = 0;
            for (uint32_t s = 0; s < ps.count; ++s) n += ps.p[s].hi - ps.p[s].lo;
            for (uint32_t s = 0; s < ps.count; ++s) {
              const bool aligned = groups_aligned(ps.p[s].base, 0, elem), fits = ps.p[s].hi >= kGroupElems;
              CHECK((ps.p[s].span != 0) == (fits && (aligned || n >= from)), "elem %zu, %u groups, %llu weights in %u tensors: %s tensor on %u row groups",
                    elem, groups, (unsigned long long)n, ps.count, aligned ? "aligned" : "misaligned", ps.p[s].span);
            }
            return static_cast<int>(ZO_OK);
          });
        }
    }
  }
}

// A shape that asks for spread tables is the one the kernel of its group count is built for (its workgroups,
// on which the chunk alignment rests), any other has the default workgroups; and tables fit the LDS.
static void check_kernels() {
  for (size_t elem : {(size_t)2, (size_t)4})
    for (uint32_t groups = 1; groups <= ZO_K_MAX / 8; ++groups) {
      const Sweep w = update_of(groups);
      const SpreadDims d = spread_dims(elem, groups);
      for (uint64_t mib : {1, 200, 300, 800, 5000, 30000}) {
        const uint64_t n = (static_cast<uint64_t>(mib) << 20) / elem;
        for (const Shape& sh : {shape_for(n, elem, w), list_shape(n, n, elem, w), list_shape(n, n / 8, elem, w)}) {
          if (sh.copies)
            CHECK(sh.copies == d.copies && sh.block == d.block && sh.wps == d.wps, "elem %zu, %u groups", elem, groups);
          else
            CHECK(sh.block == kBlock && sh.wps == 1, "elem %zu, %u groups: %u threads on shared tables", elem, groups, sh.block);
          CHECK(mib >= 256 || sh.copies == 0, "spread tables for a cache-sized buffer");
          const size_t tables = 4 * static_cast<size_t>(table_floats(groups, sh.copies));
          CHECK(tables + occupancy_lds(sh.blocks_per_cu, tables) <= 160 * 1024, "%zu bytes of tables", tables);
          if (sh.copies) CHECK(spread_groups(groups, sh.copies) * sh.copies <= 128, "more than two planes");
        }
      }
    }
}

// The buffers with which the GPU tests mean to reach four chunks per stream do.
static void check_test_sizes() {
  const struct {
    size_t elem;
    uint64_t mib;
    uint32_t groups;
  } tests[] = {{2, 1000, 6}, {2, 1000, 12}, {2, 1100, 16}, {4, 1000, 8}};
  for (auto& t : tests)
    CHECK(shape_for((t.mib << 20) / t.elem - 77, t.elem, update_of(t.groups)).chunks_per_wave == 4, "%u groups", t.groups);
}

int main() {
  check_test_sizes();
  check_kernels();
  check_lists();
  check_misaligned();
  check_rounds();
  if (!failed) std::printf("ok\n");
  return failed != 0;
}
