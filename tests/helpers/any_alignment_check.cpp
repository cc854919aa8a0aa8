// Plans of tensors stored at any weight's address (any_alignment), on the CPU: the head tiles,
// full row groups and tail tiles partition [offset, offset + n), every row group's bytes lie
// inside the tensor, and wherever planning without any_alignment has full row groups the plans agree.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>

#include "zo_plan.h"

using namespace zo;

static int failed = 0;
#define CHECK(cond)                                                                              \
  do {                                                                                           \
    if (!(cond)) {                                                                               \
      std::fprintf(stderr, "line %d: %s (n %llu offset %llu shift %llu elem %zu)\n", __LINE__, #cond, \
                   (unsigned long long)n, (unsigned long long)off, (unsigned long long)shift, elem);  \
      ++failed;                                                                                  \
    }                                                                                            \
  } while (0)

int main() {
  const uintptr_t A = 0x7f3200000000ull;
  for (size_t elem : {(size_t)2, (size_t)4})
    for (uint64_t n : {1ull, 17ull, 1023ull, 1024ull, 1025ull, 2047ull, 2049ull, 65549ull, (1ull << 39) + 5})
      for (uint64_t off : {0ull, 1ull, 1023ull, 1025ull, (1ull << 35) + 7, ~0ull - (1ull << 40)})
        for (uintptr_t shift = 0; shift < 32; shift += elem) {
          const uint32_t cg = 16;
          const zo_segment seg{reinterpret_cast<void*>(A + shift), off, n};
          int launches = 0;
          const int rc = plan_segments<1>(&seg, 1, elem, cg, 4, [&](const Plans<1>& ps) {
            ++launches;
            const Plan& pl = ps.p[0];
            const uint64_t first = (off + kGroupElems - 1) / kGroupElems, last = (off + n) / kGroupElems;
            CHECK(pl.lo == off && pl.hi == off + n);
            CHECK(pl.span == (first < last ? last - first : 0));
            uint64_t head_end = off + n, tail_begin = off + n;
            if (pl.span) {
              head_end = pl.g_lo * kGroupElems;
              tail_begin = head_end + pl.span * kGroupElems;
              CHECK(head_end >= off && head_end - off < kGroupElems && off + n - tail_begin < kGroupElems);
              const uintptr_t gb = reinterpret_cast<uintptr_t>(pl.gbase);
              CHECK(gb == A + shift + (head_end - off) * elem);
              CHECK(gb + (uintptr_t)pl.span * kGroupElems * elem <= A + shift + n * elem);
            }
            if (head_end > off) {
              CHECK(pl.head_t0 == off / kTile && (pl.head_t0 + pl.head_nt) * kTile >= head_end);
              CHECK((pl.head_t0 + pl.head_nt - 1) * kTile < head_end);
            } else {
              CHECK(pl.head_nt == 0);
            }
            if (off + n > tail_begin) {
              CHECK(pl.tail_t0 * kTile == tail_begin && (pl.tail_t0 + pl.tail_nt - 1) * kTile < off + n);
              CHECK((pl.tail_t0 + pl.tail_nt) * kTile >= off + n);
            } else {
              CHECK(pl.tail_nt == 0);
            }
            if (groups_aligned(seg.params, off, elem)) {
              Plans<1> def{};
              def.chunk_groups = cg;
              add_plan(def, make_plan(seg.params, off, n, elem, cg, false), elem, 4);
              CHECK(std::memcmp(&def, &ps, sizeof def) == 0);
            }
            return static_cast<int>(ZO_OK);
          }, true);
          CHECK(rc == ZO_OK && launches == 1);
        }
  if (!failed) std::printf("ok\n");
  return failed != 0;
}
