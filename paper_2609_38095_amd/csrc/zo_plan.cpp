// Host-side launch planning of libzo's sweeps (declared in zo_plan.h): validation, the split
// of a tensor into row groups, chunks and edge tiles, and the launch shapes. Plain C++ with
// no HIP, compiled by the host compiler into libzo.so and, with AddressSanitizer and UBSan,
// into the host checker of the tests.

#include "zo_plan.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <utility>
#include <vector>

namespace zo {
namespace {

// zo_set_max_blocks: a cap on the workgroups of every later launch in the process (0: the
// default shapes). A test hook for grid independence; atomic so that a call on another thread
// sees either value, never a torn one.
std::atomic<uint32_t> g_max_blocks{0};

uint64_t ceil_div(uint64_t a, uint64_t b) { return a / b + (a % b != 0); }

// 4 KiB chunks at full occupancy
Shape short_chunks(size_t elem) {
  const size_t group_bytes = kGroupElems * elem;
  return Shape{static_cast<uint32_t>(4096 / group_bytes), 0, 0};
}

}  // namespace

void set_max_blocks(uint32_t max_blocks) { g_max_blocks.store(max_blocks, std::memory_order_relaxed); }

// Workgroups for work_items items, per_block per workgroup of `block` threads, at most: the
// zo_set_max_blocks override if set, else kDefaultMaxBlocks, or (sized: the caller sized the
// work per workgroup itself) no cap; and always fewer than 2^32 work-items per dispatch. The
// kernels loop over whatever a smaller grid leaves.
uint32_t grid_for(uint64_t work_items, uint64_t per_block, uint32_t block, bool sized) {
  const uint64_t need = ceil_div(work_items, per_block);
  const uint32_t set = g_max_blocks.load(std::memory_order_relaxed);
  const uint64_t dispatch_cap = (1ull << 32) / block - 1;
  uint64_t cap = set ? set : sized ? dispatch_cap : kDefaultMaxBlocks;
  if (cap > dispatch_cap) cap = dispatch_cap;
  const uint64_t g = need < cap ? need : cap;
  return static_cast<uint32_t>(g ? g : 1);
}

int check_params(const void* params, zo_dtype dt, uint64_t offset, uint64_t n) {
  if (dt != ZO_F32 && dt != ZO_BF16) return ZO_ERR_ARG;
  if (n == 0) return ZO_OK;
  if (params == nullptr) return ZO_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(params) % (dt == ZO_F32 ? 4 : 2) != 0) return ZO_ERR_ARG;
  if (offset + n < offset || offset + n == 0) return ZO_ERR_ARG;  // reaches 2^64
  if (n >= ZO_N_MAX) return ZO_ERR_ARG;  // more weights than a device holds
  return ZO_OK;
}

// The address of global element 0 (params shifted back by offset elements; the subtraction may
// wrap, only its alignment is used) is 16-byte aligned when every group vector is.
bool groups_aligned(const void* params, uint64_t offset, size_t elem) {
  return ((reinterpret_cast<uintptr_t>(params) - static_cast<uintptr_t>(offset * elem)) & 15u) == 0;
}

// From how many weights of a launch on its misaligned tensors (groups_aligned false) take full row
// groups. Smaller launches are bound by the latency of one wave: a tile per lane and nothing after it
// is shorter than a chunk of row groups followed by the head and tail tiles, the more so the more
// probe groups. The element-wise path's time rises in steps of 2^20 weights (one workgroup more on each
// CU), so the lines lie there. Flat calls at an odd address with both ends ragged, element-wise against row
// groups, us: bf16, 3 groups, 0.9 M weights 9.7 / 11.3, 1.3 M 12.3 / 12.1; 4 groups, 1.8 M 12.8 / 13.8, 2.6 M
// 16.0 / 14.2; 8 groups, 40 thousand 12.3 / 19.5, 2.6 M 19.3 / 20.7, 3.6 M 22.5 / 20.7; 17 groups, 40 thousand
// 20.6 / 40.3, 3.6 M 32.9 / 41.5, 5.1 M 47.7 / 44.2; fp32, one probe, 80 thousand 6.4 / 6.5 (6.7 / 5.1 from
// a row group's start on); 2 groups, 160 thousand 8.3 / 9.2, 320 thousand 8.8 / 8.6; 8 groups, 0.9 M 14.0 / 16.3,
// 1.3 M 19.3 / 17.1; 24 groups, 2.6 M 41.0 / 48.2, 3.6 M 47.0 / 48.4, 5.1 M 68.0 / 50.5.
uint64_t any_alignment_from(size_t elem, const Sweep& w) {
  const uint64_t groups = w.update ? w.n_groups : 1;
  if (elem == 2) return std::min<uint64_t>(1 + groups / 4, 4) << 20;
  return groups <= 1 ? 0 : groups <= 3 ? 1ull << 18 : (groups <= 16 ? 1ull : 3ull) << 20;
}

// The addresses are device addresses: they are only ever offset here, never dereferenced, and
// are carried as integers until the plan holds them. Full row groups sit at any weight's address;
// without any_alignment misaligned storage has none, and n must be below 2^34, so that the edge-tile
// counts fit 32 bits.
Plan make_plan(void* params, uint64_t offset, uint64_t n, size_t elem, uint32_t chunk_groups, bool any_alignment) {
  Plan pl{};
  pl.base = static_cast<char*>(params);
  pl.lo = offset;
  pl.hi = offset + n;
  if (n == 0) return pl;
  const uintptr_t addr = reinterpret_cast<uintptr_t>(params);
  uint64_t head_end = pl.hi, tail_begin = pl.hi;
  if (any_alignment || groups_aligned(params, offset, elem)) {
    const uint64_t g_lo = ceil_div(pl.lo, kGroupElems), g_hi = pl.hi / kGroupElems;
    if (g_lo < g_hi) {  // g_hi - g_lo < 2^30: n < ZO_N_MAX is checked first
      pl.g_lo = g_lo;
      pl.span = static_cast<uint32_t>(g_hi - g_lo);
      pl.gbase = reinterpret_cast<char*>(addr + static_cast<uintptr_t>((g_lo * kGroupElems - pl.lo) * elem));
      pl.head = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(pl.gbase) / (kGroupElems * elem) % chunk_groups);
      head_end = g_lo * kGroupElems;
      tail_begin = g_hi * kGroupElems;
    }
  }
  if (head_end > pl.lo) {
    pl.head_t0 = pl.lo / kTile;
    pl.head_nt = static_cast<uint32_t>(ceil_div(head_end, kTile) - pl.head_t0);
  }
  if (pl.hi > tail_begin) {
    pl.tail_t0 = tail_begin / kTile;
    pl.tail_nt = static_cast<uint32_t>(ceil_div(pl.hi, kTile) - pl.tail_t0);
  }
  return pl;
}

// Chunk slots of a plan, the leading empty ones included (fewer than 2^30 + 2 + 16).
uint32_t plan_chunks(const Plan& pl, uint32_t chunk_groups) {
  return pl.span ? static_cast<uint32_t>(ceil_div(static_cast<uint64_t>(pl.head) + pl.span, chunk_groups)) : 0u;
}

Probe make_probe(uint32_t k, float eps) { return Probe{k / 8, k % 8, eps}; }

Gen make_gen(uint64_t seed, uint32_t step) {
  return Gen{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), step};
}

// Streaming shape of a launch over `elements` weights of `elem` bytes. HBM sustains these
// in-place sweeps best as few long sequential read-write streams: each stream walks up to
// kMaxChunkBytes of consecutive row groups with the next one or two groups in flight per wave,
// and occupancy is capped with dynamic LDS so that few streams run at once (the bf16 perturb
// on an OPT-13B shaped buffer: 6.5 TB/s at one workgroup per CU, 5.6 at full occupancy). An
// update needs more waves where its generator and table work per byte outgrows what one wave
// overlaps with its own loads: either two waves per stream (each takes every other row group
// of the chunk, so the stream keeps its length and gains a second wave to hide the work) or
// larger workgroups that share one set of spread tables. The shapes below are the fastest of
// those measured (A/B on one box) on OPT-13B shaped bf16 buffers (K <= 16), OPT-30B (K = 32),
// OPT-1.3B and Qwen3-8B (K = 60-64) and 3 G-element fp32 buffers:
//   perturb, one or two probes: 256 threads, one workgroup per CU; one fp32 probe: 128 threads, one
//     chunk per wave (1.3 G weights: 1,751 -> 1,591 us, 6.01 -> 6.62 TB/s, the rate of a plain
//     read-modify-write; a row group is twice bf16's bytes, so two waves keep as much in flight as
//     four do there; 64, 192 and 512 threads, 16 and 64 KiB chunks, one and three groups ahead and
//     other paces 1 to 50% slower; bf16 with 128 threads 38% and two fp32 probes 8 to 30% slower);
//   update, one bf16 group: one workgroup per CU, one chunk per wave (OPT-30B K = 8: 6.19 ->
//     6.53 TB/s), paced at four outstanding memory operations as the perturb (+0.5%);
//   update, two bf16 groups: 512 threads, two waves per stream, one chunk per stream, 32-copy
//     tables (OPT-13B K = 16: +0.5 to 1.8%, +2% on a GPU already busy with perturbs), paced
//     at four outstanding memory operations (+0.3 to 0.5% on three boxes; 2, 3, 5, 6 and 8,
//     three groups in flight, 16-copy tables, 256 threads and one wave per stream all equal
//     or slower);
//   update, three bf16 groups: 16-copy tables, two workgroups per CU (1.3 G weights: shared tables
//     at three per CU, the count fixed at compile time, 870 -> 853 us);
//   update, four bf16 groups: 512 threads, 16-copy tables in one plane, two workgroups per CU, one
//     chunk per wave (a 3.75 G shard, K = 32: 2,769 -> 2,681 us against 1024 threads on 32-copy
//     tables);
//   update, five to eight bf16 groups: 1024 threads sharing 16-copy tables in two planes (4 LDS
//     cycles per 64-lane read instead of 6.3), four chunks per stream (OPT-1.3B K = 64: 1.80 ->
//     1.57 ms; Qwen3-8B K = 60: 10.9 -> 9.9 ms; 1.3 G weights, against shared tables, a run-time
//     count and 4 KiB chunks: K = 40 1,410 -> 1,093 us, K = 48 1,572 -> 1,227, K = 56 1,744 ->
//     1,374). 768 threads with one group ahead were 13% faster than 1024 on zero weights run
//     back to back and 2.5% slower (1,590 against 1,550 us) on ordinary ones;
//   update, nine to sixteen bf16 groups: the first eight groups as above, the others on shared
//     tables behind them, 1024 threads up to twelve groups, else 768 (1.36 G weights, against shared tables, a
//     run-time count and 4 KiB chunks: K = 69 2,414 -> 1,781 us, K = 93 3,010 -> 2,470, K = 125 3,865 -> 3,430;
//     K = 128 with 1024 threads spills registers, 5% slower). Bound by the LDS and VALU together: 16-copy
//     tables for all would need more than the LDS holds, shared tables for all take 6.3 LDS cycles a read
//     (K = 96 on 1.3 G weights with the count fixed: 2,630 against 2,260 us);
//   fp32 updates: one workgroup per CU, 32-copy tables for one and two groups, shared ones for three
//     (the count fixed at compile time: 2,607 -> 1,630 us); four: 16-copy tables, two workgroups per CU
//     (1.3 G weights, K = 32: 1,697 against 1,647 us, in two other runs equal to 3% apart); five to eight:
//     512 threads sharing 16-copy tables (1.3 G weights: K = 40 1,911 -> 1,725 us, K = 48 2,128 ->
//     1,836, K = 56 2,161 -> 2,001, K = 64 2,169 -> 2,069; 768 and 1024 threads spill registers).
// An update with a restore probe inside its groups (Algorithm 1's schedule) is the plain
// update with that group's table changed, and takes the update's shape. Other updates (more than
// sixteen bf16 groups, or more than eight in fp32, and a restore probe outside the update's groups)
// are bound by the generator or the LDS table lookups and keep 4 KiB chunks at full occupancy. fp32
// above eight groups: 512 threads on 16-copy tables for the first eight are faster on small buffers
// only (12 groups, 0.3 GB 276 -> 225 us, 2.7 GB 1,620 -> 1,772). Above sixteen groups, beyond the 60
// to 96 probes that steps are known to use, the count stays a run-time one: a third run needs the full
// compensation, and a fixed count is twelve more kernels (trial kernels for 24 groups of 1.36 G bf16
// weights 5,777 -> 5,567 us). Perturbs smaller than the 256 MiB Infinity Cache take 4 KiB chunks at
// full occupancy too, updates of such buffers 8 KiB ones. Grids: up to
// kDefaultMaxBlocks workgroups, grid-stride beyond (in-order dispatch of many short-lived
// workgroups keeps the streams compact; a persistent grid of one workgroup per CU measured
// 5.6 TB/s), except where a number of chunks per stream is given: the bf16 perturb of one
// probe or of two in one probe group, the fp32 perturbs, the bf16 updates of one, two and four
// groups and of five and more, and the fp32 updates of five to eight. One chunk per stream: OPT-13B,
// the perturb 6.48 -> 6.67 TB/s, OPT-30B 6.20 -> 6.60; two probes in one group +1%, across two groups
// -0.3%, so those stay grid-stride; 3 G fp32 weights, the two-probe perturb 6.30 -> 6.48 across two
// probe groups.
// Four chunks per stream (each workgroup's table build serves four times the bytes) where they take no
// longer, counted in rounds of one workgroup on each of the 256 CUs: a round of four chunks lasts as
// long as four rounds of one, less the table builds (2% of it in bf16, 10% in fp32, measured where both
// fill their last round), and one started for a few last workgroups lasts as long as a full one. bf16, four
// chunks against one: eight groups at 0.94 GB (2 rounds for 8) 578 against 601 us, at 1.08 GB (3 for 9)
// 900 against 700, at 2.63 GB (5 for 20) 1,526 against 1,578; sixteen groups at 0.82 GB (3 for 9) 1,462
// against 1,146. fp32, eight groups, at 0.54 GB (3 for 9) 280 against 242, at 1.78 GB (7 for 27) 713
// against 765; five to seven groups run one always. Workgroups are counted as memory blocks touched from
// `addr`, the buffer's address: 0.40 GB in whole blocks are 3 rounds of one chunk (173 us at K = 40) or one of
// four (212), the same bytes across one more block 4 and 1.
Shape shape_for(uint64_t elements, size_t elem, const Sweep& w, uintptr_t addr) {
  const uint64_t group_bytes = kGroupElems * elem;
  if (elements * elem < kStreamBytes) {
    if (!w.update) return short_chunks(elem);
    // updates of cache-sized buffers: 8 KiB chunks, so that each workgroup's table build
    // serves twice the bytes (OPT-125M: K = 16 0.088 -> 0.084 ms, K = 60 0.201 -> 0.189 ms;
    // 16 and 32 KiB chunks measured slower at K = 16)
    return Shape{static_cast<uint32_t>(8192 / group_bytes), 0, 0};
  }
  const uint32_t chunk = static_cast<uint32_t>(kMaxChunkBytes / group_bytes);
  if (!w.update) {
    // one chunk per wave: bf16 with one probe or two in one group, fp32 with two probes
    const bool one_group_bf16 = elem == 2 && (!w.two || w.a.group == w.b.group);
    const bool two_probes_fp32 = w.two && elem == 4;
    Shape sh{chunk, 1, one_group_bf16 || two_probes_fp32 ? 1u : 0u};
    if (elem == 4 && !w.two) {
      sh.block = 128;
      sh.chunks_per_wave = 1;
    }
    return sh;
  }
  if (w.restore && !w.fold) return short_chunks(elem);
  const uint32_t g = w.n_groups;
  const SpreadDims d = spread_dims(elem, g);
  if (g > 4 && d.copies == 0) return short_chunks(elem);
  Shape sh{chunk, 1, 0, d.block, d.wps, d.copies};
  if (g == 4 || (g == 3 && elem == 2)) sh.blocks_per_cu = 2;
  if (g <= 4) {
    if (elem == 2 && g != 3) sh.chunks_per_wave = 1;
    return sh;
  }
  const uint64_t bytes = kMaxChunkBytes * (sh.block / 64);  // a workgroup's aligned block, one chunk per stream
  const uint64_t blocks = (addr % bytes + elements * elem + bytes - 1) / bytes;
  const uint64_t one = ceil_div(blocks, kCUs), four = ceil_div(ceil_div(blocks, 4), kCUs);
  sh.chunks_per_wave = (elem == 2 || g == 8) && 400 * four <= (elem == 2 ? 102 : 110) * one ? 4 : 1;
  return sh;
}

// Shape of one launch of a list call. The call's weights decide whether it streams; its launches take
// at most one chunk per stream: a tensor boundary then idles at most one chunk slot per stream of a
// workgroup (Qwen3-8B as 399 tensors, K = 60: update 10.4-10.5 -> 9.8-9.9 ms against four chunks per
// stream). Updates of five and more groups stream only where the launch's own tensors fill 256 MiB:
// one of their workgroups takes up to 512 KiB of consecutive memory, so tensors of a few MiB leave
// most of its waves idle and the chip half empty. A launch below runs as a cache-sized buffer, one
// below 32 MiB in 4 KiB chunks, which still give every CU work. bf16, K = 96, a call of 300 MiB as 150
// tensors (128 MiB a launch) 594 -> 381 us (417 in 4 KiB chunks), as 300 tensors 645 -> 428, as 600
// (32 MiB) 1,230 -> 546 (539 in 4 KiB chunks), as 1,200 2,246 -> 690 (783 in 8 KiB chunks); fp32, K = 64,
// 1.15 GB in launches of 117 MiB 700 -> 631. In launches of 267 to 384 MiB the two shapes lie within 14%
// of each other either way; of 533 MiB (2.6 GB, bf16, K = 96) the streaming one takes 2,659 us, the
// other 2,751.
Shape list_shape(uint64_t call_elements, uint64_t launch_elements, size_t elem, const Sweep& w) {
  const bool large_blocks = w.update && !(w.restore && !w.fold) && w.n_groups >= 5 &&
                            spread_dims(elem, w.n_groups).copies;
  if (large_blocks && call_elements * elem >= kStreamBytes && launch_elements * elem < kStreamBytes)
    return launch_elements * elem < kShortLaunchBytes ? short_chunks(elem) : shape_for(launch_elements, elem, w);
  Shape sh = shape_for(call_elements, elem, w);
  if (sh.chunks_per_wave > 1) sh.chunks_per_wave = 1;
  return sh;
}

// Dynamic LDS that, with `static_lds` bytes of the kernel's own, admits exactly `cap` (one or two)
// workgroups on a CU's 160 KiB (0: no cap).
size_t occupancy_lds(uint32_t cap, size_t static_lds) {
  if (cap == 0) return 0;
  const size_t per_block = cap == 1 ? 96 * 1024 : 72 * 1024;
  return per_block > static_lds ? per_block - static_lds : 0;
}

int check_sweep(const Sweep& w) {
  if (!std::isfinite(w.a.eps) || (w.two && !std::isfinite(w.b.eps))) return ZO_ERR_NONFINITE;
  if (w.update && (!std::isfinite(w.lr) || (w.restore && !std::isfinite(w.r.eps)))) return ZO_ERR_NONFINITE;
  return ZO_OK;
}

int make_update_sweep(Sweep& w, uint32_t k_base, uint32_t K, const float* c, float lr, const Probe* r) {
  if (K > ZO_K_MAX) return ZO_ERR_ARG;
  if (static_cast<uint64_t>(k_base) + K > (1ull << 32)) return ZO_ERR_ARG;
  if (K > 0 && c == nullptr) return ZO_ERR_NULL;
  if (!std::isfinite(lr) || (r && !std::isfinite(r->eps))) return ZO_ERR_NONFINITE;
  for (uint32_t j = 0; j < K; ++j)
    if (!std::isfinite(c[j])) return ZO_ERR_NONFINITE;
  w = Sweep{};
  if (K == 0) {  // nothing to sum: the restore alone, or nothing
    w.update = false;
    w.a = r ? *r : Probe{0, 0, 0.0f};
    return ZO_OK;
  }
  w.update = true;
  for (uint32_t j = 0; j < ZO_K_MAX; ++j) w.cf.c[j] = j < K ? c[j] : 0.0f;
  w.k_base = k_base;
  w.K = K;
  const uint32_t g_first = k_base / 8;
  const uint32_t g_last = static_cast<uint32_t>((static_cast<uint64_t>(k_base) + K - 1) / 8);
  w.n_groups = g_last - g_first + 1;
  w.lr = lr;
  w.restore = r != nullptr && r->eps != 0.0f;  // a zero restore changes nothing (theta + 0 = theta)
  w.r = r ? *r : Probe{0, 0, 0.0f};
  w.fold = w.restore && r->group - g_first < w.n_groups;  // wraps for a group below g_first
  return ZO_OK;
}


// A list of tensors is validated as a whole: alignment, index ranges, and no two segments
// sharing memory.
int check_segments(const zo_segment* segs, uint32_t n_segs, zo_dtype dtype) {
  if (dtype != ZO_F32 && dtype != ZO_BF16) return ZO_ERR_ARG;
  if (n_segs == 0) return ZO_OK;
  if (segs == nullptr) return ZO_ERR_NULL;
  const size_t elem = dtype == ZO_F32 ? 4 : 2;
  std::vector<std::pair<uintptr_t, uintptr_t>> spans;
  spans.reserve(n_segs);
  for (uint32_t i = 0; i < n_segs; ++i) {
    const int rc = check_params(segs[i].params, dtype, segs[i].offset, segs[i].n);
    if (rc != ZO_OK) return rc;
    if (segs[i].n == 0) continue;
    const uintptr_t a = reinterpret_cast<uintptr_t>(segs[i].params);
    if (segs[i].n > (UINTPTR_MAX - a) / elem) return ZO_ERR_ARG;
    spans.emplace_back(a, a + segs[i].n * elem);
  }
  std::sort(spans.begin(), spans.end());
  for (size_t i = 1; i < spans.size(); ++i)
    if (spans[i].first < spans[i - 1].second) return ZO_ERR_ARG;  // overlapping memory
  return ZO_OK;
}

Sweep perturb_sweep(uint32_t k_a, float eps_a, const uint32_t* k_b, float eps_b) {
  Sweep w{};
  w.a = make_probe(k_a, eps_a);
  w.two = k_b != nullptr;
  w.b = k_b ? make_probe(*k_b, eps_b) : w.a;
  return w;
}

}  // namespace zo
