"""The rules by which the host picks a kernel or its shape, compiled from the library's own sources into a small host
program (no GPU): what they promise over their whole range."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2209_07663_amd", "csrc")


def _run(tmp_path, source):
    """Compiles `source` against the library's sources and runs it; it prints what is wrong and returns how many."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs the ROCm toolchain")
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text("#include <cstdio>\n" + source)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-I", CSRC, str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE)
    assert r.returncode == 0, r.stdout.decode()


def test_walk_of_the_longest_bag_ends_at_its_last_id(tmp_path):
    """The walk of a bag goes on in steps of kIdsInRegs positions while the next one lies inside the bag: for the most
    IDs that count of a bag it has to end, and never to ask for a position outside."""
    _run(tmp_path, r"""
#include "gather.hip"
using namespace mono;
int main() {
  const BagPos most = kMostInBag;
  BagPos c = most / kIdsInRegs * kIdsInRegs;  // the last step of the walk
  for (int turns = 0; turns < 2; ++turns) {
    c += kIdsInRegs;
    if (c < most) return printf("the walk went on at position %lld of %lld\n", (long long)c, (long long)most), 1;
  }
  return 0;
}
""")


def test_pooled_rows_stay_in_the_caches_unless_they_are_large(tmp_path):
    """Pooled rows go past the caches beyond three quarters of the 256 MB cache, and never where a lane holds eight
    elements of a row."""
    _run(tmp_path, r"""
#include "gather.hip"
using namespace mono;
int main() {
  int wrong = 0;
  const unsigned long long most = 192ull << 20;
  for (unsigned dim : {4u, 32u, 36u, 64u, 256u, 512u, 1024u})
    for (unsigned long long bytes : {1ull << 20, 64ull << 20, 65ull << 20, 128ull << 20, most, most + 4 * dim, 1ull << 32}) {
      const unsigned long long bags = bytes / (4 * dim);
      if (GatherShape(dim, 4, bags).past_caches != (bags * dim * 4 > most)) printf("dim %u, %llu bags\n", dim, bags), ++wrong;
      if (GatherShape(dim, 8, bags).past_caches) printf("eight elements per lane, dim %u, %llu bags\n", dim, bags), ++wrong;
    }
  return wrong;
}
""")


def test_pooling_launches_less_than_2_to_32_threads(tmp_path):
    """However many bags there are, and however few of them a wave takes for the dimension: a launch of 2^32 threads or
    more is refused.  (Of 2^32 bags and more there is no launch, with 64 of them in a wave.)"""
    _run(tmp_path, r"""
#include "gather.hip"
using namespace mono;
int main() {
  int wrong = 0;
  const unsigned long long most = (1ull << 32) - 256;
  for (unsigned dim : {4u, 16u, 32u, 36u, 64u, 128u, 132u, 256u, 512u, 768u, 1024u})
    for (unsigned per_lane : {4u, 8u})
      for (unsigned ids : {4u, 8u})
        for (unsigned lg = 0; lg <= 32; ++lg)
          for (long long d : {-70ll, -16ll, -15ll, -1ll, 0ll, 1ll, 17ll}) {
            const long long bags = (1ll << lg) + d;
            if (bags < 1 || bags > (long long)most) continue;
            const GatherShape s(dim, per_lane, bags, ids);
            const unsigned long long threads = (s.waves + 3) / 4 * 256;
            if (threads >= 1ull << 32 || s.waves << s.bags_log2 < (unsigned long long)bags || s.bags_log2 > 6 || s.bags_log2 + s.group_log2 < 6)
              printf("dim %u, %lld bags: %llu threads\n", dim, bags, threads), ++wrong;
          }
  return wrong ? 1 : 0;
}
""")


def test_waves_of_wide_rows_are_short_and_not_a_few_more_than_run_at_a_time(tmp_path):
    """Rows that take a whole wave: at most four pieces of a wave's width to a wave, twice as many bags where the launch
    would be up to half as many waves again as the chip holds."""
    _run(tmp_path, r"""
#include "gather.hip"
using namespace mono;
template <typename Src>
int wrong(unsigned dim) {
  int bad = 0;
  const unsigned long long pieces = (dim + 64 * Src::N - 1) / (64 * Src::N);
  for (unsigned long long bags = 1; bags < 3000000; bags += 1 + bags / 400) {
    const GatherShape s(dim, Src::N, bags, Src::kIds, Src::kHeld);
    const bool few = s.waves >= 4096 || s.bags_log2 == 0, ends_alone = s.waves >= 8192 && s.waves <= 12288;
    const bool wide = (pieces << s.bags_log2) > 8 || ((pieces << s.bags_log2) > 4 && pieces != 3 && s.waves > 6145);
    if (!few || ends_alone || wide) printf("dim %u, %llu bags: %llu waves of %u bags\n", dim, bags, (unsigned long long)s.waves, 1u << s.bags_log2), ++bad;
  }
  return bad;
}
int main() {
  int bad = 0;
  for (unsigned dim : {132u, 256u, 512u, 768u, 1024u}) {
    bad += wrong<TableRows<float, 4>>(dim);
    if (dim < 512) bad += wrong<TableRows<uint16_t, 4>>(dim);
    else bad += wrong<TableRows<uint16_t, 8>>(dim);
  }
  return bad ? 1 : 0;
}
""")


def test_two_tables_eight_rows_in_flight_for_long_bags_and_for_many_of_six(tmp_path):
    """From 12 IDs a bag on (3 of narrow bf16 rows), or from 6 of rows of more than two pieces (to 8 in few
    bags) and of fp32 rows of which four or more share a wave or that are two pieces, where four IDs in flight would be more than twice the 6144 waves that the chip
    holds; and the latter are never a little more than those."""
    _run(tmp_path, r"""
#include "gather.hip"
using namespace mono;
int main() {
  int bad = 0;
  for (unsigned dim : {4u, 16u, 32u, 36u, 64u, 100u, 128u, 256u, 512u, 768u, 1024u})
    for (unsigned long long bags = 1; bags < 3000000; bags += 1 + bags / 300) {
      const unsigned lanes_log2 = dim <= 4 ? 0 : dim <= 16 ? 2 : dim <= 32 ? 3 : dim <= 64 ? 4 : dim <= 128 ? 5 : 6;
      const unsigned long long usual = lanes_log2 < 3 ? 64 : lanes_log2 == 3 ? 32 : dim == 512 ? 2 : dim > 512 ? 1 : 16;
      const bool some = lanes_log2 <= 4 || dim >= 512, many = some && bags / usual >= 12288;
      for (unsigned long long each : {1ull, 5ull, 6ull, 8ull, 9ull, 11ull, 12ull, 40ull}) {
        const unsigned long long from = many || (dim > 512 && each <= 8) ? 6 : 12;
        if (qr_takes_eight(bags * each, bags, dim, true) != (each >= (dim <= 32 ? 3 : dim > 512 ? from : 12))) printf("bf16 %u %llu %llu\n", dim, bags, each), ++bad;
        if (many != (some && (bags + usual - 1) / usual >= 12288)) continue;
        if (qr_takes_eight(bags * each, bags, dim, false) != (each >= from)) printf("%u %llu %llu\n", dim, bags, each), ++bad;
      }
      using Four = QuotRemRows<float, 4, 4>;
      const GatherShape s(dim, 4, bags, Four::kIds, Four::kHeld);
      if (lanes_log2 >= 3 && s.bags_log2 < 6 && s.waves >= 6144 && s.waves <= 9216 && s.bags_log2 + 1 < (lanes_log2 == 6 ? 3u : 7u))
        printf("dim %u, %llu bags: %llu waves\n", dim, bags, (unsigned long long)s.waves), ++bad;
    }
  return bad ? 1 : 0;
}
""")


def test_small_batches_of_many_bags_are_sorted_by_one_block(tmp_path):
    """Up to 4096 pairs in up to 16384 bags, most of them empty: one launch instead of six or nine."""
    _run(tmp_path, r"""
#include "kernels.h"
using namespace mono;
int main() {
  int wrong = 0;
  for (unsigned long long n : {1ull, 100ull, 4095ull, 4096ull, 4097ull, 8192ull, 1ull << 20, 1ull << 22})
    for (unsigned long long bags : {1ull, 4096ull, 8192ull, 8193ull, 12288ull, 16384ull, 16385ull, 1ull << 20})
      if (sorts_in_one_block(n, bags) != (n <= 4096 && bags <= 16384)) printf("%llu pairs, %llu bags\n", n, bags), ++wrong;
  return wrong;
}
""")


def test_the_workspace_holds_what_any_batch_needs_and_the_split_its_units(tmp_path):
    """The histogram workspace for batches of n pairs holds the shares and turns of every split and the histograms of every
    radix shape of any smaller batch; a block of the split's second kernel has a thread for every unit of the first; buckets
    of evenly spread rows are an eighth of what a block sorts at once; digits of nine bits from 2^24 rows in use on."""
    _run(tmp_path, r"""
#include "kernels.h"
using namespace mono;
static uint64_t words_of(uint64_t n, uint32_t rows) {
  if (n <= kSplitMost) {
    const SplitShape s = split_shape_for(n);
    const uint64_t hot = kSplitSamples[s.size] / kSplitHits;
    return sort_units(n, kSplitItems[s.size]) * (kSplitBuckets[s.size] + hot) + 2 + 2 * (hot + n / kSplitTurn);
  }
  const SortShape s = sort_shape_for(rows);
  const uint64_t groups = sort_groups(n, s.items);
  return (groups * kSortGroupUnits << s.max_bits) + (groups << s.max_bits) + (1ull << s.max_bits);
}
int main() {
  int wrong = 0;
  uint64_t sizes[200];
  int k = 0;
  for (double n = 1; n < 3e8; n *= 1.2) sizes[k++] = (uint64_t)n;
  for (uint64_t n : {1ull << 12, (1ull << 12) + 1, 1ull << 16, (1ull << 16) + 1, 1ull << 17, (1ull << 17) + 1, 1ull << 18, 1ull << 19, (1ull << 19) + 1, 1ull << 20, (1ull << 20) + 1, 1ull << 28}) sizes[k++] = n;
  for (int i = 0; i < k; ++i)
    for (int j = 0; j < k; ++j)
      for (uint32_t rows : {1u, 1u << 24, (1u << 24) + 1, 1u << 30})
        if (sizes[j] <= sizes[i] && words_of(sizes[j], rows) > sort_hist_words(sizes[i]))
          printf("%llu pairs in a workspace for %llu, %u rows\n", (unsigned long long)sizes[j], (unsigned long long)sizes[i], rows), ++wrong;
  for (uint64_t n = 1; n <= kSplitMost; n += 1 + n / 200) {
    const SplitShape s = split_shape_for(n);
    const uint64_t units = sort_units(n, kSplitItems[s.size]), most = sort_units(kSplitUpTo[s.size], kSplitItems[s.size]);
    if (n > kSplitUpTo[s.size] || units > most || most > 512 || 1u << s.buckets_log2 > kSplitBuckets[s.size]) printf("%llu: %llu units\n", (unsigned long long)n, (unsigned long long)units), ++wrong;
    if ((n >> s.buckets_log2) > 1024) printf("%llu pairs in %u buckets\n", (unsigned long long)n, 1u << s.buckets_log2), ++wrong;
  }
  for (uint32_t rows : {1u, 1u << 16, 1u << 22, 1u << 24, (1u << 24) + 1, 1u << 30}) {
    const SortShape s = sort_shape_for(rows);
    if (s.max_bits != (rows > 1u << 24 ? 9u : 8u) || s.items != 8u << s.max_bits) printf("%u rows\n", rows), ++wrong;
  }
  return wrong ? 1 : 0;
}
""")
