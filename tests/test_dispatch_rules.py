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
