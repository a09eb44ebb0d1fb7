"""The rules by which a launch hands out its electrons (paper_1901_08140_amd/csrc/swarm_internal.hpp),
built for the host with the library's own compiler: they are plain integer and float
arithmetic that host and device share."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1901_08140_amd", "csrc")

HOST_PROGRAM = r"""
#include <cstdio>
#include <cstdint>
#include <vector>
#include "swarm_internal.hpp"
using namespace swarm_impl;

// `waves` waves take electrons in turn, each for the `wanted` lanes it finds idle (all of them at
// first), and again when what it took is used up.  Prints the claims made, and the largest number
// a wave took beyond what it wanted while fewer electrons than lanes were left.
static void simulate(const char* name, uint64_t electrons, int64_t waves, uint32_t wanted, ClaimRule rule) {
  std::vector<uint32_t> end(waves, 0), held(waves, 0);
  uint64_t taken = 0, claims = 0, late = 0;
  bool first = true;
  while (taken < electrons) {
    for (int64_t w = 0; w < waves && taken < electrons; ++w) {
      const uint32_t want = first ? 64 : wanted;
      if (held[w] >= want) { held[w] -= want; continue; }
      const uint32_t n = rule.size(static_cast<uint32_t>(electrons) - end[w], want);
      if (electrons - taken < static_cast<uint64_t>(waves) * 64 && n > want && n - want > late) late = n - want;
      const uint64_t got = taken + n < electrons ? n : electrons - taken;
      end[w] = static_cast<uint32_t>(taken + got);
      taken += got;
      held[w] += static_cast<uint32_t>(got);
      held[w] -= held[w] < want ? held[w] : want;
      ++claims;
    }
    first = false;
  }
  printf("%s %llu %llu\n", name, (unsigned long long)claims, (unsigned long long)late);
}

// Launches of a run whose electrons each make `rate` secondaries per collision, the longest slice,
// and whether every limit lies in the budget and beyond the one before.
static void slices(const char* name, SlicePlan p, int64_t electrons, double rate) {
  int64_t n = 0, at = 0, longest = 0, good = 1;
  while (at < p.budget) {
    const int64_t to = p.limit(electrons);
    if (to <= at || to > p.budget) good = 0;
    if (to - at > longest) longest = to - at;
    p.launched(electrons, static_cast<int64_t>(static_cast<double>(electrons) * rate * static_cast<double>(to - at)), to, to);
    at = to;
    ++n;
    if (!good) break;
  }
  printf("%s %lld %lld %lld\n", name, (long long)n, (long long)longest, (long long)good);
}

int main() {
  simulate("real", 1000000, 4096, 2, claim_rule(64, 4096, 4, true));
  simulate("dummy", 1000000, 4096, 2, claim_rule(64, 4096, 2, false));
  for (uint32_t chunk : {64u, 1u << 20, 1u << 27, 0x7fffffc0u}) {
    const ClaimRule r = claim_rule(chunk, 8192, 2, false);
    printf("scarce%u %u\n", chunk, r.scarce);
  }
  slices("none", {20000, 262144, 100000, true}, 20000, 0.0);
  slices("many", {20000, 262144, 100000, true}, 500, 0.01);
  slices("gas", {20000, 262144, 100000, false}, 500, 0.01);
  slices("longest", {0xffffffffll, 262144, 100000, true}, 25, 0.0);
  slices("short", {40, 262144, 100000, true}, 25, 0.0);
  const ClaimRule r = claim_rule(64, 1, 4, true);
  printf("sizes %u %u %u %u\n", r.size(1u << 31, 3), r.size(257, 3), r.size(100, 3), r.size(0, 3));
  return 0;
}
"""


@pytest.fixture(scope="module")
def host_output(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_rules")
    src = d / "drv.cpp"
    src.write_text(HOST_PROGRAM)
    exe = d / "drv"
    cmd = ["hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-2000:]
    return {ln.split()[0]: [int(v) for v in ln.split()[1:]] for ln in out.stdout.splitlines()}


def test_real_generations_make_few_claims(host_output):
    """Every claim is an atomic on one address.  A generation of a few rounds takes chunks and
    then shrinking shares: of 1e6 electrons on 4096 waves at most one claim for 64 electrons while
    many are left, and then ln(64) of four shares of every wave."""
    assert host_output["real"][0] <= 1_000_000 / 64 + 4 * 4096 * 4.2


def test_dummy_launches_hold_nothing_back_at_their_end(host_output):
    assert host_output["dummy"][1] == 0


def test_the_end_of_a_launch_is_known_for_any_chunk(host_output):
    """Two chunks for each of 8192 waves, or all electrons where that is more than 32 bits hold."""
    for chunk in (64, 1 << 20, 1 << 27, 0x7fffffc0):
        assert host_output[f"scarce{chunk}"][0] == min(2 * 8192 * chunk, 0xffffffff), chunk


def test_claim_sizes(host_output):
    assert host_output["sizes"] == [64, 64, 25, 3]


def test_slices_of_the_budget(host_output):
    """Doubled from 128 without secondaries, the shortest where many are made, the whole budget
    for a gas that makes none or a budget that one slice holds."""
    assert host_output["none"] == [8, 8192, 1]          # 128 + 256 + ... + 8192 + the rest
    assert host_output["many"] == [313, 64, 1]          # 20000 / 64
    assert host_output["gas"] == [1, 20000, 1]
    assert host_output["short"] == [1, 40, 1]
    assert host_output["longest"][0] <= 26 * 33 and host_output["longest"][2] == 1
