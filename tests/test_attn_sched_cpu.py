"""The attention kernels' work split (csrc/attn_sched.hpp), compiled for the host, against 64-bit arithmetic."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "attn_sched.hpp"
#include <stdio.h>
#include <stdlib.h>
using namespace sx;
static long checked = 0, bad = 0;
static void expect(bool ok, const char* what, long a, long b, long c, long d) {
  ++checked;
  if (!ok && ++bad < 10) printf("%s: %ld %ld %ld %ld\n", what, a, b, c, d);
}
static long below(long n) { return ((static_cast<long>(rand()) << 20) ^ rand()) % n; }

// shares of a line of T granules over W workgroups
static void shares(const AttnLine& l) {
  const long T = l.T, W = l.W;
  expect(T == static_cast<long>(l.q) * W + l.r && l.q >= 1 && l.r >= 0 && l.r < W, "quotient", T, W, l.q, l.r);
  expect(attn_sched_lo(l, 0) == 0 && attn_sched_lo(l, l.W) == l.T, "ends", T, W, 0, 0);
  for (int i = 0; i < 40; ++i) {
    const long w = i < 3 ? i % W : i < 6 ? W - 1 - i % 3 % W : below(W);
    const long lo = w * T / W, hi = (w + 1) * T / W;
    expect(attn_sched_lo(l, w) == lo && attn_sched_lo(l, w + 1) == hi, "share", T, W, w, attn_sched_lo(l, w));
  }
}

// The segments of all workgroups of a launch over `len` entries (the block's n_blk included) per sequence, as the split kernels walk them:
// every unit's keys are taken once and in order, one workgroup finds the first of them and one the last (what the merging kernel is
// told), and those between take the slots between.
static void segments(const int* len, int B, int Hkv, int n_blk, int pad, int wide_from, int spread, int wgrid) {
  static int S[1025], keys[1024 * 64], first[1024 * 64], last[1024 * 64], seen[1024 * 64];
  S[0] = 0;
  for (int b = 0; b < B; ++b) S[b + 1] = S[b] + (len[b] + kAttnGran - 1) / kAttnGran;
  const AttnLine l = attn_sched_line(S[B], B, Hkv, pad, wide_from, spread, wgrid);
  for (int u = 0; u < B * Hkv; ++u) { keys[u] = seen[u] = 0; first[u] = last[u] = -1; }
  long slot = -1;
  for (int w = 0; w < l.W; ++w) {
    const int hi = attn_sched_lo(l, w + 1);
    for (int x = attn_sched_lo(l, w), b = 0; x < hi;) {
      while (b < B - 1 && static_cast<long>(Hkv) * (S[b + 1] + l.pad * (b + 1)) <= x) ++b;
      const AttnSeg s = attn_sched_cut(Hkv, n_blk, l.pad, b, S[b], S[b + 1] - S[b], len[b] - n_blk, x, hi);
      expect(s.next > x && s.next <= hi, "next", x, hi, s.next, l.W);
      x = s.next;
      if (s.s1 <= s.s0) continue;
      const int u = s.b * Hkv + s.g;
      expect(s.g >= 0 && s.g < Hkv && s.s0 == keys[u] && s.s1 <= len[b], "keys", u, s.s0, s.s1, keys[u]);
      keys[u] = s.s1;
      if (s.s0 == 0) { expect(first[u] < 0, "one first", u, first[u], w, 0); first[u] = w; }
      if (s.s1 == s.L + n_blk) { expect(last[u] < 0, "one last", u, last[u], w, 0); last[u] = w; }
      expect(first[u] >= 0 && w == first[u] + seen[u], "consecutive", u, first[u], seen[u], w);
      ++seen[u];
      expect(w + u > slot && w + u < l.W + B * Hkv, "slot", w, u, slot, l.W);
      slot = w + u;
    }
  }
  for (int u = 0; u < B * Hkv; ++u) expect(keys[u] == len[u / Hkv] && last[u] == first[u] + seen[u] - 1, "whole unit", u, keys[u], len[u / Hkv], last[u]);
}

int main() {
  srand(1);
  // the lines of launches: W from the sizes, for any lengths that the planned number of workgroups has to do for
  for (int k = 0; k < 60000; ++k) {
    const int B = k % 4 == 0 ? 1 + below(1024) : 1 + below(24), Hkv = 1 + below(k % 3 ? 8 : 64), pad = below(4);
    const int gran = B + (k % 5 == 0 ? below(1l << 20) / Hkv : below(k % 2 ? 40 : 700));
    const int wide_from = static_cast<long>(B) * Hkv >= kAttnSpread ? 0 : 1000 + below(2601), wgrid = k % 7 == 0 ? kAttnMaxGrid : k % 2 ? 256 : 512;
    const AttnLine l = attn_sched_line(gran, B, Hkv, pad, wide_from, k % 3 == 1, wgrid);
    const long bare = static_cast<long>(gran) * Hkv, T = bare + (bare > kAttnSpread ? static_cast<long>(B) * Hkv * pad : 0);
    expect(l.T == T && l.W >= 1 && l.W <= wgrid && l.W <= T, "line", gran, B, Hkv, l.W);
    if (bare > kAttnSpread && bare < wide_from)       // the middle range: no share above what 256 workgroups would have
      expect(l.W <= kAttnSpread && (T + l.W - 1) / l.W == (T + kAttnSpread - 1) / kAttnSpread, "largest share", T, l.W, B, Hkv);
    shares(l);
    // sequences of one length: where a whole number of workgroups per unit keeps the share, every unit begins a share
    const long n = gran / B + l.pad, units = static_cast<long>(B) * Hkv;
    if (gran % B == 0 && bare > kAttnSpread && bare < wide_from && l.W % units == 0)
      for (long u = 0; u < units; ++u) {
        const int w = (u * n * l.W + T - 1) / T;
        expect(attn_sched_lo(l, w) == u * n, "unit start", T, l.W, u, w);
      }
  }
  // the segments of launches: few and many sequences, empty, equal and very unequal ones, with and without padding
  static int len[1024];
  for (int k = 0; k < 6000; ++k) {
    const int B = k % 50 == 0 ? 1 + below(1024) : 1 + below(k % 2 ? 8 : 70), Hkv = 1 + below(k % 10 ? 8 : 64), n_blk = 1 + below(64);
    const int most = k % 3 == 0 ? 100 : k % 3 == 1 ? 3000 : 40000, same = below(most);
    for (int b = 0; b < B; ++b) len[b] = n_blk + (k % 4 == 0 ? same : below(5) ? below(most) : 0);
    if (k % 500 == 7 && Hkv <= 8) len[below(B)] = n_blk + (1 << 29) + below(100000);      // (more granules than the divisions by floats take)
    segments(len, B, Hkv, n_blk, below(4), static_cast<long>(B) * Hkv >= kAttnSpread ? 0 : k % 2 ? 2400 : 1000 + below(2601), k % 7 == 1, k % 11 == 0 ? kAttnMaxGrid : k % 2 ? 256 : 512);
  }
  // any line, to the limits
  for (long W = 1; W <= kAttnMaxGrid; W += W < 700 ? 1 : 37)
    for (long T : {W, W + 1, 2 * W - 1, 2 * W, 2 * W + 1, 3 * W + W / 2, W + below(4000), W + below((1l << 30) - W), (1l << 30) - 1}) {
      AttnLine l{};
      l.T = T; l.W = W; l.q = T / W; l.r = T % W;
      shares(l);
    }
  printf("%ld checks, %ld wrong\n", checked, bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_shares_and_segments_of_the_work_split(tmp_path):
    src = tmp_path / "sched.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "sched"
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-I", os.path.join(ROOT, "paper_2509_24248_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
    assert int(run.stdout.split()[0]) > 5_000_000


OWNERS = r"""
#include "kernels.hpp"
#include <stdio.h>
#include <stdlib.h>
using namespace sx;
int main() {
  srand(2);
  long checked = 0, bad = 0;
  for (int k = 0; k < 200000; ++k) {
    const long most = k % 3 == 0 ? 1l << 22 : k % 3 == 1 ? 60000 : 300;
    const long T = 1 + ((static_cast<long>(rand()) << 16) ^ rand()) % most;
    const long W = T < 4 ? 1 : 1 + rand() % (T / 2 < 1023 ? T / 2 : 1023);
    const uint32_t inv = proj_inverse(T);
    for (int i = 0; i < 12; ++i) {
      const long w = rand() % W, start = w * T / W;
      const long x = i == 0 ? 0 : i == 1 ? T - 1 : i < 6 ? start : i < 9 ? (start > 0 ? start - 1 : 0) : rand() % T;
      const long o = proj_owner(T, inv, W, x);
      ++checked;
      if (o < 0 || o >= W || o * T / W > x || (o + 1) * T / W <= x) if (++bad < 10) printf("T %ld W %ld x %ld: %ld\n", T, W, x, o);
    }
  }
  printf("%ld checks, %ld wrong\n", checked, bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_owners_of_the_projections_blocks(tmp_path):
    src = tmp_path / "owners.hip"
    src.write_text(OWNERS)
    exe = tmp_path / "owners"
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-I", os.path.join(ROOT, "paper_2509_24248_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
