"""The fragment addresses of the fp16 attention kernel, on the CPU: for sizes
that the library accepts, up to the largest, the 64-bit bases and 32-bit
offsets that the kernel adds up give the positions of the tiled layouts."""
import os
import subprocess

import pytest

from paper_2606_07878_amd import build

DRIVER = r"""
#include <cstdio>
#include "host.hpp"
using namespace still;

// One head's fragments as the kernel's waves address them; wrong ones counted.
static long head(long N, long npad, int dc, int d2, int KT, const char* what) {
  const unsigned ksteps = dc >> 4, nsteps = (unsigned)(npad >> 4), ktlast = (unsigned)(npad >> 5) - 1;
  const int KW = 32 * KT, KB = 4 * KW, FT = d2 / 128;
  long bad = 0;
  for (int w = 0; w < 4; ++w) {
    const long blocks[] = {0, KB, (N / 2) / KB * KB, (N - 1) / KB * KB};
    for (long n0 : blocks)
      for (int kt = 0; kt < KT; ++kt)
        for (unsigned js : {0u, ksteps - 1}) {
          const unsigned tile0 = xatt_ktile0((unsigned)(n0 + KW * w), ktlast);
          const long at = 2 * xatt_kbase(tile0, ksteps) + (long)xatt_koff(tile0, ktlast, kt, ksteps, js);
          const long n = std::min(n0 + KW * w + 32 * kt, npad - 32);   // tiles past the last one: the last one
          bad += at != 2 * ktile_off(0, n, 16 * (long)js, npad, dc);
        }
    for (int f = 0; f < FT; ++f)
      for (long ns : {0l, (long)nsteps / 2, (long)nsteps - 1, (long)nsteps + 3}) {
        const long at = 2 * xatt_xbase(FT * w, nsteps) + (long)xatt_xoff(f, nsteps, (unsigned)ns);
        const long k = std::min(16 * ns, npad - 16);
        bad += at != 2 * xtile_off(0, 32l * (FT * w + f), k, npad, d2);
      }
  }
  if (bad) printf("%s: %ld wrong\n", what, bad);
  return bad;
}

int main() {
  long bad = 0;
  int accepted = 0;
  for (int d : {64, 128, 256})
    for (int nc : {1, 3, 8})
      for (int dc : {128, 384, 640, 768, 1024, 2048, 1 << 20, 1 << 22, (1 << 24) - 128, 1 << 24}) {
        still_config c = {};
        c.n_kv_heads = 1;
        c.head_dim = d;
        c.latent_dim = 256;
        c.n_blocks = 1;
        c.n_cross_heads = nc;
        c.cross_head_dim = dc;
        c.compactor_rope_base = 10.0;
        c.rms_eps = 1e-6f;
        c.l2_eps = 1e-12f;
        const long span = ((1l << 31) - 1) / ((long)nc * dc);   // most keys of a head below 4 GiB
        for (long N : {1l, 300l, 4194304l, 4194305l, 5000000l, 8000000l, 128l * 65535, span})
          for (int t : {1, 65}) {
            Dims m;
            if (N < 1 || make_dims(&c, N, t, &m) != STILL_OK) continue;
            ++accepted;
            char what[128];
            snprintf(what, sizeof what, "d=%d nc=%d dc=%d N=%ld", d, nc, dc, N);
            bad += head(m.N, m.Npad, m.dc, m.d2, key_block(m) / 128, what);
          }
      }
  printf("%d sizes, %ld wrong\n", accepted, bad);
  return bad != 0 || accepted < 100;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_fragment_addresses_of_accepted_sizes(tmp_path):
    src, exe = tmp_path / "offsets.hip", tmp_path / "offsets"
    src.write_text(DRIVER)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "-o", str(exe), str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr
