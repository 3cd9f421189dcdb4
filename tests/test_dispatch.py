"""The launch rules of the linear kernels (csrc/dispatch.h) over every shape the library accepts, on the host: each
rule is compiled into a small program that walks the sizes and prints the first launch that breaks a bound of its
kernel."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_36590_amd", "csrc")

HEAD = r"""
#include "dispatch.h"
#include <cstdio>
#include <cstdlib>
using namespace seedk;
#define CHECK(c, ...) do { if (!(c)) { printf("%s: ", #c); printf(__VA_ARGS__); printf("\n"); exit(1); } } while (0)
static const int ROWS[] = {1, 2, 5, 15, 16, 17, 31, 32, 33, 40, 47, 48, 49, 63, 64};
"""


def _run(tmp_path, body):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(HEAD + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    return r.stdout


def test_decode_projections_fit_their_kernels(tmp_path):
    """Threads within the launch bounds, partial sums within LDS, every n-tile and k-range covered, and k-ranges that
    depend on the weight shape alone: hidden and ffn sizes of any multiple of 32 up to 32768 as K, N from one n-tile
    to a wide ffn, with the rows of every decode pass."""
    _run(tmp_path, r"""
int main() {
  const int wide[] = {384, 511, 512, 768, 1216, 1280, 1281, 2047, 3584, 4096};
  for (int kt = 1; kt <= 1024; ++kt)
    for (int i = 1; i <= 300 + 10; ++i) {
      const int nt = i <= 300 ? i : wide[i - 301];
      for (int epi : {EPI_QKV, EPI_RESID, EPI_SWIGLU, EPI_HEAD})
        for (int es : {2, 4})
          for (int M : ROWS) {
            const RowsPlan p = rows_plan(nt * 16, kt * 32, M, epi, es);
            CHECK(p.threads <= (p.part ? ROWS_PART_THREADS : ROWS_THREADS),
                  "N %d K %d rows %d epilogue %d: %d threads", nt * 16, kt * 32, M, epi, p.threads);
            CHECK(p.lds <= ROWS_LDS, "N %d K %d rows %d epilogue %d: %zu bytes", nt * 16, kt * 32, M, epi, p.lds);
            CHECK(p.KS >= 1 && p.KS <= std::min(kt, ROWS_KS_MAX), "N %d K %d epilogue %d: %d k-ranges", nt * 16, kt * 32, epi, p.KS);
            CHECK(p.KS == rows_plan(nt * 16, kt * 32, 1, epi, es).KS, "N %d K %d rows %d: k-ranges", nt * 16, kt * 32, M);
            CHECK(!p.part || epi == EPI_RESID, "N %d K %d epilogue %d", nt * 16, kt * 32, epi);
            CHECK(p.gx * p.NT >= nt && (p.gx - 1) * p.NT < nt, "N %d: %d workgroups of %d", nt * 16, p.gx, p.NT);
            CHECK(p.part ? p.gy * 2 >= p.KS && p.gy * 2 <= p.KS + 1 : p.gy == 1 && p.threads == 64 * p.KS,
                  "K %d: %d k-ranges in %d x %d threads", kt * 32, p.KS, p.gy, p.threads);
            CHECK(p.NT == 1 || p.NT == 2 || p.NT == 3 || (p.NT == 5 && (p.part || M <= 48)), "%d n-tiles, %d rows", p.NT, M);
          }
    }
}
""")


def test_split_wide_passes_use_all_their_partials(tmp_path):
    """k-ranges that leave none empty, and no more partials in the workspace than some shape uses."""
    _run(tmp_path, r"""
int main() {
  int most = 0;
  for (int kt = 1; kt <= 2048; ++kt)
    for (int nt = 2; nt <= 2048; ++nt) {
      const int s = wide_split(nt, kt);
      CHECK(s >= 1 && s <= kt && s <= WIDE_SPLIT_MAX, "N %d K %d: %d", nt * 16, kt * 32, s);
      most = std::max(most, s);
    }
  CHECK(most == WIDE_SPLIT_MAX, "partials for %d k-ranges, %d used", WIDE_SPLIT_MAX, most);
}
""")


def test_wide_shapes_cover_every_width(tmp_path):
    """The GPU test's wide shapes pick every number of n-tiles per wave (1 is the only one for its small shapes) in
    gate/up, the head and the residual projections, each with a wave partly filled or left empty."""
    from test_gpu_wide import MANY_TILES
    rows = ", ".join("{%s}" % ", ".join(map(str, s)) for s in MANY_TILES)
    _run(tmp_path, "static const int S[][6] = {" + rows + "};" + r"""
static unsigned seen[3];
static void add(int e, int nt, int M, int S) {
  const int ni = wide_ni(nt, M, S), last = nt % (4 * ni);
  if (last % ni || (last && last <= 3 * ni)) seen[e] |= 1u << ni;
}
int main() {
  for (auto& s : S) {
    const int nt = s[0] / 16, M = s[5];
    CHECK(M > 1024, "%d rows", M);
    add(0, 2 * s[3] / 16, M, 1);
    add(1, s[4] / 16, M, 1);
    add(2, nt, M, wide_split(nt, s[1] * 2));
    add(2, nt, M, wide_split(nt, s[3] / 32));
  }
  for (int e = 0; e < 3; ++e) CHECK((seen[e] | 2u) == 126u, "projection %d: widths %x", e, seen[e]);
}
""")


def test_heads_fit_their_kernels(tmp_path):
    """LDS of the LM head's kernels, for hidden sizes of any multiple of 32 up to 32768 and every row count: the rows
    staged whole only while they fit, chunks within the CU's LDS beside the row scales, the sums within the chunks."""
    _run(tmp_path, r"""
int main() {
  const int tiles[] = {1, 63, 64, 2000, 2047, 2048, 2049, 5119, 5120, 5121, 9496, 16384, 16385};
  for (int kt = 1; kt <= 1024; ++kt)
    for (int nt : tiles)
      for (int es : {2, 4})
        for (int M = 1; M <= 64; ++M) {
          const HeadPlan p = head_plan(nt * 16, kt * 32, M, es);
          CHECK(p.lds + (p.chunked ? 256 : 0) <= LDS_MAX, "N %d K %d rows %d: %zu bytes", nt * 16, kt * 32, M, p.lds);
          CHECK(p.chunked || M <= 16, "N %d K %d rows %d", nt * 16, kt * 32, M);
          CHECK(!p.chunked || (size_t)HEAD_NT * M * 64 <= p.lds, "rows %d: %zu bytes for the sums", M, p.lds);
          CHECK(p.grid * p.NT * HEAD_NT >= nt && (p.grid - 1) * p.NT * HEAD_NT < nt, "N %d: %d workgroups", nt * 16, p.grid);
        }
  static_assert(ROWS_LDS + 256 <= LDS_MAX, "the row kernel's sums and row scales");
}
""")


def test_attention_groups(tmp_path):
    """Positions per group for every pair of capacities: one sequence 64 up to 4096, 128 up to 8192, then 256; several
    sequences the same from 4097 positions on and 64 up to 1024, in between 64 up to 2048 while the batch capacity is
    at most 4, else up to 8192 / min(batch, 8). Decoders with the same figure give a sequence the same bits."""
    _run(tmp_path, r"""
int main() {
  for (int b = 1; b <= 64; ++b)
    for (int n = 2; n <= 20000; ++n) {
      const int s = attention_span(n, b), one = n <= 4096 ? 64 : n <= 8192 ? 128 : 256;
      const int small = b == 1 ? 4096 : b <= 4 ? 2048 : 8192 / std::min(b, 8);
      CHECK(s == (n <= small ? 64 : std::max(one, 128)), "capacity %d, batch %d: %d", n, b, s);
      CHECK((n > 1024 && n <= 4096) || s == one, "capacity %d, batch %d: %d", n, b, s);
    }
}
""")
