"""Index arithmetic of the kernels at the largest sizes that the calls accept,
run on the host: a program built from the library's own header walks the
indexes that a block forms and prints what it finds."""
from host_program import run

HEAD = '#include "fgbd_internal.h"\n'

EDGES = """
int main(int argc, char **argv) {
  // a block's edges first .. end - 1, walked as the adjoint's step does
  for (int i = 1; i + 1 < argc; i += 2) {
    const long long first = atoll(argv[i]), end = atoll(argv[i + 1]);
    long long passes = 0, stored = 0, bad = 0;
    EdgePass p;
    p.c0 = (uint32_t)first;
    p.end = (uint32_t)end;
    for (; p.more() && passes < 100000000; p.next(), ++passes) {
      const long long c0 = first + passes * kBackEdges;
      for (int q = 0; q < kBackEdges; q += (c0 + kBackEdges < end ? kBackEdges - 1 : 1)) {
        const long long want = c0 + q < end ? c0 + q : end - 1;
        bad += (long long)p.edge(q) != want || p.holds(q) != (c0 + q < end);
        stored += p.holds(q);
      }
      for (long long b : {first, c0, c0 + 1, end}) {
        const long long top = b < c0 + kBackEdges ? b : c0 + kBackEdges;
        bad += b <= end && (long long)p.below((uint32_t)b) != top - c0;
      }
    }
    printf("%lld %lld %lld\\n", passes, stored, bad);
  }
}
"""


def test_adjoint_edges_at_the_limit(tmp_path):
    """Graphs of n * k edges up to 2^31 - 1: the last block of points, a block
    that holds none, one that holds every edge, and ends around the limit."""
    top = 2**31 - 1
    step = 2048
    blocks = [(0, 0), (0, 1), (0, step), (0, step + 1), (2_147_481_600, 2_147_483_640), (top - 1, top), (top - step, top),
              (top - step - 1, top), (top - 3 * step, top - step + 5), (0, top)]
    words = run(tmp_path, HEAD, EDGES, *[v for b in blocks for v in b])
    for i, (first, end) in enumerate(blocks):
        passes, stored, bad = map(int, words[3 * i:3 * i + 3])
        assert bad == 0, (first, end)
        assert passes == -(-(end - first) // step), (first, end)
        tail = (end - first) - (passes - 1) * step if passes else 0
        assert stored == tail + 2 * max(passes - 1, 0), (first, end)


POINTS = """
int main(int argc, char **argv) {
  for (int i = 1; i < argc; ++i) {
    const int pos = atoi(argv[i]);
    const int32_t *xyz = (const int32_t *)0x10000;  // (never read)
    printf("%lld\\n", (long long)((uintptr_t)point_at(xyz, pos) - (uintptr_t)xyz));
  }
}
"""


def test_point_offsets_at_the_limit(tmp_path):
    """Coordinates are 12 bytes a point up to the largest n that the calls take."""
    at = [0, 1, 4096, 715_827_882, 715_827_883, 1_500_000_000, 2**31 - 1 - 4096]
    assert [int(w) for w in run(tmp_path, HEAD, POINTS, *at)] == [12 * p for p in at]
