"""What a context remembers of its recent calls, run on the host: sequences of
calls, the words that their launches would store, and the launches chosen."""
from host_program import run

HEAD = '#include "fgbd_adapt.h"\n'

# calls "entry clouds n needed": the call asks when nothing is outstanding, its
# words are stored at once, and the chosen count is printed
CALLS = """
int main(int argc, char **argv) {
  SweepCounts s;
  int32_t words[64] = {0};
  for (int i = 1; i + 3 < argc; i += 4) {
    const int clouds = atoi(argv[i + 1]), needed = atoi(argv[i + 3]);
    const CallKind kind = call_kind(atoi(argv[i]), clouds, atoll(argv[i + 2]));
    s.poll(words);
    if (!s.pending()) {
      const int32_t tag = s.ask(kind, clouds, words);
      for (int c = 0; c < clouds; ++c) words[c] = (c ? 1 : needed) | tag;
    }
    printf("%d\\n", s.launches(kind, 8, 64));
  }
}
"""
DENOISE, BATCHED, FILTER = 0, 1, 2


def chosen(tmp_path, calls):
    return [int(w) for w in run(tmp_path, HEAD, CALLS, *[v for c in calls for v in c])]


def test_follows_the_calls_of_one_kind(tmp_path):
    frame, batch = (DENOISE, 1, 1000000, 4), (BATCHED, 64, 262144, 31)
    got = chosen(tmp_path, [frame] * 3 + [batch] * 3 + [frame, batch] * 4 + [frame] * 2)
    assert got[:3] == [8, 5, 4]  # nothing known, one count, two that agree
    assert got[3:6] == [8, 32, 31]
    assert got[6::2][:4] == [4] * 4 and got[7::2][:4] == [31] * 4 and got[-2:] == [4, 4]


def test_kinds_are_entry_clouds_and_magnitude(tmp_path):
    kinds = [(DENOISE, 1, 5000), (FILTER, 1, 5000), (BATCHED, 1, 5000), (BATCHED, 2, 5000), (DENOISE, 1, 100000)]
    needed = [3, 7, 12, 20, 40]
    rounds = [(*k, q) for _ in range(4) for k, q in zip(kinds, needed)]
    assert chosen(tmp_path, rounds)[-5:] == needed


def test_counts_that_vary_and_the_limit(tmp_path):
    got = chosen(tmp_path, [(DENOISE, 1, 777, q) for q in (3, 9, 3, 3, 3, 3, 3, 3, 3, 3, 3, 200, 3)])
    assert got == [8, 4] + [10] * 8 + [3, 3, 64]


def test_more_kinds_than_records(tmp_path):
    """The least recently used kind is forgotten, not a wrong one taken for it."""
    many = [(BATCHED, b, 5000, b) for b in range(1, 10)]
    got = chosen(tmp_path, many * 3)
    assert all(g in (8, b[3], b[3] + 1) for g, b in zip(got, many * 3))
    assert got[-1] == 8 and chosen(tmp_path, many[:8] * 3)[-8:] == list(range(1, 9))


# a batch of 64 once, then single frames until the tags have come round, then a
# batch whose clouds are stored one by one
TAGS = """
int main(int argc, char **argv) {
  SweepCounts s;
  int32_t words[64] = {0};
  const CallKind frame = call_kind(kCallDenoise, 1, 1000), batch = call_kind(kCallBatched, 64, 4096);
  int64_t bad = 0;
  int32_t tag = s.ask(batch, 64, words);
  const int32_t first = tag;
  for (int c = 0; c < 64; ++c) words[c] = 50 | tag;
  s.poll(words);
  do {
    tag = s.ask(frame, 1, words);
    bad += tag <= 0 || (tag & 0xffff) != 0 || !s.pending() || !s.outstanding(words);
    words[0] = 4 | tag;
    bad += s.outstanding(words);
    s.poll(words);
    bad += s.pending();
  } while (tag != 0x7fff0000);  // the largest tag; the batch's own is next
  tag = s.ask(batch, 64, words);
  bad += tag != first;
  for (int c = 0; c < 64; ++c) {
    s.poll(words);
    bad += !s.pending() || !s.outstanding(words);
    words[c] = 7 | tag;
  }
  bad += s.outstanding(words);
  s.poll(words);
  bad += s.pending() || s.launches(batch, 8, 64) != 51 || s.launches(frame, 8, 64) != 4;
  printf("%lld\\n", (long long)bad);
}
"""


def test_tags_that_come_round(tmp_path):
    assert run(tmp_path, HEAD, TAGS) == ["0"]


FAILED = """
int main(int argc, char **argv) {
  int64_t bad = 0;
  const CallKind kind = call_kind(kCallDenoise, 1, 1000);
  SweepCounts s;
  int32_t words[64] = {0};
  s.ask(kind, 1, words);
  s.cancel();  // the call failed: nothing will be stored
  s.poll(words);
  bad += s.pending() || s.outstanding(words) || !s.unsure();
  for (int i = 0; i < 3; ++i) {  // later calls adapt as before
    words[0] = 5 | s.ask(kind, 1, words);
    s.poll(words);
  }
  bad += s.pending() || s.launches(kind, 8, 64) != 5;
  // a count that the failed call's launches did store is not taken for another's
  const int32_t late = 60 | s.ask(kind, 1, words);
  s.cancel();
  s.ask(kind, 1, words);
  words[0] = late;
  s.poll(words);
  bad += !s.pending() || !s.outstanding(words) || s.launches(kind, 8, 64) != 5;

  SortWatch w;
  int32_t flag[2] = {0, 0};
  bad += w.lsd(flag) || w.unsure();
  w.ask(flag);
  w.cancel();
  bad += w.pending() || w.outstanding(flag) || !w.unsure() || w.lsd(flag);
  const int32_t seq = w.ask(flag);
  bad += !w.pending() || !w.outstanding(flag) || w.lsd(flag);
  flag[0] = 1;
  flag[1] = seq;
  bad += w.outstanding(flag);
  for (int i = 0; i < SortWatch::kCalls; ++i) bad += !w.lsd(flag) || w.pending();
  bad += w.lsd(flag);
  printf("%lld\\n", (long long)bad);
}
"""


def test_a_call_that_failed(tmp_path):
    assert run(tmp_path, HEAD, FAILED) == ["0"]


TRIALS = """
int main(int argc, char **argv) {
  for (int before = 0; before < 2; ++before)
    for (int kept = 0; kept < 2; ++kept) {
      bool chosen = before;
      int during = 0;
      {
        ScheduleTrial t(chosen);
        t.start();
        during = chosen;
        if (kept) t.keep();
      }
      printf("%d%d\\n", during, (int)chosen);
    }
}
"""


def test_a_tuning_that_fails_leaves_the_mark(tmp_path):
    # (not chosen before: failed, kept; chosen before: failed, kept)
    assert run(tmp_path, HEAD, TRIALS) == ["10", "11", "11", "11"]


ROUTES = """
int main(int argc, char **argv) {
  int64_t bad = 0;
  SortWatch w;
  int32_t flag[2] = {0, 0};
  auto asked = [&](bool crowded, int32_t seq) {
    flag[0] = crowded;
    flag[1] = seq;
  };
  // nothing known: calls made ahead of the first answer keep the default
  bad += w.last_crowded(flag) || w.lsd(flag);
  int32_t seq = w.ask(flag);
  for (int i = 0; i < 50; ++i) bad += w.lsd(flag) || w.last_crowded(flag);
  asked(true, seq);
  bad += !w.last_crowded(flag);  // (a captured call: counts as no call)
  for (int round = 0; round < 3; ++round) {
    for (int i = 0; i < SortWatch::kCalls; ++i) bad += !w.lsd(flag) || w.pending();
    bad += w.lsd(flag);  // this one asks again ...
    seq = w.ask(flag);
    for (int i = 0; i < 50; ++i) bad += !w.lsd(flag) || !w.last_crowded(flag);  // ... and those ahead of its answer do not try
    asked(round < 2, seq);
  }
  for (int i = 0; i < 50; ++i) bad += w.lsd(flag) || w.last_crowded(flag) || w.pending();
  printf("%lld\\n", (long long)bad);
}
"""


def test_routes_ahead_of_the_answer(tmp_path):
    assert run(tmp_path, HEAD, ROUTES) == ["0"]
