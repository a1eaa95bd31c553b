"""The bookkeeping of the pinned memory that descriptors pass through (csrc/staging.hpp), compiled for the host with a
runtime that records what is still to be read: copies happen only when an event behind them is waited for, those of a captured
call whenever its graph is replayed, so a place that is given out or freed too early is seen."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16102_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>
#include "staging.hpp"

struct Copy { const int32_t *p; long words; bool done; };
std::vector<Copy> copies;             // of the calls, in stream order
struct Block { int32_t *p; long words; };
std::vector<Block> blocks;
struct Mark { size_t behind; };
struct Kept { const int32_t *p; long words; int32_t value; };
std::vector<Kept> kept;               // of captured calls, the newest last
constexpr int CAPTURING = 1;          // a stream that is being captured
std::vector<Mark> marks;
void need(bool ok, const char *what) { if (!ok) { std::printf("%s\n", what); std::exit(1); } }
bool meet(const int32_t *p, long n, const int32_t *q, long m) { return p < q + m && q < p + n; }

struct Fake {
  typedef int Stream;
  typedef int Event;  // 1 + index into marks
  int create(Event *e) { marks.push_back({0}); *e = (int)marks.size(); return 0; }
  int destroy(Event) { return 0; }
  int alloc(int32_t **p, long words) {
    *p = static_cast<int32_t *>(std::aligned_alloc(64, (words * 4 + 63) / 64 * 64));
    blocks.push_back({*p, words});
    return 0;
  }
  int release(int32_t *p) {
    for (size_t i = 0; i < blocks.size(); ++i)
      if (blocks[i].p == p) {
        for (const Copy &c : copies) need(c.done || !meet(c.p, c.words, p, blocks[i].words), "freed while still to be read");
        for (const Kept &k : kept) need(!meet(k.p, k.words, p, blocks[i].words), "freed under a captured call");
        blocks.erase(blocks.begin() + i);
        std::free(p);
        return 0;
      }
    need(false, "freed twice");
    return 0;
  }
  // (an event that is recorded into a capture belongs to the graph: waiting for it waits for nothing)
  int record(Event e, Stream s) { marks[e - 1].behind = s == CAPTURING ? 0 : copies.size(); return 0; }
  int capturing(Stream s, bool *yes) { *yes = s == CAPTURING; return 0; }
  int wait(Event e) { for (size_t i = 0; i < marks[e - 1].behind; ++i) copies[i].done = true; return 0; }
  int wait_all() { for (Copy &c : copies) c.done = true; return 0; }
};

int main(int argc, char **argv) {
  bs::Staging<Fake> s;
  need(s.open(4096, 10240) == 0, "open");
  for (int i = 1; i < argc; ++i) {  // a call with a descriptor of that many words, "c": captured
    const bool captured = argv[i][0] == 'c';
    const long words = (std::atol(argv[i] + captured) + 3) / 4 * 4;
    int32_t *p = nullptr;
    need(s.place(words, captured ? CAPTURING : 0, &p) == 0, "place");
    need(reinterpret_cast<uintptr_t>(p) % 16 == 0, "not on a 16-byte boundary");
    bool inside = false;
    for (const Block &b : blocks) inside = inside || (p >= b.p && p + words <= b.p + b.words);
    need(inside, "outside the buffer");
    for (const Copy &c : copies) need(c.done || !meet(c.p, c.words, p, words), "given out while still to be read");
    for (long w = 0; w < words; ++w) p[w] = i;
    if (!captured) copies.push_back({p, words, false});
    else kept.push_back({p, words, i});
    // the last four captured calls can be replayed, and as many as fit a third of the memory set aside for them
    long sum = 0;
    for (size_t k = kept.size(), n = 0; k-- > 0; ++n) {
      sum += kept[k].words;
      if (n >= 4 && 3 * sum > 10240) { kept.erase(kept.begin(), kept.begin() + k + 1); break; }
    }
    for (const Kept &k : kept)
      for (long w = 0; w < k.words; ++w) need(k.p[w] == k.value, "overwritten under a captured call");
  }
  Fake().wait_all();
  kept.clear();
  s.close();
  need(blocks.empty(), "not given back");
  return 0;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    where = tmp_path_factory.mktemp("staging")
    (where / "t.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-o", str(where / "t"), str(where / "t.cpp")])

    def go(calls):
        r = subprocess.run([str(where / "t")] + [str(c) for c in calls], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout

    return go


@pytest.mark.parametrize("calls", [
    [1, 2, 3, 5, 4096, 4093, 1, 4096],             # odd lengths; a half filled by one descriptor
    [3000] * 7, [1500] * 11, [100] * 200,
    [4097, 4097, 4097],                            # one that no half holds, and the half behind it
    [4100, 5000, 6000, 6160, 9001, 3, 9001, 9001]])
def test_descriptors_in_flight_keep_their_places(run, calls):
    run(calls)


@pytest.mark.parametrize("calls", [
    ["c900"] + [3000] * 9,                         # both halves are turned to again behind it
    ["c900", 5000, 9001],                          # a larger buffer takes the place of theirs
    [3000, "c2000", 3000, 3000, 3000],             # the capture does not fit the half that a call in flight has begun
    ["c2000"] * 9, ["c40"] * 80, ["c700", "c2048", "c12", "c1999"] * 4, ["c3000", "c3000", 900, "c9001", "c5", "c100000", "c7", "c3"]])
def test_captured_descriptors_outlive_the_calls_behind_them(run, calls):
    run(calls)
