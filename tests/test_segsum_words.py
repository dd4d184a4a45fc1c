"""The words by which Seg-Sum's waves announce pieces (csrc/segsum_words.hpp),
compiled for the host: every interleaving of the memory operations of the waves
around a cut segment, from every kind of word that an earlier call can have
left. In each, exactly one wave learns that it added a segment's last piece,
when all its pieces are stored, and a flag is seen only once its piece is."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_10045_amd", "csrc")

# A wave is a list of steps, each with one memory operation: load a word, claim
# it with what was loaded, store a piece, add to a word. "add_first" is a
# protocol that the enumeration has to reject: only the wave's own word is
# claimed, and others are added to before their tag is looked at.
MODEL = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>
#include "segsum_words.hpp"
using namespace lmz;

struct Host {
  void exchange_if(uint64_t* w, uint64_t seen, uint64_t x) const { if (*w == seen) *w = x; }
  uint64_t add(uint64_t* w, uint64_t x) const { const uint64_t o = *w; *w += x; return o; }
};
enum What { LOAD, CLAIM, STORE, FLAG, COUNT };
struct Step { What what; int word; int seg; };  // seg: of STORE and COUNT
struct Seg { int first, P; };                   // its first chunk, further pieces
using Wave = std::vector<Step>;

static const uint64_t TAG = 0x1234567;
static bool add_first = false;

struct State {
  std::vector<uint64_t> words;                // per chunk
  std::vector<uint64_t> pc, sub, cur;         // per wave; cur: what it loaded, per word
  std::vector<uint64_t> stored, finished, headed;  // per segment; headed: per chunk
  std::vector<uint64_t> key() const {
    std::vector<uint64_t> k;
    for (auto* v : {&words, &pc, &sub, &cur, &stored, &finished, &headed})
      k.insert(k.end(), v->begin(), v->end());
    return k;
  }
};

struct Model {
  std::vector<Wave> waves;
  std::vector<Seg> segs;
  std::vector<int> head;  // chunk c has a piece of a head
  std::set<std::vector<uint64_t>> seen;
  const char* bad = nullptr;

  bool step(State& s, size_t w) {
    const Step& st = waves[w][s.pc[w]];
    uint64_t* word = &s.words[st.word];
    uint64_t& cur = s.cur[w * s.words.size() + st.word];
    const uint64_t x = st.what == FLAG ? kPieceFlag : 1;
    uint64_t now = 0;
    bool done = true;
    switch (st.what) {
      case LOAD: cur = *word; break;
      case CLAIM: word_claim(Host{}, word, cur, TAG); break;
      case STORE:
        if (st.seg >= 0) ++s.stored[st.seg];
        else s.headed[st.word] = 1;
        break;
      default:
        if (!add_first) {
          now = word_add(Host{}, word, x);
        } else if (s.sub[w] == 0) {
          const uint64_t old = Host{}.add(word, x);
          now = old + x;
          if (!word_is(old, TAG)) { done = false; s.sub[w] = 1; }
        } else if (s.sub[w] == 1) {
          cur = *word;
          done = false;
          s.sub[w] = word_is(cur, TAG) ? 0 : 2;
        } else if (*word == cur) {
          now = *word = (TAG << kTagShift) | x;
        } else {
          done = false;
          s.sub[w] = 1;
        }
        if (done && st.what == COUNT) {
          const Seg& g = segs[st.seg];
          if (word_count(now) == uint64_t(g.P + 1)) {
            if (s.stored[st.seg] != uint64_t(g.P + 1)) bad = "summed before all its pieces are stored";
            ++s.finished[st.seg];
          }
        }
    }
    if (done) { ++s.pc[w]; s.sub[w] = 0; }
    for (size_t c = 0; c < s.words.size(); ++c)
      if (word_is(s.words[c], TAG) && (s.words[c] & kPieceFlag) && !s.headed[c])
        bad = "a flag without its piece";
    return !bad;
  }
  void run(const State& s) {
    if (bad || !seen.insert(s.key()).second) return;
    bool any = false;
    for (size_t w = 0; w < waves.size() && !bad; ++w) {
      if (s.pc[w] >= waves[w].size()) continue;
      any = true;
      State n = s;
      if (step(n, w)) run(n);
    }
    if (any || bad) return;
    for (size_t g = 0; g < segs.size(); ++g)
      if (s.finished[g] != 1) bad = s.finished[g] ? "summed twice" : "never summed";
    for (size_t c = 0; c < head.size(); ++c)
      if (head[c] && !(word_is(s.words[c], TAG) && (s.words[c] & kPieceFlag))) bad = "a flag is lost";
  }
};

// Chunk c's wave, from the segments: heads first[c] / starts[c], or counted ones.
static Wave wave_of(int c, const std::vector<Seg>& segs, bool ends_head, bool starts_head) {
  Wave w;
  int cont = -1, start = -1;
  for (size_t g = 0; g < segs.size(); ++g) {
    if (segs[g].first == c) start = int(g);
    else if (segs[g].first < c && c <= segs[g].first + segs[g].P) cont = int(g);
  }
  const bool other = cont >= 0 && !add_first;
  w.push_back({LOAD, c, -1});
  if (other) w.push_back({LOAD, segs[cont].first, -1});
  w.push_back({CLAIM, c, -1});
  if (other) w.push_back({CLAIM, segs[cont].first, -1});
  if (ends_head || starts_head) w.push_back({STORE, c, -1});
  if (cont >= 0) w.push_back({STORE, c, cont});
  if (start >= 0) w.push_back({STORE, c, start});
  if (ends_head) w.push_back({FLAG, c, -1});
  if (cont >= 0) w.push_back({COUNT, segs[cont].first, cont});
  if (start >= 0) w.push_back({COUNT, c, start});
  if (starts_head && !ends_head) w.push_back({FLAG, c, -1});
  return w;
}

int main(int argc, char** argv) {
  add_first = argc > 1 && atoi(argv[1]);
  struct Scene { int chunks; std::vector<Seg> segs; int ends_head, starts_head; };  // chunk or -1
  const std::vector<Scene> scenes = {
      {2, {{0, 1}}, 0, -1},          // a head ends where a segment of two pieces starts
      {3, {{0, 2}}, 0, -1},          // ... of three pieces
      {3, {{0, 1}, {1, 1}}, 0, 2},   // a segment ends where the next starts, then a head
      {3, {{0, 1}, {1, 1}}, -1, 2},
      {2, {{0, 1}}, -1, 1},
      {4, {{0, 3}}, 0, -1},
  };
  std::vector<uint64_t> stale;
  for (uint64_t tag : {TAG - 1, TAG - 2, TAG + 1, uint64_t(0), kTagMask})
    for (uint64_t flag : {uint64_t(0), kPieceFlag})
      for (uint64_t n : {uint64_t(0), uint64_t(1), uint64_t(3), kCountMask})
        stale.push_back((tag << kTagShift) | flag | n);
  size_t states = 0;
  for (size_t i = 0; i < scenes.size(); ++i) {
    const Scene& sc = scenes[i];
    for (uint64_t old : stale) {
      Model m;
      m.segs = sc.segs;
      m.head.assign(sc.chunks, 0);
      if (sc.ends_head >= 0) m.head[sc.ends_head] = 1;
      if (sc.starts_head >= 0) m.head[sc.starts_head] = 1;
      for (int c = 0; c < sc.chunks; ++c)
        m.waves.push_back(wave_of(c, sc.segs, c == sc.ends_head, c == sc.starts_head));
      State s;
      s.words.assign(sc.chunks, old);
      s.pc.assign(sc.chunks, 0);
      s.sub = s.pc;
      s.cur.assign(sc.chunks * sc.chunks, 0);
      s.stored.assign(sc.segs.size(), 0);
      s.finished = s.stored;
      s.headed.assign(sc.chunks, 0);
      m.run(s);
      states += m.seen.size();
      if (m.bad) {
        printf("scene %zu from %#llx: %s\n", i, (unsigned long long)old, m.bad);
        return 1;
      }
    }
  }
  printf("%zu states\n", states);
  return 0;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("words")
    (d / "model.cpp").write_text(MODEL)
    exe = str(d / "model")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, "-o", exe, str(d / "model.cpp")],
                   check=True)
    return exe


def test_a_word_is_wide_enough(tmp_path):
    """The tag takes all but a byte of a word, the count 16 pieces and a flag."""
    (tmp_path / "w.cpp").write_text('''#include "segsum_words.hpp"
using namespace lmz;
static_assert(kTagShift <= 8 && kCountMask >= 16 && (kPieceFlag & kCountMask) == 0);
static_assert(word_is((kTagMask << kTagShift) | kPieceFlag | kCountMask, kTagMask));
static_assert(word_count((kTagMask << kTagShift) | kPieceFlag | 16) == 16);
''')
    subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", CSRC, str(tmp_path / "w.cpp")], check=True)


def test_every_interleaving_finishes_each_segment_once(model):
    r = subprocess.run([model, "0"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 10_000, r.stdout


def test_the_enumeration_rejects_adding_before_the_tag_is_known(model):
    r = subprocess.run([model, "1"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 1 and "scene" in r.stdout, r.stdout
