// Algorithm 1 on the host: which arcs to boost for a biasing list of word sequences.
//
// Two ways, with the same results.  A graph starts with the plain search: an index word -> arcs, and the graph's own
// arrays.  What bounds it is cache misses: a list's searches meet some ten thousand states spread over hundreds of
// megabytes.  So once they have met half as many states as the graph has (some hundred lists: until then the layout costs
// about as much as it gives, and a caller with a handful of lists never pays for one), the graph is laid out for them:
// each state is one contiguous record, and a reference to a state IS the position of its record, so that a visit is one
// miss, not three (row bounds, labels, destinations), prefetched when the reference is queued.  Most visits are not made
// at all: with a reference goes a signature, 64 bits of which those are set that the words hash to which the state or
// any state behind it (through arcs without label) can output, and a search for one word goes only where that word's bit
// is set (a signature of 120 words has it by chance in 85 of 100 cases, one of 13 words in 18, one of 4 in 6: three
// visits instead of forty from each arc of the previous word, where words lie four arcs apart).  The source states of a
// word's arcs are stored with the word, and the visited set is a small hash table that stays in L1.  Independent lists
// are shared out over host threads, and so is the layout.
//
// 2M / 10M states, lists of nine sequences, 16 threads: the word index takes 22 / 114 ms (first request), the layout
// 30 / 190 to 260 ms and 130 / 640 MB; a list alone 0.6 / 1.2 ms by the plain search and 0.04 / 0.06 laid out, 128 lists in one
// request 5.1 / 8.4 ms and 0.4 / 0.5.  (A layout on one thread within whatever request came first: that one waited
// 0.4 / 2.9 s.)
#pragma once

#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <memory>
#include <new>
#include <thread>
#include <vector>

namespace cbd {

class WordIndex {
 public:
  // The arrays are the graph's own and outlive the index.
  WordIndex(int32_t S, const int32_t *row, const int32_t *dst, const int32_t *olabel)
      : S_(S), row_(row), dst_(dst), olabel_(olabel) {
    const int32_t A = row[S];
    int32_t max_word = 0;
    for (int32_t a = 0; a < A; ++a) max_word = std::max(max_word, olabel[a]);
    first_.assign((size_t)max_word + 2, 0);
    for (int32_t a = 0; a < A; ++a)
      if (olabel[a] != 0) first_[(size_t)olabel[a] + 1]++;
    for (size_t w = 1; w < first_.size(); ++w) first_[w] += first_[w - 1];
    runs_.resize((size_t)first_.back());
    std::vector<int32_t> fill(first_.begin(), first_.end() - 1);
    for (int32_t s = 0; s < S; ++s)
      for (int32_t a = row[s]; a < row[s + 1]; ++a)
        if (olabel[a] != 0) runs_[(size_t)fill[(size_t)olabel[a]]++] = WordArc{a, (uint32_t)s};
  }

  // One list after another, each on some thread: out[i] receives the arcs of list i (sorted, no repeats).
  // Sequence k is words[seq_offsets[k] .. seq_offsets[k+1]); list i has sequences [list_offsets[i], list_offsets[i+1]).
  void lists(const int32_t *words, const int32_t *seq_offsets, const int32_t *list_offsets, int32_t n_lists,
             std::vector<std::vector<int32_t>> &out) {
    out.resize((size_t)n_lists);
    for (auto &o : out) o.clear();
    std::vector<int32_t> at(list_offsets, list_offsets + n_lists);   // each list's next sequence; -1: the list is made
    std::atomic<int32_t> made{0};
    std::atomic<bool> failed{false};
    while (made.load() < n_lists) {
      if (due()) lay_out();   // (lists that were begun go on from where they are)
      std::atomic<int32_t> next{0};
      share(threads(n_lists), [&](int) {
        try {
          Search s;
          for (int32_t i; !failed.load() && !due() && (i = next.fetch_add(1)) < n_lists;) {
            int32_t &k = at[(size_t)i];
            if (k < 0) continue;
            std::vector<int32_t> &o = out[(size_t)i];
            for (; k < list_offsets[i + 1] && !due(); ++k) {
              sequence(words + seq_offsets[k], seq_offsets[k + 1] - seq_offsets[k], s, o);
              if (s.met > 0) met_ += s.met;
              s.met = 0;
            }
            if (k < list_offsets[i + 1]) break;
            std::sort(o.begin(), o.end());
            o.erase(std::unique(o.begin(), o.end()), o.end());
            k = -1;
            ++made;
          }
        } catch (...) {
          failed.store(true);   // (out of memory: reported by the caller's thread)
        }
      });
      if (failed.load()) throw std::bad_alloc();
    }
  }

  // Host threads that a request of n lists is shared over (a thread costs about as much as half a list to start).
  static int threads(int32_t n) {
    return std::max(1, std::min({(int)n / 4, 16, (int)std::thread::hardware_concurrency()}));
  }

  bool laid_out() const { return rec_ != nullptr; }

 private:
  // States (records) seen in the current step: open addressing, emptied by moving the stamp on.
  struct Seen {
    struct Slot { uint32_t key, stamp; };
    std::vector<Slot> slot = std::vector<Slot>(2048, Slot{0, 0});
    uint32_t stamp = 0, n = 0;
    void clear() {
      n = 0;
      if (++stamp == 0) { std::fill(slot.begin(), slot.end(), Slot{0, 0}); stamp = 1; }
    }
    bool insert(uint32_t key) {   // false: was there
      const uint32_t mask = (uint32_t)slot.size() - 1;
      uint32_t h = (key * 2654435761u) >> 7 & mask;
      for (; slot[h].stamp == stamp; h = (h + 1) & mask)
        if (slot[h].key == key) return false;
      slot[h] = Slot{key, stamp};
      if (++n * 2 > mask) grow();
      return true;
    }
    void grow() {
      std::vector<Slot> old(slot.size() * 4, Slot{0, 0});
      old.swap(slot);
      const uint32_t mask = (uint32_t)slot.size() - 1;
      for (const Slot &o : old) {
        if (o.stamp != stamp) continue;
        uint32_t h = (o.key * 2654435761u) >> 7 & mask;
        while (slot[h].stamp == stamp) h = (h + 1) & mask;
        slot[h] = o;
      }
    }
  };
  struct Search {
    Seen seen;
    std::vector<uint32_t> reached, next, queue;
    int64_t met = 0;   // states that plain searches met
  };

  // Runs work(0) .. work(n - 1) on n threads, or all of them on fewer.  The work throws nothing.
  template <typename Work> static void share(int n, const Work &work) {
    std::vector<std::thread> pool;
    pool.reserve((size_t)n);   // (before the first of them runs: nothing is thrown past a running thread)
    int t = 1;
    for (; t < n; ++t) {
      try {
        pool.emplace_back(work, t);
      } catch (...) {
        break;   // (no more threads or no memory for one: fewer do it)
      }
    }
    work(0);
    for (; t < n; ++t) work(t);
    for (auto &p : pool) p.join();
  }

  // A state's record (32-bit words, padded to an even number): arcs without label, arcs with one; (record it leads to,
  // that state's signature) per arc of the former; (label, arc, record of the destination) per arc of the latter.  Where
  // it starts, in pairs of words: 1 + 1.5 per arc, rounded up, and what rounding leaves over.
  uint64_t place(int32_t s) const { return 3 * ((uint64_t)row_[s] + (uint64_t)s) / 2; }

  // Plain searches have met so many states that the layout pays.
  bool due() const { return !rec_ && met_.load() > S_ / 2; }

  // Lays the graph out for the searches (top of the file).  Where there is no memory for it, or more records than can be
  // counted, the plain search goes on.
  void lay_out() {
    try {
      if (place(S_) > 0xFFFFFFFFull) { met_ = INT64_MIN; return; }
      const std::vector<uint64_t> sig = signatures();
      std::unique_ptr<uint32_t[]> rec(new uint32_t[(size_t)place(S_) * 2]);
      const int n = layout_threads();
      share(n, [&](int t) {
        for (int32_t s = part(t, n), end = part(t + 1, n); s < end; ++s) {
          uint32_t *r = rec.get() + (size_t)place(s) * 2;
          uint32_t n_u = 0, n_l = 0;
          for (int32_t a = row_[s]; a < row_[s + 1]; ++a)
            if (olabel_[a] == 0) {
              uint32_t *e = r + 2 + 3 * n_u++;
              const uint64_t g = sig[(size_t)dst_[a]];
              e[0] = (uint32_t)place(dst_[a]); e[1] = (uint32_t)g; e[2] = (uint32_t)(g >> 32);
            }
          for (int32_t a = row_[s]; a < row_[s + 1]; ++a)
            if (olabel_[a] != 0) {
              uint32_t *e = r + 2 + 3 * n_u + 3 * n_l++;
              e[0] = (uint32_t)olabel_[a]; e[1] = (uint32_t)a; e[2] = (uint32_t)place(dst_[a]);
            }
          r[0] = n_u; r[1] = n_l;
        }
      });
      share(n, [&](int t) {
        const size_t m = runs_.size();
        for (size_t k = m * (size_t)t / (size_t)n, end = m * (size_t)(t + 1) / (size_t)n; k < end; ++k)
          runs_[k].from = (uint32_t)place((int32_t)runs_[k].from);
      });
      rec_ = std::move(rec);
    } catch (const std::bad_alloc &) {
      met_ = 0;   // (tried again after as many more)
    }
  }
  int layout_threads() const { return std::max(1, std::min({S_ >> 15, 16, (int)std::thread::hardware_concurrency()})); }
  int32_t part(int t, int n) const { return (int32_t)((int64_t)S_ * t / n); }

  static uint32_t word_bit(uint32_t w) { return (w * 2654435761u) >> 26; }

  // Per state the bits of all words that it, or a state it leads to through arcs without label, can output.
  // Sweeps over all states on several threads, each state taking over what its neighbours have gathered so far, until a
  // sweep changes nothing: a handful where words lie a few arcs apart or almost every state leads to almost all others.
  // Where they don't end soon (long chains without words), one pass over the components does it.
  std::vector<uint64_t> signatures() const {
    std::vector<uint64_t> sig((size_t)S_, 0);
    const int n = layout_threads();
    share(n, [&](int t) {
      for (int32_t s = part(t, n), end = part(t + 1, n); s < end; ++s)
        for (int32_t a = row_[s]; a < row_[s + 1]; ++a)
          if (olabel_[a] != 0) sig[(size_t)s] |= 1ull << word_bit((uint32_t)olabel_[a]);
    });
    for (int sweep = 0; sweep < kSweeps; ++sweep) {
      std::atomic<bool> changed{false};
      share(n, [&](int t) {
        const int32_t b = part(t, n), e = part(t + 1, n);
        bool mine = false;
        for (int32_t i = 0; i < e - b; ++i) {
          const int32_t s = sweep & 1 ? b + i : e - 1 - i;   // (downwards first: arcs mostly lead up in a sorted graph)
          uint64_t g = __atomic_load_n(&sig[(size_t)s], __ATOMIC_RELAXED);
          if (g == ~0ull) continue;
          const uint64_t before = g;
          for (int32_t a = row_[s]; a < row_[s + 1]; ++a)
            if (olabel_[a] == 0) g |= __atomic_load_n(&sig[(size_t)dst_[a]], __ATOMIC_RELAXED);
          if (g != before) { __atomic_store_n(&sig[(size_t)s], g, __ATOMIC_RELAXED); mine = true; }
        }
        if (mine) changed.store(true);
      });
      if (!changed.load()) return sig;
    }
    return signatures_of_components(S_, row_, dst_, olabel_);
  }
  static constexpr int kSweeps = 24;

  // The same, exactly once per arc, on one thread.  States on a common cycle share theirs: one pass over the strongly
  // connected components, each finished after those it leads to.
  static std::vector<uint64_t> signatures_of_components(int32_t S, const int32_t *row, const int32_t *dst, const int32_t *olabel) {
    std::vector<uint64_t> sig((size_t)S, 0);
    std::vector<int32_t> order((size_t)S, 0), low((size_t)S, 0), open;   // order: 0 = not met, -1 = finished
    struct Frame { int32_t s, next; };
    std::vector<Frame> path;
    int32_t n = 0;
    for (int32_t root = 0; root < S; ++root) {
      if (order[(size_t)root] != 0) continue;
      path.push_back({root, row[root]});
      while (!path.empty()) {
        const int32_t s = path.back().s;
        int32_t a = path.back().next;
        if (a == row[s]) {
          if (order[(size_t)s] == 0) { order[(size_t)s] = low[(size_t)s] = ++n; open.push_back(s); }
        } else if (olabel[a - 1] == 0) {   // (back from the arc before, or seen to be finished then)
          const int32_t t = dst[a - 1];
          if (order[(size_t)t] > 0) low[(size_t)s] = std::min(low[(size_t)s], low[(size_t)t]);
          sig[(size_t)s] |= sig[(size_t)t];
        }
        if (a < row[s + 1]) {
          path.back().next = a + 1;
          if (olabel[a] != 0) sig[(size_t)s] |= 1ull << word_bit((uint32_t)olabel[a]);
          else if (order[(size_t)dst[a]] == 0) path.push_back({dst[a], row[dst[a]]});
          continue;
        }
        if (low[(size_t)s] == order[(size_t)s]) {   // s is the first of its component that was met
          uint64_t all = 0;
          size_t k = open.size();
          do all |= sig[(size_t)open[--k]]; while (open[k] != s);
          for (size_t i = k; i < open.size(); ++i) { sig[(size_t)open[i]] = all; order[(size_t)open[i]] = -1; }
          open.resize(k);
        }
        path.pop_back();
      }
    }
    return sig;
  }

  const uint32_t *record(uint32_t at) const { return rec_.get() + (size_t)at * 2; }
  static const uint32_t *labels(const uint32_t *r) { return r + 2 + 3 * (size_t)r[0]; }
  void prefetch(uint32_t at) const {
    const uint32_t *r = record(at);
    __builtin_prefetch(r);
    __builtin_prefetch(r + 15);   // (a record of three arcs is 48 bytes and may straddle a line)
  }

  // Algorithm 1 for one word sequence; arcs are appended to `out` (duplicates possible).
  void sequence(const int32_t *words, int32_t k, Search &s, std::vector<int32_t> &out) const {
    if (k <= 0) return;
    const int32_t w1 = words[0];
    if (w1 <= 0 || (size_t)w1 + 1 >= first_.size()) return;   // (no such word: nothing is reached from it)
    const size_t b = (size_t)first_[(size_t)w1], e = (size_t)first_[(size_t)w1 + 1];
    if (k == 1) {   // every arc with that label: the sequence may start anywhere (Sec. 4.1)
      for (size_t i = b; i < e; ++i) out.push_back(runs_[i].arc);
      return;
    }
    // (a 0 stands for the arcs without label: neither signatures nor records tell which arcs those are)
    if (!rec_ || std::find(words + 1, words + k, 0) != words + k) {
      sequence_plain(words, k, s, out);
      return;
    }
    // states that output w_1 (a state's arcs lie together)
    s.reached.clear();
    for (size_t i = b; i < e; ++i)
      if (s.reached.empty() || s.reached.back() != runs_[i].from) s.reached.push_back(runs_[i].from);
    for (int32_t t = 1; t < k; ++t) {
      const uint32_t w_prev = (uint32_t)words[t - 1], w_next = (uint32_t)words[t];
      // leave each state through the arcs that output the previous word, then follow arcs without output label;
      // states on the way that can output the next word are where the sequence continues.  (What one state's search
      // has seen need not be searched again from another: the result is a union.)
      s.queue.clear();
      const size_t n = s.reached.size();
      for (size_t i = 0; i < std::min<size_t>(n, 8); ++i) prefetch(s.reached[i]);
      for (size_t i = 0; i < n; ++i) {
        if (i + 8 < n) prefetch(s.reached[i + 8]);
        const uint32_t *r = record(s.reached[i]);
        for (const uint32_t *l = labels(r), *end = l + 3 * (size_t)r[1]; l != end; l += 3) {
          if (l[0] != w_prev) continue;
          out.push_back((int32_t)l[1]);
          prefetch(l[2]);
          s.queue.push_back(l[2]);
        }
      }
      s.next.clear();
      s.seen.clear();
      const uint32_t word = word_bit(w_next) >> 5, bit = 1u << (word_bit(w_next) & 31u);
      for (size_t head = 0; head < s.queue.size(); ++head) {
        const uint32_t q = s.queue[head];
        if (!s.seen.insert(q)) continue;
        const uint32_t *r = record(q);
        for (const uint32_t *u = r + 2, *end = labels(r); u != end; u += 3) {
          if (!(u[1 + word] & bit)) continue;   // nothing behind it outputs the word
          prefetch(u[0]);
          s.queue.push_back(u[0]);
        }
        for (const uint32_t *l = labels(r), *end = l + 3 * (size_t)r[1]; l != end; l += 3)
          if (l[0] == w_next) { s.next.push_back(q); break; }
      }
      s.reached.swap(s.next);
    }
    const uint32_t w_last = (uint32_t)words[k - 1];
    for (uint32_t q : s.reached) {
      const uint32_t *r = record(q);
      for (const uint32_t *l = labels(r), *end = l + 3 * (size_t)r[1]; l != end; l += 3)
        if (l[0] == w_last) out.push_back((int32_t)l[1]);
    }
  }

  // The same over the graph's own arrays, for two words or more; a word 0 after the first is followed like any other.
  void sequence_plain(const int32_t *words, int32_t k, Search &s, std::vector<int32_t> &out) const {
    auto outputs = [&](uint32_t q, int32_t w) {
      return std::find(olabel_ + row_[q], olabel_ + row_[q + 1], w) != olabel_ + row_[q + 1];
    };
    s.reached.clear();
    for (size_t i = (size_t)first_[(size_t)words[0]], e = (size_t)first_[(size_t)words[0] + 1]; i < e; ++i) {
      const uint32_t src = rec_ ? (uint32_t)(std::upper_bound(row_, row_ + S_ + 1, runs_[i].arc) - row_) - 1 : runs_[i].from;
      if (s.reached.empty() || s.reached.back() != src) s.reached.push_back(src);
    }
    for (int32_t t = 0; t < k; ++t) {
      s.queue.clear();
      for (uint32_t q : s.reached)
        for (int32_t a = row_[q]; a < row_[q + 1]; ++a) {
          if (olabel_[a] != words[t]) continue;
          out.push_back(a);
          s.queue.push_back((uint32_t)dst_[a]);
        }
      if (t + 1 == k) return;
      s.next.clear();
      s.seen.clear();
      for (size_t head = 0; head < s.queue.size(); ++head) {
        const uint32_t q = s.queue[head];
        if (!s.seen.insert(q)) continue;
        s.met += 1;
        if (outputs(q, words[t + 1])) s.next.push_back(q);
        for (int32_t a = row_[q]; a < row_[q + 1]; ++a)
          if (olabel_[a] == 0) s.queue.push_back((uint32_t)dst_[a]);
      }
      s.reached.swap(s.next);
    }
  }

  int32_t S_;
  const int32_t *row_, *dst_, *olabel_;
  struct WordArc {
    int32_t arc;
    uint32_t from;   // the state it leaves (laid out: that state's record)
  };
  std::vector<int32_t> first_;       // [words + 2] start of each word's run in runs_
  std::vector<WordArc> runs_;        // by word, each word's arcs in order
  std::unique_ptr<uint32_t[]> rec_;  // the records, once they are laid out
  std::atomic<int64_t> met_{0};      // states that plain searches have met
};

}  // namespace cbd
