// The word index (csrc/word_index.hpp) on its own, without a GPU: a C interface for tests/test_word_index.py, and with
// -DNO_MEMORY a program that lets every allocation of a request fail once.
#include "../paper_2306_15685_amd/csrc/word_index.hpp"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <new>

extern "C" {

cbd::WordIndex *word_index_make(int32_t S, const int32_t *row, const int32_t *dst, const int32_t *olabel) {
  return new cbd::WordIndex(S, row, dst, olabel);
}

void word_index_free(cbd::WordIndex *w) { delete w; }

int32_t word_index_laid_out(const cbd::WordIndex *w) { return w->laid_out(); }

// Arcs of all lists back to back; returns their number (nothing is written to arcs if it is above capacity).
int64_t word_index_lists(cbd::WordIndex *w, const int32_t *words, const int32_t *seq_offsets, const int32_t *list_offsets,
                         int32_t n_lists, int32_t *arcs, int64_t capacity, int64_t *arc_offsets) {
  std::vector<std::vector<int32_t>> out;
  w->lists(words, seq_offsets, list_offsets, n_lists, out);
  arc_offsets[0] = 0;
  for (int32_t i = 0; i < n_lists; ++i) arc_offsets[i + 1] = arc_offsets[i] + (int64_t)out[(size_t)i].size();
  if (arc_offsets[n_lists] <= capacity)
    for (int32_t i = 0; i < n_lists; ++i)
      if (!out[(size_t)i].empty()) memcpy(arcs + arc_offsets[i], out[(size_t)i].data(), 4 * out[(size_t)i].size());
  return arc_offsets[n_lists];
}

}  // extern "C"

#ifdef NO_MEMORY
static std::atomic<long> g_left{-1};   // allocations until the one that fails (below 0: none does)

__attribute__((noinline)) void *operator new(size_t n) {
  if (g_left.load() >= 0 && g_left.fetch_sub(1) == 0) throw std::bad_alloc();
  if (void *p = malloc(n)) return p;
  throw std::bad_alloc();
}
__attribute__((noinline)) void operator delete(void *p) noexcept { free(p); }
__attribute__((noinline)) void operator delete(void *p, size_t) noexcept { free(p); }

// 64 lists over a ring of 1,000 states with words 1..7.  Every request either gives the lists or throws bad_alloc.
int main() {
  std::vector<int32_t> row, dst, olabel, words, seqs{0}, lists{0};
  for (int s = 0; s < 1000; ++s) {
    row.push_back((int32_t)dst.size());
    for (int k : {1, 7}) { dst.push_back((s + k) % 1000); olabel.push_back(s % 3 == 0 ? 1 + (s + k) % 7 : 0); }
  }
  row.push_back((int32_t)dst.size());
  for (int i = 0; i < 64; ++i) {
    for (int w : {1 + i % 7, 1 + i / 7 % 7}) words.push_back(w);
    seqs.push_back((int32_t)words.size());
    lists.push_back(i + 1);
  }
  long failed = 0, served = 0;
  bool laid_out = false;
  std::vector<std::vector<int32_t>> want;
  for (long k = -1;; ++k) {
    bool thrown = false;
    std::vector<std::vector<int32_t>> out;
    g_left.store(k);
    try {
      cbd::WordIndex w(1000, row.data(), dst.data(), olabel.data());
      w.lists(words.data(), seqs.data(), lists.data(), 64, out);
      laid_out = w.laid_out();
    } catch (const std::bad_alloc &) {
      thrown = true;
    }
    const bool reached = k >= 0 && g_left.exchange(-1) < 0;
    if (k < 0) {
      if (!laid_out) { printf("no layout\n"); return 1; }
      want = out;
    } else if (!thrown && out != want) { printf("allocation %ld: other lists\n", k); return 1; }
    failed += thrown;
    served += reached && !thrown;
    if (k >= 0 && !reached) break;   // (fewer allocations than that)
  }
  printf("%ld requests ended in bad_alloc, %ld were served all the same\n", failed, served);
  return failed > 0 && served > 0 ? 0 : 1;
}
#endif
