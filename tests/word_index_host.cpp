// The word index (csrc/word_index.hpp) on its own, without a GPU: a C interface for tests/test_word_index.py.
#include "../paper_2306_15685_amd/csrc/word_index.hpp"

#include <string.h>

#include <new>

extern "C" {

cbd::WordIndex *word_index_make(int32_t S, const int32_t *row, const int32_t *dst, const int32_t *olabel) {
  return new cbd::WordIndex(S, row, dst, olabel);
}

void word_index_free(cbd::WordIndex *w) { delete w; }

// Arcs of all lists back to back; returns their number (nothing is written to arcs if it is above capacity).
int64_t word_index_lists(const cbd::WordIndex *w, const int32_t *words, const int32_t *seq_offsets, const int32_t *list_offsets,
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
