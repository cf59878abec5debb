// The lean frame: the same frame as run_frame() computes (same table, same records, same counters), for frames
// whose tables fit LDS, over rows of ordinary length and closure lists stored with the graph.  What it leaves
// out is dependent waiting and per-wave bookkeeping:
//   - the emit phase reads the tokens' rows from LDS and one arc record per lane from device memory; every
//     wave posts its minimum, one barrier, and the frame's cutoff m is final before anything reaches the table
//     (so nothing is ever marked dead afterwards).  A wave holds 128 candidates in registers; what a heavy frame
//     has beyond that counts for the minimum before the barrier and is computed again after it;
//   - the epsilon closure of a state is one contiguous list stored with the graph (depth-first, parents first,
//     each record naming its parent's position).  The lists behind a wave's committed candidates are spread
//     over its lanes, one record per lane: one read for all of them, costs handed down the lists' trees level
//     by level, one table update for all.  A list is walked for every candidate that passes the cutoff, whether
//     or not it lowered its state: a walk from a value that is not the state's final one only produces
//     candidates that the walk from the final value dominates (fp32 addition is monotone), so the fixed point
//     is the one of paper Sec. 3.2's expansion;
//   - no change log shared by the workgroup and no counter atomics: every wave logs its own commits (8 bytes
//     each) and, after the second barrier, looks up which of them is its state's value ("the winner writes" the
//     token and its back-pointer record); token indices are wave-local ordinals, made dense by a prefix sum
//     over the waves' counts.
// Whatever does not fit (a tile with more than 256 arcs, a hub row, a closure without stored list, a full table
// or log) sets Shared::redo (before the first barrier) or the wave's count in Shared::wcount to more than any table holds
// (between the barriers); each is read by all waves after the barrier that follows, and the frame is then decoded again by
// run_frame(), which handles everything.
// What bounds it: the chain of dependent LDS and device-memory reads of a frame's slowest wave, with its instructions between
// them, and three barriers at which the others wait for it (256 channels: the vector unit is active 40 % of the time its
// workgroup is resident, and waves wait for an issue slot 12 % of theirs).  So a wave goes through straight-line code for the
// 64 or 128 arcs it has (one or two slots per lane), and what lanes do is kept in lane masks.  Against the same steps with a flag per lane, an owner search by running
// maximum and shuffles for the emitting arcs, and one code for one and two slots (us): one channel x 100 frames 656 -> 562,
// 32 x 333 2,120 -> 1,792, 100 x 151 1,352 -> 1,211, 256 x 500 6,028 -> 5,625, 512 x 400 7,793 -> 7,187, 2,048 x 100 9,932 ->
// 9,048.
#pragma once

namespace cbd {

// Diagnostic build only (-DCBD_PROFILE): thread 0 stamps the phases of every lean frame with the 100 MHz counter
// and the sums go out through ChanState::spare.
#ifdef CBD_PROFILE
#define CBD_STAMP(k)                                                                                     \
  do {                                                                                                   \
    if (threadIdx.x == 0) { const long long t_ = wall_clock64(); sh->prof[k] += t_ - sh->prof_last; sh->prof_last = t_; } \
  } while (0)
// why a lean frame is given back: 0 closure stage over 64 records, 1 commit log full, 2 too many tokens, 3 other
#define CBD_WHY(k) atomicAdd(&sh->prof_why[k], 1)
#else
#define CBD_STAMP(k) do {} while (0)
#define CBD_WHY(k) do {} while (0)
#endif

constexpr uint16_t kLeanDegEscape = 0xFFFF;   // t_deg: the row is too long for the lean code
constexpr int kLeanLidBits = 10;              // a wave-local token id: wave << 10 | ordinal within the wave
constexpr int kLeanLidMask = (1 << kLeanLidBits) - 1;

// One commit as its wave logged it: slot h took (some cost, arc).  from: where the arc started, a token of the
// previous frame (kLeanFromToken set: an emitting arc) or a table slot of this frame (an epsilon-input arc).
struct __attribute__((aligned(8))) LeanLog {
  uint32_t arc;
  uint16_t h;
  uint16_t from;
};
constexpr uint16_t kLeanFromToken = 0x8000;

// The tokens' rows and the commit logs live where the general code keeps its change log.
struct LeanMem {
  int32_t *t_first;    // [tok_cap] first emitting arc of each current token's state
  uint16_t *t_deg;     // [tok_cap] number of emitting arcs
  int32_t *hrow;       // [slots] the same for the states in the table, written by whoever creates the entry
  uint8_t *hed;        // [slots]  (kEdEscape: the row is too long for the lean code)
  LeanLog *clog;       // [waves][kLeanLogPerWave]
};

constexpr int kLeanLogPerWave = 256;   // commits a wave can log per frame (more: the frame goes to the general code)
constexpr int kLeanLogEntryBytes = 8;
constexpr int kLeanRedoCount = 1 << 24;   // Shared::wcount of a wave that gave the frame up

__device__ __forceinline__ LeanMem make_lean_mem(void *log_region, int tok_cap, int slots) {
  LeanMem R;
  unsigned char *b = (unsigned char *)log_region;
  R.t_first = (int32_t *)b;
  R.t_deg = (uint16_t *)(b + (size_t)tok_cap * 4);
  b += align_up((uint32_t)tok_cap * 6u, 16u);
  R.hrow = (int32_t *)b;
  R.hed = (uint8_t *)(b + (size_t)slots * 4);
  b += align_up((uint32_t)slots * 5u, 16u);
  R.clog = (LeanLog *)b;
  return R;
}

// a register of which no one reads what it holds
__device__ __forceinline__ uint32_t any_value() { uint32_t x; asm volatile("" : "=v"(x)); return x; }

// table slot of a state: home slot first, then linear probing (same function as table_min)
__device__ __forceinline__ uint32_t lean_home(uint32_t state, uint32_t slots) {
  return __umulhi(state * 2654435761u, slots);
}

// Finds or creates the slot of `state` after a collision at its home slot.  Returns false if the table is full.
__device__ __forceinline__ bool lean_probe(const Mem<true> &M, uint32_t state, uint32_t &h, uint32_t &k) {
  uint32_t probe = 1;
  do {
    h = h + 1 == M.slots ? 0 : h + 1;
    k = atomicCAS(&M.hkey[h], kEmptyKey, state);
  } while (k != kEmptyKey && k != state && ++probe < M.slots);
  return k == kEmptyKey || k == state;
}

// A tile: up to 64 tokens of the previous frame, one per lane, and the list of their emitting arcs.
struct LeanTile {
  float cost;     // this lane's token
  int rel;        // first arc of its row minus the row's position in the arc list
  int base;       // index of lane 0's token
  int total;      // arcs in the list (uniform)
};

// What the lanes of an arc list need to know about the token that owns their position, by the tokens' ranks among those
// with arcs.  In the emit phase it lies where the wave's commit log is in the rest of the frame.
struct __attribute__((aligned(16))) LeanOwner {
  int rel;
  float cost;
  uint32_t from;   // LeanLog::from in the upper half
  uint32_t unused;
};
static_assert(64 * sizeof(LeanOwner) <= kLeanLogPerWave * sizeof(LeanLog), "a tile's owners fit the wave's log");

// Loads the tile of tokens base + lane, below tile_end (base < tile_end), prunes (step 1), and writes the heads of its arc list
// into omap (the owner of a list position is the last head at or before it) and, if kOwners, the owners by rank.
template <bool kOwners>
__device__ __forceinline__ LeanTile lean_load_tile(const AdvanceParams &p, const Mem<true> &M, const LeanMem &R,
                                                   Shared *sh, uint8_t *omap, LeanOwner *owners, int base, int tile_end,
                                                   int lane, float best, int cut, float inv, int &n_active) {
  LeanTile T;
  T.base = base;
  // (lanes beyond the last token look at that one: no branch, so what is asked of it stays in lane masks)
  const int i = min(base + lane, tile_end - 1);
  T.cost = M.t_cost[i];
  const int first = R.t_first[i];
  int deg = (int)R.t_deg[i];
  const float r = T.cost - best;
  uint64_t alive = lanes_with(base + lane < tile_end) & lanes_with(!(r > p.beam)) & lanes_with(T.cost < __builtin_inff());
  if (cut < 255) {   // uniform
    int bin = (int)floorf(r * inv);
    bin = bin > 255 ? 255 : bin;
    alive &= lanes_with(bin <= cut);
  }
  deg = lane_in(alive) ? deg : 0;
  const int incl = wave_incl_scan(deg);
  const int pos = incl - deg;
  T.total = __builtin_amdgcn_readlane(incl, 63);
  T.rel = first - pos;
  n_active += __popcll(alive);
  if (T.total > kOwnerMap) {   // uniform (a row too long for the count field, kLeanDegEscape, is one such)
    if (lane == 0) { sh->redo = 1; CBD_WHY(3); }
    T.total = 0;
    return T;
  }
  ((uint32_t *)omap)[lane] = 0;
  const uint64_t heads = lanes_with(deg > 0);
  if (lane_in(heads)) {
    omap[pos] = (uint8_t)(lane + 1);
    if (kOwners) {
      LeanOwner o;
      o.rel = T.rel; o.cost = T.cost; o.from = (uint32_t)(i | kLeanFromToken) << 16; o.unused = 0;
      owners[rank_in(heads, 0)] = o;
    }
  }
  return T;
}

// Emitting candidates, one per lane and slot: list positions jb + lane and (second slot) jb + 64 + lane.
struct LeanEmit {
  float cand[2];
  int arc[2];
  ArcRec rec[2];
  uint32_t from[2];   // LeanLog::from in the upper half
  uint64_t act[2];    // the lanes that hold one (uniform)
};

// Which lanes' arcs a[] are listed.  Every lane asks, those beyond the list of candidates too: they hold its last arc once
// more, and the costs made of it enter the frame's minimum.  A wave waits for LDS once per step for both slots, and the number
// of steps depends on the list's length alone, so a step is a read, a compare and a select per arc, with no lanes dropping out.
// (One arc after the other with a search that ends per lane: a wave waited twice per step and for the arc records before its
// second test.  32 channels x 333 frames behind the plain search 2.414 -> 2.393 ms, 8 channels x 1,000 frames 8.59 -> 8.50,
// where runs differ by 0.3 %; 2,048 channels with 1,000-arc lists behind the filter within the spread.)
template <int kSlots>
__device__ __forceinline__ void lean_listed(const Ctx &cx, const int (&a)[2], uint64_t (&in)[2]) {
  uint64_t any = 0;
#pragma unroll
  for (int q = 0; q < kSlots; ++q) in[q] = 0;
  if (cx.n == 0) return;
  if (cx.use_bitmap) {
    uint32_t w[kSlots], m[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      const uint32_t h = bloom_hash(a[q]);
      m[q] = bloom_mask(h);
      w[q] = cx.bitmap[bloom_word(h)];
    }
#pragma unroll
    for (int q = 0; q < kSlots; ++q) { in[q] = lanes_with((w[q] & m[q]) == m[q]); any |= in[q]; }
    if (any == 0) return;
  } else {
#pragma unroll
    for (int q = 0; q < kSlots; ++q) in[q] = ~0ull;
  }
  if (!cx.in_lds) {
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      bool is = false;
      if (lane_in(in[q])) is = sorted_contains(cx.g_list, cx.n, a[q]);
      in[q] = lanes_with(is);
    }
    return;
  }
  // the last entry <= a lies in [b, b + len), if there is one
  int b[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) b[q] = 0;
  for (int len = __builtin_amdgcn_readfirstlane(cx.n); len > 1;) {
    const int half = len >> 1;
    int v[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) v[q] = cx.lds_list[b[q] + half];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) b[q] = v[q] <= a[q] ? b[q] + half : b[q];
    len -= half;
  }
  int v[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) v[q] = cx.lds_list[b[q]];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) in[q] &= lanes_with(v[q] == a[q]);
}

// Costs of the candidates whose arcs and tokens' costs are known.  The records of both slots are asked for before either is
// used, and so are their scores: every lane asks, those beyond the list for what the last arc needs, so that no branch makes
// the first slot's score wait before the second's is asked for, as a condition per lane did.
template <int kSlots, bool kRowFromLds>
__device__ __forceinline__ uint32_t lean_costs(const AdvanceParams &p, const Ctx &cx, const Rows &Lrow, const float *own_cost,
                                               LeanEmit &E) {
#pragma unroll
  for (int q = 0; q < kSlots; ++q) E.rec[q] = p.arcs[E.arc[q]];
  // the bias test needs the arcs' numbers only: it runs while the records are on their way
  uint64_t listed[2];
  lean_listed<kSlots>(cx, E.arc, listed);
  float ll[kSlots];
  if (kRowFromLds && Lrow.staged) {
#pragma unroll
    for (int q = 0; q < kSlots; ++q) ll[q] = Lrow.lds[(E.rec[q].meta & 0xFFFFu) - 1u];
  } else {
    const char *row = (const char *)(Lrow.glob - 1);
#pragma unroll
    for (int q = 0; q < kSlots; ++q) ll[q] = *(const float *)(row + ((E.rec[q].meta & 0xFFFFu) << 2));
  }
  uint32_t lmin = 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    float w = E.rec[q].weight;
    w = lane_in(listed[q]) ? w + cx.offset : w;   // Sec. 4.1: boosted weight = weight + discount
    E.cand[q] = (own_cost[q] + w) - ll[q];
    lmin = umin32(lmin, f2ord(E.cand[q]));   // (lanes beyond the list have the last arc's candidate once more, offset and all)
  }
  return lmin;
}

// Emit phase: candidates of list positions [jb, jb + 64 kSlots) of tile T (T.total > jb).  heads: number of rows that begin
// before jb.  Returns the minimum (orderable bits) over the candidates computed.
template <int kSlots>
__device__ __forceinline__ uint32_t lean_candidates(const AdvanceParams &p, const Ctx &cx, const Rows &Lrow,
                                                    const uint8_t *omap, const LeanOwner *owners, int jb, int heads, int lane,
                                                    const LeanTile &T, LeanEmit &E) {
  uint32_t head[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) head[q] = omap[jb + q * 64 + lane];
  LeanOwner o[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const uint64_t hm = lanes_with(head[q] != 0);
    o[q] = owners[rank_in(hm >> 1, heads + (int)(hm & 1) - 1)];   // the last head at or before this lane
    heads += __popcll(hm);
  }
  float own_cost[kSlots];
  E.act[0] = E.act[1] = 0;
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int j = jb + q * 64 + lane;
    E.act[q] = lanes_with(j < T.total);
    E.arc[q] = o[q].rel + min(j, T.total - 1);
    own_cost[q] = o[q].cost;
    E.from[q] = o[q].from;
  }
  return lean_costs<kSlots, true>(p, cx, Lrow, own_cost, E);
}
// The number of rows of the tile in omap that begin before position jb (a multiple of 64; uniform).
__device__ __forceinline__ int lean_heads_before(const uint8_t *omap, int jb, int lane) {
  int n = 0;
  for (int b = 0; b < jb; b += 64) n += __popcll(lanes_with(omap[b + lane] != 0));
  return n;
}

// The same again after the first barrier (the commit log is in use by then: a position's owner is found by a running maximum
// over the heads, and what it has comes from its lane), both slots.
__device__ __forceinline__ void lean_candidates_again(const AdvanceParams &p, const Ctx &cx, const Rows &Lrow, const uint8_t *omap,
                                                      int jb, int lane, const LeanTile &T, LeanEmit &E) {
  int carry = 0;   // owner + 1 of the last position before jb
  for (int b = 0; b < jb; b += 64) {   // (uniform)
    const int t = __builtin_amdgcn_readlane(wave_incl_scan_max((int)omap[b + lane]), 63);
    carry = t > carry ? t : carry;
  }
  float own_cost[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int j = jb + q * 64 + lane;
    int own1 = wave_incl_scan_max((int)omap[j]);
    own1 = own1 > carry ? own1 : carry;
    carry = __builtin_amdgcn_readlane(own1, 63);
    const int owner = own1 - 1;
    E.act[q] = lanes_with(j < T.total);
    E.arc[q] = from_lane(T.rel, owner) + min(j, T.total - 1);
    own_cost[q] = from_lane(T.cost, owner);
    E.from[q] = (uint32_t)((T.base + owner) | kLeanFromToken) << 16;
  }
  lean_costs<2, false>(p, cx, Lrow, own_cost, E);
}

// Per-wave running state of the commit phase (all uniform).
struct LeanWave {
  int claimed;       // wave << kLeanLidBits | states this wave created so far
  int n_clog;        // commits it logged
  int n_cand, n_eps;
  int max_depth;
  bool redo;         // it met something this code cannot take
};

// Copies a log-likelihood row from device memory into LDS without passing through registers: every wave asks for
// 1 KB pieces (16 bytes per lane) that the memory pipeline writes straight into LDS.  The caller waits for its own
// requests (vmcnt) and passes a barrier before anyone reads the row.  Rows whose size or address is not a
// multiple of 16 bytes go 4 bytes per lane.
template <int kBlock>
__device__ __forceinline__ void stage_row_async(float *lds_row, const float *row, int num_pdfs, int wave, int lane) {
  constexpr int NW = kBlock / 64;
  typedef const __attribute__((address_space(1))) void *gptr;
  typedef __attribute__((address_space(3))) void *lptr;
  if ((num_pdfs & 3) == 0 && (((unsigned long long)row) & 15ull) == 0) {
    for (int base = wave * 256; base < num_pdfs; base += NW * 256) {   // uniform
      const int i = base + lane * 4;
      if (i < num_pdfs)
        __builtin_amdgcn_global_load_lds((gptr)(row + i), (lptr)(lds_row + base), 16, 0, 0);
    }
  } else {
    for (int base = wave * 64; base < num_pdfs; base += NW * 64) {
      const int i = base + lane;
      if (i < num_pdfs)
        __builtin_amdgcn_global_load_lds((gptr)(row + i), (lptr)(lds_row + base), 4, 0, 0);
    }
  }
}

// Asks for the table slot of `state` for lanes in ok: h, and k = what the slot held before (kEmptyKey: this
// lane created the entry).  Other lanes' h and k mean nothing.
__device__ __forceinline__ void lean_slot(const Mem<true> &M, uint64_t ok, uint32_t state, uint32_t &h, uint32_t &k) {
  h = lean_home(state, M.slots);
  k = any_value();
  if (lane_in(ok)) k = atomicCAS(&M.hkey[h], kEmptyKey, state);
}
// After a collision at the home slot: walks on.  A table without room sets W.redo.
__device__ __forceinline__ void lean_slot_collisions(const Mem<true> &M, Shared *sh, uint64_t &ok, uint32_t state,
                                                     uint32_t &h, uint32_t &k, LeanWave &W) {
  const uint64_t collided = ok & lanes_with(k != kEmptyKey) & lanes_with(k != state);
  if (collided != 0) {   // rare
    bool full = false;
    if (lane_in(collided)) full = !lean_probe(M, state, h, k);
    const uint64_t f = lanes_with(full);
    if (f != 0) { ok &= ~f; W.redo = true; if (lane_in(1ull)) CBD_WHY(3); }
  }
}

// E[state] = min key for lanes in ok (slot h, previous holder k from lean_slot), the token's wave-local id and the state's
// row if the lane created the entry, and the log entry for the look-up after the barrier.
__device__ __forceinline__ void lean_min_and_log(const Mem<true> &M, const LeanMem &R, Shared *sh, uint64_t ok, uint32_t h,
                                                 uint32_t k, uint32_t cost_ord, uint32_t arc, const ArcRec &rec, uint32_t from,
                                                 LeanLog *clog, LeanWave &W) {
  const int n_ok = __popcll(ok);
  if (W.n_clog + n_ok > kLeanLogPerWave) {   // uniform
    W.redo = true;
    if (lane_in(1ull)) CBD_WHY(1);
    return;
  }
  const uint64_t claimed = ok & lanes_with(k == kEmptyKey);
  if (lane_in(ok)) {
    atomicMin((unsigned long long *)&M.hval[h], ((unsigned long long)cost_ord << 32) | arc);
    *(uint2 *)&clog[rank_in(ok, W.n_clog)] = make_uint2(arc, h | from);   // LeanLog
  }
  if (lane_in(claimed)) {
    // this lane created the state's entry: it names the token (wave-local id, made dense after the barrier) and
    // files the state's row, which the next frame expands
    M.hidx[h] = (uint16_t)rank_in(claimed, W.claimed);
    R.hrow[h] = rec.row;
    R.hed[h] = (uint8_t)meta_ed(rec.meta);
  }
  W.claimed += __popcll(claimed);
  W.n_clog += n_ok;
}

// Commits the emitting candidates in E (the cutoff m is final) and walks the closure lists behind them.  The
// steps are ordered so that waits overlap: the table slots are asked for, then the closure records, and only
// then are the slots looked at.
// The closure stage: a lane may bring up to two lists, the stored closure lists of the states it is committing candidates
// to.  The records of all the wave's lists are spread over the lanes, one record per lane, and asked for with one read; then
// costs follow the lists' trees level by level (a record names its parent's position), a dropped record drops its subtree,
// and everything that passes is committed in one go.
template <int kSlots>
__device__ __forceinline__ void lean_commit(const AdvanceParams &p, const Mem<true> &M, const LeanMem &R, Shared *sh,
                                            const Ctx &cx, float m, int lane, LeanWave &W, uint8_t *cmap, LeanLog *clog,
                                            const LeanEmit &E, int par) {
  const float beam = p.beam;
  uint64_t pass[kSlots], any = 0;
  uint32_t h[kSlots], k[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) { pass[q] = E.act[q] & lanes_with(!(E.cand[q] - m > beam)); any |= pass[q]; }
  if (any == 0) return;   // uniform
#pragma unroll
  for (int q = 0; q < kSlots; ++q) lean_slot(M, pass[q], (uint32_t)E.rec[q].dst, h[q], k[q]);
  // the closure lists of the destinations
  int len[kSlots], mine = 0;
#pragma unroll
  for (int q = 0; q < kSlots; ++q) { len[q] = lane_in(pass[q]) ? (int)meta_cl(E.rec[q].meta) : 0; mine += len[q]; }
  const int incl = wave_incl_scan(mine);
  int total = __builtin_amdgcn_readlane(incl, 63);
  if (total >= (int)kClEscape) {   // (rare: no stored list, or more than a lane per record; the general code takes the frame)
    uint64_t esc = 0;
#pragma unroll
    for (int q = 0; q < kSlots; ++q) esc |= lanes_with(len[q] == (int)kClEscape);
    if (esc != 0 || total > 64) {
      W.redo = true;
      if (lane_in(1ull)) CBD_WHY(esc != 0 ? 3 : 0);
      total = 0;
    }
  }
  auto commit_emitting = [&]() {
#pragma unroll
    for (int q = 0; q < kSlots; ++q) lean_slot_collisions(M, sh, pass[q], (uint32_t)E.rec[q].dst, h[q], k[q], W);
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      W.n_cand += __popcll(pass[q]);
      lean_min_and_log(M, R, sh, pass[q], h[q], k[q], f2ord(E.cand[q]), (uint32_t)E.arc[q], E.rec[q], E.from[q], clog, W);
    }
    CBD_STAMP(7);   // (diagnostic: emitting candidates committed)
  };
  // A wave with closure lists has the longest way to the frame's second barrier, and the fifteen others wait for it there:
  // it goes first where waves of a SIMD could both issue, until it is past its last commit (run_frame_lean puts it back).
  // One channel x 100 frames 559 -> 556 us, 32 x 240 frames 1,791 -> 1,779, 256 streams x 500 frames 5,604 -> 5,576
  // (the runs of one side differ by 0.1 to 0.2 %); all waves with two slots first as well gives nothing more.
  if (total != 0) __builtin_amdgcn_s_setprio(2);
  if (total == 0) {   // uniform
    CBD_STAMP(6);
    commit_emitting();
    CBD_STAMP(8);
    return;
  }
  // which list a record belongs to: the last head at or before its position.  A head names its lane and which of the lane's
  // lists it is (2 lane + which + 1: later positions have larger names)
  int start[kSlots];
  start[0] = incl - mine;
  if (lane_in(0xFFFFull)) ((uint32_t *)cmap)[lane] = 0;
  if (len[0] > 0) cmap[start[0]] = (uint8_t)(kSlots * lane + 1);
  if (kSlots == 2) {
    start[1] = start[0] + len[0];
    if (len[1] > 0) cmap[start[1]] = (uint8_t)(2 * lane + 2);
  }
  const int name = wave_incl_scan_max((int)cmap[lane]) - 1;   // (position 0 is a head)
  const int owner = kSlots == 2 ? name >> 1 : name;
  const bool second = kSlots == 2 && (name & 1) != 0;
  // what the list's lane knows: where its records lie and begin in the stage, and the cost they hang from
  int at[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q)
    at[q] = E.rec[q].row + (int)meta_ed(E.rec[q].meta) + (int)meta_xd(E.rec[q].meta) - start[q];
  int rpos = from_lane(at[0], owner), o_start = from_lane(kSlots == 2 ? start[0] | (start[1] << 8) : start[0], owner);
  float o_root = from_lane(E.cand[0], owner);
  if (kSlots == 2) {
    const int rpos1 = from_lane(at[1], owner);
    const float root1 = from_lane(E.cand[1], owner);
    rpos = second ? rpos1 : rpos;
    o_root = second ? root1 : o_root;
    o_start = second ? o_start >> 8 : o_start & 0xFF;
  }
  const uint64_t act = total == 64 ? ~0ull : (1ull << total) - 1ull;
  // (lanes beyond the lists ask for the last record once more)
  rpos += min(lane, total - 1);
  const ArcRec rec = p.arcs[rpos];
  int can[2];
  can[0] = can[1] = p.canon[rpos];
  CBD_STAMP(6);   // (diagnostic: cutoff, slot requests, closure records requested)
  // now the emitting candidates' slots
  commit_emitting();

  const int o_hh = from_lane((int)(kSlots == 2 ? h[0] | (h[1] << 16) : h[0]), owner);
  W.n_eps += total;
  const int depth = (int)(rec.meta & 0xFu);   // 1..kClosureMaxDepth
  const int plane = (o_start - 1 + (int)((rec.meta >> 4) & 0x3Fu)) & 63;   // the lane that holds the parent record
  uint64_t listed[2];
  lean_listed<1>(cx, can, listed);
  float w = rec.weight;
  w = lane_in(listed[0]) ? w + cx.offset : w;   // Sec. 4.1: boosted weight = weight + discount
  const uint64_t d1 = act & lanes_with(depth == 1);
  float c = o_root + w;
  uint64_t ok = d1 & lanes_with(c < __builtin_inff()) & lanes_with(!(c - m > beam));
  c = lane_in(ok) ? c : __builtin_inff();
  int d = 1;
  for (;;) {   // uniform (a record of one level has its parent in the level before)
    const uint64_t dm = act & lanes_with(depth == d + 1);
    if (dm == 0) break;
    ++d;
    const float cc = from_lane(c, plane) + w;
    const uint64_t okd = dm & lanes_with(cc < __builtin_inff()) & lanes_with(!(cc - m > beam));
    c = lane_in(okd) ? cc : c;
    ok |= okd;
  }
  W.max_depth = max(W.max_depth, d);
  if (ok == 0) { CBD_STAMP(8); return; }   // uniform
  W.n_cand += __popcll(ok);
  const uint32_t co = f2ord(c);
  if ((ok & lanes_with(co < f2ord(m))) != 0) {
    // the frame's minimum is min(m, closure candidates): only a candidate below m can move it
    const uint32_t wmin = wave_min_u32(lane_in(ok) ? co : 0xFFFFFFFFu);
    if (lane == 0) atomicMin(&sh->lean_best[par], wmin);
  }
  uint32_t ch, ck;
  lean_slot(M, ok, (uint32_t)rec.dst, ch, ck);
  lean_slot_collisions(M, sh, ok, (uint32_t)rec.dst, ch, ck, W);
  // the source state's slot: the list's state, or the parent record's (found a moment ago by its lane)
  const uint32_t ph = (uint32_t)from_lane((int)ch, plane);
  const uint32_t o_h = kSlots == 2 ? (second ? (uint32_t)o_hh >> 16 : (uint32_t)o_hh & 0xFFFFu) : (uint32_t)o_hh;
  lean_min_and_log(M, R, sh, ok, ch, ck, co, (uint32_t)can[0], rec, (lane_in(d1) ? o_h : ph) << 16, clog, W);
  CBD_STAMP(8);   // (diagnostic: closure records committed)
}

// The thread's number in the workgroup, as a value of its own at every place that asks for it: what is derived from it
// is worked out there again (an instruction or two) instead of once ahead of the frame loop.  Kept from there, such
// values are more than the registers hold and some come back from scratch memory in every frame, a wait on the way
// (256 streams x 500 frames: 9.1 instead of 7.7 memory instructions per wave and frame).
__device__ __forceinline__ int here_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// One frame by the lean code.  Returns kFrameOk, kFrameNoTokens, kFrameRecordsFull, or kFrameRedo (then nothing
// that outlives the frame has been written, but the state table holds entries and the staged log-likelihood
// row may already be the next frame's, or on its way there: the caller waits, cleans up and runs the general code).
// par: 0 and 1 in turn from frame to frame.
template <int kBlock>
__device__ __forceinline__ int run_frame_lean(const AdvanceParams &p, const Mem<true> &M, const LeanMem &R, Shared *sh,
                                              const Ctx &cx, float *Lstage, const Rows &Lrow, const float *Lnext,
                                              uint32_t *hist, uint8_t *owner_maps, uint8_t *closure_maps, int row_buf,
                                              int2 *bp, int32_t *g_tok_state, bool last_frame, int par) {
  constexpr int NW = kBlock / 64;
  static_assert(NW <= 16, "Shared::wcount holds 16 waves");
  const int tid = here_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#ifdef CBD_PROFILE
  if (tid == 0) sh->prof_last = wall_clock64();
#endif
  const bool hist_on = p.max_active > 0 && p.beam > 0.0f && p.beam < __builtin_inff();
  const float inv = 256.0f / p.beam;
  uint8_t *omap = owner_maps + wave * kOwnerMap;
  uint8_t *cmap = closure_maps + wave * 64;
  LeanLog *clog = R.clog + wave * kLeanLogPerWave;
  LeanOwner *owners = (LeanOwner *)clog;

  // ---- emit: prune (step 1), expand (step 2).  The wave's share of the tokens is taken in tiles of 64, a tile's
  // arcs 128 at a time; tile 0's first 128 come last and stay in registers.
  const int n_tok = __builtin_amdgcn_readfirstlane(sh->n_tok);
  const float best = sh->best;
  const int cut = __builtin_amdgcn_readfirstlane(sh->cut_bin);
  const int tpw = (n_tok + NW - 1) / NW;
  const int tile0 = wave * tpw;
  const int tile_end = min(tile0 + tpw, n_tok);
  int n_active = 0, n_emit = 0;
  uint32_t lmin = 0xFFFFFFFFu;
  LeanEmit E;
  LeanTile T;
  T.total = 0;
  for (int base = tile0 + ((tile_end - 1 - tile0) & ~63); base >= tile0; base -= 64) {   // (none: tile_end <= tile0)
    T = lean_load_tile<true>(p, M, R, sh, omap, owners, base, tile_end, lane, best, cut, inv, n_active);
    if (T.total == 0) continue;   // uniform
    n_emit += T.total;
    for (int jb = (T.total - 1) & ~127; jb >= 0; jb -= 128) {   // (one round but for heavy frames)
      const int heads = lean_heads_before(omap, jb, lane);
      const uint32_t l = T.total - jb > 64 ? lean_candidates<2>(p, cx, Lrow, omap, owners, jb, heads, lane, T, E)
                                           : lean_candidates<1>(p, cx, Lrow, omap, owners, jb, heads, lane, T, E);
      lmin = umin32(lmin, l);
    }
  }
  const int n_active_frame = n_active;
  if (n_emit != 0) {   // uniform
    const uint32_t wmin = wave_min_u32(lmin);
    if (lane == 0) atomicMin(&sh->m_ord, wmin);
  }
  CBD_STAMP(0);   // emit phase of wave 0
  wg_barrier<true>();
  CBD_STAMP(1);   // its wait at the first barrier

  // ---- step 3: the emission minimum fixes the frame's cutoff
  const uint32_t m_ord = sh->m_ord;
  const int redo = sh->redo;
  if (redo) return kFrameRedo;                  // (uniform: set before the barrier, or never)
  if (m_ord == 0xFFFFFFFFu) return kFrameNoTokens;
  const float m = ord2f(m_ord);

  // ---- recombination (step 2, second half) and epsilon closure (step 4): the candidates in registers first,
  // then whatever the tiles hold beyond them, computed again (the staged row may be on its way out by then: these
  // read the row in device memory)
  LeanWave W;
  W.claimed = wave << kLeanLidBits; W.n_clog = 0; W.n_cand = 0; W.n_eps = 0; W.max_depth = 0; W.redo = false;
  if (T.total > 64) lean_commit<2>(p, M, R, sh, cx, m, lane, W, cmap, clog, E, par);
  else if (T.total > 0) lean_commit<1>(p, M, R, sh, cx, m, lane, W, cmap, clog, E, par);
  for (int base = tile0; base < tile_end; base += 64) {
    if (base > tile0) T = lean_load_tile<false>(p, M, R, sh, omap, owners, base, tile_end, lane, best, cut, inv, n_active);
    for (int jb = base > tile0 ? 0 : 128; jb < T.total; jb += 128) {
      LeanEmit X;
      lean_candidates_again(p, cx, Lrow, omap, jb, lane, T, X);
      lean_commit<2>(p, M, R, sh, cx, m, lane, W, cmap, clog, X, par);
    }
  }
  __builtin_amdgcn_s_setprio(0);   // (raised in lean_commit)
  // The emit phase is long over: the next frame's row starts its way.  (Not earlier: loads return in order, and
  // the closure stages' reads would queue behind the row.)
  // A row that is not staged is touched instead, one lane per 64 bytes: the next frame's emit phase then finds it
  // in L2.  (Touching it earlier, in the emit phase, puts it in front of the closure records: 32 to 512 channels 1.3
  // to 5 % slower.)  It falls to the last waves, which have the tokens that a frame's even split leaves over, or none.
  float touched = 0.0f;
  if (Lnext) {
    const int t = here_tid(), back = kBlock - 1 - t;
    if (Lrow.staged) stage_row_async<kBlock>(Lstage, Lnext, p.num_pdfs, back >> 6, t & 63);
    else if (back * 16 < p.num_pdfs) touched = Lnext[back * 16];
  }
  if (lane == 0) {
    sh->wcount[wave] = W.redo ? kLeanRedoCount : W.claimed & kLeanLidMask;
    if (W.max_depth) atomicMax(&sh->rounds, W.max_depth);
  }
  const int base_cur = __builtin_amdgcn_readfirstlane(sh->n_rec), base_prev = __builtin_amdgcn_readfirstlane(sh->frame_base);
  CBD_STAMP(2);   // commit phase of wave 0
  wg_barrier<true>();
  CBD_STAMP(3);   // its wait at the second barrier

  // ---- step 5 and bookkeeping: the winner of each state writes the token
  // dense token indices: prefix sums over the waves' counts (every wave computes the same numbers; lane w < NW has wave w's)
  const int my_count = sh->wcount[lane & 15];
  const int count_incl = row_incl_scan(lane < NW ? my_count : 0);
  const int wbase = count_incl - my_count;
  const int n_claim = __builtin_amdgcn_readlane(count_incl, 15);
  if (n_claim > M.tok_cap) {   // (the general code decides what an overflow means; or some wave gave the frame up)
    if (tid == 0 && n_claim < kLeanRedoCount) CBD_WHY(2);
    return kFrameRedo;
  }
  if (base_cur + n_claim > p.bp_cap) return kFrameRecordsFull;
  const bool hist_need = hist_on && n_claim > p.max_active;
  const float fbest = ord2f(umin32(m_ord, sh->lean_best[par]));
  // The frame is as good as closed: everybody has read its scalars ahead of the second barrier, so one wave writes the
  // next frame's before it looks up its entries.  Only a histogram has to wait for all winners (below).  (Left to
  // whichever wave was through last, these writes and seven counters lay between it and the third barrier: 60 frames of
  // one stream 612 -> 592 us, 32 channels x 333 frames 2.36 -> 2.28 ms, 512 channels 1.5 % faster.)
  if (wave == 0 && lane == 0) {
    sh->m_ord = 0xFFFFFFFFu;
    sh->lean_best[par ^ 1] = 0xFFFFFFFFu;   // (this frame's is still being read)
    sh->n_tok = n_claim; sh->best = fbest; sh->cut_bin = 255;
    sh->frame_base = base_cur; sh->n_rec = base_cur + n_claim;
    sh->a_lean += 1;
    sh->a_lean_tokens += (unsigned long long)n_claim;
    sh->a_maxtok = max(sh->a_maxtok, n_claim);
    sh->a_rounds += (unsigned long long)sh->rounds;
    sh->rounds = 0;
  }
  int w_surv = 0;
  // vmcnt(0): this wave's pieces of the next row have arrived in LDS; the barrier at the end of the frame tells the
  // others.  (The compiler waits for them already at the write of wcount, as it does before any LDS access behind such a
  // request; nothing here relies on that, and a frame that ends above waits in the caller.)  Here and not at that
  // barrier it is no wait for the frame's stores: the back-pointer records and long rows are read by other waves only
  // behind later barriers, which keep them in order (rows_to_device).  A row that was only touched is waited for too;
  // left on its way until the end of the frame, 1 to 512 channels are no faster (0.995 to 1.001 of the speed).
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::"v"(touched));   // (the read of the row is kept)
  // Every commit of this wave is in its log.  A state's value names its arc, so the entry whose arc is the
  // state's value is the winner and writes the token: cost, row, back-pointer record, state (last frame),
  // histogram.  An emitting arc is expanded once per frame, so its entry is unique; a closure record can have
  // been committed twice with the same (cost, arc) (two walks of one list from values that round to the same
  // sum): the compare-and-swap lets one of the two write.
  int2 *bp_cur = bp + base_cur;
  for (int j0 = 0; j0 < W.n_clog; j0 += 64) {
    // (lanes beyond the log look at its last entry: all lanes have to take part in what the waves' bases come from)
    const uint2 e = *(const uint2 *)&clog[min(j0 + lane, W.n_clog - 1)];
    const uint32_t eh = e.y & 0xFFFFu;
    // everything the winner will need is asked for together: the state's value, row and token id, and the source
    // state's token id
    const uint64_t v = M.hval[eh];
    const int row = R.hrow[eh];
    const uint32_t ed = R.hed[eh];
    const int lid = (int)M.hidx[eh];
    const bool from_token = (int)e.y < 0;
    const int from = (int)((e.y >> 16) & (kLeanFromToken - 1));
    const int plid = (int)M.hidx[from_token ? 0 : from];
    const int idx = from_lane(wbase, lid >> kLeanLidBits) + (lid & kLeanLidMask);
    const int pidx = from_lane(wbase, (plid >> kLeanLidBits) & 15) + (plid & kLeanLidMask);
    bool surv = false;
    if (j0 + lane < W.n_clog) {
      bool win = (uint32_t)v == e.x && v != kEmptyVal;
      if (win && !from_token)
        win = atomicCAS((unsigned long long *)&M.hval[eh], (unsigned long long)v, (unsigned long long)kEmptyVal) == v;
      if (win) {
        const float c = ord2f((uint32_t)(v >> 32));
        M.t_cost[idx] = c;
        R.t_first[idx] = row;
        R.t_deg[idx] = ed == kEdEscape ? kLeanDegEscape : (uint16_t)ed;
        bp_cur[idx] = make_int2((int)e.x, from_token ? base_prev + from : base_cur + pidx);
        uint32_t state = 0;
        if (last_frame || ed == kEdEscape) state = M.hkey[eh];
        if (last_frame) g_tok_state[idx] = (int)state;
        if (ed == kEdEscape) {
          // a row too long for the count field (rare): its bounds go to the row buffer in device memory, where
          // the general code, which will take the next frame, looks for them
          const int4 o = p.off2[state];
          int4 *hbm_rows = M.t_row + (size_t)row_buf * M.row_cap;
          hbm_rows[idx] = make_int4(o.x, o.y, o.z, 0);
        }
        M.hkey[eh] = kEmptyKey;
        if (from_token) M.hval[eh] = kEmptyVal;
        if (hist_need) {
          const float r = c - fbest;
          if (!(r > p.beam)) {
            surv = true;
            int bin = (int)floorf(r * inv);
            bin = bin > 255 ? 255 : bin;
            atomicAdd(&hist[bin], 1u);
          }
        }
      }
    }
    if (hist_need) w_surv += __popcll(lanes_with(surv));
  }
  if (lane == 0) {
    // (two counters to an atomic; they are taken apart when the call ends)
    atomicAdd(&sh->a_lean_pack[0], (unsigned long long)(uint32_t)n_active_frame | ((unsigned long long)(uint32_t)n_emit << 32));
    atomicAdd(&sh->a_lean_pack[1], (unsigned long long)(uint32_t)W.n_eps | ((unsigned long long)(uint32_t)W.n_cand << 32));
  }
  // ---- the histogram cut: the wave that gets here last takes it (every wave's LDS traffic of this phase lies before
  // its count, and LDS keeps a wave's operations in order)
  if (hist_need) {   // uniform
    int done = 0;
    if (lane == 0) {
      if (w_surv) atomicAdd(&sh->n_surv, w_surv);
      done = atomicAdd(&sh->n_done, 1);
    }
    if (__builtin_amdgcn_readfirstlane(done) == NW - 1) {
      int loc[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { loc[k] = (int)hist[lane * 4 + k]; hist[lane * 4 + k] = 0; }
      if (sh->n_surv > p.max_active) {
        const int sum = loc[0] + loc[1] + loc[2] + loc[3];
        int run = wave_incl_scan(sum) - sum;
        int myB = -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) { run += loc[k]; if (run <= p.max_active) myB = lane * 4 + k; }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) { const int t = __shfl_xor(myB, d, 64); myB = t > myB ? t : myB; }
        if (lane == 0) sh->cut_bin = myB < 0 ? 0 : myB;   // (behind the 255 above: that wave has counted since)
      }
      if (lane == 0) { sh->n_surv = 0; sh->n_done = 0; }
    }
  }
  CBD_STAMP(4);   // look-up phase of wave 0
  wg_barrier<true>();
  CBD_STAMP(5);   // its wait at the last barrier (with the histogram cut by the last wave)
  return kFrameOk;
}

}  // namespace cbd
