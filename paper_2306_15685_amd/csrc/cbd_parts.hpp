// Frames that outgrow the LDS tables, by parts: the same frame as run_frame() computes, for one workgroup, with the
// states split into K shares by a hash.  One share's state table fills the LDS region of the lean tables; the shares
// are recombined one after another, so that no table lives in device memory:
//
//   1  costs of all tokens are read, the live ones gathered in full groups and expanded (steps 1 and 2 of the frame);
//      candidates within the beam of the running minimum go to the queue of their destination's share (device memory,
//      16 bytes each, the memory of the general code's change log).  Rows with hundreds of arcs do not travel: their
//      arcs are sorted by share when the decoder is made, and here only count for the minimum
//   2  the minimum is final: stored closure lists of what passes are walked (spread over a wave's lanes as in lean
//      frames), closure candidates go to a second set of queues
//   3  per share: its candidates and the long rows' arcs are recombined in the LDS table (E[state] = min key), then
//      gone through once more: the one whose key is the state's value writes the token and its record.  Entries whose
//      state has a closure list then note their state's token
//   4  records of closure winners get their predecessor; histogram cut and scalars of the next frame
//
// What bounds it: vector instructions and L2 latency in turn (20,000 arcs of a hub are costed three times per frame
// rather than stored and read back).  The table in device memory that it replaces took a chain of six dependent
// device-memory accesses per candidate, most of them atomics: 160 channels x 40 frames of a 20,000-word lexicon loop
// 31.0 -> 4.0 ms (kernel time per frame 755 -> 95 us; wave 0 stamps 15 for reading and expanding tokens, 5 for the hub's
// minimum, 3 closure lists, 11 to set the tables up, 19 recombination, 27 winners, 80 together), 148 channels x 40 frames
// of 5,600 words 7.4 -> 2.0 ms.
// Who decodes so: cbd_decoder_create, from the graph and the sizes alone.  Graphs without long rows keep the general code
// for the frames that outgrow LDS, which are too few there to tell (in the kernel of kPartsFew 2,048 channels at beam 16
// take 9,840 to 10,140 us instead of 9,950 to 10,170, four other cases the same).  So do graphs with a state whose closure
// is not stored as a list, were it only one: queued entries find their closure records by the degrees in an arc's record,
// which such a state does not have.  A long row with an epsilon-input arc (a back-off) is such a state.
// A frame that does not fit (a full queue or share) leaves nothing behind and is redone by the general code, each time: to let
// such frames go there at once would refuse some that fit, since its change log counts the arcs of long rows and the queues do
// not (a second try in the frame loop behind it spilled 43 to 70 registers).
#pragma once

namespace cbd {

constexpr int kPartsMax = 8;
constexpr uint32_t kPartClosure = 0x80000000u;   // PartEntry::from: a closure candidate, the rest is its parent's entry
constexpr uint32_t kPartHasList = 0x40000000u;   // the entry's state has a closure list: its token will be asked for
constexpr uint32_t kPartMask = 0x3FFFFFFFu;

// A candidate in a queue.  from: source token of an emitting arc, or (kPartClosure) the entry of the arc's source state.
// Once its share is done: cost of an entry with kPartHasList = its state's token; arc of a closure entry = the token it
// wrote, or kArcNone.
struct __attribute__((aligned(16))) PartEntry {
  uint32_t dst;
  float cost;
  uint32_t arc;
  uint32_t from;
};
static_assert(sizeof(PartEntry) == sizeof(LogT<false>), "the queues use the change log's memory");

// A token that survived pruning, on its way to a lane.
struct LiveToken { float cost; int32_t first; int32_t deg; int32_t idx; };

// Which of k shares a state belongs to, and its home slot in that share's table (different bits of the hash).
__device__ __forceinline__ uint32_t share_hash(uint32_t state) { return state * 2654435761u; }
__device__ __forceinline__ int share_owner(uint32_t state, int k) { return (int)__umulhi(share_hash(state), (uint32_t)k); }
__device__ __forceinline__ uint32_t share_home(uint32_t state, uint32_t slots) {
  return __umulhi(share_hash(state) * 0x9E3779B1u, slots);
}

// An arc of a long row as it is laid out when the decoder is made: everything a frame needs to cost it, and the slot of
// its destination in its share's table.
struct __attribute__((aligned(16))) LongArc {
  float weight;
  uint32_t arc;       // library index
  uint32_t slot_pdf;  // bits 0..15 slot, 16..31 pdf
  int32_t row;        // first arc of the destination (long_meta: its degrees)
};

// Places in the queues of the entries' owners for up to U entries per lane: lane o adds the wave's count for owner o,
// so one LDS atomic hands out the places of all owners.
template <int U>
__device__ __forceinline__ void parts_places(int32_t *cnt, int k, const bool (&act)[U], const int (&owner)[U], int lane,
                                             int (&pos)[U]) {
  const unsigned long long below = (1ull << lane) - 1ull;
  int mine = 0, rank[U];
#pragma unroll
  for (int u = 0; u < U; ++u) rank[u] = 0;
  for (int o = 0; o < k; ++o) {   // uniform
    int n = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned long long m = __ballot(act[u] && owner[u] == o);
      if (owner[u] == o) rank[u] = n + (int)__popcll(m & below);
      n += (int)__popcll(m);
    }
    if (lane == o) mine = n;
  }
  int base = 0;
  if (mine > 0) base = atomicAdd(&cnt[lane], mine);
#pragma unroll
  for (int u = 0; u < U; ++u) pos[u] = __shfl(base, owner[u], 64) + rank[u];
}

// One workgroup per long row: its arcs sorted by the share that owns their destination, so that a share's arcs are one
// stream; those whose destination has a closure list lie behind all others (group k: they go through the queues).  The
// order inside a group does not matter.  The destinations get their slots here, once: image[share][slot] is the key table
// as every frame starts from it (all ones before; *full: a share has no slot left).  An arc of a long row is then
// recombined without a search: the shares of a frame with 20,000 such arcs in 19 instead of 33 us (5.45 -> 4.05 ms a pass).
constexpr int kPrepRowThreads = 1024;
__global__ __launch_bounds__(kPrepRowThreads) void prepare_long_rows_kernel(const ArcRec *arcs, const int4 *rows, int32_t *group,
                                                                            LongArc *out, uint32_t *out_meta, uint32_t *image,
                                                                            uint32_t slots, int32_t *full, int k) {
  __shared__ int32_t count[kPartsMax + 1], fill[kPartsMax + 1];
  const int4 row = rows[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid <= kPartsMax) count[tid] = 0;
  __syncthreads();
  // (a wave's arcs are counted, and get their places, with one atomic per group)
  for (int j0 = tid - lane; j0 < row.z; j0 += kPrepRowThreads) {   // uniform
    const int j = j0 + lane;
    const bool act[1] = {j < row.z};
    ArcRec r; r.dst = 0; r.weight = 0.0f; r.row = 0; r.meta = 0;
    if (act[0]) r = arcs[row.y + j];
    const int to[1] = {meta_cl(r.meta) ? k : share_owner((uint32_t)r.dst, k)};
    int at[1];
    parts_places<1>(count, k + 1, act, to, lane, at);
  }
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int o = 0; o <= k; ++o) { group[blockIdx.x * (k + 2) + o] = run; fill[o] = run; run += count[o]; }
    group[blockIdx.x * (k + 2) + k + 1] = run;
  }
  __syncthreads();
  for (int j0 = tid - lane; j0 < row.z; j0 += kPrepRowThreads) {   // uniform
    const int j = j0 + lane;
    const bool act[1] = {j < row.z};
    ArcRec r; r.dst = 0; r.weight = 0.0f; r.row = 0; r.meta = 0;
    if (act[0]) r = arcs[row.y + j];
    const uint32_t state = (uint32_t)r.dst;
    const int o = share_owner(state, k);
    const int to[1] = {meta_cl(r.meta) ? k : o};
    int at[1];
    parts_places<1>(fill, k + 1, act, to, lane, at);
    if (!act[0]) continue;
    uint32_t h = 0;
    if (!meta_cl(r.meta)) {
      uint32_t *keys = image + (size_t)o * slots;
      h = share_home(state, slots);
      uint32_t key = atomicCAS(&keys[h], kEmptyKey, state);
      for (uint32_t probe = 1; key != kEmptyKey && key != state && probe < slots; ++probe) {
        h = h + 1 == slots ? 0 : h + 1;
        key = atomicCAS(&keys[h], kEmptyKey, state);
      }
      if (key != kEmptyKey && key != state) *full = 1;
    }
    LongArc l;
    l.weight = r.weight; l.arc = (uint32_t)(row.y + j); l.row = r.row;
    l.slot_pdf = h | (((r.meta & 0xFFFFu) - 1u) << 16);
    out[row.w + at[0]] = l;
    out_meta[row.w + at[0]] = r.meta & 0xFFFF0000u;
  }
}

// The table of the share at hand.
struct PartTable {
  uint64_t *hval;
  uint32_t *hkey;
  uint32_t slots;
};

// E[state] = min key; returns the state's slot.  A table without a free one sets sh->redo.
__device__ __forceinline__ uint32_t part_min(const PartTable &T, Shared *sh, uint32_t state, uint64_t key) {
  uint32_t h = share_home(state, T.slots);
  uint32_t k = atomicCAS(&T.hkey[h], kEmptyKey, state);
  uint32_t probe = 1;
  while (k != kEmptyKey && k != state && probe < T.slots) {
    h = h + 1 == T.slots ? 0 : h + 1;
    k = atomicCAS(&T.hkey[h], kEmptyKey, state);
    // (a long walk means a nearly full table: stop as soon as anybody has found it full)
    if ((++probe & 63u) == 0 && __hip_atomic_load(&sh->redo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
  }
  if (k == kEmptyKey || k == state) atomicMin((unsigned long long *)&T.hval[h], (unsigned long long)key);
  else sh->redo = 1;
  return h;
}
// The slot of a state that is in the table.
__device__ __forceinline__ uint32_t part_find(const PartTable &T, uint32_t state) {
  uint32_t h = share_home(state, T.slots);
  uint32_t probe = 0;
  while (T.hkey[h] != state && probe < T.slots) { h = h + 1 == T.slots ? 0 : h + 1; ++probe; }
  return h;
}

// The closure lists of up to 64 states, one per lane (len records from pos; cost and ref: the state's candidate and its
// entry's place in the queues), spread over the lanes one record each, as many whole lists at a time as fit 64 lanes.
// What passes the cutoff goes to the closure queues.  Q2: the first of these; q2_first: its place in the queues.
__device__ __forceinline__ void parts_closures(const AdvanceParams &p, Shared *sh, const Ctx &cx, PartEntry *Q2, int q2_first,
                                               float m, uint8_t *cmap, int pos, int len, float cost, int ref, int lane,
                                               uint32_t &n_eps, uint32_t &n_cand, int &max_depth) {
  const int k = p.parts, cap = p.part_q2;
  for (;;) {
    const int incl = wave_incl_scan(len);
    if (__builtin_amdgcn_readlane(incl, 63) == 0) return;   // uniform
    const bool go = len > 0 && incl <= 64;   // (a list has at most 62 records: the first one always goes)
    const int start = incl - len;
    const unsigned long long gm = __ballot(go);
    const int total = __builtin_amdgcn_readlane(incl, 63 - __builtin_clzll(gm));
    if (lane < 16) ((uint32_t *)cmap)[lane] = 0;
    if (go) cmap[start] = (uint8_t)(lane + 1);
    int owner = wave_incl_scan_max((int)cmap[lane]) - 1;   // the lane whose list a record belongs to
    owner = owner < 0 ? 0 : owner;
    const bool act = lane < total;
    const int o_start = __shfl(start, owner, 64);
    const int rpos = __shfl(pos, owner, 64) + lane - o_start;
    ArcRec rec; rec.dst = 0; rec.weight = 0.0f; rec.row = 0; rec.meta = 0;
    int can = 0;
    if (act) { rec = p.arcs[rpos]; can = p.canon[rpos]; }
    const float o_cost = __shfl(cost, owner, 64);
    const int o_ref = __shfl(ref, owner, 64);
    const int depth = act ? (int)(rec.meta & 0xFu) : 0;
    const int plane = (o_start - 1 + (int)((rec.meta >> 4) & 0x3Fu)) & 63;   // the lane that holds the parent record
    float w = rec.weight;
    if (act && ctx_contains(cx, can)) w = w + cx.offset;   // Sec. 4.1: boosted weight = weight + discount
    float c = __builtin_inff();
    bool ok = false;
    if (depth == 1) {
      const float cc = o_cost + w;
      ok = cc < __builtin_inff() && !(cc - m > p.beam);
      if (ok) c = cc;
    }
    const int maxd = __builtin_amdgcn_readlane(wave_incl_scan_max(depth), 63);
    for (int d = 2; d <= maxd; ++d) {   // uniform
      const float pc = __shfl(c, plane, 64);
      if (depth == d) {
        const float cc = pc + w;
        ok = cc < __builtin_inff() && !(cc - m > p.beam);
        if (ok) c = cc;
      }
    }
    max_depth = max(max_depth, maxd);
    n_eps += (uint32_t)total;
    const unsigned long long om = __ballot(ok);
    if (om != 0) {
      n_cand += (uint32_t)__popcll(om);
      const uint32_t co = ok ? f2ord(c) : 0xFFFFFFFFu;
      if (__ballot(ok && co < f2ord(m)) != 0) {
        const uint32_t wmin = wave_min_u32(co);
        if (lane == 0) atomicMin(&sh->best_ord, wmin);
      }
      // candidates of one wave for one state without a list of its own (word ends lead to the hub): the least key goes
      const int fl = (int)__builtin_ctzll(om);
      const int d0 = __builtin_amdgcn_readlane(rec.dst, fl);
      if (__popcll(om) > 1 && __ballot(ok && rec.dst == d0 && meta_cl(rec.meta) == 0) == om) {
        const uint32_t mhi = wave_min_u32(co);
        const uint32_t mlo = wave_min_u32(ok && co == mhi ? (uint32_t)can : 0xFFFFFFFFu);
        ok = ok && co == mhi && (uint32_t)can == mlo;
        ok = ok && lane == (int)__builtin_ctzll(__ballot(ok));   // (two lanes can hold the same key)
      }
      const bool act1[1] = {ok};
      const int owner1[1] = {ok ? share_owner((uint32_t)rec.dst, k) : 0};
      int at[1];
      parts_places<1>(&sh->wcount[kPartsMax], k, act1, owner1, lane, at);
      const int place = owner1[0] * cap + at[0];
      const int parent = __shfl(q2_first + place, plane, 64);   // (used below depth 1: the parent record has passed too)
      if (ok) {
        if (at[0] < cap) {
          PartEntry e;
          e.dst = (uint32_t)rec.dst; e.cost = c; e.arc = (uint32_t)can;
          e.from = kPartClosure | (meta_cl(rec.meta) ? kPartHasList : 0u) | (uint32_t)(depth == 1 ? o_ref : parent);
          Q2[place] = e;
        } else {
          sh->fault = 1;
        }
      }
    }
    if (go) len = 0;
  }
}

// One frame.  region: the LDS of the lean tables, p.part_slots * 12 bytes.  cost_in / cost_out: the current tokens'
// costs and where the new ones go (apart, so that a frame can be given up at any point).  Returns kFrameOk,
// kFrameNoTokens, kFrameOverflow, kFrameRecordsFull, or kFrameRedo (the general code decodes the frame).
template <int kBlock>
__device__ __forceinline__ int run_frame_parts(const AdvanceParams &p, unsigned char *region, int c, Shared *sh, const Ctx &cx,
                                               float *Lstage, const Rows &Lrow, const float *Lnext, uint32_t *hist,
                                               uint8_t *owner_maps, uint8_t *closure_maps, int cur, int2 *bp,
                                               int32_t *g_tok_state, bool last_frame, const float *cost_in, float *cost_out) {
  constexpr int NW = kBlock / 64;
  const int tid = here_tid(), lane = tid & 63, wave = tid >> 6;
  const int k = p.parts, cap1 = p.part_q1, cap2 = p.part_q2;
  PartEntry *Q1 = (PartEntry *)(p.g_log + (size_t)c * p.g_log_cap);
  PartEntry *Q2 = Q1 + (size_t)k * cap1;
  const int4 *rows_in = p.tok_row + (size_t)c * 2 * p.g_tok_cap + (size_t)cur * p.g_tok_cap;
  int4 *rows_out = p.tok_row + (size_t)c * 2 * p.g_tok_cap + (size_t)(cur ^ 1) * p.g_tok_cap;
  uint8_t *owner_map = owner_maps + wave * kOwnerMap;
  uint8_t *cmap = closure_maps + wave * 64;
  int32_t *cnt1 = sh->wcount, *cnt2 = sh->wcount + kPartsMax;   // entries per queue
  int32_t *n_made = &sh->wbase[0];                             // tokens so far
  int32_t *n_lists = &sh->wbase[1];                            // candidates noted for step 2
  // step 2's work: (first record, records, cost, entry) of every queued candidate whose state has a closure list
  int4 *lists = (int4 *)(region + NW * 64 * sizeof(LiveToken));
  const int lists_cap = (int)((p.part_slots * 12 - NW * 64 * (int)sizeof(LiveToken)) / 16);
  const bool hist_on = p.max_active > 0 && p.beam > 0.0f && p.beam < __builtin_inff();
  const float inv = 256.0f / p.beam;
  if (tid < 16) { sh->wcount[tid] = 0; sh->wbase[tid] = 0; }
#ifdef CBD_PROFILE
  if (tid == 0) sh->prof_last = wall_clock64();
#endif
  __syncthreads();

  // ---- 1: prune and expand
  uint32_t n_active = 0, n_emit = 0, n_eps = 0, n_cand = 0;
  int max_depth = 0;
  const int n_tok = sh->n_tok;
  const float best = sh->best;
  const int cut = sh->cut_bin;
  // up to two arcs per lane, already read: candidate costs join the running minimum, what is within its beam is queued
  auto queue_arcs = [&](const bool (&act)[2], const int (&arc)[2], const ArcRec (&rec)[2], const float (&c_own)[2], const int (&src)[2]) {
    float cand[2];
    uint32_t lmin = 0xFFFFFFFFu;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      cand[q] = 0.0f;
      if (act[q]) {
        float w = rec[q].weight;
        if (ctx_contains(cx, arc[q])) w = w + cx.offset;   // Sec. 4.1
        cand[q] = (c_own[q] + w) - Lrow.at((rec[q].meta & 0xFFFFu) - 1u);
        const uint32_t o = f2ord(cand[q]);
        lmin = o < lmin ? o : lmin;
      }
    }
    const uint32_t wmin = wave_min_u32(lmin);
    if (lane == 0 && wmin != 0xFFFFFFFFu) atomicMin(&sh->m_ord, wmin);
    const float mref = ord2f(__hip_atomic_load(&sh->m_ord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    bool pass[2];
    int owner[2], at[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      pass[q] = act[q] && !(cand[q] - mref > p.beam);
      owner[q] = pass[q] ? share_owner((uint32_t)rec[q].dst, k) : 0;
    }
    if (__ballot(pass[0] || pass[1]) == 0) return;   // uniform
    parts_places<2>(cnt1, k, pass, owner, lane, at);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool list = pass[q] && meta_cl(rec[q].meta) != 0;
      const unsigned long long lm = __ballot(list);
      if (lm != 0) {   // uniform
        int first = 0;
        if (lane == 0) first = atomicAdd(n_lists, (int)__popcll(lm));
        const int i = __builtin_amdgcn_readfirstlane(first) + (int)__popcll(lm & ((1ull << lane) - 1ull));
        if (list) {
          if (i < lists_cap)
            lists[i] = make_int4(rec[q].row + (int)meta_ed(rec[q].meta) + (int)meta_xd(rec[q].meta), (int)meta_cl(rec[q].meta),
                                 (int)__float_as_uint(cand[q]), owner[q] * cap1 + at[q]);
          else sh->fault = 1;
        }
      }
      if (pass[q]) {
        if (at[q] < cap1) {
          PartEntry e;
          e.dst = (uint32_t)rec[q].dst; e.cost = cand[q]; e.arc = (uint32_t)arc[q];
          e.from = (uint32_t)src[q] | (meta_cl(rec[q].meta) ? kPartHasList : 0u);
          Q1[owner[q] * cap1 + at[q]] = e;
        } else {
          sh->fault = 1;
        }
      }
    }
  };
  {
    // Most tokens of a frame like this fall to the histogram cut: only the costs are read for all of them (eight tiles
    // of a wave at a time); the live ones are gathered in the wave's staging list and expanded 64 at a time.
    LiveToken *stage = (LiveToken *)region + wave * 64;
    auto expand_staged = [&](int n) {
      LiveToken tk; tk.cost = 0.0f; tk.first = 0; tk.deg = 0; tk.idx = 0;
      if (lane < n) {
        tk = stage[lane];
        const int2 fe = load_row_fe(&rows_in[tk.idx]);
        tk.first = fe.x; tk.deg = fe.y - fe.x;
        if (tk.deg > kBigRowArcs) {
          const int slot = atomicAdd(&sh->n_big, 1);
          if (slot < kBigRows) {
            sh->big_first[slot] = tk.first; sh->big_deg[slot] = tk.deg; sh->big_cost[slot] = tk.cost; sh->big_src[slot] = (uint32_t)tk.idx;
            tk.deg = 0;
          }
        }
      }
      const ArcList AL = make_arc_list(tk.first, tk.deg, lane, owner_map);
      n_emit += (uint32_t)AL.total;
      for (int jb = 0; jb < AL.total; jb += 128) {   // uniform
        bool act[2];
        int arc[2], src[2];
        float c_own[2];
        ArcRec rec[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j0 = jb + q * 64, j = j0 + lane;
          act[q] = j < AL.total;
          arc[q] = 0; src[q] = 0; c_own[q] = 0.0f;
          rec[q].dst = 0; rec[q].weight = 0.0f; rec[q].row = 0; rec[q].meta = 0;
          if (j0 < AL.total) {   // uniform
            const int owner = arc_owner(AL, j, j0);
            arc[q] = __shfl(AL.rel, owner, 64) + j;
            c_own[q] = __shfl(tk.cost, owner, 64);
            src[q] = __shfl(tk.idx, owner, 64);
            if (act[q]) rec[q] = p.arcs[arc[q]];
          }
        }
        queue_arcs(act, arc, rec, c_own, src);
      }
    };
    int n_staged = 0;
    for (int base = wave * 64; base < n_tok; base += 8 * kBlock) {   // uniform
      float cost[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = base + u * kBlock + lane;
        cost[u] = i < n_tok ? cost_in[i] : __builtin_inff();
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = base + u * kBlock + lane;
        const float r = cost[u] - best;
        bool alive = i < n_tok && !(r > p.beam) && cost[u] < __builtin_inff();
        if (alive && cut < 255) {
          int bin = (int)floorf(r * inv);
          bin = bin > 255 ? 255 : bin;
          alive = bin <= cut;
        }
        const unsigned long long lm = __ballot(alive);
        const int n_new = (int)__popcll(lm);
        n_active += (uint32_t)n_new;
        if (n_new == 0) continue;   // uniform
        if (n_staged + n_new > 64) { expand_staged(n_staged); n_staged = 0; }
        if (alive) {
          LiveToken tk; tk.cost = cost[u]; tk.first = 0; tk.deg = 0; tk.idx = i;
          stage[n_staged + (int)__popcll(lm & ((1ull << lane) - 1ull))] = tk;
        }
        n_staged += n_new;
      }
    }
    if (n_staged > 0) expand_staged(n_staged);
  }
  __syncthreads();
  CBD_STAMP(0);   // (diagnostic: tokens read, live ones expanded)
  const int n_big = min(sh->n_big, kBigRows);
  // an announced long row's place among the prepared ones, or -1
  auto row_id = [&](int r) {
    const int first = sh->big_first[r];
    int lo = 0, hi = p.lr.n;
    while (lo < hi) {   // uniform
      const int mid = (lo + hi) >> 1;
      if (p.lr.rows[mid].y < first) lo = mid + 1; else hi = mid;
    }
    return (lo < p.lr.n && p.lr.rows[lo].y == first) ? lo : -1;
  };
  auto long_cost = [&](const LongArc &l, float cost) {
    float w = l.weight;
    if (ctx_contains(cx, (int)l.arc)) w = w + cx.offset;   // Sec. 4.1
    return (cost + w) - Lrow.at(l.slot_pdf >> 16);
  };
  if (n_big > 0) {   // uniform
    for (int r = 0; r < n_big; ++r) {
      const int first = sh->big_first[r], deg = sh->big_deg[r], src = (int)sh->big_src[r];
      const float cost = sh->big_cost[r];
      const int id = row_id(r);
      if (wave == 0) n_emit += (uint32_t)deg;
      uint32_t lmin = 0xFFFFFFFFu;
      int queue_from = 0, queue_to = deg, first_sorted = 0;   // what goes through the queues: all of an unknown row
      if (id >= 0) {
        const int4 row = p.lr.rows[id];
        first_sorted = row.w;
        queue_from = p.lr.group[id * (k + 2) + k]; queue_to = p.lr.group[id * (k + 2) + k + 1];
        for (int t0 = tid; t0 < queue_from; t0 += 4 * kBlock) {
          LongArc l[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) l[u] = p.lr.arcs[row.w + min(t0 + u * kBlock, queue_from - 1)];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint32_t o = f2ord(long_cost(l[u], cost));   // (the last arc again and again does no harm)
            lmin = o < lmin ? o : lmin;
          }
        }
        const uint32_t wmin = wave_min_u32(lmin);
        if (lane == 0 && wmin != 0xFFFFFFFFu) atomicMin(&sh->m_ord, wmin);
      }
      for (int j0 = queue_from + wave * 128; j0 < queue_to; j0 += NW * 128) {   // uniform
        bool act[2];
        int arc[2];
        ArcRec rec[2];
        const float c_own[2] = {cost, cost};
        const int srcs[2] = {src, src};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = j0 + q * 64 + lane;
          act[q] = j < queue_to;
          arc[q] = 0;
          rec[q].dst = 0; rec[q].weight = 0.0f; rec[q].row = 0; rec[q].meta = 0;
          if (act[q]) {
            arc[q] = id >= 0 ? (int)p.lr.arcs[first_sorted + j].arc : first + j;
            rec[q] = p.arcs[arc[q]];
          }
        }
        queue_arcs(act, arc, rec, c_own, srcs);
      }
    }
    __syncthreads();
  }

  CBD_STAMP(1);   // (diagnostic: long rows' minimum)
  // ---- 2: the minimum is final; closure lists of what passes
  const uint32_t m_ord = sh->m_ord;
  if (m_ord == 0xFFFFFFFFu) return kFrameNoTokens;   // (uniform: no candidate at all)
  const float m = ord2f(m_ord);
  {
    const int n = min(*n_lists, lists_cap), per = min((n + NW - 1) / NW, 64);   // shared evenly by the waves
    for (int base = wave * per; base < n; base += NW * per) {   // uniform
      int4 w = make_int4(0, 0, 0, 0);
      if (lane < per && base + lane < n) w = lists[base + lane];
      const float cost = __uint_as_float((uint32_t)w.z);
      if (cost - m > p.beam) w.y = 0;
      parts_closures(p, sh, cx, Q2, k * cap1, m, cmap, w.x, w.y, cost, w.w, lane, n_eps, n_cand, max_depth);
    }
  }
  __syncthreads();
  if (__builtin_expect(sh->fault, 0)) {   // (uniform: set in steps 1 and 2 only) a queue is full
    if (tid == 0) sh->a_rounds += kPartsCount;
    return kFrameRedo;
  }
  CBD_STAMP(2);   // (diagnostic: closure lists)
  const float fbest = ord2f(umin32(m_ord, sh->best_ord));
  bool have_closures = false;
  for (int o = 0; o < k; ++o) have_closures = have_closures || cnt2[o] > 0;

  // ---- 3: share by share
  PartTable T;
  T.hval = (uint64_t *)region;
  T.hkey = (uint32_t *)(region + (size_t)p.part_slots * 8);
  T.slots = (uint32_t)p.part_slots;
  const int base_cur = sh->n_rec, base_prev = sh->frame_base;
  int w_surv = 0;
  // The long rows' arcs into share o, four per thread and round: fn(arcs, their places, which of them are within the cutoff,
  // costs, source token).  (Kept in registers for both passes, they spill 65 registers: 4.09 -> 4.25 ms.)
  auto for_long_arcs = [&](int o, auto &&fn) {
    for (int r = 0; r < n_big; ++r) {
      const int id = row_id(r);
      if (id < 0) continue;   // uniform
      const int4 row = p.lr.rows[id];
      const int g0 = row.w + p.lr.group[id * (k + 2) + o], g1 = row.w + p.lr.group[id * (k + 2) + o + 1];
      const float cost = sh->big_cost[r];
      const int src = (int)sh->big_src[r];
      for (int base = g0 + wave * 64; base < g1; base += 4 * kBlock) {   // uniform
        LongArc l[4];
        float cand[4];
        bool pass[4];
        int at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = base + u * kBlock + lane;
          pass[u] = t < g1;
          at[u] = min(t, g1 - 1);
          l[u] = p.lr.arcs[at[u]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          cand[u] = long_cost(l[u], cost);
          pass[u] = pass[u] && !(cand[u] - m > p.beam);
        }
        fn(l, at, pass, cand, src);
      }
    }
  };
  // the winner of a state writes the token: cost, row, state (last frame), histogram
  auto write_token = [&](int idx, uint32_t h, uint32_t state, float cost, uint32_t arc, const RowInfo &row, int prev) {
    T.hval[h] = 0xFFFFFFFF00000000ull | (uint32_t)idx;   // (no candidate's key) the state's token
    if (idx >= p.g_tok_cap) return false;
    cost_out[idx] = cost;
    rows_out[idx] = make_int4(row.first, row.eps, row.end, 0);
    if (base_cur + idx < p.bp_cap) bp[base_cur + idx] = make_int2((int)arc, prev);
    if (last_frame) g_tok_state[idx] = (int)state;
    const float r = cost - fbest;
    const bool surv = !(r > p.beam);
    if (surv && hist_on) {
      int bin = (int)floorf(r * inv);
      bin = bin > 255 ? 255 : bin;
      atomicAdd(&hist[bin], 1u);
    }
    return surv;
  };
  // places for the tokens of the lanes with win set (by whole waves)
  auto token_places = [&](unsigned long long wm) {
    int first = 0;
    if (lane == 0) first = atomicAdd(n_made, (int)__popcll(wm));
    return __builtin_amdgcn_readfirstlane(first) + (int)__popcll(wm & ((1ull << lane) - 1ull));
  };
  for (int o = 0; o < k; ++o) {
    const int n1 = min(cnt1[o], cap1), n2 = min(cnt2[o], cap2);
    PartEntry *q1 = Q1 + o * cap1, *q2 = Q2 + o * cap2;
    // (the first round's entry is asked for ahead of the table and stays in registers for both passes)
    PartEntry e0; e0.dst = 0; e0.cost = 0.0f; e0.arc = 0; e0.from = 0;
    if (tid < n1) e0 = q1[tid];
    {
      // the table starts with the keys of the long rows' destinations; everything else in it is all ones
      uint4 *t4 = (uint4 *)region;
      const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
      for (uint32_t i = tid; i < T.slots / 2; i += kBlock) t4[i] = ones;
      uint4 *k4 = (uint4 *)T.hkey;
      const uint4 *image = (const uint4 *)(p.lr.image + (size_t)o * T.slots);
      if (p.lr.n > 0) for (uint32_t i = tid; i < T.slots / 4; i += kBlock) k4[i] = image[i];
      else for (uint32_t i = tid; i < T.slots / 4; i += kBlock) k4[i] = ones;
    }
    __syncthreads();
    CBD_STAMP(3);   // (diagnostic: tables emptied)
    uint32_t h0 = 0;
    bool pass0 = false;
    for (int base = wave * 64; base < n1; base += kBlock) {   // uniform
      const int i = base + lane;
      const PartEntry e = base == wave * 64 ? e0 : q1[min(i, n1 - 1)];
      const bool pass = i < n1 && !(e.cost - m > p.beam);
      uint32_t h = 0;
      if (pass) h = part_min(T, sh, e.dst, ((uint64_t)f2ord(e.cost) << 32) | e.arc);
      if (base == wave * 64) { h0 = h; pass0 = pass; }
      n_cand += (uint32_t)__popcll(__ballot(pass));
    }
    for (int i = tid; i < n2; i += kBlock) {
      const PartEntry e = q2[i];
      part_min(T, sh, e.dst, ((uint64_t)f2ord(e.cost) << 32) | e.arc);
    }
    for_long_arcs(o, [&](const LongArc (&l)[4], const int (&)[4], const bool (&pass)[4], const float (&cand)[4], int) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (pass[u]) atomicMin((unsigned long long *)&T.hval[l[u].slot_pdf & 0xFFFFu], ((uint64_t)f2ord(cand[u]) << 32) | l[u].arc);
        n_cand += (uint32_t)__popcll(__ballot(pass[u]));
      }
    });
    __syncthreads();
    if (__builtin_expect(sh->redo, 0)) {   // (uniform: set between this barrier and the one before) the share's table is full
      if (tid == 0) sh->a_rounds += kPartsCount;
      return kFrameRedo;
    }
    CBD_STAMP(4);   // (diagnostic: shares recombined)
    // An emitting arc is expanded once per frame, so its entry is the only one with its key; a closure arc can have been
    // reached twice with the same key: there an exchange lets one of the two through.
    for (int base = wave * 64; base < n1; base += kBlock) {   // uniform
      const int i = base + lane;
      const bool first = base == wave * 64;
      const PartEntry e = first ? e0 : q1[min(i, n1 - 1)];
      const bool pass = first ? pass0 : i < n1 && !(e.cost - m > p.beam);
      uint32_t h = h0;
      if (!first && pass) h = part_find(T, e.dst);
      const bool win = pass && T.hval[h] == (((uint64_t)f2ord(e.cost) << 32) | e.arc);
      const unsigned long long wm = __ballot(win);
      if (wm == 0) continue;   // uniform
      bool surv = false;
      const int idx = token_places(wm);
      if (win) surv = write_token(idx, h, e.dst, e.cost, e.arc, row_of(p, p.arcs[e.arc]), base_prev + (int)(e.from & kPartMask));
      w_surv += (int)__popcll(__ballot(surv));
    }
    for (int base = wave * 64; base < n2; base += kBlock) {   // uniform
      const int i = base + lane;
      bool win = false, surv = false;
      uint32_t h = 0;
      PartEntry e; e.dst = 0; e.cost = 0.0f; e.arc = 0; e.from = 0;
      if (i < n2) {
        e = q2[i];
        h = part_find(T, e.dst);
        const uint64_t key = ((uint64_t)f2ord(e.cost) << 32) | e.arc;
        win = T.hval[h] == key &&
              atomicCAS((unsigned long long *)&T.hval[h], (unsigned long long)key, (unsigned long long)kEmptyVal) == key;
      }
      const unsigned long long wm = __ballot(win);
      const int idx = wm ? token_places(wm) : 0;
      // (its predecessor follows in step 4)
      if (win) surv = write_token(idx, h, e.dst, e.cost, e.arc, row_of(p, p.arcs[e.arc]), -1);
      if (i < n2) q2[i].arc = win ? (uint32_t)idx : kArcNone;
      w_surv += (int)__popcll(__ballot(surv));
    }
    for_long_arcs(o, [&](const LongArc (&l)[4], const int (&at)[4], const bool (&pass)[4], const float (&cand)[4], int src) {   // (costed once more: the same bits)
      bool win[4];
      int n = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        win[u] = pass[u] && T.hval[l[u].slot_pdf & 0xFFFFu] == (((uint64_t)f2ord(cand[u]) << 32) | l[u].arc);
        n += (int)__popcll(__ballot(win[u]));
      }
      if (n == 0) return;   // uniform
      int first = 0;
      if (lane == 0) first = atomicAdd(n_made, n);
      uint32_t meta[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) meta[u] = p.lr.meta[at[u]];
      first = __builtin_amdgcn_readfirstlane(first);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t h = l[u].slot_pdf & 0xFFFFu;
        const unsigned long long wm = __ballot(win[u]);
        bool surv = false;
        if (win[u]) {
          ArcRec rec;
          rec.dst = (int32_t)T.hkey[h]; rec.weight = 0.0f; rec.row = l[u].row; rec.meta = meta[u];
          surv = write_token(first + (int)__popcll(wm & ((1ull << lane) - 1ull)), h, (uint32_t)rec.dst, cand[u], l[u].arc, row_of(p, rec), base_prev + src);
        }
        first += (int)__popcll(wm);
        w_surv += (int)__popcll(__ballot(surv));
      }
    });
    __syncthreads();
    CBD_STAMP(5);   // (diagnostic: winners)
    if (have_closures) {   // (uniform) which token the state of an entry with a closure list has become
      for (int i = tid; i < n1; i += kBlock) {
        const PartEntry e = q1[i];
        if ((e.from & kPartHasList) && !(e.cost - m > p.beam))
          q1[i].cost = __uint_as_float((uint32_t)T.hval[part_find(T, e.dst)]);
      }
      for (int i = tid; i < n2; i += kBlock) {
        const PartEntry e = q2[i];
        if (e.from & kPartHasList) q2[i].cost = __uint_as_float((uint32_t)T.hval[part_find(T, e.dst)]);
      }
      __syncthreads();
    }
  }

  CBD_STAMP(6);   // (diagnostic: entries' tokens)
  // ---- 4: predecessors of closure winners
  if (have_closures) {
    for (int o = 0; o < k; ++o) {
      const int n2 = min(cnt2[o], cap2);
      for (int i = tid; i < n2; i += kBlock) {
        const PartEntry e = Q2[o * cap2 + i];
        if (e.arc == kArcNone || (int)e.arc >= p.g_tok_cap || base_cur + (int)e.arc >= p.bp_cap) continue;
        bp[base_cur + (int)e.arc].y = base_cur + (int)__float_as_uint(Q1[e.from & kPartMask].cost);
      }
    }
  }
  if (lane == 0 && w_surv) atomicAdd(&sh->n_surv, w_surv);
  __syncthreads();
  const int n_claim = *n_made;
  if (n_claim > p.g_tok_cap) return kFrameOverflow;
  if (base_cur + n_claim > p.bp_cap) return kFrameRecordsFull;
  if (lane == 0) {
    if (n_active) atomicAdd(&sh->a_active, (unsigned long long)n_active);
    if (n_emit) atomicAdd(&sh->a_emit, (unsigned long long)n_emit);
    if (n_eps) atomicAdd(&sh->a_eps, (unsigned long long)n_eps);
    if (n_cand) atomicAdd(&sh->a_cand, (unsigned long long)n_cand);
    if (max_depth) atomicMax(&sh->rounds, max_depth);
  }
  if (Lnext) for (int i = tid; i < p.num_pdfs; i += kBlock) Lstage[i] = Lnext[i];   // (this frame's row has been read)
  __syncthreads();
  if (wave == 0) {
    int cutb = 255;
    if (hist_on && n_claim > p.max_active && sh->n_surv > p.max_active) {
      // largest bin whose cumulative count fits max_active (0 if bin 0 alone does not)
      int loc[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) { loc[q] = (int)hist[lane * 4 + q]; sum += loc[q]; }
      int run = wave_incl_scan(sum) - sum;
      int myB = -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) { run += loc[q]; if (run <= p.max_active) myB = lane * 4 + q; }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) { const int t = __shfl_xor(myB, d, 64); myB = t > myB ? t : myB; }
      cutb = myB < 0 ? 0 : myB;
    }
    if (lane == 0) {
      sh->cut_bin = cutb;
      sh->n_tok = n_claim;
      sh->frame_base = base_cur;
      sh->n_rec = base_cur + n_claim;
      sh->best = fbest;
      atomicAdd(&sh->a_frames, kPartsCount + 1ull);
      atomicAdd(&sh->a_tokens, (unsigned long long)n_claim);
      atomicMax(&sh->a_maxtok, n_claim);
      atomicAdd(&sh->a_slow, 1);
      atomicAdd(&sh->a_impr, (unsigned long long)n_claim);
      atomicAdd(&sh->a_rounds, (unsigned long long)sh->rounds);
    }
    frame_init(sh, hist, false, lane, hist_on);   // for the next frame
  }
  __syncthreads();
  CBD_STAMP(7);   // (diagnostic: closure winners' records, next row, close)
  return kFrameOk;
}

}  // namespace cbd
