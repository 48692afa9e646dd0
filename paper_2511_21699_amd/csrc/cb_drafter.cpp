// Host-side drafter of Cacheback decoding: the leader -> follower cache table with LRU eviction in
// both domains (Section 3.1 of the paper) and the breadth-first growth of the draft-token tree
// (Section 3.2), behind the C ABI of cacheback_drafter.h.  Serial host code, no GPU involved.
//
// Table layout: leaders live in `lc` fixed slots; a hash index maps a leader's tokens to its slot;
// the slots form a doubly linked list in recency order (index links, head = least recent).  Each
// slot owns `fc` follower cells and a small array naming the cells oldest first, so that both LRU
// domains are updated with a few moves.  Nothing is allocated after a table's creation: the index is an
// open-addressed array at most half full.
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "cacheback.h"
#include "cacheback_drafter.h"

namespace {

uint32_t hash_tokens(const int32_t* p, int32_t n, uint64_t h = 0) {
  for (int32_t i = 0; i < n; i++) {  // multiplicative hashing (golden ratio), the high half folded in
    h = (h ^ (uint32_t)p[i]) * 0x9e3779b97f4a7c15ull;
    h ^= h >> 32;
  }
  return (uint32_t)h;
}
bool same_tokens(const int32_t* a, const int32_t* b, int32_t n) {  // (sequences are short: no call)
  for (int32_t i = 0; i < n; i++)
    if (a[i] != b[i]) return false;
  return true;
}

// Open-addressed index from token sequences to numbers, linear probing.  It keeps hashes and numbers; the sequences
// themselves stay with the caller, who compares them (`same`: whether a number's sequence is the one looked for).
struct TokenIndex {
  struct Cell {
    uint32_t hash;
    int32_t id;  // -1: empty
  };
  std::vector<Cell> cells;  // a power of two
  size_t mask = 0;

  void create(size_t most) {  // room for `most` entries at half load
    size_t n = 16;
    while (n < 2 * most) n *= 2;
    cells.assign(n, Cell{0, -1});
    mask = n - 1;
  }
  template <typename Same>
  size_t place(uint32_t h, Same same) const {  // the entry's cell, or the empty one it would go to
    size_t i = h & mask;
    while (cells[i].id >= 0 && !(cells[i].hash == h && same(cells[i].id))) i = (i + 1) & mask;
    return i;
  }
  void erase_at(size_t i) {  // the entries behind move up, so that no probe is cut short
    for (size_t j = (i + 1) & mask; cells[j].id >= 0; j = (j + 1) & mask) {
      if (((j - (cells[j].hash & mask)) & mask) >= ((j - i) & mask)) {
        cells[i] = cells[j];
        i = j;
      }
    }
    cells[i].id = -1;
  }
};

}  // namespace

struct cbd_table {
  int32_t ll, fl, lc, fc;
  bool frozen = false;
  std::vector<int32_t> key;    // [lc][ll] leader tokens
  std::vector<int32_t> prev, next;  // recency list over used slots
  int32_t head = -1, tail = -1;     // least / most recent leader
  std::vector<int32_t> nfol;   // followers held per slot
  std::vector<uint8_t> order;  // [lc][fc] follower cells, oldest first
  std::vector<int32_t> ftok;   // [lc][fc][fl] follower tokens
  int32_t used = 0;            // slots 0 .. used-1 have been handed out (none is ever returned: a full table evicts)
  int64_t followers = 0;
  TokenIndex index;            // leader tokens -> slot

  void unlink(int32_t s) {
    if (prev[s] >= 0) next[prev[s]] = next[s]; else head = next[s];
    if (next[s] >= 0) prev[next[s]] = prev[s]; else tail = prev[s];
  }
  void push_recent(int32_t s) {
    prev[s] = tail;
    next[s] = -1;
    if (tail >= 0) next[tail] = s; else head = s;
    tail = s;
  }
  void touch(int32_t s) {
    if (tail == s) return;
    unlink(s);
    push_recent(s);
  }
  size_t place(const int32_t* leader, uint32_t h) const {
    return index.place(h, [&](int32_t s) { return same_tokens(&key[(size_t)s * ll], leader, ll); });
  }
  int32_t find(const int32_t* leader) const { return index.cells[place(leader, hash_tokens(leader, ll))].id; }
};

namespace {

// The tree under construction.  A node's children are a linked list.
struct Tree {
  int32_t* parent;
  int32_t* token;
  int32_t* depth;
  int32_t* first;  // first child, -1: none
  int32_t* next;   // next sibling, -1: none
  int32_t n = 0;
  int32_t child(int32_t node, int32_t tk) const {
    for (int32_t c = first[node]; c >= 0; c = next[c])
      if (token[c] == tk) return c;
    return -1;
  }
  int32_t add(int32_t par, int32_t tk) {
    const int32_t id = n++;
    parent[id] = par;
    token[id] = tk;
    depth[id] = par < 0 ? 0 : depth[par] + 1;
    first[id] = next[id] = -1;
    if (par >= 0) {
      next[id] = first[par];
      first[par] = id;
    }
    return id;
  }
};

// Last `need` tokens of the root path of `node`, continued back into the context before the root
// token; returns how many there are (fewer than `need` when the context is too short).
int32_t path_tokens(const Tree& t, int32_t node, int32_t need, const int32_t* context, int64_t n_ctx, int32_t* out) {
  int32_t got = 0;
  int32_t tmp[16];
  for (int32_t x = node; x >= 0 && got < need; x = t.parent[x]) tmp[got++] = t.token[x];
  const int64_t before_root = n_ctx - 1;
  const int32_t extra = (int32_t)std::min<int64_t>(need - got, before_root);
  int32_t k = 0;
  for (int32_t i = 0; i < extra; i++) out[k++] = context[before_root - extra + i];
  for (int32_t i = got - 1; i >= 0; i--) out[k++] = tmp[i];
  return k;
}

}  // namespace

extern "C" {

int cbd_table_create(int32_t ll, int32_t fl, int32_t lc, int32_t fc, cbd_table** out) {
  if (!out || ll < 1 || fl < 1 || lc < 1 || fc < 1 || ll > 16 || fl > 16 || fc > 64) return CB_EINVAL;
  cbd_table* t = new (std::nothrow) cbd_table();
  if (!t) return CB_EINVAL;
  t->ll = ll; t->fl = fl; t->lc = lc; t->fc = fc;
  t->key.assign((size_t)lc * ll, 0);
  t->prev.assign(lc, -1);
  t->next.assign(lc, -1);
  t->nfol.assign(lc, 0);
  t->order.assign((size_t)lc * fc, 0);
  t->ftok.assign((size_t)lc * fc * fl, 0);
  t->index.create((size_t)lc);
  *out = t;
  return CB_OK;
}

void cbd_table_destroy(cbd_table* t) { delete t; }

int cbd_table_insert(cbd_table* t, const int32_t* leader, const int32_t* follower) {
  if (!t || !leader || !follower) return CB_EINVAL;
  if (t->frozen) return CB_OK;
  const int32_t ll = t->ll, fl = t->fl, fc = t->fc;
  const uint32_t h = hash_tokens(leader, ll);
  size_t at = t->place(leader, h);
  int32_t s = t->index.cells[at].id;
  if (s < 0) {
    if (t->used < t->lc) {
      s = t->used++;
    } else {  // evict the least recently used leader with all its followers
      s = t->head;
      const int32_t* old = &t->key[(size_t)s * ll];
      t->index.erase_at(t->place(old, hash_tokens(old, ll)));
      at = t->place(leader, h);  // (the cells may have moved)
      t->unlink(s);
      t->followers -= t->nfol[s];
    }
    memcpy(&t->key[(size_t)s * ll], leader, (size_t)ll * 4);
    t->index.cells[at] = TokenIndex::Cell{h, s};
    t->push_recent(s);
    t->nfol[s] = 1;
    t->order[(size_t)s * fc] = 0;
    memcpy(&t->ftok[(size_t)s * fc * fl], follower, (size_t)fl * 4);
    t->followers += 1;
    return CB_OK;
  }
  t->touch(s);  // inserting refreshes the leader
  uint8_t* ord = &t->order[(size_t)s * fc];
  int32_t* cells = &t->ftok[(size_t)s * fc * fl];
  const int32_t n = t->nfol[s];
  for (int32_t i = 0; i < n; i++) {
    if (same_tokens(&cells[(size_t)ord[i] * fl], follower, fl)) {  // present: becomes the most recent
      const uint8_t c = ord[i];
      memmove(ord + i, ord + i + 1, (size_t)(n - 1 - i));
      ord[n - 1] = c;
      return CB_OK;
    }
  }
  uint8_t cell;
  if (n < fc) {
    cell = (uint8_t)n;  // cells fill up in order; they are only recycled once all are in use
    t->nfol[s] = n + 1;
    t->followers += 1;
    ord[n] = cell;
  } else {  // evict this leader's least recent follower
    cell = ord[0];
    memmove(ord, ord + 1, (size_t)(n - 1));
    ord[n - 1] = cell;
  }
  memcpy(&cells[(size_t)cell * fl], follower, (size_t)fl * 4);
  return CB_OK;
}

int cbd_table_update(cbd_table* t, const int32_t* tokens, int64_t n, int64_t start) {
  if (!t || (!tokens && n > 0) || n < 0) return CB_EINVAL;
  for (int64_t i = std::max<int64_t>(t->ll, start); i + t->fl <= n; i++) {
    const int rc = cbd_table_insert(t, tokens + i - t->ll, tokens + i);
    if (rc) return rc;
  }
  return CB_OK;
}

int cbd_table_query(cbd_table* t, const int32_t* leader, int32_t refresh, int32_t* followers, int32_t* count) {
  if (!t || !leader || !followers || !count) return CB_EINVAL;
  *count = 0;
  const int32_t s = t->find(leader);
  if (s < 0) return CB_OK;
  if (refresh && !t->frozen) t->touch(s);
  const int32_t n = t->nfol[s], fl = t->fl;
  const uint8_t* ord = &t->order[(size_t)s * t->fc];
  const int32_t* cells = &t->ftok[(size_t)s * t->fc * fl];
  for (int32_t i = 0; i < n; i++) memcpy(followers + (size_t)i * fl, &cells[(size_t)ord[n - 1 - i] * fl], (size_t)fl * 4);
  *count = n;
  return CB_OK;
}

int cbd_table_build_frozen(int32_t ll, int32_t fl, int32_t lc, int32_t fc, const int32_t* tokens, int64_t n,
                           cbd_table** out) {
  if (!out || (!tokens && n > 0) || n < 0) return CB_EINVAL;
  cbd_table* t = nullptr;
  const int rc = cbd_table_create(ll, fl, lc, fc, &t);
  if (rc) return rc;
  // Distinct leaders, and distinct (leader, follower) pairs, numbered in order of their first window, with counts.
  struct Pair {
    int64_t first, count;  // first window
    int32_t leader, next;  // next: the pair of the same leader found before this one, -1: none
  };
  struct Leader {
    int64_t first, count;
    int32_t pairs;  // its pair found last
  };
  const int64_t windows = std::max<int64_t>(0, n - ll - fl + 1);
  if (windows >= INT32_MAX) { delete t; return CB_EINVAL; }
  std::vector<Leader> leaders;
  std::vector<Pair> pairs;
  TokenIndex by_leader, by_pair;
  by_leader.create((size_t)windows);
  by_pair.create((size_t)windows);
  for (int64_t i = ll; i + fl <= n; i++) {
    const uint32_t hl = hash_tokens(tokens + i - ll, ll);
    const size_t at = by_leader.place(hl, [&](int32_t x) { return same_tokens(tokens + leaders[x].first - ll, tokens + i - ll, ll); });
    int32_t le = by_leader.cells[at].id;
    if (le < 0) {
      le = (int32_t)leaders.size();
      leaders.push_back(Leader{i, 0, -1});
      by_leader.cells[at] = TokenIndex::Cell{hl, le};
    }
    leaders[le].count++;
    const uint32_t hp = hash_tokens(tokens + i, fl, hl);
    const size_t pt = by_pair.place(hp, [&](int32_t x) { return pairs[x].leader == le && same_tokens(tokens + pairs[x].first, tokens + i, fl); });
    int32_t pa = by_pair.cells[pt].id;
    if (pa < 0) {
      pa = (int32_t)pairs.size();
      pairs.push_back(Pair{i, 0, le, leaders[le].pairs});
      leaders[le].pairs = pa;
      by_pair.cells[pt] = TokenIndex::Cell{hp, pa};
    }
    pairs[pa].count++;
  }
  // more frequent first, then earlier first window (which is the lower number)
  std::vector<int32_t> top(leaders.size());
  for (size_t i = 0; i < top.size(); i++) top[i] = (int32_t)i;
  const size_t keep = std::min(top.size(), (size_t)lc);
  std::partial_sort(top.begin(), top.begin() + keep, top.end(), [&](int32_t a, int32_t b) {
    return leaders[a].count != leaders[b].count ? leaders[a].count > leaders[b].count : a < b;
  });
  std::vector<int32_t> fols;
  for (size_t r = keep; r-- > 0;) {  // least frequent leader first (recency is irrelevant once frozen)
    const Leader& le = leaders[top[r]];
    fols.clear();
    for (int32_t x = le.pairs; x >= 0; x = pairs[x].next) fols.push_back(x);
    std::sort(fols.begin(), fols.end(), [&](int32_t a, int32_t b) {
      return pairs[a].count != pairs[b].count ? pairs[a].count > pairs[b].count : a < b;
    });
    if ((int64_t)fols.size() > fc) fols.resize((size_t)fc);
    for (size_t k = fols.size(); k-- > 0;)  // least frequent follower first: the most frequent ends up most recent
      cbd_table_insert(t, tokens + le.first - ll, tokens + pairs[fols[k]].first);
  }
  t->frozen = true;
  *out = t;
  return CB_OK;
}

int cbd_table_freeze(cbd_table* t) {
  if (!t) return CB_EINVAL;
  t->frozen = true;
  return CB_OK;
}

int cbd_table_size(const cbd_table* t, int64_t* leaders, int64_t* followers) {
  if (!t || !leaders || !followers) return CB_EINVAL;
  *leaders = t->used;
  *followers = t->followers;
  return CB_OK;
}

int cbd_grow_tree(cbd_table* const* tables, int32_t num_tables, const int32_t* context, int64_t n_ctx,
                  int32_t node_budget, int32_t depth_cap, int32_t crt, int32_t* parent, int32_t* token,
                  int32_t* depth, int32_t* n_nodes) {
  if (!tables || num_tables < 0 || !context || n_ctx < 1 || node_budget < 1 || depth_cap < 0 || crt < 0 || !parent ||
      !token || !depth || !n_nodes)
    return CB_EINVAL;
  for (int32_t i = 0; i < num_tables; i++)
    if (!tables[i]) return CB_EINVAL;
  Tree tr;
  tr.parent = parent;
  tr.token = token;
  tr.depth = depth;
  std::vector<int32_t> scratch((size_t)node_budget * 5);  // (one allocation; every list holds a node at most once)
  tr.first = scratch.data();
  tr.next = tr.first + node_budget;
  int32_t* const leaves = tr.next + node_budget;
  int32_t* const grown = leaves + node_budget;
  int32_t* const seen = grown + node_budget;  // round in which a node was listed as a new leaf (0: never)
  int32_t n_leaves = 0, n_grown = 0;
  tr.add(-1, context[n_ctx - 1]);
  int32_t key[16];
  int32_t round_id = 0;
  for (int32_t ti = 0; ti < num_tables; ti++) {
    cbd_table* tb = tables[ti];
    const int32_t ll = tb->ll, fl = tb->fl;
    n_leaves = 0;
    for (int32_t i = 0; i < tr.n; i++)
      if (tr.first[i] < 0) leaves[n_leaves++] = i;
    bool first_round = true;
    while (n_leaves > 0 && tr.n < node_budget) {
      // the chaining-reserved tokens keep part of the budget for the second and deeper rounds
      int32_t limit = (first_round && crt > 0) ? node_budget - crt : node_budget;
      limit = std::max(limit, std::min(node_budget, tr.n + 1));
      n_grown = 0;
      round_id++;
      for (int32_t li = 0; li < n_leaves; li++) {
        const int32_t leaf = leaves[li];
        if (tr.n >= limit) break;
        if (path_tokens(tr, leaf, ll, context, n_ctx, key) < ll) continue;
        const int32_t s = tb->find(key);
        if (s < 0) continue;
        if (!tb->frozen) tb->touch(s);
        const uint8_t* const ord = &tb->order[(size_t)s * tb->fc];
        for (int32_t f = tb->nfol[s] - 1; f >= 0; f--) {  // most recent first
          const int32_t* const fol = &tb->ftok[((size_t)s * tb->fc + ord[f]) * fl];
          int32_t node = leaf;
          for (int32_t j = 0; j < fl; j++) {
            if (tr.depth[node] >= depth_cap) break;
            const int32_t tk = fol[j];
            int32_t nxt = tr.child(node, tk);
            if (nxt < 0) {  // followers that share a prefix share the nodes
              if (tr.n >= limit) break;
              nxt = tr.add(node, tk);
            }
            node = nxt;
          }
          if (node != leaf && tr.first[node] < 0 && seen[node] != round_id) {
            seen[node] = round_id;
            grown[n_grown++] = node;
          }
        }
      }
      n_leaves = 0;
      for (int32_t i = 0; i < n_grown; i++)
        if (tr.first[grown[i]] < 0) leaves[n_leaves++] = grown[i];
      first_round = false;
    }
  }
  *n_nodes = tr.n;
  return CB_OK;
}

}  // extern "C"
