// Host planner: head ranking (Eq. 3-4), budget rule (Eq. 5), removal-order
// optimisation (Alg. 1 with the cache accounting of Alg. 2 / App. A), and the
// static memory layout the kernels run on.  Pure integer work apart from the
// fp64 sums that rank the heads.  No HIP calls in this file.
#include "plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

namespace heatkv {

static thread_local std::string g_last_error;

void set_error(const std::string& msg) { g_last_error = msg; }
int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}
const char* last_error_cstr() { return g_last_error.c_str(); }

int check_shape(const heatkv_shape* s) {
  if (!s) return fail(HEATKV_EINVAL, "shape is null");
  if (!s->t) return fail(HEATKV_EINVAL, "shape.t is null");
  if (s->L < 1 || s->H < 1 || s->batch < 1) return fail(HEATKV_EINVAL, "L, H, batch must be >= 1");
  if (s->K < 1 || s->K > HEATKV_MAX_SCALES) return fail(HEATKV_EINVAL, "K out of range");
  if (s->dtype != HEATKV_F32 && s->dtype != HEATKV_BF16) return fail(HEATKV_EINVAL, "unknown dtype");
  if (s->d != 64 && s->d != 128) return fail(HEATKV_EINVAL, "head dimension must be 64 or 128");
  int64_t total = 0;
  for (int k = 0; k < s->K; ++k) {
    if (s->t[k] < 1) return fail(HEATKV_EINVAL, "t[k] must be >= 1");
    total += s->t[k];
  }
  if (total * s->H > (int64_t(1) << 30)) return fail(HEATKV_EINVAL, "sequence too long");
  return HEATKV_OK;
}

int init_shape(heatkv_plan* p, const heatkv_shape* s) {
  int rc = check_shape(s);
  if (rc) return rc;
  p->L = s->L;
  p->H = s->H;
  p->d = s->d;
  p->K = s->K;
  p->batch = s->batch;
  p->dtype = s->dtype;
  p->T = s->L * s->H;
  p->t.assign(s->t, s->t + s->K);
  p->c.resize(s->K);
  int32_t acc = 0;
  for (int k = 0; k < s->K; ++k) {
    acc += p->t[k];
    p->c[k] = acc;
  }
  return HEATKV_OK;
}

namespace {

// Bits of a double as an unsigned number that orders like the double (no distinction between the zeros).
uint64_t order_bits(double x) {
  uint64_t u;
  x += 0.0;
  std::memcpy(&u, &x, sizeof u);
  return u ^ (u >> 63 ? ~uint64_t(0) : uint64_t(1) << 63);
}

// Sorts `n` heads, given in the order of their ids (ALL: all of them), by key, then id; x, y: scratch of n each.  From a few
// hundred on a radix sort on the upper 22 bits of the range that the keys span, then the same for every run of ties of those
// bits; 8 bits where there are fewer.  No branch depends on the keys but for the ties, of which there are many where one score
// lies far from the others (a head without mass on a scale).  Scores spread over 0.1 %: 1280 heads 9.8 us, with one head at
// zero 19.5 (runs of ties sorted by comparison: 20.2), 10240 heads 136 and 215 (539).
constexpr size_t RADIX_MIN = 256;
template <bool ALL>
void sort_heads(int32_t* order, size_t n, const uint64_t* key, uint64_t* x, uint64_t* y) {
  if (n <= 16) {
    for (size_t k = 1; k < n; ++k) {
      const int32_t it = order[k];
      size_t j = k;
      for (; j > 0 && key[order[j - 1]] > key[it]; --j) order[j] = order[j - 1];
      order[j] = it;
    }
    return;
  }
  auto head = [&](size_t i) { return ALL ? uint32_t(i) : uint32_t(order[i]); };
  uint64_t least = ~uint64_t(0), most = 0;
  for (size_t i = 0; i < n; ++i) {
    least = std::min(least, key[head(i)]);
    most = std::max(most, key[head(i)]);
  }
  if (least == most) return;
  const int range = 64 - __builtin_clzll(most - least);
  int shift;
  if (n < RADIX_MIN) {
    constexpr int BITS = 8, DIGITS = 1 << BITS;
    shift = std::max(0, range - BITS);
    uint32_t first[DIGITS + 1] = {};
    for (size_t i = 0; i < n; ++i) {
      const uint64_t q = (key[head(i)] - least) >> shift;
      y[i] = q << 32 | head(i);  // digits above bit 32, head below
      ++first[q + 1];
    }
    for (int v = 0; v < DIGITS; ++v) first[v + 1] += first[v];
    for (size_t i = 0; i < n; ++i) x[first[y[i] >> 32]++] = y[i];
  } else {
    constexpr int BITS = 11, DIGITS = 1 << BITS;
    shift = std::max(0, range - 2 * BITS);
    uint32_t low[DIGITS] = {}, high[DIGITS] = {};
    for (size_t i = 0; i < n; ++i) {
      const uint64_t q = (key[head(i)] - least) >> shift;
      x[i] = q << 32 | head(i);
      ++low[q & (DIGITS - 1)];
      ++high[q >> BITS];
    }
    uint32_t a = 0, b = 0;
    for (int v = 0; v < DIGITS; ++v) {
      const uint32_t la = low[v], hb = high[v];
      low[v] = a;
      high[v] = b;
      a += la;
      b += hb;
    }
    for (size_t i = 0; i < n; ++i) y[low[x[i] >> 32 & (DIGITS - 1)]++] = x[i];
    for (size_t i = 0; i < n; ++i) x[high[y[i] >> (32 + BITS)]++] = y[i];
  }
  for (size_t i = 0; i < n; ++i) order[i] = int32_t(uint32_t(x[i]));
  if (shift == 0) return;
  for (size_t i = 0, end; i < n; i = end) {
    for (end = i + 1; end < n && x[end] >> 32 == x[i] >> 32; ++end) {}
    if (end - i > 1) sort_heads<false>(order + i, end - i, key, x + i, y + i);
  }
}

// Stable ascending order of the heads by an fp64 score; ties keep the flat head id order.
std::vector<int32_t> rank_heads(const std::vector<double>& score) {
  const size_t n = score.size();
  std::vector<int32_t> order(n);
  if (n < RADIX_MIN) {
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return score[a] < score[b]; });
    return order;
  }
  std::vector<uint64_t, UnclearedAllocator<uint64_t>> key(n), x(n), y(n);
  for (size_t i = 0; i < n; ++i) key[i] = order_bits(score[i]);
  std::iota(order.begin(), order.end(), 0);
  sort_heads<true>(order.data(), n, key.data(), x.data(), y.data());
  return order;
}

// Head scores that the orders are built from: score[i][head] for source scale i in [s, K-1), the
// un-normalised sums of Eq. 4 (scale-dependent) or Eq. 3 (binary: the same sum for every i); fp64, tau ascending.
// One pass over a head's table, row by row.
void head_scores(int K, int T, int s, bool binary, const float* beta, std::vector<std::vector<double>>& score) {
  score.assign(K, {});
  for (int i = s; i < K - 1; ++i) score[i].resize(T);
  for (int head = 0; head < T; ++head) {
    const float* b = beta + size_t(head) * K * K;
    double sum[HEATKV_MAX_SCALES] = {};
    if (binary) {
      double sc = 0.0;
      for (int tau = s; tau < K - 1; ++tau) sc += double(b[size_t(K - 1) * K + tau]);
      std::fill(sum + s, sum + std::max(s, K - 1), sc);
    } else {
      for (int tau = s + 1; tau < K; ++tau) {
        const float* r = b + size_t(tau) * K;
        int i = s;
        for (; i + 4 <= tau; i += 4) {
          sum[i] += double(r[i]);
          sum[i + 1] += double(r[i + 1]);
          sum[i + 2] += double(r[i + 2]);
          sum[i + 3] += double(r[i + 3]);
        }
        for (; i < tau; ++i) sum[i] += double(r[i]);
      }
    }
    for (int i = s; i < K - 1; ++i) score[i][head] = sum[i];
  }
}

struct Candidate {
  int32_t layer, scale, head;
};

}  // namespace

int build_sets(heatkv_plan* p, const float* beta) {
  const int K = p->K, L = p->L, H = p->H, T = p->T, s = p->sinks;
  const bool binary = (p->variant & 1) != 0, naive = (p->variant & 2) != 0;
  const int64_t cs = s > 0 ? p->c[s - 1] : 0;
  const int64_t B = p->B;

  // Eq. 5 in integers.  With B >= T c_s, N_k does not decrease with k: T - N_k = floor((B - T c_s) / (c_k - c_s)).
  p->N.assign(K > 1 ? K - 1 : 0, 0);
  for (int k = s; k < K - 1; ++k) {
    const int64_t num = int64_t(T) * p->c[k] - B, den = p->c[k] - cs;
    int64_t n = num <= 0 ? 0 : (num + den - 1) / den;
    if (n > T) return fail(HEATKV_EBUDGET, "budget is smaller than the sink scales of all heads");
    p->N[k] = int32_t(n);
  }
  if (B < int64_t(T) * cs) return fail(HEATKV_EBUDGET, "budget is smaller than the sink scales of all heads");

  // Orders.  beta[l][h][k1][k2]; sums in fp64, tau ascending.
  std::vector<std::vector<double>> score;
  head_scores(K, T, s, binary, beta, score);
  p->orders.assign(K, {});
  for (int i = s; i < K - 1; ++i) {
    if (binary && i > s) p->orders[i] = p->orders[s];
    else p->orders[i] = rank_heads(score[i]);
  }

  p->G.assign(size_t(K) * T, 0);
  p->E.assign(size_t(K) * T, 0);
  p->A.assign(size_t(K) * T, 0);
  const uint32_t all = K - 1 > s ? (1u << (K - 1)) - (1u << s) : 0u;  // source scales that can be pruned
  std::vector<int32_t> layer_of(T);
  for (int head = 0; head < T; ++head) layer_of[head] = head / H;

  // Cache size per layer: `done` with G_k applied (layers that have run), `todo` with only G_{k-1} applied (layers still
  // to run; early removals lower it).  Both follow from the step before: scale k enters, the newly pruned leave.
  std::vector<int64_t> done(L, int64_t(H) * cs), todo(L);
  std::vector<int32_t> whole(L, H);  // binary: heads of the layer that G_{k-1} leaves whole
  std::vector<int32_t> layer_end(L);
  std::vector<Candidate> cand, unsorted;
  for (int k = 0; k < K - 1; ++k) {
    // G_k: prefix of length N_k of every order O_i, i <= k (binary: of the one order, all scales).  What is new against
    // G_{k-1}, a shorter prefix, can be removed early.
    const int32_t n = p->N[k], n_before = k > s ? p->N[k - 1] : 0;
    unsorted.clear();
    uint32_t* g = &p->G[size_t(k) * T];
    if (k > 0) std::memcpy(g, g - T, T * sizeof(uint32_t));
    // Tokens that an early removal takes out of a layer that has not run.
    auto weight = [&](const Candidate& c) { return binary ? int64_t(p->c[k]) - cs : int64_t(p->t[c.scale]); };
    if (k >= s && binary) {
      for (int r = n_before; r < n; ++r) {
        const int head = p->orders[s][r];
        g[head] = all;
        unsorted.push_back({layer_of[head], 0, head});
      }
    } else if (k >= s) {
      for (int i = k; i >= s; --i)
        for (int r = i < k ? n_before : 0; r < n; ++r) {
          const int head = p->orders[i][r];
          g[head] |= 1u << i;
          unsorted.push_back({layer_of[head], i, head});
        }
    }
    for (int l = 0; l < L; ++l) {
      todo[l] = done[l] + (k < s ? 0 : int64_t(binary ? whole[l] : H) * p->t[k]);
      done[l] = todo[l];
    }
    for (const Candidate& c : unsorted) done[c.layer] -= weight(c);
    if (binary)
      for (const Candidate& c : unsorted) --whole[c.layer];

    // Removal order: last layer first, then newest source scale, then rank.  The list has the latter two already.
    std::fill(layer_end.begin(), layer_end.end(), 0);
    for (const Candidate& c : unsorted) ++layer_end[c.layer];
    for (int l = L - 1, at = 0; l >= 0; --l) {
      const int here = layer_end[l];
      layer_end[l] = at;
      at += here;
    }
    cand.resize(unsorted.size());
    for (const Candidate& c : unsorted) cand[layer_end[c.layer]++] = c;

    size_t next = 0;
    auto pop = [&]() {
      const Candidate& cd = cand[next++];
      p->E[size_t(k) * T + cd.head] |= binary ? all : 1u << cd.scale;
      todo[cd.layer] -= weight(cd);
      return cd.layer;
    };
    if (naive) {
      while (next < cand.size()) pop();
    }
    // M: layers up to l have run, the others have not.
    int64_t M = std::accumulate(todo.begin(), todo.end(), int64_t(0));
    for (int l = 0; l < L; ++l) {
      M += done[l] - todo[l];
      while (M > B) {
        if (next >= cand.size()) return fail(HEATKV_EBUDGET, "early pruning cannot reach the budget");
        const int64_t w = weight(cand[next]);
        if (pop() > l) M -= w;
      }
    }
    // A_k = G_{k-1} u E_k
    uint32_t* a = &p->A[size_t(k) * T];
    const uint32_t* e = &p->E[size_t(k) * T];
    for (int head = 0; head < T; ++head) a[head] = k > 0 ? g[head - T] | e[head] : e[head];
  }
  // Last scale: nothing is appended any more, so only the removals already decided apply.
  if (K >= 2) std::memcpy(&p->A[size_t(K - 1) * T], &p->G[size_t(K - 2) * T], T * sizeof(uint32_t));

  p->retained.resize(size_t(K) * T);
  for (int k = 0; k < K; ++k)
    for (int head = 0; head < T; ++head)
      p->retained[size_t(k) * T + head] = ((1u << k) - 1u) & ~p->A[size_t(k) * T + head];
  return HEATKV_OK;
}

int rank_scores(const heatkv_shape* shape, const float* beta, int sinks, int variant, double* scores) {
  int rc = check_shape(shape);
  if (rc) return rc;
  if (!beta || !scores) return fail(HEATKV_EINVAL, "null pointer");
  const int K = shape->K, T = shape->L * shape->H;
  if (sinks < 0 || sinks > K - 2) return fail(HEATKV_EINVAL, "sinks out of range");
  if (variant < 0 || variant > 3) return fail(HEATKV_EINVAL, "unknown variant");
  std::vector<std::vector<double>> score;
  head_scores(K, T, sinks, (variant & 1) != 0, beta, score);
  for (int i = 0; i < K; ++i)
    for (int head = 0; head < T; ++head) scores[size_t(i) * T + head] = score[i].empty() ? 0.0 : score[i][head];
  return HEATKV_OK;
}

int rank_dispersion(const heatkv_shape* shape, const float* betas, int runs, int sinks, int variant,
                    double* dispersion) {
  int rc = check_shape(shape);
  if (rc) return rc;
  if (!betas || !dispersion) return fail(HEATKV_EINVAL, "null pointer");
  if (runs < 1) return fail(HEATKV_EINVAL, "runs must be >= 1");
  const int K = shape->K, T = shape->L * shape->H;
  if (sinks < 0 || sinks > K - 2) return fail(HEATKV_EINVAL, "sinks out of range");
  if (variant < 0 || variant > 3) return fail(HEATKV_EINVAL, "unknown variant");
  const bool binary = (variant & 1) != 0;
  const size_t table = size_t(T) * K * K;
  // pos[i][run][head] = rank position of the head in that run's order O_i
  std::vector<std::vector<int32_t>> pos(K);
  for (int r = 0; r < runs; ++r) {
    std::vector<std::vector<double>> score;
    head_scores(K, T, sinks, binary, betas + size_t(r) * table, score);
    std::vector<int32_t> first;
    for (int i = sinks; i < K - 1; ++i) {
      if (pos[i].empty()) pos[i].assign(size_t(runs) * T, 0);
      std::vector<int32_t> order = (binary && i > sinks) ? first : rank_heads(score[i]);
      if (i == sinks) first = order;
      for (int rank = 0; rank < T; ++rank) pos[i][size_t(r) * T + order[rank]] = rank;
    }
  }
  for (int i = 0; i < K; ++i) dispersion[i] = 0.0;
  for (int i = sinks; i < K - 1; ++i) {
    double total = 0.0;
    for (int head = 0; head < T; ++head) {
      int64_t sum = 0;
      for (int r = 0; r < runs; ++r) sum += pos[i][size_t(r) * T + head];
      const double mean = double(sum) / runs;
      double var = 0.0;
      for (int r = 0; r < runs; ++r) {
        const double dlt = pos[i][size_t(r) * T + head] - mean;
        var += dlt * dlt;
      }
      total += std::sqrt(var / runs);
    }
    dispersion[i] = total / T;
  }
  return HEATKV_OK;
}

int load_pattern(heatkv_plan* p, const uint8_t* present) {
  const int K = p->K, T = p->T;
  p->retained.assign(size_t(K) * T, 0);
  for (int k = 0; k < K; ++k)
    for (int head = 0; head < T; ++head) {
      uint32_t m = 0;
      for (int i = 0; i < K; ++i) {
        const bool on = present[(size_t(k) * T + head) * K + i] != 0;
        if (on && i >= k) return fail(HEATKV_EINVAL, "present[k][..][i] set for i >= k");
        if (on) m |= 1u << i;
      }
      if (k > 0) {
        const uint32_t prev = p->retained[size_t(k - 1) * T + head];
        const uint32_t older = m & ((1u << (k - 1)) - 1u);
        if (older & ~prev) return fail(HEATKV_EINVAL, "a scale absent at scale k-1 is present at scale k");
      }
      p->retained[size_t(k) * T + head] = m;
    }
  return HEATKV_OK;
}

namespace {

constexpr int32_t kCopyChunkRows = 128;

// Places the layer regions of successive scales in one arena of `cap` rows as a
// FIFO: region (k+1,l) is allocated, then region (k,l) is released, in
// generation order.  A region never straddles the end of the arena.
bool place_regions(heatkv_plan* p, int64_t cap) {
  const int K = p->K, L = p->L;
  std::fill(p->region_base.begin(), p->region_base.end(), 0);
  // Live regions are those from `front` up to the one placed last: empty regions are never placed, and regions are
  // released in the order in which they were placed.
  size_t front = size_t(L), back = 0, live = 0;
  auto next_placed = [&](size_t i) {
    while (i < p->region_size.size() && p->region_size[i] == 0) ++i;
    return i;
  };
  int64_t tail = 0;
  for (size_t at = size_t(L); at < size_t(K) * L; ++at) {  // region (k+1,l); region (k,l) is L places before it
    const int64_t S = p->region_size[at];
    if (S > 0) {
      int64_t base;
      if (live == 0) {
        base = 0;
        if (S > cap) return false;
        front = at;
      } else {
        const int64_t first = p->region_base[front];
        const bool wrapped = first > p->region_base[back];
        if (!wrapped) {
          if (tail + S <= cap) base = tail;
          else if (S <= first) base = 0;
          else return false;
        } else {
          if (tail + S <= first) base = tail;
          else return false;
        }
      }
      p->region_base[at] = base;
      back = at;
      ++live;
      tail = base + S;
    }
    if (p->region_size[at - L] > 0) {
      --live;
      front = next_placed(front + 1);
    }
  }
  return true;
}

// Heads of a layer by descending run length, equal ones in index order.  Up to 64 heads: the place of each is the number
// of heads in front of it, counted without branches over keys that hold length and index.
void order_by_length(const int32_t* len, int H, int32_t* ord) {
  bool equal = true;
  int64_t longest = len[0];
  for (int h = 1; h < H; ++h) {
    equal = equal && len[h] == len[0];
    longest = std::max<int64_t>(longest, len[h]);
  }
  if (equal || H > 64 || longest >= 1 << 24) {
    std::iota(ord, ord + H, 0);
    if (!equal) std::stable_sort(ord, ord + H, [&](int32_t a, int32_t b) { return len[a] > len[b]; });
    return;
  }
  int32_t key[64];
  for (int h = 0; h < H; ++h) key[h] = len[h] * 64 + (63 - h);
  for (int h = 0; h < H; ++h) {
    const int32_t mine = key[h];
    int32_t before = 0;
    for (int j = 0; j < H; ++j) before += key[j] > mine;
    ord[before] = h;
  }
}

}  // namespace

int derive_layout(heatkv_plan* p) {
  const int K = p->K, L = p->L, H = p->H, T = p->T;
  const size_t n3 = size_t(K) * L * H, n2 = size_t(K) * L;
  p->run_len.assign(n3, 0);
  p->run_row.assign(n3, 0);
  p->head_order.assign(n3, 0);
  p->region_size.assign(n2, 0);
  p->region_base.assign(n2, 0);
  p->max_len.assign(n2, 0);

  for (int k = 0; k < K; ++k) {
    const uint32_t* m = &p->retained[size_t(k) * T];
    int32_t* len = &p->run_len[p->idx(k, 0, 0)];
    for (int head = 0; k > 0 && head < T; ++head) {  // what the scale before had, less what has left, plus that scale itself
      const uint32_t before = m[head - T];
      int32_t n = len[head - T] + ((m[head] >> (k - 1) & 1u) ? p->t[k - 1] : 0);
      for (uint32_t gone = before & ~m[head]; gone; gone &= gone - 1) n -= p->t[__builtin_ctz(gone)];
      len[head] = n;
    }
    for (int l = 0; l < L; ++l) {
      int64_t sum = 0;
      int32_t mx = 0;
      for (int h = 0; h < H; ++h) {
        sum += len[l * H + h];
        mx = std::max(mx, len[l * H + h]);
      }
      p->region_size[p->idx(k, l)] = sum;
      p->max_len[p->idx(k, l)] = mx;
      order_by_length(len + l * H, H, &p->head_order[p->idx(k, l, 0)]);
    }
  }

  // Smallest arena (searched upward from the peak of live + incoming rows) in which the FIFO fits.
  int64_t lower = 0, max_region = 0, live = 0;
  for (int k = 0; k + 1 < K; ++k)
    for (int l = 0; l < L; ++l) {
      const int64_t S = p->region_size[p->idx(k + 1, l)];
      max_region = std::max(max_region, S);
      lower = std::max(lower, live + S);
      live += S - p->region_size[p->idx(k, l)];
    }
  lower = std::max<int64_t>(lower, 1);
  const int64_t step = std::max<int64_t>(1, (max_region + 31) / 32);
  int64_t cap = lower;
  bool ok = false;
  for (int tries = 0; tries < 4096; ++tries, cap += step)
    if ((ok = place_regions(p, cap))) break;
  if (!ok) return fail(HEATKV_ENOMEM, "no arena placement found");
  if (cap * p->batch > (int64_t(1) << 31) - 1) return fail(HEATKV_EINVAL, "arena rows exceed 2^31");
  p->arena_tokens = cap;

  for (int k = 0; k < K; ++k)
    for (int l = 0; l < L; ++l) {
      int64_t row = p->region_base[p->idx(k, l)];
      for (int h = 0; h < H; ++h) {
        p->run_row[p->idx(k, l, h)] = int32_t(row);
        row += p->run_len[p->idx(k, l, h)];
      }
    }

  // Append descriptors: the move from the scale-k runs (plus the new scale) to the scale-(k+1) runs.
  p->descs.clear();
  p->desc_begin.assign(n2, 0);
  p->desc_count.assign(n2, 0);
  {
    size_t rows = 0, pieces = 0;
    for (int64_t n : p->region_size) rows += size_t(n);
    for (uint32_t m : p->retained) pieces += size_t(__builtin_popcount(m));
    p->descs.resize(rows / kCopyChunkRows + pieces);  // upper bound: every piece has at most one short descriptor
  }
  heatkv::CopyDesc* const first = p->descs.data();
  heatkv::CopyDesc* end = first;
  auto emit = [&](int32_t dst, int32_t src, int32_t rows, int32_t kind) {
    for (; rows > kCopyChunkRows; rows -= kCopyChunkRows, dst += kCopyChunkRows, src += kCopyChunkRows)
      *end++ = heatkv::CopyDesc{dst, src, kCopyChunkRows, kind};
    if (rows > 0) *end++ = heatkv::CopyDesc{dst, src, rows, kind};
  };
  for (int k = 0; k + 1 < K; ++k)
    for (int l = 0; l < L; ++l) {
      const size_t begin = size_t(end - first);
      for (int h = 0; h < H; ++h) {
        const uint32_t now = p->retained[size_t(k) * T + l * H + h];
        const uint32_t nxt = p->retained[size_t(k + 1) * T + l * H + h];
        int32_t dst = p->run_row[p->idx(k + 1, l, h)];
        int32_t src = p->run_row[p->idx(k, l, h)];
        if ((now & ~nxt) == 0) {  // nothing leaves: the run moves in one piece
          const int32_t rows = p->run_len[p->idx(k, l, h)];
          emit(dst, src, rows, 0);
          dst += rows;
        } else {
          int32_t piece = 0;  // rows kept so far that lie side by side in front of src
          for (uint32_t m = now; m; m &= m - 1) {
            const int i = __builtin_ctz(m);
            if (nxt >> i & 1u) {
              piece += p->t[i];
            } else {
              emit(dst, src - piece, piece, 0);
              dst += piece;
              piece = 0;
            }
            src += p->t[i];
          }
          emit(dst, src - piece, piece, 0);
          dst += piece;
        }
        if (nxt >> k & 1u) emit(dst, h * p->t[k], p->t[k], 1);
      }
      p->desc_begin[p->idx(k, l)] = int64_t(begin);
      p->desc_count[p->idx(k, l)] = int32_t(size_t(end - first) - begin);
    }
  p->descs.resize(size_t(end - first));
  return HEATKV_OK;
}

}  // namespace heatkv
