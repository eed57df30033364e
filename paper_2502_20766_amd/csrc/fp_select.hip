// Cumulative-attention index selection and conversion to key-block lists, for gfx950.
//
// Selection (Algorithms 3 and 4, "minimum computational budget"): for a score vector a,
// order the units by (score desc, id asc) and keep the shortest prefix whose normalised
// mass reaches gamma -- the greedy optimum of the objective equation (Appendix B).  The
// set is found without sorting: a three-digit radix select over the fp32 bit patterns
// (monotone for non-negative floats) finds the threshold key t* such that
//     mass(keys > t*) < gamma * total <= mass(keys >= t*),
// then takes the c lowest-id units with key == t* that are still needed.  Masses are
// accumulated as 2^-48 fixed-point integers, so every sum is exact and independent of
// atomic order: the selected set is bit-reproducible.  Normalisation by the explicit
// total is folded into the threshold (prefix >= gamma * total).
//
// Conversion: vertical-slash heads extend selected lines to the whole matrix (Section 3,
// vertical-slash head) at key-block granularity.  A vertical line j marks key block
// floor(j/b) for every query block at or below it; a slash line o = Delta*b + t marks the
// block diagonal Delta in every query block whose rows reach an offset-t key in it
// (t < rows of the query block), and the diagonal Delta+1 when t > 0.  Query-aware heads
// mark their selected (I, J) units.  Every row then keeps key blocks 0 and I and is
// topped up to min(m, I+1) blocks (query-aware: highest pooled score first, then lowest
// J; vertical-slash: nearest the diagonal first) -- the guards of Section 4.1.  With a
// maximum budget M, rows above M blocks keep 0, I and their other blocks in that same
// order (appendix "maximum budget limit").  Query-aware heads may instead select per query
// block (appendix "flatten ablation"); those rows, and capped query-aware rows, are
// finished by qa_rows.  With block-pooled lines the vertical-slash units are key blocks
// and offset blocks of lines (pool_lines), and a selected unit marks the tiles of all its
// lines.
#include "fp_internal.h"
#include "fp_select_dev.h"
#include "fp_sort.h"

namespace fp {

hipError_t launch_rep_scores(const SelectArgs &a, hipStream_t stream);
hipError_t launch_pattern_search(const SelectArgs &a, hipStream_t stream);
hipError_t launch_pool_q_query_aware(const SelectArgs &a, hipStream_t stream);
hipError_t launch_qa_estimate(const SelectArgs &a, hipStream_t stream);

namespace {

constexpr int kMaxNb = 8192;
constexpr int kSlice = 4096;          // units per histogram workgroup
constexpr double kFxScale = 281474976710656.0;   // 2^48

__device__ __forceinline__ unsigned long long to_fx(float x) {
  return x > 0.f ? (unsigned long long)((double)x * kFxScale) : 0ull;
}

// Inclusive scan, in thread order over the workgroup, of a (fixed-point mass, count) pair
// per thread, and the workgroup totals: a scan inside each wave through lane shuffles, then
// the NW wave totals through `wm`/`wc` (one barrier; the caller separates reuses of them
// by another).  Integer additions: the result does not depend on their order.
template <int NW>
__device__ __forceinline__ void block_incl_scan(unsigned long long &m, uint32_t &c,
                                                unsigned long long *wm, uint32_t *wc,
                                                unsigned long long &tot_m, uint32_t &tot_c) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long vm = __shfl_up(m, off);
    const uint32_t vc = __shfl_up(c, off);
    if (lane >= off) {
      m += vm;
      c += vc;
    }
  }
  if (lane == 63) {
    wm[w] = m;
    wc[w] = c;
  }
  __syncthreads();
  unsigned long long before_m = 0ull;
  uint32_t before_c = 0u;
  tot_m = 0ull;
  tot_c = 0u;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const unsigned long long x = wm[k];
    const uint32_t y = wc[k];
    if (k < w) {
      before_m += x;
      before_c += y;
    }
    tot_m += x;
    tot_c += y;
  }
  m += before_m;
  c += before_c;
}

__device__ __forceinline__ bool is_selected(const SelState &S, float x, int id) {
  const uint32_t key = __float_as_uint(x);
  return key > S.key || (key == S.key && id <= S.idcut);
}

// One radix pass over every problem: grid (slices of kSlice units, problems), 256 threads.
// A workgroup adds its slice's masses per digit to the problem's histogram; the last one of a
// problem to do so (a ticket in the problem's state) finds the digit whose bucket carries the
// cumulative mass across the threshold.  Counts are not taken per digit: pass 2 counts the
// units above its range in registers and the few units inside it by their last digit, which
// halves the LDS atomics that bound pass 0.  With the scan and the tie break in launches of
// their own the select took 51 us at 32 heads and 32k tokens (92 at 128k), so 36 (78).
// The histograms and the ticket are shared between XCDs: device-scope atomics and loads, each
// workgroup's additions waited for before its ticket.
template <int PASS>
__global__ __launch_bounds__(256) void sel_hist(SelectArgs a) {
  constexpr int NB = PASS == 2 ? kHistCounts : kHistBuckets;      // digits of this pass
  constexpr int shift = PASS == 0 ? 21 : (PASS == 1 ? 10 : 0);
  __shared__ unsigned long long mass[NB];
  __shared__ uint32_t cnt[PASS == 2 ? NB : 1];
  __shared__ unsigned long long wmass[4];
  __shared__ uint32_t wcnt[16], s_need;
  __shared__ int s_last, found;
  const int p = blockIdx.y, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  SelState S = a.sel[p];
  if (S.mode != 0) return;
  const int start = blockIdx.x * kSlice;
  if (start >= S.n) return;
  const Problem pr = problem_of(a, p);
  for (int b = tid; b < NB; b += 256) {
    mass[b] = 0ull;
    if constexpr (PASS == 2) cnt[b] = 0u;
  }
  __syncthreads();
  const int end = min(start + kSlice, S.n);
  uint32_t above = 0u;                     // units above the range of the earlier digits
  // four scores per thread are loaded before their histogram updates
  for (int base = start + tid; base < end; base += 4 * 256) {
    float xs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) xs[u] = base + u * 256 < end ? pr.scores[base + u * 256] : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (base + u * 256 >= end) break;
      const float x = xs[u];
      const uint32_t key = __float_as_uint(x);
      bool match = true;
      if (PASS == 1) match = (key >> 21) == (S.prefix >> 21);
      if (PASS == 2) {
        match = (key >> 10) == (S.prefix >> 10);
        above += (key >> 10) > (S.prefix >> 10);
      }
      const uint32_t dg = (key >> shift) & (uint32_t)(NB - 1);
      if (match) {
        const unsigned long long fx = to_fx(x);
        if (fx != 0ull) atomicAdd(&mass[dg], fx);
        if constexpr (PASS == 2) atomicAdd(&cnt[dg], 1u);
      }
    }
  }
  if constexpr (PASS == 2) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) above += __shfl_xor(above, off);
    if (lane == 0) wcnt[w] = above;
  }
  __syncthreads();
  unsigned long long *hm = a.hist_mass + (int64_t)p * kHistBuckets;
  uint32_t *hc = a.hist_cnt + (int64_t)p * kHistCounts;
  for (int b = tid; b < NB; b += 256) {
    if (mass[b]) atomicAdd(&hm[b], mass[b]);
    if constexpr (PASS == 2)
      if (cnt[b]) atomicAdd(&hc[b], cnt[b]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    const uint32_t slices = (S.n + kSlice - 1) / kSlice;
    const unsigned long long mine =
        PASS == 2 ? (unsigned long long)(wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3]) << 32 : 0ull;
    const unsigned long long done = __hip_atomic_fetch_add(&a.sel[p].ticket, mine + 1,
                                                           __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT) + mine;
    s_last = (uint32_t)done == slices - 1;
    s_need = (uint32_t)(done >> 32);
  }
  __syncthreads();
  if (!s_last) return;
  S.cnt_above = s_need;                    // (every workgroup's count, in the last one)
  // thread t owns buckets [NB - BPT (t + 1), NB - BPT t): thread order is descending key order
  constexpr int BPT = NB / 256;
  const int top = NB - BPT * tid;
  unsigned long long bm[BPT], lm = 0ull;
  uint32_t bc[BPT], lc = 0u;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    bm[i] = __hip_atomic_load(&hm[top - 1 - i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bc[i] = 0u;
    if constexpr (PASS == 2)
      bc[i] = __hip_atomic_load(&hc[top - 1 - i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    lm += bm[i];
    lc += bc[i];
  }
  // (cleared for the next pass)
  if constexpr (PASS < 2) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) hm[top - 1 - i] = 0ull;
  }
  unsigned long long im = lm, total;
  uint32_t ic = lc, count;
  block_incl_scan<4>(im, ic, wmass, wcnt, total, count);
  S.ticket = 0ull;
  if (PASS == 0) {
    S.total = total;
    if (total == 0ull) {
      S.mode = 1;
    } else {
      double t = ceil((double)a.gamma * (double)total);
      unsigned long long thr = (unsigned long long)t;
      if (thr < 1ull) thr = 1ull;
      if (thr > total) S.mode = 1;    // never reached: take every unit
      S.thr = thr;
    }
    if (S.mode == 1) {                // the same in every thread
      S.key = 0u;
      S.idcut = 0x7FFFFFFF;
      S.k = S.n;
      if (tid == 0) a.sel[p] = S;
      return;
    }
  }
  if (tid == 0) s_need = 0u;
  __syncthreads();
  unsigned long long run = S.mass_above + im - lm;
  uint32_t runc = S.cnt_above + ic - lc;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    if (run < S.thr && run + bm[i] >= S.thr) {     // exactly one bucket of all threads
      SelState T = S;
      T.prefix |= (uint32_t)(top - 1 - i) << shift;
      T.mass_above = run;
      if constexpr (PASS == 2) {
        T.cnt_above = runc;
        T.key = T.prefix;
        const unsigned long long f = bm[i] / bc[i];   // equal keys carry equal mass
        const unsigned long long need = (T.thr - run + f - 1) / f;
        T.k = (int32_t)(runc + need);
        T.idcut = 0x7FFFFFFF;
        if (need < bc[i]) {
          s_need = (uint32_t)need;
          wcnt[0] = T.key;
        }
      }
      a.sel[p] = T;
    }
    run += bm[i];
    runc += bc[i];
  }
  if constexpr (PASS == 2) {
    // lowest-id tie break, when some but not all units of the key are taken: the id of the
    // need-th unit (in id order) whose key is the threshold key
    __syncthreads();
    const uint32_t need = s_need, tkey = wcnt[0];
    if (need == 0u) return;
    uint32_t running = 0;
    if (tid == 0) found = -1;
    for (int base = 0; base < S.n; base += 1024) {
      bool f[4];
      unsigned long long bal[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = base + 256 * u + tid;
        f[u] = i < S.n && __float_as_uint(pr.scores[i]) == tkey;
        bal[u] = __ballot(f[u]);
      }
      __syncthreads();                     // the last reads of wcnt and found are done
      if (lane < 4) wcnt[4 * lane + w] = (uint32_t)__popcll(lane == 0   ? bal[0]
                                                            : lane == 1 ? bal[1]
                                                            : lane == 2 ? bal[2]
                                                                        : bal[3]);
      __syncthreads();
      uint32_t before = running;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k == w) {
            const uint32_t rank = before + (uint32_t)__popcll(bal[u] & __lanemask_lt());
            if (f[u] && rank + 1 == need) found = base + 256 * u + tid;
          }
          before += wcnt[4 * u + k];
        }
      }
      running = before;
      if (running >= need) break;          // the same in every thread
    }
    __syncthreads();
    if (tid == 0) a.sel[p].idcut = found;
  }
}

// Short problems: every selection problem of the call in one workgroup of NT threads, the
// three radix passes through an LDS histogram and the lowest-id tie break in the same
// launch -- one launch instead of the three above, the same threshold key, counts and
// tie cut (every sum is an exact integer, so the result does not depend on the path).
// A thread holds its E scores (units tid + NT e) in registers over the passes.  The LDS
// atomics bound it (many scores share a bucket), so the histogram holds masses only: units
// of the threshold key all carry that key's own mass, and the units above it are counted
// once at the end (32 heads: 15.3 -> 11.7 us at 4k tokens, 35.5 -> 26.4 at 16k).  16 scores
// per thread take 135 registers in workgroups of 256 threads (three of them a CU) and spill
// 12 at the 128 that workgroups of 1024 are held to.
constexpr int kSmallUnits = 16384;    // largest problem (units) taken by sel_small

template <int NT, int E>
__global__ __launch_bounds__(NT) void sel_small(SelectArgs a) {
  __shared__ unsigned long long mass[kHistBuckets];
  constexpr int NW = NT / 64, BPT = kHistBuckets / NT;   // waves, buckets per thread
  __shared__ unsigned long long wmass[NW];
  __shared__ unsigned long long s_run;
  __shared__ uint32_t s_digit, wcount[NW];
  __shared__ int found;
  const int p = blockIdx.x, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  SelState S = a.sel[p];
  if (S.mode != 0) return;                // the same decision in every thread
  const Problem pr = problem_of(a, p);
  float xs[E];
#pragma unroll
  for (int e = 0; e < E; ++e) xs[e] = tid + NT * e < S.n ? pr.scores[tid + NT * e] : 0.f;
  // thread t owns buckets [top - BPT, top): thread order is descending key order
  const int top = kHistBuckets - BPT * tid;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
    const uint32_t dmask = pass == 2 ? 1023u : 2047u;
    // key bits that the earlier passes fixed
    const uint32_t fixed = pass == 0 ? 0u : (pass == 1 ? ~0u << 21 : ~0u << 10);
#pragma unroll
    for (int b = 0; b < BPT; ++b) mass[tid + NT * b] = 0ull;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint32_t key = __float_as_uint(xs[e]);
      const unsigned long long fx = to_fx(xs[e]);   // 0 past the last unit
      if (fx != 0ull && ((key ^ S.prefix) & fixed) == 0u)
        atomicAdd(&mass[(key >> shift) & dmask], fx);
    }
    __syncthreads();
    unsigned long long bm[BPT], lm = 0ull;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      bm[i] = mass[top - 1 - i];
      lm += bm[i];
    }
    unsigned long long im = lm, total;
    uint32_t ic = 0u, total_c;
    block_incl_scan<NW>(im, ic, wmass, wcount, total, total_c);
    if (pass == 0) {
      S.total = total;
      if (total == 0ull) {
        S.mode = 1;
      } else {
        double t = ceil((double)a.gamma * (double)total);
        unsigned long long thr = (unsigned long long)t;
        if (thr < 1ull) thr = 1ull;
        if (thr > total) S.mode = 1;      // never reached: take every unit
        S.thr = thr;
      }
      if (S.mode == 1) {                  // the same in every thread
        S.key = 0u;
        S.idcut = 0x7FFFFFFF;
        S.k = S.n;
        if (tid == 0) a.sel[p] = S;
        return;
      }
    }
    unsigned long long run = S.mass_above + im - lm;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (run < S.thr && run + bm[i] >= S.thr) {   // exactly one bucket of all threads
        s_digit = (uint32_t)(top - 1 - i);
        s_run = run;
      }
      run += bm[i];
    }
    __syncthreads();
    S.prefix |= s_digit << shift;
    S.mass_above = s_run;
    __syncthreads();                      // every thread has read them before they are reused
  }
  S.key = S.prefix;
  const unsigned long long f = to_fx(__uint_as_float(S.key));
  const uint32_t need = (uint32_t)((S.thr - S.mass_above + f - 1) / f);   // units of the key
  // units above the key, and of the key (both at most kSmallUnits)
  uint32_t c = 0u;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t key = __float_as_uint(xs[e]);
    const bool in = tid + NT * e < S.n;
    c += (in && key > S.key ? 1u << 16 : 0u) + (in && key == S.key ? 1u : 0u);
  }
  // (a sum of at most 2^16 units per half does not carry over: S.n <= 2^14)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if (lane == 0) wcount[w] = c;
  if (tid == 0) found = -1;
  __syncthreads();
  c = 0u;
#pragma unroll
  for (int k = 0; k < NW; ++k) c += wcount[k];
  S.cnt_above = c >> 16;
  const uint32_t n_eq = c & 0xFFFFu;
  S.k = (int32_t)(S.cnt_above + need);
  S.idcut = 0x7FFFFFFF;
  // lowest-id tie break, when some but not all units of the key are taken
  if (need < n_eq) {
    uint32_t running = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (NT * e >= S.n) break;
      const int i = NT * e + tid;
      const bool f = i < S.n && __float_as_uint(xs[e]) == S.key;
      const unsigned long long bal = __ballot(f);
      __syncthreads();                    // the last reads of wcount and found are done
      if (lane == 0) wcount[w] = (uint32_t)__popcll(bal);
      __syncthreads();
      uint32_t before = 0, chunk = 0;
      for (int k = 0; k < NW; ++k) {
        if (k < w) before += wcount[k];
        chunk += wcount[k];
      }
      const uint32_t rank = running + before + (uint32_t)__popcll(bal & __lanemask_lt());
      if (f && rank + 1 == need) found = i;
      running += chunk;
    }
    __syncthreads();
    S.idcut = found;
  }
  if (tid == 0) a.sel[p] = S;
}

// ---------------------------------------------------------------- conversion to lists

// What the selected lines of a vertical-slash head reach, per key block / block diagonal.
// vertical j: column floor(j/b); slash o = D*b + t: diagonal D in full query blocks, diagonal
// D in the partial last query block when t < its rows, diagonal D+1 when t > 0.  A mark is
// only ever set, so the order of the threads does not matter.
struct LineMarks {
  uint8_t *col, *d0, *d0p, *d1;
  int stride;                            // bytes between consecutive key blocks of one array
  __device__ __forceinline__ void vertical(int J) const { col[J * stride] = 1; }
  __device__ __forceinline__ void slash(int D, int t, int last_rows, int nb) const {
    d0[D * stride] = 1;
    if (t < last_rows) d0p[D * stride] = 1;
    if (t > 0 && D + 1 < nb) d1[(D + 1) * stride] = 1;
  }
};

// Lines [j0, j1) of one (sequence, head), by nt threads.
__device__ __forceinline__ void mark_lines(const SelectArgs &a, int s, int h, const SelState S0,
                                           const SelState S1, int j0, int j1, int tid, int nt,
                                           const LineMarks &mk) {
  const int tok0 = a.st.cu[s];
  const int n = a.st.cu[s + 1] - tok0;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const int shift = a.block == 64 ? 6 : 7;
  const int last_rows = n - ((nb - 1) << shift);
  const float *av = a.a_v + (int64_t)h * a.total_tokens + tok0;
  const float *as = a.a_s + (int64_t)h * a.total_tokens + tok0;
  // four scores per thread are loaded before any mark is stored (a byte store may alias
  // the scores, so the compiler would otherwise wait for each load in turn)
  for (int base = j0 + tid; base < j1; base += 4 * nt) {
    float xv[4], xs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = base + u * nt;
      xv[u] = j < j1 ? av[j] : 0.f;
      xs[u] = j < j1 ? as[j] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = base + u * nt;
      if (j >= j1) break;
      if (is_selected(S0, xv[u], j)) mk.vertical(j >> shift);
      if (is_selected(S1, xs[u], j)) mk.slash(j >> shift, j & (a.block - 1), last_rows, nb);
    }
  }
}

// Block-pooled lines: a selected unit selects all its lines.  Key block J is a column;
// offset block D holds o = D*b (t = 0: diagonal D in every row) and, when it has more than
// one offset, o = D*b + t with t > 0 (diagonal D + 1).
__device__ __forceinline__ void mark_blocks(const SelectArgs &a, int s, int h, const SelState S0,
                                            const SelState S1, int tid, int nt,
                                            const LineMarks &mk) {
  const int n = a.st.cu[s + 1] - a.st.cu[s];
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const float *avb = a.av_blk + (int64_t)h * a.nb_total + a.st.nb_off[s];
  const float *asb = a.as_blk + (int64_t)h * a.nb_total + a.st.nb_off[s];
  for (int u = tid; u < nb; u += nt) {
    if (is_selected(S0, avb[u], u)) mk.vertical(u);
    if (is_selected(S1, asb[u], u)) {
      mk.slash(u, 0, 1, nb);
      if (n - u * a.block > 1 && u + 1 < nb) mk.d1[(u + 1) * mk.stride] = 1;
    }
  }
}

// Marks of long sequences' lines, one workgroup per (sequence, head, slice of kMarkSlice
// lines).  convert_tiles makes its own where every workgroup can afford to read the head's
// scores: sequences of up to kMarkInline tokens, and block-pooled lines of any length.
constexpr int kMarkSlice = 8192;
constexpr int kMarkInline = 8192;

// Layers whose Q is at most this large are pooled by the line pass, all heads of it: at 0.5 MB
// (two heads, 2k tokens) selection 49.2 -> 47.8 us, at 8 MB (32 heads, 1000 tokens) 63.4 ->
// 59.2; at 32 MB (4k tokens) the line pass's own workgroups wait for it: 78.7 -> 81.1.
constexpr int64_t kPoolInlineBytes = 10 << 20;

__global__ __launch_bounds__(256) void vs_marks(SelectArgs a) {
  const int s = blockIdx.x / a.hq, h = blockIdx.x % a.hq;
  if (a.pattern[s * a.hq + h] != FP_PATTERN_VERTICAL_SLASH) return;
  const int n = a.st.cu[s + 1] - a.st.cu[s];
  const int p0 = (s * a.hq + h) * 2;
  const int j0 = blockIdx.y * kMarkSlice;
  uint8_t *mk = a.vs_marks + 4 * ((int64_t)h * a.nb_total + a.st.nb_off[s]);
  const SelState S0 = a.sel[p0];
  const SelState S1 = a.sel[p0 + 1];
  mark_lines(a, s, h, S0, S1, j0, min(j0 + kMarkSlice, n), threadIdx.x,
             blockDim.x, LineMarks{mk, mk + 1, mk + 2, mk + 3, 4});
}

// Lists of one (sequence, head): grid (sequence * head, row slice); wave w of slice r
// converts rows I = 16 r + w + 16 R k.
__global__ __launch_bounds__(1024) void convert_tiles(SelectArgs a) {
  __shared__ uint8_t colsel[kMaxNb];
  __shared__ uint8_t d0[kMaxNb];
  __shared__ uint8_t d0p[kMaxNb];
  __shared__ uint8_t d1[kMaxNb + 1];
  __shared__ int added[16][FP_MAX_MIN_BUDGET];
  const int s = blockIdx.x / a.hq, h = blockIdx.x % a.hq;
  const int slice = blockIdx.y, n_slices = gridDim.y;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int n = a.st.cu[s + 1] - a.st.cu[s];
  const int b = a.block;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const int pat = a.pattern[s * a.hq + h];
  const bool vs = pat == FP_PATTERN_VERTICAL_SLASH;
  const int p0 = (s * a.hq + h) * 2;
  const SelState S0 = a.sel[p0];
  const SelState S1 = a.sel[p0 + 1];
  const float *flat = a.flat + (int64_t)h * a.tri_total + a.st.tri_off[s];
  if (slice * 16 >= nb) return;                 // no row of this (sequence, head) here

  if (vs && a.marks_inline) {
    for (int i = tid; i <= nb; i += blockDim.x) {
      if (i < nb) colsel[i] = d0[i] = d0p[i] = 0;
      d1[i] = 0;
    }
    __syncthreads();
    const LineMarks mk{colsel, d0, d0p, d1, 1};
    if (a.vs_granularity == 1) mark_blocks(a, s, h, S0, S1, tid, blockDim.x, mk);
    else mark_lines(a, s, h, S0, S1, 0, n, tid, blockDim.x, mk);
    __syncthreads();
  } else if (vs) {
    const uint32_t *mk = reinterpret_cast<const uint32_t *>(a.vs_marks) +
                         (int64_t)h * a.nb_total + a.st.nb_off[s];
    for (int i = tid; i < nb; i += blockDim.x) {
      const uint32_t m4 = mk[i];
      colsel[i] = m4 & 0xFF;
      d0[i] = (m4 >> 8) & 0xFF;
      d0p[i] = (m4 >> 16) & 0xFF;
      d1[i] = m4 >> 24;
    }
    if (tid == 0) d1[nb] = 0;
    __syncthreads();
  }
  if (tid == 0 && slice == 0) {
    // per-query-block selection accumulates its K over the rows (qa_rows, launched next)
    a.units[(s * a.hq + h) * 2 + 0] = (!vs && a.qa_mode == 1) ? 0 : S0.k;
    a.units[(s * a.hq + h) * 2 + 1] = vs ? S1.k : 0;
  }
  if (!vs && (a.qa_mode == 1 || a.max_budget > 0)) return;   // rows written by qa_rows
  const int last_rows = n - (nb - 1) * b;            // rows of the last query block

  const int m = a.min_budget;
  for (int I = slice * 16 + w; I < nb; I += 16 * n_slices) {
    const bool row_full = (I < nb - 1) || (last_rows == b);
    const int64_t tri_row = (int64_t)I * (I + 1) / 2;
    auto sel = [&](int J) -> bool {
      if (J == 0 || J == I) return true;
      if (vs) {
        const int dl = I - J;
        return colsel[J] || (row_full ? d0[dl] : d0p[dl]) || d1[dl];
      }
      return is_selected(S0, flat[tri_row + J], (int)(tri_row + J));
    };
    // selected count, only as far as the minimum budget needs it (exact whenever it stays
    // below the target, which is the only case that uses it)
    const int target = min(m, I + 1);
    int count = 0;
    for (int J0 = 0; J0 <= I && count < target; J0 += 64) {
      const int J = J0 + lane;
      count += __popcll(__ballot(J <= I && sel(J)));
    }
    int jmin = I;          // vertical-slash top-up: every unselected J in [jmin, I)
    int n_added = 0;       // query-aware top-up: added[w][0..n_added)
    if (count < target) {
      int need = target - count;
      if (vs) {
        for (int top = I - 1; top >= 0 && need > 0; top -= 64) {
          const int J = top - lane;
          const bool un = J >= 0 && !sel(J);
          const unsigned long long bal = __ballot(un);
          const int c = __popcll(bal);
          if (c >= need) {
            const int rank = __popcll(bal & __lanemask_lt());
            const unsigned long long pick = __ballot(un && rank == need - 1);
            jmin = top - (__ffsll((long long)pick) - 1);
            need = 0;
          } else {
            need -= c;
            jmin = top - 63;
          }
        }
      } else if (I < 256) {
        // rows of up to 256 blocks: the unselected blocks' scores stay in registers (-1 for
        // the others), one butterfly per added block
        float xs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int J = 64 * u + lane;
          xs[u] = J <= I ? flat[tri_row + J] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int J = 64 * u + lane;
          if (J > I || J == 0 || J == I || is_selected(S0, xs[u], (int)(tri_row + J))) xs[u] = -1.f;
        }
        for (; n_added < need; ++n_added) {
          float best = -1.f;
          int bj = 0x7FFFFFFF;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (xs[u] > best) { best = xs[u]; bj = 64 * u + lane; }
          for (int off = 32; off > 0; off >>= 1) {
            const float ob = __shfl_xor(best, off);
            const int oj = __shfl_xor(bj, off);
            if (ob > best || (ob == best && oj < bj)) { best = ob; bj = oj; }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (bj == 64 * u + lane) xs[u] = -1.f;
          if (lane == 0) added[w][n_added] = bj;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      } else {
        for (; n_added < need; ++n_added) {
          float best = -1.f;
          int bj = 0x7FFFFFFF;
          // four 64-block chunks per step, their scores loaded before the first is tested
          for (int J0 = 0; J0 <= I; J0 += 256) {
            float xs[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int J = J0 + 64 * u + lane;
              xs[u] = J <= I ? flat[tri_row + J] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int J = J0 + 64 * u + lane;
              if (J > I || J == 0 || J == I || is_selected(S0, xs[u], (int)(tri_row + J)))
                continue;
              bool taken = false;
              for (int q = 0; q < n_added; ++q) taken |= (added[w][q] == J);
              if (taken) continue;
              const float x = xs[u];
              if (x > best || (x == best && J < bj)) { best = x; bj = J; }
            }
          }
          for (int off = 32; off > 0; off >>= 1) {
            const float ob = __shfl_xor(best, off);
            const int oj = __shfl_xor(bj, off);
            if (ob > best || (ob == best && oj < bj)) { best = ob; bj = oj; }
          }
          if (lane == 0) added[w][n_added] = bj;
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
      }
    }
    auto kept = [&](int J) -> bool {
      bool f = sel(J) || (J >= jmin && J < I);
      for (int q = 0; q < n_added; ++q) f |= (added[w][q] == J);
      return f;
    };
    // maximum budget (vertical-slash rows; query-aware rows are capped in qa_rows): keep
    // blocks 0 and I and the nearest-to-diagonal others, i.e. every kept J >= jcap
    int jcap = 0;
    if (vs && a.max_budget > 0 && I > 0) {
      int total = 0;
      for (int J0 = 0; J0 <= I; J0 += 64) {
        const int J = J0 + lane;
        total += __popcll(__ballot(J <= I && kept(J)));
      }
      if (total > a.max_budget) {
        int need = a.max_budget - 2;               // others to keep, nearest I first
        jcap = I;                                    // need == 0: no other block
        for (int top = I - 1; top >= 1 && need > 0; top -= 64) {
          const int J = top - lane;
          const bool f = J >= 1 && kept(J);
          const unsigned long long bal = __ballot(f);
          const int c = __popcll(bal);
          if (c >= need) {
            const int rank = __popcll(bal & __lanemask_lt());
            const unsigned long long pick = __ballot(f && rank == need - 1);
            jcap = top - (__ffsll((long long)pick) - 1);
            need = 0;
          } else {
            need -= c;
          }
        }
      }
    }
    int32_t *out = a.kb_idx + (int64_t)h * a.tri_total + a.st.tri_off[s] + tri_row;
    int running = 0;
    // four 64-block chunks per step; a query-aware row's scores of all four are loaded
    // before the first is tested
    for (int J0 = 0; J0 <= I; J0 += 256) {
      float xs[4] = {0.f, 0.f, 0.f, 0.f};
      if (!vs) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int J = J0 + 64 * u + lane;
          if (J <= I) xs[u] = flat[tri_row + J];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int J = J0 + 64 * u + lane;
        bool f = false;
        if (J <= I) {
          bool k = (J == 0 || J == I) ? true
                   : vs               ? sel(J)
                                      : is_selected(S0, xs[u], (int)(tri_row + J));
          k = k || (J >= jmin && J < I);
          for (int q = 0; q < n_added; ++q) k |= (added[w][q] == J);
          f = k && (J == 0 || J == I || J >= jcap);
        }
        const unsigned long long bal = __ballot(f);
        if (f) out[running + __popcll(bal & __lanemask_lt())] = J;
        running += __popcll(bal);
      }
    }
    if (lane == 0) a.kb_cnt[(int64_t)h * a.nb_total + a.st.nb_off[s] + I] = running;
  }
}

// Block-pooled lines: a_v summed over each key block and a_s over each offset block, one
// wave per (query head, block); vertical-slash heads only.
__global__ __launch_bounds__(256) void pool_lines(SelectArgs a) {
  const int h = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= a.nb_total) return;
  int s = 0;
  while (s + 1 < a.st.n_seq && a.st.nb_off[s + 1] <= row) ++s;
  if (a.pattern[s * a.hq + h] != FP_PATTERN_VERTICAL_SLASH) return;
  const int u = row - a.st.nb_off[s];
  const int tok0 = a.st.cu[s];
  const int n = a.st.cu[s + 1] - tok0;
  const int lo = u * a.block, hi = min(lo + a.block, n);
  const float *av = a.a_v + (int64_t)h * a.total_tokens + tok0;
  const float *as = a.a_s + (int64_t)h * a.total_tokens + tok0;
  float sv = 0.f, ss = 0.f;
  for (int j = lo + lane; j < hi; j += 64) {
    sv += av[j];
    ss += as[j];
  }
  for (int off = 32; off > 0; off >>= 1) {
    sv += __shfl_xor(sv, off);
    ss += __shfl_xor(ss, off);
  }
  if (lane == 0) {
    a.av_blk[(int64_t)h * a.nb_total + row] = sv;
    a.as_blk[(int64_t)h * a.nb_total + row] = ss;
  }
}

// Query-aware rows when the selection is per query block (qa_mode 1) or rows are capped
// (max_budget > 0).  One workgroup per (query head, query block I): the row's pooled scores
// A_bar[I, J], J <= I, are sorted by (score desc, J asc).  The gamma-selected units of the
// row are then a prefix of that order in both modes (flattened: the head's radix
// threshold; per query block: the shortest prefix whose exact fixed-point mass reaches
// ceil(gamma * row total)).  Blocks 0 and I are always kept; the other blocks are taken
// along the same order: the selected prefix, raised to min(m, I+1) blocks in total by the
// top-up and lowered to max_budget by the cap.
constexpr int kRowWavesMax = 8;

struct RowShared {
  unsigned long long wsum[kRowWavesMax];
  uint32_t wcnt[kRowWavesMax];
  int pos0, posI, kcut;
};

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const T u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  return v;
}

// One row of NT*E >= I+1 sort slots (E a power of two).
template <int NT, int E>
__device__ void qa_row(const SelectArgs &a, unsigned long long *lds, uint8_t *keep,
                       RowShared &sh, int s, int h, int I, int row) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int len = I + 1;
  const int64_t tri_row = (int64_t)I * (I + 1) / 2;
  const float *x = a.flat + (int64_t)h * a.tri_total + a.st.tri_off[s] + tri_row;
  unsigned long long k[E];                           // (~score bits) << 32 | J
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = tid * E + e;
    k[e] = i < len ? ((unsigned long long)(~__float_as_uint(x[i])) << 32) | (uint32_t)i
                   : ~0ull;
  }
  if (tid == 0) sh.kcut = len;
  bitonic_sort<NT, E, 2>(k, lds, tid);
  auto score_of = [](unsigned long long key) { return __uint_as_float(~(uint32_t)(key >> 32)); };
  auto id_of = [](unsigned long long key) { return (int)(key & 0xFFFFFFFFu); };
  // positions of the forced blocks 0 and I in the order
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = tid * E + e;
    if (p < len) {
      const int J = id_of(k[e]);
      if (J == 0) sh.pos0 = p;
      if (J == I) sh.posI = p;
    }
  }
  int K;                                             // gamma-selected units of the row
  if (a.qa_mode == 1) {
    auto mass_at = [&](int e) {
      return tid * E + e < len ? to_fx(score_of(k[e])) : 0ull;
    };
    unsigned long long mine = 0ull;
#pragma unroll
    for (int e = 0; e < E; ++e) mine += mass_at(e);
    const unsigned long long incl = wave_incl_scan(mine, lane);
    if (lane == 63) sh.wsum[w] = incl;
    __syncthreads();
    unsigned long long run = incl - mine, total = 0ull;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
      if (q < w) run += sh.wsum[q];
      total += sh.wsum[q];
    }
    unsigned long long thr = (unsigned long long)ceil((double)a.gamma * (double)total);
    if (thr < 1ull) thr = 1ull;
    if (total > 0ull && thr <= total) {
      int cut = len;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        run += mass_at(e);
        if (cut == len && run >= thr) cut = tid * E + e + 1;
      }
      if (cut < len) atomicMin(&sh.kcut, cut);
    }
    __syncthreads();
    K = sh.kcut;
    if (tid == 0) atomicAdd(&a.units[(s * a.hq + h) * 2], K);
  } else {
    const SelState S0 = a.sel[(s * a.hq + h) * 2];
    int c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (tid * E + e < len)
        c += is_selected(S0, score_of(k[e]), (int)(tri_row + id_of(k[e])));
    c = (int)__reduce_add_sync(~0ull, (unsigned)c);
    if (lane == 0) sh.wcnt[w] = (uint32_t)c;
    __syncthreads();
    K = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) K += (int)sh.wcnt[q];
  }
  const int pos0 = sh.pos0, posI = sh.posI;
  const int f = I == 0 ? 1 : 2;                       // forced blocks
  const int in_f = (pos0 < K) + (I > 0 && posI < K);
  int k_final = K - in_f;                             // other blocks, along the order
  k_final = max(k_final, min(a.min_budget, len) - f);
  if (a.max_budget > 0) k_final = min(k_final, a.max_budget - f);
  // every J <= I sits at exactly one position p < len, so this writes all of keep[0..I]
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = tid * E + e;
    if (p < len) {
      const int J = id_of(k[e]);
      const int rank = p - (pos0 < p) - (I > 0 && posI < p);   // position among the others
      keep[J] = (J == 0 || J == I || rank < k_final) ? 1 : 0;
    }
  }
  __syncthreads();
  // ascending compaction: thread t owns blocks t*E .. t*E+E-1
  uint32_t bits = 0u;
  int cnt = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int J = tid * E + e;
    if (J < len && keep[J]) {
      bits |= 1u << e;
      ++cnt;
    }
  }
  const int incl = wave_incl_scan(cnt, lane);
  if (lane == 63) sh.wcnt[w] = (uint32_t)incl;
  __syncthreads();
  int base = incl - cnt, total = 0;
#pragma unroll
  for (int q = 0; q < NT / 64; ++q) {
    if (q < w) base += (int)sh.wcnt[q];
    total += (int)sh.wcnt[q];
  }
  int32_t *out = a.kb_idx + (int64_t)h * a.tri_total + a.st.tri_off[s] + tri_row;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if ((bits >> e) & 1u) out[base++] = tid * E + e;
  if (tid == 0) a.kb_cnt[(int64_t)h * a.nb_total + row] = total;
}

// NT threads per row, EMAX = sort slots per thread for the longest row (NT*EMAX >= max_nb).
template <int NT, int EMAX>
__global__ __launch_bounds__(NT) void qa_rows(SelectArgs a) {
  // dynamic LDS: NT*EMAX sort keys, then NT*EMAX keep flags
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  unsigned long long *lds = reinterpret_cast<unsigned long long *>(dyn);
  uint8_t *keep = dyn + (size_t)NT * EMAX * sizeof(unsigned long long);
  __shared__ RowShared sh;
  const int h = blockIdx.y;
  const int row = blockIdx.x;
  int s = 0;
  while (s + 1 < a.st.n_seq && a.st.nb_off[s + 1] <= row) ++s;
  if (a.pattern[s * a.hq + h] != FP_PATTERN_QUERY_AWARE) return;
  const int I = row - a.st.nb_off[s];
  if (I < NT) {
    qa_row<NT, 1>(a, lds, keep, sh, s, h, I, row);
  } else if (I < 2 * NT) {
    if constexpr (EMAX >= 2) qa_row<NT, 2>(a, lds, keep, sh, s, h, I, row);
  } else if (I < 4 * NT) {
    if constexpr (EMAX >= 4) qa_row<NT, 4>(a, lds, keep, sh, s, h, I, row);
  } else if (I < 8 * NT) {
    if constexpr (EMAX >= 8) qa_row<NT, 8>(a, lds, keep, sh, s, h, I, row);
  } else {
    if constexpr (EMAX >= 16) qa_row<NT, 16>(a, lds, keep, sh, s, h, I, row);
  }
}

// gamma >= 1: every causal key block, no search (full attention).
__global__ __launch_bounds__(256) void dense_lists(SelectArgs a) {
  const int h = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= a.nb_total) return;
  int s = 0;
  while (s + 1 < a.st.n_seq && a.st.nb_off[s + 1] <= row) ++s;
  const int I = row - a.st.nb_off[s];
  int32_t *out = a.kb_idx + (int64_t)h * a.tri_total + a.st.tri_off[s] + (int64_t)I * (I + 1) / 2;
  for (int J = lane; J <= I; J += 64) out[J] = J;
  if (lane == 0) a.kb_cnt[(int64_t)h * a.nb_total + row] = I + 1;
  if (I == 0 && lane == 0) {
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    a.pattern[s * a.hq + h] = FP_PATTERN_DENSE;
    a.js[s * a.hq + h] = -1.f;
    a.units[(s * a.hq + h) * 2 + 0] = nb * (nb + 1) / 2;
    a.units[(s * a.hq + h) * 2 + 1] = 0;
  }
}

}  // namespace

template <int NT, int EMAX>
hipError_t launch_qa_rows_e(const SelectArgs &a, hipStream_t stream) {
  const size_t dyn = (size_t)NT * EMAX * (sizeof(unsigned long long) + 1);
  if (dyn > 65536) {          // rows above 4096 blocks: allow the larger LDS allocation
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(qa_rows<NT, EMAX>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)dyn);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((qa_rows<NT, EMAX>), dim3(a.nb_total, a.hq), dim3(NT), dyn, stream, a);
  return hipGetLastError();
}

hipError_t launch_qa_rows(const SelectArgs &a, hipStream_t stream) {
  // row I holds I+1 <= max_nb keys in NT*E slots; at most 16 slots per thread keeps the
  // keys in registers, so the longest rows take 512 threads
  if (a.st.max_nb <= 256) return launch_qa_rows_e<256, 1>(a, stream);
  if (a.st.max_nb <= 512) return launch_qa_rows_e<256, 2>(a, stream);
  if (a.st.max_nb <= 1024) return launch_qa_rows_e<256, 4>(a, stream);
  if (a.st.max_nb <= 2048) return launch_qa_rows_e<256, 8>(a, stream);
  if (a.st.max_nb <= 4096) return launch_qa_rows_e<256, 16>(a, stream);
  if (a.st.max_nb <= 8192) return launch_qa_rows_e<512, 16>(a, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_dense_lists(const SelectArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL(dense_lists, dim3((a.nb_total + 3) / 4, a.hq), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_select_pipeline(const SelectArgs &args, hipStream_t stream) {
  SelectArgs a = args;
  int max_units = 0, max_n = 0;
  for (int s = 0; s < a.st.n_seq; ++s) {
    const int n = a.st.cu[s + 1] - a.st.cu[s];
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    max_units = max(max_units, max(n, nb * (nb + 1) / 2));
    max_n = max(max_n, n);
  }
  a.marks_inline = a.vs_granularity == 1 || max_n <= kMarkInline;
  a.small = max_units <= kSmallUnits;
  a.pool_inline = (int64_t)a.total_tokens * a.hq * a.d * 2 <= kPoolInlineBytes;
  hipError_t e;
  if ((e = launch_rep_scores(a, stream)) != hipSuccess) return e;
  if ((e = launch_pattern_search(a, stream)) != hipSuccess) return e;
  if ((e = launch_pool_q_query_aware(a, stream)) != hipSuccess) return e;
  if ((e = launch_qa_estimate(a, stream)) != hipSuccess) return e;
  const int problems = a.st.n_seq * a.hq * 2;
  const int slices = (max_units + kSlice - 1) / kSlice;
  if (a.vs_granularity == 1)
    hipLaunchKernelGGL(pool_lines, dim3((a.nb_total + 3) / 4, a.hq), dim3(256), 0, stream, a);
  if (a.small) {
    // many small problems: three workgroups of 256 threads a CU instead of one of 1024 (64
    // sequences of 8 heads: 39.4 -> 19.3 us).  The line is on the safe side: the selection of
    // packed sequences of up to 17 blocks takes 130 us with 1024 threads and 114 with 256 at
    // 528 problems, 128 and 118 at 512, 79 and 78 at 256, 65 and 63 at 64.
    if (max_units <= 4096 && problems > 512)
      hipLaunchKernelGGL((sel_small<256, 16>), dim3(problems), dim3(256), 0, stream, a);
    else if (max_units <= 4096)
      hipLaunchKernelGGL((sel_small<1024, 4>), dim3(problems), dim3(1024), 0, stream, a);
    else
      hipLaunchKernelGGL((sel_small<1024, 16>), dim3(problems), dim3(1024), 0, stream, a);
  } else {
    hipLaunchKernelGGL(sel_hist<0>, dim3(slices, problems), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(sel_hist<1>, dim3(slices, problems), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(sel_hist<2>, dim3(slices, problems), dim3(256), 0, stream, a);
  }
  {
    if (!a.marks_inline)
      hipLaunchKernelGGL(vs_marks, dim3(a.st.n_seq * a.hq, (max_n + kMarkSlice - 1) / kMarkSlice),
                         dim3(256), 0, stream, a);
    // row slices: about two workgroups per CU over all (sequence, head) pairs, and at
    // most four rows per wave on the longest sequence (packed batches mix lengths, and
    // the workgroups of short sequences end early)
    const int pairs = a.st.n_seq * a.hq;
    int slices = max((512 + pairs - 1) / pairs, (a.st.max_nb + 63) / 64);
    slices = max(1, min(slices, (a.st.max_nb + 15) / 16));
    hipLaunchKernelGGL(convert_tiles, dim3(pairs, slices), dim3(1024), 0, stream, a);
  }
  if (a.qa_mode == 1 || a.max_budget > 0) {
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_qa_rows(a, stream);
  }
  return hipGetLastError();
}

}  // namespace fp
