// Selection problems of the cumulative-mass selector: where a (sequence, head)'s scores lie
// and how its state starts (device code only; included by the HIP sources).
#pragma once
#include "fp_internal.h"

namespace fp {

struct Problem {
  const float *scores;
  int n;
  bool active;
};

// Problem `kind` of (sequence s, query head h) whose pattern is pat: kind 0 the vertical
// lines or the flattened map, kind 1 the slash lines.
__device__ __forceinline__ Problem problem_of(const SelectArgs &a, int s, int h, int kind,
                                              int pat) {
  const int tok0 = a.st.cu[s];
  const int n = a.st.cu[s + 1] - tok0;
  Problem pr{nullptr, 0, false};
  if (pat == FP_PATTERN_VERTICAL_SLASH && a.vs_granularity == 1) {
    pr.scores = (kind == 0 ? a.av_blk : a.as_blk) + (int64_t)h * a.nb_total + a.st.nb_off[s];
    pr.n = a.st.nb_off[s + 1] - a.st.nb_off[s];
    pr.active = true;
  } else if (pat == FP_PATTERN_VERTICAL_SLASH) {
    pr.scores = (kind == 0 ? a.a_v : a.a_s) + (int64_t)h * a.total_tokens + tok0;
    pr.n = n;
    pr.active = true;
  } else if (pat == FP_PATTERN_QUERY_AWARE && kind == 0 && a.qa_mode == 0) {
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    pr.scores = a.flat + (int64_t)h * a.tri_total + a.st.tri_off[s];
    pr.n = nb * (nb + 1) / 2;
    pr.active = true;
  }
  return pr;
}

// Problem p = (s * Hq + h) * 2 + kind, once the head's pattern is known.
__device__ __forceinline__ Problem problem_of(const SelectArgs &a, int p) {
  const int sh = p >> 1;
  return problem_of(a, sh / a.hq, sh % a.hq, p & 1, a.pattern[sh]);
}

// The starting state of both problems of (sequence, head), and what their kernels count up
// from: the radix histograms (not used by sel_small) and the line marks.  By nt threads.
__device__ __forceinline__ void init_problems(const SelectArgs &a, int s, int h, int pat, int tid,
                                              int nt) {
  const int p0 = (s * a.hq + h) * 2;
  if (!a.small)
    for (int b = tid; b < 2 * kHistBuckets; b += nt) {
      if (b < 2 * kHistCounts) a.hist_cnt[(int64_t)p0 * kHistCounts + b] = 0u;
      a.hist_mass[(int64_t)p0 * kHistBuckets + b] = 0ull;
    }
  if (!a.marks_inline) {
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    uint32_t *mk =
        reinterpret_cast<uint32_t *>(a.vs_marks) + (int64_t)h * a.nb_total + a.st.nb_off[s];
    for (int i = tid; i < nb; i += nt) mk[i] = 0u;
  }
  if (tid < 2) {
    const Problem pr = problem_of(a, s, h, tid, pat);
    SelState S = {};
    S.mode = pr.active ? 0 : 2;
    S.n = pr.n;
    S.idcut = -1;
    a.sel[p0 + tid] = S;
  }
}

}  // namespace fp
