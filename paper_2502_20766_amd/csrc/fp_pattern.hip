// Sparse pattern search (Algorithm 2) and the query-aware block estimate (Algorithm 4,
// first steps) for gfx950.
//
// pattern_search (or pattern_parts + pattern_decide): per (sequence, query head)
//   a_bar = softmax(scale * avgpool(Q_hat) . avgpool(K)^T)       over all key blocks
//   a_hat = block sums of the vertical line scores a_v            (= sumpool of A_hat / b')
//   D_JS  = sqrt((KL(a_bar || m) + KL(a_hat || m)) / 2), m = (a_bar + a_hat) / 2, natural log
//   pattern = query-aware iff D_JS < tau (or the forced pattern).
// The divergence is accumulated in double with a fixed reduction tree.  The same launch sets
// up the head's selection problems, whose scores its pattern names.
//
// qa_logits / qa_softmax: for query-aware heads only,
//   A_bar[I, J] = softmax over J <= I of scale * Q_bar_I . K_bar_J
// stored as the flattened causal entries (row-major, I(I+1)/2 + J), in fp32 with the
// pooled vectors kept in fp32 (pooled means rounded to bf16 would move the selection).
#include <type_traits>

#include "fp_internal.h"
#include "fp_select_dev.h"

namespace fp {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ int seq_of_block(const SeqTable &st, int blk) {
  int s = 0;
  while (s + 1 < st.n_seq && st.nb_off[s + 1] <= blk) ++s;
  return s;
}

// Sum (or max) over a workgroup of NT threads: a fixed butterfly inside each wave, then the
// wave results in wave order through `scratch` (NT / 64 values).
template <int NT, typename T, typename F>
__device__ __forceinline__ T block_reduce(T v, T *scratch, F op) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  T r = scratch[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) r = op(r, scratch[w]);
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------- Algorithm 2

// avgpool(Q_hat) into qbar[D], by 256 threads (all threads of the workgroup call it): thread
// (phase ph, chunk ch) sums rows ph, ph + PH, ... of its 8 dimensions; the phases are then
// added in order.  qpart: 256 / (D / 8) * D floats.
template <int D>
__device__ __forceinline__ void pool_qhat(const SelectArgs &a, int s, int h, float *qpart,
                                          float *qbar) {
  constexpr int CH = D / 8;                 // 16-byte chunks of a query row
  constexpr int PH = 256 / CH;              // row phases
  const int tid = threadIdx.x;
  const int tok0 = a.st.cu[s];
  const int n = a.st.cu[s + 1] - tok0;
  const int bp = min(a.block, n);
  if (tid < 256) {
    const int ch = tid % CH, ph = tid / CH;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const uint16_t *qp = a.q + ((int64_t)(tok0 + n - bp) * a.hq + h) * D + ch * 8;
#pragma unroll 8
    for (int r = ph; r < bp; r += PH) {
      const uint4 v = *reinterpret_cast<const uint4 *>(qp + (int64_t)r * a.hq * D);
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += __uint_as_float(wv[i] << 16);
        acc[2 * i + 1] += __uint_as_float(wv[i] & 0xFFFF0000u);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) qpart[ph * D + ch * 8 + i] = acc[i];
  }
  __syncthreads();
  if (tid < D) {
    float acc = 0.f;
    for (int ph = 0; ph < PH; ++ph) acc += qpart[ph * D + tid];
    qbar[tid] = acc / (float)bp;
  }
  __syncthreads();
}

// Key blocks [J0, J1) of one (sequence, head) by the NT threads of a workgroup, 16 lanes per
// block J: out(J, scale * q_bar . K_bar_J, a_hat[J]).  The lanes of a block read its pooled
// key (16-byte pieces) and its line scores (lane l tokens l, l + 16, ...) coalesced and
// whatever the sequence's alignment, all loads in flight, and add up by a fixed butterfly
// (a_hat in double).  One thread per block waits for every
// load of a sequence that does not start on a 16-byte boundary in turn: 109 us for 64 ragged
// sequences.
template <int D, int NT, typename F>
__device__ __forceinline__ void block_terms(const SelectArgs &a, int s, int h, int J0, int J1,
                                            const float *qbar, F out) {
  const int tok0 = a.st.cu[s];
  const int n = a.st.cu[s + 1] - tok0;
  const int g = h / (a.hq / a.hkv);
  const int l = threadIdx.x & 15;
  const float *av = a.a_v + (int64_t)h * a.total_tokens + tok0;
  const float4 *q4 = reinterpret_cast<const float4 *>(qbar);
  for (int J = J0 + (int)(threadIdx.x >> 4); J < J1; J += NT / 16) {
    const float4 *kb =
        reinterpret_cast<const float4 *>(a.kbar + ((int64_t)(a.st.nb_off[s] + J) * a.hkv + g) * D);
    float4 kv[D / 64];
#pragma unroll
    for (int i = 0; i < D / 64; ++i) kv[i] = kb[l + 16 * i];
    const int j0 = J * a.block, len = min(a.block, n - j0);
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = l + 16 * u < len ? av[j0 + l + 16 * u] : 0.f;
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
      const float4 qv = q4[l + 16 * i];
      dot = fmaf(qv.x, kv[i].x, dot);
      dot = fmaf(qv.y, kv[i].y, dot);
      dot = fmaf(qv.z, kv[i].z, dot);
      dot = fmaf(qv.w, kv[i].w, dot);
    }
    double ph = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) ph += (double)x[u];
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      dot += __shfl_xor(dot, off);
      ph += __shfl_xor(ph, off);
    }
    if (l == 0) out(J, dot * a.scale, ph);
  }
}

// a_bar = softmax of the logits lg, D_JS against a_hat (double, fixed reduction trees), the
// pattern, and the head's selection problems.  NT threads; scr: NT / 64 doubles.
template <int NT>
__device__ __forceinline__ void decide(const SelectArgs &a, int s, int h, int nb,
                                       const float *lg, const double *ah, double *scr) {
  const int tid = threadIdx.x;
  auto sum = [](double x, double y) { return x + y; };
  float mx = -INFINITY;
  for (int J = tid; J < nb; J += NT) mx = fmaxf(mx, lg[J]);
  mx = block_reduce<NT>(mx, reinterpret_cast<float *>(scr),
                        [](float x, float y) { return fmaxf(x, y); });
  double se = 0.0;
  for (int J = tid; J < nb; J += NT) se += (double)expf(lg[J] - mx);
  se = block_reduce<NT>(se, scr, sum);
  // JSD terms, double precision
  double jsd = 0.0;
  for (int J = tid; J < nb; J += NT) {
    const double pb = (double)expf(lg[J] - mx) / se;               // a_bar[J]
    const double ph = ah[J];                                        // a_hat[J]
    const double m = 0.5 * (pb + ph);
    if (pb > 0.0) jsd += 0.5 * pb * log(pb / m);
    if (ph > 0.0) jsd += 0.5 * ph * log(ph / m);
  }
  jsd = block_reduce<NT>(jsd, scr, sum);
  const float djs = (float)sqrt(jsd > 0.0 ? jsd : 0.0);
  int pat = (djs < a.tau) ? FP_PATTERN_QUERY_AWARE : FP_PATTERN_VERTICAL_SLASH;
  if (a.force_pattern == 0 || a.force_pattern == 1) pat = a.force_pattern;
  if (tid == 0) {
    a.js[s * a.hq + h] = djs;
    a.pattern[s * a.hq + h] = (uint8_t)pat;
  }
  init_problems(a, s, h, pat, tid, NT);
}

// Key blocks of one (sequence, head) are split over kPatSlices workgroups for the logits
// and the block sums when there are many; one workgroup per (sequence, head) then reduces
// them.
constexpr int kPatSlices = 16;
constexpr int kPatThreads = 1024;

// pattern_parts: grid (n_seq * kPatSlices, Hq).
template <int D>
__global__ __launch_bounds__(kPatThreads) void pattern_parts(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) float qbar[D];
  __shared__ float qpart[256 / (D / 8) * D];
  const int s = blockIdx.x / kPatSlices, slice = blockIdx.x % kPatSlices;
  const int h = blockIdx.y;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const int per = (nb + kPatSlices - 1) / kPatSlices;
  const int J0 = slice * per, J1 = min(nb, J0 + per);
  if (J0 >= J1) return;
  pool_qhat<D>(a, s, h, qpart, qbar);
  const int64_t at = (int64_t)h * a.nb_total + a.st.nb_off[s];
  block_terms<D, kPatThreads>(a, s, h, J0, J1, qbar, [&](int J, float logit, double ahat) {
    a.pat_logit[at + J] = logit;
    a.pat_ahat[at + J] = ahat;
  });
}

// pattern_decide: grid (n_seq, Hq).
constexpr int kDecideThreads = 1024;
__global__ __launch_bounds__(kDecideThreads) void pattern_decide(SelectArgs a) {
  extern __shared__ float dyn[];            // [max_nb] logits
  __shared__ double scr[kDecideThreads / 64];
  const int s = blockIdx.x, h = blockIdx.y;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const int64_t at = (int64_t)h * a.nb_total + a.st.nb_off[s];
  for (int J = threadIdx.x; J < nb; J += kDecideThreads) dyn[J] = a.pat_logit[at + J];
  __syncthreads();
  decide<kDecideThreads>(a, s, h, nb, dyn, a.pat_ahat + at, scr);
}

// pattern_search: both steps in one workgroup per (sequence, head), for sequences of up to
// kPatFused blocks: one launch of 8.5 us instead of 6.1 + 4.6 at 32 blocks and of 13.6 instead
// of 8.0 + 6.0 at 128 (32 heads); at 256 blocks it took 19-20 us, the two launches 17.  Grid
// (n_seq, Hq).
constexpr int kPatFused = 128;
template <int D, int NT>
__global__ __launch_bounds__(NT) void pattern_search(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) float qbar[D];
  __shared__ float qpart[256 / (D / 8) * D];
  __shared__ float lg[kPatFused];
  __shared__ double ah[kPatFused];
  __shared__ double scr[kDecideThreads / 64];
  const int s = blockIdx.x, h = blockIdx.y;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  pool_qhat<D>(a, s, h, qpart, qbar);
  block_terms<D, NT>(a, s, h, 0, nb, qbar, [&](int J, float logit, double ahat) {
    lg[J] = logit;
    ah[J] = ahat;
  });
  __syncthreads();
  decide<NT>(a, s, h, nb, lg, ah, scr);
}

// ---------------------------------------------------------------- Algorithm 4 estimate

// Softmax of the row x[0 .. I], held in one wave's registers (I < 64 R), to y[0 .. I].
template <int R>
__device__ __forceinline__ void row_softmax(const float *x, float *y, int I, int lane) {
  float xv[R];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int J = lane + 64 * u;
    xv[u] = J <= I ? x[J] : -INFINITY;
    mx = fmaxf(mx, xv[u]);
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  float se = 0.f;
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (lane + 64 * u <= I) {
      xv[u] = expf(xv[u] - mx);
      se += xv[u];
    }
  for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off);
  const float inv = 1.f / se;
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (lane + 64 * u <= I) y[lane + 64 * u] = xv[u] * inv;
}

// rows and columns of A_bar per workgroup tile: QT (16 waves, one 32x32 block each), or, where
// every sequence has at most kQtSmall blocks, one 32x32 block (four waves for the staging and
// the softmax, a quarter of the LDS)
constexpr int QT = 128;
constexpr int kQtSmall = 32;

// Tile (TI, TJ), TJ <= TI, of the logits scale * Q_bar_I . K_bar_J written into the
// flattened causal layout.  Grid x enumerates the causal tile pairs of all sequences.
// The tile's 128 Q_bar rows and 128 K_bar rows are staged in LDS with coalesced 16-byte
// loads; each wave then computes one 32x32 block with the fp32 MFMA (products and sums
// in fp32, as the vector code would): lane (l % 32, l / 32) supplies Q_bar row l % 32 and
// K_bar row l % 32 over dimensions [l / 32 * D / 2, +D / 2), so the reduction runs over the
// same dimensions for both operands.
// ROWS (every sequence in one tile, i.e. at most QT blocks): the tile holds whole rows of the
// map, so their softmax is taken here, over an LDS copy, with the operations of qa_softmax:
// 7.8 us instead of 6.5 + 4.8 at 32 blocks, 21.4 instead of 14.2 + 6.8 at 128 (32 heads).
template <int D, int QT, bool ROWS>
__global__ __launch_bounds__(QT == 128 ? 1024 : 256) void qa_logits(SelectArgs a) {
  constexpr int NT = QT == 128 ? 1024 : 256;
  constexpr int W = QT / 32;             // 32x32 blocks per side

  typedef float f32x16 __attribute__((ext_vector_type(16)));
  constexpr int P = D + 4;               // LDS row pitch in floats (16-byte rows, no conflicts)
  __shared__ __attribute__((aligned(16))) float rows[2 * QT * P];
  static_assert(2 * QT * P >= QT * (QT + 1), "the logits of a tile fit over its rows");
  float *Qs = rows, *Ks = rows + QT * P;
  const int h = blockIdx.y;
  // locate sequence and tile pair
  int t = blockIdx.x, s = 0, nt = 0;
  for (; s < a.st.n_seq; ++s) {
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    nt = (nb + QT - 1) / QT;
    const int pairs = nt * (nt + 1) / 2;
    if (t < pairs) break;
    t -= pairs;
  }
  if (s >= a.st.n_seq) return;
  if (a.pattern[s * a.hq + h] != FP_PATTERN_QUERY_AWARE) return;
  int TI = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((TI + 1) * (TI + 2) / 2 <= t) ++TI;
  while (TI * (TI + 1) / 2 > t) --TI;
  const int TJ = t - TI * (TI + 1) / 2;
  const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
  const int G = a.hq / a.hkv;
  const int g = h / G;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  // stage the rows (rows past the sequence's last block are clamped; their logits are not
  // written)
  // (every load is issued before the first store, so the loads overlap)
  constexpr int NST = QT * (D / 4) / NT;
  static_assert(NST * NT == QT * (D / 4), "staging covers the tile exactly");
  float4 qv4[NST], kv4[NST];
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const int i = tid + u * NT;
    const int row = i / (D / 4), c = i % (D / 4);
    const int I = min(TI * QT + row, nb - 1), J = min(TJ * QT + row, nb - 1);
    qv4[u] = reinterpret_cast<const float4 *>(
        a.qbar + ((int64_t)(a.st.nb_off[s] + I) * a.hq + h) * D)[c];
    kv4[u] = reinterpret_cast<const float4 *>(
        a.kbar + ((int64_t)(a.st.nb_off[s] + J) * a.hkv + g) * D)[c];
  }
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const int i = tid + u * NT;
    const int row = i / (D / 4), c = i % (D / 4);
    *reinterpret_cast<float4 *>(Qs + row * P + 4 * c) = qv4[u];
    *reinterpret_cast<float4 *>(Ks + row * P + 4 * c) = kv4[u];
  }
  __syncthreads();
  const int i0 = 32 * (w / W), j0 = 32 * (w % W);           // block within the tile
  const int I0 = TI * QT + i0, J0 = TJ * QT + j0;
  // not above the diagonal or past the end
  const bool used = w < W * W && J0 <= I0 + 31 && I0 < nb;
  if (!ROWS && !used) return;
  const float *qa = Qs + (i0 + lr) * P + lh * (D / 2);
  const float *kb = Ks + (j0 + lr) * P + lh * (D / 2);
  f32x16 acc = {};
  if (used)
#pragma unroll
  for (int c = 0; c < D / 2; c += 4) {
    const float4 qv = *reinterpret_cast<const float4 *>(qa + c);
    const float4 kv = *reinterpret_cast<const float4 *>(kb + c);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv.x, kv.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv.y, kv.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv.z, kv.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv.w, kv.w, acc, 0, 0, 0);
  }
  // lane holds column J0 + lr of rows I0 + 8 (v / 4) + 4 lh + v % 4
  float *flat = a.flat + (int64_t)h * a.tri_total + a.st.tri_off[s];
  const int J = J0 + lr;
  if constexpr (ROWS) {
    constexpr int LP = QT + 1;
    float *L = rows;                     // [row][column], once every wave is done with the rows
    __syncthreads();
    if (used)
#pragma unroll
      for (int v = 0; v < 16; ++v) L[(I0 + 8 * (v >> 2) + 4 * lh + (v & 3)) * LP + J] = acc[v] * a.scale;
    __syncthreads();
    for (int I = w; I < nb; I += NT / 64)
      row_softmax<(QT + 63) / 64>(L + I * LP, flat + (int64_t)I * (I + 1) / 2, I, lane);
    return;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int I = I0 + 8 * (v >> 2) + 4 * lh + (v & 3);
    if (I < nb && J <= I) flat[(int64_t)I * (I + 1) / 2 + J] = acc[v] * a.scale;
  }
}

// Row softmax over J <= I of the flattened logits, one wave per row (in place).
constexpr int kRowRegs = 16;   // rows up to 1024 blocks are held in registers
__global__ __launch_bounds__(kThreads) void qa_softmax(SelectArgs a) {
  const int h = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= a.nb_total) return;
  const int s = seq_of_block(a.st, row);
  if (a.pattern[s * a.hq + h] != FP_PATTERN_QUERY_AWARE) return;
  const int I = row - a.st.nb_off[s];
  float *x = a.flat + (int64_t)h * a.tri_total + a.st.tri_off[s] + (int64_t)I * (I + 1) / 2;
  if (I < 64 * kRowRegs) {
    // (same operations in the same order as the streaming form below)
    row_softmax<kRowRegs>(x, x, I, lane);
    return;
  }
  float mx = -INFINITY;
  for (int J = lane; J <= I; J += 64) mx = fmaxf(mx, x[J]);
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  float se = 0.f;
  for (int J = lane; J <= I; J += 64) se += expf(x[J] - mx);
  for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off);
  const float inv = 1.f / se;
  for (int J = lane; J <= I; J += 64) x[J] = expf(x[J] - mx) * inv;
}

}  // namespace

// Sequences of few blocks, and either very few or so many (sequence, head) pairs that
// workgroups of 1024 threads come one or two to a CU: 256 threads (64 sequences of 8 heads of
// up to 18 blocks: pattern search 18.1 -> 11.0 us, logits 30.3 -> 14.6).  The whole selection
// with 1024 threads and with 256: up to 17 blocks 65.0 and 66.0 us at 32 pairs, 79.3 and 79.5
// at 128, 128 and 126 at 256, 123 and 114 at 264, 187 and 168 at 512; up to 32 blocks 74 and
// 77 at 32, 118 and 120 at 128, 180 and 181 at 256, 185 and 179 at 264, 320 and 302 at 512.
static bool small_heads(const SelectArgs &a) {
  return a.st.max_nb <= 16 || (a.st.max_nb <= kQtSmall && a.st.n_seq * a.hq > 256);
}

hipError_t launch_pattern_search(const SelectArgs &a, hipStream_t stream) {
  if (a.st.max_nb <= kPatFused) {
    const dim3 grid(a.st.n_seq, a.hq);
    if (small_heads(a)) {
      if (a.d == 128)
        hipLaunchKernelGGL((pattern_search<128, 256>), grid, dim3(256), 0, stream, a);
      else
        hipLaunchKernelGGL((pattern_search<64, 256>), grid, dim3(256), 0, stream, a);
    } else if (a.d == 128) {
      hipLaunchKernelGGL((pattern_search<128, kDecideThreads>), grid, dim3(kDecideThreads), 0,
                         stream, a);
    } else {
      hipLaunchKernelGGL((pattern_search<64, kDecideThreads>), grid, dim3(kDecideThreads), 0,
                         stream, a);
    }
    return hipGetLastError();
  }
  const dim3 parts(a.st.n_seq * kPatSlices, a.hq);
  if (a.d == 128)
    hipLaunchKernelGGL(pattern_parts<128>, parts, dim3(kPatThreads), 0, stream, a);
  else
    hipLaunchKernelGGL(pattern_parts<64>, parts, dim3(kPatThreads), 0, stream, a);
  const size_t dyn = (size_t)a.st.max_nb * sizeof(float);
  hipLaunchKernelGGL(pattern_decide, dim3(a.st.n_seq, a.hq), dim3(kDecideThreads), dyn, stream, a);
  return hipGetLastError();
}

hipError_t launch_qa_estimate(const SelectArgs &a, hipStream_t stream) {
  int pairs = 0;
  for (int s = 0; s < a.st.n_seq; ++s) {
    const int nb = a.st.nb_off[s + 1] - a.st.nb_off[s];
    const int nt = (nb + QT - 1) / QT;
    pairs += nt * (nt + 1) / 2;
  }
  const bool rows = a.st.max_nb <= QT, small = small_heads(a);
  auto logits = [&](auto dc) {
    constexpr int D = decltype(dc)::value;
    const dim3 grid(pairs, a.hq);
    if (small)
      hipLaunchKernelGGL((qa_logits<D, kQtSmall, true>), grid, dim3(256), 0, stream, a);
    else if (rows)
      hipLaunchKernelGGL((qa_logits<D, QT, true>), grid, dim3(1024), 0, stream, a);
    else
      hipLaunchKernelGGL((qa_logits<D, QT, false>), grid, dim3(1024), 0, stream, a);
  };
  if (a.d == 128) logits(std::integral_constant<int, 128>{});
  else logits(std::integral_constant<int, 64>{});
  if (!rows)
    hipLaunchKernelGGL(qa_softmax, dim3((a.nb_total + 3) / 4, a.hq), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace fp
