// ctc_loss: the training objective of Sec. 3.2 - the negative log of Eq. 5 for a label sequence - and its gradient
// with respect to the logits, by the forward-backward recursions of the CTC paper the section cites.
//
// Two kinds of work, kept apart:
//   * the rows of logits ([V+1] floats per frame, 128 KB at V = 32000) are what costs HBM time.  Each is read
//     once and its gradient row written once, by one workgroup that holds the row in registers: ctc_row_kernel takes
//     the log-sum-exp, picks out the few log-probabilities the recursions need (the label's tokens and the
//     blank) and writes the row's softmax as the gradient; after the recursions the occupancies come off those
//     few entries.
//   * the recursions themselves are small and sequential in the frames, over the states of the extended sequence (blank,
//     y1, blank, ..., blank).  Few frames, or many sequences: ctc_short_kernel, a wavefront per sequence that runs
//     both recursions and subtracts the occupancies.  Otherwise ctc_dp_pipe_kernel, pipelined over blocks of
//     states, forward and backward at the same time; ctc_fix_kernel then forms the occupancies
//     gamma_t(s) = alpha_t(s) beta_t(s) / (p_t(z_s) P) where they are used.
// A token that occurs several times in a label has several states; their occupancies are added in label order
// by the thread of the first occurrence, so no atomic is needed and the result has the same bits on every run.
#include <type_traits>

#include "common.h"

namespace ctcspec {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) int i32x2;

constexpr int kCtcMaxLabels = 2047;  // with the blank 2048 positions: 2 per thread of ctc_row_kernel's 1024, 4 of its 512
constexpr int kCtcMaxRow = 16 * 1024 * 4;  // 65536 symbols: 16 16-byte loads per thread of a 1024-thread workgroup
constexpr int kCtcFixThreads = 256;
constexpr float kDpNarrow = -40.f;  // the recursion in doubles takes log2 p from here on

struct CtcParams {
  const float* logits;      // [B][T][Vp1]
  const int32_t* labels;    // [B][Lmax]
  const int32_t* label_len; // [B]
  const int32_t* frame_len; // [B]
  int B, T, Vp1, Lmax, blank;
  // workspace
  float* lpc;     // [B][T][Lmax + 1]: log2 p_t(y_j) for j < L, log2 p_t(blank) at Lmax
  float* ag;      // [B][T][2 Lmax + 2]: log2 alpha minus the frame's offset (state s at s; the last entry unused)
  float* bg;      // [B][T][2 Lmax + 2]: log2 beta minus the frame's offset, states counted from the last one
  double* coff_a; // [B][T][blocks]: offsets of the frame's log alpha values, one per block of pairs of states
  double* coff_b; // [B][T][blocks]: offsets of the frame's log beta values, pairs counted from the last one
  int blocks;     // blocks of pairs
  // the pipelined recursions (null otherwise)
  unsigned long long* edge;  // [B][2][T][blocks]: what a block hands to the next one, 0: not there yet
  int* wide;      // [B][T]: byte 0: a log-probability of the frame is not for the recursion in doubles, byte 1: nor in mantissas and exponents
  int* ticket;
  float wide_below;
  double* logp;   // [B]: log2 P(Y | X)
  int32_t* next;  // [B][Lmax]: next label position with the same token, -1: none
  int32_t* first; // [B][Lmax]: 1 when no earlier position holds the same token
  // outputs
  float* loss;    // [B]
  float* grad;    // [B][T][Vp1] or null
};

// The recursions run on base-2 logarithms (ctc_row_kernel hands out log2 p, the loss is turned back at the end):
// the exp2 and log2 instructions then need no scaling of their argument or result.
// log2(2^a + 2^b + 2^c) without a branch; -inf stands for an impossible state and any of the three may be -inf.
// The bare instructions carry an absolute error near 1e-7 here (the arguments of exp2 are <= 0, the argument of
// log2 is in [1, 3]; a term below 2^-126 of the largest is dropped), far below what the occupancies need.
__device__ __forceinline__ float ctc_log_add3(float a, float b, float c) {
  const float m = fmaxf(fmaxf(a, b), c);
  const float ms = m > -INFINITY ? m : 0.f;
  const float sum = __builtin_amdgcn_exp2f(a - ms) + __builtin_amdgcn_exp2f(b - ms) + __builtin_amdgcn_exp2f(c - ms);
  return ms + __builtin_amdgcn_logf(sum);  // the bare log2 instruction; sum = 0 gives -inf
}
// the reference value a frame's results are stored against: the largest value of the frame before, 0 when every
// state is impossible, so that offsets stay finite
__device__ __forceinline__ float frame_shift(float frame_max) { return frame_max > -INFINITY ? frame_max : 0.f; }
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
// floats per frame in the alpha and beta arrays: the 2 Lmax + 1 states and one more, so that pairs of states sit
// on 8-byte boundaries
__host__ __device__ __forceinline__ int ctc_state_pitch(int Lmax) { return 2 * Lmax + 2; }

// One workgroup per frame row, the row held in registers: every load of the row is in flight before the first
// is used, then log-sum-exp, the few log-probabilities the recursions need (the label's tokens and the blank),
// and the row's softmax written as the gradient.  Rows start at any multiple of 4 bytes (V + 1 is odd at
// V = 32000), so the up to three elements in front of the first 16-byte boundary and behind the last go through
// single lanes and the body through 16-byte loads and stores.
//
// Bound: HBM.  Two workgroups of 512 threads with 16 loads each share a compute unit, so that one row's loads run under
// the other's stores: 2048 x 8 rows of 32001 symbols 769 us a call (5.5 TB/s in and out) against 778 with one workgroup of
// 1024 threads.
template <int NV, int THREADS, int NY = 2>  // 16-byte loads and label positions per thread: NV * THREADS * 4 >= V + 1
__global__ __launch_bounds__(THREADS) void ctc_row_kernel(CtcParams p) {
  __shared__ float red[THREADS / 64];
  const int t = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int Tb = clampi(p.frame_len[b], 0, p.T);
  const size_t row0 = ((size_t)b * p.T + t) * p.Vp1;
  int head = (int)((4 - (row0 & 3)) & 3);
  head = head < p.Vp1 ? head : p.Vp1;
  const int nvec = (p.Vp1 - head) >> 2;
  const int tail0 = head + 4 * nvec;
  // the lane of an edge element: lanes 0..2 take the head, three others the tail
  constexpr int kTailLane = THREADS > 64 ? 64 : 32;
  int edge = -1;
  if (tid < head) edge = tid;
  else if (tid >= kTailLane && tid - kTailLane < p.Vp1 - tail0) edge = tail0 + tid - kTailLane;
  float* g = p.grad ? p.grad + row0 : nullptr;
  if (p.edge && t == 0 && b == 0 && tid == 0) *p.ticket = 0;  // whatever the sequence's length: every call counts from 0
  if (t >= Tb) {  // frames past the sequence: no gradient
    if (g) {
      f32x4* gv = (f32x4*)(g + head);
      for (int i = tid; i < nvec; i += THREADS) gv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (edge >= 0) g[edge] = 0.f;
    }
    return;
  }
  if (p.edge && tid == 0) p.wide[(size_t)b * p.T + t] = 0;  // (barriers follow before anything is set)
  const float* z = p.logits + row0;
  const f32x4* zv = (const f32x4*)(z + head);
  // the label's token ids first (Lmax < NY * THREADS), then the row, then the label's
  // logits while the row's cache lines are still on their way - asked for later they come from HBM a second time
  const int L = clampi(p.label_len[b], 0, p.Lmax);
  int yid[NY];
#pragma unroll
  for (int r = 0; r < NY; ++r) {
    const int j = tid + r * THREADS;
    yid[r] = j < L ? clampi(p.labels[(size_t)b * p.Lmax + j], 0, p.Vp1 - 1) : p.blank;
  }
  f32x4 x[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int i = tid + k * THREADS;
    x[k] = i < nvec ? zv[i] : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  }
  float xe = edge >= 0 ? z[edge] : -INFINITY;
  float zy[NY];
#pragma unroll
  for (int r = 0; r < NY; ++r) zy[r] = z[yid[r]];
  float mx = xe;
#pragma unroll
  for (int k = 0; k < NV; ++k) mx = fmaxf(fmaxf(fmaxf(mx, x[k][0]), fmaxf(x[k][1], x[k][2])), x[k][3]);
  mx = wave_max_f32(mx);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = red[0];
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) mx = fmaxf(mx, red[w]);
  // e = exp(x - max) stays in the registers: the softmax is e / sum
  xe = expf(xe - mx);
  float sum = xe;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[k][c] = expf(x[k][c] - mx);
      sum += x[k][c];
    }
  }
  sum = wave_sum_f32(sum);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = sum;
  __syncthreads();
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) sum += red[w];
  const float lse = mx + logf(sum);
  float* out = p.lpc + ((size_t)b * p.T + t) * (p.Lmax + 1);
  if (p.edge) {  // uniform
    for (int i = tid; i < 2 * p.blocks; i += THREADS) {
      const int dir = i >= p.blocks ? 1 : 0;
      p.edge[(((size_t)b * 2 + dir) * p.T + t) * p.blocks + (i - dir * p.blocks)] = 0ull;
    }
  }
  constexpr float kLog2e = 1.4426950408889634f;  // the recursions take base-2 logarithms
#pragma unroll
  for (int r = 0; r < NY; ++r) {
    const int j = tid + r * THREADS;
    const float l = (zy[r] - lse) * kLog2e;
    if (j < L) out[j] = l;
    else if (j == L) out[p.Lmax] = l;  // this thread's spare slot fetched the blank
    if (p.edge && j <= L && !(l >= kDpNarrow)) {  // cleared above; by bytes, so that no thread's mark undoes another's
      unsigned char* marks = (unsigned char*)(p.wide + (size_t)b * p.T + t);
      marks[0] = 1;
      if (l < p.wide_below && l > -INFINITY) marks[1] = 1;
    }
  }
  if (g) {
    const float inv = 1.f / sum;
    f32x4* gv = (f32x4*)(g + head);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = tid + k * THREADS;
      if (i < nvec) gv[i] = x[k] * inv;
    }
    if (edge >= 0) g[edge] = xe * inv;
  }
}

// log2(2^a + 2^b) without a branch (see ctc_log_add3)
__device__ __forceinline__ float ctc_log_add2(float a, float b) {
  const float m = fmaxf(a, b);
  const float ms = m > -INFINITY ? m : 0.f;
  const float sum = __builtin_amdgcn_exp2f(a - ms) + __builtin_amdgcn_exp2f(b - ms);
  return ms + __builtin_amdgcn_logf(sum);
}

// lane i gets lane i - 1's value, lane 0 `first`
__device__ __forceinline__ unsigned int lane_shift_up(unsigned int v, unsigned int first) {
  return (unsigned int)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}
// lane i gets lane i + 1's value, lane 63 `last`
__device__ __forceinline__ float lane_shift_down(float v, float last) {
  return __uint_as_float((unsigned int)__builtin_amdgcn_update_dpp((int)__float_as_uint(last), (int)__float_as_uint(v),
                                                                  0x130 /* wave_shl:1 */, 0xf, 0xf, false));
}

// ---- few frames, or many sequences with short labels (ctc_pipelined has the lines) -------------------------------------
// One wavefront per sequence, a lane per pair of states: pair q is the blank in front of label position q (state 2q) and
// that label's own state (2q + 1); pair L is the final blank alone.  Neighbours' values by lane shifts, no barrier.
// The forward recursion keeps its rows (in LDS when ROWS_IN_LDS, else in the workspace), the backward one forms the
// occupancies of a frame as it passes and takes them off the gradient row: one launch where the recursions, the links
// between equal tokens and the subtraction were three.  Each frame's values are held relative to the largest of the frame
// before, the offsets summed in double.  A label of 64 tokens or more cannot be reached in the fewer than 64 frames
// that ROWS_IN_LDS is for; otherwise the host sends only labels below 64 here.
// Bound: latency of the chain of frames and the scattered entries.  2048 sequences x 8 frames of 32001 symbols: 19.5 us,
// against 30 us in three kernels.
constexpr int kShortFrames = 64;  // frames that ctc_short_kernel keeps in LDS: fewer than this
constexpr int kShortBatch = 8;    // frames whose log-probabilities are fetched together

template <bool ROWS_IN_LDS>
__global__ __launch_bounds__(64) void ctc_short_kernel(CtcParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];  // [T][64] pairs, then [T] offsets
  const int b = blockIdx.x, q = threadIdx.x;
  const int L = clampi(p.label_len[b], 0, p.Lmax);
  const int Tb = clampi(p.frame_len[b], 0, p.T);
  if (Tb == 0) {
    if (q == 0) p.loss[b] = L == 0 ? 0.f : INFINITY;
    return;
  }
  const int LP = p.Lmax + 1, SP = ctc_state_pitch(p.Lmax);
  const float* __restrict__ lpc = p.lpc + (size_t)b * p.T * LP;
  const int32_t* __restrict__ y = p.labels + (size_t)b * p.Lmax;
  double logP = -(double)INFINITY;
  const bool has_label = q < L;
  const int col = has_label ? q : p.Lmax;
  const int tok = has_label ? y[q] : -1;
  const int tok_before = (int)lane_shift_up((unsigned)tok, 0u);
  const bool skip_in = q >= 1 && has_label && tok != tok_before;
  f32x2* row = ROWS_IN_LDS ? (f32x2*)rows_lds + q : (f32x2*)(p.ag + (size_t)b * p.T * SP) + q;
  double* offsets = ROWS_IN_LDS ? (double*)(rows_lds + (size_t)p.T * 64 * 8) : p.coff_a + (size_t)b * p.T;
  const size_t row_step = ROWS_IN_LDS ? 64 : SP / 2;
  const bool keeps = ROWS_IN_LDS || q <= L;
  if (L < 64) {
    float a_blank = q == 0 ? 0.f : -INFINITY, a_label = -INFINITY;  // before the first frame
    float frame_max = 0.f;
    double offset = 0.0;
    for (int t0 = 0; t0 < Tb; t0 += kShortBatch) {
      float lp[kShortBatch], lb[kShortBatch];
#pragma unroll
      for (int i = 0; i < kShortBatch; ++i) {
        const int t = t0 + i < Tb ? t0 + i : Tb - 1;
        lp[i] = lpc[(size_t)t * LP + col];
        lb[i] = lpc[(size_t)t * LP + p.Lmax];
      }
#pragma unroll
      for (int i = 0; i < kShortBatch; ++i) {
        const int t = t0 + i;
        if (t >= Tb) break;
        const float before = __uint_as_float(lane_shift_up(__float_as_uint(a_label), 0xff800000u));
        const float shift = t > 0 ? frame_shift(frame_max) : 0.f;
        offset += (double)shift;
        const float nb = ctc_log_add2(a_blank, before);
        const float nl = ctc_log_add3(a_label, a_blank, skip_in ? before : -INFINITY);
        a_blank = q <= L ? nb + (lb[i] - shift) : -INFINITY;
        a_label = has_label ? nl + (lp[i] - shift) : -INFINITY;
        if (p.grad && keeps) row[(size_t)t * row_step] = f32x2{a_blank, a_label};
        if (p.grad && q == 0) offsets[t] = offset;
        frame_max = wave_max_f32(fmaxf(a_blank, a_label));
      }
    }
    const float before = __uint_as_float(lane_shift_up(__float_as_uint(a_label), 0xff800000u));
    const float tail = __shfl(ctc_log_add2(a_blank, before), L, 64);
    logP = offset + (double)tail;  // base 2; -inf when the label cannot be reached
  } else {  // it cannot; but logits that are no numbers say so
    bool nan = false;
    for (int t = q; t < Tb; t += 64) nan |= lpc[(size_t)t * LP + p.Lmax] != lpc[(size_t)t * LP + p.Lmax];
    if (__ballot(nan) != 0ull) logP = (double)NAN;
  }
  if (q == 0) p.loss[b] = (float)(-logP * 0.6931471805599453);
  if (!p.grad) return;
  float* __restrict__ g = p.grad + (size_t)b * p.T * p.Vp1;
  if (!(logP > -(double)INFINITY)) {  // a label that cannot be reached has no gradient
    const size_t at = (size_t)b * p.T * p.Vp1, n = (size_t)Tb * p.Vp1;
    size_t head = (4 - (at & 3)) & 3;
    head = head < n ? head : n;
    const size_t body = (n - head) / 4;
    if ((size_t)q < head) g[q] = 0.f;
    f32x4* gv = (f32x4*)(g + head);
    for (size_t i = q; i < body; i += 64) gv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (head + 4 * body + q < n) g[head + 4 * body + q] = 0.f;
    return;
  }
  // positions with this lane's token: the first of them adds the occupancies of all, in label order
  unsigned long long later = 0ull;
  bool first = has_label;
  for (int i = 0; i < L; ++i) {
    const int ti = (int)readlane_u32((unsigned)tok, i);
    const bool same = has_label && ti == tok;
    if (same && i > q) later |= 1ull << i;
    if (same && i < q) first = false;
  }
  if (!first) later = 0ull;
  const bool repeats = __ballot(later != 0ull) != 0ull;
  const int entry = clampi(tok, 0, p.Vp1 - 1);
  const int tok_after = (int)__float_as_uint(lane_shift_down(__uint_as_float((unsigned)tok), 0.f));
  const bool skip_out = q + 1 < L && tok != tok_after;
  float b_blank = q == L ? 0.f : -INFINITY, b_label = -INFINITY;  // behind the last frame
  float frame_max = 0.f;
  double offset = 0.0;
  if constexpr (!ROWS_IN_LDS) __syncthreads();  // the rows have reached memory (one wavefront: its own stores)
  for (int t0 = Tb - 1; t0 >= 0; t0 -= kShortBatch) {
    float lp[kShortBatch], lb[kShortBatch];
    f32x2 ar[kShortBatch];
    double ca[kShortBatch];
#pragma unroll
    for (int i = 0; i < kShortBatch; ++i) {
      const int t = t0 - i >= 0 ? t0 - i : 0;
      lp[i] = lpc[(size_t)t * LP + col];
      lb[i] = lpc[(size_t)t * LP + p.Lmax];
      ar[i] = keeps ? row[(size_t)t * row_step] : f32x2{-INFINITY, -INFINITY};
      ca[i] = offsets[t];
    }
#pragma unroll
    for (int i = 0; i < kShortBatch; ++i) {
      const int t = t0 - i;
      if (t < 0) break;
      const float next_blank = lane_shift_down(b_blank, -INFINITY), next_label = lane_shift_down(b_label, -INFINITY);
      const float shift = t < Tb - 1 ? frame_shift(frame_max) : 0.f;
      offset += (double)shift;
      const float nb = ctc_log_add2(b_blank, b_label);
      const float nl = ctc_log_add3(b_label, next_blank, skip_out ? next_label : -INFINITY);
      b_blank = q <= L ? nb + (lb[i] - shift) : -INFINITY;  // beta_t(s) includes p_t(z_s)
      b_label = has_label ? nl + (lp[i] - shift) : -INFINITY;
      frame_max = wave_max_f32(fmaxf(b_blank, b_label));
      const float z = (float)(logP - ca[i] - offset);
      auto gamma = [&](float a, float bt, float l) {
        return (a > -INFINITY && bt > -INFINITY) ? exp2f(a + bt - l - z) : 0.f;
      };
      const float gb = gamma(ar[i][0], b_blank, lb[i]), gl = gamma(ar[i][1], b_label, lp[i]);
      // the occupancies of a frame sum to one: what is left of the recursions' rounding is mostly common to all of them
      const float blanks = wave_sum_f32(gb), total = blanks + wave_sum_f32(gl);
      const float inv = total > 0.f ? 1.f / total : 1.f;
      float tot = gl;
      if (repeats) {
        unsigned long long m = later;
        while (__ballot(m != 0ull) != 0ull) {
          const float o = __shfl(gl, m ? __ffsll((long long)m) - 1 : 0, 64);
          if (m) tot += o;
          m &= m - 1;
        }
      }
      // the entries are written, not updated: the softmax is formed again from the log-probability at hand
      float* gt = g + (size_t)t * p.Vp1;
      if (q == 0) gt[p.blank] = exp2f(lb[i]) - blanks * inv;
      if (first && entry != p.blank) gt[entry] = exp2f(lp[i]) - tot * inv;
    }
  }
}

// per sequence: links between the label positions that hold the same token.  The label is staged in LDS; one
// wavefront per position looks for the nearest later position with the same token and for any earlier one, 256
// candidates per round trip to LDS.  The positions of a sequence are dealt to `parts` workgroups; every entry
// of next and first is written by the wavefront that owns the position, so the workgroups share nothing.
__device__ void ctc_links(const CtcParams& p, int b, int part, int parts, int32_t* ytok) {
  const int tid = threadIdx.x, n = blockDim.x;
  const int lane = tid & 63, nwaves = n >> 6;
  const int wave = (tid >> 6) + nwaves * part, stride = nwaves * parts;
  const int L = clampi(p.label_len[b], 0, p.Lmax);
  int32_t* next = p.next + (size_t)b * p.Lmax;
  int32_t* first = p.first + (size_t)b * p.Lmax;
  for (int j = tid; j < L; j += n) ytok[j] = p.labels[(size_t)b * p.Lmax + j];
  __syncthreads();
  for (int j = wave; j < p.Lmax; j += stride) {
    int found = -1;
    bool earlier = false;
    if (j < L) {
      const int tok = ytok[j];
      for (int i0 = j + 1; i0 < L && found < 0; i0 += 256) {
        unsigned long long hits[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + 64 * r + lane;
          hits[r] = __ballot(i < L && ytok[i] == tok);
        }
#pragma unroll
        for (int r = 3; r >= 0; --r)
          if (hits[r]) found = i0 + 64 * r + __ffsll((long long)hits[r]) - 1;  // the lowest group with a hit wins
      }
      for (int i0 = 0; i0 < j && !earlier; i0 += 256) {
        unsigned long long any = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + 64 * r + lane;
          any |= __ballot(i < j && ytok[i] == tok);
        }
        earlier = any != 0;
      }
    }
    if (lane == 0) {
      next[j] = found;
      first[j] = (j < L && !earlier) ? 1 : 0;
    }
  }
}

// ---- the recursions, pipelined over blocks of states ---------------------------------------------------------------
// A state depends on itself and on the two states before it, in the frame before: dependences run one way through the
// states, so the states are cut into blocks of 64 pairs (a lane per pair) and a block may run as far behind the one before
// it as it likes.  A workgroup of four or six wavefronts owns a block of one sequence and direction:
//   wavefront 0 runs the recursion over kDpFrames frames, neighbours by a lane shift, no barrier between frames;
//   wavefront 1 fetches and converts the next frames' probabilities and waits for the values that the block before hands over
//               (the label state of its last pair, frame by frame);
//   the others  hand over this block's, convert the frames before to what ctc_fix_kernel reads and write them, four or
//               eight frames each (that is more instructions a frame than the recursion itself).
// One barrier per kDpFrames frames.  A value handed over is one 64-bit word (never 0) stored and loaded with relaxed
// device-scope atomics: nothing has to be fenced.  Blocks take their number from a ticket in dependence order, so the
// block that a workgroup waits for has always been started before it.
//
// The values are linear: doubles against a power of two of the state's own, which stays for the kDpFrames frames of a step.  A frame
// is three sums and two products then, with a factor - the scale of the state before against this one's - on what comes from there.
// A state's scale is its value's exponent, or the scale of a state before it less kDpDecay where that is more, so that what arrives
// within the step does not overflow (a factor of 2^40 and three terms a frame: 2^660).  With log2 p >= kDpNarrow a value that
// is at most kDpRoom below its scale keeps all of its bits in sixteen frames.  One that lies further below would be lost, and may be the one
// that counts in the end: a path that is ahead may be the only one that still reaches the last state in time, and one that waits
// may be the one whose token comes again.  A factor below 2^-1022 would lose bits too.
// Where the values before a step do not allow for it, the block takes the step in mantissas and exponents (below): one
// step in a hundred where each token is certain in one frame and at 2^-35 elsewhere, none with random logits.  (Scales of the lane, for
// both of its states, and no such look: losses off by up to a third, and infinite ones.)
//
// Sequences with a lower log-probability, one that is not a number or a probability of 0 - which may end, within a step, the larger value
// beside which another one was left out - take all steps so.  They hold mantissa and exponent (m in [0.5, 1), value m * 2^e):
// three ldexp and a sum take the place of three exp2 and a log2, the relative error of a step is 2^-24 whatever the length of
// the sequence, and no frame maximum has to be known.  An impossible state has e = kDpFloor; everything below kDpImpossible counts as
// impossible.
//
// Sequences with a finite log-probability so low that exponents could get there (wide_below: about -32768, a token that
// is masked out by a large finite number) run the same pipeline in the log domain (LOG): a block holds its values
// against a reference of its own - the larger of its largest value and of the one handed over, in the frame before - so no
// block waits for another's maximum either.  The reference is a double, the values are floats against it, and what is
// handed over is the whole value as a double.
//
// The backward recursion is the forward one over the mirrored sequence (last frame and last state first).
//
// Bound: instruction issue of wavefront 0.  Measured, 4 sequences of 2048 frames
// with up to 1024 labels and 1536 to 2048 frames: 191 us - 1.1 us a step of sixteen frames, and three steps that each block runs behind the one before; in mantissas
// and exponents, about 40 instructions a frame, 227.  One workgroup of 1024 threads per sequence and direction, log domain, a barrier and a
// frame maximum per frame took 1221 us, and its gradient was five times as far from the float64 one (5e-6 against 9e-7).
// In the log domain a frame takes about 0.25 us: 4 x 2048 frames of 1001 symbols, 1024 labels, the blank masked with -1e9,
// 585 us a call; 8 x 512 frames, 100 labels 123 us.  One workgroup per sequence and direction, a barrier and a frame
// maximum per frame: 1794 and 258 us with 1024 threads, 2400 and 223 us with 256 and the pairs in registers.
constexpr int kDpFrames = 16;
constexpr int kDpPairs = 64;
constexpr int dp_threads(int writers) { return 64 * (2 + writers); }  // writers: wavefronts that convert and write the rows
constexpr int kDpDecay = 40;               // exponents by which a state's scale may lie below that of a state before it
constexpr int kDpRoom = 1010 - kDpFrames * kDpDecay;             // ... a value below its scale
enum DpForm { kDpDouble, kDpMantissa, kDpLog };
static_assert(kDpDecay >= -kDpNarrow && kDpFrames * (kDpDecay + 2) < 1022 && kDpRoom > 0, "values stay within a double's range over a step");
constexpr int kDpFloor = -(1 << 30);
constexpr int kDpMantissas = 1 << 30;      // no exponent
constexpr int kDpZeroP = -(1 << 29);       // exponent of a probability that is 0
constexpr int kDpImpossible = -(1 << 28);
constexpr int kDpMaxPolls = 1 << 20;       // about a second; a wait is over long before

static_assert(kCtcMaxLabels * 4 <= 2 * kDpFrames * 64 * 16, "the links' label fits DpShared");
struct DpShared {
  u32x2 in[2][kDpFrames][64];   // label probability (m, e) per lane
  u32x4 uni[2][kDpFrames];      // blank probability (m, e), handed-over value (m, e) of the frame before
  u32x4 out[2][kDpFrames][64];  // blank (m, e), label (m, e) after the frame
  // kDpDouble: `in` and the first half of `uni` are doubles, `out` two of them, and
  i32x2 scale[2][64];           // the states' exponents; kDpMantissas: the step was taken in mantissas
  int highest[2];               // largest exponent handed over
  double edge[kDpFrames];       // the handed-over values against the largest exponent
};

__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// the maximum over the wavefront of each of N values, step by step side by side
template <int N>
__device__ __forceinline__ void wave_max_i32(int (&v)[N]) {
#define CTCSPEC_MAX_STEP(ROT) \
  _Pragma("unroll") for (int u = 0; u < N; ++u) v[u] = imax(v[u], (int)dpp_row_ror<ROT>((unsigned)v[u]));
  CTCSPEC_MAX_STEP(1)
  CTCSPEC_MAX_STEP(2)
  CTCSPEC_MAX_STEP(4)
  CTCSPEC_MAX_STEP(8)
#undef CTCSPEC_MAX_STEP
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int a = (int)readlane_u32((unsigned)v[u], 0), b = (int)readlane_u32((unsigned)v[u], 16);
    const int c = (int)readlane_u32((unsigned)v[u], 32), d = (int)readlane_u32((unsigned)v[u], 48);
    v[u] = imax(imax(a, b), imax(c, d));
  }
}

__device__ __forceinline__ double as_double(unsigned int lo, unsigned int hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
struct DpValue { float m; int e; };
// log2 p -> p.  Not a number stays one in m, with an exponent that sinks nothing: it is no impossible state.
__device__ __forceinline__ DpValue dp_probability(float l) {
  const float f = floorf(l);
  DpValue v;
  v.m = l == -INFINITY ? 0.5f : 0.5f * __builtin_amdgcn_exp2f(l - f);  // 2^(l - f) in [1, 2)
  v.e = l > -INFINITY ? (int)f + 1 : (l == -INFINITY ? kDpZeroP : 0);
  return v;
}
__device__ __forceinline__ DpValue dp_scaled(float sum, int e, float pm, int pe) {
  const float s = sum * pm;
  DpValue v;
  v.m = __builtin_amdgcn_frexp_mantf(s);
  v.e = imax(e + __builtin_amdgcn_frexp_expf(s) + pe, kDpFloor);
  return v;
}

// a double as mantissa and exponent, against 2^scale; zero has no exponent
__device__ __forceinline__ int dp_exponent(double v, int scale) { return v == 0.0 ? kDpFloor : __builtin_amdgcn_frexp_exp(v) + scale; }
__device__ __forceinline__ DpValue dp_value(double v, int scale) {
  DpValue r;
  r.m = v == 0.0 ? 0.5f : (float)__builtin_amdgcn_frexp_mant(v);
  r.e = dp_exponent(v, scale);
  return r;
}
__device__ __forceinline__ double lane_shift_up(double v, double first) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(v), y = (unsigned long long)__double_as_longlong(first);
  return as_double(lane_shift_up((unsigned)x, (unsigned)y), lane_shift_up((unsigned)(x >> 32), (unsigned)(y >> 32)));
}
// join over the lanes up to and with this one
template <typename F>
__device__ __forceinline__ int wave_prefix(int v, int nothing, F&& join) {
#define CTCSPEC_PREFIX(CTRL, ROWS) v = join(v, __builtin_amdgcn_update_dpp(nothing, v, CTRL, ROWS, 0xf, false));
  CTCSPEC_PREFIX(0x111, 0xf)  // row_shr:1, 2, 4, 8
  CTCSPEC_PREFIX(0x112, 0xf)
  CTCSPEC_PREFIX(0x114, 0xf)
  CTCSPEC_PREFIX(0x118, 0xf)
  CTCSPEC_PREFIX(0x142, 0xa)  // row_bcast:15 into rows 1 and 3
  CTCSPEC_PREFIX(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef CTCSPEC_PREFIX
  return v;
}

// One block of states of one sequence and direction, by a workgroup.  FORM: what holds the values (see above).
template <int FORM, int WRITERS>
__device__ __forceinline__ void ctc_block(const CtcParams& p, DpShared& sh, int directions, int block, int b, bool backward,
                                          int L, int Tb) {
  constexpr bool LOG = FORM == kDpLog, DOUBLE = FORM == kDpDouble;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool last_block = (block + 1) * kDpPairs > L;
  const int q = block * kDpPairs + lane;
  const int32_t* y = p.labels + (size_t)b * p.Lmax;
  const int j = backward ? L - 1 - q : q, jb = backward ? L - q : q - 1;  // label of the pair, of the pair before
  const bool has_label = q < L;
  const int SP = ctc_state_pitch(p.Lmax), LP = p.Lmax + 1;
  const float* lpc = p.lpc + (size_t)b * p.T * LP;
  unsigned long long* edge = p.edge + ((size_t)b * 2 + (backward ? 1 : 0)) * p.T * p.blocks;
  const int chunks = (Tb + kDpFrames - 1) / kDpFrames;
  // frame i of the recursion (0 .. Tb-1) is frame i or Tb - 1 - i of the sequence
  auto frame = [&](int i) { return backward ? Tb - 1 - i : i; };
  bool lost = false;  // a wait was given up: not a number from there on
  // a value of 0 - 0.5 * 2^kDpFloor; LOG: -inf as a double - and one that is not a number
  constexpr unsigned long long kNothing = LOG ? 0xfff0000000000000ull : ((unsigned long long)(unsigned)kDpFloor << 32) | 0x3f000000u;
  constexpr unsigned long long kLost = LOG ? 0x7ff8000000000000ull : 0x7fc00000ull;
  auto look = [&](int i) -> unsigned long long {  // per lane: the value of frame i from the block before, 0: not there yet
    if (block == 0 || i < 0 || i >= Tb) return kNothing;
    return __hip_atomic_load(edge + (size_t)frame(i) * p.blocks + (block - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto wait_for = [&](int i, unsigned long long v) -> unsigned long long {  // v: what look(i) has given before
    for (int polls = 0; !v && !lost; ++polls) {
      __builtin_amdgcn_s_sleep(1);
      v = look(i);
      lost = polls >= kDpMaxPolls;
    }
    return v ? v : kLost;
  };

  if (wave == 0) {
    const bool skip = q >= 1 && q < L && y[j] != y[jb];
    // before the first frame: all of the weight in the first blank
    float bm = 0.5f, lm = 0.5f;
    int be = q == 0 ? 1 : kDpFloor, le = kDpFloor;
    // LOG: the two states against off, the largest of the block against off
    float bl = q == 0 ? 0.f : -INFINITY, ll = -INFINITY, top = block == 0 ? 0.f : -INFINITY;
    double off = 0.0;
    // DOUBLE: the two states against 2^bscale and 2^lscale
    double db = q == 0 ? 1.0 : 0.0, dl = 0.0;
    int bscale = 0, lscale = 0;
    // the decay from the label handed over to this lane's
    const int decay = wave_prefix(skip ? kDpDecay : 2 * kDpDecay, 0, [](int x, int y) { return x + y; });
    const int skip_room = skip ? 1022 : 1 << 30;
    lds_barrier();  // LDS only: loads and stores of memory stay in flight
    // a step in doubles; false, and nothing has changed: the values do not allow for it
    auto double_frames = [&](int ch, auto partial) __attribute__((always_inline)) -> bool {
      const int buf = ch & 1;
      double pl[kDpFrames], pb[kDpFrames], edge_in[kDpFrames];
      // all of the step's probabilities are asked for first, behind what the scales need: an LDS read takes as long as a frame
      const int highest = sh.highest[buf];
      const u32x4 un = sh.uni[buf][lane & (kDpFrames - 1)];  // (four lanes a frame)
      const int handed = (int)un[3];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) {
        pl[f] = *(const double*)&sh.in[buf][f][lane];
        pb[f] = *(const double*)&sh.uni[buf][f];
      }
      __builtin_amdgcn_sched_barrier(0);
      const int be = dp_exponent(db, bscale), le = dp_exponent(dl, lscale);
      int top = imax(le, be - kDpDecay) + decay;
      top = lane == 0 ? imax(top, highest) : top;
      const int lnext = wave_prefix(top, kDpFloor, imax) - decay;
      const int before = (int)lane_shift_up((unsigned)lnext, (unsigned)highest);
      const int bnext = imax(be, before - kDpDecay);
      // by how much one is more than `room` above the other, as a number from 0 on; more than any such where it is not, or the other is a
      // value of 0 (kDpFloor)
      auto above = [](int a, int b, int room) { return (unsigned)(a - b - room); };
      auto least = [](unsigned a, unsigned b) { return a < b ? a : b; };
      const unsigned excess = least(least(above(highest, handed, kDpRoom), least(above(bnext, be, kDpRoom), above(lnext, le, kDpRoom))),
                                    least(above(bnext, before, 1022), least(above(lnext, bnext, 1022), above(lnext, before, skip_room))));
      if (__builtin_amdgcn_ballot_w64(excess < (unsigned)-kDpImpossible) != 0ull) {
        sh.scale[buf][lane] = i32x2{kDpMantissas, kDpMantissas};
        return false;
      }
      db = __builtin_amdgcn_ldexp(db, bscale - bnext);
      dl = __builtin_amdgcn_ldexp(dl, lscale - lnext);
      bscale = bnext;
      lscale = lnext;
      sh.scale[buf][lane] = i32x2{bscale, lscale};
      // factors: the label before into the blank and into the label, the blank into the label
      const double from_before = __builtin_amdgcn_ldexp(1.0, before - bscale), from_blank = __builtin_amdgcn_ldexp(1.0, bscale - lscale);
      const double from_label = skip ? __builtin_amdgcn_ldexp(1.0, before - lscale) : 0.0;
      if (lane < kDpFrames) sh.edge[lane] = handed < kDpImpossible ? 0.0 : __builtin_amdgcn_ldexp((double)__uint_as_float(un[2]), handed - highest);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) edge_in[f] = sh.edge[f];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) {
        const bool run = !decltype(partial)::value || ch * kDpFrames + f < Tb;  // frames past the end change nothing
        const double x = lane_shift_up(dl, edge_in[f]);
        const double nb = __builtin_fma(from_before, x, db) * pb[f];
        const double nl = __builtin_fma(from_label, x, __builtin_fma(from_blank, db, dl)) * pl[f];
        db = run ? nb : db;
        dl = run ? nl : dl;
        const unsigned long long vb = (unsigned long long)__double_as_longlong(db), vl = (unsigned long long)__double_as_longlong(dl);
        sh.out[buf][f][lane] = u32x4{(unsigned)vb, (unsigned)(vb >> 32), (unsigned)vl, (unsigned)(vl >> 32)};
      }
      return true;
    };
    auto frames_of = [&](int ch, auto partial) __attribute__((always_inline)) {
      const int buf = ch & 1;
      if constexpr (DOUBLE) {
        if (double_frames(ch, partial)) return;
        const DpValue vb = dp_value(db, bscale), vl = dp_value(dl, lscale);
        bm = vb.m; be = vb.e; lm = vl.m; le = vl.e;
      }
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) {
        u32x2 pr = sh.in[buf][f][lane];
        u32x4 un = sh.uni[buf][f];
        const bool run = !decltype(partial)::value || ch * kDpFrames + f < Tb;  // frames past the end change nothing
        if constexpr (DOUBLE) {  // doubles of 2^kDpNarrow and above, 0 where there is no label
          const float pl = (float)as_double(pr[0], pr[1]);
          pr = u32x2{__float_as_uint(has_label ? pl : 0.5f), has_label ? 0u : (unsigned)kDpZeroP};
          un[0] = __float_as_uint((float)as_double(un[0], un[1]));
          un[1] = 0u;
        }
        if constexpr (LOG) {
          const double h = as_double(un[2], un[3]);
          double ref = fmax(off + (double)top, h);
          ref = ref > -(double)INFINITY ? ref : off;
          // (a block without any value may be far from what arrives; the floor keeps -inf - shift what it is)
          const float shift = fmaxf((float)(ref - off), -3.0e38f), first = (float)(h - ref);
          const float b0 = bl - shift, l0 = ll - shift;
          const float before = __uint_as_float(lane_shift_up(__float_as_uint(l0), __float_as_uint(first)));
          const float nb = ctc_log_add2(b0, before) + __uint_as_float(un[0]);
          const float nl = ctc_log_add3(l0, b0, skip ? before : -INFINITY) + __uint_as_float(pr[0]);
          const float largest = wave_max_f32(fmaxf(nb, nl));
          bl = run ? nb : bl;
          ll = run ? nl : ll;
          top = run ? largest : top;
          off = run ? ref : off;
          const unsigned long long bits = (unsigned long long)__double_as_longlong(off);
          sh.out[buf][f][lane] = u32x4{__float_as_uint(bl), __float_as_uint(ll), (unsigned)bits, (unsigned)(bits >> 32)};
          continue;
        }
        const float xm = __uint_as_float(lane_shift_up(__float_as_uint(lm), un[2]));
        const int xe = (int)lane_shift_up((unsigned)le, un[3]);
        const int e0 = imax(be, xe);
        const float s0 = __builtin_amdgcn_ldexpf(bm, be - e0) + __builtin_amdgcn_ldexpf(xm, xe - e0);
        const int ke = skip ? xe : kDpFloor;
        const int e1 = imax(imax(le, be), ke);
        const float s1 = __builtin_amdgcn_ldexpf(lm, le - e1) + __builtin_amdgcn_ldexpf(bm, be - e1) +
                         __builtin_amdgcn_ldexpf(xm, ke - e1);
        const DpValue nb = dp_scaled(s0, e0, __uint_as_float(un[0]), (int)un[1]);
        const DpValue nl = dp_scaled(s1, e1, __uint_as_float(pr[0]), (int)pr[1]);
        bm = run ? nb.m : bm;
        be = run ? nb.e : be;
        lm = run ? nl.m : lm;
        le = run ? nl.e : le;
        sh.out[buf][f][lane] = u32x4{__float_as_uint(bm), (unsigned)be, __float_as_uint(lm), (unsigned)le};
      }
      if constexpr (DOUBLE) {
        db = be < kDpImpossible ? 0.0 : (double)bm;
        dl = le < kDpImpossible ? 0.0 : (double)lm;
        bscale = be;
        lscale = le;
      }
    };
    for (int ch = 0; ch <= chunks; ++ch) {
      if ((ch + 1) * kDpFrames <= Tb) frames_of(ch, std::false_type{});
      else if (ch < chunks) frames_of(ch, std::true_type{});
      lds_barrier();
    }
    if constexpr (DOUBLE) {
      const DpValue vb = dp_value(db, bscale), vl = dp_value(dl, lscale);
      bm = vb.m; be = vb.e; lm = vl.m; le = vl.e;
    }
    if (!backward && last_block) {
      // P = the last blank + the label before it
      unsigned long long v = kNothing;
      if (block > 0 && L == block * kDpPairs) v = wait_for(Tb - 1, look(Tb - 1));
      const unsigned int first0 = (unsigned)v, first1 = (unsigned)(v >> 32);
      const float xm = __uint_as_float(lane_shift_up(__float_as_uint(LOG ? ll : lm), first0));
      const int xe = (int)lane_shift_up((unsigned)le, first1);
      if (q == L) {
        double logP;
        if constexpr (LOG) {
          const double last = off + (double)bl, before = lane ? off + (double)xm : as_double(first0, first1);
          const double m = fmax(last, before);
          logP = m > -(double)INFINITY ? m + (double)__builtin_amdgcn_logf(__builtin_amdgcn_exp2f((float)(last - m)) +
                                                                           __builtin_amdgcn_exp2f((float)(before - m)))
                                       : last + before;  // -inf, or not a number
        } else {
          const int e = imax(be, xe);
          const float s = __builtin_amdgcn_ldexpf(bm, be - e) + __builtin_amdgcn_ldexpf(xm, xe - e);
          logP = e < kDpImpossible && s == s ? -(double)INFINITY : (double)e + (double)__builtin_amdgcn_logf(s);
        }
        p.loss[b] = (float)(-logP * 0.6931471805599453);
        p.logp[b] = logP;
      }
    }
  } else if (wave == 1) {
    const int col = has_label ? j : p.Lmax;
    // log-probabilities come two chunks ahead, handed-over values one: a chunk takes less than a load from memory
    float lp[2][kDpFrames], lb[2] = {0.f, 0.f};
    unsigned long long early = 0ull;
    auto fetch = [&](int ch, auto set) __attribute__((always_inline)) {
      constexpr int S = decltype(set)::value;
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) {
        const int i = ch * kDpFrames + f;
        lp[S][f] = lpc[(size_t)frame(i < Tb ? i : Tb - 1) * LP + col];
      }
      const int i = ch * kDpFrames + (lane & (kDpFrames - 1));
      lb[S] = lpc[(size_t)frame(i < Tb ? i : Tb - 1) * LP + p.Lmax];
    };
    auto look_early = [&](int ch) __attribute__((always_inline)) {
      if (lane < kDpFrames) early = look(ch * kDpFrames + lane - 1);
    };
    // chunk ch, whose log-probabilities are in set S; asks for the handed-over values of the next and fills the set again
    auto prepare = [&](int ch, auto set) __attribute__((always_inline)) {
      constexpr int S = decltype(set)::value;
      const int buf = ch & 1;
#pragma unroll
      for (int f = 0; f < kDpFrames; ++f) {
        if constexpr (LOG) {
          sh.in[buf][f][lane] = u32x2{__float_as_uint(has_label ? lp[S][f] : -INFINITY), 0u};
        } else if constexpr (DOUBLE) {
          const unsigned long long v = (unsigned long long)__double_as_longlong(has_label ? (double)__builtin_amdgcn_exp2f(lp[S][f]) : 0.0);
          sh.in[buf][f][lane] = u32x2{(unsigned)v, (unsigned)(v >> 32)};
        } else {
          const DpValue v = dp_probability(lp[S][f]);
          sh.in[buf][f][lane] = u32x2{__float_as_uint(v.m), has_label ? (unsigned)v.e : (unsigned)kDpZeroP};
        }
      }
      const DpValue vb = LOG ? DpValue{lb[S], 0} : dp_probability(lb[S]);
      if (lane < kDpFrames) {
        const unsigned long long h = wait_for(ch * kDpFrames + lane - 1, early);
        if constexpr (DOUBLE) {
          const unsigned long long v = (unsigned long long)__double_as_longlong((double)__builtin_amdgcn_exp2f(lb[S]));
          sh.uni[buf][lane] = u32x4{(unsigned)v, (unsigned)(v >> 32), (unsigned)h, (unsigned)(h >> 32)};
          int e = (int)(h >> 32);
          e = imax(e, (int)dpp_row_ror<1>((unsigned)e));
          e = imax(e, (int)dpp_row_ror<2>((unsigned)e));
          e = imax(e, (int)dpp_row_ror<4>((unsigned)e));
          e = imax(e, (int)dpp_row_ror<8>((unsigned)e));
          if (lane == 0) sh.highest[buf] = e;
        } else {
          sh.uni[buf][lane] = u32x4{__float_as_uint(vb.m), (unsigned)vb.e, (unsigned)h, (unsigned)(h >> 32)};
        }
      }
      if (ch + 1 < chunks) look_early(ch + 1);
      if (ch + 2 < chunks) fetch(ch + 2, set);
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    fetch(0, Even{});
    look_early(0);
    if (chunks > 1) fetch(1, Odd{});
    prepare(0, Even{});
    lds_barrier();
    for (int ch = 0; ch <= chunks; ch += 2) {
      if (ch + 1 < chunks) prepare(ch + 1, Odd{});
      lds_barrier();
      if (ch + 1 > chunks) break;
      if (ch + 2 < chunks) prepare(ch + 2, Even{});
      lds_barrier();
    }
  } else {
    float* g = (backward ? p.bg : p.ag) + (size_t)b * p.T * SP + 2 * q;
    double* coff = (backward ? p.coff_b : p.coff_a) + (size_t)b * p.T * p.blocks + block;
    lds_barrier();
    for (int ch = 0; ch <= chunks; ++ch) {
      if (ch > 0) {
        const int buf = (ch - 1) & 1, i0 = (ch - 1) * kDpFrames;
        if (wave == 2 && !last_block && lane < kDpFrames && i0 + lane < Tb) {
          const u32x4 v = sh.out[buf][lane][63];
          unsigned long long word = ((unsigned long long)v[3] << 32) | v[2];
          if constexpr (LOG) {
            word = (unsigned long long)__double_as_longlong(as_double(v[2], v[3]) + (double)__uint_as_float(v[1]));
            word = word ? word : 1ull << 63;  // -0.0
          }
          if constexpr (DOUBLE) {
            const int scale = sh.scale[buf][63][1];
            const DpValue l = dp_value(as_double(v[2], v[3]), scale);
            word = scale != kDpMantissas ? ((unsigned long long)(unsigned)l.e << 32) | __float_as_uint(l.m) : word;
          }
          __hip_atomic_store(edge + (size_t)frame(i0 + lane) * p.blocks + block, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (directions == 2) {  // (the loss alone needs no rows)
          constexpr int kGroup = 4;  // frames side by side: the chain of a frame is long and narrow
#pragma unroll
          for (int f0 = 0; f0 < kDpFrames / WRITERS; f0 += kGroup) {
            const int first = (wave - 2) * (kDpFrames / WRITERS) + f0;
            u32x4 v[kGroup];
            int ref[kGroup];
#pragma unroll
            for (int u = 0; u < kGroup; ++u) v[u] = sh.out[buf][first + u][lane];
            i32x2 scale = {0, 0};
            if constexpr (DOUBLE) scale = sh.scale[buf][lane];
            if (DOUBLE && __builtin_amdgcn_readfirstlane(scale[0]) != kDpMantissas) {
#pragma unroll
              for (int u = 0; u < kGroup; ++u) {
                const DpValue vb = dp_value(as_double(v[u][0], v[u][1]), scale[0]), vl = dp_value(as_double(v[u][2], v[u][3]), scale[1]);
                v[u] = u32x4{__float_as_uint(vb.m), (unsigned)vb.e, __float_as_uint(vl.m), (unsigned)vl.e};
              }
            }
#pragma unroll
            for (int u = 0; u < kGroup; ++u) ref[u] = q <= L ? imax((int)v[u][1], (int)v[u][3]) : kDpFloor;
            if constexpr (!LOG) wave_max_i32(ref);
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
              const int be = (int)v[u][1], le = (int)v[u][3];
              const f32x2 x = LOG ? f32x2{__uint_as_float(v[u][0]), __uint_as_float(v[u][1])} : f32x2{
                  be < kDpImpossible ? -INFINITY : (float)(be - ref[u]) + __builtin_amdgcn_logf(__uint_as_float(v[u][0])),
                  le < kDpImpossible ? -INFINITY : (float)(le - ref[u]) + __builtin_amdgcn_logf(__uint_as_float(v[u][2]))};
              const int i = i0 + first + u;
              const size_t t = (size_t)frame(i);
              if (i < Tb && q <= L) *(f32x2*)(g + t * SP) = x;
              if (i < Tb && lane == 0) coff[t * p.blocks] = LOG ? as_double(v[u][2], v[u][3]) : (double)ref[u];
            }
          }
        }
      }
      lds_barrier();
    }
  }
}

// Workgroups beyond the recursions' `jobs` build the links of the labels meanwhile.
template <int WRITERS>
__global__ __launch_bounds__(dp_threads(WRITERS)) void ctc_dp_pipe_kernel(CtcParams p, int directions, int jobs) {
  __shared__ DpShared sh;
  __shared__ int job_id;
  const int tid = threadIdx.x;
  if (tid == 0) job_id = atomicAdd(p.ticket, 1);
  __syncthreads();
  const int job = __builtin_amdgcn_readfirstlane(job_id);
  if ((unsigned)job >= gridDim.x) return;  // (only if something else writes the workspace meanwhile)
  if (job >= jobs) {
    const int b = (job - jobs) % p.B;
    ctc_links(p, b, (job - jobs) / p.B, ((int)gridDim.x - jobs) / p.B, (int32_t*)&sh);
    return;
  }
  const int block = job / (directions * p.B), rest = job - block * (directions * p.B);
  const int b = rest / directions;
  const bool backward = rest - b * directions != 0;
  const int L = clampi(p.label_len[b], 0, p.Lmax);
  const int Tb = clampi(p.frame_len[b], 0, p.T);
  if (block * kDpPairs > L) return;
  if (Tb == 0) {
    if (tid == 0 && !backward && block == 0) {
      p.loss[b] = L == 0 ? 0.f : INFINITY;
      p.logp[b] = L == 0 ? 0.0 : -(double)INFINITY;
    }
    return;
  }
  int wide = 0;
  for (int t = tid; t < Tb; t += dp_threads(WRITERS)) wide |= p.wide[(size_t)b * p.T + t];
  if (__syncthreads_or(wide & 0xff00)) ctc_block<kDpLog, WRITERS>(p, sh, directions, block, b, backward, L, Tb);
  else if (WRITERS == 2 || __syncthreads_or(wide)) ctc_block<kDpMantissa, WRITERS>(p, sh, directions, block, b, backward, L, Tb);
  else if constexpr (WRITERS == 4) ctc_block<kDpDouble, WRITERS>(p, sh, directions, block, b, backward, L, Tb);
}

// One wavefront per frame: the occupancies gamma_t(s) = alpha_t(s) beta_t(s) / (p_t(z_s) P) of the label's tokens
// and of the blank come off the softmax in the gradient row.  Only these few entries of the row are touched.
// The labels' occupancies are formed once and kept in LDS, where the first position of a token adds up those of all its
// positions: 256 sequences of 2048 frames, 512 labels out of 100 symbols (each five times), 2.61 ms; formed again from
// the stored rows for every position and every link, with a lane's own offsets, 5.62.
__global__ __launch_bounds__(kCtcFixThreads) void ctc_fix_kernel(CtcParams p) {
  extern __shared__ float occupancies[];  // [wavefront][Lmax]
  const int lane = threadIdx.x & 63;
  // the rows written last come first: part of them is still in the last-level cache (4 x 2048 rows of 32001: 193 -> 190 us)
  const int t = (gridDim.x - 1 - blockIdx.x) * (kCtcFixThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = gridDim.y - 1 - blockIdx.y;
  const int Tb = clampi(p.frame_len[b], 0, p.T);
  if (t >= Tb) return;  // rows past the sequence were written as zeros
  float* __restrict__ g = p.grad + ((size_t)b * p.T + t) * p.Vp1;
  const double logP = p.logp[b];
  if (!(logP > -(double)INFINITY)) {  // a label that cannot be reached has no gradient
    for (int v = lane; v < p.Vp1; v += 64) g[v] = 0.f;
    return;
  }
  const int L = clampi(p.label_len[b], 0, p.Lmax);
  const int SP = ctc_state_pitch(p.Lmax);
  const size_t frame = (size_t)b * p.T + t;
  const float* __restrict__ al = p.ag + frame * SP;
  const float* __restrict__ be = p.bg + frame * SP;
  const float* __restrict__ lp = p.lpc + frame * (p.Lmax + 1);
  // log of P over the two offsets of a state: what its stored alpha + beta - log p is measured against.  Beta's states are
  // counted from the last one: state s is its state 2 L - s, and pair q of this wavefront's group of 64 has its blank in
  // beta's pair d = L - q and its label in pair d - 1.  All 64 share alpha's block and lie in two of beta's, so the
  // offsets are the wavefront's, not the lane's.
  const double* __restrict__ ca = p.coff_a + frame * p.blocks;
  const double* __restrict__ cb = p.coff_b + frame * p.blocks;
  struct Offsets { int block; float upper, lower; };  // beta's block of pair L - q0, z there and in the block below
  auto offsets = [&](int q0) {
    const int block = (L - q0) / kDpPairs;
    const double rest = logP - ca[q0 / kDpPairs];
    return Offsets{block, (float)(rest - cb[block]), (float)(rest - cb[block > 0 ? block - 1 : 0])};
  };
  auto gamma = [&](int s, int beta_pair, float l, const Offsets& o) {
    const float a = al[s], bt = be[2 * L - s];
    const float z = beta_pair / kDpPairs == o.block ? o.upper : o.lower;
    return (a > -INFINITY && bt > -INFINITY) ? exp2f(a + bt - l - z) : 0.f;  // base-2 logarithms throughout
  };
  float* __restrict__ occ = occupancies + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * p.Lmax;
  // The occupancies of a frame sum to one (every alignment is in exactly one state at frame t).  What is left
  // of the recursions' rounding after thousands of frames is mostly common to all states of a frame - it sits in
  // z - so dividing by the computed sum removes it.  First pass: the sums, in a fixed order.
  const float lblank = lp[p.Lmax];
  float gb = 0.f, go = 0.f;
#pragma unroll 4
  for (int q0 = 0; q0 <= L; q0 += kDpPairs) {
    const Offsets o = offsets(q0);
    const int q = q0 + lane;
    if (q <= L) gb += gamma(2 * q, L - q, lblank, o);
    if (q < L) {
      const float x = gamma(2 * q + 1, L - q - 1, lp[q], o);
      occ[q] = x;
      go += x;
    }
  }
  // other lanes of this wavefront read them below: its LDS operations execute in order, the compiler must not reorder
  // them either
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_wave_barrier();
  gb = wave_sum_f32(gb);
  go = wave_sum_f32(go);
  const float total = gb + go;
  const float inv = total > 0.f ? 1.f / total : 1.f;
  // the blank: all even states
  // The entries are written, not updated: the softmax value that ctc_row_kernel left there is formed again from
  // the log-probability at hand, which saves fetching a cache line per entry.
  if (lane == 0) g[p.blank] = exp2f(lblank) - gb * inv;
  // the label's tokens: the lane of a token's first position adds the occupancies of all its positions
  const int32_t* __restrict__ y = p.labels + (size_t)b * p.Lmax;
  const int32_t* __restrict__ nx = p.next + (size_t)b * p.Lmax;
  const int32_t* __restrict__ fs = p.first + (size_t)b * p.Lmax;
#pragma unroll 4
  for (int j = lane; j < L; j += 64) {
    const int is_first = fs[j];
    const int tok = clampi(y[j], 0, p.Vp1 - 1);
    const float l = lp[j];
    float tot = occ[j];
    if (is_first) {
      for (int i = nx[j]; i >= 0; i = nx[i]) tot += occ[i];
      if (tok != p.blank) g[tok] = exp2f(l) - tot * inv;  // a label never holds the blank; ids come from the caller
    }
  }
}

struct CtcWorkspace {
  size_t lpc, ag, bg, coff_a, coff_b, logp, next, first, edge, wide, ticket, total;
};
// Which kernel runs the recursions.  A frame takes the wavefront that does all of a sequence's work alone longer than the
// pipeline's, but it needs a quarter of the wavefronts and one launch less: the pipeline is the faster one from 16 frames
// on until the sequences fill the chip, which few frames do sooner.  Whole call, 101 symbols, T / 2 labels, us pipelined /
// a wavefront each for B sequences:
//   T = 12: 14.6 / 13.5 (B = 1)      16: 15.4 / 16.3 (1), 17.4 / 18.3 (64), 20.2 / 18.5 (128)     24: 19 / 25 (64), 23 / 27 (128), 31 / 28 (256)
//   T = 32: 19 / 33 (64), 33 / 36 (256), 52 / 40 (512)       63: 20 / 54 (1), 48 / 69 (256), 76 / 82 (512), 129 / 101 (1024)
// With 64 frames and more its rows are in the workspace, and labels of 64 and more need the blocks; 80 frames of 501
// symbols, up to 20 labels, 400 / 600 / 1000 sequences: pipelined 83 / 114 / 176 us, a wavefront each 100 / 120 / 153.
constexpr int kPipeFrames = 16;  // never pipelined with fewer
static bool ctc_pipelined(int B, int T, int Lmax) {
  if (T >= kShortFrames) return Lmax >= kDpPairs || B <= 768;
  return T >= kPipeFrames && B <= 8 * T - 64;
}
// Doubles and four writers, whose workgroups take more registers, while there is a compute unit for each; beyond that the chip's
// throughput counts, and mantissas with two writers are the faster form.  us in doubles with four writers / in mantissas with two, 64
// frames, 20 labels: 128 sequences (256 workgroups) 27.8 / 28.5, 256 44.0 / 42.2, 300 51.3 / 46.2; 512 frames, 200 labels: 32 (256) 95.5 /
// 112.2, 100 253 / 246.
// Both directions count also where the loss alone is asked for, so that it has the same bits with and without its gradient.
static bool ctc_doubles(int B, int blocks) { return 2LL * B * blocks <= 256; }
static CtcWorkspace ctc_workspace(int B, int T, int Lmax) {
  CtcWorkspace w;
  size_t off = 0;
  auto carve = [&](size_t bytes) { size_t at = off; off = (off + bytes + 255) / 256 * 256; return at; };
  const size_t blocks = T >= kPipeFrames ? Lmax / kDpPairs + 1 : 1;
  w.lpc = carve((size_t)B * T * (Lmax + 1) * 4);
  // (one size for a shape whatever kernel it takes: a workspace sized for the largest batch serves the smaller ones)
  w.ag = carve((size_t)B * T * ctc_state_pitch(Lmax) * 4);
  w.bg = carve((size_t)B * T * ctc_state_pitch(Lmax) * 4);
  w.coff_a = carve((size_t)B * T * blocks * 8);
  w.coff_b = carve((size_t)B * T * blocks * 8);
  w.logp = carve((size_t)B * 8);
  w.next = carve((size_t)B * Lmax * 4);
  w.first = carve((size_t)B * Lmax * 4);
  w.edge = w.wide = w.ticket = off;
  if (T >= kPipeFrames) {
    w.edge = carve((size_t)B * 2 * T * blocks * 8);
    w.wide = carve((size_t)B * T * 4);
    w.ticket = carve(4);
  }
  w.total = off;
  return w;
}

// code of this translation unit loaded onto the current device (context creation calls this: a stage call never
// triggers a load, so it can be the first thing a stream capture records)
hipError_t prepare_ctc_loss() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, (const void*)ctc_fix_kernel);
}

}  // namespace ctcspec

using namespace ctcspec;

extern "C" size_t ctc_loss_workspace_bytes(int B, int T, int Lmax) {
  if (B < 1 || T < 1 || Lmax < 1) return 0;
  return ctc_workspace(B, T, Lmax).total;
}

extern "C" int ctc_loss(ctcspec_ctx* ctx, const float* logits, const int32_t* labels, const int32_t* label_len,
                        const int32_t* frame_len, int B, int T, int Vp1, int Lmax, int32_t blank_id, void* workspace,
                        size_t workspace_bytes, float* loss, float* grad) {
  if (!ctx) return CTCSPEC_EINVAL;
  if (const int owed = flush_deferred(ctx)) return owed;
  CTCSPEC_REQUIRE(ctx, logits && labels && label_len && frame_len && workspace && loss, CTCSPEC_EINVAL,
                  "ctc_loss: null pointer");
  CTCSPEC_REQUIRE(ctx, B > 0 && T > 0 && Vp1 > 0 && Lmax > 0, CTCSPEC_EINVAL, "ctc_loss: sizes must be positive");
  CTCSPEC_REQUIRE(ctx, blank_id >= 0 && blank_id < Vp1, CTCSPEC_EINVAL, "ctc_loss: blank_id out of range");
  CTCSPEC_REQUIRE(ctx, Lmax <= kCtcMaxLabels && Vp1 <= kCtcMaxRow && B <= 65535 && T <= 65535 * 32,
                  CTCSPEC_EUNSUPPORTED, "ctc_loss: Lmax <= %d, V+1 <= %d (a row is held in one workgroup's registers), B <= 65535",
                  kCtcMaxLabels, kCtcMaxRow);
  CTCSPEC_REQUIRE(ctx, aligned16(workspace) && aligned16(logits) && (!grad || aligned16(grad)), CTCSPEC_EINVAL,
                  "ctc_loss: logits, grad and workspace must be 16-byte aligned");
  const CtcWorkspace w = ctc_workspace(B, T, Lmax);
  CTCSPEC_REQUIRE(ctx, workspace_bytes >= w.total, CTCSPEC_EINVAL, "ctc_loss: workspace of %zu bytes needed, %zu given",
                  w.total, workspace_bytes);
  unsigned char* ws = (unsigned char*)workspace;
  CtcParams p;
  p.logits = logits; p.labels = labels; p.label_len = label_len; p.frame_len = frame_len;
  p.B = B; p.T = T; p.Vp1 = Vp1; p.Lmax = Lmax; p.blank = blank_id;
  p.lpc = (float*)(ws + w.lpc); p.ag = (float*)(ws + w.ag);
  p.bg = (float*)(ws + w.bg);
  p.coff_a = (double*)(ws + w.coff_a); p.coff_b = (double*)(ws + w.coff_b); p.logp = (double*)(ws + w.logp);
  p.next = (int32_t*)(ws + w.next); p.first = (int32_t*)(ws + w.first);
  p.loss = loss; p.grad = grad;
  const bool pipelined = ctc_pipelined(B, T, Lmax);
  p.blocks = pipelined ? Lmax / kDpPairs + 1 : 1;
  p.edge = pipelined ? (unsigned long long*)(ws + w.edge) : nullptr;
  p.wide = (int*)(ws + w.wide); p.ticket = (int*)(ws + w.ticket);
  p.wide_below = -fminf(32768.f, (float)(1 << 28) / (float)T);  // T of them stay above the pipelined recursion's floor
  const int directions = grad ? 2 : 1;
  const int link_parts = (Lmax + 31) / 32;  // eight positions per wavefront
  const long long jobs = (long long)B * directions * p.blocks, groups = jobs + (grad ? (long long)B * link_parts : 0);
  CTCSPEC_REQUIRE(ctx, !pipelined || groups <= 0x7fffffffLL, CTCSPEC_EUNSUPPORTED, "ctc_loss: grid too large");
  hipStream_t st = ctx->stream;
  // The fewest threads that hold the row with at most eight 16-byte loads each (512 threads: sixteen, see the kernel) and
  // the label with NY positions each: many short rows cost their workgroups' start and barriers (9100 rows of 616
  // symbols: the call took 64 us with 1024 threads a row, 25 with 64).
  const dim3 rows(T, B);
  auto row_launch = [&](auto threads_tag, auto ny_tag) {
    constexpr int TH = decltype(threads_tag)::value, NY = decltype(ny_tag)::value;
    const int nv = (Vp1 / 4 + TH - 1) / TH;  // 16-byte loads per thread
    if (nv <= 1) hipLaunchKernelGGL((ctc_row_kernel<1, TH, NY>), rows, dim3(TH), 0, st, p);
    else if (nv <= 2) hipLaunchKernelGGL((ctc_row_kernel<2, TH, NY>), rows, dim3(TH), 0, st, p);
    else if (nv <= 4) hipLaunchKernelGGL((ctc_row_kernel<4, TH, NY>), rows, dim3(TH), 0, st, p);
    else if (nv <= 8 || TH < 512) hipLaunchKernelGGL((ctc_row_kernel<8, TH, NY>), rows, dim3(TH), 0, st, p);
    else hipLaunchKernelGGL((ctc_row_kernel<16, (TH < 512 ? 512 : TH), NY>), rows, dim3(TH), 0, st, p);
  };
  using N2 = std::integral_constant<int, 2>;
  using N4 = std::integral_constant<int, 4>;
  if (Vp1 / 4 <= 8 * 64 && Lmax < 2 * 64) row_launch(std::integral_constant<int, 64>{}, N2{});
  else if (Vp1 / 4 <= 8 * 256 && Lmax < 2 * 256) row_launch(std::integral_constant<int, 256>{}, N2{});
  else if (Vp1 / 4 <= 16 * 512 && Lmax < 2 * 512) row_launch(std::integral_constant<int, 512>{}, N2{});
  else if (Vp1 / 4 <= 16 * 512) row_launch(std::integral_constant<int, 512>{}, N4{});
  else row_launch(std::integral_constant<int, 1024>{}, N2{});
  CTCSPEC_HIP(ctx, hipGetLastError());
  if (!pipelined) {
    if (T < kShortFrames) hipLaunchKernelGGL(ctc_short_kernel<true>, dim3(B), dim3(64), (size_t)T * (64 * 8 + 8), st, p);
    else hipLaunchKernelGGL(ctc_short_kernel<false>, dim3(B), dim3(64), 0, st, p);
    CTCSPEC_HIP(ctx, hipGetLastError());
    return CTCSPEC_OK;
  }
  if (ctc_doubles(B, p.blocks))
    hipLaunchKernelGGL(ctc_dp_pipe_kernel<4>, dim3((unsigned)groups), dim3(dp_threads(4)), 0, st, p, directions, (int)jobs);
  else
    hipLaunchKernelGGL(ctc_dp_pipe_kernel<2>, dim3((unsigned)groups), dim3(dp_threads(2)), 0, st, p, directions, (int)jobs);
  CTCSPEC_HIP(ctx, hipGetLastError());
  if (grad) {
    const int per = kCtcFixThreads / 64;
    hipLaunchKernelGGL(ctc_fix_kernel, dim3((T + per - 1) / per, B), dim3(kCtcFixThreads), (size_t)per * Lmax * 4, st, p);
    CTCSPEC_HIP(ctx, hipGetLastError());
  }
  return CTCSPEC_OK;
}
