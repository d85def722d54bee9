// np_calib.hip -- the magnitude-threshold sparsity of Sec. 3.2 (eq. 1):
//  * act_batch_kernel: activations A(i, l) = act(G x_i, U x_i) of one layer
//    over a batch of calibration tokens, on the matrix cores;
//  * pct_hist_kernel / pct_select_kernel (percentile_kernel for short rows):
//    per layer, the nearest-rank alpha-th percentile of |A| (the threshold
//    T(l, alpha)) by radix selection;
//  * threshold_active_kernel: eq. 1 as an active set, |a| >= T, in the
//    selection's mask + ascending-id layout.
#include "np_device.hpp"

namespace np {

// ---------------------------------------------------------------------------
// activations of a token batch
// ---------------------------------------------------------------------------
// The gate and up projections of a batch are two matrix products, G X^T and
// U X^T (neurons x tokens, reduction over d), so they run on MFMA with fp32
// accumulation: 16 x 16 output tiles, each a v_mfma_f32_16x16x32 (16-bit
// types) or four v_mfma_f32_16x16x4f32 (fp32) per "step" of 4*V reduction
// elements.  Lane l holds row l%16 of the A operand (a neuron's gate or up
// row) and column l%16 of the B operand (a token), each as the V consecutive
// elements starting at step*4V + V*(l/16), so the two operands pair the same
// reduction indices whatever order the unit sums them in.  The accumulator
// layout: lane l, register r holds output row 4*(l/16) + r (neuron) and
// column l%16 (token).
//
// A workgroup of 8 waves owns a block of BM neurons (2 BM weight rows) x BN
// tokens, wave (i, j) of its WGM x WGN waves MT x NT tiles of it (gate and up
// of the same neurons, so that the activation needs no exchange).  The rows
// stream through LDS in pieces of ROWB bytes, double buffered (row pitch
// ROWB + 16 bytes: the 16 rows of a fragment start 4 banks apart; bank
// conflicts are still a third of the LDS cycles).  In each
// iteration a thread writes the pieces it holds in registers to the other
// buffer, refills the registers from memory halfway through the products of
// the current buffer, and one barrier, for LDS only, ends the iteration: a
// load has at least an iteration (two with DEPTH 2) to arrive.
//
// Two regimes.  Up to 128 tokens it is HBM-bound (n flops per weight byte):
// small blocks, so that all CUs stream, long pieces (fewer barriers), the
// nontemporal hint on weights that one block reads, and two groups of four
// waves that take half of a piece's steps each, so that a wave's tiles are
// twice as large and its operands read less often.  SwiGLU 7B layer (14336 x
// 4096 f16, 235 MB of weights), 128 tokens: 58-60 us, 64 tokens 48-51 us (a
// plain read of the same rows 43.8 us); with one group of eight waves 2-5%
// more, with 128-byte pieces 64 and 51; the four-wave kernel before, whose loads the compiler had put behind the
// products they were to overlap, 76.5 and 68.7.  Beyond, it is bound by the
// matrix cores and by what feeds them: a 128 x 256 block reads 96 bytes of LDS
// a cycle for 8 waves of 128 x 64 outputs, and each weight row once per 256
// tokens.  13B layer (13824 x 5120 f16), 1999 tokens: 560-588 us (962-1011
// TFLOP/s) against 1355 in launches of 128 tokens; 4096 tokens on the SwiGLU
// layer 824-868 us (1108-1168 TFLOP/s; 2300 before; the library's square
// product of size 8192: 1112-1164 TFLOP/s).
constexpr int AB_WAVES = 8;
constexpr int AB_NT = AB_WAVES * WAVE;

struct ActBatchArgs {
  const void* w;    // one layer's [F][3d] records
  const void* x;    // [n][d] tokens
  float* acts;      // [n][F]
  uint32_t w_bytes, x_bytes;
  int F, d, n, act;
  int fb, tb;       // neuron blocks, token blocks
};

template <int MT_, int NT_, int WGM_, int WGN_, int DEPTH_, int ROWB_, int KW_ = 1>
struct AbTile {
  static constexpr int ROWB = ROWB_, PITCH = ROWB + 16;
  static constexpr int MT = MT_, NT = NT_, WGM = WGM_, WGN = WGN_, DEPTH = DEPTH_;
  static constexpr int KW = KW_;  // groups of waves, each a share of a piece's steps
  static constexpr int BM = 16 * MT * WGM, BN = 16 * NT * WGN;
  static constexpr int ROWS = 2 * BM + BN;               // LDS rows: gate, up, tokens
  static constexpr int PIECES = ROWS * (ROWB / 16);   // 16-byte pieces of an iteration
  static constexpr int PPT = PIECES / AB_NT;             // per thread
  static constexpr size_t LDS = (size_t)2 * ROWS * PITCH;
  static_assert(WGM * WGN * KW == AB_WAVES && ROWB / 64 % (2 * KW) == 0 && PIECES % AB_NT == 0 &&
                    2 * BM % (AB_NT / (ROWB / 16)) == 0,
                "whole pieces per thread, weights and tokens in separate ones");
};

template <class T, class C, bool NTW>
__global__ __launch_bounds__(AB_NT) void act_batch_kernel(ActBatchArgs a) {
  constexpr int V = T::V, ESZ = 16 / V, KC = C::ROWB / ESZ;  // KC: elements per iteration
  constexpr int ROWB = C::ROWB, PITCH = C::PITCH, LPR = ROWB / 16;  // LPR: lanes of a row piece
  constexpr int RPP = AB_NT / LPR;  // rows of a piece index
  constexpr int MT = C::MT, NT = C::NT, PPT = C::PPT, DEPTH = C::DEPTH;
  __shared__ __attribute__((aligned(16))) char ab_lds[C::LDS];
  const int t = threadIdx.x, lane = t & (WAVE - 1), w = t / WAVE, grp = lane / 16, li = lane & 15;
  constexpr int KW = C::KW, STEPS = ROWB / 64 / KW;  // steps of a piece for each wave
  const int kg = w / (C::WGM * C::WGN), wm = w / C::WGN % C::WGM, wn = w % C::WGN;
  // blocks b, b + 8, ... run on one XCD: each XCD takes a contiguous run of
  // blocks, token blocks innermost, so its L2 serves a weight panel to the
  // token blocks that share it
  const int nb = a.fb * a.tb, per = (nb + 7) / 8;
  const int blk = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (blk >= nb || (int)(blockIdx.x / 8) >= per) return;
  const int f0 = blk / a.tb * C::BM, t0 = blk % a.tb * C::BN;
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes), xr = make_rsrc(a.x, a.x_bytes);
  const uint32_t dbytes = (uint32_t)(a.d * ESZ), rec = 3u * dbytes;
  const int iters = (a.d + KC - 1) / KC;
  // piece i of this thread: row t / LPR + RPP i, 16-byte column t % LPR (gate
  // rows, up rows, tokens); rows past F or n read out of range: zeros
  const uint32_t col = (uint32_t)(t % LPR) * 16u;
  uint32_t off[PPT];
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int row = t / LPR + RPP * i;
    if (row < 2 * C::BM) {
      const int f = f0 + row % C::BM;
      off[i] = f < a.F ? (uint32_t)f * rec + (uint32_t)(row / C::BM) * dbytes : BUF_OOB;
    } else {
      const int tok = t0 + row - 2 * C::BM;
      off[i] = tok < a.n ? (uint32_t)tok * dbytes : BUF_OOB;
    }
  }
  auto load = [&](int it, u32x4_t* r) {  // past d: zeros
    const uint32_t k = (uint32_t)it * ROWB + col;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const uint32_t o = k < dbytes && off[i] != BUF_OOB ? off[i] + k : BUF_OOB;
      if (RPP * i < 2 * C::BM)  // a piece index holds weight rows only or tokens only
        r[i] = NTW ? buf_load16v_nt(wr, o, 0) : buf_load16v(wr, o, 0);
      else
        r[i] = buf_load16v(xr, o, 0);
    }
  };
  char* const st = ab_lds + (size_t)(t / LPR) * PITCH + col;
  auto store = [&](int buf, const u32x4_t* r) {
    char* p = st + (size_t)buf * C::ROWS * PITCH;
#pragma unroll
    for (int i = 0; i < PPT; ++i) *(u32x4_t*)(p + (size_t)RPP * i * PITCH) = r[i];
  };
  f32x4 accg[MT][NT], accu[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) accg[m][j][r] = accu[m][j][r] = 0.f;
  // fragment addresses: gate rows of this wave's first tile, tokens likewise
  const char* const fg = ab_lds + (size_t)(wm * MT * 16 + li) * PITCH + kg * STEPS * 64 + grp * 16;
  const char* const fx = ab_lds + (size_t)(2 * C::BM + wn * NT * 16 + li) * PITCH + kg * STEPS * 64 +
                         grp * 16;
  auto multiply = [&](int buf, int s_begin, int s_end) {
    const size_t bo = (size_t)buf * C::ROWS * PITCH;
#pragma unroll
    for (int s = s_begin; s < s_end; ++s) {
      uint4 b[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j)
        b[j] = *(const uint4*)(fx + bo + (size_t)16 * j * PITCH + s * 64);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const uint4 ag = *(const uint4*)(fg + bo + (size_t)16 * m * PITCH + s * 64);
        const uint4 au = *(const uint4*)(fg + bo + (size_t)(C::BM + 16 * m) * PITCH + s * 64);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          accg[m][j] = mfma_step<T>(ag, b[j], accg[m][j]);
          accu[m][j] = mfma_step<T>(au, b[j], accu[m][j]);
        }
      }
    }
  };
  u32x4_t pre[DEPTH][PPT];
  load(0, pre[0]);
  store(0, pre[0]);
#pragma unroll
  for (int q = 0; q < DEPTH; ++q) load(1 + q, pre[q]);
  lds_barrier();
  // iteration it: registers pre[it % DEPTH] hold piece it + 1
  for (int it = 0;; it += 2 * DEPTH) {
#pragma unroll
    for (int q = 0; q < 2 * DEPTH; ++q) {
      store((q + 1) & 1, pre[q % DEPTH]);
      multiply(q & 1, 0, STEPS / 2);
      __builtin_amdgcn_sched_barrier(0);  // neither ahead of the stores nor behind the products
      load(it + q + 1 + DEPTH, pre[q % DEPTH]);
      __builtin_amdgcn_sched_barrier(0);
      multiply(q & 1, STEPS / 2, STEPS);
      if (it + q + 1 >= iters) goto done;  // (a skipped iteration would blur the load counts)
      lds_barrier();
    }
  }
done:
  if constexpr (KW > 1) {  // the other groups' sums join group 0's, in order
    static_assert((size_t)(KW - 1) * C::BM * C::BN * 8 <= C::LDS, "the sums fit the pieces' LDS");
    f32x4* sums = reinterpret_cast<f32x4*>(ab_lds);
    const int slot = (w % (C::WGM * C::WGN)) * MT * NT * 2;
    __syncthreads();  // every wave is done with the pieces
    if (kg > 0) {
      f32x4* p = sums + (size_t)(kg - 1) * C::WGM * C::WGN * MT * NT * 2 * WAVE + lane;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          p[(size_t)(slot + 2 * (m * NT + j)) * WAVE] = accg[m][j];
          p[(size_t)(slot + 2 * (m * NT + j) + 1) * WAVE] = accu[m][j];
        }
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 0; g < KW - 1; ++g) {
      const f32x4* p = sums + (size_t)g * C::WGM * C::WGN * MT * NT * 2 * WAVE + lane;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          accg[m][j] += p[(size_t)(slot + 2 * (m * NT + j)) * WAVE];
          accu[m][j] += p[(size_t)(slot + 2 * (m * NT + j) + 1) * WAVE];
        }
    }
  }
  // acts[token][neuron]: lane l, register r holds neuron 16 m + 4 (l / 16) + r
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int tok = t0 + (wn * NT + j) * 16 + li;
    if (tok >= a.n) continue;
    float* dst = a.acts + (size_t)tok * a.F;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int f = f0 + (wm * MT + m) * 16 + 4 * grp;  // neurons f .. f + 3
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = gated(a.act, accg[m][j][e], accu[m][j][e]);
      if ((a.F & 3) == 0) {
        if (f < a.F) *(float4*)(dst + f) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (f + e < a.F) dst[f + e] = o[e];
      }
    }
  }
}

template <class T, class C, bool NTW>
static hipError_t launch_ab(const ActBatchArgs& a, hipStream_t stream) {
  ActBatchArgs b = a;
  b.fb = (a.F + C::BM - 1) / C::BM;
  b.tb = (a.n + C::BN - 1) / C::BN;
  hipLaunchKernelGGL((act_batch_kernel<T, C, NTW>), dim3((b.fb * b.tb + 7) / 8 * 8), dim3(AB_NT),
                     0, stream, b);
  return hipGetLastError();
}

template <class T>
static hipError_t act_batch_t(const np_shape& s, const void* weights, const void* x, int n,
                              float* acts, hipStream_t stream) {
  constexpr int ESZ = 16 / T::V;
  ActBatchArgs a;
  a.w = weights;
  a.x = x;
  a.acts = acts;
  a.n = n;
  a.w_bytes = (uint32_t)((size_t)s.d_ffn * 3 * s.d_model * ESZ);
  a.x_bytes = (uint32_t)((size_t)n * s.d_model * ESZ);
  a.F = s.d_ffn;
  a.d = s.d_model;
  a.act = s.act;
  // The block whose rounds over the 256 CUs cost least: the time of a round
  // of each block, relative to each other (d 4096: 119, 74, 48 and 32 us in
  // f16; fp32 is bound by its matrix rate and goes by the area alone), is the
  // same for any size within 10%: f16, n = 256, F = 14336, one round of 128 x
  // 128 takes 84 us, one of 128 x 256 115, two of 64 x 128 97; n = 1500, d 600,
  // F = 2000, one round of 128 x 128 17, one of 128 x 256 24, two of 64 x 128 21.
  struct Block {
    int bm, bn;
    float cost16, cost32;
  };
  static constexpr Block blocks[4] = {
      {128, 256, 119.f, 6.4f}, {128, 128, 74.f, 3.3f}, {64, 128, 48.f, 1.8f}, {64, 64, 32.f, 1.f}};
  int best = 0;
  float least = 0.f;
  for (int i = 0; i < 4; ++i) {
    const Block& q = blocks[i];
    const long long nb = (long long)((a.F + q.bm - 1) / q.bm) * ((n + q.bn - 1) / q.bn);
    const float c = (float)((nb + 255) / 256) * (T::dtype == NP_F32 ? q.cost32 : q.cost16);
    if (i == 0 || c < least) {
      best = i;
      least = c;
    }
  }
  // weights that a single token block reads need not stay in the caches
  const bool once = n <= blocks[best].bn;
  switch (best) {
    case 0: return launch_ab<T, AbTile<4, 4, 2, 4, 1, 128>, false>(a, stream);
    case 1: return launch_ab<T, AbTile<2, 4, 4, 2, 2, 128>, false>(a, stream);
    case 2:
      return once ? launch_ab<T, AbTile<2, 4, 2, 2, 1, 256, 2>, true>(a, stream)
                  : launch_ab<T, AbTile<2, 4, 2, 2, 1, 256, 2>, false>(a, stream);
    default:
      return once ? launch_ab<T, AbTile<2, 2, 2, 2, 1, 256, 2>, true>(a, stream)
                  : launch_ab<T, AbTile<2, 2, 2, 2, 1, 256, 2>, false>(a, stream);
  }
}

hipError_t launch_act_batch(const np_shape& s, const void* weights, const void* x, int n,
                            float* acts, hipStream_t stream) {
  switch (s.wdtype) {
    case NP_F32: return act_batch_t<TF32>(s, weights, x, n, acts, stream);
    case NP_F16: return act_batch_t<TF16>(s, weights, x, n, acts, stream);
    default: return act_batch_t<TBF16>(s, weights, x, n, acts, stream);
  }
}

// ---------------------------------------------------------------------------
// per-row nearest-rank percentile of the magnitudes
// ---------------------------------------------------------------------------
// The magnitude's bits (sign cleared) order non-negative floats like
// integers, so the m-th smallest magnitude is found digit by digit from the
// top: 11, 10 and 10 bits.  Each pass streams the row once, counts the
// values that match the digits decided so far into a histogram of the next
// digit (four LDS copies, by wave, against atomic contention on the few bins
// a narrow exponent range fills), and a prefix sum over the bins finds the
// digit that holds the m-th value.
constexpr int PCT_NT = 1024;
constexpr int PCT_BINS = 2048;
constexpr int PCT_COPIES = 4;

template <bool V4>
__global__ __launch_bounds__(PCT_NT) void percentile_kernel(const float* __restrict__ values,
                                                            int64_t n, int64_t m, float* out,
                                                            void* ws) {
  __shared__ uint32_t hist[PCT_COPIES][PCT_BINS];
  __shared__ uint32_t scan[PCT_NT / WAVE + 1];
  __shared__ uint32_t sel[2];  // chosen digit, rank left within it
  const int tid = threadIdx.x, copy = (tid / WAVE) % PCT_COPIES;
  const float* row = values + (size_t)blockIdx.x * (size_t)n;
  uint32_t prefix = 0, known = 0;  // decided high bits and their mask
  uint32_t rank = (uint32_t)m;     // 1-based rank within the matching values
  bool nan = false;
  const int shifts[3] = {20, 10, 0}, widths[3] = {11, 10, 10};
  for (int pass = 0; pass < 3; ++pass) {
    const int sh = shifts[pass], nb = 1 << widths[pass];
    for (int i = tid; i < PCT_COPIES * PCT_BINS; i += PCT_NT) (&hist[0][0])[i] = 0u;
    __syncthreads();
    auto count = [&](float v) {
      const uint32_t key = __float_as_uint(v) & 0x7FFFFFFFu;
      if (pass == 0 && key > 0x7F800000u) nan = true;
      if ((key & known) == prefix) atomicAdd(&hist[copy][(key >> sh) & (nb - 1)], 1u);
    };
    if constexpr (V4) {
      const float4* r4 = (const float4*)row;
      for (int64_t i = tid; i < n / 4; i += PCT_NT) {
        const float4 v = r4[i];
        count(v.x);
        count(v.y);
        count(v.z);
        count(v.w);
      }
    } else {
      for (int64_t i = tid; i < n; i += PCT_NT) count(row[i]);
    }
    __syncthreads();
    // thread t owns bins 2t, 2t + 1
    uint32_t c[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int b = 2 * tid + j;
      c[j] = 0u;
      if (b < nb)
#pragma unroll
        for (int cp = 0; cp < PCT_COPIES; ++cp) c[j] += hist[cp][b];
    }
    uint32_t tot;
    const uint32_t before = block_excl_scan<PCT_NT>(c[0] + c[1], scan, &tot);
    if (before < rank && rank <= before + c[0]) {
      sel[0] = 2 * tid;
      sel[1] = rank - before;
    } else if (before + c[0] < rank && rank <= before + c[0] + c[1]) {
      sel[0] = 2 * tid + 1;
      sel[1] = rank - before - c[0];
    }
    __syncthreads();
    prefix |= sel[0] << sh;
    known |= (uint32_t)(nb - 1) << sh;
    rank = sel[1];
    __syncthreads();  // sel and hist are rewritten by the next pass
  }
  if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
  if (tid == 0) out[blockIdx.x] = __uint_as_float(prefix);
}

// The same selection spread over many workgroups per row, for long rows:
// each pass is a histogram kernel over (slice, row) workgroups, which count
// their slice of the row into LDS and add the nonzero bins to the row's
// histogram in dev_ws, and a selection kernel with one workgroup per row,
// which scans that histogram, narrows the row's (prefix, known bits, rank)
// state and clears the histogram for the next pass.  The kernel boundaries
// order the passes.  dev_ws layout past the control block: state [rows][4]
// uint32, then histograms [rows][PCT_BINS] uint32.
constexpr int PCT_HNT = 512;
constexpr int PCT_HCOPIES = 4;  // LDS histogram copies, by wave

__host__ __device__ inline size_t pct_hist_offset(int rows) {
  return (WS_CTRL_BYTES + (size_t)rows * 16 + 255) & ~(size_t)255;
}
size_t percentile_ws_bytes(int rows) {
  return pct_hist_offset(rows) + (size_t)rows * PCT_BINS * 4;
}

__global__ __launch_bounds__(256) void pct_init_kernel(int64_t m, void* ws) {
  const int row = blockIdx.x;
  uint32_t* st = (uint32_t*)((char*)ws + WS_CTRL_BYTES) + 4 * (size_t)row;
  uint32_t* h = (uint32_t*)((char*)ws + pct_hist_offset(gridDim.x)) + (size_t)row * PCT_BINS;
  if (threadIdx.x == 0) {
    st[0] = 0u;  // decided high bits
    st[1] = 0u;  // their mask
    st[2] = (uint32_t)m;  // 1-based rank within the matching values
    st[3] = 0u;
  }
  for (int i = threadIdx.x; i < PCT_BINS; i += blockDim.x) h[i] = 0u;
}

// grid (slices, rows); slice s of a row covers values [s*chunk, min(n, (s+1)*chunk))
template <bool V4>
__global__ __launch_bounds__(PCT_HNT) void pct_hist_kernel(const float* __restrict__ values,
                                                           int64_t n, int64_t chunk, int pass,
                                                           int rows, void* ws) {
  __shared__ uint32_t hist[PCT_HCOPIES][PCT_BINS];
  const int tid = threadIdx.x, copy = (tid / WAVE) % PCT_HCOPIES;
  const int row = blockIdx.y;
  const uint32_t* st = (const uint32_t*)((const char*)ws + WS_CTRL_BYTES) + 4 * (size_t)row;
  const uint32_t prefix = st[0], known = st[1];
  const int sh = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
  const uint32_t nb = pass == 0 ? 2048u : 1024u;
  for (int i = tid; i < PCT_HCOPIES * PCT_BINS; i += PCT_HNT) (&hist[0][0])[i] = 0u;
  __syncthreads();
  const float* rowp = values + (size_t)row * (size_t)n;
  const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
  bool nan = false;
  auto count = [&](float v) {
    const uint32_t key = __float_as_uint(v) & 0x7FFFFFFFu;
    if (pass == 0 && key > 0x7F800000u) nan = true;
    if ((key & known) == prefix) atomicAdd(&hist[copy][(key >> sh) & (nb - 1)], 1u);
  };
  if constexpr (V4) {  // chunk and n are multiples of 4
    const float4* r4 = (const float4*)(rowp + lo);
    const int64_t n4 = (hi - lo) / 4;
    for (int64_t i = tid; i < n4; i += PCT_HNT) {
      const float4 v = r4[i];
      count(v.x);
      count(v.y);
      count(v.z);
      count(v.w);
    }
  } else {
    for (int64_t i = lo + tid; i < hi; i += PCT_HNT) count(rowp[i]);
  }
  if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
  __syncthreads();
  uint32_t* h = (uint32_t*)((char*)ws + pct_hist_offset(rows)) + (size_t)row * PCT_BINS;
  for (int b = tid; b < (int)nb; b += PCT_HNT) {
    uint32_t c = 0u;
#pragma unroll
    for (int cp = 0; cp < PCT_HCOPIES; ++cp) c += hist[cp][b];
    if (c) atomicAdd(&h[b], c);
  }
}

// one workgroup per row: the digit of this pass that holds the rank
__global__ __launch_bounds__(PCT_NT) void pct_select_kernel(int pass, int rows, float* out,
                                                            void* ws) {
  __shared__ uint32_t scan[PCT_NT / WAVE + 1];
  __shared__ uint32_t sel[2];
  const int tid = threadIdx.x, row = blockIdx.x;
  uint32_t* st = (uint32_t*)((char*)ws + WS_CTRL_BYTES) + 4 * (size_t)row;
  uint32_t* h = (uint32_t*)((char*)ws + pct_hist_offset(rows)) + (size_t)row * PCT_BINS;
  const int sh = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
  const int nb = pass == 0 ? 2048 : 1024;
  const uint32_t rank = st[2];
  uint32_t c[2];  // thread t owns bins 2t, 2t + 1
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int b = 2 * tid + j;
    c[j] = b < nb ? h[b] : 0u;
  }
  if (tid == 0) {  // a rank beyond the count (NaN rows only) keeps digit 0
    sel[0] = 0u;
    sel[1] = rank;
  }
  uint32_t tot;
  const uint32_t before = block_excl_scan<PCT_NT>(c[0] + c[1], scan, &tot);
  if (before < rank && rank <= before + c[0]) {
    sel[0] = 2 * tid;
    sel[1] = rank - before;
  } else if (before + c[0] < rank && rank <= before + c[0] + c[1]) {
    sel[0] = 2 * tid + 1;
    sel[1] = rank - before - c[0];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) h[2 * tid + j] = 0u;  // PCT_BINS = 2 * PCT_NT
  if (tid == 0) {
    const uint32_t prefix = st[0] | (sel[0] << sh);
    st[0] = prefix;
    st[1] |= (uint32_t)(nb - 1) << sh;
    st[2] = sel[1];
    if (pass == 2) out[row] = __uint_as_float(prefix);
  }
}

hipError_t launch_percentile(const float* values, int rows, int64_t n, int64_t m, float* out,
                             void* ws, size_t ws_bytes, hipStream_t stream) {
  // slices per row: about four workgroups per compute unit in all, each over
  // at least 32K values
  const int64_t want = ((int64_t)1024 + rows - 1) / rows;
  int64_t slices = std::min<int64_t>(want, (n + 32767) / 32768);
  if (slices > 65535) slices = 65535;
  if (slices >= 2 && ws_bytes >= percentile_ws_bytes(rows)) {
    int64_t chunk = (n + slices - 1) / slices;
    chunk = (chunk + 3) / 4 * 4;  // whole float4 vectors
    slices = (n + chunk - 1) / chunk;
    hipLaunchKernelGGL(pct_init_kernel, dim3(rows), dim3(256), 0, stream, m, ws);
    for (int pass = 0; pass < 3; ++pass) {
      if (n % 4 == 0)
        hipLaunchKernelGGL(pct_hist_kernel<true>, dim3((unsigned)slices, rows), dim3(PCT_HNT), 0,
                           stream, values, n, chunk, pass, rows, ws);
      else
        hipLaunchKernelGGL(pct_hist_kernel<false>, dim3((unsigned)slices, rows), dim3(PCT_HNT),
                           0, stream, values, n, chunk, pass, rows, ws);
      hipLaunchKernelGGL(pct_select_kernel, dim3(rows), dim3(PCT_NT), 0, stream, pass, rows, out,
                         ws);
    }
    return hipGetLastError();
  }
  if (n % 4 == 0)
    hipLaunchKernelGGL(percentile_kernel<true>, dim3(rows), dim3(PCT_NT), 0, stream, values, n,
                       m, out, ws);
  else
    hipLaunchKernelGGL(percentile_kernel<false>, dim3(rows), dim3(PCT_NT), 0, stream, values, n,
                       m, out, ws);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// eq. 1 as an active set
// ---------------------------------------------------------------------------
// One workgroup per row; thread t owns id words [t*WPT, t*WPT + WPT): it
// compares the word's 32 activations with the row's threshold, and a
// workgroup prefix sum over the words' popcounts places the ids in ascending
// order (the selection's layout).
template <int NT, int WPT, bool V4>
__global__ __launch_bounds__(NT) void threshold_active_kernel(
    const float* __restrict__ acts, const float* __restrict__ thr, uint32_t* __restrict__ mask,
    int32_t* __restrict__ active_ids, int32_t* __restrict__ counts, int F, int k, void* ws) {
  __shared__ uint32_t scan[NT / WAVE + 1];
  const int r = blockIdx.x, tid = threadIdx.x;
  const int W = (F + 31) / 32;
  const float T = thr[r];
  const float* row = acts + (size_t)r * F;
  uint32_t m[WPT], cnt = 0;
  bool nan = false;
#pragma unroll
  for (int i = 0; i < WPT; ++i) {
    const int word = tid * WPT + i;
    m[i] = 0u;
    if (word < W) {
      if (V4 && 32 * word + 32 <= F) {
        const float4* p = (const float4*)(row + 32 * word);
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = p[j];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float e[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            nan |= e[c] != e[c];
            if (fabsf(e[c]) >= T) m[i] |= 1u << (4 * j + c);
          }
        }
      } else {
        for (int b = 0; b < 32 && 32 * word + b < F; ++b) {
          const float e = row[32 * word + b];
          nan |= e != e;
          if (fabsf(e) >= T) m[i] |= 1u << b;
        }
      }
      mask[(size_t)r * W + word] = m[i];
    }
    cnt += __builtin_popcount(m[i]);
  }
  if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
  uint32_t tot;
  uint32_t pos = block_excl_scan<NT>(cnt, scan, &tot);
  int32_t* ids = active_ids + (size_t)r * k;
#pragma unroll
  for (int i = 0; i < WPT; ++i) {
    uint32_t bits = m[i];
    while (bits) {
      const int b = __builtin_ctz(bits);
      bits &= bits - 1;
      if (pos < (uint32_t)k) ids[pos] = 32 * (tid * WPT + i) + b;
      ++pos;
    }
  }
  if (tid == 0) {
    counts[r] = tot < (uint32_t)k ? (int32_t)tot : k;
    if (tot > (uint32_t)k) raise_error(ws, NP_DEVERR_OVERFLOW);
  }
}

hipError_t launch_threshold_active(const np_shape& s, const float* acts, int rows,
                                   const float* thr, uint32_t* mask, int32_t* active_ids,
                                   int32_t* active_counts, void* ws, hipStream_t stream) {
  const int words = (s.d_ffn + 31) / 32;
  const bool v4 = s.d_ffn % 4 == 0;
#define NP_THR_CASE(NT, W)                                                                     \
  do {                                                                                         \
    if (v4)                                                                                    \
      hipLaunchKernelGGL((threshold_active_kernel<NT, W, true>), dim3(rows), dim3(NT), 0,      \
                         stream, acts, thr, mask, active_ids, active_counts, s.d_ffn, s.k, ws); \
    else                                                                                       \
      hipLaunchKernelGGL((threshold_active_kernel<NT, W, false>), dim3(rows), dim3(NT), 0,     \
                         stream, acts, thr, mask, active_ids, active_counts, s.d_ffn, s.k, ws); \
  } while (0)
  if (words <= 256) NP_THR_CASE(256, 1);
  else if (words <= 512) NP_THR_CASE(512, 1);
  else if (words <= 1024) NP_THR_CASE(1024, 1);
  else NP_THR_CASE(1024, 2);
#undef NP_THR_CASE
  return hipGetLastError();
}

}  // namespace np
