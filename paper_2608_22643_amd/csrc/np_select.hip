// np_select.hip -- fixed-size active sets and the delta against the resident
// buffer (Sec. 3.4).  Both steps are small, latency-bound integer work: one
// workgroup per downstream layer, ids owned in contiguous runs of bits so that
// set membership, ordering and compaction are bit operations, popcounts and
// workgroup prefix sums.  The general path of either is the radix k-selection
// primitive of np_device.hpp (top-k of the scores; least-recently-used
// victims).
#include <stdlib.h>

#include "np_device.hpp"

namespace np {

// Order-preserving unsigned key of an fp32 score: larger score, larger key.
// -0.0 maps to the key of +0.0.  NaN maps to 0 (below every other key) and
// is reported through the error word.
__device__ inline uint32_t score_key(float f, bool* nan) {
  const bool bad = f != f;
  *nan |= bad;
  const uint32_t u = __float_as_uint(f + 0.f);  // -0.0 + 0.0 is +0.0, all else itself
  const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
  return bad ? 0u : key;
}

// Keys of thread tid's id words [tid*WPT, tid*WPT+WPT) of one layer's
// scores (0 past F).  Loads are unconditional (clamped index) so that all of
// them are in flight together; the range test only picks the key.  V4: the
// layer's scores are 16-byte aligned (F a multiple of 4) and read as float4.
template <int WPT, bool V4>
__device__ inline void load_score_keys(const float* __restrict__ s, int F, int tid,
                                       uint32_t (&key)[WPT][32], bool* nan) {
  if (32 * WPT * tid < F) {
#pragma unroll
    for (int w = 0; w < WPT; ++w) {
      const int word = tid * WPT + w;
      float v[32];
      if constexpr (V4) {
        const float4* s4 = reinterpret_cast<const float4*>(s);
        const int last = F / 4 - 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float4 q = s4[min(8 * word + i, last)];
          v[4 * i] = q.x;
          v[4 * i + 1] = q.y;
          v[4 * i + 2] = q.z;
          v[4 * i + 3] = q.w;
        }
      } else {
#pragma unroll
        for (int b = 0; b < 32; ++b) v[b] = s[min(32 * word + b, F - 1)];
      }
#pragma unroll
      for (int b = 0; b < 32; ++b) {
        const uint32_t kv = score_key(v[b], nan);
        key[w][b] = (32 * word + b < F) ? kv : 0u;
      }
    }
  } else {
#pragma unroll
    for (int w = 0; w < WPT; ++w)
#pragma unroll
      for (int b = 0; b < 32; ++b) key[w][b] = 0u;
  }
}

// The selected words of one layer out: the mask, and the ids in ascending
// order (a workgroup prefix sum of the words' popcounts) to `ids` and, when
// non-null, to `ids_lds` as well.
template <int NT, int WPT>
__device__ inline void write_selection(const uint32_t (&sel)[WPT], int tid, int words, int k,
                                       uint32_t* __restrict__ mask_l, int32_t* __restrict__ ids,
                                       int32_t* ids_lds, uint32_t* scan) {
  uint32_t cnt = 0;
#pragma unroll
  for (int w = 0; w < WPT; ++w) cnt += __builtin_popcount(sel[w]);
  uint32_t tot;
  uint32_t pos = block_excl_scan<NT>(cnt, scan, &tot);
#pragma unroll
  for (int w = 0; w < WPT; ++w) {
    const int word = tid * WPT + w;
    if (word < words) mask_l[word] = sel[w];
    uint32_t bits = sel[w];
    while (bits) {
      const int b = __builtin_ctz(bits);
      bits &= bits - 1;
      if (pos < (uint32_t)k) {
        ids[pos] = 32 * word + b;
        if (ids_lds) ids_lds[pos] = 32 * word + b;
      }
      ++pos;
    }
  }
}

// One workgroup of NT threads per layer; thread t owns id words
// [t*WPT, t*WPT+WPT).
template <int NT, int WPT, bool V4>
__global__ __launch_bounds__(NT) void select_kernel(const float* __restrict__ scores,
                                                    uint32_t* __restrict__ mask,
                                                    int32_t* __restrict__ active_ids, int F,
                                                    int k, void* ws) {
  __shared__ uint32_t hist[4096];
  __shared__ uint32_t scan[3 * (NT / WAVE) + 1];
  __shared__ uint32_t res[4];
  const int l = blockIdx.x, tid = threadIdx.x;
  const int words = (F + 31) / 32;
  uint32_t key[WPT][32];
  bool nan = false;
  load_score_keys<WPT, V4>(scores + (size_t)l * F, F, tid, key, &nan);
  if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
  uint32_t sel[WPT];
  block_select_largest<NT, WPT>(key, (uint32_t)k, sel, hist, scan, res);
  write_selection<NT, WPT>(sel, tid, words, k, mask + (size_t)l * words,
                           active_ids + (size_t)l * k, nullptr, scan);
}

// Order of the victims as a selection key: the smallest last_used first, so
// never (-1) has the largest key and a later token a smaller one; never 0,
// which marks rows that are no candidates.
__device__ inline uint32_t victim_key(uint32_t used) {
  const uint32_t key = ~(used + 1u);
  return key > 1u ? key : 1u;
}

// The delta of one layer, run by all NT threads of its workgroup, for any
// state, also an inconsistent one.  Thread t owns: actives j in [t*JPT,
// t*JPT+JPT), id words [t*WPT, t*WPT+WPT) and slot words [t*spt, t*spt+spt), so
// every list below comes out in ascending order from a prefix sum in thread
// order.
//   A: the layer's active ids (na of them, ascending); P, Q, U: its slot_of,
//   neuron_of and last_used, read and updated in global memory (a thread
//   reads an entry before any thread writes it).
//   amask, rmask: >= ceil(F/32) words, smask: >= ceil(C/32) words of LDS;
//   pool: >= na entries of LDS.
// Every global gather of a phase is issued unconditionally (clamped index)
// so that the phase costs one memory round trip, not one per element.
template <int NT, int WPT, int JPT>
__device__ inline void delta_layer(int l, int32_t token, const int32_t* A, int na, bool bad_count,
                                   int32_t* P, int32_t* Q, int32_t* U, const np_delta_out& out,
                                   int F, int C, int k, int spt, void* ws, uint32_t* amask,
                                   uint32_t* smask, uint32_t* rmask, uint32_t* hist,
                                   int32_t* pool, uint32_t* scan, uint32_t* res) {
  const int tid = threadIdx.x;
  const int idwords = (F + 31) / 32, slotwords = (C + 31) / 32;
  const size_t lo = (size_t)l * k;

  for (int i = tid; i < idwords; i += NT) {
    amask[i] = 0;
    rmask[i] = 0;
  }
  __syncthreads();

  // 1. hits and incoming rows, in active-list order
  int nj[JPT], pj[JPT];
  uint32_t hits = 0, incs = 0, bad = 0;
#pragma unroll
  for (int q = 0; q < JPT; ++q) nj[q] = A[min(tid * JPT + q, na > 0 ? na - 1 : 0)];
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const bool ok = nj[q] >= 0 && nj[q] < F;  // else not a neuron id: counted as a miss
    if (tid * JPT + q < na) bad |= !ok;
    if (!ok) nj[q] = -1;
    pj[q] = P[nj[q] >= 0 ? nj[q] : 0];
  }
  int qb[JPT];  // a hit's slot must hold it
#pragma unroll
  for (int q = 0; q < JPT; ++q) qb[q] = Q[(pj[q] >= 0 && pj[q] < C) ? pj[q] : 0];
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = tid * JPT + q;
    if (nj[q] < 0 || pj[q] >= C) {
      bad |= (j < na) & (pj[q] >= C) & (nj[q] >= 0);
      pj[q] = -1;
    }
    if (pj[q] >= 0 && qb[q] != nj[q]) {
      bad |= j < na;
      pj[q] = -1;
    }
    if (j < na) {
      if (nj[q] >= 0) atomicOr(&amask[nj[q] >> 5], 1u << (nj[q] & 31));
      if (pj[q] >= 0) ++hits;
      else ++incs;
    }
  }
  uint32_t tot;
  const uint32_t before = block_excl_scan<NT>(hits | (incs << 16), scan, &tot);
  const uint32_t nH = tot & 0xFFFFu, nI = tot >> 16;

  // 2. free slots and resident rows, and a consistency check of the slot
  //    map: a used slot's neuron must map back to it
  uint32_t nfree_local = 0;
  for (int q = 0; q < spt; ++q) {
    const int sw = tid * spt + q;
    if (sw >= slotwords) break;
    int qn[32];
#pragma unroll
    for (int b = 0; b < 32; ++b) qn[b] = Q[min(32 * sw + b, C - 1)];
    uint32_t bits = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // halves: 16 back-gathers in flight
      int back[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int qv = qn[16 * h + i];
        back[i] = P[(qv >= 0 && qv < F) ? qv : 0];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int b = 16 * h + i, sl = 32 * sw + b, qv = qn[b];
        if (sl < C) {
          if (qv == -1) {
            bits |= 1u << b;
          } else if (qv < 0 || qv >= F || back[i] != sl) {
            bad = 1;
          } else {
            atomicOr(&rmask[qv >> 5], 1u << (qv & 31));
          }
        }
      }
    }
    smask[sw] = bits;
    nfree_local += __builtin_popcount(bits);
  }
  uint32_t nfree;
  (void)block_excl_scan<NT>(nfree_local, scan, &nfree);  // its barriers publish rmask
  const uint32_t m = nI > nfree ? nI - nfree : 0u;

  // 3. victims: the m resident, non-active rows with the smallest
  //    (last_used, id) -- the largest victim keys, ties to lower ids.
  //    Each victim leaves the slot map here: its slot joins the pool.
  uint32_t vsel[WPT];
#pragma unroll
  for (int w = 0; w < WPT; ++w) vsel[w] = 0;
  if (m > 0) {
    uint32_t key[WPT][32];
    if (32 * WPT * tid < F) {
#pragma unroll
      for (int w = 0; w < WPT; ++w) {
        const int word = tid * WPT + w;
#pragma unroll
        for (int b = 0; b < 32; ++b) key[w][b] = (uint32_t)U[min(32 * word + b, F - 1)];
        // resident, not active, and inside the layer (rmask has no bits past F)
        const uint32_t cm = word < idwords ? (rmask[word] & ~amask[word]) : 0u;
#pragma unroll
        for (int b = 0; b < 32; ++b) key[w][b] = ((cm >> b) & 1u) ? victim_key(key[w][b]) : 0u;
      }
    } else {
#pragma unroll
      for (int w = 0; w < WPT; ++w)
#pragma unroll
        for (int b = 0; b < 32; ++b) key[w][b] = 0u;
    }
    block_select_largest<NT, WPT>(key, m, vsel, hist, scan, res);
    uint32_t cv = 0;
#pragma unroll
    for (int w = 0; w < WPT; ++w) cv += __builtin_popcount(vsel[w]);
    uint32_t vt;
    uint32_t vpos = block_excl_scan<NT>(cv, scan, &vt);
#pragma unroll
    for (int w = 0; w < WPT; ++w) {
      if (!vsel[w]) continue;
      const int word = tid * WPT + w;
      int pn[32];
#pragma unroll
      for (int b = 0; b < 32; ++b) pn[b] = P[min(32 * word + b, F - 1)];
#pragma unroll
      for (int b = 0; b < 32; ++b) {
        if (!((vsel[w] >> b) & 1u)) continue;
        const int n = 32 * word + b, old = pn[b];
        if (old < 0 || old >= C || vpos >= (uint32_t)k) {  // only with a corrupted state
          bad = 1;
          continue;
        }
        out.ev_ids[lo + vpos] = n;
        out.ev_slots[lo + vpos] = old;
        ++vpos;
        atomicOr(&smask[old >> 5], 1u << (old & 31));
        Q[old] = -1;
        P[n] = -1;
      }
    }
  }
  __syncthreads();

  // 4. the slot pool in ascending order: its first nI slots go to the
  //    incoming rows (ascending ids)
  uint32_t cs = 0;
  for (int q = 0; q < spt; ++q) {
    const int sw = tid * spt + q;
    if (sw < slotwords) cs += __builtin_popcount(smask[sw]);
  }
  uint32_t st;
  uint32_t spos = block_excl_scan<NT>(cs, scan, &st);
  const uint32_t spos_total = st < nI ? st : nI;  // slots actually handed out
  for (int q = 0; q < spt; ++q) {
    const int sw = tid * spt + q;
    if (sw >= slotwords) break;
    uint32_t bits = smask[sw];
    while (bits && spos < nI) {
      const int b = __builtin_ctz(bits);
      bits &= bits - 1;
      out.in_slots[lo + spos] = 32 * sw + b;
      pool[spos] = 32 * sw + b;
      ++spos;
    }
  }
  __syncthreads();

  // 5. incoming rows take their slots; lists and last_used
  uint32_t hb = before & 0xFFFFu, ib = before >> 16;
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = tid * JPT + q;
    if (j < na) {
      const int n = nj[q];
      int slot;
      if (pj[q] >= 0) {
        slot = pj[q];
        out.hit_ids[lo + hb] = n;
        ++hb;
      } else {
        // the pool holds at least nI slots unless the state was corrupted
        slot = ib < spos_total ? pool[ib] : -1;
        out.in_ids[lo + ib] = n;
        if (n >= 0 && slot >= 0 && slot < C) {
          P[n] = slot;
          Q[slot] = n;
        } else {
          bad = 1;
          slot = -1;
        }
        ++ib;
      }
      if (n >= 0) U[n] = token;
      out.active_slots[lo + j] = slot;
    }
  }
  if (bad || (bad_count && tid == 0)) raise_error(ws, NP_DEVERR_STATE);
  if (tid == 0) {
    out.counts[(size_t)l * 4 + 0] = (int32_t)nI;
    out.counts[(size_t)l * 4 + 1] = (int32_t)nH;
    out.counts[(size_t)l * 4 + 2] = (int32_t)m;
    out.counts[(size_t)l * 4 + 3] = (int32_t)(nI - m);
  }
}

// ---------------------------------------------------------------------------
// The selection and the delta with the layer's slot map in LDS: F <= 32768,
// C <= 16384 (slots and -1 in 16 bits), k <= 8192, 1024 threads.
//
// Bound by latency: one workgroup per layer, so the chain of barriers, LDS
// round trips and wave-wide scans is the time (the bytes, 0.15 to 0.5 MB a
// layer, take a fraction of it).  So every phase is cut to one barrier where
// it can be: prefix sums in DPP with one exchange of wave totals, histograms
// that every wave reads by itself (a coarse and a fine level, one bin a lane)
// instead of a workgroup scan, masks built with ballots from the values that
// are loaded anyway instead of LDS atomics, and the consistency of the slot map
// checked once, which frees every later step of its checks: an inconsistent
// layer takes delta_checked.  Per token before: 7B 23.3 us with 512 threads of
// 32 ids and about 45 barriers; 70B 22.3 + 21.2 us in two kernels that read the
// state from memory.  Now, a call: 7B 12.8 us, 70B 26.0 (kernel trace 12.4 and
// 26.0).  A layer that has no hint yet or misses its window runs the full
// search, and the call waits for its slowest layer: the first token takes 20.8
// and 43.8 us, a token with a miss 19 and 34 to 38 (7B: one of 31; 70B, 79
// layers: three of 11).
// ---------------------------------------------------------------------------
constexpr int SD_MAX_F = 32768;
constexpr int SD_MAX_C = 16384;
constexpr int SD_MAX_K = 8192;
constexpr int SD_BINS = 256;   // bins of the selection's window: four a lane
constexpr int SD_AGES = WAVE;  // bins of the victims' ages: one a lane
constexpr int SD_CAND = 64;    // keys of a bin resolved by one wave

// Sizes of one build: NT threads, KPT rows of 64 ids per wave, CPT slots and
// JPT active rows per thread.
template <int NT_, int KPT_, int CPT_, int JPT_>
struct Sd {
  static constexpr int NT = NT_, KPT = KPT_, CPT = CPT_, JPT = JPT_;
  static constexpr int NW = NT / WAVE, F = KPT * NT, C = CPT * NT, WORDS = F / 32;
  static_assert(KPT <= 32 && WORDS <= NT, "a row's words fit a wave's lanes, a thread owns a word");
};

// LDS of the fast path.  Key work: wave w owns KPT rows of 64 consecutive
// ids, lane i id 64 (w KPT + r) + i of row r, so loads are whole lines and a
// ballot is two mask words.  Ordered work: thread t owns mask word t.
template <class S>
struct SdLds {
  int16_t slot[S::F];              // slot_of at entry
  uint16_t ids[SD_MAX_K], pool[SD_MAX_K];  // active ids; slots for the incoming rows
  alignas(16) uint32_t smask[SD_MAX_C / 32];  // free slots, then also the victims'
  uint32_t amask[S::WORDS], rmask[S::WORDS];  // active, resident
  uint32_t gmask[S::WORDS], emask[S::WORDS];  // keys above, equal to the k-th
  alignas(16) uint32_t hist[SD_BINS];
  uint32_t vhist[SD_AGES];
  uint32_t cand[SD_CAND], scan[8][S::NW];
  uint32_t above, ncand, vmax, used, valid, nfree;
  uint32_t bad;  // set before step 2's barrier only
};
// LDS of delta_checked, when the slot map is inconsistent
struct SdChecked {
  uint32_t amask[SD_MAX_F / 32], smask[SD_MAX_F / 32], rmask[SD_MAX_F / 32], hist[256];
  int32_t pool[SD_MAX_K], held[SD_MAX_K];
  uint32_t scan[16];
};
template <class S>
union SdShared {
  SdLds<S> f;
  SdChecked g;
};

__device__ inline int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
}
template <int KPT>
__device__ inline int sd_id(int r) {
  return WAVE * (wave_id() * KPT + r) + (int)(threadIdx.x & (WAVE - 1));
}
// 32-bit loads of a layer's row of n entries: one address register for all
// rows, entries past the end read as 0 without a memory access.
struct RowLoads {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t off;
  __device__ inline RowLoads(const void* p, int n, int first)
      : rs(make_rsrc(p, (uint32_t)n * 4u)), off((uint32_t)first * 4u) {}
  __device__ inline uint32_t at(int r) const {  // entry first + 64 r
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off + 256u * (uint32_t)r), 0, 0);
  }
};

// The wave's rows of a predicate to mask words in LDS.
template <int KPT, class Fn>
__device__ inline void store_rows(uint32_t* words, Fn pred) {
  uint64_t b[KPT];
#pragma unroll
  for (int r = 0; r < KPT; ++r) b[r] = __ballot(pred(r));
  if ((threadIdx.x & (WAVE - 1)) == 0) {
    uint64_t* w = reinterpret_cast<uint64_t*>(words) + KPT * wave_id();
#pragma unroll
    for (int r = 0; r < KPT; ++r) w[r] = b[r];
  }
}

// The bin of a 256-bin histogram that holds the rem-th key counted from bin 0
// up, the keys before it, its count, and all keys; every wave by itself.
// Returns false when the histogram holds fewer than rem.
__device__ inline bool find_bin(const uint32_t* hist, uint32_t rem, uint32_t* bin,
                                uint32_t* before, uint32_t* count, uint32_t* total) {
  const int lane = threadIdx.x & (WAVE - 1);
  const uint4 h = reinterpret_cast<const uint4*>(hist)[lane];
  const uint32_t sum = h.x + h.y + h.z + h.w;
  const uint32_t incl = wave_incl_scan(sum);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
  const uint64_t hit = __ballot(incl >= rem);
  if (!hit) return false;
  // within the lane: the first of its four bins that reaches rem
  uint32_t acc = incl - sum, b = 0, c = h.x;
  if (acc + c < rem) acc += c, b = 1, c = h.y;
  if (acc + c < rem) acc += c, b = 2, c = h.z;
  if (acc + c < rem) acc += c, b = 3, c = h.w;
  const int at = __builtin_ctzll(hit);
  *bin = 4u * (uint32_t)at + (uint32_t)__builtin_amdgcn_readlane((int)b, at);
  *before = (uint32_t)__builtin_amdgcn_readlane((int)acc, at);
  *count = (uint32_t)__builtin_amdgcn_readlane((int)c, at);
  return true;
}

// The k largest keys of the layer (ties to the smaller ids), starting from a
// hint kept per layer in the workspace: the previous token's k-th key and a
// window half-width.  Scores change little from one token to the next, so the
// new k-th key usually lies in [key - half, key + half].  One pass counts the
// keys above the window and puts those inside into a histogram; every wave
// finds the k-th key's bin, and the few keys of that bin decide.  Whatever the
// hint holds, the result is the same: when the k-th key is outside the window
// or its bin holds more than SD_CAND keys, the full radix search runs.  The
// hint is updated: the new k-th key, the window halved when it held many keys
// (each costs an LDS atomic), quadrupled when the k-th key fell outside it.
// At 7B it settles between 120 and 240 keys, half-widths of 0.02 to 0.05 in
// score, against steps of the k-th key of about 0.004.
constexpr uint32_t SEL_HINT_MANY = 240;
constexpr uint32_t SEL_HINT_HALF0 = 1u << 20;  // first window half-width (fp32 keys: 0.125 at 1.0)

// Leaves the selected ids in s.amask, behind a barrier.
template <class S>
__device__ inline void select_hinted(const uint32_t (&key)[1][S::KPT], uint32_t kk, SdLds<S>& s,
                                     uint32_t* work, uint32_t* hint, uint32_t hkey,
                                     uint32_t half) {
  constexpr int KPT = S::KPT;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const uint32_t lo = hkey > half ? hkey - half : 1u;
  const uint32_t hi = hkey < 0xFFFFFFFFu - half ? hkey + half : 0xFFFFFFFFu;
  const bool window = hkey != 0u && half != 0u;
  bool use = false;
  uint32_t kth = 0, eq_take = 0, eq_all = 0, inside = 0;
  if (window) {
    const uint32_t width = hi - lo;  // bins of 2^shift keys, from the top
    const int bits = width ? 32 - __builtin_clz(width) : 0;
    const int shift = bits > 8 ? bits - 8 : 0;
    uint32_t above = 0;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const uint32_t d = hi - key[0][r];  // a key above hi wraps to more than hi >= width
      above += (uint32_t)__popcll(__ballot(d > hi));
      if (d <= width) atomicAdd(&s.hist[d >> shift], 1u);
    }
    if (lane == 0 && above) atomicAdd(&s.above, above);
    lds_barrier();
    above = s.above;
    uint32_t bin = 0, before = 0, count = 0;
    use = above < kk && find_bin(s.hist, kk - above, &bin, &before, &count, &inside) &&
          count <= SD_CAND;
    if (use) {  // the keys of the bin, in any order
      const uint32_t rem = kk - above - before;
      const uint32_t first = bin << shift, last = min((uint32_t)((1u << shift) - 1u), width - first);
#pragma unroll
      for (int r = 0; r < KPT; ++r)
        if (hi - first - key[0][r] <= last) s.cand[atomicAdd(&s.ncand, 1u)] = key[0][r];
      lds_barrier();
      const uint32_t mine = (uint32_t)lane < count ? s.cand[lane] : 0u;
      uint32_t gt = 0, eq = 0;  // keys of the bin above this lane's, equal to it
      for (uint32_t j = 0; j < count; ++j) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)j);
        gt += o > mine;
        eq += o == mine;
      }
      const int at = __builtin_ctzll(__ballot((uint32_t)lane < count && gt < rem && rem <= gt + eq));
      kth = (uint32_t)__builtin_amdgcn_readlane((int)mine, at);
      eq_take = rem - (uint32_t)__builtin_amdgcn_readlane((int)gt, at);
      eq_all = (uint32_t)__builtin_amdgcn_readlane((int)eq, at);
    }
  }
  if (!use)  // in LDS of its own: slower waves may still read the window's
    kth = block_find_kth<S::NT, 1>(key, kk, &eq_take, work, work + 4096,
                                   work + 4096 + 3 * S::NW + 1);
  if (use && eq_take == eq_all) {  // every equal key is taken (usually the one)
    store_rows<KPT>(s.amask, [&](int r) { return key[0][r] >= kth; });
    lds_barrier();
  } else {  // the first eq_take of them in id order
    store_rows<KPT>(s.gmask, [&](int r) { return key[0][r] > kth; });
    store_rows<KPT>(s.emask, [&](int r) { return key[0][r] == kth; });
    lds_barrier();
    uint32_t sel = tid < S::WORDS ? s.gmask[tid] : 0u, eq = tid < S::WORDS ? s.emask[tid] : 0u, tot;
    uint32_t n = block_excl_scan_once<S::NT>(__builtin_popcount(eq), s.scan[0], &tot);
    while (eq && n < eq_take) {
      sel |= eq & (0u - eq);
      eq &= eq - 1;
      ++n;
    }
    if (tid < S::WORDS) s.amask[tid] = sel;
    lds_barrier();
  }
  if (hint && tid == 0) {
    uint32_t h = half ? half : SEL_HINT_HALF0;
    if (use) {
      if (inside > SEL_HINT_MANY && h > 1u) h >>= 1;
    } else if (window) {
      h = h < (1u << 29) ? h << 2 : h;
    }
    hint[0] = kth;  // 0 when NaN keys were taken
    hint[1] = h;
  }
}

// slot_of of one layer to LDS, its resident bits to s.rmask, the valid entries
// counted; an entry outside {-1} and [0, C) sets bad.
template <class S>
__device__ inline void store_slots(const uint32_t (&v)[S::KPT], SdLds<S>& s, int F, int C) {
  uint32_t valid = 0, odd = 0;
  store_rows<S::KPT>(s.rmask, [&](int r) {
    const int n = sd_id<S::KPT>(r);
    s.slot[n] = (int16_t)v[r];
    const bool in = n < F;
    odd |= in ? (uint32_t)(v[r] + 1u > (uint32_t)C) : 0u;
    const bool held = in && (int)v[r] >= 0;
    valid += (uint32_t)__popcll(__ballot(held));
    return held;
  });
  if ((threadIdx.x & (WAVE - 1)) == 0 && valid) atomicAdd(&s.valid, valid);
  if (odd) s.bad = 1u;
}

// Clears the counters and histograms; a barrier must follow before their use.
template <class S>
__device__ inline void sd_clear(SdLds<S>& s) {
  const int tid = threadIdx.x;
  if (tid < SD_BINS) s.hist[tid] = 0u;
  if (tid < SD_AGES) s.vhist[tid] = 0u;
  if (tid == 0) s.above = s.ncand = s.vmax = s.used = s.valid = s.nfree = s.bad = 0u;
}

// The delta of one layer with a consistent slot map in LDS.  qv: this thread's
// neuron_of entries (slot tid + NT i); s.ids: the na active ids, ascending,
// also written to ids_out when that is not null; s.slot, s.amask, s.rmask,
// s.valid and s.bad complete behind a barrier.  Returns false, having written
// nothing, when the slot map turns out inconsistent.
template <class S>
__device__ inline bool delta_fast(int l, int32_t token, int na, const int (&qv)[S::CPT],
                                  int32_t* P, int32_t* Q, int32_t* U, int32_t* ids_out,
                                  const np_delta_out& out, int F, int C, int k, SdLds<S>& s,
                                  uint32_t* work) {
  constexpr int KPT = S::KPT, CPT = S::CPT, JPT = S::JPT, NT = S::NT;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const size_t lo = (size_t)l * k;
  // the ids' last_used, for the victims: in flight from here on, or from
  // behind step 1 where the registers do not hold both
  uint32_t key[1][KPT];
  const RowLoads used_rows(U, F, sd_id<KPT>(0));
  auto load_used = [&] {
#pragma unroll
    for (int r = 0; r < KPT; ++r) key[0][r] = used_rows.at(r);
  };
  if constexpr (KPT < 32) load_used();
  // 1. free slots, and the consistency of the map: a used slot's neuron must
  //    map back to it, and no more neurons may hold slots than slots are used
  {
    int back[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      back[i] = (uint32_t)qv[i] < (uint32_t)F ? (int)s.slot[qv[i]] : -2;
    uint32_t nfree = 0, used = 0;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      if (NT * i < C) {
        const int sl = tid + NT * i;
        const bool in = sl < C, fr = in && qv[i] == -1, us = in && qv[i] != -1;
        bad |= us && back[i] != sl;
        const uint64_t fm = __ballot(fr);
        nfree += (uint32_t)__popcll(fm);
        used += (uint32_t)__popcll(__ballot(us));
        if (lane == 0) *(uint2*)&s.smask[sl >> 5] = make_uint2((uint32_t)fm, (uint32_t)(fm >> 32));
      }
    }
    if (lane == 0) {
      if (nfree) atomicAdd(&s.nfree, nfree);
      if (used) atomicAdd(&s.used, used);
    }
    if (bad) s.bad = 1u;
  }
  if constexpr (KPT == 32) {
    __builtin_amdgcn_sched_barrier(0);
    load_used();
  }
  // 2. hits and incoming rows, in active-list order
  int nj[JPT], pj[JPT];
  uint32_t cnt = 0;  // hits | incoming << 16
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = tid * JPT + q;
    nj[q] = s.ids[min(j, na > 0 ? na - 1 : 0)];
    pj[q] = s.slot[na > 0 ? nj[q] : 0];
    if (j < na) cnt += pj[q] >= 0 ? 1u : 0x10000u;
  }
  uint32_t tot;
  const uint32_t before = block_excl_scan_once<NT>(cnt, s.scan[1], &tot);
  // uniform: nothing writes these words from the barrier on (a wave may read
  // them while another is in step 3 already)
  if (s.bad || s.used != s.valid) return false;
  const uint32_t nH = tot & 0xFFFFu, nI = tot >> 16;
  const uint32_t m = nI > s.nfree ? nI - s.nfree : 0u;
  // 3. victims: the m resident, non-active rows with the smallest (last_used,
  //    id) -- the largest victim keys, ties to lower ids; their slots join the
  //    free ones (k <= C: a consistent map holds at least m candidates)
  if (m > 0) {
    const uint32_t cw = lane < 2 * KPT ? s.rmask[2 * KPT * wave_id() + lane] &
                                             ~s.amask[2 * KPT * wave_id() + lane]
                                       : 0u;
    uint32_t mx = 0;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const uint64_t row = (uint32_t)__builtin_amdgcn_readlane((int)cw, 2 * r) |
                           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)cw, 2 * r + 1) << 32);
      const bool cand = __builtin_amdgcn_inverse_ballot_w64(row);
      key[0][r] = cand ? victim_key(key[0][r]) : 0u;
      mx = key[0][r] > mx ? key[0][r] : mx;
    }
    mx = wave_max(mx);
    if (lane == 0 && mx) atomicMax(&s.vmax, mx);
    lds_barrier();
    mx = s.vmax;
    // ages from the oldest candidate's token on, one bin each; the oldest
    // SD_AGES of them nearly always hold m rows
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const uint32_t d = mx - key[0][r];
      if (key[0][r] != 0u && d < (uint32_t)SD_AGES) atomicAdd(&s.vhist[d], 1u);
    }
    lds_barrier();
    uint32_t kth, take;
    const uint32_t ages = wave_incl_scan(s.vhist[lane]);
    const uint64_t hit = __ballot(ages >= m);
    if (hit) {
      const int at = __builtin_ctzll(hit);
      take = m - (at > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)ages, at > 0 ? at - 1 : 0) : 0u);
      kth = mx - (uint32_t)at;
    } else {
      kth = block_find_kth<NT, 1>(key, m, &take, work, work + 4096, work + 4096 + 3 * S::NW + 1);
    }
    // all older ones and the first `take` equal ones in id order; one prefix
    // sum places both
    store_rows<KPT>(s.gmask, [&](int r) { return key[0][r] > kth; });
    store_rows<KPT>(s.emask, [&](int r) { return key[0][r] == kth; });
    lds_barrier();
    uint32_t v = tid < S::WORDS ? s.gmask[tid] : 0u, eq = tid < S::WORDS ? s.emask[tid] : 0u, t2;
    const uint32_t pre = block_excl_scan_once<NT>(
        (uint32_t)__builtin_popcount(v) | ((uint32_t)__builtin_popcount(eq) << 16), s.scan[2], &t2);
    uint32_t ne = pre >> 16, vpos = (pre & 0xFFFFu) + (ne < take ? ne : take);
    while (eq && ne < take) {
      v |= eq & (0u - eq);
      eq &= eq - 1;
      ++ne;
    }
    while (v) {
      const int id = 32 * tid + __builtin_ctz(v), old = s.slot[id];
      v &= v - 1;
      out.ev_ids[lo + vpos] = id;
      out.ev_slots[lo + vpos] = old;
      ++vpos;
      atomicOr(&s.smask[old >> 5], 1u << (old & 31));
      Q[old] = -1;
      P[id] = -1;
    }
    lds_barrier();
  }
  // 4. the slot pool in ascending order: its first nI slots go to the
  //    incoming rows (ascending ids); 8 or 16 slots a thread
  {
    static_assert(CPT <= 16, "NT threads of 16 slots cover the layer");
    const int per = C <= 8 * NT ? 8 : 16;
    uint32_t bits = per * tid < C ? (s.smask[(per * tid) >> 5] >> ((per * tid) & 31)) : 0u;
    bits &= (1u << per) - 1u;
    uint32_t st;
    uint32_t pos = block_excl_scan_once<NT>(__builtin_popcount(bits), s.scan[3], &st);
    while (bits && pos < nI) {
      const int sl = per * tid + __builtin_ctz(bits);
      bits &= bits - 1;
      out.in_slots[lo + pos] = sl;
      s.pool[pos] = (uint16_t)sl;
      ++pos;
    }
  }
  __syncthreads();  // the victims' stores to P and Q come before the incoming rows'
  // 5. incoming rows take their slots; lists and last_used
  uint32_t hb = before & 0xFFFFu, ib = before >> 16;
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = tid * JPT + q;
    if (j < na) {
      const int n = nj[q];
      int slot = pj[q];
      if (slot >= 0) {
        out.hit_ids[lo + hb++] = n;
      } else {
        slot = s.pool[ib];
        out.in_ids[lo + ib++] = n;
        P[n] = slot;
        Q[slot] = n;
      }
      U[n] = token;
      if (ids_out) ids_out[j] = n;
      out.active_slots[lo + j] = slot;
    }
  }
  if (tid == 0) {
    out.counts[(size_t)l * 4 + 0] = (int32_t)nI;
    out.counts[(size_t)l * 4 + 1] = (int32_t)nH;
    out.counts[(size_t)l * 4 + 2] = (int32_t)m;
    out.counts[(size_t)l * 4 + 3] = (int32_t)(nI - m);
  }
  return true;
}

// The delta of one layer whose slot map delta_fast found inconsistent (or
// whose ids are not ascending neuron ids): delta_layer's steps and results,
// entry by entry from memory with every check, in few registers so that it
// costs the fast path none.  Thread t owns id word t, slot word t and actives
// [t*jpt, t*jpt+jpt).
template <int NT>
__device__ inline void delta_checked(int l, int32_t token, const int32_t* A, int na,
                                     bool bad_count, int32_t* P, int32_t* Q, int32_t* U,
                                     const np_delta_out& out, int F, int C, int k, void* ws,
                                     SdChecked& g) {
  const int tid = threadIdx.x, jpt = (k + NT - 1) / NT;
  const size_t lo = (size_t)l * k;
  const int j0 = min(tid * jpt, na), j1 = min(tid * jpt + jpt, na);
  __syncthreads();  // every thread is done with the LDS of the fast path
  g.amask[tid] = g.rmask[tid] = 0u;
  __syncthreads();
  uint32_t cnt = 0, bad = bad_count && tid == 0;
#pragma unroll 1
  for (int j = j0; j < j1; ++j) {  // hits and incoming rows
    const int n = A[j];
    int p = -1;
    if (n >= 0 && n < F) {
      atomicOr(&g.amask[n >> 5], 1u << (n & 31));
      p = P[n];
      if (p >= C || (p >= 0 && Q[p] != n)) {
        bad = 1;
        p = -1;
      }
    } else {
      bad = 1;
    }
    if (p < 0) p = -1;
    g.held[j] = p;
    cnt += p >= 0 ? 1u : 0x10000u;
  }
  uint32_t tot;
  const uint32_t before = block_excl_scan<NT>(cnt, g.scan, &tot);
  const uint32_t nH = tot & 0xFFFFu, nI = tot >> 16;
  uint32_t bits = 0;
#pragma unroll 1
  for (int sl = 32 * tid; sl < min(32 * tid + 32, C); ++sl) {  // free slots, resident rows
    const int q = Q[sl];
    if (q == -1) bits |= 1u << (sl & 31);
    else if (q < 0 || q >= F || P[q] != sl) bad = 1;
    else atomicOr(&g.rmask[q >> 5], 1u << (q & 31));
  }
  g.smask[tid] = bits;
  uint32_t nfree;
  (void)block_excl_scan<NT>(__builtin_popcount(bits), g.scan, &nfree);
  const uint32_t m = nI > nfree ? nI - nfree : 0u;
  if (m > 0) {  // the m largest victim keys of the resident, non-active rows
    const uint32_t cm = g.rmask[tid] & ~g.amask[tid];
    auto key = [&](int b) { return ((cm >> b) & 1u) ? victim_key((uint32_t)U[32 * tid + b]) : 0u; };
    uint32_t nz = 0;
#pragma unroll 1
    for (int b = 0; b < 32; ++b) nz += key(b) != 0u;
    (void)block_excl_scan<NT>(nz, g.scan, &nz);
    uint32_t prefix = 0, pmask = 0, rem = m >= nz ? m - nz : m;
    if (m < nz) {
#pragma unroll 1
      for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) g.hist[tid] = 0u;
        __syncthreads();
#pragma unroll 1
        for (int b = 0; b < 32; ++b) {
          const uint32_t kv = key(b);
          if (kv != 0u && (kv & pmask) == prefix) atomicAdd(&g.hist[(kv >> shift) & 255u], 1u);
        }
        __syncthreads();
        uint32_t bin = 255;
        while (bin > 0u && g.hist[bin] < rem) rem -= g.hist[bin--];
        prefix |= bin << shift;
        pmask |= 255u << shift;
        __syncthreads();
      }
    }
    uint32_t vsel = 0, eq = 0;
#pragma unroll 1
    for (int b = 0; b < 32; ++b) {
      const uint32_t kv = key(b);
      vsel |= (kv > prefix ? 1u : 0u) << b;
      eq |= (kv == prefix ? 1u : 0u) << b;
    }
    uint32_t t2;
    uint32_t ne = block_excl_scan<NT>(__builtin_popcount(eq), g.scan, &t2);
    while (eq && ne < rem) {
      vsel |= eq & (0u - eq);
      eq &= eq - 1;
      ++ne;
    }
    uint32_t vpos = block_excl_scan<NT>(__builtin_popcount(vsel), g.scan, &t2);
#pragma unroll 1
    while (vsel) {
      const int n = 32 * tid + __builtin_ctz(vsel), old = P[min(n, F - 1)];
      vsel &= vsel - 1;
      if (old < 0 || old >= C || vpos >= (uint32_t)k) {
        bad = 1;
        continue;
      }
      out.ev_ids[lo + vpos] = n;
      out.ev_slots[lo + vpos] = old;
      ++vpos;
      atomicOr(&g.smask[old >> 5], 1u << (old & 31));
      Q[old] = -1;
      P[n] = -1;
    }
  }
  __syncthreads();
  bits = g.smask[tid];
  uint32_t st;
  uint32_t pos = block_excl_scan<NT>(__builtin_popcount(bits), g.scan, &st);
  const uint32_t given = st < nI ? st : nI;  // slots actually handed out
#pragma unroll 1
  while (bits && pos < nI) {
    const int sl = 32 * tid + __builtin_ctz(bits);
    bits &= bits - 1;
    out.in_slots[lo + pos] = sl;
    g.pool[pos] = sl;
    ++pos;
  }
  __syncthreads();
  uint32_t hb = before & 0xFFFFu, ib = before >> 16;
#pragma unroll 1
  for (int j = j0; j < j1; ++j) {
    int n = A[j], slot = g.held[j];
    if (n < 0 || n >= F) n = -1;
    if (slot >= 0) {
      out.hit_ids[lo + hb++] = n;
    } else {
      slot = ib < given ? g.pool[ib] : -1;
      out.in_ids[lo + ib++] = n;
      if (n >= 0 && slot >= 0 && slot < C) {
        P[n] = slot;
        Q[slot] = n;
      } else {
        bad = 1;
        slot = -1;
      }
    }
    if (n >= 0) U[n] = token;
    out.active_slots[lo + j] = slot;
  }
  if (bad) raise_error(ws, NP_DEVERR_STATE);
  if (tid == 0) {
    out.counts[(size_t)l * 4 + 0] = (int32_t)nI;
    out.counts[(size_t)l * 4 + 1] = (int32_t)nH;
    out.counts[(size_t)l * 4 + 2] = (int32_t)m;
    out.counts[(size_t)l * 4 + 3] = (int32_t)(nI - m);
  }
}

// np_delta and np_delta_n with the slot map in LDS.  Ids that are not
// strictly ascending neuron ids go to delta_checked, as does an inconsistent
// slot map.
template <class S>
__global__ __launch_bounds__(S::NT) void delta_lds_kernel(
    int32_t token, const int32_t* __restrict__ active_ids, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ neuron_of, int32_t* __restrict__ last_used, np_delta_out out, int F,
    int C, int k, void* ws, const int32_t* __restrict__ counts) {
  __shared__ __attribute__((aligned(16))) SdShared<S> sh;
  __shared__ uint32_t work[4096 + 3 * S::NW + 1 + 4];
  constexpr int KPT = S::KPT, CPT = S::CPT, JPT = S::JPT, NT = S::NT;
  SdLds<S>& s = sh.f;
  const int l = blockIdx.x, tid = threadIdx.x;
  if (token == NP_TOKEN_AUTO) token = *(const int32_t*)((const char*)ws + WS_TOKEN);
  int32_t* P = slot_of + (size_t)l * F;
  int32_t* Q = neuron_of + (size_t)l * C;
  int32_t* U = last_used + (size_t)l * F;
  const int32_t* A = active_ids + (size_t)l * k;
  uint32_t pv[KPT];
  const RowLoads slot_rows(P, F, sd_id<KPT>(0));
#pragma unroll
  for (int r = 0; r < KPT; ++r) pv[r] = slot_rows.at(r);
  int na = k;  // active neurons of this layer: k, or a device count in [0, k]
  bool bad_count = false;
  if (counts) {
    na = counts[l];
    if (na < 0 || na > k) {
      bad_count = true;
      na = na < 0 ? 0 : k;
    }
  }
  int id[JPT], prev[JPT];
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = min(tid + NT * q, k - 1);
    id[q] = A[j];
    prev[q] = A[j > 0 ? j - 1 : 0];
  }
  int qv[CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) qv[i] = Q[min(tid + NT * i, C - 1)];
  sd_clear(s);
  if (tid < S::WORDS) s.amask[tid] = 0u;
  lds_barrier();
  store_slots<S>(pv, s, F, C);
#pragma unroll
  for (int q = 0; q < JPT; ++q) {
    const int j = tid + NT * q;
    if (j < na) {
      const bool ok = id[q] >= 0 && id[q] < F && (j == 0 || id[q] > prev[q]);
      if (ok) {
        s.ids[j] = (uint16_t)id[q];
        atomicOr(&s.amask[id[q] >> 5], 1u << (id[q] & 31));
      } else {
        s.ids[j] = 0;
        s.bad = 1u;
      }
    }
  }
  lds_barrier();
  if (!delta_fast<S>(l, token, na, qv, P, Q, U, nullptr, out, F, C, k, s, work))
    delta_checked<NT>(l, token, A, na, bad_count, P, Q, U, out, F, C, k, ws, sh.g);
  else if (bad_count && tid == 0)
    raise_error(ws, NP_DEVERR_STATE);
}

// np_delta for any size: one workgroup per layer, the state read from global
// memory.
template <int NT, int WPT, int JPT>
__global__ __launch_bounds__(NT) void delta_kernel(int32_t token,
                                                   const int32_t* __restrict__ active_ids,
                                                   int32_t* __restrict__ slot_of,
                                                   int32_t* __restrict__ neuron_of,
                                                   int32_t* __restrict__ last_used,
                                                   np_delta_out out, int F, int C, int k,
                                                   int spt, void* ws,
                                                   const int32_t* __restrict__ counts) {
  __shared__ uint32_t amask[2048];  // active set, bit n of the layer
  __shared__ uint32_t smask[2048];  // slot pool: free slots, then victims' slots
  __shared__ uint32_t rmask[2048];  // resident rows (neurons held by some slot)
  __shared__ uint32_t hist[4096];
  __shared__ int32_t pool[8192];    // the first nI pool slots, ascending
  __shared__ uint32_t scan[3 * (NT / WAVE) + 1];
  __shared__ uint32_t res[4];
  const int l = blockIdx.x;
  if (token == NP_TOKEN_AUTO) token = *(const int32_t*)((const char*)ws + WS_TOKEN);
  // active neurons of this layer: k, or a device count in [0, k]
  int na = k;
  bool bad_count = false;
  if (counts) {
    na = counts[l];
    if (na < 0 || na > k) {
      bad_count = true;
      na = na < 0 ? 0 : k;
    }
  }
  delta_layer<NT, WPT, JPT>(l, token, active_ids + (size_t)l * k, na, bad_count,
                            slot_of + (size_t)l * F, neuron_of + (size_t)l * C,
                            last_used + (size_t)l * F, out, F, C, k, spt, ws, amask, smask, rmask,
                            hist, pool, scan, res);
}

// np_select followed by np_delta in one workgroup per layer.  At entry every
// thread issues its loads at once: slot_of and the scores (the selection keys)
// of its ids and a share of neuron_of.
template <class S>
__global__ __launch_bounds__(S::NT) void select_delta_kernel(
    const float* __restrict__ scores, uint32_t* __restrict__ mask,
    int32_t* __restrict__ active_ids, int32_t token, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ neuron_of, int32_t* __restrict__ last_used, np_delta_out out, int F,
    int C, int k, void* ws) {
  __shared__ __attribute__((aligned(16))) SdShared<S> sh;
  __shared__ uint32_t work[4096 + 3 * S::NW + 1 + 4];
  constexpr int KPT = S::KPT, CPT = S::CPT, NT = S::NT;
  SdLds<S>& s = sh.f;
  const int l = blockIdx.x, tid = threadIdx.x;
  if (token == NP_TOKEN_AUTO) token = *(const int32_t*)((const char*)ws + WS_TOKEN);
  const int words = (F + 31) / 32;
  int32_t* P = slot_of + (size_t)l * F;
  int32_t* Q = neuron_of + (size_t)l * C;
  int32_t* U = last_used + (size_t)l * F;
  const float* sc = scores + (size_t)l * F;
  uint32_t pv[KPT], key[1][KPT];
  const RowLoads slot_rows(P, F, sd_id<KPT>(0)), score_rows(sc, F, sd_id<KPT>(0));
#pragma unroll
  for (int r = 0; r < KPT; ++r) pv[r] = slot_rows.at(r);
#pragma unroll
  for (int r = 0; r < KPT; ++r) key[0][r] = score_rows.at(r);
  uint32_t* hint = l < WS_SEL_HINT_LAYERS ? (uint32_t*)((char*)ws + WS_SEL_HINT) + 2 * l : nullptr;
  const uint32_t hkey = hint ? hint[0] : 0u, half = hint ? hint[1] : 0u;
  sd_clear(s);
  lds_barrier();
  store_slots<S>(pv, s, F, C);
  bool nan = false;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const uint32_t kv = score_key(__uint_as_float(key[0][r]), &nan);
    key[0][r] = sd_id<KPT>(r) < F ? kv : 0u;
  }
  if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
  int qv[CPT];  // behind the selection where the registers do not hold both
  auto load_q = [&] {
#pragma unroll
    for (int i = 0; i < CPT; ++i) qv[i] = Q[min(tid + NT * i, C - 1)];
  };
  if constexpr (KPT < 32) load_q();
  select_hinted<S>(key, (uint32_t)k, s, work, hint, hkey, half);
  if constexpr (KPT == 32) load_q();
  {  // the mask, and the ids in ascending order
    uint32_t sel = tid < S::WORDS ? s.amask[tid] : 0u, tot;
    if (tid < words) mask[(size_t)l * words + tid] = sel;
    uint32_t pos = block_excl_scan_once<NT>(__builtin_popcount(sel), s.scan[4], &tot);
    while (sel) {
      const int n = 32 * tid + __builtin_ctz(sel);
      sel &= sel - 1;
      if (pos < (uint32_t)k) s.ids[pos] = (uint16_t)n;
      ++pos;
    }
  }
  lds_barrier();  // s.ids complete
  int32_t* ids_out = active_ids + (size_t)l * k;
  if (!delta_fast<S>(l, token, k, qv, P, Q, U, ids_out, out, F, C, k, s, work)) {
    for (int j = tid; j < k; j += NT) ids_out[j] = s.ids[j];
    __syncthreads();
    __threadfence_block();  // the ids are read back from memory
    delta_checked<NT>(l, token, ids_out, k, false, P, Q, U, out, F, C, k, ws, sh.g);
  }
}

// Centroid choice and the intersected active set (Sec. 3.3-3.4), one
// workgroup per layer.  Waves 0 and 1 take the argmax of the layer's gate and
// up heads over the K logits (lane c reads c, c+64, ...; a NaN never wins and
// sets the error bit; equal values go to the smaller index).  Then thread t
// owns id words [t*WPT, t*WPT+WPT) of the AND of the two chosen masks, and a
// workgroup prefix sum places its ids in ascending order.
template <int NT, int WPT>
__global__ __launch_bounds__(NT) void centroid_active_kernel(
    const float* __restrict__ logits, const uint32_t* __restrict__ bank,
    int32_t* __restrict__ cids, uint32_t* __restrict__ mask, int32_t* __restrict__ active_ids,
    int32_t* __restrict__ counts, int L, int F, int K, int k, void* ws) {
  __shared__ int chosen[2];
  __shared__ uint32_t scan[NT / WAVE + 1];
  const int l = blockIdx.x, tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
  if (w < 2) {
    const int h = w * L + l;
    const float* lg = logits + (size_t)h * K;
    float best = 0.f;
    int bi = K;  // K: nothing seen yet
    bool nan = false;
    for (int c = lane; c < K; c += WAVE) {
      const float v = lg[c];
      if (v != v) {
        nan = true;
        continue;
      }
      if (bi == K || v > best) {  // ascending c: a lane keeps its first maximum
        best = v;
        bi = c;
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const float ob = __shfl_xor(best, off, WAVE);
      const int oi = __shfl_xor(bi, off, WAVE);
      if (oi != K && (bi == K || ob > best || (ob == best && oi < bi))) {
        best = ob;
        bi = oi;
      }
    }
    if (nan) raise_error(ws, NP_DEVERR_NAN_SCORE);
    if (lane == 0) {
      if (bi == K) bi = 0;  // every logit NaN: reported above
      chosen[w] = bi;
      cids[h] = bi;
    }
  }
  __syncthreads();
  const int W = (F + 31) / 32;
  const uint32_t* g = bank + ((size_t)l * K + chosen[0]) * W;
  const uint32_t* u = bank + (((size_t)L + l) * K + chosen[1]) * W;
  uint32_t m[WPT], cnt = 0;
#pragma unroll
  for (int i = 0; i < WPT; ++i) {
    const int word = tid * WPT + i;
    m[i] = word < W ? (g[word] & u[word]) : 0u;
    if (word == W - 1 && (F & 31)) m[i] &= (1u << (F & 31)) - 1u;
    if (word < W) mask[(size_t)l * W + word] = m[i];
    cnt += __builtin_popcount(m[i]);
  }
  uint32_t tot;
  uint32_t pos = block_excl_scan<NT>(cnt, scan, &tot);
  int32_t* ids = active_ids + (size_t)l * k;
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
    counts[l] = tot < (uint32_t)k ? (int32_t)tot : k;
    if (tot > (uint32_t)k) raise_error(ws, NP_DEVERR_OVERFLOW);
  }
}

hipError_t launch_centroid_active(const np_shape& s, const np_centroid_model& m,
                                  const float* logits, int32_t* centroid_ids, uint32_t* mask,
                                  int32_t* active_ids, int32_t* active_counts, void* ws,
                                  hipStream_t stream) {
  const int words = (s.d_ffn + 31) / 32;
#define NP_CENTROID_CASE(NT, W)                                                            \
  hipLaunchKernelGGL((centroid_active_kernel<NT, W>), dim3(s.layers), dim3(NT), 0, stream, \
                     logits, m.bank, centroid_ids, mask, active_ids, active_counts,         \
                     s.layers, s.d_ffn, m.n_centroids, s.k, ws)
  if (words <= 256) NP_CENTROID_CASE(256, 1);
  else if (words <= 512) NP_CENTROID_CASE(512, 1);
  else if (words <= 1024) NP_CENTROID_CASE(1024, 1);
  else NP_CENTROID_CASE(1024, 2);
#undef NP_CENTROID_CASE
  return hipGetLastError();
}

// Advances np_delta's step counter (NP_TOKEN_AUTO) once the delta is done.
__global__ void token_advance_kernel(void* ws) {
  if (threadIdx.x == 0) *(int32_t*)((char*)ws + WS_TOKEN) += 1;
}

__global__ void fill_state_kernel(int32_t* __restrict__ a, size_t na, int32_t* __restrict__ b,
                                  size_t nb, int32_t* __restrict__ c, size_t nc,
                                  int32_t* __restrict__ ctrl) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i = i0; i < na; i += stride) a[i] = -1;
  for (size_t i = i0; i < nb; i += stride) b[i] = -1;
  for (size_t i = i0; i < nc; i += stride) c[i] = -1;
  for (size_t i = i0; i < WS_CTRL_BYTES / 4; i += stride) ctrl[i] = 0;
}

hipError_t launch_fill_state(const np_shape& s, const np_state& st, void* ws,
                             hipStream_t stream) {
  const size_t nf = (size_t)s.layers * s.d_ffn, nc = (size_t)s.layers * s.capacity;
  hipLaunchKernelGGL(fill_state_kernel, dim3(1024), dim3(256), 0, stream, st.slot_of, nf,
                     st.neuron_of, nc, st.last_used, nf, (int32_t*)ws);
  return hipGetLastError();
}

hipError_t launch_select(const np_shape& s, const float* scores, uint32_t* mask,
                         int32_t* active_ids, void* ws, hipStream_t stream) {
  const int words = (s.d_ffn + 31) / 32;
  const bool v4 = s.d_ffn % 4 == 0;
#define NP_SELECT_CASE(NT, W)                                                                \
  do {                                                                                       \
    if (v4)                                                                                  \
      hipLaunchKernelGGL((select_kernel<NT, W, true>), dim3(s.layers), dim3(NT), 0, stream,  \
                         scores, mask, active_ids, s.d_ffn, s.k, ws);                        \
    else                                                                                     \
      hipLaunchKernelGGL((select_kernel<NT, W, false>), dim3(s.layers), dim3(NT), 0, stream, \
                         scores, mask, active_ids, s.d_ffn, s.k, ws);                        \
  } while (0)
  if (words <= 256) NP_SELECT_CASE(256, 1);
  else if (words <= 512) NP_SELECT_CASE(512, 1);
  else if (words <= 1024) NP_SELECT_CASE(1024, 1);
  else NP_SELECT_CASE(1024, 2);
#undef NP_SELECT_CASE
  return hipGetLastError();
}

template <int NT, int WPT>
static hipError_t delta_w(const np_shape& s, int32_t token, const int32_t* active_ids,
                          const np_state& st, const np_delta_out& out, void* ws,
                          hipStream_t stream, const int32_t* counts) {
  const int slotwords = (s.capacity + 31) / 32;
  const int spt = (slotwords + NT - 1) / NT;
  const int jpt = (s.k + NT - 1) / NT;
#define NP_DELTA_CASE(J)                                                                      \
  hipLaunchKernelGGL((delta_kernel<NT, WPT, J>), dim3(s.layers), dim3(NT), 0, stream, token,  \
                     active_ids, st.slot_of, st.neuron_of, st.last_used, out, s.d_ffn,        \
                     s.capacity, s.k, spt, ws, counts)
  if (jpt <= 1) NP_DELTA_CASE(1);
  else if (jpt <= 2) NP_DELTA_CASE(2);
  else if (jpt <= 4) NP_DELTA_CASE(4);
  else NP_DELTA_CASE(8);
#undef NP_DELTA_CASE
  return hipGetLastError();
}

// Whether the layer fits the kernels that keep its slot map in LDS.
static bool fits_lds(const np_shape& s) {
  return s.d_ffn <= SD_MAX_F && s.capacity <= SD_MAX_C && s.k <= SD_MAX_K;
}

// Calls f with the smallest build of the LDS kernels that holds this shape: 8
// waves for small layers, 16 from there on (7B, in-kernel: 12.2 us with 16
// waves of 12 rows, 14.8 with 8 of 24).
template <class Fn>
static void with_sd_sizes(const np_shape& s, Fn f) {
  if (s.d_ffn <= 4096 && s.k <= 2048) f(Sd<512, 8, 8, 4>());
  else if (s.d_ffn <= 12288 && s.capacity <= 8192 && s.k <= 2048) f(Sd<1024, 12, 8, 2>());
  else if (s.d_ffn <= 16384 && s.k <= 2048) f(Sd<1024, 16, 16, 2>());
  else if (s.d_ffn <= 16384) f(Sd<1024, 16, 16, 8>());
  else if (s.k <= 4096) f(Sd<1024, 32, 16, 4>());
  else f(Sd<1024, 32, 16, 8>());
}

static hipError_t advance_token(int32_t token, void* ws, hipStream_t stream) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || token != NP_TOKEN_AUTO) return e;
  hipLaunchKernelGGL(token_advance_kernel, dim3(1), dim3(64), 0, stream, ws);
  return hipGetLastError();
}

hipError_t launch_delta(const np_shape& s, int32_t token, const int32_t* active_ids,
                        const np_state& st, const np_delta_out& out, void* ws,
                        hipStream_t stream, const int32_t* counts) {
  if (fits_lds(s)) {
    with_sd_sizes(s, [&](auto z) {
      using S = decltype(z);
      hipLaunchKernelGGL((delta_lds_kernel<S>), dim3(s.layers), dim3(S::NT), 0, stream, token,
                         active_ids, st.slot_of, st.neuron_of, st.last_used, out, s.d_ffn,
                         s.capacity, s.k, ws, counts);
    });
    return advance_token(token, ws, stream);
  }
  const hipError_t e =
      s.d_ffn <= 32 * 1024 ? delta_w<1024, 1>(s, token, active_ids, st, out, ws, stream, counts)
                           : delta_w<1024, 2>(s, token, active_ids, st, out, ws, stream, counts);
  return e != hipSuccess ? e : advance_token(token, ws, stream);
}

// np_select then np_delta: one kernel where the layer fits it (unless
// NP_SELECT_DELTA_FUSED=0), else the two kernels.
hipError_t launch_select_delta(const np_shape& s, int32_t token, const float* scores,
                               uint32_t* mask, int32_t* active_ids, const np_state& st,
                               const np_delta_out& out, void* ws, hipStream_t stream) {
  const char* env = getenv("NP_SELECT_DELTA_FUSED");
  if ((env && env[0] == '0') || !fits_lds(s)) {
    hipError_t e = launch_select(s, scores, mask, active_ids, ws, stream);
    if (e != hipSuccess) return e;
    return launch_delta(s, token, active_ids, st, out, ws, stream, nullptr);
  }
  with_sd_sizes(s, [&](auto z) {
    using S = decltype(z);
    hipLaunchKernelGGL((select_delta_kernel<S>), dim3(s.layers), dim3(S::NT), 0, stream, scores,
                       mask, active_ids, token, st.slot_of, st.neuron_of, st.last_used, out,
                       s.d_ffn, s.capacity, s.k, ws);
  });
  return advance_token(token, ws, stream);
}

}  // namespace np
