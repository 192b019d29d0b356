// Robust noise statistics and normalisation (stats + normalise stage).
//
// For every (pixel, sub-band) series of n_t samples: the FP64 median and
// median absolute deviation, sigma = 1.482602218505602 * MAD, and the
// normalised series z = (x - median) / sigma formed in FP64, rounded to FP32
// and then to the store dtype (paper section 2.2: median subtraction per pixel
// and normalisation by the noise; section 3.2: a robust estimate is needed
// because wide pulses bias a plain one).
//
// Launch: one workgroup of 16 waves per (tile of 16 pixels, sub-band), one
// series per wave, held in registers (32 a lane at 2048 samples, so that two
// workgroups fit a CU: one loads while the other selects). The raw cube
// [t][s][p] (or a ring of its last n_t samples, read oldest first) is loaded in
// 16-pixel row pieces, several pixels and times a lane, and transposed through
// the LDS, 1024 samples of each series at a time. The z series is written
// time-contiguous to the search layout [p][s][t], four samples a lane.
//
// What bounds it: the strided raw read. HBM is read in requests of the piece's
// size, and a plain load of the survey cube reaches 2.0 TB/s in pieces of 32
// bytes, 2.9 in 64 and 4.2 in 128 (whole lines); 128-byte pieces of FP32 would
// need a tile of 256 KB, all a CU's registers, and nothing left to overlap with.
// With its LDS rows (8 pixels, 32-byte pieces), re-read from LDS in every pass,
// this stage took 6.86 ms of a 256 x 256 x 16 x 2048 FP32 cube (FP32 store), and
// 5.80 ms with FP16 cube and store; it now takes 5.3 (3.3 TB/s; loads and stores
// alone take 4.9) and 3.9; 64 x 64 x 16 x 256: 112 us, now 69, where the
// selections' instructions bound it.
//
// Exact selection: order statistics of FP32 keys are found by histogram rounds
// over 256 equal bins of the keys' range (a monotone map, so rank bookkeeping
// is exact whatever the rounding), keeping only the bins that hold the wanted
// ranks, until <= 64 candidates remain, which are ranked across the wave (see
// pick). A crowded bin is binned again over its own range; one whose keys are
// all equal needs no more.
//
// The median selects over the FP32 samples themselves, the MAD over the FP32
// distances |x - RN32(median)|, whose candidates' FP64 distances are then ranked
// and checked to lie inside the keys' interval (see rank_distances). For longer
// series the MAD needs no histogram of its own: the median's predicts a narrow
// bracket of distances (see mad_from_bracket). What stays undecided (a range that
// cannot be binned, a failed check) takes a general path over FP32 roundings of
// the FP64 distances: rounding is monotone, so all samples of a lower key bin have
// smaller FP64 distances than those of the bin holding the wanted rank.
//
// Normalisation divides in FP64 by Markstein's method: with r = RN(1/sigma)
// (a correctly rounded division, once per series), q0 = RN(a*r),
// e = fma(-q0, sigma, a) (exact) and q = fma(e, r, q0) is the correctly rounded
// quotient a/sigma (Markstein, IBM J. Res. Dev. 34(1), 1990); sigma far from
// 1 in exponent takes the plain division instead.
#include "device_common.h"
#include "nsfrb_internal.h"

namespace nsfrb {

// The buffers of the cubes of one launch, passed by value.
struct StatsBuffers {
  const void* x;
  const double *med_in, *sig_in;
  double *med_out, *sig_out;
  void* z;
  unsigned long long* flag_count;
};
constexpr int kStatsCubes = 16;
struct StatsCubes {
  StatsBuffers of[kStatsCubes];
};

// One workgroup takes kTile pixels of one sub-band, one wave per series.
constexpr int kTile = 16;
// Layout of a series of up to 64 V samples in its wave: x[j] of lane l holds
// sample time_of(j, l) = 64 K (j / K) + K l + j % K, so that K consecutive
// samples of a lane move in one LDS read and one store. A lane of the load
// takes K consecutive times of VP consecutive pixels, a phase of the transpose
// kPhase samples of every series.
template <int V> struct StatShape {
  static constexpr int K = V < 4 ? V : 4;
  static constexpr int VP = V / K < 4 ? V / K : 4;
  static constexpr int kPhaseRegs = V < 16 ? V : 16;
  static constexpr int kPhase = 64 * kPhaseRegs;
  static constexpr int kPhases = (V + kPhaseRegs - 1) / kPhaseRegs;
  // LDS row of a series: RS = 4 (mod 16 VP) spreads the transposing writes over
  // all banks; at least the selection's scratch (SeriesCtx), which takes the
  // row's place once the series is in registers
  static constexpr int RS = (kPhase < 896 ? 896 : kPhase) + 4;
  // two workgroups per CU: 64 VGPRs a wave, which holds a series of 2048
  // samples and its temporaries; 4096 samples leave room for one
  static constexpr int kMinWavesPerEU = V <= 32 ? 8 : 4;
  static __device__ __forceinline__ int time_of(int j, int l) { return 64 * K * (j / K) + K * l + j % K; }
};
constexpr double kMadToSigma = 1.482602218505602;

typedef const __attribute__((address_space(1))) char* gptr;   // global memory
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// N consecutive samples of E bytes as one load or store, aligned to a sample only.
template <int BYTES, int E> struct Pack;
template <> struct Pack<16, 4> { typedef u32x4 type __attribute__((aligned(4))); };
template <> struct Pack<8, 4> { typedef u32x2 type __attribute__((aligned(4))); };
template <> struct Pack<4, 4> { typedef uint32_t type; };
template <> struct Pack<8, 2> { typedef u32x2 type __attribute__((aligned(2))); };
template <> struct Pack<4, 2> { typedef uint32_t type __attribute__((aligned(2))); };
template <> struct Pack<2, 2> { typedef uint16_t type; };
template <typename T, int N> using PackOf = typename Pack<(int)sizeof(T) * N, (int)sizeof(T)>::type;

typedef __attribute__((address_space(3))) uint32_t lds_u32;
// Selection scratch of a wave, in its LDS row.
struct SeriesCtx {
  uint32_t* hist;   // 256 bins, and one word more for their prefix counts
  float* cand;      // 64 candidates
  uint32_t* slots;  // slots_of<V>() candidates of each lane
  double* list;     // 64 candidates of the general selection (in the slots' place)
  int n_t;
};
constexpr int kCandWord = 258, kSlotWord = 324;
// Up to 8 registers a lane never fill theirs; longer series have what the row holds.
template <int V> constexpr int slots_of() { return V <= 8 ? 9 : 11; }
static_assert(kSlotWord + 64 * 9 <= StatShape<1>::RS && kSlotWord + 64 * 11 <= StatShape<16>::RS,
              "scratch exceeds the LDS row");

// Result of a selection over FP32 keys: the key value, and the rank of the
// wanted element among the samples whose key equals it.
struct Sel {
  float key;
  int rank_in_ties;
};

// Keys of a series seen through an accessor key(j), j = 0..V-1, by the general
// selection: the samples, or distances formed on each read. It runs for the few
// series that the histogram rounds leave undecided, on a copy of the series in
// private memory and in rolled loops, so that it takes no registers from them.
struct RawKeys {
  const float* x;
  __device__ __forceinline__ float operator()(int j) const { return x[j]; }
};
struct DistKeys {                                  // RN32 of the FP64 distance |x - med|
  const float* x;
  double med;
  __device__ __forceinline__ float operator()(int j) const { return (float)fabs((double)x[j] - med); }
};

// k-th smallest (0-based) of the FP32 keys key(j). Registers past the end of
// the series hold NaN, which fails every comparison and is ignored by
// fminf/fmaxf, so they never take part.
template <int V, class Key>
__device__ __forceinline__ Sel select_kth_f32(const Key& key, int k, const SeriesCtx& cx) {
  const int l = lane_id();
  float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma nounroll
  for (int j = 0; j < V; ++j)
    { const float v = key(j); lo = fminf(lo, v); hi = fmaxf(hi, v); }
  lo = wave_min_f(lo);
  hi = wave_max_f(hi);
  int krem = k;                                    // rank among keys in [lo, hi]
  for (int iter = 0; iter < 48; ++iter) {
    if (!(lo < hi)) return Sel{lo, krem};
    const float scale = 256.0f / (hi - lo);
    if (!(scale > 0.0f && scale < 1e30f)) break;
    cx.hist[4 * l + 0] = 0; cx.hist[4 * l + 1] = 0; cx.hist[4 * l + 2] = 0; cx.hist[4 * l + 3] = 0;
    wave_lds_sync();
#pragma nounroll
    for (int j = 0; j < V; ++j) {
      const float v = key(j);
      if (v >= lo && v <= hi) {
        int b = (int)((v - lo) * scale);
        b = b > 255 ? 255 : b;
        atomicAdd(&cx.hist[b], 1u);
      }
    }
    wave_lds_sync();
    const uint32_t h0 = cx.hist[4 * l], h1 = cx.hist[4 * l + 1], h2 = cx.hist[4 * l + 2], h3 = cx.hist[4 * l + 3];
    const uint32_t s4 = h0 + h1 + h2 + h3;
    const uint32_t incl = wave_incl_scan(s4);
    const uint32_t excl = incl - s4;
    const uint64_t m = ballot((excl <= (uint32_t)krem) && ((uint32_t)krem < incl));
    const int L = __ffsll((long long)m) - 1;
    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)excl, L);
    const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)h0, L), a1 = (uint32_t)__builtin_amdgcn_readlane((int)h1, L);
    const uint32_t a2 = (uint32_t)__builtin_amdgcn_readlane((int)h2, L), a3 = (uint32_t)__builtin_amdgcn_readlane((int)h3, L);
    const uint32_t r = (uint32_t)krem - e;
    int bsel;
    uint32_t before, cnt;
    if (r < a0) { bsel = 0; before = 0; cnt = a0; }
    else if (r < a0 + a1) { bsel = 1; before = a0; cnt = a1; }
    else if (r < a0 + a1 + a2) { bsel = 2; before = a0 + a1; cnt = a2; }
    else { bsel = 3; before = a0 + a1 + a2; cnt = a3; }
    const int B = 4 * L + bsel;
    krem = (int)(r - before);
    if (cnt <= 64) {
      int base = 0;
#pragma nounroll
      for (int j = 0; j < V; ++j) {
        const float v = key(j);
        bool mem = false;
        if (v >= lo && v <= hi) {
          int b = (int)((v - lo) * scale);
          b = b > 255 ? 255 : b;
          mem = (b == B);
        }
        const uint64_t mm = ballot(mem);
        if (mem) cx.list[base + lanes_below(mm)] = (double)v;
        base += popc64(mm);
      }
      wave_lds_sync();
      double c = (l < (int)cnt) ? cx.list[l] : __builtin_inf();
      wave_lds_sync();
      c = wave_sort_asc(c, (int)cnt);
      const float kv = (float)readlane_d(c, krem);
      // rank among equal keys: krem minus the candidates below it
      const int below = popc64(ballot(l < (int)cnt && c < (double)kv));
      return Sel{kv, krem - below};
    }
    float nlo = __builtin_inff(), nhi = -__builtin_inff();
#pragma nounroll
    for (int j = 0; j < V; ++j) {
      const float v = key(j);
      if (v >= lo && v <= hi) {
        int b = (int)((v - lo) * scale);
        b = b > 255 ? 255 : b;
        if (b == B) { nlo = fminf(nlo, v); nhi = fmaxf(nhi, v); }
      }
    }
    lo = wave_min_f(nlo);
    hi = wave_max_f(nhi);
  }
  // Fallback: walk the distinct keys upward from lo.
  float cur = lo;
  for (;;) {
    int ceq = 0;
    float nxt = __builtin_inff();
#pragma nounroll
    for (int j = 0; j < V; ++j) {
      const float v = key(j);
      ceq += (v == cur);
      if (v > cur) nxt = fminf(nxt, v);
    }
    ceq = wave_sum(ceq);
    if (krem < ceq) return Sel{cur, krem};
    krem -= ceq;
    cur = wave_min_f(nxt);
    if (!(cur < __builtin_inff())) return Sel{cur, 0};
  }
}

// Smallest lo and largest hi of the wave, uniform (held in scalar registers).
// NaN lanes are ignored. One DPP instruction per step and value; fminf, which
// quiets its operands first, takes three.
__device__ __forceinline__ void wave_range(float& lo, float& hi) {
#define NSFRB_RANGE_STEP(C) "v_min_f32_dpp %0, %0, %0 " C "\n\tv_max_f32_dpp %1, %1, %1 " C "\n\ts_nop 0\n\t"
  float a, b;
  asm volatile("s_nop 4\n\t"                       // exec may just have been written
               NSFRB_RANGE_STEP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
               NSFRB_RANGE_STEP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
               NSFRB_RANGE_STEP("row_half_mirror row_mask:0xf bank_mask:0xf")
               NSFRB_RANGE_STEP("row_mirror row_mask:0xf bank_mask:0xf")
               NSFRB_RANGE_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
               NSFRB_RANGE_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")
               "v_readlane_b32 %2, %0, 63\n\tv_readlane_b32 %3, %1, 63\n\ts_nop 1"
               : "+v"(lo), "+v"(hi), "=&s"(a), "=&s"(b));
  lo = a;
  hi = b;
#undef NSFRB_RANGE_STEP
}

// The k-th and (k + 1)-th smallest of the candidates c of the lanes in `mask`
// (the others hold +inf; `second` is meaningless when they number k + 1). Each
// lane counts the candidates below its own; ranks shared by equal candidates
// are found at the lowest of them. For the 20 or so candidates that a selection
// ends with this needs no lane exchange through the LDS, unlike a sort (15
// dependent exchange stages of two permutes each at FP64).
__device__ __forceinline__ float readlane_t(float v, int i) { return readlane_f(v, i); }
__device__ __forceinline__ double readlane_t(double v, int i) { return readlane_d(v, i); }
template <typename T>
__device__ __forceinline__ void two_ranks(T c, uint64_t mask, int k, bool want_second, T& first, T& second) {
  int less = 0;
  first = second = readlane_t(c, __ffsll((long long)mask) - 1);
  if (ballot(c == first) == mask) return;          // one value: common where samples take few
  if ((mask & (mask + 1)) == 0) {                  // lanes [0, n)
    const int n = popc64(mask);
    for (int i = 0; i < n; i += 4) {
#pragma unroll
      for (int b = 0; b < 4; ++b) less += readlane_t(c, i + b) < c;
    }
  } else {
    for (uint64_t m = mask; m; m &= m - 1) less += readlane_t(c, __ffsll((long long)m) - 1) < c;
  }
  auto at = [&](int r) {
    uint64_t m = ballot(less == r);
    while (!m) m = ballot(less == --r);            // rank 0 is always some lane's
    return readlane_t(c, __ffsll((long long)m) - 1);
  };
  first = at(k);
  second = want_second ? at(k + 1) : first;
}

// What the histogram rounds end with: up to 64 members, one in each lane of
// `mask` in v, among which the wanted rank is krem; or no mask and the one key
// `tie` that all of them share. t_lo and t_hi bound the members' keys: those of
// all other samples lie outside.
struct Picked {
  float v, tie;
  uint64_t mask;
  int krem;
  double t_lo, t_hi;
  float scale = 0.0f;    // of the last round
  bool ok = false, one = false;   // decided; by one round over all samples (not so for equal samples, which take none)
};

// Candidates of a wave: each lane writes those among its samples to slots of its
// own and counts them by the address it writes to next, without the ballot,
// population count and lane rank per register that placing them in one list
// takes (36 instructions a register, against 4 here). One fewer than its slots
// fit a lane; the address stops at the last slot.
struct Slots {
  uint32_t addr, start, last;
};
template <int V> __device__ __forceinline__ Slots slots_begin(const SeriesCtx& cx) {
  const uint32_t a = (uint32_t)(uintptr_t)(lds_u32*)cx.slots;
  const uint32_t start = a + 4u * (uint32_t)lane_id();
  return Slots{start, start, start + 256u * (slots_of<V>() - 1)};
}
// Appends v in the lanes with lo <= |d| <= hi, and counts those with |d| < lo.
__device__ __forceinline__ void append_between(Slots& q, float d, float lo, float hi, float v, int& below) {
  uint64_t under;
  asm volatile(
      "v_cmp_lt_f32_e64 %1, |%3|, %4\n\t"
      "s_nop 1\n\t"
      "v_addc_co_u32_e64 %2, vcc, 0, %2, %1\n\t"
      "v_cmpx_le_f32_e64 vcc, |%3|, %5\n\t"
      "s_andn2_b64 exec, exec, %1\n\t"
      "ds_write_b32 %0, %6\n\t"
      "v_add_u32_e32 %0, 0x100, %0\n\t"
      "v_min_u32_e32 %0, %7, %0\n\t"
      "s_mov_b64 exec, -1"
      : "+v"(q.addr), "=&s"(under), "+v"(below)
      : "v"(d), "s"(lo), "s"(hi), "v"(v), "v"(q.last)
      : "vcc", "scc", "memory");
}
// The candidates, one in each lane of `mask` of the result and +inf elsewhere;
// an empty mask if there are none, more than 64 or more than fit.
template <int V> __device__ __forceinline__ float slots_end(const Slots& q, const SeriesCtx& cx, uint64_t& mask) {
  asm volatile("s_nop 4");                         // exec was written; lane moves by DPP follow
  const int l = lane_id();
  const uint32_t mine = (q.addr - q.start) >> 8;
  const float inf = __builtin_inff();
  mask = ballot(mine != 0);
  if (ballot(mine > 1) == 0) {                     // none has two: they stay in their lanes
    wave_lds_sync();
    return mine ? __uint_as_float(cx.slots[l]) : inf;
  }
  const uint32_t incl = wave_incl_scan(mine);
  const int n = __builtin_amdgcn_readlane((int)incl, 63);
  if (n > 64 || (V > 8 && ballot(q.addr == q.last))) {
    mask = 0;
    return inf;
  }
  wave_lds_sync();
  const uint32_t at = incl - mine;
  for (uint32_t i = 0; ballot(mine > i); ++i)
    if (mine > i) ((uint32_t*)cx.cand)[at + i] = cx.slots[64u * i + (uint32_t)l];
  wave_lds_sync();
  mask = ~0ull >> (64 - n);
  return l < n ? cx.cand[l] : inf;
}

// One sample's part of a pass of a histogram round, as asm: formed by the
// compiler, what a sample contributes to one pass (a difference, a product) is
// kept for the next, V registers at a time that the wave has not got. Key: the
// sample, or its distance |x - c|. In the lanes whose key lies in [lo, hi], if
// Checked (else it is known to, or is the NaN past the end of a series),
//   bin    counts it in its bin,
//   append adds the sample to the lane's slots if it is a member,
//   range  widens [nlo, nhi] by the key if it is a member.
struct RoundRange {
  float c, lo, hi, scale, base;   // base: 2^23 + the histogram's LDS address
  uint32_t first, width;          // members: bits(t) - first <= width
};
__device__ __forceinline__ float opaque(float v) {
  asm volatile("" : "+v"(v));
  return v;
}
#define NSFRB_KEY(X) "v_subrev_f32_e32 %[t], %[c], " X "\n\t"
#define NSFRB_IN_RANGE(K) "v_cmpx_le_f32_e64 vcc, %[lo], " K "\n\tv_cmpx_ge_f32_e64 vcc, %[hi], " K "\n\t"
#define NSFRB_BITS(K) "v_sub_f32_e64 %[t], " K ", %[lo]\n\tv_fma_f32 %[t], %[t], %[scale], %[base]\n\t"
#define NSFRB_ADD "v_and_b32_e32 %[t], 0x3fffc, %[t]\n\tds_add_u32 %[t], %[one]\n\t"
#define NSFRB_MEMBER "v_subrev_u32_e32 %[t], %[first], %[t]\n\tv_cmpx_ge_u32_e64 vcc, %[width], %[t]\n\t"
#define NSFRB_PUT "ds_write_b32 %[addr], %[x]\n\tv_add_u32_e32 %[addr], 0x100, %[addr]\n\t"
#define NSFRB_STOP "v_min_u32_e32 %[addr], %[last], %[addr]\n\t"
#define NSFRB_ALL "s_mov_b64 exec, -1"
template <bool kDistance> struct SampleOp {
  template <bool Checked> static __device__ __forceinline__ void bin(float x, const RoundRange& r) {
    float t;
    const uint32_t one = 1u;
#define NSFRB_BIN(...) \
  asm volatile(__VA_ARGS__ : [t] "=&v"(t) \
               : [x] "v"(x), [c] "s"(r.c), [lo] "s"(r.lo), [hi] "s"(r.hi), [scale] "s"(r.scale), [base] "v"(r.base), \
                 [one] "v"(one) : "vcc", "memory")
    if constexpr (kDistance && Checked)
      NSFRB_BIN(NSFRB_KEY("%[x]") NSFRB_IN_RANGE("|%[t]|") NSFRB_BITS("|%[t]|") NSFRB_ADD NSFRB_ALL);
    else if constexpr (kDistance)
      NSFRB_BIN(NSFRB_KEY("%[x]") NSFRB_BITS("|%[t]|") NSFRB_ADD);
    else if constexpr (Checked)
      NSFRB_BIN(NSFRB_IN_RANGE("%[x]") NSFRB_BITS("%[x]") NSFRB_ADD NSFRB_ALL);
    else
      NSFRB_BIN(NSFRB_BITS("%[x]") NSFRB_ADD);
  }
  template <bool Checked, bool Stop>               // Stop: the slots may not hold all of the lane's samples
  static __device__ __forceinline__ void append(float x, const RoundRange& r, Slots& q) {
    float t;
#define NSFRB_APPEND(STOP, ...) \
  asm volatile(__VA_ARGS__ NSFRB_MEMBER NSFRB_PUT STOP NSFRB_ALL : [t] "=&v"(t), [addr] "+v"(q.addr) \
               : [x] "v"(x), [c] "s"(r.c), [lo] "s"(r.lo), [hi] "s"(r.hi), [scale] "s"(r.scale), [base] "v"(r.base), \
                 [first] "s"(r.first), [width] "s"(r.width), [last] "v"(q.last) : "vcc", "memory")
    if constexpr (kDistance && Checked)
      NSFRB_APPEND(NSFRB_STOP, NSFRB_KEY("%[x]") NSFRB_IN_RANGE("|%[t]|") NSFRB_BITS("|%[t]|"));
    else if constexpr (kDistance && Stop)
      NSFRB_APPEND(NSFRB_STOP, NSFRB_KEY("%[x]") NSFRB_BITS("|%[t]|"));
    else if constexpr (kDistance)
      NSFRB_APPEND("", NSFRB_KEY("%[x]") NSFRB_BITS("|%[t]|"));
    else if constexpr (Checked)
      NSFRB_APPEND(NSFRB_STOP, NSFRB_IN_RANGE("%[x]") NSFRB_BITS("%[x]"));
    else if constexpr (Stop)
      NSFRB_APPEND(NSFRB_STOP, NSFRB_BITS("%[x]"));
    else
      NSFRB_APPEND("", NSFRB_BITS("%[x]"));
  }
  static __device__ __forceinline__ void range(float x, const RoundRange& r, float& nlo, float& nhi) {
    float t, k;
#define NSFRB_RANGE(KEY, ...) \
  asm volatile(KEY __VA_ARGS__ NSFRB_MEMBER \
               "v_min_f32_e32 %[nlo], %[k], %[nlo]\n\tv_max_f32_e32 %[nhi], %[k], %[nhi]\n\t" NSFRB_ALL \
               : [t] "=&v"(t), [k] "=&v"(k), [nlo] "+v"(nlo), [nhi] "+v"(nhi) \
               : [x] "v"(x), [c] "s"(r.c), [lo] "s"(r.lo), [hi] "s"(r.hi), [scale] "s"(r.scale), [base] "v"(r.base), \
                 [first] "s"(r.first), [width] "s"(r.width) : "vcc")
    if constexpr (kDistance)
      NSFRB_RANGE(NSFRB_KEY("%[x]") "v_and_b32_e32 %[k], 0x7fffffff, %[t]\n\t", NSFRB_IN_RANGE("%[k]") NSFRB_BITS("%[k]"));
    else
      NSFRB_RANGE("v_mov_b32_e32 %[k], %[x]\n\t", NSFRB_IN_RANGE("%[k]") NSFRB_BITS("%[k]"));
  }
};

// Members for the ranks k and, if wanted, k + 1 of the FP32 keys (the samples,
// or their distances from c), which span [lo, hi]. A round puts a key in bin bits 2..9 of round((key - lo) * 1020 /
// (hi - lo)), a monotone map. The rounded product is formed by one fma onto
// 2^23 + (LDS address of the histogram), whose low mantissa bits are then the
// bin's address: no conversion, clamp or shift. More than 64 members are binned
// again over their own range (`check`: keys outside it are masked off, as is
// the NaN in registers past the end; sent to one discard bin instead, up to 64
// lanes of an atomic would hit one address, which the LDS serialises).
template <int V, bool kDistance>
__device__ __forceinline__ Picked pick(const float (&x)[V], float c, float lo, float hi, int k, bool want_second,
                                       bool full, const SeriesCtx& cx) {
  using Op = SampleOp<kDistance>;
  const int l = lane_id();
  const uint32_t hb = (uint32_t)(uintptr_t)(lds_u32*)cx.hist;
  RoundRange r{c, lo, hi, 0.0f, 8388608.0f + (float)hb, 0u, 3u};
  u32x4* h4 = (u32x4*)cx.hist + l;
  Picked p;
  p.mask = 0;
  p.tie = lo;
  p.krem = k;
  bool check = !full;
  if (lo == hi) {                                   // all keys are equal
    p.ok = true;
    return p;
  }
#pragma nounroll
  for (int iter = 0; iter < 8; ++iter) {
    const float span = r.hi - r.lo;
    r.scale = 1020.0f * __builtin_amdgcn_rcpf(span);   // any scale that keeps the products below 1023.5 will do
    if (!(r.scale > 0.0f && r.scale < 1e30f)) break;
    *h4 = u32x4{0u, 0u, 0u, 0u};
    wave_lds_sync();
    if (!check) {
#pragma unroll
      for (int j = 0; j < V; ++j) Op::template bin<false>(x[j], r);
    } else {
#pragma unroll
      for (int j = 0; j < V; ++j) Op::template bin<true>(x[j], r);
    }
    wave_lds_sync();
    const u32x4 h = *h4;
    const uint32_t s4 = h.x + h.y + h.z + h.w;
    const uint32_t incl = wave_incl_scan(s4);
    const uint32_t excl = incl - s4;
    // bin of a rank: the first lane whose inclusive count exceeds it, then the
    // bin among that lane's four; `before` samples lie in lower bins
    auto pos = [&](uint32_t rank, int& bin, uint32_t& before, uint32_t& cnt) {
      const int L = __ffsll((long long)ballot(incl > rank)) - 1;
      before = (uint32_t)__builtin_amdgcn_readlane((int)excl, L);
      bin = 4 * L;
      cnt = (uint32_t)__builtin_amdgcn_readlane((int)h.x, L);
      const uint32_t c1 = (uint32_t)__builtin_amdgcn_readlane((int)h.y, L);
      const uint32_t c2 = (uint32_t)__builtin_amdgcn_readlane((int)h.z, L);
      const uint32_t c3 = (uint32_t)__builtin_amdgcn_readlane((int)h.w, L);
      if (before + cnt <= rank) { before += cnt; cnt = c1; ++bin; }
      if (before + cnt <= rank) { before += cnt; cnt = c2; ++bin; }
      if (before + cnt <= rank) { before += cnt; cnt = c3; ++bin; }
    };
    int bin;
    uint32_t before, cnt;
    r.width = 3u;
    pos((uint32_t)p.krem, bin, before, cnt);
    if (want_second && (uint32_t)p.krem + 1u == before + cnt) {
      // the next rank is the first of a later bin; those between are empty
      int bin2;
      uint32_t before2, cnt2;
      pos((uint32_t)p.krem + 1u, bin2, before2, cnt2);
      cnt += cnt2;
      r.width += 4u * (uint32_t)(bin2 - bin);
    }
    p.krem -= (int)before;
    p.scale = r.scale;
    p.one = iter == 0;
    const uint32_t off = 4u * (uint32_t)bin;
    r.first = 0x4b000000u + hb + off;
    if (cnt <= 64u) {                               // and no more than fit the lanes' slots
      Slots q = slots_begin<V>(cx);
      if (iter == 0) {
#pragma unroll
        for (int j = 0; j < V; ++j) Op::template append<false, (V > 8)>(x[j], r, q);   // NaN's bits lie far above
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) Op::template append<true, true>(x[j], r, q);
      }
      p.v = slots_end<V>(q, cx, p.mask);
      const double step = (double)span * (1.0 / 1020.0);
      p.t_lo = (double)r.lo + ((double)off - 0.5) * step;
      p.t_hi = (double)r.lo + ((double)(off + r.width) + 0.5) * step;
      if (__builtin_expect(iter != 0, 0)) {
        // keys outside a later round's range were masked off, however near: the
        // interval ends at the range (as a branch: the usual series, decided by its
        // first round, pays two instructions)
        p.t_lo = fmax(p.t_lo, (double)r.lo);
        p.t_hi = fmin(p.t_hi, (double)r.hi);
        asm volatile("");
      }
      p.ok = p.mask != 0;
      if (p.ok) return p;
    }
    float nlo = __builtin_inff(), nhi = -__builtin_inff();
#pragma unroll
    for (int j = 0; j < V; ++j) Op::range(x[j], r, nlo, nhi);
    wave_range(nlo, nhi);
    r.lo = nlo;
    r.hi = nhi;
    check = true;
    if (r.lo == r.hi) {
      p.tie = r.lo;
      p.ok = true;
      return p;
    }
  }
  return p;
}

// The two routes to the MAD work with FP32 keys |x - RN32(med)| and are exact or
// decide nothing. With delta = |med - RN32(med)|, a sample whose key is below
// [t_lo, t_hi] has an FP64 distance of less than t_lo + delta, one above it more
// than t_hi - delta (up to the rounding of keys and bounds, within 1 -+ 2^-20),
// so ranks found among the members are the series' own if the values keep that
// far inside. delta = 0 needs no check: rounding is monotone.
__device__ __forceinline__ bool rank_distances(float v, uint64_t mask, int krem, double t_lo, double t_hi, double med,
                                               bool even, double delta, double& mad) {
  double a, b;
  two_ranks(fabs((double)v - med), mask, krem, even, a, b);
  if (delta != 0.0 && (a < t_lo * (1.0 + 0x1p-20) + delta || b > t_hi * (1.0 - 0x1p-20) - delta)) return false;
  mad = even ? (a + b) * 0.5 : a;
  return true;
}

// MAD from histogram rounds over the keys.
template <int V>
__device__ __forceinline__ bool mad_from_keys(const float (&x)[V], double med, int k, bool even, float xmin, float xmax,
                                              bool full, const SeriesCtx& cx, double& mad) {
  const float mf = opaque((float)med);
  const double delta = fabs(med - (double)mf);
  const float dmax = fmaxf(fabsf(xmin - mf), fabsf(xmax - mf));
  const Picked p = pick<V, true>(x, mf, 0.0f, dmax, k, even, full, cx);
  if (!p.ok) return false;
  if (p.mask) return rank_distances(p.v, p.mask, p.krem, p.t_lo, p.t_hi, med, even, delta, mad);
  if (delta != 0.0) return false;
  // many equal keys: their one FP64 distance, if it is one
  double dlo = __builtin_inf(), dhi = -__builtin_inf();
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const float v = opaque(x[j]);
    if (fabsf(v - mf) == p.tie) {
      const double d = fabs((double)v - med);
      dlo = fmin(dlo, d);
      dhi = fmax(dhi, d);
    }
  }
  mad = wave_min(dlo);
  return mad == wave_max(dhi);
}

// MAD from a bracket, for longer series whose median took one round: cx.hist
// then holds the histogram of all samples. Read as a piecewise-uniform
// distribution, two parallel 64-point searches find the distance d at which the
// count of samples within d of the median reaches the middle rank, and a
// bracket around it is sized by the counting error of the two bins there (3.2
// standard deviations). One pass counts the keys below the bracket and gathers
// those inside: two compares a sample, where a round over the keys takes a
// histogram and a gather. The searches (about 350 cycles) pay from 16 registers
// a lane on.
template <int V>
__device__ __forceinline__ bool mad_from_bracket(const float (&x)[V], double med, int k, bool even, float xmin,
                                                 float xmax, float scale, const SeriesCtx& cx, double& mad) {
  const int l = lane_id();
  const float mf = opaque((float)med);
  const double delta = fabs(med - (double)mf);
  const float dmax = fmaxf(fabsf(xmin - mf), fabsf(xmax - mf));
  // exclusive prefix counts P[b] in place of the counts, P[256] = n_t
  u32x4* h4 = (u32x4*)cx.hist + l;
  const u32x4 h = *h4;
  const uint32_t s4 = h.x + h.y + h.z + h.w;
  const uint32_t e0 = wave_incl_scan(s4) - s4;
  wave_lds_sync();
  *h4 = u32x4{e0, e0 + h.x, e0 + h.x + h.y, e0 + h.x + h.y + h.z};
  if (l == 63) cx.hist[256] = (uint32_t)cx.n_t;
  wave_lds_sync();
  const float bins = 0.25f * scale;                    // bins per unit of x
  auto cdf = [&](float p) {                            // interpolated count of samples below p
    const float u = fminf(fmaxf((p - xmin) * bins, 0.0f), 255.99f);
    const int b = (int)u;
    const float pb = (float)cx.hist[b], pn = (float)cx.hist[b + 1];
    return pb + (u - (float)b) * (pn - pb);
  };
  const float target = (float)k + (even ? 1.5f : 1.0f);
  // coarse: d = dmax (i + 1) / 64; fine: 64 steps inside the first coarse step reaching the target
  const float c = dmax * (1.0f / 64.0f);
  float d = c * (float)(l + 1);
  uint64_t m = ballot(cdf(mf + d) - cdf(mf - d) >= target);
  int i = m ? __ffsll((long long)m) - 1 : 63;
  const float c0 = c * (float)i;
  d = c0 + c * (1.0f / 64.0f) * (float)(l + 1);
  m = ballot(cdf(mf + d) - cdf(mf - d) >= target);
  i = m ? __ffsll((long long)m) - 1 : 63;
  const float dh = c0 + c * (1.0f / 64.0f) * (float)(i + 1);
  auto count = [&](float p) {                          // samples in p's bin
    const float u = (p - xmin) * bins;
    if (!(u >= 0.0f && u < 256.0f)) return 0.0f;
    const int b = (int)u;
    return (float)(cx.hist[b + 1] - cx.hist[b]);
  };
  const float here = count(mf + dh) + count(mf - dh);
  const float half = here > 0.0f ? (1.6f * sqrtf(here) + 2.0f) / (here * bins) : dmax;
  const float t_lo = fmaxf(0.0f, dh - half), t_hi = dh + half;
  wave_lds_sync();
  int below = 0;
  uint64_t mask;
  Slots q = slots_begin<V>(cx);
#pragma unroll
  for (int j = 0; j < V; ++j) {
    append_between(q, x[j] - mf, t_lo, t_hi, x[j], below);   // NaN fails both tests
    if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  const float v = slots_end<V>(q, cx, mask);
  below = wave_sum(below);
  const int krem = k - below;
  if (!(krem >= 0 && krem + (even ? 1 : 0) < popc64(mask))) return false;
  return rank_distances(v, mask, krem, t_lo, t_hi, med, even, delta, mad);
}

// The (rank)-th and (rank+1)-th smallest FP64 values val(j) among the samples
// whose key equals kv; `second` is +inf when there is no (rank+1)-th tie.
template <int V, class Key, class Val>
__device__ __forceinline__ void resolve_ties(const Key& key, float kv, int rank, const Val& val,
                                             const SeriesCtx& cx, double& first, double& second) {
  const int l = lane_id();
  int base = 0;
#pragma nounroll
  for (int j = 0; j < V; ++j) {
    const bool mem = key(j) == kv;
    const uint64_t mm = ballot(mem);
    if (mem) {
      const int pos = base + lanes_below(mm);
      if (pos < 64) cx.list[pos] = val(j);
    }
    base += popc64(mm);
  }
  if (base <= 64) {
    wave_lds_sync();
    double c = (l < base) ? cx.list[l] : __builtin_inf();
    wave_lds_sync();
    c = wave_sort_asc(c, base);
    first = readlane_d(c, rank);
    second = (rank + 1 < base) ? readlane_d(c, rank + 1) : __builtin_inf();
    return;
  }
  // more than 64 equal keys: step through their distinct FP64 values
  double cur = -__builtin_inf();
  bool have_first = false;
  for (;;) {
    double nxt = __builtin_inf();
#pragma nounroll
    for (int j = 0; j < V; ++j)
      if (key(j) == kv) {
        const double v = val(j);
        if (v > cur) nxt = fmin(nxt, v);
      }
    cur = wave_min(nxt);
    if (!(cur < __builtin_inf())) { second = __builtin_inf(); return; }
    int ceq = 0;
#pragma nounroll
    for (int j = 0; j < V; ++j)
      if (key(j) == kv) ceq += (val(j) == cur);
    ceq = wave_sum(ceq);
    if (have_first) { second = cur; return; }
    if (rank < ceq) {
      first = cur;
      if (rank + 1 < ceq) { second = cur; return; }
      have_first = true;
    } else {
      rank -= ceq;
    }
  }
}

// Smallest key strictly above kv (+inf if none).
template <int V, class Key>
__device__ __forceinline__ float next_key(const Key& key, float kv, int n_t) {
  const int l = lane_id();
  float m = __builtin_inff();
#pragma nounroll
  for (int j = 0; j < V; ++j)
    { const float v = key(j); if (v > kv) m = fminf(m, v); }
  return wave_min_f(m);
}

// FP64 median of val(j) given FP32 keys with key(j) = RN32(val(j)) (rounding
// is monotone); when kExact, the keys are the values themselves.
template <bool kExact, int V, class Key, class Val>
__device__ __forceinline__ double median_via_keys(const Key& key, const Val& val, const SeriesCtx& cx) {
  const int n = cx.n_t;
  const int k1 = (n - 1) / 2;
  const Sel s = select_kth_f32<V>(key, k1, cx);
  double a, b;
  if (kExact) {
    a = (double)s.key;
    if (n & 1) return a;
    // the next order statistic: a again if another sample shares the key, else the next key
    const int l = lane_id();
    int ceq = 0;
#pragma nounroll
    for (int j = 0; j < V; ++j) ceq += key(j) == s.key;
    ceq = wave_sum(ceq);
    b = (s.rank_in_ties + 1 < ceq) ? a : (double)next_key<V>(key, s.key, n);
  } else {
    resolve_ties<V>(key, s.key, s.rank_in_ties, val, cx, a, b);
    if (n & 1) return a;
    if (!(b < __builtin_inf())) {
      const float k2 = next_key<V>(key, s.key, n);
      double dummy;
      resolve_ties<V>(key, k2, 0, val, cx, b, dummy);
    }
  }
  return (a + b) * 0.5;
}

__device__ __forceinline__ double div_markstein(double a, double b, double r) {
  const double q0 = a * r;
  const double e = __builtin_fma(-q0, b, a);
  return __builtin_fma(e, r, q0);
}

// K consecutive z samples of one lane from sample t on, those past n_t left
// out. Written with the non-temporal hint: the z cube is streamed out once (the
// search reads it back much later), so its lines should not displace the raw
// cube's, which neighbouring tiles still read.
template <int K, typename ST>
__device__ __forceinline__ void store_z(ST* zrow, int t, int n_t, bool all, const float (&zf)[K]) {
  ST v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = from_f32<ST>(zf[i]);
  if (all || t + K <= n_t) {
    PackOf<ST, K> pk;
    __builtin_memcpy(&pk, v, sizeof(pk));
    __builtin_nontemporal_store(pk, (PackOf<ST, K>*)(zrow + t));
  } else {
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (t + i < n_t) zrow[t + i] = v[i];
  }
}

// Statistics + normalisation of one series held in the wave's registers (NaN
// from n_t up to 64 V).
template <int V, typename ST>
__device__ __forceinline__ void process_series(const float (&x)[V], int p, int s, int n_t, int n_sub, int mode,
                                               const double* __restrict__ med_in, const double* __restrict__ sig_in,
                                               double* __restrict__ med_out, double* __restrict__ sig_out,
                                               ST* __restrict__ z, unsigned long long* __restrict__ flag_count,
                                               const SeriesCtx& cx) {
  using Shape = StatShape<V>;
  constexpr int K = Shape::K;
  const int l = lane_id();
  const bool full = n_t == 64 * V;                 // no NaN padding

  long long nflag = 0;
  double med = 0.0, sig = 1.0;
  bool usable = true;
  if (mode == NORM_PIXEL_SUBBAND) {
    float xmin = x[0], xmax = x[0], nf = 0.0f;
    if constexpr (V == 1) {
      nf = __builtin_fmaf(x[0], 0.0f, nf);
    } else {
#pragma unroll
      for (int j = 0; j < V; j += 2) {
        // fminf and fmaxf would first quiet every operand
        asm("v_min3_f32 %0, %1, %2, %0" : "+v"(xmin) : "v"(x[j]), "v"(x[j + 1]));
        asm("v_max3_f32 %0, %1, %2, %0" : "+v"(xmax) : "v"(x[j]), "v"(x[j + 1]));
        // stays 0 unless some sample is infinite or NaN
        nf = __builtin_fmaf(x[j], 0.0f, nf);
        nf = __builtin_fmaf(x[j + 1], 0.0f, nf);
      }
    }
    bool any_bad;
    if (full) {
      any_bad = ballot(nf != 0.0f) != 0;
    } else {
      int fin = 0;
#pragma unroll
      for (int j = 0; j < V; ++j) fin += popc64(ballot(fabsf(x[j]) < __builtin_inff()));
      any_bad = fin != n_t;
    }
    if (any_bad) {
      med = __builtin_nan(""); sig = __builtin_nan(""); usable = false;
    } else {
      wave_range(xmin, xmax);
      const int k1 = (n_t - 1) / 2;
      const bool even = (n_t & 1) == 0;
      const Picked m = pick<V, false>(x, 0.0f, xmin, xmax, k1, even, full, cx);
      double mad = 0.0;
      bool done = m.ok;
      if (done) {
        float a = m.tie, b = m.tie;
        if (m.mask) two_ranks(m.v, m.mask, m.krem, even, a, b);
        med = even ? ((double)a + (double)b) * 0.5 : (double)a;
        done = (V > 8 && m.one && mad_from_bracket<V>(x, med, k1, even, xmin, xmax, m.scale, cx, mad)) ||
               mad_from_keys<V>(x, med, k1, even, xmin, xmax, full, cx, mad);
      }
      if (!done) {
        float y[V];
#pragma unroll
        for (int j = 0; j < V; ++j) y[j] = x[j];
        med = median_via_keys<true, V>(RawKeys{y}, [&](int j) { return (double)y[j]; }, cx);
        mad = median_via_keys<false, V>(DistKeys{y, med}, [&](int j) { return fabs((double)y[j] - med); }, cx);
      }
      sig = kMadToSigma * mad;
      usable = (sig > 0.0) && (sig < __builtin_inf());
    }
    if (l == 0) {
      med_out[(size_t)p * n_sub + s] = med;
      sig_out[(size_t)p * n_sub + s] = sig;
    }
    if (!usable) nflag = 1;
  } else if (mode == NORM_EXTERNAL) {
    med = med_in[(size_t)p * n_sub + s];
    sig = sig_in[(size_t)p * n_sub + s];
    usable = __builtin_isfinite(med) && __builtin_isfinite(sig) && sig > 0.0;
    if (!usable) nflag = 1;
  }
  const double r = 1.0 / sig;
  const bool fast_div = sig > 0x1p-900 && sig < 0x1p900;
  asm volatile("" : "+v"(med));
  ST* zrow = z + ((size_t)p * n_sub + s) * n_t;
  int nbad_samples = 0;
  if (mode == NORM_PIXEL_SUBBAND && usable && fast_div) {
    // the usual case, with no per-sample branch: every sample is finite (a
    // non-finite one makes the series unusable) and the quotient is Markstein's
    auto groups = [&](bool all) {
#pragma unroll
      for (int j = 0; j < V; j += K) {
        float zf[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
          zf[i] = (float)div_markstein((double)x[j + i] - med, sig, r);
          // z is rounded to FP32 first and then to the store type; without the
          // barrier the compiler merges the two roundings into one from FP64
          asm("" : "+v"(zf[i]));
        }
        store_z<K, ST>(zrow, Shape::time_of(j, l), n_t, all, zf);
        __builtin_amdgcn_sched_barrier(0);         // bound the live FP64 temporaries
      }
    };
    if (full) groups(true);
    else groups(false);
  } else {
#pragma unroll
    for (int j = 0; j < V; j += K) {
      float zf[K];
      const int t = Shape::time_of(j, l);
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const float xj = x[j + i];
        const bool fin = __builtin_isfinite(xj);
        if (mode == NORM_NONE) {
          zf[i] = fin ? xj : 0.0f;
          nbad_samples += !fin && t + i < n_t;
        } else if (!usable) {
          zf[i] = 0.0f;
        } else if (mode == NORM_EXTERNAL && !fin) {
          zf[i] = 0.0f;
          nbad_samples += t + i < n_t;
        } else {
          const double a = (double)xj - med;
          zf[i] = (float)(fast_div ? div_markstein(a, sig, r) : a / sig);
        }
      }
      store_z<K, ST>(zrow, t, n_t, false, zf);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (mode == NORM_NONE || mode == NORM_EXTERNAL) nflag += wave_sum(nbad_samples);
  if (l == 0 && nflag) atomicAdd(flag_count, (unsigned long long)nflag);
}

template <int V, typename InT, typename ST>
__global__ __launch_bounds__(kTile * kWave)
__attribute__((amdgpu_waves_per_eu(StatShape<V>::kMinWavesPerEU))) void k_stats_norm(
    StatsCubes cubes, int n_t, int n_sub, int n_pix, int mode, int t_start) {
  const StatsBuffers& cube = cubes.of[blockIdx.z];
  const InT* __restrict__ x = (const InT*)cube.x;
  const double* __restrict__ med_in = cube.med_in;
  const double* __restrict__ sig_in = cube.sig_in;
  double* __restrict__ med_out = cube.med_out;
  double* __restrict__ sig_out = cube.sig_out;
  ST* __restrict__ z = (ST*)cube.z;
  unsigned long long* __restrict__ flag_count = cube.flag_count;
  using Shape = StatShape<V>;
  constexpr int K = Shape::K, VP = Shape::VP, RS = Shape::RS;
  using Raw = PackOf<InT, VP>;
  __shared__ __attribute__((aligned(16))) float rows[kTile * RS];

  // Workgroups are dealt to the 8 XCDs round-robin; remap so that each XCD
  // takes a contiguous run of (pixel tile, sub-band) items: neighbouring
  // tiles share 128-byte lines of the [t][s][p] rows, which then stay in one
  // L2 instead of being fetched once per XCD.
  const unsigned n_items = gridDim.x * gridDim.y;
  unsigned item = blockIdx.x + blockIdx.y * gridDim.x;
  if ((n_items & 7u) == 0) item = (item & 7u) * (n_items >> 3) + (item >> 3);
  const int s = (int)(item / gridDim.x);
  // the last tile is moved back to end at n_pix; the pixels it shares with the
  // tile before it are that one's
  const int p_own = (int)(item % gridDim.x) * kTile;
  const int p0 = max(min(p_own, n_pix - kTile), 0);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int l = lane_id();
  const size_t plane = (size_t)n_sub * n_pix;

  // ---- load: lane (g, c) of wave w takes times t0 + K g + i of phase h, K per
  // lane, and pixels c VP .. c VP + VP - 1; all of the thread's loads are issued
  // first. Rows from n_t up load a valid address and become NaN.
  constexpr int kLanesPerRow = kTile / VP, kGroups = kWave / kLanesPerRow;
  constexpr int kLoadPhases = Shape::kPhases;
  const int c = l % kLanesPerRow, g = l / kLanesPerRow;
  Raw raw[kLoadPhases][K];
  const int t_lane = w * kGroups * K + g * K;      // first row of the lane within a phase
  const char* tile = (const char*)(x + (size_t)s * n_pix + p0);
  if (n_pix < kTile) {
    // narrow plane: single samples, pixels past the end read the last one
#pragma unroll
    for (int h = 0; h < kLoadPhases; ++h)
#pragma unroll
      for (int i = 0; i < K; ++i) {
        int t = h * Shape::kPhase + t_lane + i;
        t = t < n_t ? t : 0;
        t += t_start;
        t -= t >= n_t ? n_t : 0;
        InT v[VP];
#pragma unroll
        for (int e = 0; e < VP; ++e) v[e] = x[(size_t)t * plane + (size_t)s * n_pix + min(c * VP + e, n_pix - 1)];
        __builtin_memcpy(&raw[h][i], v, sizeof(Raw));
      }
  } else if (t_start == 0 && (size_t)64 * plane * sizeof(InT) < 0x80000000u) {
    // Plain cube: the rows of a wave's load start at a uniform address, held in
    // scalar registers, to which every lane adds the same 32-bit offset for all
    // of its loads (rows past n_t: the row's, or the cube's, first).
    const uint32_t coff = (uint32_t)(c * VP * sizeof(InT));
    const uint32_t voff = coff + (uint32_t)((size_t)(g * K) * plane * sizeof(InT));
#pragma unroll
    for (int h = 0; h < kLoadPhases; ++h)
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int t_wave = h * Shape::kPhase + w * kGroups * K + i;
        gptr row = (gptr)(tile + (size_t)(t_wave < n_t ? t_wave : 0) * plane * sizeof(InT));
        asm("" : "+s"(row));
        raw[h][i] = *(const __attribute__((address_space(1))) Raw*)(row + (t_wave + g * K < n_t ? voff : coff));
      }
  } else {
    // Ring of the last n_t samples (read oldest first), or a plane too large
    // for 32-bit offsets.
#pragma unroll
    for (int h = 0; h < kLoadPhases; ++h)
#pragma unroll
      for (int i = 0; i < K; ++i) {
        int t = h * Shape::kPhase + t_lane + i;
        t = t < n_t ? t : 0;
        t += t_start;
        t -= t >= n_t ? n_t : 0;
        raw[h][i] = *(const Raw*)(tile + ((size_t)t * plane + c * VP) * sizeof(InT));
      }
  }

  // ---- transpose through the LDS, kPhase samples of each series at a time
  float xv[V];
  const bool full = n_t == 64 * V;                 // no NaN to fill in
#pragma unroll
  for (int h = 0; h < kLoadPhases; ++h) {
    if (h) __syncthreads();
    InT v[K][VP];
#pragma unroll
    for (int i = 0; i < K; ++i) __builtin_memcpy(&v[i][0], &raw[h][i], sizeof(Raw));
    const int t = h * Shape::kPhase + t_lane;
    auto put = [&](bool fill) {
#pragma unroll
      for (int e = 0; e < VP; ++e) {
        float f[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
          f[i] = to_f32(v[i][e]);
          if (fill) f[i] = t + i < n_t ? f[i] : __builtin_nanf("");
        }
        __builtin_memcpy(__builtin_assume_aligned(&rows[(c * VP + e) * RS + t_lane], 4 * K), f, sizeof(f));
      }
    };
    if (full) put(false);
    else put(true);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < Shape::kPhaseRegs; j += K)
      if (h * Shape::kPhaseRegs + j < V)
        __builtin_memcpy(&xv[h * Shape::kPhaseRegs + j],
                         __builtin_assume_aligned(&rows[w * RS + 64 * j + K * l], 4 * K), 4 * K);
  }
  if (p0 + w >= n_pix || p0 + w < p_own) return;
  // the wave's row is free from here on: histogram and candidate list
  wave_lds_sync();
  uint32_t* scratch = (uint32_t*)&rows[w * RS];
  SeriesCtx cx{scratch, (float*)scratch + kCandWord, scratch + kSlotWord, (double*)(scratch + kSlotWord), n_t};
  process_series<V, ST>(xv, p0 + w, s, n_t, n_sub, mode, med_in, sig_in, med_out, sig_out, z, flag_count, cx);
}

// ------------------------------------------------------------ launcher
// Cubes of one shape share a launch (blockIdx.z): a training batch's 16 cubes of
// 64 x 64 x 16 x 256 in 16 launches took 1,122 us a batch, each one filling and
// draining the chip, and take 1,046 in one.
template <int V, typename InT, typename ST>
static hipError_t launch_stats_v(const StatsLaunch& a, const StatsCubes& cubes, int n, hipStream_t st) {
  dim3 grid((a.n_pix + kTile - 1) / kTile, a.n_sub, n);
  hipLaunchKernelGGL((k_stats_norm<V, InT, ST>), grid, dim3(kTile * kWave), 0, st, cubes, a.n_t, a.n_sub, a.n_pix,
                     a.mode, a.t_start);
  return hipGetLastError();
}

template <typename InT, typename ST>
static hipError_t launch_stats_t(const StatsLaunch& a, const StatsCubes& cubes, int n, hipStream_t st) {
  const int v = (a.n_t + 63) / 64;
  if (v <= 1) return launch_stats_v<1, InT, ST>(a, cubes, n, st);
  if (v <= 2) return launch_stats_v<2, InT, ST>(a, cubes, n, st);
  if (v <= 4) return launch_stats_v<4, InT, ST>(a, cubes, n, st);
  if (v <= 8) return launch_stats_v<8, InT, ST>(a, cubes, n, st);
  if (v <= 16) return launch_stats_v<16, InT, ST>(a, cubes, n, st);
  if (v <= 32) return launch_stats_v<32, InT, ST>(a, cubes, n, st);
  return launch_stats_v<64, InT, ST>(a, cubes, n, st);
}

template <typename InT>
static hipError_t launch_stats_in(const StatsLaunch& a, const StatsCubes& cubes, int n, hipStream_t st) {
  switch (a.store_dtype) {
    case DT_F32: return launch_stats_t<InT, float>(a, cubes, n, st);
    case DT_F16: return launch_stats_t<InT, _Float16>(a, cubes, n, st);
    default: return launch_stats_t<InT, bf16_t>(a, cubes, n, st);
  }
}

__global__ void k_zero_u64(unsigned long long* p) {
  if (threadIdx.x == 0) p[0] = 0ull;
}

hipError_t launch_zero_u64(unsigned long long* p, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_stats(const StatsLaunch* a, int n, hipStream_t st) {
  for (int i = 0; i < n;) {
    StatsCubes cubes{};
    int m = 0;
    auto same = [&](const StatsLaunch& b) {
      return b.n_t == a[i].n_t && b.n_sub == a[i].n_sub && b.n_pix == a[i].n_pix && b.mode == a[i].mode &&
             b.in_dtype == a[i].in_dtype && b.store_dtype == a[i].store_dtype && b.t_start == a[i].t_start;
    };
    for (; i + m < n && m < kStatsCubes && same(a[i + m]); ++m) {
      const StatsLaunch& b = a[i + m];
      cubes.of[m] = StatsBuffers{b.x, b.med_in, b.sig_in, b.med_out, b.sig_out, b.z, b.flag_count};
    }
    hipError_t e;
    switch (a[i].in_dtype) {
      case DT_F32: e = launch_stats_in<float>(a[i], cubes, m, st); break;
      case DT_F16: e = launch_stats_in<_Float16>(a[i], cubes, m, st); break;
      default: e = launch_stats_in<bf16_t>(a[i], cubes, m, st);
    }
    if (e != hipSuccess) return e;
    i += m;
  }
  return hipSuccess;
}

}  // namespace nsfrb
